"""The library's GPU code as the compiler wrote it (no GPU needed).

A 64-bit shift whose amount lies in the last vector register of a wave's allocation reads another
register on the target: the compiler, which does not know this, once put the amount of a shift there
and the waves that shared a SIMD with others got wrong sums, those that did not were right.  The
sources are compiled to assembly with the library's own flags and searched for such shifts.

The hand-written instructions of a walk's eight terms write results before they have read all inputs;
that none of the two share registers is tested where their values are the same."""
import importlib.util
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIFT = re.compile(r"v_(?:lshlrev|lshrrev|ashrrev)_[bi]64\S* v\[[0-9:]+\], v(\d+),")


def shifts_from_the_last_register(assembly):
    found, body = [], []
    for line in assembly.splitlines():
        if re.match(r"^\S+:\s+; @", line):
            body = []
        body.append(line)
        m = re.search(r"amdhsa_next_free_vgpr (\d+)", line)
        if m:
            last = (int(m.group(1)) + 7) // 8 * 8 - 1          # allocated in groups of eight
            found += [b.strip() for b in body for s in [SHIFT.search(b)] if s and int(s.group(1)) == last]
            body = []
    return found


def test_the_search_finds_them():
    kernel = "k: ; @k\n v_lshlrev_b64 v[2:3], v%d, v[4:5]\n .amdhsa_next_free_vgpr %d\n"
    assert len(shifts_from_the_last_register(kernel % (79, 80))) == 1
    assert len(shifts_from_the_last_register(kernel % (71, 66))) == 1
    assert shifts_from_the_last_register(kernel % (79, 81)) == []
    assert shifts_from_the_last_register(kernel % (7, 80)) == []


def _build_module():
    spec = importlib.util.spec_from_file_location("_b", os.path.join(ROOT, "paper_cs_0408034_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    return b


def _assembly(b, source, tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    flags = [f for f in b.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    out = str(tmp_path / (source.stem + ".s"))
    subprocess.run([hipcc] + flags + ["-S", "--offload-device-only", "-o", out, str(source)], check=True,
                   capture_output=True)
    with open(out) as f:
        return f.read()


def test_no_64_bit_shift_takes_its_amount_from_the_last_register(tmp_path):
    b = _build_module()
    with ThreadPoolExecutor(len(b.SOURCES)) as pool:
        found = pool.map(lambda s: shifts_from_the_last_register(_assembly(b, s, tmp_path)), b.SOURCES)
        assert [x for f in found for x in f] == []


# A kernel in which most g hold the same values as inputs.
SAME_VALUES = """
__global__ void k(const double *in, double *out)
{
    double d[8], g[8];
    for (int i = 0; i < 8; ++i)
        d[i] = in[threadIdx.x + 64 * i];
    const double end = in[threadIdx.x + 512];
    const f64x2 ys = {in[threadIdx.x + 576], in[threadIdx.x + 640]};
    g[7] = d[0], g[6] = end, g[5] = ys.x, g[4] = ys.y, g[3] = d[2], g[2] = d[1], g[1] = d[3], g[0] = d[7];
    terms_past(d, end, ys, g);
    for (int i = 0; i < 8; ++i)
        out[threadIdx.x + 64 * i] = g[i];
}
"""


def test_the_terms_formed_again_overwrite_no_input(tmp_path):
    b = _build_module()
    kernels = (b.CSRC / "plogp_kernels.hip").read_text()
    start = kernels.index("__device__ __forceinline__ void terms_past(")
    source = tmp_path / "terms.hip"
    source.write_text("#include <hip/hip_runtime.h>\ntypedef unsigned long long u64;\n"
                      "typedef double f64x2 __attribute__((ext_vector_type(2)));\n" +
                      kernels[start:kernels.index("\n}\n", start) + 3] + SAME_VALUES)
    lines = _assembly(b, source, tmp_path).split("#ASMSTART")[1].split("#ASMEND")[0].splitlines()
    ops = [re.findall(r"v\[[0-9:]+\]", x) for x in lines if re.match(r"\s*v_", x)]
    terms = [o for o in ops if len(o) == 4]                            # v_fma_f64 g, slope, e, gap
    assert len(terms) == 8 and len(ops) == 23
    results, e = {o[0] for o in terms}, terms[0][2]
    inputs = {r for o, line in zip(ops, (x for x in lines if re.match(r"\s*v_", x)))
              for r in (o if "cmpx" in line else o[1:])} - {e}
    assert len(results) == 8 and not results & inputs
