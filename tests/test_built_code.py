"""The library's GPU code as the compiler wrote it (no GPU needed).

A 64-bit shift whose amount lies in the last vector register of a wave's allocation reads another
register on the target: the compiler, which does not know this, once put the amount of a shift there
and the waves that shared a SIMD with others got wrong sums, those that did not were right.  The
sources are compiled to assembly with the library's own flags and searched for such shifts."""
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


def test_no_64_bit_shift_takes_its_amount_from_the_last_register(tmp_path):
    spec = importlib.util.spec_from_file_location("_b", os.path.join(ROOT, "paper_cs_0408034_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    flags = [f for f in b.HIPCC_FLAGS if f not in ("-shared", "-Wall")]

    def assemble(source):
        out = str(tmp_path / (source.stem + ".s"))
        subprocess.run([hipcc] + flags + ["-S", "--offload-device-only", "-o", out, str(source)], check=True,
                       capture_output=True)
        with open(out) as f:
            return shifts_from_the_last_register(f.read())

    with ThreadPoolExecutor(len(b.SOURCES)) as pool:
        assert [x for found in pool.map(assemble, b.SOURCES) for x in found] == []
