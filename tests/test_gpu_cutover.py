"""GPU parity of the cut-over extraction: plogp_cutovers (through the C ABI)
against the CPU oracle's plain definition, record for record (integer and
index work: everything must be identical)."""
import numpy as np
import pytest

import oracle
from oracle import plogp_cutover as oc
from plogp_workloads import make_workload
from tests.gpu_util import stream_handle, torch_cuda

pytestmark = pytest.mark.gpu


def _plogp():
    from paper_cs_0408034_amd import plogp
    return plogp


def gpu_cutovers(cells, m, P, key_mode, capacity=None, d_cells=None):
    """Runs plogp_cutovers on a decision table given as a host array
    [tables][ops][m][P] (or already on the device); returns (offsets, runs, total)."""
    torch = torch_cuda()
    plogp = _plogp()
    nt, n_ops, n_m, n_P = cells.shape
    # the grid handle carries the sizes, the number of process counts and of planes
    mask = plogp.MASK_ALL if n_ops == 2 else plogp.MASK_BCAST
    grid = plogp.plogp_grid_create(m, P, [], plogp.NO_CAP, 1, mask)
    rows = plogp.plogp_cutover_rows(nt, grid)
    assert rows == nt * n_ops * n_P
    if d_cells is None:
        d_cells = torch.from_numpy(np.ascontiguousarray(cells).view(np.uint8).reshape(-1)).cuda()
    cap = cells.size if capacity is None else capacity
    d_off = torch.full((rows + 1,), -1, dtype=torch.int64, device="cuda")
    d_runs = torch.full((max(cap, 1) * 16,), 0xEE, dtype=torch.uint8, device="cuda")
    plogp.plogp_cutovers(grid, nt, d_cells.data_ptr(), key_mode, d_off.data_ptr(),
                         d_runs.data_ptr() if cap else 0, cap, stream_handle())
    torch.cuda.synchronize()
    off = d_off.cpu().numpy().view(np.uint64)
    runs = d_runs.cpu().numpy().view(plogp.RUN_DTYPE)[:cap]
    grid.free()
    return off, runs


def random_table(rng, nt, n_ops, n_m, n_P, p_change):
    """A decision table whose key changes along m with probability p_change per cell."""
    cells = np.zeros((nt, n_ops, n_m, n_P), dtype=oracle.CELL_DTYPE)
    ids = rng.integers(0, 10, size=cells.shape).astype(np.uint32)
    seg = (rng.integers(0, 3, size=cells.shape) * 8).astype(np.uint32)
    keep = rng.random(cells.shape) >= p_change
    for mi in range(1, n_m):
        ids[:, :, mi, :] = np.where(keep[:, :, mi, :], ids[:, :, mi - 1, :], ids[:, :, mi, :])
        seg[:, :, mi, :] = np.where(keep[:, :, mi, :], seg[:, :, mi - 1, :], seg[:, :, mi, :])
    cells["strategy"], cells["s"] = ids, seg
    cells["time"] = rng.random(cells.shape)
    return cells


def check(cells, m, P, key_mode):
    want_off, want_runs = oc.cutovers(cells, m, key_mode)
    off, runs = gpu_cutovers(cells, m, P, key_mode)
    assert (off == want_off).all()
    total = int(off[-1])
    assert total == len(want_runs)
    assert (runs[:total] == want_runs).all()
    # nothing is written past the last run
    assert (runs[total:].view(np.uint8) == 0xEE).all()


@pytest.mark.parametrize("key_mode", [0, 1])
@pytest.mark.parametrize("shape,p_change", [
    ((1, 1, 1, 1), 0.5),          # a single cell
    ((1, 2, 1, 7), 0.5),          # one size: every row is one run
    ((2, 2, 37, 5), 0.3),         # fewer than 64 process counts, ragged last tile of sizes
    ((1, 1, 16, 64), 1.0),        # every cell starts a run, exactly one tile
    ((1, 2, 17, 65), 0.0),        # no change at all; one process count past a wave
    ((3, 1, 100, 130), 0.1),
    ((1, 2, 1000, 3), 0.02),
    ((40, 2, 33, 24), 0.2),       # many tables, config 4's 24 process counts
])
def test_random_tables_match_the_definition(shape, p_change, key_mode):
    rng = np.random.default_rng(hash((shape, key_mode)) % (1 << 32))
    nt, n_ops, n_m, n_P = shape
    m = np.cumsum(rng.integers(1, 50, size=n_m)).astype(np.uint64)
    if n_m > 3:
        m[2] = m[1]               # a repeated size is still its own cell
    P = (np.arange(n_P) + 2).astype(np.uint32)
    check(random_table(rng, nt, n_ops, n_m, n_P, p_change), m, P, key_mode)


@pytest.mark.timeout(300)
def test_scan_over_many_groups():
    # tiles of more than 512 sizes, more than 2048 * 1024 (row, tile) pieces: the second level of the
    # prefix is a launch of its own and loops, and the table is streamed
    rng = np.random.default_rng(7)
    nt, n_ops, n_m, n_P = 500, 2, 513, 64
    cells = random_table(rng, nt, n_ops, n_m, n_P, 0.01)
    m = (np.arange(n_m) * 8 + 8).astype(np.uint64)
    P = (np.arange(n_P) + 2).astype(np.uint32)
    assert nt * n_ops * n_P * ((n_m + 15) // 16) > 2048 * 1024
    check(cells, m, P, 1)


@pytest.mark.parametrize("key_mode", [0, 1])
@pytest.mark.parametrize("shape,p_change", [
    # fewer than 256 rows per compute unit: groups of 16 rows, a thread per row and 16 sizes
    ((700, 2, 37, 24), 0.2),      # 2100 groups of a wave, its last sixteen threads without a size
    ((1100, 2, 33, 15), 0.5),     # the last group has eight rows, the third thread of a row one size
    ((300, 2, 257, 64), 0.03),    # five waves, one size in the last
    ((180, 1, 512, 200), 0.01),   # eight waves, the most sizes that are taken in groups
    ((40000, 1, 1, 1), 0.5),      # one cell per row
    ((600, 2, 64, 30), 1.0),      # every cell starts a run
    ((600, 2, 64, 30), 0.0),      # one run per row
])
def test_tables_of_many_rows_take_one_pass_and_match_the_definition(shape, p_change, key_mode):
    rng = np.random.default_rng(hash((shape, key_mode, "rows")) % (1 << 32))
    nt, n_ops, n_m, n_P = shape
    m = np.cumsum(rng.integers(1, 50, size=n_m)).astype(np.uint64)
    P = (np.arange(n_P) + 2).astype(np.uint32)
    check(random_table(rng, nt, n_ops, n_m, n_P, p_change), m, P, key_mode)


@pytest.mark.parametrize("shape,p_change", [
    # groups of 16 rows: of one per compute unit every start is kept, of more than one what LDS has room for
    ((3, 2, 512, 40), 1.0),       # 15 groups, 8192 starts in each
    ((3, 2, 241, 11), 0.4),       # four waves, one size in the last thread of a row; the fifth group has two rows
    ((400, 2, 512, 24), 0.5),     # 1200 groups whose starts do not fit: read again
    ((400, 2, 512, 24), 0.22),    # the same about as many as fit: some kept, some read again
    # from 65 536 rows on groups of 64, a thread per row and part of its sizes
    ((1400, 2, 16, 24), 1.0),     # a wave, every start kept
    ((1400, 2, 17, 24), 0.3),     # two waves, one size in the second
    ((2800, 2, 20, 24), 0.2),     # 2100 groups: four at a time where their runs are placed
    ((2200, 2, 70, 15), 1.0),     # three waves of 32, 32 and 6 sizes, read again; the last group has 16 rows
    ((2200, 2, 70, 15), 0.2),     # the same, kept
    ((1100, 2, 209, 31), 0.06),   # four waves, the last with seventeen sizes; the last group has 40 rows
    ((1100, 2, 209, 31), 0.204),  # the same about as many as fit
    ((2800, 1, 512, 24), 0.5),    # eight times sixteen sizes to a thread, read again
    ((350000, 1, 2, 3), 0.5),     # 16 407 groups: their counts go through the two-level prefix
])
@pytest.mark.timeout(300)
def test_rows_in_groups_match_the_definition(shape, p_change):
    rng = np.random.default_rng(sum(shape) + int(100 * p_change))
    nt, n_ops, n_m, n_P = shape
    m = np.cumsum(rng.integers(1, 50, size=n_m)).astype(np.uint64)
    P = (np.arange(n_P) + 2).astype(np.uint32)
    check(random_table(rng, nt, n_ops, n_m, n_P, p_change), m, P, 1)


@pytest.mark.timeout(300)
def test_full_size_of_config_4_random_decisions():
    """The shape the benchmark times: 10 000 tables x 2 operations x 256 sizes x 24 process
    counts (480 000 rows, one pass), with a run start in about 2 % of the cells as in the tuned
    table; every offset and every run against the definition."""
    rng = np.random.default_rng(41)
    nt, n_ops, n_m, n_P = 10000, 2, 256, 24
    cells = random_table(rng, nt, n_ops, n_m, n_P, 0.019)
    m = (np.arange(n_m, dtype=np.uint64) + 1) * 8
    P = (np.arange(n_P) + 2).astype(np.uint32)
    check(cells, m, P, 1)


@pytest.mark.timeout(300)
def test_more_rows_than_the_scratch_holds_go_in_slices():
    """8.55 million rows of 6 sizes, whose packed starts would take 64 bytes a row: two slices.  The second
    counts on from the first, with room for all runs, with room for some of its own and with none for them."""
    rng = np.random.default_rng(43)
    n_m, n_P = 6, 3
    cells = random_table(rng, 2_850_000, 1, n_m, n_P, 0.3)
    assert cells.size // n_m * 64 > 512 << 20
    m = (np.arange(n_m, dtype=np.uint64) + 1) * 8
    P = (np.arange(n_P) + 2).astype(np.uint32)
    want_off, want_runs = oc.cutovers(cells, m, 1)
    for cap in (len(want_runs) + 5, 2 * len(want_runs) // 3, len(want_runs) // 3):
        off, runs = gpu_cutovers(cells, m, P, 1, capacity=cap)
        assert (off == want_off).all()
        n = min(cap, len(want_runs))
        assert (runs[:n] == want_runs[:n]).all()
        assert (runs[n:].view(np.uint8) == 0xEE).all()


@pytest.mark.parametrize("n_m,p_change", [(40, 0.1), (40, 1.0), (512, 0.02)])
def test_one_grid_handle_many_rows_then_fewer_then_many_again(n_m, p_change):
    """The same handle serves a batch in groups of 64 rows, smaller ones in groups of 16 and the first again, on
    scratch laid out once: whatever a call leaves there, the next one starts clean."""
    torch = torch_cuda()
    plogp = _plogp()
    rng = np.random.default_rng(23)
    n_ops, n_P = 2, 24
    m = (np.arange(n_m) * 8 + 8).astype(np.uint64)
    P = (np.arange(n_P) + 2).astype(np.uint32)
    grid = plogp.plogp_grid_create(m, P, [], plogp.NO_CAP, 1, plogp.MASK_ALL)
    big = random_table(rng, 1500, n_ops, n_m, n_P, p_change)
    for nt in (1500, 5, 1500, 1365, 800, 1499):          # 72 000, 240, 72 000, 65 520, 38 400, 71 952 rows
        cells = big[:nt]
        want_off, want_runs = oc.cutovers(cells, m, 1)
        rows = nt * n_ops * n_P
        d_cells = torch.from_numpy(np.ascontiguousarray(cells).view(np.uint8).reshape(-1)).cuda()
        d_off = torch.full((rows + 1,), -1, dtype=torch.int64, device="cuda")
        d_runs = torch.full((cells.size * 16,), 0xEE, dtype=torch.uint8, device="cuda")
        plogp.plogp_cutovers(grid, nt, d_cells.data_ptr(), 1, d_off.data_ptr(), d_runs.data_ptr(),
                             cells.size, stream_handle())
        torch.cuda.synchronize()
        off = d_off.cpu().numpy().view(np.uint64)
        assert (off == want_off).all(), nt
        runs = d_runs.cpu().numpy().view(plogp.RUN_DTYPE)
        assert (runs[:len(want_runs)] == want_runs).all(), nt
        assert (runs[len(want_runs):].view(np.uint8) == 0xEE).all(), nt
    grid.free()


@pytest.mark.parametrize("shape,p_change", [
    ((700, 2, 20, 24), 0.3),      # groups of 16 rows, kept
    ((400, 2, 512, 24), 0.5),     # groups of 16 rows, read again
    ((1500, 2, 20, 24), 0.3),     # groups of 64 rows, kept
    ((1500, 2, 70, 24), 1.0),     # groups of 64 rows, read again
])
def test_capacity_smaller_than_the_number_of_runs_on_the_one_pass_path(shape, p_change):
    rng = np.random.default_rng(29)
    nt, n_ops, n_m, n_P = shape
    cells = random_table(rng, nt, n_ops, n_m, n_P, p_change)
    m = (np.arange(n_m) * 8 + 8).astype(np.uint64)
    P = (np.arange(n_P) + 2).astype(np.uint32)
    want_off, want_runs = oc.cutovers(cells, m, 0)
    cap = len(want_runs) // 3 + 1
    off, runs = gpu_cutovers(cells, m, P, 0, capacity=cap)
    assert (off == want_off).all() and int(off[-1]) > cap
    assert (runs == want_runs[:cap]).all()
    off, runs = gpu_cutovers(cells, m, P, 0, capacity=0)
    assert (off == want_off).all()


def test_capacity_smaller_than_the_number_of_runs_and_count_only():
    rng = np.random.default_rng(11)
    cells = random_table(rng, 2, 2, 50, 9, 0.5)
    m = (np.arange(50) * 8 + 8).astype(np.uint64)
    P = (np.arange(9) + 2).astype(np.uint32)
    want_off, want_runs = oc.cutovers(cells, m, 1)
    cap = len(want_runs) // 3
    off, runs = gpu_cutovers(cells, m, P, 1, capacity=cap)
    assert (off == want_off).all() and int(off[-1]) > cap
    assert (runs == want_runs[:cap]).all()
    off, runs = gpu_cutovers(cells, m, P, 1, capacity=0)
    assert (off == want_off).all()


@pytest.mark.parametrize("cfg,kw", [(1, {}), (2, dict(m_slice=slice(0, 1024, 4))),
                                    (4, dict(n_tables=7)), (5, dict(m_slice=slice(0, 4096, 16)))])
@pytest.mark.parametrize("key_mode", [0, 1])
def test_decision_tables_of_the_configs(cfg, kw, key_mode):
    """The oracle's decision table of a config, compressed on the GPU, equals the oracle's runs."""
    wl = make_workload(cfg, **kw)
    cells, _ = oracle.tune_workload(wl)
    check(cells, wl.m, wl.P, key_mode)


def test_tune_then_extract_on_the_device_full_config_2():
    """The headline configuration at full size: sweep and extraction chained on the device,
    checked against the oracle's runs of the oracle's table."""
    torch = torch_cuda()
    plogp = _plogp()
    wl = make_workload(2)
    tab = plogp.plogp_load_tables(wl.sizes, wl.gaps, wl.L)
    grid = plogp.plogp_grid_create(wl.m, wl.P, wl.s, wl.s_cap, wl.dtype_size, wl.strategy_mask)
    nbytes = plogp.plogp_decision_table_bytes(tab.count, grid)
    out = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    rows = plogp.plogp_cutover_rows(1, grid)
    d_off = torch.zeros(rows + 1, dtype=torch.int64, device="cuda")
    cap = nbytes // 16
    d_runs = torch.zeros(cap * 16, dtype=torch.uint8, device="cuda")
    sh = stream_handle()
    plogp.plogp_tune_grid(tab, grid, out.data_ptr(), nbytes, sh)
    plogp.plogp_cutovers(grid, 1, out.data_ptr(), 1, d_off.data_ptr(), d_runs.data_ptr(), cap, sh)
    torch.cuda.synchronize()
    want_cells, _ = oracle.tune_workload(wl)
    want_off, want_runs = oc.cutovers(want_cells, wl.m, 1)
    off = d_off.cpu().numpy().view(np.uint64)
    assert (off == want_off).all()
    runs = d_runs.cpu().numpy().view(plogp.RUN_DTYPE)[:int(off[-1])]
    assert (runs == want_runs).all()
    grid.free()
    tab.free()


def test_bad_arguments_are_refused():
    torch = torch_cuda()
    plogp = _plogp()
    grid = plogp.plogp_grid_create([8, 16], [2, 3], [], plogp.NO_CAP, 1, plogp.MASK_BCAST)
    buf = torch.zeros(1024, dtype=torch.uint8, device="cuda")
    p = buf.data_ptr()
    lib = plogp._lib
    assert lib.plogp_cutovers(grid._h, 1, p, 2, p, p, 4, None) == plogp.EINVAL        # key mode
    assert lib.plogp_cutovers(grid._h, 0, p, 0, p, p, 4, None) == plogp.EINVAL        # no table
    assert lib.plogp_cutovers(grid._h, 1, p + 8, 0, p, p, 4, None) == plogp.EINVAL    # misaligned
    assert lib.plogp_cutovers(grid._h, 1, p, 0, p, None, 4, None) == plogp.EINVAL     # no room
    assert lib.plogp_cutovers(None, 1, p, 0, p, p, 4, None) == plogp.EINVAL
    grid.free()
