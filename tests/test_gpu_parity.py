"""GPU parity: the HIP library (through its C ABI) against the CPU oracle on
the same seeded inputs.  Strategy ids and segment sizes must be identical,
predicted times within 1e-12 relative (binary64; the kernels follow the same
rounding sequence, so they are expected to be bit-identical and the tests say
when they are not)."""
import math

import numpy as np
import pytest

import oracle
from plogp_workloads import ALL_STRATEGIES_MASK, NO_CAP, SEGMENTED_IDS, Workload, make_workload
from tests.gpu_util import REL_TOL, assert_tables_equal, gpu_tune, stream_handle, torch_cuda

pytestmark = pytest.mark.gpu


def _plogp():
    from paper_cs_0408034_amd import plogp
    return plogp


def _dev(arr, dtype):
    torch = torch_cuda()
    return torch.from_numpy(np.ascontiguousarray(arr, dtype=dtype).view(
        {np.uint64: np.int64, np.uint32: np.int32}.get(dtype, dtype))).cuda()


# ------------------------------------------------------------------ step a1/a2

@pytest.mark.parametrize("cfg", [1, 2, 4, 5])
def test_slopes_and_interpolation_bit_exact(cfg):
    torch = torch_cuda()
    plogp = _plogp()
    wl = make_workload(cfg, n_tables=5) if cfg == 4 else make_workload(cfg)
    tab = plogp.plogp_load_tables(wl.sizes, wl.gaps, wl.L)
    rng = np.random.default_rng(cfg)
    for t in range(wl.n_tables):
        x, y = wl.sizes[t], wl.gaps[t]
        got = plogp.plogp_table_slopes(tab, t)
        want = oracle.slopes(x, y)
        assert (got.view(np.uint64) == want.view(np.uint64)).all()
        top = math.log2(x[-1]) + 3
        z = np.floor(2.0 ** (top * rng.random(3000))).astype(np.uint64) + np.uint64(1)
        z = np.concatenate([z, x.astype(np.uint64), x.astype(np.uint64) + np.uint64(1),
                            np.maximum(x.astype(np.uint64), 2) - np.uint64(1),
                            np.array([1, 2, 3, (1 << 53) - 1], dtype=np.uint64)])
        dz = _dev(z, np.uint64)
        dg = torch.empty(len(z), dtype=torch.float64, device="cuda")
        plogp.plogp_interp_g(tab, t, dz.data_ptr(), len(z), dg.data_ptr(), stream_handle())
        torch.cuda.synchronize()
        got = dg.cpu().numpy()
        want = np.array([oracle.g(x, y, int(v)) for v in z])
        assert (got.view(np.uint64) == want.view(np.uint64)).all()
    tab.free()


# ------------------------------------------------------------------ each row of Tables 1 and 2

@pytest.mark.parametrize("n_tables,n", [(1, 2), (1, 223), (1, 224), (2, 111), (2, 112), (89, 2), (90, 2), (1, 2047), (1, 2048)])
def test_tables_around_the_sizes_at_which_they_travel_otherwise(n_tables, n):
    # samples in the arguments of a kernel up to 448 numbers, in one copy up to 4096, in three from there on
    plogp = _plogp()
    rng = np.random.default_rng(n)
    x = np.cumsum(rng.integers(1, 900, size=(n_tables, n)), axis=1).astype(np.float64)
    y, L = rng.uniform(1.0, 90.0, size=x.shape), rng.uniform(0.0, 90.0, size=n_tables)
    tab = plogp.plogp_load_tables(x, y, L)
    for t in range(n_tables):
        slopes = np.diff(y[t]) / np.diff(x[t])
        assert (plogp.plogp_table_slopes(tab, t) == np.append(slopes, slopes[-1])).all()
    tab.free()
    wl = Workload("loaded", x, y, L, np.array([8, 800, 90000], dtype=np.uint64), np.array([2, 3, 70], dtype=np.uint32),
                  np.array([8, 64, 512], dtype=np.uint64), NO_CAP, ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "%d x %d" % (n_tables, n)), "times not bit-identical"


@pytest.mark.parametrize("cfg", [2, 5])
def test_every_strategy_at_random_points(cfg):
    torch = torch_cuda()
    plogp = _plogp()
    wl = make_workload(cfg)
    x, y, L = wl.sizes[0], wl.gaps[0], float(wl.L[0])
    tab = plogp.plogp_load_table(x, y, L)
    rng = np.random.default_rng(50 + cfg)
    n = 700
    m = rng.choice(wl.m, size=n)
    P = rng.choice(wl.P[wl.P <= 3000], size=n).astype(np.uint32)
    P[:8] = [2, 3, 64, 65, 66, 128, 129, 2049]
    s = np.array([int(rng.choice(wl.s[wl.s <= mv])) if (wl.s <= mv).any() else int(mv) for mv in m],
                 dtype=np.uint64)
    s[::7] = m[::7]                                       # k = 1 cases
    dm, dP, ds = _dev(m, np.uint64), _dev(P, np.uint32), _dev(s, np.uint64)
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    for sid in range(13):
        plogp.plogp_eval_strategy(tab, 0, sid, dm.data_ptr(), dP.data_ptr(), ds.data_ptr(), n,
                                  out.data_ptr(), stream_handle())
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        want = np.array([oracle.eval_strategy(x, y, L, sid, int(m[i]), int(P[i]), int(s[i]))
                         for i in range(n)])
        assert (np.abs(got - want) <= REL_TOL * np.abs(want)).all(), sid
        assert (got.view(np.uint64) == want.view(np.uint64)).all(), "strategy %d not bit-exact" % sid
    tab.free()


def test_eval_strategy_domain_errors_give_nan():
    torch = torch_cuda()
    plogp = _plogp()
    wl = make_workload(1)
    tab = plogp.plogp_load_table(wl.sizes[0], wl.gaps[0], 55.0)
    m = np.array([0, 64, 64, 64, 1 << 52], dtype=np.uint64)
    P = np.array([4, 1, 4, 4, 4], dtype=np.uint32)
    s = np.array([8, 8, 0, 128, 8], dtype=np.uint64)
    dm, dP, ds = _dev(m, np.uint64), _dev(P, np.uint32), _dev(s, np.uint64)
    out = torch.zeros(5, dtype=torch.float64, device="cuda")
    plogp.plogp_eval_strategy(tab, 0, 5, dm.data_ptr(), dP.data_ptr(), ds.data_ptr(), 5,
                              out.data_ptr(), stream_handle())
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.isnan(got[:4]).all() and np.isfinite(got[4])
    plogp.plogp_eval_strategy(tab, 0, 11, dm.data_ptr(), dP.data_ptr(), 0, 5, out.data_ptr(),
                              stream_handle())
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.isnan(got[0]) and np.isnan(got[1]) and np.isfinite(got[2]) and np.isnan(got[4])
    tab.free()


# ------------------------------------------------------------------ decision tables

def test_config1_full():
    wl = make_workload(1)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "cfg1"), "times not bit-identical"


def test_config2_full():
    wl = make_workload(2)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "cfg2"), "times not bit-identical"


def test_config3_full():
    wl = make_workload(3)
    got = gpu_tune(wl)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(got, want, "cfg3"), "times not bit-identical"


def test_config4_full():
    # the launch is the full 10 000-table job; the oracle recomputes every table, a
    # thousand at a time (the ragged last group of 16 tables included)
    wl = make_workload(4)
    got = gpu_tune(wl)
    exact = True
    for t0 in range(0, wl.n_tables, 1000):
        pick = slice(t0, min(t0 + 1000, wl.n_tables))
        want, _ = oracle.tune_grid(wl.sizes[pick], wl.gaps[pick], wl.L[pick], wl.m, wl.P, wl.s,
                                   wl.s_cap, wl.strategy_mask)
        exact = assert_tables_equal(got[pick], want, "cfg4 tables %d.." % t0) and exact
        print("cfg4: tables %d..%d identical to the oracle" % (t0, pick.stop - 1), flush=True)
    assert exact, "times not bit-identical"
    # every table: the properties that hold at any size
    assert (got["strategy"][:, 0] <= 9).all() and (got["strategy"][:, 1] >= 10).all()
    assert (got["strategy"][:, 1] <= 12).all()
    seg = np.isin(got["strategy"], SEGMENTED_IDS)
    assert ((got["s"] > 0) == seg).all()
    assert (got["s"][seg] <= np.broadcast_to(wl.m[None, None, :, None], got.shape)[seg]).all()
    assert np.isfinite(got["time"]).all() and (got["time"] > 0).all()
    # P = 2: the three Scatter rows tie exactly and so do Broadcast flat, chain and
    # binomial; the tie-break names the lowest id (a segmented row may still beat them)
    assert (got["strategy"][:, 1, :, 0] == 10).all()
    assert not np.isin(got["strategy"][:, 0, :, 0], (3, 7)).any()


def test_config5_full():
    wl = make_workload(5)
    got = gpu_tune(wl)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(got, want, "cfg5"), "times not bit-identical"


# ------------------------------------------------------------------ shapes, tiles, ragged tails, edge cases

def _small(cfg=2, **kw):
    wl = make_workload(cfg, **kw)
    return wl


@pytest.mark.parametrize("sid", range(13))
def test_each_strategy_alone_over_a_ragged_grid(sid):
    # one strategy enabled: the table is that row's own minimum over s
    wl = _small(2, m_slice=slice(3, 1024, 53), P_subset=[2, 3, 5, 64, 65, 66, 127, 129, 700, 1024])
    wl.strategy_mask = 1 << sid
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "only id %d" % sid)


# from 512 process counts on a lane of the sweep takes two of them, 64 apart: 512 and 640 fill
# their groups, 513 and 520 leave the second half of the last group empty, 600 and 1500 ragged
@pytest.mark.parametrize("n_P,n_m", [(1, 1), (7, 3), (255, 2), (256, 5), (257, 4), (512, 2), (513, 3),
                                     (520, 9), (600, 2), (640, 5), (1500, 3)])
def test_tile_shapes(n_P, n_m):
    rng = np.random.default_rng(n_P * 10 + n_m)
    base = make_workload(2)
    P = np.sort(rng.choice(np.arange(2, 3000), size=n_P, replace=False)).astype(np.uint32)
    m = rng.choice(base.m, size=n_m)
    wl = Workload("tiles", base.sizes, base.gaps, base.L, m, P, base.s, base.s_cap,
                  ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "tiles %d x %d" % (n_P, n_m))


@pytest.mark.parametrize("n_P", [512, 520, 577, 700])
def test_two_process_counts_per_lane_with_few_blocks(n_P):
    # consecutive process counts up to 2 + n_P: at most 32 blocks of the chain sum, so the sweep
    # adds the finished blocks itself; the last group's second half is empty, ragged or full
    base = make_workload(2, m_slice=slice(3, 1024, 97))
    wl = Workload("two", base.sizes, base.gaps, base.L, base.m, np.arange(2, 2 + n_P, dtype=np.uint32),
                  base.s, base.s_cap, ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "two per lane, %d P" % n_P)


def test_many_candidates_span_several_lds_passes():
    wl = make_workload(3, m_slice=slice(0, 1024, 171), P_subset=[2, 3, 9, 64, 4096])
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "cfg3 slice")


@pytest.mark.parametrize("mask", [1 << 2, 1 << 9, (1 << 2) | (1 << 9), 1 << 5, 0x224, ALL_STRATEGIES_MASK])
def test_many_candidates_with_exact_ties_over_s(mask):
    # g(z) = z / 4 exactly: g(s) ceil(m/s) = m / 4 for every s that divides m, so rows
    # 2 and 9 tie over many candidates and the smallest such s must be reported;
    # 600 candidates go through the lane-per-candidate sweep, 40 through the lane-per-m one
    x = np.array([[1.0, float(1 << 40)]])
    y = x / 4.0
    m = np.array([1 << 12, 3 << 11, (1 << 13) + 8, 1 << 16, 40], dtype=np.uint64)
    P = np.array([2, 3, 4, 7, 8, 9, 100, 1024], dtype=np.uint32)
    for n_s in (600, 40):
        s = np.arange(8, 8 * n_s + 1, 8, dtype=np.uint64)
        for L in (0.0, 3.0):
            wl = Workload("ties", x, y, np.array([L]), m, P, s, NO_CAP, mask)
            want, _ = oracle.tune_workload(wl)
            got = gpu_tune(wl)
            assert assert_tables_equal(got, want, "ties n_s=%d L=%g mask=%x" % (n_s, L, mask))
    if mask == 1 << 2:
        assert (got["s"][0, 0, 0] == 8).all()           # m = 4096: every power of two ties


def test_no_candidates_and_candidates_all_above_m():
    base = make_workload(2)
    m = np.array([8, 16, 64], dtype=np.uint64)
    P = np.array([2, 4, 9], dtype=np.uint32)
    for s, mask in (([], ALL_STRATEGIES_MASK), ([128, 256], ALL_STRATEGIES_MASK),
                    ([128, 256], (1 << 2) | (1 << 5) | (1 << 9)), ([8, 64], 1 << 5)):
        wl = Workload("edge", base.sizes, base.gaps, base.L, m, P, np.array(s, dtype=np.uint64),
                      NO_CAP, mask)
        want, _ = oracle.tune_workload(wl)
        got = gpu_tune(wl)
        assert_tables_equal(got, want, "edge %s %x" % (s, mask))
    assert (got["strategy"][0, 0, 0] == 5).all() and (got["s"][0, 0, 0] == 8).all()


def test_no_candidates_with_many_sizes_on_the_sweep_over_process_counts():
    # an empty candidate list with at least 32 process counts and thousands of sizes: the staged
    # path whose sweep runs its lanes over P; no per-(m, s) term may be written anywhere
    base = make_workload(2)
    rng = np.random.default_rng(77)
    m = (rng.integers(1, 1 << 20, size=3000).astype(np.uint64)) * np.uint64(8)
    P = np.unique(rng.integers(2, 3000, size=70)).astype(np.uint32)
    for mask in (ALL_STRATEGIES_MASK, 0x3FF):
        wl = Workload("no candidates", base.sizes, base.gaps, base.L, m, P, np.array([], dtype=np.uint64),
                      NO_CAP, mask)
        want, _ = oracle.tune_workload(wl)
        assert assert_tables_equal(gpu_tune(wl), want, "no candidates, mask %x" % mask)


@pytest.mark.parametrize("n_P,p_hi", [(33, 34), (63, 100), (700, 701), (150, 290)])
def test_no_candidates_where_row_5_goes_by_the_few_that_can_win(n_P, p_hi):
    # the same with process counts that lie close or, in great number, two to a lane
    base = make_workload(2)
    rng = np.random.default_rng(n_P)
    m = (rng.integers(1, 1 << 20, size=9000).astype(np.uint64)) * np.uint64(8)
    P = np.union1d(rng.choice(np.arange(2, p_hi + 1), size=n_P - 1, replace=False), [p_hi]).astype(np.uint32)
    x = np.cumsum(rng.integers(1, 3000, size=600)).astype(np.float64)[None]
    gaps = np.abs(25.0 + 0.07 * x * (1.0 + 0.3 * rng.standard_normal(x.shape)))
    for sizes, g in ((base.sizes, base.gaps), (x, gaps)):
        for mask in (ALL_STRATEGIES_MASK, 0x1FFE, 0x3FF):
            wl = Workload("no candidates", sizes, g, base.L, m, P, np.array([], dtype=np.uint64), NO_CAP, mask)
            want, _ = oracle.tune_workload(wl)
            assert assert_tables_equal(gpu_tune(wl), want, "no candidates, mask %x" % mask)


def test_cap_below_m_and_scatter_only_and_bcast_only():
    base = make_workload(2, m_slice=slice(0, 1024, 97), P_subset=[2, 6, 33, 512])
    for mask, cap in ((0x1C00, NO_CAP), (0x3FF, 4096), (ALL_STRATEGIES_MASK, 64)):
        wl = Workload("masks", base.sizes, base.gaps, base.L, base.m, base.P, base.s, cap, mask)
        want, _ = oracle.tune_workload(wl)
        assert_tables_equal(gpu_tune(wl), want, "mask %x cap %d" % (mask, cap))


def test_two_sample_table_and_non_monotone_table_and_ties():
    m = np.array([8, 4096, 4096, 1 << 20], dtype=np.uint64)        # duplicate m on purpose
    P = np.array([2, 3, 4, 5, 8, 100], dtype=np.uint32)
    s = np.array([8, 512, 4096, 1 << 16], dtype=np.uint64)
    for x, y, L in (([1.0, float(1 << 30)], [1.0, float(1 << 30)], 3.0),      # g(2s) = 2 g(s): ties over s
                    ([1.0, float(1 << 30)], [5.0, 5.0], 0.0),                  # constant gap
                    ([8.0, 64.0, 100.0, 5000.0, 1e6], [9.0, 3.0, 50.0, 20.0, 400.0], 7.0)):
        wl = Workload("tiny", np.array([x]), np.array([y]), np.array([L]), m, P, s, NO_CAP,
                      ALL_STRATEGIES_MASK)
        want, _ = oracle.tune_workload(wl)
        got = gpu_tune(wl)
        assert assert_tables_equal(got, want, "tiny table")
        assert got[0, 0, 1].tobytes() == got[0, 0, 2].tobytes()


def test_largest_sizes_before_the_range_limit():
    base = make_workload(2)
    P = np.array([2, 1000, 1 << 16], dtype=np.uint32)
    m = np.array([8, ((1 << 53) - 1) // ((1 << 16) - 1) // 8 * 8], dtype=np.uint64)
    s = np.array([8, 1 << 20, (1 << 32) - 8], dtype=np.uint64)
    wl = Workload("big", base.sizes, base.gaps, base.L, m, P, s, NO_CAP, ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "largest sizes")


def test_message_sizes_in_any_order_with_repeats():
    # the Scatter-chain sums are kept per distinct size: a grid whose sizes are shuffled and
    # repeated must give each cell the row of its own size
    base = make_workload(2, P_subset=[2, 3, 64, 65, 66, 700, 1024])
    rng = np.random.default_rng(9)
    m = rng.permutation(np.concatenate([base.m[::9], base.m[::31], base.m[5:9]]))
    wl = Workload("shuffled", base.sizes, base.gaps, base.L, m, base.P, base.s, base.s_cap,
                  base.strategy_mask)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "shuffled sizes")
    big = make_workload(5, P_subset=[2, 65, 4097, 40000, 65536])
    m5 = rng.permutation(np.concatenate([big.m[::41], big.m[100:140]]))
    wl5 = Workload("shuffled5", big.sizes, big.gaps, big.L, m5, big.P, big.s, big.s_cap,
                   big.strategy_mask)
    want5, _ = oracle.tune_workload(wl5)
    assert assert_tables_equal(gpu_tune(wl5), want5, "shuffled sizes, big table")


def test_batch_of_tables_matches_one_by_one():
    wl = make_workload(4, n_tables=37, table_offset=1000)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "cfg4 x37")


def test_batch_path_ragged_chunk_many_blocks_and_masks():
    # enough (table, m) rows for the single-kernel batch path: 300 m (one full chunk of
    # 256 and a tail of 44), 24 candidates, P up to 2048 (32 blocks of the chain sum)
    base = make_workload(4, n_tables=30, table_offset=500)
    m = np.sort(np.random.default_rng(3).choice(make_workload(4, n_m=400).m, size=300))
    P = np.array([2, 3, 63, 64, 65, 66, 128, 129, 130, 1000, 1985, 2047, 2048], dtype=np.uint32)
    s = np.array([8 << j for j in range(24)], dtype=np.uint64)
    for mask, cap in ((ALL_STRATEGIES_MASK, NO_CAP), (0x3FF, 1 << 12), (0x1C00, NO_CAP),
                      ((1 << 1) | (1 << 4) | (1 << 8) | (1 << 11), NO_CAP), (1 << 9, NO_CAP)):
        wl = Workload("batch", base.sizes, base.gaps, base.L, m, P, s, cap, mask)
        want, _ = oracle.tune_workload(wl)
        assert assert_tables_equal(gpu_tune(wl), want, "batch path mask %x" % mask)


def test_table_lane_path_on_config_4_tables():
    # 100 tables with the same sample sizes (one full group of 64 and a ragged one of 36)
    # over the whole grid of config 4: the path whose lanes run over tables
    wl = make_workload(4, n_tables=100, table_offset=2000)
    assert (wl.sizes == wl.sizes[0]).all()
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "cfg4 x100, lanes over tables")


def test_table_lane_path_ragged_many_blocks_and_masks():
    # 70 tables x 300 sizes; P up to 2048 (32 blocks of the chain sum, process counts at
    # and next to block ends), 13 process counts (a ragged chunk), 24 candidates, a cap
    base = make_workload(4, n_tables=70, table_offset=700)
    m = np.sort(np.random.default_rng(5).choice(make_workload(4, n_m=400).m, size=300))
    P = np.array([2, 3, 63, 64, 65, 66, 128, 129, 130, 1000, 1985, 2047, 2048], dtype=np.uint32)
    s = np.array([8 << j for j in range(24)], dtype=np.uint64)
    for mask, cap in ((ALL_STRATEGIES_MASK, NO_CAP), (0x3FF, 1 << 12), (0x1C00, NO_CAP),
                      ((1 << 1) | (1 << 4) | (1 << 8) | (1 << 11), NO_CAP), (1 << 9, NO_CAP),
                      ((1 << 2) | (1 << 12), NO_CAP)):
        wl = Workload("batch", base.sizes, base.gaps, base.L, m, P, s, cap, mask)
        want, _ = oracle.tune_workload(wl)
        assert assert_tables_equal(gpu_tune(wl), want, "lanes over tables, mask %x" % mask)


@pytest.mark.parametrize("n_tables,n_P", [(96, 8), (97, 3), (97, 9), (129, 12), (65, 21)])
def test_table_lane_path_half_groups_and_short_runs(n_tables, n_P):
    # the cells leave in runs of 8 process counts, 32 tables at a time: table counts that
    # end at, just after and in the middle of a half group, process counts that leave the
    # last run short or its second half empty
    base = make_workload(4, n_tables=n_tables, table_offset=900, n_m=130)
    P = np.unique(np.random.default_rng(n_P).integers(2, 700, size=64).astype(np.uint32))[:n_P]
    assert len(P) == n_P
    wl = Workload("halves", base.sizes, base.gaps, base.L, base.m, P, base.s, base.s_cap,
                  base.strategy_mask)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "lanes over tables, %d tables x %d P" % (n_tables, n_P))


def test_batch_whose_tables_do_not_share_sample_sizes():
    # one table of 128 sampled elsewhere: the batch must not take the path that assumes
    # shared sample sizes
    wl = make_workload(4, n_tables=128, table_offset=300, n_m=64)
    sizes = wl.sizes.copy()
    sizes[77, 5:9] += 1.0
    wl2 = Workload("mixed", sizes, wl.gaps, wl.L, wl.m, wl.P, wl.s, wl.s_cap, wl.strategy_mask)
    want, _ = oracle.tune_workload(wl2)
    assert assert_tables_equal(gpu_tune(wl2), want, "batch with one table sampled elsewhere")


def test_output_too_small_and_misaligned_are_refused():
    torch = torch_cuda()
    plogp = _plogp()
    wl = make_workload(1)
    tab = plogp.plogp_load_tables(wl.sizes, wl.gaps, wl.L)
    grid = plogp.plogp_grid_create(wl.m, wl.P, wl.s, wl.s_cap, 8, wl.strategy_mask)
    nbytes = plogp.plogp_decision_table_bytes(1, grid)
    buf = torch.zeros(nbytes + 64, dtype=torch.uint8, device="cuda")
    with pytest.raises(plogp.PlogpError) as e:
        plogp.plogp_tune_grid(tab, grid, buf.data_ptr(), nbytes - 16, stream_handle())
    assert e.value.status == plogp.ENOSPC
    with pytest.raises(plogp.PlogpError) as e:
        plogp.plogp_tune_grid(tab, grid, buf.data_ptr() + 8, nbytes, stream_handle())
    assert e.value.status == plogp.EINVAL
    torch.cuda.synchronize()
    assert int(buf.sum().item()) == 0                    # nothing was written
    grid.free(); tab.free()


def test_repeated_calls_on_a_side_stream_give_the_same_table():
    torch = torch_cuda()
    plogp = _plogp()
    wl = make_workload(2, m_slice=slice(0, 1024, 8))
    want, _ = oracle.tune_workload(wl)
    tab = plogp.plogp_load_tables(wl.sizes, wl.gaps, wl.L)
    grid = plogp.plogp_grid_create(wl.m, wl.P, wl.s, wl.s_cap, 8, wl.strategy_mask)
    nbytes = plogp.plogp_decision_table_bytes(1, grid)
    st = torch.cuda.Stream()
    outs = [torch.zeros(nbytes, dtype=torch.uint8, device="cuda") for _ in range(3)]
    torch.cuda.synchronize()
    for o in outs:
        plogp.plogp_tune_grid(tab, grid, o.data_ptr(), nbytes, st.cuda_stream)
    st.synchronize()
    for o in outs:
        arr = o.cpu().numpy().view(plogp.CELL_DTYPE).reshape(want.shape)
        assert assert_tables_equal(arr, want, "repeat")
    grid.free(); tab.free()


def _random_problem(rng, n_choices=(2, 3, 5, 17, 64, 65, 130, 300)):
    """A small random tuning job: table (possibly non-monotone), sizes with repeats in any
    order, ascending process counts, ascending candidates, cap, mask, one to four tables."""
    n = int(rng.choice(n_choices))
    steps = rng.integers(1, 2000, size=n).astype(np.float64)
    x = np.cumsum(steps)
    x[0] = float(rng.integers(1, 64))
    x = np.maximum.accumulate(x + 0.0)
    x = np.unique(np.floor(x))
    n = len(x)
    if n < 2:
        x = np.array([1.0, 9.0])
        n = 2
    n_tables = int(rng.choice([1, 1, 1, 2, 4]))
    gaps = np.empty((n_tables, n))
    for t in range(n_tables):
        y = 30.0 + x * rng.uniform(0.01, 0.2) * (1.0 + 0.3 * rng.standard_normal(n))
        if rng.random() < 0.5:
            y = np.maximum.accumulate(np.abs(y))
        gaps[t] = np.abs(y)
    L = rng.uniform(0.0, 200.0, size=n_tables)
    top = float(x[-1]) * float(rng.choice([0.5, 1.0, 40.0]))
    n_m = int(rng.choice([1, 3, 30, 64, 65, 129]))
    m = (np.floor(np.exp(rng.uniform(np.log(8.0), np.log(max(top, 64.0)), size=n_m)) / 8.0) * 8.0)
    m = np.maximum(m, 8.0).astype(np.uint64)
    if rng.random() < 0.5:
        m = np.concatenate([m, m[: max(1, n_m // 3)]])
    p_hi = int(rng.choice([9, 70, 700, 2500, 5000]))
    n_P = int(min(p_hi - 2, rng.choice([1, 2, 31, 32, 64, 65, 300, 513, 640])))
    P = np.sort(rng.choice(np.arange(2, p_hi), size=max(n_P, 1), replace=False)).astype(np.uint32)
    kind = int(rng.integers(0, 3))
    if kind == 0:
        s = np.array([], dtype=np.uint64)
    elif kind == 1:
        s = np.unique((rng.integers(1, 4000, size=int(rng.choice([1, 5, 34, 64, 65, 200]))) * 8)).astype(np.uint64)
    else:
        s = (np.arange(1, int(rng.choice([300, 1100])) + 1) * 8).astype(np.uint64)
    s_cap = int(rng.choice([NO_CAP, 4096, 64]))
    mask = int(rng.choice([ALL_STRATEGIES_MASK, ALL_STRATEGIES_MASK, 0x3FF, 0x1C00, 0x0A25, 0x1224,
                           int(rng.integers(1, 1 << 13))]))
    return Workload("random", np.repeat(x[None, :], n_tables, axis=0), gaps, L, m, P, s, s_cap, mask)


@pytest.mark.parametrize("seed", range(16))
def test_random_small_problems(seed):
    """Eight random problems per seed: every launch path and tile shape that the sizes select."""
    rng = np.random.default_rng(1000 + seed)
    for k in range(8):
        wl = _random_problem(rng)
        want, _ = oracle.tune_workload(wl)
        what = "random %d/%d: n=%d tables=%d m=%d P=%d s=%d cap=%d mask=%#x" % (
            seed, k, wl.sizes.shape[1], wl.n_tables, len(wl.m), len(wl.P), len(wl.s), wl.s_cap & 0xFFFFFFFF,
            wl.strategy_mask)
        print(what, flush=True)
        assert_tables_equal(gpu_tune(wl), want, what)


@pytest.mark.parametrize("seed", range(4))
def test_random_problems_with_big_tables(seed):
    """Tables of more than a thousand samples (one workgroup per CU holds the table; the
    workgroups of the chain sums also form the per-size and per-candidate terms), one to four
    of them, with every shape of grid the generator makes."""
    rng = np.random.default_rng(7000 + seed)
    for k in range(5):
        wl = _random_problem(rng, n_choices=(1100, 1500, 2300, 4096))
        want, _ = oracle.tune_workload(wl)
        what = "big table %d/%d: n=%d tables=%d m=%d P=%d s=%d cap=%d mask=%#x" % (
            seed, k, wl.sizes.shape[1], wl.n_tables, len(wl.m), len(wl.P), len(wl.s), wl.s_cap & 0xFFFFFFFF,
            wl.strategy_mask)
        print(what, flush=True)
        assert_tables_equal(gpu_tune(wl), want, what)


def _row_problem(rng):
    """A job for the path that does a whole (table, m) row in one workgroup (up to 8192 rows of 256
    process counts and more, any number from 512 on): at most 32 blocks of the chain sum (process
    counts up to 2048), at most 64 candidates, at most 512 samples.  The sizes of small jobs are
    test_small_jobs_a_row_per_workgroup's."""
    n = int(rng.choice([2, 7, 64, 200, 512]))
    x = np.unique(np.floor(np.cumsum(rng.integers(1, 3000, size=n).astype(np.float64))))
    while len(x) < 2:
        x = np.append(x, x[-1] + 7.0)
    n = len(x)
    n_tables = int(rng.choice([1, 1, 2, 5]))
    gaps = np.empty((n_tables, n))
    for t in range(n_tables):
        y = 20.0 + x * rng.uniform(0.01, 0.3) * (1.0 + 0.3 * rng.standard_normal(n))
        gaps[t] = np.abs(y) if rng.random() < 0.5 else np.maximum.accumulate(np.abs(y))
    L = rng.uniform(0.0, 100.0, size=n_tables)
    n_m = -(-256 // n_tables) + int(rng.integers(0, 70))
    top = float(x[-1]) * float(rng.choice([0.3, 2.0, 50.0]))
    m = np.maximum(np.floor(np.exp(rng.uniform(np.log(8.0), np.log(max(top, 64.0)), size=n_m)) / 8.0) * 8.0, 8.0)
    m = m.astype(np.uint64)
    if rng.random() < 0.5:
        m = np.sort(m)
    p_hi = int(rng.choice([300, 1026, 2049]))              # P below p_hi: up to 2048
    n_P = int(min(p_hi - 2, rng.choice([256, 257, 298, 512, 513, 1000])))
    P = np.sort(rng.choice(np.arange(2, p_hi), size=n_P, replace=False)).astype(np.uint32)
    if rng.random() < 0.5:
        P[-1] = p_hi - 1                                    # the largest process count allowed
        P = np.unique(P)
        while len(P) < 256:
            P = np.unique(np.append(P, rng.integers(2, p_hi - 1))).astype(np.uint32)
    n_s = int(rng.choice([0, 1, 7, 8, 9, 34, 63, 64]))
    s = np.unique(rng.integers(1, 6000, size=n_s) * 8).astype(np.uint64) if n_s else np.array([], dtype=np.uint64)
    s_cap = int(rng.choice([NO_CAP, NO_CAP, 4096, 64]))
    mask = int(rng.choice([ALL_STRATEGIES_MASK, ALL_STRATEGIES_MASK, 0x3FF, 0x1C00, 0x0A25, 0x1224, 1 << 2,
                           1 << 9, 1 << 11, 1 << 12, int(rng.integers(1, 1 << 13))]))
    return Workload("row", np.repeat(x[None, :], n_tables, axis=0), gaps, L, m, P, s, s_cap, mask)


@pytest.mark.parametrize("seed", range(10))
def test_random_whole_row_problems(seed):
    rng = np.random.default_rng(3000 + seed)
    for k in range(3):
        wl = _row_problem(rng)
        want, _ = oracle.tune_workload(wl)
        what = "row %d/%d: n=%d tables=%d m=%d P=%d (max %d) s=%d cap=%d mask=%#x" % (
            seed, k, wl.sizes.shape[1], wl.n_tables, len(wl.m), len(wl.P), int(wl.P[-1]), len(wl.s),
            wl.s_cap & 0xFFFFFFFF, wl.strategy_mask)
        print(what, flush=True)
        assert_tables_equal(gpu_tune(wl), want, what)


@pytest.mark.parametrize("p_max,n_mu,n,n_tables,n_s", [
    (6145, 128, 64, 1, 300),      # 96 blocks (the most) x 128 distinct sizes (the fewest), many candidates
    (6146, 140, 64, 1, 300),      # 97 blocks: the walk and the prefix launch instead
    (4097, 127, 64, 1, 70),       # one distinct size too few
    (2050, 70, 200, 2, 12),       # two tables share the launch; 33 blocks (a prefix is wanted)
    (2049, 200, 512, 1, 0),       # 32 blocks (block totals instead of a prefix), 512 samples, no candidates
    (65, 300, 7, 1, 5),           # two blocks, the second with one term
])
def test_chain_sums_per_row_edges(p_max, n_mu, n, n_tables, n_s):
    # the path that forms all Scatter-chain sums of a (table, m) in one workgroup, at its limits
    rng = np.random.default_rng(p_max + n_mu)
    x = np.unique(np.floor(np.cumsum(rng.integers(1, 900, size=n).astype(np.float64))))
    while len(x) < 2:
        x = np.append(x, x[-1] + 5.0)
    gaps = np.abs(25.0 + np.outer(rng.uniform(0.02, 0.2, size=n_tables), x) *
                  (1.0 + 0.2 * rng.standard_normal((n_tables, len(x)))))
    L = rng.uniform(1.0, 80.0, size=n_tables)
    mu = np.unique(rng.integers(1, 4 * int(x[-1]), size=4 * n_mu).astype(np.uint64) * 8)[:n_mu]
    assert len(mu) == n_mu
    m = np.concatenate([mu, mu[: n_mu // 3]])              # repeats: fewer distinct sizes than sizes
    rng.shuffle(m)
    P = np.unique(np.concatenate([rng.integers(2, p_max, size=40), [2, 3, 64, 65, 66, p_max - 1, p_max]])
                  ).astype(np.uint32)
    s = np.unique(rng.integers(1, 3000, size=n_s) * 8).astype(np.uint64) if n_s else np.array([], dtype=np.uint64)
    wl = Workload("chain rows", np.repeat(x[None, :], n_tables, axis=0), gaps, L, m, P, s, NO_CAP,
                  ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert_tables_equal(gpu_tune(wl), want, "chain sums per row, Pmax %d" % p_max)


@pytest.mark.parametrize("seed", range(6))
def test_random_batches(seed):
    """Batches big enough for the single-kernel paths (at least 8192 (table, m) rows), with and
    without shared sample sizes, few or many candidates, short or long chain sums."""
    rng = np.random.default_rng(2000 + seed)
    n = int(rng.choice([2, 9, 40, 64]))
    n_tables = int(rng.choice([64, 65, 100, 130]))
    n_m = -(-8192 // n_tables) + int(rng.integers(0, 40))
    x = np.unique(np.floor(np.cumsum(rng.integers(1, 3000, size=n).astype(np.float64))))
    while len(x) < 2:
        x = np.append(x, x[-1] + 7.0)
    sizes = np.repeat(x[None, :], n_tables, axis=0)
    if seed % 2 == 1:                               # tables with sample sizes of their own
        sizes = sizes + np.floor(rng.integers(0, 3, size=sizes.shape).cumsum(axis=1))
    gaps = 20.0 + sizes * rng.uniform(0.02, 0.1, size=(n_tables, 1)) * (1.0 + 0.2 * rng.random(sizes.shape))
    L = rng.uniform(1.0, 90.0, size=n_tables)
    m = (np.floor(np.exp(rng.uniform(np.log(8.0), np.log(float(x[-1]) * 20.0), size=n_m)) / 8.0) * 8.0)
    m = np.maximum(m, 8.0).astype(np.uint64)
    p_hi = int(rng.choice([40, 600, 2300]))
    P = np.sort(rng.choice(np.arange(2, p_hi), size=int(rng.choice([3, 24, 37])), replace=False)).astype(np.uint32)
    s = np.unique(rng.integers(1, 3000, size=int(rng.choice([0, 7, 21, 40]))) * 8).astype(np.uint64)
    mask = int(rng.choice([ALL_STRATEGIES_MASK, ALL_STRATEGIES_MASK, 0x3FF, 0x1C00, 0x0E24]))
    wl = Workload("batch", sizes, gaps, L, m, P, s, int(rng.choice([NO_CAP, 2048])), mask)
    want, _ = oracle.tune_workload(wl)
    what = "batch %d: n=%d tables=%d m=%d P=%d (up to %d) s=%d mask=%#x" % (
        seed, sizes.shape[1], n_tables, n_m, len(P), int(P[-1]), len(s), mask)
    print(what, flush=True)
    assert_tables_equal(gpu_tune(wl), want, what)


# ------------------------------------------------------------------ the chain row at scattered points

@pytest.mark.parametrize("n_x,n_points,p_top", [
    (2, 1, 66), (64, 255, 1026), (64, 256, 513), (64, 257, 577), (200, 1000, 129), (512, 300, 2000),
    (513, 385, 1500), (4096, 700, 1100), (64, 130, 70000),
])
def test_chain_row_at_points_around_block_ends(n_x, n_points, p_top):
    # complete blocks are dealt eight block indices at a time and the rest of a sum is walked by
    # the point's own thread: process counts at and next to the ends of blocks and of eight of
    # them, workgroups with one point, a full one and one more, both sizes of workgroup (tables
    # of up to 512 samples and larger ones), points outside the domain among the others
    torch = torch_cuda()
    plogp = _plogp()
    rng = np.random.default_rng(n_x + n_points)
    x = np.unique(np.floor(2.0 ** rng.uniform(0, 20, 6 * n_x)))
    x = np.append(x, x[-1] + 1.0 + np.arange(max(0, n_x - len(x))))[:n_x]
    y = np.abs(30.0 + 0.1 * x * (1.0 + 0.3 * rng.standard_normal(len(x))))
    edges = np.array([2, 3, 63, 64, 65, 66, 128, 129, 130, 512, 513, 514, 576, 577, 578, 1025])
    P = np.where(rng.random(n_points) < 0.5, rng.choice(edges[edges <= p_top], n_points),
                 rng.integers(2, p_top + 1, n_points)).astype(np.uint32)
    P[-1] = p_top
    m = np.maximum(np.floor(2.0 ** rng.uniform(0, 22, n_points)), 1.0).astype(np.uint64)
    if n_points > 100:
        P[5], m[6], m[7] = 1, 0, 1 << 53
        P[8], m[8] = 64, ((1 << 53) - 1) // 63                  # the largest size allowed
        P[9], m[9] = 65, ((1 << 53) - 1) // 63                  # and one process too many
    tab = plogp.plogp_load_table(x, y, 7.5)
    out = torch.empty(n_points, dtype=torch.float64, device="cuda")
    dm, dP = _dev(m, np.uint64), _dev(P, np.uint32)
    for sid in (11, 14):
        plogp.plogp_eval_strategy(tab, 0, sid, dm.data_ptr(), dP.data_ptr(), 0, n_points, out.data_ptr(),
                                  stream_handle())
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        bad = (P < 2) | (m == 0) | (m >= (1 << 53))
        bad |= (P.astype(object) - 1) * m.astype(object) >= (1 << 53)
        bad = bad.astype(bool)
        assert np.isnan(got[bad]).all() and (n_points <= 100 or bad.sum() == 4)
        want = np.array([oracle.eval_strategy(x, y, 7.5, sid, int(mv), int(pv), 0)
                         for mv, pv in zip(m[~bad], P[~bad])])
        assert (got[~bad].view(np.uint64) == want.view(np.uint64)).all(), "row %d" % sid
    tab.free()


@pytest.mark.parametrize("n_x", [64, 256, 257, 640, 641, 1500, 4096])
def test_chain_row_at_many_points(n_x):
    # more than 384 points per compute unit: from 257 samples on the rest of a sum is searched for,
    # not walked, four block indices are dealt at a time, and workgroups take 256 or 768 points.
    # Every 61st point and the last ones against the oracle, all of them against the smaller launch
    torch = torch_cuda()
    plogp = _plogp()
    rng = np.random.default_rng(n_x)
    n_points = 384 * torch.cuda.get_device_properties(0).multi_processor_count + 1
    x = np.unique(np.floor(2.0 ** rng.uniform(0, 20, 8 * n_x)))
    x = np.append(x, x[-1] + 1.0 + np.arange(max(0, n_x - len(x))))[:n_x]
    y = np.abs(30.0 + 0.1 * x * (1.0 + 0.3 * rng.standard_normal(n_x)))
    P = rng.integers(1, rng.choice([18, 66, 700], n_points)).astype(np.uint32)
    m = np.maximum(np.floor(2.0 ** rng.uniform(0, 22, n_points)), 1.0).astype(np.uint64)
    tab = plogp.plogp_load_table(x, y, 7.5)
    out = torch.empty(n_points, dtype=torch.float64, device="cuda")
    half = torch.empty(n_points, dtype=torch.float64, device="cuda")
    dm, dP = _dev(m, np.uint64), _dev(P, np.uint32)
    plogp.plogp_eval_strategy(tab, 0, 11, dm.data_ptr(), dP.data_ptr(), 0, n_points, out.data_ptr(), stream_handle())
    k = n_points // 2
    plogp.plogp_eval_strategy(tab, 0, 11, dm.data_ptr(), dP.data_ptr(), 0, k, half.data_ptr(), stream_handle())
    plogp.plogp_eval_strategy(tab, 0, 11, dm[k:].data_ptr(), dP[k:].data_ptr(), 0, n_points - k, half[k:].data_ptr(),
                              stream_handle())
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert (np.isnan(got) == (P < 2)).all()
    assert (got.view(np.uint64) == half.cpu().numpy().view(np.uint64))[P >= 2].all()
    some = np.unique(np.concatenate([np.arange(0, n_points, 61), np.arange(n_points - 300, n_points)]))
    some = some[P[some] >= 2]
    want = np.array([oracle.eval_strategy(x, y, 7.5, 11, int(mv), int(pv), 0) for mv, pv in zip(m[some], P[some])])
    assert (got[some].view(np.uint64) == want.view(np.uint64)).all()
    tab.free()


@pytest.mark.parametrize("n_x", [64, 65, 72, 73, 128, 129, 256, 257, 512, 513])
@pytest.mark.parametrize("together", [1, 13, 33, 70])
def test_complete_blocks_of_many_points_and_of_few(n_x, together):
    # from 768 points per compute unit on, and from 65 samples up to 512, the first block of a sum is walked a
    # term at a time; with fewer points it is searched for from 73 samples on, and from 129 on the others where
    # they enter many intervals.  Groups of samples one byte apart, the next 1500 on: a term enters all of a group
    torch, plogp = torch_cuda(), _plogp()
    rng = np.random.default_rng(n_x + together)
    n_points = 768 * torch.cuda.get_device_properties(0).multi_processor_count
    x = np.array([1500.0 * (1 + k // together) + k % together for k in range(n_x)])
    y = np.abs(30.0 + 0.1 * x * (1.0 + 0.3 * rng.standard_normal(n_x)))
    P = rng.integers(60, rng.choice([67, 130, 400], n_points)).astype(np.uint32)
    m = np.maximum(np.floor(2.0 ** rng.uniform(0, 15, n_points)), 1.0).astype(np.uint64)
    tab = plogp.plogp_load_table(x, y, 7.5)
    out = torch.empty(n_points, dtype=torch.float64, device="cuda")
    dm, dP = _dev(m, np.uint64), _dev(P, np.uint32)
    got = {}
    for n in (n_points, n_points - 1, 5000):
        plogp.plogp_eval_strategy(tab, 0, 11, dm.data_ptr(), dP.data_ptr(), 0, n, out.data_ptr(), stream_handle())
        torch.cuda.synchronize()
        got[n] = out.cpu().numpy().view(np.uint64)[:n]
    assert (got[n_points][:-1] == got[n_points - 1]).all() and (got[n_points][:5000] == got[5000]).all()
    some = np.append(np.arange(0, n_points, 411), n_points - 1)
    want = np.array([oracle.eval_strategy(x, y, 7.5, 11, int(mv), int(pv), 0) for mv, pv in zip(m[some], P[some])])
    assert (got[n_points][some] == want.view(np.uint64)).all()
    tab.free()


@pytest.mark.parametrize("n_m,n_P,p_hi,n_s,n", [
    (2559, 36, 1500, 13, 64), (2560, 36, 1500, 13, 64),   # 24 blocks of the chain sum: ten rows a compute unit
    (2560, 31, 1500, 13, 64), (2560, 36, 1500, 17, 64), (2560, 36, 1500, 13, 129),    # no longer one of these
    (4095, 49, 50, 16, 128), (4096, 49, 50, 25, 128),     # one block: sixteen, then the staged path
    (2600, 63, 2049, 16, 21), (3000, 64, 2049, 16, 21),   # 33 blocks; 64 process counts
    (8192, 300, 400, 25, 64), (600, 600, 700, 65, 200),   # lanes over process counts, one and two to a lane
    (5000, 127, 128, 30, 1000),                           # more workgroups of terms than the chip has room for
])
@pytest.mark.parametrize("mask", [ALL_STRATEGIES_MASK, 0x0A25])
def test_where_the_row_path_ends(n_m, n_P, p_hi, n_s, n, mask):
    rng = np.random.default_rng(n_m * 100 + n_P + n_s)
    x = np.unique(np.floor(np.cumsum(rng.integers(1, 900, size=n).astype(np.float64))))
    gaps = np.abs(25.0 + 0.07 * x[None] * (1.0 + 0.3 * rng.standard_normal((1, len(x)))))
    m = np.maximum(np.floor(np.exp(rng.uniform(np.log(8.0), np.log(40.0 * x[-1]), size=n_m)) / 8.0) * 8.0, 8.0)
    P = np.union1d(np.sort(rng.choice(np.arange(2, p_hi), size=n_P - 1, replace=False)), [p_hi]).astype(np.uint32)
    s = (8 * np.sort(rng.choice(np.arange(1, 4000), size=n_s, replace=False))).astype(np.uint64)
    wl = Workload("row end", x[None], gaps, np.array([60.0]), m.astype(np.uint64), P, s, NO_CAP, mask)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "%d x %d, mask %x" % (n_m, n_P, mask)), "times not bit-identical"


# ------------------------------------------------------------------ terms beside the sums of a big table

@pytest.mark.parametrize("n_tables,n,n_m,n_s,n_P,mask", [
    (1, 1021, 1, 0, 33, ALL_STRATEGIES_MASK), (1, 1021, 63, 1, 33, ALL_STRATEGIES_MASK), (1, 4096, 65, 63, 40, ALL_STRATEGIES_MASK),
    (1, 1500, 64, 64, 32, ALL_STRATEGIES_MASK), (2, 1100, 129, 65, 33, 0x1FFF & ~0x1000), (300, 1030, 17, 129, 32, ALL_STRATEGIES_MASK),
    (3, 2000, 4200, 5, 32, 0x0FFF), (1, 1500, 100, 256, 40, ALL_STRATEGIES_MASK), (1, 1500, 100, 257, 9, ALL_STRATEGIES_MASK),
    (1, 4096, 70, 1024, 9, 0x1A25), (1, 1500, 70, 1025, 9, ALL_STRATEGIES_MASK), (1, 1500, 257, 20, 5, ALL_STRATEGIES_MASK)])
def test_terms_beside_the_sums_of_a_big_table(n_tables, n, n_m, n_s, n_P, mask):
    # groups of 64 sizes, of 64 candidates (and none), rows of (m, s) of up to 256 candidates, each sweep
    rng = np.random.default_rng(n_m + n_s)
    x = np.cumsum(rng.integers(1, 60, size=(n_tables, n)), axis=1).astype(np.float64)
    gaps = np.abs(20.0 + x * 0.05 * (1.0 + 0.4 * rng.standard_normal(x.shape)))
    P = np.sort(rng.choice(np.arange(2, 150), size=n_P, replace=False)).astype(np.uint32)
    m = 8 * rng.choice(np.arange(1, 9000), size=n_m, replace=False)
    s = 8 * np.sort(rng.choice(np.arange(1, 3000), size=n_s, replace=False))
    wl = Workload("big", x, gaps, rng.uniform(0.0, 90.0, size=n_tables), m.astype(np.uint64), P, s.astype(np.uint64), 16000, mask)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "n=%d m=%d s=%d" % (n, n_m, n_s)), "times not bit-identical"


@pytest.mark.parametrize("n,n_tables,n_m,p_hi", [(64, 3, 5, 2200), (65, 3, 5, 2200), (65, 40, 70, 9000), (150, 100, 3, 8000),
                                                 (256, 12, 70, 5000), (257, 12, 70, 5000)])
def test_leading_blocks_of_the_sums_of_small_tables(n, n_tables, n_m, p_hi):
    # the first four blocks are items of their own from 65 samples on (the first 32 from 257), samples and
    # sizes over many octaves, so that the first block enters many intervals
    rng = np.random.default_rng(n + n_tables)
    x = np.floor(np.geomspace(1.0, 2.0 ** 22, n) * rng.uniform(1.0, 1.2, size=(n_tables, 1))) + 20.0 * np.arange(n)
    gaps = np.abs(20.0 + x * 0.05 * (1.0 + 0.3 * rng.standard_normal(x.shape)))
    m = np.unique(np.maximum(8, 8 * np.floor(np.geomspace(8, 2.0 ** 23, n_m) / 8)))
    P = np.union1d(rng.choice(np.arange(2, p_hi), size=12, replace=False), [65, 129, 257, 258, p_hi]).astype(np.uint32)
    wl = Workload("leading", x, gaps, rng.uniform(0.0, 90.0, size=n_tables), m.astype(np.uint64), P,
                  np.array([8, 64, 512], dtype=np.uint64), NO_CAP, ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "n=%d" % n), "times not bit-identical"


# ------------------------------------------------------------------ prefix of the block sums

@pytest.mark.parametrize("blocks,n_m,n_P", [(33, 15, 9), (97, 1, 300), (128, 16, 600), (129, 17, 600), (256, 5, 40), (257, 33, 40),
                                            (384, 3, 5), (385, 16, 5), (300, 7, 40), (300, 8, 40), (300, 9, 40),
                                            (513, 2, 4096), (513, 2, 4097), (65536, 1, 40),
                                            (65537, 1, 40)])
def test_prefix_of_the_block_sums_at_the_edges_of_its_tiles(blocks, n_m, n_P):
    # tiles of 128 blocks, groups of eight distinct sizes; block indices in LDS for up to 4096 process counts
    # and 65 536 blocks; the sum ends with the first term of its last block
    rng = np.random.default_rng(blocks + n_P)
    n = 700
    x = np.cumsum(rng.integers(1, 4000, size=n)).astype(np.float64)[None]
    gaps = np.abs(20.0 + x * 0.05 * (1.0 + 0.4 * rng.standard_normal(x.shape)))
    top = 64 * (blocks - 1) + 2
    P = np.union1d(rng.choice(np.arange(2, top), size=n_P - 1, replace=False), [top]).astype(np.uint32)
    m = 8 * rng.choice(np.arange(1, 9000), size=n_m, replace=False)
    wl = Workload("prefix", x, gaps, np.array([37.0]), m.astype(np.uint64), P, np.array([8, 64], dtype=np.uint64), NO_CAP,
                  ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "%d blocks" % blocks), "times not bit-identical"


@pytest.mark.parametrize("n_tables,n_m,blocks", [(1024, 8, 33), (1025, 8, 33), (513, 9, 34), (342, 17, 33), (342, 24, 129),
                                                 (260, 31, 33), (205, 33, 40)])
def test_prefix_of_the_block_sums_of_many_tables(n_tables, n_m, blocks):
    # sixteen sizes to a group where there are more than four groups of eight to a compute unit: 1024 groups,
    # 1025, and groups of one, eight and fifteen sizes behind full ones
    rng = np.random.default_rng(n_tables + n_m)
    x = np.cumsum(rng.integers(1, 9000, size=(n_tables, 20)), axis=1).astype(np.float64)
    gaps = np.abs(20.0 + x * 0.05 * (1.0 + 0.4 * rng.standard_normal(x.shape)))
    top = 64 * (blocks - 1) + 2
    P = np.union1d(rng.choice(np.arange(2, top), size=5, replace=False), [64, 65, 129, top]).astype(np.uint32)
    m = 8 * rng.choice(np.arange(1, 4000), size=n_m, replace=False)
    wl = Workload("prefix", x, gaps, rng.uniform(0.0, 90.0, size=n_tables), m.astype(np.uint64), P,
                  np.array([8, 64], dtype=np.uint64), NO_CAP, ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "%d x %d" % (n_tables, n_m)), "times not bit-identical"


# ------------------------------------------------------------------ tiles of message sizes

def _tile_problem(rng, seed):
    """A job of at least 4096 (table, m) rows (16 per compute unit; 32 with more than 512 samples) and
    at most 24 candidates whose tables have sample sizes of their own.  The kernel whose workgroups
    take a table and up to 32 message sizes takes ten of the 24 seeds: those without a Gather or
    Barrier row, of at most 32 blocks of the chain sum, up to 512 samples (and few larger tables).  The
    others go to the staged path or, from 256 process counts on, to a row per workgroup.
    test_tiles_at_the_edges_of_their_rules has the former's limits."""
    n = int([2, 3, 9, 57, 120, 300, 700, 1500][seed % 8])
    n_m = int([1, 31, 32, 33, 65, 100, 200, 47][seed % 8])
    n_tables = -(-(4096 if n <= 512 else 8192) // n_m) + int(rng.integers(0, 9))
    x = np.floor(np.cumsum(rng.integers(1, 3000 if n < 400 else 60, size=(n_tables, n)).astype(np.float64), axis=1))
    gaps = np.abs(20.0 + x * rng.uniform(0.02, 0.1, size=(n_tables, 1)) * (1.0 + 0.4 * rng.standard_normal(x.shape)))
    L = rng.uniform(0.0, 90.0, size=n_tables)
    top = float(x.max()) * float(rng.choice([0.05, 1.0, 20.0]))
    m = np.maximum(np.floor(np.exp(rng.uniform(np.log(8.0), np.log(max(top, 64.0)), size=n_m)) / 8.0) * 8.0, 8.0)
    p_hi = int([2, 66, 257, 1026, 1500, 2049, 130, 600][seed % 8])
    n_P = int(min(p_hi - 1, rng.choice([1, 5, 24, 37, 255, 256, 300])))
    P = np.sort(rng.choice(np.arange(2, p_hi + 1), size=n_P, replace=False))
    P[-1] = p_hi                                            # the last block: 1, 64, 1, 63, 32 ... terms
    P = np.unique(P).astype(np.uint32)
    s = np.unique(rng.integers(1, 4000, size=int(rng.choice([0, 1, 4, 5, 19, 24]))) * 8).astype(np.uint64)
    mask = int(rng.choice([ALL_STRATEGIES_MASK, ALL_STRATEGIES_MASK, 0x3FFFF, 0x3FFFF, 0x3FF, 0x1C00, 0x0A25, 1 << 2, 1 << 9,
                           1 << 11, 1 << 14, 0x36800, int(rng.integers(1, 1 << 18))]))
    return Workload("tile", x, gaps, L, m.astype(np.uint64), P, s, int(rng.choice([NO_CAP, NO_CAP, 2048])), mask)


@pytest.mark.parametrize("seed", range(24))
def test_random_tiles(seed):
    rng = np.random.default_rng(5000 + seed)
    wl = _tile_problem(rng, seed)
    want, _ = oracle.tune_workload(wl)
    what = "tile %d: n=%d tables=%d m=%d P=%d (max %d) s=%d mask=%#x" % (
        seed, wl.sizes.shape[1], wl.n_tables, len(wl.m), len(wl.P), int(wl.P[-1]), len(wl.s), wl.strategy_mask)
    print(what, flush=True)
    assert assert_tables_equal(gpu_tune(wl), want, what), "times not bit-identical"


@pytest.mark.parametrize("n,n_m,p_hi,n_P,mask", [
    (2, 1, 66, 5, ALL_STRATEGIES_MASK),        # a tile of one size
    (9, 31, 600, 24, ALL_STRATEGIES_MASK), (57, 33, 1026, 37, ALL_STRATEGIES_MASK), (120, 200, 2048, 250, ALL_STRATEGIES_MASK),
    (300, 32, 65, 9, ALL_STRATEGIES_MASK),     # two blocks, the second of one term: 64 items, all of them searched
    (300, 32, 129, 9, ALL_STRATEGIES_MASK),    # three blocks: 96, a lane each
    (39, 32, 400, 9, ALL_STRATEGIES_MASK), (40, 32, 400, 9, ALL_STRATEGIES_MASK),       # seven blocks, 224
    (45, 32, 512, 30, ALL_STRATEGIES_MASK), (45, 32, 514, 30, ALL_STRATEGIES_MASK),     # eight and nine
    (300, 31, 64, 40, 0x1C00),                 # one block, most of its points wanted
    (300, 33, 200, 300, ALL_STRATEGIES_MASK),  # tiles of 17 and 16; four blocks, every point wanted
    (512, 40, 256, 255, ALL_STRATEGIES_MASK),  # three workgroups' worth of LDS: tiles of fewer sizes
    (320, 64, 2049, 100, ALL_STRATEGIES_MASK), # 33 blocks: one too many
    (640, 21, 2048, 250, ALL_STRATEGIES_MASK), (1024, 21, 1500, 65, ALL_STRATEGIES_MASK),   # a big table, one tile
    (1025, 21, 1500, 64, ALL_STRATEGIES_MASK), (1025, 21, 1500, 65, ALL_STRATEGIES_MASK),   # to it
    (700, 70, 100, 31, ALL_STRATEGIES_MASK), (700, 70, 100, 32, ALL_STRATEGIES_MASK),   # several: two blocks and
    (1280, 70, 128, 6, ALL_STRATEGIES_MASK), (700, 70, 130, 6, ALL_STRATEGIES_MASK),    # few process counts (four
    (700, 130, 257, 6, ALL_STRATEGIES_MASK), (1281, 130, 129, 6, ALL_STRATEGIES_MASK),  # for many rows),
    (1100, 90, 500, 40, ALL_STRATEGIES_MASK), (1100, 90, 520, 40, ALL_STRATEGIES_MASK), # or eight blocks
    (1024, 130, 300, 30, 0x3FF), (1025, 130, 300, 30, 0x3FF),   # without chain sums: several tiles
    (2048, 65, 300, 30, 0x3FF), (2049, 65, 300, 30, 0x3FF),     # (few rows)
    (2048, 30, 300, 30, 0x13FF), (2049, 30, 300, 30, 0x13FF),   # and one
])
@pytest.mark.parametrize("dense", [True, False])
def test_tiles_at_the_edges_of_their_rules(n, n_m, p_hi, n_P, mask, dense):
    # (tables of more than 512 samples: 8192 rows, or 16 384 where n_m is 130)
    # dense: samples 8 apart, so that a block of the chain sum crosses many intervals at every size;
    # else 2000 apart, most blocks of small sizes stay in one
    rng = np.random.default_rng(n + n_m + p_hi)
    n_tables = -(-(4096 if n <= 512 else 16384 if n_m == 130 else 8192) // n_m) + 3
    step = 8 if dense else 2000
    x = np.cumsum(rng.integers(1, step + 1, size=(n_tables, n)), axis=1).astype(np.float64)
    gaps = np.abs(20.0 + x * rng.uniform(0.02, 0.1, size=(n_tables, 1)) * (1.0 + 0.4 * rng.standard_normal(x.shape)))
    m = 8 * np.sort(rng.integers(1, max(2, int(x[:, -1].max()) // 64), size=n_m))
    P = np.union1d(np.sort(rng.choice(np.arange(2, p_hi), size=min(n_P - 1, p_hi - 2), replace=False)), [p_hi])
    s = (8 * np.unique(rng.integers(1, 2000, size=17))).astype(np.uint64)
    wl = Workload("tiles", x, gaps, rng.uniform(0.0, 90.0, size=n_tables), m.astype(np.uint64), P.astype(np.uint32), s,
                  NO_CAP, mask)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "tiles n=%d m=%d P=%d" % (n, n_m, len(P))), "times not bit-identical"


@pytest.mark.parametrize("n,n_m,p_hi,n_P,n_tables", [
    (20, 22, 667, 7, 200), (60, 22, 667, 7, 200),             # 242 items, up to a wave of which enter several intervals
    (30, 24, 800, 20, 180), (30, 26, 800, 20, 170),           # 312 and 338 of one tile
    (30, 32, 1020, 16, 140), (30, 32, 1020, 17, 140), (30, 32, 1030, 16, 140),          # 512, more points, 544
    (12, 64, 667, 8, 70), (12, 96, 667, 8, 50),               # 352 in two and in three tiles
    (20, 28, 300, 9, 1500), (20, 28, 300, 9, 1560), (49, 28, 300, 9, 1560),             # workgroups that wait for others
])
def test_tiles_that_share_their_longest_items(n, n_m, p_hi, n_P, n_tables):
    # samples and message sizes spread evenly over their logarithm: most blocks enter no interval, some one,
    # the first ones several
    rng = np.random.default_rng(n + n_m + p_hi + n_P + n_tables)
    x = np.floor(np.geomspace(1.0, 2.0 ** 22, n) * rng.uniform(1.0, 1.2, size=(n_tables, 1))) + 20.0 * np.arange(n)
    gaps = np.abs(20.0 + x * rng.uniform(0.02, 0.1, size=(n_tables, 1)) * (1.0 + 0.2 * rng.standard_normal(x.shape)))
    m = np.maximum(8, 8 * np.floor(np.geomspace(8, 2.0 ** 23, n_m) / 8))
    P = np.union1d(rng.choice(np.arange(2, p_hi), size=n_P - 1, replace=False), [p_hi])
    wl = Workload("tiles", x, gaps, rng.uniform(0.0, 90.0, size=n_tables), m.astype(np.uint64), P.astype(np.uint32),
                  np.array([8, 64, 512, 4096], dtype=np.uint64), NO_CAP, ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "tiles n=%d m=%d P=%d" % (n, n_m, len(P))), "times not bit-identical"


@pytest.mark.parametrize("n,m", [(40, 192), (40, 200), (40, 224), (40, 256), (40, 512), (3, 192), (9, 2000), (300, 160),
                                 (300, 2400)])
def test_tiles_whose_terms_enter_intervals_at_an_even_pace(n, m):
    # samples 512 apart: eight terms of size m enter up to three intervals (m = 192), three or four (200,
    # 224), more (256 on); the table ends inside the sum, or inside its first block (n = 3, 9)
    rng = np.random.default_rng(n * m)
    n_tables = 1030
    x = np.tile(512.0 * np.arange(1, n + 1), (n_tables, 1))
    gaps = np.abs(20.0 + x * 0.05 * (1.0 + 0.4 * rng.standard_normal(x.shape)))
    x[:, 0] -= rng.integers(0, 500, size=n_tables)             # the tables share no sample sizes
    P = np.array([2, 3, 10, 64, 65, 66, 100, 128, 129, 200], dtype=np.uint32)
    wl = Workload("pace", x, gaps, rng.uniform(0.0, 90.0, size=n_tables), np.array([m, m, m + 8, m], dtype=np.uint64), P,
                  np.array([8, 16], dtype=np.uint64), NO_CAP, ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "n=%d m=%d" % (n, m)), "times not bit-identical"


@pytest.mark.parametrize("together", [1, 11, 12, 13, 31, 32, 33, 70])
@pytest.mark.parametrize("route", ["sums", "tiles", "points"])
def test_walks_past_samples_that_lie_together(together, route):
    # groups of samples one byte apart, 4000 from the next: a term enters all intervals of a group at once,
    # most of them without a term in them (a walk looks for the next after twelve; a wave of which some block
    # enters 32 or more, in tiles 16, or 4 from 40 samples on, searches).  Sums wanted around every eighth term
    rng = np.random.default_rng(together)
    n = {"sums": 1100, "tiles": 200, "points": 180}[route]
    n_tables = 700 if route == "tiles" else 1
    x = np.array([4000.0 * (1 + k // together) + k % together for k in range(n)])[None].repeat(n_tables, axis=0)
    x[:, 0] -= rng.integers(0, 500, size=n_tables)             # the tables share no sample sizes
    gaps = np.abs(20.0 + x * 0.05 * (1.0 + 0.4 * rng.standard_normal(x.shape)))
    m = np.array([8, 96, 328, 1000, 1992, 2000, 3992, 4000, 4008, 9000], dtype=np.uint64)
    P = np.unique(np.concatenate([64 * b + np.array([2, 8, 9, 10, 16, 17, 40, 63, 64, 65]) for b in (0, 1, 2, 5, 9)]))
    L = rng.uniform(0.0, 90.0, size=n_tables)
    if route == "points":
        torch, plogp = torch_cuda(), _plogp()
        mm, PP = [v.ravel() for v in np.meshgrid(m, P.astype(np.uint32))]
        tab = plogp.plogp_load_table(x[0], gaps[0], L[0])
        out = torch.empty(mm.size, dtype=torch.float64, device="cuda")
        dm, dP = _dev(mm, np.uint64), _dev(PP, np.uint32)
        plogp.plogp_eval_strategy(tab, 0, 11, dm.data_ptr(), dP.data_ptr(), 0, mm.size, out.data_ptr(), stream_handle())
        torch.cuda.synchronize()
        want = np.array([oracle.eval_strategy(x[0], gaps[0], L[0], 11, int(a), int(b), 0) for a, b in zip(mm, PP)])
        assert (out.cpu().numpy().view(np.uint64) == want.view(np.uint64)).all()
        tab.free()
        return
    wl = Workload("together", x, gaps, L, m, P.astype(np.uint32), np.array([8, 16], dtype=np.uint64), NO_CAP,
                  ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "%d together, %s" % (together, route)), "times not bit-identical"


# ------------------------------------------------------------------ candidates that can win row 5

@pytest.mark.parametrize("n_m,n_P,p_hi", [(9, 1, 2), (9, 1, 700), (9, 64, 65), (9, 130, 1900), (9, 513, 514), (5, 700, 2048),
                                          (4200, 33, 40), (4100, 70, 4000), (300, 520, 4000)])
@pytest.mark.parametrize("n_s", [1, 2, 63, 64, 65, 130, 256])
@pytest.mark.parametrize("table", ["noise", "flat", "falling", "line"])
def test_candidates_that_can_win_row_5(n_m, n_P, p_hi, n_s, table):
    # a row to a workgroup and lanes over process counts, one and two to a lane; up to 64 candidates in one
    # turn, more in several.  flat: equal gaps, so that candidates of the same number of segments tie;
    # falling: gaps and times below zero past the last sample; line: times that differ in their last bits
    rng = np.random.default_rng(n_m + n_P + n_s)
    n = 40
    x = np.cumsum(rng.integers(1, 3000, size=n)).astype(np.float64)[None]
    gaps = {"noise": np.abs(25.0 + 0.07 * x * (1.0 + 0.3 * rng.standard_normal(x.shape))), "flat": np.full(x.shape, 12.5),
            "falling": 30.0 * (1.0 - 0.9 * x / x[0, -1]), "line": 1.0 + x * 2.0 ** -9}[table]
    m = np.maximum(8 * np.floor(np.exp(rng.uniform(np.log(8.0), np.log(5e6), size=n_m)) / 8), 8).astype(np.uint64)
    P = np.union1d(rng.choice(np.arange(2, p_hi + 1), size=n_P - 1, replace=False), [p_hi]).astype(np.uint32)
    s = 8 * np.unique(np.concatenate([np.arange(1, n_s // 2 + 1), np.floor(np.geomspace(200, 60000, 2 * n_s))]))[:n_s]
    wl = Workload("row 5", x, gaps, np.array([0.0 if table == "line" else 40.0]), m, P, s.astype(np.uint64), NO_CAP,
                  ALL_STRATEGIES_MASK if n_s != 63 else 0x20)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "n_s=%d %s" % (n_s, table)), "times not bit-identical"


# ------------------------------------------------------------------ many candidates, chunks left out by their bounds

@pytest.mark.parametrize("n_s,n_P,shape", [
    (257, 3, "rise"), (320, 49, "noise"), (1000, 72, "flat"), (4160, 73, "fall"), (8191, 9, "rise"), (8192, 10, "tie"),
    (8193, 70, "noise"), (16448, 5, "fall"), (20000, 97, "rise"), (9000, 8, "tie"), (70000, 4, "noise"),
])
def test_many_candidates_chunks_and_passes(n_s, n_P, shape):
    # 64 candidates to a chunk, 8192 to a pass, 64 ranges of 1024 remembered: numbers of candidates
    # at and around these; gap curves whose best segment size sits at either end, wanders, or ties
    # over many sizes; sizes at which only part of a chunk or of a pass competes
    rng = np.random.default_rng(n_s + n_P)
    x = np.array([1.0, 100.0, 700.0, 5000.0, 40000.0, 300000.0])
    gaps = np.stack([{"rise": 5.0 + 0.01 * x, "flat": np.full(6, 7.0), "fall": 900.0 - 0.002 * x, "tie": x / 4.0,
                      "noise": 20.0 + 0.02 * x * rng.uniform(0.3, 2.0, 6)}[shape] * f for f in (1.0, 1.5)])
    step = 8 if n_s < 30000 else 4
    s = (step * np.arange(1, n_s + 1)).astype(np.uint64)
    top = int(s[-1])
    m = np.array([4, 8, 64, 512, 520, 1024, 4096, top // 8 * 4, top, top + 4, 3 * top, 1 << 22, 1 << 30, (1 << 40) + 4],
                 dtype=np.uint64)
    P = np.unique(np.concatenate([[2, 3, 4], rng.integers(2, 5000, size=4 * n_P)]))[:n_P].astype(np.uint32)
    for mask, cap in ((ALL_STRATEGIES_MASK, NO_CAP), (1 << 5, top // 2), ((1 << 2) | (1 << 9), NO_CAP), (0x225, 600)):
        wl = Workload("chunks", np.repeat(x[None], 2, axis=0), gaps, np.array([3.0, 0.0]), m, P, s, cap, mask)
        wl.dtype_size = 4
        want, _ = oracle.tune_workload(wl)
        assert assert_tables_equal(gpu_tune(wl), want, "%s n_s=%d mask %x" % (shape, n_s, mask)), "times not bit-identical"


@pytest.mark.parametrize("n_P", [16, 17, 32, 33, 48, 49, 72])
@pytest.mark.parametrize("n_m,n_s", [(256, 577), (257, 577), (300, 5500)])
def test_many_candidates_groups_of_process_counts(n_P, n_m, n_s):
    # a wave takes 2, 4, 6 or 9 process counts, eight waves all of them; more than 512 (table, size)
    # rows and LDS for three workgroups per compute unit (up to about 6500 candidates) take a
    # kernel of fewer registers.  577 candidates: ten chunks, two to a wave and none to the last three
    rng = np.random.default_rng(n_P * 1000 + n_m)
    x = np.array([1.0, 90.0, 2000.0, 30000.0, 500000.0])
    gaps = 20.0 + 0.02 * x * rng.uniform(0.3, 2.0, (2, 5))
    m = (8 * np.unique(np.floor(np.exp(rng.uniform(0.0, np.log(1 << 20), 2 * n_m))))[:n_m]).astype(np.uint64)
    m = np.concatenate([m, 8 * rng.integers(1, 1 << 20, n_m - len(m)).astype(np.uint64)])
    P = np.sort(rng.choice(np.arange(2, 900), size=n_P, replace=False)).astype(np.uint32)
    s = (8 * np.arange(1, n_s + 1)).astype(np.uint64)
    wl = Workload("groups", np.repeat(x[None], 2, axis=0), gaps, np.array([7.0, 60.0]), m, P, s, NO_CAP,
                  ALL_STRATEGIES_MASK)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "n_P=%d" % n_P), "times not bit-identical"


@pytest.mark.parametrize("n_s,last", [(600, 1000.0), (8192, 14000.0), (9000, 14000.0), (17000, 40000.0)])
@pytest.mark.parametrize("mask", [ALL_STRATEGIES_MASK, 0x204, 1 << 2, 1 << 9])
def test_many_candidates_whose_gap_falls_below_zero(n_s, last, mask):
    # samples are not negative, but the line through the last two goes on falling beyond them: the
    # candidates' g changes sign inside the list, and the best of rows 2 and 9 is one of large |g| k
    rng = np.random.default_rng(n_s)
    x = np.array([1.0, last])
    gaps = np.array([[104.0, 52.0], [103.64280263405897, 51.69110966029943], [80.0, 0.5], [60.0, 59.0]])
    s = (8 * np.arange(1, n_s + 1)).astype(np.uint64)
    ends = 8 * (64 * rng.integers(1, n_s // 64, 24) + 1)            # the last competing chunk holds one candidate
    m = np.unique(np.concatenate([ends, ends - 8, 8 * rng.integers(1, 3 * n_s, 24), [3080]])).astype(np.uint64)
    P = np.array([2, 3, 4, 7, 31, 64, 302, 1023, 1500], dtype=np.uint32)
    wl = Workload("falling", np.repeat(x[None], 4, axis=0), gaps, np.array([3.0, 3.0, 0.0, 900.0]), m, P, s, NO_CAP, mask)
    want, _ = oracle.tune_workload(wl)
    segmented = (want["strategy"][:, 0] == 2) | (want["strategy"][:, 0] == 9)
    assert (want["time"][:, 0][segmented] < 0.0).sum() > 100
    assert assert_tables_equal(gpu_tune(wl), want, "falling n_s=%d mask %x" % (n_s, mask)), "times not bit-identical"


@pytest.mark.parametrize("n_m,n_P,p_hi,n_s,n", [
    (1, 1, 2, 0, 2), (3, 2, 66, 1, 9), (64, 49, 50, 13, 21), (20, 63, 65, 64, 64), (33, 64, 129, 8, 200),
    (5, 65, 2048, 34, 512), (255, 16, 17, 34, 64), (257, 127, 128, 63, 64), (100, 255, 700, 9, 40),
])
@pytest.mark.parametrize("mask", [ALL_STRATEGIES_MASK, 0xA9, 0x3FF, 0x1C00, 0x0A25])
def test_small_jobs_a_row_per_workgroup(n_m, n_P, p_hi, n_s, n, mask):
    # the path whose workgroups take a (table, m) row, from one row and one process count on: lanes,
    # groups of 64 process counts and candidates at and around their limits, two tables
    rng = np.random.default_rng(n_m * 1000 + n_P)
    x = np.unique(np.floor(np.cumsum(rng.integers(1, 900, size=n).astype(np.float64))))
    gaps = np.abs(25.0 + np.outer([0.03, 0.11], x) * (1.0 + 0.3 * rng.standard_normal((2, len(x)))))
    m = np.maximum(np.floor(np.exp(rng.uniform(np.log(8.0), np.log(40.0 * x[-1]), size=n_m)) / 8.0) * 8.0, 8.0)
    P = np.sort(rng.choice(np.arange(2, p_hi + 1), size=n_P, replace=False)).astype(np.uint32)
    s = (8 * np.sort(rng.choice(np.arange(1, 4000), size=n_s, replace=False))).astype(np.uint64)
    wl = Workload("small rows", np.repeat(x[None], 2, axis=0), gaps, np.array([4.0, 60.0]), m.astype(np.uint64), P, s,
                  NO_CAP, mask)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "small rows, mask %x" % mask), "times not bit-identical"


@pytest.mark.parametrize("n_s,n_P,p_hi", [(1, 1, 2), (8, 1000, 1001), (9, 256, 300), (9, 257, 300), (24, 256, 2000), (25, 256, 2000),
                                          (12, 64, 640), (13, 64, 255), (13, 64, 256), (24, 64, 640), (25, 64, 640),
                                          (13, 65, 640), (13, 32, 127), (13, 32, 128), (25, 20, 255), (25, 20, 256),
                                          (40, 20, 499), (40, 20, 500), (64, 64, 2049)])
@pytest.mark.parametrize("mask", [ALL_STRATEGIES_MASK, 0x3FF, 0x20, 0x203FF, 0x3FFFF, 0x10024])
def test_which_rows_evaluate_every_candidate(n_s, n_P, p_hi, mask):
    # on both sides of the limits at which a workgroup per row evaluates all candidates of row 5, or leaves
    # out those that cannot win; equal gaps at the smallest sizes, so that candidates tie
    rng = np.random.default_rng(n_s * 1000 + n_P)
    x = np.cumsum(rng.integers(1, 3000, size=40)).astype(np.float64)[None]
    gaps = np.maximum(25.0 + 0.07 * x * (1.0 + 0.3 * rng.standard_normal(x.shape)), 900.0)
    m = np.maximum(8, 8 * np.floor(np.exp(rng.uniform(np.log(8.0), np.log(5e6), size=45)) / 8)).astype(np.uint64)
    P = np.union1d(rng.choice(np.arange(2, p_hi), size=n_P - 1, replace=False), [p_hi]).astype(np.uint32)
    s = (8 * np.unique(np.floor(np.geomspace(1, 60000, 2 * n_s))))[:n_s].astype(np.uint64)
    wl = Workload("row 5", x, gaps, np.array([3.0]), m, P, s, NO_CAP, mask)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "n_s=%d mask %x" % (len(s), mask)), "times not bit-identical"


@pytest.mark.parametrize("n_s,n_P,p_hi", [(4, 40, 41), (5, 40, 41), (4, 600, 700), (5, 600, 700), (24, 256, 300), (25, 255, 300),
                                          (25, 256, 300), (25, 256, 2000)])
@pytest.mark.parametrize("mask", [ALL_STRATEGIES_MASK, 0x3FF, 0x9FF])
def test_which_sweeps_evaluate_every_candidate(n_s, n_P, p_hi, mask):
    # the same of the sweep over process counts, on a table too long for a workgroup per row
    rng = np.random.default_rng(n_s * 1000 + n_P)
    x = np.cumsum(rng.integers(1, 3000, size=600)).astype(np.float64)[None]
    gaps = np.maximum(25.0 + 0.07 * x * (1.0 + 0.3 * rng.standard_normal(x.shape)), 900.0)
    m = np.maximum(8, 8 * np.floor(np.exp(rng.uniform(np.log(8.0), np.log(5e6), size=300)) / 8)).astype(np.uint64)
    P = np.union1d(rng.choice(np.arange(2, p_hi), size=n_P - 1, replace=False), [p_hi]).astype(np.uint32)
    s = (8 * np.unique(np.floor(np.geomspace(1, 60000, 2 * n_s))))[:n_s].astype(np.uint64)
    wl = Workload("row 5", x, gaps, np.array([3.0]), m, P, s, NO_CAP, mask)
    want, _ = oracle.tune_workload(wl)
    assert assert_tables_equal(gpu_tune(wl), want, "n_s=%d mask %x" % (len(s), mask)), "times not bit-identical"
