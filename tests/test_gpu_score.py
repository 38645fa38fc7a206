"""GPU parity of the scoring step (prediction against measurement, paper Section 4):
plogp_score_grid through the C ABI against the CPU oracle on the same inputs.  Predictions,
verdicts and statistics follow a fixed rounding and summation order, so everything is
compared bit for bit; the tolerance of the sweep (1e-12 relative) is asserted as well."""
import numpy as np
import pytest

import oracle
from plogp_workloads import Workload, make_measurements, make_workload
from tests.gpu_util import REL_TOL, stream_handle, torch_cuda

pytestmark = pytest.mark.gpu


def _plogp():
    from paper_cs_0408034_amd import plogp
    return plogp


def gpu_score(wl, meas, seg, table_index=0, with_seg=True):
    torch = torch_cuda()
    plogp = _plogp()
    tab = plogp.plogp_load_tables(wl.sizes, wl.gaps, wl.L)
    grid = plogp.plogp_grid_create(wl.m, wl.P, wl.s, wl.s_cap, wl.dtype_size, wl.strategy_mask)
    n_ids = plogp.plogp_score_strategies(grid)
    assert meas.shape == (n_ids, len(wl.m), len(wl.P))
    n_ops = grid.ops
    d_meas = torch.from_numpy(np.ascontiguousarray(meas)).cuda()
    d_seg = torch.from_numpy(np.ascontiguousarray(seg).view(np.int32)).cuda() if with_seg else None
    d_pred = torch.full(meas.shape, float("nan"), dtype=torch.float64, device="cuda")
    d_ver = torch.full((n_ops * meas.shape[1] * meas.shape[2] * 16,), 0xAB, dtype=torch.uint8, device="cuda")
    d_sc = torch.full((n_ids * 32,), 0xAB, dtype=torch.uint8, device="cuda")
    plogp.plogp_score_grid(tab, table_index, grid, d_meas.data_ptr(),
                           d_seg.data_ptr() if with_seg else 0, d_pred.data_ptr(), d_ver.data_ptr(),
                           d_sc.data_ptr(), stream_handle())
    torch.cuda.synchronize()
    pred = d_pred.cpu().numpy()
    ver = d_ver.cpu().numpy().view(plogp.VERDICT_DTYPE).reshape(n_ops, meas.shape[1], meas.shape[2])
    sc = d_sc.cpu().numpy().view(plogp.SCORE_DTYPE)
    grid.free()
    tab.free()
    return pred, ver, sc


def same_bits(a, b):
    return (np.ascontiguousarray(a).view(np.uint64) == np.ascontiguousarray(b).view(np.uint64)).all()


def check(wl, meas, seg, table_index=0):
    x, y, L = wl.sizes[table_index], wl.gaps[table_index], float(wl.L[table_index])
    want_p, want_v, want_s = oracle.score_grid(x, y, L, wl.m, wl.P, wl.strategy_mask, meas, seg)
    pred, ver, sc = gpu_score(wl, meas, seg, table_index)
    assert (np.abs(pred - want_p) <= REL_TOL * np.abs(want_p)).all()
    assert same_bits(pred, want_p)
    assert (ver["pred_best"] == want_v["pred_best"]).all()
    assert (ver["meas_best"] == want_v["meas_best"]).all()
    assert same_bits(ver["regret"], want_v["regret"])
    assert (sc["count"] == want_s["count"]).all() and (sc["reserved"] == 0).all()
    assert same_bits(sc["max_abs_err"], want_s["max_abs_err"])
    assert same_bits(sc["sum_abs_err"], want_s["sum_abs_err"])
    return want_p, want_v


def from_predictions(wl, seg, seed, table_index=0):
    """Measurements in the paper's two error modes around the oracle's predictions:
    a constant offset, a delay of the small messages, and seeded noise."""
    x, y, L = wl.sizes[table_index], wl.gaps[table_index], float(wl.L[table_index])
    ones = np.ones(seg.shape)
    pred, _, _ = oracle.score_grid(x, y, L, wl.m, wl.P, wl.strategy_mask, ones, seg)
    rng = np.random.default_rng(seed)
    meas = pred * (1.0 + 0.1 * rng.standard_normal(pred.shape).clip(-3, 3)) + 120.0
    small = np.asarray(wl.m)[None, :, None] < 4096
    return np.where(small, meas * 1.4, meas)


@pytest.mark.parametrize("cfg,kw", [
    (1, {}),
    (2, dict(m_slice=slice(0, 1024, 13), P_subset=[2, 3, 4, 7, 64, 65, 66, 129, 700, 1023, 1024])),
    (5, dict(m_slice=slice(0, 4096, 37), P_subset=[2, 65, 66, 4097, 40000, 65536])),
    (3, dict(m_slice=slice(0, 1024, 111), s_subset=slice(0, 8192, 4096))),
])
def test_configs_against_the_oracle(cfg, kw):
    wl = make_workload(cfg, **kw)
    _, seg = make_measurements(wl)
    meas = from_predictions(wl, seg, cfg)
    _, verdict = check(wl, meas, seg)
    # the noise flips some decisions but not all of them
    agree = (verdict["pred_best"] == verdict["meas_best"]).mean()
    assert 0.05 < agree < 1.0


def test_model_free_measurements_and_many_process_counts():
    # the generator the benchmark uses (no model in it); 300 process counts: ragged chunks
    base = make_workload(2, m_slice=slice(0, 1024, 41))
    P = np.arange(2, 302, dtype=np.uint32)
    wl = Workload("score", base.sizes, base.gaps, base.L, base.m, P, base.s, base.s_cap,
                  base.strategy_mask)
    meas, seg = make_measurements(wl, seed=3)
    check(wl, meas, seg)


@pytest.mark.parametrize("cfg,n_m,P_subset,mask", [
    # at least 2048 sizes: a wave takes a whole size and forms the error sums in the same pass
    (5, 4096, [2, 3, 65, 66, 130, 4097, 40000, 65536], 0x1FFF),                  # big table (4096 samples)
    (5, 2100, list(range(2, 72)), 0x1FFF),                                       # 70 process counts: 64 + 6
    (2, 2048, list(range(2, 131)), 0x1FFF),                                      # small table, 129 = 2 x 64 + 1
    (2, 2500, [2, 5, 64, 65, 200], (1 << 0) | (1 << 5) | (1 << 9) | (1 << 11)),  # four strategy rows
    (2, 2500, list(range(2, 67)), 0x1FFF & ~(1 << 6)),                           # twelve rows: 7 + 5
    (2, 3000, [2, 1024], 0x1C00),                                                # the Scatter plane alone
])
def test_many_sizes_take_the_one_pass_path(cfg, n_m, P_subset, mask):
    base = make_workload(cfg, n_m=n_m, P_subset=P_subset)
    wl = Workload("score", base.sizes, base.gaps, base.L, base.m, base.P, base.s, base.s_cap, mask)
    assert len(wl.m) >= 2048
    meas, seg = make_measurements(wl, seed=cfg * 100 + len(P_subset))
    check(wl, meas, seg)


@pytest.mark.timeout(300)
def test_config5_full_size_sampled_rows_and_the_statistics_from_their_definition():
    """Config 5 at full size, the launch the benchmark times (one pass, workgroups of 1024 around
    the 4096-sample table).  The oracle needs minutes for all of it, so: the predictions and
    verdicts of every 64th message size are compared with the oracle's, element by element;
    the statistics are compared with their definition applied to the library's own predictions
    (e per point, added per m in ascending P, then over ascending m, all from +0.0)."""
    wl = make_workload(5)
    meas, seg = make_measurements(wl, seed=5)
    pred, ver, sc = gpu_score(wl, meas, seg)
    rows = slice(0, len(wl.m), 64)
    sub = Workload("score", wl.sizes, wl.gaps, wl.L, wl.m[rows], wl.P, wl.s, wl.s_cap, wl.strategy_mask)
    x, y, L = wl.sizes[0], wl.gaps[0], float(wl.L[0])
    want_p, want_v, _ = oracle.score_grid(x, y, L, sub.m, sub.P, sub.strategy_mask, meas[:, rows], seg[:, rows])
    assert same_bits(pred[:, rows], want_p)
    assert (ver["pred_best"][:, rows] == want_v["pred_best"]).all()
    assert (ver["meas_best"][:, rows] == want_v["meas_best"]).all()
    assert same_bits(ver["regret"][:, rows], want_v["regret"])
    # every point has a finite, positive prediction here, and the verdicts name enabled ids
    assert np.isfinite(pred).all() and (pred > 0).all()
    assert (ver["pred_best"][0] <= 9).all() and (ver["pred_best"][1] >= 10).all()
    e = np.abs((pred - meas) / meas)
    per_m = np.cumsum(e, axis=2)[:, :, -1]                 # cumsum adds strictly left to right
    total = np.cumsum(per_m, axis=1)[:, -1]
    assert same_bits(sc["sum_abs_err"], total)
    assert same_bits(sc["max_abs_err"], e.max(axis=(1, 2)))
    assert (sc["count"] == len(wl.m) * len(wl.P)).all()


def test_unusable_segment_size_on_the_one_pass_path():
    """NaN for that point's prediction and for its strategy's sum, nothing else disturbed."""
    wl = make_workload(2, n_m=2048, P_subset=list(range(2, 70)))
    meas, seg = make_measurements(wl, seed=77)
    ids = oracle.strategy_ids(wl.strategy_mask)
    r5 = ids.index(5)
    good_p, good_v, good_s = gpu_score(wl, meas, seg)
    bad = seg.copy()
    bad[r5, 100, 67] = 0                      # the last process count: a lane of the ragged chunk
    pred, ver, sc = gpu_score(wl, meas, bad)
    assert np.isnan(pred[r5, 100, 67])
    keep = np.ones(pred.shape, dtype=bool)
    keep[r5, 100, 67] = False
    assert same_bits(pred[keep], good_p[keep])
    assert np.isnan(sc["sum_abs_err"][r5])
    others = np.arange(len(ids)) != r5
    assert same_bits(sc["sum_abs_err"][others], good_s["sum_abs_err"][others])
    assert same_bits(sc["max_abs_err"][others], good_s["max_abs_err"][others])


@pytest.mark.parametrize("cfg", [2, 5])                       # a small and a big table
@pytest.mark.parametrize("mask", [0x1FFF, 0x0224, (1 << 5) | (1 << 9) | (1 << 10)])
@pytest.mark.parametrize("unusable", [False, True])
def test_segment_sizes_that_change_along_the_process_counts(cfg, mask, unusable):
    """The one-pass path keeps g(s) and the number of segments while the segment sizes of 64 process
    counts are those of the 64 before, and takes them from the segmented row before where both rows
    have the same sizes.  Sizes here change between the groups of 64 and come back, change inside a
    group, differ between the strategies in some groups and agree in others; with `unusable`, sizes
    of zero and beyond the message fill a group or single points before usable ones."""
    base = make_workload(cfg, n_m=2050, P_subset=list(range(2, 2 + 3 * 64 + 5)))
    wl = Workload("score", base.sizes, base.gaps, base.L, base.m, base.P, base.s, base.s_cap, mask)
    rng = np.random.default_rng(cfg + mask)
    ids = oracle.strategy_ids(mask)
    meas, _ = make_measurements(wl, seed=cfg)
    n_m, n_P = len(wl.m), len(wl.P)
    m = np.asarray(wl.m).astype(np.int64)[:, None]
    group = np.arange(n_P)[None, :] // 64
    of = lambda k: np.maximum(1, m // (3 + k))                                 # noqa: E731
    seg = np.empty((len(ids), n_m, n_P), dtype=np.int64)
    kind = np.arange(n_m)[:, None] % 5
    for r in range(len(ids)):
        there_and_back = of(group % 2)
        per_row = of(np.where(group % 2 == 0, 1, r % 3))                       # agree, differ, agree, differ
        per_group_and_row = of((group + r) % 3)                                # row r has what row r + 1 gets next
        per_point = of(rng.integers(0, 3, (n_m, n_P)))
        last_of_a_group = of(np.where(np.arange(n_P)[None, :] % 64 == 63, r % 2, 2))
        seg[r] = np.choose(np.broadcast_to(kind, (n_m, n_P)),
                           [there_and_back, per_row, per_group_and_row, per_point, last_of_a_group])
    if not unusable:
        check(wl, meas, seg.astype(np.uint32))
        return
    whole = (rng.random((len(ids), n_m, 4)) < 0.3)[:, :, np.arange(n_P) // 64]
    points = rng.random(seg.shape) < 0.02
    bad = np.where(rng.random(seg.shape[:2] + (1,)) < 0.5, 0, np.minimum(2 * m, (1 << 32) - 1)[None])
    bad = np.where((whole | points) & (bad != seg) & ((bad == 0) | (bad > m[None])), bad, -1)
    segmented = np.isin(ids, (2, 5, 9))[:, None, None]
    want, _, _ = oracle.score_grid(wl.sizes[0], wl.gaps[0], float(wl.L[0]), wl.m, wl.P, mask, meas, seg.astype(np.uint32))
    pred, _, _ = gpu_score(wl, meas, np.where(bad >= 0, bad, seg).astype(np.uint32))
    nan = (bad >= 0) & segmented
    assert nan.sum() > 10000
    assert (np.isnan(pred) == nan).all()
    assert same_bits(pred[~nan], want[~nan])


@pytest.mark.parametrize("mask", [0x3FF, 0x1C00, (1 << 0) | (1 << 3) | (1 << 7), (1 << 11), (1 << 5) | (1 << 12)])
def test_masks_and_planes(mask):
    base = make_workload(2, m_slice=slice(5, 1024, 101), P_subset=[2, 5, 64, 65, 200])
    wl = Workload("score", base.sizes, base.gaps, base.L, base.m, base.P, base.s, base.s_cap, mask)
    meas, seg = make_measurements(wl, seed=mask)
    check(wl, meas, seg)


def test_second_table_of_a_batch_and_no_segment_array():
    wl4 = make_workload(4, n_tables=3, n_m=20)
    mask = (1 << 0) | (1 << 6) | (1 << 10) | (1 << 11) | (1 << 12)       # no segmented id
    wl = Workload("score", wl4.sizes, wl4.gaps, wl4.L, wl4.m, wl4.P, wl4.s, wl4.s_cap, mask)
    meas, seg = make_measurements(wl, seed=8)
    x, y, L = wl.sizes[2], wl.gaps[2], float(wl.L[2])
    want_p, want_v, want_s = oracle.score_grid(x, y, L, wl.m, wl.P, mask, meas, seg)
    pred, ver, sc = gpu_score(wl, meas, seg, table_index=2, with_seg=False)
    assert same_bits(pred, want_p) and (ver == want_v).all()
    assert same_bits(sc["sum_abs_err"], want_s["sum_abs_err"])


def test_segment_size_outside_the_domain_gives_nan_for_that_point_only():
    wl = make_workload(1)
    meas, seg = make_measurements(wl, seed=5)
    ids = oracle.strategy_ids(wl.strategy_mask)
    r5 = ids.index(5)
    good_p, _, _ = gpu_score(wl, meas, seg)
    bad = seg.copy()
    bad[r5, 3, 4] = 0
    bad[r5, 0, 0] = np.uint32(int(wl.m[0]) * 2)
    pred, ver, _ = gpu_score(wl, meas, bad)
    assert np.isnan(pred[r5, 3, 4]) and np.isnan(pred[r5, 0, 0])
    mask = np.ones(pred.shape, dtype=bool)
    mask[r5, 3, 4] = mask[r5, 0, 0] = False
    assert same_bits(pred[mask], good_p[mask])
    assert ver["pred_best"][0, 3, 4] != 5            # a NaN prediction is never the best one


def test_bad_arguments_are_refused():
    torch = torch_cuda()
    plogp = _plogp()
    wl = make_workload(1)
    tab = plogp.plogp_load_tables(wl.sizes, wl.gaps, wl.L)
    grid = plogp.plogp_grid_create(wl.m, wl.P, wl.s, wl.s_cap, wl.dtype_size, wl.strategy_mask)
    buf = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
    p = buf.data_ptr()
    lib = plogp._lib
    assert lib.plogp_score_grid(tab._h, 1, grid._h, p, p, p, p, p, None) == plogp.EINVAL      # table index
    assert lib.plogp_score_grid(tab._h, 0, grid._h, p, None, p, p, p, None) == plogp.EINVAL   # id 5 needs seg
    assert lib.plogp_score_grid(tab._h, 0, grid._h, p, p, p, p + 8, p, None) == plogp.EINVAL  # misaligned
    assert lib.plogp_score_grid(tab._h, 0, grid._h, None, p, p, p, p, None) == plogp.EINVAL
    grid.free()
    tab.free()


@pytest.mark.parametrize("seed", range(4))
def test_random_problems(seed):
    """Random tables, sizes (any order, repeats), process counts and masks; a random table of
    the batch is scored."""
    from tests.test_gpu_parity import _random_problem
    rng = np.random.default_rng(3000 + seed)
    for k in range(6):
        wl = _random_problem(rng)
        meas, seg = make_measurements(wl, seed=seed * 10 + k)
        ti = int(rng.integers(0, wl.n_tables))
        print("random %d/%d: n=%d table %d of %d, m=%d P=%d mask=%#x" % (
            seed, k, wl.sizes.shape[1], ti, wl.n_tables, len(wl.m), len(wl.P), wl.strategy_mask), flush=True)
        check(wl, meas, seg, table_index=ti)
