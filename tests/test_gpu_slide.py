"""GPU parity of the exponential maps by sliding windows along t0
(kernels_slide.hip) and of the rect prefix sums at their block edges.

Sums are FP64, so maps are held to the FP64 tolerances of checks.py whatever
the requested precision: 2F to 1e-9 of max(2F, 1) (the recurrence: 1e-8, see
TOL["recur64"]) plus the stored map's float32 rounding.  Maps by the direct
sums (an explicit tiling, or atoms that the sliding sums do not take) are held
to the FP32 tolerance.
"""
import dataclasses

import numpy as np
import pytest

import oracle
import tfsynth
from checks import TOL, check_map, check_results

pytestmark = pytest.mark.gpu

T = tfsynth.T_SFT
DENSE = 1 << 30


@pytest.fixture(scope="module")
def ctx():
    import paper_1805_05652_amd as tf
    c = tf.Context(0, arena_bytes=2 << 30)
    yield c
    c.close()


def _maps(ctx, atoms, win, prec, tiling=None):
    aid = ctx.upload_atoms(atoms)
    try:
        if tiling is not None:
            ctx.tiling_config(*tiling)
        ctx.profile_reset()
        ctx.profile(True)
        res, twoF = ctx.fmap(aid, win, prec, want_map=True)
        return res, twoF.cpu().numpy(), ctx.profile_read()["recur"][0]
    finally:
        ctx.profile(False)
        ctx.tiling_config(-1, -1)
        ctx.free(aid)


@pytest.mark.parametrize("n_bins", [1, 2, 3, 4, 5, 7, 9])
@pytest.mark.parametrize("grid", ["slots", "off", "far", "tau_wide", "same_slot", "outside"])
def test_slide_against_oracle_and_direct(ctx, n_bins, grid):
    """Every group size (1 to 4 bins, a short last group); tau tiles one tau
    short of, at and past 64; ragged last segments; rows one slot apart, off
    the slots, far apart (one row per segment), several in one slot, before
    and after the data; taus whose ends fit the LDS stage and taus too far
    apart for it, shorter than a slot and longer than the data."""
    print("case: slide %s %d bins" % (grid, n_bins), flush=True)
    atoms = tfsynth.make_atoms(9300 + n_bins, 1100, 0.15, n_bins=n_bins,
                               injections=[tfsynth.Injection(n_bins - 1, "exp", 300 * T, 60 * T, 1.0)])
    if grid == "slots":
        win = tfsynth.regular_window("exp", 0, T, 261, 2 * T, T, 63 + n_bins % 3)
    elif grid == "off":
        win = tfsynth.linspace_grid(atoms, "exp", 203, 65)
    elif grid == "far":
        win = tfsynth.regular_window("exp", 11, 97 * T, 11, T, 3 * T + 7, 64)
    elif grid == "tau_wide":
        win = tfsynth.regular_window("exp", 3 * T, 2 * T, 150, 2 * T, 13 * T, 30)
    elif grid == "same_slot":
        win = tfsynth.regular_window("exp", 40 * T + 1, 111, 150, T // 2, 2 * T - 1, 70)
    else:
        t0 = np.concatenate([-500 * T + 37 * T * np.arange(20), np.arange(3, 1300, 50) * T + 9])
        win = tfsynth.list_window("exp", np.unique(t0), [1, T - 1, T, 5 * T + 3, 40 * T, 2000 * T])
    ref = oracle.fmap_atoms(atoms, win)
    for prec in ("fp32", "fp64", "recur64"):
        res, got, n = _maps(ctx, atoms, win, prec)
        assert n == 1, "not by sliding windows"
        tol = TOL["recur64"] if prec == "recur64" else TOL["fp64"]
        check_map(got, ref, tol)
        check_results(res, ref, win, tol)
    res, direct, n = _maps(ctx, atoms, win, "fp32", (DENSE, -1))
    assert n == 0
    check_map(direct, ref, TOL["fp32"])


@pytest.mark.parametrize("n_bins,last_tau", [(1, 1000), (1, 1400), (3, 900), (3, 1000), (4, 500), (5, 700), (6, 1500)])
def test_slide_window_ends_past_the_stage(ctx, n_bins, last_tau):
    """Window ends of one tau tile spread over 3 * last_tau slots: at the edge
    of what a workgroup's LDS holds at 4, 3, 2 and 1 bins (1860, 2274, 2924 and
    4095 slots), and past it, where the ends come through the caches."""
    print("case: spread %d bins, tau to %d" % (n_bins, last_tau), flush=True)
    atoms = tfsynth.make_atoms(9350 + n_bins, 4600, 0.1, n_bins=n_bins)
    tau = np.unique(np.linspace(2, last_tau, 50).astype(np.int64) * T)
    for first in (0, -1500):   # (windows longer than the data whose ends lie inside)
        win = tfsynth.list_window("exp", 3 + first * T + 5 * T * np.arange(30), tau)
        ref = oracle.fmap_atoms(atoms, win)
        res, got, n = _maps(ctx, atoms, win, "fp32")
        assert n == 1, "not by sliding windows"
        check_map(got, ref, TOL["fp64"])
        check_results(res, ref, win, TOL["fp64"])


@pytest.mark.parametrize("n_bins", [1, 2, 3, 4, 5, 9])
@pytest.mark.parametrize("grid", ["slots", "rows17", "off", "tau_wide", "tau_far", "outside", "same_slot"])
def test_rect_tiles(ctx, n_bins, grid):
    """Every group size; tau tiles one tau short of, at and past 64; rows one
    short of, at and past a pass of sixteen waves and a tile; window ends at
    and past what the LDS stage holds at 4, 2 and 1 bins (505, 863 and 1333
    slots); windows from before the data, longer than it and empty.  A batch
    gives the same numbers."""
    print("case: rect %s %d bins" % (grid, n_bins), flush=True)
    atoms = tfsynth.make_atoms(9500 + n_bins, 2300, 0.15, n_bins=n_bins,
                               injections=[tfsynth.Injection(n_bins - 1, "rect", 300 * T, 60 * T, 1.0)])
    if grid == "slots":
        win = tfsynth.regular_window("rect", 0, T, 255 + n_bins % 3, T, T, 63 + n_bins % 3)
    elif grid == "rows17":
        win = tfsynth.regular_window("rect", 7, 3 * T, 15 + n_bins % 3, T, 5 * T + 9, 130)
    elif grid == "off":
        win = tfsynth.linspace_grid(atoms, "rect", 101, 65)
    elif grid == "tau_wide":
        win = tfsynth.regular_window("rect", 3 * T, 2 * T, 40, 2 * T, (7 + 4 * (n_bins % 4)) * T, 64)
    elif grid == "tau_far":
        win = tfsynth.regular_window("rect", 3, 2 * T, 33, 2 * T, 30 * T, 64)
    elif grid == "same_slot":
        win = tfsynth.regular_window("rect", 40 * T + 1, 111, 50, T // 2, 2 * T - 1, 70)
    else:
        t0 = np.concatenate([-2600 * T + 137 * T * np.arange(18), np.arange(3, 2500, 99) * T + 9])
        win = tfsynth.list_window("rect", np.unique(t0), [1, T - 1, T, 5 * T + 3, 40 * T, 900 * T, 2000 * T, 6000 * T])
    ref = oracle.fmap_atoms(atoms, win)
    aid = ctx.upload_atoms(atoms)
    try:
        res, twoF = ctx.fmap(aid, win, "fp32", want_map=True)
        check_map(twoF.cpu().numpy(), ref, TOL["fp64"])
        check_results(res, ref, win, TOL["fp64"])
        with ctx.batch([(aid, win), (aid, win)], "fp32") as b:
            assert b.run() == [res, res]
    finally:
        ctx.free(aid)


@pytest.mark.parametrize("slots", [1, 2, 31, 32, 33, 255, 256, 257, 513])
@pytest.mark.parametrize("kind", ["exp", "rect"])
def test_slot_count_edges(ctx, kind, slots):
    """Slot counts at the edges of the anchors' ranges (32 slots, 8 to a
    super-range) and of the prefix sums' blocks (256 slots)."""
    print("case: %s %d slots" % (kind, slots), flush=True)
    atoms = tfsynth.make_atoms(9400 + slots, slots, 0.0, n_bins=2)
    n = max(1, min(slots, 40))
    t0 = np.unique(np.linspace(0, (slots - 1) * T, n).astype(np.int64))
    win = tfsynth.list_window(kind, t0, np.unique(np.linspace(T, (slots + 1) * T, n).astype(np.int64)))
    ref = oracle.fmap_atoms(atoms, win)
    res, got, _ = _maps(ctx, atoms, win, "fp64")
    check_map(got, ref, TOL["fp64"])
    check_results(res, ref, win, TOL["fp64"])


@pytest.mark.parametrize("case", ["zero_antenna", "weak_between_strong", "one_antenna", "zero_data"])
def test_slide_weak_windows(ctx, case):
    """Windows whose A or B is nothing, or tiny, beside the slots that left
    them: SFTs with zeroed atoms, an antenna pattern 1e-6 of its neighbours'
    (collinear: every such window is degenerate), no second antenna, no data."""
    print("case: slide weak " + case, flush=True)
    base = tfsynth.make_atoms(9500, 500, 0.1, n_bins=2)
    a, b = base.a.copy(), base.b.copy()
    fa, fb = base.fa.copy(), base.fb.copy()
    hole = slice(150, 230)
    if case == "zero_antenna":
        a[hole] = b[hole] = 0.0
        fa[:, hole] = fb[:, hole] = 0.0
    elif case == "weak_between_strong":
        a[hole] *= 1e-6
        b[hole] = 2.0 * a[hole]
        fa[:, hole] *= 1e-6
        fb[:, hole] = 2.0 * fa[:, hole]
    elif case == "one_antenna":
        b[:] = 0.0
        fb[:] = 0.0
    else:
        fa[:], fb[:] = 0.0, 0.0
    atoms = dataclasses.replace(base, a=a, b=b, a2=a * a, b2=b * b, ab=a * b, fa=fa, fb=fb)
    win = tfsynth.regular_window("exp", 0, T, 300, T // 2, T // 3, 70)
    ref = oracle.fmap_atoms(atoms, win)
    for prec in ("fp64", "recur64"):
        _, got, _ = _maps(ctx, atoms, win, prec)
        # (windows across the rim of weak SFTs have D / A B down to the
        # degenerate threshold, 1e-10: neither side knows 2F to 1e-8 there)
        assert np.all(got[ref == 0.0] == 0.0)
        if case != "weak_between_strong":
            check_map(got, ref, TOL["recur64"])


@pytest.mark.parametrize("case", ["nan", "inf", "spread", "not_single"])
def test_slide_atoms_it_does_not_take(ctx, case):
    """Non-finite values (which a sliding sum would carry to the rows before
    them) and data spread beyond 2^20 keep the direct sums, cell for cell;
    atoms that are not single-precision numbers slide in FP64."""
    print("case: slide atoms " + case, flush=True)
    base = tfsynth.make_atoms(9600, 400, 0.1, n_bins=2)
    fa = base.fa.copy()
    if case == "nan":
        fa[1, 200, 0] = np.nan
    elif case == "inf":
        fa[1, 200, 1] = np.inf
    elif case == "spread":
        fa[1, :120] *= 2.0 ** -30
    else:
        fa *= 1.0 + 2.0 ** -40
    atoms = dataclasses.replace(base, fa=fa)
    win = tfsynth.regular_window("exp", 0, T, 300, 2 * T, T, 70)
    _, got, n = _maps(ctx, atoms, win, "fp32")
    _, direct, _ = _maps(ctx, atoms, win, "fp32", (DENSE, -1))
    if case == "not_single":
        assert n == 1
        check_map(got, oracle.fmap_atoms(atoms, win), TOL["fp64"])
    else:
        assert n == 0
        assert np.array_equal(got, direct, equal_nan=True)


def test_slide_in_a_short_arena():
    """An arena that cannot hold the anchors: FP32 and FP64 maps by the direct
    sums, RECUR64 with the smallest workspace, rect maps without block totals
    (bitwise the same)."""
    import paper_1805_05652_amd as tf
    print("case: slide short arena", flush=True)
    atoms = tfsynth.make_atoms(9700, 4000, 0.1, n_bins=2)
    exp = tfsynth.regular_window("exp", 0, T, 700, 2 * T, 100 * T, 3)
    rect = tfsynth.regular_window("rect", 0, T, 100, 2 * T, T, 100)
    ref = oracle.fmap_atoms(atoms, exp)
    with tf.Context(0, arena_bytes=64 << 20) as roomy:
        aid = roomy.upload_atoms(atoms)
        want_rect, _ = roomy.fmap(aid, rect, "fp64")
    # the atoms (513024 bytes) and the rect map's prefixes and tables (771584)
    with tf.Context(0, arena_bytes=513024 + 771584) as small:
        aid = small.upload_atoms(atoms)
        _, m = small.fmap(aid, exp, "recur64", want_map=True)
        check_map(m.cpu().numpy(), ref, TOL["recur64"])
        _, m = small.fmap(aid, exp, "fp32", want_map=True)
        check_map(m.cpu().numpy(), ref, TOL["fp32"])
        assert small.fmap(aid, rect, "fp64")[0] == want_rect


@pytest.mark.parametrize("cells", [1, 63, 255, 257, 2047, 2048, 2049, 16383, 16385, 18433])
@pytest.mark.parametrize("kind", ["chi2", "wide", "equal", "inf"])
def test_map_reduction_edges(ctx, cells, kind):
    """logB of a stored map at the edges of a thread's chunk (8 cells 256
    apart) and of a tile (16384 cells); values up to 2000 apart, where a power
    underflows, and -inf.  logB is a sum of at most 18433 exponentials, each to
    a few 2^-53, so 1e-12 holds whatever their order."""
    import torch
    print("case: map %s %d cells" % (kind, cells), flush=True)
    rng = np.random.default_rng(cells)
    maps = rng.chisquare(4, size=(2, 1, cells)).astype(np.float32)
    if kind == "wide":
        maps *= rng.choice(np.float32([0.0, 1.0, 200.0]), size=maps.shape)
    elif kind == "equal":
        maps[:] = maps[:, :, :1]
    elif kind == "inf" and cells > 1:
        maps[:, :, ::3] = -np.inf
        maps[:, :, -1] = 30.0
    got = ctx.logB(torch.from_numpy(maps).to("cuda:0"))
    F = maps.reshape(2, -1).astype(np.float64) / 2
    mx = F.max(axis=1)
    want = mx + np.log(np.exp(F - mx[:, None]).sum(axis=1)) - np.log(cells)
    assert np.allclose(got, want, atol=1e-12, rtol=1e-14)
