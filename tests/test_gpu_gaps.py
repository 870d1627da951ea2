"""GPU exponential maps of data with long stretches without SFTs: windows that
hold none, and windows of a few SFTs at their ends, are summed directly from
SFT to SFT."""
import types

import numpy as np
import pytest

import oracle
import tfsynth
from checks import TOL, check_map, check_results

pytestmark = pytest.mark.gpu

T = tfsynth.T_SFT


@pytest.fixture(scope="module")
def ctx():
    import paper_1805_05652_amd as tf
    c = tf.Context(0, arena_bytes=2 << 30)
    yield c
    c.close()


def cut(atoms, stretches):
    """The atoms without the SFTs of the slot ranges."""
    k = (atoms.timestamps - atoms.timestamps[0]) // T
    keep = np.ones(k.size, dtype=bool)
    for lo, hi in stretches:
        keep &= (k < lo) | (k >= hi)
    return types.SimpleNamespace(timestamps=atoms.timestamps[keep], a2=atoms.a2[keep], b2=atoms.b2[keep], ab=atoms.ab[keep],
                                 fa=atoms.fa[:, keep], fb=atoms.fb[:, keep], t_sft=T, n_bins=atoms.n_bins)


@pytest.mark.parametrize("n_bins", [1, 2, 3, 4, 5, 9])
@pytest.mark.parametrize("stretches", [[(1, 60)], [(300, 301), (400, 408), (500, 564)], [(200, 700)], [(100, 899)],
                                       [(k, k + 13) for k in range(3, 880, 14)]])
def test_maps_over_gaps(ctx, n_bins, stretches):
    """Windows that lie in a gap, end or start in one, span several, at every
    group size; SFTs alone between gaps."""
    print("case: gaps %s.. %d bins" % (stretches[0], n_bins), flush=True)
    atoms = cut(tfsynth.make_atoms(9810 + n_bins, 900, 0.05, n_bins=n_bins), stretches)
    wins = [tfsynth.regular_window("exp", -20 * T, T, 930, T // 2, T // 3, 67),
            tfsynth.regular_window("exp", 5, 3 * T, 299, 2 * T, 5 * T + 7, 70)]
    for win in wins:
        ref = oracle.fmap_atoms(atoms, win)
        aid = ctx.upload_atoms(atoms)
        try:
            for prec in ("fp32", "fp64", "recur64"):
                ctx.profile_reset()
                ctx.profile(True)
                res, twoF = ctx.fmap(aid, win, prec, want_map=True)
                ctx.profile(False)
                assert ctx.profile_read()["recur"][0] == 1, "not by sliding windows"
                tol = TOL["recur64"] if prec == "recur64" else TOL["fp64"]
                check_map(twoF.cpu().numpy(), ref, tol)
                check_results(res, ref, win, tol)
            with ctx.batch([(aid, win)], "fp64") as b:
                assert b.run()[0] == ctx.fmap(aid, win, "fp64")[0]
        finally:
            ctx.profile(False)
            ctx.free(aid)


def test_gaps_cost_no_more_than_data(ctx):
    """The kernels' time with one gap of 500 slots against none (measured: 13
    times while windows in the gap were summed slot by slot, 1.0 times from SFT
    to SFT; the least of five maps each)."""
    print("case: time over a gap", flush=True)
    base = tfsynth.make_atoms(9890, 3000, 0.1, n_bins=64)
    win = tfsynth.linspace_grid(base, "exp", 600, 700)
    ms = []
    for atoms in (cut(base, []), cut(base, [(1000, 1500)])):
        aid = ctx.upload_atoms(atoms)
        best = np.inf
        try:
            for _ in range(5):
                ctx.profile_reset()
                ctx.profile(True)
                ctx.fmap(aid, win, "fp32")
                ctx.profile(False)
                best = min(best, ctx.profile_read()["recur"][1])
        finally:
            ctx.profile(False)
            ctx.free(aid)
        ms.append(best)
    print("rows kernel: %.3f ms without, %.3f ms with the gap" % tuple(ms), flush=True)
    assert ms[1] < 3 * ms[0]
