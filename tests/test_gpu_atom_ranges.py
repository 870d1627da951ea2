"""GPU ranges of the atoms' values, found at upload: they decide whether an
exponential map is summed by sliding windows, and the FP32 plane written with
them feeds those sums."""
import dataclasses

import numpy as np
import pytest

import oracle
import tfsynth
from checks import TOL, check_map

pytestmark = pytest.mark.gpu

T = tfsynth.T_SFT


@pytest.fixture(scope="module")
def ctx():
    import paper_1805_05652_amd as tf
    c = tf.Context(0, arena_bytes=1 << 30)
    yield c
    c.close()


def slides(ctx, atoms, win, prec="fp32"):
    """(map, whether it was summed by sliding windows)"""
    aid = ctx.upload_atoms(atoms)
    try:
        ctx.profile_reset()
        ctx.profile(True)
        _, twoF = ctx.fmap(aid, win, prec, want_map=True)
        return twoF.cpu().numpy(), ctx.profile_read()["recur"][0] == 1
    finally:
        ctx.profile(False)
        ctx.free(aid)


@pytest.mark.parametrize("slots", [2, 63, 64, 65, 1023, 1024, 1025, 8193, 17000])
@pytest.mark.parametrize("n_bins", [1, 2, 3, 4, 5, 7, 8, 9, 17])
def test_ranges_at_the_edges(ctx, n_bins, slots):
    """Bins at the edges of a workgroup's eight and of the stretches a wave
    takes side by side (8, 4, 2, 1), slots at the edges of stretches (64), of a
    workgroup's sixteen waves (1024) and of more chunks: ordinary data slide;
    one value that is not finite, in the first or last slot of any bin, does
    not."""
    print("case: ranges %d bins %d slots" % (n_bins, slots), flush=True)
    base = tfsynth.make_atoms(9900 + slots + n_bins, slots, 0.0, n_bins=n_bins)
    t0 = np.unique(np.linspace(0, (slots - 1) * T, 5).astype(np.int64))
    win = tfsynth.list_window("exp", t0, np.unique([T, slots * T // 2, slots * T]))
    got, n = slides(ctx, base, win)
    assert n
    check_map(got, oracle.fmap_atoms(base, win), TOL["fp64"])
    small = tfsynth.list_window("exp", t0[:1], [T])
    for b in (0, n_bins // 2, n_bins - 1):
        for k in (0, slots - 1):
            fb = base.fb.copy()
            fb[b, k, 1] = np.inf if b else np.nan
            assert not slides(ctx, dataclasses.replace(base, fb=fb), small)[1], (b, k)


@pytest.mark.parametrize("n_bins", [1, 3, 9])
def test_weak_stretches(ctx, n_bins):
    """A column's 64-slot stretch 2^-21 below the column's largest value: not
    by sliding windows; 2^-18: by them (in single precision)."""
    print("case: weak stretches %d bins" % n_bins, flush=True)
    base = tfsynth.make_atoms(9950 + n_bins, 2300, 0.0, n_bins=n_bins)
    win = tfsynth.list_window("exp", [0, 7 * T], [5 * T])
    for shift, want in ((-18, True), (-21, False)):
        for stretch in (0, 17, 35):
            fa = base.fa.copy()
            col = fa[n_bins - 1, :, 1]
            at = slice(64 * stretch, 64 * stretch + 64)
            col[at] *= np.abs(col).max() / np.abs(col[at]).max() * 2.0 ** shift
            fa = fa.astype(np.float32).astype(np.float64)
            assert slides(ctx, dataclasses.replace(base, fa=fa), win)[1] == want, (shift, stretch)


@pytest.mark.parametrize("prec", ["fp32", "fp64", "recur64", "f16x3"])
@pytest.mark.parametrize("case", ["in_every_stretch", "one_stretch", "one_weak_slot"])
def test_strong_slots(ctx, case, prec):
    """Slots far above their neighbours in data and not in the antenna (2F of
    other windows has to come out as if they were not there): one in every 20
    slots at 2^40, which no stretch of 64 slots shows; a stretch at 2^12, which
    double precision does not slide over; a slot 2^-22 below the others.  The
    map's error is taken relative to max(2F, 1), as everywhere."""
    print("case: strong slots %s %s" % (case, prec), flush=True)
    base = tfsynth.make_atoms(9970, 640, 0.0, n_bins=2)
    fa, fb = base.fa.copy(), base.fb.copy()
    if case == "in_every_stretch":
        at, by = slice(7, None, 20), 2.0 ** 40
    elif case == "one_stretch":
        at, by = slice(320, 384), 2.0 ** 12
    else:
        at, by = slice(333, 334), 2.0 ** -22
    fa[1, at] *= by
    fb[1, at] *= by
    atoms = dataclasses.replace(base, fa=fa, fb=fb)
    win = tfsynth.regular_window("exp", 0, T, 600, T // 2, T // 5, 33)   # windows of 1 to 20 slots
    got, n = slides(ctx, atoms, win, prec)
    check_map(got, oracle.fmap_atoms(atoms, win), TOL[prec])
    assert n == (case != "in_every_stretch" and prec != "fp64")


def test_antenna_products_of_no_antenna(ctx):
    """An |ab| beyond a^2 and b^2 of every SFT (no antenna's) makes D of its
    own windows negative (2F = 0) and nothing else."""
    print("case: ab beyond a^2 and b^2", flush=True)
    base = tfsynth.make_atoms(9980, 200, 0.0, n_bins=1)
    ab = base.ab.copy()
    ab[120] = 1e200
    atoms = dataclasses.replace(base, ab=ab)
    win = tfsynth.regular_window("exp", 0, T, 190, T, T // 3, 20)
    got, n = slides(ctx, atoms, win)
    check_map(got, oracle.fmap_atoms(atoms, win), TOL["fp32"])
    assert not n


@pytest.mark.parametrize("n_bins", [1, 3, 9])
@pytest.mark.parametrize("sfts", [1, 7, 8])
def test_stretches_of_a_few_sfts(ctx, n_bins, sfts):
    """A last stretch of few SFTs has no level of its own: weak by 2^-13, seven
    SFTs slide in double precision and eight do not."""
    print("case: %d SFTs in the last stretch, %d bins" % (sfts, n_bins), flush=True)
    base = tfsynth.make_atoms(9960 + n_bins, 64 * 20 + sfts, 0.0, n_bins=n_bins)
    fa, fb = base.fa.copy(), base.fb.copy()
    b = n_bins - 1
    top = max(np.abs(fa[b]).max(), np.abs(fb[b]).max())
    at = slice(64 * 20, None)
    scale = 2.0 ** -13 * top / max(np.abs(fa[b, at]).max(), np.abs(fb[b, at]).max())
    fa[b, at] = (fa[b, at] * scale).astype(np.float32)
    fb[b, at] = (fb[b, at] * scale).astype(np.float32)
    # (every one of them above the single slots' bound, 2^-18)
    low = np.maximum(np.abs(fa[b, at]).max(axis=1), np.abs(fb[b, at]).max(axis=1))
    fa[b, at, 0] = np.where(low < 2.0 ** -17 * top, np.float32(2.0 ** -16 * top), fa[b, at, 0])
    atoms = dataclasses.replace(base, fa=fa, fb=fb)
    win = tfsynth.list_window("exp", np.arange(1200, 1280) * T, np.arange(1, 40) * T)
    got, n = slides(ctx, atoms, win, "fp64")
    check_map(got, oracle.fmap_atoms(atoms, win), TOL["fp64"])
    assert n == (sfts < 8)
    assert slides(ctx, atoms, win, "fp32")[1]


@pytest.mark.parametrize("n_bins", [1, 2, 8])
@pytest.mark.parametrize("sfts", [7, 8])
def test_a_column_of_a_few_sfts(ctx, n_bins, sfts):
    """SFTs far apart, a few a stretch, one column of one stretch 2^-24 below
    its largest as chance has it: the others bound what is left behind.  Seven
    SFTs slide, eight (a level of their own) do not."""
    print("case: one column of %d SFTs, %d bins" % (sfts, n_bins), flush=True)
    slots = 64 * 12
    base = tfsynth.make_atoms(9980 + n_bins, slots, 0.0, n_bins=n_bins)
    on = np.arange(slots) % 64 < sfts
    fa, fb = (np.where(on[None, :, None], x, 0.0).astype(np.float32) for x in (base.fa, base.fb))
    at = slice(64 * 5, 64 * 6)
    scale = 2.0 ** -24 * np.abs(fb[-1, :, 1]).max() / np.abs(fb[-1, at, 1]).max()
    fb[-1, at, 1] = (fb[-1, at, 1] * scale).astype(np.float32)
    abc = {name: np.where(on, getattr(base, name), 0.0) for name in ("a2", "b2", "ab")}
    atoms = dataclasses.replace(base, fa=fa, fb=fb, **abc)
    win = tfsynth.list_window("exp", np.arange(250, 450) * T, np.arange(1, 40) * T)
    for prec in ("fp32", "fp64"):
        got, n = slides(ctx, atoms, win, prec)
        check_map(got, oracle.fmap_atoms(atoms, win), TOL[prec])
        assert n == (sfts < 8), prec
