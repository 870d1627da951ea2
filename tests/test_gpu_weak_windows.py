"""GPU exponential maps across the rims of weak SFTs, at the bounds of each
precision where the cells are well conditioned, and at the conditioning of D
where they are not."""
import dataclasses

import numpy as np
import pytest

import oracle
import tfsynth
from checks import F32_MAP, TOL, check_map

pytestmark = pytest.mark.gpu

T = tfsynth.T_SFT


@pytest.fixture(scope="module")
def ctx():
    import paper_1805_05652_amd as tf
    c = tf.Context(0, arena_bytes=512 << 20)
    yield c
    c.close()


def _fmap(ctx, atoms, win, prec):
    aid = ctx.upload_atoms(atoms)
    try:
        return ctx.fmap(aid, win, prec, want_map=True)[1].cpu().numpy()
    finally:
        ctx.free(aid)


WIN = ("exp", 0, T, 300, T // 2, T // 3, 70)


@pytest.mark.parametrize("case", ["zero_antenna", "one_antenna", "zero_data"])
@pytest.mark.parametrize("prec", ["fp64", "recur64", "fp32", "f16x3"])
def test_nothing_beside_something(ctx, case, prec):
    """SFTs with zeroed atoms, no second antenna, no data: double precision to
    its own bound."""
    print("case: %s %s" % (case, prec), flush=True)
    base = tfsynth.make_atoms(9500, 500, 0.1, n_bins=2)
    a, b, fa, fb = (v.copy() for v in (base.a, base.b, base.fa, base.fb))
    if case == "zero_antenna":
        a[150:230] = b[150:230] = 0.0
        fa[:, 150:230] = fb[:, 150:230] = 0.0
    elif case == "one_antenna":
        b[:] = 0.0
        fb[:] = 0.0
    else:
        fa[:], fb[:] = 0.0, 0.0
    atoms = dataclasses.replace(base, a=a, b=b, a2=a * a, b2=b * b, ab=a * b, fa=fa, fb=fb)
    win = tfsynth.regular_window(*WIN)
    check_map(_fmap(ctx, atoms, win, prec), oracle.fmap_atoms(atoms, win), TOL[prec])


@pytest.mark.parametrize("weak", [1e-2, 1e-4, 1e-6])
@pytest.mark.parametrize("prec", ["fp64", "recur64"])
def test_values_across_a_rim(ctx, weak, prec):
    """A stretch of collinear SFTs (b = 2 a: D = 0 of themselves) far below
    their neighbours.  Windows across its rims have D / A B down to the
    degenerate threshold, where D keeps only what the rounding of A, B and C
    leaves it: up to some 200 terms in the window and as many steps slid, each
    to 2^-53, on both sides, so 2F may differ by 1024 * 2^-53 * A B / D
    relative to max(2F, 1) beyond the precision's own bound; cells whose D is
    decided by such a difference are left out."""
    print("case: rim %g %s" % (weak, prec), flush=True)
    base = tfsynth.make_atoms(9500, 500, 0.1, n_bins=2)
    a, b, fa, fb = (v.copy() for v in (base.a, base.b, base.fa, base.fb))
    hole = slice(150, 230)
    a[hole] *= weak
    b[hole] = 2.0 * a[hole]
    fa[:, hole] *= weak
    fb[:, hole] = 2.0 * fa[:, hole]
    atoms = dataclasses.replace(base, a=a, b=b, a2=a * a, b2=b * b, ab=a * b, fa=fa, fb=fb)
    win = tfsynth.regular_window(*WIN)
    ts = atoms.timestamps[None, None, :] - win.t0[:, None, None]
    w = np.where((ts >= 0) & (ts < 3 * win.tau[None, :, None]), np.exp(-ts / win.tau[None, :, None].astype(np.longdouble)), 0)
    A, B, C = ((w * w * v).sum(-1) for v in (atoms.a2, atoms.b2, atoms.ab))
    with np.errstate(invalid="ignore", divide="ignore"):
        cond = np.where(A * B > 0, A * B / np.abs(A * B - C * C), np.inf).astype(np.float64)
    ref = oracle.fmap_atoms(atoms, win)
    got = _fmap(ctx, atoms, win, prec).astype(np.float64)
    # (the threshold itself, D = 1e-10 A B, within the rounding of D)
    sure = np.abs(cond * 1e-10 - 1.0) > 1024 * 2.0 ** -53 * 1e10
    zero = (cond > 1e10) & sure
    assert np.all(got[:, zero] == 0.0) and np.all(ref[:, zero] == 0.0)
    ok = (cond < 1e10) & sure
    err = np.abs(got - ref) / np.maximum(np.abs(ref), 1.0)
    bound = TOL[prec] + F32_MAP + 1024 * 2.0 ** -53 * cond
    assert ok.sum() > 10000 and np.all(err[:, ok] <= bound[ok]), (err[:, ok] / bound[ok]).max()
