"""GPU exponential maps of rows far apart with short windows, which the planner
sums directly."""
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


@pytest.mark.parametrize("n_bins", [1, 5, 33])
@pytest.mark.parametrize("case", ["far", "clusters", "before_and_after"])
def test_far_rows(ctx, case, n_bins):
    """Every precision against the oracle, alone and in a batch (bitwise)."""
    print("case: far rows %s %d bins" % (case, n_bins), flush=True)
    K = 30000
    atoms = tfsynth.make_atoms(9860 + n_bins, K, 0.2, n_bins=n_bins)
    if case == "far":
        t0 = np.arange(130) * 229 * T + 7
    elif case == "clusters":
        t0 = np.concatenate([b + np.arange(9) for b in range(0, K, 2500)]) * T
    else:
        t0 = -40 * 300 * T + np.arange(180) * 300 * T + 11
    win = tfsynth.list_window("exp", t0, np.unique(np.linspace(T // 2, 9 * T, 70).astype(np.int64)))
    ref = oracle.fmap_atoms(atoms, win)
    aid = ctx.upload_atoms(atoms)
    try:
        for prec in ("fp32", "fp64", "bf16x3", "f16x3", "recur64"):
            ctx.profile_reset()
            ctx.profile(True)
            res, twoF = ctx.fmap(aid, win, prec, want_map=True)
            ctx.profile(False)
            slid = ctx.profile_read()["recur"][0]
            assert slid == (prec == "recur64") or case != "far"   # (the others lie nearer the line)
            check_map(twoF.cpu().numpy(), ref, TOL[prec])
            check_results(res, ref, win, TOL[prec])
            if prec != "recur64":
                with ctx.batch([(aid, win)], prec) as b:
                    assert b.run() == [res]
    finally:
        ctx.profile(False)
        ctx.free(aid)
