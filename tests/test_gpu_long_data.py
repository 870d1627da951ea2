"""GPU maps over long data: few SFTs in millions of slots."""
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
    c = tf.Context(0, arena_bytes=12 << 30)
    yield c
    c.close()


def sparse_atoms(seed, K, n):
    """n SFTs in K slots, in bursts of consecutive slots, the last slot among them."""
    rng = np.random.default_rng(seed)
    at = np.concatenate([np.arange(10) + s for s in np.linspace(0, K - 10, n // 10).astype(np.int64)])
    m = at.size
    assert at[-1] == K - 1
    # (antenna values of any time: independent, so that no window is degenerate by chance)
    av, bv = rng.uniform(0.3, 1.0, m), rng.uniform(-1.0, 1.0, m)
    x = rng.standard_normal((1, m, 2))
    return types.SimpleNamespace(timestamps=at * T, a2=av * av, b2=bv * bv, ab=av * bv,
                                 fa=(av[:, None] * x).astype(np.float32).astype(np.float64),
                                 fb=(bv[:, None] * x).astype(np.float32).astype(np.float64), t_sft=T, n_bins=1)


def test_rect_over_more_slots_than_a_grid_has_blocks(ctx):
    """65536 blocks of 256 slots and one slot: past the 65535 of a launch's
    second dimension, where the prefix sums run without block totals."""
    K = 65536 * 256 + 1
    print("case: rect %d slots" % K, flush=True)
    atoms = sparse_atoms(1, K, 900)
    t0 = np.concatenate([atoms.timestamps[::10] - 3 * T, [K * T // 2]])
    win = tfsynth.list_window("rect", np.unique(t0), [6 * T, 9 * T, 400000 * T, 1 + K * T // 2, K * T])
    ref = oracle.fmap_atoms(atoms, win)
    aid = ctx.upload_atoms(atoms)
    try:
        res, twoF = ctx.fmap(aid, win, "fp32", want_map=True)
    finally:
        ctx.free(aid)
    check_map(twoF.cpu().numpy(), ref, TOL["fp64"])
    check_results(res, ref, win, TOL["fp64"])


def test_rect_batch_of_more_tiles_than_a_launch_takes(ctx):
    """A batch whose map has 4.2 million tiles, past the threads of one
    launch; the same map alone gives the same numbers."""
    print("case: rect batch, 4.2 million tiles", flush=True)
    atoms = tfsynth.make_atoms(5, 6000, 0.1, n_bins=1)
    # taus 90 slots apart: the window ends of one tile exceed the stage, 64 rows a tile
    win = tfsynth.regular_window("rect", 0, 7, 40001, T, 90 * T, 430000)
    aid = ctx.upload_atoms(atoms)
    try:
        alone, _ = ctx.fmap(aid, win, "fp32")
        with ctx.batch([(aid, win)], "fp32") as b:
            assert b.stats()["n_tiles"] > 1 << 22
            assert b.run() == [alone]
    finally:
        ctx.free(aid)
