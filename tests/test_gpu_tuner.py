"""The batch autotuner where nothing of the batch runs on the persistent kernel."""
import pytest

import tfsynth

pytestmark = pytest.mark.gpu

T = tfsynth.T_SFT


@pytest.mark.parametrize("prec", ["fp32", "fp64", "f16x3"])
def test_nothing_to_tune(prec):
    """Sliding and rect maps only: the default build and width at once, the
    first time and later; a batch of the same shapes summed directly is still
    tuned, and both give the maps' own results."""
    import paper_1805_05652_amd as tf
    print("case: nothing to tune " + prec, flush=True)
    atoms = tfsynth.make_atoms(9710, 800, 0.1, n_bins=5)
    with tf.Context(0, arena_bytes=1 << 30) as c:
        aid = c.upload_atoms(atoms)
        items = [(aid, tfsynth.regular_window(k, 0, T, 300, 2 * T, T, 90)) for k in ("exp", "rect", "exp")]
        alone = [c.fmap(i, w, prec)[0] for i, w in items]
        with c.batch(items, prec) as b:
            plain = b.stats()
        for n in range(3):
            with c.batch(items, prec, tune=True) as b:
                st = b.stats()
                assert (st["variant"], st["groups"]) == (plain["variant"], plain["groups"])
                assert (st["tune_ms"] > 0.0) == (n == 0)
                assert b.run() == alone
        c.tiling_config(1 << 30, -1)
        alone = [c.fmap(i, w, prec)[0] for i, w in items]
        for n in range(2):
            with c.batch(items, prec, tune=True) as b:
                assert (b.stats()["tune_ms"] > 0.0) == (n == 0)
                assert b.run() == alone
