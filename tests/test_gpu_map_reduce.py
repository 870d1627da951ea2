"""GPU logB of stored maps with masked stretches (-inf cells)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1805_05652_amd as tf
    c = tf.Context(0, arena_bytes=64 << 20)
    yield c
    c.close()


@pytest.mark.parametrize("masked", [1, 255, 256, 1791, 1792, 1793, 2000, 2047, 2048, 2049, 2303, 2304, 4000, 16384, 18432])
@pytest.mark.parametrize("cells", [8192, 16384, 40000])
@pytest.mark.parametrize("call", ["logB", "noalloc"])
def test_logB_of_masked_stretches(ctx, call, cells, masked):
    """A stretch of masked cells at the start of a tile (16384 cells), at its
    end and over the whole map: threads that have met nothing but -inf in
    their first chunk (8 cells, 256 apart), or in all of them.  logB is a sum
    of at most 40000 exponentials, each to a few 2^-53, so 1e-12 holds
    whatever their order; a wholly masked map has logB = -inf."""
    import torch
    print("case: %s of %d cells, %d masked" % (call, cells, masked), flush=True)
    rng = np.random.default_rng(cells + masked)
    maps = rng.chisquare(4, size=(4, 1, cells)).astype(np.float32)
    maps[0, 0, :masked] = -np.inf
    maps[1, 0, -masked:] = -np.inf
    maps[2, 0, max(0, 16384 - masked):16384 + masked] = -np.inf
    maps[3] = -np.inf
    dev = torch.from_numpy(maps).to("cuda:0")
    if call == "logB":
        got = ctx.logB(dev)
    else:
        out = torch.empty(4, dtype=torch.float64, device="cuda:0")
        torch.cuda.synchronize()
        ctx.logB_noalloc(dev, out)
        ctx.stream.synchronize()
        got = out.cpu().numpy()
    want = oracle.reduce(maps[:3].astype(np.float64))[2]
    whole = np.isneginf(maps[:3]).all(axis=(1, 2))
    want[whole] = -np.inf
    assert np.allclose(got[:3], want, atol=1e-12, rtol=1e-14)
    assert np.isneginf(got[3])
