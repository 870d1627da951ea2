"""The runtime's plans of maps (host code only, through a small program built
from runtime.cpp): what a kernel reads lies inside what its plan holds, and
every plan can be launched."""
import os
import subprocess

import numpy as np
import pytest

from paper_1805_05652_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
T = 1800
PREC = {"fp64": 0, "fp32": 1, "bf16x3": 2, "recur64": 3, "f16x3": 4}


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    """plan(...) -> dict of the planned fields."""
    exe = str(tmp_path_factory.mktemp("plan") / "plan_probe")
    lib = os.path.dirname(build.library_path())
    subprocess.run([build.hipcc(), "-O1", "-std=c++17", "--cuda-host-only", "-Wno-unused-function",
                    os.path.join(ROOT, "tests", "plan_probe.cpp"), "-o", exe, "-L" + lib, "-ltfstat",
                    "-Wl,-rpath," + lib, "-lpthread"], check=True, capture_output=True)

    def plan(kind, prec, K, bins, t0, tau, exact32=True, t_sft=T):
        line = [{"rect": 0, "exp": 1}[kind], PREC[prec], K, bins, t_sft, int(exact32), len(t0), *t0, len(tau), *tau]
        out = subprocess.run([exe], input=" ".join(str(int(v)) for v in line), check=True, capture_output=True,
                             text=True).stdout
        return {k: int(v) for k, v in (f.split("=") for f in out.split())}
    return plan


def _ends(t0, tau, T_, K, factor):
    """First slots and window ends [row, tau] (clamped), as the kernels take them."""
    t0, tau = np.asarray(t0, dtype=np.int64), np.asarray(tau, dtype=np.int64) * factor
    k0 = -(-t0 // T_)
    delta = k0 * T_ - t0
    hi = np.clip(k0[:, None] + tau[None, :] // T_ + (tau[None, :] % T_ > delta[:, None]), 0, K)
    return np.clip(k0, 0, K), hi


def staged_slots(p, t0, tau, K, kind):
    """Most slots that a workgroup of the plan stages in LDS."""
    k0, hi = _ends(t0, tau, T, K, 1 if kind == "rect" else 3)
    rows = p["rect_rows"] if kind == "rect" else p["waves"] * p["seg_rows"]
    most = 0
    for n0 in range(0, len(tau), 64):
        n1 = min(n0 + 63, len(tau) - 1)
        kend = max(hi[-1, n1], p["kbeg"])
        for m0 in range(0, len(t0), rows):
            m1 = min(m0 + rows, len(t0)) - 1
            if kind == "rect":
                most = max(most, hi[m1, n1] - hi[m0, n0] + 1)
            else:
                up = max(hi[m1, n1], p["kbeg"])
                up = min(p["kbeg"] + -(-(up - p["kbeg"]) // p["range_len"]) * p["range_len"], kend)
                most = max(most, up - hi[m0, n0])
    return most


@pytest.mark.parametrize("kind", ["exp", "rect"])
@pytest.mark.parametrize("seed", range(8))
def test_stage_holds_what_the_kernel_stages(probe, kind, seed):
    """Row lists with steps of any size: rows of the last, shorter segments lie
    elsewhere than those of full ones, so that a jump can fall inside a group
    of segments that the full ones had split there."""
    rng = np.random.default_rng(seed)
    for _ in range(6):
        K = int(rng.integers(200, 9000))
        bins = int(rng.choice([1, 2, 3, 4, 5, 9, 64]))
        n = int(rng.integers(2, 400))
        step = rng.choice([7, T // 2, T, 2 * T, 11 * T, 150 * T], size=n, p=[.2, .2, .3, .2, .07, .03])
        t0 = np.cumsum(step) + int(rng.integers(-50, 50)) * T
        tau = np.unique(rng.integers(1, int(rng.choice([40, 300, 3000])) * T, size=int(rng.integers(1, 300))))
        p = probe(kind, "fp32", K, bins, t0, tau)
        if p["stage"] > 0:
            assert staged_slots(p, t0, tau, K, kind) <= p["stage"], (K, bins, n, p)


@pytest.mark.parametrize("K,split", [(256, False), (257, True), (6144 * 256, True), (6144 * 256 + 1, False),
                                     (1 << 28, False)])
def test_rect_block_totals(probe, K, split):
    """Prefix sums with block totals up to 6144 blocks of 256 slots (their
    time grows with the square of the blocks); beyond, without."""
    p = probe("rect", "fp32", K, 1, [0, 5 * T], [2 * T, 9 * T])
    assert (p["scan_blk"] > 0) == split
    assert p["scan_blk"] in (0, -(-K // 256))


@pytest.mark.parametrize("prec", ["fp32", "fp64", "recur64", "f16x3"])
@pytest.mark.parametrize("K,bins", [(65535 * 512, 1), (65535 * 512 + 1, 1), ((1 << 26) - 2, 1), ((1 << 25) - 2, 2),
                                    (1 << 24, 3), (5000, 1), (1, 1)])
def test_slide_launch_limits(probe, prec, K, bins):
    """Anchors of data as long as the sliding sums take (2 GiB of atoms): no
    more super-ranges than a grid's second dimension has blocks, and they
    cover the data."""
    t0 = [0, max(1, K // 2) * T, (K + 5) * T]
    p = probe("exp", prec, K, bins, t0, [T, K * T // 4 + 1, K * T])
    assert p["slide"] and p["range_len"] % 16 == 0 and p["n_sup"] <= 65535
    assert p["range_len"] * 8 * p["n_sup"] >= K and p["n_range"] == 8 * p["n_sup"]
