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

    def plan(kind, prec, K, bins, t0, tau, exact32=True, t_sft=T, anchor_most=-1, smaller=0):
        line = [{"rect": 0, "exp": 1}[kind], PREC[prec], K, bins, t_sft, int(exact32), anchor_most, smaller,
                len(t0), *t0, len(tau), *tau]
        out = subprocess.run([exe], input=" ".join(str(int(v)) for v in line), check=True, capture_output=True,
                             text=True).stdout
        p = dict(f.split("=") for f in out.split())
        passes = [tuple(int(v) for v in p.pop(k).split(",")) for k in list(p) if k.startswith("pass")]
        return {**{k: int(v) for k, v in p.items()}, "passes": passes}
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
    assert p["range_len"] * 8 * p["n_sup"] >= K - p["kbeg"] and p["n_range"] == 8 * p["n_sup"]


def test_anchors_only_where_windows_end(probe):
    """A few rows at the start of long data: anchors up to the last window's
    end, not to the data's (0.9 GB)."""
    p = probe("exp", "fp32", 16000000, 1, np.arange(200) * T, (2 + np.arange(64)) * T)
    assert p["slide"] and p["ws"] < 1 << 20
    last = probe("exp", "fp32", 16000000, 1, (15999800 + np.arange(200)) * T, (2 + np.arange(64)) * T)
    assert last["slide"] and last["ws"] < 1 << 20
    assert p["range_len"] * 8 * p["n_sup"] >= 200 + 3 * 66 - p["kbeg"]


@pytest.mark.parametrize("bins,n_tau", [(1, 64), (1, 700), (4, 200), (9, 130), (64, 65), (256, 500), (3, 1)])
@pytest.mark.parametrize("mib", [-1, 64, 8, 1, 0])
def test_passes_cover_every_column_once(probe, bins, n_tau, mib):
    """Tau tiles x bin groups in passes whose anchors fit the bytes they may
    take (or hold one column); the default lets common maps run in one."""
    t0, tau = np.arange(300) * T, (2 + np.arange(n_tau)) * T
    p = probe("exp", "fp32", 2500, bins, t0, tau, anchor_most=mib << 20 if mib >= 0 else -1)
    seen = np.zeros((p["n_tt"], p["n_bg"]), dtype=int)
    for tt0, tts, bg0, bgs in p["passes"]:
        assert tts >= 1 and bgs >= 1 and (tts == 1 or bgs == p["n_bg"])
        seen[tt0:tt0 + tts, bg0:bg0 + bgs] += 1
        assert tt0 + tts <= p["n_tt"] and bg0 + bgs <= p["n_bg"]
    assert (seen == 1).all()
    most = (mib if mib >= 0 else 256) << 20
    assert p["anchors"] <= most or p["passes"][0][1::2] == (1, 1)
    if mib < 0:
        assert len(p["passes"]) == 1


@pytest.mark.parametrize("prec", ["fp32", "fp64", "f16x3"])
@pytest.mark.parametrize("K,bins,n_t0,n_tau,longest", [(5000, 64, 600, 700, 1600), (5000, 1, 1000, 1000, 1600),
                                                       (4000, 2, 700, 3, 100), (9000, 16, 100, 300, 40),
                                                       (900, 5, 500, 300, 300), (3000, 256, 300, 200, 1000)])
def test_smaller_plans(probe, prec, K, bins, n_t0, n_tau, longest):
    """With less workspace a sliding map takes more passes, in no more than the
    direct sums would take; where not even one column fits that, the direct
    sums.  Nothing smaller when the direct sums would take more than all."""
    t0, tau = np.arange(n_t0) * T, np.unique(np.linspace(2 * T, longest * T, n_tau).astype(np.int64))
    full = probe("exp", prec, K, bins, t0, tau)
    direct = probe("exp", prec, K, bins, t0, tau, anchor_most=0, smaller=9)
    small = probe("exp", prec, K, bins, t0, tau, smaller=9)
    assert full["slide"] and full["smaller"] == 0
    if small["slide"]:
        assert small["smaller"] == len(small["passes"]) - 1 == 0 or small["ws"] < full["ws"]
        for k in ("bg", "n_seg", "seg_rows", "range_len", "n_range", "n_sup", "kbeg", "waves", "stage"):
            assert small[k] == full[k], k   # (the same sums)
    else:
        assert direct["ws"] == small["ws"] and small["no_slide"] == 2
    assert small["ws"] <= full["ws"]


def test_smaller_plans_of_the_recurrence(probe):
    """RECUR64 shrinks to one column a pass, then to the smallest workspace,
    then to the direct sums."""
    t0, tau = np.arange(700) * T, (2 + np.arange(130)) * T
    got = [probe("exp", "recur64", 4000, 9, t0, tau, smaller=n) for n in range(5)]
    assert [(p["slide"], p["no_slide"]) for p in got] == [(1, 0), (1, 0), (1, 1), (0, 2), (0, 2)]
    assert got[1]["passes"][0][1::2] == got[2]["passes"][0][1::2] == (1, 1)
    assert got[0]["ws"] > got[1]["ws"] > got[2]["ws"]
    assert got[4]["smaller"] == 3


@pytest.mark.parametrize("prec", ["fp32", "fp64", "f16x3", "recur64"])
@pytest.mark.parametrize("case,direct", [("long_data", True), ("far_rows", True), ("clusters", True), ("far_rows_long", False),
                                         ("clusters_long", False), ("two_rows_long", False), ("slots", False),
                                         ("days30", False), ("small", False)])
def test_sliding_where_it_is_cheaper(probe, case, direct, prec):
    """Short windows of rows far apart in long data are summed directly, long
    windows and rows near each other by sliding (the recurrence always)."""
    K, bins, t0, L, n_tau = {
        "long_data": (1000000, 1, np.arange(200) * 4999, 20, 64),
        "far_rows": (8000, 64, np.arange(100) * 80, 20, 700),
        "clusters": (8000, 64, np.concatenate([b + np.arange(40) for b in range(0, 8000, 500)]), 20, 300),
        "far_rows_long": (8000, 64, np.arange(100) * 80, 2000, 700),
        "clusters_long": (8000, 64, np.concatenate([b + np.arange(40) for b in range(0, 8000, 500)]), 2000, 300),
        "two_rows_long": (8000, 4, np.array([0, 7000]), 2000, 300),
        "slots": (2000, 256, np.arange(500), 1500, 500),
        "days30": (5000, 1, np.arange(1000), 4320, 1000),
        "small": (300, 2, np.arange(60) * 5, 20, 48)}[case]
    tau = np.unique(np.linspace(2 * T, L * T / 3, n_tau).astype(np.int64))
    p = probe("exp", prec, K, bins, t0 * T, tau)
    if case == "clusters" and prec == "fp64":
        return   # (its direct sums take three quarters of the sliding ones: near the line)
    assert p["slide"] == (prec == "recur64" or not direct)
