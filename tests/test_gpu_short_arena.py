"""GPU sliding maps where the arena cannot hold all anchors at once: more
passes, the same numbers bit for bit."""
import time

import numpy as np
import pytest

import tfsynth

pytestmark = pytest.mark.gpu

T = tfsynth.T_SFT


def _atoms_win(n_bins):
    atoms = tfsynth.make_atoms(9850 + n_bins, 2400, 0.1, n_bins=n_bins)
    return atoms, tfsynth.regular_window("exp", 3, T, 400, 2 * T, 3 * T, 330)


@pytest.fixture(scope="module")
def roomy():
    """Results and maps with room for everything, and the bytes of the atoms."""
    import paper_1805_05652_amd as tf
    out = {}
    with tf.Context(0, arena_bytes=2 << 30) as c:
        for n_bins in (1, 3, 21):
            atoms, win = _atoms_win(n_bins)
            aid = c.upload_atoms(atoms)
            for prec in ("fp32", "fp64", "f16x3", "recur64"):
                res, twoF = c.fmap(aid, win, prec, want_map=True)
                out[n_bins, prec] = res, twoF.cpu().numpy()
            c.free(aid)
    return out


def _atom_bytes(n_bins):
    up = lambda v: -(-v // 256) * 256
    return up(32 * 2401) + up(32 * 2401 * n_bins) + up(16 * 2401 * n_bins)


@pytest.mark.parametrize("n_bins", [1, 3, 21])
@pytest.mark.parametrize("prec", ["fp32", "fp64", "f16x3", "recur64"])
def test_more_passes_give_the_same_numbers(roomy, prec, n_bins):
    """Arenas from more than enough down to refusal."""
    import paper_1805_05652_amd as tf
    atoms, win = _atoms_win(n_bins)
    want, want_map = roomy[n_bins, prec]
    passes = []
    for mib in (200, 40, 20, 12, 8, 6, 5, 4, 3):
        print("case: %s %d bins, %d MiB beside the atoms" % (prec, n_bins, mib), flush=True)
        with tf.Context(0, arena_bytes=_atom_bytes(n_bins) + (mib << 20)) as c:
            aid = c.upload_atoms(atoms)
            c.profile(True)
            try:
                res, twoF = c.fmap(aid, win, prec, want_map=True)
            except tf.TfstatError as e:
                assert e.code == tf._abi.E_NOMEM
                break
            finally:
                c.profile(False)
            n = c.profile_read()["recur"][0]
            assert n >= 1, "not by sliding windows"
            passes.append(n)
            assert res == want
            assert np.array_equal(twoF.cpu().numpy(), want_map)
            with c.batch([(aid, win)], prec) if prec != "recur64" else _none() as b:
                assert b is None or b.run() == [want]
    assert passes[0] == 1
    # (where the direct sums would take more than one pass does, nothing smaller is planned)
    if n_bins == 21 or prec == "recur64" or (n_bins == 3 and prec == "fp32"):
        assert passes[-1] > 1, passes


class _none:
    def __enter__(self):
        return None

    def __exit__(self, *a):
        return False


def test_one_map_of_a_batch_in_passes(roomy):
    """A batch that does not fit makes its largest maps smaller; every map's
    numbers stay those of the map alone."""
    import paper_1805_05652_amd as tf
    print("case: batch in a short arena", flush=True)
    items = {n: _atoms_win(n) for n in (1, 3, 21)}
    beside = sum(_atom_bytes(n) for n in items)
    for mib in (400, 30, 25):
        with tf.Context(0, arena_bytes=beside + (mib << 20)) as c:
            ids = {n: c.upload_atoms(a) for n, (a, _) in items.items()}
            rect = tfsynth.regular_window("rect", 3, T, 400, 2 * T, 3 * T, 330)
            with c.batch([(ids[21], items[21][1]), (ids[1], items[1][1]), (ids[3], rect), (ids[3], items[3][1])], "fp64") as b:
                for _ in range(3):   # (the graph's replays)
                    got = b.run()
                    assert [got[0], got[1], got[3]] == [roomy[n, "fp64"][0] for n in (21, 1, 3)]
                one = b.run(timed=True)
            assert one == got


@pytest.mark.parametrize("max_batch", [1, 16])
def test_served_request_beside_a_batch(roomy, max_batch):
    """Requests that were admitted by the arena's size and meet a batch's
    memory: they run in passes instead of waiting for what nobody gives back
    (alone, and in fused admissions)."""
    import paper_1805_05652_amd as tf
    print("case: request beside a batch", flush=True)
    atoms, win = _atoms_win(21)
    rect = tfsynth.regular_window("rect", 3, T, 400, 2 * T, 3 * T, 330)
    with tf.Context(0, arena_bytes=_atom_bytes(21) + (36 << 20)) as c:
        aid = c.upload_atoms(atoms)
        # rect maps take 3.4 MB each, the request 24 MB in one pass, 8 MB in three
        with c.batch([(aid, rect)] * 6, "fp64") as b:
            c.serve_config(max_batch)
            tickets = [c.submit(aid, win, "fp64") for _ in range(3)]
            got, end = {}, time.time() + 20
            while len(got) < 3 and time.time() < end:
                for t in tickets:
                    if t not in got:
                        r = c.poll(t, 21)
                        if r is not None:
                            got[t] = r
                time.sleep(0.001)
            for t in tickets:
                if t not in got:
                    c.cancel(t)
            assert len(got) == 3, "requests wait for memory"
            assert all(r == roomy[21, "fp64"][0] for r in got.values())
            b.run()
