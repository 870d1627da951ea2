"""GPU serving from several threads at once: requests submitted, polled and
cancelled while admissions are laid out and launched."""
import threading
import time

import numpy as np
import pytest

import tfsynth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_batch", [1, 16])
def test_many_clients(max_batch):
    """Four clients with uneven requests in flight, every fifth cancelled, one
    thread uploading and freeing atoms and running maps of its own meanwhile:
    every finished request equals the map alone."""
    import paper_1805_05652_amd as tf
    print("case: many clients, max_batch %d" % max_batch, flush=True)
    with tf.Context(0, arena_bytes=2 << 30) as ctx:
        ctx.serve_config(max_batch)
        reqs = [tfsynth.candidate(i, seed_base=9600, max_slots=900, max_grid=150, max_bins=5) for i in range(8)]
        ids = [ctx.upload_atoms(a) for a, _ in reqs]
        precs = ("fp32", "f16x3", "fp64", "recur64")
        alone = {(i, p): ctx.fmap(aid, w, p)[0] for i, (aid, (_, w)) in enumerate(zip(ids, reqs)) for p in precs}
        errors, done = [], [0] * 4
        stop = threading.Event()

        def client(n):
            try:
                rng = np.random.default_rng(n)
                for _ in range(6):
                    mine = []
                    for k in range(20):
                        i, p = int(rng.integers(len(reqs))), precs[int(rng.integers(4))]
                        t = ctx.submit(ids[i], reqs[i][1], p)
                        if k % 5 == 4:
                            ctx.cancel(t)
                        mine.append((t, i, p, k % 5 == 4))
                    end = time.time() + 30
                    while mine and time.time() < end:
                        left = []
                        for t, i, p, gone in mine:
                            try:
                                r = ctx.poll(t, reqs[i][0].n_bins)
                            except tf.TfstatError as e:
                                assert gone and e.code == tf._abi.E_CANCELLED, e
                                continue
                            if r is None:
                                left.append((t, i, p, gone))
                            else:
                                assert r == alone[i, p]
                                done[n] += 1
                        mine = left
                    assert not mine, "requests did not finish"
            except BaseException as e:
                errors.append(e)

        def other():
            try:
                atoms, win = reqs[0]
                while not stop.is_set():
                    aid = ctx.upload_atoms(atoms)
                    assert ctx.fmap(aid, win, "fp32")[0] == alone[0, "fp32"]
                    ctx.free(aid)
            except BaseException as e:
                errors.append(e)

        threads = [threading.Thread(target=client, args=(n,)) for n in range(4)]
        extra = threading.Thread(target=other)
        extra.start()
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        stop.set()
        extra.join()
        if errors:
            raise errors[0]
        assert all(n >= 96 for n in done), done
