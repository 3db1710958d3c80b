"""Threads that share a context, each on its own stream, on the per-thread default
stream or all on one stream: every call's dot products as from one call alone,
whichever of them splits its K loop in the context's scratch."""
import threading

import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PER_THREAD = 2          # the handle of every thread's own default stream


def dev64(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


@pytest.mark.parametrize("streams", ["own", "per-thread", "one"])
def test_threads_share_a_context(keys, streams):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc
    from paper_2405_04463_amd.pipeline import SharedDB, SharedQueries

    q, n, rot, workers = 3, 130, list(range(-15, 16)), 3
    ctx = imc.Context(imc.Keys(*keys), max_rows=q * len(rot))
    db = SharedDB(ctx, n, parties=(2,))
    db.enroll(*(dev64(x) for x in wl.gen_codes(94, 0, n)), 0)
    qc, qm = wl.gen_codes(94, 0, q * workers, query=True)
    qs = [SharedQueries(ctx, dev64(qc[q * i:q * i + q]), dev64(qm[q * i:q * i + q]), 10 * i, keep_raw=False)
          for i in range(workers)]
    bufs = [[torch.zeros(q * len(rot), n, dtype=torch.int16, device="cuda") for _ in range(2)]
            for _ in range(2 * workers)]

    def call(i, out, tiles_stream):
        ctx.dot_shares(2, qs[i].op[2], q, imc.make_ids(10 * i, rot, 0), db.regions[2], db.capacity, n, *bufs[out], n,
                       tiles_stream)

    ctx.set_dot_tiles(imc.DOT_TILES_ROTATION_DIRECT)                # never splits
    for i in range(workers):
        call(i, workers + i, None)
    ctx.set_dot_tiles(imc.DOT_TILES_AUTO)
    torch.cuda.synchronize()
    one = torch.cuda.Stream()
    per = {"own": [torch.cuda.Stream() for _ in range(workers)], "per-thread": [PER_THREAD] * workers,
           "one": [one] * workers}[streams]

    def work(i):
        for _ in range(20):
            call(i, i, per[i])

    for _ in range(2):
        for b in bufs[:workers]:
            for t in b:
                t.zero_()
        torch.cuda.synchronize()
        ts = [threading.Thread(target=work, args=(i,)) for i in range(workers)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        torch.cuda.synchronize()
        for i in range(workers):
            assert all(torch.equal(a, b) for a, b in zip(bufs[i], bufs[workers + i])), i
    ctx.close()
