"""Calls that the plan takes apart, each on the route that its sizes name (asked
of the plan itself): the last columns, the last queries, or both go to the
rotation kernel, gathered and not, both sharings.  All outputs against the
128 x 128 expanded tiles, the first, a middle and the last entry against the
oracle."""
import numpy as np
import pytest

import oracle as orc
import workload as wl
from planlib import Plan

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return Plan(str(tmp_path_factory.mktemp("plan")))


def dev64(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


ROT = list(range(-15, 16))


@pytest.mark.parametrize("q,n,first,galois,mask,gather,pairs", [
    (20, 16390, 0, True, True, True, (16, 16384)),       # both apart
    (20, 16390, 64, False, True, True, (16, 16384)),
    (20, 16390, 64, True, True, False, (16, 16384)),
    (20, 16390, 0, False, True, False, (16, 16384)),
    (23, 16384, 0, True, True, False, (16, 16384)),      # the queries alone
    (23, 16384, 64, True, True, True, (16, 16384)),
    (19, 32800, 0, True, False, True, (16, 32768)),      # both, code dot alone
    (16, 16385, 0, False, True, True, (16, 16384)),      # the columns alone
])
def test_calls_taken_apart(keys, plan, q, n, first, galois, mask, gather, pairs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc
    from paper_2405_04463_amd.pipeline import SharedDB, SharedQueries

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert plan.plan(q, ROT, n, 2 if mask else 1, galois, cus=cus) == pairs
    dealer, party = keys
    rows, ld = q * len(ROT), n + 3
    ctx = imc.Context(imc.Keys(dealer, party), max_rows=rows)
    dc, dm = wl.gen_codes(92, first, n)
    qc, qm = wl.gen_codes(92, 0, q, query=True)
    db = SharedDB(ctx, first + n, parties=(1,), galois=galois)
    db.enroll(dev64(dc), dev64(dm), first)
    qs = SharedQueries(ctx, dev64(qc), dev64(qm), 500, keep_raw=False, galois=galois)
    ids = imc.make_ids(500, ROT, first)
    order = list(range(q))
    if gather:
        order = order[::-1]
        order[3] = order[0]
    qidx = torch.tensor(order, dtype=torch.int32, device="cuda")
    got = []
    for tiles in (imc.DOT_TILES_AUTO, imc.DOT_TILES_EXPANDED_128x128):
        ctx.set_dot_tiles(tiles)
        c = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda")
        m = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda") if mask else None
        if gather:
            ctx.dot_shares_gather(1, qs.op[1], qidx, q, ids, db.regions[1], db.capacity, n, c, m, ld, galois=galois)
        else:
            ctx.dot_shares(1, qs.op[1], q, ids, db.regions[1], db.capacity, n, c, m, ld, galois=galois)
        got.append((c, m))
    torch.cuda.synchronize()
    at = np.array([0, n // 2, n - 1])
    share, dot = (orc.galois_share, orc.galois_local_dot) if galois else (orc.share, orc.local_dot)
    ddom, qdom = ((orc.DOM_GALOIS_DB, orc.DOM_GALOIS_QUERY) if galois else (orc.DOM_SHARE_DB, orc.DOM_SHARE_QUERY))
    dsh = np.concatenate([share(dealer, ddom, dc[e:e + 1], dm[e:e + 1], first + int(e)) for e in at])
    ref = dot(1, share(dealer, qdom, qc, qm, 500)[order], ROT, dsh)
    for g, w, o in zip(*got, ref):
        if g is not None:
            assert torch.equal(g, w)                     # padding columns untouched too
            assert np.array_equal(g[:, torch.from_numpy(at).cuda()].cpu().numpy().view(np.uint16), o)
    ctx.close()
