"""The dot kernel that takes consecutive rotations in pairs (chosen for calls of
27..31 rotations with enough tiles) against the expanded kernel, all outputs,
and against the oracle's local dots on the first, last and a middle entry:
partial query tiles, ragged entry tiles, each rotation count, lists that start
anywhere, gathered queries, a code dot alone, both sharings, and calls whose
last columns or last queries go to the rotation kernel.  Sizes are about the
smallest at which a call on 256 CUs takes this kernel."""
import numpy as np
import pytest

import oracle as orc
import workload as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev64(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


@pytest.mark.parametrize("q,n,first,rot,galois,mask,gather", [
    (10, 16300, 64, range(-15, 16), False, True, False),    # one query tile of 10, ragged last entry tile
    (16, 16385, 0, range(-13, 16), True, True, False),      # 29 rotations ending at 15; the last entry goes apart
    (33, 8170, 128, range(-15, 15), False, True, False),    # 30 rotations; the last query goes apart
    (20, 16390, 0, range(-14, 14), True, True, True),       # 28, gathered with a repeat; both go apart
    (40, 10877, 0, range(-11, 16), False, False, False),    # 27 rotations, code dot alone
    (12, 16200, 0, range(-15, 16), True, True, True),       # gathered
])
def test_pairs_against_expanded_and_oracle(keys, q, n, first, rot, galois, mask, gather):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc
    from paper_2405_04463_amd.pipeline import SharedDB, SharedQueries

    dealer, party = keys
    rot = list(rot)
    rows = q * len(rot)
    ctx = imc.Context(imc.Keys(dealer, party), max_rows=rows)
    dc, dm = wl.gen_codes(91, first, n)
    qc, qm = wl.gen_codes(91, 0, q, query=True)
    db = SharedDB(ctx, first + n, parties=(1,), galois=galois)
    db.enroll(dev64(dc), dev64(dm), first)
    qs = SharedQueries(ctx, dev64(qc), dev64(qm), 500, keep_raw=False, galois=galois)
    ids = imc.make_ids(500, rot, first)
    order = list(range(q))
    if gather:
        order = order[::-1]
        order[3] = order[0]
    qidx = torch.tensor(order, dtype=torch.int32, device="cuda")
    ld = n + 3
    got = {}
    for tiles in (imc.DOT_TILES_AUTO, imc.DOT_TILES_EXPANDED_256x128):
        ctx.set_dot_tiles(tiles)
        c = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda")
        m = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda") if mask else None
        if gather:
            ctx.dot_shares_gather(1, qs.op[1], qidx, q, ids, db.regions[1], db.capacity, n, c, m, ld, galois=galois)
        else:
            ctx.dot_shares(1, qs.op[1], q, ids, db.regions[1], db.capacity, n, c, m, ld, galois=galois)
        got[tiles] = (c, m)
    torch.cuda.synchronize()
    (c, m), (ec, em) = got[imc.DOT_TILES_AUTO], got[imc.DOT_TILES_EXPANDED_256x128]
    assert torch.equal(c, ec) and (m is None or torch.equal(m, em))      # padding columns untouched too
    at = np.array([0, n // 2, n - 1])
    share, dot = (orc.galois_share, orc.galois_local_dot) if galois else (orc.share, orc.local_dot)
    ddom, qdom = ((orc.DOM_GALOIS_DB, orc.DOM_GALOIS_QUERY) if galois else (orc.DOM_SHARE_DB, orc.DOM_SHARE_QUERY))
    dsh = np.concatenate([share(dealer, ddom, dc[e:e + 1], dm[e:e + 1], first + int(e)) for e in at])
    qsh = share(dealer, qdom, qc, qm, 500)[order]
    rc, rm = dot(1, qsh, rot, dsh)
    pick = torch.from_numpy(at).cuda()
    assert np.array_equal(c[:, pick].cpu().numpy().view(np.uint16), rc)
    assert m is None or np.array_equal(m[:, pick].cpu().numpy().view(np.uint16), rm)
    ctx.close()
