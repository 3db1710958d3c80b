"""Dot products of few tiles, whose K loop is split over several workgroups, and
the tiles for few rows: every output against the oracle's local dots at the
edges of the row tiles (64, 128) and of the entry tiles, and a batch matched
against itself against a configuration that does not split."""
import numpy as np
import pytest

import oracle as orc
import workload as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev64(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def _setup(keys, q, n, first, galois, max_rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc
    from paper_2405_04463_amd.pipeline import SharedDB, SharedQueries

    ctx = imc.Context(imc.Keys(*keys), max_rows=max_rows)
    dc, dm = wl.gen_codes(93, first, n)
    qc, qm = wl.gen_codes(93, 0, q, query=True)
    db = SharedDB(ctx, first + n, parties=(2,), galois=galois)
    db.enroll(dev64(dc), dev64(dm), first)
    qs = SharedQueries(ctx, dev64(qc), dev64(qm), 40, keep_raw=False, galois=galois)
    return imc, ctx, (dc, dm, qc, qm), db, qs


@pytest.mark.parametrize("q,rot,n,first,galois,mask", [
    (1, [0], 1, 0, False, True),
    (64, [3], 129, 64, False, True),                        # the last row of a 64-row tile
    (65, [0], 128, 0, False, True),                         # one row more
    (128, [-2], 33, 0, True, True),
    (43, [-1, 0, 1], 127, 64, False, False),                # 129 rows, code dot alone
    (2, list(range(-15, 16)), 65, 128, False, True),        # rotations read in place
    (5, list(range(-6, 7)), 200, 0, True, True),
    (21, list(range(-7, 6)), 1, 0, False, True),            # 273 rows: a second row tile
])
def test_split_against_oracle(keys, q, rot, n, first, galois, mask):
    rows = q * len(rot)
    imc, ctx, (dc, dm, qc, qm), db, qs = _setup(keys, q, n, first, galois, rows)
    ids = imc.make_ids(40, rot, first)
    ld = n + 1
    c = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda")
    m = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda") if mask else None
    for _ in range(2):                                      # scratch reused
        ctx.dot_shares(2, qs.op[2], q, ids, db.regions[2], db.capacity, n, c, m, ld, galois=galois)
    torch.cuda.synchronize()
    share, dot = (orc.galois_share, orc.galois_local_dot) if galois else (orc.share, orc.local_dot)
    ddom, qdom = ((orc.DOM_GALOIS_DB, orc.DOM_GALOIS_QUERY) if galois else (orc.DOM_SHARE_DB, orc.DOM_SHARE_QUERY))
    rc, rm = dot(2, share(keys[0], qdom, qc, qm, 40), rot, share(keys[0], ddom, dc, dm, first))
    for got, want in ((c, rc), (m, rm)):
        if got is not None:
            got = got.cpu().numpy().view(np.uint16)
            assert np.array_equal(got[:, :n], want) and (got[:, n:] == 7).all()
    ctx.close()


@pytest.mark.parametrize("galois", [False, True])
def test_split_batch_against_unsplit(keys, galois):
    q, n, rot = 64, 64, list(range(-15, 16))
    imc, ctx, _, db, qs = _setup(keys, q, n, 0, galois, q * len(rot))
    ids = imc.make_ids(40, rot, 0)
    got = []
    for tiles in (imc.DOT_TILES_AUTO, imc.DOT_TILES_ROTATION_DIRECT):
        ctx.set_dot_tiles(tiles)
        c, m = (torch.zeros(q * len(rot), 64, dtype=torch.int16, device="cuda") for _ in range(2))
        ctx.dot_shares(2, qs.op[2], q, ids, db.regions[2], db.capacity, n, c, m, 64, galois=galois)
        got.append((c, m))
    torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    ctx.close()


def test_split_streams_and_capture(keys):
    """One stream's calls split; calls on another stream and captured calls give the same."""
    q, n, rot = 3, 130, list(range(-15, 16))
    imc, ctx, _, db, qs = _setup(keys, q, n, 0, False, q * len(rot))
    ids = imc.make_ids(40, rot, 0)
    bufs = [[torch.zeros(q * len(rot), n, dtype=torch.int16, device="cuda") for _ in range(2)] for _ in range(3)]

    def call(i, stream):
        ctx.dot_shares(2, qs.op[2], q, ids, db.regions[2], db.capacity, n, *bufs[i], n, stream)

    main, side = torch.cuda.current_stream(), torch.cuda.Stream()
    call(0, main)
    side.wait_stream(main)
    for _ in range(4):                                      # overlapping calls on one context
        call(0, main)
        call(1, side)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(bufs[0], bufs[1]))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(2, torch.cuda.current_stream())
    for _ in range(3):
        for b in bufs[2]:
            b.zero_()
        g.replay()
        call(0, main)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(bufs[0], bufs[2]))
    ctx.close()
