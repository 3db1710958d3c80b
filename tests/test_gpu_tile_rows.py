"""Rotation calls whose K loop is not split (a stream that does not hold the
context's scratch; groups), at each height of the tiles on 256 CUs: 64, 128 and
192 rows where tiles are few, whole ones of 256 with each height of their last
tile.  All outputs against the 128 x 128 expanded tiles, the first, a middle and
the last entry against the oracle."""
import numpy as np
import pytest

import oracle as orc
import workload as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev64(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def _rot(r):
    return [((7 * i) % 31) - 15 for i in range(r)]           # distinct, in no order


def _setup(keys, q, n, first, galois, max_rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc
    from paper_2405_04463_amd.pipeline import SharedDB, SharedQueries

    ctx = imc.Context(imc.Keys(*keys), max_rows=max_rows)
    dc, dm = wl.gen_codes(96, first, n)
    qc, qm = wl.gen_codes(96, 0, q, query=True)
    db = SharedDB(ctx, first + n, parties=(1,), galois=galois)
    db.enroll(dev64(dc), dev64(dm), first)
    qs = SharedQueries(ctx, dev64(qc), dev64(qm), 30, keep_raw=False, galois=galois)
    share = orc.galois_share if galois else orc.share
    ddom, qdom = ((orc.DOM_GALOIS_DB, orc.DOM_GALOIS_QUERY) if galois else (orc.DOM_SHARE_DB, orc.DOM_SHARE_QUERY))
    at = np.array([0, n // 2, n - 1])
    dsh = np.concatenate([share(keys[0], ddom, dc[e:e + 1], dm[e:e + 1], first + int(e)) for e in at])
    return imc, ctx, db, qs, at, dsh, share(keys[0], qdom, qc, qm, 30)


def _check(got, want, at, ref):
    for g, w, o in zip(got, want, ref):
        if g is None:
            continue
        assert torch.equal(g, w)                                # padding columns untouched too
        assert np.array_equal(g[:, torch.from_numpy(at).cuda()].cpu().numpy().view(np.uint16), o)


@pytest.mark.parametrize("q,r,n,first,galois,mask", [
    (19, 13, 64, 0, False, True),          # 64-row tiles: 247 rows
    (8, 16, 1100, 64, True, True),         # 128 rows, two row tiles
    (48, 31, 64, 0, False, True),          # 128-row tiles: 1,488 rows, the last tile of 80
    (48, 31, 60, 64, True, False),         # 24 tiles of one vector: 64 rows
    (80, 26, 64, 0, False, True),          # 192-row tiles: 2,080 rows, the last of 160
    (9, 15, 8200, 64, False, True),        # 135 rows: one tile of 192
    (5, 13, 16500, 0, False, True),        # whole tiles, the last of 65 rows
    (10, 13, 16500, 64, True, True),       # 130
    (15, 13, 16500, 0, False, True),       # 195
    (20, 13, 16500, 0, True, True),        # 260: 4, apart
    (17, 23, 16500, 64, False, True),      # 391: 135, in order
])
def test_whole_loop(keys, q, r, n, first, galois, mask):
    rows, ld = q * r, n + 3
    imc, ctx, db, qs, at, dsh, qsh = _setup(keys, q, n, first, galois, rows)
    rot = _rot(r)
    main, side = torch.cuda.current_stream(), torch.cuda.Stream()

    def call(tiles, stream, q=q, rot=rot, n=n):
        ctx.set_dot_tiles(tiles)
        c = torch.full((q * len(rot), ld), 7, dtype=torch.int16, device="cuda")
        m = torch.full((q * len(rot), ld), 7, dtype=torch.int16, device="cuda") if mask else None
        torch.cuda.synchronize()
        ctx.dot_shares(1, qs.op[1], q, imc.make_ids(30, rot, first), db.regions[1], db.capacity, n, c, m, ld, stream,
                       galois=galois)
        torch.cuda.synchronize()
        return c, m

    call(imc.DOT_TILES_ROTATION, main, 1, _rot(13), 1)          # splits: the scratch is the first stream's
    got = call(imc.DOT_TILES_ROTATION, side)
    want = call(imc.DOT_TILES_EXPANDED_128x128, side)
    _check(got, want, at, (orc.galois_local_dot if galois else orc.local_dot)(1, qsh, rot, dsh))
    ctx.close()


@pytest.mark.parametrize("groups,n,galois,persistent", [
    ([(1, 31), (2, 15)], 130, False, False),                    # 64-row tiles
    ([(20, 13), (3, 22)], 2100, True, True),                    # 128: 260 and 66 rows
    ([(20, 13), (3, 22)], 5000, False, False),                  # 192
    ([(7, 31), (0, 14), (20, 16)], 5000, True, False),          # whole
    ([(7, 31), (20, 16)], 5000, False, True),
])
def test_groups(keys, groups, n, galois, persistent):
    q = sum(g[0] for g in groups)
    rows, ld = sum(a * b for a, b in groups), n + 3
    imc, ctx, db, qs, at, dsh, qsh = _setup(keys, q, n, 0, galois, rows)
    qrow = imc.galois_query_op_bytes(1) if galois else imc.query_op_bytes(1)
    got, want = ([torch.full((rows, ld), 7, dtype=torch.int16, device="cuda") for _ in range(2)] for _ in range(2))
    args, q0, r0 = [], 0, 0
    for gq, r in groups:
        args.append((qs.op[1].data_ptr() + q0 * qrow, gq, _rot(r), *(t.data_ptr() + 2 * r0 * ld for t in got)))
        ctx.set_dot_tiles(imc.DOT_TILES_EXPANDED_128x128)
        if gq:
            ctx.dot_shares(1, args[-1][0], gq, imc.make_ids(30 + q0, _rot(r), 0), db.regions[1], db.capacity, n,
                           *(t.data_ptr() + 2 * r0 * ld for t in want), ld, galois=galois)
        q0, r0 = q0 + gq, r0 + gq * r
    ctx.set_dot_tiles(imc.DOT_PERSISTENT if persistent else 0)
    ctx.dot_shares_groups(1, args, db.regions[1], db.capacity, 0, n, ld, galois=galois)
    torch.cuda.synchronize()
    dot = orc.galois_local_dot if galois else orc.local_dot
    ref, q0 = [], 0
    for gq, r in groups:
        if gq:
            ref.append(dot(1, qsh[q0:q0 + gq], _rot(r), dsh))
        q0 += gq
    _check(got, want, at, [np.concatenate([x[v] for x in ref]) for v in (0, 1)])
    ctx.close()
