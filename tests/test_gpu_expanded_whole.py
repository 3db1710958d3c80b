"""The expanded dot kernels with their K loop whole (a stream that does not hold
the context's scratch) against the oracle, at each of their tilings and the edges
of their rows; and the persistent grid where it is smaller than the tiles."""
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
    dc, dm = wl.gen_codes(90, first, n)
    qc, qm = wl.gen_codes(90, 0, q, query=True)
    db = SharedDB(ctx, first + n, parties=(2,), galois=galois)
    db.enroll(dev64(dc), dev64(dm), first)
    qs = SharedQueries(ctx, dev64(qc), dev64(qm), 20, keep_raw=False, galois=galois)
    share = orc.galois_share if galois else orc.share
    ddom, qdom = ((orc.DOM_GALOIS_DB, orc.DOM_GALOIS_QUERY) if galois else (orc.DOM_SHARE_DB, orc.DOM_SHARE_QUERY))

    def ref(rot, at):
        dsh = np.concatenate([share(keys[0], ddom, dc[a:b], dm[a:b], first + a) for a, b in at])
        return (orc.galois_local_dot if galois else orc.local_dot)(2, share(keys[0], qdom, qc, qm, 20), rot, dsh)

    def call(tiles, stream, rot, n, ld, mask=True, q=q):
        ctx.set_dot_tiles(tiles)
        c = torch.full((q * len(rot), ld), 7, dtype=torch.int16, device="cuda")
        m = torch.full((q * len(rot), ld), 7, dtype=torch.int16, device="cuda") if mask else None
        torch.cuda.synchronize()
        ctx.dot_shares(2, qs.op[2], q, imc.make_ids(20, rot, first), db.regions[2], db.capacity, n, c, m, ld, stream,
                       galois=galois)
        torch.cuda.synchronize()
        return c, m

    return imc, ctx, ref, call


@pytest.mark.parametrize("galois", [False, True])
@pytest.mark.parametrize("q,rot,n,first,mask", [
    (1, [0], 1, 0, True),
    (9, list(range(-15, 16)), 300, 64, True),     # 279 rows
    (2, [-3, 7], 129, 0, True),
    (64, [5], 130, 0, False),                     # 64 rows: the last of the smallest tile
    (13, [0, 1, 2, 4, -15], 127, 64, True),       # 65
    (16, list(range(-4, 4)), 128, 0, True),       # 128
    (43, [-1, 15, 3], 129, 64, True),             # 129
    (12, list(range(-8, 8)), 65, 0, True),        # 192
    (193, [2], 33, 0, True),
    (64, [0, 1, 2, 3], 257, 64, True),            # 256
])
def test_whole_loop_against_oracle(keys, q, rot, n, first, mask, galois):
    imc, ctx, ref, call = _setup(keys, q, n, first, galois, q * len(rot))
    call(imc.DOT_TILES_EXPANDED_256x128, torch.cuda.current_stream(), [0], 1, 1, q=1)   # splits: the scratch is taken
    side, want = torch.cuda.Stream(), ref(rot, [(0, n)])
    for tiles in (imc.DOT_TILES_EXPANDED_256x128, imc.DOT_TILES_EXPANDED_128x128, imc.DOT_TILES_EXPANDED_SHALLOW):
        for g, w in zip(call(tiles, side, rot, n, n + 1, mask), want):
            if g is not None:
                g = g.cpu().numpy().view(np.uint16)
                assert np.array_equal(g[:, :n], w) and (g[:, n:] == 7).all(), tiles
    ctx.close()


@pytest.mark.parametrize("q,r,n,galois", [
    (60, 5, 16500, False),      # 300 rows: 272 workgroups a vector on 256 CUs
    (60, 5, 16500, True),
    (67, 8, 11000, False),      # 536 rows: 264, three row tiles
    (100, 1, 33000, True),      # 100 rows: 264 column tiles
])
def test_persistent_grid(keys, q, r, n, galois):
    rot = [((7 * i) % 31) - 15 for i in range(r)]
    imc, ctx, ref, call = _setup(keys, q, n, 0, galois, q * r)
    main, ld = torch.cuda.current_stream(), n + 3
    at = torch.tensor([0, n // 2, n - 1]).cuda()
    want = ref(rot, [(e, e + 1) for e in at.tolist()])
    plain = call(imc.DOT_TILES_EXPANDED_128x128, main, rot, n, ld)
    for tiles in (1, 2, 3):
        got = call(tiles | imc.DOT_PERSISTENT, main, rot, n, ld)
        for g, p, w in zip(got, plain, want):
            assert torch.equal(g, p), tiles
            assert np.array_equal(g[:, at].cpu().numpy().view(np.uint16), w), tiles
    ctx.close()


@pytest.mark.parametrize("q,r,n,first,galois,mask", [
    (33, 8, 16400, 64, False, True),     # 264 rows: 8 in a launch of their own
    (64, 5, 16390, 0, True, True),       # 320: 64
    (64, 6, 16385, 0, True, True),       # 384: 128
    (35, 11, 16385, 0, True, False),     # 385: 129, in the second tile
    (48, 4, 16385, 0, False, True),      # one 192-row tile
    (43, 3, 16385, 64, True, True),      # 129 rows in one
    (19, 5, 16400, 0, True, True),       # 95 in a 128-row tile
])
def test_rows_past_the_last_tile_against_oracle(keys, q, r, n, first, galois, mask):
    rot = [((7 * i) % 31) - 15 for i in range(r)]
    imc, ctx, ref, call = _setup(keys, q, n, first, galois, q * r)
    at = torch.tensor([0, 127, 128, n // 2, n - 1]).cuda()
    got = call(imc.DOT_TILES_EXPANDED_256x128, torch.cuda.current_stream(), rot, n, n + 3, mask)
    for g, w in zip(got, ref(rot, [(e, e + 1) for e in at.tolist()])):
        if g is not None:
            assert np.array_equal(g[:, at].cpu().numpy().view(np.uint16), w)
            assert (g[:, n:] == 7).all()
    ctx.close()
