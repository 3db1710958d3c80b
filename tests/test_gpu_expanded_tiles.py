"""The expanded kernel's tiles at the edges of their rows, the rows past
the last whole tile in a launch of their own (from 256 tiles on) or not,
against its 128 x 128 tiles."""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev64(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


@pytest.mark.parametrize("q,r,n,first,galois,mask", [
    (43, 3, 100, 64, False, True),       # 129 rows, the fewest of a 256-row tile; the K loop split
    (51, 5, 1000, 0, True, True),        # 255
    (32, 8, 129, 0, False, False),       # 256, code dot alone
    (32, 12, 1000, 64, True, True),      # 384, too few tiles to go apart
    (33, 8, 16400, 64, False, True),     # 264: 8 rows apart
    (64, 5, 16390, 0, True, True),       # 320: 64
    (25, 13, 16385, 0, False, True),     # 325: 69, expanded on request
    (64, 6, 16385, 0, True, True),       # 384: 128
    (35, 11, 16385, 0, True, False),     # 385: 129, in the second tile
    (48, 4, 16385, 0, False, True),      # 192-row tiles, whole
    (43, 3, 16385, 64, True, True),      # 129 in one: its last wave row idle
    (19, 5, 16400, 0, True, True),       # 128-row tiles, 95 rows
])
def test_expanded_rows(keys, q, r, n, first, galois, mask):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc
    from paper_2405_04463_amd.pipeline import SharedDB, SharedQueries

    rows, ld = q * r, n + 3
    ctx = imc.Context(imc.Keys(*keys), max_rows=rows)
    dc, dm = wl.gen_codes(99, first, n)
    qc, qm = wl.gen_codes(99, 0, q, query=True)
    db = SharedDB(ctx, first + n, parties=(2,), galois=galois)
    db.enroll(dev64(dc), dev64(dm), first)
    qs = SharedQueries(ctx, dev64(qc), dev64(qm), 70, keep_raw=False, galois=galois)
    ids = imc.make_ids(70, [((7 * i) % 31) - 15 for i in range(r)], first)
    got = []
    for tiles in (imc.DOT_TILES_EXPANDED_256x128, imc.DOT_TILES_EXPANDED_128x128):
        ctx.set_dot_tiles(tiles)
        c = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda")
        m = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda") if mask else None
        ctx.dot_shares(2, qs.op[2], q, ids, db.regions[2], db.capacity, n, c, m, ld, galois=galois)
        got.append((c, m))
    torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0]) and (not mask or torch.equal(got[0][1], got[1][1]))
    ctx.close()
