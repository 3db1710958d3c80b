"""The rotation kernel's tiles at every height a last row tile can have, alone or
after the others, whole and with the K loop split (parts of one, an odd and an
even number of segments), against the expanded kernel."""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev64(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


@pytest.mark.parametrize("q,r,n,first,galois,mask", [
    (1, 13, 1, 0, False, True),
    (4, 16, 1100, 64, False, True),        # 64 rows; 18 tiles, 14 parts of 3 segments
    (5, 13, 1100, 64, True, True),         # 65
    (8, 16, 700, 0, False, True),          # 128; parts of 2
    (10, 13, 3000, 0, True, False),        # 130, code dot alone
    (12, 16, 129, 0, False, True),         # 192; parts of 1
    (15, 13, 127, 64, True, True),         # 195
    (16, 16, 1025, 0, False, True),        # 256
    (20, 13, 1025, 0, False, True),        # 260: a last tile of 4, apart
    (16, 24, 1029, 64, True, True),        # 384: of 128, apart
    (17, 23, 1029, 64, False, True),       # 391: of 135, in order
    (25, 31, 300, 0, True, True),          # 775: four tiles, the last of 7
])
def test_rotation_tile_heights(keys, q, r, n, first, galois, mask):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc
    from paper_2405_04463_amd.pipeline import SharedDB, SharedQueries

    rows, ld = q * r, n + 3
    rot = [((7 * i) % 31) - 15 for i in range(r)]           # distinct, in no order
    ctx = imc.Context(imc.Keys(*keys), max_rows=rows)
    dc, dm = wl.gen_codes(95, first, n)
    qc, qm = wl.gen_codes(95, 0, q, query=True)
    db = SharedDB(ctx, first + n, parties=(0,), galois=galois)
    db.enroll(dev64(dc), dev64(dm), first)
    qs = SharedQueries(ctx, dev64(qc), dev64(qm), 60, keep_raw=False, galois=galois)
    ids = imc.make_ids(60, rot, first)

    def call(tiles, stream):
        ctx.set_dot_tiles(tiles)
        c = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda")
        m = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda") if mask else None
        torch.cuda.synchronize()
        ctx.dot_shares(0, qs.op[0], q, ids, db.regions[0], db.capacity, n, c, m, ld, stream, galois=galois)
        torch.cuda.synchronize()
        return c, m

    want = call(imc.DOT_TILES_EXPANDED_256x128, torch.cuda.current_stream())
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):      # split, and not: the scratch is the first's
        c, m = call(imc.DOT_TILES_ROTATION, stream)
        assert torch.equal(c, want[0]) and (m is None or torch.equal(m, want[1]))
    ctx.close()
