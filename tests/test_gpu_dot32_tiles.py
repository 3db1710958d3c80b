"""The rotation kernel over Z_2^32 at the edges of its row tiles (64 and 128 rows)
and entry tiles, for lists of the fewest and the most rotations of each staging,
against calls of up to 12 rotations, which take the kernel that reads operands
from memory."""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev64(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


@pytest.mark.parametrize("q,r,n,first", [
    (1, 13, 1, 0),
    (4, 16, 129, 64),        # 64 rows
    (5, 13, 127, 0),         # 65
    (8, 16, 1030, 0),        # 128; 9 column tiles
    (10, 13, 128, 64),       # 130: a second tile of 2
    (7, 25, 200, 0),         # 175: the most rotations of the wide staging
    (5, 26, 65, 64),         # 130: the fewest of the narrow one
    (9, 31, 1025, 0),        # 279
])
def test_dot32_tile_edges(keys, q, r, n, first):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc
    from paper_2405_04463_amd.pipeline import SharedDB32, SharedQueries32

    rot = [((7 * i) % 31) - 15 for i in range(r)]           # distinct, in no order
    ctx = imc.Context(imc.Keys(*keys), max_rows=q * r)
    dc, dm = wl.gen_codes(97, first, n)
    qc, qm = wl.gen_codes(97, 0, q, query=True)
    db = SharedDB32(ctx, first + n, vecs=(0,))
    db.enroll(dev64(dc), dev64(dm), first)
    qs = SharedQueries32(ctx, dev64(qc), dev64(qm), 80, vecs=(0,))

    def call(rots):
        ld = n + 3
        out = torch.full((q * len(rots), ld), 7, dtype=torch.int32, device="cuda")
        ctx.dot32_shares(1, qs.op[0][1], q, imc.make_ids(80, rots, first), db.regions[0][1], db.capacity, n, out, ld)
        return out.view(q, len(rots), ld)

    got = call(rot)
    want = torch.cat([call(rot[i:i + 12]) for i in range(0, r, 12)], 1)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    ctx.close()
