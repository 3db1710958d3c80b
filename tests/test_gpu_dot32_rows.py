"""The rotation kernel over Z_2^32 on both heights of its tiles (64 rows where
tiles are few, on 256 CUs), against calls of up to 12 rotations on the kernel
that reads operands from memory, and the oracle on a few entries."""
import numpy as np
import pytest

import oracle as orc
import workload as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev64(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


@pytest.mark.parametrize("q,r,n,first", [
    (8, 13, 5000, 64),       # 104 rows: 80 tiles of 64 rows
    (33, 31, 64, 0),         # 1,023 rows: 16 tiles, the last of 63
    (8, 16, 16500, 0),       # 128 rows, whole tiles
    (5, 13, 33000, 0),       # 65
    (10, 13, 16500, 64),     # 130: a second tile of 2
    (9, 31, 10900, 0),       # 279
])
def test_dot32_tile_rows(keys, q, r, n, first):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc
    from paper_2405_04463_amd.pipeline import SharedDB32, SharedQueries32

    rot = [((7 * i) % 31) - 15 for i in range(r)]           # distinct, in no order
    ctx = imc.Context(imc.Keys(*keys), max_rows=q * r)
    dc, dm = wl.gen_codes(98, first, n)
    qc, qm = wl.gen_codes(98, 0, q, query=True)
    db = SharedDB32(ctx, first + n, vecs=(1,))
    db.enroll(dev64(dc), dev64(dm), first)
    qs = SharedQueries32(ctx, dev64(qc), dev64(qm), 80, vecs=(1,))

    def call(rots):
        ld = n + 3
        out = torch.full((q * len(rots), ld), 7, dtype=torch.int32, device="cuda")
        ctx.dot32_shares(1, qs.op[1][1], q, imc.make_ids(80, rots, first), db.regions[1][1], db.capacity, n, out, ld)
        return out.view(q, len(rots), ld)

    got = call(rot)
    want = torch.cat([call(rot[i:i + 12]) for i in range(0, r, 12)], 1)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    at = np.array([0, n // 2, n - 1])
    dsh = np.concatenate([orc.share32(keys[0], orc.DOM_SHARE32_DB, dc[e:e + 1], dm[e:e + 1], first + int(e))
                          for e in at])
    _, ref = orc.local_dot32(1, orc.share32(keys[0], orc.DOM_SHARE32_QUERY, qc, qm, 80), rot, dsh)
    got = got.reshape(q * r, n + 3)[:, torch.from_numpy(at).cuda()].cpu().numpy().view(np.uint32)
    assert np.array_equal(got, ref)
    ctx.close()
