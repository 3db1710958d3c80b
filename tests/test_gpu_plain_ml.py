"""The public mask overlap and the rotated masks against numpy on the unpacked
bits: row and entry counts around the 128 x 128 tile and its 64 x 64 and
16 x 16 parts, every rotation, masks of all ones and of none, operands that
are only 8-byte aligned, and columns past n left alone."""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _ctx(keys):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc

    return imc, imc.Context(imc.Keys(*keys), max_rows=1)


@pytest.mark.parametrize("rows,n,ld", [(1, 1, 1), (16, 17, 20), (64, 65, 65), (127, 129, 131), (129, 64, 64),
                                       (200, 300, 300)])
def test_overlap(keys, rows, n, ld):
    imc, ctx = _ctx(keys)
    _, dm = wl.gen_codes(95, 0, n)
    _, rm = wl.gen_codes(95, 0, rows, query=True)
    full = np.uint64(2**64 - 1)
    dm[0] = full
    rm[0] = full
    dm[n // 2 + n % 2:n // 2 + n % 2 + 1] = 0
    rm[rows - 1] = rm[rows - 1] if rows == 1 else 0
    want = wl.unpack(rm).astype(np.int32) @ wl.unpack(dm).astype(np.int32).T
    assert want[0, 0] == wl.L
    put = lambda a: torch.cat([torch.zeros(1, dtype=torch.int64), torch.from_numpy(  # noqa: E731
        np.ascontiguousarray(a).view(np.int64)).reshape(-1)]).cuda()[1:]
    ml = torch.full((rows, ld), 7, dtype=torch.int16, device="cuda")
    r, d = put(rm), put(dm)
    assert r.data_ptr() % 16 == 8
    ctx.plain_ml(r, rows, d, n, ml, ld)
    got = ml.cpu().numpy()
    assert np.array_equal(got[:, :n], want) and (got[:, n:] == 7).all()
    ctx.close()


def test_rotated_masks(keys):
    imc, ctx = _ctx(keys)
    _, qm = wl.gen_codes(96, 0, 3, query=True)
    rot = list(range(-15, 16))
    out = torch.zeros(3 * len(rot), 200, dtype=torch.int64, device="cuda")
    ctx.rotate_masks(torch.from_numpy(qm.view(np.int64)).cuda(), 3, imc.make_ids(0, rot), out)
    got = out.cpu().numpy().view(np.uint64)
    for i in range(3):
        for j, s in enumerate(rot):
            assert np.array_equal(got[i * len(rot) + j], wl.pack(wl.rotate_bits(wl.unpack(qm[i:i + 1])[0], s)[None])[0])
    ctx.close()
