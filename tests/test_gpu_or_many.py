"""The OR-tree over many queries of few words: its components against the
oracle's where a workgroup takes several queries (the last one fewer), and its
time, which must not grow with the queries as long as they fit the GPU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from fullcheck import check_or_tree_components  # noqa: E402


def _call(keys, q, r, nw, pad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc

    ctx = imc.Context(imc.Keys(*keys), max_rows=1)
    rng = np.random.default_rng(q + r * nw)
    m = rng.integers(0, 2**64, (3, q * r, nw + pad), dtype=np.uint64)
    planes = [torch.from_numpy(np.stack([m[p], m[(p + 2) % 3]]).view(np.int64)).cuda() for p in range(3)]
    ws = torch.full((max(8, imc.or_tree_ws_bytes(q, r, nw)),), 255, dtype=torch.uint8, device="cuda")
    dup = [torch.full((2, q), 9, dtype=torch.uint8, device="cuda") for _ in range(3)]
    ids = imc.make_ids(77, [0] * r)
    return ctx, m, dup, lambda: ctx.or_tree(planes, q, nw, nw + pad, ids, ws, ws.numel(), dup)


# 256 CUs hold 2,048 workgroups of few words, 512 of the largest trees
@pytest.mark.parametrize("q,r,nw,pad", [
    (2048, 1, 1, 0), (2049, 1, 1, 1), (20001, 1, 1, 0), (140001, 1, 1, 0),   # 1, 2, 10 and 64 queries a workgroup
    (4097, 1, 2, 0), (2500, 3, 1, 1), (9001, 31, 1, 0),
    (5001, 4, 17, 2), (3001, 31, 5, 0),                   # 68 and 155 words
    (1201, 31, 16, 0), (1100, 17, 32, 1),                 # 496 words: two a workgroup; 544: one
])
def test_many_queries(keys, q, r, nw, pad):
    ctx, m, dup, run = _call(keys, q, r, nw, pad)
    run()
    check_or_tree_components(keys[1], m[:, :, :nw], [d.cpu().numpy() for d in dup], q, r, 77)
    ctx.close()


def test_time_of_many_queries(keys):
    """100,000 one-word trees are 1.8 million ChaCha12 blocks: some 20 us of the vector
    units, 57 times a call of 1,000 with a workgroup for each."""
    us = {}
    for q in (1000, 100_000):
        ctx, _, _, run = _call(keys, q, 1, 1, 0)
        run()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        best = []
        for _ in range(10):
            ev[0].record()
            for _ in range(20):
                run()
            ev[1].record()
            torch.cuda.synchronize()
            best.append(ev[0].elapsed_time(ev[1]) * 50)
        us[q] = min(best)
        ctx.close()
    assert us[100_000] < 20 * us[1000], us
