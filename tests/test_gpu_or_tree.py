"""The OR-tree's components against the oracle's at the edges of the chunks that
one workgroup reduces (1,024 words) and over one, two and three passes, with
rows longer than the words in use."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from fullcheck import check_or_tree_components  # noqa: E402


@pytest.mark.parametrize("q,r,nw,pad", [
    (3, 1, 1, 0), (2, 1, 2, 1), (1, 1, 8, 0), (2, 31, 33, 2),          # 1, 2, 8, 1,023 words
    (2, 32, 32, 0), (1, 25, 41, 0), (2, 7, 293, 1),                    # 1,024, 1,025, 2,051
    (1, 17, 964, 0), (1, 31, 33826, 0),                                # 16,388; 1,048,606: three passes
])
def test_or_tree_components(keys, q, r, nw, pad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_04463_amd as imc

    dealer, party = keys
    ctx = imc.Context(imc.Keys(dealer, party), max_rows=1)
    rng = np.random.default_rng(q + r * nw)
    m = rng.integers(0, 2**64, (3, q * r, nw + pad), dtype=np.uint64)
    planes = [torch.from_numpy(np.stack([m[p], m[(p + 2) % 3]]).view(np.int64)).cuda() for p in range(3)]
    ws = torch.full((max(8, imc.or_tree_ws_bytes(q, r, nw)),), 255, dtype=torch.uint8, device="cuda")
    dup = [torch.full((2, q), 9, dtype=torch.uint8, device="cuda") for _ in range(3)]
    ctx.or_tree(planes, q, nw, nw + pad, imc.make_ids(77, [0] * r), ws, ws.numel(), dup)
    check_or_tree_components(party, m[:, :, :nw], [d.cpu().numpy() for d in dup], q, r, 77)
    ctx.close()
