"""kvp_score_tokens at sizes of its throughput kernel and around them: what it may write."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# L, H, T, G, W: 512 rows use the largest share of the workspace; one long row; just below and above 2048 key units
@pytest.mark.parametrize("shape", [(64, 8, 256, 4, 8), (1, 1, 131100, 2, 32), (8, 8, 2048, 4, 32), (8, 8, 1984, 4, 32),
                                   (130, 8, 100, 8, 64)], ids=str)
def test_nothing_is_written_beyond_the_workspace_or_the_scores(shape):
    import paper_2512_14946_amd as kvp
    L, H, T, G, W = shape
    print("[case] score guard", shape, flush=True)
    K, _ = workloads.make_kv(L, T, H, 128, seed=6, device=DEV)
    Q = workloads.make_q(L, W, G * H, 128, seed=6, device=DEV)
    need = kvp.kvp_score_workspace_bytes(L, H, G * H, W, T)
    ws = torch.full((need + 8192,), 0xAB, dtype=torch.uint8, device=DEV)
    out = torch.full((L * H * T + 1024,), 7.0, device=DEV)
    kvp.kvp_score_tokens(Q, K, out[:L * H * T].view(L, H, T), ws=ws[:need])
    want = kvp.kvp_score_tokens(Q, K)
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0xAB).all()) and bool((out[L * H * T:] == 7.0).all())
    assert torch.equal(out[:L * H * T].view(L, H, T), want)
