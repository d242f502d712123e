"""kvp_score_tokens at sizes of its throughput kernel and around them: what it may write, views, values that are no numbers,
the scratch of the library."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# L, H, T, G, W: many short rows and one long one, chunked; the throughput kernel with a block per row, with 48 units per
# block and a launch that combines the chunks, and with one row over all blocks
@pytest.mark.parametrize("shape", [(64, 8, 256, 4, 8), (130, 8, 100, 8, 64), (1, 1, 131100, 2, 32), (32, 8, 3073, 8, 64),
                                   (2, 8, 49152, 4, 32), (1, 1, 786500, 4, 32)], ids=str)
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


# L, H, T, G, W: the throughput kernel with many rows per block and with one row over many blocks; the chunked kernel
BOTH = [(32, 8, 3073, 4, 40), (2, 8, 49152, 4, 32), (8, 8, 2000, 4, 32)]


@pytest.mark.parametrize("shape", BOTH, ids=str)
def test_strided_and_broadcast_views(shape):
    """Head-major keys, queries cut out of a longer buffer, one layer's keys and queries for all layers: the same values
    give the same scores bit for bit."""
    import paper_2512_14946_amd as kvp
    L, H, T, G, W = shape
    print("[case] score views", shape, flush=True)
    K, _ = workloads.make_kv(L, T, H, 128, seed=12, device=DEV)
    Q = workloads.make_q(L, W, G * H, 128, seed=12, device=DEV)
    want = kvp.kvp_score_tokens(Q, K)
    head_major = K.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    wide_q = torch.zeros(L, W + 3, G * H + 1, 136, dtype=torch.bfloat16, device=DEV)
    wide_q[:, 2:W + 2, 1:, :128] = Q
    assert torch.equal(kvp.kvp_score_tokens(wide_q[:, 2:W + 2, 1:, :128], head_major), want)
    one = kvp.kvp_score_tokens(Q[:1].expand(L, -1, -1, -1), K[:1].expand(L, -1, -1, -1))
    same = kvp.kvp_score_tokens(Q[:1].repeat(L, 1, 1, 1), K[:1].repeat(L, 1, 1, 1))
    assert torch.equal(one, same) and torch.equal(one[0], one[-1])


@pytest.mark.parametrize("shape", BOTH, ids=str)
def test_non_finite_keys_stay_in_their_row(shape):
    """A NaN or an infinity in a key makes scores of its own (layer, head) row NaN, whichever tile of a chunk holds it, and
    leaves every other row as it was."""
    import paper_2512_14946_amd as kvp
    L, H, T, G, W = shape
    print("[case] score non-finite", shape, flush=True)
    K, _ = workloads.make_kv(L, T, H, 128, seed=13, device=DEV)
    Q = workloads.make_q(L, W, G * H, 128, seed=13, device=DEV)
    want = kvp.kvp_score_tokens(Q, K, force_window=False)
    bad = {(0, 1): (0, float("nan")), (0, 3): (T // 2, float("nan")), (1, 2): (T - W - 1, float("nan")),
           (1, 5): (3, float("inf")), (L - 1, 7): (T // 2 + 70, float("-inf"))}
    for (l, h), (t, x) in bad.items():
        K[l, t, h, 5] = x
    got = kvp.kvp_score_tokens(Q, K, force_window=False)
    clean = torch.ones(L, H, dtype=torch.bool, device=DEV)
    for l, h in bad:
        clean[l, h] = False
        assert bool(got[l, h].isnan().any())
    assert torch.equal(got[clean], want[clean])


def test_static_scratch_of_the_throughput_kernel():
    """kvp_score_tokens_static on a shape of the throughput kernel, and on a smaller one over what that left behind."""
    import paper_2512_14946_amd as kvp
    for L, H, T, G, W in [(2, 8, 49152, 4, 32), (1, 8, 4096, 4, 32), (2, 8, 49152, 8, 64)]:
        print("[case] score static", (L, H, T, G, W), flush=True)
        assert kvp.kvp_score_workspace_bytes(L, H, G * H, W, T) <= kvp.KVP_SCORE_STATIC_SCRATCH_BYTES
        K, _ = workloads.make_kv(L, T, H, 128, seed=14, device=DEV)
        Q = workloads.make_q(L, W, G * H, 128, seed=14, device=DEV)
        got = torch.full((L, H, T), float("nan"), device=DEV)
        kvp.kvp_score_tokens_static(Q, K, got)
        assert torch.equal(got, kvp.kvp_score_tokens(Q, K))
