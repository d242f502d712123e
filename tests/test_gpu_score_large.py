"""GPU parity of kvp_score_tokens where a call is large enough for its throughput kernel (at least 2048 units of 64 keys):
chunk and unit edges, query-tile counts, masks, the fall-back of an out-of-range reference, determinism."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import torch_bits

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# L, H, T, G, W, causal, force_window
SHAPES = [
    (2, 8, 8192, 1, 1, True, True),         # 2048 units exactly, one per wave; one query row
    (3, 5, 9001, 3, 11, True, False),       # ragged rows, blocks that span two rows; M = 33: two query tiles
    (3, 5, 9001, 1, 50, False, True),       # no causal mask
    (130, 8, 100, 4, 32, True, True),       # many short rows per block; the window begins in the second unit
    (257, 8, 64, 1, 40, True, False),       # every chunk's first tile touches the window
    (1, 1, 131100, 2, 32, True, True),      # one row over all blocks: the chunk statistics get a launch of their own
    (28, 4, 1200, 7, 32, True, False),      # 7 query tiles in the instantiation for 8
    (1, 8, 16400, 8, 64, True, True),       # 512 rows, units beyond the row's end
]


def _run(Q, K, causal, fw):
    import paper_2512_14946_amd as kvp
    a = kvp.kvp_score_tokens(Q.to(DEV), K.to(DEV), causal=causal, force_window=fw)
    b = kvp.kvp_score_tokens(Q.to(DEV), K.to(DEV), causal=causal, force_window=fw)
    torch.cuda.synchronize()
    assert torch.equal(a, b)                # key units are handed out dynamically: the result must not depend on it
    return a.cpu().numpy()


def _cells(L, H, limit):
    """First, last and evenly spaced (layer, head) cells: the oracle takes up to a second per cell."""
    n = L * H
    return sorted({int(round(i)) for i in np.linspace(0, n - 1, min(n, limit))})


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_scores_of_large_calls(shape):
    L, H, T, G, W, causal, fw = shape
    print("[case] score", shape, flush=True)
    K, _ = workloads.make_kv(L, T, H, 128, seed=3)
    Q = workloads.make_q(L, W, G * H, 128, seed=3)
    got = _run(Q, K, causal, fw)
    for c in _cells(L, H, 2 if T * G * W > 1 << 21 else 24):
        l, h = divmod(c, H)
        want = oracle.score_tokens(torch_bits(Q[l:l + 1, :, h * G:(h + 1) * G]), torch_bits(K[l:l + 1, :, h:h + 1]), causal, fw)[0, 0]
        fin = np.isfinite(want)
        assert np.array_equal(np.isfinite(got[l, h]), fin)
        # logits of a few tens carry an fp32 error of a few 1e-6, and so does each exponential relative to itself
        assert np.all(np.abs(got[l, h][fin] - want[fin]) <= 2e-5 * np.abs(want[fin]) + 1e-7 * G * W / T)


def test_scores_when_later_keys_exceed_the_reference():
    """Logits that grow by thousands along a row: sums relative to the first keys overflow and the chunk starts over."""
    L, H, T, G, W = 2, 8, 8192, 1, 8
    print("[case] score overflow", flush=True)
    K, _ = workloads.make_kv(L, T, H, 128, seed=4)
    Q = workloads.make_q(L, W, G * H, 128, seed=4)
    K[0, 700, 3] = (Q[0, 2, 3].float() * 60).to(torch.bfloat16)      # one row's logit jumps to about 700
    K[1, 5000:5002, 6] = (Q[1, 0, 6].float() * 60).to(torch.bfloat16)
    got = _run(Q, K, True, False)
    for l, h in [(0, 3), (1, 6), (0, 0)]:
        want = oracle.score_tokens(torch_bits(Q[l:l + 1, :, h:h + 1]), torch_bits(K[l:l + 1, :, h:h + 1]), True, False)[0, 0]
        # a logit of 700 in fp32 is off by up to 1e-4
        assert np.all(np.abs(got[l, h] - want) <= 1e-3 * np.abs(want) + 1e-7)
