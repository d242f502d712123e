"""GPU parity of kvp_score_tokens where a call has at least 2048 units of 64 keys: chunk and unit edges, query-tile counts,
masks, determinism, in the kernel for short rows and moderate calls and in the throughput kernel (rows of at least 48
units, 10240 units and more, 24576 with fewer than 128 query rows); the fall-back of an out-of-range reference of the latter."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import torch_bits

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# L, H, T, G, W, causal, force_window
THROUGHPUT_SHAPES = [
    (2, 8, 49152, 4, 32, True, True),       # 48 units per block; 16 chunks per row: a launch combines them
    (16, 5, 9997, 3, 43, False, True),      # ragged rows, blocks that span two rows; M = 129: five query tiles; no causal mask
    (32, 8, 3073, 8, 64, True, True),       # a block per row; 512 rows; one key in the last unit
    (87, 3, 3100, 4, 40, True, False),      # chunks begin at every unit of a row, in the window too
    (67, 8, 3010, 3, 11, True, True),       # M = 33: two query tiles; a block spans three rows
    (1, 1, 786500, 4, 32, True, True),      # one row over all blocks
    (1, 8, 98311, 7, 32, True, False),      # 7 query tiles in the instantiation for 8
    (6, 8, 32768, 1, 1, True, True),        # one query row
]
SHAPES = [
    (2, 8, 8192, 1, 1, True, True),         # 2048 units exactly; one query row
    (3, 5, 9001, 3, 11, True, False),       # ragged rows; M = 33: two query tiles
    (3, 5, 9001, 1, 50, False, True),       # no causal mask
    (130, 8, 100, 4, 32, True, True),       # many short rows; the window begins in the second unit
    (257, 8, 64, 1, 40, True, False),       # every chunk's first tile touches the window
    (1, 1, 131100, 2, 32, True, True),      # one row over all blocks: the chunk statistics get a launch of their own
    (28, 4, 1200, 7, 32, True, False),      # 7 query tiles in the instantiation for 8; four or five tiles per wave
    (1, 8, 16400, 8, 64, True, True),       # 512 rows, units beyond the row's end
]


def _run(Q, K, causal, fw):
    import paper_2512_14946_amd as kvp
    a = kvp.kvp_score_tokens(Q.to(DEV), K.to(DEV), causal=causal, force_window=fw)
    b = kvp.kvp_score_tokens(Q.to(DEV), K.to(DEV), causal=causal, force_window=fw)
    torch.cuda.synchronize()
    assert torch.equal(a, b)                # pass B of the throughput kernel hands key units out dynamically: no trace of it
    return a.cpu().numpy()


def _cells(L, H, limit):
    """First, last and evenly spaced (layer, head) cells: the oracle takes up to a second per cell."""
    n = L * H
    return sorted({int(round(i)) for i in np.linspace(0, n - 1, min(n, limit))})


@pytest.mark.parametrize("shape", SHAPES + THROUGHPUT_SHAPES, ids=str)
def test_scores_of_large_calls(shape):
    L, H, T, G, W, causal, fw = shape
    print("[case] score", shape, flush=True)
    dev = DEV if shape in THROUGHPUT_SHAPES else "cpu"
    K, _ = workloads.make_kv(L, T, H, 128, seed=3, device=dev)
    Q = workloads.make_q(L, W, G * H, 128, seed=3, device=dev)
    got = _run(Q, K, causal, fw)
    for c in _cells(L, H, 2 if T * G * W > 1 << 21 else 4 if shape in THROUGHPUT_SHAPES else 24):
        l, h = divmod(c, H)
        want = oracle.score_tokens(torch_bits(Q[l:l + 1, :, h * G:(h + 1) * G]), torch_bits(K[l:l + 1, :, h:h + 1]), causal, fw)[0, 0]
        fin = np.isfinite(want)
        assert np.array_equal(np.isfinite(got[l, h]), fin)
        # logits of a few tens carry an fp32 error of a few 1e-6, and so does each exponential relative to itself
        assert np.all(np.abs(got[l, h][fin] - want[fin]) <= 2e-5 * np.abs(want[fin]) + 1e-7 * G * W / T)


@pytest.mark.parametrize("T,G,W", [(8192, 1, 8), (49152, 4, 32)])
def test_scores_when_later_keys_exceed_the_reference(T, G, W):
    """One key whose logit is about 700 behind ordinary ones: in the throughput kernel (second size) sums relative to the
    first keys of the chunk overflow, and the chunk starts over."""
    L, H = 2, 8
    print("[case] score overflow", flush=True)
    K, _ = workloads.make_kv(L, T, H, 128, seed=4)
    Q = workloads.make_q(L, W, G * H, 128, seed=4)
    K[0, 700, 3] = (Q[0, 2, 3 * G].float() * 60).to(torch.bfloat16)      # one row's logit jumps to about 700
    K[1, 5000:5002, 6] = (Q[1, 0, 6 * G].float() * 60).to(torch.bfloat16)
    got = _run(Q, K, True, False)
    for l, h in [(0, 3), (1, 6), (0, 0)]:
        want = oracle.score_tokens(torch_bits(Q[l:l + 1, :, h * G:(h + 1) * G]), torch_bits(K[l:l + 1, :, h:h + 1]), True, False)[0, 0]
        # a logit of 700 in fp32 is off by up to 1e-4
        assert np.all(np.abs(got[l, h] - want) <= 1e-3 * np.abs(want) + 1e-7)
