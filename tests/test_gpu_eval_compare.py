"""GPU parity of kvp_eval_configs where its comparison step takes several streams per block: short contexts with many
(layer, head) cells.  Covered: 1 .. 5 streams per block, a last group of fewer streams, 8 keep levels (78 KB of LDS), and
each arrangement of the attention launch's blocks."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import torch_bits

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

ALL = [(16, 0)] + [(b, g) for b in (8, 4, 2) for g in (32, 64, 128)]
LEVELS8 = (3, 9, 17, 24, 33, 40, 55, 64)

# name, (L, H, T, G, W), codecs, keep levels (a product of more than 64 is thinned out); streams per block = cells * streams / 256, at most 5
CASES = [
    ("2 per block of 10", (7, 8, 64, 2, 16), ALL, (16, 64)),
    ("3 per block of 10: a last group of one", (11, 7, 64, 2, 16), ALL, (16, 48, 64)),
    ("4 per block of 9: a last group of one", (29, 4, 64, 1, 20), ALL[:9], (20, 40)),
    ("5 per block of 6: a last group of one; 8 levels", (32, 8, 64, 2, 16), ALL[:6], LEVELS8),
    ("5 per block of 10; 8 levels and tokens nobody keeps", (16, 8, 70, 4, 8), ALL, LEVELS8),
    ("one level; the matrix-core form's reference walks on", (16, 8, 64, 2, 16), ALL[:4], (30,)),
    ("two row blocks; hidden reference", (16, 8, 64, 7, 32), ALL[1:5], (32, 50, 63)),
]


@pytest.mark.parametrize("pv", ["default", "matrix", "fp32"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: c[0])
def test_streams_per_compare_block(case, pv):
    import paper_2512_14946_amd as kvp
    name, (L, H, T, G, W), codecs, keeps = case
    print("[case] eval compare", name, pv, flush=True)
    cfgs = [(b, g, k) for b, g in codecs for k in keeps]
    cfgs = [c for i, c in enumerate(cfgs) if len(cfgs) <= 64 or i % 5 != 4]     # at most 64; every codec and level stays
    K, V = workloads.make_kv(L, T, H, 128, seed=8)
    Q = workloads.make_q(L, W, G * H, 128, seed=8)
    need = kvp.kvp_eval_workspace_bytes(L, H, G * H, W, T, len(cfgs))
    buf = torch.full((need + 4096,), 0xAB, dtype=torch.uint8, device=DEV)
    loss, part = kvp.kvp_eval_configs(Q.to(DEV), K.to(DEV), V.to(DEV), cfgs, ws=buf[:need], want_partial=True,
                                      pv_matrix_cores=pv == "matrix", pv_fp32=pv == "fp32")
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0xAB).all())
    got, got_part = loss.cpu().numpy(), part.cpu().numpy()
    want, want_part = oracle.eval_configs(torch_bits(Q), torch_bits(K), torch_bits(V), cfgs)
    # fp32 sums throughout; the default form rounds probabilities to 16 bits (2^-12 relative each, averaged over the rows)
    tol = 2e-4 if pv == "default" else 2e-5
    assert np.all(np.abs(got - want) <= tol * np.abs(want) + 1e-6)
    for c, (b, _, k) in enumerate(cfgs):
        if b == 16 and k == T:
            assert got[c] == 0.0
    want_part = np.asarray(want_part)
    assert np.all(np.abs(got_part[:, :, 1] - want_part[:, :, 1]) <= 1e-3 * want_part[:, :, 1])
