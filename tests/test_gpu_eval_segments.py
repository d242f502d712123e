"""GPU parity of kvp_eval_configs at the edges of its segments: one block attends over one keep level's new tokens, and the
levels are combined afterwards.  Losses against the oracle in every P.V form, and no write beyond the stated workspace."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import torch_bits

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# name, (L, H, T, G, W), configurations (bits, group, keep)
CASES = [
    ("one stream, tokens nobody keeps", (2, 2, 333, 4, 32), [(16, 0, 100)]),
    ("hidden reference, one short level", (1, 3, 300, 7, 32), [(4, 64, 33), (2, 32, 33)]),
    ("levels of one token, below the window, and all", (2, 1, 201, 1, 40),
     [(8, 128, 1), (8, 128, 2), (16, 0, 20), (4, 32, 40), (4, 32, 41), (2, 64, 72), (16, 0, 200), (16, 0, 201)]),
    ("every codec, two row blocks", (1, 2, 515, 8, 20),
     [(b, g, k) for b in (8, 4, 2) for g in (32, 64, 128) for k in (130, 515)] + [(16, 0, 64)]),
]


@pytest.mark.parametrize("pv", ["default", "matrix", "fp32"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: c[0])
def test_segments(case, pv):
    import paper_2512_14946_amd as kvp
    name, (L, H, T, G, W), cfgs = case
    print("[case] eval", name, pv, flush=True)
    K, V = workloads.make_kv(L, T, H, 128, seed=5)
    Q = workloads.make_q(L, W, G * H, 128, seed=5)
    need = kvp.kvp_eval_workspace_bytes(L, H, G * H, W, T, len(cfgs))
    buf = torch.full((need + 4096,), 0xAB, dtype=torch.uint8, device=DEV)
    loss, part = kvp.kvp_eval_configs(Q.to(DEV), K.to(DEV), V.to(DEV), cfgs, ws=buf[:need], want_partial=True,
                                      pv_matrix_cores=pv == "matrix", pv_fp32=pv == "fp32")
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0xAB).all())
    want, want_part = oracle.eval_configs(torch_bits(Q), torch_bits(K), torch_bits(V), cfgs)
    got = loss.cpu().numpy()
    # fp32 sums throughout; the default form rounds probabilities to 16 bits (2^-12 relative each, averaged over the rows)
    tol = 2e-4 if pv == "default" else 2e-5
    assert np.all(np.abs(got - want) <= tol * np.abs(want) + 1e-6)
    for c, (b, _, k) in enumerate(cfgs):
        if b == 16 and k == T:
            assert got[c] == 0.0                    # the identity candidate goes through the reference's own steps
    assert np.all(np.abs(part.cpu().numpy()[:, :, 1] - np.asarray(want_part)[:, :, 1]) <= 1e-3 * np.asarray(want_part)[:, :, 1])
