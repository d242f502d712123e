"""GPU parity of kvp_smooth_scores where its kernel for up to 9 taps can go wrong: ends of its 2048-token tiles, rows and
outputs off 16-byte alignment, windows that cut a group of 4, infinities; the maximum bit for bit."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kernel", [1, 3, 5, 7, 9, 11])
@pytest.mark.parametrize("T,window,pad_in,pad_out", [(1, 0, 0, 0), (3, 3, 1, 2), (2047, 31, 0, 0), (2048, 32, 0, 1), (2049, 1, 3, 0),
                                                     (2052, 5, 4, 4), (4099, 2050, 1, 0), (6144, 0, 0, 0)])
def test_smooth_edges(T, window, pad_in, pad_out, kernel):
    import paper_2512_14946_amd as kvp
    print("[case] smooth", T, window, pad_in, pad_out, kernel, flush=True)
    rng = np.random.default_rng(T + kernel)
    s = rng.standard_normal((3, T)).astype(np.float32) ** 2
    s[1] = -s[1]
    if T > window > 0:
        s[:, T - window:] = np.inf                 # never a tap of the prefix
    src = torch.zeros(3, T + pad_in, device=DEV)
    src[:, :T] = torch.from_numpy(s).to(DEV)
    for mode in ("avg", "max"):
        out = torch.full((3, T + pad_out), 7.0, device=DEV)
        kvp.kvp_smooth_scores(src[:, :T], window, kernel, mode, out=out[:, :T])
        torch.cuda.synchronize()
        want = oracle.smooth_scores(s, window, kernel, mode)
        got = out.cpu().numpy()
        assert np.all(got[:, T:] == 7.0)           # nothing beyond the row
        if mode == "max":
            assert np.array_equal(got[:, :T], want)
        else:                                      # up to 11 sums and a division in fp32 of values of one sign
            fin = np.isfinite(want)
            assert np.array_equal(np.isfinite(got[:, :T]), fin)
            assert np.all(np.abs(got[:, :T][fin] - want[fin]) <= 1e-5 * np.abs(want[fin]))
