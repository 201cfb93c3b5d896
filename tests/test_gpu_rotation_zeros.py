"""Signs of zeros through the rotated activation kernels: the lane stages of the
transform keep some values negated until the final multiply, and passes that
hold a -0 take an exact form.  A zero code's stored sign is that of the scaled
value, so every byte is compared with the oracle's for tokens of +0, of -0, of
both, with cancelling pairs, and for negative smoothing factors (which turn +0
into -0); every block size, both kernels (one workgroup per token, and tiles)."""

import numpy as np
import pytest
import torch

from oracle import qwam_oracle as O
from paper_2609_33269_amd import inputs as I
from paper_2609_33269_amd import qwam as Q

from parity_helpers import bf16_dev, bits, gpu_layer, log, oracle_factors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,r", [(24, 1024, 16), (70, 1024, 32), (70, 512, 16), (24, 768, 48), (70, 320, 16), (70, 2176, 32),
                                   (24, 80 * 64, 16)])
@pytest.mark.parametrize("deflate", [False, True])
def test_signed_zeros(M, K, r, deflate):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = I.custom(M, K, 64, r, seed=K + M, n_outliers=2)
    x = d.x.copy()
    rng = np.random.default_rng(K)
    x[0] = 0x0000                                            # +0
    x[1] = 0x8000                                            # -0
    x[2] = np.where(rng.random(K) < 0.5, 0x0000, 0x8000)     # both
    x[3, 1::2] = x[3, 0::2]                                  # a - b = 0 in the first stage
    x[4, 1::2] = x[4, 0::2] ^ 0x8000                         # a + b = 0
    x[5] = x[5, 0]                                           # constant: all but one output of a block are 0
    x[6] = np.where(rng.random(K) < 0.5, x[6, 0], x[6, 0] ^ 0x8000)
    x[7, : K // 2] = 0x8000
    x[8] = np.where(rng.random(K) < 0.02, x[8], 0x8000)
    f = oracle_factors(d, hadamard=True)
    f["lam"] = f["lam"].copy()
    f["lam"][::7] *= -1.0
    ref = O.asp_linear(x, f, deflate=deflate)
    log(f"  signed zeros M={M} K={K} r={r} block={f['hadamard']} deflate={deflate}")
    layer = gpu_layer(f)
    xq, xs, t = (Q.quantize_act_deflated if deflate else Q.quantize_act)(layer, bf16_dev(x))
    torch.cuda.synchronize()
    assert (xs.cpu().numpy() == ref["sx"].T).all(), "scales"
    bad = np.argwhere(xq.cpu().numpy() != ref["xq"])
    assert bad.size == 0, f"packed bytes differ at {bad[:5].tolist()}"
    if deflate:
        assert (bits(t) == ref["t"]).all()
