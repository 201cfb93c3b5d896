"""GPU parity of the GEMM's forms for few tokens (up to 64: operands through LDS
from K = 1088 on) and for a few hundred (tiles of 32 or 64 tokens x 64 channels
with K split over the workgroup's waves; 128 x 128 tiles with K in two halves),
at the edges of their tiles, stages and wave ranges: token remainders of one and tile - 1, N not a
multiple of the tile, fewer spans than waves, spans that fill no whole stage,
every rank, both group sizes, with and without a bias.

y against the float64 oracle: the relative Frobenius tolerance of
parity_helpers.check_y, and every element within the bound of the GEMM's
arithmetic (parity_helpers.check_y_elements)."""

import numpy as np
import pytest
import torch

from oracle import qwam_oracle as O
from paper_2609_33269_amd import inputs as I
from paper_2609_33269_amd import qwam as Q

from parity_helpers import bits, check_sampled_rows, check_y, check_y_elements, gpu_layer, log, oracle_factors, run_gpu, y_abs_terms

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    Q.lib()


SHAPES = [
    (1, 1088, 16, 16, 64, True),       # few tokens, staged: ranges of three groups, the last wave idle
    (33, 2624, 80, 48, 32, False),     # 41 groups: ranges of six, stages of four and two; one token of block 2
    (64, 4160, 112, 64, 64, True),     # 65 groups: ranges of nine
    (17, 14336, 48, 32, 32, False),    # ranges of 28: seven full stages
    # M, K, N, r, group, bias: the form the launcher's estimate picks
    (65, 64, 16, 16, 64, True),        # 32 x 64, four waves: one span, three waves idle, 16 of 64 columns
    (95, 448, 208, 32, 64, False),     # four waves, seven spans (last range one span), 31 of 32 tokens
    (97, 832, 1040, 48, 32, True),     # group 32, one token of the last tile
    (66, 7168, 80, 64, 64, True),      # 32 x 64, eight waves: deep K, ragged columns
    (127, 14336, 64, 16, 32, False),   # eight waves, group 32
    (257, 2112, 2000, 32, 64, True),   # 64 x 64, four waves: one token of the last tile, 33 spans
    (383, 1600, 2064, 64, 32, False),  # 64 x 64, group 32, rank 64, 25 spans
]


@pytest.mark.parametrize("M,K,N,r,group,bias", SHAPES)
def test_gemm_form_parity(M, K, N, r, group, bias):
    d = I.custom(M, K, N, r, seed=17 + M, n_outliers=3, with_bias=bias)
    f = dict(oracle_factors(d), group=group)
    log(f"  GEMM form M={M} K={K} N={N} r={r} group={group} bias={bias}")
    ref = O.asp_linear(d.x, f, bias_bits=d.bias)
    layer = gpu_layer(f, d.bias)
    x, xq, xs, t, y = run_gpu(layer, d.x)
    tg = bits(t)
    y_t = ref["y"] + (O.bf16_bits_to_f64(tg) - O.bf16_bits_to_f64(ref["t"])) @ O.bf16_bits_to_f64(f["L2"])
    at = y_abs_terms(ref["sx"], ref["sw"], ref["P"], tg, f["L2"], d.bias)
    check_y_elements(bits(y), y_t, at, ref["P"].shape[2], r)
    check_y(bits(y), ref["y"])
    again = Q.asp_linear(layer, xq, xs, t)
    assert torch.equal(again.view(torch.int16), y.view(torch.int16)), "the sum over the waves is in a fixed order"


@pytest.mark.parametrize("M,K,N,r,group,bias", [
    (300, 3136, 10256, 32, 64, True),   # 49 spans: 7 and 6 stages, one span in the last; 16 columns and 44 tokens of the last tiles
    (520, 1088, 6160, 48, 32, False),   # group 32, rank 48: 17 spans, 3 and 2 stages; 8 tokens of the last tile
])
def test_large_tiles_in_two_halves(M, K, N, r, group, bias):
    """128 x 128 tiles with K in two halves (tile counts of 170 to 256), on
    sampled tokens, every column."""
    d = I.custom(M, K, N, r, seed=23 + M, n_outliers=3, with_bias=bias)
    f = dict(oracle_factors(d), group=group)
    log(f"  GEMM in two halves M={M} K={K} N={N} r={r} group={group} bias={bias}")
    wq, sw, inv_lam, _ = O.pack_weights(f["R"], f["lam"], group)
    xq_ref, sx_ref, _, _, _ = O.quantize_activations(d.x, inv_lam, f["L1"], 0, group)
    layer = gpu_layer(f, d.bias)
    x, xq, xs, t, y = run_gpu(layer, d.x)
    assert (xq.cpu().numpy() == xq_ref).all() and (xs.cpu().numpy() == sx_ref.T).all()
    rows = sorted({0, 31, 32, 63, 64, 127, 128, M - 1, M - 2} | set(range(3, M, 37)))
    check_sampled_rows(layer, xq, y, xq_ref, sx_ref, bits(t), wq, sw, f["L2"], np.array(rows), d.bias)
    again = Q.asp_linear(layer, xq, xs, t)
    assert torch.equal(again.view(torch.int16), y.view(torch.int16)), "the halves are added in a fixed order"
