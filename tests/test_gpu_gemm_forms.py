"""GPU parity of the GEMM's forms: for few tokens (up to 64: operands straight
to registers, or through LDS), for a few hundred (tiles of 32 or 64 tokens x 64
channels with K split over the workgroup's waves; 128 x 128 tiles with K in two
halves) and the 128 x 128 tiles themselves, at the edges of their tiles, stages
and wave ranges: token remainders of one and tile - 1, N not a multiple of the
tile, fewer spans than waves, spans that fill no whole stage, every rank, both
group sizes, with and without a bias.  Every case asserts the form it runs.

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
    # M, K, N, r, group, bias, form
    (1, 1088, 16, 16, 64, True, "few direct"),   # ranges of three groups, the last wave idle
    (50, 2368, 48, 32, 32, True, "few direct"),  # 37 groups: ranges of five, chunks of four and one
    (31, 1280, 48, 48, 64, False, "few staged"),  # 20 groups: ranges of three, the last of two, whole lines
    (33, 2624, 80, 48, 32, False, "few staged"),  # 41 groups: ranges of six, stages of four and two; one token of block 2
    (64, 4160, 112, 64, 64, True, "few staged"),  # 65 groups: ranges of nine
    (17, 14336, 48, 32, 32, False, "few staged"),  # ranges of 28: seven full stages
    (65, 64, 16, 16, 64, True, "32x64 w4"),      # one span, three waves idle, 16 of 64 columns
    (95, 448, 208, 32, 64, False, "32x64 w4"),   # seven spans (last range one span), 31 of 32 tokens
    (97, 832, 1040, 48, 32, True, "32x64 w4"),   # group 32, one token of the last tile
    (383, 1600, 2064, 64, 32, False, "32x64 w4"),  # group 32, rank 64, 25 spans, two rounds of tiles
    (66, 7168, 80, 64, 64, True, "32x64 w8"),    # deep K, ragged columns
    (127, 14336, 64, 16, 32, False, "32x64 w8"),  # group 32
    (257, 2112, 2000, 32, 64, True, "64x64 w4"),  # one token of the last tile, 33 spans
    (300, 3136, 5136, 64, 32, True, "64x64 w4"),  # group 32, rank 64, 49 spans: the last range one span
    (513, 832, 3088, 16, 32, False, "64x64 w4"),  # group 32, rank 16: a range of one span, one token of the last tile
    (385, 1344, 4112, 48, 32, True, "64x64 w4"),  # rank 48, 21 spans, 16 columns of the last tile
]


@pytest.mark.parametrize("M,K,N,r,group,bias,form", SHAPES)
def test_gemm_form_parity(M, K, N, r, group, bias, form):
    assert Q.probe_gemm_form(M, N, K, group) == form
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


LARGE = [
    # K in two halves (tile counts of 170 to 256): 16 columns and 44 tokens of the last tiles
    (300, 5184, 10256, 32, 64, True, "128x128 halves"),   # 81 spans: 11 and 10 stages, one span in the last
    (300, 3392, 10256, 64, 64, False, "128x128 halves"),  # 53 spans: 7 and 7 stages
    (300, 3072, 10256, 16, 64, True, "128x128 halves"),   # whole stages
    (300, 1600, 10256, 48, 32, False, "128x128 halves"),  # group 32: 25 spans, 4 and 3 stages
    (300, 1344, 10256, 16, 32, True, "128x128 halves"),   # 21 spans: 3 and 3 stages
    (300, 2112, 10256, 64, 32, True, "128x128 halves"),   # 33 spans: 5 and 4 stages
    # one pipeline over K: 20 tokens and 16 columns of the last tiles, every number of spans past the unrolled eight
    (1300, 128, 2576, 16, 64, True, "128x128"),           # 2 spans
    (1300, 192, 2576, 48, 64, False, "128x128"),          # 3
    (1300, 256, 2576, 64, 64, True, "128x128"),           # 4: one stage
    (1300, 832, 2576, 32, 64, True, "128x128"),           # 8 + 5
    (1300, 896, 2576, 64, 64, False, "128x128"),          # 8 + 6
    (1300, 960, 2576, 48, 64, True, "128x128"),           # 8 + 7
    (1300, 1024, 2576, 16, 64, False, "128x128"),         # 16
    (1300, 2112, 2576, 64, 64, True, "128x128"),          # 32 + 1
    (1300, 192, 2576, 16, 32, True, "128x128"),           # group 32: a partial stage alone
    (1300, 576, 2576, 64, 32, True, "128x128"),           # three stages, one span in the last
    (1300, 960, 2576, 48, 32, False, "128x128"),          # four, three spans in the last
    (2061, 1344, 2576, 32, 32, True, "128x128"),          # six; 13 tokens of the last tiles
]


@pytest.mark.parametrize("M,K,N,r,group,bias,form", LARGE)
def test_large_tiles(M, K, N, r, group, bias, form):
    """128 x 128 tiles, on sampled tokens, every column."""
    assert Q.probe_gemm_form(M, N, K, group) == form
    d = I.custom(M, K, N, r, seed=23 + M, n_outliers=3, with_bias=bias)
    f = dict(oracle_factors(d), group=group)
    log(f"  GEMM {form} M={M} K={K} N={N} r={r} group={group} bias={bias}")
    wq, sw, inv_lam, _ = O.pack_weights(f["R"], f["lam"], group)
    xq_ref, sx_ref, _, _, _ = O.quantize_activations(d.x, inv_lam, f["L1"], 0, group)
    layer = gpu_layer(f, d.bias)
    x, xq, xs, t, y = run_gpu(layer, d.x)
    assert (xq.cpu().numpy() == xq_ref).all() and (xs.cpu().numpy() == sx_ref.T).all()
    rows = sorted({0, 31, 32, 63, 64, 127, 128, M - 1, M - 2} | set(range(3, M, 37)))
    check_sampled_rows(layer, xq, y, xq_ref, sx_ref, bits(t), wq, sw, f["L2"], np.array(rows), d.bias)
    again = Q.asp_linear(layer, xq, xs, t)
    assert torch.equal(again.view(torch.int16), y.view(torch.int16)), "the halves are added in a fixed order"


@pytest.mark.parametrize("M,K,N,r,group,form", [
    (600, 512, 2304, 32, 64, "64x64 w4"),
    (400, 1600, 2064, 32, 32, "32x64 w4"),
    (100, 4096, 1024, 16, 64, "32x64 w8"),
    (300, 3136, 10256, 32, 64, "128x128"),
    (300, 3392, 10256, 32, 64, "128x128 halves"),
    (300, 1344, 10256, 48, 32, "128x128 halves"),
])
def test_repeat_runs_of_a_form(M, K, N, r, group, form):
    """A race proxy: 20 runs on four streams, several in flight, give the same bits."""
    assert Q.probe_gemm_form(M, N, K, group) == form
    g = torch.Generator(device="cuda").manual_seed(M)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    layer = Q.make_layer(rand(N, K), rand(K).abs() + 0.5, rand(K, r).bfloat16(), rand(r, N).bfloat16(), rand(N).bfloat16(),
                         group=group)
    acts = Q.quantize_act(layer, rand(M, K).bfloat16())
    want = Q.asp_linear(layer, *acts)
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()
    ys = [torch.full_like(want, float("nan")) for _ in range(20)]
    torch.cuda.synchronize()
    for i, y in enumerate(ys):
        Q.asp_linear(layer, *acts, out=y, stream=streams[i % 4])
    torch.cuda.synchronize()
    assert all(torch.equal(y.view(torch.int16), want.view(torch.int16)) for y in ys)
