"""The native per-token calls: what they refuse goes to the checked Python path,
which names the wrong argument (on the host); on the GPU they return what the
ctypes path returns, also into given outputs, and read the layer's tensors of
the moment of the call."""

import dataclasses

import pytest
import torch

from paper_2609_33269_amd import qwam as Q


def test_wrong_arguments_are_named():
    cpu = Q.PackedLayer(64, 64, 16, *[torch.zeros(1)] * 5)
    for call in (lambda: Q.asp_layer(cpu, torch.zeros(4, 64)), lambda: Q.quantize_act(cpu, torch.zeros(4, 64)),
                 lambda: Q.asp_linear(cpu, torch.zeros(4, 32), None, None)):
        with pytest.raises(ValueError, match="wq must be a GPU tensor"):
            call()


@pytest.mark.gpu
@pytest.mark.parametrize("M", [1, 37, 130])
def test_native_calls_match_ctypes(M):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(M)
    K, N, r = 256, 192, 16
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    layer = Q.make_layer(rand(N, K), rand(K).abs() + 0.5, rand(K, r).bfloat16(), rand(r, N).bfloat16(), rand(N).bfloat16())
    x = rand(M, K).bfloat16()
    s = torch.cuda.current_stream()                     # an explicit stream takes the ctypes path
    for fn in (Q.quantize_act, Q.quantize_act_deflated):
        a, b = fn(layer, x), fn(layer, x, stream=s)
        out = tuple(torch.empty_like(t) for t in a)
        c = fn(layer, x, out=out)
        assert all(torch.equal(p, q) and torch.equal(p, w) and w is o for p, q, w, o in zip(a, b, c, out))
    y, y2 = Q.asp_linear(layer, *a), Q.asp_linear(layer, *a, stream=s)
    given = torch.empty_like(y)
    assert torch.equal(y, y2) and Q.asp_linear(layer, *a, out=given) is given and torch.equal(y, given)
    if M <= 64:
        assert torch.equal(Q.asp_layer(layer, x), Q.asp_layer(layer, x, stream=s))
    else:
        with pytest.raises(Q.QwamError, match="QWAM_ERR_UNSUPPORTED"):
            Q.asp_layer(layer, x)
    # the layer's fields count at the call, not at an earlier one
    unbiased = dataclasses.replace(layer, bias=None)
    assert torch.equal(Q.asp_linear(unbiased, *a), Q.asp_linear(unbiased, *a, stream=s))
    layer.bias = None
    assert torch.equal(Q.asp_linear(layer, *a), Q.asp_linear(unbiased, *a))
    with pytest.raises(TypeError, match="x must be torch.bfloat16"):
        Q.quantize_act(layer, x.float())
    with pytest.raises(ValueError, match="x must be contiguous"):
        Q.quantize_act(layer, rand(M, 2 * K).bfloat16()[:, ::2])
    with pytest.raises(ValueError, match="t must have shape"):
        Q.asp_linear(layer, a[0], a[1], a[2][:, :8].contiguous())
