"""The native per-token calls: what they refuse goes to the checked Python path,
which names the wrong argument (on the host); on the GPU they return what the
ctypes path returns, also into given outputs, and read the layer's tensors of
the moment of the call."""

import dataclasses
import types

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
    s = types.SimpleNamespace(cuda_stream=torch.cuda.current_stream().cuda_stream)    # a bare handle takes the ctypes path
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


@pytest.mark.gpu
@pytest.mark.parametrize("M,K", [(37, 256), (33, 4096)])     # (33, 4096): the call splits K through a workspace
def test_activation_calls_on_an_explicit_stream(M, K, monkeypatch):
    """With a torch stream an activation call is marshalled natively as without one, and runs on that stream; with a
    bare handle it asks for no workspace."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(M)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    layer = Q.make_layer(rand(64, K), rand(K).abs() + 0.5, rand(K, 32).bfloat16(), rand(32, 64).bfloat16())
    new = rand(M, K).bfloat16()
    side = torch.cuda.Stream()
    big = rand(4096, 4096)
    bare = types.SimpleNamespace(cuda_stream=side.cuda_stream)

    def unwanted(*a):
        raise AssertionError("the ctypes path")

    for fn in (Q.quantize_act, Q.quantize_act_deflated):
        want = fn(layer, new)
        x = torch.zeros_like(new)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(8):
                big @ big                             # x arrives late on the side stream
            x.copy_(new)
        with monkeypatch.context() as m:
            m.setattr(Q, "_stream_ptr", unwanted)
            got = fn(layer, x, stream=side)
        side.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(want, got))
        with monkeypatch.context() as m:
            m.setattr(Q.lib(), "qwam_quantize_act_workspace", unwanted)
            got = fn(layer, x, stream=bare)
        side.synchronize()
        assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])


@pytest.mark.gpu
def test_split_calls_on_an_explicit_stream_in_a_graph():
    """A split call with an explicit stream while that stream is captured: its workspace is the graph's."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    layer = Q.make_layer(rand(64, 4096), rand(4096).abs() + 0.5, rand(4096, 32).bfloat16(), rand(32, 64).bfloat16())
    x = rand(33, 4096).bfloat16()
    Q.quantize_act_deflated(layer, x)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        outs = [Q.quantize_act(layer, x, stream=side), Q.quantize_act_deflated(layer, x, stream=side)]
    for i in range(4):
        x.copy_(rand(33, 4096).bfloat16())
        want = [Q.quantize_act(layer, x), Q.quantize_act_deflated(layer, x)]
        junk = [torch.full((1 << 20,), float("nan"), device="cuda") for _ in range(4)]
        graph.replay()
        torch.cuda.synchronize()
        del junk
        assert all(torch.equal(a, b) for w, o in zip(want, outs) for a, b in zip(w, o)), f"replay {i}"
