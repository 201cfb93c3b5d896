"""The activation calls with K split over workgroups (few token blocks, through
the workspace of qwam_quantize_act_ws).

On the host: the workspace query and its checks.  On the GPU: the split call
against the same call without a workspace, over plain, deflated, rotated and
rotated + deflated, every rank, both group sizes and ragged splits: codes and
scales bit for bit; t bit for bit when deflated (float64 sums, one rounding),
otherwise within the float32 summation bound of parity_helpers.check_t of the
oracle's exact sum.  The outputs of the last split, the first and the padding
rows of the last token block are covered by M = 1, 17 and 47."""

import ctypes

import numpy as np
import pytest
import torch

from oracle import qwam_oracle as O
from paper_2609_33269_amd import inputs as I
from paper_2609_33269_amd import qwam as Q

from parity_helpers import bf16_dev, bits, check_t, gpu_layer, log, oracle_factors

FAKE = 0x10000          # 16-byte aligned, never dereferenced


@pytest.fixture(scope="module")
def lib():
    from paper_2609_33269_amd import build
    import os
    if not os.path.exists(Q.LIB_PATH):
        build.build()
    return Q.lib()


def _c(K, r=32, group=64, hadamard=0):
    c = Q.QwamLayerC()
    c.K, c.N, c.r, c.group, c.hadamard = K, 64, r, group, hadamard
    for f in ("wq", "ws", "wsp", "inv_smooth", "L1t", "L2t", "L1", "L1f"):
        setattr(c, f, FAKE)
    return c


def test_workspace_query_and_checks(lib):
    def need(M, defl=0, **kw):
        return lib.qwam_quantize_act_workspace(ctypes.byref(_c(**kw)), M, defl)
    assert need(4096, K=14336) == 0                       # a workgroup per CU already
    assert need(33, K=1024) == 0                          # too short to pay for a second launch
    assert need(33, K=14336) > 0 and need(33, K=14336) % (48 * 32 * 4) == 0
    assert need(33, 1, K=14336) == 2 * need(33, 0, K=14336)
    assert need(33, 1, K=1024, r=16, hadamard=1024) == 0  # one workgroup per token
    assert need(0, K=14336) == -1 and need(33, K=14336, r=24) == -1 and need(33, K=100) == -1
    n = need(33, K=14336)
    call = lambda ws, nbytes: lib.qwam_quantize_act_ws(ctypes.byref(_c(14336)), 33, 0, FAKE, FAKE, FAKE, FAKE, ws, nbytes, None)
    assert call(FAKE, n - 1) == 1 and b"workspace" in lib.qwam_last_error()
    assert call(FAKE + 8, n) == 3


def test_workspace_query_reads_only_its_fields(lib):
    """K, r, group and hadamard of the layer, as the header says: the others may be unset."""
    for kw in (dict(K=14336), dict(K=14336, r=48, group=32, hadamard=1024)):
        c = Q.QwamLayerC()
        c.K, c.r, c.group, c.hadamard = kw["K"], kw.get("r", 32), kw.get("group", 64), kw.get("hadamard", 0)
        for defl in (0, 1):
            assert lib.qwam_quantize_act_workspace(ctypes.byref(c), 33, defl) == \
                lib.qwam_quantize_act_workspace(ctypes.byref(_c(**kw)), 33, defl) > 0


def test_two_splits_need_a_longer_k(lib):
    """Plain, r <= 32, above 1360 tokens (two splits): K = 3136 takes 9.5 us unsplit and 10.5 split, K = 4096 11.2 and 10.8."""
    def need(M, K, r=32, defl=0):
        return lib.qwam_quantize_act_workspace(ctypes.byref(_c(K, r)), M, defl)
    for M in (1361, 2029, 2048):
        for r in (16, 32):
            assert need(M, 3136, r) == 0 and need(M, 3840, r) == 0
            assert need(M, 3904, r) > 0 and need(M, 3136, r, 1) > 0
        assert need(M, 3136, 48) > 0 and need(M, 3136, 64) > 0
    assert need(1360, 3136) > 0


CASES = [
    # M, K, r, group, rotated
    (1, 3072, 16, 64, False),
    (17, 4160, 32, 32, False),        # 65 groups: the last split has one
    (47, 5184, 48, 64, False),        # 81 groups
    (33, 3136, 64, 32, False),        # 49 groups
    (47, 1536, 32, 64, False),        # deflated only: the shortest K that splits
    (17, 2048, 32, 64, True),         # two tiles of 1024
    (47, 3840, 48, 32, True),         # tiles of 768
    (1, 3520, 16, 64, True),          # block 64, tiles of 704
    (2033, 2176, 64, 64, True),       # 128 token blocks, tiles of 128 in two splits
    (65, 768, 32, 64, True),          # deflated: three tiles of 256 (one of 768 does not fit in LDS)
    (33, 3840, 64, 32, True),         # the same, 15 tiles
]


@pytest.mark.gpu
@pytest.mark.parametrize("deflate", [False, True])
@pytest.mark.parametrize("M,K,r,group,rotated", CASES)
def test_split_equals_unsplit(M, K, r, group, rotated, deflate):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = I.custom(M, K, 64, r, seed=M + K, n_outliers=5)
    f = dict(oracle_factors(d, hadamard=rotated), group=group)
    layer = gpu_layer(f)
    x = bf16_dev(d.x)
    c = layer.c_struct()
    need = Q.lib().qwam_quantize_act_workspace(ctypes.byref(c), M, int(deflate))
    log(f"  split M={M} K={K} r={r} group={group} rotated={rotated} deflate={deflate}: workspace {need}")
    assert need > 0 or (not deflate and (K == 768 or (not rotated and K < 3072)))

    def call(ws):
        out = (torch.empty((M, K // 2), dtype=torch.uint8, device="cuda:0"),
               torch.empty((K // group, M), dtype=torch.float32, device="cuda:0"),
               torch.empty((M, r), dtype=torch.bfloat16, device="cuda:0"))
        st = Q.lib().qwam_quantize_act_ws(ctypes.byref(c), M, int(deflate), x.data_ptr(), *(o.data_ptr() for o in out),
                                          None if ws is None else ws.data_ptr(), 0 if ws is None else ws.numel(),
                                          torch.cuda.current_stream().cuda_stream)
        assert st == 0, Q.lib().qwam_last_error()
        torch.cuda.synchronize()
        return out

    whole = call(None)
    split = call(torch.full((max(need, 16),), 0xFF, dtype=torch.uint8, device="cuda:0"))   # NaNs the call must not read
    again = call(torch.zeros((max(need, 16),), dtype=torch.uint8, device="cuda:0"))
    assert torch.equal(whole[0], split[0]) and torch.equal(whole[1], split[1]), "codes and scales"
    assert (bits(split[2]) == bits(again[2])).all(), "a fixed summation order"
    if deflate:
        assert (bits(whole[2]) == bits(split[2])).all(), "t"
    else:
        xt = O.transformed_activations(d.x, O.inverse_smoothing(f["lam"]), int(f.get("hadamard", 0)))
        check_t(bits(split[2]), O.down_projection(xt, f["L1"]), xt, f["L1"])


@pytest.mark.gpu
@pytest.mark.parametrize("rotated", [False, True])
def test_split_calls_in_a_graph(rotated):
    """Split calls (plain and deflated) and their GEMM captured with the binding's
    workspace from the graph's pool: every replay equals the eager call, with
    eager work that takes and drops memory between the replays, also on new
    inputs."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = I.custom(35, 3072, 64, 32, seed=5, n_outliers=5)
    layer = gpu_layer(oracle_factors(d, hadamard=rotated))
    x = bf16_dev(d.x)

    def step():
        return [Q.forward(layer, x, deflate=f) for f in (False, True)]

    step()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ys = step()
    for i in range(4):
        x.copy_(bf16_dev(np.roll(d.x, i, axis=0)))
        eager = step()
        junk = [torch.full((1 << 20,), float("nan"), device="cuda:0") for _ in range(4)]
        for y in ys:
            y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        del junk
        for a, b in zip(eager, ys):
            assert (bits(a) == bits(b)).all(), f"replay {i}"
