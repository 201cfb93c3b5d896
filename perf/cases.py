"""The performance cases of the ASP W4A4 layer: what a program that serves a quantized world action model has this
library do, from one action-expert call to a full denoising-step layer, and the calibration that precedes it.

Kinds of cases (field "kind"):
  layer    one few-token layer in one call (qwam.asp_layer), launched from Python
  stack    `layers` few-token layers recorded in one HIP graph, as a sampler replays its action-expert pass: the fused
           call, or (with "forward") the two calls of the rotated / deflated / group-32 setting
  forward  one whole layer, both kernels (qwam.forward), launched from Python
  aog      one batch of probe vectors added to the action-observability Gramian (qwam.aog_accumulate)
  basis    the protected subspace from an accumulated Gramian (qwam.aog_protected_basis)
  pack     the offline weight pack of one layer (qwam.pack_weights)

Inputs are synthetic with the distributions of the layer's own workloads: bf16 activations N(0, 1) with 1% (action
expert: 2%) of the channels 10-50 times larger, weights N(0, 1/K), an orthonormal protected basis of rank r.
"""
import math

import torch

from paper_2609_33269_amd import qwam

DEV = "cuda"


def listed():
    return [
        # one action-expert projection for one action chunk of 16 tokens: the smallest call, host path and launch included
        {"name": "expert_call_m16", "kind": "layer", "M": 16, "K": 1024, "N": 1024, "r": 16},
        # the action-expert's wide and square projections for 64 action tokens, replayed as one HIP graph per sampler step
        {"name": "expert_stack_m64", "kind": "stack", "M": 64, "K": 1024, "N": 4096, "N2": 1024, "r": 16, "layers": 12,
         "group": 64, "hadamard": False, "deflate": False, "forward": False},
        # the same pass in the deployed setting (group 32, rotation, deflation), an odd number of action tokens
        {"name": "expert_stack_paper_m50", "kind": "stack", "M": 50, "K": 1024, "N": 4096, "N2": 1024, "r": 16,
         "layers": 12, "group": 32, "hadamard": True, "deflate": True, "forward": True},
        # a handful of text or state tokens through the video transformer's down-projection
        _forward("tokens_down_m33", 33, 14336, 3072),
        # a few hundred tokens (one conditioning frame) through the video transformer's QKV, rotated, with a bias
        _forward("chunk_qkv_m333", 333, 3072, 9216, hadamard=True, bias=True),
        # the same kind of chunk through its down-projection
        _forward("chunk_down_m415", 415, 14336, 3072),
        # the FFN up-projection of the headline benchmark
        _forward("ffn_up_m4096", 4096, 3072, 14336),
        # the FFN down-projection of a denoising step (8192 video tokens), the largest call
        _forward("ffn_down_m8192", 8192, 14336, 3072),
        # the QKV projection in the deployed setting: group 32, rotated, deflated
        _forward("qkv_paper_m4096", 4096, 3072, 9216, group=32, hadamard=True, deflate=True),
        # calibration: one batch of 4096 probe vectors into the Gramian of a 4096-wide layer input
        {"name": "aog_d4096", "kind": "aog", "d": 4096, "n": 4096},
        # calibration: the rank-32 protected basis of that Gramian in the smoothed, rotated coordinates
        {"name": "basis_d4096", "kind": "basis", "d": 4096, "r": 32, "iters": 10, "hadamard": True},
        # export: the FFN up-projection's weight quantized and packed
        {"name": "pack_up", "kind": "pack", "K": 3072, "N": 14336, "group": 64},
    ]


def _forward(name, M, K, N, r=32, group=64, hadamard=False, deflate=False, bias=False):
    return {"name": name, "kind": "forward", "M": M, "K": K, "N": N, "r": r, "group": group, "hadamard": hadamard,
            "deflate": deflate, "bias": bias}


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _log_step(rng, lo, hi, step):
    return max(lo, min(hi, step * round(_log(rng, lo, hi) / step)))


def draw(rng):
    """One more case of the ranges above: any layer size up to the denoising step's, every option of the layer."""
    kind = rng.choices(["layer", "stack", "forward", "aog", "basis", "pack"], [3, 3, 10, 1, 1, 1])[0]
    if kind in ("layer", "stack"):
        c = {"kind": kind, "M": rng.randint(1, 64), "K": _log_step(rng, 256, 4096, 64), "N": _log_step(rng, 256, 8192, 16),
             "r": rng.choice([16, 16, 32])}
        if kind == "stack":
            c.update(N2=_log_step(rng, 256, 4096, 16), layers=rng.randint(4, 16), group=64, hadamard=False,
                     deflate=False, forward=False)
            if rng.random() < 0.5:
                c.update(group=rng.choice([32, 64]), hadamard=True, deflate=rng.random() < 0.7, forward=True)
                c["K"] = _served_width(c)
        return c
    if kind == "aog":
        return {"kind": kind, "d": _log_step(rng, 512, 4096, 16), "n": _log_step(rng, 256, 4096, 64)}
    if kind == "basis":
        return {"kind": kind, "d": _log_step(rng, 512, 4096, 64), "r": rng.choice([16, 32, 48]), "iters": rng.randint(6, 20),
                "hadamard": rng.random() < 0.7}
    if kind == "pack":
        return {"kind": kind, "K": _log_step(rng, 256, 14336, 64), "N": _log_step(rng, 256, 9216, 16),
                "group": rng.choice([32, 64])}
    while True:
        M, K, N = round(_log(rng, 1, 8192)), _log_step(rng, 256, 14336, 64), _log_step(rng, 256, 14336, 16)
        if M * K * N <= 8192 * 14336 * 3072:
            break
    c = _forward("", M, K, N, r=rng.choice([16, 32, 32, 32, 48, 64]), group=rng.choice([32, 64]),
                 hadamard=rng.random() < 0.5, deflate=rng.random() < 0.5, bias=rng.random() < 0.5)
    del c["name"]
    c["K"] = _served_width(c)
    return c


def _served_width(c):
    """Rotated and deflated layers of rank 32 and 64 take widths in steps of 512, as the models' are (a few of the
    widths between need more LDS than a workgroup has)."""
    return max(512, c["K"] // 512 * 512) if c["hadamard"] and c["deflate"] and c["r"] in (32, 64) else c["K"]


# ---- inputs, from the seed alone ----

def _gen(seed, salt=0):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000003 + salt)


def _cpu_gen(seed, salt=0):
    return torch.Generator().manual_seed(int(seed) * 1000003 + salt)


def _orthonormal(rows, cols, seed, salt):
    q, _ = torch.linalg.qr(torch.randn(rows, cols, generator=_cpu_gen(seed, salt), dtype=torch.float64))
    return q.to(DEV)


def _block(K):
    """The rotation's block: the largest power of two dividing K, at most 1024."""
    return min(K & -K, 1024)


def _rotate(v, B, scale):
    """Rows of v times the blockwise Hadamard matrix, butterfly stages on channel bit 0, 1, .., then one multiply."""
    rows, K = v.shape
    y, h = v, 1
    while h < B:
        z = y.reshape(rows, K // (2 * h), 2, h)
        a, b = z[:, :, 0], z[:, :, 1]
        y = torch.stack((a + b, a - b), dim=2).reshape(rows, K)
        h *= 2
    return y * scale


def _layer_inputs(M, K, N, r, seed, salt=0, hadamard=False, bias=False, outliers=0.01):
    """x bf16 [M][K], lambda f32 [K], and the factors R f32 [N][K], L1 bf16 [K][r], L2 bf16 [r][N] of the split weight."""
    g = _gen(seed, salt)
    x = torch.randn(M, K, generator=g, device=DEV)
    gain = torch.ones(K, device=DEV)
    idx = torch.randperm(K, generator=g, device=DEV)[:max(1, int(outliers * K))]
    gain[idx] = 10 * torch.exp(math.log(5.0) * torch.rand(len(idx), generator=g, device=DEV))
    x = (x * gain).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g, device=DEV) / math.sqrt(K)).to(torch.bfloat16)
    xmax, wmax = gain.double() * 3, w.abs().amax(dim=0).double()
    lam = (xmax.sqrt() / wmax.sqrt()).float()
    wt = w.double() * lam.double()
    B = _block(K) if hadamard else 0
    if B:
        wt = _rotate(wt, B, B ** -0.5)
    L1 = _orthonormal(K, r, seed, salt).to(torch.bfloat16)
    L2t = (wt @ L1.double()).to(torch.bfloat16)
    R = (wt - L2t.double() @ L1.double().t().contiguous()).float()
    b = torch.randn(N, generator=g, device=DEV).to(torch.bfloat16) if bias else None
    return {"x": x, "lam": lam, "R": R, "L1": L1, "L2": L2t.t().contiguous(), "bias": b, "B": B}


def _make(f, group):
    return qwam.make_layer(f["R"], f["lam"], f["L1"], f["L2"], f["bias"], hadamard=f["B"], group=group)


def _stack_shapes(c):
    return [c["N"] if i % 2 == 0 else c["N2"] for i in range(c["layers"])]


def _probes(c, seed):
    """A batch of probe vectors, channel-major: a decaying action subspace plus noise."""
    d, n = c["d"], c["n"]
    g = _gen(seed)
    s = 0.93 ** torch.arange(96, device=DEV, dtype=torch.float32)
    z = torch.randn(96, n, generator=g, device=DEV) * s[:, None]
    u = torch.randn(d, 96, generator=g, device=DEV) / math.sqrt(d)
    return (u @ z + 0.01 / math.sqrt(d) * torch.randn(d, n, generator=g, device=DEV)).to(torch.bfloat16)


def _gramian(c, seed):
    """An accumulated Gramian [d][d] (symmetric, decaying spectrum) and the smoothing factors."""
    d = c["d"]
    u = _orthonormal(d, 96, seed, 0).float()
    g = _gen(seed)
    z = torch.randn(96, 512, generator=g, device=DEV) * (0.93 ** torch.arange(96, device=DEV))[:, None]
    f = u @ z
    A = f @ f.t().contiguous() + 1e-3 * torch.eye(d, device=DEV)
    return (A + A.t()) / 2, torch.exp(0.3 * torch.randn(d, generator=g, device=DEV))


def prepare(case, seed):
    k = case["kind"]
    if k == "layer":
        f = _layer_inputs(case["M"], case["K"], case["N"], case["r"], seed, outliers=0.02)
        return {"kind": k, "x": f["x"], "layer": _make(f, 64)}
    if k == "stack":
        calls = []
        for i, N in enumerate(_stack_shapes(case)):
            f = _layer_inputs(case["M"], case["K"], N, case["r"], seed, i + 1, case["hadamard"], outliers=0.02)
            calls.append((_make(f, case["group"]), f["x"]))

        def step():
            if case["forward"]:
                return [qwam.forward(layer, x, deflate=case["deflate"]) for layer, x in calls]
            return [qwam.asp_layer(layer, x) for layer, x in calls]

        step()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ys = step()
        return {"kind": k, "graph": graph, "ys": ys, "calls": calls}
    if k == "forward":
        f = _layer_inputs(case["M"], case["K"], case["N"], case["r"], seed, 0, case["hadamard"], case["bias"])
        return {"kind": k, "x": f["x"], "layer": _make(f, case["group"]), "deflate": case["deflate"]}
    if k == "aog":
        d = case["d"]
        return {"kind": k, "gT": _probes(case, seed), "A": torch.zeros(d, d, device=DEV)}
    if k == "basis":
        A, lam = _gramian(case, seed)
        ws = torch.empty(qwam.aog_protected_basis_workspace(case["d"], case["r"]), dtype=torch.uint8, device=DEV)
        return {"kind": k, "A": A, "lam": lam, "r": case["r"], "iters": case["iters"], "ws": ws,
                "B": _block(case["d"]) if case["hadamard"] else 0}
    f = _layer_inputs(1, case["K"], case["N"], 16, seed)
    return {"kind": k, "R": f["R"], "lam": f["lam"], "group": case["group"]}


def run(s):
    k = s["kind"]
    if k == "layer":
        return qwam.asp_layer(s["layer"], s["x"])
    if k == "stack":
        s["graph"].replay()
        return s["ys"]
    if k == "forward":
        return qwam.forward(s["layer"], s["x"], deflate=s["deflate"])
    if k == "aog":
        return qwam.aog_accumulate(s["gT"], s["A"])
    if k == "basis":
        return qwam.aog_protected_basis(s["A"], s["r"], iters=s["iters"], scale=1.0 / 512, lam=s["lam"], hadamard=s["B"],
                                        workspace=s["ws"])
    return qwam.pack_weights(s["R"], s["lam"], group=s["group"])


# ---- what one pass cannot do without ----

def _layer_work(M, K, N, r, group):
    w = N * K // 2 + 4 * N * (K // group) + 2 * N * r + 2 * K * r + 4 * K     # codes, scales, factors, 1/lambda
    return {"bytes": 2 * M * K + w + 2 * M * N, "flops": 2 * M * K * N + 2 * M * K * r + 2 * M * r * N}


def work(case):
    k = case["kind"]
    if k == "layer":
        return _layer_work(case["M"], case["K"], case["N"], case["r"], 64)
    if k == "stack":
        each = [_layer_work(case["M"], case["K"], N, case["r"], case["group"]) for N in _stack_shapes(case)]
        return {f: sum(e[f] for e in each) for f in ("bytes", "flops")}
    if k == "forward":
        return _layer_work(case["M"], case["K"], case["N"], case["r"], case["group"])
    if k == "aog":
        d, n = case["d"], case["n"]
        return {"bytes": 2 * d * n + 8 * d * d, "flops": n * d * (d + 1)}
    if k == "basis":   # one reading of the Gramian; the products of the subspace iteration on a block of r + 16 vectors
        d, r = case["d"], case["r"]
        return {"bytes": 4 * d * d + 4 * d * r, "flops": 2 * d * d * (r + 16) * (case["iters"] + 1)}
    K, N, g = case["K"], case["N"], case["group"]
    return {"bytes": 4 * N * K + N * K // 2 + 8 * N * (K // g) + 8 * K, "flops": 0}


def tolerance(case):
    k = case["kind"]
    if k == "pack":
        return "exact"                        # codes and scales are defined bit for bit
    if k == "aog":
        return {"rel": 7e-7, "max": 4e-6}     # float32 sums in another order: measured 1.7e-7 and 8e-7
    if k == "basis":
        # float32 eigenvectors: rounding over the gap of the eigenvalues; measured up to 8e-6 and 2e-4 (rank 48)
        return {"rel": 4e-5, "max": 1e-3}
    # bf16 outputs: one rounding, measured 1.7e-3 and 3.9e-3, and 1.3e-2 where an entry of t, in bf16, falls the other way
    return {"rel": 7e-3, "max": 5e-2}


# ---- the same in 64 bits, in plain torch ----

def _codes(v, group):
    """The symmetric 4-bit group quantizer in its defined float32 steps: codes (as float64) and scales [.., K / group]."""
    v = v.reshape(v.shape[0], -1, group)
    amax = v.abs().amax(dim=2)
    s = torch.where(amax < 7 * 2.0 ** -126, torch.zeros_like(amax), amax / torch.full_like(amax, 7.0))
    inv = torch.where(s == 0, torch.zeros_like(s), torch.ones_like(s) / s)
    return torch.clamp(torch.round(v * inv[:, :, None]), -8, 7).double(), s.double()


def _dequant(v, group):
    q, s = _codes(v, group)
    return (q * s[:, :, None]).reshape(v.shape[0], -1)


def _exact_layer(f, group, deflate):
    inv = torch.ones_like(f["lam"]) / f["lam"]
    xt = f["x"].float() * inv
    if f["B"]:
        xt = _rotate(xt, f["B"], float(torch.tensor(f["B"] ** -0.5, dtype=torch.float32)))
    t = (xt.to(torch.bfloat16).double() @ f["L1"].double()).to(torch.bfloat16)
    xp = xt
    if deflate:   # r rank-1 steps in float32, exact products, one rounding each
        for j in range(t.shape[1]):
            xp = xp - t[:, j:j + 1].float() * f["L1"][:, j].float()[None, :]
    y = _dequant(xp, group) @ _dequant(f["R"], group).t() + t.double() @ f["L2"].double()
    return y if f["bias"] is None else y + f["bias"].double()


def exact(case, seed):
    k = case["kind"]
    if k == "layer":
        f = _layer_inputs(case["M"], case["K"], case["N"], case["r"], seed, outliers=0.02)
        return _exact_layer(f, 64, False)
    if k == "stack":
        return [_exact_layer(_layer_inputs(case["M"], case["K"], N, case["r"], seed, i + 1, case["hadamard"], outliers=0.02),
                             case["group"], case["deflate"]) for i, N in enumerate(_stack_shapes(case))]
    if k == "forward":
        f = _layer_inputs(case["M"], case["K"], case["N"], case["r"], seed, 0, case["hadamard"], case["bias"])
        return _exact_layer(f, case["group"], case["deflate"])
    if k == "aog":
        g = _probes(case, seed).double()
        return g @ g.t().contiguous()
    if k == "basis":
        A, lam = _gramian(case, seed)
        G = lam.double()[:, None] * A.double() * lam.double()[None, :] / 512
        if case["hadamard"]:
            B = _block(case["d"])
            G = _rotate(_rotate(G, B, B ** -0.5).t().contiguous(), B, B ** -0.5)
        w, V = torch.linalg.eigh(((G + G.t()) / 2).cpu())
        w, V = w.flip(0)[:case["r"]], V.flip(1)[:, :case["r"]]
        sign = torch.sign(V.gather(0, V.abs().argmax(dim=0, keepdim=True)))
        return (V * sign, w)
    f = _layer_inputs(1, case["K"], case["N"], 16, seed)
    amax = f["R"].double().reshape(case["N"], -1, case["group"]).abs().amax(dim=2)
    return (None, (amax / 7).t().contiguous(), None, 1 / f["lam"].double())
