"""Timing cases of the framework: the calls that a pruning program makes, over the sizes it makes them at.

Six kinds of work, each through the public entry points of the binding:

  step      one inner ADMM iteration of a resident FFN module (select, both refits, a- and z-update, objective), the
            unit of work that a run repeats a few hundred to a few thousand times
  module    one module from start to end: re-bound inputs, initialisation, a few iterations on the mask of the first
            selection (what a streamed model does once per decoder layer)
  model     Alg. 1 on a whole (small) model: energies, softmax allocation per temperature, per-module ADMM, best temperature
  heads     head pruning of one attention output projection: scores per head, top-k heads, Gram of the kept channels,
            refit of W_O
  score     unit scores and layer energy of one module from its resident auxiliaries
  select    the structured mask of a score vector: one module's units, or every layer's at once (one global threshold)
  weights   weight-only importances of every layer (Alg. 2) and their inverse allocation

Shapes are those of the configurations in paper_2510_03246_amd/inputs.py (64/256, 768/3072, 2048/8192, 4096/16384, their
head counts and pruned fractions), with token counts that let three states lie in device memory, and ragged sizes
between them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2510_03246_amd import driver, inputs, strp

MODES = {"wanda": strp.WANDA, "gain": strp.GAIN}
GAMMA, RHO = 0.95, 1.5          # depth discount and attention weight of the weight-only importances

_context = None


def _ctx():
    """The one library context that a program keeps for its device; its workspace grows to the largest module seen."""
    global _context
    if _context is None:
        _context = strp.Context(0)
    return _context


def listed():
    return [
        # The smallest module the tests run end to end: nothing but launches and latency.
        dict(name="step_d64", kind="step", d=64, f=256, T=512, k=128, dtype="f32", mode="wanda"),
        # OPT-125M's module at its configured tokens, half the units kept: the factorisation chains weigh as much as the products.
        dict(name="step_d768", kind="step", d=768, f=3072, T=65536, k=1536, dtype="bf16", mode="wanda"),
        # No size a multiple of a tile (widths in eights, as the module asks), fp32 inputs (two operand planes of X), the score that needs all four token sums.
        dict(name="step_ragged_gain", kind="step", d=1000, f=2312, T=30011, k=1013, dtype="f32", mode="gain"),
        # OPT-1.3B's module at its configured 128 x 2048 tokens, 60 % pruned.
        dict(name="step_d2048", kind="step", d=2048, f=8192, T=262144, k=3277, dtype="bf16", mode="wanda"),
        # OPT-6.7B's module (the headline shape), 70 % pruned, on 64 segments of 2048 tokens.
        dict(name="step_d4096", kind="step", d=4096, f=16384, T=131072, k=4915, dtype="bf16", mode="wanda"),
        # One decoder layer of OPT-125M from inputs to refitted weights on a short calibration set.
        dict(name="module_d768", kind="module", d=768, f=3072, T=16384, k=1536, dtype="bf16", mode="wanda", iters=3),
        # Alg. 1 on a two-layer model with a grid of three temperatures and ten iterations: many small calls in a row.
        dict(name="model_d64", kind="model", L=2, d=64, f=256, T=512, dtype="f32", rbar=0.5, iters=10),
        # Head pruning of OPT-1.3B's output projection, 32 heads of 64 channels, 13 kept.
        dict(name="heads_d2048", kind="heads", heads=32, dh=64, keep=13, T=65536, dtype="bf16"),
        # Scores of an OPT-125M module by the three-tensor rule.
        dict(name="score_f3072", kind="score", d=768, f=3072, T=65536, mode="gain"),
        # The units of one OPT-6.7B module.
        dict(name="select_16384", kind="select", layers=1, n=16384, keep=0.3),
        # One threshold over all 48 layers of OPT-30B.
        dict(name="select_48x28672", kind="select", layers=48, n=28672, keep=0.3),
        # The twelve layers of OPT-125M by their weights alone: 12 heads and two fc matrices per layer.
        dict(name="weights_d768", kind="weights", L=12, d=768, f=3072, heads=12, dtype="bf16", rbar=0.5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "module", "model", "heads", "score", "select", "select", "weights"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    mode = rng.choice(["wanda", "wanda", "gain"])
    if kind in ("step", "module"):
        d = _log(rng, 64, 3000 if kind == "step" else 1200) // 8 * 8
        f = int(d * rng.uniform(2.2, 4.5)) // 8 * 8
        k = max(1, int(f * rng.uniform(0.25, 0.6)))
        # no fewer tokens than channels; at most a third of the largest listed module's tokens x units and of its products
        T = _log(rng, max(512, d), max(600, 2 * d, min(150000 if kind == "step" else 30000, int(7e8 / f), int(1e13 / (d * k * 12)))))
        case = dict(kind=kind, d=d, f=f, T=T, k=k, dtype=dtype, mode=mode)
        if kind == "module":
            case["iters"] = rng.choice([2, 3, 5])
        return case
    if kind == "model":
        d = _log(rng, 48, 200) // 8 * 8
        return dict(kind="model", L=rng.randint(2, 4), d=d, f=int(d * rng.uniform(3, 4.5)) // 8 * 8, T=_log(rng, 300, 4000), dtype=dtype,
                    rbar=round(rng.uniform(0.3, 0.7), 3), iters=rng.choice([3, 5, 10]))
    if kind == "heads":
        dh = rng.choice([64, 64, 80, 128])
        heads = rng.randint(8, 2560 // dh)
        return dict(kind="heads", heads=heads, dh=dh, keep=max(1, int(heads * rng.uniform(0.3, 0.6))), T=_log(rng, 2048, 100000), dtype=dtype)
    if kind == "score":
        f = _log(rng, 500, 12000)
        return dict(kind="score", d=max(64, f // 4), f=f, T=_log(rng, 2000, min(150000, int(6e8 / f))), mode=mode)
    if kind == "select":
        layers = rng.choice([1, 1, 12, 24, 32, 48])
        n = _log(rng, 200, 40000)
        return dict(kind="select", layers=layers, n=n, keep=round(rng.uniform(0.1, 0.9), 4))
    heads = rng.randint(4, 16)
    d = 64 * heads
    return dict(kind="weights", L=rng.randint(4, 16), d=d, f=int(d * rng.uniform(3, 4)) | 1, heads=heads, dtype=dtype, rbar=round(rng.uniform(0.3, 0.7), 3))


def _config(case, T):
    n_out = max(1, (case["d"] + 99) // 100)
    return inputs.WorkloadConfig("case", 1, case["d"], case["f"], 0, T, case["dtype"], "x20" if case["dtype"] == "f32" else "t3", n_out, 0.5, 1)


def _ffn_inputs(case, seed, layer=0):
    T = case["T"]
    return inputs.make_ffn_module(_config(case, T), layer, seed, "cuda", ld=(T + 7) // 8 * 8)


def prepare(case, seed):
    ctx = _ctx()
    kind = case["kind"]
    st = dict(case=case, ctx=ctx, kind=kind)
    if kind in ("step", "module"):
        m = _ffn_inputs(case, seed)
        mod = strp.FFNModule(ctx, m["W1hat"], m["W2hat"], m["X"], case["T"], k_max=case["k"])
        # a resident module that iterates re-selects; a module run from start to end keeps its first mask, as Alg. 1 does
        st.update(m=m, mod=mod, params=strp.Params(1.0, 1.0, 0.01, MODES[case["mode"]], int(kind == "step"), case["k"], 0))
        if kind == "step":
            mod.init(st["params"])
    elif kind == "model":
        st["modules"] = [_ffn_inputs(case, seed, layer) for layer in range(case["L"])]
        for layer, m in enumerate(st["modules"]):
            m["W2hat"] *= 1.0 + 0.3 * layer          # layers of different energies
    elif kind == "heads":
        d, T = case["heads"] * case["dh"], case["T"]
        cfg = inputs.WorkloadConfig("case", 1, d, 4 * d, case["heads"], T, case["dtype"], "t3", max(1, d // 100), 0.5, 1)
        m = inputs.make_head_module(cfg, 0, seed, "cuda", ld=(T + 7) // 8 * 8)
        Y = torch.zeros((d, m["C"].shape[1]), dtype=torch.float32, device="cuda")
        for t0 in range(0, T, 32768):                # the dense target W_O C
            Y[:, t0:t0 + 32768] = m["WOhat"].float() @ m["C"][:, t0:t0 + 32768].float()
        lam = 0.01 * float((m["C"][:, :T].float() ** 2).sum().item()) / d
        ctx.ensure_workspace(ctx.workspace_bytes(strp.ModuleDesc(d, d, T, Y.stride(0), Y.stride(0), strp.dtype_code(m["C"]), strp.BF16, d)))
        st.update(m=m, Y=Y, lam=lam, score=torch.empty(case["heads"], device="cuda"),
                  energies=torch.zeros(1, dtype=torch.float64, device="cuda"), W=torch.empty((d, d), device="cuda"))
    elif kind == "score":
        f, T, ld = case["f"], case["T"], (case["T"] + 7) // 8 * 8
        Z0 = inputs.synthetic_state(f, T, seed, "cuda", ld=ld)
        Z = (Z0 + 0.1 * inputs.synthetic_state(f, T, seed + 1, "cuda", ld=ld)).contiguous()
        A = torch.relu(Z)
        cfg = inputs.WorkloadConfig("case", 1, case["d"], f, 0, T, "bf16", "t3", 1, 0.5, 1)
        ctx.ensure_workspace(1 << 20)
        st.update(Z=Z, Z0=Z0, A=A, W2=inputs._weight(case["d"], f, cfg, seed, 0, 2, "cuda"), score=torch.empty(f, device="cuda"),
                  energies=torch.zeros(1, dtype=torch.float64, device="cuda"))
    elif kind == "select":
        # column norms x Gram diagonals: chi-square-like within a layer, another scale for each layer and some outliers
        g = torch.Generator(device="cuda").manual_seed(seed)
        L, n = case["layers"], case["n"]
        s = torch.randn((L, n), generator=g, device="cuda") ** 2 + 0.1 * torch.randn((L, n), generator=g, device="cuda") ** 2
        s *= torch.exp(0.3 * torch.randn((L, 1), generator=g, device="cuda")) * 1000.0
        s[torch.rand((L, n), generator=g, device="cuda") < 0.01] *= 50.0
        st.update(score=s.reshape(-1).contiguous(), k=max(1, int(case["keep"] * L * n)))
        ctx.ensure_workspace(max(1 << 16, int(ctx.lib.strp_topk_workspace_bytes(L * n))))
    else:
        d, f, heads, L = case["d"], case["f"], case["heads"], case["L"]
        cfg = inputs.WorkloadConfig("case", L, d, f, heads, 1, case["dtype"], "t3", 1, case["rbar"], 1)
        dh, groups = d // heads, []
        for layer in range(L):
            q, k, v, o = (inputs._weight(d, d, cfg, seed, layer, 31 + i, "cuda") for i in range(4))
            q, k, v, o = (w * (1.0 + 0.05 * layer) for w in (q, k, v, o))
            w1, w2 = inputs._weight(f, d, cfg, seed, layer, 1, "cuda"), inputs._weight(d, f, cfg, seed, layer, 2, "cuda")
            attn = [[q[h * dh:(h + 1) * dh], k[h * dh:(h + 1) * dh], v[h * dh:(h + 1) * dh], o[:, h * dh:(h + 1) * dh]] for h in range(heads)]
            groups.append((attn, [[w1], [w2]]))
        st.update(groups=groups, n_units=torch.tensor([heads, f] * L, dtype=torch.int32, device="cuda"),
                  gid=torch.tensor([0, 1] * L, dtype=torch.int32, device="cuda"))
        ctx.ensure_workspace(1 << 16)
    return st


def run(st):
    case, ctx, kind = st["case"], st["ctx"], st["kind"]
    if kind == "step":
        mod = st["mod"]
        rep = mod.step(st["params"])
        return dict(W1=mod.W1, W2=mod.W2, A=mod.A[:, :case["T"]], Z=mod.Z[:, :case["T"]], mask=mod.mask, idx=mod.idx[:case["k"]], score=mod.score,
                    terms=list(rep.terms), status=rep.status)
    if kind == "module":
        mod, m = st["mod"], st["m"]
        mod.rebind_inputs(m["W1hat"], m["W2hat"], m["X"])
        mod.init(st["params"])
        for _ in range(case["iters"]):
            rep = mod.step(st["params"])
        return dict(W1=mod.W1, W2=mod.W2, mask=mod.mask, idx=mod.idx[:case["k"]], A=mod.A[:, :case["T"]], Z=mod.Z[:, :case["T"]], Y=mod.Y[:, :case["T"]], H=mod.H,
                    terms=list(rep.terms), status=rep.status)
    if kind == "model":
        res, best = driver.prune_model(ctx, st["modules"], case["T"], case["rbar"], (0.5, 1.0, 2.0), case["iters"], keep_weights=True)
        return dict(best=best, pruned=[list(p) for p in res[best].pruned],
                    by_temperature=[dict(energies=np.array(r.energies), r=np.array(r.r), nprune=np.array(r.nprune), losses=np.array(r.losses),
                                         total=r.total) for _, r in sorted(res.items())])
    if kind == "heads":
        C, WO, T = st["m"]["C"], st["m"]["WOhat"], case["T"]
        ctx.strp_score_alloc(C, T, strp.WANDA, st["score"], st["energies"], 0, 1, group=case["dh"], What=WO)
        mask, idx, tau = ctx.strp_mask_topk(st["score"], case["keep"], case["dh"])
        G = ctx.strp_gram(C, T, idx=idx)
        W = ctx.strp_refit(strp.SIDE_FC2, G, st["lam"], st["Y"], C, T, idx, st["W"])
        return dict(score=st["score"], energies=st["energies"], mask=mask, idx=idx, tau=tau, G=G, W=W)
    if kind == "score":
        full = case["mode"] != "wanda"
        ctx.strp_score_alloc(st["A"], case["T"], MODES[case["mode"]], st["score"], st["energies"], 0, 1, What=st["W2"],
                             Z=st["Z"] if full else None, Z0=st["Z0"] if full else None)
        return dict(score=st["score"], energies=st["energies"])
    if kind == "select":
        mask, idx, tau = ctx.strp_mask_topk(st["score"], st["k"])
        return dict(mask=mask, idx=idx, tau=tau)
    energies = torch.zeros(2 * case["L"], dtype=torch.float64, device="cuda")
    for layer, (attn, mlp) in enumerate(st["groups"]):
        scale = GAMMA ** (layer + 1)
        for group in attn:
            ctx.strp_weight_energy(group, 0.1, 0.01, scale * RHO, energies[2 * layer:2 * layer + 1])
        for group in mlp:
            ctx.strp_weight_energy(group, 0.05, 0.0, scale, energies[2 * layer + 1:2 * layer + 2])
    r, nprune = ctx.strp_alloc_inverse(energies, st["n_units"], case["rbar"], 1.0, 0.95, st["gid"])
    return dict(energies=energies, r=r, nprune=nprune)


def _bytes_of(dtype):
    return 2 if dtype == "bf16" else 4


def _step_work(d, f, T, k, dtype, mode):
    xb = _bytes_of(dtype)
    # Gram of the kept rows, the two right-hand sides, residual, a- and z-update, objective's Gram; two factorisations,
    # the inverse of one system, and the two solves
    flops = T * (k * (k + 1.0) + 5 * 2.0 * d * k + d * (d + 1.0)) + (k ** 3 + 2.0 * d ** 3) / 3 + 2.0 * d * k * k + 2.0 * k * d * d + 2.0 * d * d * k
    # X, Y, the kept rows of A and every row of Z in (for the four-sum score Z0 as well), A and Z out; weights out, fp64 factor in
    nbytes = T * (xb * d + 4.0 * d + 4.0 * k + 4.0 * f + 8.0 * f + (4.0 * f if mode == "gain" else 0.0)) + 8.0 * d * f + 8.0 * d * d
    return flops, nbytes


def _init_work(d, f, T, dtype):
    xb = _bytes_of(dtype)
    flops = T * (2 * 2.0 * d * f + d * (d + 1.0)) + 2.0 * d ** 3 / 3
    nbytes = T * (xb * d + 3 * 4.0 * f + 4.0 * d) + 2.0 * xb * d * f + 12.0 * d * d + 8.0 * d * f
    return flops, nbytes


def work(case):
    kind = case["kind"]
    if kind in ("step", "module"):
        fl, by = _step_work(case["d"], case["f"], case["T"], case["k"], case["dtype"], case["mode"])
        if kind == "module":
            fi, bi = _init_work(case["d"], case["f"], case["T"], case["dtype"])
            fl, by = fi + case["iters"] * fl, bi + case["iters"] * by
    elif kind == "model":
        fs, bs = _step_work(case["d"], case["f"], case["T"], int(case["f"] * (1 - case["rbar"])), case["dtype"], "wanda")
        fi, bi = _init_work(case["d"], case["f"], case["T"], case["dtype"])
        n = case["L"] * 3
        fl, by = (n + case["L"]) * fi + n * case["iters"] * fs, (n + case["L"]) * bi + n * case["iters"] * bs
    elif kind == "heads":
        d, T, s, cb = case["heads"] * case["dh"], case["T"], case["keep"] * case["dh"], _bytes_of(case["dtype"])
        fl = T * (2.0 * d + s * (s + 1.0) + 2.0 * d * s) + s ** 3 / 3 + 2.0 * d * s * s
        by = T * (cb * d + 4.0 * d) + cb * d * d + 4.0 * d * d + 4.0 * s * s
    elif kind == "score":
        n = 3 if case["mode"] != "wanda" else 1
        fl, by = (8.0 if n == 3 else 2.0) * case["f"] * case["T"], 4.0 * n * case["f"] * case["T"] + 2.0 * case["d"] * case["f"]
    elif kind == "select":
        n = case["layers"] * case["n"]
        fl, by = 0.0, 5.0 * n + 4.0 * int(case["keep"] * n)
    else:
        n = case["L"] * (4.0 * case["d"] ** 2 + 2.0 * case["d"] * case["f"])
        fl, by = 4.0 * n, _bytes_of(case["dtype"]) * n
    return {"bytes": by, "flops": fl}


def tolerance(case):
    kind = case["kind"]
    if kind == "select":
        return "exact"
    if kind == "weights":
        return {"rel": 1e-9, "max": 1e-9}              # fp64 sums
    if kind == "score":
        return {"rel": 1e-6, "max": 1e-5}              # fp64 sums rounded once to fp32
    if kind == "heads":
        return {"rel": 1e-4, "max": 5e-3}              # fp32 sums over the tokens, a ridge system of condition 1e2 .. 1e4
    # fp32 sums through two ridge systems of condition up to 1e4, and a z rule that takes the other of two equal-cost
    # minimisers (0.7 a apart) at the few elements where rounding decides: an arithmetic error e moves Z by about sqrt(e).
    # The tests hold the same quantities to 2e-3.
    return {"rel": 1e-3, "max": 0.99}
