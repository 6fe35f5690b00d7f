"""The two refits of a small module in shared launches against the same refits called one at a time, and the two products of
the fc2 refit in one launch against a launch each."""
import ctypes as C

import pytest
import torch

from paper_2510_03246_amd import inputs, strp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f,T,k", [(8, 40, 83, 9), (64, 256, 512, 128), (72, 200, 131, 65), (128, 264, 1003, 131), (136, 520, 1003, 129)])
@pytest.mark.parametrize("prec", [strp.PREC_SPLIT, strp.PREC_FAST])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_refits_together_and_apart(d, f, T, k, prec, dtype):
    """Same products, summed in the same order: the same bits.  The workspace the library asks for holds both at a time."""
    ld = (T + 7) // 8 * 8
    cfg = inputs.WorkloadConfig("case", 1, d, f, 0, T, dtype, "t3", 3, 0.5, 1)
    m = inputs.make_ffn_module(cfg, 0, 5, "cuda", ld=ld)
    got = []
    for calls in ([strp.STAGE_REFIT2 | strp.STAGE_REFIT1 | strp.STAGE_AUPD], [strp.STAGE_REFIT2, strp.STAGE_REFIT1]):
        ctx = strp.Context(0)
        ctx.set_precision(prec)
        mod = strp.FFNModule(ctx, m["W1hat"], m["W2hat"], m["X"], T, k_max=k)
        mod.init(strp.Params(1.0, 0.7, 0.01, strp.WANDA, 1, k, 0))
        mod.Z += 0.25 * torch.randn(mod.Z.shape, generator=torch.Generator(device="cuda").manual_seed(k), device="cuda")
        mod.A.copy_(torch.relu(mod.Z))
        mod.state.sums_cached = 0
        mod.step(strp.Params(1.0, 0.7, 0.01, strp.WANDA, 1, k, strp.STAGE_SELECT))
        ctx.profile_enable(True)
        for stages in calls:
            mod.step(strp.Params(1.0, 0.7, 0.01, strp.WANDA, 0, k, stages))
        assert sum(r[0] == "chol_solve_f64" for r in ctx.profile_launches()) == len(calls)
        got.append((mod.W1.clone(), mod.W2.clone()))
        ctx.close()
    assert all(bool(w.any()) and torch.equal(w, v) for w, v in zip(*got))


@pytest.mark.parametrize("d,f,T,k", [(64, 256, 512, 128), (40, 160, 600, 159), (72, 264, 1003, 257), (128, 264, 1003, 131)])
@pytest.mark.parametrize("prec,planes", [(strp.PREC_SPLIT, None), (strp.PREC_SPLIT, (1, 2)), (strp.PREC_SPLIT, (2, 1)), (strp.PREC_FAST, None)])
def test_products_of_the_fc2_refit_together_and_apart(d, f, T, k, prec, planes):
    """The refit of fc2 alone shares a launch between the Gram matrix and the right-hand side where the workspace holds the partials of
    both.  The largest one that does not holds those of either in full, so both ways split the tokens alike: the same bits.
    planes: fp16 planes of the right-hand side's operands."""
    ld = (T + 7) // 8 * 8
    cfg = inputs.WorkloadConfig("case", 1, d, f, 0, T, "f32", "t3", 3, 0.5, 1)
    m = inputs.make_ffn_module(cfg, 0, 7, "cuda", ld=ld)
    ctx = strp.Context(0)
    ctx.set_precision(prec)
    if planes:
        ctx.set_product_planes(strp.PROD_RHS2, *planes)
    mod = strp.FFNModule(ctx, m["W1hat"], m["W2hat"], m["X"], T, k_max=k)
    mod.init(strp.Params(1.0, 0.7, 0.01, strp.WANDA, 1, k, 0))
    mod.A += 0.25 * torch.rand(mod.A.shape, generator=torch.Generator(device="cuda").manual_seed(k), device="cuda")
    mod.state.sums_cached = 0
    mod.step(strp.Params(1.0, 0.7, 0.01, strp.WANDA, 1, k, strp.STAGE_SELECT))
    space = torch.empty(1 << 24, dtype=torch.uint8, device="cuda")

    def refit(nbytes):
        """weights and products' launches, or None where the workspace is too small"""
        ctx.check(ctx.lib.strp_set_workspace(ctx.h, space.data_ptr(), nbytes))
        ctx.profile_enable(True)
        par = strp.Params(1.0, 0.7, 0.01, strp.WANDA, 0, k, strp.STAGE_REFIT2)
        status = ctx.lib.strp_admm_step(ctx.h, C.byref(mod.desc), C.byref(mod.state), C.byref(par), None)
        products = [r[0] for r in ctx.profile_launches() if r[0].startswith("gemm_")]
        assert ctx.poll() == strp.OK and status in (strp.OK, strp.ENOMEM)
        return (mod.W2.clone(), products) if status == strp.OK else None

    together, products = refit(space.numel())
    assert products == ["gemm_group"] and bool(together.any())
    lo, hi = 0, space.numel() // 256                 # the workspace in units of 256 bytes: too small for the shared launch, enough
    while hi - lo > 1:
        mid = (lo + hi) // 2
        got = refit(max(mid, 16) * 256)
        lo, hi = (lo, mid) if got is not None and got[1] == ["gemm_group"] else (mid, hi)
    apart, products = refit(lo * 256)
    assert len(products) == 2 and "gemm_group" not in products, products
    assert torch.equal(together, apart)
    ctx.close()


@pytest.mark.parametrize("d,f,T,k", [(72, 264, 1003, 131), (256, 1536, 2000, 1032), (64, 1600, 700, 1465)])
def test_rows_of_the_fc2_system_change_no_bit(d, f, T, k):
    """The system's rows are whole cache lines where the workspace holds them (host side: check_rows_of_the_fc2_system), tiles that share
    lines are read past the caches where it does not.  The smallest workspace that holds every product's partials in full, which the
    shorter rows just fit: the same bits as on the one the library asks for."""
    ld = (T + 7) // 8 * 8
    cfg = inputs.WorkloadConfig("case", 1, d, f, 0, T, "f32", "t3", 3, 0.5, 1)
    m = inputs.make_ffn_module(cfg, 0, 7, "cuda", ld=ld)
    ctx = strp.Context(0)
    mod = strp.FFNModule(ctx, m["W1hat"], m["W2hat"], m["X"], T, k_max=k)
    mod.init(strp.Params(1.0, 0.7, 0.01, strp.WANDA, 1, k, 0))
    mod.step(strp.Params(1.0, 0.7, 0.01, strp.WANDA, 1, k, strp.STAGE_SELECT))
    space = torch.empty(ctx.workspace_bytes(mod.desc), dtype=torch.uint8, device="cuda")

    def refit(nbytes):
        """weights and the bytes that the reductions read and write, or None where the workspace is too small"""
        ctx.check(ctx.lib.strp_set_workspace(ctx.h, space.data_ptr(), nbytes))
        ctx.profile_enable(True)
        par = strp.Params(1.0, 0.7, 0.01, strp.WANDA, 0, k, strp.STAGE_REFIT2)
        status = ctx.lib.strp_admm_step(ctx.h, C.byref(mod.desc), C.byref(mod.state), C.byref(par), None)
        reduced = sum(r[3] for r in ctx.profile_launches() if r[0] == "splitk_reduce")
        assert ctx.poll() == strp.OK and status in (strp.OK, strp.ENOMEM)
        return (mod.W2.clone(), reduced) if status == strp.OK else None

    want, reduced = refit(space.numel())
    lo, hi = 15, space.numel() // 256                 # the workspace in units of 256 bytes: partials cut short or none, all in full
    while hi - lo > 1:
        mid = (lo + hi) // 2
        got = refit(mid * 256)
        lo, hi = (lo, mid) if got is not None and abs(got[1] - reduced) < 1.0 else (mid, hi)
    got, _ = refit(hi * 256)
    assert bool(got.any()) and torch.equal(got, want)
    ctx.close()
