"""The two refits of a small module in shared launches against the same refits called one at a time."""
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
