"""The scoring sums that the pipelined a- and z-update leave for the rows they write, against fp64: their error is that of a balanced
tree of fp32 additions over each strip of 64 tokens (the strips are added in fp64)."""
import pytest
import torch

from paper_2510_03246_amd import inputs, strp

pytestmark = pytest.mark.gpu

F, D, T = 16384, 256, 1536


def _tree(x, y):
    """Strips of 64: a product and its fused neighbour 32 columns on, then five levels of pairs; fp32 [rows x strips]."""
    x, y = (t.reshape(t.shape[0], -1, 64) for t in (x, y))
    p = x[..., :32] * y[..., :32]
    s = (x[..., 32:].double() * y[..., 32:].double() + p.double()).float()
    while s.shape[-1] > 1:
        h = s.shape[-1] // 2
        s = s[..., :h] + s[..., h:]
    return s[..., 0]


@pytest.mark.parametrize("mode", [strp.WANDA, strp.GAIN])
def test_error_of_the_sums_of_a_strip(mode):
    """The root mean square error over 3 x 16384 rows is known to half a percent; a chain of eight additions within the strip is
    2.5 % (sum Z0 Z) and 4.4 % (sum A^2) above the tree, so 1.5 % tells them apart.  The sums are fp64 [4][f] behind the first
    256 bytes of the module's cache."""
    ctx = strp.Context(0)
    cfg = inputs.WorkloadConfig("case", 1, D, F, 0, T, "bf16", "t3", 3, 0.5, 1)
    err = {}
    for seed in range(3):
        m = inputs.make_ffn_module(cfg, 0, seed, "cuda", ld=T)
        mod = strp.FFNModule(ctx, m["W1hat"], m["W2hat"], m["X"], T, k_max=F)
        mod.init(strp.Params(1.0, 0.7, 0.01, mode, 1, F, 0))
        g = torch.Generator(device="cuda").manual_seed(seed)
        mod.Z += 0.5 * torch.randn(mod.Z.shape, generator=g, device="cuda")
        mod.step(strp.Params(1.0, 0.7, 0.01, mode, 1, F, strp.STAGE_SELECT))
        mod.W1.copy_(m["W1hat"].float() * (1.0 + 0.1 * torch.randn((F, D), generator=g, device="cuda")))
        mod.W2.copy_(m["W2hat"].float() * 0.1)
        ctx.profile_enable(True)
        mod.step(strp.Params(1.0, 0.7, 0.01, mode, 0, F, strp.STAGE_AUPD | strp.STAGE_ZUPD))
        assert {r[0] for r in ctx.profile_launches()} >= {"rowsum_reduce"}
        sums = mod.cache[256:256 + 32 * F].view(torch.float64).reshape(4, F)
        pairs = [(mod.A, mod.A)] + ([] if mode == strp.WANDA else [(mod.A, torch.relu(mod.Z0)), (mod.Z0, mod.Z)])
        for q, (x, y) in enumerate(pairs):
            exact = (x.double() * y.double()).sum(1)
            for who, got in (("kernel", sums[q]), ("tree", _tree(x, y).double().sum(1))):
                err[q, who] = err.get((q, who), 0.0) + float(((got - exact) ** 2).sum())
        del mod
    ratio = {q: (err[q, "kernel"] / err[q, "tree"]) ** 0.5 for q, who in err if who == "tree"}
    print(ratio)
    assert all(0.5 < r <= 1.015 for r in ratio.values()), ratio
    ctx.close()
