"""The a- and z-update products and split partials of the pipelined kernel (256 x 256 tiles) at sizes that are a multiple of
nothing: edges in rows, in tokens, within the four tokens of a lane, and a token count below one strip of 64 in the last tile.
The same of the 64 x 64 blocks that small products are cut into: one, two and three of them, edges in both directions, an
odd number of contraction steps.  And of the 128 x 256 tiles that two workgroups of a CU share: an odd and an even number of pairs
of stages, one row in the last tile, fewer than 64 of its 256 tokens and more, contractions that end within a pair; and of the 64 x 256
ones, with fewer pairs than they have in flight too."""
import pytest
import torch

from paper_2510_03246_amd import inputs, strp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [strp.WANDA, strp.GAIN])
@pytest.mark.parametrize("d,f,T,k", [(264, 608, 24603, 301), (256, 520, 24577, 257), (520, 768, 17001, 512), (64, 256, 512, 128),
                                       (8, 40, 83, 9), (72, 200, 131, 65), (136, 520, 1003, 129), (200, 400, 2050, 191),
                                       (200, 696, 33003, 250), (392, 800, 21845, 385), (256, 1000, 22050, 641), (1000, 1400, 8250, 1100),
                                       (72, 264, 33003, 130), (136, 400, 20003, 193), (200, 1000, 17003, 600), (520, 1704, 5003, 1100), (40, 160, 33025, 33)])
def test_update_of_the_kept_rows(d, f, T, k, mode):
    """One iteration, then the rows it kept against the formulas in fp64 from the weights it left: A_S = relu(Z_S) + W^T M^-1 E and the z
    rule on W1 X, to a quarter of the 2e-3 that the module is held to; columns past T stay as they were.  The next iteration's
    scores come out of the sums these epilogues leave: fp32 sums over 64 tokens, added in fp64, of 24-bit values: 1e-5."""
    ctx = strp.Context(0)
    ld = (T + 7) // 8 * 8
    cfg = inputs.WorkloadConfig("case", 1, d, f, 0, T, "bf16", "t3", 3, 0.5, 1)
    m = inputs.make_ffn_module(cfg, 0, 5, "cuda", ld=ld)
    mod = strp.FFNModule(ctx, m["W1hat"], m["W2hat"], m["X"], T, k_max=k)
    p = strp.Params(1.0, 0.7, 0.01, mode, 1, k, 0)
    mod.init(p)
    mod.Z += 0.25 * torch.randn(mod.Z.shape, generator=torch.Generator(device="cuda").manual_seed(k), device="cuda")
    mod.A.copy_(torch.relu(mod.Z))
    for t in (mod.Z, mod.A):
        t[:, T:] = 7.0
    z_old = mod.Z.clone()
    assert mod.step(p).status == strp.OK
    S = mod.idx[:k].long()
    W, W1 = mod.W2[:, S].double(), mod.W1[S].double()
    zs = z_old[S, :T].double()
    M = 0.7 * torch.eye(d, dtype=torch.float64, device="cuda") + W @ W.T
    E = mod.Y[:, :T].double() - W @ torch.relu(zs)
    a = torch.relu(zs) + W.T @ torch.linalg.solve(M, E)
    z1 = W1 @ m["X"][:, :T].double()
    cm, cp = z1.clamp(max=0.0), ((0.7 * a + z1) / 1.7).clamp(min=0.0)
    z = torch.where(0.7 * a ** 2 + (cm - z1) ** 2 < 0.7 * (a - cp) ** 2 + (cp - z1) ** 2, cm, cp)
    rel = lambda x, y: float((x.double() - y).norm() / y.norm())
    assert rel(mod.A[S, :T], a) <= 5e-4 and rel(mod.Z[S, :T], z) <= 5e-4
    if ld > T:
        assert bool((mod.Z[:, T:] == 7.0).all()) and bool((mod.A[:, T:] == 7.0).all())
    A, Z, Z0 = (t[:, :T].double() for t in (mod.A, mod.Z, mod.Z0))
    n2 = mod.n2
    if mode == strp.WANDA:
        want = n2 * (A ** 2).sum(1)
    else:
        # eq. (78) with b = Z, u = Z0, D = What2 A, Y = What2 relu(Z0): 2 P - Q
        want = 2.0 * ((Z0 * Z).sum(1) + n2 * (A * torch.relu(Z0)).sum(1)) - ((Z0 ** 2).sum(1) + n2 * (A ** 2).sum(1))
    p2 = strp.Params(1.0, 0.7, 0.01, mode, 1, k, 1)      # the selection alone
    mod.step(p2)
    assert rel(mod.score, want) <= 1e-5
    ctx.close()


@pytest.mark.parametrize("d,f,T,k", [(40, 168, 333, 33), (200, 800, 9000, 400), (72, 264, 70001, 131), (264, 1000, 66000, 270), (600, 1608, 5000, 800), (968, 2400, 16384, 1500)])
def test_planes_that_epilogues_write_are_whole(d, f, T, k):
    """Where d or f is no multiple of 32 the planes of E and of relu(Z0) end in groups past the last row, which the next products read: zeros, whatever the
    workspace held (each tile of E: 64x64, 128x128, 128x256, 64x256, 256x256)."""
    ctx = strp.Context(0)
    g = torch.Generator(device="cuda").manual_seed(k)
    W1, W2, X = (0.05 * torch.randn(s, generator=g, device="cuda") for s in ((f, d), (d, f), (d, (T + 7) // 8 * 8)))
    mod = strp.FFNModule(ctx, W1, W2, 20 * X, T, k_max=k)
    par, got = strp.Params(1.0, 0.7, 0.01, strp.WANDA, 1, k, 0), []
    for byte in (0, 255):                # 255: NaN in fp16, fp32 and fp64
        ctx.set_workspace(ctx.workspace_bytes(mod.desc))
        ctx.ws[256:] = byte
        mod.init(par)
        rep = mod.step(par)
        got.append([t.clone() for t in (mod.Y[:, :T], mod.A[:, :T], mod.Z[:, :T], mod.W1, mod.W2, mod.H)] + [torch.tensor(list(rep.terms))])
    assert all(torch.equal(a, b) for a, b in zip(*got)) and bool(torch.isfinite(got[0][1]).all())
    ctx.close()
