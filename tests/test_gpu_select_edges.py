"""Edges of the select's three forms (keys in registers, scores re-read by one block, several launches), of the weight
statistics' one-launch lists and of the column norms' vector loads, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import strp_oracle as orc
from paper_2510_03246_amd import strp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return strp.Context(0)


@pytest.mark.parametrize("kind", ["spread", "outlier", "ties"])
@pytest.mark.parametrize("n,k,group", [(4095, 1, 1), (4096, 2048, 1), (4097, 4096, 2), (16384, 16000, 1), (65536, 30000, 1), (65535, 65534, 2),
                                       (65537, 9, 2), (131072, 131071, 1), (300001, 150000, 1)])
def test_topk_edges(ctx, n, k, group, kind):
    """spread: many exponents; outlier: all but a few scores within a millionth of each other (one histogram bin holds
    them, more than a block ranks at once); ties: three values.  Whole numbers: exact."""
    rng = np.random.default_rng(n + k)
    if kind == "spread":
        score = (rng.normal(size=n) * np.exp(rng.normal(size=n) * 4)).astype(np.float32)
    elif kind == "outlier":
        score = (1.0 + 1e-6 * rng.random(n)).astype(np.float32)
        score[rng.integers(0, n, size=3)] = [-1e30, 1e-38, 1e30]
    else:
        score = rng.integers(0, 3, size=n).astype(np.float32)
    mask, idx, tau = ctx.strp_mask_topk(torch.from_numpy(score).cuda(), k, group)
    mo, io, to = orc.select_topk(score, k, group)
    assert np.array_equal(mask.cpu().numpy(), mo)
    assert np.array_equal(idx.cpu().numpy().astype(np.int64), io)
    assert float(tau.item()) == np.float32(to)


@pytest.mark.parametrize("at", [0, 1])
@pytest.mark.parametrize("n", [96 * 4096, 96 * 4096 + 1, 192 * 8192 + 1, 3 * 256 * 4096 + 8, 8 * 256 * 4096 + 3])
def test_topk_at_the_edges_of_its_plan(ctx, n, at):
    """One, two, three and more trips a workgroup, a last workgroup of one score, scores at an address that is no multiple of 16: many
    equal ones, so that the lower indices decide.  Whole numbers: exact, against a stable sort."""
    g = torch.Generator(device="cuda").manual_seed(n)
    score = torch.randint(-500, 500, (n + at,), generator=g, device="cuda").float()[at:]
    k = n * 3 // 10
    mask, idx, tau = ctx.strp_mask_topk(score, k)
    order = torch.sort(score, descending=True, stable=True)
    want = torch.sort(order.indices[:k]).values
    assert torch.equal(idx.long(), want)
    assert int(mask.sum()) == k and bool(mask[want].all())
    assert float(tau.item()) == float(order.values[k - 1])


def test_threshold_of_everything(ctx):
    """k = n: the lowest score that is a number, NaN where none is; k = 0: +inf."""
    s = torch.full((1500,), float("nan"), device="cuda")
    assert torch.isnan(ctx.strp_mask_topk(s, 1500)[2]).item()
    assert float(ctx.strp_mask_topk(s, 0)[2].item()) == float("inf")
    s[1400] = 3.0
    s[7] = float("inf")
    assert float(ctx.strp_mask_topk(s, 1500)[2].item()) == 3.0


@pytest.mark.parametrize("n,k,group", [(65537, 9, 2), (65600, 65599, 3), (140003, 70001, 2)])
@pytest.mark.parametrize("kind", ["spread", "ties"])
def test_topk_groups_without_workspace(n, k, group, kind):
    """A caller of groups needs no workspace at any length; one of single units does.  Whole numbers: exact."""
    rng = np.random.default_rng(n)
    score = rng.normal(size=n) * np.exp(rng.normal(size=n) * 4) if kind == "spread" else rng.integers(-1, 2, size=n)
    score = score.astype(np.float32)
    bare = strp.Context(0)
    s = torch.from_numpy(score).cuda()
    mask = torch.empty(n, dtype=torch.uint8, device="cuda")
    idx = torch.empty(k * group, dtype=torch.int32, device="cuda")
    tau = torch.empty(1, device="cuda")
    bare.check(bare.lib.strp_mask_topk(bare.h, s.data_ptr(), n, k, group, mask.data_ptr(), idx.data_ptr(), tau.data_ptr()))
    mo, io, to = orc.select_topk(score, k, group)
    assert np.array_equal(mask.cpu().numpy(), mo)
    assert np.array_equal(idx.cpu().numpy().astype(np.int64), io)
    assert float(tau.item()) == np.float32(to)
    assert bare.lib.strp_mask_topk(bare.h, s.data_ptr(), n, k, 1, mask.data_ptr(), idx.data_ptr(), tau.data_ptr()) == strp.ENOMEM


@pytest.mark.parametrize("shapes", [[(1, 1)], [(7, 13)], [(64, 768)] * 4, [(33, 40)] * 8, [(5, 8)] * 9, [(3000, 264), (2, 3), (128, 8)] * 6, [(1100, 1027)],
                                    [(3, 5)] * 7 + [(700, 1501)], [(2048, 1024), (64, 65)]])
def test_weight_energy_lists(ctx, shapes):
    """Lists below, at and above what one launch takes; aligned, unaligned and one-entry matrices of both types, alone
    and beside others of another size.  fp64
    sums of at most 5e6 terms: 1e-12."""
    g = torch.Generator(device="cuda").manual_seed(len(shapes))
    mats = []
    for i, (r, c) in enumerate(shapes):
        full = torch.randn((r, c + 8 * (i % 2) + i % 3), generator=g, device="cuda") + 0.1
        m = full.to(torch.bfloat16) if i % 2 else full
        mats.append(m[:, :c])
    energy = torch.full((1,), 2.0, dtype=torch.float64, device="cuda")
    ctx.strp_weight_energy(mats, 0.3, 0.7, 1.5, energy)
    ctx.strp_weight_energy(mats[:1], 0.3, 0.7, 1.5, energy)
    assert ctx.poll() == strp.OK

    def ref(ms):
        w = np.concatenate([m.double().cpu().numpy().ravel() for m in ms])
        return 1.5 * (np.abs(w).sum() + 0.3 * w.var() + 0.7 * np.sqrt((w * w).sum()))
    want = 2.0 + ref(mats) + ref(mats[:1])
    assert abs(float(energy.item()) - want) <= 1e-12 * want


def test_weight_energy_in_a_used_workspace(ctx):
    """The workspace is scratch: what lies in it beyond the status word does not matter to a call."""
    g = torch.Generator(device="cuda").manual_seed(1)
    mats = [torch.randn((40, 64), generator=g, device="cuda") for _ in range(9)]
    got = []
    for fill in (0, 1, 255):
        energy = torch.zeros(1, dtype=torch.float64, device="cuda")
        ctx.ensure_workspace(1 << 16)
        ctx.ws[4:].fill_(fill)
        ctx.strp_weight_energy(mats, 0.3, 0.7, 1.5, energy)
        assert ctx.poll() == strp.OK
        got.append(float(energy.item()))
    w = torch.cat([m.double().reshape(-1) for m in mats])
    want = 1.5 * float(w.abs().sum() + 0.3 * w.var(correction=0) + 0.7 * w.norm())
    assert got == [got[0]] * 3 and abs(got[0] - want) <= 1e-12 * want


@pytest.mark.parametrize("rows,cols,pad,dtype", [(1, 8, 0, torch.bfloat16), (129, 64, 0, torch.bfloat16), (300, 200, 8, torch.float32),
                                                 (130, 72, 3, torch.bfloat16), (77, 136, 0, torch.float32)])
def test_scores_with_column_norms(ctx, rows, cols, pad, dtype):
    """n2 * sum A^2 with the column norms formed by the call; one product of fp64 sums rounded to fp32."""
    g = torch.Generator(device="cuda").manual_seed(rows)
    W = torch.randn((rows, cols + pad), generator=g, device="cuda").to(dtype)[:, :cols]
    A = torch.randn((cols, 40), generator=g, device="cuda")
    ctx.ensure_workspace(1 << 20)
    score = torch.empty(cols, device="cuda")
    e = torch.zeros(1, dtype=torch.float64, device="cuda")
    ctx.strp_score_alloc(A, 37, strp.WANDA, score, e, 0, 1, What=W)
    ref = (W.double() ** 2).sum(0) * (A[:, :37].double() ** 2).sum(1)
    assert torch.allclose(score.double(), ref, rtol=1e-6, atol=0)
    assert abs(float(e.item()) - float(ref.mean().item())) <= 1e-12 * float(ref.mean().item())
