"""Tile shapes, folded triangles and K splits of the token-contraction product, through strp_gram: every entry, exactly."""
import pytest
import torch

from paper_2510_03246_amd import strp
from test_host_side import GRAMS

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = strp.Context(0)
    c.set_workspace(1 << 30)
    yield c
    c.close()


@pytest.mark.parametrize("s,T", GRAMS)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_gram_is_exact_on_small_integers(ctx, s, T, dtype):
    """Entries of at most 4: products and their sums stay below 2^24, so no step of the product rounds, in any order."""
    g = torch.Generator().manual_seed(s + T)
    ld = (T + 7) // 8 * 8
    A = torch.randint(-4, 5, (s, ld), generator=g).to(dtype).cuda()
    diag = torch.empty(s, dtype=torch.float64, device="cuda")
    G = ctx.strp_gram(A, T, diag=diag)
    assert ctx.poll() == strp.OK
    ref = A[:, :T].double() @ A[:, :T].double().T
    assert torch.equal(G.double(), ref)
    assert torch.equal(diag, ref.diagonal())


def test_gram_in_a_small_workspace():
    """Operand planes and the partials of the longest chains fit, the plan's own count of partials does not.  fp32 sums of
    8192 terms of like size and 22-bit operands: 1e-5."""
    ctx = strp.Context(0)
    s, T = 256, 65536
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.randn((s, T), generator=g, device="cuda")
    ctx.set_workspace(2 * 2 * s * T + 4 * s * s * (T // 8192) + (1 << 20))
    G = ctx.strp_gram(A, T)
    assert ctx.poll() == strp.OK
    ref = A.double() @ A.double().T
    assert float((G.double() - ref).norm() / ref.norm()) <= 1e-5
