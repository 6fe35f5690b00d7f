"""Edges of the select's three forms (keys in registers, scores re-read by one block, several launches) against the oracle."""
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
