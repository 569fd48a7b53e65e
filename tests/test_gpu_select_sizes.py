"""Selection at the edges of its variants' sizes, bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import DEV, gpu_select

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [8191, 8193, 9217, 16383, 16385, 17409, 32767, 32768, 32769, 100001])
def test_select_variant_edges(m):
    rng = np.random.default_rng(m)
    special = np.array([np.nan, -0.0, 0.0, -np.inf, np.inf])
    scores = np.exp(0.05 * rng.standard_normal(m))
    scores[rng.choice(m, m // 20, replace=False)] *= 1.6  # pooled scores: shared high bits
    mixed = rng.normal(0, 1, m) * np.exp(rng.normal(0, 30, m))
    mixed[rng.choice(m, 50, replace=False)] = np.tile(special, 10)
    for A in (scores, mixed, rng.integers(0, 3, m).astype(np.float64), np.full(m, -1.5)):
        for k in (1, m // 10, m // 2, m - 1, m):
            sel = gpu_select(torch.from_numpy(A).to(DEV), k).cpu().numpy()
            assert np.array_equal(sel, oracle.select_topk(A, k)), (m, k)
