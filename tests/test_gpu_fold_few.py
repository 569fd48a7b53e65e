"""Scoring with one to four segments per row, where the fold changes its form.

300 rows per KV head: two row blocks of which the second has one wave with rows and
three without, in the fold and, with keys far above their segment's first 32, in a
segment's exact recomputation.
"""
import math

import pytest

import paper_2601_13631_amd as ckv
from gpu_common import SCORE_RTOL_BOUND, SCORE_RTOL_UNIT
from test_gpu_score_segments import check, inputs

pytestmark = pytest.mark.gpu

CASES = [(300, 96, 64, 16), (600, 96, 64, 8), (800, 64, 64, 32), (1030, 64, 64, 4),
         (300, 96, 128, 64), (830, 64, 128, 16)]


@pytest.mark.parametrize("n,heads,d,c", CASES)
def test_few_segments(n, heads, d, c):
    check(n, 300, heads, heads, d, c, ckv.DTYPE_BF16, *inputs(n, 300, heads, heads, d, n), SCORE_RTOL_UNIT)


@pytest.mark.parametrize("n,heads,d,c", CASES)
def test_few_segments_redone(n, heads, d, c):
    q, k = inputs(n, 300, heads, heads, d, 7)
    q[:, :, 0], k[:, :, 0] = 0, 0
    q[200:, :, 0] = 8  # rows of both row blocks
    k[n - 5, -2:, 0] = 127 * math.sqrt(d) / 8
    check(n, 300, heads, heads, d, c, ckv.DTYPE_BF16, q, k, SCORE_RTOL_BOUND)
