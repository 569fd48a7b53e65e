"""Scoring over many segments per row: the fold's batches and padded rows.

Segment counts at the edges of the fold's register form (32) and of its batches
(64), up to 512; row counts that leave waves of a 256-row block without rows; and
segments redone exactly in row blocks that span several fold workgroups.  The
reference is the definition in fp64 on the GPU.
"""
import math

import pytest
import torch

from gpu_common import DEV, SCORE_RTOL_BOUND, SCORE_RTOL_UNIT, rel_err, workspace

pytestmark = pytest.mark.gpu


def scores_f64(q, k, c):
    n, Hkv, d = k.shape
    S, Hq, _ = q.shape
    G = Hq // Hkv
    tok = torch.zeros(n, dtype=torch.float64, device=DEV)
    for g in range(Hkv):
        rows = q[:, g * G:(g + 1) * G].reshape(-1, d).double()
        kk = k[:, g].double().t().contiguous()
        for r in rows.split(64):
            tok += torch.softmax((r @ kk) / math.sqrt(d), -1).sum(0)
    m = -(-n // c)
    return torch.nn.functional.pad(tok, (0, m * c - n)).view(m, c).sum(1)


def check(n, S, Hq, Hkv, d, c, dtype, q, k, rtol):
    import paper_2601_13631_amd as ckv
    print(f"case n={n} S={S} heads={Hq}/{Hkv} d={d} c={c} {dtype}", flush=True)
    dims = ckv.make_dims(n, S, Hq, Hkv, d, c, dtype)
    A = torch.full((-(-n // c),), float("nan"), dtype=torch.float64, device=DEV)
    ws = workspace(ckv.score_workspace_bytes(dims))
    ws.fill_(0xFF)  # stale scratch reads as NaN
    ckv.score_chunks(dims, q, k, A, ws)
    torch.cuda.synchronize()
    err = rel_err(A.cpu().numpy(), scores_f64(q, k, c).cpu().numpy())
    print(f"  max rel err {err:.3e}", flush=True)
    assert err <= rtol


def inputs(n, S, Hq, Hkv, d, seed, dtype=torch.bfloat16):
    gen = torch.Generator(DEV).manual_seed(seed)
    q = torch.randn((S, Hq, d), generator=gen, device=DEV).to(dtype)
    k = torch.randn((n, Hkv, d), generator=gen, device=DEV).to(dtype)
    return q, k


@pytest.mark.parametrize("n,S,Hq,Hkv,d,c", [
    (8192, 1, 1, 1, 64, 16),      # 32 segments: the last in registers
    (8448, 1, 1, 1, 64, 16),      # 33 if the workspace allows
    (16384, 3, 7, 1, 128, 32),    # 64: one batch
    (16700, 19, 7, 1, 128, 32),   # 65: two batches; 133 rows (three waves of four)
    (30011, 9, 28, 4, 128, 32),   # 63 rows (one wave)
    (131072, 2, 2, 1, 64, 8),     # 512 segments
    (12345, 50, 14, 2, 64, 4),    # 350 rows: a block of two waves behind a full one
    (20000, 64, 4, 1, 128, 16),   # 256 rows, no padding: 8-stage segments
])
def test_many_segments(n, S, Hq, Hkv, d, c):
    import paper_2601_13631_amd as ckv
    check(n, S, Hq, Hkv, d, c, ckv.DTYPE_BF16, *inputs(n, S, Hq, Hkv, d, n), SCORE_RTOL_UNIT)


@pytest.mark.parametrize("n,S,Hq,Hkv,d,c", [
    (5, 1, 4, 1, 64, 4),          # one unit
    (65, 3, 8, 2, 128, 8),        # two segments, the last of one key
    (1000, 24, 14, 2, 64, 16),    # 16 segments of one stage, a short last chunk
    (2048, 64, 28, 4, 128, 32),   # 32 segments, 256 workgroups: the most of each
    (2049, 64, 28, 4, 128, 32),   # 33 units: segments of two stages, the last of one key
    (4096, 128, 2, 1, 128, 64),   # 256 rows: no padding rows
    (4101, 8, 14, 2, 64, 8),      # 65 units: segments of three stages
    (1500, 2, 4, 2, 64, 128),     # units of two stages
    (700, 9, 4, 2, 64, 96),       # units of three stages
    (1024, 128, 40, 8, 128, 16),  # 96 workgroups of four stages become 192 of two
    (1100, 200, 40, 8, 128, 16),  # 128 become 192 of three: two-stage ones exceed one per CU
])
def test_short_segments(n, S, Hq, Hkv, d, c):
    """Launches with few workgroups, whose segments are one to three units."""
    import paper_2601_13631_amd as ckv
    check(n, S, Hq, Hkv, d, c, ckv.DTYPE_BF16, *inputs(n, S, Hq, Hkv, d, n), SCORE_RTOL_UNIT)


@pytest.mark.parametrize("n,S", [(1024, 32), (5000, 20)])
def test_fp32_segments(n, S):
    import paper_2601_13631_amd as ckv
    check(n, S, 4, 1, 64, 16, ckv.DTYPE_F32, *inputs(n, S, 4, 1, 64, n, torch.float32), SCORE_RTOL_UNIT)


@pytest.mark.parametrize("n,S,Hq,Hkv,d,c", [
    (1000, 24, 14, 2, 64, 16),    # segments of one stage
    (9000, 60, 10, 2, 64, 16),    # 300 rows: blocks of four fold workgroups and of one
    (30011, 19, 7, 1, 128, 32),   # more segments than registers
])
def test_redone_segments(n, S, Hq, Hkv, d, c):
    """Keys far above their segment's first 32 (logits of 127), for the later half
    of the queries and one KV head only, in two segments."""
    import paper_2601_13631_amd as ckv
    q, k = inputs(n, S, Hq, Hkv, d, 11)
    q[:, :, 0] = 0
    q[S // 2:, :, 0] = 8
    k[:, :, 0] = 0
    for pos in (n // 3, n - 5):
        k[pos, -1, 0] = 127 * math.sqrt(d) / 8
    check(n, S, Hq, Hkv, d, c, ckv.DTYPE_BF16, q, k, SCORE_RTOL_BOUND)
