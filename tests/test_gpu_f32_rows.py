"""The fp32 kernels at the edges of their splits, against fp64 on the GPU.

Attention: key counts around one and two steps of 128 keys, hidden indices, a short
last chunk, every unit of a step.  Scoring: row counts around a wave's 32 and a
workgroup's 64, every chunk mode, one subtile and ragged ends, and one wave of two
whose keys leave the guard.
"""
import math

import pytest
import torch

from gpu_common import (ATTN_ATOL_F32, DEV, SCORE_RTOL_BOUND, SCORE_RTOL_UNIT, workspace)
from test_gpu_attn_stages import attention_f64
from test_gpu_score_segments import check as check_scores
from test_gpu_score_segments import inputs

pytestmark = pytest.mark.gpu
D = 64


@pytest.mark.parametrize("n,S,Hq,Hkv,c,kept,hidden", [
    (60, 1, 1, 1, 4, 1, ()),
    (500, 2, 2, 1, 4, 31, ()),            # 124 + 1 and + 2 keys
    (500, 5, 4, 2, 4, 31, (3,)),          # 125 .. 129
    (1000, 3, 3, 3, 32, 8, ()),           # 257 .. 259
    (999, 40, 4, 1, 16, 63, (0, 62)),     # every chunk, the short one and the first hidden
    (3001, 9, 4, 2, 96, 32, ()),          # many steps, a short last chunk
])
def test_attention(n, S, Hq, Hkv, c, kept, hidden):
    import paper_2601_13631_amd as ckv
    print(f"case n={n} S={S} heads={Hq}/{Hkv} c={c} kept={kept}", flush=True)
    gen = torch.Generator(DEV).manual_seed(n)
    rnd = lambda *s: torch.randn(s, generator=gen, device=DEV)
    m = -(-n // c)
    sel = torch.linspace(0, m - 1, kept, device=DEV).round().to(torch.int32)
    for i in hidden:
        sel[i] = -1
    rows = sel.long()[:, None] * c + torch.arange(c, device=DEV)[None, :]
    valid = ((rows < n) & (sel[:, None] >= 0)).reshape(-1)
    q, k, v = rnd(S, Hq, D), rnd(kept * c, Hkv, D), rnd(kept * c, Hkv, D)
    ks, vs = rnd(S, Hkv, D), rnd(S, Hkv, D)
    bad = ~valid[:, None, None]
    k, v = k.masked_fill(bad, float("nan")), v.masked_fill(bad, float("inf"))  # hidden rows
    dims = ckv.make_dims(n, S, Hq, Hkv, D, c, ckv.DTYPE_F32)
    out = torch.full_like(q, float("nan"))
    ckv.sparse_prefill_attn(dims, q, k, v, sel, kept, ks, vs, out,
                            workspace(ckv.attn_workspace_bytes(dims, kept)))
    torch.cuda.synchronize()
    ref = attention_f64(q, k.masked_fill(bad, 0), v.masked_fill(bad, 0), ks, vs, valid)
    err = float((out.double() - ref).abs().max())
    print(f"  max abs err {err:.2e}", flush=True)
    assert err <= ATTN_ATOL_F32


@pytest.mark.parametrize("rows", [1, 31, 32, 33, 64, 65, 128])
@pytest.mark.parametrize("n,c", [(20, 4), (65, 8), (300, 16), (1030, 32), (777, 96)])
def test_scores(rows, n, c):
    import paper_2601_13631_amd as ckv
    check_scores(n, rows, 1, 1, D, c, ckv.DTYPE_F32, *inputs(n, rows, 1, 1, D, rows, torch.float32),
                 SCORE_RTOL_UNIT)


@pytest.mark.parametrize("c", [4, 16, 64])
def test_one_wave_redone(c):
    """A key far above its segment's first for rows 32 .. 63 only."""
    import paper_2601_13631_amd as ckv
    q, k = inputs(256, 64, 1, 1, D, c, torch.float32)
    q[:, :, 0] = 0
    q[32:, :, 0] = 8
    k[:, :, 0] = 0
    k[100, 0, 0] = 127 * math.sqrt(D) / 8
    check_scores(256, 64, 1, 1, D, c, ckv.DTYPE_F32, q, k, SCORE_RTOL_BOUND)
