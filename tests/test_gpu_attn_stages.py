"""The attention kernel's stages, unit tables and reference, against fp64.

Shapes put many 64-key stages into one workgroup's slice (many heads, so few
key splits), odd and even numbers of them, with every unit size (chunks of 4,
8, 16 and 32 or more tokens), a short last chunk, stages across the
prefix/suffix boundary, and indices that name no chunk.  Two more cases make a
slice's first reference useless: a logit far above the first keys', and a slice
whose first keys are all hidden.  The reference is the definition in fp64 on
the GPU; each element is held to the bound of gpu_common.attn_check.
"""
import math

import pytest
import torch

from gpu_common import ATTN_ATOL_BF16, BF16_U, DEV, workspace

pytestmark = pytest.mark.gpu


def attention_f64(q, k, v, ks, vs, valid):
    """Over compact prefix rows k, v (those of `valid`) and the causal suffix."""
    S, Hq, d = q.shape
    Hkv = k.shape[1]
    G = Hq // Hkv
    out = torch.empty((S, Hq, d), dtype=torch.float64, device=DEV)
    hidden = torch.cat((~valid[None, :].expand(S, -1),
                        torch.arange(S, device=DEV)[None, :] > torch.arange(S, device=DEV)[:, None]), 1)
    for h in range(Hkv):
        kk = torch.cat((k[:, h], ks[:, h])).double().t().contiguous()
        vv = torch.cat((v[:, h], vs[:, h])).double()
        for i in range(h * G, (h + 1) * G):
            x = (q[:, i].double() / math.sqrt(d)) @ kk
            x = x.masked_fill(hidden, -math.inf)
            out[:, i] = torch.softmax(x, -1) @ vv
    return out


def check(n, S, Hq, Hkv, d, c, sel, q, k, v, ks, vs):
    """k, v: the compact rows [len(sel) * c][Hkv][d] of the chunks `sel`."""
    import paper_2601_13631_amd as ckv
    m = -(-n // c)
    rows = (sel.long()[:, None] * c + torch.arange(c, device=DEV)[None, :])
    valid = ((rows < n) & (sel[:, None] >= 0) & (sel[:, None] < m)).reshape(-1)
    dims = ckv.make_dims(n, S, Hq, Hkv, d, c)
    out = torch.full_like(q, float("nan"))
    ws = workspace(ckv.attn_workspace_bytes(dims, sel.numel()))
    ckv.sparse_prefill_attn(dims, q, k, v, sel, sel.numel(), ks, vs, out, ws)
    torch.cuda.synchronize()
    k, v = k.masked_fill(~valid[:, None, None], 0), v.masked_fill(~valid[:, None, None], 0)
    ref = attention_f64(q, k, v, ks, vs, valid)
    a = attention_f64(q, k, v.abs(), ks, vs.abs(), valid)
    bound = torch.clamp(BF16_U * ref.abs() + (2 * BF16_U + 2.0 ** -11) * a + 1e-6,
                        max=max(ATTN_ATOL_BF16, 2 * BF16_U * float(a.max())))
    ratio = float(((out.double() - ref).abs() / bound).max())
    print(f"  {ratio:.2f} of its bound", flush=True)
    assert ratio <= 1.0


def inputs(S, Hq, Hkv, d, n_rows, seed):
    g = torch.Generator(DEV).manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV).to(torch.bfloat16)

    return (normal(S, Hq, d), normal(n_rows, Hkv, d), normal(n_rows, Hkv, d), normal(S, Hkv, d),
            normal(S, Hkv, d))


@pytest.mark.parametrize("n,S,Hq,Hkv,d,c,how", [
    (1300, 130, 256, 256, 64, 4, "all"),      # 23 stages in one slice, the last of them short
    (1303, 130, 256, 256, 64, 8, "third"),
    (1290, 140, 256, 256, 128, 16, "all"),
    (2500, 131, 256, 256, 128, 32, "all"),
    (2500, 140, 256, 256, 64, 96, "all"),     # chunks of three units, one of them short
    (1400, 200, 512, 256, 128, 64, "bad"),    # indices that name no chunk
    (6900, 130, 256, 256, 64, 4, "all"),      # more units than one table holds
    (64, 1, 1, 1, 128, 32, "all"), (31, 1, 2, 1, 64, 4, "all"), (1, 65, 7, 1, 128, 16, "all"),
])
def test_attention_stages(n, S, Hq, Hkv, d, c, how):
    print(f"case n={n} S={S} heads={Hq}:{Hkv} d={d} c={c} {how}", flush=True)
    m = -(-n // c)
    sel = torch.arange(m, device=DEV, dtype=torch.int32)
    if how == "third":
        sel = sel[::3].contiguous()
    elif how == "bad":
        sel[1], sel[m // 2], sel[-2] = -1, m, 2 ** 31 - 1
    q, k, v, ks, vs = inputs(S, Hq, Hkv, d, sel.numel() * c, n + S)
    check(n, S, Hq, Hkv, d, c, sel, q, k, v, ks, vs)


@pytest.mark.parametrize("d", [64, 128])
def test_attention_late_peak(d):
    """Logits 80 and more (log2 units) above those of a slice's first keys."""
    n, S, Hq, Hkv, c = 1024, 40, 4, 2, 32
    sel = torch.arange(n // c, device=DEV, dtype=torch.int32)
    q, k, v, ks, vs = inputs(S, Hq, Hkv, d, n, 3)
    u = torch.ones(d, device=DEV, dtype=torch.bfloat16)
    q += 4 * u
    for row in (200, 201, 700, 1023):  # in the middle and at the end of slices
        k[row] += (8 if d == 128 else 12) * u
    check(n, S, Hq, Hkv, d, c, sel, q, k, v, ks, vs)


@pytest.mark.parametrize("level", [0.0, -20.0])
def test_attention_hidden_first_keys(level):
    """A slice that begins in the padding of a short last chunk: its first 64
    keys are hidden, and at level -20 every logit is about -180 (log2 units)."""
    n, S, Hq, Hkv, d, c = 323, 192, 2, 1, 64, 320
    sel = torch.tensor([1], device=DEV, dtype=torch.int32)  # 3 tokens and 317 rows of padding
    q, k, v, ks, vs = inputs(S, Hq, Hkv, d, c, 4)
    u = torch.ones(d, device=DEV, dtype=torch.bfloat16)
    q += u
    k += level * u
    ks += level * u
    k[3:], v[3:] = float("nan"), float("nan")  # padding is never used
    check(n, S, Hq, Hkv, d, c, sel, q, k, v, ks, vs)
