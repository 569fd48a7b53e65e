"""Attention slices whose reference is far below their maximum, against fp64.

The numerators of a slice are taken against the largest logit of its first 32
keys.  Here one later key in every 64 stands 10 to 116 (log2 units) above those,
inside the range that is not taken again unless the outputs leave fp32, or 130,
outside, in one slice and in several that are merged; V of ordinary size and of 1.25 x 2^65, where at level 60 every slice's
outputs stay inside fp32 and a merge by weights as large as the numerators would
not.
"""
import math

import pytest
import torch

from test_gpu_attn_stages import DEV, check, inputs

pytestmark = pytest.mark.gpu


def peaked(n, S, Hq, Hkv, d, level, v_scale):
    """Small noise, and keys 40, 104, ... with logits of about `level` log2 units."""
    q, k, v, ks, vs = inputs(S, Hq, Hkv, d, n, int(level) + n)
    q, k, ks = 0.25 * q, 0.25 * k, 0.25 * ks
    q[:, :, 0], k[:, :, 0], ks[:, :, 0] = 8, 0, 0
    k[40::64, :, 0] = level * math.sqrt(d) / (8 * math.log2(math.e))
    # a column's values have one sign, so nothing cancels in a merge; that a row's
    # outputs have both keeps the sum over them, which guards a slice, small
    sign = torch.where(torch.arange(d, device=DEV) // 8 % 2 == 0, 1, -1)
    v, vs = (((1 + 0.1 * x.float().abs().clamp(max=1)) * sign * v_scale).to(x.dtype) for x in (v, vs))
    return q, k, v, ks, vs


@pytest.mark.parametrize("level", [10, 40, 60, 90, 116, 130])
@pytest.mark.parametrize("v_scale", [1.0, 1.25 * 2.0 ** 65])
@pytest.mark.parametrize("n,d", [(256, 64), (256, 128), (1024, 64), (1024, 128)])
def test_late_levels(n, d, v_scale, level):
    import paper_2601_13631_amd as ckv
    print(f"case n={n} d={d} V x {v_scale} level {level}", flush=True)
    S, Hq, Hkv, c = 40, 4, 2, 32
    k = n // c
    merged = ckv.attn_workspace_bytes(ckv.make_dims(n, S, Hq, Hkv, d, c), k) > 0
    assert merged == (n > 512)
    sel = torch.arange(k, device=DEV, dtype=torch.int32)
    check(n, S, Hq, Hkv, d, c, sel, *peaked(n, S, Hq, Hkv, d, level, v_scale))


@pytest.mark.parametrize("n,d", [(256, 64), (256, 128), (1024, 64), (1024, 128)])
def test_outputs_overflow(n, d):
    """Numerators of 2^60 times finite V of 2^70, positive and negative from peak to
    peak: a slice's sum stays inside its range while its outputs become infinite and,
    where both signs meet, NaN."""
    print(f"case n={n} d={d}", flush=True)
    S, Hq, Hkv, c = 40, 4, 2, 32
    q, k, v, ks, vs = peaked(n, S, Hq, Hkv, d, 60, 2.0 ** 70)
    v[104::128] *= -1
    check(n, S, Hq, Hkv, d, c, torch.arange(n // c, device=DEV, dtype=torch.int32), q, k, v, ks, vs)


def which_rows_differ(level):
    """Two slices of 5 stages, of which the second begins at suffix token 192, inside the
    block of rows 128..255: which rows' outputs change when row 255 has a logit of
    `level` (log2 units; the others' are a few) for key 250.  A slice that is done again
    shows in its other rows' rounding (another reference)."""
    import paper_2601_13631_amd as ckv
    n, S, d, c = 128, 512, 64, 32
    dims = ckv.make_dims(n, S, 1, 1, d, c)
    ws_bytes = ckv.attn_workspace_bytes(dims, n // c)
    assert ws_bytes == 2 * S * (d * 2 + 8)
    sel = torch.arange(n // c, device=DEV, dtype=torch.int32)
    q, k, v, ks, vs = inputs(S, 1, 1, d, n, 5)
    q[:, :, 0], k[:, :, 0], ks[:, :, 0] = 0, 0, 0
    ks[250, :, 0] = 8
    high = q.clone()
    high[255, :, 0] = level * math.sqrt(d) / (8 * math.log2(math.e))
    outs = []
    for x in (q, high):
        check(n, S, 1, 1, d, c, sel, x, k, v, ks, vs)
        outs.append(torch.empty_like(x))
        ckv.sparse_prefill_attn(dims, x, k, v, sel, n // c, ks, vs, outs[-1],
                                torch.empty(ws_bytes, dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    differ = (outs[0] != outs[1]).any(dim=-1).flatten()
    assert not differ[:192].any() and differ[255] and not differ[256:].any()
    return differ[192:255]


def test_rows_without_keys_are_not_redone():
    """The block's first rows see none of the second slice, which is no reason to do it
    again: a row that makes it so changes the others."""
    assert which_rows_differ(180).any()


def test_logits_up_to_the_guard_are_not_redone():
    """A logit far above the slice's first 32 keys, whose numerator fp32 still holds."""
    assert not which_rows_differ(100).any()
