"""The attention's split plans and the workspace of an attention in parts, on the host.

The functions are the library's own C++ ones (no part of the C ABI), by their
exported names.
"""
import ctypes
import random
import time

import pytest

import paper_2601_13631_amd as ckv


class Dims(ctypes.Structure):
    _fields_ = [("n_prefix", ctypes.c_int64)] + [(x, ctypes.c_int32) for x in (
        "n_suffix", "n_q_heads", "n_kv_heads", "head_dim", "chunk_size", "dtype")] + [
        ("sm_scale", ctypes.c_float)]


class Plan(ctypes.Structure):
    _fields_ = [("rows", ctypes.c_int32), ("n_splits", ctypes.c_int32), ("off_o", ctypes.c_size_t),
                ("off_ml", ctypes.c_size_t), ("bytes", ctypes.c_size_t)]


LIB = ctypes.CDLL(ckv.LIB_PATH)
PARTED = getattr(LIB, "_ZN3ckv18attn_parted_splitsEPK8ckv_dimsli")
PARTED.restype, PARTED.argtypes = ctypes.c_int64, [ctypes.POINTER(Dims), ctypes.c_int64, ctypes.c_int]
PLAN = getattr(LIB, "_ZN3ckv14make_attn_planEPK8ckv_dimslb")
PLAN.restype, PLAN.argtypes = Plan, [ctypes.POINTER(Dims), ctypes.c_int64, ctypes.c_bool]
SHARE = getattr(LIB, "_ZN3ckv20attn_late_part_beginElii")
SHARE.restype, SHARE.argtypes = ctypes.c_int64, [ctypes.c_int64, ctypes.c_int, ctypes.c_int]


def dims(k, s, hq, hkv, d, c):
    return Dims(max(1, k * c), s, hq, hkv, d, c, ckv.DTYPE_BF16, 0.0)


def test_parted_workspace_holds_every_division():
    rng = random.Random(1)
    for _ in range(60):
        hkv, c, k = rng.choice((1, 2, 4, 8)), rng.choice((4, 8, 16, 32, 96)), rng.randint(0, 120)
        d = dims(k, int(2 ** rng.uniform(0, 11)), hkv * rng.choice((1, 2, 5, 7)), hkv,
                 rng.choice((64, 128)), c)
        held = PARTED(d, k, 4)
        for first in range(k + 1):
            late = k - first
            parts = min(4, late)
            at = [SHARE(late, parts, i) for i in range(parts + 1)] if parts else []
            n = PLAN(d, first, True).n_splits
            n += sum(PLAN(d, b - a, False).n_splits for a, b in zip(at, at[1:]))
            assert n <= held, (d.n_suffix, d.n_q_heads, hkv, c, k, first)


@pytest.mark.parametrize("k,s,hq,hkv,d,c,most_ms", [(8192, 16, 14, 2, 64, 4, 4), (32768, 1, 1, 1, 64, 4, 30)])
def test_parted_workspace_is_quickly_sized(k, s, hq, hkv, d, c, most_ms):
    """A context of a host-resident prefix is created per request shape: 0.7 and 3.5 ms
    here, 8 and 116 with a search for the best plan at every division."""
    x = dims(k, s, hq, hkv, d, c)
    best = 1e9
    for _ in range(5):
        t = time.perf_counter()
        PARTED(x, k, 4)
        best = min(best, 1e3 * (time.perf_counter() - t))
    assert best < most_ms, best
