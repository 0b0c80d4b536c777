"""Sizes of the backward pass's workspace, which callers keep over calls of several sizes.  Host-only."""
import ctypes
import random

import pytest

import paper_2604_10103_amd as hf

LIMIT = 2 << 30   # most that is asked for stored scores


@pytest.mark.parametrize("seed", range(40))
def test_a_workspace_for_the_largest_call_serves_every_smaller_one(seed):
    """More queries or keys never ask for less, also where a call's scores pass the limit."""
    r = random.Random(seed)
    size = lambda lo, hi: int(lo * (hi / lo) ** r.random())
    dtype, d = r.choice([("f32", 128), ("f32", 64), ("bf16", 64), ("bf16", 128)])
    bq, bkv = (r.choice([1, 5, 16, 32, 48, 64, 128]) for _ in range(2))
    cfg = hf.make_config(1, size(1, 40), d, dtype, bq, bkv, r.choice([0.125, 0.25, 0.5, 1.0]), flags=r.choice([0, hf.HF_FLAG_BWD_FP32_KERNELS]))
    for which in (0, 1):
        n, other = size(1, 2000), size(1, 20000)
        last = 0
        while n < 100_000:
            args = (cfg, n, other) if which else (cfg, other, n)
            full, least = hf.hf_bwd_workspace_bytes(*args), hf.hf_bwd_least_workspace_bytes(*args)
            t_m, t_n = -(-args[1] // bq), -(-args[2] // bkv)
            assert full >= last, (args, full, last)
            assert least <= full <= least + LIMIT + cfg.heads * t_m * t_n * 4 + 256
            last, n = full, n + max(1, n // 5)


def test_a_refusal_names_the_least_size():
    cfg = hf.make_config(1, 2, 64, "f32", 64, 64, 0.25)
    least = hf.hf_bwd_least_workspace_bytes(cfg, 100, 200)
    lib, c = hf.load(), ctypes.byref(cfg)
    Q, K, V, dO, dQ, dK, dV, ws = (4096 * i for i in range(1, 9))   # (nothing is launched on an error)
    call = lambda n: lib.hf_hybrid_attn_bwd(c, Q, None, 100, K, V, 200, None, 0, None, None, None, dO, dQ, None, dK, dV, ws, n, None)
    assert call(least - 1) == -5 and str(least) in lib.hf_last_error().decode()


def test_null_and_sizes_out_of_range():
    lib, out = hf.load(), ctypes.c_size_t(0)
    c = ctypes.byref(hf.make_config(1, 2, 64, "f32", 64, 64, 0.25))
    assert lib.hf_bwd_least_workspace_bytes(c, 100, 200, None) == -1
    assert lib.hf_bwd_least_workspace_bytes(c, 0, 200, ctypes.byref(out)) == -2
    assert lib.hf_bwd_least_workspace_bytes(c, 100, (1 << 24) + 1, ctypes.byref(out)) == -2
