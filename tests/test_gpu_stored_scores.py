"""Gradients in fp32 arithmetic from stored scores (a workspace of the size that ``hf_bwd_workspace_bytes`` asks for) and from
scores that every kernel forms again (a workspace that ends where the scores would begin): both against the fp64 oracle, at tile
and block edges, for lists in any order with entries that name no block, in a cache buffer, from a workspace full of NaN.

Bounds as in test_gpu_backward: rel-L2 5e-5 in fp32, 1e-2 after the rounding to bf16."""
import re

import numpy as np
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import oracle_state, rel_l2

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [  # dtype, head_dim, heads, block_q, block_kv, n_q, n_kv, k (None: dense), capacity, queries' gain
    ("f32", 128, 2, 64, 64, 150, 300, 3, 0, 1.0),
    ("f32", 128, 3, 48, 48, 100, 250, 4, 260, 1.0),     # three tiles of sixteen in a block of two workgroups
    ("f32", 128, 2, 40, 16, 81, 65, 2, 0, 8.0),
    ("f32", 128, 2, 16, 64, 33, 129, 2, 0, 1.0),        # sixteen rows, thirty-two keys a workgroup
    ("f32", 128, 2, 64, 16, 129, 47, 3, 0, 1.0),
    ("f32", 64, 2, 24, 20, 50, 81, 3, 100, 1.0),
    ("f32", 64, 1, 1, 1, 5, 9, 4, 0, 1.0),
    ("f32", 64, 2, 64, 64, 130, 200, None, 0, 1.0),
    ("f32", 64, 1, 16, 16, 5200, 65536, 2, 0, 1.0),     # masks of the inverse lists larger than LDS
    ("bf16", 64, 2, 64, 64, 190, 333, 3, 0, 1.0),
    ("bf16", 128, 2, 32, 48, 70, 200, 3, 0, 1.0),
]


@pytest.mark.parametrize("flags", [0, hf.HF_FLAG_DKV_INDEX_ORDER])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_stored_and_recomputed_scores_match_oracle(case, flags):
    dtype, d, H, bq, bkv, n_q, n_kv, k, cap, gain = case
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    t_m, t_n = -(-n_q // bq), -(-n_kv // bkv)
    rows = cap or n_kv
    cfg = hf.make_config(1, H, d, dtype, bq, bkv, 1.0 if k is None else 0.5, keep_k=k or 0, kv_capacity=cap, flags=flags)
    mk = lambda n, s, g=1.0: wl.randn((1, H, n, d), 47_000 + s, 0.7 * g, tdt)
    Q, K, V, dO = mk(n_q, 0, gain), mk(rows, 1), mk(rows, 2), mk(n_q, 3)
    Ke, Ve = mk(40, 4), mk(40, 5)
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, Ke.to(DEV), Ve.to(DEV))
    r = np.random.default_rng(len(str(case)))
    lists = idx = None
    if k is not None:
        lists = np.stack([[r.permutation(t_n)[:k] for _ in range(t_m)] for _ in range(H)])
        lists[:, ::3, 1] = -1                             # an entry that names no block
        lists[:, 1::3, k - 1] = t_n + 7
        idx = torch.tensor(lists[None], dtype=torch.int32, device=DEV)
    small = None
    try:
        hf.hf_hybrid_attn_bwd(cfg, Q.to(DEV), K.to(DEV), V.to(DEV), idx, st, dO.to(DEV), torch.empty_like(Q, device=DEV),
                              torch.empty_like(K, device=DEV), torch.empty_like(K, device=DEV),
                              torch.empty(256, dtype=torch.uint8, device=DEV), n_kv=n_kv)
    except Exception as e:                                # the size that a call cannot do without, from the refusal
        small = int(re.search(r"workspace of (\d+) bytes needed", str(e)).group(1))
    full = hf.hf_bwd_workspace_bytes(cfg, n_q, n_kv)
    assert small is not None and full > small
    states = oracle_state([Ke], [Ve], d)
    bound = 1e-2 if dtype == "bf16" else 5e-5
    for size in (full, small):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device=DEV)
        dQ = torch.full(Q.shape, float("nan"), dtype=tdt, device=DEV)
        dK, dV = (torch.full(K.shape, 7.0, dtype=tdt, device=DEV) for _ in range(2))
        hf.hf_hybrid_attn_bwd(cfg, Q.to(DEV), K.to(DEV), V.to(DEV), idx, st, dO.to(DEV), dQ, dK, dV, ws, n_kv=n_kv)
        torch.cuda.synchronize()
        assert (dK[:, :, n_kv:] == 7.0).all() and (dV[:, :, n_kv:] == 7.0).all()
        for h in range(H):
            sel = np.tile(np.arange(t_n), (t_m, 1)) if lists is None else [[j for j in row if 0 <= j < t_n] for row in lists[h]]
            sel = np.asarray(sel, dtype=object) if lists is not None else sel
            f = lambda t, n: wl.to_f64(t)[0, h, :n]
            if n_kv <= 4096:
                q, qh, kk, v = orc.hybrid_attention_bwd(f(Q, n_q), f(K, n_kv), f(V, n_kv), states[h], bq, bkv, sel, f(dO, n_q))
            else:                                         # (the oracle's scatter over a long window, a block at a time)
                q, kk, v = (np.zeros((n, d)) for n in (n_q, n_kv, n_kv))
                for i in range(t_m):
                    s = slice(i * bq, min(n_q, (i + 1) * bq))
                    keys = np.concatenate([np.arange(j * bkv, (j + 1) * bkv) for j in sel[i]])
                    one = np.arange(len(sel[i]))[None]
                    a, b, c = orc.sparse_attention_bwd(f(Q, n_q)[s], f(K, n_kv)[keys], f(V, n_kv)[keys], one, bq, bkv, f(dO, n_q)[s])
                    q[s] = a
                    kk[keys] += b
                    v[keys] += c
                qh = orc.history_readout_bwd(f(Q, n_q), states[h][0], states[h][1], f(dO, n_q))
            for name, got, ref in (("dQ", f(dQ, n_q), q + qh), ("dK", f(dK, n_kv), kk), ("dV", f(dV, n_kv), v)):
                e = rel_l2(got, ref)
                assert e <= bound, (name, h, size == full, e)


def test_a_row_far_below_zero_ignores_an_entry_that_names_no_block():
    # scores of -400 (times log2 e): 2^(0 - lse2) of a tile that is not there would be infinite
    cfg = hf.make_config(1, 1, 64, "f32", 16, 16, 0.5, keep_k=2)
    Q = torch.full((1, 1, 16, 64), 20.0, device=DEV)
    K = -20.0 - torch.rand((1, 1, 64, 64), device=DEV, generator=torch.Generator(DEV).manual_seed(3))
    V, dO = torch.randn_like(K), torch.randn_like(Q)
    idx = torch.tensor([[[[2, -1]]]], dtype=torch.int32, device=DEV)
    ws = torch.full((hf.hf_bwd_workspace_bytes(cfg, 16, 64),), 0xFF, dtype=torch.uint8, device=DEV)
    dQ, dK, dV = torch.empty_like(Q), torch.empty_like(K), torch.empty_like(V)
    hf.hf_hybrid_attn_bwd(cfg, Q, K, V, idx, None, dO, dQ, dK, dV, ws)
    f = lambda t: wl.to_f64(t)[0, 0]
    q, k, v = orc.sparse_attention_bwd(f(Q), f(K), f(V), np.array([[2]]), 16, 16, f(dO))
    # scores of 3200 are sums of fp32 rounding 2e-4: the probabilities' relative error
    for got, ref in ((dQ, q), (dK, k), (dV, v)):
        assert torch.isfinite(got).all() and rel_l2(f(got), ref) <= 1e-2
