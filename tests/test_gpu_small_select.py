"""Selection of heads with little to pool (pooling and selection in one launch) on both sides of its limits: blocks per call,
bytes per call, ragged last blocks, rows that do not fill a workgroup, ties, and means kept for later calls."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import check_block_idx, heads_of

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [  # dtype, head_dim, block_q, block_kv, n_q, n_kv
    ("f32", 64, 16, 16, 1, 1), ("f32", 64, 16, 16, 64, 256), ("f32", 64, 16, 16, 65, 257), ("f32", 128, 64, 64, 130, 448),
    ("f32", 128, 64, 64, 64, 449), ("f32", 128, 20, 40, 41, 100), ("bf16", 128, 64, 64, 200, 640), ("bf16", 128, 64, 64, 200, 641),
    ("bf16", 64, 16, 48, 70, 140), ("bf16", 64, 128, 128, 129, 300), ("f32", 64, 16, 128, 200, 800), ("f32", 64, 16, 128, 200, 900),
]


def _select(cfg, Q, K, cached, ws, k, t_m, t_n):
    idx = torch.full((1, Q.shape[1], t_m, k), -1, dtype=torch.int32, device=DEV)
    scores = torch.full((1, Q.shape[1], t_m, t_n), float("nan"), dtype=torch.float32, device=DEV)
    hf.hf_block_select_cached(cfg, Q, K, cached, idx, scores, ws)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), scores.cpu().numpy()


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_scores_lists_and_kept_means(case):
    dtype, d, bq, bkv, n_q, n_kv = case
    H, tdt = 3, torch.bfloat16 if dtype == "bf16" else torch.float32
    cfg = hf.make_config(1, H, d, dtype, bq, bkv, 0.3)
    Q, K = (wl.randn((1, H, n, d), 81_000 + i, 0.5, tdt) for i, n in enumerate((n_q, n_kv)))
    t_m, t_n, k = -(-n_q // bq), -(-n_kv // bkv), hf.hf_select_k(cfg, n_kv)
    new_ws = lambda: torch.full((hf.hf_workspace_bytes(cfg, n_q, n_kv),), 255, dtype=torch.uint8, device=DEV)   # (NaN)
    ws = new_ws()
    idx, scores = _select(cfg, Q.to(DEV), K.to(DEV), 0, ws, k, t_m, t_n)
    for h, (q, kk) in enumerate(zip(heads_of(Q), heads_of(K))):
        A = orc.block_scores(q, kk, bq, bkv)
        assert np.abs(scores[0, h] - A).max() <= 1e-5 * max(1.0, np.abs(A).max())
        check_block_idx(idx[0, h], A, k)
    whole = n_kv // bkv
    for cached in {0, whole // 2, whole}:   # the means kept by the call before, with the keys behind them changed
        K2 = K.clone()
        K2[:, :, cached * bkv:] = K2[:, :, cached * bkv:].flip(3)
        got = _select(cfg, Q.to(DEV), K2.to(DEV), cached, ws, k, t_m, t_n)
        want = _select(cfg, Q.to(DEV), K2.to(DEV), 0, new_ws(), k, t_m, t_n)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        _select(cfg, Q.to(DEV), K.to(DEV), 0, ws, k, t_m, t_n)


def test_ties_keep_the_lower_index():
    cfg = hf.make_config(1, 2, 64, "f32", 16, 16, 1.0, keep_k=5)
    Q, K = wl.randn((1, 2, 50, 64), 82_000, 0.5, torch.float32), wl.randn((1, 2, 16, 64), 82_001, 0.5, torch.float32).repeat(1, 1, 14, 1)
    ws = torch.empty(hf.hf_workspace_bytes(cfg, 50, 224), dtype=torch.uint8, device=DEV)
    idx, _ = _select(cfg, Q.to(DEV), K.to(DEV), 0, ws, 5, 4, 14)
    assert np.array_equal(idx, np.broadcast_to(np.arange(5, dtype=np.int32), idx.shape))


# either side of the limits on workgroups (three query blocks each) and on what they read together
MANY = [  # heads, dtype, head_dim, block_kv, query blocks of 16, KV blocks, of which reused
    (12, "bf16", 128, 16, 63, 6, 0), (12, "bf16", 128, 16, 64, 6, 0), (40, "f32", 128, 64, 9, 6, 0), (40, "f32", 128, 64, 12, 6, 0),
    (48, "f32", 64, 64, 24, 7, 2), (48, "f32", 64, 64, 25, 7, 2), (255, "f32", 128, 64, 2, 6, 1), (258, "f32", 128, 64, 2, 6, 0),
    (40, "bf16", 64, 128, 12, 10, 3), (40, "bf16", 64, 128, 15, 10, 0),
]


@pytest.mark.parametrize("case", MANY, ids=lambda c: "-".join(map(str, c)))
def test_many_heads(case):
    """Three heads repeated: the oracle's scores and lists, and the same bits in every repetition and next to kept means."""
    H, dtype, d, bkv, t_m, t_n, cached = case
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    cfg = hf.make_config(1, H, d, dtype, 16, bkv, 0.5)
    n_q, n_kv = 16 * t_m - 3, bkv * t_n - 5
    Q, K = (wl.randn((1, 3, n, d), 83_000 + i, 0.5, tdt) for i, n in enumerate((n_q, n_kv)))
    q, kk = (t.repeat(1, -(-H // 3), 1, 1)[:, :H].contiguous().to(DEV) for t in (Q, K))
    k = hf.hf_select_k(cfg, n_kv)
    ws = torch.full((hf.hf_workspace_bytes(cfg, n_q, n_kv),), 255, dtype=torch.uint8, device=DEV)   # (NaN)
    idx, scores = _select(cfg, q, kk, 0, ws, k, t_m, t_n)
    for h, (a, b) in enumerate(zip(heads_of(Q), heads_of(K))):
        A = orc.block_scores(a, b, 16, bkv)
        assert np.abs(scores[0, h] - A).max() <= 1e-5 * max(1.0, np.abs(A).max())
        check_block_idx(idx[0, h], A, k)
    for h in range(H):
        assert np.array_equal(idx[0, h], idx[0, h % 3]) and np.array_equal(scores[0, h], scores[0, h % 3])
    if cached:
        kk[:, :, :cached * bkv] = float("nan")   # the means of these are not formed again
        again = _select(cfg, q, kk, cached, ws, k, t_m, t_n)
        assert np.array_equal(again[0], idx) and np.array_equal(again[1], scores)
