"""Selection inside the attention launch: rows of scores on both sides of every number of keys that a lane holds (one to four,
then the ranking of long rows), with ties across the k-th place.  Lists against the oracle's."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import check_block_idx, heads_of

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("b", [64, 128])
@pytest.mark.parametrize("t_n", [1, 2, 63, 64, 65, 128, 129, 192, 193, 256, 257])
def test_rows_of_scores(t_n, b):
    H, d, n_q, n_kv = 2, 128, b + 7, b * t_n - 5
    for keep in (0.03, 0.5):
        cfg = hf.make_config(1, H, d, "bf16", b, b, keep)
        Q, K, V = (wl.randn((1, H, n, d), 59_000 + i, 0.5, torch.bfloat16) for i, n in enumerate((n_q, n_kv, n_kv)))
        if t_n > 4:   # equal scores, which only their indices tell apart
            for j in range(0, t_n - 1, 3):
                K[:, :, b * j:b * j + b] = K[:, :, :b]
        Qd, Kd, Vd = Q.to(DEV), K.to(DEV), V.to(DEV)
        pooled = torch.empty(hf.hf_pooled_keys_bytes(cfg, n_kv), dtype=torch.uint8, device=DEV)
        k = hf.hf_select_k(cfg, n_kv)
        idx = torch.full((1, H, 2, k), -1, dtype=torch.int32, device=DEV)
        O = torch.empty_like(Qd)
        hf.hf_pool_keys(cfg, Kd, pooled)
        hf.hf_select_attn_fwd(cfg, Qd, Kd, Vd, pooled, None, None, O, idx)
        torch.cuda.synchronize()
        for h in range(H):
            q, kk, v = (heads_of(t[:, h:h + 1])[0] for t in (Q, K, V))
            rows = idx[0, h].cpu().numpy()
            check_block_idx(rows, orc.block_scores(q, kk, b, b), k)
            ref = orc.sparse_attention(q, kk, v, rows, b, b)
            got = wl.to_f64(O)[0, h]
            assert np.linalg.norm(got - ref) <= 1e-2 * np.linalg.norm(ref)
