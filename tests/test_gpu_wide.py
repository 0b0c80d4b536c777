"""The shape-generic attention kernels (fp32 arithmetic on the matrix cores; bf16 with head_dim 64) at the edges of their
tiles: one row, one key, one more or one less than a tile, block sizes that are no multiple of one, lists shorter than the
wavefronts that share them; forward with the history term, and the gradients, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import BF16_MAX_ABS, BF16_REL_L2, F32_REL_L2, heads_of, max_abs, oracle_state, rel_l2

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

SHAPES = [  # dtype, head_dim, block_q, block_kv, n_q, n_kv, keep (None: dense)
    ("f32", 128, 32, 32, 1, 1, 1.0), ("f32", 128, 64, 32, 33, 65, 0.5), ("f32", 64, 32, 64, 31, 63, 0.4),
    ("f32", 64, 96, 64, 97, 400, 0.3), ("f32", 128, 128, 128, 130, 257, None), ("f32", 64, 64, 64, 300, 900, 0.1),
    ("f32", 128, 20, 24, 41, 100, 0.5), ("f32", 64, 16, 16, 17, 129, 0.25), ("f32", 128, 200, 48, 210, 500, 0.4),
    ("bf16", 128, 32, 32, 33, 100, 0.5), ("bf16", 64, 16, 48, 70, 140, 0.5), ("bf16", 64, 64, 64, 1, 1, 1.0),
    ("bf16", 64, 64, 64, 65, 127, 0.5), ("bf16", 64, 128, 128, 200, 900, 0.3), ("bf16", 64, 64, 32, 130, 300, None),
    ("bf16", 64, 128, 48, 129, 500, 0.4), ("bf16", 64, 192, 96, 193, 450, 0.5), ("bf16", 64, 64, 64, 66, 4300, None),
    ("bf16", 64, 128, 32, 257, 33, 1.0),
]


@pytest.mark.parametrize("case", SHAPES, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("gain,phi,rope", [(1.0, hf.HF_PHI_RELU, False), (8.0, hf.HF_PHI_ELU1, True)])
def test_forward_and_gradients_at_tile_edges(case, gain, phi, rope):
    dtype, d, bq, bkv, n_q, n_kv, keep = case
    B, H = 1, 2
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    cfg = hf.make_config(B, H, d, dtype, bq, bkv, 1.0 if keep is None else keep, phi=phi)
    mk = lambda n, s, g=1.0: wl.randn((B, H, n, d), 31_000 + s, 0.5 * g, tdt)
    Q, K, V, dO = mk(n_q, 0, gain), mk(n_kv, 1), mk(n_kv, 2), mk(n_q, 3)
    Ke, Ve = mk(50, 4), mk(50, 5)
    tab = wl.rope_tables(n_q, d, first_position=9.0) if rope else (None, None)
    dev = lambda t: None if t is None else t.to(DEV)
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, dev(Ke), dev(Ve))
    t_m, t_n, k = -(-n_q // bq), -(-n_kv // bkv), hf.hf_select_k(cfg, n_kv)
    ws = torch.empty(hf.hf_workspace_bytes(cfg, n_q, n_kv), dtype=torch.uint8, device=DEV)
    idx = torch.empty((B, H, t_m, k), dtype=torch.int32, device=DEV)
    hf.hf_block_select(cfg, dev(Q), dev(K), idx, None, ws)
    use = None if keep is None else idx
    O = torch.full((B, H, n_q, d), float("nan"), dtype=tdt, device=DEV)
    hf.hf_hybrid_attn_fwd(cfg, dev(Q), dev(K), dev(V), use, st, O, ws, dev(tab[0]), dev(tab[1]))
    O0 = torch.full_like(O, float("nan"))
    hf.hf_hybrid_attn_fwd(cfg, dev(Q), dev(K), dev(V), use, None, O0)
    dQ, dK, dV = (torch.full(t.shape, float("nan"), dtype=tdt, device=DEV) for t in (Q, K, V))
    bws = torch.empty(hf.hf_bwd_workspace_bytes(cfg, n_q, n_kv), dtype=torch.uint8, device=DEV)
    hf.hf_hybrid_attn_bwd(cfg, dev(Q), dev(K), dev(V), use, st, dev(dO), dQ, dK, dV, bws, dev(tab[0]), dev(tab[1]))
    torch.cuda.synchronize()
    states = oracle_state([Ke], [Ve], d, phi)
    lists = idx.cpu().numpy() if keep is not None else np.tile(np.arange(t_n), (B, H, t_m, 1))
    tabs = tuple(None if t is None else wl.to_f64(t) for t in tab)
    rl, ma = (BF16_REL_L2, BF16_MAX_ABS) if dtype == "bf16" else (F32_REL_L2, 1e-4)
    grl, gma = (1e-2, 2e-2) if dtype == "bf16" else (5e-5, 1e-4)
    for h, (q, kk, v, g) in enumerate(zip(heads_of(Q), heads_of(K), heads_of(V), heads_of(dO))):
        for got, state in ((O, states[h]), (O0, None)):
            ref, *_ = orc.hybrid_attention(q, kk, v, state, bq, bkv, lists.shape[-1], phi, *tabs, cfg.eps, cfg.z_scale,
                                           block_idx=lists[0, h])
            x = wl.to_f64(got)[0, h]
            assert rel_l2(x, ref) <= rl and max_abs(x, ref) <= ma * max(1.0, np.abs(ref).max()), (h, rel_l2(x, ref))
        dq, dqh, dk, dv = orc.hybrid_attention_bwd(q, kk, v, states[h], bq, bkv, lists[0, h], g, phi, *tabs, cfg.eps,
                                                   cfg.z_scale)
        for name, got, ref in (("dQ", dQ, dq + dqh), ("dK", dK, dk), ("dV", dV, dv)):
            x, scale = wl.to_f64(got)[0, h], max(np.abs(ref).max(), 1e-2)
            # (with a single key the softmax is constant: the gradient through it is zero up to rounding)
            assert rel_l2(x, ref) <= grl or np.abs(ref).max() < 1e-9, (name, h, rel_l2(x, ref))
            assert max_abs(x, ref) <= gma * scale, (name, h, max_abs(x, ref), scale)
