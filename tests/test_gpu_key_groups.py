"""The bf16 attention kernel with one and with two groups of wavefronts per query block (the launch picks by the number of
workgroups): both sides of each line, lists with fewer tiles than groups and with more than one refill of the tile list, the
absorb that rides in the launch, the training by-products.  Against the fp64 oracle, a few heads of each launch."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import BF16_MAX_ABS, BF16_REL_L2, heads_of, max_abs, oracle_state, rel_l2, split_state

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [  # heads, block, n_q, n_kv, keep: workgroups
    (1, 64, 1, 20, 1.0), (2, 64, 130, 1000, 0.4), (1, 64, 65, 4400, 1.0),      # two groups: one tile, a few, more than 64 each
    (32, 64, 1024, 150, 0.5), (27, 64, 1217, 150, 0.5),                        # 512 two groups, 540 one
    (40, 64, 1601, 100, 0.6), (49, 64, 2000, 70, 1.0),                         # 1040 two groups, 1568 one
    (2, 128, 129, 400, 0.5), (32, 128, 1000, 130, 1.0), (37, 128, 830, 260, 0.4),  # block 128: 4 and 256 two groups, 259 one
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_both_sides_of_the_line(case):
    H, b, n_q, n_kv, keep = case
    d, n_ev = 128, 77
    cfg = hf.make_config(1, H, d, "bf16", b, b, keep)
    mk = lambda n, s: wl.randn((1, H, n, d), 47_000 + s, 0.5, torch.bfloat16)
    Q, K, V, Ke, Ve, Kn, Vn, dO = mk(n_q, 0), mk(n_kv, 1), mk(n_kv, 2), mk(60, 3), mk(60, 4), mk(n_ev, 5), mk(n_ev, 6), mk(n_q, 7)
    Qd, Kd, Vd = Q.to(DEV), K.to(DEV), V.to(DEV)
    byte = lambda n: torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, Ke.to(DEV), Ve.to(DEV))
    planes = byte(hf.hf_state_planes_bytes(cfg))
    hf.hf_state_planes(cfg, st, planes)
    st2, planes2 = torch.full_like(st, float("nan")), torch.empty_like(planes)
    pooled = byte(hf.hf_pooled_keys_bytes(cfg, n_kv))
    t_m, k = -(-n_q // b), hf.hf_select_k(cfg, n_kv)
    idx = torch.full((1, H, t_m, k), -1, dtype=torch.int32, device=DEV)
    O = torch.full(Q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
    hf.hf_pool_keys(cfg, Kd, pooled)
    hf.hf_step_fwd(cfg, Qd, Kd, Vd, pooled, st, planes, O, idx, Kn.to(DEV), Vn.to(DEV), st2, planes2,
                   byte(hf.hf_step_workspace_bytes(cfg, n_q, n_ev)))
    # the lists handed in, the by-products of the training forward
    Os, Ol, O0 = torch.full_like(O, float("nan")), torch.full_like(O, float("nan")), torch.full_like(O, float("nan"))
    lse2 = torch.full((H, n_q), float("nan"), dtype=torch.float32, device=DEV)
    ws = byte(hf.hf_workspace_bytes(cfg, n_q, n_kv))
    hf.hf_hybrid_attn_fwd_save(cfg, Qd, Kd, Vd, idx, st, Os, Ol, lse2, ws)
    hf.hf_hybrid_attn_fwd(cfg, Qd, Kd, Vd, idx, None, O0)
    dQ, dK, dV = torch.empty_like(Qd), torch.empty_like(Kd), torch.empty_like(Vd)
    hf.hf_hybrid_attn_bwd_saved(cfg, Qd, Kd, Vd, idx, st, dO.to(DEV), Ol, lse2, dQ, dK, dV,
                                byte(hf.hf_bwd_workspace_bytes(cfg, n_q, n_kv)))
    torch.cuda.synchronize()
    assert torch.equal(O0, Ol)
    idxc, L2, z2 = idx.cpu().numpy(), *split_state(st2, H, d)
    for h in sorted({0, H // 2, H - 1}):
        one = lambda t: heads_of(t[:, h:h + 1])[0]
        q, kk, v = one(Q), one(K), one(V)
        state = oracle_state([Ke[:, h:h + 1]], [Ve[:, h:h + 1]], d)[0]
        assert np.array_equal(idxc[0, h], orc.select_blocks(orc.block_scores(q, kk, b, b), k)[0])
        ref, *_ = orc.hybrid_attention(q, kk, v, state, b, b, k, cfg.phi, None, None, cfg.eps, cfg.z_scale, block_idx=idxc[0, h])
        loc = orc.sparse_attention(q, kk, v, idxc[0, h], b, b)
        for name, got, want in (("step", O, ref), ("save", Os, ref), ("local", Ol, loc)):
            x = wl.to_f64(got)[0, h]
            assert rel_l2(x, want) <= BF16_REL_L2 and max_abs(x, want) <= BF16_MAX_ABS, (name, h, rel_l2(x, want))
        dq, dqh, dk, dv = orc.hybrid_attention_bwd(q, kk, v, state, b, b, idxc[0, h], one(dO), cfg.phi, None, None, cfg.eps,
                                                   cfg.z_scale)
        for name, got, want in (("dQ", dQ, dq + dqh), ("dK", dK, dk), ("dV", dV, dv)):
            assert rel_l2(wl.to_f64(got)[0, h], want) <= 1e-2, (name, h)
        Ln, zn = orc.state_absorb(*state, one(Kn), one(Vn))
        assert rel_l2(L2[h], Ln) <= 1e-5 and rel_l2(z2[h], zn) <= 1e-5
