"""The bf16 attention kernel with one and with two groups of wavefronts per query block (the launch picks by the number of
workgroups): both sides of each line, lists with fewer tiles than groups and with more than one refill of the tile list, the
absorb that rides in the launch, the training by-products.  Against the fp64 oracle, a few heads of each launch."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import BF16_MAX_ABS, BF16_REL_L2, check_block_idx, heads_of, max_abs, oracle_state, rel_l2, split_state

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [  # heads, block, n_q, n_kv, keep: workgroups
    # (attending workgroups + the two absorbing ones per head that the launch counts)
    (1, 64, 1, 20, 1.0), (2, 64, 130, 1000, 0.4), (1, 64, 65, 4400, 1.0),      # two groups: one tile, a few, more than 64 each
    (32, 64, 1024, 150, 0.5), (27, 64, 1217, 150, 0.5), (32, 64, 896, 150, 0.5),  # 512 + 64 and 540 + 54 one, 448 + 64 two
    (40, 64, 1601, 100, 0.6), (49, 64, 2000, 70, 1.0),                         # 1040 + 80 two groups, 1568 + 98 one
    (2, 128, 129, 400, 0.5), (32, 128, 768, 130, 1.0),                         # block 128: 4 + 4 and 192 + 64 two groups
    (32, 128, 1000, 130, 1.0), (37, 128, 830, 260, 0.4),                       # 256 + 64 and 259 + 74 one
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


@pytest.mark.parametrize("b,heads,n_q,n_kv", [(64, 60, 640, 3000), (64, 60, 620, 64 * 262 + 9), (128, 30, 1200, 4000)])
def test_a_head_alone_and_among_many(b, heads, n_q, n_kv):
    """The same two heads in a launch of their own (two groups) and repeated to one with a single group.  Scores and lists are
    the same bits: their sums keep terms and order.  Outputs differ by the order of fp32 sums alone, P being rounded against
    the same reference: 1e-6 moves one bf16 rounding in 4000 by 2^-8, 6e-5 in all, where P rounded against another
    reference is 2.3e-3 away."""
    d = 128
    mk = lambda n, s: wl.randn((1, 2, n, d), 47_100 + s, 0.5, torch.bfloat16).to(DEV)
    Q, K, V, Ke, Ve = mk(n_q, 0), mk(n_kv, 1), mk(n_kv, 2), mk(90, 3), mk(90, 4)

    def run(H):
        cfg = hf.make_config(1, H, d, "bf16", b, b, 0.3)
        q, kk, v, ke, ve = (t.repeat(1, H // 2, 1, 1) for t in (Q, K, V, Ke, Ve))
        st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
        hf.hf_state_init(cfg, st)
        hf.hf_absorb_evicted(cfg, st, ke, ve)
        byte = lambda n: torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)
        planes, pooled = byte(hf.hf_state_planes_bytes(cfg)), byte(hf.hf_pooled_keys_bytes(cfg, n_kv))
        hf.hf_state_planes(cfg, st, planes)
        hf.hf_pool_keys(cfg, kk, pooled)
        t_m, t_n = -(-n_q // b), -(-n_kv // b)
        idx = torch.full((1, H, t_m, hf.hf_select_k(cfg, n_kv)), -1, dtype=torch.int32, device=DEV)
        scores = torch.full((1, H, t_m, t_n), float("nan"), dtype=torch.float32, device=DEV)
        O, Os, Ol = (torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(3))
        lse2 = torch.full((H, n_q), float("nan"), dtype=torch.float32, device=DEV)
        hf.hf_select_attn_fwd(cfg, q, kk, v, pooled, st, planes, O, idx, scores)
        hf.hf_hybrid_attn_fwd_save(cfg, q, kk, v, idx, st, Os, Ol, lse2, byte(hf.hf_workspace_bytes(cfg, n_q, n_kv)))
        torch.cuda.synchronize()
        return idx, scores, lse2[None], O, Os, Ol

    few, many = run(2), run(heads)
    for h in (0, heads - 2):
        pair = [t[:, h:h + 2] for t in many]
        assert torch.equal(few[1], pair[1]) and torch.equal(few[0], pair[0])
        assert (few[2] - pair[2]).abs().max().item() <= 1e-5   # log2 of fp32 sums
        for name, a, r in zip(("O", "saved O", "O_local"), few[3:], pair[3:]):
            assert rel_l2(wl.to_f64(a), wl.to_f64(r)) <= 3e-4, name


@pytest.mark.parametrize("b,heads,n_q", [(64, 25, 64 * 20), (64, 20, 64 * 50), (128, 16, 128 * 16)])
def test_an_absorb_in_the_launch_does_not_change_its_bits(b, heads, n_q):
    """Launches of just one full round (500, 1000 and 256 attending workgroups): the absorbing ones are counted either way."""
    d, n_kv, n_ev = 128, 700, 90
    cfg = hf.make_config(1, heads, d, "bf16", b, b, 0.4)
    mk = lambda n, s: wl.randn((1, heads, n, d), 47_200 + s, 0.5, torch.bfloat16).to(DEV)
    Q, K, V, Ke, Ve = mk(n_q, 0), mk(n_kv, 1), mk(n_kv, 2), mk(n_ev, 3), mk(n_ev, 4)
    byte = lambda n: torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, Ke, Ve)
    planes, pooled = byte(hf.hf_state_planes_bytes(cfg)), byte(hf.hf_pooled_keys_bytes(cfg, n_kv))
    hf.hf_state_planes(cfg, st, planes)
    hf.hf_pool_keys(cfg, K, pooled)
    out = []
    for absorb in (False, True):
        idx = torch.full((1, heads, -(-n_q // b), hf.hf_select_k(cfg, n_kv)), -1, dtype=torch.int32, device=DEV)
        O = torch.full(Q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
        if absorb:
            hf.hf_step_fwd(cfg, Q, K, V, pooled, st, planes, O, idx, Ke, Ve, torch.empty_like(st), torch.empty_like(planes),
                           byte(hf.hf_step_workspace_bytes(cfg, n_q, n_ev)))
        else:
            hf.hf_select_attn_fwd(cfg, Q, K, V, pooled, st, planes, O, idx)
        out.append((idx, O))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


# heads, block, n_q, n_kv, keep: attending workgroups + absorbing ones counted
ROTATED = [
    (40, 64, 840, 700, 0.4), (64, 64, 832, 150, 0.6),             # one group: 560 + 80 and 832 + 128
    (32, 128, 1030, 900, 0.5), (49, 128, 600, 300, 1.0),          # one group: 288 + 64 and 245 + 98
    (3, 64, 200, 700, 0.4), (2, 128, 300, 900, 0.5),              # two groups
    (40, 64, 840, 64 * 300 + 7, 0.02), (32, 128, 1030, 128 * 262 + 5, 0.02),   # one group, more than 256 KV blocks
]


@pytest.mark.parametrize("case", ROTATED, ids=lambda c: "-".join(map(str, c)))
def test_rotated_readout_on_both_sides(case):
    """ELU features, rotated queries and keys of the history term, queries of its own: by the selecting launch and, the same
    bits, from the list handed in."""
    H, b, n_q, n_kv, keep = case
    d, n_ev = 128, 70
    cfg = hf.make_config(1, H, d, "bf16", b, b, keep, phi=hf.HF_PHI_ELU1)
    mk = lambda n, s: wl.randn((1, H, n, d), 47_300 + s, 0.5, torch.bfloat16)
    Q, Qh, K, V, Ke, Ve = mk(n_q, 0), mk(n_q, 1), mk(n_kv, 2), mk(n_kv, 3), mk(n_ev, 4), mk(n_ev, 5)
    qtab, etab = wl.rope_tables(n_q, d, first_position=5.0, tokens_per_position=50), wl.rope_tables(n_ev, d, first_position=1.0)
    on = lambda *t: [x.to(DEV) for x in t]
    byte = lambda n: torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, *on(Ke, Ve, *etab))
    planes, pooled = byte(hf.hf_state_planes_bytes(cfg)), byte(hf.hf_pooled_keys_bytes(cfg, n_kv))
    hf.hf_state_planes(cfg, st, planes)
    Qd, Qhd, Kd, Vd, cos, sin = on(Q, Qh, K, V, *qtab)
    hf.hf_pool_keys(cfg, Kd, pooled)
    t_m, t_n, k = -(-n_q // b), -(-n_kv // b), hf.hf_select_k(cfg, n_kv)
    idx = torch.full((1, H, t_m, k), -1, dtype=torch.int32, device=DEV)
    scores = torch.full((1, H, t_m, t_n), float("nan"), dtype=torch.float32, device=DEV)
    O, Ol = (torch.full(Q.shape, float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    hf.hf_select_attn_fwd(cfg, Qd, Kd, Vd, pooled, st, planes, O, idx, scores, cos, sin, Qhd)
    hf.hf_hybrid_attn_fwd_planes(cfg, Qd, Kd, Vd, idx, st, planes, Ol, cos, sin, Qhd)
    torch.cuda.synchronize()
    assert torch.equal(O, Ol)
    idxc, cs, sn = idx.cpu().numpy(), wl.to_f64(qtab[0]), wl.to_f64(qtab[1])
    for h in sorted({0, H // 2, H - 1}):
        one = lambda t: heads_of(t[:, h:h + 1])[0]
        q, kk = one(Q), one(K)
        L, z = oracle_state([Ke[:, h:h + 1]], [Ve[:, h:h + 1]], d, cfg.phi, [etab])[0]
        A = orc.block_scores(q, kk, b, b)
        assert np.abs(wl.to_f64(scores)[0, h] - A).max() <= 1e-5 * max(1.0, np.abs(A).max())
        check_block_idx(idxc[0, h], A, k)
        ref = orc.sparse_attention(q, kk, one(V), idxc[0, h], b, b) + orc.history_readout(one(Qh), L, z, cfg.phi, cs, sn, cfg.eps, cfg.z_scale)
        x = wl.to_f64(O)[0, h]
        assert rel_l2(x, ref) <= BF16_REL_L2 and max_abs(x, ref) <= BF16_MAX_ABS, (h, rel_l2(x, ref))


@pytest.mark.parametrize("heads,b,n_q", [(2, 64, 130), (40, 64, 840), (2, 128, 130), (32, 128, 1030)])
def test_the_second_plane_of_the_state(heads, b, n_q):
    """Every element of L is c = 1 + 2^-8 - 2^-12, of which the high plane is 1, every element of z is 0.998 and V is zero: every
    output is c / 0.998 = 1.0057, next to 1 + 2^-7, with both planes and 1 / 0.998 = 1.002, next to 1, with one."""
    d, n_kv = 128, 300
    Q, K = (wl.randn((1, heads, n, d), 47_400, 0.5, torch.bfloat16).to(DEV) for n in (n_q, n_kv))
    for flags, want in ((hf.HF_FLAG_HISTORY_TWO_PLANES, 1 + 2.0 ** -7), (0, 1.0)):
        cfg = hf.make_config(1, heads, d, "bf16", b, b, 0.5, flags=flags)
        st = torch.full((hf.hf_state_bytes(cfg) // 4,), 1 + 2.0 ** -8 - 2.0 ** -12, dtype=torch.float32, device=DEV)
        st[heads * d * d:] = 0.998
        ws = torch.empty(hf.hf_workspace_bytes(cfg, n_q, n_kv), dtype=torch.uint8, device=DEV)
        O = torch.full(Q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
        hf.hf_hybrid_attn_fwd(cfg, Q, K, torch.zeros_like(K), None, st, O, ws)
        torch.cuda.synchronize()
        assert (O == want).all()
