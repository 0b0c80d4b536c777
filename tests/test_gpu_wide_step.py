"""Steps of small fp32 streams as one launch (selection, attention, history term and the next eviction's absorb): blocks pooled in
the launch and in front of it, windows of one to 256 KV blocks and past that, workgroups up to the limit and past it, blocks of more
rows than a workgroup, ties, rotated queries and evicted keys; steps that absorb nothing, whose lists have to be long enough for it.
Lists as the selection's own launches give them, outputs and states against those and the oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import F32_REL_L2, heads_of, oracle_state, rel_l2, split_state

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [  # heads, head_dim, block, tokens of a chunk, of the sink, slots, keep, phi
    (1, 64, 16, 1, 0, 2, 1.0, "relu"),        # a window of two tokens
    (2, 64, 16, 64, 0, 4, 0.25, "relu"),      # sixteen blocks, all pooled in the launch on the first step
    (2, 64, 16, 65, 3, 4, 0.25, "elu"),       # seventeen: not those; the chunk's own straddle their neighbours'
    (3, 128, 32, 50, 0, 3, 0.5, "relu"),
    (1, 64, 16, 341, 5, 12, 0.1, "relu"),     # 256 + 1 blocks: the separate launches
    (1, 64, 16, 341, 0, 12, 0.1, "elu"),      # 256
    (2, 128, 64, 70, 7, 3, 0.4, "elu"),       # four workgroups a block, two of them without a row in the last
    (4, 64, 16, 1024, 0, 2, 0.06, "relu"),    # 256 workgroups, the longest chunk absorbed beside them
    (1, 64, 16, 1025, 0, 2, 0.06, "relu"),    # one token more: absorbed by a launch of its own
    (1, 64, 128, 1024, 0, 2, 0.15, "elu"),    # sixteen blocks of too many bytes: pooled in front on the first step, eight not
    (1, 128, 48, 200, 0, 4, 0.3, "relu"),     # blocks that are no multiple of 32
    (48, 128, 16, 16, 0, 4, 0.5, "relu"),     # as many absorbing workgroups as ride in the launch
    (49, 128, 16, 16, 0, 28, 1.0, "relu"),    # one head more: absorbed by a launch of its own
    (5, 64, 16, 817, 0, 2, 0.06, "relu"),     # 260 workgroups: the separate launches
]


@pytest.mark.parametrize("state", [True, False, "rotated"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_steps_of_a_full_ring(case, state):
    H, d, b, n, sink, slots, keep, phi = case
    n_kv = sink + slots * n
    phi = hf.HF_PHI_RELU if phi == "relu" else hf.HF_PHI_ELU1
    cfg, packed = (hf.make_config(1, H, d, "f32", b, b, keep, phi=phi, kv_capacity=c) for c in (n_kv, 0))
    K, V, Ke, Ve, *Qs = (wl.randn((1, H, m, d), 91_000 + i, 1.0, torch.float32) for i, m in enumerate((n_kv, n_kv, 40, 40, n, n, n)))
    rot = state == "rotated"   # tables for the queries, which are others than the window's, and for the evicted chunk
    tabs, tabs_ev = (wl.rope_tables(n, d, first_position=p) if rot else (None, None) for p in (3.0, 1.5))
    (cq, sq), (ce, se) = ([None if t is None else t.to(DEV) for t in ts] for ts in (tabs, tabs_ev))
    t64, te64 = (tuple(None if t is None else wl.to_f64(t) for t in ts) for ts in (tabs, tabs_ev))
    K[:, :, -1] = K[:, :, 0]
    if n_kv >= 6 * b:   # whole blocks alike: ties
        K[:, :, 2 * b:3 * b] = K[:, :, :b]
        K[:, :, 4 * b:5 * b] = K[:, :, :b]
    Kd, Vd = K.to(DEV), V.to(DEV)
    st = None
    if state:
        st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
        hf.hf_state_init(cfg, st)
        hf.hf_absorb_evicted(packed, st, Ke.to(DEV), Ve.to(DEV))
    st2 = torch.full((hf.hf_state_bytes(cfg) // 4,), float("nan"), device=DEV)
    byte = lambda m: torch.full((max(int(m), 256),), 255, dtype=torch.uint8, device=DEV)   # (NaN)
    ws, sws = byte(hf.hf_workspace_bytes(cfg, n, n_kv)), byte(max(hf.hf_step_workspace_bytes(cfg, n, n), hf.hf_absorb_workspace_bytes(cfg, n)))
    ring = hf.make_ring(sink, n)
    ring.n_filled, ring.cur_slot, ring.next_slot, ring.absorbed_ahead = slots, slots - 1, 0, 0
    k, t_m = hf.hf_select_k(cfg, n_kv), -(-n // b)
    at = sink + (slots - 1) * n
    for i, Q in enumerate(Qs):
        Qd, O, O2 = Q.to(DEV), *(torch.full(Q.shape, float("nan"), device=DEV) for _ in range(2))
        idx, idx2 = (torch.full((1, H, t_m, k), -1, dtype=torch.int32, device=DEV) for _ in range(2))
        Qh = Q.flip(2).contiguous() if rot else None
        Qhd = None if Qh is None else Qh.to(DEV)
        if i:   # the chunk's keys of this step
            Kd[:, :, at:] = Kd[:, :, at:].flip(3)
        if i < 2:
            hf.hf_ring_step(cfg, ring, Qd, Kd, Vd, i, idx, st, O, ws, cq, sq, Qhd)
        else:
            assert hf.hf_ring_last_step(cfg, ring, Qd, Kd, Vd, i, idx, st, O, ws, st2, sws, cq, sq, Qhd, ce, se)
        ws2 = byte(hf.hf_workspace_bytes(packed, n, n_kv))
        hf.hf_block_select(packed, Qd, Kd, idx2, None, ws2)
        hf.hf_hybrid_attn_fwd(packed, Qd, Kd, Vd, idx2, st, O2, ws2, cq, sq, Qhd)
        torch.cuda.synchronize()
        assert torch.equal(idx, idx2)
        for h in sorted({0, H - 1}):
            assert rel_l2(wl.to_f64(O)[0, h], wl.to_f64(O2)[0, h]) <= F32_REL_L2
            one = lambda t: heads_of(t.cpu()[:, h:h + 1])[0]
            s0 = oracle_state([Ke[:, h:h + 1]], [Ve[:, h:h + 1]], d, phi=cfg.phi)[0] if state else None
            ref = orc.sparse_attention(one(Q), one(Kd), one(Vd), idx[0, h].cpu().numpy(), b, b)
            if state:
                ref = ref + orc.history_readout(one(Q if Qh is None else Qh), *s0, cfg.phi, *t64, cfg.eps, cfg.z_scale)
            assert rel_l2(wl.to_f64(O)[0, h], ref) <= F32_REL_L2
    L, z = split_state(st2, H, d)
    for h in sorted({0, H - 1}):
        s0 = oracle_state([Ke[:, h:h + 1]], [Ve[:, h:h + 1]], d, phi=cfg.phi)[0] if state else orc.state_zero(d)
        ke, ve = (wl.to_f64(t[0, h, sink:sink + n].cpu()) for t in (Kd, Vd))
        Lr, zr = orc.state_absorb(*s0, ke, ve, cfg.phi, *te64)
        assert rel_l2(L[h], Lr) <= 1e-5 and rel_l2(z[h], zr) <= 1e-5
    assert ring.absorbed_ahead == 1
    assert np.isfinite(wl.to_f64(st2)).all()


# head_dim, block of keys, of queries, window, tokens of the chunk, keep: lists on both sides of the line at head_dim 128 (26 tiles of 16
# keys for query blocks of 16, 27 of 32, 35 of 128; 25 at 64 for chunks of more than fifteen blocks), every block or a part of them
# pooled in the launch, blocks of two sizes
STREAMS = [(128, 16, 16, 400, 37, 1.0), (128, 16, 16, 416, 37, 1.0), (128, 32, 32, 416, 60, 1.0), (128, 32, 32, 450, 60, 1.0),
           (128, 128, 128, 500, 130, 1.0), (128, 128, 128, 640, 130, 1.0), (64, 16, 16, 1552, 40, 0.01), (64, 16, 16, 1552, 40, 0.25),
           (64, 16, 16, 1600, 250, 0.24), (64, 16, 16, 1600, 250, 0.25),
           (64, 256, 256, 2000, 256, 0.1), (64, 48, 20, 700, 90, 0.3), (128, 20, 48, 900, 90, 0.8), (128, 16, 300, 1300, 320, 0.9)]


@pytest.mark.parametrize("case", STREAMS, ids=lambda c: "-".join(map(str, c)))
def test_steps_that_absorb_nothing(case):
    d, b, bq, n_kv, n, keep = case
    cfg, packed = (hf.make_config(1, 2, d, "f32", bq, b, keep, kv_capacity=c) for c in (n_kv, 0))
    K, V, Ke, Ve, *Qs = (wl.randn((1, 2, m, d), 95_000 + i, 1.0, torch.float32).to(DEV) for i, m in enumerate((n_kv, n_kv, 40, 40, n, n)))
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(packed, st, Ke, Ve)
    ws, ws2 = (torch.full((hf.hf_workspace_bytes(cfg, n, n_kv),), 255, dtype=torch.uint8, device=DEV) for _ in range(2))   # (NaN)
    win = hf.hf_window(0, n_kv)
    for i, Q in enumerate(Qs):
        O, O2 = (torch.full_like(Q, float("nan")) for _ in range(2))
        idx, idx2 = (torch.full((1, 2, -(-n // bq), hf.hf_select_k(cfg, n_kv)), -1, dtype=torch.int32, device=DEV) for _ in range(2))
        if i:
            K[:, :, -n:] = K[:, :, -n:].flip(3)
        hf.hf_stream_step(cfg, win, Q, K, V, i, idx, st, O, ws)
        hf.hf_block_select(packed, Q, K, idx2, None, ws2)
        hf.hf_hybrid_attn_fwd(packed, Q, K, V, idx2, st, O2, ws2)
        torch.cuda.synchronize()
        assert torch.equal(idx, idx2)
        assert rel_l2(wl.to_f64(O), wl.to_f64(O2)) <= F32_REL_L2
