"""Steps of streams and rings whose window has more KV blocks than the attention launch selects from (1024): the selection's own
launches, then attention with the state's planes that the chunk's first step leaves in the workspace.  Every step of two chunks, the
state changed in between, against the separate calls, which form the history term anew: the same bits."""
import pytest
import torch

import paper_2604_10103_amd as hf
import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("driver", ["ring", "stream"])
@pytest.mark.parametrize("H,bq,n,slots,phi,rope", [(1, 64, 2051, 8, "relu", False), (2, 128, 1100, 16, "elu", True),
                                                   (1, 64, 8200, 2, "elu", True), (4, 128, 8300, 2, "relu", False)])
def test_every_step_of_two_chunks(driver, H, bq, n, slots, phi, rope):
    d, b, n_kv = 128, 16, slots * n
    assert 1024 < -(-n_kv // b) <= 1100
    phi = hf.HF_PHI_RELU if phi == "relu" else hf.HF_PHI_ELU1
    cfg, packed = (hf.make_config(1, H, d, "bf16", bq, b, 0.02, phi=phi, kv_capacity=c) for c in (n_kv, 0))
    byte = lambda m: torch.full((max(int(m), 256),), 255, dtype=torch.uint8, device=DEV)   # (NaN)
    mk = lambda m, s: wl.randn((1, H, m, d), 83_000 + s, 0.5, torch.bfloat16).to(DEV)
    K, V = mk(n_kv, 0), mk(n_kv, 1)
    tabs = tuple(t.to(DEV) for t in wl.rope_tables(n, d, first_position=3.0)) if rope else (None, None)
    ws, ws2 = byte(hf.hf_workspace_bytes(cfg, n, n_kv)), byte(hf.hf_workspace_bytes(packed, n, n_kv))
    sws = byte(max(hf.hf_step_workspace_bytes(cfg, n, n), hf.hf_absorb_workspace_bytes(cfg, n)))
    st, st2 = (torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV) for _ in range(2))
    idx, idx2 = (torch.empty((1, H, -(-n // bq), hf.hf_select_k(cfg, n_kv)), dtype=torch.int32, device=DEV) for _ in range(2))
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(packed, st, mk(60, 2), mk(60, 3))
    ring, win = hf.make_ring(0, n), hf.hf_window(0, n_kv)
    ring.n_filled, ring.cur_slot, ring.next_slot, ring.absorbed_ahead = slots, slots - 1, 0, 0
    for chunk in range(2):
        at = (n_kv - n) if driver == "stream" else n * ring.cur_slot
        for step in range(3):
            Q = mk(n, 10 + 4 * chunk + step)
            K[:, :, at:at + n] = K[:, :, at:at + n].flip(3)
            O, O2, O0 = (torch.full_like(Q, float("nan")) for _ in range(3))
            if driver == "stream":
                hf.hf_stream_step(cfg, win, Q, K, V, step, idx, st, O, ws, *tabs)
            elif step < 2:
                hf.hf_ring_step(cfg, ring, Q, K, V, step, idx, st, O, ws, *tabs)
            else:
                assert hf.hf_ring_last_step(cfg, ring, Q, K, V, step, idx, st, O, ws, st2, sws, *tabs)
            hf.hf_block_select(packed, Q, K, idx2, None, ws2)
            hf.hf_hybrid_attn_fwd(packed, Q, K, V, idx2, st, O2, ws2, *tabs)
            hf.hf_hybrid_attn_fwd(packed, Q, K, V, idx2, None, O0, ws2)
            torch.cuda.synchronize()
            assert torch.equal(idx, idx2)
            assert torch.isfinite(O).all() and torch.equal(O, O2), (driver, chunk, step)
            assert not torch.equal(O2, O0)   # (the state is seen)
        if driver == "stream":
            hf.hf_absorb_evicted(packed, st, mk(100, 4), mk(100, 5))
        else:
            st, st2 = st2, st
            hf.hf_ring_open_chunk(cfg, ring, K, V, st, workspace=sws)
