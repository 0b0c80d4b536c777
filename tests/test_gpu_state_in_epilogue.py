"""The history term from the fp32 state itself (small launches of the calls that keep no planes) against the call with kept
planes: the same bits, for one and several groups of wavefronts, with lists and dense, both sides of the line, and in the
training forward, whose O_local is staged where the plane lies."""
import pytest
import torch

import paper_2604_10103_amd as hf
import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("H,b,n_q,n_kv", [(3, 64, 70, 400), (8, 64, 4096, 130), (9, 64, 4096, 130), (5, 128, 300, 700),
                                          (16, 128, 2048, 130), (17, 128, 2048, 130), (240, 64, 129, 1930)])
@pytest.mark.parametrize("phi", ["relu", "elu"])
def test_same_bits_as_kept_planes(H, b, n_q, n_kv, dense, phi):
    d = 128
    cfg = hf.make_config(1, H, d, "bf16", b, b, 0.4, phi=hf.HF_PHI_RELU if phi == "relu" else hf.HF_PHI_ELU1)
    Q, K, V, Ke, Ve = (wl.randn((1, H, n, d), 61_000 + i, 0.5, torch.bfloat16).to(DEV) for i, n in enumerate((n_q, n_kv, n_kv, 60, 60)))
    byte = lambda n: torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, Ke, Ve)
    planes, ws = byte(hf.hf_state_planes_bytes(cfg)), byte(hf.hf_workspace_bytes(cfg, n_q, n_kv))
    hf.hf_state_planes(cfg, st, planes)
    idx = None
    if not dense:
        idx = torch.empty((1, H, -(-n_q // b), hf.hf_select_k(cfg, n_kv)), dtype=torch.int32, device=DEV)
        hf.hf_block_select(cfg, Q, K, idx, None, ws)
    O, Op, Os, Ol = (torch.full_like(Q, float("nan")) for _ in range(4))
    lse2 = torch.empty((H, n_q), dtype=torch.float32, device=DEV)
    hf.hf_hybrid_attn_fwd(cfg, Q, K, V, idx, st, O, ws)
    hf.hf_hybrid_attn_fwd_planes(cfg, Q, K, V, idx, st, planes, Op)
    hf.hf_hybrid_attn_fwd_save(cfg, Q, K, V, idx, st, Os, Ol, lse2, ws)
    O0 = torch.full_like(Q, float("nan"))
    hf.hf_hybrid_attn_fwd(cfg, Q, K, V, idx, None, O0)
    torch.cuda.synchronize()
    assert torch.isfinite(O).all()
    assert torch.equal(O, Op) and torch.equal(O, Os) and torch.equal(O0, Ol)
