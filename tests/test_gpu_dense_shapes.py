"""The dense window (no block list) in bf16 at head_dim 128: every workgroup shape that the launch picks from (wavefronts of
rows x groups of keys), with ragged rows and keys, alone and with the history term.  Against the fp64 oracle, a few heads."""
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import BF16_MAX_ABS, BF16_REL_L2, heads_of, max_abs, oracle_state, rel_l2

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [  # heads, block, n_q, n_kv, phi: shape
    (300, 64, 70, 90, "relu"),       # 2 x 1
    (60, 64, 130, 130, "elu"),       # 2 x 2
    (3, 64, 70, 1000, "elu"),        # 2 x 4
    (1, 64, 33, 4401, "relu"),       # the same, more than 64 tiles in a group's list
    (2, 128, 200, 2000, "elu"),      # 2 x 4 at block 128
    (256, 64, 130, 130, "relu"),     # 2 x 1 in two rounds
    (250, 64, 300, 130, "relu"),     # 4 x 1
    (60, 64, 500, 1001, "elu"),      # 4 x 2
    (240, 64, 250, 1930, "relu"),    # 8 x 1, rows short of a workgroup's
    (240, 48, 250, 1930, "elu"),     # the same with KV blocks of one and a half tiles
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_dense_shapes(case):
    H, b, n_q, n_kv, phi = case
    d, bq = 128, 64 if b == 48 else b
    cfg = hf.make_config(1, H, d, "bf16", bq, b, 1.0, phi=hf.HF_PHI_RELU if phi == "relu" else hf.HF_PHI_ELU1)
    mk = lambda n, s: wl.randn((1, H, n, d), 53_000 + s, 0.5, torch.bfloat16)
    Q, K, V, Ke, Ve = mk(n_q, 0), mk(n_kv, 1), mk(n_kv, 2), mk(60, 3), mk(60, 4)
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, Ke.to(DEV), Ve.to(DEV))
    ws = torch.empty(max(int(hf.hf_workspace_bytes(cfg, n_q, n_kv)), 256), dtype=torch.uint8, device=DEV)
    O, O0 = (torch.full(Q.shape, float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    Qd, Kd, Vd = Q.to(DEV), K.to(DEV), V.to(DEV)
    hf.hf_hybrid_attn_fwd(cfg, Qd, Kd, Vd, None, st, O, ws)
    hf.hf_hybrid_attn_fwd(cfg, Qd, Kd, Vd, None, None, O0)
    torch.cuda.synchronize()
    assert torch.isfinite(O).all() and torch.isfinite(O0).all()
    for h in sorted({0, H // 2, H - 1}):
        one = lambda t: heads_of(t[:, h:h + 1])[0]
        q, kk, v = one(Q), one(K), one(V)
        state = oracle_state([Ke[:, h:h + 1]], [Ve[:, h:h + 1]], d, phi=cfg.phi)[0]
        loc = orc.dense_attention(q, kk, v)
        ref = loc + orc.history_readout(q, *state, cfg.phi, None, None, cfg.eps, cfg.z_scale)
        for name, got, want in (("hybrid", O, ref), ("local", O0, loc)):
            x = wl.to_f64(got)[0, h]
            assert rel_l2(x, want) <= BF16_REL_L2 and max_abs(x, want) <= BF16_MAX_ABS, (name, h, rel_l2(x, want))
