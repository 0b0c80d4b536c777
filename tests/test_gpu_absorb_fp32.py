"""Eq. 2 in fp32 arithmetic (fp32 inputs, bf16 with head_dim 64) at the edges of its runs and slices: one token, one more or
less than a wavefront's 16, than a round's 128, than the 1024 tokens that one workgroup per tile takes without atomics."""
import numpy as np
import pytest
import torch

import paper_2604_10103_amd as hf
import workloads as wl
from parity import oracle_state, rel_l2

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("n", [1, 15, 17, 127, 129, 1024, 1025, 2600])
@pytest.mark.parametrize("phi,rope", [(hf.HF_PHI_RELU, False), (hf.HF_PHI_ELU1, True)])
def test_absorb_matches_the_oracle_at_edges(dtype, d, n, phi, rope):
    B, H = 1, 3
    cfg = hf.make_config(B, H, d, dtype, 64, 64, 0.5, phi=phi)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K, V = (wl.randn((B, H, n, d), 52_000 + i, 0.5, tdt) for i in range(2))
    tabs = wl.rope_tables(n, d, first_position=3.0) if rope else (None, None)
    st = torch.full((hf.hf_state_bytes(cfg) // 4,), 0.25, dtype=torch.float32, device=DEV)   # a state that holds something
    hf.hf_absorb_evicted(cfg, st, K.to(DEV), V.to(DEV), *(None if t is None else t.to(DEV) for t in tabs))
    torch.cuda.synchronize()
    ref = oracle_state([K], [V], d, phi, [tabs] if rope else None)
    got = st.cpu().double().numpy()
    L, z = got[:B * H * d * d].reshape(B * H, d, d), got[B * H * d * d:].reshape(B * H, d)
    # fp32 sums over n tokens: sqrt(n) 2^-24 of the sum's size, far inside the bound of the other absorb tests
    assert rel_l2(L, np.stack([r[0] for r in ref]) + 0.25) <= 1e-5
    assert rel_l2(z, np.stack([r[1] for r in ref]) + 0.25) <= 1e-5
