"""Small evicted chunks are absorbed beside the attention by two workgroups a head, each for half of the value features: at the
edges of their 16-token stages, of the slices whose order the sums keep, and of the range that takes them."""
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import rel_l2, split_state

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# one stage and less, one slice and two, a short last stage, the longest chunk of this path and the shortest of the other
@pytest.mark.parametrize("n_ev", [1, 15, 17, 64, 256, 257, 700, 1023, 1024, 1025])
@pytest.mark.parametrize("heads,block,n_q", [(3, 64, 130), (5, 128, 200)])
def test_state_beside_the_attention(n_ev, heads, block, n_q):
    """fp32 sums of exact products: 1e-6 of the state's norm.  The rows behind a head's evicted tokens are not read."""
    cfg = hf.make_config(1, heads, 128, "bf16", block, block, 0.5)
    n_kv, stride = 2 * n_q, n_ev + 5
    Q, K, V = (wl.randn((1, heads, n, 128), 41_000 + i, 0.5, torch.bfloat16).to(DEV) for i, n in enumerate((n_q, n_kv, n_kv)))
    Kev, Vev = (wl.randn((1, heads, stride, 128), 42_000 + i, 1.0, torch.bfloat16) for i in range(2))
    K0, V0 = (wl.randn((1, heads, 300, 128), 43_000 + i, 1.0, torch.bfloat16) for i in range(2))
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    planes = torch.empty(hf.hf_state_planes_bytes(cfg), dtype=torch.uint8, device=DEV)
    hf.hf_absorb_evicted_planes(cfg, st, K0.to(DEV), V0.to(DEV), planes)
    pooled = torch.empty(hf.hf_pooled_keys_bytes(cfg, n_kv), dtype=torch.uint8, device=DEV)
    hf.hf_pool_keys(cfg, K, pooled)
    k = hf.hf_select_k(cfg, n_kv)
    idx = torch.empty((1, heads, -(-n_q // block), k), dtype=torch.int32, device=DEV)
    ws = torch.empty(hf.hf_step_workspace_bytes(cfg, n_q, n_ev), dtype=torch.uint8, device=DEV)
    kd, vd = Kev.to(DEV), Vev.to(DEV)
    kd[:, :, n_ev:], vd[:, :, n_ev:] = float("nan"), float("nan")
    outs = []
    for _ in range(2):
        O, st_out = torch.empty_like(Q), torch.full_like(st, float("nan"))
        pl_out = torch.empty_like(planes)
        hf.hf_step_fwd(cfg, Q, K, V, pooled, st, planes, O, idx, kd, vd, st_out, pl_out, ws, n_ev=n_ev)
        torch.cuda.synchronize()
        outs.append((O, st_out, pl_out))
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    L, z = split_state(st_out, heads, 128)
    for h in range(heads):
        Lr, zr = orc.state_absorb(*orc.state_zero(128), wl.to_f64(K0[0, h]), wl.to_f64(V0[0, h]))
        Lr, zr = orc.state_absorb(Lr, zr, wl.to_f64(Kev[0, h, :n_ev]), wl.to_f64(Vev[0, h, :n_ev]))
        assert rel_l2(L[h], Lr) <= 1e-6 and rel_l2(z[h], zr) <= 1e-6, (h, rel_l2(L[h], Lr), rel_l2(z[h], zr))
    ref = torch.empty_like(planes)
    hf.hf_state_planes(cfg, st_out, ref)
    torch.cuda.synchronize()
    assert torch.equal(pl_out, ref)
