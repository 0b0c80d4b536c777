"""fp32-arithmetic gradients from workspaces with room for stored scores and from the least that a call takes: what the one way is
held to holds for the other."""
import pytest
import torch

import paper_2604_10103_amd as hf
import workloads as wl
from parity import rel_l2

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
NAN, INF = float("nan"), float("inf")


BAD = [("K", NAN), ("K", INF), ("K", -INF), ("V", NAN), ("V", INF), ("Q", NAN), ("Q", INF), ("dO", NAN), ("dO", -INF)]


@pytest.mark.parametrize("which,bad", BAD)
@pytest.mark.parametrize("dtype,d,bq,bkv", [("f32", 128, 64, 64), ("f32", 64, 48, 40), ("f32", 128, 16, 16), ("bf16", 64, 64, 32)])
def test_what_is_not_finite_reaches_as_far(which, bad, dtype, d, bq, bkv):
    """One element of one row is bad.  The same gradients are not finite, and the others are the same numbers (5e-5 in fp32, two
    roundings to bf16 in bf16).  In particular a row without a finite sum of probabilities gives nothing to the values' gradients
    of the other keys on its list."""
    n_q, n_kv = 2 * bq + 5, 4 * bkv + 7
    cfg = hf.make_config(1, 2, d, dtype, bq, bkv, 0.5)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    T = {n: wl.randn((1, 2, r, d), 71_000 + i, 0.5, td).to(DEV) for i, (n, r) in enumerate((("Q", n_q), ("K", n_kv), ("V", n_kv), ("dO", n_q)))}
    T[which][:, :, bkv + 3 if which in "KV" else bq + 3, 5] = bad
    idx = torch.tensor([[0, 1], [1, 3], [2, 4]], dtype=torch.int32, device=DEV).expand(1, 2, 3, 2).contiguous()
    out = []
    for size in (hf.hf_bwd_workspace_bytes(cfg, n_q, n_kv), hf.hf_bwd_least_workspace_bytes(cfg, n_q, n_kv)):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device=DEV)
        grads = [torch.full_like(T[n], 7.0) for n in ("Q", "K", "V")]
        hf.hf_hybrid_attn_bwd(cfg, T["Q"], T["K"], T["V"], idx, None, T["dO"], *grads, ws)
        torch.cuda.synchronize()
        out.append(grads)
    for name, a, b in zip(("dQ", "dK", "dV"), *out):
        assert torch.equal(a.isfinite(), b.isfinite()), (name, (a.isfinite() != b.isfinite()).sum().item())
        f = a.isfinite()
        assert f.any() and rel_l2(wl.to_f64(a[f]), wl.to_f64(b[f])) <= (8e-3 if dtype == "bf16" else 5e-5), name


def _gradients(cfg, T, idx, st, room, n_q, n_kv):
    """Gradients from the least workspace and `room` bytes behind the lists' places, and what lies behind that room afterwards."""
    places = -(-cfg.batch * cfg.heads * -(-n_q // cfg.block_q) * -(-n_kv // cfg.block_kv) * 4 // 256) * 256
    least = hf.hf_bwd_least_workspace_bytes(cfg, n_q, n_kv)
    ws = torch.full((least + places + room + 4096,), 0xFF, dtype=torch.uint8, device=DEV)
    grads = [torch.full_like(T[n], 7.0) for n in ("Q", "K", "V")]
    hf.hf_hybrid_attn_bwd(cfg, T["Q"], T["K"], T["V"], idx, st, T["dO"], *grads, ws[:least + places + room], n_kv=n_kv)
    torch.cuda.synchronize()
    return grads, ws[least + places:least + places + room], ws[least + places + room:]


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("dtype,d,b", [("f32", 64, 32), ("f32", 128, 16), ("bf16", 64, 48)])
def test_heads_a_few_at_a_time(dtype, d, b, dense):
    """70 heads, in groups from 256 query-side workgroups on: the same bits whatever the room, nothing written behind it; with less the
    scores' place is left alone and the gradients are those within the rounding of fp32 sums (5e-5; bf16: two roundings)."""
    heads, n_q, n_kv = 70, 9 * b + 3, 13 * b + 5
    cfg = hf.make_config(2, heads // 2, d, dtype, b, b, 0.3, kv_capacity=n_kv + 9)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    T = {n: wl.randn((2, heads // 2, r, d), 73_000 + i, 0.7, td).to(DEV) for i, (n, r) in
         enumerate((("Q", n_q), ("K", n_kv + 9), ("V", n_kv + 9), ("dO", n_q)))}
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(hf.make_config(2, heads // 2, d, dtype, b, b, 0.3), st, T["Q"], T["dO"])
    k, t_m = hf.hf_select_k(cfg, n_kv), -(-n_q // b)
    idx = None
    if not dense:
        idx = torch.empty((2, heads // 2, t_m, k), dtype=torch.int32, device=DEV)
        hf.hf_block_select(cfg, T["Q"], T["K"], idx, None, torch.empty(hf.hf_workspace_bytes(cfg, n_q, n_kv), dtype=torch.uint8, device=DEV),
                           n_kv=n_kv)
    tile = -(-b // 16)
    head = t_m * (-(-n_kv // b) if dense else k) * tile * tile * 2048
    per_head = t_m * (-(-b // 32) if -(-b // 32) * 96 <= 4 * b else tile)   # query-side workgroups
    few = -(-256 // per_head)
    few = next(n for n in range(few, heads) if heads // -(-heads // n) * per_head >= 256)   # (groups of a size)
    want, room, _ = _gradients(cfg, T, idx, st, heads * head, n_q, n_kv)
    assert not (room == 0xFF).all()
    for n in (heads - 1, few):
        got, room, behind = _gradients(cfg, T, idx, st, n * head + head // 2, n_q, n_kv)
        assert not (room == 0xFF).all() and (behind == 0xFF).all()
        assert all(torch.equal(a, r) for a, r in zip(got, want)), n
    for n in (0, 1, few // 2):
        got, room, behind = _gradients(cfg, T, idx, st, n * head, n_q, n_kv)
        assert (room == 0xFF).all() and (behind == 0xFF).all()
        for a, r in zip(got, want):
            assert rel_l2(wl.to_f64(a), wl.to_f64(r)) <= (8e-3 if dtype == "bf16" else 5e-5), n


@pytest.mark.parametrize("heads,n_kv", [(1, (1 << 23) + 100), (4, (1 << 21) + 100)])
def test_more_key_blocks_than_a_launch_of_eight_wavefronts_has_workgroups(heads, n_kv):
    """2^23 workgroups of 512 threads are 2^32 threads, more than a launch may have; of 256 they fit.  One query, one key on its list:
    P = 1, so that dV of that key is dO and all else is zero."""
    cfg = hf.make_config(1, heads, 64, "f32", 1, 1, 0.5)
    Q, dO = (torch.randn((1, heads, 1, 64), device=DEV, generator=torch.Generator(DEV).manual_seed(s)) for s in (1, 2))
    K = torch.ones((1, heads, n_kv, 64), device=DEV)
    idx = torch.full((1, heads, 1, 1), n_kv - 3, dtype=torch.int32, device=DEV)
    ws = torch.empty(hf.hf_bwd_workspace_bytes(cfg, 1, n_kv), dtype=torch.uint8, device=DEV)
    dQ, dK, dV = torch.full_like(Q, 7.0), torch.full_like(K, 7.0), torch.full_like(K, 7.0)
    hf.hf_hybrid_attn_bwd(cfg, Q, K, K, idx, None, dO, dQ, dK, dV, ws)
    torch.cuda.synchronize()
    assert dQ.abs().max() <= 1e-6 and dK.abs().max() <= 1e-5
    assert torch.allclose(dV[:, :, n_kv - 3], dO[:, :, 0], rtol=1e-6) and (dV[:, :, :n_kv - 3] == 0).all() and (dV[:, :, n_kv - 2:] == 0).all()
