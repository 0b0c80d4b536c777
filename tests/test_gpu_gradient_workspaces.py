"""fp32-arithmetic gradients from workspaces with room for stored scores and from the least that a call takes: what the one way is
held to holds for the other."""
import re

import pytest
import torch

import paper_2604_10103_amd as hf
import workloads as wl
from parity import rel_l2

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
NAN, INF = float("nan"), float("inf")


def least_bytes(cfg, n_q, n_kv):
    """The size that a call cannot do without, from its refusal."""
    t = torch.empty(256, dtype=torch.uint8, device=DEV)
    td = torch.bfloat16 if cfg.dtype == hf.HF_BF16 else torch.float32
    q, k, v, g, dq, dk, dv = (torch.empty((cfg.batch, cfg.heads, n, cfg.head_dim), dtype=td, device=DEV)
                              for n in (n_q, n_kv, n_kv, n_q, n_q, n_kv, n_kv))
    with pytest.raises(Exception, match="workspace of") as e:
        hf.hf_hybrid_attn_bwd(cfg, q, k, v, None, None, g, dq, dk, dv, t)
    return int(re.search(r"workspace of (\d+) bytes needed", str(e.value)).group(1))


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
    for size in (hf.hf_bwd_workspace_bytes(cfg, n_q, n_kv), least_bytes(cfg, n_q, n_kv)):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device=DEV)
        grads = [torch.full_like(T[n], 7.0) for n in ("Q", "K", "V")]
        hf.hf_hybrid_attn_bwd(cfg, T["Q"], T["K"], T["V"], idx, None, T["dO"], *grads, ws)
        torch.cuda.synchronize()
        out.append(grads)
    for name, a, b in zip(("dQ", "dK", "dV"), *out):
        assert torch.equal(a.isfinite(), b.isfinite()), (name, (a.isfinite() != b.isfinite()).sum().item())
        f = a.isfinite()
        assert f.any() and rel_l2(wl.to_f64(a[f]), wl.to_f64(b[f])) <= (8e-3 if dtype == "bf16" else 5e-5), name
