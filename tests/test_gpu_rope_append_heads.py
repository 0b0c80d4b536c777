"""hf_rope_append_keys with two heads a workgroup (more than 2048 workgroups of one): an odd number of heads, a block that holds cached
tokens too, with and without tables; the same keys and means as head by head, where a workgroup has one."""
import pytest
import torch

import paper_2604_10103_amd as hf
import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("rope", [False, True])
def test_two_heads_a_workgroup(dtype, d, rope):
    H, b, first, n_new = 37, 16, 41, 1000
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    n_kv = first + n_new
    K, X = (wl.randn((1, H, n, d), 73_000 + i, 1.0, td).to(DEV) for i, n in enumerate((n_kv, n_new)))
    cos, sin = (t.to(DEV) for t in wl.rope_tables(n_new, d, first_position=2.0)) if rope else (None, None)
    cfg, one = (hf.make_config(1, h, d, dtype, b, b, 0.5) for h in (H, 1))
    assert H * -(-n_new // b) > 2048
    pooled = torch.full((hf.hf_pooled_keys_bytes(cfg, n_kv) // 4,), -1.0, device=DEV)
    W = K.clone()
    hf.hf_rope_append_keys(cfg, X, cos, sin, W, first, pooled.view(torch.uint8))
    t_n = -(-n_kv // b)
    for h in (0, 1, H - 2, H - 1):
        w, p = K[:, h:h + 1].clone(), torch.full((hf.hf_pooled_keys_bytes(one, n_kv) // 4,), -1.0, device=DEV)
        hf.hf_rope_append_keys(one, X[:, h:h + 1].contiguous(), cos, sin, w, first, p.view(torch.uint8))
        torch.cuda.synchronize()
        assert torch.equal(W[:, h:h + 1], w)
        assert torch.equal(pooled[h * t_n * d:(h + 1) * t_n * d], p[:t_n * d])
