"""hf_rope_append_keys with two heads a workgroup (with tables, blocks of at least 8192 values, more than 2048 workgroups of one head; of
at least 16384, more than 1024) and with one in as long launches: an odd number of heads, a block that holds cached tokens too, with and
without tables; the same keys and means as head by head."""
import pytest
import torch

import paper_2604_10103_amd as hf
import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("values,blocks", [(None, 63), (8192, 56), (8192, 55), (16384, 28), (16384, 27)])
def test_two_heads_a_workgroup(dtype, d, rope, values, blocks):
    H, first, b = 37, 41, 16 if values is None else values // d
    n_new = 1000 if values is None else b * blocks - first - 5
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    n_kv = first + n_new
    K, X = (wl.randn((1, H, n, d), 73_000 + i, 1.0, td).to(DEV) for i, n in enumerate((n_kv, n_new)))
    cos, sin = (t.to(DEV) for t in wl.rope_tables(n_new, d, first_position=2.0)) if rope else (None, None)
    cfg, one = (hf.make_config(1, h, d, dtype, b, b, 0.5) for h in (H, 1))
    n_blocks = -(-n_kv // b) - first // b
    assert (H * n_blocks > (1024 if values == 16384 else 2048)) == (blocks not in (55, 27))
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
