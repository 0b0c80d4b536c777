"""Steps of small fp32 rings select in their attention workgroups: windows of up to 64 blocks by every wavefront for itself, longer
ones together, both by the comparisons that the selection of its own makes, equal scores by index."""
import pytest
import torch

import paper_2604_10103_amd as hf
import workloads as wl
from parity import rel_l2

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("ties", [False, True])
# blocks: one, two, a wavefront's lanes but one, all of them, one more; ragged last blocks; blocks longer than 32 rows; head_dim 128
@pytest.mark.parametrize("d,block,slots,chunk", [(64, 16, 1, 16), (64, 16, 2, 13), (64, 16, 7, 143), (64, 16, 8, 128), (64, 16, 5, 207),
                                                 (64, 32, 4, 70), (64, 48, 4, 60), (128, 16, 8, 127), (128, 16, 5, 206)])
def test_lists_of_a_step_are_the_selections(d, block, slots, chunk, ties):
    """The list is the same, bit for bit, and the output that of the separate calls but for the order of fp32 sums (1e-5)."""
    heads, n_kv = 3, slots * chunk
    cfg = hf.make_config(1, heads, d, "f32", block, block, 0.3, kv_capacity=n_kv)
    Q, K, V = (wl.randn((1, heads, n, d), 61_000 + i, 1.0, torch.float32).to(DEV) for i, n in enumerate((chunk, n_kv, n_kv)))
    if ties:   # whole blocks alike: every score occurs several times
        K = K[:, :, :block].repeat(1, 1, -(-n_kv // block), 1)[:, :, :n_kv].contiguous()
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, K, V)
    ring = hf.make_ring(0, chunk)
    ring.n_filled, ring.cur_slot, ring.next_slot, ring.absorbed_ahead = slots, slots - 1, 0, 1
    ws = torch.empty(max(hf.hf_workspace_bytes(cfg, chunk, n_kv), 256), dtype=torch.uint8, device=DEV)
    k = hf.hf_select_k(cfg, n_kv)
    shape = (1, heads, -(-chunk // block), k)
    idx, ref = (torch.full(shape, -1, dtype=torch.int32, device=DEV) for _ in range(2))
    O, Or = torch.empty_like(Q), torch.empty_like(Q)
    for step in range(2):   # the first pools the window's blocks, the second those of its chunk
        hf.hf_ring_step(cfg, ring, Q, K, V, step, idx, st, O, ws)
        torch.cuda.synchronize()
        hf.hf_block_select(cfg, Q, K, ref, None, torch.empty_like(ws), n_kv=n_kv)
        hf.hf_hybrid_attn_fwd(cfg, Q, K, V, ref, st, Or, torch.empty_like(ws), n_kv=n_kv)
        torch.cuda.synchronize()
        assert torch.equal(idx, ref)
        assert rel_l2(wl.to_f64(O), wl.to_f64(Or)) <= 1e-5
        idx.fill_(-1)
