"""Evicted chunks beside the attention of small launches: up to which length two workgroups a head absorb them without an exchange
(the workspace is not written then), and that their sums are, bit for bit, those of slices that meet in the workspace."""
import pytest
import torch

import paper_2604_10103_amd as hf
import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _step(heads, block, n_q, n_ev, seed=51_000):
    """(new state, its planes, the workspace behind the counters) of a step; head h's inputs depend on h alone."""
    cfg = hf.make_config(1, heads, 128, "bf16", block, block, 0.5)
    head = lambda i, n: wl.randn((1, 3, n, 128), seed + i, 1.0, torch.bfloat16).repeat(1, -(-heads // 3), 1, 1)[:, :heads].contiguous().to(DEV)
    Q, K, V, Ke, Ve = (head(i, n) for i, n in enumerate((n_q, 2 * n_q, 2 * n_q, n_ev, n_ev)))
    L, z = (wl.randn((3, n), seed + 10 + i, 30.0, torch.float32).repeat(-(-heads // 3), 1)[:heads] for i, n in enumerate((128 * 128, 128)))
    st = torch.cat([L.reshape(-1), z.abs().reshape(-1)]).to(DEV)
    planes = torch.empty(hf.hf_state_planes_bytes(cfg), dtype=torch.uint8, device=DEV)
    hf.hf_state_planes(cfg, st, planes)
    pooled = torch.empty(hf.hf_pooled_keys_bytes(cfg, 2 * n_q), dtype=torch.uint8, device=DEV)
    hf.hf_pool_keys(cfg, K, pooled)
    idx = torch.empty((1, heads, -(-n_q // block), hf.hf_select_k(cfg, 2 * n_q)), dtype=torch.int32, device=DEV)
    ws = torch.full((hf.hf_step_workspace_bytes(cfg, n_q, n_ev),), 0xFF, dtype=torch.uint8, device=DEV)
    O, st_out, pl_out = torch.empty_like(Q), torch.empty_like(st), torch.empty_like(planes)
    hf.hf_step_fwd(cfg, Q, K, V, pooled, st, planes, O, idx, Ke, Ve, st_out, pl_out, ws)
    torch.cuda.synchronize()
    return st_out, pl_out, ws[-(-heads * 8 // 256) * 256:]


# longest chunk of two workgroups a head and shortest of slices; blocks of 128 have the shorter limit where heads are few
@pytest.mark.parametrize("heads,block,longest", [(3, 64, 1024), (3, 128, 839), (12, 128, 884), (40, 128, 1024)])
def test_which_chunks_meet_in_the_workspace(heads, block, longest):
    assert (_step(heads, block, 130, longest)[2] == 0xFF).all()
    assert not (_step(heads, block, 130, longest + 1)[2] == 0xFF).all()


# many heads: one group of wavefronts and as many slices a head
@pytest.mark.parametrize("block,n_q,many", [(64, 330, 102), (128, 200, 102)])
@pytest.mark.parametrize("n_ev", [1, 17, 256, 257, 511, 700, 767, 768])
def test_sums_are_those_of_slices(block, n_q, many, n_ev):
    few, few_planes, few_ws = _step(3, block, n_q, n_ev)
    st, planes, ws = _step(many, block, n_q, n_ev)
    assert (few_ws == 0xFF).all() and (n_ev <= 256 or not (ws == 0xFF).all())
    D = 128
    assert torch.equal(st[:3 * D * D], few[:3 * D * D]) and torch.equal(st[many * D * D:][:3 * D], few[3 * D * D:])
    assert torch.equal(planes[:few_planes.numel()], few_planes)
