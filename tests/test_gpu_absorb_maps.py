"""Keys as they are, rotated or under ELU + 1 with a workspace (one launch, quadrants or halves of the state): counts of tokens around a
tile and a pair of tiles, one slice (which exchanges nothing) and many, heads in one round of the chip and in several; the planes
are those of the state.  Against the fp64 oracle."""
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import rel_l2, split_state

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("heads,n", [(1, 1), (2, 31), (3, 33), (1, 64), (2, 65), (130, 127), (300, 129), (1, 9000), (34, 3000), (64, 1290)])
@pytest.mark.parametrize("phi,rope", [(hf.HF_PHI_RELU, False), (hf.HF_PHI_ELU1, False), (hf.HF_PHI_RELU, True), (hf.HF_PHI_ELU1, True)])
def test_maps(heads, n, phi, rope):
    """A feature rounded to bf16 is off by 2^-9 of itself at most, 2^-9 / sqrt(3) in the mean, of either sign; z is not rounded.
    Twice, on a state that holds something: the second call finds the workspace as the first left it."""
    two = min(heads, 2)
    K, V = (wl.randn((1, two, n, 128), 71_000 + i, 1.0, torch.bfloat16) for i in range(2))
    cfg = hf.make_config(1, heads, 128, "bf16", 64, 64, 0.5, phi=phi)
    cos, sin = wl.rope_tables(n, 128, first_position=3.0) if rope else (None, None)
    k, v = (t.repeat(1, -(-heads // two), 1, 1)[:, :heads].contiguous().to(DEV) for t in (K, V))
    cd, sd = (None if t is None else t.to(DEV) for t in (cos, sin))
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    ws = torch.empty(hf.hf_absorb_workspace_bytes(cfg, n), dtype=torch.uint8, device=DEV)
    planes, again = (torch.empty(hf.hf_state_planes_bytes(cfg), dtype=torch.uint8, device=DEV) for _ in range(2))
    hf.hf_absorb_evicted(cfg, st, k, v, cd, sd, workspace=ws)
    hf.hf_absorb_evicted_planes(cfg, st, k, v, planes, cd, sd, workspace=ws)
    hf.hf_state_planes(cfg, st, again)
    torch.cuda.synchronize()
    assert torch.equal(planes, again)
    L, z = split_state(st, heads, 128)
    tabs = tuple(None if t is None else wl.to_f64(t) for t in (cos, sin))
    for h in sorted({0, min(1, heads - 1), heads - 1}):
        Lr, zr = orc.state_absorb(*orc.state_zero(128), wl.to_f64(K[0, h % two]), wl.to_f64(V[0, h % two]), phi, *tabs)
        assert rel_l2(L[h], 2 * Lr) <= 2.5e-3 and rel_l2(z[h], 2 * zr) <= 1e-6, (h, rel_l2(L[h], 2 * Lr), rel_l2(z[h], 2 * zr))
