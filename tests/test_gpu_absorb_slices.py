"""Rotated and ELU + 1 keys are absorbed in slices of one or more runs of 320 tokens: the rounding of the sums does not grow with
the runs of a slice, and the state is the oracle's."""
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import rel_l2, split_state

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# the longest slices: 19 runs (as many heads as compute units), four, two and a short one
@pytest.mark.parametrize("heads,n", [(256, 6000), (40, 10800), (13, 6401)])
@pytest.mark.parametrize("phi,rope", [(hf.HF_PHI_ELU1, False), (hf.HF_PHI_RELU, True), (hf.HF_PHI_ELU1, True)])
def test_sums_of_longer_slices(heads, n, phi, rope):
    """Against 64 bits, on keys whose features are exact in bf16 (multiples of 1/64 below one, turned by right angles): what is
    left is the rounding of fp32 sums of positive terms.  N additions of a growing sum, each off by 2^-23.5 / sqrt(12) of it,
    make sqrt(N / 3) of that: 0.9e-7 for the 20 products of a run and 19 runs, 2.7e-7 for 375 in a row.  Bound 2e-7."""
    g = torch.Generator().manual_seed(5)
    K = (torch.randint(0, 64, (1, 2, n, 128), generator=g) / 64).bfloat16()
    V = torch.rand((1, 2, n, 128), generator=g).bfloat16()
    cfg = hf.make_config(1, heads, 128, "bf16", 64, 64, 0.5, phi=phi)
    turn = torch.arange(n)[:, None] % 4 + torch.zeros((1, 64), dtype=torch.int64)
    cos, sin = (torch.tensor(t)[turn].contiguous() for t in ((1.0, 0.0, -1.0, 0.0), (0.0, 1.0, 0.0, -1.0))) if rope else (None, None)
    k, v = (t.repeat(1, -(-heads // 2), 1, 1)[:, :heads].contiguous().to(DEV) for t in (K, V))
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    ws = torch.empty(hf.hf_absorb_workspace_bytes(cfg, n), dtype=torch.uint8, device=DEV)
    hf.hf_absorb_evicted(cfg, st, k, v, *(None if t is None else t.to(DEV) for t in (cos, sin)), workspace=ws)
    torch.cuda.synchronize()
    L, z = split_state(st, heads, 128)
    tabs = tuple(None if t is None else wl.to_f64(t) for t in (cos, sin))
    for h in (0, 1, heads - 1):
        Lr, zr = orc.state_absorb(*orc.state_zero(128), wl.to_f64(K[0, h % 2]), wl.to_f64(V[0, h % 2]), phi, *tabs)
        assert rel_l2(L[h], Lr) <= 2e-7 and rel_l2(z[h], zr) <= 2e-7, (h, rel_l2(L[h], Lr))


@pytest.mark.parametrize("heads,n", [(13, 6401), (40, 2300), (2, 321)])
@pytest.mark.parametrize("phi,rope", [(hf.HF_PHI_ELU1, False), (hf.HF_PHI_RELU, True), (hf.HF_PHI_ELU1, True)])
def test_longer_slices_against_the_oracle(heads, n, phi, rope):
    """A feature rounded to bf16 is off by 2^-9 of itself at most; of values of either sign, so is the sum (2.0e-3).  z is not
    rounded."""
    K, V = (wl.randn((1, 2, n, 128), 96_000 + i, 1.0, torch.bfloat16) for i in range(2))
    cfg = hf.make_config(1, heads, 128, "bf16", 64, 64, 0.5, phi=phi)
    cos, sin = wl.rope_tables(n, 128, first_position=3.0) if rope else (None, None)
    k, v = (t.repeat(1, -(-heads // 2), 1, 1)[:, :heads].contiguous().to(DEV) for t in (K, V))
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    ws = torch.empty(hf.hf_absorb_workspace_bytes(cfg, n), dtype=torch.uint8, device=DEV)
    hf.hf_absorb_evicted(cfg, st, k, v, *(None if t is None else t.to(DEV) for t in (cos, sin)), workspace=ws)
    torch.cuda.synchronize()
    L, z = split_state(st, heads, 128)
    tabs = tuple(None if t is None else wl.to_f64(t) for t in (cos, sin))
    for h in (0, 1, heads - 1):
        Lr, zr = orc.state_absorb(*orc.state_zero(128), wl.to_f64(K[0, h % 2]), wl.to_f64(V[0, h % 2]), phi, *tabs)
        assert rel_l2(L[h], Lr) <= 2.5e-3 and rel_l2(z[h], zr) <= 1e-6, (h, rel_l2(L[h], Lr), rel_l2(z[h], zr))
