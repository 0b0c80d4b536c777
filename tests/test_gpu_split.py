"""fp32 attention in bf16 products of values split in three (launches of more than 128 blocks of 64 rows): one, two and four
groups of wavefronts at both head sizes, ragged rows and keys, empty parts of blocks, lists that the groups do not divide, the
history term, the statistics the backward pass takes; NaN, infinities and the type's lowest value among the keys."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2604_10103_amd as hf
import workloads as wl
from parity import F32_REL_L2, max_abs, oracle_state, rel_l2

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
NAN, INF, LOWEST = float("nan"), float("inf"), torch.finfo(torch.float32).min


def _tensors(heads, n, d, seed, gain=1.0):
    """Three heads repeated: what the oracle has to follow."""
    return [(wl.randn((1, 3, m, d), 71_000 + seed + i, gain, torch.float32)).repeat(1, heads // 3, 1, 1) for i, m in enumerate(n)]


def _attend(cfg, Q, K, V, idx, st=None, tab=(None, None)):
    O = torch.full_like(Q, 7.0)
    ws = torch.empty(max(hf.hf_workspace_bytes(cfg, Q.shape[2], K.shape[2]), 256), dtype=torch.uint8, device=DEV)
    hf.hf_hybrid_attn_fwd(cfg, Q, K, V, idx, st, O, ws, *tab)
    torch.cuda.synchronize()
    return O


# heads, head_dim, block_q, block_kv, n_q, n_kv, keep (None: dense); the groups follow the blocks of 64 rows and the list's keys
SHAPES = [
    (66, 128, 64, 64, 65, 100, 1.0), (45, 128, 128, 32, 130, 257, 0.5), (129, 128, 64, 96, 1, 96 * 3 + 1, 0.5),
    (150, 128, 64, 32, 129, 33, 1.0), (300, 128, 64, 64, 70, 300, None), (390, 128, 64, 64, 100, 200, 0.5),
    (270, 128, 128, 64, 200, 130, 0.4), (66, 64, 64, 64, 65, 100, 1.0), (45, 64, 192, 32, 200, 300, 0.3),
    (390, 64, 64, 96, 100, 200, None), (270, 64, 64, 32, 193, 65, 0.4),
    # (129 to 256 blocks and more than 320 keys: four groups; up to 512 two; up to 768 by 256 keys; 1025 to 1664 by 128 keys)
    (66, 128, 64, 64, 65, 400, 1.0), (45, 128, 128, 32, 130, 700, 0.5), (129, 128, 64, 96, 1, 96 * 8 + 1, 0.5), (66, 128, 64, 64, 65, 321, None),
    (66, 128, 64, 64, 65, 320, None), (300, 128, 64, 64, 70, 200, 0.6), (270, 128, 128, 64, 200, 300, 0.6), (300, 64, 64, 64, 70, 200, 0.6),
    (300, 64, 64, 64, 70, 300, None),
    # (smaller launches: fp32 products)
    (90, 128, 64, 64, 33, 300, 0.4), (201, 128, 32, 32, 40, 100, 0.5), (90, 64, 64, 32, 40, 200, 0.5), (201, 64, 32, 64, 33, 150, None),
]


@pytest.mark.parametrize("case", SHAPES, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("gain,phi,rope", [(1.0, hf.HF_PHI_RELU, False), (4.0, hf.HF_PHI_ELU1, True)])
def test_forward_and_gradients(case, gain, phi, rope):
    heads, d, bq, bkv, n_q, n_kv, keep = case
    cfg = hf.make_config(1, heads, d, "f32", bq, bkv, 1.0 if keep is None else keep, phi=phi)
    Q, K, V, dO, Ke, Ve = _tensors(heads, (n_q, n_kv, n_kv, n_q, 50, 50), d, 0, 0.5)
    Q = Q * gain
    tab = wl.rope_tables(n_q, d, first_position=9.0) if rope else (None, None)
    dtab = tuple(None if t is None else t.to(DEV) for t in tab)
    q, k, v, g = (t.to(DEV) for t in (Q, K, V, dO))
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, Ke.to(DEV), Ve.to(DEV))
    t_m, t_n, kk = -(-n_q // bq), -(-n_kv // bkv), hf.hf_select_k(cfg, n_kv)
    idx = torch.empty((1, heads, t_m, kk), dtype=torch.int32, device=DEV)
    ws = torch.empty(hf.hf_workspace_bytes(cfg, n_q, n_kv), dtype=torch.uint8, device=DEV)
    hf.hf_block_select(cfg, q, k, idx, None, ws)
    use = None if keep is None else idx
    O, O0 = _attend(cfg, q, k, v, use, st, dtab), _attend(cfg, q, k, v, use)
    dQ, dK, dV = (torch.full_like(t, NAN) for t in (q, k, v))
    bws = torch.empty(hf.hf_bwd_workspace_bytes(cfg, n_q, n_kv), dtype=torch.uint8, device=DEV)
    hf.hf_hybrid_attn_bwd(cfg, q, k, v, use, st, g, dQ, dK, dV, bws, *dtab)
    torch.cuda.synchronize()
    states = oracle_state([Ke[:, :3]], [Ve[:, :3]], d, phi)
    lists = idx.cpu().numpy() if keep is not None else np.tile(np.arange(t_n), (1, heads, t_m, 1))
    tabs = tuple(None if t is None else wl.to_f64(t) for t in tab)
    for h in (0, 1, heads - 1):
        a = [wl.to_f64(t[0, h]) for t in (Q, K, V, dO)]
        for got, state in ((O, states[h % 3]), (O0, None)):
            ref, *_ = orc.hybrid_attention(*a[:3], state, bq, bkv, lists.shape[-1], phi, *tabs, cfg.eps, cfg.z_scale,
                                           block_idx=lists[0, h])
            x = wl.to_f64(got[0, h])
            assert rel_l2(x, ref) <= F32_REL_L2 and max_abs(x, ref) <= 1e-4 * max(1.0, np.abs(ref).max()), (h, rel_l2(x, ref))
        dq, dqh, dk, dv = orc.hybrid_attention_bwd(*a[:3], states[h % 3], bq, bkv, lists[0, h], a[3], phi, *tabs, cfg.eps, cfg.z_scale)
        for name, got, ref in (("dQ", dQ, dq + dqh), ("dK", dK, dk), ("dV", dV, dv)):   # (bounds as in test_gpu_wide.py)
            x = wl.to_f64(got[0, h])
            assert rel_l2(x, ref) <= 5e-5 and max_abs(x, ref) <= 1e-4 * max(np.abs(ref).max(), 1e-2), (name, h, rel_l2(x, ref))


# three query blocks of 64 rows a head, lists of two KV blocks: two, four, two and one group; two and one; fp32 products
BAD = [(66, 128, 64), (66, 128, 192), (150, 128, 64), (300, 128, 64), (66, 64, 64), (390, 64, 64), (30, 128, 64), (30, 64, 64)]


def _bad_case(heads, d, bkv):
    b, n_kv = 64, bkv * 3 + 10
    cfg = hf.make_config(1, heads, d, "f32", b, bkv, 0.5)
    Q, K, V = (t.to(DEV) for t in _tensors(heads, (2 * b + 5, n_kv, n_kv), d, 20))
    idx = torch.tensor([[0, 3], [1, 2], [2, 3]], dtype=torch.int32, device=DEV).expand(1, heads, 3, 2).contiguous()
    return cfg, Q, K, V, idx


@pytest.mark.parametrize("heads,d,bkv", BAD)
@pytest.mark.parametrize("bad", [NAN, INF, LOWEST])
def test_an_unselected_block_is_not_read(heads, d, bkv, bad):
    cfg, Q, K, V, idx = _bad_case(heads, d, bkv)
    want = _attend(cfg, Q, K, V, idx)
    K[:, :, :bkv] = bad
    V[:, :, :bkv] = bad
    assert want.isfinite().all() and torch.equal(_attend(cfg, Q, K, V, idx)[:, :, 64:], want[:, :, 64:])


@pytest.mark.parametrize("heads,d,bkv", BAD)
def test_values_without_a_finite_remainder(heads, d, bkv):
    """A selected infinite value stays one; a key of an infinitely small score, or of the lowest finite one, has no weight."""
    cfg, Q, K, V, idx = _bad_case(heads, d, bkv)
    Q[..., 0] = Q[..., 0].abs() + 0.1
    n_kv = K.shape[2]
    for value in (-INF, LOWEST):
        K2 = K.clone()
        K2[:, :, n_kv - 1, 0] = value          # the last key of block 3: query blocks 0 and 2
        short, V2 = K2[:, :, :n_kv - 1].contiguous(), V[:, :, :n_kv - 1].contiguous()
        got, want = _attend(cfg, Q, K2, V, idx), _attend(cfg, Q, short, V2, idx)
        assert want.isfinite().all() and ((got - want).norm() / want.norm()).item() <= F32_REL_L2
    V[:, :, n_kv - 1, 3] = INF
    V[:, :, n_kv - 1, 40] = LOWEST
    O = _attend(cfg, Q, K, V, idx)
    assert (O[:, :, :64, 3] == INF).all() and (O[:, :, 128:, 3] == INF).all() and O[:, :, 64:128].isfinite().all()
    assert (O[:, :, :64, 40] < -1e30).all() and (O[:, :, 128:, 40] < -1e30).all()
    K[:, :, n_kv - 1, 0] = INF                 # a score of +infinity: no softmax
    assert _attend(cfg, Q, K, V, idx)[:, :, :64].isnan().all()


@pytest.mark.parametrize("heads,d,bkv", BAD)
def test_infinities_of_the_state(heads, d, bkv):
    """An infinite entry of the state (of an infinite value that was absorbed) is one of its feature's outputs, two of either
    sign make NaN there; the other features keep their bits.  phi = ELU + 1, which is positive."""
    cfg, Q, K, V, idx = _bad_case(heads, d, bkv)
    cfg.phi = hf.HF_PHI_ELU1
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, K, V)
    want = _attend(cfg, Q, K, V, idx, st)
    L = st[:heads * d * d].view(1, heads, d, d)
    L[:, :, 5, 3], L[:, :, 9, 40], L[:, :, 5, d - 1], L[:, :, d - 2, d - 1] = INF, -INF, INF, -INF
    O = _attend(cfg, Q, K, V, idx, st)
    same = [f for f in range(d) if f not in (3, 40, d - 1)]
    assert want.isfinite().all() and torch.equal(O[..., same], want[..., same])
    assert (O[..., 3] == INF).all() and (O[..., 40] == -INF).all() and O[..., d - 1].isnan().all()


@pytest.mark.parametrize("d", [128, 64])
def test_a_nan_does_not_make_a_call_serial(d):
    """Rows that are not finite are done again in tiles: about three times the time of a call without one, whatever the list's
    length (key after key it was 35 times).  The bound leaves a factor of three."""
    cfg = hf.make_config(1, 12, d, "f32", 64, 64, 1.0)
    Q, K, V = (t.to(DEV) for t in _tensors(12, (1560, 4096, 4096), d, 60))
    O = torch.empty_like(Q)

    def us():
        t = [torch.cuda.Event(enable_timing=True) for _ in range(5)]
        hf.hf_hybrid_attn_fwd(cfg, Q, K, V, None, None, O)
        for e in t:
            e.record()
            hf.hf_hybrid_attn_fwd(cfg, Q, K, V, None, None, O)
        torch.cuda.synchronize()
        return min(a.elapsed_time(b) for a, b in zip(t, t[1:]))

    clean = us()
    V[:, :, 77, 5] = NAN
    assert us() <= 9 * clean


def _low_bits(n, seed):
    """n values in [1, 1.25) whose parts behind the first eight bits are as large as they get: the upper bits random, then ones."""
    g = torch.Generator().manual_seed(seed)
    return (1.0 + torch.randint(0, 32, (n,), generator=g) / 128.0 + (2.0 ** 16 - 1) / 2.0 ** 23).float()


@pytest.mark.parametrize("heads,d,bkv", BAD)
def test_products_are_as_exact_as_one_rounding(heads, d, bkv):
    """A product of the window's two contractions or the history term is off by no more than 2^-24 of itself, half a unit of
    fp32's last place (what is left out of cut-off parts is up to 2^-21).  Single products, so that nothing averages out."""
    n_q, n_kv = 130, 64 if bkv == 64 else 2 * bkv
    scale = np.float32(16.0 / np.float32(1.4426950408889634))
    assert scale * np.float32(1.4426950408889634) == 16.0   # (the queries' low bits are not touched)
    cfg = hf.make_config(1, heads, d, "f32", 64, 64, 1.0, softmax_scale=float(scale))
    x = [_low_bits(heads * m, 40 + i).view(1, heads, m) for i, m in enumerate((n_q, 1, d, d))]
    Q, K, V = (torch.zeros((1, heads, m, d)) for m in (n_q, n_kv, n_kv))
    # scores: key 0 has one of zero, key 1 one product of about -17, the others none (2^-1000)
    Q[..., 0], K[:, :, 1, 0], K[:, :, 2:, 0], V[:, :, 1] = x[0], -x[1][..., 0], -60.0, 1.0
    got = wl.to_f64(_attend(cfg, Q.to(DEV), K.to(DEV), V.to(DEV), None))[0]
    s = 16.0 * wl.to_f64(x[0])[0] * wl.to_f64(x[1])[0]
    p = 2.0 ** -s
    # the score: left out 2^-24 of it, rounded 2^-20 (its last place is 2^-19); then the exponential, 1 + p, 1 / l and the product
    bound = np.log(2) * (s.max() * 2.0 ** -24 + 2.0 ** -20) + 5 * 2.0 ** -24
    assert np.abs(got / (p / (1 + p))[..., None] - 1).max() <= bound
    # values: one key of any weight w next to one without a value; O = w x, w from a feature whose value is one
    V[:, :, 1] = x[2]
    V[:, :, 1, 5] = 1.0
    K[:, :, 1, 0] = -x[1][..., 0] / 64.0
    got = wl.to_f64(_attend(cfg, Q.to(DEV), K.to(DEV), V.to(DEV), None))[0]
    want = got[..., 5:6] * wl.to_f64(V)[0, :, 1:2]
    assert np.abs(got / want - 1).max() <= 5 * 2.0 ** -24   # left out, rounded to fp32, scaled by 1 / l here and there
    # history: no value in the window, a state of one row, denominator one: O is the product
    st = torch.zeros(hf.hf_state_bytes(cfg) // 4)
    st[:heads * d * d].view(heads, d, d)[:, 0] = x[3][0]
    cfg.eps = 1.0
    got = wl.to_f64(_attend(cfg, Q.to(DEV), K.to(DEV), torch.zeros_like(V).to(DEV), None, st.to(DEV)))[0]
    want = wl.to_f64(x[0])[0][..., None] * wl.to_f64(x[3])[0][:, None]
    assert np.abs(got / want - 1).max() <= 2.01 * 2.0 ** -24


@pytest.mark.parametrize("bad", [NAN, INF])
@pytest.mark.parametrize("bq,bkv,n_kv", [(64, 32, 300), (128, 96, 96 * 3 + 10)])
def test_bf16_at_head_dim_64_beyond_small_launches(bq, bkv, n_kv, bad):
    """More than 64 blocks of 64 rows take the kernel that splits the probabilities: infinite values of selected keys stay
    infinite in their feature alone, unselected blocks are not read."""
    heads, n_q = 33, 2 * bq + 5
    cfg = hf.make_config(1, heads, 64, "bf16", bq, bkv, 0.5)
    Q, K, V = (t.bfloat16().to(DEV) for t in _tensors(heads, (n_q, n_kv, n_kv), 64, 40, 0.5))
    last = (n_kv - 1) // bkv
    idx = torch.tensor([[1, last], [last, 2], [1, 2]], dtype=torch.int32, device=DEV).expand(1, heads, 3, 2).contiguous()
    want = _attend(cfg, Q, K, V, idx)
    K[:, :, :bkv] = bad
    V[:, :, :bkv] = bad
    V[:, :, n_kv - 1, 3] = INF
    V[:, :, n_kv - 1, 40] = -INF
    O = _attend(cfg, Q, K, V, idx)
    same = [f for f in range(64) if f not in (3, 40)]
    assert want.isfinite().all() and torch.equal(O[..., same], want[..., same]) and torch.equal(O[:, :, 2 * bq:], want[:, :, 2 * bq:])
    assert (O[:, :, :2 * bq, 3] == INF).all() and (O[:, :, :2 * bq, 40] == -INF).all()


@pytest.mark.parametrize("dtype,d,heads,n_q", [("f32", 128, 9, 64), ("f32", 64, 9, 64), ("f32", 128, 7, 33), ("bf16", 64, 5, 64)])
def test_rows_that_do_not_exist_choose_no_kernel(dtype, d, heads, n_q):
    """A query block far longer than the queries has the kernel, and so the bits, of a block they fill."""
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    Q, K, V, Ke = (wl.randn((1, heads, n, d), 72_000 + i, 0.5, td).to(DEV) for i, n in enumerate((n_q, 200, 200, 50)))
    cfg, long = (hf.make_config(1, heads, d, dtype, bq, 64, 1.0) for bq in (64, 1024))
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, Ke, Ke)
    assert torch.equal(_attend(cfg, Q, K, V, None, st), _attend(long, Q, K, V, None, st))


# fp32 products with 32 rows a workgroup: 129 to 256 of them with lists of more than 192 keys, more than 384 of any; sixteen rows in
# all others (heads, head_dim, block_q, block_kv, n_q, n_kv, keep)
SHAPES_32 = [
    (90, 128, 64, 64, 33, 300, None), (75, 128, 32, 32, 40, 300, 0.8), (126, 64, 64, 32, 40, 300, 0.8), (66, 64, 32, 64, 50, 257, None),
    (195, 128, 32, 32, 33, 100, 0.5), (129, 64, 96, 64, 97, 200, 0.4), (150, 128, 32, 64, 40, 300, 0.5),
]


@pytest.mark.parametrize("case", SHAPES_32, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("gain,phi,rope", [(1.0, hf.HF_PHI_RELU, False), (4.0, hf.HF_PHI_ELU1, True)])
def test_fp32_products_at_either_number_of_rows(case, gain, phi, rope):
    test_forward_and_gradients(case, gain, phi, rope)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("bad", [NAN, INF, LOWEST])
def test_what_is_not_finite_in_32_rows_a_workgroup(d, bad):
    """Block 0 is selected by nobody, the infinite value of the last key by query blocks 0 and 2."""
    heads, b, n_kv = 30, 64, 64 * 4 + 10   # 150 workgroups of 32 rows, 202 keys and more a list
    cfg = hf.make_config(1, heads, d, "f32", b, b, 0.8)
    Q, K, V = (t.to(DEV) for t in _tensors(heads, (2 * b + 5, n_kv, n_kv), d, 30))
    idx = torch.tensor([[1, 2, 3, 4], [1, 2, 3, 3], [1, 2, 3, 4]], dtype=torch.int32, device=DEV).expand(1, heads, 3, 4).contiguous()
    want = _attend(cfg, Q, K, V, idx)
    K[:, :, :64], V[:, :, :64], V[:, :, n_kv - 1, 3] = bad, bad, INF
    O = _attend(cfg, Q, K, V, idx)
    same = [f for f in range(d) if f != 3]
    assert want.isfinite().all() and torch.equal(O[..., same], want[..., same]) and torch.equal(O[:, :, 64:128], want[:, :, 64:128])
    assert (O[:, :, :64, 3] == INF).all() and (O[:, :, 128:, 3] == INF).all()


@pytest.mark.parametrize("heads,d,bkv", BAD)
def test_small_values_keep_their_bits(heads, d, bkv):
    """Values around 2^-100 and below have parts under bf16's smallest.  Powers of two change no rounding above fp32's smallest
    normal value, so that outputs are those of the values times 2^s, up to fp32 sums in two orders (6e-7 at most)."""
    cfg, Q, K, V, idx = _bad_case(heads, d, bkv)
    want = _attend(cfg, Q, K, V, idx).double()
    for s in (90, 104, 110, 120):
        got = _attend(cfg, Q, K, V * 2.0 ** -s, idx).double() * 2.0 ** s
        assert ((got - want).norm() / want.norm()).item() <= 1e-6, s
    W = V.clone()
    W[..., 5] *= 2.0 ** -118                    # one feature of a row is enough
    got = _attend(cfg, Q, K, W, idx).double()[..., 5] * 2.0 ** 118
    assert ((got - want[..., 5]).norm() / want[..., 5].norm()).item() <= 1e-6
    W[..., 5] = 0.0
    assert (_attend(cfg, Q, K, W, idx)[..., 5] == 0).all()


@pytest.mark.parametrize("dtype,d", [("f32", 128), ("f32", 64), ("bf16", 64)])
def test_a_head_alone_and_among_many(dtype, d):
    """Launch sizes choose kernels: a head's lists and scores keep their bits, its output differs by rounding (of fp32 products and
    sums; in bf16 of the stored value, whose last bit is 2^-8 of it)."""
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    Q, K, V, Ke = (wl.randn((1, 1, n, d), 74_000 + i, 0.5, td).to(DEV) for i, n in enumerate((130, 330, 330, 50)))
    outs = []
    for heads in (1, 30, 47, 80, 200, 300, 420):
        cfg = hf.make_config(1, heads, d, dtype, 64, 64, 0.7)
        q, k, v, e = (t.expand(1, heads, -1, -1).contiguous() for t in (Q, K, V, Ke))
        st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
        hf.hf_state_init(cfg, st)
        hf.hf_absorb_evicted(cfg, st, e, e)
        idx = torch.empty((1, heads, 3, hf.hf_select_k(cfg, 330)), dtype=torch.int32, device=DEV)
        scores = torch.empty((1, heads, 3, 6), dtype=torch.float32, device=DEV)
        hf.hf_block_select(cfg, q, k, idx, scores, torch.empty(hf.hf_workspace_bytes(cfg, 130, 330), dtype=torch.uint8, device=DEV))
        O = _attend(cfg, q, k, v, idx, st)
        assert (O == O[:, :1]).all() and (idx == idx[:, :1]).all() and (scores == scores[:, :1]).all()
        outs.append((idx[:, 0].clone(), scores[:, 0].clone(), O[:, 0].double()))
    for idx, scores, O in outs[1:]:
        assert torch.equal(idx, outs[0][0]) and torch.equal(scores, outs[0][1])
        assert ((O - outs[0][2]).norm() / O.norm()).item() <= (2e-6 if dtype == "f32" else 1e-3)


# four groups of one value block, two of two at head_dim 128, two of one at 64, ragged rows: what keeps a query's features
@pytest.mark.parametrize("case", [(66, 128, 64, 64, 65, 400, 1.0), (300, 128, 64, 64, 70, 200, 0.6), (300, 64, 64, 64, 70, 200, 0.6)],
                         ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("phi", [hf.HF_PHI_RELU, hf.HF_PHI_ELU1])
def test_history_without_rotation(case, phi):
    test_forward_and_gradients(case, 4.0, phi, False)


@pytest.mark.parametrize("heads,d,bkv", BAD)
def test_sums_of_the_history_term(heads, d, bkv):
    """History term alone (no value in the window), positive terms.  A rounding at full size is off by 2.5e-8 of the result (2^-24
    over a mantissa of 1 to 2); the products' sum, the normaliser's, its reciprocal and the scaling are about ten of them: 8.0e-8.
    With the normaliser's 64 or 32 terms of a lane in one chain, or 32 products in one, it was 9.2e-8 and 11.3e-8."""
    cfg = hf.make_config(1, heads, d, "f32", 64, 64, 1.0)
    g = torch.Generator().manual_seed(heads)
    Q, K = torch.randn(1, heads, 130, d, generator=g), torch.zeros(1, heads, 64 if bkv == 64 else 2 * bkv, d)
    st = torch.rand(hf.hf_state_bytes(cfg) // 4, generator=g) + 0.5
    L, z = st[:heads * d * d].view(heads, d, d).double(), st[heads * d * d:heads * d * (d + 1)].view(heads, 1, d).double()
    phi = Q[0].double().clamp(min=0)
    want = (phi @ L) / (cfg.z_scale * (phi * z).sum(-1, keepdim=True) + cfg.eps)
    got = _attend(cfg, Q.to(DEV), K.to(DEV), K.to(DEV), None, st.to(DEV))[0].cpu().double()
    assert ((got - want).norm() / want.norm()).item() <= 8.4e-8
