"""NaN and infinities among the valid tokens reach the rows that select their block and no others, whatever parts of short
blocks and ends of lists the kernels pad their tiles with.  A call on poisoned inputs is compared bit for bit with the same
call on finite ones."""
import pytest
import torch

import paper_2604_10103_amd as hf
import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
NAN, INF = float("nan"), float("inf")


def _inputs(dtype, d, n_q, n_kv, seed):
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    mk = lambda n, s: wl.randn((1, 2, n, d), 61_000 + seed + s, 0.5, td).to(DEV)
    return mk(n_q, 0), mk(n_kv, 1), mk(n_kv, 2), mk(n_q, 3)


def _lists(rows):
    return torch.tensor(rows, dtype=torch.int32, device=DEV).expand(1, 2, len(rows), len(rows[0])).contiguous()


def _attend(cfg, Q, K, V, idx):
    O = torch.full_like(Q, 7.0)
    ws = torch.empty(max(hf.hf_workspace_bytes(cfg, Q.shape[2], K.shape[2]), 256), dtype=torch.uint8, device=DEV)
    hf.hf_hybrid_attn_fwd(cfg, Q, K, V, idx, None, O, ws)
    torch.cuda.synchronize()
    return O


# dtype, head_dim, block_q, block_kv, keys, list of a query block without block 0
FORWARD = {
    "mfma_groups": ("bf16", 128, 64, 32, 300, [2, 5, 8]),          # two groups of wavefronts, an odd number of tiles
    "mfma_groups_b128": ("bf16", 128, 128, 32, 300, [2, 5, 9]),
    "d64": ("bf16", 64, 64, 32, 300, [2, 5, 8]),
    "d64_short": ("bf16", 64, 128, 96, 96 * 3 + 10, [1, 2, 3]),    # the last block's parts 1 and 2 are empty
    "wide_f32": ("f32", 128, 48, 48, 48 * 3 + 10, [1, 2, 3]),      # fp32 arithmetic, 16-key tiles: likewise
    "wide_f32_d64": ("f32", 64, 20, 40, 40 * 3 + 5, [1, 3]),
    "wide_bf16": ("bf16", 128, 48, 40, 40 * 3 + 5, [1, 2, 3]),
    "wide_bf16_d64": ("bf16", 64, 40, 33, 33 * 3 + 10, [1, 2, 3]),
    "wide32_f32": ("f32", 128, 64, 64, 64 * 3 + 10, [1, 3]),
}


@pytest.mark.parametrize("case", FORWARD, ids=str)
@pytest.mark.parametrize("bad", [NAN, INF])
def test_an_unselected_block_is_not_read(case, bad):
    dtype, d, bq, bkv, n_kv, sel = FORWARD[case]
    n_q = 2 * bq + 5
    cfg = hf.make_config(1, 2, d, dtype, bq, bkv, 0.5)
    Q, K, V, _ = _inputs(dtype, d, n_q, n_kv, 0)
    idx = _lists([sel] * 3)
    want = _attend(cfg, Q, K, V, idx)
    K[:, :, :min(bkv, 32)] = bad
    V[:, :, :min(bkv, 32)] = bad
    assert want.isfinite().all() and torch.equal(_attend(cfg, Q, K, V, idx), want)


@pytest.mark.parametrize("heads,bq,bkv,n_kv,sel", [
    (180, 64, 32, 300, [2, 5, 8]), (100, 128, 32, 300, [2, 5, 9]),   # one group of wavefronts (540 and 300 workgroups)
    (2, 192, 64, 64 * 4 + 10, [1, 2, 4]), (2, 256, 48, 48 * 3 + 10, [1, 2, 3]),   # larger query blocks
])
@pytest.mark.parametrize("bad", [NAN, INF])
def test_an_unselected_block_is_not_read_by_the_other_bf16_kernels(heads, bq, bkv, n_kv, sel, bad):
    n_q = 2 * bq + 5
    cfg = hf.make_config(1, heads, 128, "bf16", bq, bkv, 0.5)
    Q, K, V, _ = (t.repeat(1, heads // 2, 1, 1) for t in _inputs("bf16", 128, n_q, n_kv, 40))
    idx = _lists([sel] * 3).repeat(1, heads // 2, 1, 1)
    want = _attend(cfg, Q, K, V, idx)
    K[:, :, :bkv] = bad
    V[:, :, :bkv] = bad
    assert want.isfinite().all() and torch.equal(_attend(cfg, Q, K, V, idx), want)


@pytest.mark.parametrize("case", ["mfma_groups", "wide_f32", "wide_f32_d64", "wide_bf16", "wide_bf16_d64", "wide32_f32"])
def test_a_selected_infinity_stays_one(case):
    """In the last key of a short tile: nothing repeats that row with weight zero (zero times infinity is NaN)."""
    dtype, d, bq, bkv, n_kv, sel = FORWARD[case]
    n_q = 2 * bq + 5
    cfg = hf.make_config(1, 2, d, dtype, bq, bkv, 0.5)
    Q, K, V, _ = _inputs(dtype, d, n_q, n_kv, 10)
    last = (n_kv - 1) // bkv
    idx = _lists([[0, last], [1, last], [0, 1]])
    want = _attend(cfg, Q, K, V, idx)
    V[:, :, n_kv - 1] = INF
    O = _attend(cfg, Q, K, V, idx)
    assert (O[:, :, :2 * bq] == INF).all() and torch.equal(O[:, :, 2 * bq:], want[:, :, 2 * bq:])


@pytest.mark.parametrize("case,head_stride", [("d64", 0), ("d64_short", 400)])
def test_a_selected_infinity_at_head_dim_64(case, head_stride):
    """Probabilities are split into terms of which some are zero or negative: no NaN comes of an infinite value.  Features 3
    and 40 (one of either group of wavefronts) of two keys; the other features and the rows of other blocks keep their bits."""
    dtype, d, bq, bkv, n_kv, _ = FORWARD[case]
    n_q = 2 * bq + 5
    cfg = hf.make_config(1, 2, d, dtype, bq, bkv, 0.5, kv_capacity=head_stride)
    Q, K, V, Qh = _inputs(dtype, d, n_q, head_stride or n_kv, 30)
    st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
    hf.hf_state_init(cfg, st)
    hf.hf_absorb_evicted(cfg, st, Qh[:, :, :bq].contiguous(), Q[:, :, :bq].contiguous())
    last = (n_kv - 1) // bkv
    idx = _lists([[0, last], [last, 2], [0, 1]])

    def attend():
        O = torch.full_like(Q, 7.0)
        ws = torch.empty(max(hf.hf_workspace_bytes(cfg, n_q, n_kv), 256), dtype=torch.uint8, device=DEV)
        hf.hf_hybrid_attn_fwd(cfg, Q, K, V, idx, st, O, ws, n_kv=n_kv if head_stride else None)
        torch.cuda.synchronize()
        return O

    want = attend()
    V[:, :, n_kv - 1, 3] = INF
    V[:, :, n_kv - 1, 40] = -INF
    V[:, 1, 2 * bkv, 40] = INF       # block 2, head 1: rows of query block 1 meet both signs
    O = attend()
    same = [f for f in range(d) if f not in (3, 40)]
    assert torch.equal(O[..., same], want[..., same]) and torch.equal(O[:, :, 2 * bq:], want[:, :, 2 * bq:])
    assert (O[:, :, :2 * bq, 3] == INF).all()
    assert (O[:, 0, :2 * bq, 40] == -INF).all() and (O[:, 1, :bq, 40] == -INF).all() and O[:, 1, bq:2 * bq, 40].isnan().all()


@pytest.mark.parametrize("bad", [NAN, INF])
@pytest.mark.parametrize("dtype,d,b", [("f32", 128, 48), ("f32", 64, 40), ("f32", 64, 64), ("bf16", 128, 48), ("bf16", 64, 33), ("bf16", 128, 64)])
def test_gradients_of_other_blocks(dtype, d, b, bad):
    """Keys and values of block 0 and queries and output gradients of query block 0 are bad.  Query blocks 1 and 2 select
    neither, KV blocks 2 and 3 are selected by neither; the last block on either side is short, with empty parts behind it."""
    n_q, n_kv = 2 * b + 10, 3 * b + 10
    cfg = hf.make_config(1, 2, d, dtype, b, b, 0.5)
    Q, K, V, dO = _inputs(dtype, d, n_q, n_kv, 20)
    idx = _lists([[0, 1], [1, 3], [2, 3]])

    def gradients():
        out = [torch.full_like(t, 7.0) for t in (Q, K, V)]
        ws = torch.empty(hf.hf_bwd_workspace_bytes(cfg, n_q, n_kv), dtype=torch.uint8, device=DEV)
        hf.hf_hybrid_attn_bwd(cfg, Q, K, V, idx, None, dO, *out, ws)
        torch.cuda.synchronize()
        return [t[:, :, n:] for t, n in zip(out, (b, 2 * b, 2 * b))]

    want = gradients()
    K[:, :, :16] = bad
    V[:, :, :16] = bad
    Q[:, :, :16] = bad
    dO[:, :, :16] = bad
    for name, a, r in zip(("dQ", "dK", "dV"), gradients(), want):
        assert r.isfinite().all() and torch.equal(a, r), name
