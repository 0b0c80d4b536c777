"""The work that users of the hybrid-attention library have it do, as measurable cases.

A case is a dict of plain values.  ``kind`` names the pass through the public entry points:

    ring      one chunk of the streaming inference algorithm on the ring cache: open the chunk, its denoising steps, the
              last of which absorbs the chunk that is evicted next
    rope      one chunk of a model that rotates its keys (relative RoPE): tables, eviction of rotated keys into the state,
              rotation of the cached window, then per denoising step the rotation of queries and new keys and the attention
    step      one layer call of one chunk: pool, select, attend, history term, absorb of an evicted chunk
    prefill   the linear state built from a long run of tokens at once
    attend    selection and attention as separate calls: any storage type, head size and block size
    dense     sliding-window attention over every block
    train     selection, forward and backward of the one denoising step per chunk that carries gradients

Sizes: ``tokens`` per latent frame, frames per ``chunk`` and ``window`` (the chunk included), ``heads`` of ``head_dim``
features, KV and query ``block``, fraction of blocks to ``keep``.  Inputs are Gaussian, as in the benchmark.
"""
import math

import torch

import paper_2604_10103_amd as hf

DEV = "cuda"


def _case(name, kind, **kw):
    base = dict(name=name, kind=kind, dtype="bf16", batch=1, heads=12, head_dim=128, tokens=1560, chunk=3, window=6, sink=0,
                block=64, keep=0.25, steps=1, phi="relu", rope=False, state_frames=15)
    base.update(kw)
    return base


def listed():
    return [
        # the tiny fp32 stream (2 heads of 64, 256 tokens in the window): a chunk is a handful of launches on little data
        _case("ring_tiny_f32", "ring", dtype="f32", heads=2, head_dim=64, tokens=64, chunk=1, window=4, block=16, steps=2,
              state_frames=8),
        # a small stream with ragged blocks (200 tokens a frame), four denoising steps
        _case("ring_small", "ring", heads=3, tokens=200, chunk=2, window=6, steps=4, state_frames=4),
        # one layer of the 832x480 stream over a whole chunk: three sink frames, six cached or current ones, four steps
        _case("ring_832x480", "ring", window=9, sink=3, steps=4),
        # the same layer in a model that rotates its keys
        _case("rope_832x480", "rope", steps=4),
        # one layer call, the benchmark's step
        _case("step_832x480", "step"),
        # the large model's layer call
        _case("step_1280x720", "step", heads=40, tokens=3600, block=128, state_frames=30),
        # the state of one layer from fifteen frames at once (a stream that resumes or starts from given frames)
        _case("prefill_832x480", "prefill", chunk=15, window=15),
        # dense sliding window of the same length: the layers, or the comparison, without sparsity
        _case("dense_832x480", "dense", keep=1.0),
        # twice the heads at half the width
        _case("attend_832x480_d64", "attend", heads=24, head_dim=64),
        # the layer in fp32, as for checking a bf16 model
        _case("attend_832x480_f32", "attend", dtype="f32"),
        # the training step of one layer
        _case("train_832x480", "train"),
        # the same in fp32 on a quarter of the frame (416x240)
        _case("train_416x240_f32", "train", dtype="f32", tokens=390),
    ]


# the most products (forward flops) that a drawn case may have: the largest listed case of its kernels' class
_CAP = {"fast": 1.2e12, "train": 1.4e11, "wide": 7.0e10, "train_f32": 5.5e9}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["ring", "ring", "rope", "step", "step", "prefill", "attend", "attend", "dense", "train", "train"])
        c = _case("", kind, heads=_log_int(rng, 2, 40), tokens=_log_int(rng, 64, 3600), chunk=rng.choice([1, 2, 3]),
                  block=rng.choice([64, 64, 128]), keep=round(math.exp(rng.uniform(math.log(0.125), math.log(0.5))), 3),
                  state_frames=4)
        del c["name"]
        if kind == "ring":
            c.update(steps=rng.choice([1, 2, 4]), sink=rng.choice([0, 1, 3]))
            c["window"] = c["sink"] + c["chunk"] * rng.choice([2, 3])
        elif kind == "prefill":
            c["chunk"] = c["window"] = rng.choice([1, 3, 9, 15])
            c.update(phi=rng.choice(["relu", "relu", "elu"]), rope=rng.choice([False, True]))
        else:
            c["window"] = c["chunk"] * rng.choice([2, 3])
        if kind == "rope":
            c["steps"] = rng.choice([2, 4])
        if kind == "dense":
            c["keep"] = 1.0
        if kind in ("attend", "train") and rng.random() < 0.4:
            c.update(dtype="f32", block=rng.choice([16, 32, 64, 128]))
        if kind == "attend":
            c.update(head_dim=rng.choice([64, 128]), phi=rng.choice(["relu", "relu", "elu"]))
        if kind == "ring" and rng.random() < 0.3:   # small fp32 streams
            c.update(dtype="f32", head_dim=64, heads=_log_int(rng, 1, 4), tokens=_log_int(rng, 32, 256), block=rng.choice([16, 32]))
        z = _sizes(c)
        cap = ("wide" if c["dtype"] == "f32" or c["head_dim"] == 64 else "fast") if kind != "train" else \
            ("train_f32" if c["dtype"] == "f32" else "train")
        if c["steps"] * z["attn_flops"] <= _CAP[cap] and z["t_n"] <= 1000:
            return c


# ------------------------------------------------------------------------------------------------ sizes and work
def _sizes(c):
    n_q, n_kv = c["tokens"] * c["chunk"], c["tokens"] * c["window"]
    t_m, t_n = -(-n_q // c["block"]), -(-n_kv // c["block"])
    k = min(t_n, max(1, math.ceil(c["keep"] * t_n - 1e-9)))
    bh, d = c["batch"] * c["heads"], c["head_dim"]
    return dict(n_q=n_q, n_kv=n_kv, t_m=t_m, t_n=t_n, k=k, bh=bh, d=d, es=2 if c["dtype"] == "bf16" else 4,
                attn_flops=4.0 * d * n_q * min(n_kv, k * c["block"]) * bh, state=bh * (d * d + d) * 4)


def work(case):
    z = _sizes(case)
    d, bh, n_q, n_kv, es, st = z["d"], z["bh"], z["n_q"], z["n_kv"], z["es"], z["state"]
    row = bh * d * es                                   # bytes of one token of every head
    readout = 2.0 * bh * n_q * d * d                    # products of the history term, and of absorbing as many tokens
    idx = bh * z["t_m"] * z["k"] * 4
    kind, steps = case["kind"], case["steps"]
    if kind == "prefill":
        return {"bytes": 2 * n_kv * row + 3 * st, "flops": 2.0 * bh * n_kv * d * d}
    if kind == "dense":
        return {"bytes": (2 * n_q + 2 * n_kv) * row, "flops": z["attn_flops"]}
    if kind == "attend":
        return {"bytes": (2 * n_q + 2 * n_kv) * row + st + idx, "flops": z["attn_flops"] + readout}
    if kind == "step":
        return {"bytes": (2 * n_q + 2 * n_kv + 2 * n_q) * row + 3 * st + idx, "flops": z["attn_flops"] + 2 * readout}
    if kind == "ring":
        return {"bytes": (steps * 2 * n_q + 2 * n_kv) * row + 2 * st + steps * idx,
                "flops": steps * (z["attn_flops"] + readout) + readout}
    if kind == "rope":
        # the window's keys are read once un-rotated and written once rotated; per step Q, the new keys and O
        return {"bytes": (steps * 3 * n_q + 3 * n_kv + 2 * n_q) * row + 3 * st + steps * idx + 2 * n_kv * d * 2,
                "flops": steps * (z["attn_flops"] + readout) + readout}
    # train: forward, and five products of its size backward
    return {"bytes": (4 * n_q + 4 * n_kv) * row + st + idx, "flops": 3.5 * z["attn_flops"] + 3 * readout}


def tolerance(case):
    # A selection may differ where two scores agree to the last bits of their fp32 sums ("differ").
    if case["kind"] == "prefill":
        # fp32 sums next to their bf16 planes; rotated or ELU keys are rounded to bf16 for the products
        return {"rel": 5e-3 if case["rope"] or case["phi"] != "relu" else 1e-3}
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "differ": 2e-3}            # bf16 outputs, probabilities rounded to bf16 for the second product
    # fp32 sums; the gradients subtract numbers of the size of one
    return {"rel": 5e-5 if case["kind"] == "train" else 1e-5, "differ": 2e-3}


# ------------------------------------------------------------------------------------------------ what a program keeps
class _Gauss:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(int(seed))

    def __call__(self, shape, scale, dtype):
        return (torch.randn(shape, generator=self.g, device=DEV, dtype=torch.float32) * scale).to(dtype)


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def _grid(tokens):
    rows = int(math.isqrt(tokens))
    while tokens % rows:
        rows -= 1
    return rows, tokens // rows


def _pairs(d):
    return (d // 2 - 2 * (d // 6), d // 6, d // 6)


def prepare(case, seed):
    c, z = case, _sizes(case)
    gauss = _Gauss(seed)
    td = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    B, H, d, n_q, n_kv = c["batch"], c["heads"], z["d"], z["n_q"], z["n_kv"]
    scale = 0.5 if c["dtype"] == "bf16" else 1.0
    kind = c["kind"]
    phi = hf.HF_PHI_RELU if c["phi"] == "relu" else hf.HF_PHI_ELU1
    cfg = hf.make_config(B, H, d, c["dtype"], c["block"], c["block"], c["keep"], phi=phi,
                         kv_capacity=n_kv if kind == "ring" else 0)
    s = {"kind": kind, "cfg": cfg, "case": c, "n_q": n_q, "n_kv": n_kv}
    qs, ks = (B, H, n_q, d), (B, H, n_kv, d)

    def filled_state():
        """A state that holds some frames already, absorbed as a stream does."""
        st = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
        hf.hf_state_init(cfg, st)
        n = c["tokens"] * c["state_frames"]
        ws = _bytes(hf.hf_absorb_workspace_bytes(cfg, n))
        shape = (B, H, n, d)
        hf.hf_absorb_evicted(cfg, st, gauss(shape, scale, td), gauss(shape, scale, td), workspace=ws)
        return st

    if kind == "prefill":
        s["K"], s["V"] = gauss(ks, scale, td), gauss(ks, scale, td)
        s["state"] = torch.empty(hf.hf_state_bytes(cfg) // 4, dtype=torch.float32, device=DEV)
        s["planes"] = _bytes(hf.hf_state_planes_bytes(cfg))
        s["ws"] = _bytes(hf.hf_absorb_workspace_bytes(cfg, n_kv))
        s["cos"] = s["sin"] = None
        if c["rope"]:
            s["cos"] = torch.empty((n_kv, d // 2), dtype=torch.float32, device=DEV)
            s["sin"] = torch.empty_like(s["cos"])
            hf.hf_rope_tables(list(range(c["window"])), *_grid(c["tokens"]), _pairs(d), s["cos"], s["sin"])
        return s

    s["K"], s["V"] = gauss(ks, scale, td), gauss(ks, scale, td)
    s["Q"] = [gauss(qs, scale, td) for _ in range(c["steps"])]
    s["O"] = [torch.empty(qs, dtype=td, device=DEV) for _ in range(c["steps"])]
    if kind == "dense":
        return s
    s["idx"] = [torch.empty((B, H, z["t_m"], hf.hf_select_k(cfg, n_kv)), dtype=torch.int32, device=DEV)
                for _ in range(c["steps"])]
    s["state"] = filled_state()

    if kind == "ring":
        s["ws"] = _bytes(hf.hf_workspace_bytes(cfg, n_q, n_kv))
        s["step_ws"] = _bytes(max(hf.hf_step_workspace_bytes(cfg, n_q, n_q), hf.hf_absorb_workspace_bytes(cfg, n_q)))
        s["state2"] = torch.empty_like(s["state"])
        # the cache is full, and the chunk before has absorbed the slot that comes next (as hf_ring_last_step leaves it)
        slots = (c["window"] - c["sink"]) // c["chunk"]
        ring = hf.make_ring(c["sink"] * c["tokens"], n_q)
        ring.n_filled, ring.cur_slot, ring.next_slot, ring.absorbed_ahead = slots, slots - 1, 0, 1
        s["ring"] = ring
    elif kind == "rope":
        s["n_old"] = n_kv - n_q
        s["grid"], s["pairs"] = _grid(c["tokens"]), _pairs(d)
        s["K_new"] = [gauss(qs, scale, td) for _ in range(c["steps"])]
        s["K_ev"], s["V_ev"] = gauss(qs, scale, td), gauss(qs, scale, td)
        s["K_rot"], s["Q_rot"] = torch.empty_like(s["K"]), torch.empty_like(s["Q"][0])
        s["cos"] = torch.empty((n_kv, d // 2), dtype=torch.float32, device=DEV)
        s["sin"] = torch.empty_like(s["cos"])
        s["cos_ev"] = torch.empty((n_q, d // 2), dtype=torch.float32, device=DEV)
        s["sin_ev"] = torch.empty_like(s["cos_ev"])
        s["planes"] = _bytes(hf.hf_state_planes_bytes(cfg))
        s["absorb_ws"] = _bytes(hf.hf_absorb_workspace_bytes(cfg, n_q))
        s["pooled"] = _bytes(hf.hf_pooled_keys_bytes(cfg, n_kv))
    elif kind == "step":
        s["K_ev"], s["V_ev"] = gauss(qs, scale, td), gauss(qs, scale, td)
        s["planes"] = _bytes(hf.hf_state_planes_bytes(cfg))
        hf.hf_state_planes(cfg, s["state"], s["planes"])
        s["state2"], s["planes2"] = torch.empty_like(s["state"]), torch.empty_like(s["planes"])
        s["pooled"] = _bytes(hf.hf_pooled_keys_bytes(cfg, n_kv))
        s["step_ws"] = _bytes(hf.hf_step_workspace_bytes(cfg, n_q, n_q))
    else:
        s["ws"] = _bytes(hf.hf_workspace_bytes(cfg, n_q, n_kv))
        if kind == "train":
            s["dO"] = gauss(qs, 1.0, td)
            s["dQ"], s["dK"], s["dV"] = torch.empty_like(s["dO"]), torch.empty_like(s["K"]), torch.empty_like(s["V"])
            s["bwd_ws"] = _bytes(hf.hf_bwd_workspace_bytes(cfg, n_q, n_kv))
            if c["dtype"] == "bf16":   # the saving forward and the backward from its by-products cover bf16
                s["O_local"] = torch.empty_like(s["dO"])
                s["lse2"] = torch.empty((B * H, n_q), dtype=torch.float32, device=DEV)
    return s


# ------------------------------------------------------------------------------------------------ one pass
def _run_ring(s):
    cfg, ring, steps = s["cfg"], s["ring"], len(s["Q"])
    hf.hf_ring_open_chunk(cfg, ring, s["K"], s["V"], s["state"], workspace=s["step_ws"])
    for i in range(steps - 1):
        hf.hf_ring_step(cfg, ring, s["Q"][i], s["K"], s["V"], i, s["idx"][i], s["state"], s["O"][i], s["ws"])
    i = steps - 1
    if hf.hf_ring_last_step(cfg, ring, s["Q"][i], s["K"], s["V"], i, s["idx"][i], s["state"], s["O"][i], s["ws"], s["state2"],
                            s["step_ws"]):
        s["state"], s["state2"] = s["state2"], s["state"]
    return {"O": s["O"], "idx": s["idx"], "state": s["state"]}


def _run_rope(s):
    cfg, n_old, frames = s["cfg"], s["n_old"], s["case"]["window"]
    # the stream is past the cap of its temporal index: the window's frames keep their distances to the newest
    idx = hf.hf_rope_window_indices(200, frames, 21)
    hf.hf_rope_tables(idx, *s["grid"], s["pairs"], s["cos"], s["sin"])
    chunk = s["case"]["chunk"]
    hf.hf_rope_tables([idx[0] - chunk + f for f in range(chunk)], *s["grid"], s["pairs"], s["cos_ev"], s["sin_ev"])
    hf.hf_absorb_evicted_planes(cfg, s["state"], s["K_ev"], s["V_ev"], s["planes"], s["cos_ev"], s["sin_ev"],
                                workspace=s["absorb_ws"])
    hf.hf_rope_apply(cfg, s["K"], s["cos"], s["sin"], s["K_rot"])
    hf.hf_pool_keys(cfg, s["K_rot"], s["pooled"])
    cq, sq = s["cos"][n_old:], s["sin"][n_old:]
    for Q, K_new, O, bi in zip(s["Q"], s["K_new"], s["O"], s["idx"]):
        hf.hf_rope_append_keys(cfg, K_new, cq, sq, s["K_rot"], n_old, s["pooled"])
        hf.hf_rope_apply(cfg, Q, cq, sq, s["Q_rot"])
        hf.hf_select_attn_fwd(cfg, s["Q_rot"], s["K_rot"], s["V"], s["pooled"], s["state"], s["planes"], O, bi,
                              rope_cos_q=cq, rope_sin_q=sq, Q_hist=Q)
    return {"O": s["O"], "idx": s["idx"], "state": s["state"], "K_rot": s["K_rot"]}


def _run_step(s):
    cfg = s["cfg"]
    hf.hf_pool_keys(cfg, s["K"], s["pooled"])
    hf.hf_step_fwd(cfg, s["Q"][0], s["K"], s["V"], s["pooled"], s["state"], s["planes"], s["O"][0], s["idx"][0], s["K_ev"],
                   s["V_ev"], s["state2"], s["planes2"], s["step_ws"])
    return {"O": s["O"], "idx": s["idx"], "state": s["state2"], "planes": s["planes2"].view(torch.bfloat16)}


def _run_prefill(s):
    hf.hf_state_init(s["cfg"], s["state"])
    hf.hf_absorb_evicted_planes(s["cfg"], s["state"], s["K"], s["V"], s["planes"], s["cos"], s["sin"], workspace=s["ws"])
    # (the planes hold the high part of the state and the remainder, which is rounding: the first is what is compared)
    return {"state": s["state"], "planes": s["planes"].view(torch.bfloat16).view(-1, 2, 128, 128)[:, 0]}


def _run_dense(s):
    hf.hf_hybrid_attn_fwd(s["cfg"], s["Q"][0], s["K"], s["V"], None, None, s["O"][0])
    return s["O"][0]


def _run_attend(s):
    cfg = s["cfg"]
    hf.hf_block_select(cfg, s["Q"][0], s["K"], s["idx"][0], None, s["ws"])
    hf.hf_hybrid_attn_fwd(cfg, s["Q"][0], s["K"], s["V"], s["idx"][0], s["state"], s["O"][0], s["ws"])
    return {"O": s["O"][0], "idx": s["idx"][0]}


def _run_train(s):
    cfg, Q, idx = s["cfg"], s["Q"][0], s["idx"][0]
    hf.hf_block_select(cfg, Q, s["K"], idx, None, s["ws"])
    if "lse2" in s:
        hf.hf_hybrid_attn_fwd_save(cfg, Q, s["K"], s["V"], idx, s["state"], s["O"][0], s["O_local"], s["lse2"], s["ws"])
        hf.hf_hybrid_attn_bwd_saved(cfg, Q, s["K"], s["V"], idx, s["state"], s["dO"], s["O_local"], s["lse2"], s["dQ"],
                                    s["dK"], s["dV"], s["bwd_ws"])
    else:
        hf.hf_hybrid_attn_fwd(cfg, Q, s["K"], s["V"], idx, s["state"], s["O"][0], s["ws"])
        hf.hf_hybrid_attn_bwd(cfg, Q, s["K"], s["V"], idx, s["state"], s["dO"], s["dQ"], s["dK"], s["dV"], s["bwd_ws"])
    return {"O": s["O"][0], "idx": idx, "dQ": s["dQ"], "dK": s["dK"], "dV": s["dV"]}


_RUN = {"ring": _run_ring, "rope": _run_rope, "step": _run_step, "prefill": _run_prefill, "dense": _run_dense,
        "attend": _run_attend, "train": _run_train}


def run(state):
    return _RUN[state["kind"]](state)
