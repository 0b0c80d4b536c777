"""Binding of libhf.so: same names as the C ABI, argument marshalling only.

Every function takes torch tensors that already live on the GPU, checks dtype / shape /
contiguity, and passes raw device pointers plus the current HIP stream.  The checks and the
call are native (csrc/hf_marshal.cpp); here stand the signatures.  No step of the
method runs in Python or in torch; torch is used for device memory and streams.
There is no fallback: a missing library or a failed call raises.
"""
from __future__ import annotations

import ctypes
import os

import torch

HF_BF16, HF_F32 = 0, 1
HF_PHI_RELU, HF_PHI_ELU1 = 0, 1
HF_FLAG_READOUT_KERNEL, HF_FLAG_HISTORY_TWO_PLANES, HF_FLAG_BWD_FP32_KERNELS, HF_FLAG_DKV_INDEX_ORDER = 1, 2, 4, 8
HF_OK = 0

_LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libhf.so")
_lib = None
_native = None   # the marshalling module, bound to the loaded library


class HFError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"hf error {code}: {msg}")
        self.code = code


class hf_config(ctypes.Structure):
    _fields_ = [
        ("batch", ctypes.c_int32),
        ("heads", ctypes.c_int32),
        ("head_dim", ctypes.c_int32),
        ("dtype", ctypes.c_int32),
        ("block_q", ctypes.c_int32),
        ("block_kv", ctypes.c_int32),
        ("keep_ratio", ctypes.c_float),
        ("keep_k", ctypes.c_int32),
        ("phi", ctypes.c_int32),
        ("eps", ctypes.c_float),
        ("z_scale", ctypes.c_float),
        ("softmax_scale", ctypes.c_float),
        ("kv_capacity", ctypes.c_int32),
        ("flags", ctypes.c_int32),
    ]


class hf_window(ctypes.Structure):
    _fields_ = [("n_sink", ctypes.c_int32), ("n_tokens", ctypes.c_int32)]


class hf_ring(ctypes.Structure):
    _fields_ = [("n_sink", ctypes.c_int32), ("n_chunk", ctypes.c_int32), ("n_filled", ctypes.c_int32),
                ("next_slot", ctypes.c_int32), ("cur_slot", ctypes.c_int32), ("absorbed_ahead", ctypes.c_int32)]


def make_config(batch, heads, head_dim, dtype, block_q, block_kv, keep_ratio=1.0, keep_k=0,
                phi=HF_PHI_RELU, eps=1e-6, z_scale=1.0, softmax_scale=0.0, kv_capacity=0, flags=0) -> hf_config:
    if isinstance(dtype, str):
        dtype = {"bf16": HF_BF16, "f32": HF_F32}[dtype]
    elif isinstance(dtype, torch.dtype):
        dtype = {torch.bfloat16: HF_BF16, torch.float32: HF_F32}[dtype]
    return hf_config(batch, heads, head_dim, dtype, block_q, block_kv, keep_ratio, keep_k, phi, eps,
                     z_scale, softmax_scale, kv_capacity, flags)


def lib_path() -> str:
    return _LIB_PATH


def load():
    """Load libhf.so (built in-tree by ``python -m paper_2604_10103_amd.build``)."""
    global _lib, _native
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise RuntimeError(f"{_LIB_PATH} is missing: build it with `python -m paper_2604_10103_amd.build`")
    lib = ctypes.CDLL(_LIB_PATH)
    P, I, SZ = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
    CP = ctypes.POINTER(hf_config)
    lib.hf_last_error.restype = ctypes.c_char_p
    lib.hf_last_error.argtypes = []
    lib.hf_version.restype = ctypes.c_char_p
    lib.hf_version.argtypes = []
    lib.hf_state_bytes.argtypes = [CP, ctypes.POINTER(SZ)]
    lib.hf_state_init.argtypes = [CP, P, P]
    lib.hf_state_fold_linear.argtypes = [CP, P, P, P, P]
    lib.hf_absorb_evicted.argtypes = [CP, P, P, P, I, P, P, P, SZ, P]
    lib.hf_absorb_workspace_bytes.argtypes = [CP, I, ctypes.POINTER(SZ)]
    lib.hf_state_planes_bytes.argtypes = [CP, ctypes.POINTER(SZ)]
    lib.hf_state_planes.argtypes = [CP, P, P, P]
    lib.hf_absorb_evicted_planes.argtypes = [CP, P, P, P, I, P, P, P, SZ, P, P]
    lib.hf_hybrid_attn_fwd_planes.argtypes = [CP, P, P, I, P, P, I, P, I, P, P, P, P, P, P]
    lib.hf_window_advance.argtypes = [CP, P, P, I, I, P, P, P, P, SZ, P]
    lib.hf_window_evict.argtypes = [CP, P, P, I, I, I, P, P, P, P, SZ, P]
    WP = ctypes.POINTER(hf_window)
    lib.hf_stream_open_chunk.argtypes = [CP, WP, I, P, P, P, P, P, P, SZ, ctypes.POINTER(I), ctypes.POINTER(I), P]
    lib.hf_stream_step.argtypes = [CP, WP, P, P, I, P, P, I, P, P, P, P, P, P, SZ, P]
    RP = ctypes.POINTER(hf_ring)
    lib.hf_ring_open_chunk.argtypes = [CP, RP, P, P, P, P, P, P, SZ, ctypes.POINTER(I), ctypes.POINTER(I), P]
    lib.hf_ring_step.argtypes = [CP, RP, P, P, P, P, I, P, P, P, P, P, P, SZ, P]
    lib.hf_select_k.argtypes = [CP, I, ctypes.POINTER(I)]
    lib.hf_workspace_bytes.argtypes = [CP, I, I, ctypes.POINTER(SZ)]
    lib.hf_block_select.argtypes = [CP, P, I, P, I, P, P, P, SZ, P]
    lib.hf_block_select_cached.argtypes = [CP, P, I, P, I, I, P, P, P, SZ, P]
    lib.hf_block_select_static.argtypes = [CP, P, I, P, I, P, P, P]
    lib.hf_pooled_keys_bytes.argtypes = [CP, I, ctypes.POINTER(ctypes.c_size_t)]
    lib.hf_pool_keys.argtypes = [CP, P, I, I, P, P]
    lib.hf_select_attn_fwd.argtypes = [CP, P, P, I, P, P, I, P, P, P, P, P, P, P, P, P]
    lib.hf_ring_last_step.argtypes = [CP, ctypes.POINTER(hf_ring), P, P, P, P, I, P, P, P, P, P, P, SZ, P, P, P, P, SZ,
                                      ctypes.POINTER(ctypes.c_int32), P]
    lib.hf_step_workspace_bytes.argtypes = [CP, I, I, ctypes.POINTER(SZ)]
    lib.hf_step_fwd.argtypes = [CP, P, P, I, P, P, I, P, P, P, P, P, P, P, P, P, P, I, I, P, P, P, SZ, P]
    lib.hf_hybrid_attn_fwd.argtypes = [CP, P, I, P, P, I, P, I, P, P, P, P, P, SZ, P]
    lib.hf_hybrid_attn_fwd_split.argtypes = [CP, P, P, I, P, P, I, P, I, P, P, P, P, P, SZ, P]
    lib.hf_hybrid_attn_fwd_save.argtypes = [CP, P, P, I, P, P, I, P, I, P, P, P, P, P, P, P, SZ, P]
    lib.hf_bwd_workspace_bytes.argtypes = [CP, I, I, ctypes.POINTER(SZ)]
    lib.hf_bwd_least_workspace_bytes.argtypes = [CP, I, I, ctypes.POINTER(SZ)]
    lib.hf_hybrid_attn_bwd.argtypes = [CP, P, P, I, P, P, I, P, I, P, P, P, P, P, P, P, P, P, SZ, P]
    lib.hf_hybrid_attn_bwd_saved.argtypes = [CP, P, P, I, P, P, I, P, I, P, P, P, P, P, P, P, P, P, P, P, SZ, P]
    lib.hf_rope_window_indices.argtypes = [I, I, I, ctypes.POINTER(I)]
    lib.hf_rope_tables.argtypes = [ctypes.POINTER(I), I, I, I, I, I, I, ctypes.c_double, I, P, P, P]
    lib.hf_rope_apply.argtypes = [CP, P, I, P, P, P, P]
    lib.hf_rope_append_keys.argtypes = [CP, P, I, P, P, P, I, I, P, P]
    lib.hf_probe_mfma_bf16.argtypes = [I, P, ctypes.POINTER(ctypes.c_double), P]
    for name in ("hf_state_bytes", "hf_state_init", "hf_state_fold_linear", "hf_window_advance", "hf_absorb_evicted", "hf_absorb_workspace_bytes", "hf_select_k",
                 "hf_workspace_bytes",
                 "hf_block_select", "hf_block_select_cached", "hf_block_select_static", "hf_hybrid_attn_fwd",
                 "hf_hybrid_attn_fwd_split",
                 "hf_rope_window_indices", "hf_rope_tables", "hf_rope_apply", "hf_window_evict", "hf_stream_open_chunk",
                 "hf_stream_step", "hf_bwd_workspace_bytes", "hf_bwd_least_workspace_bytes", "hf_hybrid_attn_bwd", "hf_state_planes_bytes",
                 "hf_state_planes", "hf_absorb_evicted_planes", "hf_hybrid_attn_fwd_planes", "hf_probe_mfma_bf16",
                 "hf_ring_open_chunk", "hf_ring_step", "hf_pooled_keys_bytes", "hf_pool_keys", "hf_select_attn_fwd",
                 "hf_step_workspace_bytes", "hf_step_fwd", "hf_rope_append_keys", "hf_ring_last_step"):
        getattr(lib, name).restype = ctypes.c_int
    try:
        from . import _marshal
    except ImportError as e:
        raise RuntimeError(f"the marshalling module does not load ({e}): build it with `python -m paper_2604_10103_amd.build`") from e
    _marshal.bind({name: ctypes.cast(getattr(lib, name), ctypes.c_void_p).value for name in _marshal.entry_names()}, HFError,
                  hf_config, hf_window, hf_ring)
    _lib, _native = lib, _marshal
    return lib


def _call():
    if _native is None:
        load()
    return _native


def _check(code: int):
    if code != HF_OK:
        raise HFError(code, load().hf_last_error().decode())


# ------------------------------------------------------------------------------ host helpers
def hf_version() -> str:
    return load().hf_version().decode()


def hf_state_bytes(cfg: hf_config) -> int:
    out = ctypes.c_size_t(0)
    _check(load().hf_state_bytes(ctypes.byref(cfg), ctypes.byref(out)))
    return out.value


def hf_window_advance(cfg: hf_config, K_win, V_win, n_evict: int, state, rope_cos=None, rope_sin=None,
                      workspace=None, n_sink: int = 0, n_kv=None) -> None:
    """Absorb the oldest n_evict tokens behind the first n_sink of the window buffers into the state and move
    the rest down (hf_window_evict; n_sink = 0 is hf_window_advance)."""
    _call().window_evict(cfg, K_win, V_win, n_evict, state, rope_cos, rope_sin, workspace, n_sink, n_kv)


def hf_select_k(cfg: hf_config, n_kv: int) -> int:
    out = ctypes.c_int32(0)
    _check(load().hf_select_k(ctypes.byref(cfg), n_kv, ctypes.byref(out)))
    return out.value


def hf_absorb_workspace_bytes(cfg: hf_config, n_tokens: int) -> int:
    out = ctypes.c_size_t(0)
    _check(load().hf_absorb_workspace_bytes(ctypes.byref(cfg), n_tokens, ctypes.byref(out)))
    return out.value


def hf_workspace_bytes(cfg: hf_config, n_q: int, n_kv: int) -> int:
    out = ctypes.c_size_t(0)
    _check(load().hf_workspace_bytes(ctypes.byref(cfg), n_q, n_kv, ctypes.byref(out)))
    return out.value


# ------------------------------------------------------------------------------ device calls
def hf_state_init(cfg: hf_config, state: torch.Tensor) -> None:
    """state: fp32 GPU tensor of hf_state_bytes(cfg)/4 elements, zeroed in place."""
    _call().state_init(cfg, state)


def hf_state_fold_linear(cfg: hf_config, state_in, W, state_out) -> None:
    """state_out = state_in with L[b,h] replaced by L[b,h] @ W[h]; W: fp32 GPU tensor [H, d, d]."""
    _call().state_fold_linear(cfg, state_in, W, state_out)


def hf_absorb_evicted(cfg: hf_config, state, K_ev, V_ev, rope_cos=None, rope_sin=None, workspace=None) -> None:
    """workspace: optional uint8 GPU buffer of hf_absorb_workspace_bytes(cfg, n) bytes (atomic-free path)."""
    _call().absorb_evicted(cfg, state, K_ev, V_ev, rope_cos, rope_sin, workspace)


def hf_state_planes_bytes(cfg: hf_config) -> int:
    """Bytes of the caller-kept bf16 planes of the state (0: the configuration has no such path)."""
    out = ctypes.c_size_t(0)
    _check(load().hf_state_planes_bytes(ctypes.byref(cfg), ctypes.byref(out)))
    return out.value


def hf_state_planes(cfg: hf_config, state, planes_out) -> None:
    """planes_out (uint8 GPU buffer of hf_state_planes_bytes(cfg) bytes) = the bf16 planes of state."""
    _call().state_planes(cfg, state, planes_out)


def hf_absorb_evicted_planes(cfg: hf_config, state, K_ev, V_ev, planes_out, rope_cos=None, rope_sin=None,
                             workspace=None) -> None:
    """hf_absorb_evicted that also writes the planes of the updated state into planes_out."""
    _call().absorb_evicted_planes(cfg, state, K_ev, V_ev, planes_out, rope_cos, rope_sin, workspace)


def hf_block_select(cfg: hf_config, Q, K_win, block_idx, scores=None, workspace=None, n_kv=None) -> None:
    """block_idx: int32 [B,H,T_m,k] out; scores: optional fp32 [B,H,T_m,T_n] out; workspace: uint8 buffer."""
    _call().block_select(cfg, Q, K_win, None, block_idx, scores, workspace, n_kv)


HF_STATIC_SCRATCH_BYTES = 8 << 20


def hf_block_select_static(cfg: hf_config, Q, K_win, block_idx, scores=None, n_kv=None) -> None:
    """hf_block_select without a workspace: the pooled means live in the library's built-in per-GPU buffer."""
    _call().block_select_static(cfg, Q, K_win, block_idx, scores, n_kv)


def hf_block_select_cached(cfg: hf_config, Q, K_win, n_cached_kv_blocks: int, block_idx, scores=None,
                           workspace=None, n_kv=None) -> None:
    """As hf_block_select; the pooled means of the first n_cached_kv_blocks KV blocks are reused from the
    previous call on the same workspace (the caller guarantees those tokens did not change)."""
    _call().block_select(cfg, Q, K_win, int(n_cached_kv_blocks), block_idx, scores, workspace, n_kv)


def hf_hybrid_attn_fwd(cfg: hf_config, Q, K_win, V_win, block_idx, state, O, workspace=None,
                       rope_cos_q=None, rope_sin_q=None, Q_hist=None, n_kv=None) -> None:
    """block_idx None = dense window attention; state None = no history term; Q_hist: the history branch's
    queries when they are not Q (hf_hybrid_attn_fwd_split)."""
    _call().hybrid_attn_fwd(cfg, Q, K_win, V_win, block_idx, state, O, workspace, rope_cos_q, rope_sin_q, Q_hist, n_kv)


def hf_hybrid_attn_fwd_planes(cfg: hf_config, Q, K_win, V_win, block_idx, state, planes, O, rope_cos_q=None,
                              rope_sin_q=None, Q_hist=None, n_kv=None) -> None:
    """hf_hybrid_attn_fwd with the state's planes kept by the caller (hf_absorb_evicted_planes /
    hf_state_planes): no workspace, no conversion launch."""
    _call().hybrid_attn_fwd_planes(cfg, Q, K_win, V_win, block_idx, state, planes, O, rope_cos_q, rope_sin_q, Q_hist, n_kv)


def hf_pooled_keys_bytes(cfg: hf_config, n_kv: int) -> int:
    out = ctypes.c_size_t(0)
    _check(load().hf_pooled_keys_bytes(ctypes.byref(cfg), n_kv, ctypes.byref(out)))
    return out.value


def hf_pool_keys(cfg: hf_config, K_win, pooled_K, n_cached_kv_blocks: int = 0, n_kv=None) -> None:
    """Pooled keys of the window (Eq. 4's k-bar) for hf_select_attn_fwd; the first n_cached_kv_blocks keep their values."""
    _call().pool_keys(cfg, K_win, pooled_K, n_cached_kv_blocks, n_kv)


def hf_select_attn_fwd(cfg: hf_config, Q, K_win, V_win, pooled_K, state, planes, O, block_idx_out, scores=None,
                       rope_cos_q=None, rope_sin_q=None, Q_hist=None, n_kv=None) -> None:
    """Top-K selection (Eq. 4), sparse attention (Eq. 5) and history term (Eq. 3, 6) in one launch; the chosen
    blocks are written to block_idx_out [B, H, T_m, k]."""
    _call().select_attn_fwd(cfg, Q, K_win, V_win, pooled_K, state, planes, O, block_idx_out, scores, rope_cos_q, rope_sin_q,
                            Q_hist, n_kv)


def hf_step_workspace_bytes(cfg: hf_config, n_q: int, n_ev: int) -> int:
    out = ctypes.c_size_t(0)
    _check(load().hf_step_workspace_bytes(ctypes.byref(cfg), n_q, n_ev, ctypes.byref(out)))
    return out.value


def hf_step_fwd(cfg: hf_config, Q, K_win, V_win, pooled_K, state_in, planes, O, block_idx_out, K_ev, V_ev, state_out,
                planes_out, workspace, scores=None, rope_cos_q=None, rope_sin_q=None, Q_hist=None, n_kv=None,
                n_ev=None) -> None:
    """hf_select_attn_fwd with workgroups of their own that absorb K_ev, V_ev (Eq. 2) into state_out / planes_out
    = state_in + their contribution, in the same launch.  n_ev: tokens of every head of K_ev to absorb (default:
    all of its third dimension, which is also the head stride)."""
    _call().step_fwd(cfg, Q, K_win, V_win, pooled_K, state_in, planes, O, block_idx_out, K_ev, V_ev, state_out, planes_out,
                     workspace, scores, rope_cos_q, rope_sin_q, Q_hist, n_kv, n_ev)


def hf_hybrid_attn_fwd_save(cfg: hf_config, Q, K_win, V_win, block_idx, state, O, O_local_out, lse2_out, workspace=None,
                            rope_cos_q=None, rope_sin_q=None, Q_hist=None, n_kv=None) -> None:
    """hf_hybrid_attn_fwd that also writes O_local and the softmax row statistic lse2 [B*H, n_q] (fp32) for
    hf_hybrid_attn_bwd_saved."""
    _call().hybrid_attn_fwd_save(cfg, Q, K_win, V_win, block_idx, state, O, O_local_out, lse2_out, workspace, rope_cos_q,
                                 rope_sin_q, Q_hist, n_kv)


def hf_probe_mfma_bf16(iters: int, scratch) -> float:
    """Enqueue the MFMA issue-rate probe; returns the floating-point operations of the launch (time it with events)."""
    flops = ctypes.c_double(0.0)
    if not scratch.is_cuda or scratch.dtype != torch.float32:
        raise TypeError("scratch must be a float32 GPU tensor")
    if not scratch.is_contiguous():
        raise ValueError("scratch must be contiguous")
    _check(load().hf_probe_mfma_bf16(int(iters), scratch.data_ptr(), ctypes.byref(flops),
                                     torch.cuda.current_stream().cuda_stream))
    return flops.value


def hf_rope_window_indices(i_newest: int, n_frames: int, t0: int) -> list:
    """Eq. 7 with the cache re-based to the current chunk: temporal indices of the last n_frames frames."""
    return _call().rope_window_indices(i_newest, n_frames, t0)


def hf_rope_tables(frame_idx, height: int, width: int, pairs, cos_out, sin_out, theta: float = 10000.0,
                   temporal_only: bool = False) -> None:
    """cos_out, sin_out: fp32 GPU tensors [len(frame_idx) * height * width, sum(pairs)]."""
    _call().rope_tables(frame_idx, height, width, pairs, cos_out, sin_out, theta, temporal_only)


def hf_rope_append_keys(cfg: hf_config, K_new, rope_cos, rope_sin, K_win, first: int, pooled_K, n_kv=None) -> None:
    """K_new [B, H, n_new, d], rotated by its tables (None: copied), becomes tokens first .. first + n_new - 1 of the
    window buffer K_win; the pooled keys of the KV blocks those tokens touch are rewritten in pooled_K."""
    _call().rope_append_keys(cfg, K_new, rope_cos, rope_sin, K_win, first, pooled_K, n_kv)


def hf_rope_apply(cfg: hf_config, X, rope_cos, rope_sin, Y) -> None:
    """Y = X with adjacent feature pairs of every token turned by the tables [n, d/2]; Y may be X."""
    _call().rope_apply(cfg, X, rope_cos, rope_sin, Y)


def hf_stream_open_chunk(cfg: hf_config, win: hf_window, n_chunk: int, K_win, V_win, state, rope_cos_ev=None,
                         rope_sin_ev=None, workspace=None):
    """Evict what the next chunk of n_chunk tokens pushes out of the cache into the state and reserve the
    chunk's slot; returns (token offset of the slot, tokens evicted) and updates ``win``."""
    return _call().stream_open_chunk(cfg, win, n_chunk, K_win, V_win, state, rope_cos_ev, rope_sin_ev, workspace)


def hf_stream_step(cfg: hf_config, win: hf_window, Q, K_win, V_win, step_in_chunk: int, block_idx, state, O,
                   workspace, rope_cos_q=None, rope_sin_q=None, Q_hist=None) -> None:
    """Selection (pooled keys of the unchanged blocks reused after the chunk's first step) and hybrid attention
    over the valid tokens of the cache."""
    _call().stream_step(cfg, win, Q, K_win, V_win, step_in_chunk, block_idx, state, O, workspace, rope_cos_q, rope_sin_q, Q_hist)


def make_ring(n_sink: int, n_chunk: int) -> hf_ring:
    return hf_ring(int(n_sink), int(n_chunk), 0, 0, -1, 0)


def hf_ring_open_chunk(cfg: hf_config, ring: hf_ring, K_cache, V_cache, state, rope_cos_ev=None, rope_sin_ev=None,
                       workspace=None):
    """Hand the next chunk slot of the ring to a new chunk; the chunk it held (if any) goes into the state where it
    lies.  Returns (token offset of the slot, tokens evicted) and updates ``ring``."""
    return _call().ring_open_chunk(cfg, ring, K_cache, V_cache, state, rope_cos_ev, rope_sin_ev, workspace)


def hf_ring_last_step(cfg: hf_config, ring: hf_ring, Q, K_cache, V_cache, step_in_chunk: int, block_idx, state, O, workspace,
                      state_out, step_workspace, rope_cos_q=None, rope_sin_q=None, Q_hist=None, rope_cos_ev=None,
                      rope_sin_ev=None) -> bool:
    """hf_ring_step for the chunk's last denoising step; if the next hf_ring_open_chunk would evict a chunk, that chunk
    is absorbed now into state_out (= state + its contribution) and True is returned: state_out is the state from the
    next chunk on."""
    return _call().ring_last_step(cfg, ring, Q, K_cache, V_cache, step_in_chunk, block_idx, state, O, workspace, state_out,
                                  step_workspace, rope_cos_q, rope_sin_q, Q_hist, rope_cos_ev, rope_sin_ev)


def hf_ring_step(cfg: hf_config, ring: hf_ring, Q, K_cache, V_cache, step_in_chunk: int, block_idx, state, O, workspace,
                 rope_cos_q=None, rope_sin_q=None, Q_hist=None) -> None:
    """Selection and hybrid attention of one denoising step over the ring's valid tokens, in storage order."""
    _call().ring_step(cfg, ring, Q, K_cache, V_cache, step_in_chunk, block_idx, state, O, workspace, rope_cos_q, rope_sin_q, Q_hist)


def hf_bwd_workspace_bytes(cfg: hf_config, n_q: int, n_kv: int) -> int:
    out = ctypes.c_size_t(0)
    _check(load().hf_bwd_workspace_bytes(ctypes.byref(cfg), n_q, n_kv, ctypes.byref(out)))
    return out.value


def hf_bwd_least_workspace_bytes(cfg: hf_config, n_q: int, n_kv: int) -> int:
    """The least that hf_hybrid_attn_bwd takes (hf_bwd_workspace_bytes: what it makes use of)."""
    out = ctypes.c_size_t(0)
    _check(load().hf_bwd_least_workspace_bytes(ctypes.byref(cfg), n_q, n_kv, ctypes.byref(out)))
    return out.value


def hf_hybrid_attn_bwd(cfg: hf_config, Q, K_win, V_win, block_idx, state, dO, dQ, dK, dV, workspace,
                       rope_cos_q=None, rope_sin_q=None, Q_hist=None, dQ_hist=None, n_kv=None) -> None:
    """Gradients of hf_hybrid_attn_fwd's output with respect to Q (and Q_hist), K_win, V_win for a fixed mask
    and a constant state.  dK, dV are laid out like K_win, V_win."""
    _call().hybrid_attn_bwd(cfg, Q, K_win, V_win, block_idx, state, dO, dQ, dK, dV, workspace, rope_cos_q, rope_sin_q, Q_hist,
                            dQ_hist, n_kv)


def hf_hybrid_attn_bwd_saved(cfg: hf_config, Q, K_win, V_win, block_idx, state, dO, O_local, lse2, dQ, dK, dV, workspace,
                             rope_cos_q=None, rope_sin_q=None, Q_hist=None, dQ_hist=None, n_kv=None) -> None:
    """hf_hybrid_attn_bwd from O_local and lse2 as hf_hybrid_attn_fwd_save wrote them (no recomputed forward)."""
    _call().hybrid_attn_bwd_saved(cfg, Q, K_win, V_win, block_idx, state, dO, O_local, lse2, dQ, dK, dV, workspace, rope_cos_q,
                                  rope_sin_q, Q_hist, dQ_hist, n_kv)
