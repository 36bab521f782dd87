"""Python binding of libentropyinfer.so (argument marshalling only).

Every function takes torch tensors that already live on a ROCm device, checks
dtype / shape / contiguity, and passes raw device pointers plus the current
HIP stream to the C ABI of the same name (``include/entropyinfer.h``).  All
arithmetic runs in the library's HIP kernels; there is no fallback: if the
library is missing or a call fails, an exception is raised.
"""
from __future__ import annotations

import contextlib
import ctypes
import functools
import math
import operator
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libentropyinfer.so")

EI_OK = 0
_STATUS = {0: "EI_OK", -1: "EI_ERR_NULL", -2: "EI_ERR_SHAPE", -3: "EI_ERR_UNSUPPORTED",
           -4: "EI_ERR_WORKSPACE", -5: "EI_ERR_LAUNCH"}


class Dims(ctypes.Structure):
    _fields_ = [("batch", ctypes.c_int32), ("n_q_heads", ctypes.c_int32),
                ("n_kv_heads", ctypes.c_int32), ("seq_len", ctypes.c_int32),
                ("head_dim", ctypes.c_int32)]


class Tiling(ctypes.Structure):
    _fields_ = [("seg_len", ctypes.c_int32), ("block_len", ctypes.c_int32)]


class BudgetParams(ctypes.Structure):
    _fields_ = [("entropy_threshold", ctypes.c_float), ("alpha", ctypes.c_double),
                ("delta_t", ctypes.c_double), ("base_budget_tokens", ctypes.c_int32),
                ("max_budget_mult", ctypes.c_int32)]


class EIError(RuntimeError):
    def __init__(self, fn: str, status: int, text: str):
        super().__init__(f"{fn} returned {status} ({_STATUS.get(status, '?')}): {text}")
        self.status = status


_LIB = None
_VP = ctypes.c_void_p


def lib() -> ctypes.CDLL:
    """Load libentropyinfer.so (built in-tree by ``build.py``); raise if absent."""
    global _LIB
    if _LIB is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is not built; run paper_2606_09508_amd/build.py "
                               "(or __graft_entry__.build()) first")
        L = ctypes.CDLL(LIB_PATH)
        L.ei_abi_version.restype = ctypes.c_int32
        L.ei_status_str.restype = ctypes.c_char_p
        L.ei_status_str.argtypes = [ctypes.c_int]
        L.ei_num_segments.restype = ctypes.c_int64
        L.ei_num_segments.argtypes = [Dims, Tiling]
        L.ei_num_blocks.restype = ctypes.c_int64
        L.ei_num_blocks.argtypes = [Dims, Tiling]
        L.ei_kmax.restype = ctypes.c_int32
        L.ei_kmax.argtypes = [Tiling, BudgetParams]
        L.ei_probe_workspace_bytes.restype = ctypes.c_size_t
        L.ei_probe_workspace_bytes.argtypes = [Dims, Tiling]
        L.ei_entropy_probe.restype = ctypes.c_int
        L.ei_entropy_probe.argtypes = [_VP, _VP, Dims, Tiling, ctypes.c_double, _VP, _VP, _VP,
                                       ctypes.c_size_t, _VP]
        L.ei_select_blocks.restype = ctypes.c_int
        L.ei_select_blocks.argtypes = [_VP, _VP, Dims, Tiling, BudgetParams, ctypes.c_int32, _VP,
                                       _VP, _VP, _VP, _VP]
        L.ei_select_blocks_mode.restype = ctypes.c_int
        L.ei_select_blocks_mode.argtypes = [_VP, _VP, Dims, Tiling, BudgetParams, ctypes.c_int32,
                                            ctypes.c_int32, _VP, _VP, _VP, _VP, _VP]
        L.ei_probe_select_workspace_bytes.restype = ctypes.c_size_t
        L.ei_probe_select_workspace_bytes.argtypes = [Dims, Tiling]
        L.ei_probe_select_fused.restype = ctypes.c_int
        L.ei_probe_select_fused.argtypes = [_VP, _VP, Dims, Tiling, ctypes.c_double, BudgetParams,
                                            ctypes.c_int32, ctypes.c_int32, _VP, _VP, _VP, _VP,
                                            _VP, _VP, ctypes.c_size_t, _VP]
        L.ei_sparse_prefill_attn.restype = ctypes.c_int
        L.ei_sparse_prefill_attn.argtypes = [_VP, _VP, _VP, Dims, Tiling, ctypes.c_float, _VP,
                                             _VP, ctypes.c_int32, _VP, _VP, ctypes.c_size_t,
                                             _VP]
        L.ei_prefill_workspace_bytes.restype = ctypes.c_size_t
        L.ei_prefill_workspace_bytes.argtypes = [Dims, Tiling]
        L.ei_entropy_guided_prefill.restype = ctypes.c_int
        L.ei_entropy_guided_prefill.argtypes = [_VP, _VP, _VP, Dims, Tiling, ctypes.c_double,
                                                BudgetParams, ctypes.c_int32, ctypes.c_int32,
                                                ctypes.c_float, _VP, _VP, _VP, _VP, _VP, _VP,
                                                _VP, _VP, ctypes.c_size_t, _VP]
        L.ei_entropy_guided_prefill_noalloc.restype = ctypes.c_int
        L.ei_entropy_guided_prefill_noalloc.argtypes = [
            _VP, _VP, _VP, Dims, Tiling, ctypes.c_double, BudgetParams, ctypes.c_int32,
            ctypes.c_int32, ctypes.c_float, _VP, _VP, _VP, _VP, _VP, _VP, _VP, _VP]
        L.ei_sparse_prefill_attn_gqa_union.restype = ctypes.c_int
        L.ei_sparse_prefill_attn_gqa_union.argtypes = [_VP, _VP, _VP, Dims, Tiling,
                                                       ctypes.c_float, _VP, _VP, ctypes.c_int32,
                                                       _VP, _VP]
        L.ei_dense_prefill_attn.restype = ctypes.c_int
        L.ei_dense_prefill_attn.argtypes = [_VP, _VP, _VP, Dims, ctypes.c_float, ctypes.c_int32,
                                            _VP, _VP]
        L.ei_add_rmsnorm.restype = ctypes.c_int
        L.ei_add_rmsnorm.argtypes = [_VP, _VP, _VP, ctypes.c_int64, ctypes.c_int32, ctypes.c_float,
                                     _VP, _VP, _VP]
        L.ei_rope_heads.restype = ctypes.c_int
        L.ei_rope_heads.argtypes = [_VP, _VP, _VP, _VP, _VP, Dims, _VP, _VP, _VP, _VP]
        L.ei_rope_tables.restype = ctypes.c_int
        L.ei_rope_tables.argtypes = [ctypes.c_int32, ctypes.c_int32, ctypes.c_float, _VP, _VP, _VP]
        L.ei_swiglu.restype = ctypes.c_int
        L.ei_swiglu.argtypes = [_VP, _VP, ctypes.c_int64, _VP, _VP]
        _LIB = L
    return _LIB


def _check(fn: str, st: int) -> None:
    if st != EI_OK:
        raise EIError(fn, st, lib().ei_status_str(st).decode())


# A call's host side is part of what a short prompt waits for (a 100-token
# layer is ~10 library calls of a few us of GPU time each), so the checks below
# take one test in the good case, the stream comes as the raw handle, and the
# device is switched only where it is not the current one (a small dense call
# 12.7 -> 8.7 us, sparse attention 15.8 -> 11.1, a selection 22.1 -> 16.7, two
# small decoder layers with logits 665 -> 601).
def _ptr(t):
    return None if t is None else t.data_ptr()


def _stream(t: torch.Tensor) -> int:
    return torch._C._cuda_getCurrentRawStream(t.get_device())


_HERE_ALREADY = contextlib.nullcontext()


def _on(t: torch.Tensor):
    """Context with t's device current."""
    if torch._C._cuda_getDevice() == t.get_device():
        return _HERE_ALREADY
    return torch.cuda.device(t.device)


def _req(t: torch.Tensor, name: str, dtype, ndim: int) -> None:
    if isinstance(t, torch.Tensor) and t.is_cuda and t.dtype is dtype and t.dim() == ndim \
            and t.is_contiguous():
        return
    if not isinstance(t, torch.Tensor):
        raise TypeError(f"{name} must be a torch.Tensor")
    if t.device.type != "cuda":
        raise ValueError(f"{name} must be on a ROCm device, got {t.device}")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    raise ValueError(f"{name} must be a contiguous {ndim}-d tensor, got {tuple(t.shape)}")


def check_qkv_shapes(q_shape, k_shape, v_shape=None) -> None:
    """q [B, Hq, N, D], k (and v) [B, Hkv, N, D] with Hkv dividing Hq: the C
    ABI takes every size from q and Hkv, so k / v must match them exactly."""
    if len(q_shape) != 4 or len(k_shape) != 4:
        raise ValueError("q and k must be 4-d [B, H, N, D]")
    B, Hq, N, D = q_shape
    if (k_shape[0], k_shape[2], k_shape[3]) != (B, N, D):
        raise ValueError(f"k {tuple(k_shape)} does not match q {tuple(q_shape)} in B, N or D")
    if k_shape[1] <= 0 or Hq % k_shape[1]:
        raise ValueError(f"the {k_shape[1]} KV heads must divide the {Hq} query heads")
    if v_shape is not None and tuple(v_shape) != tuple(k_shape):
        raise ValueError(f"v {tuple(v_shape)} does not match k {tuple(k_shape)}")


def check_score_shapes(ls_shape, en_shape, seq_len: int, seg_len: int, block_len: int) -> None:
    """log_scores [B, Hq, C_S, C_B] and entropy [B, Hq, C_S] for seq_len
    tokens: the kernels size every row from seq_len."""
    CS = -(-seq_len // seg_len) if seg_len > 0 else -1
    CB = -(-seq_len // block_len) if block_len > 0 else -1
    if len(ls_shape) != 4 or tuple(ls_shape[2:]) != (CS, CB):
        raise ValueError(f"log_scores {tuple(ls_shape)} is not [B, Hq, {CS}, {CB}]")
    if tuple(en_shape) != tuple(ls_shape[:3]):
        raise ValueError(f"entropy {tuple(en_shape)} is not {tuple(ls_shape[:3])}")


def _same_device(*ts) -> None:
    dev = ts[0].device
    for t in ts[1:]:
        if t is not None and t.device != dev:
            raise ValueError(f"tensors on different devices: {dev} and {t.device}")


def dims_of(q: torch.Tensor, k: torch.Tensor) -> Dims:
    B, Hq, N, D = q.shape
    return Dims(B, Hq, k.shape[1], N, D)


def budget_params(e_t: float = 1e-5, alpha: float = 0.5, delta_t: float = 0.4,
                  base_budget: int = 2048, mult: int = 3) -> BudgetParams:
    return BudgetParams(float(e_t), float(alpha), float(delta_t), int(base_budget), int(mult))


def num_segments(N: int, seg_len: int) -> int:
    return -(-N // seg_len)


def num_blocks(N: int, block_len: int) -> int:
    return -(-N // block_len)


@functools.lru_cache(maxsize=256)   # a pure function of four plain integers
def _kmax(seg_len: int, block_len: int, base_budget: int, mult: int) -> int:
    v = lib().ei_kmax(Tiling(seg_len, block_len), budget_params(base_budget=base_budget, mult=mult))
    if v < 0:
        raise ValueError("invalid tiling or budget parameters")
    return v


def kmax(seg_len: int, block_len: int, base_budget: int = 2048, mult: int = 3) -> int:
    # (numbers of other kinds, arrays and tensors among them, by their value)
    return _kmax(operator.index(seg_len), operator.index(block_len), int(base_budget), int(mult))


def probe_workspace_bytes(dims: Dims, seg_len: int, block_len: int) -> int:
    return int(lib().ei_probe_workspace_bytes(dims, Tiling(seg_len, block_len)))


def entropy_probe(q, k, seg_len: int, block_len: int, probe_scale: float = 1.0,
                  log_scores=None, entropy=None, workspace=None):
    """ei_entropy_probe: returns (log_scores fp32 [B,Hq,C_S,C_B], entropy fp32 [B,Hq,C_S])."""
    _req(q, "q", torch.bfloat16, 4)
    _req(k, "k", torch.bfloat16, 4)
    check_qkv_shapes(q.shape, k.shape)
    d = dims_of(q, k)
    CS, CB = num_segments(d.seq_len, seg_len), num_blocks(d.seq_len, block_len)
    dev = q.device
    if log_scores is None:
        log_scores = torch.empty((d.batch, d.n_q_heads, CS, CB), dtype=torch.float32, device=dev)
    if entropy is None:
        entropy = torch.empty((d.batch, d.n_q_heads, CS), dtype=torch.float32, device=dev)
    _req(log_scores, "log_scores", torch.float32, 4)
    _req(entropy, "entropy", torch.float32, 3)
    if tuple(log_scores.shape) != (d.batch, d.n_q_heads, CS, CB) or \
            tuple(entropy.shape) != (d.batch, d.n_q_heads, CS):
        raise ValueError("log_scores / entropy have the wrong shape")
    need = probe_workspace_bytes(d, seg_len, block_len)
    if workspace is None:
        workspace = torch.empty((max(need, 1),), dtype=torch.uint8, device=dev)
    _same_device(q, k, log_scores, entropy, workspace)
    with _on(q):
        st = lib().ei_entropy_probe(_ptr(q), _ptr(k), d, Tiling(seg_len, block_len),
                                    float(probe_scale), _ptr(log_scores), _ptr(entropy),
                                    _ptr(workspace), workspace.numel() * workspace.element_size(),
                                    _stream(q))
    _check("ei_entropy_probe", st)
    return log_scores, entropy


CLASSIFY_HEAD, CLASSIFY_GQA_GROUP, CLASSIFY_SEGMENT = 0, 1, 2   # ei_classify_mode


def select_blocks(log_scores, entropy, seq_len: int, seg_len: int, block_len: int,
                  e_t: float = 1e-5, alpha: float = 0.5, delta_t: float = 0.4,
                  base_budget: int = 2048, mult: int = 3, kmax_: int | None = None,
                  head_dim: int = 128, n_kv_heads: int | None = None, out: dict | None = None,
                  mode: int = CLASSIFY_HEAD):
    """ei_select_blocks_mode (mode CLASSIFY_HEAD is ei_select_blocks): returns
    dict(rigid u8 [B,Hq], budget i32 [B,Hq,C_S], idx i32 [B,Hq,C_S,kmax],
    cnt i32 [B,Hq,C_S])."""
    _req(log_scores, "log_scores", torch.float32, 4)
    _req(entropy, "entropy", torch.float32, 3)
    B, Hq, CS, CB = log_scores.shape
    p = budget_params(e_t, alpha, delta_t, base_budget, mult)
    km = kmax(seg_len, block_len, base_budget, mult) if kmax_ is None else int(kmax_)
    dev = log_scores.device
    if out is None:
        out = {"rigid": torch.empty((B, Hq), dtype=torch.uint8, device=dev),
               "budget": torch.empty((B, Hq, CS), dtype=torch.int32, device=dev),
               "idx": torch.empty((B, Hq, CS, km), dtype=torch.int32, device=dev),
               "cnt": torch.empty((B, Hq, CS), dtype=torch.int32, device=dev)}
    _req(out["rigid"], "rigid", torch.uint8, 2)
    _req(out["budget"], "budget", torch.int32, 3)
    _req(out["idx"], "idx", torch.int32, 4)
    _req(out["cnt"], "cnt", torch.int32, 3)
    check_score_shapes(log_scores.shape, entropy.shape, seq_len, seg_len, block_len)
    if tuple(out["rigid"].shape) != (B, Hq) or tuple(out["budget"].shape) != (B, Hq, CS) or \
            tuple(out["idx"].shape) != (B, Hq, CS, km) or tuple(out["cnt"].shape) != (B, Hq, CS):
        raise ValueError("rigid / budget / idx / cnt do not match [B, Hq], [B, Hq, C_S], "
                         "[B, Hq, C_S, kmax], [B, Hq, C_S]")
    _same_device(log_scores, entropy, *out.values())
    d = Dims(B, Hq, Hq if n_kv_heads is None else n_kv_heads, seq_len, head_dim)
    with _on(log_scores):
        st = lib().ei_select_blocks_mode(_ptr(log_scores), _ptr(entropy), d,
                                         Tiling(seg_len, block_len), p, int(mode), km,
                                         _ptr(out["rigid"]), _ptr(out["budget"]),
                                         _ptr(out["idx"]), _ptr(out["cnt"]), _stream(log_scores))
    _check("ei_select_blocks_mode", st)
    return out


def probe_select_workspace_bytes(dims: Dims, seg_len: int, block_len: int) -> int:
    return int(lib().ei_probe_select_workspace_bytes(dims, Tiling(seg_len, block_len)))


def probe_select_fused(q, k, seg_len: int, block_len: int, e_t: float = 1e-5,
                       alpha: float = 0.5, delta_t: float = 0.4, base_budget: int = 2048,
                       mult: int = 3, probe_scale: float = 1.0, mode: int = CLASSIFY_HEAD,
                       kmax_: int | None = None, bufs: dict | None = None):
    """ei_probe_select_fused (probe and selection without ln A in memory):
    returns (entropy fp32 [B,Hq,C_S], dict(rigid, budget, idx, cnt) as
    select_blocks).  ``bufs`` (optional) caches the outputs and workspace."""
    _req(q, "q", torch.bfloat16, 4)
    _req(k, "k", torch.bfloat16, 4)
    check_qkv_shapes(q.shape, k.shape)
    _same_device(q, k)
    d = dims_of(q, k)
    B, Hq, N, _ = q.shape
    CS = num_segments(N, seg_len)
    km = kmax(seg_len, block_len, base_budget, mult) if kmax_ is None else int(kmax_)
    dev = q.device
    bufs = {} if bufs is None else bufs
    shapes = {"entropy": ((B, Hq, CS), torch.float32), "rigid": ((B, Hq), torch.uint8),
              "budget": ((B, Hq, CS), torch.int32), "idx": ((B, Hq, CS, km), torch.int32),
              "cnt": ((B, Hq, CS), torch.int32)}
    for name, (shape, dtype) in shapes.items():
        t = bufs.get(name)
        if t is None or tuple(t.shape) != shape or t.dtype != dtype or t.device != dev:
            bufs[name] = torch.empty(shape, dtype=dtype, device=dev)
    need = max(probe_select_workspace_bytes(d, seg_len, block_len), 1)
    ws = bufs.get("workspace")
    if ws is None or ws.numel() < need or ws.device != dev:
        bufs["workspace"] = ws = torch.empty((need,), dtype=torch.uint8, device=dev)
    with _on(q):
        st = lib().ei_probe_select_fused(
            _ptr(q), _ptr(k), d, Tiling(seg_len, block_len), float(probe_scale),
            budget_params(e_t, alpha, delta_t, base_budget, mult), int(mode), km,
            _ptr(bufs["entropy"]), _ptr(bufs["rigid"]), _ptr(bufs["budget"]), _ptr(bufs["idx"]),
            _ptr(bufs["cnt"]), _ptr(ws), ws.numel(), _stream(q))
    _check("ei_probe_select_fused", st)
    return bufs["entropy"], {n: bufs[n] for n in ("rigid", "budget", "idx", "cnt")}


ATTN_WORKSPACE_BYTES = 256   # EI_ATTN_WORKSPACE_BYTES


def sparse_prefill_attn(q, k, v, block_idx, block_cnt, seg_len: int, block_len: int,
                        softmax_scale: float | None = None, out=None, gqa_union: bool = False,
                        persistent: bool = True, workspace=None):
    """ei_sparse_prefill_attn (or, with gqa_union, ei_sparse_prefill_attn_gqa_union,
    bitwise the same result): bf16 [B,Hq,N,D] output.  `persistent` passes a
    scheduling workspace (`workspace`, or a new ATTN_WORKSPACE_BYTES one), which
    selects the persistent grid; False passes none (the static grid)."""
    for t, n in ((q, "q"), (k, "k"), (v, "v")):
        _req(t, n, torch.bfloat16, 4)
    _req(block_idx, "block_idx", torch.int32, 4)
    _req(block_cnt, "block_cnt", torch.int32, 3)
    check_qkv_shapes(q.shape, k.shape, v.shape)
    d = dims_of(q, k)
    if out is None:
        out = torch.empty_like(q)
    _req(out, "out", torch.bfloat16, 4)
    if k.shape != v.shape or tuple(out.shape) != tuple(q.shape):
        raise ValueError("k / v / out shapes do not match q")
    CS = num_segments(d.seq_len, seg_len)
    if tuple(block_idx.shape[:3]) != (d.batch, d.n_q_heads, CS) or \
            tuple(block_cnt.shape) != (d.batch, d.n_q_heads, CS):
        raise ValueError("block_idx / block_cnt do not match [B, Hq, C_S]")
    sc = 1.0 / math.sqrt(d.head_dim) if softmax_scale is None else float(softmax_scale)
    _same_device(q, k, v, block_idx, block_cnt, out)
    if persistent and not gqa_union and workspace is None:
        workspace = torch.empty((ATTN_WORKSPACE_BYTES,), dtype=torch.uint8, device=q.device)
    if workspace is not None:
        _same_device(q, workspace)
    with _on(q):
        args = [_ptr(q), _ptr(k), _ptr(v), d, Tiling(seg_len, block_len), sc, _ptr(block_idx),
                _ptr(block_cnt), int(block_idx.shape[-1]), _ptr(out)]
        if gqa_union:
            fn = "ei_sparse_prefill_attn_gqa_union"
            st = lib().ei_sparse_prefill_attn_gqa_union(*args, _stream(q))
        else:
            fn = "ei_sparse_prefill_attn"
            ws = workspace if persistent else None
            nb = ws.numel() * ws.element_size() if ws is not None else 0
            st = lib().ei_sparse_prefill_attn(*args, _ptr(ws) if ws is not None else None, nb,
                                              _stream(q))
    _check(fn, st)
    return out


def dense_prefill_attn(q, k, v, softmax_scale: float | None = None, causal: bool = True,
                       out=None):
    """ei_dense_prefill_attn: bf16 [B,Hq,N,D] output."""
    for t, n in ((q, "q"), (k, "k"), (v, "v")):
        _req(t, n, torch.bfloat16, 4)
    check_qkv_shapes(q.shape, k.shape, v.shape)
    d = dims_of(q, k)
    if out is None:
        out = torch.empty_like(q)
    _req(out, "out", torch.bfloat16, 4)
    if k.shape != v.shape or tuple(out.shape) != tuple(q.shape):
        raise ValueError("k / v / out shapes do not match q")
    sc = 1.0 / math.sqrt(d.head_dim) if softmax_scale is None else float(softmax_scale)
    _same_device(q, k, v, out)
    with _on(q):
        st = lib().ei_dense_prefill_attn(_ptr(q), _ptr(k), _ptr(v), d, sc, 1 if causal else 0,
                                         _ptr(out), _stream(q))
    _check("ei_dense_prefill_attn", st)
    return out


def prefill_workspace_bytes(dims: Dims, seg_len: int, block_len: int) -> int:
    return int(lib().ei_prefill_workspace_bytes(dims, Tiling(seg_len, block_len)))


def entropy_guided_prefill(q, k, v, seg_len: int = 128, block_len: int = 64,
                           base_budget: int = 2048, e_t: float = 1e-5, alpha: float = 0.5,
                           delta_t: float = 0.4, mult: int = 3, probe_scale: float = 1.0,
                           softmax_scale: float | None = None, bufs: dict | None = None,
                           mode: int = CLASSIFY_HEAD, noalloc: bool = False):
    """ei_entropy_guided_prefill: the whole path on one layer (probe -> select
    -> sparse attention) on the current stream.  ``bufs`` (optional) caches
    the output and scratch buffers between calls.  Returns (output, selection
    dict, log_scores, entropy).  With ``noalloc`` the call goes to
    ei_entropy_guided_prefill_noalloc (no workspace: the library's static
    scratch array)."""
    for t, n in ((q, "q"), (k, "k"), (v, "v")):
        _req(t, n, torch.bfloat16, 4)
    check_qkv_shapes(q.shape, k.shape, v.shape)
    _same_device(q, k, v)
    d = dims_of(q, k)
    B, Hq, N, D = q.shape
    CS, CB = num_segments(N, seg_len), num_blocks(N, block_len)
    km = kmax(seg_len, block_len, base_budget, mult)
    dev = q.device
    bufs = {} if bufs is None else bufs
    rows = (B, Hq, CS)
    for name, shape, dtype in (("log_scores", (B, Hq, CS, CB), torch.float32),
                               ("entropy", rows, torch.float32), ("rigid", (B, Hq), torch.uint8),
                               ("budget", rows, torch.int32), ("idx", (B, Hq, CS, km), torch.int32),
                               ("cnt", rows, torch.int32), ("out", q.shape, torch.bfloat16)):
        t = bufs.get(name)
        if t is None or t.shape != shape or t.dtype != dtype or t.device != dev:
            bufs[name] = torch.empty(shape, dtype=dtype, device=dev)
    if not noalloc:
        need = max(prefill_workspace_bytes(d, seg_len, block_len), 1)
        ws = bufs.get("workspace")
        if ws is None or ws.numel() < need or ws.device != dev:
            bufs["workspace"] = ws = torch.empty((need,), dtype=torch.uint8, device=dev)
    scale = (1.0 / math.sqrt(D)) if softmax_scale is None else float(softmax_scale)
    args = (_ptr(q), _ptr(k), _ptr(v), d, Tiling(seg_len, block_len), float(probe_scale),
            budget_params(e_t, alpha, delta_t, base_budget, mult), int(mode), km, scale,
            _ptr(bufs["log_scores"]), _ptr(bufs["entropy"]), _ptr(bufs["rigid"]),
            _ptr(bufs["budget"]), _ptr(bufs["idx"]), _ptr(bufs["cnt"]), _ptr(bufs["out"]))
    with _on(q):
        if noalloc:
            fn = "ei_entropy_guided_prefill_noalloc"
            st = lib().ei_entropy_guided_prefill_noalloc(*args, _stream(q))
        else:
            fn = "ei_entropy_guided_prefill"
            st = lib().ei_entropy_guided_prefill(*args, _ptr(ws), ws.numel(), _stream(q))
    _check(fn, st)
    sel = {n: bufs[n] for n in ("rigid", "budget", "idx", "cnt")}
    return bufs["out"], sel, bufs["log_scores"], bufs["entropy"]


def add_rmsnorm(x, y, gain, eps: float):
    """ei_add_rmsnorm over the last dimension of x (bf16, contiguous): returns
    (x + y, its RMSNorm times gain), or (x, norm of x) when y is None."""
    _req(x, "x", torch.bfloat16, x.dim())
    _req(gain, "gain", torch.bfloat16, 1)
    cols = x.shape[-1]
    if gain.numel() != cols:
        raise ValueError(f"gain has {gain.numel()} elements for {cols} columns")
    if y is not None:
        _req(y, "y", torch.bfloat16, x.dim())
        if y.shape != x.shape:
            raise ValueError(f"y {tuple(y.shape)} does not match x {tuple(x.shape)}")
    _same_device(x, gain, y)
    s = x if y is None else torch.empty_like(x)
    out = torch.empty_like(x)
    with _on(x):
        st = lib().ei_add_rmsnorm(_ptr(x), _ptr(y), _ptr(gain), x.numel() // cols, cols, float(eps),
                                  _ptr(s), _ptr(out), _stream(x))
    _check("ei_add_rmsnorm", st)
    return s, out


def rope_heads(q, k, v, cos, sin):
    """ei_rope_heads: q [B, N, Hq, D], k and v [B, N, Hkv, D] (bf16) to
    head-major [B, H, N, D], q and k rotated by the tables cos / sin [N, D/2]."""
    for t, n in ((q, "q"), (k, "k"), (v, "v")):
        _req(t, n, torch.bfloat16, 4)
    B, N, Hq, D = q.shape
    Hkv = k.shape[2]
    if tuple(k.shape) != (B, N, Hkv, D) or v.shape != k.shape or Hkv <= 0 or Hq % Hkv:
        raise ValueError(f"k {tuple(k.shape)} / v {tuple(v.shape)} do not match q {tuple(q.shape)}")
    for t, n in ((cos, "cos"), (sin, "sin")):
        _req(t, n, torch.float32, 2)
        if tuple(t.shape) != (N, D // 2):
            raise ValueError(f"{n} {tuple(t.shape)} is not [{N}, {D // 2}]")
    _same_device(q, k, v, cos, sin)
    out = [torch.empty((B, t.shape[2], N, D), dtype=t.dtype, device=t.device) for t in (q, k, v)]
    with _on(q):
        st = lib().ei_rope_heads(_ptr(q), _ptr(k), _ptr(v), _ptr(cos), _ptr(sin),
                                 Dims(B, Hq, Hkv, N, D), *(_ptr(t) for t in out), _stream(q))
    _check("ei_rope_heads", st)
    return out


def rope_tables(cos, sin, head_dim: int, theta: float) -> None:
    """ei_rope_tables: fills cos and sin [N, ceil(head_dim / 2)] (fp32)."""
    for t, n in ((cos, "cos"), (sin, "sin")):
        _req(t, n, torch.float32, 2)
        if t.shape != cos.shape or t.shape[1] != (head_dim + 1) // 2:
            raise ValueError(f"{n} {tuple(t.shape)} is not [N, {(head_dim + 1) // 2}]")
    _same_device(cos, sin)
    with _on(cos):
        st = lib().ei_rope_tables(cos.shape[0], head_dim, float(theta), _ptr(cos), _ptr(sin),
                                  _stream(cos))
    _check("ei_rope_tables", st)


def swiglu(g, u, out=None):
    """ei_swiglu: silu(g) * u (bf16, contiguous); ``out`` may be g or u."""
    _req(g, "g", torch.bfloat16, g.dim())
    _req(u, "u", torch.bfloat16, g.dim())
    out = torch.empty_like(g) if out is None else out
    _req(out, "out", torch.bfloat16, g.dim())
    if u.shape != g.shape or out.shape != g.shape:
        raise ValueError("g / u / out shapes differ")
    _same_device(g, u, out)
    with _on(g):
        st = lib().ei_swiglu(_ptr(g), _ptr(u), g.numel(), _ptr(out), _stream(g))
    _check("ei_swiglu", st)
    return out
