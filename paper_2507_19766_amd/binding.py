"""Binding of libulorl: argument marshalling only.

Every function here has the name of the C entry point it wraps (minus the ``ulorl_`` prefix)
and does nothing but check tensors (device, dtype, contiguity), allocate outputs with torch
and pass raw pointers plus the current HIP stream; the calls of a training step do that in an extension module
(``csrc/torch_marshal.cpp``), the rest through ctypes.  All arithmetic of these calls runs in the HIP kernels.
"""
from __future__ import annotations

import ctypes
import importlib.util
import os
from dataclasses import dataclass
from typing import Optional

import torch

F32, BF16 = 0, 1
IS_SAIS, IS_POIS = 0, 1
GATE_PER_RESPONSE, GATE_GLOBAL, GATE_ALWAYS, GATE_NEVER = 0, 1, 2, 3
STATUS_BAD_TOKEN, STATUS_NONFINITE, STATUS_BAD_CU, STATUS_SYNC = 1, 2, 4, 8
LAUNCH_PER_ROW = 1
LAUNCH_DENSE_ROWS = 2

_HERE = os.path.dirname(os.path.abspath(__file__))


class UlorlError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__("%s: %s (status %d)" % (where, status_string(status), status))


class _CParams(ctypes.Structure):
    _fields_ = [("eps_low", ctypes.c_float), ("eps_high", ctypes.c_float),
                ("tau", ctypes.c_float), ("sigma", ctypes.c_float),
                ("is_mode", ctypes.c_int32), ("gate_mode", ctypes.c_int32),
                ("seg_len", ctypes.c_int32), ("reserved", ctypes.c_int32),
                ("denominator", ctypes.c_double)]


class _CLaunch(ctypes.Structure):
    _fields_ = [("flags", ctypes.c_uint32), ("sync_spins", ctypes.c_int32), ("gemm_tile", ctypes.c_int32),
                ("gemm_group_m", ctypes.c_int32), ("reserved", ctypes.c_int32 * 4)]


class _CSegStats(ctypes.Structure):
    _fields_ = [("K", ctypes.c_int32), ("reserved", ctypes.c_int32),
                ("count", ctypes.c_void_p), ("ratio_sum", ctypes.c_void_p), ("ratio_max", ctypes.c_void_p),
                ("clipped", ctypes.c_void_p), ("kl_sum", ctypes.c_void_p), ("ent_sum", ctypes.c_void_p),
                ("masked", ctypes.c_void_p), ("out_of_range", ctypes.c_void_p),
                ("workspace", ctypes.c_void_p), ("workspace_bytes", ctypes.c_size_t)]


@dataclass
class Launch:
    """Per-call launch options (ulorl_launch); the defaults are the library's."""
    per_row: bool = False
    dense_rows: bool = False
    sync_spins: int = 0
    gemm_tile: int = 0
    gemm_group_m: int = 0

    def to_c(self) -> _CLaunch:
        return _CLaunch((LAUNCH_PER_ROW if self.per_row else 0) | (LAUNCH_DENSE_ROWS if self.dense_rows else 0), self.sync_spins, self.gemm_tile, self.gemm_group_m,
                        (ctypes.c_int32 * 4)(0, 0, 0, 0))


def _launch_ref(launch: Optional["Launch"]):
    """(pointer argument, object to keep alive) for an optional Launch."""
    if launch is None:
        return None, None
    c = launch.to_c()
    return ctypes.byref(c), c


@dataclass
class Params:
    """Scalar parameters; defaults are the paper's (tau = 0.99, sigma = 0.2, Sec. 4.1)."""
    eps_low: float = 0.2
    eps_high: float = 0.2
    tau: float = 0.99
    sigma: float = 0.2
    is_mode: int = IS_SAIS
    gate_mode: int = GATE_PER_RESPONSE
    seg_len: int = 0
    denominator: float = 0.0

    def to_c(self) -> _CParams:
        return _CParams(self.eps_low, self.eps_high, self.tau, self.sigma, self.is_mode,
                        self.gate_mode, self.seg_len, 0, self.denominator)


def _structs(params: Optional["Params"], launch: Optional["Launch"]):
    return (params or Params()).to_c(), launch.to_c() if launch is not None else None


def _addr(struct) -> int:
    return ctypes.addressof(struct) if struct is not None else 0


def lib_path() -> str:
    return os.path.join(_HERE, "lib", "libulorl.so")


_lib = None


def load_library(build_if_missing: bool = True):
    """Load lib/libulorl.so (building it once if it is absent)."""
    global _lib
    if _lib is not None:
        return _lib
    path = lib_path()
    if not os.path.exists(path):
        if not build_if_missing:
            raise FileNotFoundError(path)
        from . import build as _build
        _build.build()
    lib = ctypes.CDLL(path)
    c = ctypes
    lib.ulorl_version.restype = c.c_int32
    lib.ulorl_status_string.restype = c.c_char_p
    lib.ulorl_status_string.argtypes = [c.c_int32]
    lib.ulorl_token_loss_workspace_bytes.restype = c.c_size_t
    lib.ulorl_token_loss_workspace_bytes.argtypes = [c.c_int64, c.c_int64, c.c_int32]
    vp = c.c_void_p
    lib.ulorl_token_loss_fwd.restype = c.c_int32
    lib.ulorl_token_loss_fwd.argtypes = [
        vp, c.c_int32, c.c_int64, c.c_int64, c.c_int64,      # logits, dt, N, V, stride
        vp, vp, c.c_int32,                                   # token_ids, cu_seqlens, R
        vp, vp, vp,                                          # segment_ids, old_logp, advantages
        c.POINTER(_CParams),
        vp, vp, vp, vp, vp,                                  # loss, logp, entropy, lse, gcoef
        vp, vp, vp,                                          # mpt_mask, ratio, segment_out
        vp, vp, vp,                                          # resp_entropy, resp_gate, counters
        vp,                                                  # seg_stats
        vp, c.c_size_t, vp, vp]                              # workspace, bytes, launch, stream
    lib.ulorl_token_loss_fwd_bwd.restype = c.c_int32
    lib.ulorl_token_loss_fwd_bwd.argtypes = [
        vp, c.c_int32, c.c_int64, c.c_int64, c.c_int64,      # logits, dt, N, V, stride
        vp, vp, c.c_int32,                                   # token_ids, cu_seqlens, R
        vp, vp, vp,                                          # segment_ids, old_logp, advantages
        c.POINTER(_CParams), c.c_float,                      # params, grad_out
        vp, vp, vp, vp, vp,                                  # loss, logp, entropy, lse, gcoef
        vp, vp, vp,                                          # mpt_mask, ratio, segment_out
        vp, vp, vp,                                          # resp_entropy, resp_gate, counters
        vp,                                                  # seg_stats
        vp, vp, c.c_size_t, vp, vp]                          # dlogits, workspace, bytes, launch, stream
    lib.ulorl_init.restype = c.c_int32
    lib.ulorl_init.argtypes = []
    lib.ulorl_static_scratch_bytes.restype = c.c_size_t
    lib.ulorl_static_scratch_bytes.argtypes = []
    lib.ulorl_token_loss_fwd_bwd_static.restype = c.c_int32
    lib.ulorl_token_loss_fwd_bwd_static.argtypes = lib.ulorl_token_loss_fwd_bwd.argtypes[:-4] + [vp, vp]
    lib.ulorl_lmhead_workspace_bytes.restype = c.c_size_t
    lib.ulorl_lmhead_workspace_bytes.argtypes = [c.c_int64, c.c_int64, c.c_int64, c.c_int32, c.c_int32]
    lib.ulorl_lmhead_token_loss_fwd.restype = c.c_int32
    lib.ulorl_lmhead_token_loss_fwd.argtypes = [
        vp, vp, c.c_int64, c.c_int64, c.c_int64, c.c_int32,  # hidden, W, N, Hd, V, chunk
        vp, vp, c.c_int32, vp, vp, vp, c.POINTER(_CParams),
        vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp,
        vp, vp, c.c_size_t, vp, vp]                          # seg_stats, workspace, bytes, launch, stream
    lib.ulorl_lmhead_token_loss_bwd.restype = c.c_int32
    lib.ulorl_lmhead_token_loss_bwd.argtypes = [
        vp, vp, c.c_int64, c.c_int64, c.c_int64, c.c_int32, vp, vp, vp, c.c_float, vp, vp, vp, c.c_size_t, vp, vp]
    lib.ulorl_gemm_tn_bf16.restype = c.c_int32
    lib.ulorl_gemm_tn_bf16.argtypes = [vp, c.c_int64, vp, c.c_int64, c.c_int64, c.c_int64, c.c_int64, vp, c.c_int64, vp, vp]
    lib.ulorl_advantage_prep.restype = c.c_int32
    lib.ulorl_advantage_prep.argtypes = [vp, vp, vp, c.c_int32, c.c_int32, c.c_int64, c.c_float, c.c_int32,
                                         vp, vp, vp, vp, vp]
    lib.ulorl_segment_diagnostics_workspace_bytes.restype = c.c_size_t
    lib.ulorl_segment_diagnostics_workspace_bytes.argtypes = [c.c_int64, c.c_int32]
    lib.ulorl_segment_diagnostics.restype = c.c_int32
    lib.ulorl_segment_diagnostics.argtypes = [c.c_int64, c.c_int32, vp, vp, vp, vp, vp, vp, vp, c.c_float, c.c_float,
                                              vp, vp, vp, vp, vp, vp, vp, vp, vp, c.c_size_t, vp]
    lib.ulorl_segment_pool_step.restype = c.c_int32
    lib.ulorl_segment_pool_step.argtypes = [c.c_int32, vp, vp, vp, c.c_int32, c.c_int32, vp, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.ulorl_token_loss_bwd.restype = c.c_int32
    lib.ulorl_token_loss_bwd.argtypes = [
        vp, c.c_int32, c.c_int64, c.c_int64, c.c_int64, vp, vp, vp, c.c_float, vp, vp]
    _lib = lib
    return lib


def version() -> int:
    return int(load_library().ulorl_version())


def status_string(status: int) -> str:
    return load_library().ulorl_status_string(status).decode()


def token_loss_workspace_bytes(N: int, V: int, R: int) -> int:
    return int(load_library().ulorl_token_loss_workspace_bytes(N, V, R))


# ------------------------------------------------------------------------------------ helpers

_marshal = None


def native():
    """The extension module that turns tensors into arguments (lib/_marshal.so, built with the library if it is absent)."""
    global _marshal
    if _marshal is None:
        load_library()
        path = os.path.join(_HERE, "lib", "_marshal.so")
        if not os.path.exists(path):
            from . import build as _build
            _build.build()
        spec = importlib.util.spec_from_file_location("_marshal", path)
        module = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(module)
        module.set_status_error(UlorlError)
        _marshal = module
    return _marshal


def _p(t: Optional[torch.Tensor]):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _stream(dev) -> ctypes.c_void_p:
    return ctypes.c_void_p(torch.cuda.current_stream(dev).cuda_stream)


@dataclass
class FwdResult:
    loss: Optional[torch.Tensor]
    logp: torch.Tensor
    entropy: torch.Tensor
    lse: torch.Tensor
    gcoef: Optional[torch.Tensor] = None
    mpt_mask: Optional[torch.Tensor] = None
    ratio: Optional[torch.Tensor] = None
    segment_out: Optional[torch.Tensor] = None
    resp_entropy: Optional[torch.Tensor] = None
    resp_gate: Optional[torch.Tensor] = None
    counters: Optional[torch.Tensor] = None
    segment_stats: Optional[dict] = None      # per-segment diagnostics, when asked for (segments=K)


SEGMENT_FIELDS = ("count", "ratio_sum", "ratio_max", "clipped", "kl_sum", "ent_sum", "masked", "out_of_range", "_workspace")


def _fields(out: Optional[FwdResult], stats_only: bool):
    """A caller's tensors; a stats-only pass looks at the three that it writes."""
    if out is None:
        return None
    if stats_only:
        return [None, out.logp, out.entropy, out.lse] + [None] * 7
    return [out.loss, out.logp, out.entropy, out.lse, out.gcoef, out.mpt_mask, out.ratio, out.segment_out, out.resp_entropy,
            out.resp_gate, out.counters]


def _result(out: Optional[FwdResult], fields, segments, stats_only: bool = False) -> FwdResult:
    """The call's tensors as a FwdResult: a new one, or the caller's with what was missing filled in."""
    if out is None:
        out = FwdResult(*fields)
    elif not stats_only:
        (out.loss, out.logp, out.entropy, out.lse, out.gcoef, out.mpt_mask, out.ratio, out.segment_out, out.resp_entropy,
         out.resp_gate, out.counters) = fields
    if segments:
        out.segment_stats = dict(zip(SEGMENT_FIELDS, segments))
    return out


def token_loss_fwd(logits, token_ids, cu_seqlens, advantages, old_logp=None, params: Params = None,
                   segment_ids=None, out: Optional[FwdResult] = None,
                   workspace: Optional[torch.Tensor] = None, launch: Optional[Launch] = None,
                   segments: int = 0) -> FwdResult:
    """ulorl_token_loss_fwd.  ``advantages=None`` selects the stats-only pass.
    ``out``/``workspace`` let a caller reuse buffers (nothing is allocated then).
    ``segments=K`` asks for the per-segment diagnostics of ids 0..K-1 (``out.segment_stats``)."""
    with_params, with_launch = _structs(params, launch)
    fields, seg = native().token_loss_fwd(logits, token_ids, cu_seqlens, advantages, old_logp, segment_ids, _addr(with_params),
                                          _addr(with_launch), _fields(out, advantages is None), workspace, segments)
    return _result(out, fields, seg, advantages is None)


def token_loss_fwd_bwd(logits, token_ids, cu_seqlens, advantages, old_logp=None, params: Params = None,
                       segment_ids=None, grad_out: float = 1.0, dlogits: Optional[torch.Tensor] = None,
                       inplace: bool = False, out: Optional[FwdResult] = None,
                       workspace: Optional[torch.Tensor] = None, launch: Optional[Launch] = None,
                       segments: int = 0):
    """ulorl_token_loss_fwd_bwd -> (FwdResult, dlogits).  ``inplace=True`` overwrites ``logits``."""
    with_params, with_launch = _structs(params, launch)
    fields, seg, d = native().token_loss_fwd_bwd(logits, token_ids, cu_seqlens, advantages, old_logp, segment_ids, _addr(with_params),
                                                 _addr(with_launch), float(grad_out), dlogits, bool(inplace), False,
                                                 _fields(out, False), workspace, segments)
    return _result(out, fields, seg), d


def init() -> None:
    """ulorl_init: resolve the static scratch array of the current device (set-up time)."""
    rc = load_library().ulorl_init()
    if rc != 0:
        raise UlorlError(rc, "ulorl_init")


def static_scratch_bytes() -> int:
    return int(load_library().ulorl_static_scratch_bytes())


def token_loss_fwd_bwd_static(logits, token_ids, cu_seqlens, advantages, old_logp=None, params: Params = None,
                              segment_ids=None, grad_out: float = 1.0, dlogits: Optional[torch.Tensor] = None,
                              inplace: bool = False, out: Optional[FwdResult] = None,
                              launch: Optional[Launch] = None):
    """ulorl_token_loss_fwd_bwd_static -> (FwdResult, dlogits): the one-call path on the library's
    static scratch array (the C call allocates nothing; pass ``out`` and ``dlogits`` to keep this
    wrapper from allocating outputs either)."""
    with_params, with_launch = _structs(params, launch)
    fields, _, d = native().token_loss_fwd_bwd(logits, token_ids, cu_seqlens, advantages, old_logp, segment_ids, _addr(with_params),
                                               _addr(with_launch), float(grad_out), dlogits, bool(inplace), True,
                                               _fields(out, False), None, 0)
    return _result(out, fields, None), d


def row_stats(logits, token_ids, out: Optional[FwdResult] = None, launch: Optional[Launch] = None) -> FwdResult:
    """Stats-only forward: lse, chosen-token log-prob and entropy per row."""
    return token_loss_fwd(logits, token_ids, None, None, out=out, launch=launch)


def token_loss_bwd(logits, token_ids, lse, gcoef, grad_out: float = 1.0,
                   dlogits: Optional[torch.Tensor] = None, inplace: bool = False) -> torch.Tensor:
    """ulorl_token_loss_bwd.  ``inplace=True`` overwrites ``logits`` with the gradient."""
    return native().token_loss_bwd(logits, token_ids, lse, gcoef, float(grad_out), dlogits, bool(inplace))


# ------------------------------------------------------------------------------------ lm_head variant

def lmhead_workspace_bytes(N: int, Hd: int, V: int, R: int, vocab_chunk: int) -> int:
    return int(load_library().ulorl_lmhead_workspace_bytes(N, Hd, V, R, vocab_chunk))


def lmhead_token_loss_fwd(hidden, weight, token_ids, cu_seqlens, advantages, old_logp=None,
                          params: Params = None, segment_ids=None, vocab_chunk: int = 8192,
                          out: Optional[FwdResult] = None, workspace: Optional[torch.Tensor] = None,
                          launch: Optional[Launch] = None, segments: int = 0) -> FwdResult:
    """ulorl_lmhead_token_loss_fwd."""
    with_params, with_launch = _structs(params, launch)
    fields, seg = native().lmhead_fwd(hidden, weight, token_ids, cu_seqlens, advantages, old_logp, segment_ids, _addr(with_params),
                                      _addr(with_launch), vocab_chunk, _fields(out, advantages is None), workspace, segments)
    return _result(out, fields, seg, advantages is None)


def lmhead_token_loss_bwd(hidden, weight, token_ids, lse, gcoef, grad_out: float = 1.0, vocab_chunk: int = 8192,
                          d_hidden: Optional[torch.Tensor] = None, d_weight: Optional[torch.Tensor] = None,
                          workspace: Optional[torch.Tensor] = None, launch: Optional[Launch] = None):
    """ulorl_lmhead_token_loss_bwd -> (d_hidden [N, Hd] bf16, d_weight [Hd, V] bf16)."""
    with_launch = launch.to_c() if launch is not None else None
    return native().lmhead_bwd(hidden, weight, token_ids, lse, gcoef, float(grad_out), vocab_chunk, d_hidden, d_weight, workspace,
                               _addr(with_launch))


def gemm_tn_bf16(a: torch.Tensor, b: torch.Tensor, out: Optional[torch.Tensor] = None,
                 launch: Optional[Launch] = None) -> torch.Tensor:
    """ulorl_gemm_tn_bf16: a [M, K] . b [N, K]^T -> fp32 [M, N]."""
    lib = load_library()
    if not (a.is_cuda and b.is_cuda) or a.dtype != torch.bfloat16 or b.dtype != torch.bfloat16:
        raise TypeError("a and b must be bfloat16 device tensors")
    if a.dim() != 2 or b.dim() != 2 or a.stride(1) != 1 or b.stride(1) != 1 or a.shape[1] != b.shape[1]:
        raise ValueError("a is [M, K], b is [N, K], unit stride along K")
    M, K = a.shape
    N = b.shape[0]
    if out is None:
        out = torch.empty(M, N, dtype=torch.float32, device=a.device)
    lref, _keep = _launch_ref(launch)
    rc = lib.ulorl_gemm_tn_bf16(_p(a), a.stride(0), _p(b), b.stride(0), M, N, K, _p(out), out.stride(0), lref,
                                _stream(a.device))
    if rc != 0:
        raise UlorlError(rc, "ulorl_gemm_tn_bf16")
    return out


# ------------------------------------------------------------------------------------ neighbours of the hot path

def advantage_prep(rewards, cu_seqlens, group_size: int, truncated=None, eps: float = 1e-6, unbiased: bool = False):
    """ulorl_advantage_prep -> (resp_adv [R], group_keep [R/G], token_adv [N], kept_tokens [1] int64)."""
    return native().advantage_prep(rewards, truncated, cu_seqlens, group_size, float(eps), bool(unbiased))


def segment_diagnostics(res: FwdResult, advantages, old_logp, K: int, eps_low: float = 0.2, eps_high: float = 0.2,
                        segment_ids=None):
    """ulorl_segment_diagnostics on the outputs of a forward call -> dict of per-segment tensors."""
    seg = res.segment_out if segment_ids is None else segment_ids
    return dict(zip(SEGMENT_FIELDS[:-1], native().segment_diagnostics(K, seg, res.ratio, res.logp, old_logp, res.entropy, res.mpt_mask,
                                                                      advantages, float(eps_low), float(eps_high))))


def segment_pool_step(prev_len, new_len, hit_eos, seg_len: int, max_len: int):
    """ulorl_segment_pool_step -> dict of device tensors: state, total_len, segments [B];
    unfinished_idx, experience_idx, exp_truncated [B] and exp_cu_seqlens [B+1] (only the leading
    counts[0] / counts[1] (+1) entries are meaningful); counts [5] int64."""
    return dict(zip(("state", "total_len", "segments", "unfinished_idx", "experience_idx", "exp_cu_seqlens", "exp_truncated", "counts"),
                    native().segment_pool_step(prev_len, new_len, hit_eos, int(seg_len), int(max_len))))
