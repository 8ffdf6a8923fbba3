"""Binding of libpicospec.so with the same names as the C ABI (include/picospec.h).

Argument marshalling only: torch supplies device memory and the current stream, every step of
the path runs in the library's HIP kernels.  What runs on every call (tensors to pointers, outputs and
scratch, entering the C ABI) is native code (``_native``, csrc/native.cpp); ``lib`` is the library itself through ctypes.
Calls of few rows get scratch in which the library spreads every row over many workgroups (``scratch_bytes``): ids are the same
as with one workgroup per row, sums (probabilities, masses, statistics) agree to rounding, so their bits depend on the number of
rows in the call.  Scratch comes from torch's allocator on the current stream: capture such calls with ``torch.cuda.graph``, whose
pool keeps it for the replays.
Outputs that a call allocates by itself (the wire messages', sample_draft's, row_stats') share one allocation as far as they are
small (64 KB each): one that is kept keeps the other small ones of its call, torch.save writes them with it, and an in-place resize_
beyond its size runs into them; clone() it for any of these.  Larger outputs stand alone.
There is no fallback: if the library has not been built (``python -m paper_2603_19133_amd.build``) importing this module raises.
"""
from __future__ import annotations

import ctypes as C
import os
from dataclasses import dataclass

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libpicospec.so")

F32, BF16 = 0, 1
OK, EINVAL, EWORKSPACE, EDTYPE, EHIP, EUNSUPPORTED, ESCRATCH = 0, -1, -2, -3, -4, -5, -6
FLAG_TOKEN_NOT_IN_SUPPORT, FLAG_NONFINITE, FLAG_RESIDUAL_EMPTY, FLAG_BAD_INPUT = 1, 2, 4, 8
CALL_COMPRESS, CALL_SAMPLE_DRAFT, CALL_VERIFY, CALL_SAMPLE_RESIDUAL = 0, 1, 2, 3
CALL_COMPRESS_REJECTED, CALL_RESAMPLE_SPARSE, CALL_ROUND, CALL_VERIFY_SAMPLE, CALL_ROW_STATS = 4, 5, 6, 7, 8
LIMIT_MAX_K, LIMIT_MAX_V = 0, 1
WIRE_FP32, WIRE_FP16, WIRE_BF16 = 0, 1, 2
WIRE_BAD_HEADER, WIRE_BAD_BATCH, WIRE_CLAMPED, WIRE_TRUNCATED = 1, 2, 4, 8

EXPORTS = ("picospec_round", "picospec_verify_sample", "picospec_verify_sample_static", "picospec_static_scratch_bytes", "picospec_compress", "picospec_sample_draft", "picospec_verify", "picospec_verify_range", "picospec_sample_residual", "picospec_sample_residual_ws",
           "picospec_row_stats", "picospec_row_stats_ws", "picospec_compress_rejected", "picospec_resample_sparse",
           "picospec_pack_downlink", "picospec_unpack_downlink", "picospec_pack_uplink", "picospec_unpack_uplink",
           "picospec_downlink_bytes_max", "picospec_uplink_bytes", "picospec_max_load_byte", "picospec_check_device", "picospec_probe_clock",
           "picospec_workspace_bytes", "picospec_scratch_bytes", "picospec_one_launch_bytes", "picospec_limit", "picospec_strerror", "picospec_version")

if not os.path.exists(LIB_PATH):
    raise ImportError(f"{LIB_PATH} is missing: build it with `python -m paper_2603_19133_amd.build` "
                      "(there is no CPU fallback)")

lib = C.CDLL(LIB_PATH)

try:
    from . import _native as _nat
except ImportError as e:
    raise ImportError(f"{os.path.join(_HERE, '_native.so')} is missing or does not load: build it with "
                      "`python -m paper_2603_19133_amd.build` (there is no CPU fallback)") from e

_p, _i32, _i64, _f, _sz = C.c_void_p, C.c_int32, C.c_int64, C.c_float, C.c_size_t
lib.picospec_compress.argtypes = [_p, C.c_int, _i64, _i32, _i32, _f, _i32, _f, _p, _p, _p, _p, _p, _p, _sz, _p]
lib.picospec_sample_draft.argtypes = [_p, _p, _p, _p, _i32, _i32, _p, _p, _p, _p]
lib.picospec_verify.argtypes = [_p, C.c_int, _i64, _i32, _f, _i32, _i32, _p, _p, _p, _p, _p, _p, _i32, C.c_int,
                                _p, _p, _p, _p, _p, _p, _p, _p, _p, _p, _sz, _p]
lib.picospec_verify_range.argtypes = [_p, C.c_int, _i64, _i32, _f, _i32, _i32, _p, _p, _p, _p, _p, _p, _i32, C.c_int,
                                      _p, _p, _p, _p, _i32, _p, _p, _p, _p, _p, _p, _p, _p, _sz, _p]
lib.picospec_round.argtypes = [_p, _p, C.c_int, _i64, _i64, _i32, _f, _i32, _i32, _p, _p, _i32, _f, C.c_int, _p,
                               _p, _p, _p, _p, _p, _p, _p, _p, _p, _p, _p, _p, _p, _p, _p, _p, _sz, _p]
lib.picospec_verify_sample.argtypes = [_p, C.c_int, _i64, _i32, _f, _i32, _i32, _p, _p, _p, _p, _p, _p, _i32, C.c_int, _p,
                                       _p, _p, _p, _p, _p, _p, _p, _p, _p, _p, _p, _sz, _p]
lib.picospec_verify_sample.restype = C.c_int
lib.picospec_verify_sample_static.argtypes = lib.picospec_verify_sample.argtypes[:-3] + [_p]
lib.picospec_verify_sample_static.restype = C.c_int
lib.picospec_static_scratch_bytes.argtypes = []
lib.picospec_static_scratch_bytes.restype = _i64
lib.picospec_sample_residual.argtypes = [_p, C.c_int, _i64, _i32, _f, _i32, _i32, _p, _p, _p, _p, _p, _p, _p, _p,
                                         _i32, C.c_int, _p, _p, _p, _p, _p, _sz, _p]
lib.picospec_sample_residual_ws.argtypes = lib.picospec_sample_residual.argtypes
lib.picospec_row_stats.argtypes = [_p, C.c_int, _i64, _i32, _i32, _f, _p, _p, _p, _p]
lib.picospec_row_stats_ws.argtypes = [_p, C.c_int, _i64, _i32, _i32, _f, _p, _p, _p, _p, _sz, _p]
lib.picospec_compress_rejected.argtypes = [_p, C.c_int, _i64, _i32, _f, _i32, _i32, _p, _p, _i32, _f,
                                           _p, _p, _p, _p, _p, _p, _sz, _p]
lib.picospec_resample_sparse.argtypes = [_p, C.c_int, _i64, _i32, _f, _i32, _i32, _p, _p, _p, _p, _p, _p, _p, _p,
                                         _i32, C.c_int, _p, _p, _p, _p, _p, _sz, _p]
lib.picospec_pack_downlink.argtypes = [_i32, _p, _p, _p, _p, _p, _p, _i32, C.c_int, _p, _i64, _p, _p, _p]
lib.picospec_unpack_downlink.argtypes = [_p, _i64, _i32, _i32, _p, _p, _p, _p, _p, _p, _p, _p]
lib.picospec_pack_uplink.argtypes = [_i32, _i32, _p, _p, _p, C.c_int, _p, _i64, _p, _p]
lib.picospec_unpack_uplink.argtypes = [_p, _i64, _i32, _i32, _p, _p, _p, _p, _p]
lib.picospec_downlink_bytes_max.argtypes = [_i32, _i32, C.c_int]
lib.picospec_downlink_bytes_max.restype = _i64
lib.picospec_uplink_bytes.argtypes = [_i32, _i32, C.c_int]
lib.picospec_uplink_bytes.restype = _i64
lib.picospec_max_load_byte.argtypes = [C.c_int, C.c_int, _i32, _i32]
lib.picospec_max_load_byte.restype = _i64
lib.picospec_check_device.argtypes = [_p, _sz, _p, _p]
lib.picospec_check_device.restype = C.c_int
lib.picospec_probe_clock.argtypes = [_p, _p]
lib.picospec_probe_clock.restype = C.c_int
lib.picospec_workspace_bytes.argtypes = [C.c_int, C.c_int, _i32, _i32, _i32]
lib.picospec_workspace_bytes.restype = _sz
lib.picospec_scratch_bytes.argtypes = [C.c_int, C.c_int, _i32, _i32, _i32, _i32]
lib.picospec_scratch_bytes.restype = _sz
lib.picospec_one_launch_bytes.argtypes = [C.c_int, C.c_int, _i32, _i32, _i32, _i32]
lib.picospec_one_launch_bytes.restype = _sz
lib.picospec_limit.argtypes = [C.c_int]
lib.picospec_limit.restype = _i64
lib.picospec_strerror.argtypes = [C.c_int]
lib.picospec_strerror.restype = C.c_char_p
for _n in ("picospec_compress", "picospec_sample_draft", "picospec_verify", "picospec_sample_residual", "picospec_sample_residual_ws",
           "picospec_row_stats", "picospec_row_stats_ws", "picospec_compress_rejected", "picospec_resample_sparse", "picospec_version",
           "picospec_pack_downlink", "picospec_unpack_downlink", "picospec_pack_uplink", "picospec_unpack_uplink",
           "picospec_verify_range", "picospec_round"):
    getattr(lib, _n).restype = C.c_int


class PicoSpecError(RuntimeError):
    def __init__(self, code: int):
        self.code = code
        super().__init__(f"picospec error {code}: {lib.picospec_strerror(code).decode()}")


def _check(rc: int) -> None:
    if rc != OK:
        raise PicoSpecError(rc)


def alloc_workspace(dtype: torch.dtype, rows: int, V: int, device, which: int = CALL_VERIFY, k: int = 0, n_draft: int = 0) -> torch.Tensor:
    """The optional workspace of verify / sample_residual / verify_sample / round for `rows` = n_draft + B target rows.  With the
    record length k and n_draft, a round's also holds the scratch that spreads its draft rows (else a round that has a use for
    it allocates it)."""
    code = F32 if dtype == torch.float32 else BF16
    n = int(lib.picospec_workspace_bytes(which, code, rows, V, 0))
    if which == CALL_VERIFY:                     # (with what lets a verification of few rows go out in one launch, however many sequences)
        n = max(n, int(lib.picospec_one_launch_bytes(which, code, 0, rows, V, 0)))
    if k and n_draft:
        n = max(n, int(lib.picospec_scratch_bytes(which, code, n_draft, rows - n_draft, V, k)))
    return torch.empty(max(n, 16), dtype=torch.uint8, device=device)


# the current stream's handle without building a Stream object for it (two microseconds a call)
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream() -> int:
    if _raw_stream is None or not torch.cuda.is_initialized():
        return torch.cuda.current_stream().cuda_stream
    return _raw_stream(torch.cuda.current_device())


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return F32
    if t.dtype == torch.bfloat16:
        return BF16
    raise PicoSpecError(EDTYPE)


def _logits_2d(t: torch.Tensor):
    """(dtype code, stride of a row, rows) of a 2-d device tensor with contiguous rows."""
    r = _nat.rows2d(t)
    if r.__class__ is int:
        raise PicoSpecError(r)
    return r


@dataclass
class Compressed:
    idx: torch.Tensor     # int32 [rows, k]
    prob: torch.Tensor    # float32 [rows, k]
    count: torch.Tensor   # int32 [rows]
    mass: torch.Tensor    # float32 [rows]
    lse: torch.Tensor     # float32 [rows]
    k: int


def alloc_compressed(rows: int, k: int, device) -> Compressed:
    e = lambda *s, dt=torch.float32: torch.empty(*s, dtype=dt, device=device)
    return Compressed(e(rows, k, dt=torch.int32), e(rows, k), e(rows, dt=torch.int32), e(rows), e(rows), k)


def _split_stats(which: int, dt: int, n_draft: int, B: int, V: int) -> bool:
    """Whether the library has a use for a table of its own in a call that was given none."""
    return _nat.scratch_bytes(which, dt, n_draft, B, V, 0) > 0


def _table(workspace, which: int, dt: int, n_draft: int, B: int, V: int, like):
    """The workspace of a call that was given none: such a call then spreads its rows over many workgroups."""
    if workspace is not None or not _split_stats(which, dt, n_draft, B, V):
        return workspace
    return _nat.scratch(like, which, dt, n_draft, B, V, 0)


def compress(logits: torch.Tensor, V: int, temperature: float, k: int, top_p: float = 0.0,
             out: Compressed | None = None) -> Compressed:
    """picospec_compress on [rows, >=V] fp32/bf16 device logits."""
    dt, ld, rows = _logits_2d(logits)
    out = out or alloc_compressed(rows, k, logits.device)
    _check(_nat.compress(logits, dt, ld, rows, V, temperature, k, top_p, out.idx, out.prob, out.count, out.mass, out.lse,
                       _nat.scratch(logits, CALL_COMPRESS, dt, rows, 0, V, k), _stream()))
    return out


def sample_draft(q: Compressed, uniforms: torch.Tensor, tok: torch.Tensor | None = None,
                 q_scalar: torch.Tensor | None = None):
    """picospec_sample_draft -> (tok int32 [rows], q_scalar float32 [rows])."""
    rows = q.idx.shape[0]
    if tok is None:
        tok, = _nat.empty(q.idx, "i", rows)
    if q_scalar is None:
        q_scalar, = _nat.empty(q.idx, "f", rows)
    _check(_nat.sample_draft(q.idx, q.prob, q.count, q.mass, q.k, rows, uniforms, tok, q_scalar, _stream()))
    return tok, q_scalar


@dataclass
class Verified:
    n_accept: torch.Tensor   # int32 [B]
    p_tok: torch.Tensor      # float32 [N]
    q_tok: torch.Tensor      # float32 [N]
    tgt_max: torch.Tensor    # float32 [N+B]
    tgt_sum: torch.Tensor    # float32 [N+B]
    tgt_lse: torch.Tensor    # float32 [N+B]
    flags: torch.Tensor      # int32 (bit pattern of uint32) [B]


def alloc_verified(B: int, N: int, device) -> Verified:
    e = lambda n, dt=torch.float32: torch.empty(n, dtype=dt, device=device)
    return Verified(e(B, torch.int32), e(N), e(N), e(N + B), e(N + B), e(N + B), e(B, torch.int32))


def verify(tgt_logits: torch.Tensor, V: int, temperature: float, seq_off: torch.Tensor, n_draft: int,
           draft_tok: torch.Tensor, q: Compressed | None, uniforms: torch.Tensor, renorm: int = 1,
           q_scalar: torch.Tensor | None = None, out: Verified | None = None,
           workspace: torch.Tensor | None = None) -> Verified:
    """picospec_verify; seq_off int32 [B+1] on device, n_draft = seq_off[B] known on the host.  `workspace`
    (alloc_workspace) receives the target rows' segment table for sample_residual."""
    dt, ld, _ = _logits_2d(tgt_logits)
    B = seq_off.shape[0] - 1
    out = out or alloc_verified(B, n_draft, tgt_logits.device)
    rec = (q.idx, q.prob, q.count, q.mass, q.k) if q else _NO_RECORDS
    _check(_nat.verify(tgt_logits, dt, ld, V, temperature, B, n_draft, seq_off, draft_tok, *rec, renorm, q_scalar, uniforms,
                     out.n_accept, out.p_tok, out.q_tok, out.tgt_max, out.tgt_sum, out.tgt_lse, out.flags,
                     _table(workspace, CALL_VERIFY, dt, n_draft, B, V, tgt_logits), _stream()))
    return out


_NO_RECORDS = (None, None, None, None, 0)


def verify_range(tgt_logits: torch.Tensor, V: int, temperature: float, seq_off: torch.Tensor, n_draft: int,
                 draft_tok: torch.Tensor, q: Compressed | None, uniforms: torch.Tensor,
                 pos_begin: torch.Tensor | None, pos_end: torch.Tensor | None, gamma_max: int, renorm: int = 1,
                 q_scalar: torch.Tensor | None = None, out: Verified | None = None) -> Verified:
    """picospec_verify_range: the draft positions pos_begin[b] <= t < pos_end[b] only; `out` from an earlier
    call keeps its entries outside the range."""
    dt, ld, _ = _logits_2d(tgt_logits)
    B = seq_off.shape[0] - 1
    out = out or alloc_verified(B, n_draft, tgt_logits.device)
    rec = (q.idx, q.prob, q.count, q.mass, q.k) if q else _NO_RECORDS
    _check(_nat.verify_range(tgt_logits, dt, ld, V, temperature, B, n_draft, seq_off, draft_tok, *rec, renorm, q_scalar, uniforms,
                           pos_begin, pos_end, gamma_max,
                           out.n_accept, out.p_tok, out.q_tok, out.tgt_max, out.tgt_sum, out.tgt_lse, out.flags,
                           _table(None, CALL_VERIFY, dt, n_draft, B, V, tgt_logits), _stream()))
    return out


def round(draft_logits: torch.Tensor, tgt_logits: torch.Tensor, V: int, temperature: float, seq_off: torch.Tensor,
          n_draft: int, draft_tok: torch.Tensor, k: int, uniforms: torch.Tensor, top_p: float = 0.0, renorm: int = 1,
          q: "Compressed | None" = None, ver: "Verified | None" = None, res: "Residual | None" = None,
          workspace: torch.Tensor | None = None):
    """picospec_round -> (Compressed, Verified, Residual): the whole round in one call."""
    dt, ld_d, _ = _logits_2d(draft_logits) if n_draft else (_dtype_code(tgt_logits), V, 0)
    dt_t, ld_t, _ = _logits_2d(tgt_logits)
    if dt != dt_t:
        raise PicoSpecError(EDTYPE)
    B = seq_off.shape[0] - 1
    dev = tgt_logits.device
    q = q or alloc_compressed(n_draft, k, dev)
    ver = ver or alloc_verified(B, n_draft, dev)
    res = res or alloc_residual(B, dev)
    # few draft rows: a buffer for the segment table and the split kernels' scratch, unless the caller's holds both
    own = _nat.scratch(tgt_logits, CALL_ROUND, dt, n_draft, B, V, k, workspace)
    _check(_nat.round(draft_logits, tgt_logits, dt, ld_d, ld_t, V, temperature, B, n_draft, seq_off, draft_tok, k, top_p, renorm,
                    uniforms, q.idx, q.prob, q.count, q.mass, q.lse,
                    ver.n_accept, ver.p_tok, ver.q_tok, ver.tgt_max, ver.tgt_sum, ver.tgt_lse, ver.flags,
                    res.out_tok, res.resid_mass, res.flags, workspace, own, _stream()))
    return q, ver, res


def verify_sample(tgt_logits: torch.Tensor, V: int, temperature: float, seq_off: torch.Tensor, n_draft: int,
                  draft_tok: torch.Tensor, q: "Compressed", uniforms: torch.Tensor, renorm: int = 1,
                  ver: "Verified | None" = None, res: "Residual | None" = None, workspace: torch.Tensor | None = None):
    """picospec_verify_sample -> (Verified, Residual): verification and draw on records that exist."""
    dt, ld, _ = _logits_2d(tgt_logits)
    B = seq_off.shape[0] - 1
    dev = tgt_logits.device
    ver = ver or alloc_verified(B, n_draft, dev)
    res = res or alloc_residual(B, dev)
    _check(_nat.verify_sample(tgt_logits, dt, ld, V, temperature, B, n_draft, seq_off, draft_tok,
                            q.idx, q.prob, q.count, q.mass, q.k, renorm, uniforms,
                            ver.n_accept, ver.p_tok, ver.q_tok, ver.tgt_max, ver.tgt_sum, ver.tgt_lse, ver.flags,
                            res.out_tok, res.resid_mass, res.flags, _table(workspace, CALL_VERIFY_SAMPLE, dt, n_draft, B, V, tgt_logits), _stream()))
    return ver, res


@dataclass
class Residual:
    out_tok: torch.Tensor     # int32 [B]
    resid_mass: torch.Tensor  # float32 [B]
    flags: torch.Tensor       # int32 [B]


def alloc_residual(B: int, device) -> Residual:
    return Residual(torch.empty(B, dtype=torch.int32, device=device),
                    torch.empty(B, dtype=torch.float32, device=device),
                    torch.empty(B, dtype=torch.int32, device=device))


def verify_sample_static(tgt_logits: torch.Tensor, V: int, temperature: float, seq_off: torch.Tensor, n_draft: int,
                         draft_tok: torch.Tensor, q: "Compressed", uniforms: torch.Tensor, ver: "Verified", res: "Residual",
                         renorm: int = 1) -> None:
    """picospec_verify_sample_static into `ver` and `res` (the caller's: this wrapper allocates nothing either)."""
    dt, ld, _ = _logits_2d(tgt_logits)
    B = seq_off.shape[0] - 1
    _check(_nat.verify_sample_static(tgt_logits, dt, ld, V, temperature, B, n_draft, seq_off, draft_tok,
                                   q.idx, q.prob, q.count, q.mass, q.k, renorm, uniforms,
                                   ver.n_accept, ver.p_tok, ver.q_tok, ver.tgt_max, ver.tgt_sum, ver.tgt_lse, ver.flags,
                                   res.out_tok, res.resid_mass, res.flags, _stream()))


def static_scratch_bytes() -> int:
    return int(lib.picospec_static_scratch_bytes())


def sample_residual(tgt_logits: torch.Tensor, V: int, temperature: float, seq_off: torch.Tensor, n_draft: int,
                    ver: Verified, q: Compressed, uniforms: torch.Tensor, renorm: int = 1,
                    out: Residual | None = None, n_accept: torch.Tensor | None = None,
                    workspace: torch.Tensor | None = None) -> Residual:
    """picospec_sample_residual from the statistics and first-rejection indices of `ver` (and, if given, from the
    segment table that verify left in `workspace`)."""
    dt, ld, _ = _logits_2d(tgt_logits)
    B = seq_off.shape[0] - 1
    out = out or alloc_residual(B, tgt_logits.device)
    call = _nat.sample_residual
    if workspace is None:                        # (the draw may make a table of the rows it draws from)
        workspace = _nat.scratch(tgt_logits, CALL_SAMPLE_RESIDUAL, dt, n_draft, B, V, q.k)
        if workspace is not None:
            call = _nat.sample_residual_ws
    _check(call(tgt_logits, dt, ld, V, temperature, B, n_draft, seq_off,
                ver.n_accept if n_accept is None else n_accept, ver.tgt_max, ver.tgt_sum,
                q.idx, q.prob, q.count, q.mass, q.k, renorm, uniforms, out.out_tok, out.resid_mass, out.flags,
                workspace, _stream()))
    return out


def row_stats(logits: torch.Tensor, V: int, temperature: float):
    """picospec_row_stats -> (row_max, row_sum, row_lse), float32 [rows] each."""
    dt, ld, rows = _logits_2d(logits)
    mx, sm, ls = _nat.empty(logits, "fff", rows, rows, rows)
    _check(_nat.row_stats(logits, dt, ld, rows, V, temperature, mx, sm, ls, _table(None, CALL_ROW_STATS, dt, rows, 0, V, logits), _stream()))
    return mx, sm, ls


def compress_rejected(tgt_logits: torch.Tensor, V: int, temperature: float, seq_off: torch.Tensor, n_draft: int,
                      n_accept: torch.Tensor, k: int, top_p: float = 0.0, out: Compressed | None = None) -> Compressed:
    """picospec_compress_rejected: the downlink record of every sequence's rejected (or bonus) target row."""
    dt, ld, _ = _logits_2d(tgt_logits)
    B = seq_off.shape[0] - 1
    out = out or alloc_compressed(B, k, tgt_logits.device)
    _check(_nat.compress_rejected(tgt_logits, dt, ld, V, temperature, B, n_draft, seq_off, n_accept, k, top_p,
                                out.idx, out.prob, out.count, out.mass, out.lse,
                                _nat.scratch(tgt_logits, CALL_COMPRESS_REJECTED, dt, n_draft, B, V, k), _stream()))
    return out


def resample_sparse(draft_logits: torch.Tensor, V: int, temperature: float, seq_off: torch.Tensor, n_draft: int,
                    n_accept: torch.Tensor, draft_max: torch.Tensor, draft_sum: torch.Tensor, p: Compressed,
                    uniforms: torch.Tensor, renorm: int = 0, out: Residual | None = None) -> Residual:
    """picospec_resample_sparse: the edge's local draw from norm(max(0, P_j - Q_j)) on the record's slots."""
    dt, ld, _ = _logits_2d(draft_logits)
    B = seq_off.shape[0] - 1
    out = out or alloc_residual(B, draft_logits.device)
    _check(_nat.resample_sparse(draft_logits, dt, ld, V, temperature, B, n_draft, seq_off, n_accept, draft_max, draft_sum,
                              p.idx, p.prob, p.count, p.mass, p.k, renorm, uniforms, out.out_tok, out.resid_mass, out.flags,
                              _stream()))
    return out


def downlink_bytes_max(B: int, k: int, prob_format: int) -> int:
    return lib.picospec_downlink_bytes_max(B, k, prob_format)


def uplink_bytes(B: int, n_draft: int, prob_format: int) -> int:
    return lib.picospec_uplink_bytes(B, n_draft, prob_format)


def pack_downlink(seq_off: torch.Tensor, n_accept: torch.Tensor, token: torch.Tensor | None,
                  rec: Compressed | None, prob_format: int, wire: torch.Tensor | None = None):
    """picospec_pack_downlink -> (wire uint8 [capacity], wire_bytes int64 [1], status int32 [1]), all on device."""
    B = seq_off.shape[0] - 1
    k = rec.k if rec is not None else 0
    if wire is None:
        wire = torch.empty(downlink_bytes_max(B, k, prob_format), dtype=torch.uint8, device=seq_off.device)
    nbytes, status = _nat.empty(seq_off, "li", 1, 1)
    idx, prob, count = (rec.idx, rec.prob, rec.count) if rec else (None, None, None)
    _check(_nat.pack_downlink(B, seq_off, n_accept, token, idx, prob, count, k, prob_format, wire, wire.numel(), nbytes, status, _stream()))
    return wire, nbytes, status


@dataclass
class Downlink:
    n_accept: torch.Tensor   # int32 [B]
    token: torch.Tensor      # int32 [B]
    rec: Compressed          # idx/prob [B,k], count, mass (lse unused)
    status: torch.Tensor     # int32 [1]


def unpack_downlink(wire: torch.Tensor, wire_bytes: int, B: int, k: int) -> Downlink:
    """picospec_unpack_downlink; `wire_bytes` is the received length (a host value)."""
    na, tok, idx, prob, count, mass, lse, status = _nat.empty(wire, "iiififfi", B, B, (B, k), (B, k), B, B, B, 1)
    _check(_nat.unpack_downlink(wire, wire_bytes, B, k, na, tok, idx, prob, count, mass, status, _stream()))
    return Downlink(na, tok, Compressed(idx, prob, count, mass, lse, k), status)


def pack_uplink(seq_off: torch.Tensor, n_draft: int, draft_tok: torch.Tensor, q_scalar: torch.Tensor,
                prob_format: int, wire: torch.Tensor | None = None):
    """picospec_pack_uplink -> (wire uint8, wire_bytes int64 [1]) on device."""
    B = seq_off.shape[0] - 1
    if wire is None:
        wire = torch.empty(uplink_bytes(B, n_draft, prob_format), dtype=torch.uint8, device=seq_off.device)
    nbytes, = _nat.empty(seq_off, "l", 1)
    _check(_nat.pack_uplink(B, n_draft, seq_off, draft_tok, q_scalar, prob_format, wire, wire.numel(), nbytes, _stream()))
    return wire, nbytes


def unpack_uplink(wire: torch.Tensor, wire_bytes: int, B: int, n_max: int):
    """picospec_unpack_uplink -> (seq_off int32 [B+1], draft_tok int32 [n_max], q_scalar float32 [n_max], status)."""
    seq_off, tok, q, status = _nat.empty(wire, "iifi", B + 1, n_max, n_max, 1)
    _check(_nat.unpack_uplink(wire, wire_bytes, B, n_max, seq_off, tok, q, status, _stream()))
    return seq_off, tok, q, status


def check_device(device) -> int:
    """picospec_check_device -> status word (0: the device's buffer loads range-check as the row kernels assume)."""
    ws = torch.empty(64 * 1024, dtype=torch.uint8, device=device)
    status = torch.full((1,), -1, dtype=torch.int32, device=device)
    _check(lib.picospec_check_device(ws.data_ptr(), ws.numel(), status.data_ptr(), _stream()))
    return int(status.item()) & 0xFFFFFFFF


def probe_clock(ticks: torch.Tensor) -> None:
    """picospec_probe_clock into `ticks` (int64 [2], device): 100 * ticks[0] / ticks[1] = shader clock in MHz."""
    _check(lib.picospec_probe_clock(ticks.data_ptr(), _stream()))


def max_load_byte(which: int, dtype: int, V: int, misalign_bytes: int) -> int:
    return int(lib.picospec_max_load_byte(which, dtype, V, misalign_bytes))


def workspace_bytes(which: int, dtype: int, rows: int, V: int, k: int) -> int:
    return int(lib.picospec_workspace_bytes(which, dtype, rows, V, k))


def scratch_bytes(which: int, dtype: int, n_draft: int, B: int, V: int, k: int) -> int:
    return int(lib.picospec_scratch_bytes(which, dtype, n_draft, B, V, k))


def limit(which: int) -> int:
    return int(lib.picospec_limit(which))


def version() -> int:
    return int(lib.picospec_version())
