"""ctypes binding of include/hydra_ops.h (argument marshalling only).

Arguments are torch CUDA tensors (device memory is PyTorch's job here); every
function enqueues the named C entry point on torch's current stream.
"""
from __future__ import annotations

import ctypes as C
import struct
from array import array

from .hydra import HydraError, lib

F32, BF16 = 0, 1
EPI_NONE, EPI_RELU, EPI_GELU = 0, 1, 2


class hydra_gemm_desc(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("dtype", "M", "N", "K", "x_kmajor", "w_kmajor", "ldx", "ldw", "ldo", "ldg", "ldr",
                                       "act", "out_f32", "tile", "G")] + \
               [(n, C.c_void_p) for n in ("X", "W", "bias", "out", "pre", "gate", "resid", "rowsum", "ws")] + \
               [("ws_bytes", C.c_size_t)]


# A small product takes less time than ctypes needs for its arguments: tables are made as one array of addresses and the
# descriptor is packed (3 tables of forward, bias and pre-activation: 4.1 -> 2.0 us, of which reading the addresses is 1.1).
_desc = struct.Struct("15i9PN").pack           # the fields of hydra_gemm_desc


_ready = False


def _L():
    global _ready
    L = lib()
    if not _ready:
        vp = pp = C.c_void_p                       # tables go by address, descriptors as bytes or by reference
        L.hydra_op_gemm.argtypes = [vp, vp]
        L.hydra_op_gemm_update.argtypes = [vp, C.c_int, pp, pp, pp, pp, vp, vp]
        L.hydra_op_colsum.argtypes = [C.c_int] * 5 + [pp, pp, pp, vp]
        L.hydra_op_colsum_part_floats.argtypes = [C.c_int, C.c_int]
        L.hydra_op_colsum_part_floats.restype = C.c_size_t
        L.hydra_op_colsum_noalloc.argtypes = [C.c_int] * 5 + [pp, pp, vp]
        L.hydra_op_colsum_noalloc_max_floats.argtypes = []
        L.hydra_op_colsum_noalloc_max_floats.restype = C.c_size_t
        L.hydra_op_gemm_split_k.argtypes = [C.c_int] * 3
        L.hydra_op_gemm_split_ws_bytes.argtypes = [C.c_int] * 4
        L.hydra_op_gemm_split_ws_bytes.restype = C.c_size_t
        L.hydra_op_softmax_ce.argtypes = [C.c_int] * 5 + [C.c_float, C.c_int, pp, vp, pp, pp, pp, vp]
        L.hydra_op_optim.argtypes = [C.c_int, C.c_size_t, C.c_int, pp, pp, pp, pp, pp, vp, vp]
        L.hydra_op_init_uniform.argtypes = [vp, C.c_size_t, C.c_uint64, C.c_uint64, C.c_float, vp]
        L.hydra_op_cast_bf16.argtypes = [vp, vp, C.c_size_t, vp]
        L.hydra_op_layernorm_fwd.argtypes = [C.c_int] * 4 + [C.c_float, C.c_int] + [pp] * 6 + [vp]
        L.hydra_op_layernorm_bwd.argtypes = [C.c_int] * 5 + [pp] * 10 + [vp]
        L.hydra_op_layernorm_part_floats.argtypes = [C.c_int, C.c_int]
        L.hydra_op_layernorm_part_floats.restype = C.c_size_t
        L.hydra_op_attention_fwd.argtypes = [C.c_int] * 7 + [C.c_float, C.c_int, pp, pp, pp, vp]
        L.hydra_op_attention_bwd.argtypes = [C.c_int] * 7 + [C.c_float, C.c_int] + [pp] * 6 + [vp]
        L.hydra_op_embed_fwd.argtypes = [C.c_int] * 6 + [vp, pp, pp, pp, vp]
        L.hydra_op_embed_bwd.argtypes = [C.c_int] * 8 + [vp, vp, pp, pp, pp, vp]
        L.hydra_op_empty_launches.argtypes = [C.c_int, vp]
        L.hydra_ops_last_error.restype = C.c_char_p
        _ready = True
    return L


def _stream():
    """torch's current stream on the current device (the raw handle: building a Stream object costs several us)."""
    import torch
    return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())


def _tabs(*tables):
    """[keep, a, b, ...]: the addresses of all tables' tensors in one array, which the caller keeps over the call, and the address of
    each table in it (None for none)."""
    keep = array("Q", [x.data_ptr() for t in tables if t is not None for x in t])
    at, out = keep.buffer_info()[0], [keep]
    for t in tables:
        if t is None:
            out.append(None)
        else:
            out.append(at)
            at += 8 * len(t)
    return out


def _hp(hp_rows, problems):
    """Hyper-parameters of all problems as doubles, six to a problem, and their address: zeros where fewer are given, more are refused."""
    try:
        flat = array("d", [x for row in hp_rows for x in row])
    except TypeError:  # what only float() makes a number of
        flat = array("d", [float(x) for row in hp_rows for x in row])
    missing = 6 * problems - len(flat)
    if missing:
        if missing < 0:
            raise IndexError(f"{len(flat)} hyper-parameters for {problems} problems")
        flat.extend([0.0] * missing)
    return flat, flat.buffer_info()[0]


def _nbytes(ws):
    return 0 if ws is None else min(t.numel() * t.element_size() for t in ws)


def _check(st: int):
    if st != 0:
        raise HydraError(st, _L().hydra_ops_last_error().decode())


def hydra_op_gemm(dtype, M, N, K, X, W, out, *, x_kmajor, w_kmajor, ldx, ldw, ldo, bias=None, pre=None, gate=None,
                  resid=None, ldg=0, ldr=0, act=EPI_NONE, out_f32=False, tile=0, rowsum=None, ws=None):
    """ws: optional per-problem scratch tensors (uint8, hydra_op_gemm_split_ws_bytes bytes) that allow a split sum over k."""
    keep, *at = _tabs(X, W, bias, out, pre, gate, resid, rowsum, ws)
    d = _desc(dtype, M, N, K, int(x_kmajor), int(w_kmajor), ldx, ldw, ldo, ldg, ldr, act, int(out_f32), tile, len(X),
              *[a or 0 for a in at], _nbytes(ws))
    _check(_L().hydra_op_gemm(d, _stream()))


def hydra_op_gemm_split_k(M, N, K) -> int:
    return int(_L().hydra_op_gemm_split_k(M, N, K))


def hydra_op_gemm_split_ws_bytes(M, N, K, ldo) -> int:
    return int(_L().hydra_op_gemm_split_ws_bytes(M, N, K, ldo))


def hydra_op_gemm_update(dtype, M, N, K, X, W, opt, p, m, v, w16, hp_rows, *, ldx, ldw, ldo, out=None, tile=0, rowsum=None,
                         ws=None):
    """Weight gradient dW[M,N] = sum_k X(k,m) W(k,n) with the optimizer step of hydra_op_optim in its epilogue."""
    keep, tx, tw, to, tr, ts, tp, tm, tv, t16 = _tabs(X, W, out, rowsum, ws, p, m, v, w16)
    d = _desc(dtype, M, N, K, 0, 0, ldx, ldw, ldo, 0, 0, EPI_NONE, 1, tile, len(X), tx or 0, tw or 0, 0, to or 0, 0, 0, 0, tr or 0, ts or 0,
              _nbytes(ws))
    flat, hp = _hp(hp_rows, len(p))
    _check(_L().hydra_op_gemm_update(d, opt, tp, tm, tv, t16, hp, _stream()))


def hydra_op_colsum_part_floats(M, N) -> int:
    return int(_L().hydra_op_colsum_part_floats(M, N))


def hydra_op_colsum(dtype, M, N, ld, src, out, part=None):
    keep, *at = _tabs(src, out, part)
    _check(_L().hydra_op_colsum(dtype, M, N, ld, len(src), *at, _stream()))


def hydra_op_empty_launches(n: int):
    _check(_L().hydra_op_empty_launches(n, _stream()))


def hydra_op_colsum_noalloc(dtype, M, N, ld, src, out):
    keep, *at = _tabs(src, out)
    _check(_L().hydra_op_colsum_noalloc(dtype, M, N, ld, len(src), *at, _stream()))


def hydra_op_colsum_noalloc_max_floats() -> int:
    return int(_L().hydra_op_colsum_noalloc_max_floats())


def hydra_op_softmax_ce(dtype, M, Cn, ldz, lddz, inv_n, logits, labels, dz, rowloss, loss):
    keep, tz, *at = _tabs(logits, dz, rowloss, loss)
    _check(_L().hydra_op_softmax_ce(dtype, M, Cn, ldz, lddz, inv_n, len(logits), tz, labels.data_ptr(), *at, _stream()))


def hydra_op_optim(opt, n, p, g, m, v, w16, hp_rows):
    """hp_rows: per problem (lr, b1, b2, eps, bc1, bc2)."""
    keep, *at = _tabs(p, g, m, v, w16)
    flat, hp = _hp(hp_rows, len(p))
    _check(_L().hydra_op_optim(opt, n, len(p), *at, hp, _stream()))


def hydra_op_init_uniform(dst, n, seed, stream_id, a):
    _check(_L().hydra_op_init_uniform(C.c_void_p(dst.data_ptr()), n, C.c_uint64(seed), C.c_uint64(stream_id), a, _stream()))


def hydra_op_cast_bf16(src, dst, n):
    _check(_L().hydra_op_cast_bf16(C.c_void_p(src.data_ptr()), C.c_void_p(dst.data_ptr()), n, _stream()))


def hydra_op_layernorm_fwd(dtype, rows, d, ld, eps, x, y, gamma, beta, mean, rstd):
    keep, *at = _tabs(x, y, gamma, beta, mean, rstd)
    _check(_L().hydra_op_layernorm_fwd(dtype, rows, d, ld, eps, len(x), *at, _stream()))


def hydra_op_layernorm_part_floats(rows, d) -> int:
    return int(_L().hydra_op_layernorm_part_floats(rows, d))


def hydra_op_layernorm_bwd(dtype, rows, d, ld, x, dy, add, dx, gamma, mean, rstd, part, dgamma, dbeta):
    keep, *at = _tabs(x, dy, add, dx, gamma, mean, rstd, part, dgamma, dbeta)
    _check(_L().hydra_op_layernorm_bwd(dtype, rows, d, ld, len(x), *at, _stream()))


def hydra_op_attention_fwd(B, S, H, DH, ld_qkv, ld_o, causal, scale, qkv, o, lse):
    keep, *at = _tabs(qkv, o, lse)
    _check(_L().hydra_op_attention_fwd(B, S, H, DH, ld_qkv, ld_o, int(causal), scale, len(qkv), *at, _stream()))


def hydra_op_attention_bwd(B, S, H, DH, ld_qkv, ld_o, causal, scale, qkv, o, dout, lse, delta, dqkv):
    keep, *at = _tabs(qkv, o, dout, lse, delta, dqkv)
    _check(_L().hydra_op_attention_bwd(B, S, H, DH, ld_qkv, ld_o, int(causal), scale, len(qkv), *at, _stream()))


def hydra_op_embed_fwd(dtype, tokens, S, d, ld, ids, tok, pos, x):
    keep, *at = _tabs(tok, pos, x)
    _check(_L().hydra_op_embed_fwd(dtype, tokens, S, d, ld, len(x), ids.data_ptr(), *at, _stream()))


def hydra_op_embed_bwd(dtype, V, S, S_table, B, d, ld, row_ptr, positions, dx, dtok, dpos):
    keep, *at = _tabs(dx, dtok, dpos)
    _check(_L().hydra_op_embed_bwd(dtype, V, S, S_table, B, d, ld, len(dx), row_ptr.data_ptr(), positions.data_ptr(), *at, _stream()))
