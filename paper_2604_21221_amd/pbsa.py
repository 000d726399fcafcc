"""Thin ctypes binding of libpbsa.so: argument marshalling only, same names as include/pbsa.h.

Tensor arguments are torch tensors living on the GPU (their data_ptr() is passed through) or plain
integers holding a device address.  Nothing is computed here and there is no fallback: if the HIP
library is missing the import of the library fails loudly.
"""
from __future__ import annotations

import ctypes
import os

import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libpbsa.so")

PBSA_OK, PBSA_EINVAL, PBSA_ESHAPE, PBSA_EALIGN, PBSA_EWS, PBSA_EHIP = 0, -1, -2, -3, -4, -5
PBSA_MAX_N_LOC, PBSA_MAX_C, PBSA_MAX_C_ATTEND, PBSA_MAX_K = 672, 64, 336, 672
PBSA_MAX_N_LOC_AUX, PBSA_MAX_C_AUX, PBSA_MAX_K_AUX = 512, 192, 512
PBSA_STATIC_WS_BYTES = 4 << 20

class pbsa_params(ctypes.Structure):
    _fields_ = [("size", ctypes.c_uint32), ("H", ctypes.c_int32), ("d", ctypes.c_int32), ("B", ctypes.c_int32),
                ("Nq", ctypes.c_int32), ("nqb", ctypes.c_int32), ("n_loc", ctypes.c_int32),
                ("n_loc_cap", ctypes.c_int32), ("C", ctypes.c_int32), ("n_sink", ctypes.c_int32),
                ("k", ctypes.c_int32), ("causal", ctypes.c_int32), ("n_evict", ctypes.c_int32),
                ("pool_from", ctypes.c_int32), ("scale", ctypes.c_float),
                ("q_stride_h", ctypes.c_int64), ("q_stride_t", ctypes.c_int64),
                ("o_stride_h", ctypes.c_int64), ("o_stride_t", ctypes.c_int64)]


def make_params(H, d, B, Nq, n_loc, n_loc_cap, C, k, scale, n_sink=0, causal=1, n_evict=0, pool_from=0,
                q_strides=None, o_strides=None) -> pbsa_params:
    qs = q_strides or (Nq * d, d)
    os_ = o_strides or (Nq * d, d)
    return pbsa_params(ctypes.sizeof(pbsa_params), H, d, B, Nq, -(-Nq // B), n_loc, n_loc_cap, C, n_sink, k, causal,
                       n_evict, pool_from, scale, qs[0], qs[1], os_[0], os_[1])


class pbsa_grid(ctypes.Structure):
    _fields_ = [("size", ctypes.c_uint32), ("T", ctypes.c_int32), ("Hs", ctypes.c_int32), ("Ws", ctypes.c_int32),
                ("Bt", ctypes.c_int32), ("Bh", ctypes.c_int32), ("Bw", ctypes.c_int32), ("H", ctypes.c_int32),
                ("d", ctypes.c_int32), ("B", ctypes.c_int32)]


def make_grid(T, Hs, Ws, Bt, Bh, Bw, H, d, B) -> pbsa_grid:
    return pbsa_grid(ctypes.sizeof(pbsa_grid), T, Hs, Ws, Bt, Bh, Bw, H, d, B)


class PbsaError(RuntimeError):
    def __init__(self, code: int):
        self.code = code
        super().__init__(f"pbsa error {code}: {pbsa_strerror(code)}")


# The library's functions and the kinds of their arguments: p / g a pbsa_params / pbsa_grid by reference, t a tensor (or a
# device address, or None), i / l / z an int32 / int64 / size, w an address that is none of a tensor's (workspace, stream),
# P / L a host array of pointers / of int64, o a size to be filled in.
_SIGNATURES = {
    "pbsa_workspace_bytes": "po",
    "pbsa_attention_workspace_bytes": "po",
    "pbsa_mass_workspace_bytes": "po",
    "pbsa_bwd_workspace_bytes": "po",
    "pbsa_pool_blocks": "pttitw",
    "pbsa_summary_view": "p" + 5 * "t" + "w",
    "pbsa_append_chunk": "pttlllliitttw",
    "pbsa_append_chunk_pool": "pttlllliittttlltw",
    "pbsa_append_select": "pttlllliitttttttt" + "w",
    "pbsa_select_pooled": "ptttttw",
    "pbsa_select_blocks": "p" + 8 * "t" + "wzw",
    "pbsa_select_blocks_apply": "p" + 8 * "t" + "p" + 6 * "t" + "wzw",
    "pbsa_attention_fwd": "p" + 11 * "t" + "wzw",
    "pbsa_attention_fwd_split": "p" + 11 * "t" + "wzw",
    "pbsa_attention_fwd_plan": "p" + 20 * "t" + "wzw",
    "pbsa_attention_fwd_plan_split": "p" + 20 * "t" + "wzwzw",
    "pbsa_attention_fwd_mass": "p" + 12 * "t" + "wzw",
    "pbsa_attention_fwd_mass_split": "p" + 12 * "t" + "wzwzw",
    "pbsa_attention_mass": "p" + 9 * "t" + "w",
    "pbsa_attention_bwd": "p" + 17 * "t" + "wzw",
    "pbsa_memory_update": "p" + 17 * "t" + "wzw",
    "pbsa_memory_update_static": "p" + 17 * "t" + "w",
    "pbsa_memory_update_plan": "p" + 12 * "t" + "wzw",
    "pbsa_memory_update_apply": "p" + 7 * "t" + "wzw",
    "pbsa_memory_update_fine": "p" + 16 * "t" + "wzw",
    "pbsa_blockify": "giPPLw",
    "pbsa_unblockify": "gtltw",
}
EXPORTS = (*_SIGNATURES, "pbsa_strerror", "pbsa_version")

_lib = None


def lib() -> ctypes.CDLL:
    """Load libpbsa.so (built in-tree by paper_2604_21221_amd/build.py).  No fallback."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(f"{LIB_PATH} is missing: build it with `python -m paper_2604_21221_amd.build` "
                              "(there is no CPU fallback)")
        L = ctypes.CDLL(LIB_PATH)
        L.pbsa_version.restype = ctypes.c_int
        L.pbsa_version.argtypes = []
        L.pbsa_strerror.restype = ctypes.c_char_p
        L.pbsa_strerror.argtypes = [ctypes.c_int]
        ref = ctypes.POINTER
        types = dict(p=ref(pbsa_params), g=ref(pbsa_grid), t=ctypes.c_void_p, w=ctypes.c_void_p, i=ctypes.c_int32, l=ctypes.c_int64,
                     z=ctypes.c_size_t, o=ref(ctypes.c_size_t), P=ref(ctypes.c_void_p), L=ref(ctypes.c_int64))
        for name, kinds in _SIGNATURES.items():
            fn = getattr(L, name)
            fn.restype = ctypes.c_int
            fn.argtypes = [types[k] for k in kinds]
        _lib = L
    return _lib


def _ptr(x):
    """Device address of a tensor (must be on the GPU), or an int / None passed through."""
    if x is None:
        return None
    if isinstance(x, int):
        return ctypes.c_void_p(x)
    if not x.is_cuda:
        raise TypeError("pbsa: tensor arguments must live on the GPU")
    if not x.is_contiguous() and x.dim() < 3:
        raise TypeError("pbsa: small tensors must be contiguous")
    return ctypes.c_void_p(x.data_ptr())


def _stream(stream):
    if stream is None:
        # what torch.cuda.current_stream().cuda_stream says, without the Stream object (3 us)
        return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
    if isinstance(stream, int):
        return stream
    return stream.cuda_stream


def _ws(ws):
    if ws is None:
        return None, 0
    if isinstance(ws, tuple):
        return ws[0], ws[1]
    return ws.data_ptr(), ws.numel() * ws.element_size()


class _Functions(dict):
    """Address and argument kinds of each library function, looked up (and the library loaded) on first use."""

    def __missing__(self, name):
        self[name] = f = (ctypes.cast(getattr(lib(), name), ctypes.c_void_p).value, _SIGNATURES[name].encode())
        return f


_F = _Functions()


def _invoke(*args):
    """Calls the function at address args[0] with the rest (csrc/pbsa_host.cpp)."""
    global _invoke
    try:
        from ._pbsa_host import invoke, setup
    except ImportError as e:
        raise ImportError("the binding's native half is missing: build it with `python -m paper_2604_21221_amd.build`") from e
    setup(pbsa_params, pbsa_grid, ctypes.Array)
    _invoke = invoke
    return invoke(*args)


def plain_rows(*args):
    """plain_rows(Kl, Vl, H, Nq, d, watched, *tensors) -> bool (csrc/pbsa_host.cpp)"""
    global plain_rows
    from ._pbsa_host import plain_rows as native
    plain_rows = native
    return native(*args)


def _through_ctypes(name, args):
    """The call for what the native half leaves alone: anything but plain tensors, integers and the structures themselves.
    ctypes and _ptr take it or refuse it."""
    conv = dict(p=ctypes.byref, g=ctypes.byref, t=_ptr, w=ctypes.c_void_p)
    return getattr(lib(), name)(*[conv[k](a) if k in conv else a for k, a in zip(_SIGNATURES[name], args)])


def _call(name, *args):
    rc = _invoke(*_F[name], *args)
    _check(_through_ctypes(name, args) if rc is NotImplemented else rc)


def _size(name, p):
    out = ctypes.c_size_t(0)
    _check(getattr(lib(), name)(ctypes.byref(p), ctypes.byref(out)))
    return out.value


def _check(rc: int):
    if rc != PBSA_OK:
        raise PbsaError(rc)


def pbsa_version() -> int:
    return lib().pbsa_version()


def pbsa_strerror(code: int) -> str:
    return lib().pbsa_strerror(code).decode()


def pbsa_workspace_bytes(p: pbsa_params) -> int:
    return _size("pbsa_workspace_bytes", p)


def pbsa_attention_workspace_bytes(p: pbsa_params) -> int:
    return _size("pbsa_attention_workspace_bytes", p)


def pbsa_pool_blocks(p, X, length, n_blocks, out, stream=None):
    _call("pbsa_pool_blocks", p, X, length, n_blocks, out, _stream(stream))


def pbsa_summary_view(p, S_sum, S_cnt, Kp, Vp, p_len, stream=None):
    _call("pbsa_summary_view", p, S_sum, S_cnt, Kp, Vp, p_len, _stream(stream))


def pbsa_append_chunk(p, K, V, slot0, zero_tail, Kl, Vl, Kc_l=None, stream=None, Q=None, Qc=None):
    """K, V: [H][Nq][d] bf16 with a contiguous last dimension, or None.  Q, Qc: the queries are pooled along
    (pbsa_append_chunk_pool), for a pbsa_select_blocks with pooled=True."""
    ks, vs = (x.stride() if x is not None else (0, 0, 1) for x in (K, V))
    if Q is not None:
        qs = Q.stride()
        _call("pbsa_append_chunk_pool", p, K, V, ks[0], ks[1], vs[0], vs[1], slot0, int(zero_tail), Kl, Vl, Kc_l, Q, qs[0], qs[1],
              Qc, _stream(stream))
        return
    _call("pbsa_append_chunk", p, K, V, ks[0], ks[1], vs[0], vs[1], slot0, int(zero_tail), Kl, Vl, Kc_l, _stream(stream))


def pbsa_append_select(p, K, V, slot0, zero_tail, Q, Kl, Vl, l_map, Kc_l, Qc, sel, Zl=None, stream=None):
    """K, V: [H][Nq][d] bf16 with a contiguous last dimension; Q has p's strides."""
    ks, vs = K.stride(), V.stride()
    _call("pbsa_append_select", p, K, V, ks[0], ks[1], vs[0], vs[1], slot0, int(zero_tail), Q, Kl, Vl, l_map, Kc_l, Qc, sel, Zl,
          _stream(stream))


def pbsa_select_blocks(p, Q, Kl, l_len, l_map, Kc_l, Qc, sel, Zl=None, ws=None, stream=None, pooled=False):
    """pooled: Qc and all of Kc_l have been written already (pbsa_select_pooled)."""
    if pooled:
        _call("pbsa_select_pooled", p, l_map, Kc_l, Qc, sel, Zl, _stream(stream))
        return
    w, wb = _ws(ws)
    _call("pbsa_select_blocks", p, Q, Kl, l_len, l_map, Kc_l, Qc, sel, Zl, w, wb, _stream(stream))


def pbsa_select_blocks_apply(p, Q, Kl, l_len, l_map, Kc_l, Qc, sel, Zl, p_upd, Kp, Vp, p_len, S_sum, S_cnt, Vl, ws,
                             stream=None):
    w, wb = _ws(ws)
    _call("pbsa_select_blocks_apply", p, Q, Kl, l_len, l_map, Kc_l, Qc, sel, Zl, p_upd, Kp, Vp, p_len, S_sum, S_cnt, Vl, w,
          wb, _stream(stream))


def pbsa_attention_fwd(p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse=None, ws=None, stream=None):
    w, wb = _ws(ws)
    _call("pbsa_attention_fwd", p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, w, wb, _stream(stream))


def pbsa_attention_fwd_split(p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, ws, stream=None):
    """pbsa_attention_fwd with pbsa_attention_workspace_bytes(p) bytes of scratch."""
    w, wb = _ws(ws)
    _call("pbsa_attention_fwd_split", p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, w, wb, _stream(stream))


def pbsa_memory_update(p, Qc, Kc_l, Zl, Kp, Vp, Kc_p, p_len, p_id, S_sum, S_cnt, Kl, Vl, l_len, l_map, l_id, scores,
                       slot_src, ws, stream=None):
    w, wb = _ws(ws)
    _call("pbsa_memory_update", p, Qc, Kc_l, Zl, Kp, Vp, Kc_p, p_len, p_id, S_sum, S_cnt, Kl, Vl, l_len, l_map, l_id, scores,
          slot_src, w, wb, _stream(stream))


def pbsa_memory_update_static(p, Qc, Kc_l, Zl, Kp, Vp, Kc_p, p_len, p_id, S_sum, S_cnt, Kl, Vl, l_len, l_map, l_id, scores,
                              slot_src, stream=None):
    _call("pbsa_memory_update_static", p, Qc, Kc_l, Zl, Kp, Vp, Kc_p, p_len, p_id, S_sum, S_cnt, Kl, Vl, l_len, l_map, l_id,
          scores, slot_src, _stream(stream))


def pbsa_memory_update_plan(p, Qc, Kc_l, Zl, Kc_p, p_len, p_id, S_cnt, l_len, l_map, l_id, scores, slot_src, ws,
                            stream=None):
    w, wb = _ws(ws)
    _call("pbsa_memory_update_plan", p, Qc, Kc_l, Zl, Kc_p, p_len, p_id, S_cnt, l_len, l_map, l_id, scores, slot_src, w, wb,
          _stream(stream))


def pbsa_attention_fwd_plan(p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, Qc, Kc_l, Zl, Kc_p, p_id, S_cnt, l_id,
                            scores, slot_src, ws, stream=None):
    w, wb = _ws(ws)
    _call("pbsa_attention_fwd_plan", p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, Qc, Kc_l, Zl, Kc_p, p_id, S_cnt,
          l_id, scores, slot_src, w, wb, _stream(stream))


def pbsa_attention_fwd_plan_split(p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, Qc, Kc_l, Zl, Kc_p, p_id, S_cnt,
                                  l_id, scores, slot_src, ws, split_ws, stream=None):
    w, wb = _ws(ws)
    v, vb = _ws(split_ws)
    _call("pbsa_attention_fwd_plan_split", p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, Qc, Kc_l, Zl, Kc_p, p_id,
          S_cnt, l_id, scores, slot_src, w, wb, v, vb, _stream(stream))


def pbsa_memory_update_apply(p, Kp, Vp, p_len, S_sum, S_cnt, Kl, Vl, ws, stream=None):
    w, wb = _ws(ws)
    _call("pbsa_memory_update_apply", p, Kp, Vp, p_len, S_sum, S_cnt, Kl, Vl, w, wb, _stream(stream))


def pbsa_attention_mass(p, Q, Kp, p_len, Kl, l_len, l_map, sel, lse, Mt, stream=None):
    _call("pbsa_attention_mass", p, Q, Kp, p_len, Kl, l_len, l_map, sel, lse, Mt, _stream(stream))


def pbsa_mass_workspace_bytes(p: pbsa_params) -> int:
    return _size("pbsa_mass_workspace_bytes", p)


def pbsa_attention_fwd_mass(p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, Mt, ws, stream=None):
    w, wb = _ws(ws)
    _call("pbsa_attention_fwd_mass", p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, Mt, w, wb, _stream(stream))


def pbsa_attention_fwd_mass_split(p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, Mt, ws, split_ws, stream=None):
    w, wb = _ws(ws)
    v, vb = _ws(split_ws)
    _call("pbsa_attention_fwd_mass_split", p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, Mt, w, wb, v, vb,
          _stream(stream))


def pbsa_memory_update_fine(p, Mt, Kc_l, Kp, Vp, Kc_p, p_len, p_id, S_sum, S_cnt, Kl, Vl, l_len, l_map, l_id, scores,
                            slot_src, ws, stream=None):
    w, wb = _ws(ws)
    _call("pbsa_memory_update_fine", p, Mt, Kc_l, Kp, Vp, Kc_p, p_len, p_id, S_sum, S_cnt, Kl, Vl, l_len, l_map, l_id,
          scores, slot_src, w, wb, _stream(stream))


def pbsa_bwd_workspace_bytes(p: pbsa_params) -> int:
    return _size("pbsa_bwd_workspace_bytes", p)


def pbsa_attention_bwd(p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, dO, lse, dQ, dKp, dVp, dKl, dVl, ws, stream=None):
    w, wb = _ws(ws)
    _call("pbsa_attention_bwd", p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, dO, lse, dQ, dKp, dVp, dKl, dVl, w, wb,
          _stream(stream))


def pbsa_blockify(g, X, Xblk, blk_stride_h, stream=None):
    """X, Xblk: sequences of tensors (or device addresses), blk_stride_h: sequence of ints, one per tensor."""
    n = len(X)
    xs = (ctypes.c_void_p * n)(*[_ptr(x) for x in X])
    bs = (ctypes.c_void_p * n)(*[_ptr(x) for x in Xblk])
    st = (ctypes.c_int64 * n)(*[int(v) for v in blk_stride_h])
    _call("pbsa_blockify", g, n, xs, bs, st, _stream(stream))


def pbsa_unblockify(g, Xblk, blk_stride_h, X, stream=None):
    _call("pbsa_unblockify", g, Xblk, int(blk_stride_h), X, _stream(stream))
