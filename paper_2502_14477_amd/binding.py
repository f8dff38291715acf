"""Python binding over libesa.so: argument marshalling only.

Every function has the name and meaning of its C entry point (include/esa.h).  Tensors are
torch CUDA tensors (torch provides device memory and the current stream, nothing else); a
leading batch dimension is optional.  The marshalling itself (sizes and strides, output and workspace
allocation, the call) is native code, csrc/binding.cpp: a step is a few tens of microseconds of kernels, and host
time per call is part of what it takes.  The C entry points remain reachable as `lib.esa_*` (ctypes).
Nothing in this module computes: with the library missing, import fails.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Tuple

import torch

ESA_F32, ESA_BF16 = 0, 1
ESA_W_ROWMAJOR, ESA_W_PACKED = 0, 1
_PKG = os.path.dirname(os.path.abspath(__file__))


class EsaError(RuntimeError):
    def __init__(self, code: int, text: str):
        super().__init__("libesa error %d: %s" % (code, text))
        self.code = code


def lib_path() -> str:
    return os.path.join(_PKG, "libesa.so")


def _load() -> ctypes.CDLL:
    path = lib_path()
    if not os.path.exists(path):
        raise ImportError(
            "%s is missing: build it with `python -m paper_2502_14477_amd.build` "
            "(there is no fallback path)" % path)
    L = ctypes.CDLL(path)
    i32, i64, vp, sz, f32 = ctypes.c_int, ctypes.c_int64, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_float
    L.esa_version.restype = i32
    L.esa_version.argtypes = []
    L.esa_last_error.restype = ctypes.c_char_p
    L.esa_last_error.argtypes = []
    L.esa_segments.restype = i32
    L.esa_segments.argtypes = [i64, i64, i64, ctypes.POINTER(i64), ctypes.POINTER(i64)]
    L.esa_compress.restype = i32
    L.esa_pack_weights.restype = i32
    L.esa_pack_weights.argtypes = [vp, i64, i32, i32, vp, vp]
    L.esa_compress.argtypes = [vp, i64, i64, i64, vp, i32, vp, i32, vp, i64, i32, i32, i64, i64, vp]
    L.esa_compress_qk.restype = i32
    L.esa_compress_qk.argtypes = [vp, i64, i64, vp, vp, vp, i64, i64, i64, vp, i64, i64, vp, vp, vp, i64, i64, i64,
                                  i64, i32, i32, i32, i32, vp]
    L.esa_score_workspace_bytes.restype = sz
    L.esa_score_workspace_bytes.argtypes = [i32, i64, i32, i32]
    L.esa_score.restype = i32
    L.esa_score.argtypes = [vp, i32, vp, i64, i64, i32, i32, vp, i32, i32, i64, i64, i64, vp, sz, vp]
    L.esa_select_topk_workspace_bytes.restype = sz
    L.esa_select_topk_workspace_bytes.argtypes = [i64, i32, i32]
    L.esa_select_topk.restype = i32
    L.esa_select_topk.argtypes = [vp, i64, i32, i64, vp, i32, i64, i64, vp, sz, vp]
    L.esa_score_select_gather_workspace_bytes.restype = sz
    L.esa_score_select_gather_workspace_bytes.argtypes = [i32, i64, i32, i32, i32]
    L.esa_score_select_gather.restype = i32
    L.esa_score_select_gather.argtypes = [vp, i32, vp, i64, i64, i32, i32, i32, vp, vp, vp, vp, i64, i32, i32, vp, vp, i32, i32,
                                          i64, i64, i64, i64, i64, i64, vp, sz, vp]
    L.esa_select_topk_static_capacity.restype = sz
    L.esa_select_topk_static_capacity.argtypes = []
    L.esa_select_topk_static_prepare.restype = i32
    L.esa_select_topk_static_prepare.argtypes = []
    L.esa_select_topk_static.restype = i32
    L.esa_select_topk_static.argtypes = [vp, i64, i32, i64, vp, i32, i64, i64, vp]
    L.esa_gather_kv.restype = i32
    L.esa_gather_kv.argtypes = [vp, vp, i64, vp, i32, i32, i32, vp, vp, i32, i32, i64, i64, i64, vp]
    L.esa_attend_workspace_bytes.restype = sz
    L.esa_attend_workspace_bytes.argtypes = [i32, i32, i32, i32, i32, i32]
    L.esa_attend.restype = i32
    L.esa_attend.argtypes = [vp, i32, i32, i32, i32, vp, vp, i64, i64, i64, i64, vp, vp, i32, f32, vp, vp,
                             i32, i32, i64, i64, i64, i64, vp, sz, vp]
    L.esa_attend_indexed_workspace_bytes.restype = sz
    L.esa_attend_indexed_workspace_bytes.argtypes = [i32, i32, i32, i32, i32, i32, i32]
    L.esa_attend_indexed.restype = i32
    L.esa_attend_indexed.argtypes = [vp, i32, i32, i32, i32, vp, vp, i64, i64, i64, i64, vp, i32, i64, f32, vp, vp,
                                     i32, i32, i64, i64, i64, vp, sz, vp]
    L.esa_attend_finish.restype = i32
    L.esa_attend_finish.argtypes = [vp, i32, i32, i32, i32, vp, vp, i64, i64, i64, i64, vp, vp, i32, f32, i32, vp, vp,
                                    i32, i32, i64, i64, i64, i64, vp, sz, vp]
    L.esa_attend_local.restype = i32
    L.esa_attend_local.argtypes = [vp, i32, i32, i32, i32, vp, vp, i64, i64, i64, i64, f32, i32, i32, i32, i64, i64,
                                   vp, sz, vp]
    f64 = ctypes.c_double
    L.esa_rope.restype = i32
    L.esa_rope.argtypes = [vp, i64, i32, i32, i64, f64, f64, f64, vp, i64, i32, i32, i64, i64, vp]
    L.esa_attend_reencoded_workspace_bytes.restype = sz
    L.esa_attend_reencoded_workspace_bytes.argtypes = [i32, i32, i32, i32, i32, i32, i64]
    L.esa_attend_reencoded.restype = i32
    L.esa_attend_reencoded.argtypes = [vp, i32, i32, i32, i32, vp, vp, i64, i64, i64, i64, vp, vp, i32, f32, f64, f64,
                                       vp, vp, i32, i32, i64, i64, i64, i64, vp, sz, vp]
    return L


lib = _load()
from . import _native  # noqa: E402  (links against the library loaded above)

EXPORTS = ("esa_version", "esa_last_error", "esa_segments", "esa_pack_weights", "esa_compress", "esa_score_workspace_bytes",
           "esa_score", "esa_select_topk_workspace_bytes", "esa_select_topk", "esa_gather_kv",
           "esa_attend_workspace_bytes", "esa_attend", "esa_attend_local", "esa_attend_finish",
           "esa_attend_indexed_workspace_bytes", "esa_attend_indexed", "esa_rope",
           "esa_attend_reencoded_workspace_bytes", "esa_attend_reencoded", "esa_compress_qk",
           "esa_select_topk_static_capacity", "esa_select_topk_static_prepare", "esa_select_topk_static",
           "esa_score_select_gather_workspace_bytes", "esa_score_select_gather")


_native.set_error_class(EsaError)


def _check(code: int) -> None:
    if code != 0:
        raise EsaError(code, lib.esa_last_error().decode())


def esa_version() -> int:
    return lib.esa_version()


def esa_segments(t0: int, l_i: int, l_l: int) -> Tuple[int, int]:
    return _native.segments(t0, l_i, l_l)


class PackedWeights:
    """Compression weights in the packed layout [d_c, d_in] (see esa_pack_weights)."""

    def __init__(self, data: torch.Tensor, d_in: int, d_c: int):
        self.data, self.d_in, self.d_c = data, d_in, d_c


def esa_pack_weights(W: torch.Tensor) -> PackedWeights:
    """W [d_in, d_c] -> packed weights; done once per layer."""
    d_in, d_c = W.shape
    assert W.is_contiguous()
    dtype = {torch.float32: ESA_F32, torch.bfloat16: ESA_BF16}.get(W.dtype)
    if dtype is None:
        raise EsaError(-2, "unsupported torch dtype %s" % W.dtype)
    out = torch.empty((d_c, d_in), dtype=W.dtype, device=W.device)
    _check(lib.esa_pack_weights(W.data_ptr(), d_in, d_c, dtype, out.data_ptr(), torch.cuda.current_stream().cuda_stream))
    return PackedWeights(out, d_in, d_c)


def esa_compress(x: torch.Tensor, W, bias: Optional[torch.Tensor] = None,
                 out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """x [B?, n_tok, heads, d] or [B?, n_tok, d_in] -> [B?, n_tok, d_c].  W is a [d_in, d_c] tensor or
    PackedWeights.  `out` may be a row-strided view (e.g. rows t0.. of the compressed-key cache)."""
    if isinstance(W, PackedWeights):
        return _native.compress(x, W.data, ESA_W_PACKED, W.d_in, W.d_c, bias, out)
    d_in, d_c = W.shape
    return _native.compress(x, W, ESA_W_ROWMAJOR, d_in, d_c, bias, out)


def esa_compress_qk(xq: torch.Tensor, Wq, xk: torch.Tensor, Wk, bias_q: Optional[torch.Tensor] = None,
                    bias_k: Optional[torch.Tensor] = None, out_q: Optional[torch.Tensor] = None,
                    out_k: Optional[torch.Tensor] = None):
    """Both compressions of Eq. 5 in one call (shapes per tensor as esa_compress; `out_k` is typically the rows
    t0.. of the compressed-key cache).  Returns (q', k')."""
    if isinstance(Wq, PackedWeights):
        assert isinstance(Wk, PackedWeights), "both weight matrices in the same layout"
        assert Wq.d_c == Wk.d_c
        return _native.compress_qk(xq, Wq.data, Wq.d_in, xk, Wk.data, Wk.d_in, ESA_W_PACKED, Wq.d_c, bias_q, bias_k, out_q, out_k)
    assert not isinstance(Wk, PackedWeights), "both weight matrices in the same layout"
    (dq, dc), (dk, dck) = Wq.shape, Wk.shape
    assert dc == dck
    return _native.compress_qk(xq, Wq, dq, xk, Wk, dk, ESA_W_ROWMAJOR, dc, bias_q, bias_k, out_q, out_k)


def esa_score(qc: torch.Tensor, kc_cache: torch.Tensor, m_lo: int, m_hi: int, eps: int = 0,
              out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """qc [B?, l_c, d_c], kc_cache [B?, S, d_c] -> score [B?, m_hi-m_lo] fp32."""
    return _native.score(qc, kc_cache, m_lo, m_hi, eps, out)


def esa_select_topk(score: torch.Tensor, k: int, base: int = 0) -> torch.Tensor:
    """score [B?, n] fp32 -> idx [B?, min(k, n)] int32, ascending absolute positions."""
    return _native.select_topk(score, k, base)


def esa_score_select_gather(qc: torch.Tensor, kc_cache: torch.Tensor, m_lo: int, m_hi: int, k: int,
                            k_cache: Optional[torch.Tensor] = None, v_cache: Optional[torch.Tensor] = None, eps: int = 0):
    """esa_score + esa_select_topk (+ esa_gather_kv when the caches are given) in one call.
    Returns (score or None, idx, k_sel, v_sel); k_sel / v_sel are None without caches."""
    return _native.score_select_gather(qc, kc_cache, m_lo, m_hi, k, k_cache, v_cache, eps)


def esa_select_topk_static_capacity() -> int:
    return lib.esa_select_topk_static_capacity()


def esa_select_topk_static_prepare() -> None:
    _check(lib.esa_select_topk_static_prepare())


def esa_select_topk_static(score: torch.Tensor, k: int, base: int = 0, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """esa_select_topk on the library's own scratch.  With `out` given ([B?, min(k, n)] int32) this
    function allocates nothing either."""
    return _native.select_topk_static(score, k, base, out)


def esa_gather_kv(k_cache: torch.Tensor, v_cache: torch.Tensor, idx: torch.Tensor):
    """caches [B?, S, h_kv, d] (GPU memory, or pinned host memory for an offloaded cache), idx [B?, n_sel]
    int32 on the GPU -> (k_sel, v_sel) [B?, n_sel, h_kv, d] on the GPU."""
    return _native.gather_kv(k_cache, v_cache, idx)


ESA_SPLIT_I_EARLY, ESA_SPLIT_ALGORITHM1 = 0, 1


def esa_attend_indexed(q: torch.Tensor, k_cache: torch.Tensor, v_cache: torch.Tensor, t0: int, l_i: int, l_l: int,
                       idx: Optional[torch.Tensor], scale: Optional[float] = None, return_lse: bool = False):
    """esa_gather_kv + esa_attend in one call: idx [B?, n_sel] int32 positions of the selected tokens."""
    return _native.attend_indexed(q, k_cache, v_cache, t0, l_i, l_l, idx, scale, return_lse)


def esa_rope(x: torch.Tensor, pos0: float, pos_step: float, base: float, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Rotary encoding of x [B?, n_tok, heads, d]: row i goes to position pos0 + i*pos_step.  `out` may be
    x itself (in place) or a view with the same shape (e.g. rows of a cache)."""
    return _native.rope(x, pos0, pos_step, base, out)


def esa_attend_reencoded(q: torch.Tensor, k_cache: torch.Tensor, v_cache: torch.Tensor, t0: int, l_i: int, l_l: int,
                         k_sel: Optional[torch.Tensor], v_sel: Optional[torch.Tensor], w: float, rope_base: float,
                         scale: Optional[float] = None, return_lse: bool = False):
    """Section 3.2's attention on un-encoded q, key cache and gathered keys (shapes as esa_attend)."""
    return _native.attend_reencoded(q, k_cache, v_cache, t0, l_i, l_l, k_sel, v_sel, w, rope_base, scale, return_lse)


def esa_attend_local(q: torch.Tensor, k_cache: torch.Tensor, v_cache: torch.Tensor, t0: int, l_i: int, l_l: int,
                     scale: Optional[float] = None, split: int = ESA_SPLIT_I_EARLY) -> None:
    """First half of the two-call form of esa_attend: the keys that do not depend on the selection
    ([I, L, C], or [L, C] with split = ESA_SPLIT_ALGORITHM1).  Leaves partial results in a buffer that the device's
    two-call attentions share, for esa_attend_finish (same sizes and split, ordered after it, with no other
    esa_attend_local of the device between the two)."""
    _native.attend_local(q, k_cache, v_cache, t0, l_i, l_l, scale, split)


def esa_attend_finish(q, k_cache, v_cache, t0, l_i, l_l, k_sel, v_sel, scale=None, return_lse=False,
                      split: int = ESA_SPLIT_I_EARLY):
    """Second half of the two-call form: the selected keys (with the initial tokens if split =
    ESA_SPLIT_ALGORITHM1), then the merge.  Arguments as esa_attend."""
    return esa_attend(q, k_cache, v_cache, t0, l_i, l_l, k_sel, v_sel, scale, return_lse, _split=split)


def esa_attend(q: torch.Tensor, k_cache: torch.Tensor, v_cache: torch.Tensor, t0: int, l_i: int, l_l: int,
               k_sel: Optional[torch.Tensor], v_sel: Optional[torch.Tensor], scale: Optional[float] = None,
               return_lse: bool = False, _split: Optional[int] = None):
    """q [B?, l_c, h, d]; caches [B?, S, h_kv, d] holding the current tokens at rows t0..; gathered
    buffers [B?, n_sel, h_kv, d] -> out [B?, l_c, h, d] (and lse [B?, l_c, h] fp32)."""
    return _native.attend(q, k_cache, v_cache, t0, l_i, l_l, k_sel, v_sel, scale, return_lse, _split)
