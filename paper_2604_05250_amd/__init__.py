"""MI355X-native hot path of one DualDiffusion draft-then-verify step.

Thin binding over the C ABI in ``include/dd.h`` (``libdd.so``, hand-written
gfx950 HIP kernels).  The functions here have the C entry points' names and only
marshal arguments: torch tensors supply device memory and the current stream, every
step of the computation runs in the library's kernels.  The marshalling itself is native
(``csrc/binding.cpp``); the C ABI is also reachable through ``lib()`` (ctypes).  There is no CPU
fallback: if a library cannot be loaded, the first call raises.
"""
from __future__ import annotations

import ctypes as C
import os
from typing import Optional

F32, BF16, FP8_E4M3 = 0, 1, 2
TRUST, KL_THRESH, CONF_THRESH, KL_PROB, CONF_PROB, KL_TOPK, CONF_TOPK = 0, 1, 2, 3, 4, 5, 6
UNMASK_THRESH, UNMASK_TOPK = 0, 1

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libdd.so")
BINDING_PATH = os.path.join(_HERE, "_binding.so")
_lib = None
_native = None


class DDError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {lib().dd_strerror(status).decode()} (status {status})")


def lib():
    """The loaded C-ABI library (built on first use only when no built library exists)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        from .build import build_library
        build_library(force=True)
    # torch ships its own copy of the HIP runtime (same soname).  It has to be mapped first so
    # that this library binds to that copy: streams and device pointers handed over by torch
    # are only valid inside the runtime instance that created them.
    import torch  # noqa: F401
    L = C.CDLL(LIB_PATH)
    vp, i, sz = C.c_void_p, C.c_int, C.c_size_t
    L.dd_strerror.restype = C.c_char_p
    L.dd_strerror.argtypes = [i]
    L.dd_version.restype = i
    L.dd_bidir_attention.restype = i
    L.dd_bidir_attention.argtypes = [vp, vp, vp, vp, i, i, i, i, i, i, i, vp, vp, vp, sz, vp]
    L.dd_bidir_attention_workspace_bytes.restype = sz
    L.dd_bidir_attention_workspace_bytes.argtypes = [i, i, i, i, i, i, i]
    L.dd_block_attention_cached.restype = i
    L.dd_block_attention_cached.argtypes = [vp, vp, vp, vp, i, i, vp, vp, i, i, i, i, i, i, i, vp, vp, vp, sz, vp]
    L.dd_block_attention_cached_workspace_bytes.restype = sz
    L.dd_block_attention_cached_workspace_bytes.argtypes = [i, i, i, i, i, i, i, i]
    L.dd_bidir_attention_fp8v.restype = i
    L.dd_bidir_attention_fp8v.argtypes = [vp, vp, vp, vp, i, i, i, i, i, vp, vp, vp, vp]
    L.dd_bidir_attention_mx.restype = i
    L.dd_bidir_attention_mx.argtypes = [vp, vp, vp, vp, vp, vp, vp, i, i, i, i, i, vp]
    L.dd_block_attention_cached_fp8v.restype = i
    L.dd_block_attention_cached_fp8v.argtypes = [vp, vp, vp, vp, i, i, vp, vp, i, i, i, i, i, vp, vp, vp, vp, sz, vp]
    L.dd_block_attention_cached_fp8v_workspace_bytes.restype = sz
    L.dd_block_attention_cached_fp8v_workspace_bytes.argtypes = [i, i, i, i, i, i]
    L.dd_verify_remask.restype = i
    L.dd_verify_remask.argtypes = [vp, vp, vp, i, C.c_float, C.c_uint64, vp, vp, vp, i, i, i, i, vp, sz, vp]
    L.dd_verify_remask_workspace_bytes.restype = sz
    L.dd_verify_remask_workspace_bytes.argtypes = [i, i, i, i]
    L.dd_verify_remask_static.restype = i
    L.dd_verify_remask_static.argtypes = [vp, vp, vp, i, C.c_float, C.c_uint64, vp, vp, vp, i, i, i, i, vp]
    L.dd_unmask.restype = i
    L.dd_unmask.argtypes = [vp, vp, i, C.c_float, vp, vp, vp, vp, i, i, i, i, vp, sz, vp]
    L.dd_unmask_workspace_bytes.restype = sz
    L.dd_unmask_workspace_bytes.argtypes = [i, i, i, i]
    L.dd_block_attention_refresh.restype = i
    L.dd_block_attention_refresh.argtypes = [vp, vp, vp, vp, i, i, vp, vp, i, i, i, i, i, i, i, vp, vp, vp, sz, vp]
    L.dd_block_attention_refresh_workspace_bytes.restype = sz
    L.dd_block_attention_refresh_workspace_bytes.argtypes = [i, i, i, i, i, i, i, i]
    L.dd_block_attention_window.restype = i
    L.dd_block_attention_window.argtypes = [vp, vp, vp, vp, i, i, i, i, vp, vp, i, i, i, i, i, i, i, vp, vp, vp, sz, vp]
    L.dd_block_attention_window_workspace_bytes.restype = sz
    L.dd_block_attention_window_workspace_bytes.argtypes = [i, i, i, i, i, i, i, i, i]
    L.dd_block_attention_batched.restype = i
    L.dd_block_attention_batched.argtypes = [vp, vp, vp, vp, vp, i, vp, vp, i, i, i, i, i, i, i, vp, vp, vp, sz, vp]
    L.dd_block_attention_batched_workspace_bytes.restype = sz
    L.dd_block_attention_batched_workspace_bytes.argtypes = [i, i, i, i, i, i, i, i]
    L.dd_cache_insert_rows.restype = i
    L.dd_cache_insert_rows.argtypes = [vp, vp, vp, vp, vp, i, i, i, i, i, i, i, vp]
    L.dd_verify_scores.restype = i
    L.dd_verify_scores.argtypes = [vp, vp, vp, vp, vp, vp, vp, i, i, i, vp, sz, vp]
    L.dd_verify_scores_workspace_bytes.restype = sz
    L.dd_verify_scores_workspace_bytes.argtypes = [i, i, i]
    _lib = L
    return L


EXPORTS = ("dd_strerror", "dd_version", "dd_bidir_attention", "dd_bidir_attention_workspace_bytes",
           "dd_block_attention_cached", "dd_block_attention_cached_workspace_bytes",
           "dd_verify_remask", "dd_verify_remask_workspace_bytes", "dd_verify_remask_static", "dd_unmask", "dd_unmask_workspace_bytes",
           "dd_verify_scores", "dd_verify_scores_workspace_bytes",
           "dd_block_attention_refresh", "dd_block_attention_refresh_workspace_bytes",
           "dd_block_attention_window", "dd_block_attention_window_workspace_bytes", "dd_cache_insert_rows",
           "dd_block_attention_batched", "dd_block_attention_batched_workspace_bytes",
           "dd_bidir_attention_fp8v", "dd_block_attention_cached_fp8v", "dd_block_attention_cached_fp8v_workspace_bytes",
           "dd_bidir_attention_mx")


# ---------------------------------------------------------------- marshalling (csrc/binding.cpp)
def native():
    """The binding's native module (built on first use only when no built one exists)."""
    global _native
    if _native is not None:
        return _native
    lib()                                         # first: it brings torch's HIP runtime with it
    if not os.path.exists(BINDING_PATH):
        from .build import build_binding
        build_binding()
    from importlib.machinery import ExtensionFileLoader
    from importlib.util import module_from_spec, spec_from_file_location
    name = __name__ + "._binding"
    spec = spec_from_file_location(name, BINDING_PATH, loader=ExtensionFileLoader(name, BINDING_PATH))
    mod = module_from_spec(spec)
    spec.loader.exec_module(mod)
    mod.set_error_class(DDError)
    _native = mod
    return mod


def reset_workspace_peak() -> None:
    native().reset_workspace_peak()


def workspace_peak() -> int:
    """The largest scratch size any call has asked for since reset_workspace_peak()."""
    return native().workspace_peak()


class fixed_workspace:
    """Context manager: calls of the binding inside it use `tensor` (uint8, on the GPU) as their scratch memory
    instead of the per-stream cached one; they must all be ordered on one stream.  For graph capture: the
    tensor is allocated before the capture and kept alive by whoever keeps the graph."""

    def __init__(self, tensor):
        self.tensor = tensor

    def __enter__(self):
        self.prev = native().set_fixed_workspace(self.tensor)
        return self.tensor

    def __exit__(self, *exc):
        native().set_fixed_workspace(self.prev)
        return False


# ---------------------------------------------------------------- entry points
def dd_bidir_attention_workspace_bytes(B, H, Hkv, N, d, qk_dtype, v_dtype) -> int:
    return lib().dd_bidir_attention_workspace_bytes(B, H, Hkv, N, d, qk_dtype, v_dtype)


def dd_bidir_attention(Q, K, V, O=None, q_scale=None, k_scale=None, qk_dtype: Optional[int] = None,
                       v_dtype: Optional[int] = None):
    """Verifier attention over all positions.  Q [B,H,N,d], K,V [B,Hkv,N,d] -> O [B,H,N,d] (V's type)."""
    return native().bidir(Q, K, V, O, q_scale, k_scale, qk_dtype, v_dtype)


def dd_block_attention_cached_workspace_bytes(block_len, B, H, Hkv, N, d, qk_dtype, v_dtype) -> int:
    return lib().dd_block_attention_cached_workspace_bytes(block_len, B, H, Hkv, N, d, qk_dtype, v_dtype)


def dd_block_attention_cached(Qblk, Kc, Vc, block_start: int, O=None, Kblk=None, Vblk=None, q_scale=None,
                              k_scale=None, qk_dtype: Optional[int] = None, v_dtype: Optional[int] = None,
                              _refresh: bool = False):
    """Drafter attention: the active block's queries over cached K/V.
    Qblk [B,H,bl,d], Kc,Vc [B,Hkv,N,d], optional Kblk,Vblk [B,Hkv,bl,d] -> O [B,H,bl,d]."""
    return native().block(1 if _refresh else 0, Qblk, Kc, Vc, block_start, 0, 0, O, Kblk, Vblk, q_scale, k_scale,
                          qk_dtype, v_dtype)


def dd_bidir_attention_fp8v(Q, K, V, q_scale, k_scale, v_scale, O=None):
    """Verifier attention with Q, K and V all stored as e4m3 codes (uint8) and per-head fp32 scales -> O bf16
    (as int16 bit patterns unless O is given)."""
    return native().bidir_fp8v(Q, K, V, q_scale, k_scale, v_scale, O)


def dd_bidir_attention_mx(Q, Qs, K, Ks, V, Vs, O=None):
    """Verifier attention on block-scaled inputs: Q [B,H,N,d], K [B,Hkv,N,d] e4m3 codes, V [B,Hkv,N,d/2] packed e2m1
    codes, each with E8M0 scales [..., d/32] (all uint8) -> O bf16 (as int16 bit patterns unless O is given)."""
    return native().bidir_mx(Q, Qs, K, Ks, V, Vs, O)


def dd_block_attention_cached_fp8v(Qblk, Kc, Vc, block_start: int, q_scale, k_scale, v_scale, O=None, Kblk=None, Vblk=None):
    """Drafter attention with every operand stored as e4m3 codes; shapes as for dd_block_attention_cached -> O bf16."""
    return native().block_fp8v(Qblk, Kc, Vc, block_start, q_scale, k_scale, v_scale, O, Kblk, Vblk)


def dd_block_attention_refresh_workspace_bytes(block_len, B, H, Hkv, N, d, qk_dtype, v_dtype) -> int:
    return lib().dd_block_attention_refresh_workspace_bytes(block_len, B, H, Hkv, N, d, qk_dtype, v_dtype)


def dd_block_attention_refresh(Qblk, Kc, Vc, block_start: int, Kblk, Vblk, O=None, q_scale=None, k_scale=None,
                               qk_dtype: Optional[int] = None, v_dtype: Optional[int] = None):
    """Drafter attention of a completed block: as dd_block_attention_cached with Kblk/Vblk, and rows
    [block_start, block_start + bl) of Kc / Vc are overwritten with Kblk / Vblk in the same call."""
    return dd_block_attention_cached(Qblk, Kc, Vc, block_start, O=O, Kblk=Kblk, Vblk=Vblk, q_scale=q_scale,
                                     k_scale=k_scale, qk_dtype=qk_dtype, v_dtype=v_dtype, _refresh=True)


def dd_block_attention_window_workspace_bytes(block_len, win_len, B, H, Hkv, N, d, qk_dtype, v_dtype) -> int:
    return lib().dd_block_attention_window_workspace_bytes(block_len, win_len, B, H, Hkv, N, d, qk_dtype, v_dtype)


def dd_block_attention_window(Qblk, Kc, Vc, block_start: int, win_start: int, win_len: int, O=None, Kblk=None,
                              Vblk=None, q_scale=None, k_scale=None, qk_dtype: Optional[int] = None,
                              v_dtype: Optional[int] = None):
    """Drafter attention over the key rows [win_start, win_start + win_len) of the cache only.
    Shapes as for dd_block_attention_cached (Kc, Vc are the whole cache)."""
    return native().block(2, Qblk, Kc, Vc, block_start, win_start, win_len, O, Kblk, Vblk, q_scale, k_scale,
                          qk_dtype, v_dtype)


def dd_block_attention_batched(Qblk, Kc, Vc, block_starts, Kblk, Vblk, O=None, q_scale=None, k_scale=None,
                               qk_dtype: Optional[int] = None, v_dtype: Optional[int] = None):
    """Drafter attention with one block position per batch entry: block_starts [B] i32 on the device."""
    return native().block(3, Qblk, Kc, Vc, block_starts, 0, 0, O, Kblk, Vblk, q_scale, k_scale, qk_dtype, v_dtype)


def dd_cache_insert_rows(Kc, Vc, Krows, Vrows, positions, qk_dtype: Optional[int] = None, v_dtype: Optional[int] = None):
    """Kc/Vc [B,Hkv,N,d] <- rows of Krows/Vrows [B,Hkv,n,d] at positions [B,n] (i32, on the device; entries outside
    [0, N) skip their row).  In place; returns None."""
    native().cache_insert(Kc, Vc, Krows, Vrows, positions, qk_dtype, v_dtype)


def dd_verify_remask_workspace_bytes(B, G, V, logit_dtype) -> int:
    return lib().dd_verify_remask_workspace_bytes(B, G, V, logit_dtype)


def dd_verify_remask(logits_d, logits_v, mask, mode: int, threshold: float, seed: int, B: int, G: int,
                     out_mask=None, out_tokens=None, out_scores=None, logit_dtype: Optional[int] = None):
    """Verification rule over the vocabulary.  logits [B*G, V]; mask [B*G] u8 (1 = still masked).
    Returns (out_mask u8, out_tokens i32, out_scores f32)."""
    return native().verify_remask(0, logits_d, logits_v, mask, mode, threshold, seed, B, G, out_mask, out_tokens, out_scores,
                                  logit_dtype)


def dd_verify_remask_static(logits_d, logits_v, mask, mode: int, threshold: float, seed: int, B: int, G: int,
                            out_mask, out_tokens, out_scores, logit_dtype: Optional[int] = None):
    """dd_verify_remask without a workspace: the library's static device array holds the partial states.  The
    three output tensors are the caller's (nothing is allocated here either).  Returns them."""
    return native().verify_remask(1, logits_d, logits_v, mask, mode, threshold, seed, B, G, out_mask, out_tokens, out_scores,
                                  logit_dtype)


def dd_unmask_workspace_bytes(B, G, V, logit_dtype) -> int:
    return lib().dd_unmask_workspace_bytes(B, G, V, logit_dtype)


def dd_unmask(logits_d, mask, mode: int, threshold: float, B: int, G: int, x_tokens=None, out_mask=None,
              out_tokens=None, out_conf=None, logit_dtype: Optional[int] = None):
    """One drafter unmasking step.  logits_d [B*G, V]; mask [B*G] u8 (1 = still masked); x_tokens [B*G] i32
    (optional, updated in place where a position is revealed).  Returns (out_mask u8, out_tokens i32, out_conf f32)."""
    return native().unmask(logits_d, mask, mode, threshold, B, G, x_tokens, out_mask, out_tokens, out_conf, logit_dtype)


def dd_verify_scores_workspace_bytes(P, V, logit_dtype) -> int:
    return lib().dd_verify_scores_workspace_bytes(P, V, logit_dtype)


def dd_verify_scores(logits_d, logits_v, drafter: bool = True, logit_dtype: Optional[int] = None):
    """Divergence, both confidences and both argmax tokens of every row in one pass.  logits_d, logits_v [P, V].
    Returns (kl f32, conf_v f32, tok_v i32, conf_d f32 | None, tok_d i32 | None)."""
    return native().verify_scores(logits_d, logits_v, drafter, logit_dtype)