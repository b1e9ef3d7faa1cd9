"""Python binding of include/hydra_attn.h.  Argument marshalling only, in native code (csrc/torch_binding.cpp):
tensors in, raw device pointers and sizes out; every step of the computation runs in the HIP kernels.  There is no
fallback: if the shared library or its binding is missing, loading raises."""
from __future__ import annotations

import ctypes
import importlib.util
import os
from typing import Optional

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libhydra_attn.so")
_NATIVE_PATH = os.path.join(_HERE, "_hydra_torch.so")
_lib = None
_native = None

HYDRA_OK = 0


class HydraError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {hydra_status_string(status)} (status {status})")


def library_path() -> str:
    return _LIB_PATH


def load_library() -> ctypes.CDLL:
    """dlopen the in-tree library and its native binding; returns the library through ctypes, for callers that pass raw
    pointers.  Raises if they have not been built (python -m paper_2505_12658_amd.build)."""
    global _lib, _native
    if _lib is None:
        for path in (_LIB_PATH, _NATIVE_PATH):
            if not os.path.exists(path):
                raise ImportError(f"{path} is missing: build it with `python -m paper_2505_12658_amd.build`; "
                                  "there is no CPU or PyTorch fallback for this library")
        lib = ctypes.CDLL(_LIB_PATH)
        vp, i32, i64, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_size_t
        lib.hydra_attn_varlen_fwd.restype = ctypes.c_int
        lib.hydra_attn_varlen_fwd.argtypes = [vp, vp, vp, vp, i64, i64, i64, vp, i32, i32, i32, i32, i32, i32, i32, ctypes.c_float,
                                              vp, sz, vp]
        lib.hydra_attn_varlen_fwd_prebuilt.restype = ctypes.c_int
        lib.hydra_attn_varlen_fwd_prebuilt.argtypes = lib.hydra_attn_varlen_fwd.argtypes
        lib.hydra_attn_varlen_fwd_shared.restype = ctypes.c_int
        lib.hydra_attn_varlen_fwd_shared.argtypes = lib.hydra_attn_varlen_fwd.argtypes[:-1] + [i32, vp]
        lib.hydra_attn_varlen_fwd_static.restype = ctypes.c_int
        lib.hydra_attn_varlen_fwd_static.argtypes = lib.hydra_attn_varlen_fwd.argtypes[:-3] + [vp]
        lib.hydra_attn_build_worklist.restype = ctypes.c_int
        lib.hydra_attn_build_worklist.argtypes = [vp, i32, i32, i32, i32, i32, i32, i32, vp, sz, vp]
        lib.hydra_kv_cache_write.restype = ctypes.c_int
        lib.hydra_kv_cache_write.argtypes = [vp, vp, i64, i64, vp, vp, vp, i32, i32, i32, i32, i64, vp]
        lib.hydra_attn_paged_fwd.restype = ctypes.c_int
        lib.hydra_attn_paged_fwd.argtypes = [vp, vp, i64, vp, vp, vp, i32, vp, vp, i32, i32, i32, i32, i32, i32, i32, i64, ctypes.c_float, vp, sz, vp]
        lib.hydra_attn_paged_workspace_bytes.restype = sz
        lib.hydra_attn_paged_workspace_bytes.argtypes = [i32] * 5
        lib.hydra_page_cache_write.restype = ctypes.c_int
        lib.hydra_page_cache_write.argtypes = [vp, i64, vp, vp, i32, i32, i64, vp]
        lib.hydra_page_cache_gather.restype = ctypes.c_int
        lib.hydra_page_cache_gather.argtypes = [vp, vp, vp, i64, i32, i32, i64, vp]
        lib.hydra_attn_workspace_bytes.restype = sz
        lib.hydra_attn_workspace_bytes.argtypes = [i32] * 6
        lib.hydra_status_string.restype = ctypes.c_char_p
        lib.hydra_status_string.argtypes = [ctypes.c_int]
        spec = importlib.util.spec_from_file_location("_hydra_torch", _NATIVE_PATH)
        native = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(native)
        native.load(_LIB_PATH, HydraError)
        _native, _lib = native, lib  # (_lib last: it is what other threads look at)
    return _lib


def _calls():
    if _lib is None:
        load_library()
    return _native


def hydra_status_string(status: int) -> str:
    return load_library().hydra_status_string(int(status)).decode()


def hydra_attn_workspace_bytes(batch: int, total_tokens: int, max_seqlen: int, n_q_heads: int, n_kv_heads: int, head_dim: int) -> int:
    return int(load_library().hydra_attn_workspace_bytes(batch, total_tokens, max_seqlen, n_q_heads, n_kv_heads, head_dim))


def hydra_attn_paged_workspace_bytes(batch: int, n_kv_heads: int, head_dim: int, max_blocks_per_seq: int, block_size: int) -> int:
    return int(load_library().hydra_attn_paged_workspace_bytes(batch, n_kv_heads, head_dim, max_blocks_per_seq, block_size))


def hydra_attn_varlen_fwd(q: torch.Tensor, k: torch.Tensor, v: torch.Tensor, cu_seqlens: torch.Tensor, max_seqlen: int, causal: bool,
                          softmax_scale: float, out: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None,
                          stream: Optional[torch.cuda.Stream] = None) -> torch.Tensor:
    """q [N, Hq, d], k/v [N, Hkv, d] bf16 (token-strided views allowed), cu_seqlens int32 [B+1] on the device."""
    return _calls().attn_varlen_fwd(q, k, v, cu_seqlens, max_seqlen, causal, softmax_scale, out, workspace, stream)


def hydra_attn_varlen_fwd_static(q: torch.Tensor, k: torch.Tensor, v: torch.Tensor, cu_seqlens: torch.Tensor, max_seqlen: int, causal: bool,
                                 softmax_scale: float, out: torch.Tensor, stream: Optional[torch.cuda.Stream] = None) -> torch.Tensor:
    """hydra_attn_varlen_fwd with the work list in the library's own static device array: nothing is allocated,
    here or in the library, so `out` is the caller's."""
    return _calls().attn_varlen_fwd_static(q, k, v, cu_seqlens, max_seqlen, causal, softmax_scale, out, stream)


def hydra_attn_build_worklist(cu_seqlens: torch.Tensor, total_tokens: int, max_seqlen: int, n_q_heads: int, n_kv_heads: int, head_dim: int,
                              causal: bool, workspace: Optional[torch.Tensor] = None, stream: Optional[torch.cuda.Stream] = None) -> torch.Tensor:
    """Builds the tile work list for one packed batch into `workspace` (allocated if None) and returns it."""
    return _calls().attn_build_worklist(cu_seqlens, total_tokens, max_seqlen, n_q_heads, n_kv_heads, head_dim, causal, workspace, stream)


def hydra_attn_varlen_fwd_prebuilt(q: torch.Tensor, k: torch.Tensor, v: torch.Tensor, cu_seqlens: torch.Tensor, max_seqlen: int,
                                   causal: bool, softmax_scale: float, out: torch.Tensor, workspace: torch.Tensor,
                                   stream: Optional[torch.cuda.Stream] = None) -> torch.Tensor:
    """Attention against a work list built earlier by hydra_attn_build_worklist for the same batch."""
    return _calls().attn_varlen_fwd_prebuilt(q, k, v, cu_seqlens, max_seqlen, causal, softmax_scale, out, workspace, None, stream)


def hydra_attn_varlen_fwd_shared(q: torch.Tensor, k: torch.Tensor, v: torch.Tensor, cu_seqlens: torch.Tensor, max_seqlen: int,
                                 causal: bool, softmax_scale: float, out: torch.Tensor, workspace: torch.Tensor, workgroups_per_cu: int,
                                 stream: Optional[torch.cuda.Stream] = None) -> torch.Tensor:
    """hydra_attn_varlen_fwd_prebuilt with at most `workgroups_per_cu` persistent workgroups per compute unit, for a caller
    that runs another kernel beside it on a second stream."""
    return _calls().attn_varlen_fwd_prebuilt(q, k, v, cu_seqlens, max_seqlen, causal, softmax_scale, out, workspace, int(workgroups_per_cu), stream)


def hydra_kv_cache_write(k: torch.Tensor, v: torch.Tensor, k_cache: torch.Tensor, v_cache: torch.Tensor, slot_mapping: torch.Tensor,
                         stream: Optional[torch.cuda.Stream] = None) -> None:
    """k/v [N, Hkv, d] bf16; caches [num_blocks, block_size, Hkv, d] bf16 contiguous; slot_mapping int64 [N]."""
    _calls().kv_cache_write(k, v, k_cache, v_cache, slot_mapping, stream)


def hydra_attn_paged_fwd(q: torch.Tensor, k_cache: torch.Tensor, v_cache: torch.Tensor, block_tables: torch.Tensor,
                         cu_seqlens_q: torch.Tensor, kv_lens: torch.Tensor, max_q_len: int, softmax_scale: float,
                         out: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None, use_workspace: bool = True,
                         stream: Optional[torch.cuda.Stream] = None) -> torch.Tensor:
    """q [Nq, Hq, d] bf16 (new tokens of all requests, packed); caches [num_blocks, block_size, Hkv, d] bf16 contiguous;
    block_tables int32 [B, max_blocks_per_seq]; cu_seqlens_q int32 [B+1]; kv_lens int32 [B] (context lengths, new tokens included).
    workspace: uint8 tensor for the split of decode contexts over workgroups (allocated at the size the library asks for when
    None and use_workspace; use_workspace=False runs without splitting)."""
    return _calls().attn_paged_fwd(q, k_cache, v_cache, block_tables, cu_seqlens_q, kv_lens, max_q_len, softmax_scale, out, workspace,
                                   use_workspace, stream)


def hydra_page_cache_write(rows: torch.Tensor, cache: torch.Tensor, slot_mapping: torch.Tensor, stream: Optional[torch.cuda.Stream] = None) -> None:
    """rows [n, row_elems] bf16 (row-strided view allowed) -> cache [pages, page_rows, row_elems] at slot_mapping (int64 [n], < 0 skips)."""
    _calls().page_cache_write(rows, cache, slot_mapping, stream)


def hydra_page_cache_gather(cache: torch.Tensor, slot_mapping: torch.Tensor, rows: torch.Tensor, stream: Optional[torch.cuda.Stream] = None) -> None:
    """cache rows at slot_mapping -> rows [n, row_elems] bf16 (row-strided view allowed); rows with a negative slot keep their contents."""
    _calls().page_cache_gather(cache, slot_mapping, rows, stream)
