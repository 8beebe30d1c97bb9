"""Binding of libdream.so: same names and argument order as include/dream.h.

Device buffers are torch tensors (only their data_ptr() crosses the boundary); sizes are Python
ints; `stream` is a torch.cuda.Stream or None (= torch's current stream).  Every wrapper raises
DreamError on a non-zero status.  Nothing is computed here.  The calls that work on tensors go through the
extension built from csrc/call.cpp, the host-only ones through ctypes.
"""
from __future__ import annotations

import ctypes as C
import os
from typing import Optional, Sequence

import numpy as np
import torch

F32, BF16 = 0, 1
_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libdream.so")

EXPORTED_SYMBOLS = (
    "dream_init", "dream_tree_verify_attn_workspace", "dream_tree_verify_attn",
    "dream_draft_xattn_workspace", "dream_draft_xattn", "dream_visual_compress_workspace",
    "dream_visual_compress", "dream_accept_path_workspace", "dream_accept_path",
    "dream_tree_validate_host", "dream_last_error", "dream_set_kv_splits", "dream_set_q_tiles", "dream_set_tile_waves", "dream_set_accept_spin", "dream_attn_variants",
    "dream_attn_plan_describe", "dream_stream_read", "dream_kv_commit",
    "dream_tree_expand_workspace", "dream_tree_expand_level", "dream_tree_finalize",
    "dream_attention_entropy_workspace", "dream_attention_entropy", "dream_spec_accept_workspace", "dream_spec_accept",
    "dream_project_rows", "dream_project_rows_multi", "dream_accept_path_static", "dream_accept_static_init",
)


_raw_stream = torch._C._cuda_getCurrentRawStream
_current_device = torch.cuda.current_device


class DreamError(RuntimeError):
    def __init__(self, status: int, message: str):
        super().__init__(f"libdream status {status}: {message}")
        self.status = status


class AttnDesc(C.Structure):
    _fields_ = [("batch", C.c_int32), ("n_q_heads", C.c_int32), ("n_kv_heads", C.c_int32),
                ("head_dim", C.c_int32), ("dtype", C.c_int32), ("scale", C.c_float), ("s_max", C.c_int64)]


def attn_desc(batch: int, n_q_heads: int, n_kv_heads: int, head_dim: int, dtype: int, s_max: int,
              scale: float = 0.0) -> AttnDesc:
    return AttnDesc(batch, n_q_heads, n_kv_heads, head_dim, dtype, scale, s_max)


_lib: Optional[C.CDLL] = None


def library_path() -> str:
    return _LIB_PATH


def load() -> C.CDLL:
    """Load libdream.so.  Raises if it has not been built (python -m paper_2505_19201_amd.build)."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise FileNotFoundError(f"{_LIB_PATH} is missing: build it with `python -m paper_2505_19201_amd.build`; "
                                    "there is no fallback path")
        lib = C.CDLL(_LIB_PATH)
        for name in EXPORTED_SYMBOLS:
            getattr(lib, name)
        for name in ("dream_tree_verify_attn_workspace", "dream_draft_xattn_workspace",
                     "dream_visual_compress_workspace", "dream_accept_path_workspace", "dream_tree_expand_workspace",
                     "dream_attention_entropy_workspace", "dream_spec_accept_workspace"):
            getattr(lib, name).restype = C.c_size_t
        lib.dream_last_error.restype = C.c_char_p
        lib.dream_set_kv_splits.restype = None
        lib.dream_set_q_tiles.restype = None
        lib.dream_set_tile_waves.restype = None
        lib.dream_set_accept_spin.restype = None
        _lib = lib
    return _lib


_call = None


def _native():
    """The extension that converts arguments and calls the library (built with it)."""
    global _call
    if _call is None:
        load()
        from . import _call as module
        _call = module
    return _call


def _dev(t: Optional[torch.Tensor]):
    if t is None:
        return None
    if not t.is_cuda:
        raise ValueError("device tensor expected")
    if not t.is_contiguous():
        raise ValueError("contiguous tensor expected")
    return t.data_ptr()


def _stream(stream) -> int:
    # torch.cuda.current_stream() would build a Stream object: the raw handle of the same stream costs a tenth of it
    return _raw_stream(_current_device()) if stream is None else stream.cuda_stream


def _check(status: int) -> None:
    if status != 0:
        raise DreamError(status, load().dream_last_error().decode())


def dream_last_error() -> str:
    return load().dream_last_error().decode()


def dream_set_kv_splits(n_splits: int) -> None:
    load().dream_set_kv_splits(C.c_int32(n_splits))


def dream_set_q_tiles(q_tiles: int) -> None:
    load().dream_set_q_tiles(C.c_int32(q_tiles))


def dream_set_tile_waves(waves: int) -> None:
    load().dream_set_tile_waves(C.c_int32(waves))


def dream_set_accept_spin(polls: int) -> None:
    load().dream_set_accept_spin(C.c_int32(polls))


def dream_stream_read(src: torch.Tensor, nbytes: int, sink: torch.Tensor, offset_bytes: int = 0, stream=None) -> None:
    if offset_bytes < 0 or offset_bytes + nbytes > src.numel() * src.element_size():
        raise ValueError("range outside the source tensor")
    _check(load().dream_stream_read(C.c_void_p(src.data_ptr() + offset_bytes), C.c_size_t(nbytes), C.c_void_p(_dev(sink)), C.c_void_p(_stream(stream))))


def dream_attn_variants() -> list:
    buf = C.create_string_buffer(4096)
    _check(load().dream_attn_variants(buf, C.c_size_t(4096)))
    return buf.value.decode().split(";")


def dream_attn_plan_describe(desc: "AttnDesc", n_q: int, max_kv_len: int) -> str:
    buf = C.create_string_buffer(256)
    _check(load().dream_attn_plan_describe(C.byref(desc), C.c_int32(n_q), C.c_int64(max_kv_len), buf, C.c_size_t(256)))
    return buf.value.decode()


def dream_init() -> None:
    _check(load().dream_init())


def alloc_workspace(nbytes: int, device="cuda") -> torch.Tensor:
    """Device scratch of at least nbytes (allocation is the caller's job in C; the content needs no initialisation)."""
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=device)


def to_device(a: np.ndarray, dtype: Optional[str] = None, device="cuda") -> torch.Tensor:
    """Upload a host array; uint16 arrays tagged "bf16" become torch.bfloat16 views of the same bits."""
    if dtype == "bf16" or (dtype is None and a.dtype == np.uint16):
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).to(device).view(torch.bfloat16)
    if a.dtype == np.uint64:
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to(device)
    return torch.from_numpy(np.ascontiguousarray(a)).to(device)


def dream_tree_verify_attn_workspace(desc: AttnDesc, n_tree: int, max_kv_len: int) -> int:
    return int(load().dream_tree_verify_attn_workspace(C.byref(desc), C.c_int32(n_tree), C.c_int64(max_kv_len)))


def dream_tree_verify_attn(desc: AttnDesc, q, k_cache, v_cache, prefix_len, n_tree: int, parent, tree_mask,
                           max_kv_len: int, out, lse, workspace, stream=None) -> None:
    _check(_native().dream_tree_verify_attn(desc, q, k_cache, v_cache, prefix_len, n_tree, parent, tree_mask, max_kv_len, out, lse,
                                            workspace, workspace, _stream(stream)))


def dream_draft_xattn_workspace(desc: AttnDesc, n_q: int, max_kv_len: int) -> int:
    return int(load().dream_draft_xattn_workspace(C.byref(desc), C.c_int32(n_q), C.c_int64(max_kv_len)))


def dream_draft_xattn(desc: AttnDesc, q, kx_cache, vx_cache, prefix_len, n_tree: int, parent, n_q: int, q_node,
                      max_kv_len: int, out, workspace, stream=None) -> None:
    _check(_native().dream_draft_xattn(desc, q, kx_cache, vx_cache, prefix_len, n_tree, parent, n_q, q_node, max_kv_len, out, workspace,
                                       workspace, _stream(stream)))


def dream_visual_compress_workspace(desc: AttnDesc, n_q: int, vis_len: int) -> int:
    return int(load().dream_visual_compress_workspace(C.byref(desc), C.c_int32(n_q), C.c_int32(vis_len)))


def dream_visual_compress(desc: AttnDesc, q, q_pos, n_q: int, k_cache, n_keys: int, vis_start: int, vis_len: int,
                          keep_num: int, keep_den: int, scores_in, scores_out, kept_idx, gather_src, n_rows_src: int,
                          gather_dst, row_elems: int, workspace, stream=None, row_lse_in=None) -> int:
    """Returns k, the kept count the library reports through its host out-parameter."""
    n_kept = C.c_int32(-1)
    _check(_native().dream_visual_compress(desc, q, q_pos, n_q, k_cache, n_keys, vis_start, vis_len, keep_num, keep_den, scores_in,
                                           row_lse_in, scores_out, kept_idx, n_kept, gather_src, n_rows_src, gather_dst, row_elems,
                                           workspace, workspace, _stream(stream)))
    return int(n_kept.value)


def dream_accept_path_workspace(batch: int, n_tree: int, vocab: int) -> int:
    return int(load().dream_accept_path_workspace(C.c_int32(batch), C.c_int32(n_tree), C.c_int32(vocab)))


def dream_accept_path(logits, logits_dtype: int, batch: int, n_tree: int, vocab: int, token, parent, max_depth: int,
                      node_argmax, accept_len, accept_path, bonus_token, workspace, stream=None) -> None:
    _check(_native().dream_accept_path(logits, logits_dtype, batch, n_tree, vocab, token, parent, max_depth, node_argmax, accept_len,
                                       accept_path, bonus_token, workspace, workspace, _stream(stream)))


def dream_accept_static_init() -> None:
    _check(load().dream_accept_static_init())


def dream_accept_path_static(logits, logits_dtype: int, batch: int, n_tree: int, vocab: int, token, parent, max_depth: int,
                             node_argmax, accept_len, accept_path, bonus_token, stream=None) -> None:
    _check(_native().dream_accept_path_static(logits, logits_dtype, batch, n_tree, vocab, token, parent, max_depth, node_argmax,
                                              accept_len, accept_path, bonus_token, _stream(stream)))


def dream_kv_commit(desc: AttnDesc, caches: Sequence[torch.Tensor], prefix_len: torch.Tensor, n_tree: int,
                    accept_path: torch.Tensor, accept_len: torch.Tensor, prefix_len_out: Optional[torch.Tensor] = None,
                    stream=None) -> None:
    caches = tuple(caches)     # the count handed over is that of the pointers, whatever kind of sequence this is
    _check(_native().dream_kv_commit(desc, caches, len(caches), prefix_len, n_tree, accept_path, accept_path.shape[-1], accept_len,
                                     prefix_len_out, _stream(stream)))


def dream_project_rows(desc: AttnDesc, x, n_rows: int, hidden: int, w, n_heads: int, row_base, row_index, out, stream=None) -> None:
    _check(_native().dream_project_rows(desc, x, n_rows, hidden, w, n_heads, row_base, row_index, out, _stream(stream)))


class ProjJob(C.Structure):
    """The C layout of a job (dream_proj_job), for callers of the library itself."""
    _fields_ = [("x", C.c_void_p), ("w", C.c_void_p), ("n_heads", C.c_int32), ("row_base", C.c_void_p),
                ("row_index", C.c_void_p), ("out", C.c_void_p)]


def dream_project_rows_multi(desc: AttnDesc, jobs, n_rows: int, hidden: int, stream=None) -> None:
    """jobs: sequence of (x, w, n_heads, row_base, row_index, out)."""
    jobs = tuple(jobs)         # (see dream_kv_commit)
    _check(_native().dream_project_rows_multi(desc, jobs, len(jobs), n_rows, hidden, _stream(stream)))


def dream_spec_accept_workspace(batch: int, n_tree: int, vocab: int) -> int:
    return int(load().dream_spec_accept_workspace(C.c_int32(batch), C.c_int32(n_tree), C.c_int32(vocab)))


def dream_spec_accept(target_logits, draft_logits, logits_dtype: int, batch: int, n_tree: int, vocab: int, token, parent,
                      u_accept, u_bonus, max_depth: int, temperature: float, accept_len, accept_path, bonus_token, workspace,
                      stream=None) -> None:
    _check(_native().dream_spec_accept(target_logits, draft_logits, logits_dtype, batch, n_tree, vocab, token, parent, u_accept,
                                       u_bonus, max_depth, temperature, accept_len, accept_path, bonus_token, workspace, workspace,
                                       _stream(stream)))


def dream_attention_entropy_workspace(desc: AttnDesc, n_q: int) -> int:
    return int(load().dream_attention_entropy_workspace(C.byref(desc), C.c_int32(n_q)))


def dream_attention_entropy(desc: AttnDesc, q, q_pos, n_q: int, k_cache, n_keys: int, row_entropy, ae, workspace, stream=None) -> None:
    _check(_native().dream_attention_entropy(desc, q, q_pos, n_q, k_cache, n_keys, row_entropy, ae, workspace, workspace,
                                             _stream(stream)))


def dream_tree_expand_workspace(batch: int, n_frontier: int, vocab: int, k: int) -> int:
    return int(load().dream_tree_expand_workspace(C.c_int32(batch), C.c_int32(n_frontier), C.c_int32(vocab), C.c_int32(k)))


def dream_tree_expand_level(logits: torch.Tensor, logits_dtype: int, batch: int, n_frontier: int, vocab: int,
                            cum_in: torch.Tensor, k: int, cand_token: torch.Tensor, cand_score: torch.Tensor,
                            next_frontier: torch.Tensor, workspace: torch.Tensor, stream=None) -> None:
    _check(_native().dream_tree_expand_level(logits, logits_dtype, batch, n_frontier, vocab, cum_in, k, cand_token, cand_score,
                                             next_frontier, workspace, workspace, _stream(stream)))


def dream_tree_finalize(pool_score: torch.Tensor, pool_parent: torch.Tensor, pool_token: torch.Tensor, batch: int, n_pool: int,
                        budget: int, tree_parent: torch.Tensor, tree_token: torch.Tensor, tree_pool_index: torch.Tensor,
                        stream=None) -> int:
    n_tree = C.c_int32(0)
    _check(_native().dream_tree_finalize(pool_score, pool_parent, pool_token, batch, n_pool, budget, tree_parent, tree_token,
                                         tree_pool_index, n_tree, _stream(stream)))
    return int(n_tree.value)


def dream_tree_validate_host(parent_host: np.ndarray) -> int:
    """Host-side validation of one parent array; returns the maximum depth."""
    p = np.ascontiguousarray(parent_host, dtype=np.int32)
    depth = C.c_int32(0)
    _check(load().dream_tree_validate_host(p.ctypes.data_as(C.c_void_p), C.c_int32(p.shape[0]), C.byref(depth)))
    return int(depth.value)
