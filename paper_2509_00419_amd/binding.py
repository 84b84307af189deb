"""Binding of liblvlm.so: argument marshalling only.

Every step of the path runs in the library's HIP kernels; this module turns
torch tensors (used for device memory and streams) into the pointers, strides
and plain structs of include/lvlm.h and raises on any non-zero status.  The
calls of the path are native (csrc/torch_binding.cpp, built beside the
library); the descriptors and helper calls here go through ctypes.  There is
no fallback: if a shared library is missing the import fails.
"""
from __future__ import annotations

import ctypes as C
import importlib.util
import os
from typing import Optional

import torch

HERE = os.path.dirname(os.path.abspath(__file__))
# the in-tree build, or another build of the same sources named by LVLM_LIBRARY (e.g. one with a sanitized host side)
LIB_PATH = os.environ.get("LVLM_LIBRARY") or os.path.join(HERE, "liblvlm.so")
TORCH_BINDING_PATH = os.environ.get("LVLM_TORCH_BINDING")       # ... and of the extension module beside it

# ---- enums (include/lvlm.h) ----
BF16, F32, I32 = 0, 1, 2
OP_SCORE, OP_MERGE, OP_KV_COMPRESS, OP_DECODE_ATTN, OP_MERGE_SIMILAR, OP_SCORE_PROBS, OP_PREFILL_ATTN = 0, 1, 2, 3, 4, 5, 6
MERGE_LINEAR_RANK, MERGE_PAIRWISE, MERGE_LINEAR_RAW = 0, 1, 2
RULE_WEIGHTED, RULE_TOP = 0, 1
KV_THRESHOLD, KV_BUDGET = 0, 1
ORDER_STABLE, ORDER_FILL = 0, 1
KIND_PROTECTED, KIND_IMAGE, KIND_GENERATED = 0, 1, 2
MAX_PLANES = 8
STATUS = {0: "LVLM_OK", 1: "LVLM_ERR_INVALID_ARG", 2: "LVLM_ERR_UNSUPPORTED", 3: "LVLM_ERR_WORKSPACE",
          4: "LVLM_ERR_HIP"}

_DTYPE = {torch.bfloat16: BF16, torch.float32: F32, torch.int32: I32}


class ScoreDesc(C.Structure):
    _fields_ = [("dtype", C.c_int32), ("B", C.c_int32), ("N", C.c_int32), ("T", C.c_int32),
                ("q_pos0", C.c_int32), ("Hq", C.c_int32), ("Hkv", C.c_int32), ("hd", C.c_int32),
                ("img_begin", C.c_int32), ("n_img", C.c_int32), ("causal", C.c_int32), ("scale", C.c_float),
                ("q_stride_b", C.c_int64), ("q_stride_t", C.c_int64), ("q_stride_h", C.c_int64),
                ("k_stride_b", C.c_int64), ("k_stride_n", C.c_int64), ("k_stride_h", C.c_int64),
                ("sh_stride_b", C.c_int64), ("sh_stride_h", C.c_int64)]


class ProbsDesc(C.Structure):
    _fields_ = [("dtype", C.c_int32), ("B", C.c_int32), ("N", C.c_int32), ("T", C.c_int32),
                ("Hq", C.c_int32), ("Hkv", C.c_int32), ("img_begin", C.c_int32), ("n_img", C.c_int32),
                ("p_stride_b", C.c_int64), ("p_stride_h", C.c_int64), ("p_stride_t", C.c_int64),
                ("sh_stride_b", C.c_int64), ("sh_stride_h", C.c_int64)]


class PrefillDesc(C.Structure):
    _fields_ = [("dtype", C.c_int32), ("B", C.c_int32), ("N", C.c_int32), ("Hq", C.c_int32), ("Hkv", C.c_int32),
                ("hd", C.c_int32), ("causal", C.c_int32), ("scale", C.c_float), ("T", C.c_int32),
                ("img_begin", C.c_int32), ("n_img", C.c_int32),
                ("q_stride_b", C.c_int64), ("q_stride_n", C.c_int64), ("q_stride_h", C.c_int64),
                ("k_stride_b", C.c_int64), ("k_stride_n", C.c_int64), ("k_stride_h", C.c_int64),
                ("v_stride_b", C.c_int64), ("v_stride_n", C.c_int64), ("v_stride_h", C.c_int64),
                ("o_stride_b", C.c_int64), ("o_stride_n", C.c_int64), ("o_stride_h", C.c_int64),
                ("sh_stride_b", C.c_int64), ("sh_stride_h", C.c_int64)]


class Plane(C.Structure):
    _fields_ = [("src", C.c_void_p), ("dst", C.c_void_p), ("src_stride_b", C.c_int64),
                ("dst_stride_b", C.c_int64), ("row_elems", C.c_int32), ("dtype", C.c_int32),
                ("merge_rule", C.c_int32), ("reserved", C.c_int32)]


class MergeDesc(C.Structure):
    _fields_ = [("B", C.c_int32), ("N", C.c_int32), ("img_begin", C.c_int32), ("n_img", C.c_int32),
                ("n_keep", C.c_int32), ("n_planes", C.c_int32)]


class MergeQuery(C.Structure):
    _fields_ = [("desc", C.POINTER(MergeDesc)), ("planes", C.POINTER(Plane))]


class KvDesc(C.Structure):
    _fields_ = [("dtype", C.c_int32), ("B", C.c_int32), ("Hkv", C.c_int32), ("hd", C.c_int32),
                ("Lmax", C.c_int32), ("len_bound", C.c_int32), ("mode", C.c_int32), ("order", C.c_int32),
                ("budget", C.c_int32), ("n_recent", C.c_int32), ("beta", C.c_double)]


class AttnDesc(C.Structure):
    _fields_ = [("dtype", C.c_int32), ("B", C.c_int32), ("Hq", C.c_int32), ("Hkv", C.c_int32),
                ("hd", C.c_int32), ("Lmax", C.c_int32), ("len_bound", C.c_int32), ("new_kind", C.c_int32),
                ("new_pos", C.c_int32), ("scale", C.c_float), ("score_decay", C.c_float),
                ("evict_budget", C.c_int32), ("evict_recent", C.c_int32)]


class ProfileEntry(C.Structure):
    _fields_ = [("name", C.c_char * 48), ("calls", C.c_int32), ("total_ms", C.c_float), ("min_ms", C.c_float),
                ("max_ms", C.c_float)]


class LvlmError(RuntimeError):
    def __init__(self, status: int, message: str):
        super().__init__(f"{STATUS.get(status, status)}: {message}")
        self.status = status


def _load():
    if not os.path.exists(LIB_PATH):
        raise ImportError(f"{LIB_PATH} is missing: run `python -c 'import __graft_entry__ as g; g.build()'` "
                          "(the HIP library is the only implementation; there is no fallback)")
    lib = C.CDLL(LIB_PATH)
    vp, i32p, f32p = C.c_void_p, C.c_void_p, C.c_void_p
    lib.lvlm_create.argtypes = [C.POINTER(C.c_void_p), C.c_int]
    lib.lvlm_destroy.argtypes = [C.c_void_p]
    lib.lvlm_last_error.argtypes = [C.c_void_p]
    lib.lvlm_last_error.restype = C.c_char_p
    lib.lvlm_workspace_bytes.argtypes = [C.c_void_p, C.c_int, C.c_void_p, C.POINTER(C.c_size_t)]
    lib.lvlm_set_workspace.argtypes = [C.c_void_p, C.c_void_p, C.c_size_t]
    lib.lvlm_schedule.argtypes = [C.c_int, C.c_double, C.c_int, C.POINTER(C.c_int)]
    lib.lvlm_merge_weights.argtypes = [C.c_int, C.c_int, C.POINTER(C.c_float)]
    lib.lvlm_score_tokens.argtypes = [vp, vp, C.POINTER(ScoreDesc), vp, vp, f32p, f32p, f32p]
    lib.lvlm_score_plan.argtypes = [vp, C.POINTER(ScoreDesc), C.POINTER(C.c_int32)]
    lib.lvlm_score_few_rows.argtypes = [vp, C.POINTER(ScoreDesc), C.c_int, C.POINTER(C.c_int32)]
    lib.lvlm_score_shares.argtypes = lib.lvlm_score_few_rows.argtypes
    lib.lvlm_score_from_probs.argtypes = [vp, vp, C.POINTER(ProbsDesc), vp, f32p, f32p]
    lib.lvlm_prefill_attn.argtypes = [vp, vp, C.POINTER(PrefillDesc), vp, vp, vp, vp, f32p, f32p, f32p]
    lib.lvlm_merge_compact.argtypes = [vp, vp, C.POINTER(MergeDesc), f32p, f32p, C.POINTER(Plane), i32p, i32p]
    lib.lvlm_merge_similar.argtypes = [vp, vp, C.POINTER(MergeDesc), f32p, C.POINTER(Plane), f32p, f32p, i32p, i32p]
    lib.lvlm_kv_compress.argtypes = [vp, vp, C.POINTER(KvDesc), vp, vp, f32p, vp, i32p, i32p, i32p]
    lib.lvlm_decode_attn.argtypes = [vp, vp, C.POINTER(AttnDesc), vp, vp, vp, vp, vp, f32p, vp, i32p, i32p, vp]
    lib.lvlm_decode_attn_static.argtypes = lib.lvlm_decode_attn.argtypes
    lib.lvlm_decode_plan.argtypes = [vp, C.POINTER(AttnDesc), C.POINTER(C.c_int32), C.POINTER(C.c_int32), C.POINTER(C.c_int32)]
    lib.lvlm_stream_probe.argtypes = [vp, vp, vp, C.c_size_t, C.c_int32, vp]
    lib.lvlm_profile.argtypes = [C.c_void_p, C.c_int]
    lib.lvlm_profile_read.argtypes = [C.c_void_p, C.POINTER(ProfileEntry), C.c_int, C.POINTER(C.c_int)]
    for name in ("lvlm_profile", "lvlm_profile_read", "lvlm_create", "lvlm_destroy", "lvlm_workspace_bytes", "lvlm_set_workspace", "lvlm_schedule",
                 "lvlm_merge_weights", "lvlm_score_tokens", "lvlm_score_plan", "lvlm_score_few_rows", "lvlm_score_shares", "lvlm_score_from_probs", "lvlm_prefill_attn", "lvlm_merge_compact",
                 "lvlm_merge_similar",
                 "lvlm_kv_compress",
                 "lvlm_decode_attn", "lvlm_decode_attn_static", "lvlm_decode_plan", "lvlm_stream_probe"):
        getattr(lib, name).restype = C.c_int
    return lib


lib = _load()


def _load_calls():
    try:
        if TORCH_BINDING_PATH:
            spec = importlib.util.spec_from_file_location(__package__ + "._torch_binding", TORCH_BINDING_PATH)
            _torch_binding = importlib.util.module_from_spec(spec)
            spec.loader.exec_module(_torch_binding)
        else:
            from . import _torch_binding
    except ImportError as e:
        raise ImportError("the native side of the binding is missing or does not fit this torch: run "
                          f"`python -c 'import __graft_entry__ as g; g.build()'` ({e})") from e
    address = lambda name: C.cast(getattr(lib, name), C.c_void_p).value          # noqa: E731
    _torch_binding.setup(LvlmError, *(address("lvlm_" + n) for n in (
        "last_error", "workspace_bytes", "set_workspace", "score_tokens", "score_from_probs", "prefill_attn", "merge_compact",
        "merge_similar", "kv_compress", "decode_attn", "decode_attn_static")))
    return _torch_binding.ContextCalls


_ContextCalls = _load_calls()


def _ptr(t: Optional[torch.Tensor]):
    return None if t is None else C.c_void_p(t.data_ptr())


def _stream() -> C.c_void_p:
    return C.c_void_p(torch.cuda.current_stream().cuda_stream)


def schedule(n_img: int, final_keep: float, n_stages: int = 3):
    out = (C.c_int * n_stages)()
    st = lib.lvlm_schedule(n_img, float(final_keep), n_stages, out)
    if st:
        raise LvlmError(st, "lvlm_schedule")
    return list(out)


def merge_weights(mode: int, m: int) -> torch.Tensor:
    out = (C.c_float * m)()
    st = lib.lvlm_merge_weights(mode, m, out)
    if st:
        raise LvlmError(st, "lvlm_merge_weights")
    return torch.tensor(list(out), dtype=torch.float32)


class Context(_ContextCalls):
    """One lvlm_ctx plus a grow-only workspace tensor (device memory via torch)."""

    def __init__(self, device: int = 0):
        self._h = C.c_void_p()
        st = lib.lvlm_create(C.byref(self._h), device)
        if st:
            raise LvlmError(st, "lvlm_create")
        self.device = device
        self._attach(self._h.value, device)

    def close(self):
        if self._h:
            self._attach(0, self.device)
            lib.lvlm_destroy(self._h)
            self._h = C.c_void_p()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _check(self, st: int):
        if st:
            raise LvlmError(st, lib.lvlm_last_error(self._h).decode())

    def workspace_bytes(self, op: int, desc) -> int:
        n = C.c_size_t()
        self._check(lib.lvlm_workspace_bytes(self._h, op, C.byref(desc), C.byref(n)))
        return n.value

    def set_workspace(self, ws: Optional[torch.Tensor]):
        self._ws = ws
        self._check(lib.lvlm_set_workspace(self._h, _ptr(ws), 0 if ws is None else ws.numel()))

    def stream_probe(self, src: torch.Tensor, n_workgroups: int, sink: torch.Tensor):
        """lvlm_stream_probe: a read-only pass over src (diagnostic)."""
        self._check(lib.lvlm_stream_probe(self._h, _stream(), _ptr(src), src.numel() * src.element_size(), n_workgroups,
                                          _ptr(sink)))

    def profile(self, enable: bool):
        """lvlm_profile: bracket every kernel launch with HIP events (eager mode only)."""
        self._check(lib.lvlm_profile(self._h, int(enable)))

    def profile_read(self):
        """lvlm_profile_read -> {kernel name: (calls, total_ms, min_ms, max_ms)}; clears the record."""
        arr = (ProfileEntry * 64)()
        n = C.c_int()
        self._check(lib.lvlm_profile_read(self._h, arr, 64, C.byref(n)))
        return {arr[i].name.decode(): (arr[i].calls, arr[i].total_ms, arr[i].min_ms, arr[i].max_ms)
                for i in range(n.value)}

    # score_tokens, score_from_probs, prefill_attn, merge_compact, merge_similar, kv_compress and decode_attn are
    # native (csrc/torch_binding.cpp), with the argument names and defaults that help(Context) shows.

    # ---- step 1 ----
    def score_desc(self, q, k, *, q_pos0, img_begin, n_img, scale=None, causal=True, score_head=None) -> ScoreDesc:
        B, T, Hq, hd = q.shape
        _, N, Hkv, _ = k.shape
        assert q.stride(3) == 1 and k.stride(3) == 1, "head dimension must be contiguous"
        return ScoreDesc(_DTYPE[q.dtype], B, N, T, q_pos0, Hq, Hkv, hd, img_begin, n_img, int(causal),
                         float(hd ** -0.5 if scale is None else scale),
                         q.stride(0), q.stride(1), q.stride(2), k.stride(0), k.stride(1), k.stride(2),
                         0 if score_head is None else score_head.stride(0),
                         0 if score_head is None else score_head.stride(1))

    def score_plan(self, desc: ScoreDesc) -> int:
        """lvlm_score_plan: 0 = two-pass kernels, 1 = one launch (a chunk per workgroup), 2 = one launch (shared tiles),
        3 = the shared-tile kernel with the keys cut into runs (one launch per sweep)."""
        form = C.c_int32()
        self._check(lib.lvlm_score_plan(self._h, C.byref(desc), C.byref(form)))
        return form.value

    def score_few_rows(self, desc: ScoreDesc, lse_given: bool = False) -> int:
        """lvlm_score_few_rows: chunks of 16 query rows per KV head where the kernel for few query rows takes the place of
        form 0 or 1 (every key read and multiplied once, one launch), else 0."""
        chunks = C.c_int32()
        self._check(lib.lvlm_score_few_rows(self._h, C.byref(desc), int(lse_given), C.byref(chunks)))
        return chunks.value

    def score_shares(self, desc: ScoreDesc, lse_given: bool = False) -> int:
        """lvlm_score_shares: shares the keys are dealt out in where the kernel for much work takes the place of form 0, 2 or 3
        (a launch per sweep), else 0."""
        shares = C.c_int32()
        self._check(lib.lvlm_score_shares(self._h, C.byref(desc), int(lse_given), C.byref(shares)))
        return shares.value

    # ---- step 6 ----
    def decode_plan(self, desc: AttnDesc):
        """lvlm_decode_plan: (n_split, split_len, form); form 0 = one tile per wave, 1 = some wave has a second tile,
        2 = whole 128-entry splits plus one entry taken by one wave."""
        n, sl, form = C.c_int32(), C.c_int32(), C.c_int32()
        self._check(lib.lvlm_decode_plan(self._h, C.byref(desc), C.byref(n), C.byref(sl), C.byref(form)))
        return n.value, sl.value, form.value
