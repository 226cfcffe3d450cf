"""Thin binding of libppv_hip.so: argument marshalling only, through ctypes for the calls that are made once per
constraint set and through the native extension _ppv_call for those that are made at every step (ctypes and tensor
attributes read from Python took 10 to 12 us per call, longer than the GPU needs for a small batch).

Same names as the C ABI in include/ppv.h.  Tensors are torch tensors on the GPU (torch provides
device memory and the current stream, nothing else); every step of the path runs in the library's
own kernels.  There is no fallback: if the library is missing or a call fails, this raises.
"""
from __future__ import annotations

import ctypes as C
import os
from typing import Optional, Tuple

import numpy as np
import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libppv_hip.so")
CALL_PATH = os.path.join(_PKG, "_ppv_call.so")

PPV_OK = 0
PPV_F32, PPV_BF16 = 0, 1
PPV_MAX_VOCAB = 262144
PPV_TOPM_MAX = 1024

PPV_STATE_WORDS = 8

SYMBOLS = ("ppv_status_string", "ppv_build_index", "ppv_index_info", "ppv_index_export", "ppv_free_index",
           "ppv_index_save", "ppv_index_load",
           "ppv_next_token_mask", "constrained_sample", "ppv_decode_begin", "ppv_decode_step", "ppv_decode_loop", "ppv_topm_mask",
           "ppv_disc_select", "ppv_tuning_set", "ppv_tuning_get", "constrained_sample_noalloc",
           "ppv_sample_next", "ppv_decode_begin_empty", "ppv_decode_first_step")
PPV_NOALLOC_MAX_ROWS = 512

# tuning / test switches (ppv_tuning_set)
(PPV_TUNE_WAVES_PER_ROW, PPV_TUNE_TOPM_WAVES, PPV_TUNE_TOPM_STREAMING, PPV_TUNE_LOOKUP, PPV_TUNE_LOOKUP_WEAK,
 PPV_TUNE_ROW_SPLIT) = range(6)

_lib = None
_call = None     # the native extension, bound to the library's entry points when the library is loaded


class PPVError(RuntimeError):
    def __init__(self, status: int, what: str):
        self.status = status
        super().__init__(f"{what}: status {status} ({status_string(status)})")


def load_library() -> C.CDLL:
    """Load libppv_hip.so (built by paper_2504_09135_amd.build); raises if it is not there."""
    global _lib, _call
    if _lib is not None:
        return _lib
    for path in (LIB_PATH, CALL_PATH):
        if not os.path.exists(path):
            raise FileNotFoundError(f"{path} is missing: run `python -m paper_2504_09135_amd.build` "
                                    "(or __graft_entry__.build()) first; there is no fallback path")
    lib = C.CDLL(LIB_PATH)
    p, i32, i64 = C.c_void_p, C.c_int32, C.c_int64
    lib.ppv_status_string.restype = C.c_char_p
    lib.ppv_status_string.argtypes = [C.c_int]
    lib.ppv_build_index.restype = C.c_int
    lib.ppv_build_index.argtypes = [p, p, i64, i32, C.POINTER(p)]
    lib.ppv_index_info.restype = C.c_int
    lib.ppv_index_info.argtypes = [p, C.POINTER(i64), C.POINTER(i32), C.POINTER(i32), C.POINTER(i64), C.POINTER(i64)]
    lib.ppv_index_export.restype = C.c_int
    lib.ppv_index_export.argtypes = [p, p, p, C.POINTER(i64)]
    lib.ppv_index_save.restype = C.c_int
    lib.ppv_index_save.argtypes = [p, C.c_char_p]
    lib.ppv_index_load.restype = C.c_int
    lib.ppv_index_load.argtypes = [C.c_char_p, C.POINTER(p)]
    lib.ppv_free_index.restype = None
    lib.ppv_free_index.argtypes = [p]
    lib.ppv_next_token_mask.restype = C.c_int
    lib.ppv_next_token_mask.argtypes = [p, p, i32, p, i32, p, p, p, p, p]
    lib.constrained_sample.restype = C.c_int
    lib.constrained_sample.argtypes = [p, C.c_int, i64, p, p, i32, i32, p, p, p, C.c_float, p]
    lib.constrained_sample_noalloc.restype = C.c_int
    lib.constrained_sample_noalloc.argtypes = lib.constrained_sample.argtypes
    lib.ppv_sample_next.restype = C.c_int
    lib.ppv_sample_next.argtypes = [p, p, i32, p, i32, p, C.c_int, i64, p, p, p, C.c_float, p]
    lib.ppv_decode_begin.restype = C.c_int
    lib.ppv_decode_begin.argtypes = [p, p, i32, p, i32, p, p, p, p]
    lib.ppv_decode_begin_empty.restype = C.c_int
    lib.ppv_decode_begin_empty.argtypes = [p, i32, p, p, p, p, p]
    lib.ppv_decode_step.restype = C.c_int
    lib.ppv_decode_step.argtypes = [p, p, i32, p, p, p, p, C.c_int, i64, p, i32, p, p, p, C.c_float, p]
    lib.ppv_decode_first_step.restype = C.c_int
    lib.ppv_decode_first_step.argtypes = [p, p, i32, p, p, p, p, C.c_int, i64, p, i32, p, p, p, C.c_float, p]
    lib.ppv_decode_loop.restype = C.c_int
    lib.ppv_decode_loop.argtypes = [p, p, i32, p, p, p, p, C.c_int, i64, i64, p, i32, i32, p, p, p, C.c_float, p]
    lib.ppv_topm_mask.restype = C.c_int
    lib.ppv_topm_mask.argtypes = [p, p, i32, p, p, C.c_int, i64, i32, i32, p, p, p, p]
    lib.ppv_disc_select.restype = C.c_int
    lib.ppv_disc_select.argtypes = [p, i32, i32, i32, p, p, i32, p, p, p, p]
    lib.ppv_tuning_set.restype = C.c_int
    lib.ppv_tuning_set.argtypes = [i32, i32]
    lib.ppv_tuning_get.restype = C.c_int
    lib.ppv_tuning_get.argtypes = [i32, C.POINTER(i32)]
    from . import _ppv_call
    _ppv_call.bind({name: C.cast(getattr(lib, name), p).value for name in SYMBOLS})
    _call = _ppv_call
    _lib = lib
    return lib


def _native():
    """The native extension, with the library loaded."""
    load_library()
    return _call


def status_string(status: int) -> str:
    return load_library().ppv_status_string(int(status)).decode()


def _check(status: int, what: str):
    if status != PPV_OK:
        raise PPVError(status, what)


class PPVIndex:
    """Owner of a ppv_index_t handle."""

    def __init__(self, handle: int):
        self._h = C.c_void_p(handle)
        self._address = handle      # what the native calls read; None once the index is freed
        self.n_distinct, self.l_max, self.vocab, self.n_prefixes, self.device_bytes = ppv_index_info(self)
        self.n_words = (self.vocab + 31) // 32

    @property
    def handle(self) -> C.c_void_p:
        if not self._h:
            raise ValueError("index already freed")
        return self._h

    def free(self):
        if self._h:
            self._address = None
            load_library().ppv_free_index(self._h)
            self._h = None

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


def ppv_build_index(tokens: np.ndarray, offsets: np.ndarray, vocab: int) -> PPVIndex:
    """S as host CSR arrays (int32 tokens, int64 offsets) -> device index."""
    lib = load_library()
    tokens = np.ascontiguousarray(tokens, dtype=np.int32)
    offsets = np.ascontiguousarray(offsets, dtype=np.int64)
    out = C.c_void_p()
    st = lib.ppv_build_index(tokens.ctypes.data_as(C.c_void_p), offsets.ctypes.data_as(C.c_void_p),
                             int(offsets.shape[0]) - 1, int(vocab), C.byref(out))
    _check(st, "ppv_build_index")
    return PPVIndex(out.value)


def ppv_index_save(index: PPVIndex, path: str) -> None:
    """Write the index to a file (ppv_index_load reads it back)."""
    _check(load_library().ppv_index_save(index.handle, os.fsencode(path)), "ppv_index_save")


def ppv_index_load(path: str) -> PPVIndex:
    """Read an index written by ppv_index_save onto the current device."""
    out = C.c_void_p()
    _check(load_library().ppv_index_load(os.fsencode(path), C.byref(out)), "ppv_index_load")
    return PPVIndex(out.value)


def ppv_index_info(index: PPVIndex) -> Tuple[int, int, int, int, int]:
    n, l, v, g, by = C.c_int64(), C.c_int32(), C.c_int32(), C.c_int64(), C.c_int64()
    _check(load_library().ppv_index_info(index.handle, C.byref(n), C.byref(l), C.byref(v), C.byref(g), C.byref(by)),
           "ppv_index_info")
    return n.value, l.value, v.value, g.value, by.value


def ppv_index_export(index: PPVIndex) -> Tuple[np.ndarray, np.ndarray]:
    """Sorted, de-duplicated S as host CSR arrays."""
    lib = load_library()
    nt = C.c_int64()
    _check(lib.ppv_index_export(index.handle, None, None, C.byref(nt)), "ppv_index_export")
    tokens = np.empty(nt.value, dtype=np.int32)
    offsets = np.empty(index.n_distinct + 1, dtype=np.int64)
    _check(lib.ppv_index_export(index.handle, tokens.ctypes.data_as(C.c_void_p),
                                offsets.ctypes.data_as(C.c_void_p), None), "ppv_index_export")
    return tokens, offsets


def ppv_free_index(index: PPVIndex) -> None:
    index.free()


def ppv_next_token_mask(index: PPVIndex, prefixes: torch.Tensor, lens: torch.Tensor, mask: torch.Tensor,
                        range_lo: Optional[torch.Tensor] = None, range_hi: Optional[torch.Tensor] = None,
                        member: Optional[torch.Tensor] = None, stream=None) -> None:
    """prefixes int32 [B, stride], lens int32 [B] -> mask int32 [B, ceil(V/32)] (bit pattern of
    uint32 words), range_lo/range_hi int32 [B] (bit pattern of uint32), member uint8 [B]."""
    st = (_call or _native()).next_token_mask(index, prefixes, lens, mask, range_lo, range_hi, member, stream)
    if st:
        _check(st, "ppv_next_token_mask")


def constrained_sample(logits: torch.Tensor, mask: torch.Tensor, uniforms: torch.Tensor, ids: torch.Tensor,
                       logZ_valid: torch.Tensor, logZ_all: Optional[torch.Tensor] = None, stream=None,
                       temperature: float = 1.0, _noalloc: bool = False) -> None:
    """logits [B, V] f32/bf16, mask int32 [B, ceil(V/32)], uniforms f32 [B] -> ids int32 [B],
    logZ_valid f32 [B], logZ_all f32 [B] (optional); P = softmax(logits / temperature)."""
    st = (_call or _native()).sample(logits, mask, uniforms, ids, logZ_valid, logZ_all, stream, temperature, _noalloc)
    if st:
        _check(st, "constrained_sample_noalloc" if _noalloc else "constrained_sample")


def constrained_sample_noalloc(logits: torch.Tensor, mask: torch.Tensor, uniforms: torch.Tensor, ids: torch.Tensor,
                               logZ_valid: torch.Tensor, logZ_all: Optional[torch.Tensor] = None, stream=None,
                               temperature: float = 1.0) -> None:
    """constrained_sample through the entry point that allocates nothing (at most PPV_NOALLOC_MAX_ROWS rows)."""
    constrained_sample(logits, mask, uniforms, ids, logZ_valid, logZ_all, stream, temperature, _noalloc=True)


def ppv_decode_begin(index: PPVIndex, prefixes: torch.Tensor, lens: torch.Tensor, state: torch.Tensor,
                     active: torch.Tensor, logx: Optional[torch.Tensor] = None, stream=None) -> None:
    """Locate every row's current prefix once: writes state int32 [B, PPV_STATE_WORDS], active uint8 [B]
    and zeroes logx f32 [B]."""
    st = (_call or _native()).decode_begin(index, prefixes, lens, state, active, logx, stream)
    if st:
        _check(st, "ppv_decode_begin")


def ppv_decode_begin_empty(index: PPVIndex, lens: torch.Tensor, state: torch.Tensor, active: torch.Tensor,
                           logx: Optional[torch.Tensor] = None, stream=None) -> None:
    """SampleCandidate initialisation from the empty candidate for every row: lens int32 [B] (written 0),
    state int32 [B, PPV_STATE_WORDS], active uint8 [B], logx f32 [B] (optional) are written."""
    st = (_call or _native()).decode_begin_empty(index, lens, state, active, logx, stream)
    if st:
        _check(st, "ppv_decode_begin_empty")


def ppv_decode_step(index: PPVIndex, prefixes: torch.Tensor, lens: torch.Tensor, active: torch.Tensor,
                    logits: torch.Tensor, uniforms: torch.Tensor, ids: Optional[torch.Tensor] = None,
                    logZ_valid: Optional[torch.Tensor] = None, logx: Optional[torch.Tensor] = None,
                    state: Optional[torch.Tensor] = None, stream=None, temperature: float = 1.0,
                    _first: bool = False) -> None:
    """One fused constrained decoding step, in place on prefixes / lens / active / logx (and on
    state int32 [B, PPV_STATE_WORDS] from ppv_decode_begin when given); P = softmax(logits / temperature)."""
    st = (_call or _native()).decode_step(index, prefixes, lens, active, logits, uniforms, ids, logZ_valid, logx, state,
                                          stream, temperature, _first)
    if st:
        _check(st, "ppv_decode_first_step" if _first else "ppv_decode_step")


def ppv_decode_first_step(index: PPVIndex, prefixes: torch.Tensor, lens: torch.Tensor, active: torch.Tensor,
                          logits: torch.Tensor, uniforms: torch.Tensor, ids: Optional[torch.Tensor] = None,
                          logZ_valid: Optional[torch.Tensor] = None, logx: Optional[torch.Tensor] = None,
                          state: Optional[torch.Tensor] = None, stream=None, temperature: float = 1.0) -> None:
    """ppv_decode_begin_empty and the first ppv_decode_step in one launch (state is required)."""
    st = (_call or _native()).decode_step(index, prefixes, lens, active, logits, uniforms, ids, logZ_valid, logx, state,
                                          stream, temperature, True)
    if st:
        _check(st, "ppv_decode_first_step")


def ppv_decode_loop(index: PPVIndex, prefixes: torch.Tensor, lens: torch.Tensor, active: torch.Tensor,
                    logits: torch.Tensor, uniforms: torch.Tensor, ids: Optional[torch.Tensor] = None,
                    logZ_valid: Optional[torch.Tensor] = None, logx: Optional[torch.Tensor] = None,
                    state: Optional[torch.Tensor] = None, stream=None, temperature: float = 1.0) -> None:
    """The whole decode loop in one launch: logits [n_steps, B, V] (f32/bf16), uniforms f32 [n_steps, B],
    ids int32 / logZ_valid f32 [n_steps, B] (optional); everything else as ppv_decode_step."""
    st = (_call or _native()).decode_loop(index, prefixes, lens, active, logits, uniforms, ids, logZ_valid, logx, state,
                                          stream, temperature)
    if st:
        _check(st, "ppv_decode_loop")


def ppv_topm_mask(index: PPVIndex, prefixes: torch.Tensor, lens: torch.Tensor, logits: torch.Tensor, M: int,
                  mask: torch.Tensor, top_ids: Optional[torch.Tensor] = None, mask_V: Optional[torch.Tensor] = None,
                  stream=None) -> None:
    """Algorithm 2 with M candidates: prefixes int32 [B, stride], lens int32 [B], logits [B, V] f32/bf16 ->
    mask int32 [B, ceil(V/32)], top_ids int32 [B, M] (optional), mask_V uint8 [B, M] (optional)."""
    st = (_call or _native()).topm_mask(index, prefixes, lens, logits, M, mask, top_ids, mask_V, stream)
    if st:
        _check(st, "ppv_topm_mask")


def ppv_disc_select(logx: torch.Tensor, K: int, accept_u: torch.Tensor, resample_u: torch.Tensor,
                    chosen: torch.Tensor, n_draws: Optional[torch.Tensor] = None,
                    accepted: Optional[torch.Tensor] = None, reuse_rejected: bool = False, stream=None) -> None:
    """DISC accept/reject rounds + importance-resampling fallback: logx f32 [n_candidates, Q], accept_u f32 [K, Q],
    resample_u f32 [Q] -> chosen int32 [Q], n_draws int32 [Q], accepted uint8 [Q]."""
    st = (_call or _native()).disc_select(logx, K, accept_u, resample_u, chosen, n_draws, accepted, reuse_rejected,
                                          stream)
    if st:
        _check(st, "ppv_disc_select")


def ppv_tuning_set(knob: int, value: int) -> None:
    """Set a process-wide tuning / test switch (PPV_TUNE_*)."""
    _check(load_library().ppv_tuning_set(int(knob), int(value)), "ppv_tuning_set")


def ppv_tuning_get(knob: int) -> int:
    v = C.c_int32()
    _check(load_library().ppv_tuning_get(int(knob), C.byref(v)), "ppv_tuning_get")
    return v.value


def ppv_sample_next(index: PPVIndex, prefixes: torch.Tensor, lens: torch.Tensor, logits: torch.Tensor,
                    uniforms: torch.Tensor, ids: torch.Tensor, logZ_valid: Optional[torch.Tensor] = None, stream=None,
                    temperature: float = 1.0) -> None:
    """Mask + sample fused, nothing of the caller's rows changed: prefixes int32 [B, stride], lens int32 [B],
    logits [B, V] f32/bf16, uniforms f32 [B] -> ids int32 [B], logZ_valid f32 [B] (optional)."""
    st = (_call or _native()).sample_next(index, prefixes, lens, logits, uniforms, ids, logZ_valid, stream, temperature)
    if st:
        _check(st, "ppv_sample_next")
