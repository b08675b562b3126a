"""ctypes binding of ``include/moe_hub.h``: same names, argument marshalling only."""
from __future__ import annotations

import ctypes
import os

try:
    import torch
except ImportError:  # the library's path, its symbols and last_error() need no torch
    torch = None

HERE = os.path.dirname(os.path.abspath(__file__))
# MOE_HUB_LIBRARY selects another build of the same library (A/B timing of two builds)
_LIB_PATH = os.environ.get("MOE_HUB_LIBRARY") or os.path.join(HERE, "libmoe_hub.so")

BF16, F32 = 0, 1
SCORE_SOFTMAX_TOPK, SCORE_SIGMOID_TOPK = 0, 1
OP_ROUTE, OP_DISPATCH_LAYOUT, OP_GROUPED_FFN = 0, 1, 2

_ERR_NAMES = {-1: "MOE_ERR_ARG", -2: "MOE_ERR_UNSUPPORTED", -3: "MOE_ERR_WORKSPACE", -4: "MOE_ERR_LAUNCH",
              -5: "MOE_ERR_STATE"}

_c_i64, _c_int, _c_vp, _c_sz = ctypes.c_int64, ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t

# name -> (restype, argtypes), exactly the declarations of include/moe_hub.h
_SIGNATURES = {
    "moe_last_error": (ctypes.c_char_p, []),
    "moe_workspace_bytes": (_c_sz, [_c_int, _c_i64, _c_i64, _c_int, _c_int, _c_int, _c_i64, _c_int]),
    "moe_route": (_c_int, [_c_vp, _c_int, _c_i64, _c_i64, _c_vp, _c_vp, _c_int, _c_int, _c_int,
                           _c_vp, _c_vp, _c_vp, _c_vp, _c_sz, _c_vp]),
    "moe_dispatch_layout": (_c_int, [_c_vp, _c_i64, _c_int, _c_int, _c_int, _c_vp, _c_vp, _c_vp, _c_vp,
                                     _c_vp, _c_vp, _c_vp, _c_sz, _c_vp]),
    "moe_dispatch_layout_static": (_c_int, [_c_vp, _c_i64, _c_int, _c_int, _c_int, _c_vp, _c_vp, _c_vp,
                                            _c_vp, _c_vp, _c_vp, _c_vp]),
    "moe_dispatch_layout_arrival": (_c_int, [_c_vp, _c_i64, _c_int, _c_int, _c_int, _c_vp, _c_vp, _c_vp,
                                             _c_vp, _c_vp, _c_vp, _c_vp]),
    "moe_route_resolve_arrival": (_c_int, [_c_vp, _c_int, _c_i64, _c_i64, _c_vp, _c_vp, _c_int, _c_int, _c_int,
                                           _c_int, _c_vp, _c_vp, _c_vp, _c_vp, _c_vp, _c_vp, _c_vp, _c_vp, _c_vp,
                                           _c_vp, _c_sz, _c_vp]),
    "moe_permute": (_c_int, [_c_vp, _c_int, _c_i64, _c_i64, _c_int, _c_vp, _c_vp, _c_vp, _c_vp]),
    "moe_grouped_ffn": (_c_int, [_c_vp, _c_int, _c_i64, _c_i64, _c_i64, _c_int, _c_vp, _c_vp, _c_vp,
                                 _c_vp, _c_vp, _c_vp, _c_sz, _c_vp]),
    "moe_ffn_schedule": (_c_int, [_c_int, _c_i64, _c_i64, _c_i64, _c_int, _c_vp, _c_vp, _c_sz, _c_vp]),
    "moe_ffn_gate_up_down": (_c_int, [_c_vp, _c_int, _c_i64, _c_i64, _c_i64, _c_int, _c_vp, _c_vp, _c_vp,
                                      _c_vp, _c_vp, _c_vp, _c_sz, _c_i64, _c_vp]),
    "moe_ffn_status": (_c_int, [_c_int, _c_i64, _c_i64, _c_i64, _c_int, _c_vp, _c_sz, _c_vp]),
    "moe_ffn_gate_up": (_c_int, [_c_vp, _c_int, _c_i64, _c_i64, _c_i64, _c_int, _c_vp, _c_vp, _c_vp,
                                 _c_vp, _c_sz, _c_vp]),
    "moe_ffn_gate_up_gather": (_c_int, [_c_vp, _c_int, _c_i64, _c_int, _c_i64, _c_i64, _c_int, _c_vp, _c_vp,
                                        _c_vp, _c_vp, _c_vp, _c_sz, _c_vp]),
    "moe_ffn_down_combine": (_c_int, [_c_int, _c_i64, _c_int, _c_i64, _c_i64, _c_int, _c_vp, _c_vp, _c_vp, _c_vp,
                                      _c_vp, _c_vp, _c_vp, _c_sz, _c_vp]),
    "moe_ffn_down": (_c_int, [_c_int, _c_i64, _c_i64, _c_i64, _c_int, _c_vp, _c_vp, _c_vp, _c_vp, _c_sz, _c_vp]),
    "moe_combine": (_c_int, [_c_vp, _c_int, _c_i64, _c_i64, _c_int, _c_vp, _c_vp, _c_vp, _c_vp]),
}

_lib = None


class MoEHubError(RuntimeError):
    def __init__(self, code: int, message: str):
        super().__init__(f"{_ERR_NAMES.get(code, code)}: {message}")
        self.code = code


def lib_path() -> str:
    return _LIB_PATH


def exported_symbols():
    return sorted(_SIGNATURES)


def load_library(build_if_missing: bool = True):
    """Loads libmoe_hub.so (building it with hipcc when it does not exist yet)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        if not build_if_missing:
            raise FileNotFoundError(f"{_LIB_PATH} is not built; run python -m paper_2605_05888_amd.build")
        from . import build as _build
        _build.build(verbose=False)
    lib = ctypes.CDLL(_LIB_PATH)
    for name, (res, args) in _SIGNATURES.items():
        fn = getattr(lib, name)          # AttributeError if a declared symbol is missing
        fn.restype, fn.argtypes = res, args
    _lib = lib
    return lib


def last_error() -> str:
    return load_library().moe_last_error().decode()


def _check(rc: int):
    if rc != 0:
        raise MoEHubError(rc, last_error())


def _ptr(t):
    return None if t is None else t.data_ptr()


def _stream():
    # the handle itself where this torch hands it out (the name is private to it); torch.cuda.current_stream() builds a
    # Stream object around it at every call
    try:
        raw = torch._C._cuda_getCurrentRawStream
    except AttributeError:
        return torch.cuda.current_stream().cuda_stream
    return raw(torch.cuda.current_device())


def _dtype_code(t) -> int:
    if t.dtype == torch.bfloat16:
        return BF16
    if t.dtype == torch.float32:
        return F32
    raise TypeError(f"unsupported activation dtype {t.dtype}")


def _need(t, dtype, name):
    if not t.is_cuda or not t.is_contiguous() or t.dtype != dtype:
        raise TypeError(f"{name} must be a contiguous device tensor of {dtype}")


def _need_layout(E, G, R, *arrays):
    # One pass without a call per array where all is well: a layer of one token is bound by the host.  With torch imported once
    # and pointers taken without a call, 256 fp32 rows (five calls) take 32.2 us instead of 33.4, 13.2 -> 12.0 of them here.
    i32 = torch.int32
    sizes = (E, E + 1, G, G + 1, R, R)
    for t, n in zip(arrays, sizes):
        if t.dtype != i32 or not t.is_cuda or not t.is_contiguous() or t.numel() != n:
            break
    else:
        return
    names = ("expert_counts", "expert_offsets", "dest_counts", "dest_offsets", "slot_of_row", "row_of_slot")
    for name, t, n in zip(names, arrays, sizes):
        _need(t, i32, name)
        assert t.numel() == n, name


def workspace_bytes(op: int, N: int = 0, H: int = 0, E: int = 0, K: int = 0, G: int = 1, F: int = 0,
                    dtype: int = BF16) -> int:
    return int(load_library().moe_workspace_bytes(op, N, H, E, K, G, F, dtype))


def _ws_args(ws):
    if ws is None:
        return None, 0
    return ws.data_ptr(), ws.numel() * ws.element_size()


def moe_route(x, W_r, bias, K: int, score_mode: int, topk_idx, topk_w, logits=None, ws=None):
    N, H = x.shape
    E = W_r.shape[1]
    _need(W_r, torch.float32, "W_r")
    _need(topk_idx, torch.int32, "topk_idx")
    _need(topk_w, torch.float32, "topk_w")
    assert W_r.shape[0] == H and x.is_contiguous()
    assert topk_idx.numel() == N * K and topk_w.numel() == N * K
    assert logits is None or (logits.numel() == N * E and logits.dtype == torch.float32)
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_route(x.data_ptr(), _dtype_code(x), N, H, W_r.data_ptr(), _ptr(bias), E, K, score_mode,
                         topk_idx.data_ptr(), topk_w.data_ptr(), _ptr(logits), wp, wb, _stream()))


def moe_dispatch_layout(topk_idx, E: int, G: int, expert_counts, expert_offsets, dest_counts, dest_offsets,
                        slot_of_row, row_of_slot, ws):
    N, K = topk_idx.shape
    _need_layout(E, G, N * K, expert_counts, expert_offsets, dest_counts, dest_offsets, slot_of_row, row_of_slot)
    _need(topk_idx, torch.int32, "topk_idx")
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_dispatch_layout(topk_idx.data_ptr(), N, K, E, G, expert_counts.data_ptr(),
                                   expert_offsets.data_ptr(), dest_counts.data_ptr(), dest_offsets.data_ptr(),
                                   slot_of_row.data_ptr(), row_of_slot.data_ptr(), wp, wb, _stream()))


def moe_dispatch_layout_static(topk_idx, E: int, G: int, expert_counts, expert_offsets, dest_counts,
                               dest_offsets, slot_of_row, row_of_slot):
    N, K = topk_idx.shape
    _need_layout(E, G, N * K, expert_counts, expert_offsets, dest_counts, dest_offsets, slot_of_row, row_of_slot)
    _need(topk_idx, torch.int32, "topk_idx")
    lib = _lib or load_library()
    _check(lib.moe_dispatch_layout_static(topk_idx.data_ptr(), N, K, E, G, expert_counts.data_ptr(),
                                          expert_offsets.data_ptr(), dest_counts.data_ptr(), dest_offsets.data_ptr(),
                                          slot_of_row.data_ptr(), row_of_slot.data_ptr(), _stream()))


def moe_dispatch_layout_arrival(topk_idx, E: int, G: int, expert_counts, expert_offsets, dest_counts,
                                dest_offsets, slot_of_row, row_of_slot):
    N, K = topk_idx.shape
    _need_layout(E, G, N * K, expert_counts, expert_offsets, dest_counts, dest_offsets, slot_of_row, row_of_slot)
    _need(topk_idx, torch.int32, "topk_idx")
    lib = _lib or load_library()
    _check(lib.moe_dispatch_layout_arrival(topk_idx.data_ptr(), N, K, E, G, expert_counts.data_ptr(),
                                           expert_offsets.data_ptr(), dest_counts.data_ptr(), dest_offsets.data_ptr(),
                                           slot_of_row.data_ptr(), row_of_slot.data_ptr(), _stream()))


def moe_route_resolve_arrival(x, W_r, bias, K: int, G: int, score_mode: int, topk_idx, topk_w, expert_counts,
                              expert_offsets, dest_counts, dest_offsets, slot_of_row, row_of_slot, logits=None,
                              ws=None):
    N, H = x.shape
    E = W_r.shape[1]
    _need(W_r, torch.float32, "W_r")
    _need(topk_idx, torch.int32, "topk_idx")
    _need(topk_w, torch.float32, "topk_w")
    assert W_r.shape[0] == H and x.is_contiguous()
    assert topk_idx.numel() == N * K and topk_w.numel() == N * K
    assert logits is None or (logits.numel() == N * E and logits.dtype == torch.float32)
    _need_layout(E, G, N * K, expert_counts, expert_offsets, dest_counts, dest_offsets, slot_of_row, row_of_slot)
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_route_resolve_arrival(x.data_ptr(), _dtype_code(x), N, H, W_r.data_ptr(), _ptr(bias), E, K, G,
                                         score_mode, topk_idx.data_ptr(), topk_w.data_ptr(), _ptr(logits),
                                         expert_counts.data_ptr(), expert_offsets.data_ptr(), dest_counts.data_ptr(),
                                         dest_offsets.data_ptr(), slot_of_row.data_ptr(), row_of_slot.data_ptr(), wp,
                                         wb, _stream()))


def moe_permute(x, K: int, slot_of_row, row_of_slot, xp):
    N, H = x.shape
    assert x.is_contiguous() and xp.is_contiguous() and xp.dtype == x.dtype and xp.numel() == N * K * H
    assert slot_of_row.numel() == N * K and row_of_slot.numel() == N * K
    lib = _lib or load_library()
    _check(lib.moe_permute(x.data_ptr(), _dtype_code(x), N, H, K, slot_of_row.data_ptr(), row_of_slot.data_ptr(),
                           xp.data_ptr(), _stream()))


def moe_grouped_ffn(xp, seg_offsets, W_gate, W_up, W_down, y, ws):
    M, H = xp.shape
    E_local, F, H2 = W_gate.shape
    assert H2 == H and tuple(W_up.shape) == (E_local, F, H) and tuple(W_down.shape) == (E_local, H, F)
    assert W_gate.dtype == W_up.dtype == W_down.dtype == xp.dtype == y.dtype
    for t in (xp, W_gate, W_up, W_down, y):
        assert t.is_cuda and t.is_contiguous()
    _need(seg_offsets, torch.int32, "seg_offsets")
    assert seg_offsets.numel() == E_local + 1 and y.numel() == M * H
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_grouped_ffn(xp.data_ptr(), _dtype_code(xp), M, H, F, E_local, seg_offsets.data_ptr(),
                               W_gate.data_ptr(), W_up.data_ptr(), W_down.data_ptr(), y.data_ptr(), wp, wb, _stream()))


def moe_ffn_schedule(dtype: int, M: int, H: int, F: int, seg_offsets, ws):
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_ffn_schedule(dtype, M, H, F, seg_offsets.numel() - 1, seg_offsets.data_ptr(), wp, wb, _stream()))


def moe_ffn_gate_up_down(xp, seg_offsets, W_gate, W_up, W_down, y, ws, wait_limit: int = 0):
    M, H = xp.shape
    E_local, F, H2 = W_gate.shape
    assert H2 == H and tuple(W_up.shape) == (E_local, F, H) and tuple(W_down.shape) == (E_local, H, F)
    assert W_gate.dtype == W_up.dtype == W_down.dtype == xp.dtype == y.dtype
    for t in (xp, W_gate, W_up, W_down, y):
        assert t.is_cuda and t.is_contiguous()
    _need(seg_offsets, torch.int32, "seg_offsets")
    assert seg_offsets.numel() == E_local + 1 and y.numel() == M * H
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_ffn_gate_up_down(xp.data_ptr(), _dtype_code(xp), M, H, F, E_local, seg_offsets.data_ptr(),
                                    W_gate.data_ptr(), W_up.data_ptr(), W_down.data_ptr(), y.data_ptr(), wp, wb,
                                    wait_limit, _stream()))


def moe_ffn_status(dtype: int, M: int, H: int, F: int, E_local: int, ws):
    """Waits for the current stream; raises MoEHubError(MOE_ERR_STATE) if a GEMM step found no schedule."""
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_ffn_status(dtype, M, H, F, E_local, wp, wb, _stream()))


def moe_ffn_gate_up(xp, seg_offsets, W_gate, W_up, ws):
    M, H = xp.shape
    E_local, F, _ = W_gate.shape
    assert tuple(W_up.shape) == tuple(W_gate.shape) and W_gate.shape[2] == H
    assert xp.is_contiguous() and W_gate.is_contiguous() and W_up.is_contiguous()
    assert seg_offsets.numel() == E_local + 1
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_ffn_gate_up(xp.data_ptr(), _dtype_code(xp), M, H, F, E_local, seg_offsets.data_ptr(),
                               W_gate.data_ptr(), W_up.data_ptr(), wp, wb, _stream()))


def moe_ffn_gate_up_gather(x, K: int, seg_offsets, row_of_slot, W_gate, W_up, ws):
    N, H = x.shape
    E_local, F, _ = W_gate.shape
    assert tuple(W_up.shape) == tuple(W_gate.shape) and W_gate.shape[2] == H
    assert x.is_contiguous() and W_gate.is_contiguous() and W_up.is_contiguous()
    assert seg_offsets.numel() == E_local + 1
    _need(row_of_slot, torch.int32, "row_of_slot")
    assert row_of_slot.numel() == N * K
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_ffn_gate_up_gather(x.data_ptr(), _dtype_code(x), N, K, H, F, E_local, seg_offsets.data_ptr(),
                                      row_of_slot.data_ptr(), W_gate.data_ptr(), W_up.data_ptr(), wp, wb, _stream()))


def moe_ffn_down(seg_offsets, W_down, y, ws):
    M, H = y.shape
    E_local, H2, F = W_down.shape
    assert H2 == H and y.is_contiguous() and W_down.is_contiguous() and W_down.dtype == y.dtype
    assert seg_offsets.numel() == E_local + 1
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_ffn_down(_dtype_code(y), M, H, F, E_local, seg_offsets.data_ptr(), W_down.data_ptr(), y.data_ptr(),
                            wp, wb, _stream()))


def moe_ffn_down_combine(K: int, seg_offsets, W_down, row_of_slot, topk_w, sums, out, ws):
    N, H = out.shape
    E_local, H2, F = W_down.shape
    assert H2 == H and out.is_contiguous() and W_down.is_contiguous() and W_down.dtype == out.dtype
    assert seg_offsets.numel() == E_local + 1
    _need(row_of_slot, torch.int32, "row_of_slot")
    _need(topk_w, torch.float32, "topk_w")
    _need(sums, torch.float32, "sums")
    assert row_of_slot.numel() == N * K and topk_w.numel() == N * K and sums.numel() == N * H
    wp, wb = _ws_args(ws)
    lib = _lib or load_library()
    _check(lib.moe_ffn_down_combine(_dtype_code(out), N, K, H, F, E_local, seg_offsets.data_ptr(), W_down.data_ptr(),
                                    row_of_slot.data_ptr(), topk_w.data_ptr(), sums.data_ptr(), out.data_ptr(), wp, wb,
                                    _stream()))


def moe_combine(y, K: int, slot_of_row, topk_w, out):
    N, H = out.shape
    assert y.is_contiguous() and out.is_contiguous() and y.dtype == out.dtype and y.numel() == N * K * H
    _need(topk_w, torch.float32, "topk_w")
    assert slot_of_row.numel() == N * K and topk_w.numel() == N * K
    lib = _lib or load_library()
    _check(lib.moe_combine(y.data_ptr(), _dtype_code(y), N, H, K, slot_of_row.data_ptr(), topk_w.data_ptr(),
                           out.data_ptr(), _stream()))
