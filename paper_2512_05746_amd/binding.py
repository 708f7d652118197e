"""Python face of libhq.so: one function per C entry point declared in ``include/hq.h``.

Tensors are PyTorch tensors used purely as device buffers, and the work is enqueued on PyTorch's
current HIP stream.  The library is loaded with ctypes; the checks of the arguments, the allocation of
results and the calls themselves are native (``csrc/marshal.cpp``).  There is no fallback: if a library
cannot be loaded or a call is refused, an exception is raised.
"""
from __future__ import annotations

import ctypes
from typing import Optional, Tuple

import torch

from . import build as _build

SYMBOLS = ("hq_status_string", "hq_quantize_weights", "hq_act_hadamard_quant",
           "hq_int_linear", "hq_int_conv2d", "hq_act_hadamard_quant_static",
           "hq_int_linear_static", "hq_int_conv2d_static",
           "hq_quantize_weights_single", "hq_int_linear_single",
           "hq_act_hadamard_quant_width", "hq_int_conv2d_width",
           "hq_int_linear_i8", "hq_int_conv2d_i8", "hq_act_hadamard_quant_i8",
           "hq_act_quant_int_conv2d", "hq_act_quant_int_linear")
# entry points that do not return a status
INFO_SYMBOLS = ("hq_int_conv2d_kernel_name",)


class HqError(RuntimeError):
    def __init__(self, fn: str, code: int, text: str):
        super().__init__("%s failed: %s (status %d)" % (fn, text, code))
        self.code = code


_lib = None
_marshal = None      # the native module, bound to the loaded library


def _native():
    """The native module; loads the library on first use."""
    if _marshal is None:
        load_library()
    return _marshal


def load_library(path: Optional[str] = None) -> ctypes.CDLL:
    """Loads libhq.so.  The in-tree library is built first if it is missing or older than one of
    its sources (a child-process compile; nothing here touches the GPU before that)."""
    global _lib, _marshal
    if _lib is not None and path is None:
        return _lib
    if path is None:
        path = _build.LIB
        if _build.is_stale():
            _build.build_lib()
    lib = ctypes.CDLL(path)
    vp, i32, i64 = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64
    lib.hq_status_string.argtypes = [i32]
    lib.hq_status_string.restype = ctypes.c_char_p
    lib.hq_quantize_weights.argtypes = [vp, i32, i32, i32, i32, i32, i32, vp, vp, vp]
    lib.hq_act_hadamard_quant.argtypes = [vp, i32, i64, i32, i32, i32, vp, vp, vp]
    lib.hq_int_linear.argtypes = [vp, vp, vp, vp, vp, i64, i32, i32, vp, i32, vp]
    lib.hq_int_conv2d.argtypes = [vp] * 5 + [i32] * 9 + [vp, i32, vp]
    lib.hq_act_hadamard_quant_static.argtypes = [vp, i32, i64, i32, i32, i32, vp, vp, vp]
    lib.hq_int_linear_static.argtypes = lib.hq_int_linear.argtypes
    lib.hq_int_conv2d_static.argtypes = lib.hq_int_conv2d.argtypes
    lib.hq_quantize_weights_single.argtypes = [vp, i32, i32, i32, i32, i32, vp, vp, vp]
    lib.hq_int_linear_single.argtypes = [vp, vp, vp, vp, vp, i64, i32, i32, i32, vp, i32, vp]
    lib.hq_act_hadamard_quant_width.argtypes = [vp, i32, i32, i32, i32, i32, i32, i32, vp, vp, vp]
    lib.hq_int_conv2d_width.argtypes = [vp] * 5 + [i32] * 10 + [vp, i32, vp]
    lib.hq_int_linear_i8.argtypes = lib.hq_int_linear.argtypes
    lib.hq_act_hadamard_quant_i8.argtypes = lib.hq_act_hadamard_quant.argtypes
    lib.hq_int_conv2d_i8.argtypes = lib.hq_int_conv2d.argtypes
    lib.hq_act_quant_int_conv2d.argtypes = [vp, i32, vp, vp, vp] + [i32] * 11 + [vp, i32, vp, vp, vp]
    lib.hq_act_quant_int_linear.argtypes = [vp, i32, vp, vp, vp, i64, i32, i32, i32, i32, vp, i32, vp, vp, vp]
    for name in SYMBOLS[1:]:
        getattr(lib, name).restype = i32
    lib.hq_int_conv2d_kernel_name.argtypes = [i32] * 11
    lib.hq_int_conv2d_kernel_name.restype = ctypes.c_char_p
    from . import _marshal as marshal
    marshal.bind({name: ctypes.cast(getattr(lib, name), ctypes.c_void_p).value for name in SYMBOLS}, HqError)
    _lib, _marshal = lib, marshal
    return lib


def hq_int_conv2d_kernel_name(nb: int, h: int, w: int, c_in: int, c_out: int, ksize: int = 3, stride: int = 1,
                              pad: Optional[int] = None, static_scale: bool = False, bits: int = 4) -> str:
    """Name of the kernel the convolution calls run for this geometry, and its tile (host logic only)."""
    pad = (ksize - 1) // 2 if pad is None else pad
    return load_library().hq_int_conv2d_kernel_name(nb, h, w, c_in, c_out, ksize, ksize, stride, pad,
                                                    1 if static_scale else 0, bits).decode()


def status_string(code: int) -> str:
    return load_library().hq_status_string(code).decode()


def hq_quantize_weights(w: torch.Tensor, had_block: int = 64, w_bits: int = 4
                        ) -> Tuple[torch.Tensor, torch.Tensor]:
    """w [n_out, taps, k_in] fp16/fp32 -> (wq uint8 [n_out, taps, k_in/2], w_scale fp32 [n_out]);
    w_bits = 8: wq int8 [n_out, taps, k_in], one code per byte."""
    return _native().quantize_weights(w, had_block, w_bits)


def hq_act_hadamard_quant(x: torch.Tensor, had_block: int = 64, a_bits: int = 4,
                          out: Optional[Tuple[torch.Tensor, torch.Tensor]] = None
                          ) -> Tuple[torch.Tensor, torch.Tensor]:
    """x [..., k] fp16/fp32 -> (xq uint8 [..., k/2], x_scale fp32 [...]); a_bits = 8: xq int8 [..., k]."""
    return _native().act_hadamard_quant(x, had_block, a_bits, out)


def hq_int_linear(xq: torch.Tensor, x_scale: Optional[torch.Tensor], wq: torch.Tensor,
                  w_scale: Optional[torch.Tensor], bias: Optional[torch.Tensor] = None,
                  y_dtype: torch.dtype = torch.float16, out: Optional[torch.Tensor] = None
                  ) -> torch.Tensor:
    """xq [m, k/2], wq [n, k/2] (or [n, 1, k/2]) -> y [m, n]; y_dtype int32 returns the raw sums."""
    return _native().linear(xq, x_scale, wq, w_scale, bias, y_dtype, out)


def hq_int_conv2d(xq: torch.Tensor, x_scale: Optional[torch.Tensor], wq: torch.Tensor,
                  w_scale: Optional[torch.Tensor], bias: Optional[torch.Tensor] = None,
                  ksize: int = 3, stride: int = 1, pad: Optional[int] = None,
                  y_dtype: torch.dtype = torch.float16, out: Optional[torch.Tensor] = None
                  ) -> torch.Tensor:
    """xq [nb, h, w, cin/2], wq [cout, ksize*ksize, cin/2] -> y [nb, ho, wo, cout] (same size for
    stride 1; ksize 3, stride 2, pad 1 halves it, rounding up); y_dtype int32 returns the per-tap
    sums [nb, ho, wo, ksize*ksize, cout]."""
    return _native().conv2d(xq, x_scale, wq, w_scale, bias, ksize, stride, pad, y_dtype, out)


def hq_act_quant_int_conv2d(x: torch.Tensor, wq: torch.Tensor, w_scale: Optional[torch.Tensor],
                            bias: Optional[torch.Tensor] = None, had_block: int = 64, a_bits: int = 4,
                            ksize: int = 3, stride: int = 1, pad: Optional[int] = None,
                            y_dtype: torch.dtype = torch.float16, out: Optional[torch.Tensor] = None,
                            codes_out: Optional[Tuple[torch.Tensor, torch.Tensor]] = None) -> torch.Tensor:
    """The whole 3x3 layer in one launch: x [nb, h, w, cin] fp16, wq [cout, 9, cin/2] -> y [nb, h, w, cout]
    (y_dtype int32: per-tap sums [nb, h, w, 9, cout]).  codes_out = (xq uint8 [nb, h, w, cin/2],
    x_scale fp32 [nb, h, w]) receives the codes and scales the kernel used."""
    return _native().act_quant_conv2d(x, wq, w_scale, bias, had_block, a_bits, ksize, stride, pad, y_dtype, out,
                                      codes_out)


def hq_act_quant_int_linear(x: torch.Tensor, wq: torch.Tensor, w_scale: Optional[torch.Tensor],
                            bias: Optional[torch.Tensor] = None, had_block: int = 64, a_bits: int = 4,
                            y_dtype: torch.dtype = torch.float16, out: Optional[torch.Tensor] = None,
                            codes_out: Optional[Tuple[torch.Tensor, torch.Tensor]] = None) -> torch.Tensor:
    """A linear layer / 1x1 convolution in one launch: x [..., k] fp16, wq [n, k/2] (or [n, 1, k/2]) ->
    y [..., n] (y_dtype int32: the integer sums).  codes_out = (xq uint8 [..., k/2], x_scale fp32 [...])
    receives the codes and scales the kernel used."""
    return _native().act_quant_linear(x, wq, w_scale, bias, had_block, a_bits, y_dtype, out, codes_out)


def hq_act_hadamard_quant_static(x: torch.Tensor, x_scale: torch.Tensor, had_block: int = 64,
                                 a_bits: int = 4, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """x [..., k] fp16/fp32, x_scale one fp32 on the device -> xq uint8 [..., k/2]."""
    return _native().act_hadamard_quant_static(x, x_scale, had_block, a_bits, out)


def hq_int_linear_static(xq: torch.Tensor, x_scale: Optional[torch.Tensor], wq: torch.Tensor,
                         w_scale: Optional[torch.Tensor], bias: Optional[torch.Tensor] = None,
                         y_dtype: torch.dtype = torch.float16, out: Optional[torch.Tensor] = None
                         ) -> torch.Tensor:
    """As hq_int_linear with one activation scale (a device tensor holding one float32)."""
    return _native().linear_static(xq, x_scale, wq, w_scale, bias, y_dtype, out)


def hq_int_conv2d_static(xq: torch.Tensor, x_scale: Optional[torch.Tensor], wq: torch.Tensor,
                         w_scale: Optional[torch.Tensor], bias: Optional[torch.Tensor] = None,
                         ksize: int = 3, stride: int = 1, pad: Optional[int] = None,
                         y_dtype: torch.dtype = torch.float16, out: Optional[torch.Tensor] = None
                         ) -> torch.Tensor:
    """As hq_int_conv2d with one activation scale; y_dtype int32 returns the sums over all
    taps and input channels, [nb, h, w, cout]."""
    return _native().conv2d_static(xq, x_scale, wq, w_scale, bias, ksize, stride, pad, y_dtype, out)


# ---- Single scheme: un-transformed quantised weights, integer H folded into digit planes -------

def hq_quantize_weights_single(w: torch.Tensor, had_block: int = 64, w_bits: int = 4
                               ) -> Tuple[torch.Tensor, torch.Tensor]:
    """w [n_out, k_in] fp16/fp32 -> (wq3 uint8 [n_out, 3, k_in/2] digit planes, w_scale fp32 [n_out])."""
    return _native().quantize_weights_single(w, had_block, w_bits)


def hq_int_linear_single(xq: torch.Tensor, x_scale: Optional[torch.Tensor], wq3: torch.Tensor,
                         w_scale: Optional[torch.Tensor], bias: Optional[torch.Tensor] = None,
                         had_block: int = 64, y_dtype: torch.dtype = torch.float16,
                         out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """xq [m, k/2], wq3 [n, 3, k/2] -> y [m, n]; y_dtype int32 returns the three sums [m, 3, n]."""
    return _native().linear_single(xq, x_scale, wq3, w_scale, bias, had_block, y_dtype, out)


# ---- width-axis convolution: the paper's own convolution ---------------------------------------

def hq_act_hadamard_quant_width(x: torch.Tensor, x_scale: torch.Tensor, had_block: int, a_bits: int = 4,
                                out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """x [N, H, W, C] fp16/fp32, x_scale one fp32 on the device -> xu3 uint8 [3, N, H, W, C/2]
    (digit planes of the codes taken back along the width axis with the +-1 matrix)."""
    return _native().act_hadamard_quant_width(x, x_scale, had_block, a_bits, out)


def hq_int_conv2d_width(xu3: torch.Tensor, x_scale: Optional[torch.Tensor], wq: torch.Tensor,
                        w_scale: Optional[torch.Tensor], bias: Optional[torch.Tensor] = None,
                        had_block: int = 64, y_dtype: torch.dtype = torch.float16,
                        out: Optional[torch.Tensor] = None, stride: int = 1) -> torch.Tensor:
    """xu3 [3, N, H, W, Cin/2], wq [Cout, 9, Cin/2] (or [Cout, 3, 3, Cin/2]) -> y [N, Ho, Wo, Cout]
    (same size for stride 1; stride 2 halves it, rounding up); y_dtype int32 returns the exact integer sums.  The
    integers in the planes must lie within 8 * had_block, as those of hq_act_hadamard_quant_width do."""
    return _native().conv2d_width(xu3, x_scale, wq, w_scale, bias, had_block, y_dtype, out, stride)


# ---- 8-bit codes (W8A8): int8 operands, one code per byte ---------------------------------------

def hq_act_hadamard_quant_i8(x: torch.Tensor, had_block: int = 64, a_bits: int = 4
                             ) -> Tuple[torch.Tensor, torch.Tensor]:
    """x [..., k] fp16/fp32 -> (xq int8 [..., k] with codes of a_bits bits, x_scale fp32 [...])."""
    return _native().act_hadamard_quant_i8(x, had_block, a_bits)


def hq_int_linear_i8(xq: torch.Tensor, x_scale: Optional[torch.Tensor], wq: torch.Tensor,
                     w_scale: Optional[torch.Tensor], bias: Optional[torch.Tensor] = None,
                     y_dtype: torch.dtype = torch.float16, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """xq int8 [m, k], wq int8 [n, k] (or [n, 1, k]) -> y [m, n]; y_dtype int32 returns the raw sums."""
    return _native().linear_i8(xq, x_scale, wq, w_scale, bias, y_dtype, out)


def hq_int_conv2d_i8(xq: torch.Tensor, x_scale: Optional[torch.Tensor], wq: torch.Tensor,
                     w_scale: Optional[torch.Tensor], bias: Optional[torch.Tensor] = None,
                     ksize: int = 3, y_dtype: torch.dtype = torch.float16,
                     out: Optional[torch.Tensor] = None, stride: int = 1) -> torch.Tensor:
    """xq int8 [N, H, W, Cin], wq int8 [Cout, ksize*ksize, Cin] -> y [N, Ho, Wo, Cout] (same size for
    stride 1; ksize 3 at stride 2 halves it, rounding up); y_dtype int32 returns the per-tap sums
    [N, Ho, Wo, ksize*ksize, Cout]."""
    return _native().conv2d_i8(xq, x_scale, wq, w_scale, bias, ksize, stride, None, y_dtype, out)
