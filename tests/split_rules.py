"""The library's own choices between kernels and grids, asked through the functions that its launchers ask.  No GPU."""
import ctypes

from paper_1901_07988_amd import binding as B


class Geom(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("N", "H", "W", "Cin", "Cout", "R", "S", "stride", "pad", "Ho", "Wo")]


def geom(N, H, W, cin, cout, R):
    return Geom(N, H, W, cin, cout, R, R, 1, (R - 1) // 2, H, W)   # 'same', stride 1


def _fn(name, res, *args):
    f = getattr(B.lib, name)
    f.restype, f.argtypes = res, [ctypes.POINTER(Geom), *args]
    return f


_i, _b = ctypes.c_int, ctypes.c_bool
_blocks = _fn("_ZN3abl17split_conv_blocksERKNS_8ConvGeomEibb", _i, _i, _b, _b)
_forward3 = _fn("_ZN3abl14split_forward3ERKNS_8ConvGeomEPi", _i, ctypes.POINTER(_i))
_parts_pay = _fn("_ZN3abl9parts_payERKNS_8ConvGeomEibb", _b, _i, _b, _b)
_beats_image = _fn("_ZN3abl17split_beats_imageERKNS_8ConvGeomEi", _b, _i)


def rows(s, mode, bf16=False, sums=False):
    """Blocks along the pixels of the split convolution that the layer takes, 0 = another kernel."""
    return _blocks(ctypes.byref(geom(*s)), mode, bf16, sums)


def fused_rows(s):
    """Blocks along the pixels of the 3x3 forward with the prologue (0: it does not run; -1: a pass of its own in front)."""
    n = _i(0)
    path = _forward3(ctypes.byref(geom(*s)), ctypes.byref(n))
    return n.value if path > 0 else path


def parts_pay(s, mode, bf16=False, own_launch=False):
    """Whether the weights of a layer are split once per call instead of by its blocks."""
    return _parts_pay(ctypes.byref(geom(*s)), mode, bf16, own_launch)


def beats_image(s, mode):
    """Whether a 3x3 layer with bf16 operands prefers the split convolution to the image-resident kernel."""
    return _beats_image(ctypes.byref(geom(*s)), mode)
