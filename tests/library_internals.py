"""The library's inner functions that a test asks or calls by themselves, and a handle that needs no GPU: its shape and layout, with
no arrays behind it, for the functions that choose a kernel on the host."""
import ctypes
from ctypes import c_bool, c_int, c_int64, c_size_t, c_void_p

from paper_2310_02065_amd import binding


class Layout(ctypes.Structure):
    _fields_ = [("R", c_int64), ("K", c_int64), ("G", c_int64), ("Rb", c_int64), ("W", c_int64), ("steps", c_int64), ("vt", c_int),
                ("Rbp", c_int64), ("rec_bytes", c_int64), ("packed", c_bool), ("off_values", c_size_t), ("off_columns", c_size_t),
                ("off_meta", c_size_t), ("off_arec", c_size_t), ("off_rowidx", c_size_t), ("off_status", c_size_t), ("total", c_size_t)]


class HostHandle(ctypes.Structure):
    _fields_ = [("R", c_int64), ("K", c_int64), ("V", c_int), ("N", c_int), ("M", c_int), ("lay", Layout), ("ws", c_void_p)]


def inner(name, restype, *argtypes):
    f = getattr(binding.lib(), name)
    f.argtypes, f.restype = list(argtypes), restype
    return f


def host_handle(R, K, V, M):
    make_layout = inner("_ZN5venom11make_layoutEllii", Layout, c_int64, c_int64, c_int, c_int)
    h = HostHandle(R, K, V, 2, M, make_layout(R, K, V, M), None)
    n = c_size_t(0)
    assert binding.lib().venom_workspace_bytes(R, K, V, 2, M, ctypes.byref(n)) == 0 and n.value == h.lay.total   # (the same layout)
    return h


# how a product of few columns, or a layer of few tokens that reads X in place, is dealt to workgroups
NONE, WHOLE, SPLIT, PAIR = -1, 0, 1, 2


def layer_form(h, X, ldx, tokens, Y, ldy, dtype=0, units=256):
    f = inner("_ZN5venom12skinny_layerERK12venom_handlePKvllS4_lii", c_int, c_void_p, c_void_p, c_int64, c_int64, c_void_p, c_int64,
              c_int, c_int)
    return f(ctypes.byref(h), X, ldx, tokens, Y, ldy, dtype, units)


def product_form(h, ldb, cols, units=256):
    f = inner("_ZN5venom14skinny_productERK12venom_handlelli", c_int, c_void_p, c_int64, c_int64, c_int)
    return f(ctypes.byref(h), ldb, cols, units)
