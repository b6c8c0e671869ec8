"""The launch rules of libps, called in the built library by their C++ names, so
that tests take the sizes of a rule's line from the rule itself."""

import ctypes

from paper_1705_08210_amd import ps

I32, I64, P = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p


def _rule(name, res, *args):
    f = getattr(ps.lib, name)
    f.restype, f.argtypes = res, list(args)
    return f


# int small3(int64_t n_f, int64_t n_v, int32_t nchunks, const ps_opts*)
_small3 = _rule("_ZN2ps6small3ElliPK7ps_opts", I32, I64, I64, I32, P)


def small3(n_f, n_v, nchunks, tile=0):
    """Waves of the 3-way 32 x 32 tiles, 0: the 64 x 64 tiles."""
    return _small3(n_f, n_v, nchunks, ctypes.byref(ps._opts(tile=tile)))
