"""The launch rules of libps, called in the built library by their C++ names, so
that tests take the sizes of a rule's line from the rule itself."""

import ctypes

from paper_1705_08210_amd import ps

I32, I64, P = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p


def _rule(name, res, *args):
    f = getattr(ps.lib, name)
    f.restype, f.argtypes = res, list(args)
    return f


# int bp2_rows(int64_t n_v): rows of the tiles of planes of bits
bp2_rows = _rule("_ZN2ps8bp2_rowsEl", I32, I64)

# int small3(int64_t n_f, int64_t n_v, int32_t nchunks, const ps_opts*)
_small3 = _rule("_ZN2ps6small3ElliPK7ps_opts", I32, I64, I64, I32, P)


def small3(n_f, n_v, nchunks, tile=0):
    """Waves of the 3-way 32 x 32 tiles, 0: the 64 x 64 tiles."""
    return _small3(n_f, n_v, nchunks, ctypes.byref(ps._opts(tile=tile)))


class _Split(ctypes.Structure):
    _fields_ = [("nchunks", I32), ("chunk_tiles", I64)]


# int choose_cfg(int32_t dt, int32_t way, int32_t path, int64_t n_f, int64_t n_v, const ps_opts*)
_choose_cfg = _rule("_ZN2ps10choose_cfgEiiillPK7ps_opts", I32, I32, I32, I32, I64, I64, P)
# Split plan_split(int32_t dt, int64_t n_f, int64_t n_v, int cfg, const ps_opts*)
_plan_split = _rule("_ZN2ps10plan_splitEilliPK7ps_opts", _Split, I32, I64, I64, I32, P)
# int small2(int32_t dt, int64_t n_f, int64_t n_v, int cfg, int32_t nchunks, const ps_opts*)
_small2 = _rule("_ZN2ps6small2EilliiPK7ps_opts", I32, I32, I64, I64, I32, I32, P)


def pairs_2way(dtype, n_f, n_v):
    """(waves of the 32 x 32 tiles or 0, field chunks) of a 2-way call on the VALU."""
    dt, o = ps.DTYPES[dtype], ctypes.byref(ps._opts())
    cfg = _choose_cfg(dt, 2, ps.PATH["valu"], n_f, n_v, o)
    chunks = _plan_split(dt, n_f, n_v, cfg, o).nchunks
    return _small2(dt, n_f, n_v, cfg, chunks, o), chunks


def line(rule, lo, hi):
    """The first n in (lo, hi] at which rule(n) differs from rule(lo); a rule with
    one line in the range."""
    first = rule(lo)
    assert rule(hi) != first
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if rule(mid) == first else (lo, mid)
    return hi
