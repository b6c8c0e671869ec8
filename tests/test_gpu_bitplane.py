"""Planes of bits on the fp4 matrix cores (bitplane.hip): bit for bit against
the oracle, or against the byte VALU path where the oracle would be slow, at
the edges of the packing (fields per word, per 16-byte chunk, per stage), of
the tiles and of the tile shapes, with rows of any alignment, and on both sides
of the bound below which the quotient is taken in FP32."""

import numpy as np
import pytest

import oracle
import workloads
from psx import announce, check_exact_f32, host, need_gpu, slab_off, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _levels(n_v, n_f, L, seed, pad=0):
    """n_v x n_f values 0..L in rows of n_f + pad bytes, the pad 255."""
    V = workloads.levels(n_v, n_f + pad, seed=seed, probs=np.full(L + 1, 1.0 / (L + 1)))
    V[:, n_f:] = 255
    if n_v > 2:
        V[n_v // 2, :n_f] = 0      # an all-zero vector
    return V


def _opt(L, binary):
    return dict(path="bits", levels=1) if binary else dict(path="mfma_fp4", levels=L)


# (n_v, n_f, L, pad): field edges of the word (32), chunk (128 bits), group
# (256) and stage (512), planes that end inside a stage, row alignments
FIELDS = [(70, 1, 1, 0), (70, 31, 1, 0), (70, 32, 1, 16), (70, 33, 3, 0), (70, 127, 1, 1),
          (70, 128, 1, 0), (70, 129, 5, 0), (70, 511, 1, 0), (70, 512, 1, 0), (70, 513, 1, 3),
          (70, 1025, 2, 7), (70, 4000, 7, 0), (70, 2049, 15, 0), (70, 96, 127, 4)]
# tile edges of the 64-wide shape
TILES = [(2, 40, 3, 0), (3, 200, 3, 0), (63, 100, 2, 0), (64, 100, 2, 0), (65, 100, 2, 0),
         (129, 700, 3, 0), (257, 300, 1, 0)]


@pytest.mark.parametrize("n_v,n_f,L,pad", FIELDS + TILES)
def test_2way(n_v, n_f, L, pad):
    from paper_1705_08210_amd import ps
    big = _levels(n_v, n_f, L, seed=n_v + n_f, pad=pad)
    V = np.ascontiguousarray(big[:, :n_f])
    Vd = to_dev(big)[:, :n_f]
    ref, rn2 = oracle.c2_all(V, with_n2=True)
    for kw in [_opt(L, False)] + ([_opt(L, True)] if L == 1 else []):
        announce(f"bit planes 2-way {n_v}x{n_f} pad={pad} {kw}")
        c2, n2 = ps.ps2(Vd, want_n2=True, **kw)
        check_exact_f32(host(c2), ref, "c2")
        assert np.array_equal(host(n2).astype(np.float64), rn2)
        s, _ = ps.vector_sums(Vd)
        given, _ = ps.ps2(Vd, s=s, **kw)
        assert np.array_equal(host(given).view(np.uint32), host(c2).view(np.uint32))


@pytest.mark.parametrize("n_v", [1536, 1537, 5632, 5700])
def test_2way_tile_shapes(n_v):
    """The last size of one tile shape and the first of the next."""
    from paper_1705_08210_amd import ps
    V = to_dev(_levels(n_v, 150, 3, seed=n_v))
    announce(f"bit planes 2-way shape n_v={n_v}")
    a, na = ps.ps2(V, want_n2=True, path="mfma_fp4", levels=3)
    b, nb = ps.ps2(V, want_n2=True, path="valu")
    assert bool((a == b).all()) and bool((na == nb).all())


@pytest.mark.parametrize("n_f", [4_190_000, 8_388_607, 8_388_609])
def test_2way_quotient_bound(n_f):
    """2 n2 on both sides of 2^24: FP32 and FP64 quotients."""
    from paper_1705_08210_amd import ps
    V = _levels(3, n_f, 1, seed=9)
    V[0, :] = 1
    announce(f"bit planes quotient n_f={n_f}")
    c2, _ = ps.ps2(to_dev(V), path="bits", levels=1)
    check_exact_f32(host(c2), oracle.c2_all(V), "c2")


@pytest.mark.parametrize("n_v,n_f,L,pad", FIELDS[::2] + [(3, 64, 3, 0), (4, 300, 2, 1),
                                                        (130, 200, 3, 0), (300, 520, 1, 0)])
def test_3way(n_v, n_f, L, pad):
    from paper_1705_08210_amd import ps
    big = _levels(n_v, n_f, L, seed=n_v + 2 * n_f, pad=pad)
    V = np.ascontiguousarray(big[:, :n_f])
    Vd = to_dev(big)[:, :n_f]
    ref = oracle.c3_all(V)
    for kw in [_opt(L, False)] + ([_opt(L, True)] if L == 1 else []):
        announce(f"bit planes 3-way {n_v}x{n_f} pad={pad} {kw}")
        check_exact_f32(host(ps.ps3(Vd, **kw)), ref, "c3")
        s, _ = ps.vector_sums(Vd)
        _, n2 = ps.ps2(Vd, s=s, want_c2=False, want_n2=True, **kw)
        jb, je = max(1, n_v // 3), max(2, min(n_v - 1, 2 * n_v // 3))
        lo, hi = int(slab_off(n_v, jb)), int(slab_off(n_v, je))
        part = ps.ps3(Vd, s=s, n2=n2, j_begin=jb, j_end=je, **kw)
        check_exact_f32(host(part), ref[lo:hi], f"stage [{jb}, {je})")


@pytest.mark.parametrize("n_f", [2_796_000, 2_796_400])
def test_3way_quotient_bound(n_f):
    """6 n_f on both sides of 2^24."""
    from paper_1705_08210_amd import ps
    V = _levels(4, n_f, 1, seed=10)
    V[0, :] = 1
    announce(f"bit planes 3-way quotient n_f={n_f}")
    check_exact_f32(host(ps.ps3(to_dev(V), path="bits", levels=1)), oracle.c3_all(V), "c3")


def test_auto_levels_take_the_planes():
    """AUTO on integer levels: planes of bits for the 3-way slices and the
    larger triangles, the same bits as the other paths."""
    from paper_1705_08210_amd import ps
    assert ps.path_choice(np.uint8, 3, 333, 150, levels=2) == ps.PATH["mfma_fp4"]
    V = to_dev(_levels(150, 333, 2, seed=5))
    announce("bit planes auto 3-way")
    a = host(ps.ps3(V, levels=2))
    for path in ("mfma", "valu"):
        b = host(ps.ps3(V, path=path, levels=2))
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


def test_noalloc_auto_without_room_for_planes():
    """ps3_noalloc where the planes do not fit the static scratch: AUTO runs
    the int8 path, which has none."""
    from paper_1705_08210_amd import ps
    import torch
    n_v, n_f = 300, 200_000       # planes: 300 x 3 x 100 KB
    V = to_dev(_levels(n_v, n_f, 3, seed=6))
    s, _ = ps.vector_sums(V)
    _, n2 = ps.ps2(V, s=s, want_c2=False, want_n2=True, path="valu")
    c3 = torch.empty(ps.stage_size(n_v, 100, 102), device=V.device)
    announce("bit planes noalloc without room")
    ps.ps3_noalloc(V, c3, s=s, n2=n2, j_begin=100, j_end=102, levels=3)
    ref = ps.ps3(V, s=s, n2=n2, j_begin=100, j_end=102, path="mfma", levels=3)
    assert bool((c3 == ref).all())


def _shape_sizes():
    """The last and first sizes of every tile shape, and for the widest one a last
    row block of one row, of half a block, of one row more, and all but one row."""
    import librules
    a = librules.line(librules.bp2_rows, 64, 4096)
    b = librules.line(librules.bp2_rows, a, 16384)
    assert [librules.bp2_rows(n) for n in (a - 1, a, b - 1, b)] == [64, 128, 128, 256]
    c = -(-b // 256) * 256
    return [a - 1, a, b - 1, b, c + 1, c + 128, c + 129, c + 255]


@pytest.mark.parametrize("k", range(8))
def test_2way_shape_edges(k):
    from paper_1705_08210_amd import ps
    n_v = _shape_sizes()[k]
    for L, kw in ((3, dict(path="mfma_fp4", levels=3)), (1, dict(path="bits", levels=1))):
        V = to_dev(_levels(n_v, 150, L, seed=n_v))
        announce(f"bit planes 2-way shape edge n_v={n_v} {kw}")
        a, na = ps.ps2(V, want_n2=True, **kw)
        b, nb = ps.ps2(V, want_n2=True, path="valu")
        assert bool((a == b).all()) and bool((na == nb).all())
