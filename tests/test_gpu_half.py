"""The FP16 tiles whose sums run on the matrix cores (mgemm_half.h): every tile
configuration at the edges of the tiles, the field tiles and the 16-byte chunks,
with rows of any alignment, against the oracle on the FP16 values (at most 4200
terms, FP32 sums: 1e-5); and a vector with infinities and NaN, which must not
touch the pairs of the others."""

import itertools

import numpy as np
import pytest

import oracle
import workloads
from psx import announce, check_rel, colex, host, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _half(n_v, n_f, seed):
    return workloads.to_f16(workloads.gwas_like(n_v, n_f, seed=seed))


@pytest.mark.parametrize("tile", [1, 2, 3])
@pytest.mark.parametrize("n_v,n_f", [(2, 1), (64, 7), (65, 8), (127, 9), (128, 32), (129, 33),
                                     (200, 64), (257, 65), (300, 129), (130, 4201)])
def test_2way_and_batched(n_v, n_f, tile):
    from paper_1705_08210_amd import ps
    V = _half(n_v, n_f, seed=n_v + n_f)
    announce(f"half 2-way {n_v}x{n_f} tile={tile}")
    Vd = to_dev(V)
    ref = oracle.c2_all(V.astype(np.float32))
    c2, _ = ps.ps2(Vd, acc="plain", tile=tile)
    check_rel(host(c2), ref, 1e-5, "c2")
    for pad in (1, 3, 8):     # 2-, 2- and 16-byte row alignment: the same sums
        wide = to_dev(np.pad(V, ((0, 0), (0, pad)), constant_values=9))[:, :n_f]
        other, _ = ps.ps2(wide, acc="plain", tile=tile)
        assert np.array_equal(host(other).view(np.uint32), host(c2).view(np.uint32))
    outs = ps.ps2_batched([Vd, Vd], acc="plain", tile=tile)
    assert np.array_equal(host(outs[1][0]).view(np.uint32), host(c2).view(np.uint32))


@pytest.mark.parametrize("tile", [1, 2, 3])
@pytest.mark.parametrize("n_v,n_f", [(3, 5), (40, 33), (131, 65), (140, 130)])
def test_3way(n_v, n_f, tile):
    from paper_1705_08210_amd import ps
    V = _half(n_v, n_f, seed=n_v + n_f)
    announce(f"half 3-way {n_v}x{n_f} tile={tile}")
    c3 = host(ps.ps3(to_dev(V), tile=tile))
    check_rel(c3, oracle.c3_all(V.astype(np.float32)), 1e-5, "c3")


@pytest.mark.parametrize("tile", [1, 2, 3])
def test_non_finite_vector_leaves_the_others(tile):
    from paper_1705_08210_amd import ps
    V = _half(150, 300, seed=8)
    announce(f"half non-finite tile={tile}")
    clean = host(ps.ps2(to_dev(V), tile=tile)[0])
    V[70, 10:20] = np.inf
    V[70, 30] = np.nan
    V[90, 10:15] = np.inf
    got = host(ps.ps2(to_dev(V), tile=tile)[0])
    i, j = np.triu_indices(150, 1)
    others = ~(np.isin(i, (70, 90)) | np.isin(j, (70, 90)))
    idx = colex(i[others], j[others])
    assert np.array_equal(got[idx].view(np.uint32), clean[idx].view(np.uint32))


@pytest.mark.parametrize("tile", [1, 2, 3])
def test_infinities_of_either_sign_leave_the_others(tile):
    """Out-of-domain vectors as rows and as columns of a tile, and inside it:
    2-way, batched and 3-way outputs of the other vectors keep their bits."""
    from paper_1705_08210_amd import ps
    from psx import jslab
    bad = (0, 70, 149)
    V = _half(150, 300, seed=9)
    W = V.copy()
    for v in bad:
        W[v, 10:20] = -np.inf
        W[v, 25] = np.inf
        W[v, 30] = np.nan
        W[v, 40] = -1.0
    W[70] = -np.inf
    announce(f"half infinities tile={tile}")
    Vd, Wd = to_dev(V), to_dev(W)
    i, j = np.triu_indices(150, 1)
    ok = ~(np.isin(i, bad) | np.isin(j, bad))
    idx = colex(i[ok], j[ok])
    for f in (lambda X: ps.ps2(X, tile=tile)[0], lambda X: ps.ps2_batched([X], tile=tile)[0][0]):
        clean, got = host(f(Vd))[idx], host(f(Wd))[idx]
        assert np.array_equal(got.view(np.uint32), clean.view(np.uint32))
    i, j, k = np.array([t for t in itertools.combinations(
        [v for v in range(150) if v not in bad], 3)]).T
    idx = jslab(150, i, j, k)
    clean = host(ps.ps3(Vd, tile=tile))[idx]
    got = host(ps.ps3(Wd, tile=tile))[idx]
    assert np.array_equal(got.view(np.uint32), clean.view(np.uint32))
