"""The 32 x 32 field-split tiles of small problems (mgemm_small.h): every
storage type at the edges of the tile (32 vectors), of a stage (32 or 64 words),
of the field chunks and of the rules that choose them, against the oracle.
Floating sums are at most 20000 terms, each rounding 2^-24 relative: 1e-5 as
everywhere; FP64 data is exact up to the output's rounding (2^-24) and the
sums' 1e-12; integers are bit-exact."""

import numpy as np
import pytest

import oracle
import workloads
from psx import announce, check_exact_f32, check_rel, host, need_gpu, slab_off, to_dev

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "f16": 1e-5, "f64": 2.0 ** -24 + 1e-12}


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _data(kind, n_v, n_f, seed):
    if kind == "u8":
        return np.random.default_rng(seed).integers(0, 256, (n_v, n_f), dtype=np.uint8)
    V = workloads.gwas_like(n_v, n_f, seed=seed)
    V[n_v // 2] = 0.0
    return {"f32": V, "f16": workloads.to_f16(V), "f64": V.astype(np.float64) * 1.1}[kind]


def _check(got, ref, kind, what):
    if kind == "u8":
        check_exact_f32(got, ref, what)
    else:
        check_rel(got, ref, TOL[kind], what)


@pytest.mark.parametrize("kind", ["f32", "f16", "f64", "u8"])
@pytest.mark.parametrize("n_v,n_f", [(2, 1), (31, 5), (32, 64), (33, 127), (65, 257), (96, 1025),
                                     (200, 700), (300, 4100), (64, 9000)])
def test_2way(kind, n_v, n_f):
    from paper_1705_08210_amd import ps
    V = _data(kind, n_v, n_f, seed=n_v + n_f)
    announce(f"small 2-way {kind} {n_v}x{n_f}")
    Vd = to_dev(V)
    c2, n2 = ps.ps2(Vd, want_n2=True)
    ref, rn2 = oracle.c2_all(V, with_n2=True)
    _check(host(c2), ref, kind, "c2")
    if kind == "u8":
        assert np.array_equal(host(n2).astype(np.float64), rn2)
    # given sums, and rows of another alignment: the same field order, the same bits
    s, _ = ps.vector_sums(Vd)
    given, _ = ps.ps2(Vd, s=s)
    wide = to_dev(np.pad(V, ((0, 0), (0, 3)), constant_values=7))[:, :n_f]
    pitch, _ = ps.ps2(wide)
    for other in (given, pitch):
        assert np.array_equal(host(other).view(np.uint32), host(c2).view(np.uint32))


@pytest.mark.parametrize("kind,n_v,n_f", [("f32", 1090, 1001), ("f32", 1100, 1001),
                                          ("f64", 2112, 40), ("f64", 2113, 40),
                                          ("u8", 1536, 100), ("u8", 1537, 100)])
def test_2way_rule_edges(kind, n_v, n_f):
    """The last size of the small tiles and the first of the 64 x 64 ones; the
    shards of a call together give its bits on both sides."""
    import torch
    from paper_1705_08210_amd import ps
    V = _data(kind, n_v, n_f, seed=3)
    announce(f"small rule {kind} {n_v}x{n_f}")
    Vd = to_dev(V)
    full, _ = ps.ps2(Vd)
    _check(host(full), oracle.c2_all(V), kind, "c2")
    union = torch.full_like(full, float("nan"))
    for k in range(3):
        ps.ps2_shard(Vd, k, 3, c2=union)
    assert np.array_equal(host(union).view(np.uint32), host(full).view(np.uint32))


@pytest.mark.parametrize("kind", ["f32", "f16", "f64", "u8"])
@pytest.mark.parametrize("n_v,n_f", [(3, 1), (5, 40), (34, 65), (96, 385), (97, 130), (130, 5000),
                                     (208, 70), (209, 70)])
def test_3way(kind, n_v, n_f):
    from paper_1705_08210_amd import ps
    V = _data(kind, n_v, n_f, seed=n_v + 3 * n_f)
    announce(f"small 3-way {kind} {n_v}x{n_f}")
    Vd = to_dev(V)
    full = host(ps.ps3(Vd))
    _check(full, oracle.c3_all(V), kind, "c3")
    # stages concatenate to the same bits, the numerators given
    s, _ = ps.vector_sums(Vd)
    _, n2 = ps.ps2(Vd, s=s, want_c2=False, want_n2=True)
    cuts = sorted({1, 2, 2 * n_v // 5, n_v // 2, n_v - 1} & set(range(1, n_v)))
    parts = [host(ps.ps3(Vd, s=s, n2=n2, j_begin=a, j_end=b)) for a, b in zip(cuts, cuts[1:])]
    assert sum(p.size for p in parts) == int(slab_off(n_v, n_v - 1))
    assert np.array_equal(np.concatenate(parts).view(np.uint32), full.view(np.uint32))


@pytest.mark.parametrize("kind", ["f32", "f16"])
@pytest.mark.parametrize("n_v,n_f", [(120, 17361), (120, 17362), (208, 6111), (208, 6112)])
def test_3way_rule_edges_of_split_sums(kind, n_v, n_f):
    """The last field counts of the small tiles (more than three field chunks, and
    up to three) and the first of the 64 x 64 ones; stages keep the run's bits."""
    import librules
    from paper_1705_08210_amd import ps
    small = librules.small3(n_f, n_v, -(-n_f // 4096)) > 0
    assert small == (n_f in (17361, 6111))
    V = _data(kind, n_v, n_f, seed=n_f)
    announce(f"small 3-way rule {kind} {n_v}x{n_f}")
    Vd = to_dev(V)
    full = host(ps.ps3(Vd))
    _check(full, oracle.c3_all(V), kind, "c3")
    s, _ = ps.vector_sums(Vd)
    _, n2 = ps.ps2(Vd, s=s, want_c2=False, want_n2=True)
    cuts = [1, 2, n_v // 2, n_v - 1]
    parts = [host(ps.ps3(Vd, s=s, n2=n2, j_begin=a, j_end=b)) for a, b in zip(cuts, cuts[1:])]
    assert np.array_equal(np.concatenate(parts).view(np.uint32), full.view(np.uint32))


RULE_N_F = {"f32": 1001, "f16": 1001, "f64": 40, "u8": 100}


def _rule_edges(kind):
    """Sizes around the lines of the 2-way rule: eight waves to four, and the last of
    the small tiles to the first of the 64 x 64 ones."""
    import librules
    import torch
    dt = {"f32": torch.float32, "f16": torch.float16, "f64": torch.float64,
          "u8": torch.uint8}[kind]

    def waves(n_v):
        return librules.pairs_2way(dt, RULE_N_F[kind], n_v)[0]
    eight = max(n for n in range(2, 1200) if waves(n) == 8)
    last = max(n for n in range(eight, 4000) if waves(n))
    assert [waves(n) for n in (eight, eight + 1, last, last + 1)] == [8, 4, 4, 0]
    chunks = librules.pairs_2way(dt, RULE_N_F[kind], last)[1]
    assert (chunks > 1) == (kind in ("f32", "f16"))   # the sums ride along, or not
    return [eight, eight + 1, last, last + 1]


@pytest.mark.parametrize("kind", ["f32", "f16", "f64", "u8"])
@pytest.mark.parametrize("k", range(4))
def test_2way_at_the_lines_of_the_rule(kind, k):
    """Against the oracle, the sums inside; the shards of a call together write its
    bits once, whether the sums are given or not."""
    import torch
    from paper_1705_08210_amd import ps
    n_v = _rule_edges(kind)[k]
    V = _data(kind, n_v, RULE_N_F[kind], seed=n_v)
    announce(f"small rule line {kind} {n_v}x{RULE_N_F[kind]}")
    Vd = to_dev(V)
    full, n2 = ps.ps2(Vd, want_n2=True)
    _check(host(full), oracle.c2_all(V), kind, "c2")
    s, _ = ps.vector_sums(Vd)
    for given in (None, s):
        union, nun = torch.full_like(full, float("nan")), torch.full_like(n2, -1)
        for r in range(3):
            before = union.clone()
            ps.ps2_shard(Vd, r, 3, s=given, c2=union, n2=nun)
            written = torch.isnan(before)
            assert bool((union[~written] == before[~written]).all())
        assert np.array_equal(host(union).view(np.uint32), host(full).view(np.uint32))
        assert bool((nun == n2).all())
