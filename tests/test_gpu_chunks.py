"""Field-split sums whose last chunk is short, at tile counts around the line
from which every XCD takes all chunks of its share of the tiles (256 tiles),
against 64-bit references."""

import math

import pytest
import torch

from paper_1705_08210_amd import ps

pytestmark = pytest.mark.gpu

N_F = 4100   # chunks of 4096 and 4 fields
TOL = N_F * 2.0 ** -24   # every rounded FP32 addition at its worst


# 64 x 64 tiles: 253 (the chunk-major list), 276 (not a multiple of 8), 351, 528 (66 x 8)
@pytest.mark.parametrize("n_v", [1408, 1409, 1664, 2001])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("nshards", [1, 2])
def test_split_pairs(n_v, dtype, nshards):
    g = torch.Generator(device="cuda").manual_seed(n_v)
    V = torch.rand((n_v, N_F), device="cuda", generator=g).to(dtype)
    c2 = torch.full((n_v * (n_v - 1) // 2,), -1.0, device="cuda")
    n2 = torch.full_like(c2, -1.0)
    for r in range(nshards):
        if nshards == 1:
            ps.ps2(V, c2=c2, n2=n2, tile=2, acc="blocked")
        else:
            ps.ps2_shard(V, r, nshards, c2=c2, n2=n2, tile=2, acc="blocked")
    assert bool((n2 >= 0).all()) and bool((c2 >= 0).all())
    W = V.double()
    for j in (1, 63, 64, 65, n_v // 2, n_v - 65, n_v - 1):
        ref = torch.minimum(W[j], W[:j]).sum(-1)
        got = n2[j * (j - 1) // 2: j * (j - 1) // 2 + j].double()
        assert bool(((got - ref).abs() <= TOL * ref).all())


# 64 x 64 tiles of pairs against vectors: below 256 of them, and above
@pytest.mark.parametrize("n_v", [40, 150, 171])
def test_split_triples(n_v):
    g = torch.Generator(device="cuda").manual_seed(n_v)
    V = torch.rand((n_v, N_F), device="cuda", generator=g)
    got = ps.ps3(V, tile=2, acc="blocked").double()
    W = V.double()
    s = W.sum(-1)
    assert got.numel() == math.comb(n_v, 3) and bool((got > 0).all())
    for j in (1, 2, n_v // 3, n_v // 2, n_v - 2):
        # slabs of the middle index j; in a slab k, then i fastest
        pos = sum(m * (n_v - 1 - m) for m in range(1, j))
        x = torch.minimum(W[j], W[:j])
        nij = x.sum(-1)
        for k in range(j + 1, n_v):
            nik = torch.minimum(W[:j], W[k]).sum(-1)
            njk = torch.minimum(W[j], W[k]).sum()
            n3p = torch.minimum(x, W[k]).sum(-1)
            ref = 1.5 * (nij + nik + njk - n3p) / (s[:j] + s[j] + s[k])
            # four sums of relative error TOL, each at most the numerator
            assert bool(((got[pos:pos + j] - ref).abs() <= 5 * TOL * ref).all())
            pos += j
