"""Path AUTO on integer levels where there is no room for its planes of bits: a
workspace of the size that the paths without planes need is accepted, by the C
ABI and by the binding, and the results are the same bits."""

import ctypes

import numpy as np
import pytest
import torch

import workloads
from psx import announce, host, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _levels(n_v, n_f, L, seed):
    return to_dev(workloads.levels(n_v, n_f, seed=seed, probs=np.full(L + 1, 1.0 / (L + 1))))


def _same(a, b):
    return np.array_equal(host(a).view(np.uint32), host(b).view(np.uint32))


@pytest.mark.parametrize("L", [1, 3, 12])
@pytest.mark.parametrize("tile", [0, 2])
def test_2way_workspace_without_planes(L, tile):
    from paper_1705_08210_amd import ps
    n_v, n_f = 1100, 333
    V = _levels(n_v, n_f, L, seed=L)
    s, _ = ps.vector_sums(V)
    ref, _ = ps.ps2(V, path="valu")
    o = ps._opts(levels=L, tile=tile)
    full = ps.lib.ps2_workspace_size(2, n_f, n_v, 1, ctypes.byref(o))
    assert full > 0
    ws = torch.empty(full, dtype=torch.uint8, device=V.device)
    st = torch.cuda.current_stream().cuda_stream
    for nbytes, given, room in ((0, True, None), (full - 1, True, ws), (full, True, ws),
                                (8960, False, ws)):   # 8960: the sums alone
        announce(f"2-way levels={L} tile={tile} workspace {nbytes}, sums given {given}")
        c2 = torch.full_like(ref, float("nan"))
        assert ps.lib.ps2_compute(V.data_ptr(), 2, n_f, n_v, n_f, ps._ptr(s) if given else None,
                                  c2.data_ptr(), None, ps._ptr(room), nbytes, ctypes.byref(o),
                                  st) == 0
        assert _same(c2, ref)


@pytest.mark.parametrize("L", [2, 11])
def test_3way_workspace_without_planes(L):
    from paper_1705_08210_amd import ps
    n_v, n_f = 150, 270
    V = _levels(n_v, n_f, L, seed=L)
    ref = ps.ps3(V, path="valu")
    o, o1 = ps._opts(levels=L), ps._opts(levels=L, path="valu")
    size = [ps.lib.ps3_workspace_size(2, n_f, n_v, 0, 0, 1, n_v - 1, ctypes.byref(q))
            for q in (o, o1)]
    assert size[0] > size[1]
    ws = torch.empty(size[0], dtype=torch.uint8, device=V.device)
    st = torch.cuda.current_stream().cuda_stream
    for nbytes in size:
        announce(f"3-way levels={L} workspace {nbytes}")
        c3 = torch.full_like(ref, float("nan"))
        assert ps.lib.ps3_compute(V.data_ptr(), 2, n_f, n_v, n_f, None, None, 1, n_v - 1,
                                  c3.data_ptr(), ws.data_ptr(), nbytes, ctypes.byref(o), st) == 0
        assert _same(c3, ref)
    assert ps.lib.ps3_compute(V.data_ptr(), 2, n_f, n_v, n_f, None, None, 1, n_v - 1,
                              c3.data_ptr(), ws.data_ptr(), size[1] - 256, ctypes.byref(o),
                              st) == 3   # PS_ERR_WORKSPACE


def test_binding_without_memory_for_planes(monkeypatch):
    from paper_1705_08210_amd import ps
    V = _levels(1100, 400, 3, seed=5)
    W = V[:140]
    two, _ = ps.ps2(V, path="valu")
    three = ps.ps3(W, path="valu")
    plain, asked = ps._workspace, []

    def scarce(nbytes, device):
        asked.append(nbytes)
        if len(asked) % 2:
            raise torch.OutOfMemoryError("no room")
        return plain(nbytes, device)
    monkeypatch.setattr(ps, "_workspace", scarce)
    announce("binding without memory for planes")
    assert _same(ps.ps2(V, levels=3)[0], two)
    assert _same(ps.ps3(W, levels=3), three)
    plan = ps.Plan3(W, levels=3)
    assert _same(plan.run(), three)
    plan.close()
    assert len(asked) == 6 and all(b < a for a, b in zip(asked[::2], asked[1::2]))
    for kw in (dict(path="mfma_fp4", levels=3), dict(path="valu")):   # no other path to take
        with pytest.raises(torch.OutOfMemoryError):
            ps.ps3(W, **kw)
        asked.append(0)


def test_noalloc_planes_past_the_static_scratch():
    from paper_1705_08210_amd import ps
    n_v, n_f = 300, 400_000       # planes of bits: 300 x 3 x 50 KB
    V = _levels(n_v, n_f, 3, seed=6)
    s, _ = ps.vector_sums(V)
    _, n2 = ps.ps2(V, s=s, want_c2=False, want_n2=True, path="valu")
    o = ps._opts(levels=3)
    assert ps.lib.ps3_workspace_size(2, n_f, n_v, 1, 1, 100, 102, ctypes.byref(o)) > \
        ps.noalloc_scratch_bytes()
    c3 = torch.empty(ps.stage_size(n_v, 100, 102), device=V.device)
    announce("noalloc, planes past the static scratch")
    ps.ps3_noalloc(V, c3, s=s, n2=n2, j_begin=100, j_end=102, levels=3)
    assert _same(c3, ps.ps3(V, s=s, n2=n2, j_begin=100, j_end=102, path="valu"))
