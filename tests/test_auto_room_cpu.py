"""What path AUTO reserves for the planes of bits of integer levels: the planes
themselves, one bit per value and level, and nothing below the sizes from which
it takes them."""

import ctypes

import pytest

ps = pytest.importorskip("paper_1705_08210_amd.ps")


def _opts(**kw):
    return ctypes.byref(ps._opts(**kw))


def _planes(n_v, n_f, levels):
    """n_v rows of `levels` planes of 32-bit words, in whole 16-byte chunks."""
    words = -(-levels * -(-n_f // 32) // 4) * 4
    return -(-n_v * words * 4 // 256) * 256


@pytest.mark.parametrize("n_v,n_f,levels", [(32768, 8192, 3), (1025, 100, 1), (2000, 4097, 15),
                                            (5000, 1, 7), (1400, 12000, 2), (1024, 4096, 3)])
def test_2way(n_v, n_f, levels):
    assert ps.path_choice(ps.torch.uint8, 2, n_f, n_v, levels=levels) == ps.PATH["mfma_fp4"]
    assert ps.lib.ps2_workspace_size(2, n_f, n_v, 1, _opts(levels=levels)) == \
        _planes(n_v, n_f, levels)


def test_2way_small_triangles_reserve_nothing():
    for n_v in (2, 300, 1023):
        assert ps.lib.ps2_workspace_size(2, 4096, n_v, 1, _opts(levels=3)) == 0


@pytest.mark.parametrize("n_v,n_f,levels", [(1024, 4096, 3), (50, 100, 1), (700, 12000, 15)])
def test_3way(n_v, n_f, levels):
    def size(path):
        return ps.lib.ps3_workspace_size(2, n_f, n_v, 1, 1, 1, n_v - 1,
                                         _opts(path=path, levels=levels))
    assert size("auto") - size("valu") == _planes(n_v, n_f, levels)
