"""As test_gpu_multilaunch, for the launches whose work items carry more than a
tile: the small tiles with the sums of the vectors appended, the small slices, the
planes of bits (2-way and slices), and split sums, whose tiles are dealt to the
XCDs chunk after chunk.  A child process capped at 64 blocks a launch must give
this process's bits."""

import os
import subprocess
import sys
import textwrap

import numpy as np
import pytest

from psx import announce, need_gpu

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CASES = textwrap.dedent("""
    import sys, numpy as np, torch
    sys.path.insert(0, {root!r})
    import workloads
    from paper_1705_08210_amd import ps
    def dev(V):
        return torch.from_numpy(np.ascontiguousarray(V)).cuda()
    out = {{}}
    F = workloads.sparse_uniform(400, 1001, seed=90)
    for name, V in (("f32", F), ("f16", workloads.to_f16(F)), ("f64", F.astype(np.float64)),
                    ("u8", workloads.levels(400, 1001, seed=91))):
        W = dev(V)
        out["small2_" + name] = ps.ps2(W)[0]
        out["small3_" + name] = ps.ps3(W[:120])
    G = dev(workloads.sparse_uniform(2001, 4100, seed=92))   # 528 tiles x 2 chunks
    out["chunks2"] = ps.ps2(G, acc="blocked", tile=2)[0]
    out["chunks3"] = ps.ps3(G[:175], acc="blocked", tile=2)
    H = G[:1409].half()                                      # 276 tiles, not a multiple of 8
    out["chunks2_f16"] = ps.ps2(H, acc="blocked", tile=2)[0]
    B = dev(workloads.binary(1500, 700, seed=93, dtype=np.uint8))
    out["bits2"] = ps.ps2(B, path="bits", levels=1)[0]
    out["bits3"] = ps.ps3(B[:300], path="bits", levels=1)
    L = dev(workloads.levels(2100, 300, seed=94))
    out["planes2"] = ps.ps2(L, levels=3)[0]                  # 128 x 128 tiles
    out["planes3"] = ps.ps3(L[:300], levels=3)
    torch.cuda.synchronize()
    np.savez({path!r}, **{{k: v.cpu().numpy() for k, v in out.items()}})
""")


def test_multi_launch_equals_single_launch(tmp_path):
    need_gpu()
    path = str(tmp_path / "out.npz")
    announce("multi-launch child process (PS_MAX_GRID_BLOCKS=64), small tiles, planes, chunks")
    env = dict(os.environ, PS_MAX_GRID_BLOCKS="64")
    r = subprocess.run([sys.executable, "-c", CASES.format(root=ROOT, path=path)], env=env,
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    child = np.load(path)
    announce("multi-launch: same cases in this process")
    single_path = str(tmp_path / "single.npz")
    exec(CASES.format(root=ROOT, path=single_path), {})
    single = np.load(single_path)
    assert sorted(child.files) == sorted(single.files) and len(single.files) == 15
    for k in child.files:
        assert np.array_equal(child[k].view(np.uint32), single[k].view(np.uint32)), k
