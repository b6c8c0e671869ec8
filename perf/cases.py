"""The measured work of the library: what its users have it do, through the
public entry points of ``paper_1705_08210_amd``.

``listed()`` holds the fixed cases; ``draw(rng)`` gives further ones of the
same kinds and ranges.  A case is a dict of plain values:

  kind "ps2"       one 2-way call over all pairs (sums inside, unless
                   "sums": then ``vector_sums`` with its domain check first,
                   as a program does with data it has just read)
  kind "ps3"       one 3-way call over a stage [j0, j1) of middle indices,
                   or over all triples; "given": the sums and pair numerators
                   are the caller's (a later stage of a run); "plan": that
                   stage captured once and replayed
  kind "batched"   a batch of uneven independent 2-way problems, eager or as
                   a captured plan
  kind "campaign"  a whole staged 3-way run that delivers bytes or a
                   thresholded list to host memory

Inputs follow the value distributions of ``workloads``: GWAS-like strengths
(70% exact zeros, exponential nonzeros), half-zero uniforms, exponentials,
integer levels (genotype-like) and binary presence data, drawn on the GPU.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_1705_08210_amd import campaign, ps

DTYPES = {"f32": torch.float32, "f16": torch.float16, "f64": torch.float64,
          "u8": torch.uint8}
BYTES = {"f32": 4, "f16": 2, "f64": 8, "u8": 1}
# a drawn case's size limit: comparisons of the largest listed case of about
# the same time, per storage type and path
LIMIT = {"f32": 1.2e12, "f16": 1.2e12, "f64": 4e11, "u8": 3e12}


def listed():
    return [
        # the smallest call in ordinary use: a few hundred vectors, one panel
        # of fields; launches and latency count
        {"name": "ps2_f32_small", "kind": "ps2", "dtype": "f32", "data": "uniform",
         "n_v": 256, "n_f": 1024, "path": "auto", "levels": 0, "sums": False},
        # many vectors of few fields (385, the paper's sample problem): odd
        # sizes, rows that are not 16-byte aligned, output heavy
        {"name": "ps2_f32_ragged", "kind": "ps2", "dtype": "f32", "data": "gwas",
         "n_v": 6001, "n_f": 385, "path": "auto", "levels": 0, "sums": True},
        # the 2-way run at scale: the bench workload
        {"name": "ps2_f32_large", "kind": "ps2", "dtype": "f32", "data": "gwas",
         "n_v": 16384, "n_f": 20000, "path": "auto", "levels": 0, "sums": True},
        # the same data in FP16 storage, an odd number of vectors
        {"name": "ps2_f16", "kind": "ps2", "dtype": "f16", "data": "gwas",
         "n_v": 8191, "n_f": 20000, "path": "auto", "levels": 0, "sums": True},
        # the paper's double-precision build (5000 fields)
        {"name": "ps2_f64", "kind": "ps2", "dtype": "f64", "data": "gwas",
         "n_v": 4096, "n_f": 5000, "path": "auto", "levels": 0, "sums": True},
        # integer levels 0..3 at scale, the library's own choice of path
        {"name": "ps2_levels", "kind": "ps2", "dtype": "u8", "data": "levels",
         "n_v": 32768, "n_f": 8192, "path": "auto", "levels": 3, "sums": False},
        # binary presence data (the Sorensen case) on its own path, odd sizes
        {"name": "ps2_bits", "kind": "ps2", "dtype": "u8", "data": "binary",
         "n_v": 20001, "n_f": 8190, "path": "bits", "levels": 1, "sums": False},
        # a small 3-way call, everything computed inside: latency
        {"name": "ps3_f32_small", "kind": "ps3", "dtype": "f32", "data": "sparse",
         "n_v": 96, "n_f": 385, "path": "auto", "levels": 0, "j0": 1, "j1": 95,
         "given": False, "plan": False},
        # the full tetrahedron in FP32: the 3-way bench workload
        {"name": "ps3_f32", "kind": "ps3", "dtype": "f32", "data": "sparse",
         "n_v": 1024, "n_f": 4096, "path": "auto", "levels": 0, "j0": 1, "j1": 1023,
         "given": False, "plan": False},
        # the full tetrahedron on integer levels
        {"name": "ps3_levels", "kind": "ps3", "dtype": "u8", "data": "levels",
         "n_v": 1024, "n_f": 4096, "path": "auto", "levels": 3, "j0": 1, "j1": 1023,
         "given": False, "plan": False},
        # a batch of uneven problems (the batched workload's ranges), captured
        # once and replayed
        {"name": "batched_f32", "kind": "batched", "dtype": "f32", "data": "exponential",
         "count": 16, "nv_lo": 500, "nv_hi": 8000, "nf_lo": 1000, "nf_hi": 20000,
         "shape_seed": 0, "plan": True},
        # a staged 3-way run over genotype data, one byte per triple delivered
        # to host memory
        {"name": "campaign_u8", "kind": "campaign", "dtype": "u8", "data": "genotype",
         "n_v": 700, "n_f": 5000, "path": "auto", "levels": 2, "stages": 8, "reduce": "u8"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(c):
    """Comparisons of a case, as a bound on its time."""
    if c["kind"] == "batched":
        return float(sum(f * v * (v - 1) // 2 for v, f in _shapes(c)))
    pairs = c["n_v"] * (c["n_v"] - 1) // 2
    if c["kind"] == "ps2":
        return float(c["n_f"]) * pairs
    triples = (math.comb(c["n_v"], 3) if c["kind"] == "campaign"
               else ps.stage_size(c["n_v"], c["j0"], c["j1"]))
    # an output or a delivered byte of few fields still costs its store
    return max(float(c["n_f"]), 400.0) * (triples + pairs)


def _u8_choice(rng):
    """Integer data: bytes without a level bound, levels, or binary."""
    what = rng.choice(["bytes", "levels", "levels", "bits"])
    if what == "bytes":
        return {"data": "bytes", "path": "auto", "levels": 0}
    if what == "bits":
        return {"data": "binary", "path": "bits", "levels": 1}
    lv = rng.choice([1, 2, 2, 3, 3, 5, 7])
    return {"data": {1: "binary", 2: "genotype", 3: "levels"}.get(lv, "deep"),
            "path": "auto", "levels": lv}


def _float_choice(rng):
    dt = rng.choice(["f32", "f32", "f16", "f64"])
    return {"dtype": dt, "data": rng.choice(["gwas", "sparse", "uniform"]), "path": "auto",
            "levels": 0}


def draw(rng):
    while True:
        kind = rng.choice(["ps2", "ps2", "ps2", "ps3", "ps3", "batched", "campaign"])
        if kind == "ps2":
            c = {"kind": "ps2"}
            c.update(_float_choice(rng) if rng.random() < 0.55
                     else {"dtype": "u8", **_u8_choice(rng)})
            c["n_v"] = _log(rng, 64, 24000 if c["dtype"] == "u8" else 16384)
            c["n_f"] = _log(rng, 200, 20000)
            c["sums"] = rng.random() < 0.5
        elif kind == "ps3":
            c = {"kind": "ps3"}
            c.update(_float_choice(rng) if rng.random() < 0.55
                     else {"dtype": "u8", **_u8_choice(rng)})
            c["n_v"] = _log(rng, 48, 1400)
            c["n_f"] = _log(rng, 200, 12000)
            if rng.random() < 0.5:
                c["j0"], c["j1"] = 1, c["n_v"] - 1
                c["given"] = c["plan"] = False
            else:   # one stage of a longer run
                a = rng.randrange(1, c["n_v"] - 2)
                c["j0"], c["j1"] = a, min(c["n_v"] - 1, a + rng.randrange(1, c["n_v"] // 3 + 2))
                c["given"] = True
                c["plan"] = rng.random() < 0.5
        elif kind == "batched":
            c = {"kind": "batched", "dtype": rng.choice(["f32", "f32", "f16", "u8"]),
                 "count": rng.randrange(4, 33), "nv_lo": _log(rng, 50, 600),
                 "nf_lo": _log(rng, 200, 1500), "shape_seed": rng.randrange(1 << 20),
                 "plan": rng.random() < 0.5}
            c["nv_hi"] = _log(rng, c["nv_lo"] * 4, 8000)
            c["nf_hi"] = _log(rng, c["nf_lo"] * 4, 20000)
            c["data"] = "bytes" if c["dtype"] == "u8" else "exponential"
        else:
            lv = rng.choice([1, 2, 3])
            c = {"kind": "campaign", "dtype": "u8",
                 "data": {1: "binary", 2: "genotype", 3: "levels"}[lv],
                 "n_v": _log(rng, 60, 800), "n_f": _log(rng, 300, 12000), "path": "auto",
                 "levels": lv, "stages": rng.randrange(2, 13),
                 "reduce": rng.choice(["u8", "u8", "threshold"])}
        if _cost(c) <= LIMIT[c["dtype"]]:
            return c


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------

PROBS = {"levels": (0.6, 0.2, 0.15, 0.05), "genotype": (0.55, 0.33, 0.12),
         "binary": (0.7, 0.3)}


def _values(shape, data, dtype, levels, g):
    """One matrix, rows drawn in slabs to bound the temporaries."""
    n_v, n_f = shape
    V = torch.empty(shape, dtype=DTYPES[dtype], device="cuda")
    rows = max(1, (1 << 27) // max(n_f, 1))
    for r in range(0, n_v, rows):
        m = (min(rows, n_v - r), n_f)
        if data == "bytes":
            x = torch.randint(0, 256, m, device="cuda", dtype=torch.uint8, generator=g)
        elif data == "deep":
            x = torch.randint(0, levels + 1, m, device="cuda", dtype=torch.uint8, generator=g)
        elif dtype == "u8":
            u = torch.rand(m, device="cuda", generator=g)
            x = torch.zeros(m, dtype=torch.uint8, device="cuda")
            acc = 0.0
            for p in PROBS[data][:-1]:
                acc += p
                x += (u >= acc).to(torch.uint8)
        else:
            fdt = torch.float64 if dtype == "f64" else torch.float32
            x = torch.rand(m, device="cuda", dtype=fdt, generator=g)
            if data in ("gwas", "exponential"):
                x = -torch.log1p(-x) * (2.0 if data == "gwas" else 1.0)
            zeros = {"gwas": 0.7, "sparse": 0.5}.get(data, 0.0)
            if zeros:
                x *= torch.rand(m, device="cuda", generator=g) >= zeros
        V[r:r + m[0]] = x
    return V


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _shapes(case):
    """(n_v, n_f) of the problems of a batch, log-uniform."""
    g = np.random.default_rng(case["shape_seed"])

    def one(lo, hi):
        return int(math.exp(g.uniform(math.log(lo), math.log(hi))))
    return [(one(case["nv_lo"], case["nv_hi"]), one(case["nf_lo"], case["nf_hi"]))
            for _ in range(case["count"])]


def _inputs(case, seed):
    g = _generator(seed)
    lv = case.get("levels", 0)
    if case["kind"] == "batched":
        return [_values(sh, case["data"], case["dtype"], lv, g) for sh in _shapes(case)]
    return _values((case["n_v"], case["n_f"]), case["data"], case["dtype"], lv, g)


def prepare(case, seed):
    V = _inputs(case, seed)
    st = {"case": case, "V": V}
    kind = case["kind"]
    if kind == "ps3" and case["given"]:
        st["s"], _ = ps.vector_sums(V, want_bad=False)
        _, st["n2"] = ps.ps2(V, s=st["s"], want_c2=False, want_n2=True, path=case["path"],
                             levels=case["levels"])
        if case["plan"]:
            st["plan"] = ps.Plan3(V, s=st["s"], n2=st["n2"], j_begin=case["j0"],
                                  j_end=case["j1"], path=case["path"], levels=case["levels"])
    elif kind == "batched" and case["plan"]:
        st["plan"] = ps.BatchedPlan(V)
    elif kind == "campaign":
        total = campaign.expected_bytes(case["n_v"])
        if case["reduce"] == "u8":
            st["out"] = torch.empty(total, dtype=torch.uint8)
        else:   # about the top hundredth, by the metrics of a few vectors
            head = ps.ps3(V[:48], path=case["path"], levels=case["levels"])
            st["threshold"] = float(torch.quantile(head, 0.99))
            st["cap"] = max(1024, total // 50)
            n = len(campaign.stage_bounds(case["n_v"], case["stages"]))
            st["idx"] = torch.empty(n * st["cap"], dtype=torch.int64)
            st["val"] = torch.empty(n * st["cap"])
    return st


def run(state):
    case, V = state["case"], state["V"]
    kind = case["kind"]
    if kind == "ps2":
        opt = {"path": case["path"], "levels": case["levels"]}
        if not case["sums"]:
            c2, _ = ps.ps2(V, **opt)
            return {"c2": c2}
        s, bad = ps.vector_sums(V)
        c2, _ = ps.ps2(V, s=s, **opt)
        return {"s": s, "bad": bad, "c2": c2}
    if kind == "ps3":
        if case["plan"]:
            return {"c3": state["plan"].run()}
        return {"c3": ps.ps3(V, s=state.get("s"), n2=state.get("n2"), j_begin=case["j0"],
                             j_end=case["j1"], path=case["path"], levels=case["levels"])}
    if kind == "batched":
        outs = state["plan"].run() if case["plan"] else ps.ps2_batched(V)
        return {"c2": [c2 for c2, _, _ in outs]}
    if case["reduce"] == "u8":
        out = state["out"]

        def sink(st):
            out[st.first:st.first + st.size] = st.u8
        campaign.run3(V, case["stages"], sink, reduce="u8", path=case["path"],
                      levels=case["levels"])
        return {"u8": out}
    idx, val, kept, dropped = state["idx"], state["val"], [0], []

    def keep(st):
        o, m = kept[0], len(st.idx)
        idx[o:o + m] = st.idx
        val[o:o + m] = st.val
        kept[0] = o + m
        dropped.append(st.dropped)
    campaign.run3(V, case["stages"], keep, reduce="threshold",
                  threshold=state["threshold"], cap=state["cap"], path=case["path"],
                  levels=case["levels"])
    idx[kept[0]:] = -1
    val[kept[0]:] = 0.0
    return {"idx": idx, "val": val, "kept": kept[0],
            "dropped": torch.tensor(dropped, dtype=torch.int64)}


def work(case):
    """Comparisons (a min and an add each) and the bytes in and out."""
    kind, esz = case["kind"], BYTES[case["dtype"]]
    if kind == "batched":
        sh = _shapes(case)
        return {"bytes": sum(v * f * esz + v * (v - 1) // 2 * 4 for v, f in sh),
                "flops": sum(2 * f * (v * (v - 1) // 2) for v, f in sh)}
    n_v, n_f = case["n_v"], case["n_f"]
    pairs, vin = n_v * (n_v - 1) // 2, n_v * n_f * esz
    if kind == "ps2":
        return {"bytes": vin + pairs * 4 + (n_v * 8 if case["sums"] else 0),
                "flops": 2 * n_f * pairs}
    n2 = 2 * n_f * pairs
    if kind == "ps3":
        t = ps.stage_size(n_v, case["j0"], case["j1"])
        if case["given"]:
            return {"bytes": vin + n_v * 8 + pairs * (8 if case["dtype"] == "f64" else 4) + 4 * t,
                    "flops": 2 * n_f * t}
        return {"bytes": vin + 4 * t, "flops": 2 * n_f * t + n2}
    t = math.comb(n_v, 3)
    out = t if case["reduce"] == "u8" else 12 * max(1024, t // 50)
    return {"bytes": vin + out, "flops": 2 * n_f * t + n2}


# ---------------------------------------------------------------------------
# The definitions of the metric in 64 bits, in plain torch.
# ---------------------------------------------------------------------------

def _min_sums(A, B, levels=0):
    """sum_q min(A[i, q], B[j, q]) in FP64, blocked over rows; for integers
    up to `levels`, min(a, b) = the number of t with a >= t and b >= t."""
    if levels:
        return sum((A >= t).to(torch.float64) @ (B >= t).to(torch.float64).t()
                   for t in range(1, levels + 1))
    out = torch.empty((A.shape[0], B.shape[0]), dtype=torch.float64, device=A.device)
    blk = max(1, (1 << 27) // max(1, B.shape[0] * A.shape[1]))
    if B.shape[0] * A.shape[1] > (1 << 28):   # long rows: block the columns as well
        step = max(1, (1 << 27) // A.shape[1])
        for c in range(0, B.shape[0], step):
            for r in range(A.shape[0]):
                out[r, c:c + step] = torch.minimum(A[r], B[c:c + step]).sum(-1)
        return out
    for r in range(0, A.shape[0], blk):
        out[r:r + blk] = torch.minimum(A[r:r + blk, None, :], B[None]).sum(-1)
    return out


def _ratio(num, den):
    return torch.where(den > 0, num / den.clamp_min(1e-300), torch.zeros_like(num))


def _exact2(V, levels=0):
    """s and colex c2."""
    W = V.to(torch.float64)
    s = W.sum(-1)
    n = V.shape[0]
    cols = []
    rows = max(1, (1 << 27) // max(1, W.shape[1] * 8))
    for j0 in range(1, n, rows):
        j1 = min(n, j0 + rows)
        n2 = _min_sums(W[j0:j1], W[:j1], levels)
        c = _ratio(2.0 * n2, s[j0:j1, None] + s[None, :j1])
        cols += [c[j - j0, :j] for j in range(j0, j1)]
    return s, (torch.cat(cols) if cols else W.new_zeros(0))


def _exact3(V, j0, j1):
    """c3 of the triples of middle indices [j0, j1), j-slab order."""
    W = V.to(torch.float64)
    s = W.sum(-1)
    n2 = _min_sums(W, W)
    out = []
    for j in range(j0, j1):
        n3p = _min_sums(torch.minimum(W[j + 1:], W[j]), W[:j])       # (k, i)
        n3 = n2[:j, j][None] + n2[j + 1:, :j] + n2[j + 1:, j][:, None] - n3p
        d3 = s[:j][None] + s[j] + s[j + 1:][:, None]
        out.append(_ratio(3.0 * n3, 2.0 * d3).reshape(-1))
    return torch.cat(out)


def exact(case, seed):
    if case["kind"] == "campaign":   # bytes and selections: whole numbers
        return None
    # about 1e11 comparisons a second, faster where levels make it a product
    if _cost(case) > (6e12 if case["kind"] == "ps2" and case["levels"] else 1.2e12):
        return None
    V = _inputs(case, seed)
    if case["kind"] == "ps2":
        s, c2 = _exact2(V, case["levels"])
        return {"s": s, "bad": None, "c2": c2} if case["sums"] else {"c2": c2}
    if case["kind"] == "ps3":
        return {"c3": _exact3(V, case["j0"], case["j1"])}
    return {"c2": [_exact2(X)[1] for X in V]}
