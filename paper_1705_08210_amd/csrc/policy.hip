// policy.hip -- launch policy of the tile kernels: the tile configurations,
// the tuning table that overrides the defaults, the accumulation mode and
// field-chunk split, and the path choice.  The kernels' work and traffic
// follow from these choices and from the kernel sources alone.
#include <stdlib.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "ps_internal.h"

namespace ps {

const TileCfg kValuCfgs[kNumValuCfgs] = {
    {8, 8, 32},   // 128 x 128 output tile, 32-word field tile
    {4, 4, 32},   // 64 x 64
    {8, 8, 16},   // 128 x 128, 16-word field tile
};

// ---------------------------------------------------------------------------
// Tuning table.
// ---------------------------------------------------------------------------
struct TuneEntry {
    int32_t dt, way, path;
    int64_t nf_lo, nf_hi, nv_lo, nv_hi;
    int32_t idx;
};
static std::mutex g_tune_mu;
static std::vector<TuneEntry> g_tune;

static int default_cfg(int32_t way, int64_t n_v) {
    // 128x128 output tiles with 16-word field tiles (measured fastest on the
    // large problems: 126 registers, 4 waves per SIMD) once the tiles fill
    // the chip a few times over; 64x64 tiles below that
    if (way == 2) return tri_tiles(n_v, 128) >= 1024 ? 2 : 1;
    return n_v >= 256 ? 2 : 1;
}

int choose_cfg(int32_t dt, int32_t way, int32_t path, int64_t n_f, int64_t n_v,
                      const ps_opts* o) {
    if (o && o->tile > 0) return o->tile - 1;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        for (auto it = g_tune.rbegin(); it != g_tune.rend(); ++it)
            if (it->dt == dt && it->way == way && it->path == path && n_f >= it->nf_lo &&
                n_f < it->nf_hi && n_v >= it->nv_lo && n_v < it->nv_hi)
                return it->idx;
    }
    if (dt == PS_F64) return 1;   // 64x64 tiles: the 128x128 FP64 tiles need >= 256 registers
    return default_cfg(way, n_v);
}

// The 32 x 32 field-split tiles pay while the 64 x 64 tiles (x field chunks)
// leave the chip short of workgroups; past that their double operand traffic
// per output shows, the sooner the more fields a tile sums at a time.  Whole calls,
// us, 64 x 64 / 32 x 32 with four waves:
//   FP32, FP16 (split over field chunks; line 1200 items).  Below: 1001 fields, 1024
//     vectors 48 / 38 (1088 items; FP16 39 / 35); 12000 fields, 256 vectors 74 / 63
//     (750; FP16 49 / 38).  Above: 12000 fields, 384 vectors 99 / 94 (1575), 512
//     121 / 127 (1944); 4096 fields, 700 vectors 78 / 81 (2112); but 1001 fields,
//     1500 vectors 77 / 70 (2100), 2048 113 / 108; 300 fields, 2500 vectors 70 / 65
//   FP64 (never split; line 560 tiles).  Below: 5000 fields, 2048 vectors 1187 / 888
//     (528).  Above: 413 fields, 3000 vectors 167 / 172 (1128), 5830 499 / 603; but
//     5000 fields, 2500 vectors 1496 / 1254 (820), 4096 3131 / 3063, 5000 4425 / 4518
//   uint8 (never split; line 300 tiles below 2048 fields, else 560).  Below: 1001
//     fields, 1500 vectors 39 / 34 (300); 4096 fields, 2048 vectors 137 / 102 (528).
//     Above: 1001 fields, 2048 vectors 49 / 51; but 4096 fields, 3000 203 / 188
// The number of items alone does not separate the two sides: each line lies where no
// depth of fields loses yet, and leaves up to a fifth beyond it to a finer rule.
// Eight waves while all workgroups find a CU of their own (FP64, 4096 fields:
// 700 vectors 119 against 162 with four, 1024 324 against 276).
int small2(int32_t dt, int64_t n_f, int64_t n_v, int cfg, int32_t nchunks, const ps_opts* o) {
    if ((o && o->tile > 0) || cfg != 1) return 0;
    const int64_t limit = dt == PS_F32 || dt == PS_F16 ? 1200
                          : dt == PS_U8 && n_f < 2048  ? 300
                                                       : 560;
    if (tri_tiles(n_v, 64) * nchunks > limit) return 0;
    return tri_tiles(n_v, 32) * nchunks <= 320 ? 8 : 4;
}

// As small2 for the slices.  The rule looks at the whole run (n_v vectors, nchunks
// field chunks), never at the stage, so that a stage sums as the whole run does.
// Unsplit sums take the small tiles up to 208 vectors at any number of fields: the
// 64 x 64 tiles are too few there.  Whole calls, us, 64 x 64 / 32 x 32:
//   FP32 385 fields, 64 vectors 79 / 25, 150 85 / 44, 200 95 / 61, 255 134 / 121;
//   4096 fields, 208 vectors 601 / 499
//   FP64 4000 fields, 208 vectors 903 / 819; uint8 40000 fields, 208 vectors 1848 / 995
// Field chunks bring the 64 x 64 tiles more workgroups, and past the work at which
// they fill the chip the doubled operand traffic of the small ones loses:
//   FP32 (two, three chunks) 6000 fields, 208 vectors 608 / 562; 8192, 180 727 / 706,
//   190 725 / 779; 12000, 130 622 / 530, 160 745 / 692, 170 852 / 871, 208 1139 / 1302
//   FP32 (more) 20000 fields, 110 vectors 660 / 615, 120 653 / 725; 40000 fields, 80
//   737 / 496, 130 1152 / 1583, 208 2967 / 4064
//   FP16 12000 fields, 160 vectors 437 / 406, 208 716 / 742; 40000, 120 595 / 744
// One stage of few slabs is still faster in small tiles beyond the line (12000
// fields, 208 vectors, one slab 548 / 152), at the price of other sums than the run's.
// Eight waves up to 96 vectors, where the tiles leave CUs idle (four / eight waves,
// FP32: 385 fields, 48 vectors 28 / 23, 96 28 / 25, 100 30 / 30, 128 35 / 39; 4000
// fields, 96 vectors 144 / 103, 100 155 / 163, 150 295 / 254, 180 376 / 364).
int small3(int64_t n_f, int64_t n_v, int32_t nchunks, const ps_opts* o) {
    if ((o && o->tile > 0) || n_v > 208) return 0;
    const int64_t limit = nchunks > 3 ? 30000000000 : 55000000000;
    if (nchunks > 1 && n_v * n_v * n_v > limit / n_f) return 0;
    return n_v <= 96 ? 8 : 4;
}

int choose_acc(int64_t n_f, const ps_opts* o) {
    const int a = o ? o->acc : PS_ACC_AUTO;
    if (a == PS_ACC_PLAIN || a == PS_ACC_BLOCKED) return a;
    return n_f > kChunkFields ? PS_ACC_BLOCKED : PS_ACC_PLAIN;
}

// Number of field chunks of the blocked (split) accumulation; 1 = no split.
// kChunkFields is a multiple of every configuration's field-tile depth.
int32_t split_chunks(int32_t dt, int64_t n_f, int acc) {
    if (dt == PS_U8 || dt == PS_F64 || acc != PS_ACC_BLOCKED) return 1;   // exact or FP64
    const int64_t n = ceil_div(n_f, kChunkFields);
    return n > 1 ? (int32_t)n : 1;
}

// Field tiles per chunk: a field tile is bkw words of word_bytes(dt) bytes.
int64_t chunk_tiles(int32_t dt, int cfg) {
    return kChunkFields / ((int64_t)kValuCfgs[cfg].bkw * word_bytes(dt) / elem_size(dt));
}

// Field-chunk plan of a 2-way launch (see Split in ps_internal.h).
Split plan_split(int32_t dt, int64_t n_f, int64_t n_v, int cfg, const ps_opts* o) {
    Split sp{split_chunks(dt, n_f, choose_acc(n_f, o)), chunk_tiles(dt, cfg)};
    const int acc_req = o ? o->acc : PS_ACC_AUTO;
    if (dt == PS_U8 || dt == PS_F64 || acc_req != PS_ACC_AUTO || n_v < 2) return sp;
    const int64_t ftiles = ceil_div(n_f * elem_size(dt), (int64_t)kValuCfgs[cfg].bkw * 4);
    const int64_t tiles = tri_tiles(n_v, kValuCfgs[cfg].bm());
    if (tiles * sp.nchunks >= kMinItems) return sp;
    const int64_t want = std::min(ceil_div(kMinItems, tiles), ftiles / kMinChunkTiles);
    if (want > sp.nchunks) {
        sp.chunk_tiles = ceil_div(ftiles, want);
        sp.nchunks = (int32_t)ceil_div(ftiles, sp.chunk_tiles);
    }
    return sp;
}

// Tile configuration of a batched launch: a tuning entry registered for
// way 0 and the field count of the largest problem, else 128x128 tiles with
// 16-word field tiles.
int batch_cfg(const ps_problem* p, int32_t n, int32_t dt, const ps_opts* o) {
    if (o && o->tile > 0) return o->tile - 1;
    // representative shape: the field count of the largest problem by work
    int64_t best = -1, nf = 0;
    for (int32_t i = 0; i < n; ++i) {
        const int64_t w = p[i].n_f * p[i].n_v * p[i].n_v;
        if (w > best) best = w, nf = p[i].n_f;
    }
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (auto it = g_tune.rbegin(); it != g_tune.rend(); ++it)
        if (it->dt == dt && it->way == 0 && nf >= it->nf_lo && nf < it->nf_hi)
            return it->idx;
    return 2;
}

int64_t max_grid_blocks(int threads, int64_t multiple) {
    static const int64_t env_cap = [] {
        const char* e = getenv("PS_MAX_GRID_BLOCKS");
        const long long v = e ? atoll(e) : 0;
        return v > 0 ? (int64_t)v : (int64_t)0;
    }();
    int64_t cap = (int64_t)0xffffffffu / threads;
    if (env_cap > 0 && env_cap < cap) cap = env_cap;
    cap = cap / multiple * multiple;
    return cap > 0 ? cap : multiple;
}

bool is_mfma(int path) { return path == PS_PATH_MFMA || path == PS_PATH_MFMA_FP4; }

// Whether a matrix-core path can take the shape (exact sums, 32-bit offsets).
static bool mfma_can(int path, int way, int64_t n_f, int64_t n_v, int levels, int wide,
                     int64_t ld) {
    if (path == PS_PATH_MFMA_FP4)
        return bp_exact(n_f, levels) && mfma_row_fits(n_f, levels, 1);
    if (mfma_fused(n_f, levels, 0, wide))
        return mfma_ld_fits(ld) && (way != 3 || mfma3_nv_fits(n_v));
    return (int64_t)levels * n_f < ((int64_t)1 << 31) && mfma_row_fits(n_f, levels, 0);
}

// AUTO keeps triangles of up to this many vectors on a path without a plane
// workspace, so that their size query stays 0 (with the sums given): the VALU path
// with its small tiles, int8 only where the byte sums do not fit 32 bits.  What that
// costs or gains, us, VALU / planes of bits: three levels, 4096 fields, 512 vectors
// 22 / 19, 1023 44 / 20; 12000 fields, 512 52 / 44, 1023 114 / 47; one level, 12000
// fields, 1023 114 / 21; fifteen levels, 12000 fields, 512 52 / 182, 1023 114 / 181;
// 300 fields 14 / 14.  (int8, three levels: 4096 fields, 512 vectors 115; 12000
// fields, 1024 vectors 220: its 256-row tiles leave most of the chip idle.)
static constexpr int64_t kBpMinVectors = 1024;

// A tuned entry for (dt, way, path) covering the shape, or -1.
static int tuned(int32_t dt, int way, int32_t path, int64_t n_f, int64_t n_v) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (auto it = g_tune.rbegin(); it != g_tune.rend(); ++it)
        if (it->dt == dt && it->way == way && it->path == path && n_f >= it->nf_lo &&
            n_f < it->nf_hi && n_v >= it->nv_lo && n_v < it->nv_hi)
            return it->idx;
    return -1;
}

int choose_path(int32_t dt, const ps_opts* o, int way, int64_t n_f, int64_t n_v, int64_t ld) {
    const int p = o ? o->path : PS_PATH_AUTO;
    if (p == PS_PATH_VALU || p == PS_PATH_MFMA || p == PS_PATH_MFMA_FP4 || p == PS_PATH_BITS)
        return p;
    if (dt != PS_U8 || !o || o->levels < 1 || o->levels > 15) return PS_PATH_VALU;
    const int wide = way == 2 && o->tile == 2;   // 3-way: tile 2 picks the slab tiles
    const int t = tuned(dt, way, PS_PATH_AUTO, n_f, n_v);
    if (t == PS_PATH_VALU) return PS_PATH_VALU;
    if ((t == PS_PATH_MFMA || t == PS_PATH_MFMA_FP4) &&
        mfma_can(t, way, n_f, n_v, o->levels, wide, ld))
        return t;
    if (way == 2 && n_v <= kBpMinVectors && 255 * n_f < ((int64_t)1 << 31)) return PS_PATH_VALU;
    if (mfma_can(PS_PATH_MFMA_FP4, way, n_f, n_v, o->levels, wide, ld) &&
        (way == 2 ? n_v > kBpMinVectors : bp3_fits(n_f, n_v, o->levels)))
        return PS_PATH_MFMA_FP4;
    return mfma_can(PS_PATH_MFMA, way, n_f, n_v, o->levels, wide, ld) ? PS_PATH_MFMA
                                                                      : PS_PATH_VALU;
}

int path_without_planes(int32_t dt, const ps_opts* o, int way, int64_t n_f, int64_t n_v,
                        int64_t ld) {
    const int levels = o ? o->levels : 0;
    const int wide = way == 2 && o && o->tile == 2;
    return dt == PS_U8 && mfma_fused(n_f, levels, 0, wide) &&
                   mfma_can(PS_PATH_MFMA, way, n_f, n_v, levels, wide, ld)
               ? PS_PATH_MFMA
               : PS_PATH_VALU;
}

// AUTO reserves the planes of bits themselves.  Path FP4 by name reserves half a
// byte per value and level, four times as much, which programs may have computed
// for themselves, and so does a tuned entry that takes it for a triangle below
// kBpMinVectors.
size_t plane_bytes(const ps_opts* o, int way, int path, int64_t n_f, int64_t n_v) {
    const int levels = o ? o->levels : 0;
    if (path == PS_PATH_MFMA_FP4 && o && o->path == PS_PATH_AUTO &&
        (way == 3 || n_v >= kBpMinVectors))
        return bp_bytes(n_f, n_v, levels);
    return mfma_workspace_bytes(n_f, n_v, levels, path == PS_PATH_MFMA_FP4 ? 1 : 0,
                                way == 2 && o && o->tile == 2);
}

int mfma_group(int64_t n_f, int64_t n_v) {
    const int t = tuned(PS_U8, 2, PS_PATH_MFMA, n_f, n_v);
    return 1 << (t >= 0 ? t : 2);
}

}  // namespace ps

using namespace ps;

extern "C" {

int32_t ps_tile_config(int32_t dtype, int32_t way, int32_t path, int32_t idx, int32_t* bm,
                       int32_t* bn, int32_t* bk) {
    if (elem_size(dtype) == 0 || (way != 2 && way != 3)) return 0;
    if (path == PS_PATH_MFMA && way == 3) {   // tilings of the fused 3-way int8 slices
        if (dtype != PS_U8) return 0;
        if (idx >= 0 && idx < 2) {
            if (bm) *bm = kMfmaTile;
            if (bn) *bn = kMfmaTile;
            if (bk) *bk = 128;
        }
        return 2;
    }
    if (path == PS_PATH_MFMA) {   // tile orders of the 2-way int8 kernel, 256 x 256 x 128
        if (dtype != PS_U8 || way != 2) return 0;
        if (idx >= 0 && idx < kNumMfmaCfgs) {
            if (bm) *bm = kMfmaTile;
            if (bn) *bn = kMfmaTile;
            if (bk) *bk = 128;
        }
        return kNumMfmaCfgs;
    }
    if (is_mfma(path)) return 0;
    if (idx >= 0 && idx < kNumValuCfgs) {
        if (bm) *bm = kValuCfgs[idx].bm();
        if (bn) *bn = kValuCfgs[idx].bn();
        if (bk) *bk = kValuCfgs[idx].bkw * word_bytes(dtype) / elem_size(dtype);  // fields
    }
    return kNumValuCfgs;
}

ps_status ps_tune_register(int32_t dtype, int32_t way, int32_t path, int64_t nf_lo,
                           int64_t nf_hi, int64_t nv_lo, int64_t nv_hi, int32_t idx) {
    if (elem_size(dtype) == 0) return fail(PS_ERR_DTYPE, "unknown dtype %d", dtype);
    if (way != 0 && way != 2 && way != 3)
        return fail(PS_ERR_ARG, "way must be 2, 3 (or 0 for batched)");
    if (path == PS_PATH_AUTO) {   // the path AUTO takes for integer data
        if (dtype != PS_U8 || way == 0)
            return fail(PS_ERR_ARG, "path choices are tuned for PS_U8, way 2 or 3");
        if (idx != PS_PATH_VALU && idx != PS_PATH_MFMA && idx != PS_PATH_MFMA_FP4)
            return fail(PS_ERR_ARG, "path choice %d is not VALU, MFMA or MFMA_FP4", idx);
    } else if (path == PS_PATH_MFMA) {
        if (idx < 0 || idx >= kNumMfmaCfgs)
            return fail(PS_ERR_ARG, "MFMA tile order %d out of range", idx);
    } else if (idx < 0 || idx >= kNumValuCfgs) {
        return fail(PS_ERR_ARG, "tile index %d out of range", idx);
    }
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune.push_back(TuneEntry{dtype, way, path, nf_lo, nf_hi, nv_lo, nv_hi, idx});
    return PS_OK;
}

int32_t ps_path_choice(int32_t dtype, int32_t way, int64_t n_f, int64_t n_v, int64_t ld,
                       const ps_opts* opts) {
    if (elem_size(dtype) == 0 || (way != 2 && way != 3) || n_f < 0 || n_v < 0) return -1;
    return choose_path(dtype, opts, way, n_f, n_v, ld < n_f ? n_f : ld);
}

void ps_tune_clear(void) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune.clear();
}

}  // extern "C"
