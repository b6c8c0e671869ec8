// mgemm_small.h -- the VALU min-product for problems whose 64 x 64 tiles would
// leave most of the chip idle.
//
// What bounds a small call is the serial chain of one tile: load, stage,
// barrier, 32 words of arithmetic by lone waves, per field tile.  Here a
// workgroup computes a 32 x 32 tile (four times as many workgroups) in stages of
// 8 words per wave that its four or eight waves share (every wave over the whole
// 32 x 32 outputs); stages are loaded kSmAhead ahead into
// registers and staged into alternating LDS buffers (one barrier per stage), and
// the partial sums of an output are added through LDS at the end.  A
// pair's sum thus has a fixed order that does not depend on its tile or the
// 3-way stage.
//
// 3-way tiles are enumerated as row tiles x the most column tiles any row tile
// has (a workgroup past its row's last tile returns at once), so no prefix
// launch is needed, and Eq. 1 runs here: no finish launch either.
//
// Whole calls: 256 vectors x 1024 fields FP32, 26.0 -> 15.3 us (three launches -> two); 96 x 385
// FP32 3-way, 110 -> 24.6 us (seven launches -> three).
#pragma once

#include "sums.h"

namespace ps {

constexpr int kSmB = 32;         // tile rows and columns
constexpr int kSmMine = 8;       // words of a stage per wave: NW waves, 8 NW words
constexpr int kSmAhead = 4;      // stages in flight (even)
constexpr int kSmLd = kSmB + 4;  // LDS pitch of a word's row (words)

// Words of LDS: two buffers of both operands, reused for the partial sums.
template <int DT, int NW>
constexpr int sm_lds_words() {
    constexpr int stage = 2 * 2 * kSmMine * NW * kSmLd;
    constexpr int red = NW * kSmB * kSmB * (int)sizeof(typename Ops<DT>::Acc) /
                        (int)sizeof(typename Ops<DT>::Word);
    return stage > red ? stage : red;
}

// This thread's 16-byte chunks of one operand's stage: row t % 32, chunks t / 32
// (+ 2 NW): word-major in LDS, S[w * kSmLd + row].  With XJ each chunk is min-ed
// with the same chunk of a second row, when it is stored (so that the loads of
// later stages are not waited for).
template <int DT, int NW, bool XJ, bool VEC>
struct SmChunks {
    using Word = typename Ops<DT>::Word;
    static constexpr int kWpc = 16 / (int)sizeof(Word);
    static constexpr int kChunks = kSmB * (kSmMine * NW / kWpc);
    static constexpr int kCh = kChunks / (64 * NW);
    static_assert(kCh * 64 * NW == kChunks, "stage split");
    uint4 v[kCh], x[XJ ? kCh : 1];
    // rows at byte offsets ro (< 0: none, zeros) and, with XJ, xo; kb: the stage's
    // first byte; fields end at byte `end`
    __device__ __forceinline__ void load(const char* V, int64_t ro, int64_t xo, int64_t kb,
                                         int64_t end) {
        using S = Stager<kSmB, 32, Word>;
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            const int64_t b0 = kb + (threadIdx.x / kSmB + c * (2 * NW)) * 16;
            v[c] = make_uint4(0, 0, 0, 0);
            if constexpr (XJ) x[c] = v[c];
            if (ro >= 0) {
                v[c] = S::template load_chunk<Ops<DT>::kEsz, VEC>(V + ro, b0, end);
                if constexpr (XJ) x[c] = S::template load_chunk<Ops<DT>::kEsz, VEC>(V + xo, b0, end);
            }
        }
    }
    __device__ __forceinline__ void store(Word* S) const {
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            uint4 r = v[c];
            if constexpr (XJ) r = xmin_chunk<DT>(r, x[c]);
            const int ch = threadIdx.x / kSmB + c * (2 * NW);
            Word* w = S + ch * kWpc * kSmLd + threadIdx.x % kSmB;
            if constexpr (sizeof(Word) == 8) {
                w[0] = ((uint64_t)r.y << 32) | r.x;
                w[kSmLd] = ((uint64_t)r.w << 32) | r.z;
            } else {
                w[0] = r.x;
                w[kSmLd] = r.y;
                w[2 * kSmLd] = r.z;
                w[3 * kSmLd] = r.w;
            }
        }
    }
};

// The 32 x 32 sums over bytes [b0, b1) of the rows; A rows at offset ao (XJ: min
// with the row at xo), B rows at bo, one row per thread as in SmChunks.  Threads
// t < 256 receive out[0..3], four consecutive entries along the fast side
// (fastrow: rows 4 (t % 8) .., column t / 8; else columns 4 (t % 8) .., row t / 8).
template <int DT, int NW, bool XJ, bool VEC>
__device__ __forceinline__ void sm_tile(const char* V, int64_t ao, int64_t xo, int64_t bo,
                                        int64_t b0, int64_t b1, bool fastrow,
                                        typename Ops<DT>::Word* lds,
                                        typename Ops<DT>::Acc (&out)[4]) {
    using Word = typename Ops<DT>::Word;
    using Acc = typename Ops<DT>::Acc;
    constexpr int64_t kStage = kSmMine * NW * (int64_t)sizeof(Word);
    constexpr int kBuf = kSmMine * NW * kSmLd;
    constexpr int kV = (int)sizeof(Word) / 4;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int lx = lane % 8, ly = lane / 8;
    Acc acc[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = Acc(0);
    SmChunks<DT, NW, XJ, VEC> sa[kSmAhead];
    SmChunks<DT, NW, false, VEC> sb[kSmAhead];
#pragma unroll
    for (int u = 0; u < kSmAhead; ++u)
        if (b0 + u * kStage < b1) {
            sa[u].load(V, ao, xo, b0 + u * kStage, b1);
            sb[u].load(V, bo, 0, b0 + u * kStage, b1);
        }
    for (int64_t kb = b0; kb < b1; kb += kSmAhead * kStage) {
#pragma unroll
        for (int u = 0; u < kSmAhead; ++u) {
            const int64_t k = kb + u * kStage;
            if (k >= b1) break;
            Word* As = lds + (u & 1) * 2 * kBuf;
            Word* Bs = As + kBuf;
            sa[u].store(As);
            sb[u].store(Bs);
            if (k + kSmAhead * kStage < b1) {
                sa[u].load(V, ao, xo, k + kSmAhead * kStage, b1);
                sb[u].load(V, bo, 0, k + kSmAhead * kStage, b1);
            }
            __syncthreads();   // this stage is in LDS; everyone is done with the one before
#pragma unroll
            for (int w = 0; w < kSmMine; ++w) {
                const int ww = wave * kSmMine + w;
                Word a[4], b[4];
#pragma unroll
                for (int h = 0; h < kV; ++h) {
                    ((uint4*)a)[h] = ((const uint4*)&As[ww * kSmLd + lx * 4])[h];
                    ((uint4*)b)[h] = ((const uint4*)&Bs[ww * kSmLd + ly * 4])[h];
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[r][c] = Ops<DT>::step(acc[r][c], a[r], b[c]);
            }
        }
    }
    __syncthreads();
    // partial sums [wave][slow][fast]
    Acc* red = (Acc*)lds;
    const int slow0 = (fastrow ? ly : lx) * 4, fast0 = (fastrow ? lx : ly) * 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        Acc* p = red + (wave * kSmB + slow0 + s) * kSmB + fast0;
#pragma unroll
        for (int f = 0; f < 4; ++f) p[f] = fastrow ? acc[f][s] : acc[s][f];
    }
    __syncthreads();
    if (threadIdx.x >= 256) return;
    const Acc* p = red + threadIdx.x * 4;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        out[f] = p[f];
#pragma unroll
        for (int w = 1; w < NW; ++w) out[f] += p[f + w * kSmB * kSmB];
    }
}

// Bytes [b0, b1) of a launch's field chunk: chunk_tiles field tiles of 32 words
// (the 64 x 64 configuration's), or all of the row.
template <int DT>
__device__ __forceinline__ void sm_range(int64_t nbytes, int32_t nchunks, int64_t chunk_tiles,
                                         int64_t chunk, int64_t& b0, int64_t& b1) {
    const int64_t len = chunk_tiles * 32 * (int64_t)sizeof(typename Ops<DT>::Word);
    b0 = nchunks > 1 ? chunk * len : 0;
    b1 = nchunks > 1 && b0 + len < nbytes ? b0 + len : nbytes;
}

// 2-way: work items (field chunk, 32 x 32 tile of the upper triangle), then,
// with a.s_out, blocks of NW vectors to sum (nothing in this launch reads
// the sums then: raw chunk sums, or numerators alone).
template <int DT, int NW, bool VEC>
__global__ __launch_bounds__(64 * NW, 2) void ps_sm2_kernel(Mg2Call a, int64_t ntiles,
                                                             int64_t item0) {
    using Word = typename Ops<DT>::Word;
    using Acc = typename Ops<DT>::Acc;
    constexpr int ESZ = Ops<DT>::kEsz;
    __shared__ __attribute__((aligned(16))) Word lds[sm_lds_words<DT, NW>()];
    const int64_t ldb = a.ld * ESZ, nbytes = a.n_f * ESZ;
    const char* V = (const char*)a.V;
    const int64_t w = item0 + blockIdx.x, nitems = ntiles * a.nchunks;
    if (w >= nitems) {
        const int64_t i = (w - nitems) * NW + threadIdx.x / 64;
        if (a.s_out && i < a.n_v) {
            int bad;
            const double x = wave_row_sum<DT>(V + i * ldb, a.n_f, VEC, bad);
            if (threadIdx.x % 64 == 0) a.s_out[i] = x;
        }
        return;
    }
    const int64_t chunk = w / ntiles;
    int64_t bi, bj;
    tri_decode(w % ntiles, bi, bj);
    // a tile shard is counted in the configuration's 64 x 64 tiles
    if (a.nshards > 1 && ((bj / 2) * (bj / 2 + 1) / 2 + bi / 2) % a.nshards != a.shard0) return;
    const int64_t row0 = bi * kSmB, col0 = bj * kSmB;
    const int64_t ra = row0 + threadIdx.x % kSmB, rb = col0 + threadIdx.x % kSmB;
    int64_t b0, b1;
    sm_range<DT>(nbytes, a.nchunks, a.chunk_tiles, chunk, b0, b1);
    Acc out[4];
    sm_tile<DT, NW, false, VEC>(V, ra < a.n_v ? ra * ldb : -1, 0, rb < a.n_v ? rb * ldb : -1, b0, b1,
                            true, lds, out);
    if (threadIdx.x >= 256) return;
    const int64_t j = col0 + threadIdx.x / 8, i0 = row0 + 4 * (threadIdx.x % 8);
    if (j >= a.n_v) return;
    const int64_t base = j * (j - 1) / 2;
    if constexpr (DT != PS_F64) {
        if (a.nchunks > 1) {
            uint32_t* dst = (uint32_t*)a.partial + chunk * (a.n_v * (a.n_v - 1) / 2) + base;
#pragma unroll
            for (int f = 0; f < 4; ++f)
                if (i0 + f < j) dst[i0 + f] = __builtin_bit_cast(uint32_t, out[f]);
            return;
        }
    }
    const bool sums = !a.s_out;   // with s_out: numerators that need no sums
    const double sj = sums ? a.s[j] : 0.0;
#pragma unroll
    for (int f = 0; f < 4; ++f)
        if (i0 + f < j)
            store_pair<DT>(out[f], sums ? a.s[i0 + f] : 0.0, sj, base + i0 + f, a.c2, a.n2);
}

// One triple (Eq. 1, Section 2.2) from its slice sum, with the pair (x, y) that
// was staged and the single vector z: nxy their numerator.
template <int DT>
__device__ __forceinline__ void sm3_store(const Mg3Launch& a, typename Ops<DT>::Acc acc,
                                          int64_t i, int64_t j, int64_t k, PairT<DT> nxy,
                                          double sz, int64_t idx, int64_t chunk, int64_t stage) {
    if (DT != PS_F64 && DT != PS_U8 && a.nchunks > 1) {
        a.partial[chunk * stage + idx] = (float)acc;   // FP32 chunk sums, finished later
        return;
    }
    const PairT<DT>* N2 = (const PairT<DT>*)a.n2;
    const double nij = (double)N2[j * (j - 1) / 2 + i], nik = (double)N2[k * (k - 1) / 2 + i],
                 njk = (double)N2[k * (k - 1) / 2 + j];
    double n3p;
    if constexpr (DT == PS_U8) n3p = (double)(int32_t)u8_min_sum(acc, nxy, sz);
    else n3p = (double)acc;
    const double n3 = ((nij + nik) + njk) - n3p;
    const double d3 = (a.s[i] + a.s[j]) + a.s[k];
    a.c3[idx] = d3 > 0.0 ? (float)((3.0 * n3) / (2.0 * d3)) : 0.0f;
}

// Row and column tiles of the two parts of the split tiling (split3).
struct Sm3Grid {
    int64_t rows0, cols0, rows1, cols1;
    int64_t items() const { return rows0 * cols0 + rows1 * cols1; }
};

// 3-way: work items (field chunk, row tile of 32 pairs, column tile of 32
// vectors).  Part 0: colex pairs (i, j) of the slabs below js against k from
// the row tile's smallest j + 1; part 1: lex pairs (j, k) of the others
// against i.
template <int DT, int NW, bool VEC>
__global__ __launch_bounds__(64 * NW, 2) void ps_sm3_kernel(Mg3Launch a, Sm3Grid g, int64_t nitems,
                                                     int64_t item0) {
    using Word = typename Ops<DT>::Word;
    using Acc = typename Ops<DT>::Acc;
    constexpr int ESZ = Ops<DT>::kEsz;
    __shared__ __attribute__((aligned(16))) Word lds[sm_lds_words<DT, NW>()];
    const int64_t w = item0 + blockIdx.x;
    if (w >= nitems * a.nchunks) return;
    const int64_t chunk = w / nitems, t = w % nitems;
    const int64_t n = a.n_v;
    const bool lex = t >= g.rows0 * g.cols0;
    const int64_t u = lex ? t - g.rows0 * g.cols0 : t;
    const int64_t rt = u / (lex ? g.cols1 : g.cols0), ct = u % (lex ? g.cols1 : g.cols0);
    int64_t r0, rend, col0;
    if (!lex) {
        r0 = a.j_begin * (a.j_begin - 1) / 2 + rt * kSmB;
        rend = a.js * (a.js - 1) / 2;
        col0 = pair_j(r0) + 1 + ct * kSmB;
        if (col0 >= n) return;
    } else {
        r0 = lex_first(n, a.js) + rt * kSmB;
        rend = lex_first(n, a.j_end);
        col0 = ct * kSmB;
        int64_t jz, kz;
        lex_pair(n, r0 + kSmB - 1 < rend ? r0 + kSmB - 1 : rend - 1, jz, kz);
        if (col0 >= jz) return;
    }
    const int64_t ldb = a.ld * ESZ, nbytes = a.n_f * ESZ;
    // this thread's staged pair and vector, -1 past the part's end
    const int64_t r = r0 + threadIdx.x % kSmB, rr = r < rend ? r : rend - 1;
    int64_t x, y;
    if (!lex) {
        y = pair_j(rr);
        x = rr - y * (y - 1) / 2;
    } else {
        lex_pair(n, rr, x, y);
    }
    const int64_t z = col0 + threadIdx.x % kSmB;
    int64_t b0, b1;
    sm_range<DT>(nbytes, a.nchunks, a.chunk_tiles, chunk, b0, b1);
    Acc out[4];
    sm_tile<DT, NW, true, VEC>((const char*)a.V, r < rend ? x * ldb : -1, y * ldb,
                           z < n ? z * ldb : -1, b0, b1, !lex, lds, out);
    if (threadIdx.x >= 256) return;
    const int64_t ob = slab_offset(n, a.j_begin), stage = slab_offset(n, a.j_end) - ob;
    const PairT<DT>* N2 = (const PairT<DT>*)a.n2;
    const int fast = 4 * (threadIdx.x % 8), slow = threadIdx.x / 8;
    if (!lex) {
        const int64_t k = col0 + slow, p0 = r0 + fast;
        if (k >= n || p0 >= rend) return;
        const double sz = DT == PS_U8 ? a.s[k] : 0.0;
        int64_t j = pair_j(p0), i = p0 - j * (j - 1) / 2;
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            if (p0 + f < rend && k > j)
                sm3_store<DT>(a, out[f], i, j, k, DT == PS_U8 ? N2[p0 + f] : PairT<DT>(0), sz,
                              slab_offset(n, j) - ob + (k - j - 1) * j + i, chunk, stage);
            if (++i == j) {   // the next pair in colex order
                i = 0;
                ++j;
            }
        }
    } else {
        const int64_t q = r0 + slow, i0 = col0 + fast;
        if (q >= rend) return;
        int64_t j, k;
        lex_pair(n, q, j, k);
        const int64_t base = slab_offset(n, j) - ob + (k - j - 1) * j;
        const PairT<DT> njk = DT == PS_U8 ? N2[k * (k - 1) / 2 + j] : PairT<DT>(0);
#pragma unroll
        for (int f = 0; f < 4; ++f)
            if (i0 + f < j)
                sm3_store<DT>(a, out[f], i0 + f, j, k, njk, DT == PS_U8 ? a.s[i0 + f] : 0.0,
                              base + i0 + f, chunk, stage);
    }
}

// waves: of a workgroup, 4 or 8.
template <int DT, class Go>
hipError_t sm_dispatch(const void* V, int64_t ld, int waves, Go go) {
    const bool vec = (uintptr_t)V % 16 == 0 && ld * Ops<DT>::kEsz % 16 == 0;
    using std::integral_constant;
    if (waves == 8)
        return vec ? go(integral_constant<int, 8>{}, std::true_type{})
                   : go(integral_constant<int, 8>{}, std::false_type{});
    return vec ? go(integral_constant<int, 4>{}, std::true_type{})
               : go(integral_constant<int, 4>{}, std::false_type{});
}

template <int DT>
hipError_t go_sm2(const Mg2Call& a, hipStream_t st) {
    const int64_t T = tri_tiles(a.n_v, kSmB);
    return sm_dispatch<DT>(a.V, a.ld, a.small, [&](auto nw, auto vec) {
        constexpr int NW = decltype(nw)::value;
        const int64_t n = T * a.nchunks + (a.s_out ? ceil_div(a.n_v, NW) : 0);
        return launch_items(n, 64 * NW, 1, [&](unsigned grid, int64_t item0) {
            hipLaunchKernelGGL((ps_sm2_kernel<DT, NW, decltype(vec)::value>), dim3(grid),
                               dim3(64 * NW), 0, st, a, T, item0);
        });
    });
}

template <int DT>
hipError_t go_sm3(const Mg3Launch& a, hipStream_t st) {
    Sm3Grid g;
    g.rows0 = flat_row_tiles(a.j_begin, a.js, kSmB);
    g.cols0 = ceil_div(a.n_v - 1 - a.j_begin, kSmB);   // the first row tile's
    g.rows1 = lex_row_tiles(a.n_v, a.js, a.j_end, kSmB);
    g.cols1 = ceil_div(a.j_end - 1, kSmB);             // the last row tile's
    return sm_dispatch<DT>(a.V, a.ld, a.mode == kSlabSmall8 ? 8 : 4, [&](auto nw, auto vec) {
        constexpr int NW = decltype(nw)::value;
        return launch_items(g.items() * a.nchunks, 64 * NW, 1, [&](unsigned grid, int64_t item0) {
            hipLaunchKernelGGL((ps_sm3_kernel<DT, NW, decltype(vec)::value>), dim3(grid),
                               dim3(64 * NW), 0, st, a, g, g.items(), item0);
        });
    });
}

}  // namespace ps
