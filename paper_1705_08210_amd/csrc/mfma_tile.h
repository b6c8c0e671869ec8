// mfma_tile.h -- pieces shared by the matrix-core tile kernels (mfma.hip: int8
// thermometer planes of bytes; bitplane.hip: planes of bits on fp4): launch
// arguments, the LDS stage layout and hand-over, and the 3-way epilogues of
// the split tiling.
#pragma once

#include <type_traits>

#include "ps_internal.h"

namespace ps {

typedef unsigned v4u_t __attribute__((ext_vector_type(4)));
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef int v16i_t __attribute__((ext_vector_type(16)));
typedef float v16f_t __attribute__((ext_vector_type(16)));

constexpr int kMB = kMfmaTile;   // output tile rows and columns

// n / d correctly rounded, for integers 0 <= n < 2^24 and 1 <= d < 2^24 held
// in floats (the FP32 quotients of Section 2.1 and Eq. 1): the reciprocal
// refinement and the two remainder corrections of the IEEE division
// sequence, without its range scaling and special-case fix-up.  No
// operand, reciprocal, partial quotient or remainder here is denormal,
// infinite or needs scaling, so those steps are identities and the result
// is the sequence's own, the correctly rounded quotient.
__device__ __forceinline__ float div_u24(float n, float d) {
    const float y0 = __builtin_amdgcn_rcpf(d);
    const float y = __builtin_fmaf(__builtin_fmaf(-d, y0, 1.0f), y0, y0);
    const float q0 = n * y;
    const float q1 = __builtin_fmaf(__builtin_fmaf(-d, q0, n), y, q0);
    return __builtin_fmaf(__builtin_fmaf(-d, q1, n), y, q1);
}

// Dword 3 of a raw buffer descriptor on gfx950: 32-bit data format, offset
// addressing, no swizzle (loads past num_records return zero).
constexpr int kRsrcWord3 = 0x00020000;

struct LvArgs {
    const uint8_t* V;
    int64_t ld, n_f, n_v;
    int levels;
    int group;            // 2-way: block columns per tile-order group
    int64_t nk;           // field tiles
    const double* s;
    float* c2;
    int32_t* n2;
    int64_t nb, ntiles;
    // 3-way
    int64_t j_begin, j_end;
    const int64_t* prefix;
    uint32_t* c3;
    int64_t item0;
    int32_t mode, ob;
    int32_t f32div;       // the quotient's operands are integers below 2^24 (FP32 division)
    // split 3-way tiling, part p = 0, 1: its tiles, row tiles, the prefix of
    // their column-tile counts, and its pairs [r_begin, r_end) (colex indices
    // for the (i, j) part, lex indices for the (j, k) part); tiles
    // [0, nt[0]) of a launch are part 0's, the next nt[1] part 1's
    int64_t nt[2], nrt[2], r_begin[2], r_end[2];
    const int64_t* pre[2];
};

constexpr int kLvdMK = 64;
constexpr int kLvdStages = 3;

// Chunk swizzle of 64-byte rows: for every chunk c, the slots of any 8
// consecutive rows are distinct modulo 128 bytes and those of any 16
// consecutive rows distinct modulo 256 bytes (b128 fragment reads free of
// bank conflicts whether the LDS serves 8 or 16 lanes at once); rows r and
// r + 32 share a swizzle.
__device__ __forceinline__ int lvd_swz(int r) { return ((r >> 1) ^ (r >> 3)) & 3; }

// This wave's stage loads but the N most recent have landed and its LDS
// accesses are done, then the barrier; the empty asm statements keep the
// compiler from moving memory accesses across.
template <int N>
__device__ __forceinline__ void lvd_sync() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (0x7 << 4) | ((N >> 4) << 14));   // lgkmcnt 0
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Part 0 epilogue (Eq. 1 as in lv3_epilogue): a lane's two columns are pairs
// (i, j) with their own j, so n2(j, k) is gathered per element like n2(i, k);
// 2 s_k of the tile's rows is staged in LDS.  Stores go through a buffer
// resource from the tile's first entry (0, jmin, k0) to the end of the last
// pair's slab; an element outside i < j < k < n_v gets an offset past it.
template <bool F32, typename AccT>
__device__ __forceinline__ void lvs_epilogue0(const LvArgs& a, const AccT (&acc)[4][2],
                                              int64_t p0, int64_t k0, int wr, int wc,
                                              bool active, int8_t* lds) {
    using R = typename std::conditional<F32, float, double>::type;
    constexpr int TB = kMB, WN = 2, WM = 4;
    const int lane = threadIdx.x % 64;
    const int64_t n = a.n_v;
    const double* __restrict__ S = a.s;
    const int32_t* __restrict__ N2 = a.n2;
    R* rs2 = (R*)lds;   // 2 s_k
    if (threadIdx.x < TB) {
        const int64_t k = k0 + threadIdx.x;
        rs2[threadIdx.x] = k < n ? (R)(2.0 * S[k]) : (R)0;
    }
    __syncthreads();
    if (!active) return;
    const int64_t pe = a.r_end[0];
    const int64_t jmin = pair_j(p0);
    const int64_t jlast = pair_j(p0 + TB - 1 < pe ? p0 + TB - 1 : pe - 1);
    const int64_t ob = slab_offset(n, a.j_begin);
    const int64_t base0 = slab_offset(n, jmin) - ob + (k0 - jmin - 1) * jmin;
    const __amdgpu_buffer_rsrc_t rc3 = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.c3 + base0), (short)0, (int)((slab_offset(n, jlast + 1) - ob - base0) * 4),
        kRsrcWord3);
    const __amdgpu_buffer_rsrc_t rn2 = __builtin_amdgcn_make_buffer_rsrc(
        (void*)N2, (short)0, (int)(n * (n - 1) / 2 * 4), kRsrcWord3);
    R ls2[WN];            // 2 (s_i + s_j)
    uint32_t nij[WN];     // n2(i, j)
    int ii[WN], jj[WN];   // the column's pair; jj = n_v when past the part
    uint32_t sb[WN];      // entry (i, j, k) - base0 = sb + k j (mod 2^32)
#pragma unroll
    for (int nn = 0; nn < WN; ++nn) {
        const int64_t p = p0 + wc + nn * 32 + lane % 32;
        const bool vp = p < pe;
        const int64_t pp = vp ? p : pe - 1;
        const int64_t j = pair_j(pp), i = pp - j * (j - 1) / 2;
        ls2[nn] = (R)2 * ((R)S[i] + (R)S[j]);
        nij[nn] = (uint32_t)N2[pp];
        ii[nn] = (int)i;
        jj[nn] = vp ? (int)j : (int)n;
        sb[nn] = (uint32_t)(slab_offset(n, j) - ob - base0 - (j + 1) * j + i);
    }
    constexpr int RB = 4, NB = WM * 16 / RB;
    auto row_dk = [&](int b, int q) {
        const int m = b / (16 / RB), r = (b % (16 / RB)) * RB + q;
        return wr + m * 32 + (r / 4) * 8 + (lane / 32) * 4 + (r % 4);
    };
    struct Batch {
        uint32_t nik[RB][WN], njk[RB][WN];
    };
    const int kb = (int)k0;
    auto load_batch = [&](int b, Batch& o) {
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            const uint32_t k = (uint32_t)(kb + row_dk(b, q));
            const uint32_t ck = (k * (k - 1)) >> 1;   // k < 2^16: the table is below 2^31 bytes
#pragma unroll
            for (int nn = 0; nn < WN; ++nn) {
                o.nik[q][nn] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                    rn2, (int)((ck + (uint32_t)ii[nn]) * 4), 0, 0);
                o.njk[q][nn] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                    rn2, (int)((ck + (uint32_t)jj[nn]) * 4), 0, 0);
            }
        }
    };
    auto store_batch = [&](int b, const Batch& o) {
        const int m = b / (16 / RB);
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            const int r = (b % (16 / RB)) * RB + q;
            const int dk = row_dk(b, q);
            const int k = kb + dk;
            const R rk = rs2[dk];
#pragma unroll
            for (int nn = 0; nn < WN; ++nn) {
                const bool ok = k > jj[nn] && k < (int)n;
                const uint32_t n3 = nij[nn] + o.nik[q][nn] + o.njk[q][nn] - (uint32_t)acc[m][nn][r];
                const R d = ls2[nn] + rk;
                const R dd = d > (R)0 ? d : (R)1;
                float qv;
                if constexpr (F32)
                    qv = div_u24((float)(3u * n3), dd);
                else
                    qv = (float)((3.0 * (double)n3) / dd);
                const float c = d > (R)0 ? qv : 0.0f;
                const uint32_t off = ok ? (sb[nn] + __umul24((uint32_t)k, (uint32_t)jj[nn])) * 4u
                                        : 0x80000000u;
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, c), rc3,
                                                      (int)off, 0, 0);
            }
        }
    };
    Batch bt[2];
    load_batch(0, bt[0]);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b + 1 < NB) load_batch(b + 1, bt[(b + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        store_batch(b, bt[b & 1]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Part 1 epilogue (TB rows): a row is a pair (j, k); its 2 (s_j + s_k), n2(j, k), the
// pair-table offsets of rows j and k, j and its output row offset are staged
// in LDS once per tile; n2(i, j) and n2(i, k) are gathered per element
// (contiguous in i).  Stores from the tile's first pair's entry i = 0 to the
// end of the last pair's slab; columns i >= j get an offset past it.
template <bool F32, int TB, typename AccT>
__device__ __forceinline__ void lvs_epilogue1(const LvArgs& a, const AccT (&acc)[4][2],
                                              int64_t q0, int64_t i0, int wr, int wc,
                                              bool active, int8_t* lds) {
    using R = typename std::conditional<F32, float, double>::type;
    constexpr int WN = 2, WM = 4;   // TB rows (pairs) from q0
    const int lane = threadIdx.x % 64;
    const int64_t n = a.n_v;
    const double* __restrict__ S = a.s;
    const int32_t* __restrict__ N2 = a.n2;
    const int64_t qe = a.r_end[1];
    const int64_t ob = slab_offset(n, a.j_begin);
    int64_t jf, kf, jl, kl;
    lex_pair(n, q0 < qe ? q0 : qe - 1, jf, kf);   // (a half past the part stores nothing)
    lex_pair(n, q0 + TB - 1 < qe ? q0 + TB - 1 : qe - 1, jl, kl);
    const int64_t base0 = slab_offset(n, jf) - ob + (kf - jf - 1) * jf;
    int4* rowi = (int4*)lds;                         // {c(j), c(k), j, output row offset}
    R* rs2 = (R*)(lds + TB * sizeof(int4));           // 2 (s_j + s_k)
    int32_t* rnj = (int32_t*)(lds + TB * (sizeof(int4) + sizeof(R)));   // n2(j, k)
    if (threadIdx.x < TB) {
        const int64_t q = q0 + threadIdx.x;
        const bool vq = q < qe;
        int64_t j, k;
        lex_pair(n, vq ? q : qe - 1, j, k);
        const int64_t cj = j * (j - 1) / 2, ck = k * (k - 1) / 2;
        rowi[threadIdx.x] = make_int4((int)cj, (int)ck, vq ? (int)j : 0,
                                      (int)(slab_offset(n, j) - ob + (k - j - 1) * j - base0));
        rs2[threadIdx.x] = (R)2 * ((R)S[j] + (R)S[k]);
        rnj[threadIdx.x] = N2[ck + j];
    }
    __syncthreads();
    if (!active) return;
    const __amdgpu_buffer_rsrc_t rc3 = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.c3 + base0), (short)0, (int)((slab_offset(n, jl + 1) - ob - base0) * 4),
        kRsrcWord3);
    const __amdgpu_buffer_rsrc_t rn2 = __builtin_amdgcn_make_buffer_rsrc(
        (void*)N2, (short)0, (int)(n * (n - 1) / 2 * 4), kRsrcWord3);
    R ls[WN];        // 2 s_i
    int ii[WN];
#pragma unroll
    for (int nn = 0; nn < WN; ++nn) {
        const int64_t i = i0 + wc + nn * 32 + lane % 32;
        ls[nn] = (R)(2.0 * S[i < n ? i : n - 1]);
        ii[nn] = (int)i;
    }
    constexpr int RB = 4, NB = WM * 16 / RB;
    auto row_dk = [&](int b, int q) {
        const int m = b / (16 / RB), r = (b % (16 / RB)) * RB + q;
        return wr + m * 32 + (r / 4) * 8 + (lane / 32) * 4 + (r % 4);
    };
    struct Batch {
        uint32_t nij[RB][WN], nik[RB][WN];
        int4 ri[RB];
    };
    auto load_batch = [&](int b, Batch& o) {
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            const int4 ri = rowi[row_dk(b, q)];
            o.ri[q] = ri;
#pragma unroll
            for (int nn = 0; nn < WN; ++nn) {
                o.nij[q][nn] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                    rn2, (int)(((uint32_t)ri.x + (uint32_t)ii[nn]) * 4), 0, 0);
                o.nik[q][nn] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                    rn2, (int)(((uint32_t)ri.y + (uint32_t)ii[nn]) * 4), 0, 0);
            }
        }
    };
    auto store_batch = [&](int b, const Batch& o) {
        const int m = b / (16 / RB);
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            const int r = (b % (16 / RB)) * RB + q;
            const int dk = row_dk(b, q);
            const R rr = rs2[dk];
            const uint32_t njk = (uint32_t)rnj[dk];
            const int4 ri = o.ri[q];
#pragma unroll
            for (int nn = 0; nn < WN; ++nn) {
                const bool ok = ii[nn] < ri.z;
                const uint32_t n3 = o.nij[q][nn] + o.nik[q][nn] + njk - (uint32_t)acc[m][nn][r];
                const R d = ls[nn] + rr;
                const R dd = d > (R)0 ? d : (R)1;
                float qv;
                if constexpr (F32)
                    qv = div_u24((float)(3u * n3), dd);
                else
                    qv = (float)((3.0 * (double)n3) / dd);
                const float c = d > (R)0 ? qv : 0.0f;
                const uint32_t off =
                    ok ? ((uint32_t)ri.w + (uint32_t)ii[nn]) * 4u : 0x80000000u;
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, c), rc3,
                                                      (int)off, 0, 0);
            }
        }
    };
    Batch bt[2];
    load_batch(0, bt[0]);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b + 1 < NB) load_batch(b + 1, bt[(b + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        store_batch(b, bt[b & 1]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

}  // namespace ps
