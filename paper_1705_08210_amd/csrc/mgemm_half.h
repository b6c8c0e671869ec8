// mgemm_half.h -- the FP16 tile core: minima on the vector ALUs, their sums on
// the matrix cores.
//
// On the vector ALUs alone a pair of fields costs a packed min and a
// v_dot2c_f32_f16, both at half rate, and the matrix cores idle.  Here the eight
// mins of one output over a 16-byte chunk of fields are the A operand of
// v_mfma_f32_16x16x32_f16: lane l is row l % 16, k-group l / 16 of A, and B is a
// 0/1 selection, column n taking k-group n % 4 alone, for the outputs g = n / 4
// (sel[g]: zero in the other columns).  Four matrix instructions with g = 0..3
// thus add eight mins to each of four outputs of every lane, and one FP32
// accumulator block D holds the four:
//   D[row m][column 4 g + k] = the sum of lane m + 16 k's output g.
// Products with 1 are exact and the sums are FP32, eight terms per rounding
// chain where the dot product takes two.  A product with 0 must not be NaN, or an
// infinity of one vector would spread to pairs of others: when staged, the A rows
// are clamped from below and the B rows from both sides to the finite range (a
// NaN becomes an end of it), so that no min is infinite or NaN; finite data is
// unchanged.  What a pair with such a vector itself gets is unspecified.  The
// clamps cost 0.3 to 1% (B rows alone, from above: 14.97 against 15.01 ms at
// 20000 x 8191, 17.96 against 18.11 ms at 4096 x 1024 3-way), but a negative
// infinity then reached other pairs.
//
// Per 512 comparisons the wave issues four packed mins and one matrix
// instruction instead of eight half-rate vector instructions; measured in
// isolation 5.0e13 comparisons/s against 3.88e13 (the mins and the matrix
// instruction's issue slots bound it).  20000 x 8191 2-way 19.3 -> 15.5 ms (4.3e13/s),
// 4096 x 1024 3-way 22.3 -> 18.0 ms.
#pragma once

#include "ps_internal.h"

namespace ps {

typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));

// Staging of one field tile of 16 TM rows x BKW words: 16-byte chunks, chunk-major
// in LDS (chunk ch of row r at ch * kPitch + r), two buffers.  Consecutive threads
// take the chunks of a row in turn; the pitch spreads the chunks of 16 lanes
// over the banks, and fragment reads take eight consecutive rows.
template <int TM, int BKW>
struct HalfGeom {
    static constexpr int BM = 16 * TM;
    static constexpr int kCpr = BKW / 4;
    static constexpr int kCh = BM * kCpr / kThreads;
    static constexpr int kPitch = BM + 16 / kCpr;
    static constexpr int kBuf = kCpr * kPitch;          // chunks per buffer
    static constexpr int kLdsWords = 2 * kBuf * 4;
    static_assert(BM * kCpr % kThreads == 0 && 16 % kCpr == 0, "tile not divisible");
    __device__ static int row(int c) { return (threadIdx.x + c * kThreads) / kCpr; }
    __device__ static int ch(int c) { return (threadIdx.x + c * kThreads) % kCpr; }
};

__device__ __forceinline__ uint4 half_min(uint4 a, uint4 b) {
    return __builtin_bit_cast(uint4, __builtin_elementwise_min(__builtin_bit_cast(h8_t, a),
                                                               __builtin_bit_cast(h8_t, b)));
}
__device__ __forceinline__ uint4 half_max(uint4 a, uint4 b) {
    return __builtin_bit_cast(uint4, __builtin_elementwise_max(__builtin_bit_cast(h8_t, a),
                                                               __builtin_bit_cast(h8_t, b)));
}

// The sums of a 16 TM x 16 TM tile (run_tile / run_tile_flat in mgemm_core.h):
// byte offsets of this thread's staged rows, ra (with XJ min-ed with xa) and rb
// (rows past the end repeat a valid one: their outputs are not stored); field
// tiles [kt0, nk).  D[r][c / 4] holds the outputs of the lane's rows 8 r + l % 8
// and columns 8 c + l / 8 as described above.  LoadChunk: (pointer,
// bytes left in the row) -> uint4, zeros past the row's end; it serves the last field tile, the
// others are plain loads (their address arithmetic and tests would cost 8% of
// the vector instructions).
template <int TM, int BKW, bool XJ, bool VEC, class LoadChunk>
__device__ __forceinline__ void half_tile(const char* Vb, int64_t nbytes,
                                          const int64_t (&ra)[HalfGeom<TM, BKW>::kCh],
                                          const int64_t (&xa)[HalfGeom<TM, BKW>::kCh],
                                          const int64_t (&rb)[HalfGeom<TM, BKW>::kCh],
                                          bool active, uint4* As, uint4* Bs,
                                          f4_t (&D)[TM][TM / 4], int64_t kt0, int64_t nk,
                                          LoadChunk load_chunk) {
    using G = HalfGeom<TM, BKW>;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int fa = (wave & 1) * (8 * TM) + lane % 8;    // first A row of the lane
    const int fb = (wave >> 1) * (8 * TM) + lane / 8;   // first B row
#pragma unroll
    for (int r = 0; r < TM; ++r)
#pragma unroll
        for (int c = 0; c < TM / 4; ++c) D[r][c] = (f4_t){};
    h8_t sel[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const _Float16 x = (_Float16)(lane % 16 == 4 * g + lane / 16 ? 1.0f : 0.0f);
        sel[g] = (h8_t){x, x, x, x, x, x, x, x};
    }
    uint4 va[G::kCh], vx[XJ ? G::kCh : 1], vb[G::kCh];
    const char* pa[G::kCh];
    const char* px[XJ ? G::kCh : 1];
    const char* pb[G::kCh];
#pragma unroll
    for (int c = 0; c < G::kCh; ++c) {
        const int64_t o = kt0 * (BKW * 4) + G::ch(c) * 16;
        pa[c] = Vb + ra[c] + o;
        if constexpr (XJ) px[c] = Vb + xa[c] + o;
        pb[c] = Vb + rb[c] + o;
    }
    auto load16 = [](const char* p) {
        if constexpr (VEC) return *(const uint4*)p;
        uint4 v;
        __builtin_memcpy(&v, p, 16);
        return v;
    };
    auto load = [&](int64_t kt) {   // called for kt0, kt0 + 1, ... in turn
        if ((kt + 1) * (BKW * 4) <= nbytes) {
#pragma unroll
            for (int c = 0; c < G::kCh; ++c) {
                va[c] = load16(pa[c]);
                if constexpr (XJ) vx[c] = load16(px[c]);
                vb[c] = load16(pb[c]);
                pa[c] += BKW * 4;
                if constexpr (XJ) px[c] += BKW * 4;
                pb[c] += BKW * 4;
            }
        } else {   // the last one
#pragma unroll
            for (int c = 0; c < G::kCh; ++c) {
                const int64_t left = nbytes - kt * (BKW * 4) - G::ch(c) * 16;
                va[c] = load_chunk(pa[c], left);
                if constexpr (XJ) vx[c] = load_chunk(px[c], left);
                vb[c] = load_chunk(pb[c], left);
            }
        }
    };
    const uint32_t big2 = 0x7bff7bffu;   // 65504 twice
    const uint4 big = make_uint4(big2, big2, big2, big2);
    const uint32_t low2 = 0xfbfffbffu;   // -65504 twice
    const uint4 low = make_uint4(low2, low2, low2, low2);
    auto store = [&](int buf) {
#pragma unroll
        for (int c = 0; c < G::kCh; ++c) {
            const int o = buf * G::kBuf + G::ch(c) * G::kPitch + G::row(c);
            if constexpr (XJ)
                As[o] = half_max(half_min(va[c], vx[c]), low);
            else
                As[o] = half_max(va[c], low);
            Bs[o] = half_min(half_max(vb[c], low), big);
        }
    };
    if (kt0 >= nk) return;
    load(kt0);
    store(0);
    if (kt0 + 1 < nk) load(kt0 + 1);
    __syncthreads();
    int cur = 0;
    for (int64_t kt = kt0; kt < nk; ++kt) {
        // the next field tile to the other buffer (its last readers passed the
        // barrier below), the one after into registers
        if (kt + 1 < nk) store(cur ^ 1);
        if (kt + 2 < nk) load(kt + 2);
        if (active) {
            constexpr int kUnroll = TM == 8 && BKW == 16 ? 1 : 2;
#pragma unroll kUnroll
            for (int ch = 0; ch < G::kCpr; ++ch) {
                const uint4* A = As + cur * G::kBuf + ch * G::kPitch + fa;
                const uint4* B = Bs + cur * G::kBuf + ch * G::kPitch + fb;
                h8_t a[TM];
#pragma unroll
                for (int r = 0; r < TM; ++r) a[r] = __builtin_bit_cast(h8_t, A[8 * r]);
#pragma unroll
                for (int c = 0; c < TM; ++c) {
                    const h8_t b = __builtin_bit_cast(h8_t, B[8 * c]);
#pragma unroll
                    for (int r = 0; r < TM; ++r)
                        D[r][c / 4] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            __builtin_elementwise_min(a[r], b), sel[c % 4], D[r][c / 4], 0, 0, 0);
                }
            }
        }
        __syncthreads();   // kt + 1 staged; everyone is done with kt
        cur ^= 1;
    }
}

}  // namespace ps
