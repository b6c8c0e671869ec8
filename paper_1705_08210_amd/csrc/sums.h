// sums.h -- the sum of one vector's fields by one wave, shared by the sums
// kernels and the launches that carry the sums along.
#pragma once

#include "mgemm_core.h"

namespace ps {

// ---------------------------------------------------------------------------
// Per-vector sums s_i = sum_q v_{i,q} in FP64 (exact integers for PS_U8),
// plus the count of entries outside the domain v >= 0 (negative, NaN, Inf).
// One wave per vector; 16-byte coalesced loads along the fields.
// ---------------------------------------------------------------------------
template <int DT>
__device__ __forceinline__ void sum_word(uint32_t w, double& acc, uint64_t& iacc, int& bad) {
    if constexpr (DT == PS_F32) {
        acc += (double)as_f32(w);
        bad += ((w & 0x7f800000u) == 0x7f800000u) | ((w >> 31) & (w != 0x80000000u));
    } else if constexpr (DT == PS_F16) {
        const h2_t h = as_h2(w);
        acc += (double)(float)h.x;
        acc += (double)(float)h.y;
        const uint32_t lo = w & 0xffffu, hi = w >> 16;
        bad += ((lo & 0x7c00u) == 0x7c00u) | ((lo >> 15) & (lo != 0x8000u));
        bad += ((hi & 0x7c00u) == 0x7c00u) | ((hi >> 15) & (hi != 0x8000u));
    } else {
        iacc += (w & 0xffu) + ((w >> 8) & 0xffu) + ((w >> 16) & 0xffu) + (w >> 24);
    }
}

// One FP64 element: its value and whether it is outside v >= 0 (negative
// other than -0, NaN or Inf).
__device__ __forceinline__ void sum_f64(uint64_t x, double& acc, int& bad) {
    acc += __builtin_bit_cast(double, x);
    bad += ((x & 0x7ff0000000000000ull) == 0x7ff0000000000000ull) |
           (int)((x >> 63) & (x != 0x8000000000000000ull));
}

template <int DT>
__device__ __forceinline__ void sum_row(const char* row, int64_t n_f, bool vec,
                                        double& acc, uint64_t& iacc, int& bad) {
    constexpr int ESZ = Ops<DT>::kEsz;
    const int lane = threadIdx.x % 64;
    const int64_t nbytes = n_f * ESZ;
    int64_t done = 0;
    if (vec) {
        const int64_t full = nbytes / 16 * 16;
        for (int64_t b = (int64_t)lane * 16; b < full; b += 64 * 16) {
            const uint4 v = *(const uint4*)(row + b);
            if constexpr (DT == PS_F64) {
                sum_f64(((uint64_t)v.y << 32) | v.x, acc, bad);
                sum_f64(((uint64_t)v.w << 32) | v.z, acc, bad);
            } else {
                sum_word<DT>(v.x, acc, iacc, bad);
                sum_word<DT>(v.y, acc, iacc, bad);
                sum_word<DT>(v.z, acc, iacc, bad);
                sum_word<DT>(v.w, acc, iacc, bad);
            }
        }
        done = full / ESZ;
    }
    if constexpr (DT == PS_F64) {   // whole 8-byte elements
        for (int64_t q = done + lane; q < n_f; q += 64)
            sum_f64(*(const uint64_t*)(row + 8 * q), acc, bad);
    } else {
        for (int64_t q = done + lane; q < n_f; q += 64) {
            uint32_t w;
            if (ESZ == 4) w = *(const uint32_t*)(row + 4 * q);
            else if (ESZ == 2) w = *(const unsigned short*)(row + 2 * q);
            else w = *(const unsigned char*)(row + q);
            sum_word<DT>(w, acc, iacc, bad);  // zero upper parts contribute 0
        }
    }
}

__device__ __forceinline__ void wave_reduce(double& acc, uint64_t& iacc, int& bad) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        acc += __shfl_xor(acc, off);
        iacc += __shfl_xor(iacc, off);
        bad += __shfl_xor(bad, off);
    }
}

// The sum of row[0 .. n_f) in every lane of a wave; bad: the wave's count of
// entries outside the domain.
template <int DT>
__device__ __forceinline__ double wave_row_sum(const char* row, int64_t n_f, bool vec, int& bad) {
    double acc = 0.0;
    uint64_t iacc = 0;
    bad = 0;
    sum_row<DT>(row, n_f, vec, acc, iacc, bad);
    wave_reduce(acc, iacc, bad);
    return DT == PS_U8 ? (double)iacc : acc;
}

}  // namespace ps
