// bitplane.hip -- integer levels and binary data as planes of BITS on the fp4
// matrix cores.
//
// For integer values 0 <= v <= L, min(a, b) = sum_{t=1..L} [a >= t] [b >= t]
// (Section 3.1's min-product; L = 1 is the Sorensen case of Section 2.3, where
// min is AND).  A pass over V writes every row as L planes of one bit per
// field (an eighth of a byte plane, a quarter of an fp4 plane), so a row of
// 8192 fields and three levels is 3 KB and the whole operand stays in the
// caches.  The contraction runs on v_mfma_f32_32x32x64_f8f6f4 with e2m1
// operands formed in registers: a word holds 32 fields, a nibble four of them,
// and one AND with 0x1, 0x2 or 0x4 per nibble leaves one field per nibble as
// 0.5, 1 or 2 (e2m1).  The other operand takes the reciprocal weight (a shift
// and an AND), so every product of two set bits is exactly 1, no scale factors
// are needed, and the FP32 sums are integers below 2^24 (checked on the host):
// exact.  Which bit of which word a field lies in is the same for every row
// and otherwise free.
//
// Cost: 136 vector instructions form the operands of 32 matrix instructions (4
// x 2 blocks of 32 x 32, 256 bits deep), and those hide about six apiece:
// measured in isolation, 9.25 POP/s (the bare instruction's spec rate is 10.1).
//
// Against the paths it replaces (whole calls): binary 2-way 8190 x 20001, AND +
// popcount on the vector ALUs, 3.40 -> 0.645 ms; three levels 2-way 8192 x
// 32768, int8 planes formed in registers, 7.74 -> 3.99 ms (6.6 POP/s); three
// levels 3-way 4096 x 1024, 1.714 -> 0.884 ms.  The matrix cores bound the
// 2-way calls; the 3-way slices spend about as long on Eq. 1 and the stores.
//
// Kernels:
//   ps_bp_pack_kernel   V -> bit planes (and the per-vector sums): HBM-bound
//   ps_bp2_kernel       upper-triangle tiles, 2-way epilogue
//   ps_bp3_kernel       split tiling of the 3-way slices (pair rows are the AND
//                       of two rows: [min(a,b) >= t] = [a >= t] [b >= t]),
//                       Eq. 1 in the epilogue
#include <type_traits>

#include "mfma_tile.h"

namespace ps {

// Words of one row: the planes one after the other, each ceil(n_f / 32) words,
// padded to whole 16-byte chunks at the end.
int64_t bp_row_words(int64_t n_f, int levels) {
    return ceil_div((int64_t)levels * ceil_div(n_f, kBitsPerWord), 4) * 4;
}

// ---------------------------------------------------------------------------
// Packing.  One wave per row (waves stride over the rows): lane l forms word
// w of every plane from bytes 32 w .. 32 w + 31, bit 8 b + k = byte b of dword
// k, so four bytes are thresholded and placed per three or four instructions.
// The last word of a row whose length is not a multiple of 32 reads the row's
// last 32 bytes and clears those that belong to the word before (rows shorter
// than 32 bytes are read byte by byte).  For levels > 1 values are at most
// 127: (v | 0x80) - t keeps bit 7 iff v >= t and never borrows; for one level
// ((v & 0x7f) + 0x7f) | v has bit 7 set iff v != 0.
// ---------------------------------------------------------------------------
template <bool BIN>
__device__ __forceinline__ uint32_t bp_word(const uint32_t (&u)[8], uint32_t t) {
    uint32_t bits = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t f = BIN ? ((u[k] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | u[k]
                               : (u[k] | 0x80808080u) - t * 0x01010101u;
        bits |= (f & 0x80808080u) >> (7 - k);
    }
    return bits;
}

template <bool VEC>
__device__ __forceinline__ void bp_load32(const uint8_t* p, uint32_t (&u)[8]) {
    if constexpr (VEC) {
        const uint4 a = *(const uint4*)p, b = *(const uint4*)(p + 16);
        u[0] = a.x; u[1] = a.y; u[2] = a.z; u[3] = a.w;
        u[4] = b.x; u[5] = b.y; u[6] = b.z; u[7] = b.w;
    } else {   // byte-aligned 16-byte loads (the hardware takes any alignment)
        __builtin_memcpy(u, p, 16);
        __builtin_memcpy(u + 4, p + 16, 16);
    }
}

template <bool BIN, bool VEC>
__global__ __launch_bounds__(256) void ps_bp_pack_kernel(const uint8_t* V, int64_t n_f,
                                                         int64_t n_v, int64_t ld, int levels,
                                                         int64_t W, uint32_t* P, double* s) {
    const int lane = threadIdx.x % 64;
    const int64_t wf = (n_f + kBitsPerWord - 1) / kBitsPerWord;
    for (int64_t i = (int64_t)blockIdx.x * 4 + threadIdx.x / 64; i < n_v;
         i += (int64_t)gridDim.x * 4) {
        const uint8_t* row = V + i * ld;
        uint32_t* out = P + i * W;
        uint64_t sum = 0;
        for (int64_t w = lane; w < wf; w += 64) {
            const int64_t q0 = w * kBitsPerWord;
            uint32_t u[8];
            if (q0 + 32 <= n_f) {
                bp_load32<VEC>(row + q0, u);
            } else if (n_f >= 32) {
                bp_load32<false>(row + n_f - 32, u);
                const int skip = (int)(32 - (n_f - q0));   // bytes of the word before
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int z = skip - 4 * k;
                    u[k] &= z <= 0 ? 0xffffffffu : z >= 4 ? 0u : ~0u << (8 * z);
                }
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) u[k] = 0;
                for (int e = 0; e < (int)n_f; ++e) {
                    const uint32_t v = (uint32_t)row[e] << (8 * (e % 4));
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        if (e / 4 == k) u[k] |= v;
                }
            }
            uint32_t part = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) part = __builtin_amdgcn_sad_u8(u[k], 0u, part);
            sum += part;
            if constexpr (BIN) {
                out[w] = bp_word<true>(u, 1);
            } else {
                for (int t = 1; t <= levels; ++t)
                    out[(int64_t)(t - 1) * wf + w] = bp_word<false>(u, (uint32_t)t);
            }
        }
        for (int64_t w = levels * wf + lane; w < W; w += 64) out[w] = 0;
        if (s) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
            if (lane == 0) s[i] = (double)sum;
        }
    }
}

hipError_t launch_bp_pack(const uint8_t* V, int64_t n_f, int64_t n_v, int64_t ld, int levels,
                          uint32_t* P, double* s, hipStream_t st) {
    if (n_v <= 0) return hipSuccess;
    const dim3 grid((unsigned)(n_v < (int64_t)4 << 20 ? ceil_div(n_v, 4) : (int64_t)1 << 20));
    const int64_t W = bp_row_words(n_f, levels);
    const bool vec = (uintptr_t)V % 16 == 0 && ld % 16 == 0;
    auto go = [&](auto bin, auto al) {
        hipLaunchKernelGGL((ps_bp_pack_kernel<decltype(bin)::value, decltype(al)::value>), grid,
                           dim3(256), 0, st, V, n_f, n_v, ld, levels, W, P, s);
        return hipGetLastError();
    };
    using T = std::true_type;
    using F = std::false_type;
    if (levels == 1) return vec ? go(T{}, T{}) : go(T{}, F{});
    return vec ? go(F{}, T{}) : go(F{}, F{});
}

// ---------------------------------------------------------------------------
// Tile core.
// ---------------------------------------------------------------------------
constexpr int kBpMK = 64;   // bytes of a row per LDS stage (512 bits), the lvd_swz layout

// 64 zero bytes: the source of the chunks past a row's end in its last stage.
static __device__ uint4 bp_zeros[4];

// One stage of a wave's 32 WM x 32 WN block: A rows wr .., B rows wc .. of LDS
// regions of 64-byte rows; two 256-bit groups, four matrix k-steps each.  The
// second group's fragments are read while the first runs, and mid() (the
// loads of a later stage) is issued between the two.
template <int WM, int WN, class MID>
__device__ __forceinline__ void bp_stage(const int8_t* A, const int8_t* B, int wr, int wc,
                                         v16f_t (&acc)[WM][WN], MID mid) {
    constexpr int MK = kBpMK;
    const int lane = threadIdx.x % 64;
    const int fr = lane % 32, hk = lane / 32;
    const int sw = lvd_swz(fr);   // the swizzle of rows wr + m 32 + fr and wc + n 32 + fr
    auto frag = [&](int g, v4i_t (&fa)[WM], v4i_t (&fb)[WN]) {
        const int co = ((g * 2 + hk) ^ sw) * 16;
#pragma unroll
        for (int m = 0; m < WM; ++m) fa[m] = *(const v4i_t*)(A + (wr + m * 32 + fr) * MK + co);
#pragma unroll
        for (int n = 0; n < WN; ++n) fb[n] = *(const v4i_t*)(B + (wc + n * 32 + fr) * MK + co);
    };
    v4i_t fa[2][WM], fb[2][WN];
    frag(0, fa[0], fb[0]);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        if (g == 0) frag(1, fa[1], fb[1]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v8i_t xa[WM], xb[WN];   // e2m1: 0x1 = 0.5, 0x2 = 1, 0x4 = 2
            const v4i_t m1 = 0x11111111, m2 = 0x22222222, m4 = 0x44444444;
#pragma unroll
            for (int m = 0; m < WM; ++m) {
                const v4i_t f = fa[g][m];
                const v4i_t x = k == 0 ? f & m1 : k == 1 ? f & m2 : k == 2 ? f & m4 : (f >> 2) & m2;
                xa[m] = (v8i_t){x.x, x.y, x.z, x.w, 0, 0, 0, 0};
            }
#pragma unroll
            for (int n = 0; n < WN; ++n) {
                const v4i_t f = fb[g][n];
                const v4i_t x = k == 0   ? (f << 2) & m4
                                : k == 1 ? f & m2
                                : k == 2 ? (f >> 2) & m1
                                         : (f >> 2) & m2;
                xb[n] = (v8i_t){x.x, x.y, x.z, x.w, 0, 0, 0, 0};
            }
#pragma unroll
            for (int m = 0; m < WM; ++m)
#pragma unroll
                for (int n = 0; n < WN; ++n)   // zero scale operands: the form without scales
                    acc[m][n] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        xa[m], xb[n], acc[m][n], 4, 4, 0, 0, 0, 0);
        }
        if (g == 0) {
            asm volatile("" ::: "memory");
            mid();
            asm volatile("" ::: "memory");
        }
    }
}

// Stage hand-over before stage s of ns with stages issued AHEAD ahead, NU
// loads each: stage s has landed, and every wave is past stage s - 1.
template <int NU, int AHEAD>
__device__ __forceinline__ void bp_sync(int64_t s, int64_t ns) {
    if (s + AHEAD <= ns)
        lvd_sync<NU*(AHEAD - 1)>();
    else
        lvd_sync<0>();
}

// ---------------------------------------------------------------------------
// 2-way.  Workgroups of 2 x 2 waves, a wave 32 WM rows j by 32 WN columns i;
// stages of 64 bytes of the tile's 64 (WM + WN) rows go straight into a ring of
// S LDS slots (global_load_lds_dwordx4, 16 rows per wave instruction), S - 1
// stages ahead.  Rows past n_v load row n_v - 1 (their outputs are never
// stored), chunks past a row's end load zeros.
// ---------------------------------------------------------------------------

// c2 (and n2) of a wave's block: D[row][col] of a 32 x 32 block has col = lane
// % 32 and row = (r / 4) * 8 + (lane / 32) * 4 + r % 4; rows are j, columns i.
// ssj: s_j of the tile's rows.  F32: 2 n2 and s_i + s_j are integers below
// 2^24, and the FP32 quotient is the FP64 quotient's rounding (div_u24);
// otherwise FP64.  INNER: every i < j < n_v in the block.
// One of the two outputs at a time and no branch inside a full block: with a
// branch per element around either store each quotient ran as a serial chain
// (8192 x 32768, three levels, 4.31 -> 4.17 ms; 8190 x 20001 binary 0.666 -> 0.656;
// 400 x 6000, two levels, 34 -> 30 us; 400 x 20001 binary, bound by the stores,
// 210 -> 218 us).
template <int WM, int WN, bool F32, bool INNER, bool C2, typename R>
__device__ __forceinline__ void bp_store2(const LvArgs& a, const v16f_t (&acc)[WM][WN], int64_t i0,
                                          int64_t jw, int wr, const R* ssj) {
    const int lane = threadIdx.x % 64;
    const int64_t i = i0 + lane % 32;
    R si[WN];
    if constexpr (C2) {
#pragma unroll
        for (int n = 0; n < WN; ++n) {
            const int64_t ii = i + n * 32;
            si[n] = (R)a.s[INNER || ii < a.n_v ? ii : a.n_v - 1];
        }
    }
#pragma unroll
    for (int m = 0; m < WM; ++m)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int dr = m * 32 + g * 8 + (lane / 32) * 4;
            const int64_t j = jw + dr;
            int64_t row = j * (j - 1) / 2 + i;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float c[WN];
                if constexpr (C2) {
                    const R sj = ssj[wr + dr + e];
#pragma unroll
                    for (int n = 0; n < WN; ++n) {
                        const float num = acc[m][n][g * 4 + e];
                        const R d = si[n] + sj;
                        if constexpr (F32)
                            c[n] = div_u24(2.0f * num, d > 0.0f ? d : 1.0f);
                        else
                            c[n] = (float)((2.0 * (double)num) / (d > 0.0 ? d : 1.0));
                        c[n] = d > (R)0 ? c[n] : 0.0f;
                    }
                }
#pragma unroll
                for (int n = 0; n < WN; ++n) {
                    if (!INNER && (j + e >= a.n_v || i + n * 32 >= j + e)) continue;
                    if constexpr (C2)
                        a.c2[row + n * 32] = c[n];
                    else
                        a.n2[row + n * 32] = (int32_t)acc[m][n][g * 4 + e];
                }
                row += j + e;
            }
        }
}

template <int WM, int WN, bool F32, typename R>
__device__ __forceinline__ void bp_epilogue2(const LvArgs& a, const v16f_t (&acc)[WM][WN],
                                             int64_t i0, int64_t j0, int wr, int wc, bool active,
                                             int8_t* lds) {
    R* ssj = (R*)lds;
    for (int t = threadIdx.x; t < 64 * WM; t += 256)
        ssj[t] = (R)a.s[j0 + t < a.n_v ? j0 + t : a.n_v - 1];
    __syncthreads();
    if (!active) return;
    const int64_t iw = i0 + wc, jw = j0 + wr;
    const bool inner = iw + 32 * WN <= jw && jw + 32 * WM <= a.n_v;
    if (a.c2) {
        if (inner)
            bp_store2<WM, WN, F32, true, true, R>(a, acc, iw, jw, wr, ssj);
        else
            bp_store2<WM, WN, F32, false, true, R>(a, acc, iw, jw, wr, ssj);
    }
    if (a.n2) {
        if (inner)
            bp_store2<WM, WN, F32, true, false, R>(a, acc, iw, jw, wr, ssj);
        else
            bp_store2<WM, WN, F32, false, false, R>(a, acc, iw, jw, wr, ssj);
    }
}

template <int WM, int WN, int S>
__global__ __launch_bounds__(256, 2) void ps_bp2_kernel(LvArgs a) {
    constexpr int MK = kBpMK, RA = 64 * WM, RB = 64 * WN, HALVES = RA / RB;
    constexpr int kStageBytes = (RA + RB) * MK;
    constexpr int NU = kStageBytes / 1024 / 4;       // wave instructions per stage
    constexpr int AHEAD = S - 1;
    static_assert(NU * 4 * 1024 == kStageBytes && NU * AHEAD < 64, "stage split");
    __shared__ __attribute__((aligned(1024))) int8_t lds[S * kStageBytes];
    const int64_t t2 = a.item0 + (int64_t)(blockIdx.x % kXcds) * (gridDim.x / kXcds) +
                       blockIdx.x / kXcds;
    if (t2 >= HALVES * a.ntiles) return;
    int64_t bi, bj;
    grouped_tri_decode_rt(t2 / HALVES, a.nb, a.group, bi, bj);
    const int64_t i0 = bi * RA + (t2 % HALVES) * RB, j0 = bj * RA;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int wr = (wave % 2) * 32 * WM;    // j offset of the wave's block (A rows)
    const int wc = (wave / 2) * 32 * WN;    // i offset (B rows)
    const bool active =
        (i0 + wc < a.n_v) && (j0 + wr < a.n_v) && (i0 + wc + 1 < j0 + wr + 32 * WM);
    const uint8_t* src[NU];
    int cb[NU];                             // byte offset of the lane's chunk in a stage
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int row = (wave + 4 * u) * 16 + lane / 4;
        const int c = (lane % 4) ^ lvd_swz(row);
        int64_t g = row < RA ? j0 + row : i0 + (row - RA);
        if (g >= a.n_v) g = a.n_v - 1;
        cb[u] = c * 16;
        src[u] = a.V + g * a.ld + c * 16;
    }
    const int64_t ns = a.nk;
    auto issue = [&](int64_t s, int slot) {
        const int64_t left = a.ld - s * MK;   // bytes of the rows from this stage on
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const void* p = cb[u] < left ? (const void*)(src[u] + s * MK) : (const void*)bp_zeros;
            __builtin_amdgcn_global_load_lds(
                p, (void*)(lds + slot * kStageBytes + (wave + 4 * u) * 1024), 16, 0, 0);
        }
    };
    v16f_t acc[WM][WN];
#pragma unroll
    for (int m = 0; m < WM; ++m)
#pragma unroll
        for (int n = 0; n < WN; ++n) acc[m][n] = (v16f_t){};
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)
        if (s < ns) issue(s, s);
    // one loop for waves with work, one for the rest (a branch inside the loop
    // would carry the accumulators across it)
    auto run = [&](auto compute) {
        int slot = 0;
        for (int64_t s = 0; s < ns; ++s) {
            bp_sync<NU, AHEAD>(s, ns);
            const int sn = slot == 0 ? S - 1 : slot - 1;
            compute(slot, [&]() {
                if (s + AHEAD < ns) issue(s + AHEAD, sn);
            });
            slot = slot == S - 1 ? 0 : slot + 1;
        }
    };
    if (active)
        run([&](int slot, auto mid) {
            const int8_t* A = lds + slot * kStageBytes;
            bp_stage<WM, WN>(A, A + RA * MK, wr, wc, acc, mid);
        });
    else
        run([](int, auto mid) { mid(); });
    // the epilogue's sums go to the slot of stage ns - 2, which every wave
    // left before the barrier of stage ns - 1
    int8_t* ep = lds + (int)((ns + S - 2) % S) * kStageBytes;
    if (a.f32div)
        bp_epilogue2<WM, WN, true, float>(a, acc, i0, j0, wr, wc, active, ep);
    else
        bp_epilogue2<WM, WN, false, double>(a, acc, i0, j0, wr, wc, active, ep);
}

// ---------------------------------------------------------------------------
// 3-way: half h of tile t of part PART of the split tiling (split3), 256 plain
// rows by 128 pair rows.  Part 0: output rows are k from the row tile's
// smallest j + 1, output columns the colex pairs (i, j); part 1: output rows
// are the lex pairs (j, k), output columns i.  The plain rows go straight into
// a ring of three LDS slots, two stages ahead; a pair row is the AND of its two
// rows, formed in registers and written into the same slots.  Four waves of
// 128 x 64, two workgroups per CU (one's barriers and epilogue overlap the
// other's multiply-adds).
// ---------------------------------------------------------------------------
template <int PART>
__device__ __forceinline__ void bp3_tile(const LvArgs& a, int64_t t, int h, int8_t* lds) {
    constexpr int TB = kMB, WN = 2, HB = TB / 2, MK = kBpMK, S = kLvdStages;
    constexpr int kStageBytes = (TB + HB) * MK;
    constexpr int NU = TB * MK / 1024 / 4;   // plain-row wave instructions per stage
    constexpr int NP = HB * MK / 16 / 256;   // pair-row chunks per thread per stage
    static_assert(NU * 4 * 1024 == TB * MK && NP * 256 * 16 == HB * MK, "stage split");
    const int64_t* pre = a.pre[PART];
    int64_t lo = 0, hi = a.nrt[PART];
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) / 2;
        if (pre[mid] <= t) lo = mid; else hi = mid;
    }
    const int64_t ct = t - pre[lo];
    const int64_t n = a.n_v;
    const int64_t r0 = a.r_begin[PART] + lo * TB, re = a.r_end[PART];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    int64_t g0;        // first plain row
    int64_t k0 = 0, i0 = 0, qa = 0;
    int wr, wl, wc;    // the wave's A rows, B rows (LDS) and output columns in the tile
    bool active;
    int ox[NP], oy[NP], pc[NP];   // this thread's pair chunks: rows and byte offset in a stage
    auto pair_offsets = [&](auto pair) {
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            const int q = (int)threadIdx.x + 256 * c;
            int64_t x, y;
            pair(q / 4, x, y);
            pc[c] = (q % 4) * 16;
            ox[c] = (int)(x * a.ld) + pc[c];
            oy[c] = (int)(y * a.ld) + pc[c];
        }
    };
    if constexpr (PART == 0) {
        k0 = pair_j(r0) + 1 + ct * TB;
        g0 = k0;
        wr = (wave % 2) * (TB / 2);
        wl = (wave / 2) * 32 * WN;
        wc = h * HB + wl;
        const int64_t pq = r0 + wc;
        const int64_t kq = k0 + wr + TB / 2 - 1 < n - 1 ? k0 + wr + TB / 2 - 1 : n - 1;
        active = k0 + wr < n && pq < re && pair_j(pq) < kq;
        pair_offsets([&](int r, int64_t& x, int64_t& y) {
            const int64_t p = r0 + h * HB + r < re ? r0 + h * HB + r : re - 1;
            y = pair_j(p);
            x = p - y * (y - 1) / 2;
        });
    } else {
        i0 = ct * TB;
        g0 = i0;
        qa = r0 + h * HB;
        const int64_t qz = qa + HB - 1 < re ? qa + HB - 1 : re - 1;
        wr = 0;
        wl = wave * 32 * WN;
        wc = wl;
        int64_t jz, kz;
        lex_pair(n, qz, jz, kz);
        active = qa < re && i0 + wl < jz;
        pair_offsets([&](int r, int64_t& x, int64_t& y) {
            lex_pair(n, qa + r < re ? qa + r : re - 1, x, y);
        });
    }
    const uint8_t* src[NU];
    int cb[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int row = (wave + 4 * u) * 16 + lane / 4;
        const int c = (lane % 4) ^ lvd_swz(row);
        const int64_t g = g0 + row < n ? g0 + row : n - 1;
        cb[u] = c * 16;
        src[u] = a.V + g * a.ld + c * 16;
    }
    int pd[NP];   // LDS byte offsets of this thread's pair chunks within a slot
#pragma unroll
    for (int c = 0; c < NP; ++c) {
        const int q = (int)threadIdx.x + 256 * c, r = q / 4;
        pd[c] = (TB + r) * MK + ((q % 4) ^ lvd_swz(r)) * 16;
    }
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)a.V, (short)0, (int)(n * a.ld), kRsrcWord3);
    v4u_t px[NP], py[NP];
    auto issue = [&](int64_t s, int slot) {
        const int64_t left = a.ld - s * MK;
#pragma unroll
        for (int c = 0; c < NP; ++c) {   // a chunk past the rows' end reads zero (out of range)
            const int so = pc[c] < left ? (int)s * MK : (int)0x80000000;
            px[c] = __builtin_amdgcn_raw_buffer_load_b128(rs, ox[c] + so, 0, 0);
            py[c] = __builtin_amdgcn_raw_buffer_load_b128(rs, oy[c] + so, 0, 0);
        }
        asm volatile("" ::: "memory");   // pair loads first: their wait leaves the DMA in flight
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const void* p = cb[u] < left ? (const void*)(src[u] + s * MK) : (const void*)bp_zeros;
            __builtin_amdgcn_global_load_lds(
                p, (void*)(lds + slot * kStageBytes + (wave + 4 * u) * 1024), 16, 0, 0);
        }
    };
    auto pstore = [&](int slot) {
#pragma unroll
        for (int c = 0; c < NP; ++c)
            *(v4u_t*)(lds + slot * kStageBytes + pd[c]) = px[c] & py[c];
    };
    v16f_t acc[4][WN];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int nn = 0; nn < WN; ++nn) acc[m][nn] = (v16f_t){};
    const int64_t ns = a.nk;
    issue(0, 0);
    pstore(0);
    if (ns > 1) {
        issue(1, 1);
        pstore(1);
    }
    auto run = [&](auto compute) {
        int slot = 0;
        for (int64_t s = 0; s < ns; ++s) {
            bp_sync<NU, 2>(s, ns);
            const int sn = slot == 0 ? S - 1 : slot - 1;
            compute(slot, [&]() {
                if (s + 2 < ns) issue(s + 2, sn);
            });
            if (s + 2 < ns) pstore(sn);
            slot = slot == S - 1 ? 0 : slot + 1;
        }
    };
    if (active)
        run([&](int slot, auto mid) {
            const int8_t* P = lds + slot * kStageBytes;   // plain rows
            const int8_t* Q = P + TB * MK;                 // pair rows
            if constexpr (PART == 0)
                bp_stage<4, WN>(P, Q, wr, wl, acc, mid);
            else
                bp_stage<4, WN>(Q, P, wr, wl, acc, mid);
        });
    else
        run([](int, auto mid) { mid(); });
    // the epilogue's row data goes to slot (ns + 1) % 3, last read by stage
    // ns - 2 before the barrier of stage ns - 1
    int8_t* ep = lds + (int)((ns + 1) % S) * kStageBytes;
    if constexpr (PART == 0) {
        if (a.f32div)
            lvs_epilogue0<true>(a, acc, r0, k0, wr, wc, active, ep);
        else
            lvs_epilogue0<false>(a, acc, r0, k0, wr, wc, active, ep);
    } else {
        if (a.f32div)
            lvs_epilogue1<true, HB>(a, acc, qa, i0, 0, wl, active, ep);
        else
            lvs_epilogue1<false, HB>(a, acc, qa, i0, 0, wl, active, ep);
    }
}

__global__ __launch_bounds__(256, 2) void ps_bp3_kernel(LvArgs a) {
    __shared__ __attribute__((aligned(1024))) int8_t lds[kLvdStages * (kMB + kMB / 2) * kBpMK];
    const int64_t t2 = a.item0 + (int64_t)(blockIdx.x % kXcds) * (gridDim.x / kXcds) +
                       blockIdx.x / kXcds;
    if (t2 >= 2 * a.ntiles) return;
    const int64_t t = t2 / 2;
    const int h = (int)(t2 % 2);
    if (t < a.nt[0])
        bp3_tile<0>(a, t, h, lds);
    else
        bp3_tile<1>(a, t - a.nt[0], h, lds);
}

// ---------------------------------------------------------------------------
// Launches.
// ---------------------------------------------------------------------------
static LvArgs bp_args(const BpLaunch& b) {
    LvArgs a{};
    a.V = (const uint8_t*)b.planes;
    a.ld = bp_row_words(b.n_f, b.levels) * 4;   // a row of planes, in bytes
    a.n_f = b.n_f;
    a.n_v = b.n_v;
    a.levels = b.levels;
    a.group = 4;
    a.nk = a.ld > kBpMK ? ceil_div(a.ld, kBpMK) : 1;
    a.s = b.s;
    a.c2 = b.c2;
    a.n2 = b.n2;
    return a;
}

// The widest shape that still leaves about a workgroup per half CU: 64 x 64
// tiles, 128 x 128 once there are 128 of them, 256 x 128 once there are
// 1024 (whole calls, us, three levels of 8000 fields; 256 x 128 / 128 x 128
// / 64 x 64): 1536 vectors 88 / 57 / 45, 2048 89 / 58 / 64, 4096 136 / 118 /
// 142, 6000 199 / 186 / 271, 8192 315 / 316 / 482; 400 to 20000 fields and
// one level cross at the same sizes.
int bp2_rows(int64_t n_v) {
    if (tri_tiles(n_v, 256) * 2 >= 1024) return 256;
    return tri_tiles(n_v, 128) >= 128 ? 128 : 64;
}

hipError_t launch_bp2(const BpLaunch& b, hipStream_t st) {
    if (b.n_v < 2) return hipSuccess;
    LvArgs a = bp_args(b);
    a.f32div = 2 * (int64_t)b.levels * b.n_f < ((int64_t)1 << 24);
    auto go = [&](auto wm, auto wn, auto slots) {
        constexpr int WM = decltype(wm)::value, WN = decltype(wn)::value;
        a.nb = ceil_div(b.n_v, 64 * WM);
        a.ntiles = a.nb * (a.nb + 1) / 2;
        return launch_items(WM / WN * a.ntiles, 256, kXcds, [&](unsigned grid, int64_t item0) {
            LvArgs c = a;
            c.item0 = item0;
            hipLaunchKernelGGL((ps_bp2_kernel<WM, WN, decltype(slots)::value>), dim3(grid),
                               dim3(256), 0, st, c);
        });
    };
    using std::integral_constant;
    switch (bp2_rows(b.n_v)) {
    case 256:
        return go(integral_constant<int, 4>{}, integral_constant<int, 2>{},
                  integral_constant<int, 3>{});
    case 128:
        return go(integral_constant<int, 2>{}, integral_constant<int, 2>{},
                  integral_constant<int, 4>{});
    default:
        return go(integral_constant<int, 1>{}, integral_constant<int, 1>{},
                  integral_constant<int, 8>{});
    }
}

hipError_t launch_bp3(const BpLaunch& b, hipStream_t st) {
    if (b.n_v < 3 || b.j_end <= b.j_begin) return hipSuccess;
    const int64_t n = b.n_v, jb = b.j_begin, je = b.j_end, js = split3(n, jb, je);
    LvArgs a = bp_args(b);   // a.n2: the pair numerators of Eq. 1
    a.j_begin = jb;
    a.j_end = je;
    a.f32div = 6 * (int64_t)b.levels * b.n_f < ((int64_t)1 << 24);
    a.c3 = (uint32_t*)b.c3;
    a.nrt[0] = flat_row_tiles(jb, js, kMB);
    a.nrt[1] = lex_row_tiles(n, js, je, kMB);
    a.pre[0] = b.prefix;
    a.pre[1] = b.prefix + a.nrt[0] + 1;
    a.r_begin[0] = jb * (jb - 1) / 2;
    a.r_end[0] = js * (js - 1) / 2;
    a.r_begin[1] = lex_first(n, js);
    a.r_end[1] = lex_first(n, je);
    a.nt[0] = a.nrt[0] > 0 ? flat_tiles(n, jb, js, kMB) : 0;
    a.nt[1] = a.nrt[1] > 0 ? lex_tiles(n, js, je, kMB) : 0;
    hipError_t e = launch_prefix3_split(n, jb, js, je, kMB, b.prefix, b.prefix + a.nrt[0] + 1, st);
    if (e != hipSuccess) return e;
    a.ntiles = a.nt[0] + a.nt[1];
    return launch_items(2 * a.ntiles, 256, kXcds, [&](unsigned grid, int64_t item0) {
        LvArgs c = a;
        c.item0 = item0;
        hipLaunchKernelGGL(ps_bp3_kernel, dim3(grid), dim3(256), 0, st, c);
    });
}

}  // namespace ps
