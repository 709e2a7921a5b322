// Shared skeleton of the prepared bit-vector searches (Hamming, ADC): the
// shape of a workgroup's LDS ring and the FP4 query operand.
#pragma once

#include "hdc_device.h"

namespace hdc {

// Shape per class-tile count: query tiles (32 queries) per wave, words per
// window, LDS stages.  Two stages keep the LDS footprint small enough for
// several workgroups per CU: the other waves on each SIMD cover one wave's
// operand building, LDS waits and barriers, which pays more than deeper
// prefetch.
template <int KT> struct HmShape {
    static constexpr int QT = KT == 4 ? 1 : 2;
    static constexpr int W = KT == 1 ? 8 : 4;          // words per window (divides kHmWin)
    static constexpr int U = W / 2;                    // 16-byte units per query row
    static constexpr int RPL = 64 / U;                 // query rows per 1 KiB load
    static constexpr int SWZ = U == 2 ? 3 : 2;         // row shift of the unit swizzle
    static constexpr int ROWS = kWaves * QT * 32;      // queries per workgroup
    static constexpr int QB = ROWS * W * 8;            // query bytes per stage
    static constexpr int TB = W * KT * 1024;           // class operand bytes per window
    static constexpr int NST = 2;                      // LDS stages
    static constexpr int NQL = QB / 1024 / kWaves;     // query loads per wave per window
    static constexpr int NTL = TB / 1024 / kWaves;     // class loads per wave per window
    static constexpr int SB = QB + TB;                 // bytes per stage
};
constexpr int kHmWin = 8;   // the class operand is padded to whole 8-word windows

// Query bits of one dword as the FP4 B operand (0.5 per set bit): register
// r, nibble j = bit 4j + r.  The upper half of the operand is unused by FP4.
__device__ __forceinline__ v8i query_nibbles(uint32_t d)
{
    v8i b = {};
#pragma unroll
    for (int r = 0; r < 4; ++r)
        b[r] = (int)((d >> r) & 0x11111111u);
    return b;
}

// Query bits of one dword as bipolar FP4 values: +1.0 (0x2) for a clear bit,
// -1.0 (0xA) for a set one, in the same nibble order as query_nibbles (the bit
// of nibble j goes straight to the nibble's sign: a shift and one and-or).
__device__ __forceinline__ v8i query_bipolar(uint32_t d)
{
    v8i b = {};
#pragma unroll
    for (int r = 0; r < 4; ++r)
        b[r] = (int)(((d << (3 - r)) & 0x88888888u) | 0x22222222u);
    return b;
}

// Class operand table of the FP4 searches: for word w (from w_lo) and class
// tile kt, 64 lanes x 16 bytes where lane l, nibble j of dword r holds, for
// class kt*32 + l%32 at dimension d = 64w + 32*(l/32) + 4j + r, the code
// POS (class bit 0) or NEG (class bit 1) when d is in S, else 0.
//
// Built dword by dword: the dword's dimensions in S as a bit mask (set_mask),
// its nibble-spaced quarters times POS, and the class bits in the signs (NEG
// has POS's magnitude): a few operations per register instead of a remainder
// by the stride per dimension (K = 26, D = 10240: 11 us and 6 for the counts,
// 3.6 for both in one launch).  The first KT * 32 workgroups count each class's
// -1 elements over S where popc is given.
template <uint32_t POS, uint32_t NEG>
__global__ __launch_bounds__(256) void k_sign_table(const uint64_t *__restrict__ C, int K, int64_t ldc, int start,
                                                    int end, int stride, int w_lo, int KT, int64_t total,
                                                    int8_t *__restrict__ tab, int32_t *__restrict__ popc)
{
    static_assert(NEG == (POS | 8u), "codes of one magnitude");
    const int nk = popc ? 32 * KT : 0;
    if ((int)blockIdx.x < nk) {
        class_popc(C, K, ldc, start, end, stride, (int)blockIdx.x, popc);
        return;
    }
    const int64_t idx = (int64_t)((int)blockIdx.x - nk) * 256 + threadIdx.x;
    if (idx >= total)
        return;
    const int lane = (int)(idx & 63);
    const int kt = (int)((idx >> 6) % KT);
    const int64_t w = w_lo + (idx >> 6) / KT;
    const int k = kt * 32 + (lane & 31), g = lane >> 5;
    uint32_t o[4] = {0, 0, 0, 0};
    const uint32_t m = set_mask((int)(64 * w + 32 * g), start, end, stride);
    if (k < K && m) {
        const uint32_t c = (uint32_t)(C[k * ldc + w] >> (32 * g)) & m;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            o[r] = ((m >> r) & 0x11111111u) * POS | ((c >> r) & 0x11111111u) << 3;
    }
    *(uint4 *)(tab + idx * 16) = make_uint4(o[0], o[1], o[2], o[3]);
}

// Query row r of a stage is W words = U 16-byte units; unit hh of the
// window sits in slot hh ^ ((r >> SWZ) & (U - 1)), which keeps the 16-byte
// reads of 16 consecutive rows on distinct banks.
template <int KT> __device__ __forceinline__ int hm_slot(int r, int hh)
{
    typedef HmShape<KT> S;
    return hh ^ ((r >> S::SWZ) & (S::U - 1));
}

// Searches of few queries.  The streaming kernels take 128 or 256 queries per
// workgroup through every word in turn, so a few thousand queries leave most
// of the device idle (6238 queries, 26 classes, 10240 dimensions: 25
// workgroups, 19 us).  Here a workgroup takes 32 queries and its four waves a
// quarter of the word pairs each, queries and class operand straight from
// global memory, kFewPairs pairs' loads in flight; the waves' sums meet in LDS.
// Measured at 10240 x 26 / 8192 x 100: Hamming 18 / 24 us streaming against
// 11 / 12 at 6238 queries, 18 / 25 against 12 / 18 at 16384, 19 / 26 against
// 17 / 30 at 24000; cosine 31 / 73 against 16 / 26 and, at 24000, 35 / 76
// against 31 / 74.
constexpr int64_t kFewQueries = 16384;
constexpr int kFewPairs = 4;

// Calls op(p, p1, u) for this wave's pairs of words [.., p1) from w_lo, pairs
// p .. p + kFewPairs - 1 at a time with the query's words in u, the query
// being row blockIdx.x * 32 + lane % 32 (rows past n: row n - 1).  u is zero
// for pairs from p1 on.
template <class Op>
__device__ __forceinline__ void few_pairs(const uint64_t *__restrict__ Q, int64_t n, int64_t ldq, int w_lo, int w_hi,
                                          const Op &op)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t q = (int64_t)blockIdx.x * 32 + (lane & 31);
    const uint64_t *row = Q + (q < n ? q : n - 1) * ldq + w_lo;
    const int np = (w_hi - w_lo + 1) / 2;                     // pairs (ldq is even: the last is in the row)
    const int per = (np + kWaves - 1) / kWaves;
    const int p0 = wave * per, p1 = p0 + per < np ? p0 + per : np;
    for (int p = p0; p < p1; p += kFewPairs) {
        v4i u[kFewPairs];
#pragma unroll
        for (int i = 0; i < kFewPairs; ++i) {
            const int pc = p + i < p1 ? p + i : p1 - 1;
            u[i] = *(const v4i *)(row + 2 * pc);
            if (p + i >= p1)
                u[i] = v4i{0, 0, 0, 0};
        }
        op(p, p1, u);
    }
}

}  // namespace hdc
