// Cosine similarity of bipolar query hypervectors against non-binarised
// (integer) class accumulators, on the matrix cores.
//
// With q'_d in {0,1} the query bit (1 = element -1) and a_kd the class
// accumulator, the dot product over S is
//     dot_k = sum_S a_kd - 2 * sum_S q'_d * a_kd.
// The second sum runs as int8 MFMAs (rows = classes, columns = queries,
// K = 32 dimensions): a_kd = 256 * hi + lo with hi, lo in [-128, 127]
// (|a| <= 32639), one MFMA per part; the query operand holds the bits as
// bytes {0, 1}, two operations per register (see spread_bits).
// score_k = (double)dot_k * rinv_k with rinv_k = 1 / sqrt(sum_S a_kd^2)
// (0 for an all-zero class), both roundings correctly rounded, so the
// scores equal a plain double computation bit for bit; label = first class
// with the largest score.  An accumulator entry over S outside [-32639,
// 32639] does not fit the split: _prepare then clears a flag in the
// workspace and every label of the search is -1, every score NaN.
//
// Prepared operand (hdc_cosine_prepare): for word w (from the even word at
// or below the first word of S, padded to whole 8-word windows), dword half
// h, part p (lo, hi) and class tile kt, 64 lanes x 16 bytes: lane l, byte
// b = 4r + i holds part p of a_kd for class kt*32 + l%32 at dimension
// 64w + 32h + 4*(l/32) + r + 8i (0 outside S), the order in which the
// query operand takes the dword's bits (register r of lane half g =
// (dword >> (4g + r)) & 0x01010101); then T_k = sum_S a_kd (int64)
// and rinv_k (double) for 128 classes, max |a_kd| over S per class (int32)
// and the range flag.
//
// Accumulators of at most 255 over S (sums of up to 255 training rows) take a
// faster operand, chosen by _prepare from the classes' largest entries (flag
// 2): a_kd = 16 * h + l with 4-bit magnitudes of a's sign, as FP6 (E2M3 holds
// n / 8 for n = 0..15 in the codes 0..15) against the query bits as FP4 (0.5),
// block scales 2^4 and 2^8, both parts into one fp32 accumulator: every
// product is an integer and |sum| <= 255 * 65536 < 2^24, so the sums are
// exact.  Twice the K per instruction at the same cycles, one accumulator
// instead of two (two query tiles per wave with four class tiles), 3 KiB per
// word and class tile instead of 4: for word w, [part (l, h)][kt] 64 lanes x
// 16 bytes, then [part][kt] 64 lanes x 8 bytes, the 192 bits of lane l being
// 32 codes of class kt*32 + l%32, code i for dimension 64w + 32*(l/32) +
// 4*(i%8) + i/8 (the order of the query nibbles).
//
// Streaming as in the prepared Hamming search: query words and operand
// windows go from global memory straight into a two-stage LDS ring
// (global_load_lds), one barrier per window.
#include <limits.h>

#include "hdc_stream.h"

namespace hdc {

template <int KT, int QT_> struct CosShape {
    static constexpr int QT = KT == 4 ? 1 : QT_;
    static constexpr int W = KT == 4 ? 2 : 4;          // words per window (divides kCosWin)
    static constexpr int U = W / 2;                    // 16-byte units per query row
    static constexpr int RPL = 64 / U;                 // query rows per 1 KiB load
    static constexpr int ROWS = kWaves * QT * 32;      // queries per workgroup
    static constexpr int QB = ROWS * W * 8;            // query bytes per stage
    static constexpr int TB = W * 4 * KT * 1024;       // operand bytes per window
    static constexpr int NST = KT == 1 ? 3 : 2;        // LDS stages
    // loads per wave (a short last one: its waves past QB load nothing)
    static constexpr int NQL = (QB / 1024 + kWaves - 1) / kWaves;
    static constexpr int NTL = TB / 1024 / kWaves;
    static constexpr int SB = QB + TB;
    static_assert(NST == 2 || QB % (1024 * kWaves) == 0, "waits count the loads of a window");
};
constexpr int kCosWin = 8;
// Up to here the workgroups take 128 queries, one tile per wave: at 256 they
// would be fewer than the CUs (50000 x 8192 against 50 classes: 56 us at 256,
// 36 here; 25000 x 6208 against 10: 24 and 14).  Past it two tiles share each
// operand read.
constexpr int64_t kCosNarrow = 65536;
// The few-queries kernel (see few_pairs) with four class tiles: its registers
// leave one workgroup per CU, so past 256 workgroups it takes a second round
// (16000 x 8192 against 100 int8 classes: 71 us, 66 streaming; 1000: 32 and
// 62).
constexpr int64_t cos_few_queries(int kt) { return kt == 4 ? 8192 : kFewQueries; }
constexpr int kCosMaxAcc = 32639;   // |a| bound of the two-byte split
constexpr int kCosMaxF6 = 255;      // of the two FP6 digits
enum CosFlag : int32_t { COS_OUT_OF_RANGE = 0, COS_I8 = 1, COS_F6 = 2 };

struct CosLayout {
    int w_lo, w_hi, nwin, KT;
    size_t off_T, off_rinv, off_amax, off_flag, total;
    CosLayout(int start, int end, int K)
    {
        w_lo = (start >> 6) & ~1;
        w_hi = (end + 63) >> 6;
        nwin = (w_hi - w_lo + kCosWin - 1) / kCosWin;
        KT = class_tiles(K);
        off_T = (size_t)nwin * kCosWin * 4 * KT * 1024;
        off_rinv = off_T + 128 * 8;
        off_amax = off_rinv + 128 * 8;
        off_flag = off_amax + 128 * 4;
        total = off_flag + 16;
    }
};

size_t cos_workspace_bytes(int start, int end, int K) { return CosLayout(start, end, K).total; }

__device__ __forceinline__ bool in_set(int64_t d, int start, int end, int stride)
{
    return d >= start && d < end && (d - start) % stride == 0;
}

// The FP6 operand of (word, class tile, lane), both digits: index idx counts the
// entries of the int8 table (four per word, tile and lane); here one of the four
// works.  A lane's 32 entries are one run of its class's sums: read without
// branches (those outside the set read one inside and count 0), all in flight
// (entry by entry, each digit for itself and with a remainder by the stride: 100
// classes x 16384 35 us, 8 so).
__device__ __forceinline__ void f6_entry(const int32_t *__restrict__ acc, int K, int64_t lda, int start, int end,
                                         int stride, int w_lo, int KT, int64_t idx, int8_t *__restrict__ tab)
{
    const int lane = (int)(idx & 63);
    const int kt = (int)((idx >> 6) % KT);
    const int64_t whp = (idx >> 6) / KT;
    if (whp & 3)
        return;
    const int64_t wi = whp >> 2;
    const int k = kt * 32 + (lane & 31), g = lane >> 5;
    const int d0 = (int)((w_lo + wi) * 64) + 32 * g;
    uint32_t o[2][6] = {};
    const uint32_t m = k < K ? set_mask(d0, start, end, stride) : 0u;
    if (m) {
        const int32_t *row = acc + k * lda + d0;
        const int in = __builtin_ctz(m);
        int a[32];
        if (m == ~0u) {   // (16-byte loads at 4-byte alignment)
            typedef int v4i4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
            for (int j = 0; j < 32; j += 4) {
                const v4i4 v = *(const v4i4 *)(row + j);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    a[j + e] = v[e];
            }
        } else {
#pragma unroll
            for (int j = 0; j < 32; ++j)
                a[j] = row[(m >> j) & 1u ? j : in];
        }
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const int j = 4 * (i & 7) + (i >> 3), bit = 6 * i;
            const int v = (m >> j) & 1u ? a[j] : 0;
            const uint32_t u = (uint32_t)(v < 0 ? -v : v), sign = v < 0 ? 0x20u : 0u;
#pragma unroll
            for (int part = 0; part < 2; ++part) {
                const uint32_t c = (part ? u >> 4 : u & 15u) | sign;
                o[part][bit >> 5] |= c << (bit & 31);
                if ((bit & 31) > 26)
                    o[part][(bit >> 5) + 1] |= c >> (32 - (bit & 31));
            }
        }
    }
    int8_t *word = tab + wi * (3072 * KT);
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        *(uint4 *)(word + (part * KT + kt) * 1024 + lane * 16) = make_uint4(o[part][0], o[part][1], o[part][2], o[part][3]);
        *(uint2 *)(word + 2048 * KT + (part * KT + kt) * 512 + lane * 8) = make_uint2(o[part][4], o[part][5]);
    }
}

__global__ __launch_bounds__(256) void k_cos_table(const int32_t *__restrict__ acc, int K, int64_t lda, int start,
                                                   int end, int stride, int w_lo, int KT, int64_t total,
                                                   const int32_t *__restrict__ flag, int8_t *__restrict__ tab)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total)
        return;
    if (flag[0] == COS_F6) {
        f6_entry(acc, K, lda, start, end, stride, w_lo, KT, idx, tab);
        return;
    }
    const int lane = (int)(idx & 63);
    const int kt = (int)((idx >> 6) % KT);
    const int64_t whp = (idx >> 6) / KT;   // (word * 2 + half) * 2 + part
    const int part = (int)(whp & 1);
    const int h = (int)((whp >> 1) & 1);
    const int64_t w = w_lo + (whp >> 2);
    const int k = kt * 32 + (lane & 31), g = lane >> 5;
    uint32_t o[4] = {0, 0, 0, 0};
    if (k < K) {
#pragma unroll
        for (int b = 0; b < 16; ++b) {
            const int64_t d = w * 64 + 32 * h + 4 * g + (b >> 2) + 8 * (b & 3);
            if (in_set(d, start, end, stride)) {
                const int a = acc[k * lda + d];
                const int hi = (a + 128) >> 8;
                const int v = part ? hi : a - 256 * hi;
                o[b >> 2] |= ((uint32_t)v & 0xffu) << (8 * (b & 3));
            }
        }
    }
    *(uint4 *)(tab + idx * 16) = make_uint4(o[0], o[1], o[2], o[3]);
}

// T_k, rinv_k and max |a_kd| over S, one workgroup per class (classes past
// K get 0).  It is the first to read the sums: eight loads in flight a thread (one:
// 100 classes x 16384 20 us, 7.5 so).
__global__ __launch_bounds__(256) void k_cos_norms(const int32_t *__restrict__ acc, int K, int64_t lda, int start,
                                                   int end, int stride, int64_t *__restrict__ T,
                                                   double *__restrict__ rinv, int32_t *__restrict__ amax)
{
    __shared__ long long ps[256], pq[256], pm[256];
    const int k = blockIdx.x, t = threadIdx.x;
    long long s = 0, q = 0, m = 0;
    if (k < K)
        for (int64_t d = start + (int64_t)t * stride; d < end; d += (int64_t)(8 * 256) * stride) {
            int v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t du = d + (int64_t)(u * 256) * stride;
                v[u] = acc[k * lda + (du < end ? du : d)];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const long long a = d + (int64_t)(u * 256) * stride < end ? v[u] : 0;
                s += a;
                q += a * a;
                m = a > m ? a : (-a > m ? -a : m);
            }
        }
    ps[t] = s;
    pq[t] = q;
    pm[t] = m;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) {
            ps[t] += ps[t + h];
            pq[t] += pq[t + h];
            pm[t] = pm[t + h] > pm[t] ? pm[t + h] : pm[t];
        }
        __syncthreads();
    }
    if (t == 0) {
        T[k] = ps[0];
        rinv[k] = pq[0] > 0 ? __ddiv_rn(1.0, __dsqrt_rn((double)pq[0])) : 0.0;
        amax[k] = pm[0] > INT_MAX ? INT_MAX : (int32_t)pm[0];
    }
}

__global__ __launch_bounds__(128) void k_cos_flag(const int32_t *__restrict__ amax, int32_t *__restrict__ flag)
{
    __shared__ int bad, wide;
    if (threadIdx.x == 0)
        bad = wide = 0;
    __syncthreads();
    if (amax[threadIdx.x] > kCosMaxAcc)
        atomicOr(&bad, 1);
    if (amax[threadIdx.x] > kCosMaxF6)
        atomicOr(&wide, 1);
    __syncthreads();
    if (threadIdx.x == 0)
        flag[0] = bad ? COS_OUT_OF_RANGE : wide ? COS_I8 : COS_F6;
}

// Query bits as bytes {0, 1}: register r of lane half g holds, in byte i,
// bit 4g + r + 8i of the dword (two operations per register).
__device__ __forceinline__ v4i spread_bits(uint32_t d, uint32_t sh)
{
    const uint32_t e = d >> sh;
    v4i b;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        b[r] = (int)((e >> r) & 0x01010101u);
    return b;
}

// One search on the int8 operand: the workgroup's CosShape ROWS queries from
// rbase.
template <int KT, int QT_>
__device__ __forceinline__ void cosine_i8(uint8_t *smem, int64_t rbase, const uint64_t *__restrict__ Q, int64_t n,
                                          int64_t ldq, int K, int w_lo, int w_hi, int nwin,
                                          const int8_t *__restrict__ tab, const int64_t *__restrict__ T,
                                          const double *__restrict__ rinv, const int32_t *__restrict__ flag,
                                          int32_t *__restrict__ label, double *__restrict__ max_score,
                                          double *__restrict__ scores)
{
    typedef CosShape<KT, QT_> S;
    constexpr int QT = S::QT, W = S::W, NST = S::NST;
    constexpr int G = S::NQL + S::NTL;                 // loads per window and wave
    lds_u8 *L = (lds_u8 *)smem;
    const int lane = threadIdx.x & 63, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t sh = 4u * (uint32_t)g;
    const uint64_t *Qwg = Q + rbase * ldq;

    // query loads: load i of a wave fills rows RPL*j .. (j = i*4 + wave),
    // lane l -> row RPL*j + l/U, unit l%U of the window (rows past n
    // re-read row n-1; 16-byte units of 2 words, no swizzle needed for the
    // 8-byte reads below)
    int qrow[S::NQL], qunit[S::NQL];
#pragma unroll
    for (int i = 0; i < S::NQL; ++i) {
        const int j = i * kWaves + wave;
        int r = S::RPL * j + lane / S::U;
        qunit[i] = lane % S::U;
        if (rbase + r >= n)
            r = (int)(n - 1 - rbase);
        qrow[i] = r;
    }
    auto issue = [&](int v, int st) {
        const int vc = v < nwin ? v : nwin - 1;
        lds_u8 *sq = L + st * S::SB;
#pragma unroll
        for (int i = 0; i < S::NQL; ++i) {
            int w = w_lo + vc * W + 2 * qunit[i];
            if (w >= w_hi)
                w = w_lo;
            if (S::QB % (1024 * kWaves) == 0 || (i * kWaves + wave) * 1024 < S::QB)
                lds_dma16(Qwg, (uint32_t)(((int64_t)qrow[i] * ldq + w) * 8), sq + (i * kWaves + wave) * 1024);
        }
#pragma unroll
        for (int i = 0; i < S::NTL; ++i) {
            const int j = i * kWaves + wave;
            lds_dma16(tab, (uint32_t)(vc * S::TB + j * 1024 + lane * 16), sq + S::QB + j * 1024);
        }
    };

    v16i alo[KT][QT], ahi[KT][QT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            alo[kt][qt] = v16i{};
            ahi[kt][qt] = v16i{};
        }

    // ring of NST stages: window v lives in stage v % NST; loads run NST-1
    // windows ahead, and vector memory operations complete in order, so
    // vmcnt(G*(NST-2)) leaves only the newer windows in flight
#pragma unroll
    for (int v = 0; v < NST - 1; ++v)
        issue(v, v);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(G * (NST - 2)) : "memory");
    int st = 0;
    for (int v = 0; v < nwin; ++v) {
        issue(v + NST - 1, st == 0 ? NST - 1 : st - 1);
        const lds_u8 *sq = L + st * S::SB;
        const lds_u8 *stb = sq + S::QB;
#pragma unroll
        for (int ww = 0; ww < W; ++ww) {
            uint64_t q[QT];
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) {
                const int r = (wave * QT + qt) * 32 + (lane & 31);
                q[qt] = *(const HDC_LDS uint64_t *)(sq + (r * W + ww) * 8);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v4i flo[KT], fhi[KT];
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    flo[kt] = *(const lds_v4i *)(stb + ((((ww * 2 + h) * 2 + 0) * KT + kt) * 64 + lane) * 16);
                    fhi[kt] = *(const lds_v4i *)(stb + ((((ww * 2 + h) * 2 + 1) * KT + kt) * 64 + lane) * 16);
                }
#pragma unroll
                for (int qt = 0; qt < QT; ++qt) {
                    const v4i bf = spread_bits(h ? (uint32_t)(q[qt] >> 32) : (uint32_t)q[qt], sh);
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt) {
                        alo[kt][qt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(flo[kt], bf, alo[kt][qt], 0, 0, 0);
                        ahi[kt][qt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fhi[kt], bf, ahi[kt][qt], 0, 0, 0);
                    }
                }
            }
        }
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(G * (NST - 2)) : "memory");
        st = st == NST - 1 ? 0 : st + 1;
    }
    __builtin_amdgcn_s_waitcnt(0);

    // argmax: lane holds query l%32 of each tile and classes 8(v/4)+4g+v%4
    const bool in_range = flag[0] != 0;
    const double nan = __builtin_nan("");
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        const int64_t q = rbase + (wave * QT + qt) * 32 + (lane & 31);
        double best = -1.0 / 0.0;
        int bk = 0;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = kt * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                if (k < K) {
                    const long long s = 256ll * ahi[kt][qt][v] + alo[kt][qt][v];
                    const double sc = in_range ? __dmul_rn((double)(T[k] - 2 * s), rinv[k]) : nan;
                    if (sc > best) { best = sc; bk = k; }
                    if (scores && q < n)
                        scores[q * K + k] = sc;
                }
            }
        const double ob = __shfl_xor(best, 32);
        const int obk = __shfl_xor(bk, 32);
        if (ob > best || (ob == best && obk < bk)) { best = ob; bk = obk; }
        if (g == 0 && q < n) {
            label[q] = in_range ? bk : -1;
            if (max_score)
                max_score[q] = in_range ? best : nan;
        }
    }
}

// The search on the FP6 operand (flag 2).  With one class tile eight words a
// window: a row's 64 bytes, half a line; with four the search of queries that
// come from HBM reads each line four times over (147537 x 8292 against 14
// classes: 102 us, 78 with eight).
template <int KT, int QT_> struct F6Shape {
    static constexpr int QT = QT_;
    static constexpr int W = 8 / KT;                   // words per window (divides kCosWin)
    static constexpr int U = W / 2;                    // 16-byte units per query row
    static constexpr int RPL = 64 / U;                 // query rows per 1 KiB load
    static constexpr int ROWS = kWaves * QT * 32;      // queries per workgroup
    static constexpr int QB = ROWS * W * 8;            // query bytes per stage
    static constexpr int WB = 3072 * KT;               // operand bytes per word
    static constexpr int TB = W * WB;
    static constexpr int NST = 2;
    // loads per wave (a short last one: its waves past QB load nothing)
    static constexpr int NQL = (QB / 1024 + kWaves - 1) / kWaves;
    static constexpr int NTL = TB / 1024 / kWaves;
    static constexpr int SB = QB + TB;
    // unit hh of row r sits in slot hh ^ (r / 8 % U): 16 rows' reads on
    // distinct banks
    static __device__ __forceinline__ int slot(int r, int hh) { return hh ^ ((r >> 3) & (U - 1)); }
};

template <int KT, int QT_>
__device__ __forceinline__ void cosine_f6(uint8_t *smem, int64_t rbase, const uint64_t *__restrict__ Q, int64_t n,
                                          int64_t ldq, int K, int w_lo, int w_hi, int nwin,
                                          const int8_t *__restrict__ tab, const int64_t *__restrict__ T,
                                          const double *__restrict__ rinv, int32_t *__restrict__ label,
                                          double *__restrict__ max_score, double *__restrict__ scores)
{
    typedef F6Shape<KT, QT_> S;
    constexpr int QT = S::QT, W = S::W;
    lds_u8 *L = (lds_u8 *)smem;
    const int lane = threadIdx.x & 63, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t *Qwg = Q + rbase * ldq;

    // query loads: load i of a wave fills rows RPL*j .. (j = i*4 + wave);
    // rows past n re-read row n-1, words past w_hi the first pair
    uint32_t qoff[S::NQL];
    int qunit[S::NQL];
#pragma unroll
    for (int i = 0; i < S::NQL; ++i) {
        const int r = S::RPL * (i * kWaves + wave) + lane / S::U;
        qunit[i] = 2 * S::slot(r, lane % S::U);
        qoff[i] = (uint32_t)((rbase + r < n ? r : n - 1 - rbase) * ldq * 8);
    }
    auto issue = [&](int v, int st) {
        const int vc = v < nwin ? v : nwin - 1;
        lds_u8 *sq = L + st * S::SB;
#pragma unroll
        for (int i = 0; i < S::NQL; ++i) {
            const int w = w_lo + vc * W + qunit[i];
            if ((i * kWaves + wave) * 1024 < S::QB)
                lds_dma16(Qwg, qoff[i] + 8u * (uint32_t)(w < w_hi ? w : w_lo), sq + (i * kWaves + wave) * 1024);
        }
#pragma unroll
        for (int i = 0; i < S::NTL; ++i)
            lds_dma16(tab + (int64_t)vc * S::TB + (i * kWaves + wave) * 1024, (uint32_t)lane * 16,
                      sq + S::QB + (i * kWaves + wave) * 1024);
    };

    v16f acc[KT][QT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
            acc[kt][qt] = v16f{};
    issue(0, 0);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    int st = 0;
    for (int v = 0; v < nwin; ++v) {
        issue(v + 1, st ^ 1);
        const lds_u8 *sq = L + st * S::SB;
        const lds_u8 *stb = sq + S::QB;
        v4i qv[QT][S::U];
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            const int r = (wave * QT + qt) * 32 + (lane & 31);
#pragma unroll
            for (int hh = 0; hh < S::U; ++hh)
                qv[qt][hh] = *(const lds_v4i *)(sq + r * (W * 8) + 16 * S::slot(r, hh));
        }
#pragma unroll
        for (int ww = 0; ww < W; ++ww) {
            v8i bf[QT];
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) {
                const v4i u = qv[qt][ww >> 1];
                bf[qt] = query_nibbles((uint32_t)(g ? u[2 * (ww & 1) + 1] : u[2 * (ww & 1)]));
            }
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int part = 0; part < 2; ++part) {
                    typedef int v2i __attribute__((ext_vector_type(2)));
                    const lds_u8 *e = stb + ww * S::WB;
                    const v4i lo = *(const lds_v4i *)(e + (part * KT + kt) * 1024 + lane * 16);
                    const v2i hi = *(const HDC_LDS v2i *)(e + 2048 * KT + (part * KT + kt) * 512 + lane * 8);
                    const v8i af = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], 0, 0};
                    // A: E2M3 (format 2) scaled by 2^4 or 2^8, B: E2M1 (4)
#pragma unroll
                    for (int qt = 0; qt < QT; ++qt)
                        acc[kt][qt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                            af, bf[qt], acc[kt][qt], 2, 4, 0, part ? 127 + 8 : 127 + 4, 0, 127);
                }
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        st ^= 1;
    }

    // argmax: lane holds query l%32 of each tile and classes 8(v/4)+4g+v%4
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        const int64_t q = rbase + (wave * QT + qt) * 32 + (lane & 31);
        double best = -1.0 / 0.0;
        int bk = 0;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = kt * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                if (k < K) {
                    const long long sum = (long long)(int)acc[kt][qt][v];
                    const double sc = __dmul_rn((double)(T[k] - 2 * sum), rinv[k]);
                    if (sc > best) { best = sc; bk = k; }
                    if (scores && q < n)
                        scores[q * K + k] = sc;
                }
            }
        const double ob = __shfl_xor(best, 32);
        const int obk = __shfl_xor(bk, 32);
        if (ob > best || (ob == best && obk < bk)) { best = ob; bk = obk; }
        if (g == 0 && q < n) {
            label[q] = bk;
            if (max_score)
                max_score[q] = best;
        }
    }
}

// The streaming search on the operand _prepare chose.  Two workgroups per CU:
// one's LDS waits and barriers under the other's MFMAs.  100003 x 16384
// against 100 classes: 518 us on the int8 operand (its four products per 64
// dimensions and class tile the bound), 218 on FP6, the matrix cores busy 0.43 of
// the cycles, the rest the operand's LDS reads (24 bytes per lane and two
// products) and the barriers.  One kernel for both operands: a launch of each, the
// unwanted one returning at once, cost 2 us.
template <int KT, int QT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_cosine(const uint64_t *__restrict__ Q, int64_t n, int64_t ldq, int K, int w_lo, int w_hi, int words,
              const int8_t *__restrict__ tab, const int64_t *__restrict__ T, const double *__restrict__ rinv,
              const int32_t *__restrict__ flag, int32_t *__restrict__ label, double *__restrict__ max_score,
              double *__restrict__ scores)
{
    typedef CosShape<KT, QT> S8;
    typedef F6Shape<KT, QT> S6;
    constexpr int B8 = S8::NST * S8::SB, B6 = S6::NST * S6::SB;
    __shared__ __align__(16) uint8_t smem[B8 > B6 ? B8 : B6];
    const int64_t rbase = (int64_t)blockIdx.x * S6::ROWS;
    if (flag[0] == COS_F6) {
        cosine_f6<KT, QT>(smem, rbase, Q, n, ldq, K, w_lo, w_hi, words / S6::W, tab, T, rinv, label, max_score, scores);
        return;
    }
    for (int64_t r = rbase; r < rbase + S6::ROWS && r < n; r += S8::ROWS) {
        cosine_i8<KT, QT>(smem, r, Q, n, ldq, K, w_lo, w_hi, words / S8::W, tab, T, rinv, flag, label, max_score, scores);
        __syncthreads();   // LDS reads done before the next rows' loads
    }
}

// The search of few queries (see few_pairs) on either operand: one kernel, the
// sums of the int8 parts taken as 256 * hi + lo.
template <int KT>
__global__ __launch_bounds__(256) void k_cosine_few(const uint64_t *__restrict__ Q, int64_t n, int64_t ldq, int K,
                                                    int w_lo, int w_hi, const int8_t *__restrict__ tab,
                                                    const int64_t *__restrict__ T, const double *__restrict__ rinv,
                                                    const int32_t *__restrict__ flag, int32_t *__restrict__ label,
                                                    double *__restrict__ max_score, double *__restrict__ scores)
{
    __shared__ long long sums[KT * 32][33];
    __shared__ double best[8][32];
    __shared__ int bestk[8][32];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 5;
    const int fl = flag[0];
    long long s[KT][16];
    if (fl == COS_F6) {
        v16f acc[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
            acc[kt] = v16f{};
        few_pairs(Q, n, ldq, w_lo, w_hi, [&](int p, int p1, const v4i (&u)[kFewPairs]) {
#pragma unroll
            for (int i = 0; i < kFewPairs; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    typedef int v2i __attribute__((ext_vector_type(2)));
                    const int w = 2 * (p + i < p1 ? p + i : p1 - 1) + h;
                    const int8_t *e = tab + (int64_t)w * (3072 * KT);
                    const v8i bf = query_nibbles((uint32_t)(g ? u[i][2 * h + 1] : u[i][2 * h]));
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                        for (int part = 0; part < 2; ++part) {
                            const v4i lo = *(const v4i *)(e + (part * KT + kt) * 1024 + lane * 16);
                            const v2i hi = *(const v2i *)(e + 2048 * KT + (part * KT + kt) * 512 + lane * 8);
                            acc[kt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], 0, 0}, bf, acc[kt], 2, 4, 0,
                                part ? 127 + 8 : 127 + 4, 0, 127);
                        }
                }
        });
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                s[kt][v] = (long long)(int)acc[kt][v];
    } else {
        v16i alo[KT], ahi[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            alo[kt] = v16i{};
            ahi[kt] = v16i{};
        }
        few_pairs(Q, n, ldq, w_lo, w_hi, [&](int p, int p1, const v4i (&u)[kFewPairs]) {
#pragma unroll
            for (int i = 0; i < kFewPairs; ++i)
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const int64_t wh = 4 * (int64_t)(p + i < p1 ? p + i : p1 - 1) + h;   // dword of the words
                    const v4i bf = spread_bits((uint32_t)u[i][h], 4u * (uint32_t)g);
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt) {
                        const v4i lo = *(const v4i *)(tab + (((wh * 2) * KT + kt) * 64 + lane) * 16);
                        const v4i hi = *(const v4i *)(tab + (((wh * 2 + 1) * KT + kt) * 64 + lane) * 16);
                        alo[kt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(lo, bf, alo[kt], 0, 0, 0);
                        ahi[kt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(hi, bf, ahi[kt], 0, 0, 0);
                    }
                }
        });
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                s[kt][v] = 256ll * ahi[kt][v] + alo[kt][v];
    }
    // the waves' sums, one after the other
    for (int w = 0; w < kWaves; ++w) {
        if (wave == w) {
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    long long &x = sums[kt * 32 + 8 * (v >> 2) + 4 * g + (v & 3)][lane & 31];
                    x = w == 0 ? s[kt][v] : x + s[kt][v];
                }
        }
        __syncthreads();
    }
    const int c = t & 31, slot = t >> 5;
    const int64_t q = (int64_t)blockIdx.x * 32 + c;
    const bool in_range = fl != COS_OUT_OF_RANGE;
    const double nan = __builtin_nan("");
    double b = -1.0 / 0.0;
    int bk = 0;
    for (int k = slot; k < K; k += 8) {
        const double sc = in_range ? __dmul_rn((double)(T[k] - 2 * sums[k][c]), rinv[k]) : nan;
        if (sc > b) {
            b = sc;
            bk = k;
        }
        if (scores && q < n)
            scores[q * K + k] = sc;
    }
    best[slot][c] = b;
    bestk[slot][c] = bk;
    __syncthreads();
    if (t < 32 && q < n) {
#pragma unroll
        for (int w = 1; w < 8; ++w)
            if (best[w][c] > b || (best[w][c] == b && bestk[w][c] < bk)) {
                b = best[w][c];
                bk = bestk[w][c];
            }
        label[q] = in_range ? bk : -1;
        if (max_score)
            max_score[q] = in_range ? b : nan;
    }
}

hipError_t launch_cos_prepare(const int32_t *acc, int K, int64_t lda, int start, int end, int stride, uint8_t *ws,
                              hipStream_t st)
{
    const CosLayout L(start, end, K);
    const int64_t total = (int64_t)L.nwin * kCosWin * 4 * L.KT * 64;
    hipLaunchKernelGGL(k_cos_norms, dim3(128), dim3(256), 0, st, acc, K, lda, start, end, stride,
                       (int64_t *)(ws + L.off_T), (double *)(ws + L.off_rinv), (int32_t *)(ws + L.off_amax));
    hipLaunchKernelGGL(k_cos_flag, dim3(1), dim3(128), 0, st, (const int32_t *)(ws + L.off_amax),
                       (int32_t *)(ws + L.off_flag));
    hipLaunchKernelGGL(k_cos_table, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, acc, K, lda, start, end,
                       stride, L.w_lo, L.KT, total, (const int32_t *)(ws + L.off_flag), (int8_t *)ws);
    return hipGetLastError();
}

hipError_t launch_cos_prepared(const uint64_t *Q, int64_t n, int64_t ldq, int K, int start, int end,
                               const uint8_t *ws, int32_t *label, double *max_score, double *scores, hipStream_t st)
{
    const CosLayout L(start, end, K);
    const int8_t *tab = (const int8_t *)ws;
    const int64_t *T = (const int64_t *)(ws + L.off_T);
    const double *rinv = (const double *)(ws + L.off_rinv);
    const int32_t *flag = (const int32_t *)(ws + L.off_flag);
#define HDC_COS_CASE(KT_)                                                                                      \
    if (L.KT == KT_ && n <= cos_few_queries(KT_)) {                                                             \
        hipLaunchKernelGGL(k_cosine_few<KT_>, dim3((unsigned)((n + 31) / 32)), dim3(256), 0, st, Q, n, ldq, K,   \
                           L.w_lo, L.w_hi, tab, T, rinv, flag, label, max_score, scores);                      \
        return hipGetLastError();                                                                              \
    }                                                                                                          \
    if (L.KT == KT_ && n <= kCosNarrow) {                                                                      \
        hipLaunchKernelGGL((k_cosine<KT_, 1>), dim3((unsigned)((n + 127) / 128)), dim3(256), 0, st, Q, n, ldq,   \
                           K, L.w_lo, L.w_hi, L.nwin * kCosWin, tab, T, rinv, flag, label, max_score, scores); \
        return hipGetLastError();                                                                              \
    }                                                                                                          \
    if (L.KT == KT_) {                                                                                         \
        hipLaunchKernelGGL((k_cosine<KT_, 2>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, Q, n, ldq,   \
                           K, L.w_lo, L.w_hi, L.nwin * kCosWin, tab, T, rinv, flag, label, max_score, scores); \
        return hipGetLastError();                                                                              \
    }
    HDC_COS_CASE(1)
    HDC_COS_CASE(2)
    HDC_COS_CASE(4)
#undef HDC_COS_CASE
    return hipErrorInvalidValue;
}

}  // namespace hdc
