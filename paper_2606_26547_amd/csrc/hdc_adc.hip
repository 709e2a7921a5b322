// ADC-chunked dot-product similarity: the similarity an in-memory
// accelerator computes when every 128-element array chunk's partial dot
// product is digitised by an ADC before accumulation.  For query i, class k
// and chunk c (dimensions [128c, 128c+128) that lie in S), the partial of
// the bipolar vectors is s = n_c - 2 * popc((q ^ c_k) & mask), n_c the
// chunk's dimensions in S; the ADC maps s to value(s) (clip to [floor,
// ceil], nearest of 2^res levels floor + step*j, ties up), read from a
// 257-entry table in LDS; score = sum of values, label = first class with
// the largest score.  One query per lane, 16-word windows (8 chunks) of the
// queries and of the masked class words staged through LDS as in the
// Hamming kernel.
#include <limits.h>

#include "hdc_stream.h"

namespace hdc {

constexpr int kAdcWin = 16;            // words per window (8 chunks)
constexpr int kAdcMaxWords = 1024;     // hypervectors up to 65536 bits

template <int KB>
__global__ __launch_bounds__(256) void k_adc_argmax(const uint64_t *__restrict__ Q, int64_t n, int64_t ldq,
                                                    const uint64_t *__restrict__ C, int K, int64_t ldc, int start,
                                                    int end, int stride, int res, int step, int floor_, int ceil_,
                                                    int32_t *__restrict__ label, int32_t *__restrict__ max_score,
                                                    int32_t *__restrict__ scores)
{
    __shared__ uint64_t qs[kWaves][64][kAdcWin + 1];
    __shared__ uint64_t cls[KB][kAdcWin];
    __shared__ uint64_t msk[kAdcMaxWords];
    __shared__ int lut[257];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int w_lo = (start >> 7) * 2, w_hi = (end + 63) >> 6;   // chunk-aligned first word
    for (int w = w_lo + t; w < w_hi; w += 256) {
        uint64_t m = 0;
        const int64_t lo = (int64_t)w * 64 > start ? (int64_t)w * 64 : start;
        const int64_t hi = (int64_t)w * 64 + 64 < end ? (int64_t)w * 64 + 64 : end;
        for (int64_t d = start + ((lo - start + stride - 1) / stride) * (int64_t)stride; d < hi; d += stride)
            m |= 1ull << (d & 63);
        msk[w - w_lo] = m;
    }
    for (int i = t; i < 257; i += 256) {   // value of every partial s in [-128, 128]
        const int s = i - 128;
        const int64_t x = s < floor_ ? floor_ : (s > ceil_ ? ceil_ : s);
        int64_t code = (2 * (x - floor_) + step) / (2 * (int64_t)step);
        const int64_t top = (1ll << res) - 1;
        if (code > top)
            code = top;
        lut[i] = (int)(floor_ + step * code);
    }

    const int64_t rbase = (int64_t)blockIdx.x * 256 + wave * 64;
    int sc[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k)
        sc[k] = 0;

    for (int w0 = w_lo; w0 < w_hi; w0 += kAdcWin) {
        __syncthreads();   // masks / table ready, previous window consumed
#pragma unroll
        for (int p = 0; p < 16; ++p) {
            const int r = 4 * p + (lane >> 4), ww = lane & 15;
            const int64_t row = rbase + r;
            uint64_t v = 0;
            if (row < n && w0 + ww < w_hi)
                v = Q[row * ldq + w0 + ww];
            qs[wave][r][ww] = v;
        }
        for (int i = t; i < KB * kAdcWin; i += 256) {
            const int k = i / kAdcWin, ww = i % kAdcWin;
            uint64_t v = 0;
            if (k < K && w0 + ww < w_hi)
                v = C[(int64_t)k * ldc + w0 + ww] & msk[w0 + ww - w_lo];
            cls[k][ww] = v;
        }
        __syncthreads();
        for (int cc = 0; cc < kAdcWin / 2; ++cc) {
            const int wa = w0 + 2 * cc;
            const uint64_t m0 = wa < w_hi ? msk[wa - w_lo] : 0ull;
            const uint64_t m1 = wa + 1 < w_hi ? msk[wa + 1 - w_lo] : 0ull;
            const int nc = __popcll(m0) + __popcll(m1);
            if (nc == 0)   // uniform: a chunk without a dimension of S is not converted
                continue;
            const uint64_t q0 = qs[wave][lane][2 * cc] & m0, q1 = qs[wave][lane][2 * cc + 1] & m1;
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                const int h = __popcll(q0 ^ cls[k][2 * cc]) + __popcll(q1 ^ cls[k][2 * cc + 1]);
                sc[k] += lut[nc - 2 * h + 128];
            }
        }
    }

    const int64_t row = rbase + lane;
    if (row >= n)
        return;
    int best = INT_MIN, bk = 0;
#pragma unroll
    for (int k = 0; k < KB; ++k)
        if (k < K) {
            if (sc[k] > best) { best = sc[k]; bk = k; }
            if (scores)
                scores[row * K + k] = sc[k];
        }
    label[row] = bk;
    if (max_score)
        max_score[row] = best;
}

#define HDC_ADC_CASE(KB_)                                                                                      \
    if (K <= KB_) {                                                                                            \
        hipLaunchKernelGGL(k_adc_argmax<KB_>, grid, block, 0, st, Q, n, ldq, C, K, ldc, start, end, stride, res, \
                           step, floor_, ceil_, label, max_score, scores);                                     \
        return hipGetLastError();                                                                              \
    }

hipError_t launch_adc_argmax(const uint64_t *Q, int64_t n, int64_t ldq, const uint64_t *C, int K, int64_t ldc,
                             int start, int end, int stride, int res, int step, int floor_, int ceil_,
                             int32_t *label, int32_t *max_score, int32_t *scores, hipStream_t st)
{
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    HDC_ADC_CASE(4)
    HDC_ADC_CASE(12)
    HDC_ADC_CASE(28)
    HDC_ADC_CASE(64)
    HDC_ADC_CASE(128)
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------ prepared
// The same similarity on the matrix cores.  Each chunk partial s is the
// FP4 product of the bipolar query (+-1.0 nibbles) with the class signs
// (+-1.0, 0 outside S) over the chunk's two words: two 32x32x64 MFMAs into
// a fresh fp32 accumulator (|s| <= 128, exact), then every partial goes
// through the ADC table and adds to an int32 score; chunks with no
// dimension of S (uniform) are skipped.  Streaming as in the prepared
// Hamming search (query words and class operand windows into an LDS ring).
//
// Workspace: the class operand (k_sign_table with codes +-1.0) from the
// chunk-aligned word w_lo = 2*floor(start/128), padded to whole windows,
// then the number of dimensions of S in each chunk (int32).
struct AdcLayout {
    int w_lo, w_hi, nwin, KT;
    size_t off_nc, total;
    AdcLayout(int start, int end, int K)
    {
        w_lo = (start >> 7) * 2;
        w_hi = (end + 63) >> 6;
        nwin = (w_hi - w_lo + kHmWin - 1) / kHmWin;
        KT = class_tiles(K);
        off_nc = (size_t)nwin * kHmWin * KT * 1024;
        total = off_nc + (size_t)nwin * (kHmWin / 2) * 4;
    }
};

size_t adc_workspace_bytes(int start, int end, int K) { return AdcLayout(start, end, K).total; }

__global__ __launch_bounds__(256) void k_adc_chunks(int start, int end, int stride, int c_lo, int nchunk,
                                                    int32_t *__restrict__ nc)
{
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= nchunk)
        return;
    const int64_t lo = (int64_t)(c_lo + c) * 128, hi = lo + 128;
    int cnt = 0;
    if (hi > start && lo < end) {
        const int64_t a = lo > start ? lo : start, b = hi < end ? hi : end;
        const int64_t first = start + (a - start + stride - 1) / stride * (int64_t)stride;
        if (first < b)
            cnt = (int)((b - 1 - first) / stride + 1);
    }
    nc[c] = cnt;
}

hipError_t launch_adc_prepare(const uint64_t *C, int K, int64_t ldc, int start, int end, int stride, uint8_t *ws,
                              hipStream_t st)
{
    const AdcLayout L(start, end, K);
    const int64_t total = (int64_t)L.nwin * kHmWin * L.KT * 64;
    // E2M1 +1.0 / -1.0
    hipLaunchKernelGGL((k_sign_table<0x2u, 0xAu>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, C, K,
                       ldc, start, end, stride, L.w_lo, L.KT, total, (int8_t *)ws, (int32_t *)nullptr);
    const int nchunk = L.nwin * (kHmWin / 2);
    hipLaunchKernelGGL(k_adc_chunks, dim3((unsigned)((nchunk + 255) / 256)), dim3(256), 0, st, start, end, stride,
                       L.w_lo / 2, nchunk, (int32_t *)(ws + L.off_nc));
    return hipGetLastError();
}

// The converter.  A table read per partial kept LDS busy (16 reads of 64
// scattered words per chunk and tile), so partials go through packed
// half-precision arithmetic where that gives the table's value for every one
// of the 257 partials (checked by each workgroup, entry by entry; else the
// table is read): with code = round((x - floor) / step) of the clipped partial
// x, at most cmax,
//     t = clamp(s * k + c, 0, 1),   1024 + code = t * r + 1024 (rounded to the
// integer by the addition), r = min((ceil - floor) / step, 2^res - 1), two
// partials per operation, four operations.  The 16-bit patterns 0x6400 + code
// are summed as integers for up to kAdcFlush chunks (1023 * 64 < 2^16) and
// then added to the 32-bit code sums; score = floor * chunks + step * codes.
// 262144 x 10240 against 26 classes, 6 bits: 132 us by the table, 106 so; the
// conversion's vector operations, four a partial, bound it.
constexpr int kAdcFlush = 64;
// (see few_pairs; 24000 x 10240 against 26 classes: 37 us streaming, 21 so; 16384
// x 8192 against 100, from where on the few-queries kernel only grows: 45 and 45)
constexpr int64_t adc_few_queries(int kt) { return kt == 1 ? 32768 : 16384; }
struct AdcConv {
    uint32_t k, c, r;            // each a packed pair of one half
    static __device__ __forceinline__ uint32_t pair(float x)
    {
        typedef __fp16 h2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(uint32_t, h2{(__fp16)x, (__fp16)x});
    }
    __device__ __forceinline__ AdcConv(int res, int step, int floor_, int ceil_)
    {
        const float top = (float)((1ll << res) - 1);
        float range = (float)((int64_t)ceil_ - floor_) / (float)step;
        range = range < top ? range : top;
        range = range > 0.0f ? range : 1.0f;
        const float inv = 1.0f / ((float)step * range);
        k = pair(inv);
        c = pair((0.25f - (float)floor_) * inv);   // a quarter step up: ties round up
        r = pair(range);
    }
    // bits of 1024 + code (halves) of two partials
    __device__ __forceinline__ uint32_t operator()(float a, float b) const
    {
        const uint32_t s = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
        uint32_t t, m;
        asm("v_pk_fma_f16 %0, %1, %2, %3 clamp" : "=v"(t) : "v"(s), "v"(k), "v"(c));
        asm("v_pk_fma_f16 %0, %1, %2, %3" : "=v"(m) : "v"(t), "v"(r), "v"(0x64006400u));
        return m;
    }
};

// Fills the table with the value of every partial s in [-128, 128]; returns
// whether the arithmetic gives all of them (a workgroup barrier).
__device__ __forceinline__ bool adc_table(int *lut, int t, const AdcConv &conv, int res, int step, int floor_,
                                          int ceil_)
{
    int ok = 1;
    for (int i = t; i < 257; i += 256) {
        const int s = i - 128;
        const int64_t x = s < floor_ ? floor_ : (s > ceil_ ? ceil_ : s);
        int64_t code = (2 * (x - floor_) + step) / (2 * (int64_t)step);
        const int64_t top = (1ll << res) - 1;
        if (code > top)
            code = top;
        lut[i] = (int)(floor_ + step * code);
        ok &= code < 1024 && conv((float)s, (float)s) == 0x64006400u + (uint32_t)code * 0x10001u;
    }
    return __syncthreads_and(ok);
}

// The code sums of one tile: 16 partials per lane in packed halves, moved to
// 32 bits every kAdcFlush chunks.
struct AdcCodes {
    uint32_t h[8];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            h[i] = 0;
    }
    __device__ __forceinline__ void add(const AdcConv &conv, const v16f &part)
    {
        typedef unsigned short v2us __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < 8; ++i)
            h[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2us, h[i]) +
                                                    __builtin_bit_cast(v2us, conv(part[2 * i], part[2 * i + 1])));
    }
    // chunks: those added since the last call
    __device__ __forceinline__ void flush(v16i &sum, int chunks)
    {
        const uint32_t base = (uint32_t)chunks * 0x6400u;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            sum[2 * i] += (int)((h[i] - base) & 0xffffu);
            sum[2 * i + 1] += (int)(((h[i] >> 16) - base) & 0xffffu);
            h[i] = 0;
        }
    }
};

// The streaming search of one workgroup, its partials converted by arithmetic or
// (not ARITH) by the table: a loop of its own each, the table's as it was before
// the arithmetic (both in one loop: 200000 x 8192 against 100 classes, 12 bits, 257
// us -> 362; so 247).
template <int KT, bool ARITH>
__device__ __forceinline__ void adc_stream(uint8_t *smem, const int *lut, const AdcConv &conv,
                                           const uint64_t *__restrict__ Q, int64_t n, int64_t ldq, int K, int w_lo,
                                           int w_hi, int nwin, const int8_t *__restrict__ tab,
                                           const int32_t *__restrict__ nc, int step, int floor_,
                                           int32_t *__restrict__ label, int32_t *__restrict__ max_score,
                                           int32_t *__restrict__ scores)
{
    typedef HmShape<KT> S;
    constexpr int QT = S::QT, W = S::W, ROWS = S::ROWS, NST = S::NST;
    // a group's tiles (registers for two waves per SIMD)
    constexpr int QG = KT == 2 || !ARITH ? 1 : QT, KG = ARITH ? KT : 1;
    lds_u8 *L = (lds_u8 *)smem;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 5;
    const int64_t rbase = (int64_t)blockIdx.x * ROWS;
    const uint64_t *Qwg = Q + rbase * ldq;

    int qrow[S::NQL], qhalf[S::NQL];
#pragma unroll
    for (int i = 0; i < S::NQL; ++i) {
        const int j = i * kWaves + wave;
        int r = S::RPL * j + lane / S::U;
        qhalf[i] = hm_slot<KT>(r, lane % S::U);
        if (rbase + r >= n)
            r = (int)(n - 1 - rbase);
        qrow[i] = r;
    }
    auto issue = [&](int v, int st) {
        const int vc = v < nwin ? v : nwin - 1;
        lds_u8 *sq = L + st * S::SB;
#pragma unroll
        for (int i = 0; i < S::NQL; ++i) {
            int w = w_lo + vc * W + 2 * qhalf[i];
            if (w >= w_hi)
                w = w_lo;
            lds_dma16(Qwg, (uint32_t)(((int64_t)qrow[i] * ldq + w) * 8), sq + (i * kWaves + wave) * 1024);
        }
#pragma unroll
        for (int i = 0; i < S::NTL; ++i) {
            const int j = i * kWaves + wave;
            lds_dma16(tab, (uint32_t)(vc * S::TB + j * 1024 + lane * 16), sq + S::QB + j * 1024);
        }
    };
    constexpr int G = S::NQL + S::NTL;

    v16i sc[KT][QT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
            sc[kt][qt] = v16i{};
    AdcCodes codes[KT][QT];   // (ARITH)
    if constexpr (ARITH) {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int qt = 0; qt < QT; ++qt)
                codes[kt][qt].clear();
    }
    int pending = 0, chunks = 0;   // chunks in codes, and converted in all
    auto flush = [&]() {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int qt = 0; qt < QT; ++qt)
                codes[kt][qt].flush(sc[kt][qt], pending);
        pending = 0;
    };

#pragma unroll
    for (int v = 0; v < NST - 1; ++v)
        issue(v, v);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(G * (NST - 2)) : "memory");

    // whether each chunk of the window is converted, read a window ahead (a
    // scalar load per chunk, waited for on the spot, held up the whole wave)
    bool conv_now[W / 2], conv_next[W / 2];
    auto read_nc = [&](int v) {
#pragma unroll
        for (int cc = 0; cc < W / 2; ++cc)
            conv_next[cc] = nc[(v < nwin ? v : nwin - 1) * (W / 2) + cc] != 0;
    };
    read_nc(0);
    int st = 0;
    for (int v = 0; v < nwin; ++v) {
        issue(v + NST - 1, st == 0 ? NST - 1 : st - 1);
#pragma unroll
        for (int cc = 0; cc < W / 2; ++cc)
            conv_now[cc] = conv_next[cc];
        read_nc(v + 1);
        const lds_u8 *sq = L + st * S::SB;
        const lds_u8 *stb = sq + S::QB;
        v4i qv[QT][S::U];
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            const int r = (wave * QT + qt) * 32 + (lane & 31);
#pragma unroll
            for (int hh = 0; hh < S::U; ++hh)
                qv[qt][hh] = *(const lds_v4i *)(sq + r * (W * 8) + 16 * hm_slot<KT>(r, hh));
        }
#pragma unroll
        for (int cc = 0; cc < W / 2; ++cc) {
            if (!conv_now[cc])   // uniform: not converted
                continue;
            ++pending;
            ++chunks;
            v8i af[2][KT];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    const v4i a4 = *(const lds_v4i *)(stb + (((2 * cc + h) * KT + kt) * 64 + lane) * 16);
                    af[h][kt] = v8i{a4[0], a4[1], a4[2], a4[3], 0, 0, 0, 0};
                }
            // a group of tiles' products first: a tile's conversion runs while
            // the next ones' products are on the matrix cores
#pragma unroll
            for (int q0 = 0; q0 < QT; q0 += QG) {
                v8i bq[QG][2];
#pragma unroll
                for (int qt = 0; qt < QG; ++qt) {
                    const v4i u = qv[q0 + qt][cc];   // the chunk's two words: dwords 0-1 and 2-3
                    bq[qt][0] = query_bipolar((uint32_t)(g ? u[1] : u[0]));
                    bq[qt][1] = query_bipolar((uint32_t)(g ? u[3] : u[2]));
                }
#pragma unroll
                for (int k0 = 0; k0 < KT; k0 += KG) {
                    v16f part[QG][KG];
#pragma unroll
                    for (int qt = 0; qt < QG; ++qt)
#pragma unroll
                        for (int kt = 0; kt < KG; ++kt) {
                            part[qt][kt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                af[0][k0 + kt], bq[qt][0], v16f{}, 4, 4, 0, 0, 0, 0);
                            part[qt][kt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                af[1][k0 + kt], bq[qt][1], part[qt][kt], 4, 4, 0, 0, 0, 0);
                        }
#pragma unroll
                    for (int qt = 0; qt < QG; ++qt)
#pragma unroll
                        for (int kt = 0; kt < KG; ++kt) {
                            if constexpr (ARITH) {
                                codes[k0 + kt][q0 + qt].add(conv, part[qt][kt]);
                            } else {
#pragma unroll
                                for (int e = 0; e < 16; ++e)
                                    sc[k0 + kt][q0 + qt][e] += lut[(int)part[qt][kt][e] + 128];
                            }
                        }
                }
            }
        }
        if (ARITH && pending > kAdcFlush - W / 2)
            flush();
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(G * (NST - 2)) : "memory");
        st = st == NST - 1 ? 0 : st + 1;
    }
    __builtin_amdgcn_s_waitcnt(0);
    const int mul = ARITH ? step : 1, add = ARITH ? floor_ * chunks : 0;   // codes to values
    if (ARITH)
        flush();

    // argmax: lane holds query l%32 of each tile and classes 8(v/4)+4g+v%4
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        const int64_t q = rbase + (wave * QT + qt) * 32 + (lane & 31);
        int best = INT_MIN, bk = 0;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int k = kt * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
                if (k < K) {
                    const int val = sc[kt][qt][e] * mul + add;
                    if (val > best) { best = val; bk = k; }
                    if (scores && q < n)
                        scores[q * K + k] = val;
                }
            }
        const int ob = __shfl_xor(best, 32), obk = __shfl_xor(bk, 32);
        if (ob > best || (ob == best && obk < bk)) { best = ob; bk = obk; }
        if (g == 0 && q < n) {
            label[q] = bk;
            if (max_score)
                max_score[q] = best;
        }
    }
}

// ARITH: by arithmetic if that gives the table's values, else by the table; the
// registers of the arithmetic (two waves per SIMD from 33 classes on) slow the
// table's loop, so where the table is foreseen (adc_arith) it has its own kernel
// with three.
template <int KT, bool ARITH>
__global__ __launch_bounds__(256) void k_adc_mfma(const uint64_t *__restrict__ Q, int64_t n, int64_t ldq, int K,
                                                  int w_lo, int w_hi, int nwin, const int8_t *__restrict__ tab,
                                                  const int32_t *__restrict__ nc, int res, int step, int floor_,
                                                  int ceil_, int32_t *__restrict__ label,
                                                  int32_t *__restrict__ max_score, int32_t *__restrict__ scores)
{
    typedef HmShape<KT> S;
    __shared__ __align__(16) uint8_t smem[S::NST * S::SB];
    __shared__ int lut[257];
    const AdcConv conv(res, step, floor_, ceil_);
    const bool arith = adc_table(lut, threadIdx.x, conv, res, step, floor_, ceil_);   // uniform
    if constexpr (ARITH) {
        if (arith) {
            adc_stream<KT, true>(smem, lut, conv, Q, n, ldq, K, w_lo, w_hi, nwin, tab, nc, step, floor_, label,
                                 max_score, scores);
            return;
        }
    }
    adc_stream<KT, false>(smem, lut, conv, Q, n, ldq, K, w_lo, w_hi, nwin, tab, nc, step, floor_, label, max_score,
                          scores);
}

// The same for few queries (see few_pairs): a pair of words is a chunk; the
// pairs a block lacks fall on chunk slots that are not converted.
template <int KT>
__global__ __launch_bounds__(256) void k_adc_few(const uint64_t *__restrict__ Q, int64_t n, int64_t ldq, int K,
                                                 int w_lo, int w_hi, const int8_t *__restrict__ tab,
                                                 const int32_t *__restrict__ nc, int res, int step, int floor_,
                                                 int ceil_, int32_t *__restrict__ label,
                                                 int32_t *__restrict__ max_score, int32_t *__restrict__ scores)
{
    __shared__ int32_t sums[kWaves][KT * 32][33];
    __shared__ int lut[257];
    __shared__ int best[8][32], bestk[8][32];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 5;
    const AdcConv conv(res, step, floor_, ceil_);
    const bool arith = adc_table(lut, t, conv, res, step, floor_, ceil_);
    v16i sc[KT];
    AdcCodes codes[KT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
        sc[kt] = v16i{};
        codes[kt].clear();
    }
    int pending = 0, chunks = 0;   // chunks in codes, and converted by this wave
    auto flush = [&]() {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
            codes[kt].flush(sc[kt], pending);
        pending = 0;
    };
    few_pairs(Q, n, ldq, w_lo, w_hi, [&](int p, int p1, const v4i (&u)[kFewPairs]) {
#pragma unroll
        for (int i = 0; i < kFewPairs; ++i) {
            if (p + i >= p1 || nc[p + i] == 0)   // uniform: not converted
                continue;
            ++pending;
            ++chunks;
            const v8i b0 = query_bipolar((uint32_t)(g ? u[i][1] : u[i][0]));
            const v8i b1 = query_bipolar((uint32_t)(g ? u[i][3] : u[i][2]));
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                const int8_t *e = tab + ((int64_t)(2 * (p + i)) * KT + kt) * 1024 + lane * 16;
                const v4i a0 = *(const v4i *)e, a1 = *(const v4i *)(e + KT * 1024);
                v16f part = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                    v8i{a0[0], a0[1], a0[2], a0[3], 0, 0, 0, 0}, b0, v16f{}, 4, 4, 0, 0, 0, 0);
                part = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(v8i{a1[0], a1[1], a1[2], a1[3], 0, 0, 0, 0}, b1,
                                                                       part, 4, 4, 0, 0, 0, 0);
                if (arith) {
                    codes[kt].add(conv, part);
                } else {
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        sc[kt][v] += lut[(int)part[v] + 128];
                }
            }
        }
        if (arith && pending > kAdcFlush - kFewPairs)
            flush();
    });
    const int mul = arith ? step : 1, add = arith ? floor_ * chunks : 0;   // codes to values
    if (arith)
        flush();
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            sums[wave][kt * 32 + 8 * (v >> 2) + 4 * g + (v & 3)][lane & 31] = sc[kt][v] * mul + add;
    __syncthreads();
    const int c = t & 31, slot = t >> 5;
    const int64_t q = (int64_t)blockIdx.x * 32 + c;
    int b = INT_MIN, bk = INT_MAX;
    for (int k = slot; k < K; k += 8) {
        const int v = sums[0][k][c] + sums[1][k][c] + sums[2][k][c] + sums[3][k][c];
        if (scores && q < n)
            scores[q * K + k] = v;
        if (bk == INT_MAX || v > b) {
            b = v;
            bk = k;
        }
    }
    best[slot][c] = b;
    bestk[slot][c] = bk;
    __syncthreads();
    if (t < 32 && q < n) {
#pragma unroll
        for (int s = 1; s < 8; ++s)
            if (bestk[s][c] != INT_MAX && (best[s][c] > b || (best[s][c] == b && bestk[s][c] < bk))) {
                b = best[s][c];
                bk = bestk[s][c];
            }
        label[q] = bk;
        if (max_score)
            max_score[q] = b;
    }
}

// Whether the arithmetic of AdcConv gives the table's values: the same check in
// single precision, its results rounded to halves' 11 bits, to choose the kernel
// (which checks for itself).  Settings whose codes pass 1023, and about one in
// fifty others, take the table.
static bool adc_arith(int res, int step, int floor_, int ceil_)
{
    auto half = [](float v) {
        const float g = v * 8193.0f;
        return g - (g - v);
    };
    const float top = (float)((1ll << res) - 1);
    float range = (float)((int64_t)ceil_ - floor_) / (float)step;
    range = range < top ? range : top;
    range = range > 0.0f ? range : 1.0f;
    const float inv = 1.0f / ((float)step * range);
    const float k = half(inv), c = half((0.25f - (float)floor_) * inv), r = half(range);
    // (single precision and without exits: four values at a time)
    const float lo = (float)floor_, hi = (float)ceil_, two = 2.0f * (float)step;
    int bad = 0;
    for (int s = -128; s <= 128; ++s) {
        const float x = (float)s < lo ? lo : (float)s > hi ? hi : (float)s;
        const float v = (2.0f * (x - lo) + (float)step) / two;
        const float code = (float)(int)(v < top ? v : top);
        float t = half((float)s * k + c);
        t = t < 0.0f ? 0.0f : t > 1.0f ? 1.0f : t;
        bad |= !(code < 1024.0f) | !(half(t * r + 1024.0f) == 1024.0f + code);
    }
    return !bad;
}

hipError_t launch_adc_prepared(const uint64_t *Q, int64_t n, int64_t ldq, int K, int start, int end, int res,
                               int step, int floor_, int ceil_, const uint8_t *ws, int32_t *label,
                               int32_t *max_score, int32_t *scores, hipStream_t st)
{
    const AdcLayout L(start, end, K);
    const int8_t *tab = (const int8_t *)ws;
    const int32_t *nc = (const int32_t *)(ws + L.off_nc);
#define HDC_ADCP_CASE(KT_)                                                                                     \
    if (L.KT == KT_ && n <= adc_few_queries(KT_)) {                                                            \
        hipLaunchKernelGGL(k_adc_few<KT_>, dim3((unsigned)((n + 31) / 32)), dim3(256), 0, st, Q, n, ldq, K, L.w_lo, \
                           L.w_hi, tab, nc, res, step, floor_, ceil_, label, max_score, scores);               \
        return hipGetLastError();                                                                              \
    }                                                                                                          \
    if (L.KT == KT_) {                                                                                         \
        typedef HmShape<KT_> S;                                                                                \
        constexpr int NW = kHmWin / S::W;                                                                      \
        const dim3 grid((unsigned)((n + S::ROWS - 1) / S::ROWS));                                              \
        if (adc_arith(res, step, floor_, ceil_))                                                               \
            hipLaunchKernelGGL((k_adc_mfma<KT_, true>), grid, dim3(256), 0, st, Q, n, ldq, K, L.w_lo, L.w_hi,    \
                               L.nwin * NW, tab, nc, res, step, floor_, ceil_, label, max_score, scores);      \
        else                                                                                                   \
            hipLaunchKernelGGL((k_adc_mfma<KT_, false>), grid, dim3(256), 0, st, Q, n, ldq, K, L.w_lo, L.w_hi,   \
                               L.nwin * NW, tab, nc, res, step, floor_, ceil_, label, max_score, scores);      \
        return hipGetLastError();                                                                              \
    }
    HDC_ADCP_CASE(1)
    HDC_ADCP_CASE(2)
    HDC_ADCP_CASE(4)
#undef HDC_ADCP_CASE
    return hipErrorInvalidValue;
}

}  // namespace hdc
