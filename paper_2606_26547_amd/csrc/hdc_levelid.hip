// Encode-side kernels beside random projection: the feature-column gather
// that perforates the encoding's reduction over features, the level
// quantiser and Level-ID encoding.
//
// Level-ID: bit d of a row's hypervector is set when more than half of the
// F bound pairs ID_f xor LV_level(f) have bit d set (the bipolar sum is
// F - 2*count; a zero sum gives +1).  A lane owns two 64-bit words of a few
// rows; per feature it takes the level words from LDS and adds them, bound to
// the ID words, to a bit-sliced counter through a carry-save tree (see
// k_level_id).
#include <type_traits>

#include "hdc_device.h"

namespace hdc {

// ------------------------------------------------------------------ gather
// Y[i][j] = X[i][start + j*stride] for j < nf, 0 for nf <= j < ldy; each
// thread writes 16 bytes of one row.
template <typename T>
__global__ __launch_bounds__(256) void k_gather_cols(const T *__restrict__ X, int64_t n, int64_t ldx, int start,
                                                     int stride, int nf, T *__restrict__ Y, int64_t ldy)
{
    constexpr int E = 16 / sizeof(T);
    const int64_t per_row = ldy / E;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n * per_row)
        return;
    const int64_t i = idx / per_row;
    const int j0 = (int)(idx - i * per_row) * E;
    const T *x = X + i * ldx + start;
    T v[E];
#pragma unroll
    for (int e = 0; e < E; ++e)
        v[e] = j0 + e < nf ? x[(int64_t)(j0 + e) * stride] : T(0);
    *(uint4 *)(Y + i * ldy + j0) = *(const uint4 *)v;
}

hipError_t launch_gather_cols(const void *X, int elem, int64_t n, int64_t ldx, int start, int stride, int nf,
                              void *Y, int64_t ldy, hipStream_t st)
{
    const int64_t total = n * (ldy * elem / 16);
    const dim3 grid((unsigned)((total + 255) / 256));
    if (elem == 1)
        hipLaunchKernelGGL(k_gather_cols<uint8_t>, grid, dim3(256), 0, st, (const uint8_t *)X, n, ldx, start,
                           stride, nf, (uint8_t *)Y, ldy);
    else
        hipLaunchKernelGGL(k_gather_cols<float>, grid, dim3(256), 0, st, (const float *)X, n, ldx, start, stride,
                           nf, (float *)Y, ldy);
    return hipGetLastError();
}

// --------------------------------------------------------------- quantiser
// level = floor((x - lo) * L / (hi - lo)) in binary32, each step rounded to
// nearest even (no contraction), 0 for an empty range, a value at or below
// lo, or NaN; L - 1 at or above the top level.
//
// Streaming bound: a thread takes one feature of kLqRows rows, all its loads
// in flight, the range read once (one element per thread, with a 64-bit
// division to find it, took 41 us for 32768 x 617; the bytes take 25).  A
// workgroup's lanes cover FW features of 256 / FW rows: 64, or for narrow rows
// the power of two that holds them, so that no lane is without a feature (4194304
// x 1: 197 us with 64, 17.6 so).
constexpr int kLqRows = 8;
template <int FW>
__device__ __forceinline__ void quantize_rows(const float *__restrict__ X, int64_t n, int64_t ldx, float l0, float w,
                                              int64_t i0, int64_t f, int L, uint16_t *__restrict__ lev, int64_t ldl)
{
    constexpr int RW = 256 / FW;
    float x[kLqRows];
#pragma unroll
    for (int r = 0; r < kLqRows; ++r)
        x[r] = X[(i0 + r * RW < n ? i0 + r * RW : n - 1) * ldx + f];
#pragma unroll
    for (int r = 0; r < kLqRows; ++r) {
        const float v = __fdiv_rn(__fmul_rn(__fsub_rn(x[r], l0), (float)L), w);
        int level;
        if (!(w > 0.0f) || !(v > 0.0f))
            level = 0;
        else if (v >= (float)(L - 1))
            level = L - 1;
        else
            level = (int)floorf(v);
        if (i0 + r * RW < n)
            lev[(i0 + r * RW) * ldl + f] = (uint16_t)level;
    }
}

// STRIDE: more rows or features than a grid holds (the loops cost 5 to 10%).
template <int FW, bool STRIDE>
__global__ __launch_bounds__(256) void k_level_quantize(const float *__restrict__ X, int64_t n, int F, int64_t ldx,
                                                        const float *__restrict__ lo, const float *__restrict__ hi,
                                                        int L, uint16_t *__restrict__ lev, int64_t ldl)
{
    constexpr int64_t ROWS = 256 / FW * kLqRows;
    const int64_t i0 = (int64_t)blockIdx.x * ROWS + threadIdx.x / FW;
    if constexpr (STRIDE) {
        for (int64_t f = (int64_t)blockIdx.y * FW + threadIdx.x % FW; f < F; f += (int64_t)gridDim.y * FW)
            for (int64_t i = i0; i < n; i += (int64_t)gridDim.x * ROWS)
                quantize_rows<FW>(X, n, ldx, lo[f], __fsub_rn(hi[f], lo[f]), i, f, L, lev, ldl);
    } else {
        const int f = blockIdx.y * FW + threadIdx.x % FW;
        if (f < F)
            quantize_rows<FW>(X, n, ldx, lo[f], __fsub_rn(hi[f], lo[f]), i0, f, L, lev, ldl);
    }
}

template <int FW>
static void launch_lq(const float *X, int64_t n, int F, int64_t ldx, const float *lo, const float *hi, int L,
                      uint16_t *lev, int64_t ldl, hipStream_t st)
{
    constexpr int64_t rows = 256 / FW * kLqRows;
    const int64_t x = (n + rows - 1) / rows, y = ((int64_t)F + FW - 1) / FW;
    const dim3 grid((unsigned)(x < (1 << 22) ? x : 1 << 22), (unsigned)(y < 65535 ? y : 65535));
    if (x > grid.x || y > grid.y)
        hipLaunchKernelGGL((k_level_quantize<FW, true>), grid, dim3(256), 0, st, X, n, F, ldx, lo, hi, L, lev, ldl);
    else
        hipLaunchKernelGGL((k_level_quantize<FW, false>), grid, dim3(256), 0, st, X, n, F, ldx, lo, hi, L, lev, ldl);
}

hipError_t launch_level_quantize(const float *X, int64_t n, int F, int64_t ldx, const float *lo, const float *hi,
                                 int L, uint16_t *lev, int64_t ldl, hipStream_t st)
{
    if (F <= 1)
        launch_lq<1>(X, n, F, ldx, lo, hi, L, lev, ldl, st);
    else if (F <= 2)
        launch_lq<2>(X, n, F, ldx, lo, hi, L, lev, ldl, st);
    else if (F <= 4)
        launch_lq<4>(X, n, F, ldx, lo, hi, L, lev, ldl, st);
    else if (F <= 8)
        launch_lq<8>(X, n, F, ldx, lo, hi, L, lev, ldl, st);
    else if (F <= 16)
        launch_lq<16>(X, n, F, ldx, lo, hi, L, lev, ldl, st);
    else if (F <= 32)
        launch_lq<32>(X, n, F, ldx, lo, hi, L, lev, ldl, st);
    else
        launch_lq<64>(X, n, F, ldx, lo, hi, L, lev, ldl, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------- Level-ID
constexpr int kLidFeat = 32;    // features per ripple of the counters
constexpr int kLidBig = 6;      // planes of the weight-32 counter (F <= 1024 -> count / 32 <= 32)

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// acc + x + y: parity to acc, majority returned
__device__ __forceinline__ uint32_t csa(uint32_t &acc, uint32_t x, uint32_t y)
{
    const uint32_t c = __builtin_amdgcn_bitop3_b32(acc, x, y, 0xE8);
    acc = xor3(acc, x, y);
    return c;
}

// acc + (a xor i) + (b xor j) in three operations: with u = acc ^ a ^ i and
// s = u ^ b ^ j the carry is the second input where u is set (b ^ j = ~s
// there), else acc.
__device__ __forceinline__ uint32_t csa_bound(uint32_t &acc, uint32_t a, uint32_t i, uint32_t b, uint32_t j)
{
    const uint32_t u = xor3(acc, a, i), s = xor3(u, b, j);
    const uint32_t c = __builtin_amdgcn_bitop3_b32(u, s, acc, 0x3A);   // u ? ~s : acc
    acc = s;
    return c;
}

struct LidCounter {
    uint32_t ones[4], twos[4], fours[4], eights[4], sixteens[4], big[kLidBig][4];
    uint32_t f[4], e[4], h[4];   // pending carries of weight 4, 8 and 16

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            ones[k] = twos[k] = fours[k] = eights[k] = sixteens[k] = f[k] = e[k] = h[k] = 0;
#pragma unroll
            for (int p = 0; p < kLidBig; ++p)
                big[p][k] = 0;
        }
    }
    // dword k's carry of weight 4 from group q of 8
    __device__ __forceinline__ void carry(int q, int k, uint32_t c4)
    {
        if (q % 2 == 0) {
            f[k] = c4;
            return;
        }
        const uint32_t c8 = csa(fours[k], f[k], c4);
        if (q % 4 == 1) {
            e[k] = c8;
            return;
        }
        const uint32_t c16 = csa(eights[k], e[k], c8);
        if (q == 3) {
            h[k] = c16;
            return;
        }
        uint32_t c = csa(sixteens[k], h[k], c16);
#pragma unroll
        for (int p = 0; p < kLidBig; ++p) {
            const uint32_t nc = big[p][k] & c;
            big[p][k] ^= c;
            c = nc;
        }
    }
    // a group without features
    __device__ __forceinline__ void add0(int q)
    {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            carry(q, k, 0);
    }
    // four features (level words a, identity words id), group q of 8
    __device__ __forceinline__ void add4(int q, const v4i (&a)[4], const v4i (&id)[4])
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t t0 = csa_bound(ones[k], (uint32_t)a[0][k], (uint32_t)id[0][k], (uint32_t)a[1][k],
                                          (uint32_t)id[1][k]);
            const uint32_t t1 = csa_bound(ones[k], (uint32_t)a[2][k], (uint32_t)id[2][k], (uint32_t)a[3][k],
                                          (uint32_t)id[3][k]);
            carry(q, k, csa(twos[k], t0, t1));
        }
        // in order: later reads, or these sums, moved across here would not
        // fit the registers
        asm volatile("" : "+v"(ones[0]), "+v"(ones[1]), "+v"(ones[2]), "+v"(ones[3]), "+v"(twos[0]), "+v"(twos[1]),
                     "+v"(twos[2]), "+v"(twos[3])::"memory");
        if (q % 2 == 1)
            asm volatile("" : "+v"(fours[0]), "+v"(fours[1]), "+v"(fours[2]), "+v"(fours[3]));
        __builtin_amdgcn_sched_barrier(0);
    }
    // plane p of dword k: the counts' bit of weight 2^p
    __device__ __forceinline__ uint32_t &plane(int p, int k)
    {
        return p == 0 ? ones[k] : p == 1 ? twos[k] : p == 2 ? fours[k] : p == 3 ? eights[k] : p == 4 ? sixteens[k]
                                                                                                     : big[p - 5][k];
    }
    // bit set where count > T
    __device__ __forceinline__ uint32_t greater(int k, uint32_t T) const
    {
        uint32_t cnt[5 + kLidBig] = {ones[k], twos[k], fours[k], eights[k], sixteens[k]};
#pragma unroll
        for (int p = 0; p < kLidBig; ++p)
            cnt[5 + p] = big[p][k];
        uint32_t gt = 0, eq = ~0u;
#pragma unroll
        for (int p = 5 + kLidBig - 1; p >= 0; --p) {
            if ((T >> p) & 1u) {
                eq &= cnt[p];
            } else {
                gt |= eq & cnt[p];
                eq &= ~cnt[p];
            }
        }
        return gt;
    }
};

// Shape of a launch: LPR lanes of two words share a row (a window of 2 * LPR
// words), each lane takes R rows.  With LPR = 16 the 16 lanes that LDS
// serves at a time read one whole 256-byte level row, all 64 banks, whatever
// its level (8 lanes of one word met bank conflicts).  Identity words come
// from L2, a group of features ahead: through LDS as well, the two rows'
// reads would keep LDS busy longer than the vector units.  These bound it: 2.8
// operations per dword and feature in the tree (the bound inputs enter it in
// 1.5, see csa_bound; 32 features per ripple) and 1.25 per level address and
// lane, against 13 per 64-bit word and feature for plain xor and majority on
// one word per lane.  32768 x 617, 10240 dimensions, 128 levels, with the
// quantiser: 1372 us on one word and row per lane, 792 so, the vector units
// busy four fifths of it; without it 779 so, 876 with one row per lane.
//
// Few rows (FS): the four waves of a workgroup take a quarter of the features
// each of the same rows, and their counts meet in LDS.  A wave alone on its SIMD
// takes 70 ns a feature whatever its rows, so ten rows left it at 43 us (one word
// per lane: 32); split, 17 (617 features, 128 levels, 10240 dimensions).
template <int LPR, int R, bool FS = false> struct LidShape {
    static constexpr int W = 2 * LPR;                      // words per window
    static constexpr int RPW = 64 / LPR;                   // rows per wave at a time
    static constexpr int ROWS = (FS ? 1 : kWaves) * RPW * R;   // rows per workgroup
    static constexpr int PITCH = W * 8 + (LPR == 16 ? 0 : 16);   // bytes per level row in LDS
    static constexpr int SUMS = FS ? (kWaves - 1) * R * (5 + kLidBig) * 4 * 64 * 4 : 0;   // other waves' counts
    static size_t lds(int L)
    {
        const size_t levels = (size_t)(L + 1) * PITCH;
        return levels > SUMS ? levels : SUMS;
    }
};

// base + pitch * the low (HI: high) half of the level pair
template <bool HI> __device__ __forceinline__ uint32_t lid_addr(uint32_t pair, uint32_t pitch, uint32_t base)
{
    uint32_t r;
    if constexpr (HI)
        asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(pair), "v"(pitch), "v"(base));
    else
        asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(r) : "v"(pair), "v"(pitch), "v"(base));
    return r;
}

template <int LPR, int R, bool FS, bool PASSES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FS ? 1 : R == 1 ? 3 : 2)))
void k_level_id(const uint16_t *__restrict__ lev, int64_t n, int F, int64_t ldl, const uint64_t *__restrict__ ID,
                int64_t ldid, const uint64_t *__restrict__ LV, int L, int64_t ldlv, int D, uint64_t *__restrict__ H,
                int64_t ldh)
{
    typedef LidShape<LPR, R, FS> S;
    typedef unsigned short v2us __attribute__((ext_vector_type(2)));
    extern __shared__ __align__(16) uint8_t lid_lds[];
    lds_u8 *slv = (lds_u8 *)lid_lds;
    typedef HDC_LDS uint64_t lds_u64;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int W = (D + 63) / 64, w0 = blockIdx.y * S::W;
    const int nw = W - w0 < S::W ? W - w0 : S::W;

    // level rows of the window, then a row of zeros (the level of features
    // past F, whose identity words are zero too)
    for (int e = t; e < (L + 1) * S::W; e += 256) {
        const int r = e / S::W, w = e % S::W;
        *(lds_u64 *)(slv + r * S::PITCH + w * 8) = r < L && w < nw ? LV[(int64_t)r * ldlv + w0 + w] : 0;
    }
    const int wl = lane % LPR;                             // this lane's words: w0 + 2 wl, + 1
    int64_t row0 = (int64_t)blockIdx.x * S::ROWS + (FS ? 0 : wave * (S::RPW * R)) + lane / LPR;
    // this wave's features: all, or (FS) whole blocks of 32
    const int per = FS ? (F + kLidFeat * kWaves - 1) / (kLidFeat * kWaves) * kLidFeat : F;
    const int fb = FS ? __builtin_amdgcn_readfirstlane(wave) * per : 0, fe = fb + per < F ? fb + per : F;
    const uint16_t *lrow[R];
    // eight levels of each row from feature f on (past the row: its first)
    auto lev_load = [&](uint4 (&l)[R], int f) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            l[r] = *(const uint4 *)(lrow[r] + (f < F ? f : 0));
    };
    // this lane's identity words of features f .. f + 3, zero past the row
    // (a buffer of one row's words: no address past its end is read) or past F
    auto id_load = [&](v4i (&id)[4], int f) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int fu = f + u;
            const __amdgpu_buffer_rsrc_t row = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(ID + (int64_t)(fu < F ? fu : 0) * ldid), 0, fu < F ? W * 8 : 0, 0x00020000);
            id[u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(row, (w0 + 2 * wl) * 8, 0, 0));
        }
    };
    LidCounter cnt[R];
    const uint32_t lbase = (uint32_t)(uintptr_t)slv + wl * 16;
    const uint32_t lmax = (uint32_t)(L - 1) * 0x10001u;
    uint4 lv[2][R];
    v4i id[2][4];
    // a pass over ROWS rows starts
    auto start = [&]() {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t row = row0 + r * S::RPW;
            lrow[r] = lev + (row < n ? row : n - 1) * ldl;
            cnt[r].clear();
        }
        lev_load(lv[0], fb);
        id_load(id[0], fb);
    };
    start();
    __syncthreads();
    // one block of 32 features; TAIL: features past F take the zero row, and
    // groups past it only pass the carries on (8231 rows, 65 features, 7530
    // dimensions: 54 us with whole blocks, 45 so)
    auto block = [&](int f0, auto tail) {
        constexpr bool TAIL = decltype(tail)::value;
#pragma unroll
        for (int q = 0; q < 8; ++q) {                      // groups of four features
            if constexpr (TAIL) {
                if (f0 + 4 * q >= F) {   // uniform: nothing to read or bind
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        cnt[r].add0(q);
                    continue;
                }
            }
            if (q % 2 == 0)
                lev_load(lv[(q / 2 + 1) & 1], f0 + 4 * q + 8);
            id_load(id[(q + 1) & 1], f0 + 4 * q + 4);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint4 &l4 = lv[(q / 2) & 1][r];
                v4i a[4];
#pragma unroll
                for (int u = 0; u < 4; u += 2) {
                    const uint32_t p0 = q % 2 ? (u ? l4.w : l4.z) : (u ? l4.y : l4.x);
                    uint32_t pr = __builtin_bit_cast(
                        uint32_t, __builtin_elementwise_min(__builtin_bit_cast(v2us, p0), __builtin_bit_cast(v2us, lmax)));
                    if constexpr (TAIL) {
                        const int f = f0 + 4 * q + u;
                        if (f >= F)
                            pr = (uint32_t)L * 0x10001u;
                        else if (f + 1 >= F)
                            pr = (pr & 0xffffu) | ((uint32_t)L << 16);
                    }
                    a[u] = *(const lds_v4i *)(uintptr_t)lid_addr<false>(pr, S::PITCH, lbase);
                    a[u + 1] = *(const lds_v4i *)(uintptr_t)lid_addr<true>(pr, S::PITCH, lbase);
                }
                cnt[r].add4(q, a, id[q & 1]);
            }
        }
    };
    for (int64_t rb = blockIdx.x;;) {
        int f0 = fb;
        for (; f0 + kLidFeat <= fe; f0 += kLidFeat)
            block(f0, std::integral_constant<bool, false>{});
        if (f0 < fe)
            block(f0, std::integral_constant<bool, true>{});
        if constexpr (FS) {   // (one pass)
            constexpr int NP = 5 + kLidBig;
            lds_i32 *sums = (lds_i32 *)slv;
            __syncthreads();   // the level words are done with
            if (wave > 0) {
#pragma unroll
                for (int i = 0; i < R * NP * 4; ++i)
                    sums[((wave - 1) * (R * NP * 4) + i) * 64 + lane] = (int)cnt[i / (NP * 4)].plane(i / 4 % NP, i % 4);
            }
            __syncthreads();
            if (wave > 0)
                return;
#pragma unroll
            for (int w = 0; w < kWaves - 1; ++w)
#pragma unroll
                for (int rk = 0; rk < R * 4; ++rk) {
                    uint32_t c = 0;
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        const uint32_t x = (uint32_t)sums[(w * (R * NP * 4) + rk / 4 * (NP * 4) + p * 4 + rk % 4) * 64 + lane];
                        c = csa(cnt[rk / 4].plane(p, rk % 4), x, c);
                    }
                }
        }

#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t row = row0 + r * S::RPW;
            if (row >= n)
                continue;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int w = w0 + 2 * wl + i;
                if (w >= W)
                    continue;
                uint64_t v = (uint64_t)cnt[r].greater(2 * i, (uint32_t)F >> 1) |
                             ((uint64_t)cnt[r].greater(2 * i + 1, (uint32_t)F >> 1) << 32);
                if (w == W - 1 && (D & 63))
                    v &= (1ull << (D & 63)) - 1ull;
                H[row * ldh + w] = v;
            }
        }
        rb += gridDim.x;
        if (!PASSES || rb * S::ROWS >= n)
            break;
        row0 += (int64_t)gridDim.x * S::ROWS;
        start();
    }
}

template <int LPR, int R, bool FS, bool PASSES>
static hipError_t launch_level_id_grid(const dim3 &grid, const uint16_t *lev, int64_t n, int F, int64_t ldl,
                                       const uint64_t *ID, int64_t ldid, const uint64_t *LV, int L, int64_t ldlv, int D,
                                       uint64_t *H, int64_t ldh, hipStream_t st)
{
    // once per process and shape (thread-safe static initialisation)
    static const hipError_t attr = hipFuncSetAttribute((const void *)k_level_id<LPR, R, FS, PASSES>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess)
        return attr;
    hipLaunchKernelGGL((k_level_id<LPR, R, FS, PASSES>), grid, dim3(256), (LidShape<LPR, R, FS>::lds(L)), st, lev, n, F,
                       ldl, ID, ldid, LV, L, ldlv, D, H, ldh);
    return hipGetLastError();
}

template <int LPR, int R, bool FS>
static hipError_t launch_level_id_rows(const uint16_t *lev, int64_t n, int F, int64_t ldl, const uint64_t *ID,
                                       int64_t ldid, const uint64_t *LV, int L, int64_t ldlv, int D, uint64_t *H,
                                       int64_t ldh, hipStream_t st)
{
    typedef LidShape<LPR, R, FS> S;
    const int W = (D + 63) / 64;
    // Where staging the levels costs like half a pass or more, and their LDS leaves
    // too few workgroups per CU to hide it, a workgroup takes several passes of
    // rows, as many as leave two per CU (20000 rows x 20 features, 256 levels, 4096
    // dimensions: 42 us with one pass, 23 so; 60000 x 60, 2000 dimensions 87 and 51;
    // but 8000 x 40, 100 levels, 10000 dimensions, four per CU: 28 and 31).  Else one
    // pass (without the loop, whose registers cost 5%), up to 2^22 workgroups (a grid
    // takes 2^24).
    const int64_t blocks = (n + S::ROWS - 1) / S::ROWS, wins = (W + S::W - 1) / S::W;
    const bool stage = !FS && S::lds(L) > 40 * 1024 && (int64_t)(L + 1) * S::W > 64ll * F * R;
    const int64_t most = stage ? (512 + wins - 1) / wins : 1 << 22;
    const dim3 grid((unsigned)(blocks < most ? blocks : most), (unsigned)wins);
    if constexpr (!FS) {
        if (blocks > most)
            return launch_level_id_grid<LPR, R, FS, true>(grid, lev, n, F, ldl, ID, ldid, LV, L, ldlv, D, H, ldh, st);
    }
    return launch_level_id_grid<LPR, R, FS, false>(grid, lev, n, F, ldl, ID, ldid, LV, L, ldlv, D, H, ldh, st);
}

// Two rows per lane (each identity word read serves both, two waves per SIMD)
// once they make four rounds of the device's 512 workgroups; below, one row
// and three waves per SIMD fill the last rounds better (5555 rows x 389
// features, 5450 dimensions: 110 us with two rows, 75 with one; 32768 x 617,
// 10240: 779 and 876, without the quantiser).  While the rows, four to sixteen a workgroup, leave the
// device half idle, the waves split the features.
template <int LPR>
static hipError_t launch_level_id_shape(const uint16_t *lev, int64_t n, int F, int64_t ldl, const uint64_t *ID,
                                        int64_t ldid, const uint64_t *LV, int L, int64_t ldlv, int D, uint64_t *H,
                                        int64_t ldh, hipStream_t st)
{
    typedef LidShape<LPR, 2> S;
    typedef LidShape<LPR, 1, true> SF;
    const int W = (D + 63) / 64;
    if (F > kLidFeat && (n + SF::ROWS - 1) / SF::ROWS * ((W + S::W - 1) / S::W) <= 128)
        return launch_level_id_rows<LPR, 1, true>(lev, n, F, ldl, ID, ldid, LV, L, ldlv, D, H, ldh, st);
    if ((n + S::ROWS - 1) / S::ROWS * ((W + S::W - 1) / S::W) >= 2048)
        return launch_level_id_rows<LPR, 2, false>(lev, n, F, ldl, ID, ldid, LV, L, ldlv, D, H, ldh, st);
    return launch_level_id_rows<LPR, 1, false>(lev, n, F, ldl, ID, ldid, LV, L, ldlv, D, H, ldh, st);
}

// Windows of 32, 16 or 8 words: the widest whose level rows leave room for
// two workgroups per CU (up to 319, 567 levels; 8 words beyond) and
// whose last window is not mostly empty (an idle lane costs as much as a busy
// one).
hipError_t launch_level_id(const uint16_t *lev, int64_t n, int F, int64_t ldl, const uint64_t *ID, int64_t ldid,
                           const uint64_t *LV, int L, int64_t ldlv, int D, uint64_t *H, int64_t ldh, hipStream_t st)
{
    const int W = (D + 63) / 64;
    auto padded = [&](int w) { return (W + w - 1) / w * w; };
    const size_t half = 80 * 1024;
    int w = 8;
    if (LidShape<8, 2>::lds(L) <= half && padded(16) * 8 <= padded(8) * 9)
        w = 16;
    if (LidShape<16, 2>::lds(L) <= half && padded(32) * 8 <= padded(w) * 9)
        w = 32;
    if (w == 32)
        return launch_level_id_shape<16>(lev, n, F, ldl, ID, ldid, LV, L, ldlv, D, H, ldh, st);
    if (w == 16)
        return launch_level_id_shape<8>(lev, n, F, ldl, ID, ldid, LV, L, ldlv, D, H, ldh, st);
    return launch_level_id_shape<4>(lev, n, F, ldl, ID, ldid, LV, L, ldlv, D, H, ldh, st);
}

}  // namespace hdc
