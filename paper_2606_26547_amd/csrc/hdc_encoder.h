// The gfx950 random-projection encoder: one 256-thread workgroup = 4
// waves, each wave owning QT tiles of 32 queries whose features stay in
// VGPRs (converted once to the compute type) for the whole launch.  The
// workgroup walks the selected dimensions in chunks of one or two row tiles
// of 32: the gathered projection rows go through LDS, copied straight into a
// ring of stages (byte features) or through registers, converted, into a
// double buffer (fp32 features and the sweep's other bodies), while an
// earlier chunk is multiplied on the matrix cores (rows = dimensions, columns =
// queries).  The 32x32 accumulator of each query tile then goes through one
// of two epilogues, which run between the MFMAs of the following chunk:
//   M_ENCODE   sign -> packed bits, one uint32 half-word per query per chunk
//   M_CLASSIFY sign -> {0,-1} bytes laid out as the B operand of a second
//              int8 MFMA against the +-1 class bytes of the same 32
//              dimensions (staged in LDS with the chunk), accumulating
//              sum_d c_kd * m_qd; after the last chunk the Hamming distance
//              is popc_k - acc and the argmin is taken across the lanes.
// The encoder body is a device function so the persistent configuration
// sweep can run it per work item.
#pragma once

#include <type_traits>

#include "hdc_device.h"

namespace hdc {

// Projection rows as the direct-staged kernels read them (their SRC
// parameter): W_ROWS multiplies the bytes as they are (int8 features on the
// int8 path, the shifted projections, E4M3 rows); W_ALT is int8 +-1 rows with
// uint8 features on the int8 path (column sums), or converted to E4M3 as
// each fragment is read on the E4M3 paths.
enum Weights : int { W_ROWS = 0, W_ALT = 1 };

template <int CT, int XF, int QT, int KS, int KT, int MODE, int WV = 0, bool DMA = false, int RT = 1,
          int SRC = W_ROWS>
struct Encoder {
    typedef Tr<CT> T;
    typedef typename T::frag frag;
    typedef typename T::xfrag xfrag;
    typedef typename T::acc acc_t;
    static constexpr int KSTEP = T::KSTEP;
    static constexpr int KB = KSTEP * T::ESZ;              // LDS bytes per K-step per row
    static constexpr int RSB = KS * KB + 16;               // LDS row stride (16 B skew)
    static constexpr int PIECES = (KS * KSTEP + 15) / 16;  // 16-byte int8 pieces per row (max)
    static constexpr int MP = (PIECES + 7) / 8;            // pieces per thread (8 threads / row)
    // DMA: projection rows and class fragments go from global memory
    // straight into LDS (global_load_lds, 16 bytes per lane), a ring of three
    // to six stages.  Each load fills 1 KiB of LDS contiguously, so a stage is NIW
    // loads per wave (the last ones repeat its last KiB) and the units past
    // the chunk's rows land in the stage's slack.  The rows are copied as they
    // are (bytes on every path).
    // A chunk is RT row tiles of 32 dimensions (one or two, direct staging
    // only); its class operand is RT * KT KiB.
    static_assert(!DMA || (XF == 0 && (CT == C_I8 || CT == C_FP8 || CT == C_FP8S)),
                  "direct LDS staging is for integer features on the int8 and E4M3 paths");
    static_assert(RT == 1 || (RT == 2 && DMA), "two row tiles per chunk need direct LDS staging");
    static_assert(SRC == W_ROWS || DMA, "weight forms are for direct staging");
    static_assert(!(DMA && CT == C_I8 && SRC == W_ALT) || RT == 1, "column sums: a barrier per row tile");
    static constexpr bool U8 = DMA && CT == C_I8 && SRC == W_ALT;    // uint8 features: column sums
    static constexpr bool CVT = DMA && CT != C_I8 && SRC == W_ALT;   // int8 rows, E4M3 on read
    static constexpr int CH = kDimChunk * RT;              // dimensions per chunk
    static constexpr int UPR = RSB / 16;                   // 16-byte units per LDS row
    static constexpr int NIW = (CH * UPR + 64 * kWaves - 1) / (64 * kWaves);
    static constexpr int NCT = RT * KT;                    // class tiles per chunk
    static constexpr int NCW = (NCT + kWaves - 1) / kWaves;   // class-tile loads per wave
    static constexpr int NU = (CH * UPR + 63) / 64;        // 1 KiB pieces of a stage
    static constexpr int SSZ = DMA ? NU * 1024 : CH * RSB; // bytes per stage
    // LDS stages: chunks of one row tile are short, and the first touch of a
    // projection row comes from behind the L2, so where one workgroup has the
    // LDS to itself chunks are loaded up to five ahead (else two)
    static constexpr int CSZ = MODE == M_CLASSIFY ? NCT * 1024 : 0;
    static constexpr bool stages_fit(int n) { return RT == 1 && QT * KS > 20 && n * (SSZ + CSZ) + 512 <= 160 * 1024; }
    static constexpr int NBUF = !DMA ? 2 : stages_fit(6) ? 6 : stages_fit(5) ? 5 : U8 || stages_fit(4) ? 4 : 3;
    // chunks past the current one whose loads a pass's barrier waits for (the
    // uint8 kernels sum the columns of the tile two ahead), and the loads that
    // may stay in flight there
    static constexpr int VIS = U8 ? 2 : 1;
    static constexpr int OFF_C = NBUF * SSZ;
    static constexpr int OFF_CS = OFF_C + (MODE == M_CLASSIFY ? NBUF * NCT * 1024 : 0);
    static constexpr int LDS = OFF_CS + (!DMA ? NBUF * kDimChunk * 4 : U8 ? 2 * kDimChunk * 4 : 0);
    static_assert(LDS <= 160 * 1024, "LDS of one workgroup");
    static constexpr int QPW = QT * 32;                    // queries per wave
    // Waves per SIMD the kernel is compiled for (WV, or by default two where
    // the resident query operand leaves room, so that one wave's stalls are
    // covered by the other's MFMAs, else one).
    static constexpr int WAVES = WV ? WV
                                    : ((QT == 1 && RT == 1 && KT == 1 &&
                                        ((CT == C_I8 && KS <= 20) || (CT == C_BF16 && KS <= 16) ||
                                         (CT == C_F32 && KS <= 64))) ? 2 : 1);
    static constexpr int QPB = QPW * kWaves;               // queries per workgroup
    // Waves per SIMD the registers are kept to: the E4M3 path up to 320 features
    // and two class tiles (the shifted one: one) is near two already (200000 x
    // 300, 4096 dimensions, 40 classes: 375 us with 259 registers, 281 with 256;
    // shifted, 10 classes: 275 with 262, 212 with 254).
    static constexpr int REGW = DMA && CT == C_FP8 && QT == 2 && KS <= 5 && KT <= (SRC == W_ROWS ? 1 : 2) ? 2 : WAVES;

    // ---------------------------------------------------------------- X
    // One K step of byte features (16 bytes at k0 on the int8 path, 32 on
    // the E4M3 ones, 8 for bf16) converted to the B operand, features past F
    // cleared.
    static constexpr int XW = XF == 0 ? KSTEP / 8 : 0;   // feature dwords per lane and K step
    static __device__ __forceinline__ xfrag conv_bytes(const uint32_t (&d)[XW ? XW : 1], int k0, int F, bool sgn)
    {
        xfrag r;
        if constexpr (CT == C_I8) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t x = keep_bytes(d[e], k0 + 4 * e, F);
                if constexpr (U8)
                    x ^= 0x80808080u;            // x - 128; -128 past F (see SumHook)
                else if (!sgn)
                    x = keep_bytes(d[e] ^ 0x80808080u, k0 + 4 * e, F);
                r[e] = (int)x;
            }
        } else if constexpr (CT == C_FP8) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint32_t x = keep_bytes(d[e], k0 + 4 * e, F);
                r[e] = (int)fp8x4_raw(byte_value(x, 0, sgn), byte_value(x, 1, sgn), byte_value(x, 2, sgn),
                                      byte_value(x, 3, sgn));
            }
        } else if constexpr (CT == C_FP8S) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint32_t hi, lo;
                fp8_split4(keep_bytes(d[e], k0 + 4 * e, F), sgn, &hi, &lo);
                r[e] = (int)hi;
                r[8 + e] = (int)lo;
            }
        } else {   // C_BF16
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t x = keep_bytes(d[e], k0 + 4 * e, F);
                r[2 * e] = (int)bf16x2(byte_value(x, 0, sgn), byte_value(x, 1, sgn));
                r[2 * e + 1] = (int)bf16x2(byte_value(x, 2, sgn), byte_value(x, 3, sgn));
            }
        }
        return r;
    }

    // A K step past the features.
    static __device__ __forceinline__ xfrag no_features()
    {
        xfrag f{};
        if constexpr (U8) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                f[e] = (int)0x80808080u;
        }
        return f;
    }

    static __device__ __forceinline__ xfrag load_frag(const EncodeArgs &a, int64_t q, int s, int g)
    {
        const int k0 = s * KSTEP + g * (KSTEP / 2);
        if constexpr (XF == 0) {
            const uint8_t *row = (const uint8_t *)a.X + q * a.ldx;
            uint32_t d[XW];
            if constexpr (XW == 2) {
                const uint2 w = *(const uint2 *)(row + k0);
                d[0] = w.x;
                d[1] = w.y;
            } else {
#pragma unroll
                for (int i = 0; i < XW / 4; ++i) {
                    const uint4 w = *(const uint4 *)(row + k0 + 16 * i);
                    d[4 * i] = w.x;
                    d[4 * i + 1] = w.y;
                    d[4 * i + 2] = w.z;
                    d[4 * i + 3] = w.w;
                }
            }
            return conv_bytes(d, k0, a.F, a.x_type == X_INT8);
        } else {
            static_assert(CT != C_FP8S, "the split E4M3 type is for integer features");
            const float *row = (const float *)a.X + q * a.ldx;
            auto val = [&](int k) { return k < a.F ? row[k] : 0.0f; };
            if constexpr (CT == C_F32) {
                return val(k0);
            } else if constexpr (CT == C_FP8) {
                v8i r;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float4 f = *(const float4 *)(row + k0 + 4 * e);
                    int k = k0 + 4 * e;
                    r[e] = (int)fp8x4(k < a.F ? f.x : 0.f, k + 1 < a.F ? f.y : 0.f,
                                      k + 2 < a.F ? f.z : 0.f, k + 3 < a.F ? f.w : 0.f);
                }
                return r;
            } else {   // C_BF16
                v4i r;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    float4 f = *(const float4 *)(row + k0 + 4 * e);
                    int k = k0 + 4 * e;
                    r[2 * e] = (int)bf16x2(k < a.F ? f.x : 0.f, k + 1 < a.F ? f.y : 0.f);
                    r[2 * e + 1] = (int)bf16x2(k + 2 < a.F ? f.z : 0.f, k + 3 < a.F ? f.w : 0.f);
                }
                (void)val;
                return r;
            }
        }
    }

    static __device__ __forceinline__ void load_x(xfrag (&xr)[QT][KS], const EncodeArgs &a,
                                                  int64_t qbase, int lane, int ks_used)
    {
        // Branch-free: out-of-range rows / steps load an in-bounds address
        // (row n-1, step 0), so all loads are in flight at once; the steps
        // hold no features.
        const int g = lane >> 5;
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            const int64_t q = qbase + qt * 32 + (lane & 31);
            const int64_t qc = q < a.n ? q : a.n - 1;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const bool v = s < ks_used;
                xfrag f = load_frag(a, qc, v ? s : 0, g);
                if (!v)
                    f = no_features();
                xr[qt][s] = f;
            }
        }
    }

    // Direct-staged features.  Reading fragments straight from global memory
    // touches 32 rows per load (16 bytes of each) and takes every 128-byte
    // line four times through an L1 it does not fit: 13.6 thousand cycles for
    // a workgroup's 256 x 640 bytes.  Instead each wave copies its own rows
    // into its part of the ring past stage 0 (which is receiving the first
    // chunk meanwhile) with full-line loads, in pieces of one 128-byte line of
    // each row of a query tile, XNB pieces in flight, and takes the fragments
    // from LDS.
    // Rows past n re-read row n - 1 (their results are not stored, or stored
    // over row n - 1 with the same value).
    static constexpr int XAREA = (NBUF - 1) * SSZ / kWaves / 1024 * 1024;   // bytes per wave
    static constexpr int KSX = KS * KSTEP < 128 ? KS : 128 / KSTEP;   // K steps per piece
    static constexpr int UPX = KSX * KSTEP / 16 + 1;       // 16-byte units per row (one of skew)
    static constexpr int NXL = (32 * UPX + 63) / 64;       // loads per piece
    static constexpr int NPQ = (KS + KSX - 1) / KSX;       // pieces per query tile
    static constexpr int XNB0 = XAREA / (NXL * 1024);
    static constexpr int XNB = XNB0 < QT * NPQ ? XNB0 : QT * NPQ;
    static constexpr bool XLDS = DMA && XNB > 0;           // else (64 features, one tile) directly
    // waits until at most `pieces` pieces are in flight
    static __device__ __forceinline__ void wait_loads(int pieces)
    {
        switch (pieces) {
        case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        case 1: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NXL) : "memory"); break;
        case 2: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NXL) : "memory"); break;
        case 3: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NXL) : "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * NXL) : "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(5 * NXL) : "memory"); break;
        }
    }
    static __device__ __forceinline__ void load_x_lds(xfrag (&xr)[QT][KS], const EncodeArgs &a, lds_u8 *area,
                                                      int64_t qbase, int lane, int ks_used)
    {
        const int g = lane >> 5;
        const bool sgn = a.x_type == X_INT8;
        const int npx = ks_used * KSTEP / 16;              // 16-byte pieces of a row holding features
        const int64_t q0 = qbase < a.n ? qbase : a.n - 1;
        const int last = a.n - q0 < QPW ? (int)(a.n - q0) - 1 : QPW - 1;
        const uint8_t *xb = (const uint8_t *)a.X + q0 * a.ldx;
        // A wave with all its rows and 32-bit offsets within them: offsets of a
        // piece's units computed once, the piece in the scalar base; units past
        // the row's features read on (cut at the last row's end), and are
        // cleared below with the rest of the bytes past F.  Otherwise unit by
        // unit, to the byte.
        const bool full = qbase + QPW <= a.n && a.ldx < (1 << 24);
        uint32_t off[NXL];
#pragma unroll
        for (int i = 0; i < NXL; ++i) {
            const int u = i * 64 + lane;
            off[i] = (uint32_t)__umul24(u / UPX < 32 ? u / UPX : 31, (int)a.ldx) + 16u * (uint32_t)(u % UPX);
        }
        auto issue = [&](int j) {
            const int qt = j / NPQ, kp = j % NPQ;
            lds_u8 *dst = area + (j % XNB) * (NXL * 1024);
            if (full) {
                const uint32_t po = (uint32_t)__umul24(qt * 32, (int)a.ldx) + kp * (KSX * KSTEP);
                const uint32_t lim = (uint32_t)__umul24(QPW - 1, (int)a.ldx) + 16u * (uint32_t)(npx - 1) - po;
#pragma unroll
                for (int i = 0; i < NXL; ++i)
                    lds_dma16(xb + po, off[i] < lim ? off[i] : lim, dst + i * 1024);
            } else {
                int r = qt * 32 + lane / UPX, p = lane % UPX;  // unit i * 64 + lane of the piece
#pragma unroll 1
                for (int i = 0; i < NXL; ++i) {
                    const int row = r < last ? r : last;
                    const int pc = p + kp * (UPX - 1);
                    lds_dma16(xb + row * a.ldx + (pc < npx ? 16 * pc : 0), dst + i * 1024);
                    r += 64 / UPX;
                    p += 64 % UPX;
                    if (p >= UPX) {
                        p -= UPX;
                        ++r;
                    }
                }
            }
        };
#pragma unroll
        for (int j = 0; j < XNB; ++j)
            issue(j);
#pragma unroll
        for (int j = 0; j < QT * NPQ; ++j) {
            const int qt = j / NPQ, kp = j % NPQ;
            wait_loads(QT * NPQ - 1 - j < XNB - 1 ? QT * NPQ - 1 - j : XNB - 1);
            lds_u8 *xrow = area + (j % XNB) * (NXL * 1024) + (lane & 31) * (UPX * 16);
            // clear the bytes past F
            constexpr int PB = KSX * KSTEP;
            const int f0 = a.F - kp * PB;                  // first such byte of the piece
            const int fe = (KS - kp * KSX < KSX ? KS - kp * KSX : KSX) * KSTEP;
            if (f0 < fe) {
                const int o = f0 > 0 ? f0 : 0;
                if ((o & 3) && g == 0) {
                    lds_i32 *w = (lds_i32 *)(xrow + (o & ~3));
                    *w = *w & (int)((1u << (8 * (o & 3))) - 1u);
                }
#pragma unroll 1
                for (int w = (o + 3) / 4 + g; w < fe / 4; w += 2)
                    ((lds_i32 *)xrow)[w] = 0;
                __builtin_amdgcn_wave_barrier();           // (LDS operations of a wave are in order)
            }
            const lds_u8 *src = xrow + g * (KSTEP / 2);
#pragma unroll
            for (int s = 0; s < KSX; ++s) {
                if (kp * KSX + s >= KS)
                    break;
                uint32_t d[XW];
#pragma unroll
                for (int i = 0; i < XW / 4; ++i) {
                    const v4i w = *(const lds_v4i *)(src + s * KSTEP + 16 * i);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        d[4 * i + e] = (uint32_t)w[e];
                }
                xr[qt][kp * KSX + s] = conv_bytes(d, 0, KSTEP, sgn);   // already cleared past F
            }
            // the reads are done before the next piece lands on them
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (j + XNB < QT * NPQ)
                issue(j + XNB);
        }
    }

    // Start of chain 0 of each query tile on the int8 path: with the
    // shifted projection (weights p + 1 in {0, 2}, poff set) the MFMAs add
    // sum_i x_i (p_i + 1) = y + sum_i x_i, so the chain starts from minus
    // the query's feature sum and ends at y exactly (integer arithmetic);
    // otherwise from 0.  Lane l holds half of every K step of query l % 32
    // (features past F are zero in xr); the two halves are added across the
    // lane pair.  Shifted weights are mostly zero bits: the matrix cores
    // switch far fewer of them than on +-1 (0x01 / 0xFF) and hold a higher
    // clock under full load.  The E4M3 path (weights 0 / 2.0) takes minus
    // the sum of its rounded features from the matrix cores (an all -1.0
    // operand against the query fragments; integers below 2^24, exact in
    // fp32).  Only the shapes the shifted types launch take the shifted
    // projection (shift_tile with two query tiles, shift8_tile); the others
    // start from 0.
    static constexpr bool kShift = DMA && SRC == W_ROWS && ((QT == 2 && CT == C_I8 && shift_tile(KS, KT)) ||
                                                            (CT == C_FP8 && shift8_tile(KS, KT)));
    static __device__ __forceinline__ void shift_start(acc_t (&x0)[QT], const xfrag (&xr)[QT][KS], int poff)
    {
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            x0[qt] = acc_t{};
            if (!kShift || !poff)
                continue;
            if constexpr (kShift && CT == C_FP8) {
                frag neg;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    neg[i] = (int)0xB8B8B8B8u;   // E4M3 -1.0 bytes
#pragma unroll
                for (int k = 0; k < KS; ++k)
                    mma(x0[qt], neg, xr[qt][k]);
            } else if constexpr (kShift) {
                int s = 0;
#pragma unroll
                for (int k = 0; k < KS; ++k)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        s = __builtin_amdgcn_sdot4(xr[qt][k][e], 0x01010101, s, false);
                s += __shfl_xor(s, 32);
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    x0[qt][i] = -s;
            }
        }
    }

    // ---------------------------------------------------------------- P
    // Thread t stages row t/8 of the chunk, pieces t%8 + 8m.
    static __device__ __forceinline__ void stage_load(uint4 (&pr)[MP], const EncodeArgs &a, int c,
                                                      int t, int npc)
    {
        // Branch-free: rows past the dimension list re-read row S_0 and
        // pieces past the row re-read piece 0; stage_store discards both.
        const int r = t >> 3, sub = t & 7;
        const int dl = c * kDimChunk + r;
        const int dlc = dl < a.nd ? dl : 0;
        const int8_t *rowp = a.P + (int64_t)(a.s0 + (int64_t)dlc * a.stride) * a.ldp;
#pragma unroll
        for (int m = 0; m < MP; ++m) {
            const int j = sub + 8 * m;
            pr[m] = *(const uint4 *)(rowp + 16 * (j < npc ? j : 0));
        }
    }

    // Zero the part of every LDS row past the staged pieces (both buffers),
    // so that the fixed-length K loop multiplies zero features by finite
    // weights there.  Disjoint from what stage_store writes.
    static __device__ __forceinline__ void zero_tails(lds_u8 *lp0, lds_u8 *lp1, int t, int npc)
    {
        const int r = t >> 3, sub = t & 7;
        const int used16 = npc * T::ESZ, tot16 = KS * KB / 16;
        for (int u = used16 + sub; u < tot16; u += 8) {
            lds_st16(lp0 + r * RSB + 16 * u, make_uint4(0, 0, 0, 0));
            lds_st16(lp1 + r * RSB + 16 * u, make_uint4(0, 0, 0, 0));
        }
    }

    static __device__ __forceinline__ void stage_store(lds_u8 *lp, lds_i32 *lcs, const uint4 (&pr)[MP],
                                                       const EncodeArgs &a, int c, int t, int npc,
                                                       bool colsum)
    {
        const int r = t >> 3, sub = t & 7;
        const bool valid = c * kDimChunk + r < a.nd;
        lds_u8 *rowl = lp + r * RSB;
        int cs = 0;
#pragma unroll
        for (int m = 0; m < MP; ++m) {
            const int j = sub + 8 * m;
            if (j >= npc)
                continue;
            uint32_t d[4] = {pr[m].x, pr[m].y, pr[m].z, pr[m].w};
            if (colsum) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // sum of the +-1 weights of features < F in this dword
                    int k0 = 16 * j + 4 * e;
                    int nv = a.F - k0;
                    nv = nv < 0 ? 0 : (nv > 4 ? 4 : nv);
                    uint32_t neg = d[e] & 0x80808080u & (nv >= 4 ? 0xffffffffu : ((1u << (8 * nv)) - 1u));
                    cs += valid ? nv - 2 * __popc(neg) : 0;
                }
            }
            if constexpr (CT == C_I8) {
                lds_st16(rowl + 16 * j, valid ? pr[m] : make_uint4(0, 0, 0, 0));
            } else if constexpr (CT == C_FP8 || CT == C_FP8S) {
                uint4 o;
                uint32_t *op = (uint32_t *)&o;
#pragma unroll
                for (int e = 0; e < 4; ++e)   // +1 -> 0x38, -1 -> 0xB8 (E4M3)
                    op[e] = valid ? ((d[e] & 0x80808080u) | 0x38383838u) : 0u;
                lds_st16(rowl + 16 * j, o);
            } else if constexpr (CT == C_BF16) {
                // 16 weights -> 16 bf16: +1 -> 0x3F80, -1 -> 0xBF80
                uint32_t o[8];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t sg = d[e] & 0x80808080u;
                    o[2 * e] = valid ? (0x3F803F80u | ((sg & 0x80u) << 8) | ((sg & 0x8000u) << 16)) : 0u;
                    o[2 * e + 1] = valid ? (0x3F803F80u | ((sg >> 8) & 0x8000u) | (sg & 0x80000000u)) : 0u;
                }
                lds_st16(rowl + 32 * j, make_uint4(o[0], o[1], o[2], o[3]));
                lds_st16(rowl + 32 * j + 16, make_uint4(o[4], o[5], o[6], o[7]));
            } else {   // C_F32
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t s = d[e] & 0x80808080u;
                    uint4 o = valid ? make_uint4(0x3F800000u | ((s & 0x80u) << 24), 0x3F800000u | ((s & 0x8000u) << 16),
                                                 0x3F800000u | ((s & 0x800000u) << 8), 0x3F800000u | (s & 0x80000000u))
                                    : make_uint4(0, 0, 0, 0);
                    lds_st16(rowl + 64 * j + 16 * e, o);
                }
            }
        }
        if (colsum) {
            cs += __shfl_xor(cs, 1);
            cs += __shfl_xor(cs, 2);
            cs += __shfl_xor(cs, 4);
            if (sub == 0)
                lcs[r] = cs;
        }
    }

    // ------------------------------------------------------------ classes
    static __device__ __forceinline__ uint4 class_load(const EncodeArgs &a, int c, int t)
    {
        // threads past the table re-read entry 0 (discarded by class_store)
        const int tc = t < KT * 64 ? t : 0;
        return *(const uint4 *)(a.ctab + ((int64_t)c * KT * 64 + tc) * 16);
    }
    static __device__ __forceinline__ void class_store(lds_u8 *lc, uint4 v, int t)
    {
        if (t < KT * 64)
            lds_st16(lc + t * 16, v);
    }

    // ------------------------------------------------------------ compute
    // Accumulator chains of a row tile, K step s in chain s % KC, added in the
    // epilogue.  fp32 features round, so their order is that of the width
    // (fp32_chains).  Integer features are exact in any order; there a
    // single-tile wave alternates between two, so that a product does not wait
    // for the one before it (back to back the int8 32x32x32 form keeps its 32
    // cycles in one chain as well; with LDS waits between them two chains
    // measured faster), unless it is register staged and compiled for two waves
    // per SIMD, which has no room for the second set and relies on the other
    // wave instead; two query tiles are two chains already.
    // The split E4M3 type always has two: its high parts accumulate in the
    // first, its low parts in the second (|sums| < 2^24, exact).
    static constexpr int KC = XF == 1         ? fp32_chains(CT, KS)
                              : CT == C_FP8S ? 2
                              : (QT == 1 && (WAVES == 1 || DMA) && KS >= 2) ? 2 : 1;
    typedef acc_t Parts[QT][KC];             // accumulators of one row tile
    static constexpr int kPhases = 4 * QT;   // epilogue phases (see Epilogue)

    // Work interleaved with a pass: at(s) runs after the MFMAs of K step s,
    // tail() after the loop.
    struct NoHook {
        __device__ __forceinline__ void at(int) const {}
        __device__ __forceinline__ void tail() const {}
    };

    // One pass over a row tile (32 dimensions) in LDS: a fixed-length,
    // branch-free K loop with PD projection fragments in flight (steps past
    // the feature count read zero-filled or finite LDS against zero
    // features).  Chain 0 of every query tile starts from x0 (minus the
    // query's feature sum on the shifted projection, else 0), or from the
    // uint8 correction 128 * sum_i p_i of its rows.  The hook's work (the
    // previous row tile's epilogue, the next chunk's loads) issues between
    // the MFMAs, while the matrix core is busy.
    template <class Hook>
    static __device__ __forceinline__ void tile_mma(Parts &part, const xfrag (&xr)[QT][KS], const lds_u8 *lp,
                                                    const lds_i32 *lcs, bool colsum, int lane, const Hook &hook,
                                                    const acc_t (&x0)[QT])
    {
        const int g = lane >> 5, row = lane & 31;
        const lds_u8 *base = lp + row * RSB + g * (KB / 2);
        constexpr int PDW = (CT == C_I8 && (WAVES == 1 || DMA)) ? 4 : (CT == C_F32 ? 4 : 2);
        constexpr int PD = KS < PDW ? KS : PDW;
        frag f[PD];
#pragma unroll
        for (int s = 0; s < PD; ++s)
            f[s] = *(const HDC_LDS frag *)(base + s * KB);
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll
            for (int k = 0; k < KC; ++k)
                part[qt][k] = k == 0 ? x0[qt] : acc_t{};
        if constexpr (CT == C_I8) {
            if (colsum) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const v4i cs = *(const lds_v4i *)(lcs + 8 * j + 4 * g);
#pragma unroll
                    for (int qt = 0; qt < QT; ++qt)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            part[qt][0][4 * j + i] = 128 * cs[i];
                }
            }
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const frag cur = f[s % PD];
            if (s + PD < KS)
                f[s % PD] = *(const HDC_LDS frag *)(base + (s + PD) * KB);
            if constexpr (CT == C_FP8S) {
#pragma unroll
                for (int qt = 0; qt < QT; ++qt)
                    mma(part[qt][0], cur, split_hi(xr[qt][s]));
#pragma unroll
                for (int qt = 0; qt < QT; ++qt)
                    mma(part[qt][1], cur, split_lo(xr[qt][s]));
            } else {
#pragma unroll
                for (int qt = 0; qt < QT; ++qt)
                    mma(part[qt][s % KC], cur, xr[qt][s]);
            }
            hook.at(s);
            __builtin_amdgcn_sched_barrier(0);
        }
        hook.tail();
    }

    // Epilogue of row tile w (dimensions S_{32w .. 32w+31}) split into
    // phases; per query tile qt:
    //   4qt     adds the KC partial accumulators
    //   classify: 4qt+1, 4qt+2 turn the signs into {0,-1} bytes (the B
    //             operand), 4qt+3 runs the Hamming MFMAs against the class
    //             fragments of the tile
    //   encode:   4qt+1, 4qt+2 pack the 16 signs of the lane, join the two
    //             lane halves and clear dimensions past the end, 4qt+3
    //             stores the 32-bit word
    struct Epilogue {
        const EncodeArgs &a;
        Parts &part;
        v16i (&dacc)[KT][QT];
        const v4i (&cf)[KT];
        int w, lane, g;
        int64_t qbase;
        mutable v4i mb[QT];
        mutable uint32_t bits[QT];

        __device__ __forceinline__ void operator()(int p) const
        {
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) {
                const int ph = p - 4 * qt;
                const acc_t &y = part[qt][0];
                if (ph == 0) {
                    if constexpr (CT == C_FP8 || CT == C_FP8S) {
                        // The 16-pass E4M3 MFMA's accumulator was observed to
                        // be read one wait state early by the compiler-inserted
                        // hazard padding; extra wait states keep the read clear.
                        __builtin_amdgcn_sched_barrier(0);
                        asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (KC == 2)
                        part[qt][0] += part[qt][1];
                } else if (ph == 1 || ph == 2) {
                    if constexpr (MODE == M_CLASSIFY) {
#pragma unroll
                        for (int e = 2 * (ph - 1); e < 2 * ph; ++e) {
                            // bytes: 0xFF where the projection is negative, else 0
                            const uint32_t t0 = __builtin_amdgcn_perm(sign_word(y[4 * e + 1]),
                                                                      sign_word(y[4 * e]), 0x0C0C0B09u);
                            const uint32_t t1 = __builtin_amdgcn_perm(sign_word(y[4 * e + 3]),
                                                                      sign_word(y[4 * e + 2]), 0x0B090C0Cu);
                            mb[qt][e] = (int)(t0 | t1);
                        }
                    } else {
                        uint32_t b = ph == 1 ? 0u : bits[qt];
#pragma unroll
                        for (int v = 8 * (ph - 1); v < 8 * ph; ++v)
                            b |= (sign_word(y[v]) >> 31) << (8 * (v >> 2) + (v & 3));
                        if (ph == 2) {
                            b <<= 4 * g;
                            b |= (uint32_t)__shfl_xor((int)b, 32);
                            const int nv = a.nd - w * kDimChunk;   // dimensions of this tile
                            if (nv < 32)
                                b &= nv > 0 ? (1u << nv) - 1u : 0u;
                        }
                        bits[qt] = b;
                    }
                } else if (ph == 3) {
                    if constexpr (MODE == M_CLASSIFY) {
#pragma unroll
                        for (int kt = 0; kt < KT; ++kt)
                            mma(dacc[kt][qt], cf[kt], mb[qt]);
                    } else {
                        const int64_t q = qbase + qt * 32 + (lane & 31);
                        if (g == 0 && q < a.n)
                            a.H32[q * a.ldh32 + w] = bits[qt];
                    }
                }
            }
        }
    };

    static __device__ __forceinline__ void run_epilogue(const Epilogue &epi)
    {
#pragma unroll
        for (int p = 0; p < kPhases; ++p)
            epi(p);
    }

    // The epilogue as a pass hook: phase p after K step p * SP.
    static constexpr int SP = KS >= 2 * kPhases ? 2 : 1;
    struct EpiHook {
        Epilogue epi;
        __device__ __forceinline__ void at(int s) const
        {
            if (s % SP == 0 && s / SP < kPhases)
                epi(s / SP);
        }
        __device__ __forceinline__ void tail() const
        {
#pragma unroll
            for (int p = (KS + SP - 1) / SP; p < kPhases; ++p)
                epi(p);
        }
    };
    template <class H1, class H2> struct Both;
    template <class H1, class H2>
    static __device__ __forceinline__ Both<H1, H2> both(const H1 &h1, const H2 &h2)
    {
        return Both<H1, H2>{h1, h2};
    }
    template <class H1, class H2>
    struct Both {
        H1 h1;
        H2 h2;
        __device__ __forceinline__ void at(int s) const
        {
            h1.at(s);
            h2.at(s);
        }
        __device__ __forceinline__ void tail() const
        {
            h1.tail();
            h2.tail();
        }
    };

    // ------------------------------------------------------------ body
    // Runs the whole dimension loop for the queries of this workgroup.
    // Returns the class accumulators (classify mode) through dacc.
    static __device__ __forceinline__ void run(const EncodeArgs &a, uint8_t *smem, int64_t qblock,
                                               v16i (&dacc)[KT][QT])
    {
        if constexpr (DMA)
            run_dma(a, smem, qblock, dacc);
        else
            run_db(a, smem, qblock, dacc);
    }

    // Register-staged loop over a double-buffered LDS stage: step c
    // prefetches chunk c+1 into registers, multiplies chunk c while chunk
    // c-1's epilogue runs between its MFMAs, reads chunk c's class fragments
    // into registers, stores chunk c+1 into the other buffer and
    // synchronises once.  The two accumulator sets alternate, so the loop is
    // unrolled by two.
    static __device__ __forceinline__ void run_db(const EncodeArgs &a, uint8_t *smem, int64_t qblock,
                                                  v16i (&dacc)[KT][QT])
    {
        const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 5;
        const int64_t qbase = qblock + (int64_t)wave * QPW;
        const int ks_used = (a.F + KSTEP - 1) / KSTEP;
        const int npc = (ks_used * KSTEP + 15) / 16;
        const int NC = (a.nd + kDimChunk - 1) / kDimChunk;
        const bool colsum = CT == C_I8 && XF == 0 && a.x_type == X_UINT8;

        xfrag xr[QT][KS];
        load_x(xr, a, qbase, lane, ks_used);
        const acc_t x0[QT] = {};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int qt = 0; qt < QT; ++qt)
                dacc[kt][qt] = v16i{};

        lds_u8 *L = (lds_u8 *)smem;
        lds_u8 *lp[2] = {L, L + kDimChunk * RSB};
        lds_u8 *lc[2] = {L + OFF_C, L + OFF_C + KT * 1024};
        lds_i32 *lcs[2] = {(lds_i32 *)(L + OFF_CS), (lds_i32 *)(L + OFF_CS) + kDimChunk};

        uint4 pr[MP];
        uint4 cr = make_uint4(0, 0, 0, 0);
        zero_tails(lp[0], lp[1], t, npc);
        stage_load(pr, a, 0, t, npc);
        if constexpr (MODE == M_CLASSIFY)
            cr = class_load(a, 0, t);
        stage_store(lp[0], lcs[0], pr, a, 0, t, npc, colsum);
        if constexpr (MODE == M_CLASSIFY)
            class_store(lc[0], cr, t);
        __syncthreads();

        v4i cf[KT];
        auto step = [&](int c, int b, Parts &cur, const auto &hook) {
            const bool more = c + 1 < NC;
            // prefetch the next chunk (the last step re-reads in-bounds data
            // and discards it, keeping the loop free of branches)
            stage_load(pr, a, c + 1, t, npc);
            if constexpr (MODE == M_CLASSIFY)
                cr = class_load(a, more ? c + 1 : c, t);
            tile_mma(cur, xr, lp[b], lcs[b], colsum, lane, hook, x0);
            if constexpr (MODE == M_CLASSIFY) {
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
                    cf[kt] = *(const lds_v4i *)(lc[b] + (kt * 64 + lane) * 16);
            }
            if (more) {
                stage_store(lp[b ^ 1], lcs[b ^ 1], pr, a, c + 1, t, npc, colsum);
                if constexpr (MODE == M_CLASSIFY)
                    class_store(lc[b ^ 1], cr, t);
            }
            __syncthreads();
        };

        Parts P0, P1;
        step(0, 0, P0, NoHook{});
        for (int c = 1;; c += 2) {
            if (c >= NC) {
                run_epilogue(Epilogue{a, P0, dacc, cf, c - 1, lane, g, qbase});
                break;
            }
            step(c, 1, P1, EpiHook{Epilogue{a, P0, dacc, cf, c - 1, lane, g, qbase}});
            if (c + 1 >= NC) {
                run_epilogue(Epilogue{a, P1, dacc, cf, c, lane, g, qbase});
                break;
            }
            step(c + 1, 0, P0, EpiHook{Epilogue{a, P1, dacc, cf, c, lane, g, qbase}});
        }
        if constexpr (MODE == M_ENCODE) {
            if (NC & 1) {   // high half of the last word holds no dimension
#pragma unroll
                for (int qt = 0; qt < QT; ++qt) {
                    const int64_t q = qbase + qt * 32 + (lane & 31);
                    if (g == 0 && q < a.n)
                        a.H32[q * a.ldh32 + NC] = 0u;
                }
            }
        }
    }

    // ------------------------------------------------------------ DMA
    // Source of each of this lane's NIW loads: LDS unit u = piece * 64 +
    // lane of a stage is row u / UPR, piece u % UPR; the skew unit and
    // pieces past the features re-read piece 0 (finite weights against zero
    // features), units past the chunk's rows land in slack.  Row r of chunk c
    // is dimension S_{c*CH + r}.  Each chunk is a buffer of its own, from its
    // first row to the last dimension's last piece (row_window): offsets past
    // it are refused by the load's range check, which covers the per-lane
    // offset, so no address outside the projection is formed; those rows'
    // results are masked, or meet zero class bytes.  (The chunk offset in the
    // scalar offset instead, over one buffer of all rows, is not known to be
    // checked.)  Byte offsets fit 32 bits: the projection is below 2^32 bytes.
    struct Loader {
        const EncodeArgs &a;
        uint32_t off0[NIW];   // offset of load i in a chunk
        const int8_t *first;  // row of the set's first dimension
        uint32_t rstep, rbytes;
        int NC, lane, wave;

        __device__ __forceinline__ Loader(const EncodeArgs &a_, int NC_, int npc, int wave_, int lane_)
            : a(a_), first(a_.P + (uint32_t)a_.s0 * (uint32_t)a_.ldp),
              rstep((uint32_t)a_.stride * (uint32_t)a_.ldp), rbytes(16u * (uint32_t)npc), NC(NC_), lane(lane_),
              wave(wave_)
        {
#pragma unroll
            for (int i = 0; i < NIW; ++i) {
                const int u = piece(i) * 64 + lane;
                const int r = u / UPR < CH ? u / UPR : CH - 1, p = u % UPR;
                off0[i] = (uint32_t)r * rstep + 16u * (uint32_t)(p < npc ? p : 0);
            }
        }
        // KiB of the stage that load i of this wave fills
        __device__ __forceinline__ int piece(int i) const
        {
            return i * kWaves + kWaves <= NU || i * kWaves + wave < NU ? i * kWaves + wave : NU - 1;
        }
        // Chunk c, or the last chunk from there on (the class table holds a
        // whole number of chunks, zero rows past nd), as scalars.
        struct Chunk {
            uint32_t cc;
            v4i rows;
        };
        __device__ __forceinline__ Chunk chunk(int c) const
        {
            const RowWindow w = row_window(c, CH, a.nd, rstep, rbytes);
            return Chunk{(uint32_t)(c < NC ? c : NC - 1), raw_buffer(first + w.off, w.bytes)};
        }
        // Load i (< NIW + NCW) of a chunk: the projection rows, then the class
        // fragments (wave w loads class tiles (w + 4j) % NCT; duplicate tiles
        // write the same bytes).
        __device__ __forceinline__ void issue(int i, const Chunk &c, lds_u8 *stage, lds_u8 *lcls) const
        {
            if (i < NIW) {
                lds_dma16(c.rows, off0[i], stage + piece(i) * 1024);
            } else if constexpr (MODE == M_CLASSIFY) {
                const int tile = (wave + kWaves * (i - NIW)) % NCT;   // rt * KT + kt
                lds_dma16(a.ctab + (c.cc * NCT + tile) * 1024, (uint32_t)(lane * 16), lcls + tile * 1024);
            }
        }
        __device__ __forceinline__ void all(int c, lds_u8 *stage, lds_u8 *lcls) const
        {
            const Chunk ch = chunk(c);
#pragma unroll
            for (int i = 0; i < NIW + (MODE == M_CLASSIFY ? NCW : 0); ++i)
                issue(i, ch, stage, lcls);
        }
    };
    static constexpr int NLOADS = NIW + (MODE == M_CLASSIFY ? NCW : 0);   // loads per wave per chunk

    // MFMAs are issued in order and each holds the matrix core for 32 (int8)
    // or 64 cycles, so between two of them a wave can issue about 7 (15) other
    // instructions for free and more than that stalls it.  The work beside
    // the MFMAs is therefore cut into pieces of a few instructions, handed
    // out by slot: slot s * MPS + m follows MFMA m of K step s; the first
    // fragments of the next pass are read before this one ends, so passes
    // follow each other without an LDS wait.  Per MFMA of 32 cycles at 617
    // features: 42 cycles with a loop that drained at each row tile, 38 so
    // (classify), 52 and 37 (encode); on large batches the clock, which falls
    // as the cores fill, takes most of that back (262144 x 617, 10240
    // dimensions: 1209 us, 1160 so).
    static constexpr int MPS = CT == C_FP8S ? 2 : QT;      // MFMAs per K step
    static_assert(!DMA || CT != C_FP8S || QT == 1, "the split E4M3 type takes one query tile");
    static constexpr int SLOTS = KS * MPS;

    // The loads of one chunk as a pass hook: load i in slot SL + i * MPS (the
    // slots that hold no piece of the epilogue).
    template <int SL> struct LoadHook {
        const Loader &ld;
        typename Loader::Chunk c;
        lds_u8 *stage, *lcls;
        static constexpr int LSP = MPS;
        static constexpr int IN = SL < SLOTS ? (SLOTS - SL + LSP - 1) / LSP : 0;   // loads in slots
        __device__ __forceinline__ void at(int s) const
        {
            if (s >= SL && (s - SL) % LSP == 0 && (s - SL) / LSP < NLOADS)
                ld.issue((s - SL) / LSP, c, stage, lcls);
        }
        __device__ __forceinline__ void tail() const
        {
#pragma unroll
            for (int i = IN; i < NLOADS; ++i)
                ld.issue(i, c, stage, lcls);
        }
    };

    // Wait until at most G of this wave's vector memory operations are in
    // flight (they complete in issue order, so everything older is done) and
    // meet the other waves; with DRAIN also for this wave's LDS reads.
    template <int G, bool DRAIN>
    static __device__ __forceinline__ void dma_barrier()
    {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (DRAIN)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(G) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(G) : "memory");
        __builtin_amdgcn_sched_barrier(0);
    }

    // ------------------------------------------------ direct-staged passes
    // Projection fragments in flight (the ring f): KS * RT (RT * KS over the
    // two unrolled steps with RT = 1) is a multiple of PDD, so every pass
    // starts at a fixed slot.
    static constexpr int PDD = KS < 4 ? KS : (CT == C_I8 ? 4 : 2);
    // A pass takes its first PDD fragments from the previous pass, which
    // reads them between its last MFMAs, so the matrix cores do not wait for
    // LDS at a row tile's start.  With one row tile per chunk the barrier
    // that makes the next chunk visible then has to come inside the pass,
    // after K step BAR (> PDD: by then every LDS read of the previous chunk
    // has been waited for) and before the first of those reads; shorter
    // passes synchronise between the chunks instead.
    static constexpr int BAR = PDD + 1;
    static constexpr bool XPF = RT == 2 || BAR < KS - PDD;

    static __device__ __forceinline__ frag read_frag(const lds_u8 *p) { return *(const HDC_LDS frag *)p; }

    // The A operand of a fragment: int8 +-1 bytes become E4M3 +-1.0 (0x38 /
    // 0xB8) on the converting kernels: one operation per dword, in the shadow
    // of the MFMAs it feeds.
    static __device__ __forceinline__ frag weights(frag f)
    {
        if constexpr (CVT) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                f[i] = (int)(((uint32_t)f[i] & 0x80808080u) | 0x38383838u);
        }
        return f;
    }

    // uint8 features are multiplied as x - 128, so a row tile's sums start
    // from 128 * sum_i p_i of each dimension.  The four waves share these sums
    // as a pass hook two tiles ahead: each takes 8 of the tile's 32 rows, 8
    // lanes a row, a few 16-byte reads spread over the pass, and leaves them
    // in LDS, two buffers in turn; the next pass's barrier makes them visible
    // and that pass reads them as the accumulators of the one after.  Vector
    // instructions cost about 3 cycles each beside the MFMAs (dot products
    // 15), so bytes are summed as sad(b ^ 0x80, 0) = b + 128, two operations
    // per dword, and the shared sums come without any per accumulator: 51.8
    // cycles per MFMA at 784 features before, 43.8 now.  The sum covers
    // every byte multiplied, pad columns included: there the query operand is
    // -128 and the two terms cancel.
    static constexpr int SJ = (KS * KSTEP / 16 + 7) / 8;   // reads per lane and tile
    struct SumHook {
        const lds_u8 *row;           // this lane's row and first piece of the tile
        lds_i32 *out;                // its sum's place
        bool last;                   // the last read is within the row
        bool write;
        mutable v4i f;
        mutable uint32_t c;
        // after the barrier: read j in slot S0 + j * PER, summed two dwords at
        // a time in slots S0 + j * PER + PER - 2 and the next
        static constexpr int S0 = XPF ? (BAR + 1) * MPS : SLOTS;
        static constexpr int PER = (SLOTS - S0) / SJ > 4 ? (SLOTS - S0) / SJ : 4;
        __device__ __forceinline__ void read(int j) const { f = *(const lds_v4i *)(row + j * 128); }
        __device__ __forceinline__ void add(int j, int e) const
        {
            uint32_t t = j == 0 && e == 0 ? 0u : c;
            t = __builtin_amdgcn_sad_u8((uint32_t)f[e] ^ 0x80808080u, 0u, t);
            t = __builtin_amdgcn_sad_u8((uint32_t)f[e + 1] ^ 0x80808080u, 0u, t);
            c = j < SJ - 1 || last ? t : c;
        }
        __device__ __forceinline__ void at(int s) const
        {
            if (s < S0 || (s - S0) / PER >= SJ)
                return;
            const int j = (s - S0) / PER, r = (s - S0) % PER;
            if (r == 0)
                read(j);
            if (r == PER - 2)
                add(j, 0);
            if (r == PER - 1)
                add(j, 2);
        }
        __device__ __forceinline__ void tail() const
        {
#pragma unroll
            for (int j = 0; j < SJ; ++j) {
                if (S0 + j * PER >= SLOTS)
                    read(j);
                if (S0 + j * PER + PER - 2 >= SLOTS)
                    add(j, 0);
                if (S0 + j * PER + PER - 1 >= SLOTS)
                    add(j, 2);
            }
            // over the row's 8 lanes: lane ^ 1, lane ^ 2, mirrored eights
            int t = (int)c;
            t += __builtin_amdgcn_update_dpp(0, t, 0xB1, 0xF, 0xF, true);
            t += __builtin_amdgcn_update_dpp(0, t, 0x4E, 0xF, 0xF, true);
            t += __builtin_amdgcn_update_dpp(0, t, 0x141, 0xF, 0xF, true);
            if (write)
                *out = (t - 128 * KS * KSTEP) * 128;
        }
        __device__ __forceinline__ void all() const
        {
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                at(s);
            tail();
        }
    };

    // One pass over a row tile in LDS (base) that ends with the first PDD
    // fragments of the next one (nbase) in the ring; OFF is the ring slot of
    // the pass's first fragment.
    template <int OFF, class Hook>
    static __device__ __forceinline__ void tile_pass(Parts &part, const xfrag (&xr)[QT][KS], frag (&f)[PDD],
                                                     const lds_u8 *base, const lds_u8 *nbase, const Hook &hook, const acc_t (&x0)[QT])
    {
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll
            for (int k = 0; k < KC; ++k)
                part[qt][k] = k == 0 ? x0[U8 ? 0 : qt] : acc_t{};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const frag cur = weights(f[(OFF + s) % PDD]);
            if (s + PDD < KS)
                f[(OFF + s) % PDD] = read_frag(base + (s + PDD) * KB);
            else if constexpr (XPF)
                f[(OFF + s) % PDD] = read_frag(nbase + (s + PDD - KS) * KB);
#pragma unroll
            for (int m = 0; m < MPS; ++m) {
                if constexpr (CT == C_FP8S) {
                    if (m == 0)
                        mma(part[0][0], cur, split_hi(xr[0][s]));
                    else
                        mma(part[0][1], cur, split_lo(xr[0][s]));
                } else {
                    mma(part[m][s % KC], cur, xr[m][s]);
                }
                hook.at(s * MPS + m);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        hook.tail();
    }

    // Epilogue of row tile w in phases of a few instructions: per query tile,
    // EPG of them take four (or, where there is more to do than signs, two)
    // dimensions each (adding the partial accumulators, then the signs: bytes {0, -1} of the Hamming MFMA's B
    // operand, or bits), a last one runs the Hamming MFMAs or finishes the
    // word.  Encoding: a lane holds half the signs of a dimension tile for one
    // query of each query tile; one lane-half swap gives the lower lanes the
    // first tile's words and the upper lanes the second's, the 32-bit word of
    // an even tile (LO) waits in hw, and the odd tile's last phase stores
    // both as one 64-bit word per query (always issued, so that the barriers
    // can count it).
    static constexpr int EPG = KC == 2 ? 8 : 4;
    static constexpr int EPH = (EPG + 1) * QT;
    template <bool LO> struct EpiD {
        const EncodeArgs &a;
        Parts &part;
        v16i (&dacc)[KT][QT];
        const v4i (&cf)[KT];
        uint32_t &hw;
        uint32_t *hrow;              // packed row of this lane's query
        int w, lane;
        mutable v4i mb[QT];
        mutable uint32_t bits[QT];
        __device__ __forceinline__ void phase(int p) const
        {
            const int qt = p / (EPG + 1), ph = p % (EPG + 1);
            acc_t &y = part[qt][0];
            if (CT != C_I8 && ph == 0) {
                // The 16-pass E4M3 MFMA's accumulator was observed to be read
                // one wait state early by the compiler-inserted hazard
                // padding; extra wait states keep the read clear.
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
            if (ph < EPG) {
                constexpr int NV = 16 / EPG;
                const int v0 = 16 - NV * (ph + 1);         // registers v0 .. v0 + NV - 1
#pragma unroll
                for (int v = v0; v < v0 + NV; ++v) {
                    if constexpr (KC == 2)
                        y[v] += part[qt][1][v];
                }
                if constexpr (MODE == M_CLASSIFY) {
                    // bytes: 0xFF where the projection is negative, else 0
                    // (two registers to bytes 0, 1 or 2, 3)
#pragma unroll
                    for (int v = v0; v < v0 + NV; v += 2) {
                        const uint32_t t = __builtin_amdgcn_perm(sign_word(y[v + 1]), sign_word(y[v]),
                                                                 v & 2 ? 0x0B090C0Cu : 0x0C0C0B09u);
                        const int e = v >> 2;
                        mb[qt][e] = (v & 2) == (NV == 2 ? 2 : 0) ? (int)t : mb[qt][e] | (int)t;
                    }
                } else {
                    // signs shifted in from the top: register v lands on bit
                    // 8 * (v / 4) + v % 4
                    uint32_t b = ph == 0 ? 0u : bits[qt];
#pragma unroll
                    for (int v = v0 + NV - 1; v >= v0; --v) {
                        if (v % 4 == 3 && v < 15)
                            b <<= 4;
                        b = __builtin_amdgcn_alignbit(b, sign_word(y[v]), 31);
                    }
                    bits[qt] = b;
                }
            } else if constexpr (MODE == M_CLASSIFY) {
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
                    mma(dacc[kt][qt], cf[kt], mb[qt]);
            } else if (qt == QT - 1) {
                // lane half g holds bits 4g.. of every byte
                typedef unsigned v2u __attribute__((ext_vector_type(2)));
                const v2u sw = __builtin_amdgcn_permlane32_swap(bits[0], bits[QT - 1], false, false);
                const int nv = a.nd - w * kDimChunk;       // dimensions of this tile
                const uint32_t b = (sw[0] | (sw[1] << 4)) & (nv >= 32 ? ~0u : nv > 0 ? (1u << nv) - 1u : 0u);
                if constexpr (LO)
                    hw = b;
                else if (QT == 2 || lane < 32)             // the word of tiles w - 1 and w
                    *(uint2 *)(hrow + (w - 1)) = make_uint2(hw, b);
            }
        }
        __device__ __forceinline__ void all() const
        {
#pragma unroll
            for (int p = 0; p < EPH; ++p)
                phase(p);
        }
        // as a pass hook: phase p in slot E0 + p * SPD, the slot after a K
        // step's last MFMA
        static constexpr int E0 = MPS - 1;
        static constexpr int SPA = (SLOTS - E0) / EPH / MPS * MPS;
        static constexpr int SPD = SPA > MPS ? SPA : MPS;
        __device__ __forceinline__ void at(int s) const
        {
            if (s >= E0 && (s - E0) % SPD == 0 && (s - E0) / SPD < EPH)
                phase((s - E0) / SPD);
        }
        __device__ __forceinline__ void tail() const
        {
#pragma unroll
            for (int p = (SLOTS - E0 + SPD - 1) / SPD; p < EPH; ++p)
                phase(p);
        }
    };

    // The barrier of a one-row-tile pass; uint8: and, after it, the read of
    // the next tile's start values.
    static constexpr int BG = (NBUF - 2 - VIS) * NLOADS;   // loads it leaves in flight
    struct BarHook {
        const lds_i32 *sums;
        acc_t &start;
        __device__ __forceinline__ void read_start() const
        {
            if constexpr (U8) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const v4i v = *(const lds_v4i *)(sums + 8 * j);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        start[4 * j + i] = v[i];
                }
            }
        }
        __device__ __forceinline__ void at(int s) const
        {
            if (XPF && s == BAR * MPS + MPS - 1)
                dma_barrier<BG, false>();
            if (XPF && s == (BAR + 2) * MPS + MPS - 1)
                read_start();
        }
        __device__ __forceinline__ void tail() const
        {
            if (!XPF) {
                dma_barrier<BG, true>();
                read_start();
            }
        }
    };

    // Staged loop.  Pass by pass over the row tiles: each has the previous
    // tile's epilogue and (with two row tiles per chunk: the second pass; with
    // one: after the barrier) the loads of the chunk NBUF - 1 ahead between
    // its MFMAs, and reads its class fragments after its last one.  One
    // barrier per chunk, between the two passes or inside the only one: it
    // waits for the loads of the next chunk, issued NBUF - 2 chunks ago (only
    // younger ones may be in flight), and releases the stage of the previous
    // chunk.  Two accumulator sets alternate.
    static __device__ __forceinline__ void run_dma(const EncodeArgs &a, uint8_t *smem, int64_t qblock,
                                                   v16i (&dacc)[KT][QT])
    {
        const int lane = threadIdx.x & 63, g = lane >> 5;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // in a scalar register
        const int64_t qbase = qblock + (int64_t)wave * QPW;
        const int ks_used = (a.F + KSTEP - 1) / KSTEP;
        const int npc = (ks_used * KB + 15) / 16;   // 16-byte pieces of a row holding features
        const int NC = (a.nd + 63) / 64 * (64 / CH);   // whole 64-dimension words

        lds_u8 *L = (lds_u8 *)smem;
        auto lp = [&](int i) { return L + i * SSZ; };
        auto lc = [&](int i) { return L + OFF_C + i * (NCT * 1024); };
        const Loader ld(a, NC, npc, wave, lane);
        ld.all(0, lp(0), lc(0));
        xfrag xr[QT][KS];
        if constexpr (XLDS)
            load_x_lds(xr, a, L + SSZ + wave * XAREA, qbase, lane, ks_used);
        else
            load_x(xr, a, qbase, lane, ks_used);
        dma_barrier<0, true>();
#pragma unroll
        for (int c = 1; c < NBUF - 1; ++c)
            ld.all(c, lp(c), lc(c));
        acc_t x0[QT];
        shift_start(x0, xr, a.poff);
        if constexpr (kShift && CT == C_FP8) {
            // the E4M3 start values come from 16-pass MFMAs: wait states
            // before anything reads them (as in the epilogue)
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int qt = 0; qt < QT; ++qt)
                dacc[kt][qt] = v16i{};

        // this lane's packed output row: query g * 32 + l % 32 of the wave
        // (one query tile: l % 32); rows past n repeat row n - 1's store
        uint32_t *hrow = nullptr;
        uint32_t hw = 0;
        if constexpr (MODE == M_ENCODE) {
            const int64_t q = qbase + (QT == 2 ? lane : (lane & 31));
            hrow = a.H32 + (q < a.n ? q : a.n - 1) * a.ldh32;
        }

        const int loff = (lane & 31) * RSB + g * (KB / 2);
        frag f[PDD];
        auto fill = [&](const lds_u8 *base) {
#pragma unroll
            for (int s = 0; s < PDD; ++s)
                f[s] = read_frag(base + s * KB);
        };
        fill(lp(0) + loff);

        v4i cf[KT];
        int b = 0;   // stage of the chunk being multiplied
        auto nxt = [&](int i) { return i == NBUF - 1 ? 0 : i + 1; };
        auto base = [&](int st, int rt) { return lp(st) + rt * kDimChunk * RSB + loff; };
        // start values of tile w: buffer w % 2; lane l reads 8 j + 4 (l / 32)
        // .. + 3, and sums row 8 * wave + l / 8
        lds_i32 *lcs = (lds_i32 *)(L + OFF_CS);
        const int srow = 8 * wave + lane / 8;
        const lds_u8 *sbase = L + srow * RSB + (lane & 7) * 16;
        const bool slast = (SJ - 1) * 8 + (lane & 7) < KS * KSTEP / 16;
        auto sum = [&](int w, int st) {
            return SumHook{sbase + st * SSZ, lcs + (w & 1) * kDimChunk + srow, slast, (lane & 7) == 0};
        };
        auto bar = [&](int c) { return BarHook{lcs + ((c + 1) & 1) * kDimChunk + 4 * g, x0[0]}; };
        // after a pass: its class fragments
        auto after = [&](int rt) {
            if constexpr (MODE == M_CLASSIFY) {
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
                    cf[kt] = *(const lds_v4i *)(lc(b) + ((rt * KT + kt) * 64 + lane) * 16);
            }
        };
        auto loads = [&](int c, auto s0) {   // loads of chunk c + NBUF - 1 into the stage before b
            const int b2 = __builtin_amdgcn_readfirstlane(b == 0 ? NBUF - 1 : b - 1);   // (kept scalar)
            return LoadHook<decltype(s0)::value>{ld, ld.chunk(c + NBUF - 1), lp(b2), lc(b2)};
        };
        auto epi = [&](auto lo, Parts &prev, int w) {
            return EpiD<decltype(lo)::value>{a, prev, dacc, cf, hw, hrow, w, lane};
        };
        typedef std::integral_constant<bool, true> Lo;
        typedef std::integral_constant<bool, false> Hi;

        Parts P0, P1;
        if constexpr (RT == 2) {
            typedef std::integral_constant<int, 0> S0;
            constexpr int O1 = KS % PDD;
            // stores the barrier of a step may leave in flight: the one of
            // the epilogue between the awaited loads and the barrier
            constexpr int G = MODE == M_ENCODE ? 1 : 0;
            auto second = [&](int c) {
                tile_pass<O1>(P1, xr, f, base(b, 1), base(nxt(b), 0),
                              both(epi(Lo{}, P0, 2 * c), loads(c, S0{})), x0);
                after(1);
                b = nxt(b);
            };
            tile_pass<0>(P0, xr, f, base(b, 0), base(b, 1), NoHook{}, x0);
            after(0);
            dma_barrier<0, false>();
            second(0);
            for (int c = 1; c < NC; ++c) {
                tile_pass<0>(P0, xr, f, base(b, 0), base(b, 1), epi(Hi{}, P1, 2 * c - 1), x0);
                after(0);
                dma_barrier<G, false>();
                second(c);
            }
            epi(Hi{}, P1, 2 * NC - 1).all();
        } else {
            // tiles in pairs (an odd last one with a masked partner), so that
            // the two accumulator sets alternate without exits in between
            typedef std::integral_constant<int, (XPF ? (BAR + 1) * MPS : SLOTS)> S0;
            typedef std::integral_constant<int, (XPF ? KS % PDD : 0)> O1;
            typedef std::integral_constant<int, 0> O0;
            auto step = [&](auto off, Parts &cur, int c, const auto &e) {
                if constexpr (U8)
                    tile_pass<decltype(off)::value>(cur, xr, f, base(b, 0), base(nxt(b), 0),
                                                    both(both(both(e, bar(c)), sum(c + 2, nxt(nxt(b)))), loads(c, S0{})), x0);
                else
                    tile_pass<decltype(off)::value>(cur, xr, f, base(b, 0), base(nxt(b), 0),
                                                    both(both(e, bar(c)), loads(c, S0{})), x0);
                after(0);
                b = nxt(b);
                if constexpr (!XPF)
                    fill(base(b, 0));
            };
            if constexpr (U8) {   // start values of the first two tiles
                dma_barrier<(NBUF - 3) * NLOADS, false>();
                sum(0, 0).all();
                sum(1, 1).all();
                dma_barrier<(NBUF - 3) * NLOADS, true>();
                bar(-1).read_start();
            }
            step(O0{}, P0, 0, NoHook{});
            step(O1{}, P1, 1, epi(Lo{}, P0, 0));
            for (int c = 2; c < NC; c += 2) {
                step(O0{}, P0, c, epi(Hi{}, P1, c - 1));
                step(O1{}, P1, c + 1, epi(Lo{}, P0, c));
            }
            epi(Hi{}, P1, NC - 1).all();
        }
        // no load may still be writing this workgroup's LDS when it exits
        __builtin_amdgcn_s_waitcnt(0);
    }

    // Argmin over the class accumulators; returns the label of this lane's
    // query (valid in lanes 0..31 of each tile) and optionally writes dists.
    static __device__ __forceinline__ void finish(const EncodeArgs &a, int64_t qblock,
                                                  const v16i (&dacc)[KT][QT], int32_t (&lab)[QT])
    {
        const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 5;
        const int64_t qbase = qblock + (int64_t)wave * QPW;
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            const int64_t q = qbase + qt * 32 + (lane & 31);
            int bd = 0x7fffffff, bk = 0;
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int k = kt * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                    if (k < a.K) {
                        const int d = a.cpop[k] - dacc[kt][qt][v];
                        if (d < bd) { bd = d; bk = k; }
                        if (a.dists && q < a.n)
                            a.dists[q * a.K + k] = d;
                    }
                }
            const int od = __shfl_xor(bd, 32), ok = __shfl_xor(bk, 32);
            if (od < bd || (od == bd && ok < bk)) { bd = od; bk = ok; }
            lab[qt] = bk;
        }
    }
};

}  // namespace hdc
