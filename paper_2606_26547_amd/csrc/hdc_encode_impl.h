// Kernel entry points and launch dispatch of the encoder for one compute
// type.  Each hdc_encode_<type>.hip defines HDC_CT and includes this file,
// so the instantiations of the four compute types compile in parallel.
#pragma once

#include "hdc_encoder.h"

namespace hdc {

// Whether a split launch's partial sums are [z][n][K] (else [z][K][n]): from 65
// classes on, and from 33 on for few queries.  With the classes apart every
// workgroup of the argmin touches a line per class and split, however few its
// queries (60 x 64 E4M3, 10240 dimensions, 100 classes, 40 splits: 18.4 us with
// the encoder, 14 so; 1500 x 617 int8, 8192 dimensions, 128 classes 40 and 34); 50
// classes gain 2% below 1024 queries and lose 3% above.
constexpr int64_t kRowQueries = 1024;
__host__ __device__ __forceinline__ bool part_rows(int KT, int64_t n)
{
    return KT == 4 || (KT == 2 && n < kRowQueries);
}
// Place of (split, class, query) in them.
__device__ __forceinline__ int64_t part_at(const EncodeArgs &a, int KT, int z, int k, int64_t q)
{
    return part_rows(KT, a.n) ? ((int64_t)z * a.n + q) * a.K + k : ((int64_t)z * a.K + k) * a.n + q;
}

// Grid: query blocks, or (dimension split, query block) when the launch
// splits its dimensions (a.nsplit = Z > 1).  Split z of Z takes the whole
// 64-dimension words [z * per, (z + 1) * per) of the dimension list: its
// projection rows, its half-words of the packed output and its part of the
// class operand.  Workgroups are dealt to the XCDs in turn by linear id, so
// with the split index fastest each XCD's L2 holds the projection rows of
// its splits only, not all of them.  In classify mode every split adds its
// own part of the class sums, so a split launch writes them to
// part (part_rows) and k_split_argmin or k_split_argmin_rows finishes.
template <int CT, int XF, int QT, int KS, int KT, int MODE, bool DMA, int RT, int SRC>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(Encoder<CT, XF, QT, KS, KT, MODE, 0, DMA, RT, SRC>::REGW)))
void k_encode(EncodeArgs a)
{
    typedef Encoder<CT, XF, QT, KS, KT, MODE, 0, DMA, RT, SRC> E;
    __shared__ __align__(16) uint8_t smem[E::LDS];
    const int Z = a.nsplit;
    const int z = Z > 1 ? (int)blockIdx.x : 0;
    const int64_t qblock = (int64_t)(Z > 1 ? blockIdx.y : blockIdx.x) * E::QPB;
    if (Z > 1) {
        const int per = split_units(a.nd, Z);
        const int d0 = 64 * z * per;                    // first dimension (list index) of the split
        const int nd = a.nd - d0 < 64 * per ? a.nd - d0 : 64 * per;
        a.s0 += d0 * a.stride;
        a.nd = nd;
        if constexpr (MODE == M_ENCODE)
            a.H32 += d0 / 32;
        else
            a.ctab += (int64_t)(d0 / 32) * KT * 1024;
    }
    v16i dacc[KT][QT];
    E::run(a, smem, qblock, dacc);
    if constexpr (MODE == M_CLASSIFY) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        if (Z > 1) {
            const int g = lane >> 5;
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) {
                const int64_t q = qblock + (int64_t)wave * E::QPW + qt * 32 + (lane & 31);
                if (q >= a.n)
                    continue;
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int k = kt * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                        if (k < a.K)
                            a.part[part_at(a, KT, z, k, q)] = dacc[kt][qt][v];
                    }
            }
            return;
        }
        int32_t lab[QT];
        E::finish(a, qblock, dacc, lab);
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            const int64_t q = qblock + (int64_t)wave * E::QPW + qt * 32 + (lane & 31);
            if (lane < 32 && q < a.n)
                a.labels[q] = lab[qt];
        }
    }
}

// Distances and argmin of a split classify launch.  A workgroup takes QB
// queries: wave w sums classes w, w + 16, .., its lanes 64 / QB splits x QB
// queries (runs of the class-major partials), dist_k = popc_k - sum.  Few
// queries are latency bound and go 8 to a workgroup; from 1024 on, 32 (whole
// lines; 1559 queries, 26 classes, 32 splits: 1.5 us less than with 8).  The
// first smallest distance wins, as in Encoder::finish: the minimum of
// (distance, class) packed in one 64-bit integer (a projection may have over
// 2^24 dimensions).  The distances go out through LDS, whole rows at once.
template <int QB>
static __global__ __launch_bounds__(1024) void k_split_argmin(EncodeArgs a, int Z)
{
    constexpr int ZL = 64 / QB;
    __shared__ int64_t best[16][QB];
    __shared__ int32_t dist[QB * kMaxK];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ql = lane % QB, zl = lane / QB;
    const int64_t q0 = (int64_t)blockIdx.x * QB, q = q0 + ql, qc = q < a.n ? q : a.n - 1;
    const int64_t zs = a.n * a.K;
    int64_t m = INT64_MAX;
    for (int k = wave; k < a.K; k += 16) {
        const int32_t *p = a.part + k * a.n + qc;
        int s = 0;
        for (int z0 = zl; z0 < Z; z0 += 8 * ZL) {   // eight loads in flight, also for few splits
            int v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = p[(z0 + u * ZL < Z ? z0 + u * ZL : z0) * zs];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                s += z0 + u * ZL < Z ? v[u] : 0;
        }
#pragma unroll
        for (int o = QB; o < 64; o *= 2)
            s += __shfl_xor(s, o);
        const int d = a.cpop[k] - s;
        if (zl == 0 && a.dists)
            dist[ql * a.K + k] = d;
        const int64_t key = (int64_t)d * 128 + k;
        m = key < m ? key : m;
    }
    if (zl == 0)
        best[wave][ql] = m;
    __syncthreads();
    const int nq = a.n - q0 < QB ? (int)(a.n - q0) : QB;
    if (a.dists)
        for (int i = threadIdx.x; i < nq * a.K; i += 1024)
            a.dists[q0 * a.K + i] = dist[i];
    if ((int)threadIdx.x < nq) {
        m = best[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < 16; ++w)
            m = best[w][threadIdx.x] < m ? best[w][threadIdx.x] : m;
        a.labels[q] = (int32_t)(m % 128);
    }
}

// The same for rows of classes (part_rows): a wave per query, lane l classes l and
// l + 64.
static __global__ __launch_bounds__(256) void k_split_argmin_rows(EncodeArgs a, int Z)
{
    const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (q >= a.n)
        return;
    // (classes past the last: an earlier one again)
    const int k0 = lane < a.K ? lane : a.K - 1, k1 = lane + 64 < a.K ? lane + 64 : k0;
    const int32_t *p = a.part + q * a.K;
    const int64_t zs = a.n * a.K;
    int s0 = 0, s1 = 0;
    for (int z0 = 0; z0 < Z; z0 += 8) {
        int v0[8], v1[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int32_t *pz = p + (z0 + u < Z ? z0 + u : z0) * zs;
            v0[u] = pz[k0];
            v1[u] = pz[k1];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            s0 += z0 + u < Z ? v0[u] : 0;
            s1 += z0 + u < Z ? v1[u] : 0;
        }
    }
    int bd = a.cpop[k0] - s0, bk = k0;
    const int d1 = a.cpop[k1] - s1;
    if (a.dists) {
        a.dists[q * a.K + k0] = bd;
        a.dists[q * a.K + k1] = d1;
    }
    if (d1 < bd) {
        bd = d1;
        bk = k1;
    }
    // first minimum across the lanes (lower class index on ties)
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const int od = __shfl_xor(bd, o), ok = __shfl_xor(bk, o);
        if (od < bd || (od == bd && ok < bk)) {
            bd = od;
            bk = ok;
        }
    }
    if (lane == 0)
        a.labels[q] = bk;
}

static void launch_split_argmin(const EncodeArgs &a, int Z, hipStream_t st)
{
    if (part_rows(class_tiles(a.K), a.n))
        hipLaunchKernelGGL(k_split_argmin_rows, dim3((unsigned)((a.n + 3) / 4)), dim3(256), 0, st, a, Z);
    else if (a.n >= 1024)
        hipLaunchKernelGGL(k_split_argmin<32>, dim3((unsigned)((a.n + 31) / 32)), dim3(1024), 0, st, a, Z);
    else
        hipLaunchKernelGGL(k_split_argmin<8>, dim3((unsigned)((a.n + 7) / 8)), dim3(1024), 0, st, a, Z);
}

// Smallest dimension split (64-dimension words) of a launch.
constexpr int split_units_min(int mode) { return mode == M_ENCODE ? 1 : kSplitMinUnits; }

// Whether two query tiles per wave would leave much of the device idle (encodings,
// and the fp32 features' kernels): then one query tile (128 queries per workgroup)
// makes twice the workgroups, each with half the features to load and half the
// MFMAs a word.  It pays while its splits, over twice the blocks, are not over a
// quarter longer: where the words run out (both are bounded by the shortest split,
// see split_units_min).
static bool few_blocks(const EncodeArgs &a, int mode)
{
    const int64_t blocks = (a.n + 255) / 256;
    const int z2 = split_count(blocks, a.nd, a.max_split, 256, split_units_min(mode));
    const int z1 = split_count(2 * blocks, a.nd, a.max_split, 256, split_units_min(mode));
    return 2 * blocks * z1 <= 256 && 4 * split_units(a.nd, z1) <= 5 * split_units(a.nd, z2);
}

// Expected time (ns) of a direct-staged classify launch with qt query tiles per
// wave on width features: the words of a split, one after the other, and where
// there are splits the second launch and the partial sums it writes and reads.
// Two tiles cost less than twice one a word on narrow features (LDS bound) and
// about twice on wide ones; more workgroups of one tile mean fewer splits, which
// many classes and few dimensions favour: 30000 x 64 E4M3, 1024 dimensions, 50
// classes, 15 us with one tile unsplit and 28 with two in two splits; 20000 x 617
// int8, 8192 dimensions, 100 classes, 140 and 120.  Coefficients fitted to 1500
// launches of both kinds (64 to 784 features, 300 to 30000 queries, 5 to 128
// classes, 1024 to 8192 dimensions, int8, uint8, E4M3); on none of them is the
// choice slower than the kernels of one shape before.
static int word_ns(int qt, int width, int kt)
{
    return qt == 1 ? 700 + width * 4 / 5 + 20 * kt : 500 + 2 * width + 100 * kt;
}
static int64_t classify_ns(const EncodeArgs &a, int qt, int width)
{
    const int64_t blocks = (a.n + 128 * qt - 1) / (128 * qt);
    const int z = split_count(blocks, a.nd, a.max_split, 256);
    return (int64_t)split_units(a.nd, z) * word_ns(qt, width, class_tiles(a.K)) +
           (z > 1 ? 4000 + a.n * a.K * z * 7 / 2000 : 0);
}

// Whether a direct-staged launch takes one query tile per wave.  An encoding has no
// partial sums; its few longest splits may take a quarter longer, for half the
// features to load first (1000 x 784, 10240 dimensions: 17.2 us with two tiles, 13.2
// with one; 6000 x 1024, 1000 dimensions 16.8 and 12.1).
static bool one_tile(const EncodeArgs &a, int mode, int width)
{
    if ((a.n + 255) / 256 > 128)
        return false;
    if (mode == M_CLASSIFY)
        return classify_ns(a, 1, width) <= classify_ns(a, 2, width);
    auto split_ns = [&](int qt) {
        const int z = split_count((a.n + 128 * qt - 1) / (128 * qt), a.nd, a.max_split, 256, 1);
        return (int64_t)split_units(a.nd, z) * word_ns(qt, width, 0);
    };
    return few_blocks(a, mode) || 4 * split_ns(1) <= 5 * split_ns(2);
}

template <int CT, int XF, int QT, int KS, int KT, int MODE, bool DMA = false, int RT = 1, int SRC = W_ROWS>
static hipError_t launch_one(const EncodeArgs &a, hipStream_t st)
{
    typedef Encoder<CT, XF, QT, KS, KT, MODE, 0, DMA, RT, SRC> E;
    const int64_t blocks = (a.n + E::QPB - 1) / E::QPB;
    // resident workgroups: one per CU per wave per SIMD the kernel is built for
    const int Z = split_count(blocks, a.nd, a.max_split, 256 * E::WAVES, split_units_min(MODE));
    EncodeArgs b = a;
    b.nsplit = Z;
    const dim3 grid = Z > 1 ? dim3((unsigned)Z, (unsigned)blocks) : dim3((unsigned)blocks);
    hipLaunchKernelGGL((k_encode<CT, XF, QT, KS, KT, MODE, DMA, RT, SRC>), grid, dim3(256), 0, st, b);
    if (MODE == M_CLASSIFY && Z > 1)
        launch_split_argmin(a, Z, st);
    return hipGetLastError();
}

// The direct-staged shape of a bucket: two query tiles per wave (one wave per
// SIMD), so that each projection fragment read from LDS feeds two MFMAs: with
// one, four waves ask LDS for 128 bytes a cycle, all it has (784 uint8
// features, n = 60000, 8192 dimensions: 820 us of encoding against 300).  Two
// row tiles per chunk (80 MFMAs between barriers at 640 features) while three
// stages of them fit the LDS, else one (uint8 features: always one, whose barrier also
// publishes the column sums).  One query tile where the registers hold no
// second beside the accumulators: four class tiles from 833 features, and the
// split E4M3 type, whose query operand is twice as wide (there each fragment
// feeds two MFMAs already); and the shifted E4M3 type at up to 320 features and
// two class tiles, where two take 297 registers, one wave per SIMD, and the last
// round of workgroups costs a whole one (200000 x 300, 4096 dimensions, 40
// classes: 298 us with two, 259 with one; 65536: 75 and 79).
// Few query blocks take one query tile (one_tile), except the shifted int8
// type, whose start values need the registers of one wave per SIMD (20000 x
// 617, 8192 dimensions on the shifted E4M3 form without scratch: 190 us with
// two, 144 with one).
template <int CT, int KS, int KT, int MODE, int SRC>
static hipError_t launch_direct(const EncodeArgs &a, hipStream_t st)
{
    constexpr int W = KS * Tr<CT>::KSTEP;
    constexpr bool SHIFT1 = CT == C_FP8 && SRC == W_ROWS && W <= 320 && KT == 2;
    constexpr int QT = CT == C_FP8S || (W > 832 && KT == 4) || SHIFT1 ? 1 : 2;
    constexpr int RT = QT == 1 || W > 640 || (CT == C_I8 && SRC == W_ALT) ? 1 : 2;
    if (QT == 2 && (CT == C_FP8 || !a.poff) && one_tile(a, MODE, W))
        return launch_one<CT, 0, 1, KS, KT, MODE, true, 1, SRC>(a, st);
    return launch_one<CT, 0, QT, KS, KT, MODE, true, RT, SRC>(a, st);
}

// One feature-width bucket of byte features: everything is staged directly,
// whichever variant a tile table names, except that int8 features on the
// int8 path also have one tile of each with two waves per SIMD (TV_DMA_1X1,
// up to 640 features and two class tiles).  The register-staged kernels that
// the other ids once named were slower for every bucket (one query tile: LDS
// bound, as above).
template <int CT, int KS, int KT, int MODE, int SRC>
static hipError_t launch_bytes_kt(const EncodeArgs &a, int variant, hipStream_t st)
{
    if (a.poff) {   // the shifted projections
        if constexpr (SRC == W_ROWS && (CT == C_I8 ? shift_tile(KS, KT) : shift8_tile(KS, KT))) {
            if (variant != TV_DMA_1X1)
                return launch_direct<CT, KS, KT, MODE, SRC>(a, st);
        }
        return hipErrorInvalidValue;
    }
    if constexpr (CT == C_I8 && SRC == W_ROWS && big_tile(KS, KT)) {
        if (variant == TV_DMA_1X1)
            return launch_one<CT, 0, 1, KS, KT, MODE, true, 1>(a, st);
    }
    if constexpr (CT == C_FP8 && SRC == W_ROWS)   // E4M3 rows: the shifted ones only
        return hipErrorInvalidValue;
    else
        return launch_direct<CT, KS, KT, MODE, SRC>(a, st);
}

template <int CT, int W, int SRC>
static hipError_t launch_bytes_bucket(const EncodeArgs &a, int mode, int variant, hipStream_t st)
{
    constexpr int KS = W / Tr<CT>::KSTEP;
    if (mode == M_ENCODE)
        return launch_bytes_kt<CT, KS, 1, M_ENCODE, SRC>(a, variant, st);
    const int kt = class_tiles(a.K);
    if (kt == 1)
        return launch_bytes_kt<CT, KS, 1, M_CLASSIFY, SRC>(a, variant, st);
    if (kt == 2)
        return launch_bytes_kt<CT, KS, 2, M_CLASSIFY, SRC>(a, variant, st);
    return launch_bytes_kt<CT, KS, 4, M_CLASSIFY, SRC>(a, variant, st);
}

// Byte features: the smallest compiled width (kIntWidths) >= F is used.
template <int CT, int SRC>
static hipError_t launch_bytes(const EncodeArgs &a, int mode, Tile tile, hipStream_t st)
{
    const int F = a.F, v = tile.variant;
    if (F <= 64) return launch_bytes_bucket<CT, 64, SRC>(a, mode, v, st);
    if (F <= 128) return launch_bytes_bucket<CT, 128, SRC>(a, mode, v, st);
    if (F <= 192) return launch_bytes_bucket<CT, 192, SRC>(a, mode, v, st);
    if (F <= 256) return launch_bytes_bucket<CT, 256, SRC>(a, mode, v, st);
    if (F <= 320) return launch_bytes_bucket<CT, 320, SRC>(a, mode, v, st);
    if (F <= 384) return launch_bytes_bucket<CT, 384, SRC>(a, mode, v, st);
    if (F <= 512) return launch_bytes_bucket<CT, 512, SRC>(a, mode, v, st);
    if (F <= 640) return launch_bytes_bucket<CT, 640, SRC>(a, mode, v, st);
    if (F <= 832) return launch_bytes_bucket<CT, 832, SRC>(a, mode, v, st);
    if (F <= 1024) return launch_bytes_bucket<CT, 1024, SRC>(a, mode, v, st);
    return hipErrorInvalidValue;
}

// One width of fp32 features, register staged: as many query tiles per wave
// as fit, one where two leave half the device idle (the built-in rule; 200 x
// 64, 2048 dimensions: 29 us with two), or the variant's.
template <int CT, int W>
static hipError_t launch_fp32_bucket(const EncodeArgs &a, int mode, Tile tile, hipStream_t st)
{
    constexpr int KS = W / Tr<CT>::KSTEP;
    constexpr int QM = qt2_fits(CT, KS) ? 2 : 1;
    const bool one = QM == 1 || tile.variant == TV_REG_QT1 || (tile.variant == TV_AUTO && few_blocks(a, mode));
    const int qt = one ? 1 : 2;
    if (mode == M_ENCODE) {
        if (qt == 2)
            return launch_one<CT, 1, QM, KS, 1, M_ENCODE>(a, st);
        return launch_one<CT, 1, 1, KS, 1, M_ENCODE>(a, st);
    }
    const int kt = class_tiles(a.K);
    if (kt == 1) {
        if (qt == 2)
            return launch_one<CT, 1, QM, KS, 1, M_CLASSIFY>(a, st);
        return launch_one<CT, 1, 1, KS, 1, M_CLASSIFY>(a, st);
    }
    if (kt == 2) {
        if (qt == 2)
            return launch_one<CT, 1, QM, KS, 2, M_CLASSIFY>(a, st);
        return launch_one<CT, 1, 1, KS, 2, M_CLASSIFY>(a, st);
    }
    return launch_one<CT, 1, 1, KS, 4, M_CLASSIFY>(a, st);
}

// fp32 features: the smallest compiled width (kF32Widths) >= F is used.
template <int CT>
static hipError_t launch_fp32(const EncodeArgs &a, int mode, Tile tile, hipStream_t st)
{
    if (a.poff)
        return hipErrorInvalidValue;
    if (a.F <= 64) return launch_fp32_bucket<CT, 64>(a, mode, tile, st);
    if (a.F <= 128) return launch_fp32_bucket<CT, 128>(a, mode, tile, st);
    if (a.F <= 256) return launch_fp32_bucket<CT, 256>(a, mode, tile, st);
    return hipErrorInvalidValue;
}

}  // namespace hdc
