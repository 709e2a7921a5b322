// Encoder instantiations for the fp32 compute type (fp32 features), and its
// classifier for few queries.
#include "hdc_encode_impl.h"

namespace hdc {

// Split classification of few queries in fp32: a workgroup takes 32 queries
// and one dimension split, its four waves the split's row tiles in turn.  The
// scratch bounds the splits (one per kSplitMinUnits words), and with 128
// queries per workgroup 200 queries at 2048 dimensions ran on 16 workgroups,
// each wave through 8 row tiles of 32 MFMAs of 64 cycles (17.5 us); here 56
// workgroups with two row tiles per wave.  Projection rows and class operand
// come straight from global memory (each is read once per workgroup), the
// int8 +-1 weights become fp32 as they are multiplied, and the K steps go to the
// encoder's chains in the encoder's order (fp32_chains), so the signs are the
// same bit for bit.  The four waves' class sums meet in LDS.
template <int KS, int KT>
__global__ __launch_bounds__(256) void k_classify_f32_few(EncodeArgs a)
{
    __shared__ int32_t sums[kWaves][KT * 32][33];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 5, c = lane & 31;
    const int Z = (int)gridDim.x, z = (int)blockIdx.x;
    const int64_t qb = (int64_t)blockIdx.y * 32, q = qb + c < a.n ? qb + c : a.n - 1;
    const int per = split_units(a.nd, Z), t0 = 2 * z * per;
    const int nt = (a.nd + kDimChunk - 1) / kDimChunk, t1 = t0 + 2 * per < nt ? t0 + 2 * per : nt;

    float x[KS];
    const float *xrow = (const float *)a.X + q * a.ldx;
#pragma unroll
    for (int s = 0; s < KS; ++s)
        x[s] = 2 * s + g < a.F ? xrow[2 * s + g] : 0.0f;
    v16i dacc[KT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
        dacc[kt] = v16i{};
    const int nw = (a.F + 15) / 16;                        // 16-byte pieces of a row holding features
    for (int t = t0 + wave; t < t1; t += kWaves) {
        const int dl = t * kDimChunk + c < a.nd ? t * kDimChunk + c : a.nd - 1;
        const int8_t *row = a.P + (int64_t)(a.s0 + (int64_t)dl * a.stride) * a.ldp;
        v4i cf[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
            cf[kt] = *(const v4i *)(a.ctab + ((int64_t)t * KT + kt) * 1024 + lane * 16);
        constexpr int KC = fp32_chains(C_F32, KS);
        v16f y{}, y1{};                                    // chains of the even and odd K steps (KC == 2)
        constexpr int NB = KS / 8 < 8 ? KS / 8 : 8;        // pieces in flight
#pragma unroll
        for (int j0 = 0; j0 < KS / 8; j0 += NB) {
            uint4 w[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j)
                w[j] = *(const uint4 *)(row + 16 * (j0 + j < nw ? j0 + j : 0));
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // weight 2s + g is byte 2 (s % 2) + g of its dword
                    const uint32_t d = (e == 0 ? w[j].x : e == 1 ? w[j].y : e == 2 ? w[j].z : w[j].w) << (8 * (1 - g));
                    const int s = 8 * (j0 + j) + 2 * e;
                    mma(y, __uint_as_float(((d << 16) & 0x80000000u) | 0x3F800000u), x[s]);
                    mma(KC == 2 ? y1 : y, __uint_as_float((d & 0x80000000u) | 0x3F800000u), x[s + 1]);
                }
        }
        if constexpr (KC == 2)
            y += y1;
        v4i mb;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // bytes: 0xFF where the projection is negative, else 0
            const uint32_t lo = __builtin_amdgcn_perm(sign_word(y[4 * e + 1]), sign_word(y[4 * e]), 0x0C0C0B09u);
            const uint32_t hi = __builtin_amdgcn_perm(sign_word(y[4 * e + 3]), sign_word(y[4 * e + 2]), 0x0B090C0Cu);
            mb[e] = (int)(lo | hi);
        }
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
            mma(dacc[kt], cf[kt], mb);
    }
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            sums[wave][kt * 32 + 8 * (v >> 2) + 4 * g + (v & 3)][c] = dacc[kt][v];
    __syncthreads();
    auto sum = [&](int k, int col) {
        if (qb + col < a.n)
            a.part[part_at(a, KT, z, k, qb + col)] = sums[0][k][col] + sums[1][k][col] + sums[2][k][col] + sums[3][k][col];
    };
    if (part_rows(KT, a.n)) {   // a query's classes in turn
        for (int i = threadIdx.x; i < KT * 32 * 32; i += 256)
            if (i % (KT * 32) < a.K)
                sum(i % (KT * 32), i / (KT * 32));
    } else {
        for (int k = threadIdx.x >> 5; k < a.K; k += 8)
            sum(k, threadIdx.x & 31);
    }
}

// Class tiles and width of the kernel for few queries.
template <int KS>
static hipError_t launch_f32_few(const EncodeArgs &a, int Z, hipStream_t st)
{
    const dim3 grid((unsigned)Z, (unsigned)((a.n + 31) / 32));
    const int kt = class_tiles(a.K);
    if (kt == 1)
        hipLaunchKernelGGL((k_classify_f32_few<KS, 1>), grid, dim3(256), 0, st, a);
    else if (kt == 2)
        hipLaunchKernelGGL((k_classify_f32_few<KS, 2>), grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_classify_f32_few<KS, 4>), grid, dim3(256), 0, st, a);
    launch_split_argmin(a, Z, st);
    return hipGetLastError();
}

hipError_t launch_encode_f32(const EncodeArgs &a, int mode, Tile tile, hipStream_t st)
{
    if (mode == M_CLASSIFY && tile.variant == TV_AUTO && a.F <= 256 && few_blocks(a, mode)) {
        const int Z = split_count((a.n + 255) / 256, a.nd, a.max_split, 256);
        // four class tiles: two workgroups per CU, and each writes 16 KiB of sums;
        // past two rounds the encoder's 128 queries a workgroup are faster (1000 x
        // 64, 10240 dimensions, 100 classes: 45 us, 42)
        if (Z > 1 && (class_tiles(a.K) < 4 || (a.n + 31) / 32 * Z <= 1024)) {
            if (a.F <= 64)
                return launch_f32_few<32>(a, Z, st);
            return a.F <= 128 ? launch_f32_few<64>(a, Z, st) : launch_f32_few<128>(a, Z, st);
        }
    }
    return launch_fp32<C_F32>(a, mode, tile, st);
}
}  // namespace hdc
