// Index arithmetic of the kernels that has to hold over every size the entry
// points take, apart from them so that the host can run it: plain functions of
// integers.
#pragma once

#include <stdint.h>

namespace hdc {

// Dimensions of the set {start + j * stride < end} among d0 .. d0 + 31, as a
// bit mask.  d0, start >= 0 and stride >= 1, any of them and end up to the
// largest int: offsets from d0, unsigned, never pass 2^31 + 31.
__host__ __device__ inline uint32_t set_mask(int d0, int start, int end, int stride)
{
    if (d0 >= end || start - d0 >= 32)
        return 0u;
    const uint32_t lim = end - d0 < 32 ? (uint32_t)(end - d0) : 32u;
    uint32_t o = 0;   // the set's first dimension at or past d0
    if (d0 < start) {
        o = (uint32_t)(start - d0);
    } else if (stride > 1) {
        const uint32_t r = (uint32_t)(d0 - start) % (uint32_t)stride;
        o = r ? (uint32_t)stride - r : 0u;
    }
    if (stride == 1)
        return (lim < 32 ? (1u << lim) - 1u : ~0u) & ~0u << o;
    uint32_t m = 0;
    for (; o < lim; o += (uint32_t)stride)
        m |= 1u << o;
    return m;
}

// Set bits of the dimensions of {start + j * stride < end} in a packed row,
// over its dwords first + k * step, first counted from the start's word: the
// share of one of `step` threads.  (The dwords are counted, not their
// dimensions: 32 * dword passes the largest int within a step of an end there.)
__host__ __device__ inline int set_popc(const uint64_t *row, int start, int end, int stride, int first, int step)
{
    const int n = (end - 1) / 32 + 1;
    int s = 0;
    for (int h = 2 * (start >> 6) + first; h < n; h += step)
        s += __builtin_popcount((uint32_t)(row[h >> 1] >> (32 * (h & 1))) & set_mask(32 * h, start, end, stride));
    return s;
}

// The projection rows a direct-staged kernel reads for a chunk of ch dimensions:
// offset of the chunk's first row from the row of the set's first dimension,
// and the bytes from there to the end of the last dimension's row.  rstep is
// the offset from one dimension's row to the next, row_bytes what is read of a
// row.  A chunk past the last dimension (the partner of an odd last one, or one
// loaded ahead) gives the last chunk that holds one.  A buffer of `bytes` at
// `off` thus lies within the projection whatever the offsets into it, which are
// checked against its size (a chunk's rows past the last dimension are past its
// end, or wrap to others of its rows).
struct RowWindow {
    uint32_t off, bytes;
};
__host__ __device__ inline RowWindow row_window(int c, int ch, int nd, uint32_t rstep, uint32_t row_bytes)
{
    const int last = (nd - 1) / ch, cc = c < last ? c : last;
    return RowWindow{(uint32_t)(cc * ch) * rstep, (uint32_t)(nd - 1 - cc * ch) * rstep + row_bytes};
}

}  // namespace hdc
