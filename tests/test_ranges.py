"""Index arithmetic of the kernels (csrc/hdc_ranges.h), compiled for the host
and compared with its definition in unbounded integers, at the ends of what the
entry points take."""
import ctypes as C
import os
import random
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_26547_amd", "csrc")
SOURCE = r"""
#include "hdc_ranges.h"
using namespace hdc;
extern "C" uint32_t t_set_mask(int d0, int start, int end, int stride) { return set_mask(d0, start, end, stride); }
extern "C" void t_row_window(int c, int ch, int nd, uint32_t rstep, uint32_t row_bytes, uint32_t *out)
{
    const RowWindow w = row_window(c, ch, nd, rstep, row_bytes);
    out[0] = w.off;
    out[1] = w.bytes;
}
extern "C" int t_set_popc(const uint64_t *row, int start, int end, int stride, int threads)
{
    int s = 0;
    for (int t = 0; t < threads; ++t)
        s += set_popc(row, start, end, stride, t, threads);
    return s;
}
"""
MAX = 2 ** 31 - 1


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("ranges")
    (d / "t.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-fPIC", "-shared", "-D__host__=", "-D__device__=",
                    "-I", CSRC, "-o", str(d / "t.so"), str(d / "t.cpp")], check=True)
    L = C.CDLL(str(d / "t.so"))
    L.t_set_mask.restype = C.c_uint32
    return L


def _mask(d0, start, end, stride):
    return sum(1 << i for i in range(32) if start <= d0 + i < end and (d0 + i - start) % stride == 0)


def test_set_mask(lib):
    r = random.Random(1)
    strides = [1, 2, 3, 5, 31, 32, 33, 63, 64, 65, 1000, 10241, 2147418113, MAX - 10240, 2147483000, MAX - 1, MAX]
    for stride in strides:
        for start, end in [(0, 10240), (70, 10001), (1, 33), (31, 64), (5, 6), (64, 65536)]:
            for d0 in list(range(0, 256, 32)) + [32 * r.randrange(2048) for _ in range(40)]:
                assert lib.t_set_mask(d0, start, end, stride) == _mask(d0, start, end, stride), (d0, start, end, stride)
        # sets that end at the largest int
        for _ in range(200):
            end = MAX - r.randrange(100)
            start = r.choice([0, 1, r.randrange(end), end - 1 - r.randrange(90)])
            d0 = r.choice([start // 32 * 32, end // 32 * 32, (end - 64) // 32 * 32, 32 * r.randrange(2 ** 26)])
            assert lib.t_set_mask(d0, start, end, stride) == _mask(d0, start, end, stride), (d0, start, end, stride)


@pytest.mark.timeout(60)
@pytest.mark.parametrize("end", [1, 64, 10240, MAX - 8192, MAX - 31, MAX])
def test_set_popc_ends(lib, end):
    """Counts over the last dimensions of a row, up to the longest: every
    thread's loop ends, within the row."""
    first = max(0, end - 5000) // 64 * 64
    W = (end + 63) // 64 - first // 64
    row = np.random.default_rng(end).integers(-2 ** 63, 2 ** 63, size=W, dtype=np.int64)
    bits = np.unpackbits(row.view(np.uint8), bitorder="little")
    base = row.ctypes.data - first // 8          # dwords before the start's word are not read
    for start in {first, min(first + 70, end - 1)}:
        for stride in (1, 3, 4999, MAX):
            want = int(bits[start - first:end - first:stride].sum())
            assert lib.t_set_popc(C.c_void_p(base), start, end, stride, 256) == want, (start, stride)


def test_row_window(lib):
    """The buffer of every chunk a direct-staged kernel loads (chunks past the
    last one among them) lies within the projection, so no offset its range
    check lets through reaches past it; the rows that count are all in it, at
    their place."""
    r = random.Random(2)
    out = (C.c_uint32 * 2)()
    for i in range(4000):
        F = r.choice([1, 64, 65, 617, 640, 641, 1000, 1024])
        ldp = (F + 63) // 64 * 64 + 16 * r.choice([0, 0, 4, 1000])
        D = r.choice([r.randrange(1, 200), r.randrange(200, 20000), (2 ** 32 - 1 - ldp) // ldp])
        start = r.choice([0, 0, r.randrange(D)])
        end = D if r.random() < 0.5 else r.randrange(start + 1, D + 1)
        stride = r.choice([1, 1, 2, 3, 17, r.randrange(1, 2 * D), MAX])
        nd = (end - start + stride - 1) // stride
        rb = (F + 31) // 32 * 32
        base, rstep = start * ldp, stride * ldp % 2 ** 32
        for ch in (32, 64):
            chunks = (nd + 63) // 64 * (64 // ch)             # whole 64-dimension words
            for c in {0, 1, nd // ch - 1, nd // ch, chunks - 2, chunks - 1, chunks, chunks + 6}:
                if c < 0:
                    continue
                lib.t_row_window(c, ch, nd, rstep, rb, out)
                off, size = out
                assert size >= rb and base + off + size <= (D - 1) * ldp + rb, (F, ldp, D, start, end, stride, ch, c)
                for d in range(c * ch, min((c + 1) * ch, nd)):
                    at = (d - c * ch) * rstep                 # the lane's offset
                    assert at < 2 ** 32 and at + rb <= size and base + off + at == (start + d * stride) * ldp
