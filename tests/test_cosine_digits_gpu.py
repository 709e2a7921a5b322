"""The cosine search's two operands at the bound between them: accumulators up
to 255 over S (two FP6 digits, one fp32 sum), from 256 on (two signed bytes),
and the largest sums the FP6 operand can reach (65536 dimensions of +-255 with
every query bit set, where the fp32 sum must still be exact).  Scores equal the
oracle's bit for bit."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu

CASES = [
    # n, nbits, K, perf, accumulator bound
    (1, 64, 1, (0, 64, 1), 255), (255, 2048, 10, (0, 2048, 1), 255), (257, 2048, 32, (65, 2047, 2), 256),
    (256, 10240, 33, (0, 10240, 1), 240), (31, 4032, 64, (130, 4001, 3), 255), (300, 1088, 65, (0, 1088, 1), 255),
    (513, 16384, 100, (0, 16384, 1), 240), (40, 640, 128, (1, 640, 1), 255), (40, 640, 128, (1, 640, 1), 256),
]


def _check(Q, acc, perf):
    from paper_2606_26547_amd import hdc
    s, e, k = perf
    ref = O.cosine_scores(Q, acc, s, e, k)
    lref, mref = O.argmax_f64(ref)
    lab, mx, sc = hdc.CosinePrepared(torch.as_tensor(acc).cuda(), s, e, k)(
        torch.as_tensor(Q.view(np.int64)).cuda(), True, True)
    assert np.array_equal(sc.cpu().numpy().view(np.uint64), ref.view(np.uint64))
    assert np.array_equal(lab.cpu().numpy(), lref)
    assert np.array_equal(mx.cpu().numpy().view(np.uint64), mref.view(np.uint64))


@pytest.mark.parametrize("case", CASES, ids=str)
def test_cosine_digits(case):
    O.build()
    n, nbits, K, perf, lim = case
    print("[case] cosine", case, flush=True)
    g = np.random.default_rng(n + nbits + K)
    Q = g.integers(-2 ** 63, 2 ** 63, size=(n, (nbits + 63) // 64), dtype=np.int64).view(np.uint64)
    acc = g.integers(-lim, lim + 1, size=(K, nbits), dtype=np.int32)
    acc[0, perf[0]] = -lim                                # the bound itself
    if perf[2] > 1:
        acc[K - 1, perf[0] + 1] = 100000                  # outside S
    if K >= 5:
        acc[4] = 0
        acc[3] = acc[1]
    _check(Q, acc, perf)


def test_cosine_largest_sums():
    O.build()
    g = np.random.default_rng(5)
    D = 65536
    acc = np.full((6, D), 255, dtype=np.int32)
    acc[1] = -255
    acc[2, ::2] = 1                                       # small terms beside a large running sum
    acc[3, 1:] = 1
    acc[4] = g.integers(-255, 256, size=D)
    acc[5, 40000:] = -1
    Q = np.full((33, D // 64), 0xFFFFFFFFFFFFFFFF, dtype=np.uint64)
    Q[1:] |= 0
    Q[2] = g.integers(-2 ** 63, 2 ** 63, size=D // 64, dtype=np.int64).view(np.uint64)
    Q[3, 700:] = 1
    _check(Q, acc, (0, D, 1))
