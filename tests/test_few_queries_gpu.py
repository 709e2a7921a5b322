"""The prepared searches on both sides of the rules on the number of queries
(16384; the ADC search's 32768 up to 32 classes; the cosine search's 8192 from
65 classes and 65536):
the kernel that splits words over a workgroup's waves and the streaming ones,
at every class-tile count, dimension sets that start and end inside words, and
ragged last blocks.  Labels, minima / maxima and all scores equal the oracle's
exactly."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu

NS = [1, 33, 8192, 8193, 16384, 16385, 16700, 32768, 32769, 65536, 65537]
SETS = [  # nbits, K, (start, end, stride)
    (1088, 3, (0, 1088, 1)), (2048, 40, (65, 2001, 2)), (640, 100, (130, 639, 1)), (64, 32, (0, 64, 1)),
]


def _inputs(n, nbits, K):
    g = np.random.default_rng(n + nbits + K)
    W = (nbits + 63) // 64
    W += W % 2
    Q = g.integers(-2 ** 63, 2 ** 63, size=(n, W), dtype=np.int64)
    C = g.integers(-2 ** 63, 2 ** 63, size=(K, (nbits + 63) // 64), dtype=np.int64)
    C[K // 2] = C[0]
    return g, Q, C, torch.as_tensor(Q).cuda(), torch.as_tensor(C).cuda()


@pytest.mark.parametrize("n", NS)
@pytest.mark.parametrize("case", SETS, ids=str)
def test_searches_match_oracle(case, n):
    from paper_2606_26547_amd import hdc
    O.build()
    nbits, K, (s, e, k) = case
    print("[case] few", case, n, flush=True)
    g, Q, C, Qd, Cd = _inputs(n, nbits, K)
    Qu, Cu = Q.view(np.uint64), C.view(np.uint64)
    lab, mn, dist = hdc.HammingPrepared(Cd, s, e, k)(Qd, True, True)
    dref = O.hamming(Qu, Cu, s, e, k)
    assert np.array_equal(dist.cpu().numpy(), dref) and np.array_equal(lab.cpu().numpy(), dref.argmin(1))
    assert np.array_equal(mn.cpu().numpy(), dref.min(1))
    for adc in ((8, 2, -3, 128), (6, 9, -3, 128)):
        lab, mx, sc = hdc.AdcPrepared(Cd, s, e, k)(Qd, adc, True, True)
        sref = O.adc_scores(Qu, Cu, s, e, k, *adc)
        alab, amx = O.argmax(sref)
        assert np.array_equal(sc.cpu().numpy(), sref) and np.array_equal(lab.cpu().numpy(), alab)
        assert np.array_equal(mx.cpu().numpy(), amx)
    for lim in (255, 20000):
        acc = g.integers(-lim, lim + 1, size=(K, nbits), dtype=np.int32)
        acc[0, s] = lim
        lab, mx, sc = hdc.CosinePrepared(torch.as_tensor(acc).cuda(), s, e, k)(Qd, True, True)
        cref = O.cosine_scores(Qu, acc, s, e, k)
        clab, cmx = O.argmax_f64(cref)
        assert np.array_equal(sc.cpu().numpy().view(np.uint64), cref.view(np.uint64))
        assert np.array_equal(lab.cpu().numpy(), clab) and np.array_equal(mx.cpu().numpy(), cmx)
