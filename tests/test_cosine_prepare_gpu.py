"""The cosine search's FP6 operand from rows of sums at every alignment (odd row
pitches, bases off 16 bytes), sets that start, end and stride inside a dword,
and rows that end where the allocation's data do.  Scores and labels equal the
oracle's exactly."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(0, 1001, 1), (70, 990, 1), (3, 1001, 3), (31, 33, 1), (0, 1001, 64)], ids=str)
@pytest.mark.parametrize("K", [1, 33, 100])
def test_digit_operand(K, dims):
    from paper_2606_26547_amd import hdc
    O.build()
    print("[case] cosine prepare", K, dims, flush=True)
    n, nbits = 40, 1001
    g = np.random.default_rng(K)
    Q = g.integers(-2 ** 63, 2 ** 63, size=(n, 16), dtype=np.int64)
    buf = g.integers(-255, 256, size=K * nbits + 3, dtype=np.int32)
    bufd = torch.as_tensor(buf).cuda()
    for base in (0, 1, 3):
        acc = buf[base:base + K * nbits].reshape(K, nbits)
        accd = bufd[base:base + K * nbits].view(K, nbits)
        lab, mx, sc = hdc.CosinePrepared(accd, *dims)(torch.as_tensor(Q).cuda(), True, True)
        cref = O.cosine_scores(Q.view(np.uint64), np.ascontiguousarray(acc), *dims)
        clab, cmx = O.argmax_f64(cref)
        assert np.array_equal(sc.cpu().numpy().view(np.uint64), cref.view(np.uint64))
        assert np.array_equal(lab.cpu().numpy(), clab) and np.array_equal(mx.cpu().numpy(), cmx)
