"""The E4M3 kernels on both sides of the rule on query tiles: few query blocks
(one tile per wave), many (two), and the shifted projection at 320 features and
two class tiles (one always), one feature width past it.  Labels and distances
equal the oracle's exactly, shifted and not."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2606_26547_amd import datagen as dg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [70, 9000, 33000])
@pytest.mark.parametrize("F, K", [(257, 5), (320, 33), (300, 64), (321, 40), (617, 26)])
def test_fp8_query_tiles(n, F, K):
    from paper_2606_26547_amd import hdc
    O.build()
    print("[case] fp8", n, F, K, flush=True)
    D = 200
    X, P = dg.random_case(n, F, D, "int8", seed=n + F)
    C = np.random.default_rng(K).integers(0, 2 ** 63, size=(K, 4), dtype=np.int64)
    C[:, -1] &= (1 << (D % 64)) - 1
    lref, dref = O.classify(X, P, C.view(np.uint64), "fp8", with_dists=True)
    Xd, Pd, Cd = hdc.pad_cols(X), hdc.pad_cols(P), torch.as_tensor(C).cuda()
    for compute, Pc in (("fp8", Pd), ("fp8shift", hdc.shift_projection(Pd, F, compute="fp8shift"))):
        for split in (True, False):
            lab, dists = hdc.classify(Xd, F, Pc, D, Cd, compute, with_dists=True, split=split)
            assert np.array_equal(dists.cpu().numpy(), dref), (compute, split)
            assert np.array_equal(lab.cpu().numpy(), lref), (compute, split)
        H = hdc.encode(Xd, F, Pc, D, compute)
        assert np.array_equal(H.cpu().numpy().view(np.uint64), O.encode(X, P, "fp8")), compute
