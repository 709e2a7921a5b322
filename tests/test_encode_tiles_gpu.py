"""Encodings on both sides of the choice of query tiles, which depends on the
queries, the features and the dimensions: codes equal the oracle's exactly."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_26547_amd import datagen as dg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, D", [(1, 2000), (300, 2000), (1000, 4096), (6000, 200), (12000, 130), (33000, 70)])
@pytest.mark.parametrize("F, xt, compute", [(64, "int8", "int8"), (64, "uint8", "int8"), (617, "int8", "fp8"),
                                            (784, "int8", "int8"), (1000, "uint8", "int8"), (1000, "int8", "fp8")])
def test_encode_tiles(n, D, F, xt, compute):
    from paper_2606_26547_amd import hdc
    O.build()
    print("[case] encode tiles", n, D, F, xt, compute, flush=True)
    X, P = dg.random_case(n, F, D, xt, seed=n + F)
    H = hdc.encode(hdc.pad_cols(X), F, hdc.pad_cols(P), D, compute)
    assert np.array_equal(H.cpu().numpy().view(np.uint64), O.encode(X, P, compute))
