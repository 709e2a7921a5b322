"""Level-ID encoding in every shape of its kernel (windows of 32, 16 and 8
words, one and two rows per lane): row counts on both sides of the two-row
rule, odd word counts (identity rows off 16-byte alignment), partial last
windows, feature counts around the 32-feature blocks, and levels past the
last one (clamped).  Bits equal the oracle's exactly."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2606_26547_amd import datagen as dg

pytestmark = pytest.mark.gpu

CASES = [
    # n, F, L, D
    (65600, 9, 5, 2000),        # 32-word windows, two rows per lane
    (131100, 3, 400, 1000),     # 16-word windows, two rows
    (262200, 2, 600, 500),      # 8-word windows, two rows
    (45, 31, 319, 2112), (45, 32, 320, 2112), (45, 65, 128, 64 * 33 - 5), (33, 64, 567, 1985), (33, 63, 568, 1985),
    (70, 97, 1024, 129), (3, 1024, 7, 4160),
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_level_id_shapes(case):
    from paper_2606_26547_amd import hdc
    O.build()
    n, F, L, D = case
    print("[case] level-id", case, flush=True)
    g = np.random.default_rng(n + F + L + D)
    ID, LV = dg.id_hypervectors(F, D, 5), dg.level_hypervectors(L, D, 6)
    lev = g.integers(0, L, size=(n, F)).astype(np.uint16)
    given = lev.copy()
    past = (lev == L - 1) & (g.random((n, F)) < 0.5)
    given[past] = g.integers(L, 65536, size=int(past.sum())).astype(np.uint16)
    H = hdc.level_id_encode(torch.as_tensor(given.view(np.int16)).cuda(), torch.as_tensor(ID.view(np.int64)).cuda(),
                            torch.as_tensor(LV.view(np.int64)).cuda(), D)
    assert np.array_equal(H.cpu().numpy().view(np.uint64), O.level_id_encode(lev, ID, LV, D))
