"""Level-ID encoding of few rows, where a workgroup's waves split the features:
feature counts around the waves' blocks of 32 (waves with part of a block and
with none), every window width, level counts small and large, and row counts on
both sides of the rule (128 workgroups of 4, 8 or 16 rows).  Bits equal the
oracle's exactly."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2606_26547_amd import datagen as dg

pytestmark = pytest.mark.gpu

CASES = [
    # n, F, L, D
    (1, 33, 2, 64), (3, 64, 16, 2048), (7, 65, 128, 10240), (10, 617, 128, 10240), (5, 96, 100, 2112), (4, 129, 5, 1985),
    (9, 1024, 400, 1000), (17, 1000, 1024, 129), (2, 1024, 1024, 8192), (33, 160, 600, 500), (102, 300, 7, 10240),
    (104, 300, 7, 10240), (512, 40, 3, 2000), (513, 40, 3, 2000), (1024, 70, 400, 900), (1030, 70, 400, 900),
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_few_rows(case):
    from paper_2606_26547_amd import hdc
    O.build()
    n, F, L, D = case
    print("[case] level-id few", case, flush=True)
    ID, LV = dg.id_hypervectors(F, D, 5), dg.level_hypervectors(L, D, 6)
    lev = np.random.default_rng(n + F + L + D).integers(0, L, size=(n, F)).astype(np.uint16)
    lev[0] = 0
    H = hdc.level_id_encode(torch.as_tensor(lev.view(np.int16)).cuda(), torch.as_tensor(ID.view(np.int64)).cuda(),
                            torch.as_tensor(LV.view(np.int64)).cuda(), D)
    assert np.array_equal(H.cpu().numpy().view(np.uint64), O.level_id_encode(lev, ID, LV, D))
