"""The shared sweep's search at its edges: the class-tile counts (32, 64 and 128
classes and one past each), as many ends per chain as are ranked together and
one more (8 / 4 / 2 by class tiles) up to more than one item holds, ends on and
beside word and chunk boundaries, and query counts around a block.  Correct
counts equal the oracle's."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu

CASES = [  # n, K, D, ends per chain, (start, stride) pairs
    (1, 1, 64, 1, [(0, 1)]), (32, 32, 2112, 8, [(0, 1), (65, 3)]), (33, 33, 2112, 4, [(0, 1)]),
    (63, 32, 4160, 9, [(0, 2)]), (65, 64, 2112, 5, [(31, 1), (0, 64)]), (40, 65, 2112, 2, [(0, 1)]),
    (31, 128, 2112, 3, [(1, 7)]), (100, 26, 4160, 17, [(0, 1), (2, 100)]),
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_shared_search_edges(case):
    from paper_2606_26547_amd import hdc
    O.build()
    n, K, D, nends, chains = case
    print("[case] shared search", case, flush=True)
    g = np.random.default_rng(n + K + D)
    F = 24
    X = g.integers(-127, 128, size=(n, F), dtype=np.int8)
    P = (2 * g.integers(0, 2, size=(D, F), dtype=np.int8) - 1).astype(np.int8)
    C = g.integers(-2 ** 63, 2 ** 63, size=(K, (D + 63) // 64), dtype=np.int64)
    y = g.integers(0, K, size=n).astype(np.int32)
    edge = [D, 64, 63, 65, 128, 2047, 2048, 2049, 1984, 2112, 96, 160, 1, 2000, 127, 129, 1000]
    cfgs = []
    for s, k in chains:
        ends = [d for d in edge if s < d <= D][:nends]
        cfgs += [(d, k, s, t) for d in ends for t in ("int8", "fp8", "bf16")]
    res = hdc.eval_configs(hdc.pad_cols(X), F, torch.as_tensor(y).cuda(), hdc.pad_cols(P), D,
                           torch.as_tensor(C).cuda(), cfgs, tile=4)
    assert np.array_equal(res["correct"], O.eval_configs(X, y, P, C.view(np.uint64), cfgs))
    assert (res["n"] == n).all()
