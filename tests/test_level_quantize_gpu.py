"""The level quantiser at every feature width its workgroups are shaped for,
row counts around a workgroup's, and sizes past one grid's limits: levels equal
the oracle's exactly."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 33, 2049, 70001])
@pytest.mark.parametrize("F", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 130])
def test_widths(n, F):
    from paper_2606_26547_amd import hdc
    O.build()
    g = np.random.default_rng(n + F)
    X = g.standard_normal((n, F)).astype(np.float32)
    X[g.random(X.shape) < 0.01] = np.nan
    lo, hi = np.full(F, -1.5, np.float32), g.uniform(0.5, 2.0, F).astype(np.float32)
    hi[0] = lo[0] if F > 1 else hi[0]           # an empty range
    out = torch.full((n, F + 3), -7, dtype=torch.int16, device="cuda")
    hdc.level_quantize(torch.as_tensor(X).cuda(), torch.as_tensor(lo).cuda(), torch.as_tensor(hi).cuda(), 100,
                       out=out[:, :F])
    got = out.cpu().numpy().view(np.uint16)
    assert np.array_equal(got[:, :F], O.level_quantize(X, lo, hi, 100)) and bool((out[:, F:] == -7).all())


@pytest.mark.parametrize("n, F", [(2, 64 * 65535 + 70), (2 ** 29 + 77, 1)])
def test_past_one_grid(n, F):
    """More 64-feature blocks than a grid's second dimension takes, and more
    rows than its first in workgroups of 32: rows of 0, 1, 2, .. levels."""
    from paper_2606_26547_amd import hdc
    print("[case] quantise", n, F, flush=True)
    L = 1000
    want = (torch.arange(n * F, device="cuda", dtype=torch.int32) % L).to(torch.int16).view(n, F)
    X = want.to(torch.float32).add_(0.5)
    lo, hi = torch.zeros(F, device="cuda"), torch.full((F,), float(L), device="cuda")
    out = torch.full((n, F), -1, dtype=torch.int16, device="cuda")
    assert torch.equal(hdc.level_quantize(X, lo, hi, L, out=out), want)
