"""fp32 features round as they are summed, so a sign can depend on the order
of the sum; the library's order is one per compute type and feature width.
Features that cancel (a sum's large terms meet each other or the small ones
first, depending on the order) give the same bits in every kernel shape: an
encoding does not depend on the batch it is in, and hdc_classify equals
hdc_encode followed by the Hamming search for every batch size, tile variant,
class-tile count, with dimension splits and without."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

D = 1100            # four dimension splits, the last word ragged


def _inputs(F, K, compute, n=64):
    """Rows of paired large features of both signs and small ones, at random
    places; the first dimensions' weights are all +1, where every pair
    cancels, the others random."""
    g = np.random.default_rng(F + K)
    big, small = (448.0, 2.0 ** -9) if compute == "fp8" else (2.0 ** 24, 0.5)
    X = np.zeros((n, F), dtype=np.float32)
    for i in range(n):
        at = g.permutation(F)
        m = 2 * (F // 6)
        X[i, at[:m]] = np.repeat([big, -big], m // 2)
        X[i, at[m:]] = small * g.choice([-2.0, -1.0, 1.0, 2.0], F - m)
    # two chains on alternate K steps give +0.5, one chain -0.5
    X[0] = 0
    X[0, [0, 2, 4, 6]] = [big, 2 * small, -big, -small]
    P = g.choice(np.array([-1, 1], dtype=np.int8), (D, F))
    P[:64] = 1
    C = g.integers(-2 ** 63, 2 ** 63, size=(K, (D + 63) // 64), dtype=np.int64)
    C[:, -1] &= (1 << (D % 64)) - 1
    return X, P, C


@pytest.mark.parametrize("K", [10, 40, 100])
@pytest.mark.parametrize("F", [64, 128, 130, 256])
@pytest.mark.parametrize("compute", ["fp32", "bf16", "fp8"])
def test_every_shape_sums_in_one_order(compute, F, K):
    from paper_2606_26547_amd import hdc
    print("[case] fp32 order", compute, F, K, flush=True)
    X, P, C = _inputs(F, K, compute)
    Xd, Pd, Cd = hdc.pad_cols(X), hdc.pad_cols(P), torch.as_tensor(C).cuda()
    H = hdc.encode(Xd, F, Pd, D, compute)
    # the same rows in a batch that fills the device
    big = Xd.repeat(33024 // X.shape[0], 1)
    Hb = hdc.encode(big, F, Pd, D, compute).view(-1, *H.shape)
    assert torch.equal(Hb, H.expand_as(Hb))
    assert torch.equal(hdc.encode(Xd[:1], F, Pd, D, compute), H[:1])
    for v in hdc.tile_variants("encode", "fp32", compute, F, 1):
        assert torch.equal(hdc.encode(Xd, F, Pd, D, compute, tile=v), H), v
    lab, _, dist = hdc.HammingPrepared(Cd, 0, D, 1)(H, with_dists=True)
    for v in [0] + hdc.tile_variants("classify", "fp32", compute, F, K):
        for split in (True, False):
            for x, l, d in ((Xd, lab, dist), (Xd[:1], lab[:1], dist[:1])):
                cl, cd = hdc.classify(x, F, Pd, D, Cd, compute, with_dists=True, split=split, tile=v)
                assert torch.equal(cd, d) and torch.equal(cl, l), (v, split, x.shape[0])
    cl, cd = hdc.classify(big, F, Pd, D, Cd, compute, with_dists=True)
    assert torch.equal(cd.view(-1, *dist.shape), dist.expand(big.shape[0] // X.shape[0], -1, -1))
    assert torch.equal(cl.view(-1, lab.shape[0]), lab.expand(big.shape[0] // X.shape[0], -1))
