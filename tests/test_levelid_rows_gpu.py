"""Level-ID encoding of more rows than one grid holds (2^24 workgroups of 128;
a launch takes 2^22): rows of one feature, whose encoding is the level's word bound to the
identity's."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_rows_past_one_launch():
    from paper_2606_26547_amd import hdc
    n, L, D = 2 ** 31 + 300, 5, 50
    print("[case] level-id rows", n, flush=True)
    g = torch.Generator(device="cuda").manual_seed(1)
    ID = torch.randint(0, 2 ** 50, (1, 1), dtype=torch.int64, device="cuda", generator=g)
    LV = torch.randint(0, 2 ** 50, (L, 1), dtype=torch.int64, device="cuda", generator=g)
    lev = torch.zeros((n, 8), dtype=torch.int16, device="cuda")
    for i in range(0, n, 2 ** 27):
        lev[i:i + 2 ** 27, 0] = torch.arange(i, min(i + 2 ** 27, n), device="cuda") % L
    H = torch.full((n, 1), -1, dtype=torch.int64, device="cuda")
    hdc.level_id_encode(lev[:, :1], ID, LV, D, out=H)
    bound = (LV ^ ID)[:, 0]
    for i in range(0, n, 2 ** 27):
        assert torch.equal(H[i:i + 2 ** 27, 0], bound[lev[i:i + 2 ** 27, 0].long()])
