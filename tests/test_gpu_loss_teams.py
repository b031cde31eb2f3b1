"""The loss at batches of every way of sharing them out (sets of waves, teams of one, two or four groups, a team with no
positions, a second turn of the blocks): quarters of a batch, launched alone, differ from it by the mean's 1/n, a
factor of exactly 4 (the smaller launches are compared with the oracle in test_gpu_loss_groups.py)."""
import numpy as np
import pytest
import torch

from test_gpu_loss_groups import FORMATS
from util import ensure_built
from paper_2407_09543_amd import ntbc

pytestmark = pytest.mark.gpu


# 40,000: 2,500 groups of 16; 65,640 = 65,536 + 104: past one turn of 256 blocks of 256 positions, the last group ragged;
# 81,940: ragged in the quarters too; 104,000: teams for three textures
@pytest.mark.parametrize("formats", FORMATS + ["ccsss"])
@pytest.mark.parametrize("quarter", [10000, 16410, 20485, 26000])
def test_quarters(formats, quarter):
    ensure_built()
    side, n = 64, 4 * quarter
    rng = np.random.default_rng(len(formats) + quarter)
    fmts = [1 if f == "c" else 4 for f in formats]
    tex = [torch.from_numpy(rng.integers(0, 256, (side, side, 3) if f == 1 else (side, side), dtype=np.uint8)).cuda()
           for f in fmts]
    targets = ntbc.Targets(torch.stack([ntbc.encode_ref(t, f) for t, f in zip(tex, fmts)]), tex)
    desc = ntbc.make_desc(2, 8, 4, False, 64, 2, fmts, side // 4, side // 4)
    ids = torch.from_numpy(rng.integers(0, (side // 4) ** 2, n).astype(np.int32)).cuda()
    y = torch.from_numpy(rng.random((n, ntbc.model_sizes(desc)[1]), dtype=np.float32)).cuda()
    losses, dh = ntbc.loss_grad(desc, targets, y, ids)
    parts = [ntbc.loss_grad(desc, targets, y[k:k + quarter], ids[k:k + quarter].contiguous()) for k in range(0, n, quarter)]
    assert torch.equal(4 * dh, torch.cat([d for _, d in parts]))
    # sums of up to 16 * 81,940 * 24 squares in another order: float32 rounding of a few hundred additions each
    assert torch.allclose(4 * losses, sum(l for l, _ in parts), rtol=1e-5, atol=0)
