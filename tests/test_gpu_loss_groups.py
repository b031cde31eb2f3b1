"""The loss over every mix of formats and both ways its blocks share out the positions (one group of 16 positions
a block, or several), ragged batches included, against the FP64 oracle."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from cases import near_tie_positions
from util import ensure_built
from oracle import bc as OB
from oracle import ntbc as ON
from paper_2407_09543_amd import ntbc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()
    assert torch.cuda.is_available()


# waves idle, equal and unequal shares, seven colour textures whose rows fill the LDS of one group
FORMATS = ["c", "s", "cs", "sss", "scscs", "ccssss", "ccccccc", "ssssssss"]


@pytest.mark.parametrize("formats", FORMATS)
@pytest.mark.parametrize("n", [1, 33])
def test_loss_groups(formats, n):
    rng = np.random.default_rng(len(formats) * 100 + n % 97)
    fmts = [1 if f == "c" else 4 for f in formats]
    side, texels, blocks = 64, [], []
    for f in fmts:
        t = rng.integers(0, 256, (side, side, 3 if f == 1 else 1), dtype=np.uint8)
        t[:, :8] = 0  # blocks whose distances to a black prediction are exactly zero
        texels.append(t if f == 1 else t[..., 0])
        blocks.append(OB.image_to_blocks(t))
    ref = [OB.bc1_encode_ref(b) if f == 1 else OB.bc4_encode_ref(b[..., 0]) for b, f in zip(blocks, fmts)]
    oracle = ON.Targets(fmts, ref, blocks)
    tex = [torch.from_numpy(t).cuda() for t in texels]
    targets = ntbc.Targets(torch.stack([ntbc.encode_ref(t, f) for t, f in zip(tex, fmts)]), tex)
    desc = ntbc.make_desc(2, 8, 4, False, 64, 2, fmts, side // 4, side // 4)
    ids = rng.integers(0, (side // 4) ** 2, n).astype(np.int32)
    y = rng.random((n, oracle.lay.E + 16 * oracle.lay.C), dtype=np.float32)
    y[ids % (side // 4) < 2] *= rng.integers(0, 2)
    losses, dh = ntbc.loss_grad(desc, targets, torch.from_numpy(y).cuda(), torch.from_numpy(ids).cuda())
    l_or, dy_or = ON.loss_and_grad(y.astype(np.float64), oracle, ids)
    losses = losses.cpu().numpy()
    assert losses[4] == 0.0 and np.allclose(losses[:4], l_or, rtol=2e-5, atol=1e-9)
    keep = ~near_tie_positions(SimpleNamespace(tg_oracle=oracle), y.astype(np.float64), ids)
    assert keep.mean() > 0.5 or n == 1  # all-zero BC4 predictions sit on the mode switch and are left out
    if keep.any():
        assert np.abs(dh.cpu().numpy() - dy_or)[keep].max() <= 1e-4 * np.abs(dy_or).max()


@pytest.mark.parametrize("formats", FORMATS)
def test_several_groups_a_block(formats):
    # a batch of which a block takes several groups, and its halves, of which it takes one: the mean's 1/n is the only
    # difference, a factor of exactly 2 (8,205 = 16 * 512 + 13: the last group is ragged both ways)
    half, side = 8205, 64
    rng = np.random.default_rng(len(formats))
    fmts = [1 if f == "c" else 4 for f in formats]
    tex = [torch.from_numpy(rng.integers(0, 256, (side, side, 3) if f == 1 else (side, side), dtype=np.uint8)).cuda()
           for f in fmts]
    targets = ntbc.Targets(torch.stack([ntbc.encode_ref(t, f) for t, f in zip(tex, fmts)]), tex)
    desc = ntbc.make_desc(2, 8, 4, False, 64, 2, fmts, side // 4, side // 4)
    ids = torch.from_numpy(rng.integers(0, (side // 4) ** 2, 2 * half).astype(np.int32)).cuda()
    y = torch.from_numpy(rng.random((2 * half, ntbc.model_sizes(desc)[1]), dtype=np.float32)).cuda()
    losses, dh = ntbc.loss_grad(desc, targets, y, ids)
    parts = [ntbc.loss_grad(desc, targets, y[k:k + half], ids[k:k + half].contiguous()) for k in (0, half)]
    assert torch.equal(2 * dh, torch.cat([d for _, d in parts]))
    # the sums of 16 * 16,410 squares are added in another order: float32 rounding, as between two runs
    assert torch.allclose(2 * losses, parts[0][0] + parts[1][0], rtol=1e-5, atol=0)
