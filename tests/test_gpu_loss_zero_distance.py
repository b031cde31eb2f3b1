"""The loss where predicted palette entries coincide with the texel (distance 0, subgradient 0) at temperatures
whose reciprocal is far beyond 2^63: the gradient is finite and the FP64 oracle's."""
import numpy as np
import pytest
import torch

from util import ensure_built
from oracle import bc as OB
from oracle import ntbc as ON
from paper_2407_09543_amd import ntbc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("formats", ["c", "cs"])
@pytest.mark.parametrize("temperature", [1e-2, 1e-20, 1e-22, 1e-30])
def test_zero_distance(formats, temperature):
    # texels of black and white, both predicted endpoints black: the four predicted entries of a BC1 block are one
    # colour, at distance 0 from its black texels (in both branches: the predicted colours are the texels), and the
    # softmax ties, so the straight-through factor is of the size of 1/T
    ensure_built()
    rng = np.random.default_rng(7)
    fmts = [1 if f == "c" else 4 for f in formats]
    side = 32
    bw = rng.integers(0, 2, (side, side), dtype=np.uint8) * 255
    texels = [np.repeat(bw[..., None], 3, axis=2) if f == 1 else bw for f in fmts]
    blocks = [OB.image_to_blocks(t) for t in texels]
    ref = [OB.bc1_encode_ref(b) if f == 1 else OB.bc4_encode_ref(b[..., 0]) for b, f in zip(blocks, fmts)]
    oracle = ON.Targets(fmts, ref, blocks)
    tex = [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in texels]
    targets = ntbc.Targets(torch.stack([ntbc.encode_ref(t, f) for t, f in zip(tex, fmts)]), tex)
    desc = ntbc.make_desc(2, 8, 4, False, 64, 2, fmts, side // 4, side // 4)
    ids = np.arange((side // 4) ** 2, dtype=np.int32)
    lay = oracle.lay
    y = np.zeros((len(ids), lay.E + 16 * lay.C), np.float32)
    y[:, lay.E:] = oracle.c[ids].reshape(len(ids), -1)
    losses, dh = ntbc.loss_grad(desc, targets, torch.from_numpy(y).cuda(), torch.from_numpy(ids).cuda(), temperature)
    l_or, dy = ON.loss_and_grad(y.astype(np.float64), oracle, ids, temperature)
    losses, dh = losses.cpu().numpy(), dh.cpu().numpy()
    assert losses[4] == 0.0 and np.isfinite(dh).all()
    assert np.allclose(losses[:4], l_or, rtol=2e-5, atol=1e-9)
    # beside the bound of the loss's other comparisons, what 1/T makes of float32's x - c: off by 2^-22 for values up
    # to 1, so g by twice that over N_cd, and a term's 1/(4 T) (G_n - mean G) by six times g's; 16 texels, 4 entries
    n_cd = len(ids) * 16 * lay.C
    slack = 16 * 4 * 6 * 2 * 2.0 ** -22 / (4 * temperature * n_cd)
    assert np.abs(dh - dy).max() <= 1e-4 * np.abs(dy).max() + slack
