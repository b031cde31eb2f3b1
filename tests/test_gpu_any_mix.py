"""The any-mix register epilogue and the resident-weight kernels (bfloat16 and half, one or two middle layers, at
most ten colour channels): every width, input width, texture mix and order of textures; ragged ranges, ranges
of one position and of more tiles than the chip has waves for in one round.  Heads against the oracle's
emulation of the format (the bounds of test_gpu_infer.py), packing bit-exact on the kernel's own heads, and the
same blocks from the batched decode."""
import numpy as np
import pytest
import torch

from cases import model_inputs, oracle_levels
from util import ensure_built, u64
from oracle import ntbc as ON
from paper_2407_09543_amd import ntbc, synth

pytestmark = pytest.mark.gpu

CASES = [  # hidden, hidden layers, levels, features, formats, blocks w, h, first, count, uint8 grid
    (64, 2, 2, 4, (4,), 7, 5, 0, 35, False), (64, 3, 5, 4, (1, 4), 64, 64, 1, 4000, True),
    (64, 2, 5, 8, (4, 1, 4, 1), 33, 40, 100, 1, True), (64, 3, 8, 8, (1, 1, 1, 4), 128, 300, 5, 38001, True),
    (32, 2, 3, 4, (4, 4, 4), 50, 20, 999, 1, False), (128, 2, 2, 8, (1,), 30, 30, 3, 800, True),
    (128, 3, 3, 8, (4, 4, 1, 4, 4, 4, 4), 40, 44, 0, 1760, True), (128, 2, 6, 8, (1, 4, 1), 64, 64, 31, 33, False),
    (128, 3, 8, 8, (4,) * 8, 256, 256, 7, 65000, True), (96, 3, 7, 8, (1, 4, 4), 37, 29, 0, 37 * 29, True),
    (256, 2, 2, 8, (4, 1), 20, 20, 0, 400, True), (256, 3, 4, 8, (1, 1), 33, 9, 2, 290, False),
    (256, 2, 5, 8, (4, 1, 1), 41, 41, 0, 1681, True), (256, 3, 8, 8, (1, 4, 1, 4, 4), 64, 64, 0, 4096, True),
    (192, 3, 8, 8, (1, 1, 1, 4), 24, 24, 1, 500, True)]


@pytest.mark.parametrize("precision", ["bf16", "fp16"])
@pytest.mark.parametrize("hidden,n_hidden,levels,feats,formats,bw,bh,first,count,u8", CASES)
def test_any_mix(precision, hidden, n_hidden, levels, feats, formats, bw, bh, first, count, u8):
    ensure_built()
    cfg = synth.ModelConfig(levels, 8, feats, u8, hidden, n_hidden, formats, bw, bh)
    flat, layers, g = model_inputs(cfg, hidden + count, u8=u8)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    grid = [t(g["codes"]), t(g["scale"]), t(g["zero"])] if u8 else [t(g["grid"])]
    m = ntbc.Model(ntbc.desc_from_config(cfg), t(flat), *grid)
    prec = ntbc.PRECISIONS[precision]
    words, heads = m.infer(prec, first, count, heads=True)
    assert torch.equal(m.infer(prec, first, count), words)
    batch = ntbc.Batch([(m, m.desc, first, count)], prec, tiles={})
    assert torch.equal(batch.run()[0], words)
    pick = np.unique(np.concatenate([np.arange(min(count, 40)), np.random.default_rng(1).integers(0, count, 1500), [count - 1]]))
    hs = heads[torch.from_numpy(pick).cuda()].cpu().numpy()
    assert np.array_equal(u64(words)[:, pick], ON.pack(hs, formats, "f32"))
    dy = np.abs(hs - ON.heads(cfg, oracle_levels(cfg, g), layers, first + pick, precision))
    top, p99 = (1e-2, 2e-3) if precision == "bf16" else (2e-3, 4e-4)
    assert dy.max() <= top and np.percentile(dy, 99) <= p99 and np.median(dy) <= 1e-6
