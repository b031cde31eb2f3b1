"""Inference shapes outside the streaming kernels, in 16 bits (more than 64 inputs or heads wider than 192): the first
layer's operands pass through the place in LDS that later holds a wave's heads, which is larger than the heads
for few channels and smaller for many.  The bounds of test_gpu_infer.py; packing exact on the kernel's heads."""
import numpy as np
import pytest
import torch

from cases import model_inputs, oracle_levels
from util import ensure_built, u64
from oracle import ntbc as ON
from paper_2407_09543_amd import ntbc, synth

pytestmark = pytest.mark.gpu

# hidden, hidden layers, levels, features, formats, blocks w, h, uint8 grid
CASES = [(96, 1, 5, 16, (4,), 9, 7, True), (128, 2, 9, 8, (1, 4), 33, 20, False), (64, 3, 4, 4, (1,) * 8, 20, 21, True),
         (128, 2, 6, 8, (1, 1, 1, 1, 1, 4), 64, 64, True), (128, 4, 9, 2, (1,) * 6, 17, 30, False),
         (256, 3, 8, 8, (1, 1, 1, 1, 1, 4), 40, 44, True), (256, 1, 10, 16, (4,), 25, 31, True),
         (192, 2, 8, 16, (4, 4, 1, 1, 1, 1), 64, 32, False), (256, 2, 7, 1, (1,) * 5, 13, 13, True)]


@pytest.mark.parametrize("precision", ["bf16", "fp16"])
@pytest.mark.parametrize("hidden,n_hidden,levels,feats,formats,bw,bh,u8", CASES)
def test_wide_shapes(precision, hidden, n_hidden, levels, feats, formats, bw, bh, u8):
    ensure_built()
    cfg = synth.ModelConfig(levels, 2, feats, u8, hidden, n_hidden, formats, bw, bh)
    flat, layers, g = model_inputs(cfg, hidden + levels, u8=u8)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    grid = [t(g["codes"]), t(g["scale"]), t(g["zero"])] if u8 else [t(g["grid"])]
    m = ntbc.Model(ntbc.desc_from_config(cfg), t(flat), *grid)
    words, heads = m.infer(ntbc.PRECISIONS[precision], 1, bw * bh - 2, heads=True)
    hs = heads.cpu().numpy()
    assert np.array_equal(u64(words), ON.pack(hs, formats, "f32"))
    dy = np.abs(hs - ON.heads(cfg, oracle_levels(cfg, g), layers, np.arange(1, bw * bh - 1), precision))
    top, p99 = (1e-2, 2e-3) if precision == "bf16" else (2e-3, 4e-4)
    assert dy.max() <= top and np.percentile(dy, 99) <= p99 and np.median(dy) <= 1e-6
