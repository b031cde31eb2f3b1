"""Every texture mix of the paper-layout inference kernel (one instance per number of BC1 and BC4 slots of a
lane group, odd and even texture counts, interleaved formats) on a block grid that is no power of two,
against the oracle: packing bit-exact on the kernel's own heads, heads as in test_gpu_faithful.py."""
import numpy as np
import pytest

from util import ensure_built, u64
from oracle import faithful as F
from oracle import ntbc as ON
from oracle.ntbc import BC1, BC4
from test_gpu_faithful import _model

pytestmark = pytest.mark.gpu

# (BC1 textures, BC4 textures): every (slots, slots) with at most eight textures
MIXES = [(0, 1), (0, 4), (0, 5), (0, 8), (1, 0), (1, 1), (2, 3), (2, 6), (1, 7), (3, 0), (4, 2), (3, 4), (3, 5), (5, 0),
         (6, 2), (5, 3), (7, 0), (7, 1)]


@pytest.mark.parametrize("nb1,nb4", MIXES)
def test_slot_instances(nb1, nb4):
    ensure_built()
    rng = np.random.default_rng(17 * nb1 + nb4)
    formats = [int(f) for f in rng.permutation([BC1] * nb1 + [BC4] * nb4)]
    bw, bh, first, n = 37, 21, 3, 37 * 21 - 3 - 5
    m, (el, ew, cl, cw) = _model(rng, formats, bw, bh, (nb1 + nb4) % 2 == 0)
    words, heads = m.infer(first, n, heads=True)
    assert np.array_equal(u64(m.infer(first, n)), u64(words))  # without the heads
    heads = heads.cpu().numpy()
    assert np.array_equal(u64(words), ON.pack(heads, formats, "f32"))
    ids = np.arange(first, first + n)
    dy = np.abs(heads - F.block_heads(formats, el, ew, cl, cw, ids % bw, ids // bw, bw, bh, "fp16"))
    assert dy.max() <= 2e-3 and np.median(dy) <= 1e-6
