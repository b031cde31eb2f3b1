"""The narrow networks' backward with their weight products (k_f32_bwd_dw) against the FP64 oracle, at one to
three tiles of endpoint outputs and one and two of colours, and batches from one block (one group of 16 texels, a
sixteenth of a group of blocks) to more than a workgroup's share, and the coarse grid scatter of their texel blocks.  Bound 1e-4 of the 2-norm, the two-network
layout's bound; bitwise repeatable."""
import numpy as np
import pytest
import torch

from test_gpu_faithful_train import COL, EP, Problem, SIZE, _rel
from util import ensure_built
from oracle import bc as OB
from oracle import faithful as F
from oracle import ntbc as ON
from oracle.ntbc import BC1
from paper_2407_09543_amd import ntbc, synth

pytestmark = pytest.mark.gpu


class Mix(Problem):
    def __init__(self, formats, seed, size=SIZE, col=COL):
        self.col, self.formats = col, [1 if f == "c" else 4 for f in formats]
        pick = {t.fmt == BC1: t.texels for t in synth.material_small(SIZE, seed).textures}
        texels = [np.ascontiguousarray(np.roll(pick[f == BC1], 5 * k, axis=0)[:size, :size]) for k, f in enumerate(self.formats)]
        blocks = [OB.image_to_blocks(t) for t in texels]
        ref = [OB.bc1_encode_ref(b) if f == BC1 else OB.bc4_encode_ref(b[..., 0]) for b, f in zip(blocks, self.formats)]
        self.tg_oracle = ON.Targets(self.formats, ref, blocks)
        self.tex = [torch.from_numpy(t).cuda() for t in texels]
        self.tg_gpu = ntbc.Targets(torch.stack([ntbc.encode_ref(t, f) for t, f in zip(self.tex, self.formats)]), self.tex)
        rng = np.random.default_rng(seed)
        e, c = F.output_nodes(self.formats)
        self.ew, self.cw = self._net(rng, 2 * EP["n_levels"], e), self._net(rng, 2 * col["n_levels"], c)
        self.eg = rng.uniform(-0.5, 0.5, (F.grid_vertices(EP), 2)).astype(np.float32)
        self.cg = rng.uniform(-0.5, 0.5, (F.grid_vertices(col), 2)).astype(np.float32)
        self.bw = self.bh = size // 4


@pytest.mark.parametrize("formats", ["s", "ccssss", "cccccccc"])
@pytest.mark.parametrize("n", [1, 17, 300])
def test_weight_products(formats, n):
    ensure_built()
    pb = Mix(formats, 11)
    ids = pb.clean_ids(12, n, False)
    runs = []
    for _ in range(2):
        tr = pb.trainer(n, 100, deterministic=True)
        assert tr.step(torch.from_numpy(ids).cuda(), 0)[4] == 0
        runs.append([g.clone() for g in (tr.d_ep_grid, tr.d_col_grid, tr.d_ep_weights, tr.d_col_weights)])
    assert all(torch.equal(a, b) for a, b in zip(*runs))
    _, dge, dle, dgc, dlc, _ = pb.oracle(ids, False)
    want = (dge, dgc, Problem.flat(dle), Problem.flat(dlc))
    assert max(_rel(g.cpu().numpy().reshape(-1), np.asarray(w, np.float64).reshape(-1)) for g, w in zip(runs[0], want)) <= 1e-4


# the coarse levels' sums of whole blocks: the finest of them below, at and beyond the texel grid's 32 x 32 (beyond:
# texel by texel), with the fixed-point sums' smaller share of levels too
@pytest.mark.parametrize("col", [dict(n_levels=2, base_res=12, n_features=2), dict(n_levels=2, base_res=16, n_features=2),
                                 dict(n_levels=1, base_res=33, n_features=2)], ids=["24", "32", "33"])
@pytest.mark.parametrize("qat,det", [(False, False), (True, True)])
def test_coarse_levels_of_texel_blocks(col, qat, det):
    ensure_built()
    pb = Mix("cs", 13, 32, col)
    ids = pb.clean_ids(14, 40, qat)
    tr = pb.trainer(len(ids), 100, deterministic=det)
    assert tr.step(torch.from_numpy(ids).cuda(), 0, qat=qat)[4] == 0
    _, dge, _, dgc, _, _ = pb.oracle(ids, qat)
    assert _rel(tr.d_col_grid.cpu().numpy(), dgc) <= 1e-4 and _rel(tr.d_ep_grid.cpu().numpy(), dge) <= 1e-4
