"""The narrow networks' backward with their weight products (k_f32_bwd_dw) against the FP64 oracle, at one to
three tiles of endpoint outputs and one and two of colours, and batches from one block (one group of 16 texels, a
sixteenth of a group of blocks) to more than a workgroup's share.  Bound 1e-4 of the 2-norm, the two-network
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
    def __init__(self, formats, seed):
        self.col, self.formats = COL, [1 if f == "c" else 4 for f in formats]
        pick = {t.fmt == BC1: t.texels for t in synth.material_small(SIZE, seed).textures}
        texels = [np.ascontiguousarray(np.roll(pick[f == BC1], 5 * k, axis=0)) for k, f in enumerate(self.formats)]
        blocks = [OB.image_to_blocks(t) for t in texels]
        ref = [OB.bc1_encode_ref(b) if f == BC1 else OB.bc4_encode_ref(b[..., 0]) for b, f in zip(blocks, self.formats)]
        self.tg_oracle = ON.Targets(self.formats, ref, blocks)
        self.tex = [torch.from_numpy(t).cuda() for t in texels]
        self.tg_gpu = ntbc.Targets(torch.stack([ntbc.encode_ref(t, f) for t, f in zip(self.tex, self.formats)]), self.tex)
        rng = np.random.default_rng(seed)
        e, c = F.output_nodes(self.formats)
        self.ew, self.cw = self._net(rng, 2 * EP["n_levels"], e), self._net(rng, 2 * COL["n_levels"], c)
        self.eg = rng.uniform(-0.5, 0.5, (F.grid_vertices(EP), 2)).astype(np.float32)
        self.cg = rng.uniform(-0.5, 0.5, (F.grid_vertices(COL), 2)).astype(np.float32)
        self.bw = self.bh = SIZE // 4


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
