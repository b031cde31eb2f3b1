"""The two-network layout's training step with grids of more than eight levels (more than 16 inputs, beyond the narrow
kernels) in either network or both, against the FP64 oracle at that layout's bounds (losses 1e-5, gradients 1e-4
of the 2-norm: float32 products and sums)."""
import numpy as np
import pytest
import torch

from test_gpu_faithful_train import Problem, _rel
from util import ensure_built
from oracle import faithful as F
from paper_2407_09543_amd import ntbc

pytestmark = pytest.mark.gpu


class Levels(Problem):
    def __init__(self, ep_levels, col_levels, seed):
        super().__init__("all", seed)
        self.ep = dict(n_levels=ep_levels, base_res=2, n_features=2)
        self.col = dict(n_levels=col_levels, base_res=2, n_features=2)
        rng = np.random.default_rng(seed)
        e, c = F.output_nodes(self.formats)
        self.ew, self.cw = self._net(rng, 2 * ep_levels, e), self._net(rng, 2 * col_levels, c)
        self.eg, self.cg = (rng.uniform(-0.5, 0.5, (F.grid_vertices(g), 2)).astype(np.float32) for g in (self.ep, self.col))

    def trainer(self, batch, total, **kw):
        t = lambda a: torch.from_numpy(a).cuda()
        return ntbc.FaithfulTrainer(self.formats, self.bw, self.bh, t(self.eg), t(self.cg), t(self.flat(self.ew)),
                                    t(self.flat(self.cw)), self.tg_gpu, batch, total, ep_levels=self.ep["n_levels"],
                                    ep_base_res=2, col_levels=self.col["n_levels"], col_base_res=2, **kw)

    def oracle(self, ids, qat):
        return F.gradients(self.formats, self.eg, self.ew, self.cg, self.cw, self.tg_oracle, ids, self.bw, self.bh,
                           qat, ep_cfg=self.ep, col_cfg=self.col)


@pytest.mark.parametrize("ep,col", [(9, 5), (3, 10), (9, 9), (8, 8)])
@pytest.mark.parametrize("qat,det", [(False, False), (True, True)])
def test_more_than_eight_levels(ep, col, qat, det):
    ensure_built()
    pb = Levels(ep, col, 21)
    ids = pb.clean_ids(22, 200, qat)
    tr = pb.trainer(len(ids), 100, deterministic=det)
    before = [t.clone() for t in tr.params]
    losses = tr.step(torch.from_numpy(ids).cuda(), 0, qat=qat).cpu().numpy()
    l_or, dge, dle, dgc, dlc, _ = pb.oracle(ids, qat)
    assert losses[4] == 0 and np.allclose(losses[:4], l_or, rtol=1e-5, atol=1e-9)
    want = (dge, dgc, Problem.flat(dle), Problem.flat(dlc))
    got = (tr.d_ep_grid, tr.d_col_grid, tr.d_ep_weights, tr.d_col_weights)
    assert max(_rel(g.cpu().numpy().reshape(-1), np.asarray(w, np.float64).reshape(-1)) for g, w in zip(got, want)) <= 1e-4
    assert all(not torch.equal(a, b) for a, b in zip(before, tr.params))  # and the four parameter sets moved


def test_non_finite_weights_beyond_eight_levels():
    # a step that sees a NaN leaves the parameters as they are and says so
    ensure_built()
    pb = Levels(9, 9, 23)
    ids = torch.arange(64, dtype=torch.int32, device="cuda")
    tr = pb.trainer(64, 100)
    tr.col_weights[5] = float("nan")
    before = [t.clone() for t in tr.params]
    assert tr.step(ids, 0)[4] == 1
    assert all(torch.equal(a[~a.isnan()], b[~b.isnan()]) for a, b in zip(before, tr.params))
