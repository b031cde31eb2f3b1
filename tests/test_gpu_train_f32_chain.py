"""Edges of the chained FP32 training path (k_f32_fwd, k_f32_bwd, k_f32_dw) against the FP64 oracle through
ntbc_forward and ntbc_backward: batches around the 16- and 64-position tiles, input widths that are no
multiple of 4 or 16, one to four hidden layers at each width, small and full heads.  Heads within 1e-5 (the
FP32 path's bound), gradients within 1e-5 of the oracle's in the 2-norm; hidden pre-activations within 1e-5 of
zero are left out (float32 may take the other side of the ReLU there) by dropping their positions."""
import numpy as np
import pytest
import torch

from util import ensure_built
from oracle import grid as G
from oracle import mlp
from oracle import ntbc as ON
from paper_2407_09543_amd import ntbc, synth

CASES = [  # hidden, hidden layers, levels, features, formats, batch
    (64, 1, 5, 1, (4,), 1), (64, 2, 4, 4, (1, 4), 15), (64, 4, 7, 2, (4, 4), 17), (64, 3, 8, 8, (1, 1, 4, 4, 4), 63),
    (128, 1, 3, 2, (1,), 64), (128, 3, 6, 8, (1, 1, 4, 4, 4), 65), (128, 2, 5, 4, (4,), 333), (128, 4, 7, 8, (1, 4), 16),
    (256, 1, 4, 8, (1, 1), 129), (256, 3, 8, 8, (1, 1, 4, 4, 4), 200), (256, 4, 3, 1, (4, 1), 31), (256, 2, 6, 4, (1,), 1000)]


def _config(hidden, n_hidden, levels, feats, formats):
    return synth.ModelConfig(levels, 4, feats, False, hidden, n_hidden, formats, 37, 29)


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,n_hidden,levels,feats,formats,n", CASES)
def test_forward_backward(hidden, n_hidden, levels, feats, formats, n):
    ensure_built()
    cfg = _config(hidden, n_hidden, levels, feats, formats)
    rng = np.random.default_rng(hidden + 10 * n_hidden + n)
    layers = [(w, (0.1 * rng.standard_normal(len(b))).astype(np.float32)) for w, b in synth.init_weights(cfg, n)]
    grid = synth.random_grid(cfg, n, 0.5)
    ids = rng.integers(0, cfg.n_positions, 4 * n + 64)
    x = G.features(ON.grid_levels(cfg, grid=grid), ids % 37, ids // 37, 37, 29)
    _, (_, zs) = mlp.forward(layers, x)
    clear = np.all([np.abs(z).min(axis=1) > 1e-5 for z in zs[:-1]], axis=0)
    ids = ids[clear][:n].astype(np.int32)
    assert len(ids) == n
    x = G.features(ON.grid_levels(cfg, grid=grid), ids % 37, ids // 37, 37, 29)
    y, cache = mlp.forward(layers, x)
    dy = rng.standard_normal(y.shape).astype(np.float32)
    dws, dbs, dx = mlp.backward(layers, cache, dy.astype(np.float64), y)
    dgrid = G.features_backward(dx, ids % 37, ids // 37, 37, 29, levels, 4, feats)
    desc = ntbc.desc_from_config(cfg)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    g, w, i = t(grid), t(synth.flatten_weights(layers)), t(ids)
    heads = ntbc.forward(desc, g, w, i).cpu().numpy()
    assert np.abs(heads - y).max() <= 1e-5
    dg, dw = ntbc.backward(desc, g, w, i, t(dy))
    want = np.concatenate([np.concatenate([a.ravel(), b]) for a, b in zip(dws, dbs)])
    for got, ref in ((dg.cpu().numpy().ravel(), dgrid.ravel()), (dw.cpu().numpy(), want)):
        assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)
    # the weight products add their ranges in a fixed order
    assert torch.equal(ntbc.backward(desc, g, w, i, t(dy))[1], dw)


def test_workspace_grows_with_the_batch():
    ensure_built()
    for hidden, n_hidden in ((128, 3), (256, 3), (96, 2)):
        desc = ntbc.desc_from_config(_config(hidden, n_hidden, 6, 8, (1, 1, 4, 4, 4)))
        sizes = [ntbc.workspace_size(desc, ntbc.FP32, b) for b in range(1, 1500)]
        assert all(a <= b for a, b in zip(sizes, sizes[1:]))
