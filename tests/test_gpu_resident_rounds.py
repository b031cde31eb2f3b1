"""Narrow networks with resident weights (k_infer_res, and the batch's width-64 instance) over more positions than the
chip's waves take in one round: a wave's later rounds read the weights that it already has.  Ragged ends, so
that the last workgroup stops inside a round.  The words are those of the same range in one-round pieces, and
at sampled positions those of the oracle's packing of the kernel's own heads, which are the emulation's."""
import numpy as np
import pytest
import torch

from cases import model_inputs, oracle_levels
from util import ensure_built, u64
from oracle import ntbc as ON
from paper_2407_09543_amd import ntbc, synth

pytestmark = pytest.mark.gpu


def model(hidden, n_hidden, levels, formats, bw, bh, seed):
    cfg = synth.ModelConfig(levels, 8, 8, True, hidden, n_hidden, formats, bw, bh)
    flat, layers, g = model_inputs(cfg, seed, u8=True)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return cfg, layers, g, ntbc.Model(ntbc.desc_from_config(cfg), t(flat), t(g["codes"]), t(g["scale"]), t(g["zero"]))


def sampled(cfg, layers, g, m, prec, name, words, heads, first, count):
    pick = np.unique(np.concatenate([np.random.default_rng(3).integers(0, count, 1500), np.arange(count - 40, count)]))
    hs = heads[torch.from_numpy(pick).cuda()].cpu().numpy()
    assert np.array_equal(u64(words)[:, pick], ON.pack(hs, cfg.formats, "f32"))
    dy = np.abs(hs - ON.heads(cfg, oracle_levels(cfg, g), layers, first + pick, name))
    top, p99 = (1e-2, 2e-3) if name == "bf16" else (2e-3, 4e-4)  # the bounds of test_gpu_infer.py
    assert dy.max() <= top and np.percentile(dy, 99) <= p99 and np.median(dy) <= 1e-6


# 65,536 positions are one round of 256 workgroups of eight waves of 32; rounds: two with a ragged last one, four and a bit
@pytest.mark.parametrize("bw,bh,first", [(300, 300, 7), (540, 500, 3)], ids=["two", "five"])
@pytest.mark.parametrize("precision", ["bf16", "fp16"])
@pytest.mark.parametrize("hidden,n_hidden", [(64, 2), (64, 3), (128, 2), (128, 3)])
def test_rounds(hidden, n_hidden, precision, bw, bh, first):
    ensure_built()
    cfg, layers, g, m = model(hidden, n_hidden, 6, (4, 1, 4), bw, bh, hidden + bw)
    count, prec = bw * bh - first - 5, ntbc.PRECISIONS[precision]
    words, heads = m.infer(prec, first, count, heads=True)
    piece = 60001
    for p in range(0, count, piece):
        n = min(piece, count - p)
        w, h = m.infer(prec, first + p, n, heads=True)
        assert torch.equal(w, words[:, p:p + n]) and torch.equal(h, heads[p:p + n])
    sampled(cfg, layers, g, m, prec, precision, words, heads, first, count)


@pytest.mark.parametrize("precision", ["bf16", "fp16"])
def test_batch_rounds(precision):
    # width 64: 512 workgroups of four waves are resident, so 65,536 positions are one round; two items of more
    ensure_built()
    prec = ntbc.PRECISIONS[precision]
    made = [model(64, 3, 8, (1, 4, 4), 300, 300, 1), model(64, 3, 8, (4, 1, 4, 4), 411, 205, 2)]
    ranges = [(11, 300 * 300 - 11 - 3), (0, 411 * 205)]
    batch = ntbc.Batch([(m, m.desc, *r) for (_, _, _, m), r in zip(made, ranges)], prec, tiles={})
    assert len(batch.groups()) == 1
    want = [m.infer(prec, *r, heads=True) for (_, _, _, m), r in zip(made, ranges)]
    for waves in (4, 2, 8) if precision == "bf16" else (4,):
        batch.set_waves(0, waves)
        for o in batch.outputs:
            o.zero_()
        assert all(torch.equal(o, w) for o, (w, _) in zip(batch.run(), want)), waves
    for (cfg, layers, g, m), (w, h), r in zip(made, want, ranges):
        sampled(cfg, layers, g, m, prec, precision, w, h, *r)
