"""A batch decodes materials of widths 64 and 128 with the instance of their mix or, small ones together, with the any-mix
one: the same words, from the same packed weights (the order of the head rows does not depend on the choice)."""
import ctypes

import pytest
import torch

from cases import model_inputs
from util import ensure_built
from paper_2407_09543_amd import ntbc, synth

pytestmark = pytest.mark.gpu


def models(hidden, n_hidden):
    out = []
    # formats out of order, too: the BC1 textures come first in the packed rows, in their place in the words
    for k, (formats, bw, bh) in enumerate((((1, 1, 4), 45, 33), ((1, 4, 1, 4), 64, 64), ((4, 1, 4, 1, 4), 70, 20), ((4, 1, 4), 31, 17))):
        cfg = synth.ModelConfig(8, 2, 8, True, hidden, n_hidden, formats, bw, bh)
        flat, _, g = model_inputs(cfg, 10 * hidden + k, u8=True)
        t = [torch.from_numpy(x).cuda() for x in (flat, g["codes"], g["scale"], g["zero"])]
        out.append(ntbc.Model(ntbc.desc_from_config(cfg), *t))
    return out


@pytest.mark.parametrize("n_hidden", [2, 3])
@pytest.mark.parametrize("hidden", [64, 128])
def test_same_words_by_either_instance(hidden, n_hidden):
    ensure_built()
    ms = models(hidden, n_hidden)
    entries = [(m, m.desc, 0, m.desc.blocks_w * m.desc.blocks_h) for m in ms]
    together = ntbc.Batch(entries, ntbc.BF16)
    assert len(together.groups()) == 1
    got = [o.clone() for o in together.run()]
    for e, o in zip(entries, got):
        alone = ntbc.Batch([e], ntbc.BF16)
        assert alone.groups()[0]["nb1"] == (2 if e[0].desc.n_textures != 3 or e is entries[0] else -2)
        assert torch.equal(alone.run()[0], o) and torch.equal(e[0].infer(ntbc.BF16), o)


@pytest.mark.parametrize("hidden", [64, 128])
def test_replanned_without_packing_again(hidden):
    # the ranges change which instance decodes a mix; the weights that lie in the workspace still serve
    ensure_built()
    ms = models(hidden, 3)[:2]
    small = ntbc.Batch([(m, m.desc, 0, m.desc.blocks_w * m.desc.blocks_h) for m in ms], ntbc.BF16)
    assert [g["nb1"] for g in small.groups()] == [-2]
    large = []
    for m in ms:
        d = ntbc.ModelDesc.from_buffer_copy(m.desc)
        d.blocks_w, d.blocks_h = 600, 500
        large.append((m, d, 0, 300000))
    large = ntbc.Batch(large, ntbc.BF16)
    assert sorted(g["nb4"] for g in large.groups()) == [1, 2]
    want = [o.clone() for o in large.run()]
    # the same plan over the small batch's workspace, packed for the any-mix instance
    n, tb, ws = 2, len(large.table), ctypes.c_size_t()
    table = (ctypes.c_uint8 * tb)()
    lib, at = ntbc.lib(), ctypes.addressof(table)
    assert lib.ntbc_batch_plan(ctypes.addressof(large._arr), n, ntbc.BF16, small.ws.data_ptr(), at, tb, ctypes.byref(ws)) == 0
    assert ws.value <= small.ws.numel()
    dev = torch.frombuffer(bytearray(bytes(table)), dtype=torch.uint8).cuda()
    for o in large.outputs:
        o.zero_()
    assert lib.ntbc_infer_batch(at, dev.data_ptr(), small.ws.data_ptr(), small.ws.numel(), None, None) == 0
    torch.cuda.synchronize()
    assert all(torch.equal(o, w) for o, w in zip(large.outputs, want))
