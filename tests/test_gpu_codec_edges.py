"""Edges of the packed integer codec against the oracle (bit-exact): textures whose base or pitch is not
a multiple of four bytes (byte loads and stores instead of words), narrow and flat single-channel blocks
(every value range from every base), and the quotients by constants over their whole ranges."""
import ctypes

import numpy as np
import pytest
import torch

from util import ensure_built, u64
from oracle import bc
from paper_2407_09543_amd import ntbc


def test_constant_quotients():
    # the codec's reciprocals: one product and a shift, exact over the stated ranges
    for mul, shift, div, top in ((0xAAAB, 17, 3, 1 << 16), (0x8081, 23, 255, 1 << 16), (13108, 16, 5, 1792),
                                 (9363, 16, 7, 1792)):
        x = np.arange(top, dtype=np.uint64)
        assert np.array_equal((x * mul) >> shift, x // div)
        assert int(x[-1]) * mul < 1 << 32


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", [1, 4])
@pytest.mark.parametrize("base,extra", [(0, 0), (1, 0), (0, 3), (2, 5)])
def test_unaligned_textures(fmt, base, extra):
    ensure_built()
    rng = np.random.default_rng(100 * fmt + 10 * base + extra)
    ch, h, w = (3 if fmt == 1 else 1), 24, 52
    pitch = w * ch + extra
    raw = rng.integers(0, 256, base + h * pitch, dtype=np.uint8)
    tex = np.lib.stride_tricks.as_strided(raw[base:], (h, w, ch), (pitch, ch, 1)).copy()
    blocks = bc.image_to_blocks(tex)
    dev = torch.from_numpy(raw).cuda()
    n = (h // 4) * (w // 4)
    out = torch.empty(n, dtype=torch.int64, device="cuda")
    sse = torch.empty(n, dtype=torch.int32, device="cuda")
    lib, p = ntbc.lib(), ctypes.c_void_p
    src = p(dev.data_ptr() + base)
    assert lib.ntbc_bc_encode_ref(src, w, h, pitch, fmt, p(out.data_ptr()), p(sse.data_ptr()), ntbc._stream()) == 0
    words, want_sse = (bc.bc1_encode_ref(blocks, return_sse=True) if fmt == 1 else
                       bc.bc4_encode_ref(blocks[..., 0], return_sse=True))
    assert np.array_equal(u64(out), words) and np.array_equal(sse.cpu().numpy(), want_sse)
    sse.zero_()
    assert lib.ntbc_block_sse(p(out.data_ptr()), src, w, h, pitch, fmt, p(sse.data_ptr()), ntbc._stream()) == 0
    assert np.array_equal(sse.cpu().numpy(), want_sse)
    # decode into a buffer of the same alignment: the texels arrive, the bytes between the rows stay
    dst = torch.full((base + h * pitch,), 7, dtype=torch.uint8, device="cuda")
    assert lib.ntbc_bc_decode(p(out.data_ptr()), w, h, fmt, p(dst.data_ptr() + base), pitch, ntbc._stream()) == 0
    ref = bc.bc1_decode(words) if fmt == 1 else bc.bc4_decode(words)[..., None]
    want = np.full(base + h * pitch, 7, dtype=np.uint8)
    np.lib.stride_tricks.as_strided(want[base:], (h, w, ch), (pitch, ch, 1))[:] = bc.blocks_to_image(ref, h, w).reshape(h, w, ch)
    assert np.array_equal(dst.cpu().numpy(), want)


@pytest.mark.gpu
def test_bc4_ranges():
    # blocks over [lo, lo + span] for every lo and small and large spans, with and without 0 and 255
    ensure_built()
    rng = np.random.default_rng(4)
    rows = []
    for span in (0, 1, 2, 3, 4, 5, 6, 7, 8, 13, 40, 100, 254, 255):
        for lo in range(256 - span):
            b = rng.integers(lo, lo + span + 1, 16)
            b[:2] = lo, lo + span
            rows.append(b)
            c = b.copy()
            c[rng.integers(0, 16, 5)] = rng.choice([0, 255], 5)
            rows.append(c)
    blocks = np.array(rows, dtype=np.uint8)
    blocks = blocks[:len(blocks) // 16 * 16, :, None]
    tex = bc.blocks_to_image(blocks, 4 * (len(blocks) // 16), 64)[..., 0]
    words, sse = ntbc.encode_ref(torch.from_numpy(np.ascontiguousarray(tex)).cuda(), 4, return_sse=True)
    want, want_sse = bc.bc4_encode_ref(bc.image_to_blocks(tex)[..., 0], return_sse=True)
    assert np.array_equal(u64(words), want) and np.array_equal(sse.cpu().numpy(), want_sse)
