"""Which materials of a batched decode share a launch (ntbc_batch_plan, host only): mixes with a kernel instance of their
own keep it where their positions repay the launch, small ones go together to the any-mix instance.  Device pointers
are placeholders; the plan reads none."""
import ctypes

import pytest

from util import ensure_built
from paper_2407_09543_amd import ntbc

ANY = (-2, 0)


def groups(mats, precision=ntbc.BF16, empty=()):
    """mats: (width, hidden layers, mix, texture size); one item each.  {(width, nh, nb1, nb4): items}"""
    ensure_built()
    arr = (ntbc.BatchItemC * len(mats))()
    for i, (hidden, n_hidden, mix, size) in enumerate(mats):
        arr[i].desc = ntbc.make_desc(8, 8, 8, True, hidden, n_hidden, [1 if c == "c" else 4 for c in mix], size // 4, size // 4)
        arr[i].params.grid = arr[i].params.weights = arr[i].params.grid_scale = arr[i].params.grid_zero = 1 << 20
        arr[i].n_blocks = 0 if i in empty else (size // 4) ** 2
        arr[i].blocks_out = 1 << 20
        arr[i].model_id = i
    tb, ws, n = ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_int32()
    lib = ntbc.lib()
    assert lib.ntbc_batch_table_size(len(mats), ctypes.byref(tb)) == 0
    table = (ctypes.c_uint8 * tb.value)()
    at = ctypes.addressof(table)
    assert lib.ntbc_batch_plan(ctypes.addressof(arr), len(mats), precision, None, at, tb.value, ctypes.byref(ws)) == 0
    buf = (ctypes.c_int32 * 256)()
    assert lib.ntbc_batch_groups(at, buf, 32, ctypes.byref(n)) == 0
    return {(buf[8 * g + 1], buf[8 * g + 3], buf[8 * g + 4], buf[8 * g + 5]): buf[8 * g + 7] for g in range(n.value)}


@pytest.mark.parametrize("hidden", [64, 128])
def test_small_mixes_share_a_launch(hidden):
    three = [(hidden, 3, m, 512) for m in ("ccs", "ccss", "ccsss")]
    assert groups(three) == {(hidden, 2, *ANY): 3}
    # alone, a mix keeps its instance: there is no launch to save
    for m in three:
        nb4 = len(m[2]) - 2
        assert groups([m]) == {(hidden, -1, 2, nb4): 1}
    # unless another mix launches the any-mix instance anyway
    assert groups([three[0], (hidden, 3, "cs", 512)]) == {(hidden, 2, *ANY): 2}
    # networks of different depth do not share one
    assert groups([three[0], (hidden, 2, "ccss", 512)]) == {(hidden, -1, 2, 1): 1, (hidden, -1, 2, 2): 1}


@pytest.mark.parametrize("hidden", [64, 128])
def test_large_mixes_keep_their_instances(hidden):
    big = [(hidden, 3, m, 4096) for m in ("ccs", "ccss", "ccsss")]
    assert groups(big) == {(hidden, -1, 2, k): 1 for k in (1, 2, 3)}
    # a small one beside a large one of its mix goes with it; one beside large ones of other mixes launches by itself
    assert groups(big + [(hidden, 3, "ccs", 64)]) == {(hidden, -1, 2, 1): 2, (hidden, -1, 2, 2): 1, (hidden, -1, 2, 3): 1}
    # two small mixes beside a large one share the any-mix launch
    assert groups([big[0], (hidden, 3, "ccss", 256), (hidden, 3, "ccsss", 256)]) == {(hidden, -1, 2, 1): 1, (hidden, 2, *ANY): 2}


def test_three_bc4_at_128_pay_off_late():
    # its two epilogues differ by 5%: 1536^2 (147,456 positions) goes with the others, which keep theirs
    mats = [(128, 3, m, 2048) for m in ("ccs", "ccss", "ccsss", "cs")]
    assert groups(mats) == {(128, -1, 2, 1): 1, (128, -1, 2, 2): 1, (128, 2, *ANY): 2}


def test_what_has_no_choice():
    # width 256 and half precision as before; four hidden layers have no any-mix instance; empty items add nothing
    assert groups([(256, 3, m, 256) for m in ("ccs", "ccss")]) == {(256, 2, 2, 1): 1, (256, 2, 2, 2): 1}
    assert groups([(64, 3, m, 4096) for m in ("ccs", "ccss")], ntbc.FP16) == {(64, 2, *ANY): 2}
    assert groups([(64, 4, m, 256) for m in ("ccs", "ccss")]) == {(64, -1, 2, 1): 1, (64, -1, 2, 2): 1}
    assert groups([(64, 3, "ccs", 256), (64, 3, "cs", 256)], empty=(1,)) == {(64, -1, 2, 1): 1, (64, 2, *ANY): 0}
