"""CPU check of the push kernel's workgroup numbering (csrc/push_order.h): every (row block,
instance, slice of the targets) exactly once, whatever the batch; the XCDs evenly loaded when
budgets repeat every eight instances, and the 32 compute units of an XCD when only few of the row
blocks have work; the rule that picks the form."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2504_21411_amd", "csrc")
SOURCE = """
#include "push_order.h"
extern "C" long long workgroups(long long rb, long long B, int js, int run) { return gs::push_workgroups(rb, B, js, run); }
extern "C" int run_of(long long rb, int by) { return gs::push_run(rb, by != 0); }
extern "C" int by_instance(long long bytes, int B) { return gs::push_by_instance(bytes, B); }
extern "C" int row_groups(int S, int bp, long long tiles, int by) { return gs::push_row_groups(S, bp != 0, tiles, by != 0); }
extern "C" void items(unsigned n, int js, int B, int run, int *out) {
  for (unsigned i = 0; i < n; ++i) {
    const gs::PushItem it = gs::push_item(i, js, B, run);
    out[3 * i] = it.b; out[3 * i + 1] = it.row_block; out[3 * i + 2] = it.slice;
  }
}
"""


@pytest.fixture(scope="module")
def order(tmp_path_factory):
    d = tmp_path_factory.mktemp("push_order")
    (d / "order.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    str(d / "order.cpp"), "-o", str(d / "order.so")], check=True)
    lib = ctypes.CDLL(str(d / "order.so"))
    lib.workgroups.restype = ctypes.c_longlong
    lib.workgroups.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    lib.run_of.argtypes = [ctypes.c_longlong, ctypes.c_int]
    lib.row_groups.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.c_int]
    lib.by_instance.argtypes = [ctypes.c_longlong, ctypes.c_int]

    def items(B, row_blocks, jsplit, by):
        run = lib.run_of(row_blocks, by)
        n = lib.workgroups(row_blocks, B, jsplit, run)
        out = np.empty((n, 3), np.int32)
        lib.items(ctypes.c_uint(n), jsplit, B, run, out.ctypes.data_as(ctypes.c_void_p))
        return out
    return lib, items


@pytest.mark.parametrize("by", [0, 1])
@pytest.mark.parametrize("B", [1, 2, 7, 8, 9, 13, 64, 70, 259, 1024])
@pytest.mark.parametrize("row_blocks", [1, 2, 8, 9, 33])
@pytest.mark.parametrize("jsplit", [1, 3, 8])
def test_every_item_exactly_once(order, B, row_blocks, jsplit, by):
    it = order[1](B, row_blocks, jsplit, by)
    assert it.min() >= 0 and it[:, 2].max() < jsplit
    it = it[(it[:, 0] < B) & (it[:, 1] < row_blocks)]
    key = (it[:, 0].astype(np.int64) * row_blocks + it[:, 1]) * jsplit + it[:, 2]
    assert np.array_equal(np.sort(key), np.arange(B * row_blocks * jsplit))
    # the slices of an item on one XCD: workgroup i runs on XCD i % 8
    full = order[1](B, row_blocks, jsplit, by).reshape(-1, jsplit, 8, 3)
    assert (full[:, :, :, :2] == full[:, :1, :, :2]).all()


@pytest.mark.parametrize("B", [256, 259, 512, 2048])
@pytest.mark.parametrize("row_blocks", [8, 9, 16])
def test_budgets_that_repeat_fill_the_xcds_alike(order, B, row_blocks):
    """Budgets of 1/8 to 8/8, one after the other: no XCD more than an eighth above the average."""
    it = order[1](B, row_blocks, 1, 1)
    work = np.where((it[:, 0] < B) & (it[:, 1] < row_blocks), it[:, 0] % 8 + 1, 0)
    load = work.reshape(-1, 8).sum(0)
    assert load.max() <= 1.125 * load.mean()


@pytest.mark.parametrize("row_blocks", [4, 8, 9, 12, 16, 32])
@pytest.mark.parametrize("working", [0.125, 0.5])
def test_few_working_row_blocks_use_all_compute_units(order, row_blocks, working):
    """An XCD's workgroups go to its 32 compute units in turn: no unit gets more than twice the
    average when only the first eighth, or the middle half, of every instance's row blocks works."""
    it = order[1](2048, row_blocks, 1, 1).reshape(-1, 8, 3)[:, 0]
    first = 0 if working < 0.5 else row_blocks // 4
    last = first + max(1, round(working * row_blocks))
    work = ((it[:, 0] < 2048) & (it[:, 1] >= first) & (it[:, 1] < last)).astype(int)
    load = np.bincount(np.arange(len(work)) % 32, weights=work, minlength=32)
    assert load.max() <= 2 * load.mean()


def test_row_groups_of_a_wave(order):
    """Few strategies on many tiles take four (up to 1.5 times the speed of two), and no count asks for a
    form that is not built: four up to 8 strategies, two up to 48."""
    groups = order[0].row_groups
    assert groups(3, 0, 215000, 1) == 4 and groups(3, 1, 54000, 0) == 4 and groups(1, 0, 8192, 0) == 4
    assert groups(4, 1, 43000, 0) == 4 and groups(4, 0, 255000, 1) == 2
    assert groups(6, 0, 28000, 0) == 4 and groups(6, 1, 28000, 0) == 2
    assert groups(3, 0, 8191, 0) == 2 and groups(3, 0, 4095, 0) == 1
    for S in range(1, 129):
        for tiles in (1, 4096, 8192, 12288, 16384, 24576, 1 << 20):
            for bp in (0, 1):
                for by in (0, 1):
                    assert groups(S, bp, tiles, by) in ((1, 2, 4) if S <= 8 else (1, 2) if S <= 48 else (1,))


def test_which_batches_are_numbered_by_instance(order):
    MB = 1 << 20
    by = order[0].by_instance
    assert by(64 * MB, 8) and by(384 * MB, 2048) and by(70 * MB, 259) and by(64 * MB, 38)
    assert not by(64 * MB - 1, 2048) and not by(10 * MB, 8)        # the memory-side cache holds it
    assert not by(400 * MB, 9) and not by(400 * MB, 15) and not by(400 * MB, 65)  # XCDs would idle
