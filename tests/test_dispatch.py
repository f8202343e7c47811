"""Which form a pass takes (whole items, half items, persistent workgroups), asked of the scheduler's own rules on the host."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import dispatch_packs as packs
from paper_2504_20490_amd import build as lib_build

SHIM = """
#include "schedule.hpp"
using namespace hspmd;
extern "C" int packed_form(int kind, const int* cu, int n, int hq, int hkv, int d) {
    const auto k = (hspmd_list_kind)kind;
    return (int)pass_dispatch(k, pass_load(k, cu, n, hq, hkv), (int64_t)build_work_list(k, cu, n, hq, hkv, kNumXcd).size(), d, false);
}
extern "C" int block_form(int kind, const int* cq, const int* ck, const int* qp, const int* kp, int n, int hq, int hkv, int d) {
    const auto k = (hspmd_list_kind)kind;
    return (int)pass_dispatch(k, block_pass_load(k, cq, ck, qp, kp, n, hq, hkv),
                              (int64_t)build_block_list(k, cq, ck, qp, kp, n, hq, hkv, kNumXcd).size(), d, true);
}
"""


@pytest.fixture(scope="module")
def scheduler(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("dispatch")
    src, so = tmp / "shim.cpp", tmp / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", lib_build.CSRC, "-o", str(so), str(src),
                    os.path.join(lib_build.CSRC, "schedule.cpp")], check=True)
    return ctypes.CDLL(str(so))


def _ints(a):
    return (ctypes.c_int32 * len(a))(*[int(x) for x in a])


def _cu(lengths):
    return _ints(np.concatenate([[0], np.cumsum(lengths)]))


def _packed(lib, lengths, hq, hkv, d):
    return tuple(lib.packed_form(kind, _cu(lengths), len(lengths), hq, hkv, d) for kind in range(3))


@pytest.mark.parametrize("lengths,hq,hkv,d,rows,dkv", packs.PACKED + packs.PERSISTENT_PACKS)
def test_packed_packs(scheduler, lengths, hq, hkv, d, rows, dkv):
    assert _packed(scheduler, lengths, hq, hkv, d) == (rows, rows, dkv)


@pytest.mark.parametrize("hq,hkv,d,rows,dkv", packs.BLOCKS)
def test_block_packs(scheduler, hq, hkv, d, rows, dkv):
    ql, kl, qp, kp = packs.GEOMETRY
    form = tuple(scheduler.block_form(kind, _cu(ql), _cu(kl), _ints(qp), _ints(kp), len(ql), hq, hkv, d) for kind in range(3))
    assert form == (rows, rows, dkv)


def test_packs_of_the_other_form(scheduler):
    """The edges on which half items are compared with the oracle, and the many short items of the persistent pass."""
    from test_gpu_split_items import EDGES, MANY_SHORT
    for lengths in (EDGES, [449], [700, 64], [1100], [449, 70, 129]):
        for hq, hkv, d in ((2, 2, 128), (3, 1, 128), (2, 1, 104), (2, 2, 96), (4, 2, 64), (2, 1, 64), (2, 2, 40)):
            assert _packed(scheduler, lengths, hq, hkv, d) == (packs.HALVES,) * 3, (lengths, hq, hkv, d)
    for hq, hkv, d in ((8, 8, 128), (16, 8, 104), (8, 8, 72)):
        assert _packed(scheduler, MANY_SHORT, hq, hkv, d)[2] == packs.PERSISTENT
    assert _packed(scheduler, [2048] * 8, 32, 32, 128) == (packs.WHOLE,) * 3


@pytest.mark.parametrize("lengths,hq,hkv,d", [([512] * 3, 16, 16, 128), ([512] * 3, 16, 16, 64), ([256] * 5, 16, 16, 96),
                                              ([100] * 9, 16, 16, 64), ([64] * 2, 4, 4, 128)])
def test_short_items_on_many_units_stay_whole(scheduler, lengths, hq, hkv, d):
    """Halves of them are more than the chip has units, or too short for what halves cost."""
    assert _packed(scheduler, lengths, hq, hkv, d)[:2] == (packs.WHOLE, packs.WHOLE)


@pytest.mark.parametrize("lengths,heads,d,form", [
    ([512] * 10, 4, 128, packs.WHOLE),            # 160 items: halves would come in two rounds
    ([16384], 2, 64, packs.WHOLE),                # two whole items fit a unit, halves do not
    ([64] * 43, 24, 128, packs.WHOLE), ([300] * 67, 8, 128, packs.WHOLE), ([1300] * 5, 24, 128, packs.WHOLE),
    ([400] * 33, 16, 128, packs.PERSISTENT), ([512] * 78, 16, 128, packs.PERSISTENT),
    ([1024] * 7, 40, 128, packs.WHOLE), ([1024] * 7, 40, 104, packs.PERSISTENT), ([16384], 1, 128, packs.HALVES)])
def test_form_of_the_dkv_pass(scheduler, lengths, heads, d, form):
    assert _packed(scheduler, lengths, heads, heads, d)[2] == form
