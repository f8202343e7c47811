"""dK/dV items of grouped heads that are dealt out by query heads: what the shares cover, on the CPU, and the outputs on the GPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2504_20490_amd import build as lib_build

LONG = [2500, 449, 1, 64, 130, 127]
# (lengths, q heads, kv heads, head_dim, half pieces)
PACKS = [(LONG, 6, 2, d, 1) for d in (40, 64, 80, 96, 104, 128)]
PACKS += [([3200, 1500, 900, 65, 1], 28, 7, d, 0) for d in (80, 96, 104, 128)] + [([3200, 900, 65, 1], 32, 4, 64, 0)]
PACKS += [([700, 300, 128], 6, 2, 128, 1), ([512], 8, 2, 128, 1), ([449], 5, 1, 72, 1)]
# no longest item that outlasts the rest, or heads that are not grouped
ORDINARY = [([2048] * 4, 32, 8, 128), ([3000, 500], 8, 8, 128), ([64] * 40, 8, 4, 128), ([256], 4, 1, 128), ([], 8, 2, 128)]

SHIM = """
#include "schedule.hpp"
#include <cstring>
using namespace hspmd;
static PieceList list;
extern "C" int build(const int* cu, int n, int hq, int hkv, int d) {
    const PassLoad load = pass_load(HSPMD_LIST_DKV, cu, n, hq, hkv);
    return build_piece_list(cu, n, hq, hkv, kNumXcd, load, (int64_t)build_work_list(HSPMD_LIST_DKV, cu, n, hq, hkv, kNumXcd).size(), d, list);
}
extern "C" void sizes(long long* out) { out[0] = list.items.size(); out[1] = list.sums.size(); out[2] = list.areas; out[3] = list.halves; }
extern "C" void copy(int* items, int* sums) {
    memcpy(items, list.items.data(), list.items.size() * sizeof(HeadPiece));
    memcpy(sums, list.sums.data(), list.sums.size() * sizeof(PieceSum));
}
"""


@pytest.fixture(scope="module")
def pieces(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("pieces")
    src, so = tmp / "shim.cpp", tmp / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", lib_build.CSRC, "-o", str(so), str(src),
                    os.path.join(lib_build.CSRC, "schedule.cpp")], check=True)
    lib = ctypes.CDLL(str(so))

    def call(lengths, hq, hkv, d):
        cu = (ctypes.c_int32 * (len(lengths) + 1))(*np.concatenate([[0], np.cumsum(lengths)]).astype(int).tolist())
        if not lib.build(cu, len(lengths), hq, hkv, d):
            return None
        size = (ctypes.c_longlong * 4)()
        lib.sizes(size)
        items, sums = np.zeros((size[0], 8), np.int32), np.zeros((size[1], 8), np.int32)
        lib.copy(items.ctypes.data_as(ctypes.c_void_p), sums.ctypes.data_as(ctypes.c_void_p))
        return items, sums, size[2], size[3]
    return call


@pytest.mark.parametrize("lengths,hq,hkv,d,halves", PACKS)
def test_shares_cover_every_head_of_every_item_once(pieces, lengths, hq, hkv, d, halves):
    items, sums, areas, in_halves = pieces(lengths, hq, hkv, d)
    assert in_halves == halves and len(items) % 8 == 0
    starts = np.concatenate([[0], np.cumsum(lengths)])
    seen, parts = set(), {}
    for start, length, tile, head, first, n, area, _ in items[items[:, 2] >= 0]:
        assert length in lengths and start in starts and 128 * tile < length and 0 <= head < hkv
        for h in range(first, first + n):
            assert (start, tile, head, h) not in seen and 0 <= h < hq // hkv
            seen.add((start, tile, head, h))
        if area < 0:
            assert (first, n) == (0, hq // hkv)
        else:
            parts.setdefault((start, tile, head), []).append((first, area))
    assert len(seen) == sum(-(-n // 128) for n in lengths) * hq
    assert sorted(a for p in parts.values() for _, a in p) == list(range(areas))
    # the areas of an item follow each other in the order of its heads
    want = {}
    for (start, tile, head), p in parts.items():
        p.sort()
        assert [a for _, a in p] == list(range(p[0][1], p[0][1] + len(p)))
        length = lengths[int(np.where(starts == start)[0][0])] if start else lengths[0]
        want[(start + 128 * tile, head)] = (min(128, length - 128 * tile), 128 * tile, p[0][1], len(p))
    got = {(r, h): (rows, pos, first, n) for r, rows, h, pos, first, n, _, _ in sums}
    assert got == want and len(sums) == len(want) > 0


@pytest.mark.parametrize("lengths,hq,hkv,d", ORDINARY)
def test_other_packs_keep_their_items(pieces, lengths, hq, hkv, d):
    assert pieces(lengths, hq, hkv, d) is None


@pytest.mark.gpu
@pytest.mark.parametrize("lengths,hq,hkv,d,halves", PACKS)
def test_outputs(lengths, hq, hkv, d, halves):
    """Sampled rows and keys against the oracle; bf16 and rotated gradients against the fp32 ones."""
    import test_gpu_whole_items
    test_gpu_whole_items.test_persistent_dkv_pass_on_long_items(lengths, hq, hkv, d, None, None)


@pytest.mark.gpu
def test_refills_of_one_plan():
    """From a pack without shares to packs with few and with many of them and back: what a plan of its own gives, every time."""
    import torch
    import paper_2504_20490_amd as A
    from gpu_util import GpuRun, make_case
    hq, hkv, d = 8, 2, 128
    packs = [[100, 60], [512, 40], [4096, 300], [100, 60], [4096, 300], [2048] * 3]
    cu = [A.build_cu_seqlens(p)[0] for p in packs]
    plan = A.Plan(cu[0], hq, hkv, d)
    for lengths, offsets in zip(packs, cu):
        q, k, v, do = make_case(lengths, hq, hkv, d, seed=31)
        run = GpuRun(lengths, q, k, v, do).run()
        want = [getattr(run, n).clone() for n in ("dq", "dk", "dv")]
        plan.update(offsets)
        run.plan = plan
        for n in ("dq", "dk", "dv"):
            getattr(run, n).fill_(float("nan"))
        run.backward()
        torch.cuda.synchronize()
        assert all(torch.equal(getattr(run, n), x) for n, x in zip(("dq", "dk", "dv"), want)), lengths
