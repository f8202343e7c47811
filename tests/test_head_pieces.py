"""dK/dV items that are dealt out by query heads and tiles: what the shares cover, on the CPU, and the outputs on the GPU."""
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
# shares of one head's tiles: whole, with the list in the arguments and on the device
PACKS += [([2438, 32], 2, 2, 64, 0), ([2681], 3, 3, 96, 0), ([1769, 473], 3, 3, 128, 0), ([4466, 410], 5, 5, 64, 0), ([7617, 1702, 1436], 4, 4, 128, 0)]
# half shares, the last of heads
PACKS += [([1967], 2, 2, d, 1) for d in (64, 40)] + [([1411], 1, 1, d, 1) for d in (80, 96, 104, 128)]
PACKS += [([4500, 300, 1], 1, 1, d, 1) for d in (80, 104, 128)] + [([8000, 129], 2, 1, 96, 1)]
# no longest item that outlasts the rest by what the sums cost; lists in the arguments that shares which pay would not fit into
ORDINARY = [([4500, 300, 1], 1, 1, 64), ([8200, 64], 2, 2, 64), ([2048] * 4, 32, 8, 128), ([2048], 8, 8, 128), ([2048] * 8, 32, 32, 128), ([1024] * 2, 8, 8, 64), ([64] * 40, 8, 4, 128), ([256], 4, 1, 128), ([], 8, 2, 128)]

SHIM = """
#include <algorithm>
#include "schedule.hpp"
using namespace hspmd;
static PieceList list;
static int group;
extern "C" int build(const int* cu, int n, int hq, int hkv, int d, long long most) {
    const PassLoad load = pass_load(HSPMD_LIST_DKV, cu, n, hq, hkv);
    const size_t rows = build_work_list(HSPMD_LIST_FWD, cu, n, hq, hkv, kNumXcd).size(), keys = build_work_list(HSPMD_LIST_DKV, cu, n, hq, hkv, kNumXcd).size();
    if (most == 0) most = std::max(rows, keys) <= 240 ? 240 : 1 << 30;   // as a plan, whose lists are all in the arguments or none is
    group = hq / hkv;
    return build_piece_list(cu, n, hq, hkv, kNumXcd, load, (int64_t)keys, d, most, list);
}
extern "C" void sizes(long long* out) { out[0] = list.items.size(); out[1] = list.areas; out[2] = list.halves; }
extern "C" void copy(int* out) {
    for (const HeadPiece& x : list.items) {
        const bool pad = x.padding();
        const int fields[] = {x.token_start, x.seq_len, pad ? -1 : x.tile(), x.head(), pad ? 0 : x.first_head(), pad ? 0 : x.n_heads(group),
                              pad ? 0 : x.first_tile(), pad ? 0 : x.end_tile(), x.index(), pad ? 0 : x.shares(group), x.area()};
        for (int f : fields) *out++ = f;
    }
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

    def call(lengths, hq, hkv, d, most=0):
        cu = (ctypes.c_int32 * (len(lengths) + 1))(*np.concatenate([[0], np.cumsum(lengths)]).astype(int).tolist())
        if not lib.build(cu, len(lengths), hq, hkv, d, ctypes.c_longlong(most)):
            return None
        size = (ctypes.c_longlong * 3)()
        lib.sizes(size)
        items = np.zeros((size[0], 11), np.int32)
        lib.copy(items.ctypes.data_as(ctypes.c_void_p))
        return items, size[1], size[2]
    return call


@pytest.mark.parametrize("lengths,hq,hkv,d,halves", PACKS)
def test_shares_cover_every_head_of_every_item_once(pieces, lengths, hq, hkv, d, halves):
    items, areas, in_halves = pieces(lengths, hq, hkv, d)
    assert in_halves == halves and len(items) % 8 == 0
    starts = np.concatenate([[0], np.cumsum(lengths)])
    seen, parts = set(), {}
    for start, length, tile, head, first, n, first_tile, end_tile, index, shares, area in items[items[:, 2] >= 0]:
        assert length in lengths and start in starts and 128 * tile < length and 0 <= head < hkv
        diagonal, end = 2 * tile, -(-length // 64)
        assert (first_tile, end_tile) == (diagonal, end) or (n == hq // hkv == 1 and diagonal <= first_tile < end_tile - 1 < end)
        for h in range(first, first + n):
            assert 0 <= h < hq // hkv
            rows = {(start, tile, head, h, t) for t in range(first_tile, end_tile)}
            assert not rows & seen
            seen |= rows
        parts.setdefault((start, tile, head), []).append((first, first_tile, index, shares, area))
    assert len(seen) == sum(-(-n // 64) - 2 * t for n in lengths for t in range(-(-n // 128))) * hq
    # the areas of an item follow each other in the order of its heads and tiles, from its first share's on
    used = []
    for p in parts.values():
        p.sort()
        assert [x[2] for x in p] == list(range(p[0][3])) and all(x[3] == len(p) for x in p)
        if len(p) > 1:
            assert [x[4] for x in p] == list(range(p[0][4], p[0][4] + len(p)))
            used += [x[4] for x in p]
    assert sorted(used) == list(range(areas)) and areas > 0


@pytest.mark.parametrize("lengths,hq,hkv,d", ORDINARY)
def test_other_packs_keep_their_items(pieces, lengths, hq, hkv, d):
    assert pieces(lengths, hq, hkv, d) is None


def test_no_more_shares_than_asked_for(pieces):
    few = pieces([3000, 500], 8, 2, 128, 240)
    assert few is not None and len(few[0]) <= 240 and pieces([3000, 500], 8, 2, 128, 60) is None


@pytest.mark.gpu
@pytest.mark.parametrize("lengths,hq,hkv,d,halves", PACKS)
def test_outputs(lengths, hq, hkv, d, halves):
    """Sampled rows and keys against the oracle; bf16 and rotated gradients against the fp32 ones; every key against the pass that walks
    whole items, and no sum read that was not written."""
    import torch
    import test_gpu_whole_items
    from gpu_util import GpuRun, make_case
    test_gpu_whole_items.test_persistent_dkv_pass_on_long_items(lengths, hq, hkv, d, None, None)
    q, k, v, do = make_case(lengths, hq, hkv, d, seed=41)
    run = GpuRun(lengths, q, k, v, do)
    run.ws = torch.full((run.plan.bwd_workspace_bytes() // 4,), float("nan"), dtype=torch.float32, device="cuda")
    run.run()
    dealt = run.dk.clone(), run.dv.clone()
    assert run.ws.numel() > 2 * hq * sum(lengths) + 16
    run.ws = torch.full((2 * hq * sum(lengths) + 16,), float("nan"), dtype=torch.float32, device="cuda")
    run.dk.fill_(float("nan")), run.dv.fill_(float("nan"))
    run.backward()
    torch.cuda.synchronize()
    for got, whole in zip(dealt, (run.dk, run.dv)):
        # fp32 sums in another order; a weight whose fp32 value then lies on the other side of a rounding edge differs by a bf16 step, 2^-8 of
        # it at most; a key may have a single row, or rows that cancel (hence the mean).  (NaN compares false.)
        difference, size = (got - whole).norm(dim=2), whole.norm(dim=2)
        assert bool((difference <= 2.0 ** -8 * (size + size.mean())).all()), float((difference / (size + size.mean())).max())


@pytest.mark.gpu
def test_refills_of_one_plan():
    """From a pack without shares to packs with few and with many of them and back: what a plan of its own gives, every time; and with a
    workspace that has no room for the sums, what they sum to."""
    import torch
    import paper_2504_20490_amd as A
    from gpu_util import GpuRun, make_case
    hq, hkv, d = 8, 2, 128
    packs = [[100, 60], [512, 40], [4096, 300], [100, 60], [4096, 300], [2048] * 3]
    cu = [A.build_cu_seqlens(p)[0] for p in packs]
    plan, dealt = A.Plan(cu[0], hq, hkv, d), 0
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
        # the statistics alone
        least = (2 * hq * sum(lengths) + 16) * 4
        dealt += plan.bwd_workspace_bytes() > least
        run.ws = torch.empty(least, dtype=torch.uint8, device="cuda")
        run.backward()
        torch.cuda.synchronize()
        for n, x in zip(("dq", "dk", "dv"), want):
            # the order of fp32 sums over the group's rows, and P and dS of another 32-row block's partial products
            assert (getattr(run, n) - x).norm() <= 1e-5 * x.norm(), (lengths, n)
        with pytest.raises(A.HspmdError):
            run.ws = torch.empty(least - 4, dtype=torch.uint8, device="cuda")
            run.backward()
    assert dealt >= 2
