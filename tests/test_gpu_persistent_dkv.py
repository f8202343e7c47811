"""Persistent dK/dV workgroups on packs of long items: the same bits as one workgroup per item.

A block plan of whole sequences runs the same arithmetic with one workgroup per item, and takes the row statistics that the packed
pass left, so dK and dV have to agree exactly.  The packs are the smallest that the rule takes, with items of every length from one
tile up, and widths with kernels of their own."""
import ctypes
import os
import subprocess

import pytest

from gpu_util import make_case, to_dev
from paper_2504_20490_amd import build as lib_build

PACKS = [([1300] * 7, 20, 20, 128), ([1300, 64, 1, 777, 2000, 129] * 3, 14, 14, 104), ([900, 1025] * 8, 12, 12, 128),
         ([1300, 650] * 4, 24, 24, 80)]


@pytest.mark.gpu
@pytest.mark.parametrize("lengths,hq,hkv,d", PACKS)
def test_same_bits_as_one_workgroup_per_item(lengths, hq, hkv, d):
    import torch
    import paper_2504_20490_amd as A
    T = sum(lengths)
    q, k, v, do = (to_dev(x) for x in make_case(lengths, hq, hkv, d, seed=60 + d))
    cu, _, _ = A.build_cu_seqlens(lengths)
    plan = A.Plan(cu, hq, hkv, d)
    assert plan.num_items(A.LIST_DKV) >= 1536
    o, lse = torch.empty(T, hq, d, dtype=torch.bfloat16, device="cuda"), torch.empty(hq, T, dtype=torch.float32, device="cuda")
    full = lambda h: torch.full((T, h, d), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(plan.bwd_workspace_bytes(), dtype=torch.uint8, device="cuda")
    A.attn_varlen_fwd(plan, q, k, v, o, lse)
    results = []
    for _ in range(3):                                   # the draw counters start from zero again
        dq, dk, dv = full(hq), full(hkv), full(hkv)
        A.attn_varlen_bwd(plan, q, k, v, o, lse, do, dq, dk, dv, ws, grad_dtype=A.GRAD_F32)
        results.append((dk, dv))
    blocks = A.BlockPlan(cu, cu, [0] * len(lengths), [0] * len(lengths), hq, hkv, d)
    dq, dk, dv = full(hq), full(hkv), full(hkv)
    A.attn_block_bwd(blocks, q, k, v, None, None, do, dq, dk, dv, ws, reuse_statistics=True)
    torch.cuda.synchronize()
    assert not torch.isnan(dk).any() and not torch.isnan(dv).any()
    for i, (a, b) in enumerate(results):
        assert torch.equal(a, dk) and torch.equal(b, dv), i


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("persistent")
    src, so = tmp / "rule.cpp", tmp / "rule.so"
    src.write_text('#include "schedule.hpp"\nusing namespace hspmd;\n'
                   'extern "C" int rule(int form, long total, long heaviest, long slots, int group, int d) {\n'
                   '    PassLoad l; l.total = total; l.heaviest = heaviest; return persistent_dkv((Dispatch)form, l, slots, group, d); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", lib_build.CSRC, "-o", str(so), str(src),
                    os.path.join(lib_build.CSRC, "schedule.cpp")], check=True)
    fn = ctypes.CDLL(str(so)).rule
    fn.argtypes = [ctypes.c_int, ctypes.c_long, ctypes.c_long, ctypes.c_long, ctypes.c_int, ctypes.c_int]
    return fn


@pytest.mark.parametrize("slots,total,heaviest,d,persistent", [
    (1536, 1536 * 17, 32, 128, True), (1528, 1528 * 17, 32, 128, False), (1536, 4916, 4, 104, True), (1536, 4915, 4, 104, False),
    (1536, 1536 * 17, 112, 128, True), (1536, 1536 * 17, 113, 128, False), (4096, 4096 * 64, 170, 65, True),
    (4096, 4096 * 49, 170, 113, False), (4096, 4096 * 17, 32, 64, False)])
def test_rule(rule, slots, total, heaviest, d, persistent):
    assert rule(0, total, heaviest, slots, 1, d) == persistent
    assert rule(0, total, heaviest, slots, 2, d) == 0       # items of several heads
    assert rule(1, total, heaviest, slots, 1, d) == 0       # half items stay half items
