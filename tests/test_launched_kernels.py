"""Which kernels a pack launches, asked of the library itself (no GPU: see launch_recorder)."""
import pytest

import dispatch_packs as packs
import launch_recorder as rec


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    return rec.build_stand_in(tmp_path_factory.mktemp("recorder"))


def launched(stand_in, cases):
    """Per case (lengths or block geometry, q heads, kv heads, head_dim): the kernels of its forward and backward."""
    program = """
for pack, hq, hkv, d in args[0]:
    plan = BlockPlan(*pack, hq, hkv, d) if isinstance(pack[0], list) else Plan(pack, hq, hkv, d)
    calls(); plan.forward(); plan.backward()
    out([name for what, name, _ in calls() if what == "launch"])
"""
    return [[rec.kernel(name) for name in names] for names in rec.record(stand_in, program, cases)]


def _steps(d):
    return 4 if d <= 64 else max(5, -(-d // 16))


# (fifth argument of the dK/dV kernel: persistent workgroups; sixth: the walk for items of several query heads)
@pytest.mark.parametrize("pack,hq,hkv,d,block,persistent,groups", [
    (packs.RAGGED, 24, 12, 128, False, False, True), (packs.RAGGED, 24, 12, 96, False, False, False),
    ([4096] * 4, 32, 16, 112, False, False, False), ([16384], 32, 8, 120, False, False, True),
    (packs.GEOMETRY, 24, 12, 128, True, False, False), (packs.GEOMETRY, 12, 12, 128, True, False, False),
    (packs.RAGGED, 24, 12, 64, False, False, False), (packs.RAGGED, 8, 8, 128, False, False, False),
    ([1 + (i * 37) % 131 for i in range(40)] + [449] * 24, 16, 8, 104, False, True, False), ([2048] * 8, 32, 32, 128, False, True, False)])
def test_walk_of_the_dkv_pass(stand_in, pack, hq, hkv, d, block, persistent, groups):
    (names,) = launched(stand_in, [(pack, hq, hkv, d)])
    width = 64 if d <= 64 else 128
    assert names[-1] == ("bwd_dkv_kernel", (width, block, _steps(d), False, persistent, groups, False))


def test_packs_of_the_persistent_pass(stand_in):
    from test_gpu_persistent_dkv import PACKS
    for (lengths, hq, hkv, d), names in zip(PACKS, launched(stand_in, PACKS)):
        assert names[-1] == ("bwd_dkv_kernel", (128, False, _steps(d), False, True, False, False)), (lengths, d)
    # fewer than six items per compute unit: one workgroup each
    few = [([1300] * 5, 24, 24, 128), ([1300] * 8, 16, 16, 104), ([2440] * 7, 8, 8, 128)]
    for pack, names in zip(few, launched(stand_in, few)):
        assert names[-1] == ("bwd_dkv_kernel", (128, False, _steps(pack[3]), False, False, False, False)), pack


HALVES = {"fwd_kernel": 3, "bwd_dq_kernel": 3, "bwd_dkv_kernel": 3}      # the template argument that says half items


def test_half_items_of_either_kind_of_list(stand_in):
    long_lists, short_lists = packs.HALF_LONG_PACKS + packs.HALF_LONG_BLOCKS, [c for c in packs.SHORT_PACKS if c[0] is packs.EDGES]
    short_lists += [c for c in packs.SHORT_BLOCKS if c[0] is packs.HALF_GEOMETRY]
    for cases, in_arguments in ((long_lists, False), (short_lists, True)):
        for case, names in zip(cases, launched(stand_in, cases)):
            names = [k for k in names if k[0] in HALVES]
            assert len(names) == 3
            for name, args in names:
                assert args[3] and args[-1] == in_arguments, (case, name, args)


def test_every_attention_kernel_is_compared_with_the_oracle(stand_in):
    """The packs of the GPU tests, those named in dispatch_packs and those of teams and shares, reach every instance of the attention
    kernels that the library holds."""
    import test_head_pieces
    import test_teams
    from test_gpu_split_items import MANY_SHORT
    cases = [c[:4] for c in packs.PACKED + packs.PERSISTENT_PACKS] + [(packs.GEOMETRY, *c[:3]) for c in packs.BLOCKS]
    cases += packs.HALF_LONG_PACKS + packs.HALF_LONG_BLOCKS + packs.SHORT_PACKS + packs.SHORT_BLOCKS + [(MANY_SHORT, 16, 8, 104)]
    cases += [c[:4] for c in test_head_pieces.PACKS + test_teams.PACKS]
    seen = {k for names in launched(stand_in, cases) for k in names}
    program = """
name, names = ctypes.c_char_p(), []
for i in range(fake.fake_kernels(0, ctypes.byref(name))):
    fake.fake_kernels(i, ctypes.byref(name))
    names.append(name.value.decode())
out(names)
"""
    held = {rec.kernel(n) for n in rec.record(stand_in, program)[0]}
    attention = {k for k in held if k[0] in HALVES or k[0] == "bwd_piece_sums_kernel"}
    assert len(attention) > 100 and all(sum(mark in k[1] for k in attention) > 10 for mark in ("TwoTeams", "HeadPieces"))
    assert not attention - seen, sorted(attention - seen)


def test_packs_of_shares_launch_the_form_that_they_declare(stand_in):
    """Whole and half shares, at either tile width, with the list in the arguments and on the device."""
    from test_head_pieces import ORDINARY, PACKS
    forms = {1: set(), 2: set()}   # of single heads, of groups
    for (lengths, hq, hkv, d, halves), names in zip(PACKS, launched(stand_in, [c[:4] for c in PACKS])):
        in_arguments = names[-1][1][-1]
        width = 64 if d <= 64 else 128
        assert names[-2:] == [("bwd_dkv_kernel", (width, False, _steps(d), bool(halves), False, False, "HeadPieces", in_arguments)),
                              ("bwd_piece_sums_kernel", (in_arguments,))], (lengths, d)
        forms[1 if hq == hkv else 2].add((width, halves, in_arguments))
    assert {(w, 0, a) for w in (64, 128) for a in (False, True)} <= forms[1] and {(w, 1, True) for w in (64, 128)} <= forms[1]
    assert {(w, h, False) for w in (64, 128) for h in (0, 1)} <= forms[2] and (128, 1, True) in forms[2]
    ordinary = [c for c in ORDINARY if c[0]]
    for case, names in zip(ordinary, launched(stand_in, ordinary)):
        assert names[-1][0] == "bwd_dkv_kernel" and "HeadPieces" not in names[-1][1], case


def test_static_workspace_takes_the_same_kernels(stand_in):
    """The entry point without a workspace launches what the one with a workspace launches, also where the sums of items that are dealt
    out are more than the statistics leave of the array."""
    from test_head_pieces import ORDINARY, PACKS
    cases = [c[:4] for c in PACKS + ORDINARY if c[0]] + [([3000, 500], 8, 2, 128), ([700, 45, 260, 1, 129, 1500], 8, 2, 128),
                                                         ([12000] + [128] * 150, 8, 1, 128), ([29082, 18500], 8, 2, 128)]
    program = """
for pack, hq, hkv, d in args[0]:
    plan = Plan(pack, hq, hkv, d)
    calls(); plan.backward(); both = calls(); plan.backward_static()
    out([[c for c in x if c[0] == "launch"] for x in (both, calls())])
"""
    for case, (with_workspace, without) in zip(cases, rec.record(stand_in, program, cases)):
        assert with_workspace == without, case


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (8, 1, 64), (4, 4, 104), (32, 8, 128), (24, 24, 128), (15, 15, 64), (6, 3, 80), (1, 1, 128)])
def test_one_workspace_serves_every_pack_of_a_plan(stand_in, hq, hkv, d):
    """Its size follows from the number of tokens, is never less for more of them, and is enough for what any pack launches."""
    import random
    rng = random.Random(hq + hkv)
    packs_of = {}
    for tokens in (1, 192, 449, 700, 2048, 4096, 20000, 65536):
        for mean in (tokens, 40, 300, 2000):
            lengths = []
            while sum(lengths) < tokens:
                lengths.append(min(1 + int(rng.expovariate(1 / mean)) if mean < tokens else tokens, tokens - sum(lengths)))
            packs_of.setdefault(tokens, []).append(lengths)
    program = """
packs, hq, hkv, d = args
plan = None
for lengths in packs:
    plan = plan or Plan(lengths, hq, hkv, d)
    plan.update(lengths)
    calls(); plan.backward(); own = calls(); plan.backward(1 << 40)
    launches = [[c for c in x if c[0] == "launch"] for x in (own, calls())]
    out([lib.hspmd_attn_bwd_workspace_bytes(plan.h), *launches])
"""
    found = rec.record(stand_in, program, [p for group in packs_of.values() for p in group], hq, hkv, d)
    sizes = []
    for tokens, group in packs_of.items():
        of_tokens, found = found[:len(group)], found[len(group):]
        assert len({size for size, *_ in of_tokens}) == 1, (tokens, [size for size, *_ in of_tokens])
        assert all(own == with_any for _, own, with_any in of_tokens), tokens
        sizes.append(of_tokens[0][0])
    assert sizes == sorted(sizes) and sizes[-1] <= 8 * hq * 65536 + 320 + (64 << 20)


@pytest.mark.parametrize("long,short,count,hq,hkv,d", [(16000, 33, 1000, 4, 2, 128), (9000, 100, 578, 8, 1, 128), (5000, 1, 3000, 32, 4, 64)])
def test_sums_are_looked_for_among_the_items_that_have_some(stand_in, long, short, count, hq, hkv, d):
    """Few of a long list's items are dealt out: those of the long sequence."""
    program = """
pack, hq, hkv, d = args
plan = Plan(pack, hq, hkv, d)
calls(); plan.backward(); out([c for c in calls() if c[0] == "launch"])
"""
    (found,) = rec.record(stand_in, program, [long] + [short] * count, hq, hkv, d)
    _, name, workgroups = found[-1]
    assert rec.kernel(name)[0] == "bwd_piece_sums_kernel" and 0 < workgroups <= 8 * hkv * -(-long // 128)


@pytest.mark.parametrize("lengths,hq,hkv,d", [
    ([3596], 16, 8, 128), ([2893, 2545], 10, 5, 80), ([3524], 16, 8, 96), ([2332], 27, 9, 128), ([1585, 482, 970], 20, 10, 104), ([3100], 16, 8, 128),
    ([7158, 1551, 3781, 1094], 40, 5, 128), ([6735, 5618, 13278], 21, 3, 128), ([13846], 4, 2, 128), ([5113, 5915, 5569, 7671], 24, 3, 104),
    ([1331, 426, 176, 433, 682, 390, 246, 77, 677, 287, 413, 341, 436, 509, 595, 487, 1391], 21, 3, 128)])
def test_items_stay_whole_where_shares_would_take_longer(stand_in, lengths, hq, hkv, d):
    program = """
pack, hq, hkv, d = args
plan = Plan(pack, hq, hkv, d)
calls(); plan.backward(); out([c[1] for c in calls() if c[0] == "launch"])
"""
    (names,) = rec.record(stand_in, program, lengths, hq, hkv, d)
    name, arguments = rec.kernel(names[-1])
    assert name == "bwd_dkv_kernel" and "HeadPieces" not in arguments


@pytest.mark.parametrize("lengths,heads,d,fwd,dq", [
    # lists without padding: (forward, dQ) of two teams
    ([2835], 8, 64, False, False), ([3582], 8, 64, False, False), ([3281, 344, 534], 8, 64, False, False), ([4800], 8, 64, False, False),
    ([233, 918, 6919, 480, 837, 1553, 1293, 549], 8, 128, False, False), ([415, 2508, 656, 7878], 8, 104, False, False),
    ([4096], 8, 128, False, False), ([5900], 8, 64, True, False), ([6850], 8, 128, True, False), ([16001], 5, 128, True, True)])
def test_items_keep_one_team_where_two_would_take_longer(stand_in, lengths, heads, d, fwd, dq):
    program = """
pack, h, d = args
plan = Plan(pack, h, h, d)
calls(); plan.forward(); plan.backward(); out([c[1] for c in calls() if c[0] == "launch"])
"""
    (names,) = rec.record(stand_in, program, lengths, heads, d)
    kernels = [rec.kernel(n) for n in names[:2]]
    assert [name for name, _ in kernels] == ["fwd_kernel", "bwd_dq_kernel"]
    assert ["TwoTeams" in arguments for _, arguments in kernels] == [fwd, dq]
