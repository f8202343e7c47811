"""Forward and dQ passes whose items two teams of waves share.

The forward's tile loop, walked on the host as in `test_fwd_tile_order`: a team copies and reads its own buffers, and the barriers
are the whole workgroup's, so every wave of both teams has to pass the same number of them.  The packs that take teams, asked of the
scheduler, and their outputs against the oracle on the GPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import test_fwd_tile_order as one_team
from paper_2504_20490_amd import build as lib_build

SHIM = """
#include "fwd_tiles.hpp"
extern "C" void tiles(int split, int lq, int l, int off, int q_row0, int row_block, int key_block, int team, int* out) {
    const hspmd::FwdTiles t = hspmd::fwd_tiles(split != 0, lq, l, off, q_row0, row_block, key_block, 2, team);
    out[0] = t.n_passes; out[1] = t.n_tiles; out[2] = t.n_tiles_w; out[3] = t.n_plain; out[4] = t.n_spread; out[5] = t.reuses_first_k();
}
"""
BK = one_team.BK


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("team_tiles")
    src, so = tmp / "shim.cpp", tmp / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", lib_build.CSRC, "-o", str(so), str(src)], check=True)
    lib = ctypes.CDLL(str(so))

    def call(*args):
        out = (ctypes.c_int * 6)()
        lib.tiles(*args, out)
        return tuple(out)
    return call


def _walk(t, issue, read):
    n_passes, n_tiles, n_tiles_w, _, n_spread, reuses_first_k = t
    epoch = 0
    if n_tiles > 0:
        issue("K", 0, epoch), issue("V", 0, epoch)
    if n_tiles > 1:
        issue("K", 1, epoch)
    epoch += 1
    if n_tiles_w > 0:
        read("K", 0, epoch)
    if reuses_first_k:
        epoch += 1
    for kt in range(n_passes):
        if kt > 0:
            epoch += 1
        if kt < n_spread or kt + 2 < n_tiles:
            issue("K", kt + 2, epoch)
        if kt < n_spread or kt + 1 < n_tiles:
            issue("V", kt + 1, epoch)
        if kt < n_tiles_w:
            read("V", kt, epoch)
        if kt + 1 < n_tiles_w:
            read("K", kt + 1, epoch)
    return epoch


def _check_item(tiles, split, lq, l, off, q_row0):
    rows = 64 if split else 128
    ends, barriers, item_tiles = set(), set(), max(0, -(-min(l, min(lq, q_row0 + rows) + off) // BK))
    for team in range(2):
        issues, reads, owned = {}, {}, set()
        for wave in range(4):
            row_block, key_block = (wave & 1, wave >> 1) if split else (wave, 0)
            t = tiles(split, lq, l, off, q_row0, row_block, key_block, team)
            where = (split, lq, l, off, q_row0, team, wave, t)
            barriers.add((t[0], t[5]))
            assert t[0] == -(-item_tiles // 2) and t[1] == (item_tiles + 1 - team) // 2, where
            assert t[4] <= max(t[3], 0) and t[3] < max(t[2], 1) and t[2] <= t[1], where
            assert t[4] == 0 or (2 * (t[4] + 1) + team + 1) * BK <= l, where
            # every key that a row of the wave sees lies in a tile that the wave takes, and tiles without a mask hold no other
            first_row, last_row = q_row0 + row_block * 32, min(lq, q_row0 + row_block * 32 + 32) - 1
            for kt in range(t[1]):
                lowest = (2 * kt + team) * BK + key_block * 32
                seen = last_row >= first_row and lowest < l and lowest <= last_row + off
                assert seen == (kt < t[2]), where
                if kt < t[3]:
                    highest = lowest + (31 if split else 63)
                    assert highest <= first_row + off and highest < l, where
            if t[0] == 0:
                continue
            owned.add(t[1])
            ends.add(_walk(t, lambda x, n, e, w=wave: issues.setdefault((x, n), []).append((w, e)),
                           lambda x, n, e, w=wave: reads.setdefault((x, n), []).append((w, e))))
        for (x, n), copied in issues.items():
            first, last = min(e for _, e in copied), max(e for _, e in copied)
            assert all(e > last for _, e in reads.get((x, n), [])), ("read before its barrier", split, lq, l, off, q_row0, team, x, n)
            assert all(e < first for _, e in reads.get((x, n - 2), [])), ("copy onto a tile in use", split, lq, l, off, q_row0, team, x, n)
            assert {n + 1 <= o for o in owned} == {True} and sorted(w for w, _ in copied) == [0, 1, 2, 3]
        assert set(reads) <= set(issues)
    assert len(barriers) == 1 and len(ends) <= 1, (split, lq, l, off, q_row0)


@pytest.mark.parametrize("split", [0, 1])
def test_packed_items(tiles, split):
    for l in [*range(1, 460), 511, 512, 513, 640, 1023, 1025, 2048, 4111]:
        for q_row0 in range(0, l, 64 if split else 128):
            _check_item(tiles, split, l, l, 0, q_row0)


@pytest.mark.parametrize("split", [0, 1])
def test_block_items(tiles, split):
    import random
    rng = random.Random(7)
    for _ in range(1500):
        lq, l = rng.randint(1, 420), rng.randint(1, 700)
        off = rng.choice([0, 1, l - lq, l, rng.randint(-lq - 5, 800), rng.choice([64, 128, 192]) - rng.randint(0, 2)])
        for q_row0 in range(0, lq, 64 if split else 128):
            _check_item(tiles, split, lq, l, off, q_row0)


# (lengths, q heads, kv heads, head_dim, (halves, teams) of the forward, of the dQ pass)
HALF, WHOLE = (1, 2), (0, 2)
LONG, LONG_GROUPS = [3200, 70, 1, 64], [3199, 65]
PACKS = [(LONG, 2, 2, d, HALF, HALF) for d in (40, 64, 80, 96, 104, 128)] + [(LONG_GROUPS, 2, 1, d, HALF, HALF) for d in (64, 128)]
PACKS += [([6465], 10, 10, d, WHOLE, WHOLE) for d in (64, 80, 96, 104, 128)]
# whole items with the list in the arguments
PACKS += [([3000], 7, 7, 64, WHOLE, (1, 1))]

FORM_SHIM = """
#include "schedule.hpp"
using namespace hspmd;
extern "C" int rows(int kind, const int* cu, int n, int hq, int hkv, int d) {
    const auto k = (hspmd_list_kind)kind;
    const int64_t slots = (int64_t)build_work_list(k, cu, n, hq, hkv, kNumXcd).size();
    const RowsForm f = rows_form(k, pass_load(k, cu, n, hq, hkv), slots, hq / hkv, d, slots <= 240);
    return 10 * f.halves + f.teams;
}
extern "C" int slots(const int* cu, int n, int hq, int hkv) { return (int)build_work_list(HSPMD_LIST_FWD, cu, n, hq, hkv, kNumXcd).size(); }
"""


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("team_forms")
    src, so = tmp / "shim.cpp", tmp / "shim.so"
    src.write_text(FORM_SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", lib_build.CSRC, "-o", str(so), str(src),
                    os.path.join(lib_build.CSRC, "schedule.cpp")], check=True)
    lib = ctypes.CDLL(str(so))

    def call(lengths, hq, hkv, d):
        cu = (ctypes.c_int32 * (len(lengths) + 1))(*np.concatenate([[0], np.cumsum(lengths)]).tolist())
        form = tuple(divmod(lib.rows(kind, cu, len(lengths), hq, hkv, d), 10) for kind in range(2))
        return form, lib.slots(cu, len(lengths), hq, hkv)
    return call


@pytest.mark.parametrize("lengths,hq,hkv,d,fwd,dq", PACKS)
def test_packs_take_teams(forms, lengths, hq, hkv, d, fwd, dq):
    assert forms(lengths, hq, hkv, d)[0] == (fwd, dq)


def test_packs_cover_every_kernel(forms):
    """Whole items in device lists, half items in lists in the arguments; at width 64 whole items in those too."""
    reached = set()
    for lengths, hq, hkv, d, *_ in PACKS:
        (fwd, dq), slots = forms(lengths, hq, hkv, d)
        reached |= {(name, max(64, -(-d // 16) * 16), form[0], slots <= 240) for name, form in (("fwd", fwd), ("dq", dq)) if form[1] == 2}
    widths = (64, 80, 96, 104 + 8, 128)
    whole, halves = ({(name, w, h, inline) for name in ("fwd", "dq") for w in widths} for h, inline in ((0, False), (1, True)))
    assert reached == whole | halves | {("fwd", 64, 0, True)}


def test_other_packs_keep_one_team(forms):
    """Short items, more half items than compute units, few rounds of equal items."""
    for lengths, heads, d in (([1024] * 2, 8, 128), ([512], 4, 128), ([2048] * 8, 32, 128), ([8192], 12, 128), ([1024] * 4, 8, 64)):
        assert all(teams == 1 for _, teams in forms(lengths, heads, heads, d)[0]), (lengths, heads, d)


@pytest.mark.gpu
@pytest.mark.parametrize("lengths,hq,hkv,d,fwd,dq", PACKS)
def test_outputs(lengths, hq, hkv, d, fwd, dq):
    import test_gpu_whole_items
    test_gpu_whole_items.test_persistent_dkv_pass_on_long_items(lengths, hq, hkv, d, None, None)
