"""Copies, reads and barriers of the forward's tile loop, walked on the host from the kernel's own index arithmetic.

A K or V tile lives in one of two LDS buffers.  Between the last read of a buffer's old tile, by any wave, and the first copy
onto it, by any wave, there must be a workgroup barrier, and one between a tile's copies and its reads.  The waves of a
workgroup have different tile ranges on the diagonal, so what one wave skips another may still be doing."""
import ctypes
import os
import random
import subprocess

import pytest

from paper_2504_20490_amd import build as lib_build

SHIM = """
#include "fwd_tiles.hpp"
extern "C" void tiles(int split, int lq, int l, int off, int q_row0, int row_block, int key_block, int* out) {
    const hspmd::FwdTiles t = hspmd::fwd_tiles(split != 0, lq, l, off, q_row0, row_block, key_block);
    out[0] = t.n_tiles; out[1] = t.n_tiles_w; out[2] = t.n_plain; out[3] = t.n_spread; out[4] = t.reuses_first_k();
}
"""
BK = 64


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("fwd_tiles")
    src, so = tmp / "shim.cpp", tmp / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", lib_build.CSRC, "-o", str(so), str(src)], check=True)
    lib = ctypes.CDLL(str(so))

    def call(*args):
        out = (ctypes.c_int * 5)()
        lib.tiles(*args, out)
        return tuple(out)
    return call


def _walk(t, issue, read):
    """One wave's way through an item (the loops of fwd_kernel); an epoch is what lies between two barriers."""
    n_tiles, n_tiles_w, _, n_spread, reuses_first_k = t
    epoch = 0
    issue("K", 0, epoch), issue("V", 0, epoch)
    if n_tiles > 1:
        issue("K", 1, epoch)
    epoch += 1
    if n_tiles_w > 0:
        read("K", 0, epoch)
    if reuses_first_k:
        epoch += 1
    for kt in range(n_tiles):
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
    issues, reads, ends, plans = {}, {}, [], []
    for wave in range(4):
        t = tiles(split, lq, l, off, q_row0, wave & 1 if split else wave, wave >> 1 if split else 0)
        where = (split, lq, l, off, q_row0, wave, t)
        plans.append(t)
        if t[0] == 0:
            continue
        assert t[3] <= max(t[2], 0) and t[2] < max(t[1], 1) and t[1] <= t[0], where
        # copies from inside an iteration have no bounds check: K(kt+2) and V(kt+1) are whole tiles
        assert t[3] == 0 or (t[3] + 2) * BK <= l, where
        ends.append(_walk(t, lambda x, n, e, w=wave: issues.setdefault((x, n), []).append((w, e)),
                          lambda x, n, e, w=wave: reads.setdefault((x, n), []).append((w, e))))
    assert len({(t[0], t[4]) for t in plans}) == 1 and len(set(ends)) <= 1, (split, lq, l, off, q_row0, plans)
    for (x, n), copied in issues.items():
        where = (split, lq, l, off, q_row0, x, n, plans)
        first, last = min(e for _, e in copied), max(e for _, e in copied)
        for _, e in reads.get((x, n), []):
            assert e > last, ("read before the barrier that publishes the tile", where)
        for _, e in reads.get((x, n - 2), []):
            assert e < first, ("copy onto a tile that another wave may still read", where)
        assert n < plans[0][0] and sorted(w for w, _ in copied) == [0, 1, 2, 3], ("a copy that not every wave shares", where)
    assert set(reads) <= set(issues)


@pytest.mark.parametrize("split", [0, 1])
def test_packed_items(tiles, split):
    rows = 64 if split else 128
    for l in [*range(1, 460), 511, 512, 513, 640, 1023, 1025, 2048, 4111]:
        for q_row0 in range(0, l, rows):
            _check_item(tiles, split, l, l, 0, q_row0)


@pytest.mark.parametrize("split", [0, 1])
def test_block_items(tiles, split):
    rng = random.Random(5)
    rows = 64 if split else 128
    for _ in range(1500):
        lq, l = rng.randint(1, 420), rng.randint(1, 700)
        off = rng.choice([0, 1, l - lq, l, rng.randint(-lq - 5, 800), rng.choice([64, 128, 192]) - rng.randint(0, 2)])
        for q_row0 in range(0, lq, rows):
            _check_item(tiles, split, lq, l, off, q_row0)
