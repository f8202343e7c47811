"""Refit the coefficients of hspmd_attn_estimate_ms on the GPU at hand.

Runs forward + backward of a set of synthetic packs (uniform and log-normal length mixes, one to forty heads, with and without
groups) at every width that has kernels of its own, with per-kernel event timing, takes what the model knows of a pass (PassFeatures in
csrc/schedule.hpp: its form, the inner steps and items of the eight XCD queues, the heaviest item) from the scheduler's own sources, and
fits all widths of a pass together by relative least squares: first the passes that one team of waves takes item by item, then, with those
coefficients kept, the shares of the passes that two teams take and what the sums of dealt-out dK/dV items cost.  Prints the tables that
go into csrc/schedule.cpp, and how far the model that the library holds is from the same measurements.

    python -m paper_2504_20490_amd.fit_cost_model [--head-dim 64 96 ...]
"""
from __future__ import annotations

import argparse
import ctypes
import os
import subprocess
import tempfile

import numpy as np

WIDTHS = {64: 0, 80: 1, 96: 2, 104: 3, 128: 4}      # a head_dim of every width class, in the order of the tables
PASSES = ["fwd_kernel", "bwd_dq_kernel", "bwd_dkv_kernel"]   # in the order of the list kinds


def _packs(rng):
    for hq, hkv in [(16, 16), (32, 8), (8, 8), (40, 40)]:
        for length, count in [(512, 32), (1024, 16), (4096, 4), (16384, 1), (256, 64), (8192, 4), (128, 256)]:
            yield [length] * count, hq, hkv
    for _ in range(12):
        n = int(rng.integers(2, 30))
        lens = [int(x) for x in np.clip(np.exp(rng.normal(7.0, 1.2, n)), 16, 20000)]
        yield lens, int(rng.choice([8, 16, 24, 32])), 8


def _small_packs(rng):
    """Packs of which one item takes a large part of a pass: few sequences, few heads, large groups."""
    for hq, hkv in [(1, 1), (2, 2), (5, 5), (8, 2), (32, 8), (40, 40)]:
        for lens in ([16384], [24000], [2048], [512] * 3, [300] * 12, [1024] * 6, [1500, 400, 153], [4000, 300, 200, 90],
                     [6000, 1000, 500] * 2):
            yield list(lens), hq, hkv
    for _ in range(30):
        n = int(rng.integers(1, 20))
        lens = [int(x) for x in np.clip(np.exp(rng.normal(rng.uniform(4.5, 7.5), 1.0, n)), 16, 16384)]
        hkv = int(rng.choice([1, 2, 3, 4, 8]))
        yield lens, hkv * int(rng.choice([1, 1, 2, 4])), hkv


def _measure(A, torch, lengths, hq, hkv, d):
    T = sum(lengths)
    g = torch.Generator(device="cuda")
    g.manual_seed(0)
    mk = lambda h: torch.randn(T, h, d, device="cuda", generator=g).to(torch.bfloat16)
    q, k, v, do = mk(hq), mk(hkv), mk(hkv), mk(hq)
    o = torch.empty_like(q)
    lse = torch.empty(hq, T, dtype=torch.float32, device="cuda")
    dq = torch.empty(T, hq, d, dtype=torch.float32, device="cuda")
    dk = torch.empty(T, hkv, d, dtype=torch.float32, device="cuda")
    dv = torch.empty_like(dk)
    cu, _, _ = A.build_cu_seqlens(lengths)
    plan = A.Plan(cu, hq, hkv, d)
    ws = torch.empty(plan.bwd_workspace_bytes(), dtype=torch.uint8, device="cuda")

    def step():
        A.attn_varlen_fwd(plan, q, k, v, o, lse)
        A.attn_varlen_bwd(plan, q, k, v, o, lse, do, dq, dk, dv, ws, grad_dtype=A.GRAD_F32)

    for _ in range(3):
        step()
    torch.cuda.synchronize()
    A.profile_enable(True)
    for _ in range(8):
        step()
    torch.cuda.synchronize()
    A.profile_enable(False)
    return {name: ms / n * 1e3 for name, (ms, n) in A.profile_read().items()}   # microseconds


# what a plan's passes are to the model, asked of the scheduler itself
_SHIM = """
#include "schedule.hpp"
extern "C" void features(const int* cu, int n, int hq, int hkv, int head_dim, double* out) {
    hspmd::PassFeatures f[3];
    hspmd::pack_features(cu, n, hq, hkv, head_dim, f);
    for (const hspmd::PassFeatures& x : f) {
        *out++ = x.halves, *out++ = x.teams, *out++ = (double)x.areas, *out++ = x.heaviest;
        for (double steps : x.queue_steps) *out++ = steps;
        for (double items : x.queue_items) *out++ = items;
    }
}
"""
_VALUES = 4 + 2 * 8


def _scheduler(folder):
    from paper_2504_20490_amd import build
    source, library = os.path.join(folder, "features.cpp"), os.path.join(folder, "features.so")
    with open(source, "w") as f:
        f.write(_SHIM)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O2", "-shared", "-fPIC", "-I", build.CSRC, "-o", library, source,
                    os.path.join(build.CSRC, "schedule.cpp")], check=True)
    return ctypes.CDLL(library)


def _features(scheduler, lengths, hq, hkv, head_dim):
    """Per pass, in the order of the list kinds: halves, teams, areas, heaviest item, steps and items of each queue."""
    cu = np.ascontiguousarray(np.concatenate([[0], np.cumsum(lengths)]), dtype=np.int32)
    out = np.zeros((3, _VALUES))
    as_ = lambda x, kind: x.ctypes.data_as(ctypes.POINTER(kind))
    scheduler.features(as_(cu, ctypes.c_int), len(lengths), hq, hkv, head_dim, as_(out, ctypes.c_double))
    return out


class _Passes:
    """All measured passes of one kind as arrays; `time` is the model (estimate_pass_us in csrc/schedule.cpp)."""

    def __init__(self, kind, features, rows):
        f = features[:, kind]
        self.halves, self.teams, self.areas, self.heaviest = f[:, 0] > 0, f[:, 1], f[:, 2], f[:, 3]
        self.steps, self.items = f[:, 4:12], f[:, 12:20]
        self.width = np.array([WIDTHS[d] for *_, d, _ in rows])
        narrow = np.array([d <= 64 for *_, d, _ in rows])
        per_unit = np.where(narrow & ~self.halves, 2, 1) if kind == 2 else np.where(narrow & (kind == 1), 3, 2)
        self.slots = 32.0 * per_unit
        self.measured = np.array([t[PASSES[kind]] for *_, t in rows])
        self.plain = (self.teams == 1) & (self.areas == 0)

    def time(self, launch, table, shares):
        """shares: of a whole item's step, step alone and fixed time, one row per pass."""
        step, item, alone = table[self.width].T
        share_step, share_alone, share_item = shares.T
        two = np.where(self.halves, 2.0, 1.0)
        load = (self.steps * (two * share_step * step)[:, None] + self.items * (two * share_item * item)[:, None]).max(axis=1) / self.slots
        single = self.heaviest * share_alone * alone + share_item * item
        return launch + (load ** 4 + single ** 4) ** 0.25


def _least(residual, start):
    from scipy.optimize import least_squares
    return np.abs(least_squares(residual, start, loss="soft_l1", f_scale=0.1, max_nfev=4000).x)


def _fit(kind, passes):
    """(launch_us, halves[3], table[width][3], {(halves): shares[3]} of two teams, (fixed, per area) of the sums, relative errors)."""
    y, halves, plain = passes.measured, passes.halves, passes.plain

    def base(p):
        p = np.abs(p)
        shares = np.where(halves[:, None], p[1:4], 1.0)
        return p[0], p[4:].reshape(-1, 3), shares

    start = np.concatenate([[8.0, 0.6, 0.65, 0.7], np.tile([1.6, 8.0, 1.2], len(WIDTHS))])
    p = _least(lambda p: (passes.time(*base(p)) / y - 1.0)[plain], start)
    launch, table, shares = base(p)
    teams = {}
    for half in (False, True):
        these = (passes.teams == 2) & (halves == half)
        if these.sum() < 10:
            continue
        of = lambda q: np.where(these[:, None], np.abs(q), shares)
        teams[half] = _least(lambda q: (passes.time(launch, table, of(q)) / y - 1.0)[these], np.array([0.9, 0.6, 1.0]))
        shares = of(teams[half])
    time, sums = passes.time(launch, table, shares), None
    dealt = passes.areas > 0
    if dealt.sum() >= 10:
        cost = lambda q: np.where(dealt, abs(q[0]) + abs(q[1]) * passes.areas, 0.0)
        sums = _least(lambda q: ((time + cost(q)) / y - 1.0)[dealt], np.array([5.0, 0.03]))
        time = time + cost(sums)
    return launch, p[1:4], table, teams, sums, np.abs(time / y - 1.0)


def _errors(err):
    return f"mean |error| {err.mean():.3f}, 95 % below {np.quantile(err, 0.95):.2f}, max {err.max():.2f}"


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--head-dim", type=int, nargs="*", default=list(WIDTHS), choices=list(WIDTHS))
    args = ap.parse_args()
    import torch
    import paper_2504_20490_amd as A
    A.load_library()
    packs = list(_packs(np.random.default_rng(7))) + list(_small_packs(np.random.default_rng(11)))
    rows = []
    for d in args.head_dim:
        rows += [(lens, hq, hkv, d, _measure(A, torch, lens, hq, hkv, d)) for lens, hq, hkv in packs]
        print(f"// head_dim {d}: {len(packs)} packs", flush=True)
    with tempfile.TemporaryDirectory() as folder:
        scheduler = _scheduler(folder)
        features = np.stack([_features(scheduler, lens, hq, hkv, d) for lens, hq, hkv, d, _ in rows])
    held = np.array([A.estimate_ms(np.concatenate([[0], np.cumsum(lens)]), hq, hkv, d) for lens, hq, hkv, d, _ in rows]) * 1e3
    measured = np.array([[t[PASSES[0]], t[PASSES[1]] + t[PASSES[2]]] for *_, t in rows])
    for name, err in zip(("forward", "backward"), np.abs(held / measured - 1.0).T):
        print(f"// the library's model, {name}: {_errors(err)}")
    for kind, name in enumerate(PASSES):
        passes = _Passes(kind, features, rows)
        launch, halves, table, teams, sums, err = _fit(kind, passes)
        print(f"// {name}: {_errors(err)}; {passes.plain.sum()} of {len(rows)} passes are the base fit's")
        print(f"{{{launch:.1f}, {', '.join(f'{x:.2f}' for x in halves)}}},")
        print("{" + ", ".join(f"{{{s:.3f}, {i:.2f}, {a:.3f}}}" for s, i, a in table) + "},")
        for half, shares in teams.items():
            print(f"// two teams, {'half' if half else 'whole'} items: {{{', '.join(f'{x:.2f}' for x in shares)}}}")
        if sums is not None:
            print(f"// sums of dealt-out items: {sums[0]:.1f} us and {sums[1]:.3f} each area")
    return 0


if __name__ == "__main__":
    raise SystemExit(main())
