"""Refit the coefficients of hspmd_attn_estimate_ms on the GPU at hand.

Runs forward + backward of a set of synthetic packs (uniform and log-normal length mixes, one to forty heads, with and without
groups) at every width that has kernels of its own, with per-kernel event timing, takes the features that the model uses --
inner steps and items of the eight XCD queues, the heaviest item, whole or half items -- from the host scheduler, and fits
all widths of a pass together by relative least squares.  Prints the tables that go into csrc/schedule.cpp.

    python -m paper_2504_20490_amd.fit_cost_model [--head-dim 64 96 ...]
"""
from __future__ import annotations

import argparse

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


class _Features:
    """What the model knows of one pass over one pack (all eight queues)."""

    def __init__(self, A, kind, lengths, hq, hkv, head_dim):
        cu = np.concatenate([[0], np.cumsum(lengths)])
        items = A.schedule(kind, cu, hq, hkv)
        length, tile = items[:, 1].astype(np.int64), items[:, 2].astype(np.int64)
        real = tile >= 0
        rows = A.tile_rows(kind)
        if kind == A.LIST_DKV:
            steps = np.where(real, -(-(length - tile * rows) // 64) * (hq // hkv), 0)
        else:
            steps = np.where(real, -(-np.minimum(length, (tile + 1) * rows) // 64), 0)
        # the scheduler's own rules (pass_dispatch in csrc/schedule.cpp)
        heaviest, total, n, narrow = float(steps.max()), float(steps.sum()), len(items), head_dim <= 64
        if kind == A.LIST_DKV:
            full = 1.6 if narrow else 1.3
            whole = max(heaviest + 8, (total + 8 * n) / (512 if narrow else 256))
            tail = 0.25 * (0.5 * full * total / n + 8) if 2 * n > 256 else 0.0
            self.halves = max(0.68 * heaviest + 8, (full * total + 16 * n) / 256 + tail) < 0.9 * whole
            per_unit = 2 if narrow and not self.halves else 1
        else:
            if kind == A.LIST_FWD:
                least = max(5, (6 if narrow else 5) + 0.08 * (n - 96))
            else:
                least = 8 + 0.05 * (n - 128) if n > 128 else 2
            self.halves = heaviest + 6 >= 2 * (total + 12 * n) / 512 and heaviest >= least
            per_unit = 3 if narrow and kind == A.LIST_DQ else 2
        self.slots = 32.0 * per_unit
        self.queue_steps = np.array([steps[x::8].sum() for x in range(8)], dtype=float)
        self.queue_items = np.array([real[x::8].sum() for x in range(8)], dtype=float)
        self.heaviest = heaviest


def _fit(A, rows, kind):
    """rows: (lengths, q heads, kv heads, head_dim, {kernel: microseconds}).  Returns (launch_us, halves[3], table[width][3],
    relative errors)."""
    from scipy.optimize import least_squares
    f = [_Features(A, kind, lens, hq, hkv, d) for lens, hq, hkv, d, _ in rows]
    y = np.array([t[PASSES[kind]] for *_, t in rows])
    width = np.array([WIDTHS[d] for *_, d, _ in rows])
    S, N = np.stack([x.queue_steps for x in f]), np.stack([x.queue_items for x in f])
    H, slots, halves = (np.array([getattr(x, name) for x in f]) for name in ("heaviest", "slots", "halves"))

    def model(p):
        p = np.abs(p)
        half_step, half_alone, half_item = (np.where(halves, x, 1.0) for x in p[1:4])
        step, item, alone = p[4:].reshape(-1, 3)[width].T
        two = np.where(halves, 2.0, 1.0)
        load = ((S * (two * half_step * step)[:, None] + N * (two * half_item * item)[:, None]).max(axis=1)) / slots
        single = H * half_alone * alone + half_item * item
        return p[0] + (load ** 4 + single ** 4) ** 0.25

    start = np.concatenate([[8.0, 0.6, 0.65, 0.7], np.tile([1.6, 8.0, 1.2], len(WIDTHS))])
    found = least_squares(lambda p: model(p) / y - 1.0, start, loss="soft_l1", f_scale=0.1, max_nfev=4000)
    p = np.abs(found.x)
    return p[0], p[1:4], p[4:].reshape(-1, 3), np.abs(model(found.x) / y - 1.0)


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
    for kind, name in enumerate(PASSES):
        launch, halves, table, err = _fit(A, rows, kind)
        print(f"// {name}: mean |error| {err.mean():.3f}, 95 % below {np.quantile(err, 0.95):.2f}, max {err.max():.2f}")
        print(f"{{{launch:.1f}, {{{', '.join(f'{x:.2f}' for x in halves)}}}}},")
        print("{" + ", ".join(f"{{{s:.3f}, {i:.2f}, {a:.3f}}}" for s, i, a in table) + "},")
    return 0


if __name__ == "__main__":
    raise SystemExit(main())
