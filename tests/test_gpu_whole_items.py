"""Parity of the kernels that large packs run: whole items in every pass, persistent dK/dV workgroups on items long enough for
every loop, packed and block plans, at every width that has kernels of its own.  The packs are small enough for the oracle and
chosen for the form of their passes, which `test_dispatch.py` checks on the CPU."""
import numpy as np
import pytest

import dispatch_packs as packs
import gpu_util
import oracle
from gpu_util import GpuRun, LSE_ABS, assert_close, default_scale, f64, magnitude_bound, make_case
from oracle import rope as orope
from test_gpu_block import _check_single_block
from test_gpu_parity import _full_check
from test_gpu_rope import BASE, _bwd_rope, _table

pytestmark = pytest.mark.gpu


def _assert_turned_back(name, got, plain, positions):
    """The rotary epilogue alone: the plain pass's fp32 gradients, turned back in fp64, differ by fp32 rounding only."""
    want = orope.rope_transposed(plain, positions, BASE)
    assert np.max(np.abs(got - want)) <= 2e-6 * max(1.0, float(np.max(np.abs(want)))), name


def _check_other_stores(run, lengths):
    """The remaining epilogues on the same pack, against its fp32 gradients: bf16 gradients are those rounded once, rotated
    ones those turned back."""
    import torch
    A = run.A
    plain = {n: getattr(run, n).clone() for n in ("dq", "dk", "dv")}
    run.dq, run.dk, run.dv = (torch.full_like(plain[n], float("nan"), dtype=torch.bfloat16) for n in ("dq", "dk", "dv"))
    run.grad_dtype = A.GRAD_BF16
    run.backward()
    torch.cuda.synchronize()
    for n in plain:
        assert torch.equal(getattr(run, n), plain[n].to(torch.bfloat16)), n
    run.dq, run.dk, run.dv = (torch.full_like(plain[n], float("nan")) for n in ("dq", "dk", "dv"))
    d = plain["dq"].shape[2]
    _bwd_rope(run, _table(max(lengths), d), max(lengths), A.GRAD_F32)
    pos = orope.positions_of(lengths)
    for n in ("dq", "dk"):
        _assert_turned_back(n, run.host(n), plain[n].cpu().numpy().astype(np.float64), pos)
    assert torch.equal(run.dv, plain["dv"])


@pytest.mark.parametrize("lengths,hq,hkv,d,rows,dkv", packs.PACKED)
def test_packed_whole_items(lengths, hq, hkv, d, rows, dkv):
    run = _full_check(lengths, hq, hkv, d, seed=1100 + d + hq, magnitude_slack=True)
    _check_other_stores(run, lengths)


@pytest.mark.parametrize("lengths,hq,hkv,d,rows,dkv", packs.PERSISTENT_PACKS)
def test_persistent_dkv_pass_on_long_items(lengths, hq, hkv, d, rows, dkv):
    """Sampled rows and keys, the first and last of every sequence among them."""
    gpu_util.CONTEXT["case"] = f"persistent d{d}"
    q, k, v, do = make_case(lengths, hq, hkv, d, seed=1200 + d)
    run = GpuRun(lengths, q, k, v, do).run()
    s = default_scale(d)
    ends = np.cumsum(lengths)
    rng = np.random.default_rng(d)
    rows = np.unique(np.concatenate([rng.integers(0, ends[-1], 24), ends - 1, ends[:-1], [0]])).astype(np.int32)
    heads, kvh = rng.integers(0, hq, len(rows)).astype(np.int32), rng.integers(0, hkv, len(rows)).astype(np.int32)
    ro, rlse, rdq = oracle.attn_rows(f64(q), f64(k), f64(v), f64(do), lengths, s, rows, heads)
    rdk, rdv = oracle.attn_keys(f64(q), f64(k), f64(v), f64(do), lengths, s, rows, kvh)
    assert np.max(np.abs(run.host("lse")[heads, rows] - rlse)) <= LSE_ABS
    for name, got, ref in (("O rows", run.host("o")[rows, heads], ro), ("dQ rows", run.host("dq")[rows, heads], rdq),
                           ("dK keys", run.host("dk")[rows, kvh], rdk), ("dV keys", run.host("dv")[rows, kvh], rdv)):
        assert_close(name, got, ref, max_abs=magnitude_bound(ref))
    gpu_util.CONTEXT["slack"] = None
    for n in ("o", "dq", "dk", "dv"):
        assert not np.isnan(run.host(n)).any(), n
    _check_other_stores(run, lengths)


@pytest.mark.parametrize("hq,hkv,d,rows,dkv", packs.BLOCKS)
def test_block_whole_items(hq, hkv, d, rows, dkv):
    import torch
    ql, kl, qp, kp = packs.GEOMETRY
    r, _, (o_dev, lse_dev) = _check_single_block(ql, kl, qp, kp, hq, hkv, d, 1300 + d, f"block_whole_d{d}", magnitude_slack=True)
    A = r.A
    # accumulation into dQ and statistics from the workspace: dQ doubles, dK and dV are rewritten as they were
    plain = {n: getattr(r, n).clone() for n in ("dq", "dk", "dv")}
    r.dk.fill_(float("nan")), r.dv.fill_(float("nan"))
    A.attn_block_bwd(r.plan, r.q, r.k, r.v, None, None, r.do, r.dq, r.dk, r.dv, r.ws, dq_accumulate=True, reuse_statistics=True)
    torch.cuda.synchronize()
    assert torch.equal(r.dq, 2 * plain["dq"]) and torch.equal(r.dk, plain["dk"]) and torch.equal(r.dv, plain["dv"])
    # the rotary epilogue, written and accumulated
    positions = max(max(p + n for p, n in zip(qp, ql)), max(p + n for p, n in zip(kp, kl)))
    pos_q, pos_k = (np.concatenate([p + np.arange(n) for p, n in zip(ps, ns)]).astype(np.int64) for ps, ns in ((qp, ql), (kp, kl)))
    host = {n: t.cpu().numpy().astype(np.float64) for n, t in plain.items()}
    for accumulate in (False, True):
        for n in ("dk", "dv") if accumulate else ("dq", "dk", "dv"):
            getattr(r, n).fill_(float("nan"))
        A.attn_block_bwd_rope(r.plan, r.q, r.k, r.v, o_dev, lse_dev, r.do, r.dq, r.dk, r.dv, r.ws, _table(positions, d), positions,
                              dq_accumulate=accumulate)
        torch.cuda.synchronize()
        _assert_turned_back("dq", r.host("dq"), (2 if accumulate else 1) * host["dq"], pos_q)
        _assert_turned_back("dk", r.host("dk"), host["dk"], pos_k)
        assert torch.equal(r.dv, plain["dv"])
