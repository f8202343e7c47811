"""Host-side properties of hspmd_attn_estimate_ms (the prediction's accuracy is a GPU test)."""
import numpy as np
import pytest

import paper_2504_20490_amd as A


def _cu(lengths):
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)


def test_empty_pack_costs_nothing():
    assert A.estimate_ms([0], 4, 2, 128) == (0.0, 0.0)
    assert A.estimate_ms([0, 0, 0], 4, 2, 64) == (0.0, 0.0)


def test_longer_and_more_sequences_cost_more():
    prev = (0.0, 0.0)
    for L in (256, 1024, 4096, 16384):
        cur = A.estimate_ms(_cu([L] * 4), 16, 16, 128)
        assert cur[0] > prev[0] and cur[1] > prev[1]
        prev = cur
    a = A.estimate_ms(_cu([4096] * 4), 16, 16, 128)
    b = A.estimate_ms(_cu([4096] * 8), 16, 16, 128)
    assert b[0] > a[0] and b[1] > a[1]


def test_quadratic_in_length_and_linear_in_heads_for_large_packs():
    """Large packs are dominated by the step term: one 32k sequence costs about 4x one 16k sequence, and twice the
    heads about twice the time; backward is between 2x and 4x forward."""
    f16, b16 = A.estimate_ms(_cu([16384]), 32, 32, 128)
    f32, b32 = A.estimate_ms(_cu([32768]), 32, 32, 128)
    assert 3.5 < f32 / f16 < 4.2 and 3.5 < b32 / b16 < 4.2
    fh, bh = A.estimate_ms(_cu([16384]), 64, 64, 128)
    assert 1.8 < fh / f16 < 2.1 and 1.8 < bh / b16 < 2.1
    assert 2.0 < b16 / f16 < 4.0


def test_head_dim_64_is_cheaper():
    f128, b128 = A.estimate_ms(_cu([3000, 500, 9000]), 16, 8, 128)
    f64, b64 = A.estimate_ms(_cu([3000, 500, 9000]), 16, 8, 64)
    assert f64 < f128 and b64 < b128


def test_validation():
    with pytest.raises(A.HspmdError):
        A.estimate_ms([0, 10], 3, 2, 128)
    with pytest.raises(A.HspmdError):
        A.estimate_ms([0, 10], 2, 2, 100)
    with pytest.raises(A.HspmdError):
        A.estimate_ms([0, 10, 5], 2, 2, 128)


@pytest.mark.parametrize("lengths,hq,hkv", [([64] * 1000, 32, 4), ([2048] * 16, 32, 32)])
def test_an_estimate_costs_little_more_than_the_two_work_lists(lengths, hq, hkv):
    """The shortest of many runs of either, through the C ABI: each list is built once."""
    import ctypes
    import time
    lib, offsets = ctypes.CDLL(A.library_path()), _cu(lengths)
    cu, items, count, ms = (ctypes.c_int32 * len(offsets))(*offsets), (ctypes.c_int32 * (4 << 18))(), ctypes.c_int64(), (ctypes.c_double * 2)()

    def lists():
        for kind in (A.LIST_FWD, A.LIST_DKV):
            assert lib.hspmd_attn_schedule(kind, cu, len(lengths), hq, hkv, 8, items, ctypes.c_int64(1 << 18), ctypes.byref(count)) == 0

    def estimate():
        assert lib.hspmd_attn_estimate_ms(cu, len(lengths), hq, hkv, 128, ms, ctypes.byref(ms, 8)) == 0

    def shortest(call):
        times = []
        for _ in range(40):
            start = time.perf_counter()
            call()
            times.append(time.perf_counter() - start)
        return min(times)
    # (1.3 to 1.5; building the forward's list once per pass and once more for the dK/dV pass 2.6 to 3)
    assert shortest(estimate) < 2.0 * shortest(lists)


def test_refit_knows_the_forms_of_the_passes():
    """Given the library's own predictions for measurements, the refit finds a model that gives them back: its features and formula are
    the library's, passes of two teams and dealt-out items among them."""
    import tempfile
    from paper_2504_20490_amd import fit_cost_model as fit
    packs = list(fit._packs(np.random.default_rng(7))) + list(fit._small_packs(np.random.default_rng(11)))
    rows = []
    for d in (64, 104, 128):
        for lengths, hq, hkv in packs:
            forward, _ = A.estimate_ms(_cu(lengths), hq, hkv, d)
            rows.append((lengths, hq, hkv, d, {name: forward * 1e3 for name in fit.PASSES}))
    with tempfile.TemporaryDirectory() as folder:
        scheduler = fit._scheduler(folder)
        features = np.stack([fit._features(scheduler, lengths, hq, hkv, d) for lengths, hq, hkv, d, _ in rows])
    forward, dkv = fit._Passes(0, features, rows), fit._Passes(2, features, rows)
    assert min((forward.teams == 2).sum(), (dkv.areas > 0).sum(), forward.plain.sum()) > 20
    *_, errors = fit._fit(0, forward)
    assert errors.max() < 1e-3
    # the dK/dV pass from coefficients of its kind: the sums' cost is found again
    table = np.tile([1.6, 13.0, 1.1], (len(fit.WIDTHS), 1))
    shares = np.where(dkv.halves[:, None], [0.52, 0.70, 0.84], 1.0)
    dkv.measured = dkv.time(0.0, table, shares) + np.where(dkv.areas > 0, 5.0 + 0.03 * dkv.areas, 0.0)
    *_, sums, errors = fit._fit(2, dkv)
    assert errors.max() < 0.02 and abs(sums[0] - 5.0) < 0.5 and abs(sums[1] - 0.03) < 0.005
