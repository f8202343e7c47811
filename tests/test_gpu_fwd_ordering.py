"""The forward's item loop: its buffers and its slot hand-over must not depend on how far the waves of a workgroup run apart."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [128, 64])
def test_last_tiles_with_one_wave_of_rows_are_bit_identical_from_run_to_run(d):
    """Sequences of 257 .. 288 tokens end in a tile of five key tiles in which three of four waves own no row: those waves
    skip the first product and reach the copy of the third K tile long before the first wave has read the tile it lands on.
    Their first tile, of two key tiles, is the case in which no wave may copy a third at all (test_fwd_tile_order.py).
    Which items suffer is chance, so the pack holds hundreds of them and runs many times; every run must give the same bits."""
    import torch
    import paper_2504_20490_amd as A
    lengths = [257 + (i * 7) % 32 for i in range(48)]
    hq, hkv = 32, 8
    T = sum(lengths)
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(T, h, d, generator=gen, device="cuda").to(torch.bfloat16) for h in (hq, hkv, hkv))
    plan = A.Plan(A.build_cu_seqlens(lengths)[0], hq, hkv, d)
    first = None
    for _ in range(40):
        o = torch.full((T, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((hq, T), float("nan"), dtype=torch.float32, device="cuda")
        A.attn_varlen_fwd(plan, q, k, v, o, lse)
        torch.cuda.synchronize()
        if first is None:
            first = (o, lse)
            assert not torch.isnan(o).any() and not torch.isnan(lse).any()
        else:
            assert torch.equal(o.view(torch.int16), first[0].view(torch.int16)) and torch.equal(lse, first[1])


def test_items_without_a_visible_key_in_a_row():
    """A block wholly in the future: every item of the persistent loop only writes zeros and draws its successor, without
    any barrier of a tile loop in between."""
    import torch
    import paper_2504_20490_amd as A
    lengths = [700, 1, 129, 64, 3000, 255] * 4
    hq, hkv, d = 12, 4, 128
    T = sum(lengths)
    cu = np.concatenate([[0], np.cumsum(lengths)])
    gen = torch.Generator(device="cuda").manual_seed(4)
    q, k, v = (torch.randn(T, h, d, generator=gen, device="cuda").to(torch.bfloat16) for h in (hq, hkv, hkv))
    plan = A.BlockPlan(cu, cu, [0] * len(lengths), [4096] * len(lengths), hq, hkv, d)
    for _ in range(5):
        o = torch.full((T, hq, d), float("nan"), device="cuda")
        lse = torch.full((hq, T), float("nan"), device="cuda")
        A.attn_block_fwd(plan, q, k, v, o, lse)
        torch.cuda.synchronize()
        assert bool((o == 0).all()) and bool((lse == -float("inf")).all())
