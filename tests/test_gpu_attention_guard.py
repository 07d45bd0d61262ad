"""Stage 3 (Eq. 3-4) where the scores of some rows rise far above those of the first keys: the per-row shift is
raised in the step that holds them.  The rise sits around the edges of steps (32 keys), tiles (64), pieces and key
groups, in one key, in stairs, over half of the keys, or builds up over many keys; the neighbouring rows of the
same wave stay as they are.  Whole tiles, pieces and key groups, both key conventions, against the oracle's
attention."""
import numpy as np
import pytest
import torch

import paper_2511_21317_amd as httm
from oracle import httm_oracle as orc
from gpu_util import require_gpu, f32, check_output

pytestmark = pytest.mark.gpu

# rows, keys, scratch: 128-row tiles; 256-row tiles of one key group; 44 tiles in pieces; four key groups of 64 and of
# 128 rows, two of 256
SHAPES = {
    "small_tiles": (301, 700, False),
    "whole_tiles": (256 * 513 + 31, 230, False),
    "pieces": (256 * 299 + 77, 3000, True),
    "four_groups_64": (300, 1089, False),
    "four_groups_128": (8192, 2113, False),
    "two_groups_256": (256 * 200, 2113, False),
}
# log2 units by which the keys from .. to rise in the rows that see them (the channel's q is 1)
RISES = {
    "one_key_31": lambda n: [(31, 32, 90)],
    "one_key_32": lambda n: [(32, 33, 70)],
    "one_key_63": lambda n: [(63, 64, 2000)],
    "one_key_64": lambda n: [(64, 65, 61)],
    "one_key_mid": lambda n: [(n // 2 + 1, n // 2 + 2, 300)],
    "last_key": lambda n: [(n - 1, n, 100)],
    "first_half_low": lambda n: [(0, n // 2, -1500)],
    "first_keys_low": lambda n: [(0, 33, -250)],
    "last_half_low": lambda n: [(n // 2, n, -1500)],
    "stairs": lambda n: [(i, min(i + 45, n), 62 * (i // 45)) for i in range(0, n, 45)],
    "many_keys": lambda n: [(40, n, 53)],          # no key is far above the shift, their sum outgrows it
}


@pytest.mark.parametrize("log2", [True, False], ids=["log2_keys", "plain_keys"])
@pytest.mark.parametrize("rise", RISES)
@pytest.mark.parametrize("shape", SHAPES)
def test_rows_whose_scores_rise_match_the_oracle(shape, rise, log2):
    require_gpu()
    mq, mk, with_scratch = SHAPES[shape]
    gen = torch.Generator().manual_seed(8900 + mq % 991 + mk)
    q, k, v = (torch.randn((n, 64), generator=gen) for n in (mq, mk, mk))
    sees = torch.arange(mq) % 3 == 1
    q[:, 0] = sees.float()
    k[:, 0] = 0
    unit = 1.0 if log2 else 8 / 1.4426950408889634          # a key's channel value per log2 unit of the score
    k[:, 1:] *= float(httm.LOG2_KEY_SCALE) if log2 else 1.0
    for a, b, units in RISES[rise](mk):
        k[a:b, 0] = units * unit
    qm, km, vm = (t.to(torch.bfloat16).cuda() for t in (q, k, v))
    got = torch.full_like(qm, float("nan"))
    scratch = torch.full((httm.attention_scratch_bytes(1),), 0xFF, dtype=torch.uint8, device="cuda") if with_scratch else None
    if log2:
        httm.attention_log2(qm, km, vm, got, [0, mq], [0, mk], scratch=scratch)
    else:
        httm.attention(qm, km, vm, got, [0, mq], [0, mk], 0.125, scratch=scratch)
    torch.cuda.synchronize()
    got, qf, vf = f32(got), f32(qm), f32(vm)
    kf = f32(km) / np.float32(httm.LOG2_KEY_SCALE) if log2 else f32(km)
    assert np.count_nonzero(~np.isfinite(got)) == 0
    rows = np.unique(np.concatenate([np.arange(0, mq, max(1, mq // 300)), np.arange(mq - 140, mq)]))
    check_output(got[rows], orc.attention(qf, kf, vf, rows=rows), f"{shape}, {rise}", relative_to_magnitude=True)


@pytest.mark.parametrize("rise,again", [("last_half_low", False), ("first_half_low", False), ("one_key_mid", True), ("all_low", True)])
def test_pieces_without_shifts_are_judged_by_the_sums_of_their_rows(rise, again):
    """Unshifted weights of a piece may be small if those of the rest of the row are not: such a piece keeps its shift
    of zero.  It takes shifts of its own where its weights are too large, or all of the row's are small."""
    require_gpu()
    mq, mk, _ = SHAPES["pieces"]
    gen = torch.Generator().manual_seed(8960)
    q, k, v = (torch.randn((n, 64), generator=gen) for n in (mq, mk, mk))
    q[:, 0] = (torch.arange(mq) % 3 == 1).float()
    k[:, 0] = 0
    k[:, 1:] *= float(httm.LOG2_KEY_SCALE)
    for a, b, units in [(0, mk, -1500)] if rise == "all_low" else RISES[rise](mk):
        k[a:b, 0] = units
    qm, km, vm = (t.to(torch.bfloat16).cuda() for t in (q, k, v))
    got = torch.full_like(qm, float("nan"))
    scratch = torch.full((httm.attention_scratch_bytes(1),), 0xFF, dtype=torch.uint8, device="cuda")
    httm.attention_log2(qm, km, vm, got, [0, mq], [0, mk], scratch=scratch)
    torch.cuda.synchronize()
    # the scratch holds, for every slot, 256 x 64 sums, then 256 row sums a slot, then 256 shifts a slot
    slots = httm.attention_split_plan([0, mq], [0, mk], torch.cuda.get_device_properties(0).multi_processor_count)["slots"]
    assert slots > 0
    shifts = scratch.view(torch.float32)[slots * 256 * 65:slots * 256 * 66]
    shifts = shifts[~torch.isnan(shifts)]                # (slots and rows that stay unused keep their NaN)
    assert shifts.numel() > 0 and bool((shifts != 0).any()) == again
    rows = np.arange(mq - 300, mq, 7)
    want = orc.attention(f32(qm), f32(km) / np.float32(httm.LOG2_KEY_SCALE), f32(vm), rows=rows)
    check_output(f32(got)[rows], want, rise, relative_to_magnitude=True)


def test_a_row_with_nan_leaves_its_neighbours_alone():
    """Row sums of two query tiles come out of one instruction, where NaN times zero is NaN: the rows beside one with
    NaN are taken again on their own."""
    require_gpu()
    gen = torch.Generator().manual_seed(8950)
    for mq, mk, log2 in ((301, 700, False), (300, 1089, False), (8192, 2113, False), (301, 700, True), (300, 1089, True)):
        q, k, v = (torch.randn((n, 64), generator=gen) for n in (mq, mk, mk))
        q[5] = float("nan")
        q[100, 3] = float("inf")
        scale = np.float32(httm.LOG2_KEY_SCALE) if log2 else np.float32(1.0)
        qm, km, vm = (t.to(torch.bfloat16).cuda() for t in (q, k * float(scale), v))
        got = torch.full_like(qm, 7.0)
        if log2:
            httm.attention_log2(qm, km, vm, got, [0, mq], [0, mk])
        else:
            httm.attention(qm, km, vm, got, [0, mq], [0, mk], 0.125)
        torch.cuda.synchronize()
        got = f32(got)
        assert np.isnan(got[[5, 100]]).all()
        rows = np.setdiff1d(np.arange(min(mq, 400)), [5, 100])
        check_output(got[rows], orc.attention(f32(qm), f32(km) / scale, f32(vm), rows=rows), f"{mq} x {mk}")
