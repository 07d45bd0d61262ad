"""Stage 3 (Eq. 3-4) where rows leave the range of their weights: per-row shifts are raised in the step that needs
it (plain keys), tiles and pieces without shifts are taken again with shifts, inside the same launch (log2 keys).
Both key conventions, key counts around the step (32) and tile (64) sizes, against the oracle's attention."""
import numpy as np
import pytest
import torch

import paper_2511_21317_amd as httm
from oracle import httm_oracle as orc
from gpu_util import require_gpu, f32, check_output

pytestmark = pytest.mark.gpu

KEY_SCALE = np.float32(httm.LOG2_KEY_SCALE)


def _run(q, k, v, mq, mk, log2, scratch=False):
    qm = q.to(torch.bfloat16).cuda()
    km = (k * float(KEY_SCALE) if log2 else k).to(torch.bfloat16).cuda()
    vm = v.to(torch.bfloat16).cuda()
    om = torch.full_like(qm, float("nan"))
    room = torch.full((httm.attention_scratch_bytes(1),), 0xFF, dtype=torch.uint8, device="cuda") if scratch else None
    if log2:
        httm.attention_log2(qm, km, vm, om, [0, mq], [0, mk], scratch=room)
    else:
        httm.attention(qm, km, vm, om, [0, mq], [0, mk], 0.125, scratch=room)
    torch.cuda.synchronize()
    kk = f32(km) / KEY_SCALE if log2 else f32(km)
    return f32(om), f32(qm), kk, f32(vm)


@pytest.mark.parametrize("log2", [True, False], ids=["log2_keys", "plain_keys"])
@pytest.mark.parametrize("mk", [1, 31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 191, 192, 193, 257, 320])
def test_key_counts_around_steps_and_tiles_with_and_without_running_maxima(mk, log2):
    require_gpu()
    gen = torch.Generator().manual_seed(8100 + mk)
    mq = 301                                     # 128-row tiles, the last one partial
    q, k, v = (torch.randn((n, 64), generator=gen) for n in (mq, mk, mk))
    got, qf, kf, vf = _run(q, k, v, mq, mk, log2)
    check_output(got, orc.attention(qf, kf, vf), f"{mk} keys")
    q[130:140] *= 40                             # rows of the second tile leave the range (either way)
    k[mk // 2:] *= 30
    got, qf, kf, vf = _run(q, k, v, mq, mk, log2)
    assert np.isfinite(got).all()
    check_output(got, orc.attention(qf, kf, vf), f"{mk} keys, out of range", relative_to_magnitude=True)


@pytest.mark.parametrize("log2", [True, False], ids=["log2_keys", "plain_keys"])
@pytest.mark.parametrize("case", ["one_piece_high", "one_piece_low", "all_pieces_low"])
def test_pieces_of_a_split_tile_keep_their_own_shifts(case, log2):
    """300 tiles on 256 CUs: 44 run in pieces.  Keys in one stretch make the weights of the pieces that hold
    them leave the range (too large; or, without shifts, sums below 2^-64), the other pieces stay in it."""
    require_gpu()
    gen = torch.Generator().manual_seed(8200)
    mq, mk = 256 * 299 + 77, 6000
    base = torch.randn((1, 64), generator=gen)
    q = base + 0.3 * torch.randn((mq, 64), generator=gen)      # rows that agree on a direction
    k = 0.3 * torch.randn((mk, 64), generator=gen)
    v = torch.randn((mk, 64), generator=gen)
    if case == "one_piece_high":
        k[2000:2100] += 12 * base
    elif case == "one_piece_low":
        k[1000:3500] -= 12 * base
    else:
        k -= 12 * base
    plan = httm.attention_split_plan([0, mq], [0, mk], torch.cuda.get_device_properties(0).multi_processor_count)
    assert plan["n_tiles"] == 44
    got, qf, kf, vf = _run(q, k, v, mq, mk, log2, scratch=True)
    assert np.isfinite(got).all()
    rows = np.unique(np.concatenate([np.arange(0, mq, 997), np.arange(mq - 44 * 256, mq, 41), np.arange(mq - 77, mq)]))
    want = orc.attention(qf, kf, vf, rows=rows)
    check_output(got[rows], want, case, relative_to_magnitude=True)
