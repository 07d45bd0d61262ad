"""Stage 3 (Eq. 3-4) on rows whose every score is near the lowest float: a channel that masks all keys of
some rows (q = 1, k = the lowest bf16) leaves them uniform weights, so their result is the mean of the
values.  Whole tiles, tiles in pieces and key groups, both key conventions; the other rows of the same tiles
against the oracle's attention."""
import numpy as np
import pytest
import torch

import paper_2511_21317_amd as httm
from oracle import httm_oracle as orc
from gpu_util import require_gpu, f32, check_output

pytestmark = pytest.mark.gpu

LOWEST = float(torch.finfo(torch.bfloat16).min)

# rows and keys per head, scratch.  On 256 CUs: 128-row tiles; 256-row tiles of one key group; 44 tiles in
# pieces; 64- and 128-row tiles with four key groups, 256-row tiles with two.
CASES = {
    "small_tiles": ([301, 77], [700, 65], False),
    "whole_tiles": ([256 * 300 + 31, 256 * 300], [130, 97], False),
    "pieces": ([256 * 299 + 77], [6000], True),
    "four_groups_64": ([300, 17], [1089, 64], False),
    "four_groups_128": ([8192, 65], [2113, 31], False),
    "two_groups_256": ([256 * 200, 257], [2113, 129], False),
}


@pytest.mark.parametrize("log2", [True, False], ids=["log2_keys", "plain_keys"])
@pytest.mark.parametrize("case", CASES)
def test_rows_of_the_lowest_scores_have_uniform_weights(case, log2):
    require_gpu()
    mq, mk, with_scratch = CASES[case]
    qo, ko = ([int(x) for x in np.concatenate([[0], np.cumsum(n)])] for n in (mq, mk))
    gen = torch.Generator().manual_seed(8600 + sum(mq) % 991)
    q, k, v = (torch.randn((n, 64), generator=gen) for n in (qo[-1], ko[-1], ko[-1]))
    masked = torch.zeros(qo[-1], dtype=torch.bool)
    masked[::37] = True
    masked[-13:] = True                     # and the end of the last tile
    q[:, 0] = masked.float()
    k[:, 0] = LOWEST
    if log2:
        k[:, 1:] *= float(np.float32(httm.LOG2_KEY_SCALE))
    qm, km, vm = (t.to(torch.bfloat16).cuda() for t in (q, k, v))
    assert torch.isfinite(km).all()
    got = torch.full_like(qm, float("nan"))
    scratch = torch.full((httm.attention_scratch_bytes(len(mq)),), 0xFF, dtype=torch.uint8, device="cuda") if with_scratch else None
    if log2:
        httm.attention_log2(qm, km, vm, got, qo, ko, scratch=scratch)
    else:
        httm.attention(qm, km, vm, got, qo, ko, 0.125, scratch=scratch)
    torch.cuda.synchronize()
    got, qf, kf, vf, masked = f32(got), f32(qm), f32(km), f32(vm), masked.numpy()
    qf[:, 0] = kf[:, 0] = 0                 # what the other rows see of the channel: 0 * lowest
    if log2:
        kf /= np.float32(httm.LOG2_KEY_SCALE)
    assert np.count_nonzero(~np.isfinite(got)) == 0
    for h in range(len(mq)):
        n, m = got[qo[h]:qo[h + 1]], masked[qo[h]:qo[h + 1]]
        vh = vf[ko[h]:ko[h + 1]]
        mean = np.broadcast_to(vh.astype(np.float64).mean(axis=0), n[m].shape)
        check_output(n[m], mean, f"{case}, head {h}, masked rows")
        rows = np.flatnonzero(~m)
        rows = rows[:: max(1, rows.size // 200)]
        want = orc.attention(qf[qo[h]:qo[h + 1]], kf[ko[h]:ko[h + 1]], vh, rows=rows)
        check_output(n[rows], want, f"{case}, head {h}, other rows")
