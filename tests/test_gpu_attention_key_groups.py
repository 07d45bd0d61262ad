"""Stage 3 (Eq. 3-4) with the keys cut among the waves of a workgroup: heads of few rows (64- and 128-row
tiles, four key groups; 256-row tiles, two), and what is left after whole rounds of 256-row tiles.  Both key
conventions, key counts around the dispatch's limits and where the groups' shares are unequal, one
group with rows out of range, an empty head, against the oracle's attention."""
import numpy as np
import pytest
import torch

import paper_2511_21317_amd as httm
from oracle import httm_oracle as orc
from gpu_util import require_gpu, f32, check_output

pytestmark = pytest.mark.gpu

# rows and keys per head.  On 256 CUs: 64-row tiles from 768 keys, the others from 2048, the rounds from 512 full tiles.
CASES = {
    "four_groups_limit": ([64, 65, 1, 256], [768, 767, 705, 768]),
    "four_groups_unequal": ([300, 17], [1089, 64]),           # 18 key tiles; a single one: three groups without keys
    "four_groups_empty_heads": ([100, 0, 40, 33], [900, 500, 0, 1]),
    "eight_waves_128_limit": ([8192, 8065, 1], [2048, 2047, 1985]),
    "eight_waves_128_one_tile": ([16384, 130], [2113, 31]),
    "eight_waves_256_limit": ([256 * 100, 256 * 100 + 1, 300, 200], [2048, 2047, 65, 1]),
    "eight_waves_256_unequal": ([256 * 200, 257], [2113, 129]),
    "rounds_and_four_groups": ([256 * 256 + 100, 256 * 256 + 65, 77], [400, 333, 129]),
    "rounds_and_eight_waves": ([256 * 400, 256 * 200 + 3], [200, 321]),
}


def _off(n):
    return [int(x) for x in np.concatenate([[0], np.cumsum(n)])]


@pytest.mark.parametrize("log2", [True, False], ids=["log2_keys", "plain_keys"])
@pytest.mark.parametrize("out_of_range", [False, True], ids=["in_range", "out_of_range"])
@pytest.mark.parametrize("case", CASES)
def test_key_groups_match_the_oracle(case, out_of_range, log2):
    require_gpu()
    mq, mk = CASES[case]
    qo, ko = _off(mq), _off(mk)
    gen = torch.Generator().manual_seed(8300 + sum(mq) % 997)
    q, k, v = (torch.randn((n, 64), generator=gen) for n in (qo[-1], ko[-1], ko[-1]))
    if out_of_range:      # keys of the last group (and of a head's only tile) draw some rows out of the range
        for h in range(len(mq)):
            k[ko[h + 1] - min(5, mk[h]):ko[h + 1]] *= 30
            q[qo[h + 1] - min(70, mq[h]):qo[h + 1]] *= 20
    scale = np.float32(httm.LOG2_KEY_SCALE)
    qm, vm = q.to(torch.bfloat16).cuda(), v.to(torch.bfloat16).cuda()
    km = (k * float(scale) if log2 else k).to(torch.bfloat16).cuda()
    got = torch.full_like(qm, float("nan"))
    if log2:
        httm.attention_log2(qm, km, vm, got, qo, ko)
    else:
        httm.attention(qm, km, vm, got, qo, ko, 0.125)
    torch.cuda.synchronize()
    got, qf, vf = f32(got), f32(qm), f32(vm)
    kf = f32(km) / scale if log2 else f32(km)
    assert np.isfinite(got).all()
    for h in range(len(mq)):
        g = got[qo[h]:qo[h + 1]]
        if mq[h] == 0 or mk[h] == 0:
            assert not g.any()
            continue
        rows = np.unique(np.concatenate([np.arange(0, mq[h], max(1, mq[h] // 300)), np.arange(max(0, mq[h] - 140), mq[h])]))
        want = orc.attention(qf[qo[h]:qo[h + 1]], kf[ko[h]:ko[h + 1]], vf[ko[h]:ko[h + 1]], rows=rows)
        check_output(g[rows], want, f"{case}, head {h}", relative_to_magnitude=out_of_range or mk[h] < 64)
