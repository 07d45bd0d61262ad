"""Stage 3 (Eq. 3-4) on few rows: tiles of 32, 64 and 128 rows whose waves of 32 rows share the keys in four, four and
two groups.  Row counts around the tiles' edges, key counts that leave groups without a key tile or with unequal
ones, both key conventions, rows that leave the range of the unshifted weights, against the oracle's attention."""
import numpy as np
import pytest
import torch

import paper_2511_21317_amd as httm
from oracle import httm_oracle as orc
from gpu_util import require_gpu, f32, check_output

pytestmark = pytest.mark.gpu

# rows and keys per head; on 256 CUs by the number of tiles and the longest head's keys
CASES = {
    "rows32": ([1, 31, 32, 33, 64, 65, 0, 97], [300, 64, 65, 255, 256, 257, 9, 1]),
    "rows32_many_heads": ([470, 481, 460, 512] * 4, [439, 449, 128, 193] * 4),
    "rows64": ([1000, 961, 1024, 1, 1023, 63, 65, 2000] * 2, [500, 1000, 449, 65, 700, 1, 64, 513] * 2),
    "rows128": ([2000, 1921, 1, 2048, 2047, 1500, 127, 129] * 2, [1400, 1409, 64, 1, 1000, 129, 200, 1345] * 2),
}


@pytest.mark.parametrize("log2", [True, False], ids=["log2_keys", "plain_keys"])
@pytest.mark.parametrize("out_of_range", [False, True], ids=["in_range", "out_of_range"])
@pytest.mark.parametrize("case", CASES)
def test_small_tiles_match_the_oracle(case, out_of_range, log2):
    require_gpu()
    print(f"[case] {case} log2={log2} out_of_range={out_of_range}", flush=True)
    mq, mk = CASES[case]
    qo, ko = ([int(x) for x in np.concatenate([[0], np.cumsum(n)])] for n in (mq, mk))
    gen = torch.Generator().manual_seed(9100 + sum(mq) % 997)
    q, k, v = (torch.randn((n, 64), generator=gen) for n in (qo[-1], ko[-1], ko[-1]))
    if out_of_range:
        for h in range(len(mq)):
            k[ko[h + 1] - min(5, mk[h]):ko[h + 1]] *= 30
            q[qo[h + 1] - min(40, mq[h]):qo[h + 1]] *= 20
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
    for h in range(min(8, len(mq))):
        if mq[h] == 0:
            continue
        rows = np.unique(np.concatenate([np.arange(0, mq[h], max(1, mq[h] // 200)), np.arange(max(0, mq[h] - 70), mq[h])]))
        want = orc.attention(qf[qo[h]:qo[h + 1]], kf[ko[h]:ko[h + 1]], vf[ko[h]:ko[h + 1]], rows=rows)
        check_output(got[qo[h]:qo[h + 1]][rows], want, f"{case}, head {h}", relative_to_magnitude=out_of_range or mk[h] < 64)
