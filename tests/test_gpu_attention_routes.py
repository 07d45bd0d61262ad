"""Stage 3 (Eq. 3-4) with scratch memory where there are few query rows: a launch against many keys runs in
segments (they keep every CU busy), one against fewer keys in key groups, which touch no scratch.  Shapes to either
side of the line, on 256 CUs, both key conventions, against the oracle's attention."""
import numpy as np
import pytest
import torch

import paper_2511_21317_amd as httm
from oracle import httm_oracle as orc
from gpu_util import require_gpu, f32, check_output

pytestmark = pytest.mark.gpu

# heads, rows, keys, runs in segments
SHAPES = [
    (16, 64, 2500, False), (16, 64, 6000, True), (8, 250, 12000, True), (16, 250, 12000, True), (1, 1000, 2000, False),
    (1, 1000, 30000, True), (1, 256, 28700, True), (16, 500, 4000, False), (16, 500, 9000, True), (1, 30000, 9000, False),
    (16, 2000, 8192, False), (12, 2800, 28000, True), (16, 3000, 12000, False),
]


@pytest.mark.parametrize("log2", [True, False], ids=["log2_keys", "plain_keys"])
@pytest.mark.parametrize("H,mq,mk,segments", SHAPES)
def test_few_rows_take_segments_against_many_keys_only(H, mq, mk, segments, log2):
    require_gpu()
    print(f"[case] {H} heads of {mq} rows x {mk} keys, log2={log2}", flush=True)
    lens_q = [mq - (h % 3) for h in range(H)]
    lens_k = [mk - 5 * (h % 4) for h in range(H)]
    qo, ko = ([int(x) for x in np.concatenate([[0], np.cumsum(n)])] for n in (lens_q, lens_k))
    gen = torch.Generator().manual_seed(8700 + mq + mk)
    q, k, v = (torch.randn((n, 64), generator=gen) for n in (qo[-1], ko[-1], ko[-1]))
    scale = np.float32(httm.LOG2_KEY_SCALE) if log2 else np.float32(1.0)
    qm, km, vm = (t.to(torch.bfloat16).cuda() for t in (q, k * float(scale), v))
    got = torch.full_like(qm, float("nan"))
    scratch = torch.full((httm.attention_scratch_bytes(H),), 0xFF, dtype=torch.uint8, device="cuda")
    if log2:
        httm.attention_log2(qm, km, vm, got, qo, ko, scratch=scratch)
    else:
        httm.attention(qm, km, vm, got, qo, ko, 0.125, scratch=scratch)
    torch.cuda.synchronize()
    assert bool((scratch != 0xFF).any()) == segments
    got, qf, kf, vf = f32(got), f32(qm), f32(km) / scale, f32(vm)
    assert np.count_nonzero(~np.isfinite(got)) == 0
    for h in sorted({0, H // 2, H - 1}):
        rows = np.unique(np.concatenate([np.arange(0, lens_q[h], max(1, lens_q[h] // 60)), np.arange(max(0, lens_q[h] - 20), lens_q[h])]))
        want = orc.attention(qf[qo[h]:qo[h + 1]], kf[ko[h]:ko[h + 1]], vf[ko[h]:ko[h + 1]], rows=rows)
        check_output(got[qo[h]:qo[h + 1]][rows], want, f"head {h}")


def test_the_static_entry_point_takes_a_launch_in_key_groups_whatever_its_segments_would_need():
    """128 tiles of 256 rows against 40000 keys: segments would need 41 MiB of partial results, more than the library's
    array holds, but the launch runs in key groups and needs none."""
    require_gpu()
    mq, mk = 128 * 256, 40000
    gen = torch.Generator().manual_seed(8800)
    q, k, v = (torch.randn((n, 64), generator=gen) for n in (mq, mk, mk))
    scale = np.float32(httm.LOG2_KEY_SCALE)
    qm, km, vm = (t.to(torch.bfloat16).cuda() for t in (q, k * float(scale), v))
    got, want = torch.full_like(qm, float("nan")), torch.full_like(qm, float("nan"))
    httm.attention_log2_static(qm, km, vm, got, [0, mq], [0, mk])
    scratch = torch.full((httm.attention_scratch_bytes(1),), 0xFF, dtype=torch.uint8, device="cuda")
    httm.attention_log2(qm, km, vm, want, [0, mq], [0, mk], scratch=scratch)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16)) and bool((scratch == 0xFF).all())
    rows = np.arange(0, mq, 613)
    check_output(f32(got)[rows], orc.attention(f32(qm), f32(km) / scale, f32(vm), rows=rows), "static, key groups")
