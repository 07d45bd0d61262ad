"""Stage 3 (Eq. 3-4) in 512-row tiles: long launches with log2 keys, against the oracle on rows either side of the edges of
tiles, slots and waves, and against the same call without scratch, whose rows of whole tiles have the same sums."""
import numpy as np
import pytest
import torch

import paper_2511_21317_amd as httm
from oracle import httm_oracle as orc
from gpu_util import require_gpu, f32, check_output

pytestmark = pytest.mark.gpu

LIMIT = httm.attention_scratch_bytes(1)


def _run(mq, mk, seed, change=None):
    qo, ko = ([int(x) for x in np.concatenate([[0], np.cumsum(n)])] for n in (mq, mk))
    plan = httm.attention_wide_plan(qo, ko, torch.cuda.get_device_properties(0).multi_processor_count)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = (torch.randn((n, 64), generator=gen, device="cuda") for n in (qo[-1], ko[-1], ko[-1]))
    if change is not None:
        change(q, k, qo, ko)
    q, v, k2 = q.bfloat16(), v.bfloat16(), (k * httm.LOG2_KEY_SCALE).bfloat16()
    scratch = torch.full((LIMIT,), 0xFF, dtype=torch.uint8, device="cuda")      # NaN bit patterns
    out, plain = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    httm.attention_log2(q, k2, v, out, qo, ko, scratch=scratch)
    httm.attention_log2(q, k2, v, plain, qo, ko)
    torch.cuda.synchronize()
    return plan, q, k2, v, qo, ko, out, plain


def _check_rows(q, k2, v, qo, ko, out, heads):
    rng = np.random.default_rng(7)
    for h in heads:
        n = qo[h + 1] - qo[h]
        if n == 0:
            continue
        last = n // 512 * 512
        rows = [0, 1, 63, 64, 127, 128, 255, 256, 383, 384, 511, 512, last - 1, last, last + 127, last + 255, last + 256, last + 257, n - 1]
        rows = np.unique([r for r in rows + list(rng.integers(0, n, 60)) if 0 <= r < n])
        kk = f32(k2[ko[h]:ko[h + 1]]) / np.float32(httm.LOG2_KEY_SCALE)
        want = orc.attention(f32(q[qo[h]:qo[h + 1]][rows.tolist()]), kk, f32(v[ko[h]:ko[h + 1]]))
        check_output(f32(out[qo[h]:qo[h + 1]][rows.tolist()]), want, f"head {h} of {n} rows")


# whole rounds; partial tiles of few rows with units of two key tiles, of one and 256 rows; partial tiles with two slots;
# both kinds; a head without rows; ragged keys, a last key tile of one key
CASES = [
    ([16384] * 16, [4096] * 16, 0),
    ([28700] * 16, [14401] * 16, 144),
    ([28160 + (1 if h % 2 else 256) for h in range(16)], [12033] * 16, None),
    ([28650] * 16, [17001] * 16, 128),
    ([24000 + 411 * h for h in range(16)], [14000 - 20 * h for h in range(16)], None),
    ([43968] * 6 + [0] + [46080] * 6, [9216 + 17 * h for h in range(13)], None),
]


@pytest.mark.parametrize("mq,mk,n_tiles", CASES, ids=["whole", "few_rows", "one_or_256_rows", "two_slots", "ragged", "no_rows"])
def test_wide_tiles_match_the_oracle(mq, mk, n_tiles):
    require_gpu()
    print(f"[case] {mq} {mk}", flush=True)
    plan, q, k2, v, qo, ko, out, plain = _run(mq, mk, 6100 + len(mq) + mq[0] % 100)
    assert plan is not None and (plan["n_tiles"] > 0 if n_tiles is None else plan["n_tiles"] == n_tiles)
    _check_rows(q, k2, v, qo, ko, out, [0, 1, len(mq) // 2, len(mq) - 1])
    pieces = torch.zeros(qo[-1], dtype=torch.bool, device="cuda")
    for _, h, q0, *_ in plan["segments"].tolist():
        pieces[qo[h] + q0:min(qo[h] + q0 + 512, qo[h + 1])] = True
    d = (out.float() - plain.float()).abs()
    assert bool((d <= 2.0 ** -7 * plain.float().abs() + 1e-5).all()), float(d.max())     # fp32 rounding of the pieces' sums
    if len(httm.attention_route(qo, ko, 256, 0)["tiles"]) == 1:     # (else some of its rows run in key groups)
        assert torch.equal(out[~pieces], plain[~pieces])


def test_rows_out_of_the_unshifted_range():
    """Whole tiles and pieces whose weights leave the range of the pass without shifts, above in a few keys and below in all
    of them, and pieces that hold masked keys only, which keep their sums of (almost) nothing."""
    require_gpu()

    def change(q, k, qo, ko):
        k[ko[3] + 6000:ko[3] + 6100] *= 60.0                  # head 3: far above, in one piece of its tiles
        k[ko[5]:ko[6]] *= 0.0                                 # head 5: all weights 1
        for h in (7, 9, 15):
            q[qo[h]:qo[h + 1], 0] = 16.0
        for h, first in ((7, 6000), (9, 0), (15, 6000)):
            k[ko[h] + first:ko[h + 1], 0] = -100.0            # 7, 15: half of the keys masked; 9: all scores low
        k[ko[14] + 100, :] = 40.0 * torch.sign(q[qo[15] - 1, :])      # head 14: one key that some rows like

    plan, q, k2, v, qo, ko, out, plain = _run([28700] * 16, [14401] * 16, 6200, change)
    assert plan is not None and plan["n_tiles"] == 144
    assert bool(torch.isfinite(out.float()).all())
    _check_rows(q, k2, v, qo, ko, out, [0, 3, 5, 7, 9, 14, 15])


def test_only_the_half_with_a_row_out_of_range_is_taken_again():
    """One key that only single rows see brings these out of the range: their 256-row halves of the tiles are taken again with
    shifts; every other row keeps the bits it has without that key's channel."""
    require_gpu()
    mq, mk = 28650, 17001
    # (head, row): whole tiles, first and last rows of either half; a partial tile in pieces; a full tile in pieces
    bad = [(1, 512 * 10), (1, 512 * 13 + 255), (2, 512 * 20 + 256), (4, 512 * 9 + 511), (5, 512 * 3 + 7), (5, 512 * 3 + 300),
           (0, mq - 1), (3, mq // 512 * 512 + 30), (15, 512 * 50 + 3), (14, 512 * 52 + 400)]

    def change(key_value):
        def set_channel(q, k, qo, ko):
            q[:, 0] = 0
            k[:, 0] = 0
            for h, r in bad:
                q[qo[h] + r, 0] = 1.0
            k[torch.tensor(ko[:-1]) + 9000, 0] = key_value
        return set_channel

    plan, *_, calm, _ = _run([mq] * 16, [mk] * 16, 6250, change(0.0))
    pieces = {(h, q0) for _, h, q0, *_ in plan["segments"].tolist()}
    assert (0, mq // 512 * 512) in pieces and (15, 512 * 50) in pieces and (1, 512 * 10) not in pieces
    _, q, k2, v, qo, ko, out, _ = _run([mq] * 16, [mk] * 16, 6250, change(1200.0))
    again = torch.zeros(qo[-1], dtype=torch.bool, device="cuda")
    for h, r in bad:
        again[qo[h] + r // 256 * 256:min(qo[h] + r // 256 * 256 + 256, qo[h + 1])] = True
        kk = f32(k2[ko[h]:ko[h + 1]]) / np.float32(httm.LOG2_KEY_SCALE)
        rows = [x for x in (r - 1, r, r + 1, r // 256 * 256, r // 256 * 256 + 255) if 0 <= x < mq]
        want = orc.attention(f32(q[qo[h]:qo[h + 1]][rows]), kk, f32(v[ko[h]:ko[h + 1]]))
        check_output(f32(out[qo[h]:qo[h + 1]][rows]), want, f"head {h}, rows around {r}", relative_to_magnitude=True)
    assert bool(torch.isfinite(out.float()).all())
    assert torch.equal(out[~again], calm[~again])


def test_the_library_s_own_scratch_gives_the_same_bits():
    require_gpu()
    plan, q, k2, v, qo, ko, out, _ = _run([28700] * 16, [14401] * 16, 6300)
    assert plan["slots"] * 256 * 66 * 4 > 32 << 20
    own = torch.full_like(q, float("nan"))
    httm.attention_log2_static(q, k2, v, own, qo, ko)
    torch.cuda.synchronize()
    assert torch.equal(own, out)


def test_a_layer_s_outlier_queries_behind_wide_tiles():
    """100 frames of 37 x 37, a tenth of the queries outliers: merged rows and outliers in one launch of 512-row tiles, the
    pieces behind both.  The same bits as the separate calls (which are checked against the oracle elsewhere)."""
    require_gpu()
    S, H = 100, 16
    plan = httm.Plan(httm.make_geom(S, 37, 37, 4, 4, 0.8, 0.8, H=H, log2_keys=True, outlier_frac=0.1))
    off = [h * plan.M_q for h in range(H + 1)]
    assert httm.attention_wide_plan(off, [h * plan.M_k for h in range(H + 1)])["n_tiles"] > 0
    gen = torch.Generator(device="cuda").manual_seed(6400)
    q, k, v = (torch.randn((H, plan.N, 64), generator=gen, device="cuda").bfloat16() for _ in range(3))
    out = torch.full((plan.N, H * 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = httm.alloc_workspace(plan)
    httm.layer_forward(plan, q, k, v, out, ws)
    w = httm.workspace_views(plan, ws)
    o_m, o_out = torch.empty_like(w["o_m"]), torch.empty_like(w["o_out"])
    scratch = torch.empty(LIMIT, dtype=torch.uint8, device="cuda")
    httm.attention_log2(w["q_m"], w["k_m"], w["v_m"], o_m, off, [h * plan.M_k for h in range(H + 1)], scratch=scratch)
    httm.attention_outliers(plan, w["q_out"], w["k_m"], w["v_m"], o_out)
    torch.cuda.synchronize()
    assert torch.equal(o_m, w["o_m"])
    want = torch.empty_like(out)
    httm.unmerge_filtered(plan, o_m, o_out, w["assign_q"], want)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    plan.close()
