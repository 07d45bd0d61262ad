"""Stage 4 at the end of stage 3's tiles (httm_layer_forward) against the stage-4 kernel on the same merged
outputs and assignments: the copies must agree bit for bit, whatever the tile size, the blocks and the row counts."""
import pytest
import torch

import paper_2511_21317_amd as httm
from gpu_util import merged_attention, require_gpu

pytestmark = pytest.mark.gpu

# name, S, Hp, Wp, b, T, rho_q, rho_kv, H, options
CASES = [
    ("one_token", 1, 1, 1, 1, 1, 0.0, 0.0, 1, {}),                                   # a tile with a single row
    ("groups32", 2, 16, 16, 4, 2, 0.5, 0.5, 16, {}),                                 # keys shared in four groups
    ("groups32_span_of_one_block", 2, 16, 16, 16, 2, 0.6, 0.2, 3, {}),               # 512-token blocks: a tile inside one
    ("groups64", 3, 19, 23, 4, 2, 0.5, 0.5, 16, {}),
    ("groups128", 7, 20, 21, 4, 2, 0.5, 0.4, 16, {}),
    ("groups128_wide", 20, 21, 21, 4, 2, 0.5, 0.5, 5, {}),
    ("tiles128", 9, 25, 24, 4, 2, 0.5, 0.9, 16, {}),
    ("groups256", 9, 29, 31, 4, 2, 0.55, 0.5, 15, {}),
    ("segments", 8, 37, 35, 4, 2, 0.5, 0.5, 16, {}),
    ("segments_plain_keys", 8, 37, 35, 4, 2, 0.5, 0.5, 16, {"log2_keys": False}),
    ("unmerged", 8, 21, 19, 4, 2, 0.0, 0.0, 16, {"variant": "none"}),                # exact spans, no search
    ("top_r", 6, 25, 27, 8, 4, 0.4, 0.4, 8, {"dst_frac": 0.25}),
    ("top_r_nothing_merges", 4, 17, 16, 8, 2, 0.0, 0.0, 6, {"dst_frac": 0.25}),      # all clusters, not in order
    ("uniform", 5, 22, 20, 5, 3, 0.6, 0.5, 12, {"variant": "uniform"}),
    ("big_blocks", 31, 9, 37, 128, 30, 0.9, 0.7, 4, {"chunked_blocks": True}),
    ("big_blocks_little_merged", 30, 8, 17, 128, 30, 0.1, 0.5, 3, {"chunked_blocks": True}),
    ("outliers", 9, 21, 22, 5, 3, 0.7, 0.6, 8, {"outlier_frac": 0.1}),
    ("outliers_few", 9, 21, 22, 5, 3, 0.7, 0.6, 8, {"outlier_frac": 0.0003}),
    ("outliers_segments", 8, 37, 35, 4, 2, 0.5, 0.5, 16, {"outlier_frac": 0.05}),
    ("outliers_big_blocks", 20, 9, 31, 128, 20, 0.8, 0.7, 4, {"chunked_blocks": True, "outlier_frac": 0.1}),
    ("anchored", 6, 18, 17, 4, 3, 0.8, 0.8, 7, {"anchor_first_frame": True}),
    # many queries against few keys: whole rounds of tiles, then the heads' last rows in a launch of their own
    ("rounds", 13, 37, 37, 8, 4, 0.5, 0.9, 16, {}),
    ("rounds_plain_keys", 13, 37, 37, 8, 4, 0.5, 0.9, 16, {"log2_keys": False}),
    ("rounds_head_in_both", 19, 28, 37, 4, 2, 0.5, 0.9, 16, {}),
    ("rounds_queries_unmerged", 9, 37, 37, 4, 2, 0.0, 0.9, 12, {}),
    ("rounds_24_heads", 9, 37, 37, 4, 2, 0.5, 0.85, 24, {}),
    ("rounds_outliers", 13, 37, 37, 8, 4, 0.5, 0.9, 16, {"outlier_frac": 0.05}),
    ("rounds_outliers_plain_keys", 19, 28, 37, 4, 2, 0.5, 0.9, 16, {"outlier_frac": 0.002, "log2_keys": False}),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_layer_outputs_are_the_stage_kernels_copies(case):
    require_gpu()
    name, S, Hp, Wp, b, T, rho_q, rho_kv, H, opts = case
    print(f"[case] {name}", flush=True)
    plan = httm.Plan(httm.make_geom(S, Hp, Wp, b, T, rho_q, rho_kv, H=H, **{"log2_keys": True, **opts}))
    gen = torch.Generator(device="cuda").manual_seed(len(name))
    q, k, v = (torch.randn((H, plan.N, 64), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    out = torch.full((plan.N, H * 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = httm.alloc_workspace(plan)
    for _ in range(2):                                   # (the second call finds the first one's workspace)
        out.fill_(float("nan"))
        httm.layer_forward(plan, q, k, v, out, ws)
    views = httm.workspace_views(plan, ws)
    want = torch.empty_like(out)
    if plan.outlier_cap:
        httm.unmerge_filtered(plan, views["o_m"], views["o_out"], views["assign_q"], want)
    else:
        httm.unmerge(plan, views["o_m"], views["assign_q"], want)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), want.view(torch.int16))
    assert bool(torch.isfinite(out.float()).all())
    plan.close()


# the outlier queries in the merged rows' tiles, behind them in one launch, or in tiles and a launch of their own
FILTERED = [
    ("groups32", 5, 19, 17, 4, 2, 0.86, 0.86, 8, {"outlier_frac": 0.05, "log2_keys": False}),
    ("groups64", 3, 33, 19, 4, 4, 0.34, 0.73, 8, {"outlier_frac": 0.005}),
    ("groups128", 4, 20, 17, 4, 1, 0.24, 0.24, 16, {"outlier_frac": 0.02}),
    ("groups128_apart", 5, 28, 19, 4, 4, 0.38, 0.35, 16, {"outlier_frac": 0.1}),
    ("groups128_wide", 25, 21, 17, 5, 3, 0.65, 0.49, 8, {"outlier_frac": 0.005}),
    ("groups256", 4, 37, 31, 5, 3, 0.41, 0.41, 16, {"outlier_frac": 0.1}),
    ("groups256_plain_keys", 33, 29, 15, 6, 6, 0.7, 0.7, 8, {"outlier_frac": 0.02, "log2_keys": False}),
    ("groups256_apart", 19, 27, 34, 4, 4, 0.73, 0.73, 12, {"outlier_frac": 0.05}),
    ("tiles128", 3, 32, 26, 8, 4, 0.47, 0.89, 16, {"outlier_frac": 0.1, "log2_keys": False}),
    ("rounds", 11, 33, 30, 4, 2, 0.25, 0.91, 16, {"outlier_frac": 0.02}),
    ("rounds_apart", 19, 31, 21, 6, 6, 0.21, 0.89, 16, {"outlier_frac": 0.02, "log2_keys": False}),
]


@pytest.mark.parametrize("case", FILTERED, ids=[c[0] for c in FILTERED])
def test_filtered_layer_outputs_are_those_of_the_stage_calls(case):
    require_gpu()
    name, S, Hp, Wp, b, T, rho_q, rho_kv, H, opts = case
    print(f"[case] filtered {name}", flush=True)
    plan = httm.Plan(httm.make_geom(S, Hp, Wp, b, T, rho_q, rho_kv, H=H, **{"log2_keys": True, **opts}))
    gen = torch.Generator(device="cuda").manual_seed(100 + len(name))
    q, k, v = (torch.randn((H, plan.N, 64), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    out, want = (torch.full((plan.N, H * 64), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    httm.layer_forward(plan, q, k, v, out, httm.alloc_workspace(plan))
    staged = httm.workspace_views(plan, httm.alloc_workspace(plan))
    httm.reorder_match_merge_filtered(plan, q, k, v, staged["q_m"], staged["k_m"], staged["v_m"], staged["assign_q"],
                                      staged["assign_k"], staged["eps_q"], staged["q_out"])
    merged_attention(plan, staged["q_m"], staged["k_m"], staged["v_m"], staged["o_m"])
    httm.attention_outliers(plan, staged["q_out"], staged["k_m"], staged["v_m"], staged["o_out"])
    httm.unmerge_filtered(plan, staged["o_m"], staged["o_out"], staged["assign_q"], want)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), want.view(torch.int16))
    assert bool(torch.isfinite(out.float()).all())
    plan.close()
