"""Stage 2 in blocks of at most 16 tokens, of 257 to 448 tokens (eight waves whose tiles go round) and, by the general rule, of
one wave (merging tokens picked by counting): exact ties and zero rows, block sizes around the limits, one-token
blocks.  The checks are those of the tests of ties, of the general rule and of the whole layer."""
import pytest

import test_gpu_random_geometries
import test_gpu_ties
import test_gpu_topr
from synth.vggt_tokens import Workload
from test_gpu_block_sizes import _runs_of

pytestmark = pytest.mark.gpu

# name, index, S, Hp, Wp, b, T, rho_q, shift; rho_kv
TIES = [
    (Workload("ties_block16", 48, 4, 8, 8, 4, 1, 0.5, 1, H=2), 0.25),            # k = 8 / 12
    (Workload("ties_block294", 49, 6, 14, 14, 7, 6, 0.6, 1, H=2), 0.3),          # 10 tiles of 32 over 8 waves
    (Workload("ties_block384", 50, 6, 16, 16, 8, 6, 0.6, 1, H=2), 0.3),
    (Workload("ties_block448", 51, 7, 16, 16, 8, 7, 0.7, 1, H=2), 0.4),
]
TOPR_TIES = [
    Workload("topr_ties_block16", 52, 4, 8, 8, 4, 1, 0.5, 1, H=2, dst_frac=0.25),
    Workload("topr_ties_block64", 53, 4, 16, 16, 4, 4, 0.5, 1, H=2, dst_frac=0.25),
    Workload("topr_ties_block384", 54, 6, 16, 16, 8, 6, 0.5, 1, H=2, dst_frac=0.25),
]


@pytest.mark.parametrize("w,rho_kv", TIES, ids=[w.name for w, _ in TIES])
def test_exact_ties(w, rho_kv):
    test_gpu_ties.test_exact_ties_and_zero_vectors_follow_the_lowest_cluster_rule(w, rho_kv)


@pytest.mark.parametrize("w", TOPR_TIES, ids=lambda w: w.name)
def test_exact_ties_under_the_general_rule(w):
    test_gpu_ties.test_top_r_selection_breaks_ties_at_its_boundary_by_position(w)


@pytest.mark.parametrize("n", [1, 2, 15, 17])
def test_layer_in_blocks_around_sixteen_tokens(n):
    test_gpu_random_geometries._check_layer(_runs_of(n), 0.5, "headwise", n % 2 == 0)


@pytest.mark.parametrize("n", [15, 16, 17, 48, 63])
def test_top_r_rule_in_blocks_of_one_wave(n):
    test_gpu_topr.test_top_r_rule_matches_the_oracle(_runs_of(n, dst_frac=0.25), "headwise")
