"""Stage 2 at the block sizes where its kernel instances meet (32, 64, 128, ... 512 tokens, and one token to
either side): runs of n patch tokens of one frame, the last run of a frame partial.  The checks are
those of the tests of the whole layer, of the general rule and of the outlier filter."""
import pytest

import test_gpu_outliers
import test_gpu_random_geometries
import test_gpu_topr
from synth.vggt_tokens import Workload

pytestmark = pytest.mark.gpu

EDGES = [16, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 319, 320, 321, 383, 384, 385, 447, 448,
         449, 511, 512]


def _runs_of(n, dst_frac=0.0):
    # two frames of two whole runs and a partial one of a third of a run
    Wp = 16
    Hp = -(-(2 * n + n // 3) // Wp)
    return Workload(f"runs_of_{n}", 2000 + n, 2, Hp, Wp, n, 1, 0.6, 1, H=2, n_special=5, chunked=True, dst_frac=dst_frac)


@pytest.mark.parametrize("n", EDGES)
def test_layer_at_instance_edges(n):
    test_gpu_random_geometries._check_layer(_runs_of(n), 0.75, "headwise", n % 2 == 0)


@pytest.mark.parametrize("n", [32, 33, 65, 192, 300, 512])
def test_head_uniform_layer_at_instance_edges(n):
    test_gpu_random_geometries._check_layer(_runs_of(n), 0.5, "uniform", True)


@pytest.mark.parametrize("n", [31, 32, 64, 65, 128, 192, 193, 320, 384, 448, 512])
def test_top_r_rule_at_instance_edges(n):
    test_gpu_topr.test_top_r_rule_matches_the_oracle(_runs_of(n, dst_frac=0.25), "headwise")


@pytest.mark.parametrize("n", [32, 33, 65, 128, 192, 193, 320, 384, 448, 512])
def test_outlier_filter_at_instance_edges(n):
    test_gpu_outliers.test_filtered_stages_match_the_oracle(_runs_of(n), 0.1)
