"""Host-side check of the tiles stage 3 (Eq. 3-4) runs a launch in (httm_attention_route evaluates the launch's own
decision): the launches take every row of every head exactly once, in tiles whose edges stage 4 at their end can look
up, and many rows against few keys run in two launches.  No GPU needed."""
import numpy as np
import pytest

import paper_2511_21317_amd as httm
from test_gpu_layer_unmerge import CASES, FILTERED


def _check_rows(mq, mk, scratch_bytes=None):
    qo, ko = ([int(x) for x in np.concatenate([[0], np.cumsum(n)])] for n in (mq, mk))
    r = httm.attention_route(qo, ko, 256, scratch_bytes)
    for h, m in enumerate(mq):
        end = 0
        for launch in range(len(r["tiles"])):
            first, count = (int(x) for x in r["rows"][launch, h])
            if count == 0:
                continue
            assert first == end and first % 32 == 0, (h, launch, first, end)
            end = first + count
        assert end == m
    return r


def _layer_rows(case):
    name, S, Hp, Wp, b, T, rho_q, rho_kv, H, opts = case
    s = httm.geom_sizes(httm.make_geom(S, Hp, Wp, b, T, rho_q, rho_kv, H=H, **opts))
    return [int(s.M_q)] * H, [int(s.M_k)] * H


# the cases of test_gpu_layer_unmerge.py that are there for the tiles their names begin with
KINDS = ("groups128_wide", "groups128", "groups32", "groups64", "groups256", "tiles128", "segments", "rounds")
BY_KIND = [(c, next(kind for kind in KINDS if c[0].startswith(kind))) for c in CASES + FILTERED if c[0].startswith(KINDS)]


def test_every_kind_of_tile_has_a_layer():
    assert {kind for _, kind in BY_KIND} == set(KINDS)


@pytest.mark.parametrize("case,kind", BY_KIND, ids=["-".join(str(x) for x in c[:1] + c[9:]) for c, _ in BY_KIND])
def test_layers_run_in_the_tiles_their_names_say(case, kind):
    mq, mk = _layer_rows(case)
    r = _check_rows(mq, mk)
    off = lambda n: [h * n[0] for h in range(len(n) + 1)]  # noqa: E731
    if kind == "rounds":
        # the second launch begins inside heads: their first rows ran in the first one
        assert len(r["tiles"]) == 2 and r["tiles"][0] == "tiles256"
        assert ((r["rows"][1, :, 0] > 0) & (r["rows"][1, :, 1] > 0)).any()
        if "head_in_both" in case[0]:
            assert ((r["rows"][0, :, 1] > 0) & (r["rows"][1, :, 1] > 256)).any()
    elif kind == "segments":
        assert r["tiles"] == ["tiles256"] and httm.attention_split_plan(off(mq), off(mk))["n_tiles"] > 0
    else:
        assert r["tiles"] == [kind]


# many queries against few keys, in layers: frames, grid, block, frames a block, merged shares, heads
@pytest.mark.parametrize("geom", [(32, 21, 37, 8, 4, 0.6, 0.9, 16), (32, 28, 18, 4, 2, 0.38, 0.89, 16), (19, 28, 37, 4, 2, 0.5, 0.9, 16)])
def test_layers_of_many_rows_and_few_keys_take_every_row_once(geom):
    mq, mk = _layer_rows(("", *geom, {}))
    assert len(_check_rows(mq, mk)["tiles"]) == 2


@pytest.mark.parametrize("seed", range(100))
def test_random_launches_take_every_row_once(seed):
    rng = np.random.default_rng(4700 + seed)
    H = int(rng.integers(1, 25))
    if seed % 2:
        mq, mk = [int(rng.integers(1, 16000))] * H, [int(rng.integers(1, 4000))] * H
    else:
        mq, mk = ([int(x) for x in rng.integers(0, n, H)] for n in (16000, 4000))
    _check_rows(mq, mk)
    _check_rows(mq, mk, 0)


# heads, rows, keys of launches whose segments would need more than the 32 MiB of httm_attention_log2_static: in key
# groups where those are no slower, which need nothing of it (None: segments, refused there)
@pytest.mark.parametrize("H,mq,mk,tiles", [(1, 29824, 35072, "groups128_wide"), (2, 15376, 33474, "groups128_wide"),
                                           (32, 950, 86828, "groups128_wide"), (8, 3935, 91614, "groups128_wide"),
                                           (1, 55294, 21770, "groups256"), (24, 2346, 56082, "groups256"),
                                           (1, 456 * 256, 20000, None), (1, 10418, 105994, None), (27, 557, 48900, None)])
def test_launches_with_long_segments_run_in_key_groups_where_they_are_no_slower(H, mq, mk, tiles):
    off = lambda n: [h * n for h in range(H + 1)]  # noqa: E731
    r, p = _check_rows([mq] * H, [mk] * H), httm.attention_split_plan(off(mq), off(mk))
    if tiles:
        assert r["tiles"] == [tiles] and p["slots"] == 0
    else:
        assert r["tiles"] == ["tiles256"] and p["slots"] * 256 * 66 * 4 > 32 << 20


# few rows a head against many keys, where key groups would read every head's keys once per tile: in segments; and a
# launch whose 64-row tiles fit the CUs but not, as they are dealt out, the first XCD's
@pytest.mark.parametrize("H,mq,mk,segments", [(24, 68, 6785, True), (64, 90, 19556, True), (32, 141, 8058, True), (16, 41, 4702, True),
                                              (3, 5423, 23452, True), (16, 250, 3000, False), (12, 929, 4000, False)])
def test_few_rows_a_head(H, mq, mk, segments):
    off = lambda n: [h * n for h in range(H + 1)]  # noqa: E731
    assert (httm.attention_split_plan(off(mq), off(mk))["n_tiles"] > 0) == segments
    assert (_check_rows([mq] * H, [mk] * H)["tiles"] == ["tiles256"]) == segments


# against two key tiles: heads of at most 64 rows leave half of a 128-row tile's waves idle, longer ones do not; full tiles
# of many heads look theirs up
@pytest.mark.parametrize("H,mq,mk,tiles", [(16, 40, 73, "tiles128"), (32, 64, 128, "tiles128"), (48, 43, 65, "tiles128"), (16, 65, 128, "groups32"),
                                           (64, 66, 69, "tiles128"), (3, 181, 80, "groups32"),
                                           (16, 200, 100, "groups32"), (16, 40, 129, "groups32"), (16, 500, 64, "tiles128")])
def test_few_rows_against_few_keys(H, mq, mk, tiles):
    assert _check_rows([mq] * H, [mk] * H)["tiles"] == [tiles]
