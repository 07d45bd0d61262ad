"""Host-side check of stage 3's (Eq. 3-4) launches in 512-row tiles: which launches with log2 keys run in them, and that the
segments of the tiles in excess cover every (query row, key tile) pair once, in slots nobody else writes, inside the
scratch the library asks for.  No GPU needed."""
import numpy as np
import pytest

import paper_2511_21317_amd as httm

ROWS, SLOT_ROWS, SLOT_BYTES = 512, 256, 256 * 66 * 4


def _offsets(n):
    return [int(x) for x in np.concatenate([[0], np.cumsum(n)])]


def check_wide_plan(mq, mk, scratch_bytes=None):
    H = len(mq)
    p = httm.attention_wide_plan(_offsets(mq), _offsets(mk), 256, scratch_bytes)
    if p is None:
        return None
    full, ragged = [m // ROWS for m in mq], [h for h in range(H) if mq[h] % ROWS]
    T = sum(full) + len(ragged)
    assert T >= 256
    if p["n_tiles"] == 0:
        return p
    assert p["n_tiles"] == T % 256
    assert p["slots"] * SLOT_BYTES <= (httm.attention_scratch_bytes(H) if scratch_bytes is None else scratch_bytes)
    flat = [(h, t * ROWS) for h in range(H) for t in range(full[h])]
    tiles = [(h, full[h] * ROWS) for h in ragged[:p["split_ragged"]]] + flat[p["kept_full"]:]
    assert len(tiles) == p["n_tiles"]
    seen, owner, shares = {t: 0 for t in tiles}, {}, set()
    for share, h, q0, t0, t1, slot in p["segments"].tolist():
        kt, rows = -(-mk[h] // 64), min(ROWS, mq[h] - q0)
        assert t0 == seen[(h, q0)] and t0 < t1 <= kt + 1 and (t1 <= kt or rows <= SLOT_ROWS)     # in key order, without a gap
        seen[(h, q0)] = min(t1, kt)
        shares.add(share)
        for s in range(slot, slot + -(-rows // SLOT_ROWS)):
            assert s not in owner and s < p["slots"]
            owner[s] = share
    assert all(seen[(h, q0)] == -(-mk[h] // 64) for h, q0 in tiles)
    assert shares == set(range(p["shares"])) and p["shares"] <= 256
    return p


@pytest.mark.parametrize("H,mq,mk,n_tiles", [
    (16, 28650, 28650, 128), (16, 28700, 28700, 144), (16, 28700, 83140, 144), (16, 43968, 17600, 96), (16, 16384, 4096, 0),
    (16, 16384, 2000, None), (16, 5516, 5516, None), (16, 10992, 10992, None), (16, 9000, 9000, None), (16, 28700, 2048, None)])
def test_which_launches_run_in_512_row_tiles(H, mq, mk, n_tiles):
    p = check_wide_plan([mq] * H, [mk] * H)
    assert (p["n_tiles"] if p else None) == n_tiles


def test_one_tile_more_than_an_xcd_has_cus_is_another_round():
    """256 tiles, 246 full and 10 partial ones: the grid deals 31 and 2 of them to the first XCD's 32 CUs."""
    rows = [12900] * 9 + [11000]
    assert sum(-(-m // ROWS) for m in rows) == 256 and check_wide_plan(rows, [4000] * 10) is None
    assert check_wide_plan([12900] * 9 + [11264 - 512], [4000] * 10) is None       # 255: not a round
    assert check_wide_plan([16384] * 8, [16384] * 8)["n_tiles"] == 0               # 256 full ones: dealt evenly


def test_heads_of_few_tiles_against_few_keys_do_not():
    assert check_wide_plan([3685] * 40, [18667] * 40) is None
    assert check_wide_plan([3685] * 40, [45000] * 40)["n_tiles"] == 64


def test_heads_of_different_key_lengths_do_not():
    assert check_wide_plan([28700] * 16, [28700] * 15 + [30000]) is None
    assert check_wide_plan([28700] * 15 + [0], [28700] * 15 + [512]) is not None      # (a head without rows has no say)


def test_without_scratch_only_whole_rounds():
    assert check_wide_plan([28700] * 16, [28700] * 16, 0) is None
    assert check_wide_plan([16384] * 16, [16384] * 16, 0)["n_tiles"] == 0


@pytest.mark.parametrize("H,mq,mk", [(20, 8942, 50208), (16, 12404, 72887), (48, 3762, 63618), (16, 28700, 28700), (16, 28650, 28650), (16, 17600, 17600)])
def test_shares_take_equal_times(H, mq, mk):
    """A tile of at most 256 rows takes 0.62 of the time of a larger one per key tile (alone on a CU): shares of such tiles
    have that many key tiles more."""
    p = check_wide_plan([mq] * H, [mk] * H)
    time = np.zeros(p["shares"])
    for share, _, q0, t0, t1, _ in p["segments"].tolist():
        time[share] += (t1 - t0) * (0.62 if mq - q0 <= SLOT_ROWS else 1.0)
    assert time[:-1].max() <= 1.02 * time[:-1].mean() + 1, (time.max(), time[:-1].mean())


@pytest.mark.parametrize("rows,n_tiles,slots", [(28650, 128, 766), (28700, 144, 764), (29142, 144, 798), (30166, 176, 862), (31190, 208, 926), (23500, 224, 958)])
def test_a_plan_needs_room_for_all_its_slots(rows, n_tiles, slots):
    """Tiles in excess are cut if there is room for all of the plan's slots and not otherwise (then all tiles run whole, or none has
    512 rows); what the library asks for holds 767, which the plans of a quarter of the long launches exceed."""
    off = [h * rows for h in range(17)]
    p = check_wide_plan([rows] * 16, [rows] * 16, slots * SLOT_BYTES)
    assert (p["n_tiles"], p["slots"]) == (n_tiles, slots)
    cut = lambda q: q is not None and q["n_tiles"] > 0      # noqa: E731
    assert not cut(check_wide_plan([rows] * 16, [rows] * 16, slots * SLOT_BYTES - 1))
    assert cut(httm.attention_wide_plan(off, off)) == (slots <= 767)
    assert httm.attention_scratch_bytes(16) == 767 * SLOT_BYTES


@pytest.mark.parametrize("room", [None, 1020 * SLOT_BYTES], ids=["as_asked_for", "more"])
@pytest.mark.parametrize("family", ["equal", "ragged", "few_rows"])
def test_random_launches_are_covered_exactly_once(family, room):
    rng = np.random.default_rng({"equal": 51200, "ragged": 51300, "few_rows": 51400}[family])
    split = whole = 0
    for _ in range(400):
        H = int(rng.integers(1, 24))
        if family == "equal":
            mq, mk = [int(rng.integers(9000, 60000))] * H, [int(rng.integers(2048, 60000))] * H
        elif family == "ragged":      # some heads without rows
            mq = [max(0, int(x)) for x in rng.integers(-7000, 70000, H)]
            mk = [30000 + int(x) for x in rng.integers(0, 900, H)]
        else:                         # every head's last tile has at most 256 rows
            mq = [int(ROWS * rng.integers(10, 120) + rng.integers(1, 257)) for _ in range(H)]
            mk = [12000 + int(x) for x in rng.integers(0, 300, H)]
        p = check_wide_plan(mq, mk, room)
        split += p is not None and p["n_tiles"] > 0
        whole += p is not None and p["n_tiles"] == 0
        if split >= 40:
            break
    assert split >= 40, (split, whole)
