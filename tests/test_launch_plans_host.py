"""Which kernel form a call takes, and the plan it is launched with, through dfa_launch_describe: 64-row tiles of the
short launches, 32-row tiles and cut lists of the fp32 kernels, split and packed launches, all against the operator's
definition.  Host code only: nothing here launches a kernel."""
import os

import numpy as np
import pytest

import helpers


@pytest.fixture(scope="module")
def B():
    from paper_2403_09195_amd import binding, build
    if not os.path.exists(build.LIB_PATH):
        build.build()
    binding.lib()
    return binding


def _check_launched_plan(B, Bsz, H, N, branches, offs, dtype_code, backward):
    """Every row is stored by one slot of one tile, and the multiplicities of the keys its 32-row block walks are those of
    the definition; blocks, tiles and items are within what the form's kernels take."""
    p = B.launch_describe(Bsz, H, N, branches, offs, dtype_code, backward, arrays=True)
    rows, segs, bm = p["rows"], p["segs"], p["block_mult"]
    short = p["form"] == B.FORM_SHORT
    assert p["threads"] < 2 ** 32
    forward_bf16 = dtype_code == B.DFA_BF16 and not backward
    most_blocks = None if not short else 64 if forward_bf16 else 256
    mult = [helpers.multiplicity_matrix(N, h, branches, offs) for h in range(H)]
    seen = np.zeros((H, N), dtype=np.int32)
    for (h, rb, nr, sb, ns, _) in p["tiles"]:
        assert 1 <= nr <= (64 if short else 256)
        if p["cut"]:
            assert most_blocks is None or ns <= most_blocks
            lst = segs[sb:sb + ns]
            assert np.all((lst[:, 2] >= 1) & (lst[:, 2] <= 32)) and np.all(lst[lst[:, 2] == 1, 1] == 0)
        tile_rows = rows[rb:rb + nr]
        assert forward_bf16 or np.all(tile_rows >= 0)                # only the bf16 forward packs tiles
        for blk in range((nr + 31) // 32):
            mine = np.zeros(N, dtype=np.int64)
            for s in range(sb, sb + ns):
                key0, stride, count, m = (int(x) for x in segs[s])
                m = int(bm[s, blk]) if forward_bf16 else m
                assert 0 <= key0 and key0 + stride * (count - 1) < N
                mine[key0 + stride * np.arange(count)] += m
            slots = tile_rows[32 * blk:32 * blk + 32]
            real = slots[slots >= 0]
            seen[h, real] += 1
            assert np.all(mult[h][np.where(slots < 0, ~slots, slots)] == mine)
    assert np.all(seen == 1)
    live = p["items"][p["items"][:, 0] >= 0]
    assert len(p["items"]) % 8 == 0 and len(set(map(tuple, live.tolist()))) == len(live) == len(p["tiles"]) * Bsz
    return p


PROBLEMS = [
    (1, 12, 256, [(64, 1), (128, 2), (256, 4)], None),
    (3, 6, 1500, [(400, 1), (750, 3), (1500, 5)], [[(3 * h + x + 1) % r for h in range(6)] for x, r in enumerate((1, 3, 5))]),
    (1, 3, 1000, [(625, 1), (1250, 2), (2500, 4)], None),
    (2, 2, 130, [(65, 2)], None),                                    # uncovered rows
    (40, 2, 96, [(32, 4), (96, 1)], None),
    (2, 3, 50, [(16, 3), (7, 2), (64, 5)], None),
    (1, 2, 1025, [(1024, 1), (300, 7)], [[0, 0], [6, 2]]),
    (1, 2, 512, [(256, 2), (256, 2), (512, 1)], None),               # keys that count double
    (600, 1, 64, [(64, 1)], None),
    (1, 1, 2100, [(2100, 1)], None),                                 # a list of 66 blocks
]


# A little more than one round of 64-row workgroups: the rests of row groups share tiles where that saves the second round
# (six 800^2 images of two heads: 528 -> 480 workgroups; three of 1500 tokens: 540 -> at most 512), or than one workgroup to a CU.
@pytest.mark.parametrize("Bsz,H,N,branches,offs,most", [
    (6, 2, 2500, [(625, 1), (1250, 2), (2500, 4)], None, 512),
    (3, 6, 1500, [(400, 1), (750, 3), (1500, 5)], [[(3 * h + x + 1) % r for h in range(6)] for x, r in enumerate((1, 3, 5))], 512),
    (3, 2, 2500, [(625, 1), (1250, 2), (2500, 4)], None, 256),
])
def test_rests_of_row_groups_share_tiles(B, Bsz, H, N, branches, offs, most):
    p = _check_launched_plan(B, Bsz, H, N, branches, offs, B.DFA_BF16, False)
    assert p["form"] == B.FORM_SHORT and p["packed"] and p["n_items"] <= most


# Launches of 577 to 1152 workgroups of 64 rows: the short form where its estimate is the shorter one, the form of before elsewhere
# (one image: split; windows: whole tiles; lists of few steps: packed tiles; one workgroup more than fits).
@pytest.mark.parametrize("Bsz,H,N,branches,offs,form", [
    (2, 8, 2107, [(526, 1), (1053, 2), (2107, 4)], None, "SHORT"),
    (3, 6, 2053, [(511, 1), (1029, 3), (2053, 5)], [[(3 * h + x + 1) % r for h in range(6)] for x, r in enumerate((1, 3, 5))], "SHORT"),
    (1, 12, 4096, [(1024, 1), (2048, 2), (4096, 4)], None, "SPLIT"), (1, 20, 2048, [(512, 1), (1024, 2), (2048, 4)], None, "SPLIT"),
    (1, 16, 2170, [(271, 1), (542, 2), (1085, 4), (2170, 8)], None, "SHORT"),
    (3, 8, 1441, [(288, 1)], None, "TILES"),
    (16, 8, 505, [(126, 1), (252, 2), (505, 4)], None, "TILES"),
    (1153, 1, 64, [(64, 1)], None, "TILES"),
])
def test_launches_of_two_rounds_of_row_groups(B, Bsz, H, N, branches, offs, form):
    p = B.launch_describe(Bsz, H, N, branches, offs)
    if N == 2053: _check_launched_plan(B, Bsz, H, N, branches, offs, B.DFA_BF16, False)
    assert p["form"] == getattr(B, "FORM_" + form)
    assert form != "SHORT" or 576 < p["n_items"] <= 1152


# Where the estimates choose: part-filled tiles go to the short form, split or not; tiles of one step stay, and so do workgroups with keys that fit one
# round beside many without.
@pytest.mark.parametrize("Bsz,H,N,branches,form", [
    (7, 3, 1152, [(144, 1), (288, 2), (576, 4), (1152, 8)], "SHORT"), (1, 8, 4736, [(1184, 3)], "SHORT"), (3, 12, 1024, [(256, 1), (512, 2), (1024, 4)], "SHORT"), (6, 12, 1024, [(256, 1), (512, 2), (1024, 4)], "TILES"),
    (7, 16, 133, [(33, 1), (66, 2), (133, 4)], "TILES"), (23, 4, 98, [(12, 1), (24, 2)], "TILES"), (10, 9, 66, [(8, 1), (16, 2)], "TILES"),
    (16, 8, 298, [(149, 3)], "TILES"), (6, 6, 256, [(32, 1)], "TILES"), (6, 8, 1280, [(640, 2)], "TILES"), (10, 6, 959, [(191, 1)], "TILES"),
])
def test_form_with_the_shorter_estimate(B, Bsz, H, N, branches, form):
    p = _check_launched_plan(B, Bsz, H, N, branches, None, B.DFA_BF16, False)
    assert p["form"] == getattr(B, "FORM_" + form)


@pytest.mark.parametrize("Bsz,H,N,branches,form", [
    (8, 8, 326, [(40, 1)], "SHORT"), (2, 8, 3520, [(1173, 3)], "SHORT"), (4, 6, 1024, [(256, 1), (512, 2), (1024, 4)], "SHORT"),
    (64, 8, 64, [(64, 1)], "SHORT"), (256, 2, 33, [(33, 1)], "SHORT"), (400, 8, 64, [(64, 1)], "TILES"), (64, 8, 128, [(128, 1)], "TILES"), (16, 12, 4096, [(1024, 1), (2048, 2), (4096, 4)], "TILES"),
])
def test_backward_form_with_the_shorter_estimate(B, Bsz, H, N, branches, form):
    p = _check_launched_plan(B, Bsz, H, N, branches, None, B.DFA_BF16, True)
    assert p["form"] == getattr(B, "FORM_" + form)


# Sharing does not take a plan out of the short form: padded for the dies it would have 592 workgroups here, apart it has 568 (and the
# form in its place takes 1.4 times as long).
def test_sharing_does_not_leave_the_short_form(B):
    p = _check_launched_plan(B, 3, 6, 1222, [(305, 1), (611, 2), (1222, 4)], None, B.DFA_BF16, False)
    assert p["form"] == B.FORM_SHORT and p["n_items"] <= 576


@pytest.mark.parametrize("Bsz,H,N,branches,offs", PROBLEMS)
@pytest.mark.parametrize("dtype,backward", [("bf16", False), ("bf16", True), ("f32", False)])
def test_launched_plan_covers_the_definition(B, Bsz, H, N, branches, offs, dtype, backward):
    _check_launched_plan(B, Bsz, H, N, branches, offs, B.DFA_BF16 if dtype == "bf16" else B.DFA_F32, backward)


@pytest.mark.parametrize("seed", range(16))
def test_launched_plans_of_random_problems(B, seed):
    rng = np.random.default_rng(250 + seed)
    Bsz, H, N, nb = int(rng.integers(1, 40)), int(rng.integers(1, 7)), int(rng.integers(1, 500)), int(rng.integers(1, 6))
    branches, offs = [], []
    for _ in range(nb):
        r = int(rng.integers(1, 8))
        branches.append((int(rng.integers(1, 2 * N + 1)), r))
        offs.append([int(rng.integers(0, r)) for _ in range(H)])
    for code, backward in ((B.DFA_BF16, False), (B.DFA_BF16, True), (B.DFA_F32, False)):
        _check_launched_plan(B, Bsz, H, N, branches, offs if seed % 2 else None, code, backward)


def test_each_form_is_taken_where_it_should_be(B):
    """One shape per form, far from where the library's estimates meet."""
    sam = [(1024, 1), (2048, 2), (4096, 4)]
    form = lambda *a, **k: B.launch_describe(*a, **k)["form"]
    assert form(16, 12, 4096, sam) == B.FORM_TILES and form(16, 12, 4096, sam, backward=True) == B.FORM_TILES
    assert form(1, 12, 4096, sam) == B.FORM_SPLIT
    assert form(1, 6, 4096, sam) == B.FORM_SHORT and form(1, 6, 4096, sam, backward=True) == B.FORM_SHORT
    small = B.launch_describe(2, 6, 1024, [(256, 1), (512, 2), (1024, 4)], dtype_code=B.DFA_F32, arrays=True)
    assert small["cut"] and int(small["tiles"][:, 2].max()) == 32            # part-filled 256-row tiles: 32-row tiles
    one = B.launch_describe(1, 12, 4096, sam, dtype_code=B.DFA_F32, arrays=True)
    assert one["cut"] and int(one["tiles"][:, 2].max()) == 256
    assert not B.launch_describe(1, 1, 16384, [(16384, 1), (16, 1)], dtype_code=B.DFA_F32)["cut"]     # 2^19 blocks of lists


@pytest.mark.parametrize("Bsz,H,N,branches", [
    (1, 9, 4096, [(512, 1)]),            # 576 workgroups, a second round of them
    (6, 4, 1500, [(512, 1)]),
    (8, 16, 200, [(50, 1)]),             # 512 workgroups, lists of two blocks
    (3, 9, 1024, [(128, 1)]),            # lists of four
    (8, 2, 1024, [(256, 4)]),            # a single dilated branch, lists of one whole step
])
def test_short_lists_in_whole_tiles_keep_them(B, Bsz, H, N, branches):
    """Launches whose 256-row tiles walk a few steps and are done before the short form has merged its shares (measured
    1.2 to 1.6 times as long)."""
    assert B.launch_describe(Bsz, H, N, branches)["form"] == B.FORM_TILES


@pytest.mark.parametrize("Bsz,H,N,branches", [
    (1, 9, 4096, [(1024, 1), (2048, 2), (4096, 4)]),
    (3, 6, 1500, [(400, 1), (750, 3), (1500, 5)]),
    (2, 5, 2048, [(512, 1)]),
    (1, 12, 256, [(64, 1), (128, 2), (256, 4)]),
    (2, 2, 512, [(512, 1)]),
    (1, 1, 33, [(33, 1)]),               # one workgroup to a CU, lists that do not fill their last 64-key step
    (2, 7, 550, [(55, 1)]),
])
def test_launches_that_stay_with_the_short_form(B, Bsz, H, N, branches):
    assert B.launch_describe(Bsz, H, N, branches)["form"] == B.FORM_SHORT


def test_short_backward_of_millions_of_tiles_stays_within_a_grid(B):
    """60 000 images of 96 short tiles each, three workgroups of 256 threads per tile: more threads than one grid holds,
    so the launch has to come in slices."""
    d = B.launch_describe(60000, 3, 1024, [(32, 1), (1024, 1)], backward=True)
    assert d["form"] == B.FORM_SHORT and 3 * 256 * d["n_items"] >= 2 ** 32
    assert d["threads"] < 2 ** 32


@pytest.mark.parametrize("Bsz,H,N,branches,offs", PROBLEMS + [
    (1, 4, 2048, [(512, 1), (1024, 2), (2048, 4)], None),            # walks long enough to split, taken by the short form
    (3, 6, 1500, [(400, 1), (750, 3), (1500, 5)], None),
    (1, 20, 2048, [(512, 1), (1024, 2), (2048, 4)], None),           # split
    (1, 2, 4224, [(1056, 1), (2112, 2), (4224, 4)], None),
    (1, 12, 4096, [(1024, 1), (2048, 2), (4096, 4)], None),
])
def test_only_split_launches_ask_for_a_workspace(B, Bsz, H, N, branches, offs):
    """Partial results are written by split launches alone: no other form asks for room for them."""
    d = B.launch_describe(Bsz, H, N, branches, offs)
    need = B.workspace_bytes(Bsz, H, N, 64, B.DFA_BF16, branches, offs)
    assert need == (d["threads"] // 256 * 256 * (64 * 2 + 8) if d["form"] == B.FORM_SPLIT else 0)


# Fewer (image, head) units than the dies can be dealt evenly: every die has a run of tiles that follow one another, no longer than the others'.
@pytest.mark.parametrize("Bsz,H,N,branches,dtype,backward", [
    (1, 12, 4096, [(1024, 1), (2048, 2), (4096, 4)], "bf16", False), (1, 12, 2500, [(625, 1), (1250, 2), (2500, 4)], "bf16", True),
    (2, 6, 1024, [(256, 1), (512, 2), (1024, 4)], "f32", False), (3, 6, 1500, [(400, 1), (750, 3), (1500, 5)], "bf16", False),
])
def test_dies_take_runs_of_tiles(B, Bsz, H, N, branches, dtype, backward):
    p = B.launch_describe(Bsz, H, N, branches, None, B.DFA_BF16 if dtype == "bf16" else B.DFA_F32, backward, arrays=True)
    live = int(np.sum(p["items"][:, 0] >= 0))
    dies = []
    for d in range(8):
        items = [it for it in p["items"][d::8].tolist() if it[0] >= 0]
        assert len(items) in (live // 8, -(-live // 8))
        keys = sorted((b, int(p["tiles"][t][0]), int(p["rows"][p["tiles"][t][1]])) for t, b in (it[:2] for it in items))
        dies.append((keys[0], keys[-1]))
    assert all(a[1] <= b[0] for a, b in zip(dies, dies[1:]))


# bf16 forward, all workgroups at once: those that share a compute unit (i and i + 32 of a die's list) are a long and a short one, and a
# longest list that has a unit to itself exists wherever units are left over.
@pytest.mark.parametrize("Bsz,H,N,branches", [(2, 9, 467, [(116, 1), (233, 2), (467, 4)]), (3, 6, 1500, [(400, 1), (750, 3), (1500, 5)]),
                                              (4, 16, 211, [(26, 1), (52, 2), (105, 4), (211, 8)]), (1, 12, 256, [(64, 1), (128, 2), (256, 4)])])
def test_long_walks_share_a_unit_with_short_ones(B, Bsz, H, N, branches):
    p = B.launch_describe(Bsz, H, N, branches, arrays=True)
    for d in range(8):
        steps = [int(p["tiles"][it[0]][5]) for it in p["items"][d::8].tolist() if it[0] >= 0]
        assert len(steps) <= 64
        twos = max(len(steps) - 32, 0)
        alone, first, second = steps[twos:32], steps[:twos], steps[32:]
        assert alone == sorted(alone, reverse=True) and (not twos or not alone or min(alone) >= max(first + second))
        assert first == sorted(first, reverse=True) and second == sorted(second) and (not twos or first[-1] >= second[-1])


# What a split launch reads: its shares cover every item's steps once, each with a block of partial results of its own; every die has as many as the
# others, and no compute unit walks longer than if every length were dealt out in turn; and which of several tiles with equally long shares gets one more goes by the tiles (most pairs, then the
# first tile, then the first image; where units are dealt whole, every die's first unit before its second), not by where the launch runs them.
@pytest.mark.parametrize("Bsz,H,N,branches", [
    (1, 12, 4096, [(1024, 1), (2048, 2), (4096, 4)]),                # 32 tiles of 32 steps have four shares, 16 of them three
    (2, 6, 4096, [(1024, 1), (2048, 2), (4096, 4)]), (1, 20, 2048, [(512, 1), (1024, 2), (2048, 4)]),
    (1, 2, 4224, [(1056, 1), (2112, 2), (4224, 4)]), (4, 1, 8448, [(8448, 1)]), (4, 3, 4032, [(4032, 1)]), (1, 3, 9664, [(2416, 1), (4832, 2), (9664, 4)]),
    (2, 1, 8043, [(4021, 1)]),                                       # 256 shares of 15 or 16 steps, two of one step
    (1, 8, 6464, [(6464, 1)]), (2, 8, 3072, [(3072, 1)]),            # units dealt whole, one and two to a die
    (1, 8, 5568, [(1391, 1), (2778, 3), (5568, 5)]), (2, 10, 2486, [(2486, 1)]),
])
def test_shares_of_a_split_launch(B, Bsz, H, N, branches):
    p = B.launch_describe(Bsz, H, N, branches, arrays=True)
    image, data = B.launch_image(Bsz, H, N, branches)
    assert p["form"] == B.FORM_SPLIT and image["n_shares"] == p["threads"] // 256
    ints = lambda at, rows, cols: data[at:at + 4 * rows * cols].view(np.int32).reshape(rows, cols)
    tiles, items = p["tiles"], ints(image["items"], len(p["items"]), 8)
    assert np.array_equal(items[:, :2], p["items"])
    shares, share_items = ints(image["shares"], image["n_shares"], 3), ints(image["share_items"], image["n_shares"], 8)
    first, parts = ints(image["item_parts"], len(items), 2).T
    total = int(parts.sum())
    real = shares[:, 0] >= 0
    assert int(real.sum()) == total <= 512 and np.all(share_items[~real, 0] < 0) and len(shares) - total < 8
    assert np.array_equal(share_items[real], items[shares[real, 0]])
    assert sorted(shares[real, 2].tolist()) == list(range(total))                # a block each
    for item, part_nparts, block in shares[real].tolist():
        part, nparts = part_nparts & 0xffff, part_nparts >> 16
        assert nparts == parts[item] and 0 <= part < nparts and block == first[item] + part
    steps = tiles[np.maximum(items[:, 0], 0), 5]
    dies = [[int(steps[i]) / int(parts[i]) for i in shares[d::8, 0] if i >= 0] for d in range(8)]
    assert all(v == sorted(v, reverse=True) for v in dies) and max(map(len, dies)) - min(map(len, dies)) <= 1
    walks = lambda dies: max(sum(v[cu::32]) for v in dies for cu in range(min(32, len(v))))      # of a compute unit's workgroups
    in_turn = sorted(sum(dies, []), reverse=True)
    assert walks(dies) <= walks([in_turn[d::8] for d in range(8)])
    # the same by the rule
    pairs = np.zeros(len(tiles), dtype=np.int64)
    for t, (_, rb, nr, sb, ns, _) in enumerate(tiles.tolist()):
        slots = p["rows"][rb:rb + nr]
        rows = np.array([int((slots[32 * w:32 * w + 32] >= 0).sum()) for w in range(8)])
        pairs[t] = int((p["segs"][sb:sb + ns, 2].astype(np.int64) * ((p["block_mult"][sb:sb + ns] > 0) @ rows)).sum())
    units = Bsz * H
    if units >= 32 or (units >= 8 and -(-units // 8) * 64 <= 9 * units):
        def place(i):
            t, unit = items[i, 0], items[i, 1] * H + tiles[items[i, 0], 0]
            rank = int(sum(tiles[u, 0] == tiles[t, 0] and (-pairs[u], u) < (-pairs[t], t) for u in range(len(tiles))))
            return (tiles[t, 4] <= 1, unit // 8, rank, unit % 8)
    else:
        place = lambda i: (-pairs[items[i, 0]], items[i, 0], items[i, 1])
    live = sorted((i for i in range(len(items)) if items[i, 0] >= 0), key=place)
    want = np.zeros(len(items), dtype=np.int64)
    want[live] = 1
    while want.sum() < 512:
        able = [i for i in live if want[i] < 4 and steps[i] // (want[i] + 1) >= 8]
        if not able:
            break
        want[max(able, key=lambda i: -(-int(steps[i]) // int(want[i])))] += 1     # the first of the longest
    assert np.array_equal(want, parts)


# What a short forward reads, one record of start_bytes per workgroup: its item, the tokens of its 64 slots, and for each of the four waves the blocks
# wave, wave + 4, ... of the tile's list, then at least one record without a valid key (the last block again, for the copies that run ahead).
@pytest.mark.parametrize("Bsz,H,N,branches,offs", [(2, 3, 32 * n - 7, [(32 * n - 7, 1)], None) for n in range(1, 10)] + [
    (2, 3, 2048, [(2048, 1)], None),                                 # the longest lists: 16 records a wave
    (1, 12, 256, [(64, 1), (128, 2), (256, 4)], None),               # filler slots, skipped blocks, multiplicities up to 3
    (2, 3, 300, [(20, 1), (60, 3), (300, 5)], None),
    (2, 2, 130, [(65, 2)], None),                                    # rows without keys
    (3, 6, 1500, [(400, 1), (750, 3), (1500, 5)], [[(3 * h + x + 1) % r for h in range(6)] for x, r in enumerate((1, 3, 5))]),
    (6, 2, 2500, [(625, 1), (1250, 2), (2500, 4)], None),
])
def test_starts_of_a_short_forward(B, Bsz, H, N, branches, offs):
    p = B.launch_describe(Bsz, H, N, branches, offs, arrays=True)
    image, data = B.launch_image(Bsz, H, N, branches, offs)
    assert p["form"] == B.FORM_SHORT and len(data) == image["start_bytes"] * p["n_items"]
    longest = int(p["tiles"][:, 4].max())
    per_wave = -(-longest // 4) + 1
    assert image["start_bytes"] == 4 * (8 + 64) + 16 * 4 * per_wave and per_wave <= 64
    starts = data.reshape(p["n_items"], image["start_bytes"])
    for start, (tile, b) in zip(starts, p["items"].tolist()):
        item = start[:32].view(np.int32)
        assert item[0] == tile
        if tile < 0:
            continue
        assert item[1] == b and np.array_equal(item[2:], p["tiles"][tile])
        _, rb, nr, sb, ns, _ = p["tiles"][tile].tolist()
        assert np.array_equal(start[32:288].view(np.int32), p["rows"][rb + np.minimum(np.arange(64), nr - 1)])
        if ns == 0:
            assert not start[288:].any()
            continue
        ints = start[288:].view(np.uint32).reshape(4, per_wave, 4)
        mult = start[288:].view(np.float32).reshape(4, per_wave, 4)[:, :, 2:]
        with np.errstate(divide="ignore"):
            want = np.log2(p["block_mult"][sb:sb + ns, :2].astype(np.float32))
        for wave in range(4):
            mine = np.arange(wave, ns, 4)
            stride, count, turn = ints[wave, :, 1] & 0xffffff, ints[wave, :, 1] >> 24 & 0x3f, ints[wave, :, 1] >> 31
            assert len(mine) < per_wave                                          # every share is followed by one without keys
            n, segs = len(mine), p["segs"][sb + mine]
            assert np.array_equal(np.stack((ints[wave, :n, 0], stride[:n], count[:n])).T, segs[:, :3])
            assert np.array_equal(mult[wave, :n], want[mine])
            changes = np.any(want[mine][1:] != want[mine][:-1], axis=1)
            assert np.array_equal(turn[:n], np.concatenate(([True], changes))[:n] | (count[:n] < 32))
            last = mine[-1] if n else 0                                          # a valid source for copies, masked as a whole
            assert np.all(count[n:] == 0) and np.all(turn[n:] == 1)
            assert np.all(ints[wave, n:, 0] == p["segs"][sb + last, 0]) and np.all(stride[n:] == p["segs"][sb + last, 1])
            assert np.array_equal(mult[wave, n:], np.broadcast_to(want[last], (per_wave - n, 2)))
