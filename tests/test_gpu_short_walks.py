"""The short-launch kernels (64 rows per workgroup, 32 for dk and dv; four waves that take every fourth 32-row block of the
list, the forward two blocks at a time) at the edges of their tiles, blocks and shares, against the fp64 oracle.  Bars as
everywhere on the bf16 path: out 2e-2 / 2e-3, lse per row (see gpu_util), gradients by the size of the terms an element is
a sum of (the bound of the random problems in test_gpu_random_shapes)."""
import numpy as np
import pytest

import helpers
from gpu_util import check_lse_bf16, error_stats, make_qkv, to_device, to_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2403_09195_amd import binding
    binding.lib()
    return binding


EDGES = [(n, [(n, 1)]) for n in (1, 31, 33, 64, 65, 96, 127, 129, 161, 256, 257, 2016, 2048)] + [
    (2080, [(2080, 1)]),                           # one block more than the forward takes: the split launch
    (128, [(64, 1), (96, 1)]),                     # a full block or two for some rows, more for others
    (130, [(65, 2)]),                              # one block and one row, uncovered rows
    (384, [(96, 1), (192, 2), (384, 4)]),          # row groups that share a tile, skipping blocks, several multiplicities
    (300, [(20, 1), (60, 3), (300, 5)]),           # many groups of a few rows, many progressions of a few keys
]


@pytest.mark.parametrize("N,branches", EDGES)
@pytest.mark.parametrize("packed", [False, True])
def test_edges(B, oracle, N, branches, packed):
    import torch
    from paper_2403_09195_amd import synth
    # one full step is a short walk in 256-row tiles too, and faster there
    forward = {64: B.FORM_TILES, 2080: B.FORM_SPLIT}.get(N, B.FORM_SHORT)
    assert B.launch_describe(2, 3, N, branches)["form"] == forward
    assert B.launch_describe(2, 3, N, branches, backward=True)["form"] == B.FORM_SHORT
    (q, k, v), ex = make_qkv(1300 + N, 2, N, 3, 64, "bf16")
    if packed:                                     # views of one buffer, row pitch 3 * H * D
        q, k, v = torch.stack((q, k, v), dim=2).unbind(2)
    out, lse = B.forward(q, k, v, branches, 0.125)
    o_ref, l_ref = oracle.forward(*ex, branches, 0.125)
    mx, mean = error_stats(to_f64(out), o_ref)
    assert mx <= 2e-2 and mean <= 2e-3, (mx, mean)
    check_lse_bf16(to_f64(lse), oracle, ex, branches, 0.125, l_ref)
    st, ge = synth.tensor(1300 + N, 7, (2, N, 3, 64), "bf16")
    grads = B.backward(q, k, v, out, lse, to_device(st), branches, 0.125)
    refs = oracle.backward(*ex, ge, branches, 0.125)
    bounds = helpers.multiset_attention_backward(*ex, ge, 0.125, branches)[3:]
    dead = np.isneginf(l_ref).transpose(0, 2, 1)
    eps = 2.0 ** -9
    for name, got, ref, absum in zip(("dq", "dk", "dv"), grads, refs, bounds):
        d = np.abs(to_f64(got) - ref)
        assert np.all(d <= 2.0 ** -8 * np.abs(ref) + 4 * eps * absum + 1e-6), name
        assert d.mean() <= eps * absum.mean() + 1e-7, name
        assert np.all(to_f64(got)[dead] == 0.0)


@pytest.mark.parametrize("N", [33, 96, 100, 160])
def test_infinite_value_stays_in_its_column(B, N):
    """A value row of infinities at the end of a list whose blocks, or whose shares, are not filled: its own column is
    infinite, and the slots past the end make no NaN of it."""
    import torch
    assert B.launch_describe(1, 1, N, [(N, 1)])["form"] == B.FORM_SHORT
    (q, k, v), _ = make_qkv(78, 1, N, 1, 64, "bf16")
    v[:, N - 1, :, 5] = float("inf")
    out, lse = B.forward(q, k, v, [(N, 1)], 0.125)
    assert bool(torch.isposinf(out[..., 5]).all())
    rest = torch.cat((out[..., :5], out[..., 6:]), dim=-1)
    assert bool(torch.isfinite(rest).all()) and bool(torch.isfinite(lse).all())


def test_one_key_carries_the_row(B, oracle):
    """Scores of very different size (scale 4): reference exponents that move late, waves whose share weighs nothing."""
    (q, k, v), ex = make_qkv(1400, 1, 384, 2, 64, "bf16")
    branches = [(96, 1), (384, 3)]
    assert B.launch_describe(1, 2, 384, branches)["form"] == B.FORM_SHORT
    out, lse = B.forward(q, k, v, branches, 4.0)
    o_ref, l_ref = oracle.forward(*ex, branches, 4.0)
    # a weight is off by 2^-8 at most, an output by that times its two largest values (|v| <= 4.5) and its own rounding
    assert np.abs(to_f64(out) - o_ref).max() <= 2.0 ** -8 * (2 * 4.5 + 4.5)
    assert np.abs(to_f64(lse) - l_ref).max() <= 3.95e-3 + 4e-6 * np.abs(l_ref).max()


@pytest.mark.parametrize("N,form", [(8133, "short"), (8160, "short"), (8192, "short"), (8193, "tiles"), (8224, "tiles")])
def test_backward_of_the_longest_lists(B, N, form):
    """255 and 256 blocks, the most a short launch takes (64 records a wave), and 257, which go to the general kernels:
    against fp64 by the definition, bounds as in test_edges."""
    import torch
    assert B.launch_describe(1, 1, N, [(N, 1)], backward=True)["form"] == {"short": B.FORM_SHORT, "tiles": B.FORM_TILES}[form]
    (q, k, v), _ = make_qkv(1500, 1, N, 1, 64, "bf16")
    g = torch.empty_like(q).normal_(generator=torch.Generator(device="cuda").manual_seed(8))
    out, lse = B.forward(q, k, v, [(N, 1)], 0.125)
    grads = B.backward(q, k, v, out, lse, g, [(N, 1)], 0.125)
    q6, k6, v6, g6 = (t[0, :, 0].double() for t in (q, k, v, g))
    p = torch.softmax(0.125 * (q6 @ k6.T.contiguous()), 1)
    go = g6 * (p @ v6)
    dp = g6 @ v6.T.contiguous()
    ds = 0.125 * p * (dp - go.sum(1, keepdim=True))
    w = 0.125 * p * (dp.abs() + go.abs().sum(1, keepdim=True))
    refs = (ds @ k6, ds.T.contiguous() @ q6, p.T.contiguous() @ g6)
    sums = (w @ k6.abs(), w.T.contiguous() @ q6.abs(), p.T.contiguous() @ g6.abs())
    eps = 2.0 ** -9
    for name, got, ref, absum in zip(("dq", "dk", "dv"), grads, refs, sums):
        d = (got[0, :, 0].double() - ref).abs()
        assert bool((d <= 2.0 ** -8 * ref.abs() + 4 * eps * absum + 1e-6).all()), name
        assert float(d.mean()) <= eps * float(absum.mean()) + 1e-7, name


def test_backward_launch_of_more_than_one_slice(B):
    """More tiles than one slice of the launch takes (2^19): every gradient as from four calls of a quarter of the images,
    bit for bit (a tile's arithmetic does not depend on the launch around it)."""
    import torch
    Bsz, N, H, branches = 5600, 1024, 3, [(32, 1), (1024, 1)]
    whole = B.launch_describe(Bsz, H, N, branches, backward=True)
    quarter = B.launch_describe(Bsz // 4, H, N, branches, backward=True)
    assert whole["form"] == quarter["form"] == B.FORM_SHORT and whole["n_items"] > 2 ** 19 > quarter["n_items"]
    gen = torch.Generator(device="cuda").manual_seed(31)
    q, k, v, g = (torch.empty((Bsz, N, H, 64), dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(4))
    out, lse = B.forward(q, k, v, branches, 0.125)
    grads = B.backward(q, k, v, out, lse, g, branches, 0.125)
    for b in range(0, Bsz, Bsz // 4):
        sl = slice(b, b + Bsz // 4)
        for got, ref in zip(grads, B.backward(q[sl], k[sl], v[sl], out[sl], lse[sl], g[sl], branches, 0.125)):
            assert torch.equal(got[sl], ref), b
    assert all(bool(torch.isfinite(t[-1].float()).all()) for t in grads)


# Backward tiles of a few rows, without a second dk/dv workgroup (33 rows: with one), and lists of one to twelve blocks, so that no wave, some or
# all have one.  A call of NaN before it leaves them in LDS, where the places of rows and waves are that the call does not fill.
@pytest.mark.parametrize("Bsz,N,branches,most", [
    (3, 7, [(3, 1), (7, 2)], 2), (3, 32, [(32, 1)], 32), (3, 33, [(33, 1)], 33), (3, 34, [(4, 1), (8, 2), (17, 4), (34, 8)], 2), (3, 64, [(16, 1), (64, 1)], 16),
    (3, 96, [(24, 1), (96, 1)], 24), (3, 160, [(32, 1), (160, 1)], 32), (3, 165, [(33, 1), (165, 1)], 33), (3, 340, [(17, 1), (340, 1)], 17),
    (105, 33, [(33, 1)], 33), (110, 63, [(63, 1)], 63), (102, 64, [(64, 1)], 64),          # images of a tile each, more than a round of them
])
def test_backward_of_tiles_of_few_rows(B, oracle, Bsz, N, branches, most):
    from paper_2403_09195_amd import synth
    import torch
    plan = B.launch_describe(Bsz, 5, N, branches, backward=True, arrays=True)
    assert plan["form"] == B.FORM_SHORT and int(plan["tiles"][:, 2].max()) == most
    assert plan["threads"] == 256 * (2 if most <= 32 else 3) * plan["n_items"]
    (q, k, v), ex = make_qkv(1600 + N, Bsz, N, 5, 64, "bf16")
    out, lse = B.forward(q, k, v, branches, 0.125)
    st, ge = synth.tensor(1600 + N, 7, (Bsz, N, 5, 64), "bf16")
    nan = torch.full((4, 1024, 6, 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    assert B.launch_describe(4, 6, 1024, [(1024, 1)], backward=True)["form"] == B.FORM_SHORT
    B.backward(nan, nan, nan, nan, nan[..., 0].transpose(1, 2).float().contiguous(), nan, [(1024, 1)], 0.125)
    grads = B.backward(q, k, v, out, lse, to_device(st), branches, 0.125)
    refs = oracle.backward(*ex, ge, branches, 0.125)
    bounds = helpers.multiset_attention_backward(*ex, ge, 0.125, branches)[3:]
    eps = 2.0 ** -9
    for name, got, ref, absum in zip(("dq", "dk", "dv"), grads, refs, bounds):
        d = np.abs(to_f64(got) - ref)
        assert np.all(d <= 2.0 ** -8 * np.abs(ref) + 4 * eps * absum + 1e-6), name
        assert d.mean() <= eps * absum.mean() + 1e-7, name


# launches of more than a round of workgroups: in place of whole tiles (ragged, offsets) and of a split launch
@pytest.mark.parametrize("Bsz,H,N,branches,offs", [
    (3, 6, 2053, [(511, 1), (1029, 3), (2053, 5)], [[(3 * h + x + 1) % r for h in range(6)] for x, r in enumerate((1, 3, 5))]),
    (1, 16, 2170, [(271, 1), (542, 2), (1085, 4), (2170, 8)], None),
])
def test_two_rounds_of_row_groups(B, oracle, Bsz, H, N, branches, offs):
    plan = B.launch_describe(Bsz, H, N, branches, offs, arrays=True)
    assert plan["form"] == B.FORM_SHORT and plan["n_items"] > 576
    (q, k, v), ex = make_qkv(1700 + N, Bsz, N, H, 64, "bf16")
    out, lse = B.forward(q, k, v, branches, 0.125, offs)
    o_ref, l_ref = oracle.forward(*ex, branches, 0.125, offs)
    mx, mean = error_stats(to_f64(out), o_ref)
    assert mx <= 2e-2 and mean <= 2e-3, (mx, mean)
    check_lse_bf16(to_f64(lse), oracle, ex, branches, 0.125, l_ref, offs)


def _attends(N, H, branches, offs, t):
    """[H, N]: does row n of head h hold token t as a key (the definition, branch by branch)?"""
    n = np.arange(N)
    res = np.zeros((H, N), dtype=bool)
    for h in range(H):
        for x, (w, r) in enumerate(branches):
            o = offs[x][h] if offs else h % r
            pos = n % w - o
            kept = (pos >= 0) & (pos % r == 0)
            if kept[t]:
                res[h] |= kept & (n // w == t // w)
    return res


# Tiles whose 32-row blocks walk keys that only some of them attend to: the rests of row groups (an 800^2 image; ragged, offsets) and small
# groups.  What is not finite at such a key reaches exactly the rows that hold it.
@pytest.mark.parametrize("Bsz,H,N,branches,offs", [
    (6, 2, 2500, [(625, 1), (1250, 2), (2500, 4)], None),
    (3, 6, 1500, [(400, 1), (750, 3), (1500, 5)], [[(3 * h + x + 1) % r for h in range(6)] for x, r in enumerate((1, 3, 5))]),
    (1, 4, 256, [(64, 1), (128, 2), (256, 4)], None),
])
def test_not_finite_stays_with_the_rows_that_hold_it(B, oracle, Bsz, H, N, branches, offs):
    plan = B.launch_describe(Bsz, H, N, branches, offs, arrays=True)
    assert plan["form"] == B.FORM_SHORT and plan["packed"]
    skipped = [int(plan["segs"][s, 0]) for h, _, nrows, seg, nseg, _ in plan["tiles"] for s in range(seg, seg + nseg)
               if any(plan["block_mult"][s, x] == 0 for x in range((nrows + 31) // 32))]
    t = skipped[len(skipped) // 2]
    (q, k, v), ex = make_qkv(1800 + N, Bsz, N, H, 64, "bf16")
    o_ref, l_ref = oracle.forward(*ex, branches, 0.125, offs)
    holds = _attends(N, H, branches, offs, t).T                       # [N, H]
    assert holds.any() and not holds.all()
    for value in (float("inf"), float("nan")):
        bad = v.clone()
        bad[:, t, :, 7] = value
        out, lse = (to_f64(x) for x in B.forward(q, k, bad, branches, 0.125, offs))
        check_lse_bf16(lse, oracle, ex, branches, 0.125, l_ref, offs)
        d = np.abs(np.delete(out - o_ref, 7, axis=3))
        assert d.max() <= 2e-2 and d.mean() <= 2e-3
        assert np.abs((out - o_ref)[:, ~holds]).max() <= 2e-2 and not np.isfinite(out[:, holds][..., 7]).any()
        bad = k.clone()
        bad[:, t, :, 7] = value
        out, lse = (to_f64(x) for x in B.forward(q, bad, v, branches, 0.125, offs))
        assert np.abs((out - o_ref)[:, ~holds]).max() <= 2e-2
        assert np.abs(lse - l_ref)[:, ~holds.T][np.isfinite(l_ref[:, ~holds.T])].max() <= 3.95e-3 + 4e-6 * np.abs(l_ref[np.isfinite(l_ref)]).max()
        if value != value:
            assert np.isnan(out[:, holds]).all() and np.isnan(lse[:, holds.T]).all()
