"""The fp32 kernels at the edges of their blocks (32 rows per workgroup, 32 walked rows per step, four waves that take
every fourth step) against the fp64 oracle.  Bars as everywhere on the fp32 path: 1e-5 on out and lse (sums of at most a
few hundred fp32 products, measured 1e-6), 2e-5 of the largest gradient."""
import numpy as np
import pytest

from gpu_util import check_lse, make_qkv, to_device, to_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2403_09195_amd import binding
    binding.lib()
    return binding


EDGES = [(n, [(n, 1)]) for n in (1, 31, 32, 33, 96, 127, 128, 129, 160, 257)] + [
    (130, [(65, 2)]),                              # one block and one row, uncovered rows
    (384, [(96, 1), (192, 2), (384, 4)]),          # progressions of several multiplicities, shorter than four blocks
    (320, [(40, 1), (320, 8)]),                    # many short progressions for some rows
]


@pytest.mark.parametrize("N,branches", EDGES)
@pytest.mark.parametrize("packed", [False, True])
def test_f32_edges(B, oracle, N, branches, packed):
    import torch
    from paper_2403_09195_amd import synth
    (q, k, v), ex = make_qkv(900 + N, 2, N, 3, 64, "f32")
    st, ge = synth.tensor(900 + N, 7, (2, N, 3, 64), "f32")
    g = to_device(st)
    if packed:                                     # views of one buffer, row pitch 3 * H * D
        q, k, v = torch.stack((q, k, v), dim=2).unbind(2)
    out, lse = B.forward(q, k, v, branches, 0.125)
    grads = B.backward(q, k, v, out, lse, g, branches, 0.125)
    o_ref, l_ref = oracle.forward(*ex, branches, 0.125)
    assert np.abs(to_f64(out) - o_ref).max() <= 1e-5
    check_lse(to_f64(lse), l_ref, atol=1e-5, rtol=1e-5)
    for got, ref in zip(grads, oracle.backward(*ex, ge, branches, 0.125)):
        assert np.abs(to_f64(got) - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())


@pytest.mark.parametrize("N", [33, 100])
def test_f32_infinite_value_stays_in_its_column(B, N):
    """A value row of infinities at the end of a ragged list: its own column is infinite, and the slots past the end of
    the list (which hold the last row again, with weight 0) make no NaN of it."""
    import torch
    (q, k, v), _ = make_qkv(77, 1, N, 1, 64, "f32")
    v[:, N - 1, :, 5] = float("inf")
    out, lse = B.forward(q, k, v, [(N, 1)], 0.125)
    assert bool(torch.isposinf(out[..., 5]).all())
    rest = torch.cat((out[..., :5], out[..., 6:]), dim=-1)
    assert bool(torch.isfinite(rest).all()) and bool(torch.isfinite(lse).all())


def test_f32_masked_block(B, oracle):
    """Scores of -inf over whole blocks (keys of -inf against positive queries) weigh nothing."""
    import torch
    (q, k, v), ex = make_qkv(78, 1, 160, 1, 64, "f32")
    q = q.abs() + 0.1
    k[:, 32:96] = -float("inf")
    out, lse = B.forward(q, k, v, [(160, 1)], 0.125)
    keep = list(range(32)) + list(range(96, 160))
    s = 0.125 * to_f64(q)[0, :, 0] @ to_f64(k)[0, keep, 0].T
    w = np.exp(s - s.max(1, keepdims=True))
    ref = (w / w.sum(1, keepdims=True)) @ to_f64(v)[0, keep, 0]
    assert np.abs(to_f64(out)[0, :, 0] - ref).max() <= 1e-5
    assert np.abs(to_f64(lse)[0, 0] - (s.max(1) + np.log(w.sum(1)))).max() <= 1e-5 * 10


def test_f32_launch_of_more_than_one_slice(B):
    """More workgroups than one grid takes (windows of one token: 9 * 16 * 4096 tiles): every row is its own value, bit
    for bit, and its lse the scaled dot product with its own key."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.empty((9, 4096, 16, 64), device="cuda").normal_(generator=gen) for _ in range(3))
    out, lse = B.forward(q, k, v, [(1, 1)], 0.125)
    assert torch.equal(out, v)
    ref = (q.double() * k.double()).sum(-1).mul(0.125).transpose(1, 2)
    assert float((lse.double() - ref).abs().max()) <= 1e-5
    # the backward likewise: P is 1, dv is dout; dq and dk are scale times a key or query (below 6) times dP - delta, which is the
    # rounding of two sums of 64 products (terms below 100 in all: 64 * 2^-24 * 100 at worst), where a wrong row gives about 1
    g = torch.empty_like(q).normal_(generator=gen)
    dq, dk, dv = B.backward(q, k, v, out, lse, g, [(1, 1)], 0.125)
    assert float((dv - g).abs().max()) <= 1e-5 * float(g.abs().max())
    bar = 0.125 * 6 * 2 * 64 * 2.0 ** -24 * 100
    assert float(dq.abs().max()) <= bar and float(dk.abs().max()) <= bar


@pytest.mark.parametrize("window,cut", [(16, False), (64, True)])
def test_f32_lists_whole_and_cut(B, window, cut):
    """Many row groups with long lists: past 2^18 blocks of lists (4 MB of records) the plan keeps them whole, and the
    kernels count through the progressions instead.  Against fp64 by the definition: keys of the row's own window count
    twice.  Sums of 16384 products, 1e-5 as above for out (of size 1e-2); gradients 2e-5 of the largest."""
    import torch
    N, br = 16384, [(16384, 1), (window, 1)]
    plan = B.plan_describe(1, 1, N, br)
    tiles, segs = plan["tiles"], plan["segs"]
    blocks = sum(-(-int(segs[x][2]) // 32) for begin, n in {(int(t[3]), int(t[4])) for t in tiles} for x in range(begin, begin + n))
    assert (blocks <= 1 << 18) == cut
    (q, k, v), _ = make_qkv(79, 1, N, 1, 64, "f32")
    g = torch.empty_like(q).normal_(generator=torch.Generator(device="cuda").manual_seed(6))
    out, lse = B.forward(q, k, v, br, 0.125)
    grads = B.backward(q, k, v, out, lse, g, br, 0.125)
    same, same_lse = B.forward_static(q, k, v, br, 0.125)
    assert torch.equal(same, out) and torch.equal(same_lse, lse)

    q6, k6, v6, g6 = (t[0, :, 0].double() for t in (q, k, v, g))
    ref, ref_lse, dq = torch.empty_like(q6), torch.empty(N, dtype=torch.float64, device="cuda"), torch.empty_like(q6)
    dk, dv = torch.zeros_like(q6), torch.zeros_like(q6)
    own = torch.arange(N, device="cuda") // window
    for n0 in range(0, N, 4096):
        r = slice(n0, n0 + 4096)
        s = 0.125 * (q6[r] @ k6.T.contiguous()) + torch.log((own[r, None] == own[None]).double() + 1.0)
        ref_lse[r] = torch.logsumexp(s, 1)
        p = torch.exp(s - ref_lse[r, None])
        ref[r] = p @ v6
        ds = p * (g6[r] @ v6.T.contiguous() - (g6[r] * ref[r]).sum(1, keepdim=True)) * 0.125
        dq[r] = ds @ k6
        dk += ds.T.contiguous() @ q6[r]
        dv += p.T.contiguous() @ g6[r]
    assert float((out[0, :, 0] - ref).abs().max()) <= 1e-5
    assert float((lse[0, 0] - ref_lse).abs().max()) <= 1e-5 * float(ref_lse.abs().max())
    for got, want in zip(grads, (dq, dk, dv)):
        assert float((got[0, :, 0] - want).abs().max()) <= 2e-5 * max(1.0, float(want.abs().max()))


# The products of the fp32 path are sums of bf16 products of the operands' parts; operands that parts cannot hold take fp32
# products.  Values so small that their low parts are not normal bf16 numbers (1e-37 is 2^-123), small and large ones that parts do
# hold, and ones that round up to 2^128 in bf16: everything is linear in v (forward) and in dout (backward), so the bars are
# those of ordinary values times the factor.
@pytest.mark.parametrize("factor", [2.0 ** -121, 2.0 ** -100, 2.0 ** -60, 2.0 ** 90])
def test_f32_range_of_values(B, oracle, factor):
    N, branches = 200, [(50, 1), (100, 2), (200, 4)]
    (q, k, v), ex = make_qkv(311, 2, N, 3, 64, "f32")
    from paper_2403_09195_amd import synth
    st, ge = synth.tensor(311, 7, (2, N, 3, 64), "f32")
    out, lse = B.forward(q, k, v * factor, branches, 0.125)
    o_ref, l_ref = oracle.forward(*ex, branches, 0.125)
    assert np.abs(to_f64(out) / factor - o_ref).max() <= 1e-5
    check_lse(to_f64(lse), l_ref, atol=1e-5, rtol=1e-5)
    out, lse = B.forward(q, k, v, branches, 0.125)
    grads = B.backward(q, k, v, out, lse, to_device(st) * factor, branches, 0.125)
    for got, ref in zip(grads, oracle.backward(*ex, ge, branches, 0.125)):
        assert np.abs(to_f64(got) / factor - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())


def test_f32_values_next_to_the_largest(B, oracle):
    """A value at fp32's largest: bf16 rounds it up to infinity, its share of every weighted mean is finite."""
    N, top = 96, float(np.finfo(np.float32).max)
    (q, k, v), ex = make_qkv(312, 1, N, 2, 64, "f32")
    v[:, 50, :, 9] = top
    ex[2][:, 50, :, 9] = top
    out, _ = B.forward(q, k, v, [(N, 1)], 0.125)
    o_ref, _ = oracle.forward(*ex, [(N, 1)], 0.125)
    scale = np.where(np.arange(64) == 9, top, 1.0)
    assert np.abs(to_f64(out) / scale - o_ref / scale).max() <= 1e-5


def test_f32_infinities_and_nan(B):
    """An infinite key component makes the scores of its key infinite: NaN rows where the score is +inf, weight 0 where it is
    -inf.  A NaN value row is NaN in its column only."""
    import torch
    N = 70
    (q, k, v), _ = make_qkv(313, 1, N, 1, 64, "f32")
    k2 = k.clone()
    k2[:, 40, :, 3] = float("inf")
    out, lse = B.forward(q, k2, v, [(N, 1)], 0.125)
    up = q[0, :, 0, 3] > 0                          # rows whose score with key 40 is +inf
    assert bool(torch.isnan(out[0, up]).all())
    keep = [n for n in range(N) if n != 40]
    o_ref, l_ref = B.forward(q[:, keep].contiguous(), k[:, keep].contiguous(), v[:, keep].contiguous(), [(N - 1, 1)], 0.125)
    down = torch.tensor([n for n in keep if not bool(up[n])])
    at = torch.tensor([keep.index(int(n)) for n in down])
    assert float((out[0, down.cuda()] - o_ref[0, at.cuda()]).abs().max()) <= 1e-5
    assert float((lse[0, 0, down.cuda()] - l_ref[0, 0, at.cuda()]).abs().max()) <= 1e-5
    v2 = v.clone()
    v2[:, 11, :, 60] = float("nan")
    out, lse = B.forward(q, k, v2, [(N, 1)], 0.125)
    assert bool(torch.isnan(out[..., 60]).all()) and bool(torch.isfinite(out[..., :60]).all()) and bool(torch.isfinite(lse).all())


# Small operands against large ones: the result is an ordinary number and says nothing of the low parts that 2^-120 has lost (scores; dP;
# ds k and ds q).  Every gradient is its ordinary value times the powers of two of its operands.
@pytest.mark.parametrize("e_q,e_v,e_g", [(-120, 0, 0), (120, 0, 0), (0, -121, 110), (0, 110, -121)])
def test_f32_small_operands_against_large_ones(B, oracle, e_q, e_v, e_g):
    N, branches = 200, [(50, 1), (100, 2), (200, 4)]
    (q, k, v), ex = make_qkv(314, 1, N, 3, 64, "f32")
    from paper_2403_09195_amd import synth
    st, ge = synth.tensor(314, 7, (1, N, 3, 64), "f32")
    q, k, v, g = q * 2.0 ** e_q, k * 2.0 ** -e_q, v * 2.0 ** e_v, to_device(st) * 2.0 ** e_g
    out, lse = B.forward(q, k, v, branches, 0.125)
    o_ref, l_ref = oracle.forward(*ex, branches, 0.125)
    assert np.abs(to_f64(out) / 2.0 ** e_v - o_ref).max() <= 1e-5
    check_lse(to_f64(lse), l_ref, atol=1e-5, rtol=1e-5)
    grads = B.backward(q, k, v, out, lse, g, branches, 0.125)
    for got, ref, e in zip(grads, oracle.backward(*ex, ge, branches, 0.125), (e_v + e_g - e_q, e_v + e_g + e_q, e_g)):
        assert np.abs(to_f64(got) / 2.0 ** e - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())


def test_f32_one_small_operand(B, oracle):
    """One walked row whose values parts do not hold, at weight 1 for its own segment: the other lists and tiles keep the split."""
    N, w = 128, 64
    (q, k, v), ex = make_qkv(315, 1, N, 2, 64, "f32")
    v[:, :w] *= 2.0 ** -120
    out, lse = B.forward(q, k, v, [(w, 1)], 0.125)
    o_ref, l_ref = oracle.forward(*ex, [(w, 1)], 0.125)
    got = to_f64(out)
    got[:, :w] *= 2.0 ** 120
    assert np.abs(got - o_ref).max() <= 1e-5
    check_lse(to_f64(lse), l_ref, atol=1e-5, rtol=1e-5)


def test_f32_small_scale(B, oracle):
    """A scale whose product with 2^-60 is no normal number, against queries as much larger."""
    N = 100
    (q, k, v), ex = make_qkv(316, 1, N, 2, 64, "f32")
    from paper_2403_09195_amd import synth
    st, ge = synth.tensor(316, 7, (1, N, 2, 64), "f32")
    for e in (-50, -80):
        out, lse = B.forward(q * 2.0 ** -e, k, v, [(N, 1)], 0.125 * 2.0 ** e)
        o_ref, l_ref = oracle.forward(*ex, [(N, 1)], 0.125)
        assert np.abs(to_f64(out) - o_ref).max() <= 1e-5
        check_lse(to_f64(lse), l_ref, atol=1e-5, rtol=1e-5)
        grads = B.backward(q * 2.0 ** -e, k, v, out, lse, to_device(st), [(N, 1)], 0.125 * 2.0 ** e)
        for got, ref, x in zip(grads, oracle.backward(*ex, ge, [(N, 1)], 0.125), (e, 0, 0)):
            assert np.abs(to_f64(got) / 2.0 ** x - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())


# lists of one block each: windows and dilated windows of up to 32 keys, a shorter last one, rows that no branch keeps; a window of 33 and
# windows beside longer ones take the other form
@pytest.mark.parametrize("N,branches", [(32, [(32, 1)]), (100, [(32, 1)]), (96, [(31, 1)]), (130, [(64, 2)]), (96, [(33, 1)]), (128, [(32, 1), (128, 2)])])
def test_f32_lists_of_one_block(B, oracle, N, branches):
    (q, k, v), ex = make_qkv(317 + N, 2, N, 3, 64, "f32")
    out, lse = B.forward(q, k, v, branches, 0.125)
    o_ref, l_ref = oracle.forward(*ex, branches, 0.125)
    assert np.abs(to_f64(out) - o_ref).max() <= 1e-5
    check_lse(to_f64(lse), l_ref, atol=1e-5, rtol=1e-5)
    assert np.all(to_f64(out)[np.isneginf(l_ref).transpose(0, 2, 1)] == 0.0)
