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
