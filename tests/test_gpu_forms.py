"""The kernels of 256-row tiles (forward whole, packed and split; backward) on shapes that the rules leave to them, with the
edges that small problems otherwise take to the short-launch kernels.  Every test asserts the form its shape takes
(launch_describe), so that a change of a rule cannot turn it into a test of another kernel.  Bars as everywhere on the
bf16 path: out 2e-2 / 2e-3, lse per row (see gpu_util), gradients by the size of the terms an element is a sum of (the
bound of the random problems in test_gpu_random_shapes)."""
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


def _forward(B, oracle, q, k, v, ex, branches, offs, workspace="auto"):
    out, lse = B.forward(q, k, v, branches, 0.125, head_offsets=offs, workspace=workspace)
    o_ref, l_ref = oracle.forward(*ex, branches, 0.125, head_offsets=offs)
    mx, mean = error_stats(to_f64(out), o_ref)
    assert mx <= 2e-2 and mean <= 2e-3, (mx, mean)
    check_lse_bf16(to_f64(lse), oracle, ex, branches, 0.125, l_ref, offs)
    assert np.all(to_f64(out)[np.isneginf(l_ref).transpose(0, 2, 1)] == 0.0)
    return out, lse, l_ref


def _backward(B, oracle, q, k, v, ex, out, lse, l_ref, branches, offs, seed):
    from paper_2403_09195_amd import synth
    st, ge = synth.tensor(seed, 7, tuple(q.shape), "bf16")
    grads = B.backward(q, k, v, out, lse, to_device(st), branches, 0.125, head_offsets=offs)
    refs = oracle.backward(*ex, ge, branches, 0.125, head_offsets=offs)
    bounds = helpers.multiset_attention_backward(*ex, ge, 0.125, branches, offs)[3:]
    dead = np.isneginf(l_ref).transpose(0, 2, 1)
    eps = 2.0 ** -9
    for name, got, ref, absum in zip(("dq", "dk", "dv"), grads, refs, bounds):
        d = np.abs(to_f64(got) - ref)
        assert np.all(d <= 2.0 ** -8 * np.abs(ref) + 4 * eps * absum + 1e-6), name
        assert d.mean() <= eps * absum.mean() + 1e-7, name
        assert np.all(to_f64(got)[dead] == 0.0)


# forward: lists around the 32-key beat and the 64-key stage, walks of one step to a few, tiles of a row to full ones
@pytest.mark.parametrize("count,r", [(1, 1), (2, 1), (31, 1), (32, 1), (33, 1), (63, 2), (64, 1), (65, 3), (95, 1), (96, 2),
                                     (97, 1), (128, 1), (129, 2), (257, 1)])
def test_forward_whole_tiles_key_counts(B, oracle, count, r):
    w = count * r
    Bsz, N, H = 160, 2 * w, 3
    (q, k, v), ex = make_qkv(2300 + count, Bsz, N, H, 64, "bf16")
    for br in ([(w, r), (2 * w, 2 * r)], [(w, r)]):
        assert B.launch_describe(Bsz, H, N, br)["form"] == B.FORM_TILES
        _forward(B, oracle, q, k, v, ex, br, None)


# forward, split: ragged lists and tiles, shares of several progressions, packed tiles, rows kept by nothing
@pytest.mark.parametrize("H,N,branches,offs,packed", [
    (1, 2113, [(2113, 1)], None, False),
    (3, 2200, [(2200, 1)], None, True),
    (2, 2400, [(2400, 1), (600, 4)], [[0, 0], [3, 1]], False),
    (2, 4224, [(1056, 1), (2112, 2), (4224, 4)], None, True),
    (2, 3000, [(100, 1), (3000, 1)], None, False),
    (2, 4500, [(4500, 2)], [[1, 0]], False),
])
def test_forward_split(B, oracle, H, N, branches, offs, packed):
    import torch
    assert B.launch_describe(1, H, N, branches, offs)["form"] == B.FORM_SPLIT
    (q, k, v), ex = make_qkv(2400 + N, 1, N, H, 64, "bf16")
    if packed:                                     # views of one buffer, row pitch 3 * H * D
        q, k, v = torch.stack((q, k, v), dim=2).unbind(2)
    out, _, _ = _forward(B, oracle, q, k, v, ex, branches, offs)
    whole, _, _ = _forward(B, oracle, q, k, v, ex, branches, offs, workspace=None)
    assert not torch.equal(out, whole)             # the workspace did change the kernel


# backward: tiles of 1, 63 to 65, 127 to 129 and 191 to 257 rows (a second dk/dv workgroup without rows, with a few, full),
# walks of one step to five against the ring of four stages, ragged last stages
@pytest.mark.parametrize("count", [1, 31, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257])
@pytest.mark.parametrize("packed", [False, True])
def test_backward_whole_tiles_list_lengths(B, oracle, count, packed):
    import torch
    Bsz, N, H, branches = (400 if count <= 64 else 64), count, 8, [(count, 1)]
    assert B.launch_describe(Bsz, H, N, branches, backward=True)["form"] == B.FORM_TILES
    (q, k, v), ex = make_qkv(2500 + count, Bsz, N, H, 64, "bf16")
    if packed:
        q, k, v = torch.stack((q, k, v), dim=2).unbind(2)
    out, lse, l_ref = _forward(B, oracle, q, k, v, ex, branches, None)
    _backward(B, oracle, q, k, v, ex, out, lse, l_ref, branches, None, 2500 + count)


@pytest.mark.parametrize("Bsz,N,H,branches,offs", [
    (64, 390, 4, [(195, 2)], None),                                  # rows kept by nothing, tiles of 97 and 98 rows
    (160, 260, 4, [(130, 2)], [[1, 0, 1, 1]]),
    (96, 600, 2, [(300, 1), (600, 2)], [[0, 0], [1, 0]]),            # two ragged progressions, pairs that count double
    (48, 512, 4, [(256, 2), (256, 2), (512, 1)], None),              # multiplicities up to 3
    (96, 700, 2, [(350, 1), (700, 3)], [[0, 0], [2, 1]]),
])
def test_backward_whole_tiles_branches(B, oracle, Bsz, N, H, branches, offs):
    assert B.launch_describe(Bsz, H, N, branches, offs, backward=True)["form"] == B.FORM_TILES
    (q, k, v), ex = make_qkv(2600 + N, Bsz, N, H, 64, "bf16")
    out, lse, l_ref = _forward(B, oracle, q, k, v, ex, branches, offs)
    _backward(B, oracle, q, k, v, ex, out, lse, l_ref, branches, offs, 2600 + N)


def _problem(seed):
    """Random branches, offsets and sizes, at the smallest batch at which both directions run 256-row tiles."""
    rng = np.random.default_rng(4100 + seed)
    H, N, nb = int(rng.integers(1, 6)), int(rng.integers(40, 420)), int(rng.integers(1, 4))
    branches, offs = [], []
    for _ in range(nb):
        r = int(rng.integers(1, 4))
        branches.append((int(rng.integers(max(r, 8), 2 * N)), r))
        offs.append([int(rng.integers(0, r)) for _ in range(H)])
    return H, N, branches, (offs if seed % 2 else None)


@pytest.mark.parametrize("seed", [0, 1, 4, 7, 8, 10, 12, 13, 17, 22, 25, 29, 30, 34, 36, 40, 52, 54])
def test_random_problems_of_whole_tiles(B, oracle, seed):
    H, N, branches, offs = _problem(seed)
    Bsz = next(b for b in (16, 32, 64, 128, 256) if B.launch_describe(b, H, N, branches, offs)["form"] == B.FORM_TILES
               and B.launch_describe(b, H, N, branches, offs, backward=True)["form"] == B.FORM_TILES)
    print(f"[whole tiles {seed}] B={Bsz} N={N} H={H} branches={branches} offsets={offs}", flush=True)
    (q, k, v), ex = make_qkv(2700 + seed, Bsz, N, H, 64, "bf16")
    out, lse, l_ref = _forward(B, oracle, q, k, v, ex, branches, offs)
    _backward(B, oracle, q, k, v, ex, out, lse, l_ref, branches, offs, 2700 + seed)
