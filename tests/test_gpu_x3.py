"""The exact gradient of fp32 layers as three bf16 or two fp16 pieces on the matrix core, and of bf16 layers as one: the shapes
where its tiles, its staging and its result tile have edges, the inputs that the pieces cannot represent, and its error
against fp64."""
import numpy as np
import pytest

import oracle
from paper_1908_05460_amd import binding as B
from tests.gpu_util import TOL, normwise_err, oracle_shape, rand_inputs, to_gpu
from tests.x3_shapes import PLANS, plan

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride_h, stride_w, pad_h, pad_w; N such that the shape takes this form: 0.03 GFLOP, with at most 16
# channels on a side 0.5, and any size where rows or planes are odd or rows too long for the streaming form
EDGES = [
    (3, 33, 32, 32, 65, 3, 3, 1, 1, 1, 1),      # one channel and one output channel over a 32 tile
    (8, 31, 16, 16, 31, 3, 3, 1, 1, 1, 1),      # one under
    (9, 64, 8, 8, 64, 3, 3, 1, 1, 1, 1),        # a last tile of one image
    (73, 40, 4, 4, 40, 3, 3, 1, 1, 1, 1),       # a last tile of one image, position by position in fp32
    (2, 32, 27, 27, 32, 3, 3, 1, 1, 1, 1),      # a row's last chunk holds three columns; last tile of three rows
    (1, 32, 5, 300, 32, 3, 3, 1, 1, 1, 1),      # rows cut into column tiles: neighbour words on both sides
    (1, 64, 9, 130, 64, 3, 3, 1, 1, 1, 1),      # the last column tile holds two columns
    (160, 20, 7, 4, 20, 3, 3, 1, 1, 1, 1),      # the narrowest rows
    (2, 20, 6, 7, 20, 3, 3, 1, 1, 0, 0),        # no padding: the output starts left of the input's first column
    (2, 20, 6, 7, 20, 3, 3, 1, 1, 3, 4),        # more padding than the filter needs
    (2, 20, 9, 21, 24, 3, 3, 2, 2, 1, 1),       # strides, odd width
    (2, 20, 9, 20, 24, 3, 3, 3, 2, 0, 2),
    (40, 20, 9, 20, 24, 3, 3, 2, 1, 1, 1),      # stride in rows alone
    (500, 3, 20, 12, 80, 3, 3, 1, 1, 1, 1),     # (channel, filter row) columns
    (2, 9, 12, 13, 40, 3, 3, 1, 1, 1, 1),
    (2, 33, 11, 14, 18, 5, 5, 1, 1, 2, 2),
    (40, 32, 16, 16, 32, 3, 3, 1, 1, 1, 1),     # several workgroups share the reduction
    (1, 1, 5, 5, 1, 3, 3, 1, 1, 1, 1),
    (73, 40, 6, 4, 40, 3, 3, 1, 1, 1, 1),       # rows of half a chunk
    (130, 65, 4, 4, 65, 3, 3, 1, 1, 1, 1),      # position by position: one channel over both tiles, the last stage has two images
    (40, 64, 4, 4, 64, 3, 3, 1, 1, 1, 1),       # whole tiles
    (257, 33, 2, 2, 100, 3, 3, 1, 1, 1, 1),     # 2x2: the last stage has one image
    (36, 200, 2, 2, 63, 3, 3, 1, 1, 1, 1),      # the last stage's second group of images is empty
]


def mk(t, dtype="fp32"):
    N, C, H, W, K, R, S, sh, sw, ph, pw = t
    return B.desc(N, C, H, W, K, R, S, stride=sh, pad=ph, stride_w=sw, pad_w=pw, dtype=B.BF16 if dtype == "bf16" else B.F32)


def torch_nan(d):
    import torch
    return torch.full((d.K, d.C, d.R, d.S), float("nan"), device="cuda")


def run(d, X, dY):
    return B.conv_wgrad_exact(d, X, dY, dW=torch_nan(d)).cpu().numpy()


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("t", EDGES)
def test_edges_match_the_oracle(t, dtype):
    d = mk(t, dtype)
    X, dY = rand_inputs(d, 99, dtype)
    want = oracle.wgrad_exact(oracle_shape(d), X, dY)
    # fp32 sums of exact products: far inside the fp32 tolerance (a lost piece would cost 4e-3, 2e-5 or 1e-7)
    assert normwise_err(run(d, to_gpu(X), to_gpu(dY)), want) < TOL["fp32"] / 50


@pytest.mark.parametrize("variant, t, dtype, halo", PLANS)
def test_every_variant_matches_the_oracle(variant, t, dtype, halo):
    """Several tiles to a workgroup: the next tile's loads, LDS reuse, neighbour words and uneven shares of a reduction;
    then with infinities and NaNs, which only what they meet may show."""
    d = mk(t, dtype)
    X, dY = rand_inputs(d, 99, dtype)
    want = oracle.wgrad_exact(oracle_shape(d), X, dY)
    got = run(d, to_gpu(X), to_gpu(dY))
    assert normwise_err(got, want) < TOL["fp32"] / 50
    size = np.sqrt(np.mean(want * want))
    bits = {np.inf: 0x7F80, -np.inf: 0xFF80, np.nan: 0x7FC0}
    ends = ((0, 0, 0, 0), (-1, -1, -1, -1), (-1, 1, 0, -1), (0, -1, -1, 0))
    for bad, where in ((np.inf, X), (-np.inf, dY), (np.nan, dY)):
        kept = [where[at] for at in ends]
        for at in ends:
            where[at] = bits[bad] if dtype == "bf16" else bad
        with np.errstate(all="ignore"):
            want = oracle.wgrad_exact(oracle_shape(d), X, dY)
        got = run(d, to_gpu(X), to_gpu(dY))
        fine = np.isfinite(want)
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[~fine], want[~fine].astype(np.float32), equal_nan=True)
        if fine.any():
            assert np.abs(got[fine] - want[fine]).max() < TOL["fp32"] * size
        for at, v in zip(ends, kept):
            where[at] = v


@pytest.mark.parametrize("t", [EDGES[4], EDGES[5], EDGES[12], EDGES[13], EDGES[15], EDGES[19], EDGES[20], EDGES[21]])
def test_tensors_aligned_to_their_elements_only(t):
    import torch
    d = mk(t)
    X, dY = rand_inputs(d, 5)
    Xu = torch.empty(X.size + 1, device="cuda")[1:].view(X.shape).copy_(to_gpu(X))
    dYu = torch.empty(dY.size + 3, device="cuda")[3:].view(dY.shape).copy_(to_gpu(dY))
    assert np.array_equal(run(d, Xu, dYu), run(d, to_gpu(X), to_gpu(dY)))


@pytest.mark.parametrize("t", [EDGES[1], EDGES[4], EDGES[13]])
def test_bf16_tensors_aligned_to_their_elements_only(t):
    """Whole rows are read in 8-byte pieces; a tensor that starts at any even address takes the older kernels."""
    import torch
    d = mk(t, "bf16")
    X, dY = (to_gpu(a) for a in rand_inputs(d, 5, "bf16"))
    Xu = torch.empty(X.numel() + 1, dtype=torch.bfloat16, device="cuda")[1:].view(X.shape).copy_(X)
    dYu = torch.empty(dY.numel() + 3, dtype=torch.bfloat16, device="cuda")[3:].view(dY.shape).copy_(dY)
    assert normwise_err(run(d, Xu, dYu), run(d, X, dY).astype(np.float64)) < TOL["fp32"] / 50


@pytest.mark.parametrize("t", [EDGES[0], EDGES[4], EDGES[6]])
@pytest.mark.parametrize("where", ["X", "dY"])
@pytest.mark.parametrize("bad", [0x7F80, 0xFF80, 0x7FC0])
def test_bf16_infinities_and_nans(t, where, bad):
    d = mk(t, "bf16")
    X, dY = rand_inputs(d, 7, "bf16")
    a = X if where == "X" else dY
    for at in ((0, 0, 0, 0), (-1, -1, -1, -1), (0, 1 % a.shape[1], a.shape[2] // 2, a.shape[3] // 2)):
        a[at] = bad
    want = oracle.wgrad_exact(oracle_shape(d), X, dY)
    got = run(d, to_gpu(X), to_gpu(dY))
    fine = np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[~fine], want[~fine].astype(np.float32), equal_nan=True)
    assert normwise_err(got[fine], want[fine]) < TOL["fp32"] / 50


@pytest.mark.parametrize("t", [EDGES[0], EDGES[3], EDGES[4], EDGES[6], EDGES[10], EDGES[13], EDGES[18], EDGES[19], EDGES[21]])
@pytest.mark.parametrize("where", ["X", "dY"])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 3.4e38])
def test_values_the_pieces_cannot_hold(t, where, bad):
    """An infinity meets zeros and both signs in its pieces' products, and 3.4e38 rounds to infinity as bf16: the result
    is the definition's all the same, infinities where it has them and everything untouched by the value finite."""
    d = mk(t)
    X, dY = rand_inputs(d, 7)
    a = X if where == "X" else dY
    for at in ((0, 0, 0, 0), (-1, -1, -1, -1), (0, 1 % a.shape[1], a.shape[2] // 2, a.shape[3] // 2)):
        a[at] = bad
    with np.errstate(all="ignore"):
        want = oracle.wgrad_exact(oracle_shape(d), X, dY)
        want32 = want.astype(np.float32)
    got = run(d, to_gpu(X), to_gpu(dY))
    assert np.array_equal(np.isnan(got), np.isnan(want32))
    assert np.array_equal(got[np.isinf(want32)], want32[np.isinf(want32)])
    fine = np.isfinite(want32)
    # entries that sum the huge value are compared at their own size, the rest at theirs
    big = fine & (np.abs(want) > 1e30)
    for part in (big, fine & ~big):
        if part.any():
            assert normwise_err(got[part], want[part]) < TOL["fp32"]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("t", [
    (2, 20, 6, 7, 24, 3, 3, 1, 1, 3, 4),
    (3, 64, 32, 32, 64, 3, 3, 1, 1, 3, 3),
    (2, 20, 9, 21, 24, 3, 3, 2, 2, 5, 5),
    (2, 33, 11, 14, 18, 5, 5, 1, 1, 6, 7),
])
def test_nan_in_a_column_that_sees_only_padding(t, dtype):
    """Padding as wide as the filter: the outermost columns of dY meet nothing but zeros, and a NaN there is still a
    NaN of every entry of its output channel."""
    d = mk(t, dtype)
    X, dY = rand_inputs(d, 3, dtype)
    Xg = to_gpu(X)
    for w in range(d.Wo):
        bad = dY.copy()
        bad[0, 1, d.Ho // 2, w] = 0x7FC0 if dtype == "bf16" else np.nan
        if w in (0, d.Wo // 2):
            assert np.array_equal(np.isnan(oracle.wgrad_exact(oracle_shape(d), X, bad)).all(axis=(1, 2, 3)), np.arange(d.K) == 1)
        got = run(d, Xg, to_gpu(bad))
        assert np.isnan(got[1]).all() and np.isfinite(np.delete(got, 1, axis=0)).all(), w


@pytest.mark.parametrize("t", [EDGES[0], EDGES[4], EDGES[10], EDGES[19], EDGES[21]])
@pytest.mark.parametrize("scale", [(1e15, 1e15), (1e-12, 1e-12), (1e-20, 1e18), (1e25, 1e-25), (1e31, 1e-3), (1e30, 1e-32),
                                   (1e30, 1e-34), (1e30, 1e-36), (1e-36, 1e30), (1e30, 1e-39), (1e-40, 1e36)])
def test_scales_far_from_one(t, scale):
    """Down to tensors of subnormal numbers: the pieces hold every fp32 number whole."""
    d = mk(t)
    X, dY = rand_inputs(d, 11)
    X, dY = X * np.float32(scale[0]), dY * np.float32(scale[1])
    want = oracle.wgrad_exact(oracle_shape(d), X, dY)
    assert normwise_err(run(d, to_gpu(X), to_gpu(dY)), want) < TOL["fp32"] / 50


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("t", [(2, 17, 6, 40, 24, 3, 3, 1, 1, 9, 1), (2, 33, 6, 40, 70, 3, 3, 1, 1, 9, 1), (1, 33, 5, 300, 40, 3, 3, 1, 1, 8, 1),
                               (2, 17, 6, 41, 24, 3, 3, 1, 1, 9, 1), (3, 17, 5, 40, 24, 3, 3, 2, 2, 9, 1)])
def test_rows_of_padding_behind_the_last_plane(t, dtype):
    """Padding so high that a tile's first input row lies behind the tensor's last: nothing is left to read there."""
    d = mk(t, dtype)
    X, dY = rand_inputs(d, 41, dtype)
    assert normwise_err(run(d, to_gpu(X), to_gpu(dY)), oracle.wgrad_exact(oracle_shape(d), X, dY)) < TOL["fp32"] / 50


def test_wide_range_of_magnitudes_within_a_tensor():
    """Output channels of 2^-40 .. 2^40 side by side, each of them uniform (16-wide tiles in bf16 pieces): one of small gradients is as
    exact as one of large ones.  Magnitudes that differ within a channel: test_small_numbers_beside_large_ones_that_meet_zeros."""
    d = mk((4, 32, 12, 12, 64, 3, 3, 1, 1, 1, 1))
    X, dY = rand_inputs(d, 13)
    dY *= np.exp2(np.linspace(-40, 40, d.K)).astype(np.float32)[None, :, None, None]
    want = oracle.wgrad_exact(oracle_shape(d), X, dY)
    got = run(d, to_gpu(X), to_gpu(dY))
    for k in range(d.K):
        assert normwise_err(got[k], want[k]) < TOL["fp32"] / 50


def test_error_is_that_of_fp32_sums():
    """64 -> 64 @ 32x32 at N = 128: the fp32 matrix core's kernel is 6.5e-7 of the result (2-norm) off."""
    d = mk((128, 64, 32, 32, 64, 3, 3, 1, 1, 1, 1))
    X, dY = rand_inputs(d, 17)
    want = oracle.wgrad_exact(oracle_shape(d), X, dY)
    got = run(d, to_gpu(X), to_gpu(dY))
    assert np.linalg.norm(got - want) < 6.5e-7 * np.linalg.norm(want)


@pytest.mark.parametrize("t, dtype, bound", [
    ((128, 16, 32, 32, 16, 3, 3, 1, 1, 1, 1), "fp32", 1.84e-7),
    ((100, 33, 24, 24, 100, 3, 3, 1, 1, 1, 1), "fp32", 2.92e-7),
    ((135, 4, 133, 8, 278, 3, 3, 2, 2, 1, 1), "fp32", 2.46e-7),
    ((5, 5, 66, 170, 22, 5, 5, 1, 1, 2, 2), "fp32", 1.70e-7),
    ((35, 24, 11, 148, 122, 3, 3, 1, 1, 1, 1), "fp32", 2.90e-7),
    ((216, 29, 39, 39, 21, 3, 3, 1, 1, 1, 1), "fp32", 3.34e-7),
    ((61, 182, 22, 8, 211, 3, 3, 1, 1, 1, 1), "bf16", 1.45e-7),
])
def test_error_is_that_of_fp32_sums_and_centred(t, dtype, bound):
    """The bounds are what the fp32 matrix core's kernels are off (2-norm); bf16 1.1 times that.  The bf16 core rounds
    what it adds to a larger sum downwards: the error's mean, which no length of the sum may let grow, stays a
    fraction of it (unsigned sums: 4.8e-7 of the result's size in the sixth shape)."""
    d = mk(t, dtype)
    X, dY = rand_inputs(d, 17, dtype)
    want = oracle.wgrad_exact(oracle_shape(d), X, dY)
    err = run(d, to_gpu(X), to_gpu(dY)) - want
    size = np.sqrt(np.mean(want * want))
    assert np.sqrt(np.mean(err * err)) < bound * size
    assert abs(err.mean()) < 5e-8 * size


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_run_of_layers_equals_the_single_calls_to_rounding(dtype):
    """Layers of several variants, and of one variant more groups (9) and layers (24) than a launch carries, in one run."""
    import torch
    many = [(5, 64 + 16 * i, 17, 17, 64, 3, 3, 1, 1, 1, 1) for i in range(10)]      # ten groups of three
    assert len({plan(t, dtype)[0].variant for t in many}) == 1 and all(plan(t, dtype)[1] == 2 for t in many)
    shapes = EDGES + many * 3 + [(40, 128, 16, 16, 128, 3, 3, 1, 1, 1, 1)] * 3
    # 2x2 planes that alone are a plain matrix product and, two of a shape in a run, are not
    shapes += [(70, 512, 2, 2, 512, 3, 3, 1, 1, 1, 1), (140, 272, 2, 2, 528, 3, 3, 1, 1, 1, 1)] * 2
    shapes += [(66, 512, 2, 2, 512, 3, 3, 1, 1, 1, 1)]           # one of a shape: as alone
    ds = [mk(t, dtype) for t in shapes]
    data = [tuple(to_gpu(a) for a in rand_inputs(d, 100 + i, dtype)) for i, d in enumerate(ds)]
    out = [torch.full((d.K, d.C, d.R, d.S), float("nan"), device="cuda") for d in ds]
    s = B.Schedule(ds, [x for x, _ in data], [y for _, y in data], out)
    m = [B.EXACT] * len(ds)
    s.run(m, B.alloc_workspace(s.workspace_bytes(m)))
    for d, (X, dY), got in zip(ds, data, out):
        assert normwise_err(got.cpu().numpy(), run(d, X, dY).astype(np.float64)) < TOL["fp32"] / 50


def test_infinities_in_a_run_of_layers():
    """2x2 planes of whole tiles take the position form in a run only, two or more of a shape."""
    shapes = [EDGES[0], EDGES[4], EDGES[19]]
    shapes += [(70, 512, 2, 2, 512, 3, 3, 1, 1, 1, 1), (140, 272, 2, 2, 528, 3, 3, 1, 1, 1, 1)] * 2
    ds = [mk(t) for t in shapes]
    data = [rand_inputs(d, 200 + i) for i, d in enumerate(ds)]
    for X, dY in data:
        dY[0, 0, 0, 0], dY[-1, 5, -1, -1], X[1, 3, 0, 0] = np.inf, np.nan, -np.inf
    out = [torch_nan(d) for d in ds]
    s = B.Schedule(ds, [to_gpu(x) for x, _ in data], [to_gpu(y) for _, y in data], out)
    m = [B.EXACT] * len(ds)
    s.run(m, B.alloc_workspace(s.workspace_bytes(m)))
    for d, (X, dY), got in zip(ds, data, out):
        with np.errstate(all="ignore"):
            want = oracle.wgrad_exact(oracle_shape(d), X, dY)
        got, fine = got.cpu().numpy(), np.isfinite(want)
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[~fine], want[~fine].astype(np.float32), equal_nan=True)
        assert normwise_err(got[fine], want[fine]) < TOL["fp32"]


# Two fp16 pieces to a number: 32-wide tiles (whole rows, cut rows, ragged rows, (channel, filter row) columns) and 4x4 planes in
# sums of twelve stages and more
HALVES = [t for v, t, _, _ in PLANS if v in (0, 1, 2, 9, 10)] + [(97, 1000, 4, 4, 1040, 3, 3, 1, 1, 1, 1)]


@pytest.mark.parametrize("t", HALVES)
@pytest.mark.parametrize("how", ["growing", "shrinking", "channels", "hidden"])
def test_scales_of_fp16_pieces(t, how):
    """The scales of a workgroup's channels change along its sum, differ between the channels of both tensors, or are set by
    one huge number that meets only zeros, beside which the others would have no bits left: those are summed as they are."""
    d = mk(t)
    X, dY = rand_inputs(d, 23)
    n = np.arange(d.N)[:, None, None, None]
    if how in ("growing", "shrinking"):
        dY *= np.exp2((1 if how == "growing" else -1) * (7 * n % 41) * 1.0).astype(np.float32)
        X *= np.exp2((1 if how == "growing" else -1) * (5 * n % 23) * 0.5).astype(np.float32)
    elif how == "channels":
        dY *= np.exp2(np.linspace(-60, 60, d.K)).astype(np.float32)[None, :, None, None]
        X *= np.exp2(np.linspace(50, -50, d.C)).astype(np.float32)[None, :, None, None]
    else:
        X[0] = 0
        dY[0, ::3] *= np.float32(1e25)
    want = oracle.wgrad_exact(oracle_shape(d), X, dY)
    got = run(d, to_gpu(X), to_gpu(dY))
    if how == "channels":
        want, got = want.reshape(d.K * d.C, -1), got.reshape(d.K * d.C, -1)
        assert (np.abs(got - want).max(1) / np.abs(want).max(1)).max() < TOL["fp32"] / 5    # (of the nine taps of a pair)
    else:
        assert normwise_err(got, want) < TOL["fp32"] / 50
        for k in range(d.K):
            assert normwise_err(got[k], want[k]) < TOL["fp32"] / 25


@pytest.mark.parametrize("t", HALVES)
@pytest.mark.parametrize("where, factor", [("images", f) for f in (14, 18, 22, 26, 30, 40, 66)] + [("columns", f) for f in (22, 40, 66)])
def test_small_numbers_beside_large_ones_that_meet_zeros(t, where, factor):
    """Every other image of dY, or its first column, is 2^factor times the rest and meets only zeros of X: the result consists of numbers
    far below their channel's largest, in which an fp16 piece has few bits left or none, and is as exact as without the others."""
    d = mk(t)
    X, dY = rand_inputs(d, 29)
    if where == "images":
        X[::2] = 0
        dY[::2] *= np.float32(2.0 ** factor)
    else:
        X[..., :max(0, d.S - d.pad_w)] = 0
        dY[..., 0] *= np.float32(2.0 ** factor)
    want = oracle.wgrad_exact(oracle_shape(d), X, dY)
    got = run(d, to_gpu(X), to_gpu(dY))
    for k in range(d.K):
        assert normwise_err(got[k], want[k]) < TOL["fp32"] / 50


@pytest.mark.parametrize("t", HALVES)
def test_single_results_of_small_numbers(t):
    """Channels of X that are zero but for one number, whose partner in a few channels of dY is far below those channels' largest: a few
    results of a workgroup consist of such a product alone, and are as exact as any."""
    d = mk(t)
    X, dY = rand_inputs(d, 37)
    n, h, w = d.N - 1, d.Ho - 1, d.Wo // 2
    y, x = h * d.stride_h + d.R // 2 - d.pad_h, w * d.stride_w + d.S // 2 - d.pad_w     # what the middle tap sees from there
    few = [(5, 1), (11, 1), (d.K - 1, d.C - 2), (8, d.C - 2), (9, d.C - 2)]
    for k, c in few:
        X[:, c] = 0
        X[n, c, y, x] = 1.7
        dY[n, k, h, w] = 0.3 * 2.0 ** -(24 + 2 * k % 37)
    want = oracle.wgrad_exact(oracle_shape(d), X, dY)
    got = run(d, to_gpu(X), to_gpu(dY))
    assert normwise_err(got, want) < TOL["fp32"] / 50
    for k, c in few:
        assert abs(got[k, c, d.R // 2, d.S // 2] - want[k, c, d.R // 2, d.S // 2]) <= 2.0 ** -23 * abs(want[k, c, d.R // 2, d.S // 2]) and want[k, c, d.R // 2, d.S // 2] != 0


@pytest.mark.parametrize("t", HALVES)
@pytest.mark.parametrize("how", ["numbers", "images", "sparse"])
def test_every_result_of_numbers_of_many_magnitudes(t, how):
    """Magnitudes over 2^40 from number to number or image to image, or over 2^30 in products so rare that many results are a few or none:
    no result is further off than an fp32 sum of its products may be, a rounding of 2^-24 of their magnitudes or two for each."""
    d = mk(t)
    X, dY = rand_inputs(d, 41)
    rng = np.random.default_rng(43)
    if how == "images":
        dY *= np.exp2(-40 * rng.random((d.N, 1, 1, 1), np.float32))
    elif how == "sparse":
        X *= rng.random(X.shape) < 4 / (d.N * d.H * d.W)
        dY *= np.exp2(-30 * rng.random(dY.shape, np.float32))
    else:
        X *= np.exp2(-40 * rng.random(X.shape, np.float32)) * (rng.random(X.shape) < 0.5)
        dY *= np.exp2(-40 * rng.random(dY.shape, np.float32)) * (rng.random(dY.shape) < 0.5)
    g = oracle_shape(d)
    want, size = oracle.wgrad_exact(g, X, dY), oracle.wgrad_exact(g, np.abs(X), np.abs(dY))
    got = run(d, to_gpu(X), to_gpu(dY))
    p = plan(t, "fp32")[0]
    # products of a workgroup's sum (4x4 planes: eight images a stage); of the rare ones sixteen at most, two of them on average
    terms = 8 if how == "sparse" else -(-p.tiles // p.splits) * (p.nch * 8 if p.nch else 128)
    assert (np.abs(got - want) <= 2 * terms * 2.0 ** -24 * size).all()
    assert np.median(np.abs(got - want)[size > 0] / size[size > 0]) < 2.0 ** -23


# ResNet-20's layers with a stride and its first one beside the others in one launch; from N = 74 on with fp16 pieces in the long sums
@pytest.mark.parametrize("bad", [False, True, "hidden"])
@pytest.mark.parametrize("N", [31, 128])
def test_layers_of_several_kinds_in_one_launch(N, bad):
    shapes = [(N, 3, 32, 32, 16, 3, 3, 1, 1, 1, 1)] + [(N, 16, 32, 32, 16, 3, 3, 1, 1, 1, 1)] * 7 + [(N, 16, 32, 32, 32, 3, 3, 2, 2, 1, 1)] \
        + [(N, 32, 16, 16, 32, 3, 3, 1, 1, 1, 1)] * 6 + [(N, 32, 16, 16, 64, 3, 3, 2, 2, 1, 1)] + [(N, 64, 8, 8, 64, 3, 3, 1, 1, 1, 1)] * 5
    ds = [mk(t) for t in shapes]
    kept = (0, 1, 8, 9, 15, 16)                                     # the first layer of each kind is compared with the oracle
    data = {i: rand_inputs(ds[i], 300 + i) for i in kept}
    for X, dY in data.values():
        if bad == "hidden":                                         # (as above)
            X[::2] = 0
            dY[::2] *= np.float32(2.0 ** 28)
        elif bad:
            dY[0, 0, 0, 0], dY[-1, 5, -1, -1], X[1, 2, 0, 0] = np.inf, np.nan, -np.inf
    on_gpu = {i: (to_gpu(X), to_gpu(dY)) for i, (X, dY) in data.items()}
    of = [max(i for i in kept if i <= j) for j in range(len(ds))]
    out = [torch_nan(d) for d in ds]
    s = B.Schedule(ds, [on_gpu[i][0] for i in of], [on_gpu[i][1] for i in of], out)
    m = [B.EXACT] * len(ds)
    s.run(m, B.alloc_workspace(s.workspace_bytes(m)))
    for i in kept:
        with np.errstate(all="ignore"):
            want = oracle.wgrad_exact(oracle_shape(ds[i]), *data[i])
        fine = np.isfinite(want)
        for j, got in enumerate(o.cpu().numpy() for k, o in enumerate(out) if of[k] == i):
            assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[~fine], want[~fine].astype(np.float32), equal_nan=True)
            assert normwise_err(got[fine], want[fine]) < TOL["fp32"] / (1 if bad is True else 50), (i, j)


# ResNet-20's shapes in runs, on both sides of the lines for short layers: 0.14 GFLOP for two layers of a shape, 0.5 for one and
# for strides
@pytest.mark.parametrize("N", [29, 30, 48, 107])
def test_short_layers_in_runs(N):
    import torch
    shapes = [(N, 16, 32, 32, 16, 3, 3, 1, 1, 1, 1)] * 2 + [(N, 32, 16, 16, 32, 3, 3, 1, 1, 1, 1)] * 3 \
        + [(N, 64, 8, 8, 64, 3, 3, 1, 1, 1, 1), (N, 16, 32, 32, 32, 3, 3, 2, 2, 1, 1)]
    ds = [mk(t) for t in shapes]
    data = [rand_inputs(d, 90 + i) for i, d in enumerate(ds)]
    out = [torch_nan(d) for d in ds]
    S = B.Schedule(ds, [to_gpu(x) for x, _ in data], [to_gpu(y) for _, y in data], out)
    mask = np.full(len(ds), B.EXACT, np.uint8)
    S.run(mask, B.alloc_workspace(S.workspace_bytes(mask)))
    torch.cuda.synchronize()
    for d, (X, dY), got in zip(ds, data, out):
        assert normwise_err(got.cpu().numpy(), oracle.wgrad_exact(oracle_shape(d), X, dY)) < TOL["fp32"] / 10


@pytest.mark.parametrize("N", [33, 48])
def test_short_layers_in_runs_with_enough_of_them(N):
    """2 GFLOP of short layers in all, which the three-piece form then takes, beside layers that it does not."""
    import torch
    from tests.test_run_forms import X3_RUN, forms
    assert forms([(B.EXACT, "fp32", N, 16, 32, 16, 7), (B.EXACT, "fp32", N, 32, 16, 32, 7), (B.EXACT, "fp32", N, 3, 32, 16, 1)]) == [X3_RUN, X3_RUN, 0]
    shapes = [(N, 16, 32, 32, 16, 3, 3, 1, 1, 1, 1)] * 7 + [(N, 32, 16, 16, 32, 3, 3, 1, 1, 1, 1)] * 7 + [(N, 3, 32, 32, 16, 3, 3, 1, 1, 1, 1)]
    ds = [mk(t) for t in shapes]
    data = [rand_inputs(d, 130 + i) for i, d in enumerate(ds)]
    out = [torch_nan(d) for d in ds]
    S = B.Schedule(ds, [to_gpu(x) for x, _ in data], [to_gpu(y) for _, y in data], out)
    mask = np.full(len(ds), B.EXACT, np.uint8)
    S.run(mask, B.alloc_workspace(S.workspace_bytes(mask)))
    torch.cuda.synchronize()
    for d, (X, dY), got in zip(ds, data, out):
        assert normwise_err(got.cpu().numpy(), oracle.wgrad_exact(oracle_shape(d), X, dY)) < TOL["fp32"] / 10
