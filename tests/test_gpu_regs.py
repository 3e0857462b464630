"""Approximated fp32 layers on 8x8, 4x4 and 2x2 planes, whose planes lie in registers: tiles of four and of eight wavefronts, one image,
stages that end early, batch chunks, strides, alone and in runs, against the oracle on every dW entry."""
import numpy as np
import pytest

import oracle
from paper_1908_05460_amd import binding as B
from tests.gpu_util import TOL, normwise_err, oracle_shape, rand_inputs, to_gpu

pytestmark = pytest.mark.gpu

# (N, C, HW, K, stride): a stage is 2 images of 8x8 planes, 4 of 4x4 or 16 of 2x2 ones; K = 160 has no whole tile of eight wavefronts
SHAPES = [(1, 64, 4, 128, 1), (5, 64, 4, 160, 1), (16, 128, 4, 128, 2), (67, 192, 4, 256, 1), (128, 64, 4, 128, 1),
          (1, 64, 2, 128, 1), (17, 64, 2, 160, 1), (33, 128, 2, 128, 2), (70, 192, 2, 256, 1),
          (1, 64, 8, 128, 1), (5, 64, 8, 160, 1), (16, 128, 8, 128, 2), (43, 192, 8, 256, 1), (128, 64, 8, 128, 1)]
BOUND = TOL["fp32"] / 50        # fp32 sums of up to 128 products


def desc(t):
    N, C, HW, K, stride = t
    return B.desc(N, C, HW, HW, K, R=3, S=3, stride=stride, pad=1)


def run_approx(ds, data):
    import torch
    out = [torch.full((d.K, d.C, 3, 3), float("nan"), device="cuda") for d in ds]
    S = B.Schedule(ds, [to_gpu(x) for x, _ in data], [to_gpu(y) for _, y in data], out)
    mask = np.full(len(ds), B.APPROX, np.uint8)
    S.run(mask, B.alloc_workspace(S.workspace_bytes(mask)), scale=0.25)
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("t", SHAPES)
def test_alone_matches_the_oracle(t):
    import torch
    d = desc(t)
    X, dY = rand_inputs(d, 5)
    want, want_idx, _ = oracle.wgrad_approx(oracle_shape(d), X, dY)
    idx = torch.full((d.N, d.K), -1, dtype=torch.int32, device="cuda")
    got = B.conv_wgrad_approx(d, to_gpu(X), to_gpu(dY), idx_out=idx).cpu().numpy()
    assert normwise_err(got, want) < BOUND
    assert np.array_equal(idx.cpu().numpy(), want_idx)


@pytest.mark.parametrize("shapes", [SHAPES, [SHAPES[4], SHAPES[8], SHAPES[4]], [SHAPES[3]] * 9 + SHAPES])
def test_runs_match_the_oracle(shapes):
    """Several shapes and layers of one shape in one launch, more groups than a launch carries.  (2x2 planes take the form beside
    4x4 ones only.)"""
    ds = [desc(t) for t in shapes]
    data = [rand_inputs(d, 60 + i) for i, d in enumerate(ds)]
    for d, (X, dY), got in zip(ds, data, run_approx(ds, data)):
        assert normwise_err(got * 4, oracle.wgrad_approx(oracle_shape(d), X, dY)[0]) < BOUND


@pytest.mark.parametrize("hw", [2, 4, 8])
def test_unaligned_tensors(hw):
    """A tensor that does not begin at a multiple of 16 bytes takes another form, in the same workspace."""
    import torch
    d = desc((9, 64, hw, 128, 1))
    X, dY = rand_inputs(d, 8)
    buf = torch.zeros(X.size + 1, device="cuda")
    buf[1:] = to_gpu(X).flatten()
    got = B.conv_wgrad_approx(d, buf[1:].view(X.shape), to_gpu(dY)).cpu().numpy()
    assert normwise_err(got, oracle.wgrad_approx(oracle_shape(d), X, dY)[0]) < BOUND


@pytest.mark.parametrize("hw", [2, 4, 8])
def test_infinities(hw):
    """An infinity of X reaches only the taps whose kept position sees it."""
    ds = [desc((6, 64, hw, 128, 1)), desc((7, 64, 4, 128, 1))]
    data = [rand_inputs(d, 9) for d in ds]
    data[0][0][2, 3, hw - 1, 0] = np.inf
    data[0][0][5, 60, 0, hw - 1] = -np.inf
    with np.errstate(all="ignore"):
        want = oracle.wgrad_approx(oracle_shape(ds[0]), *data[0])[0]
    got = run_approx(ds, data)[0] * 4
    fine = np.isfinite(want)
    assert not fine.all() and np.array_equal(got[~fine], want[~fine].astype(np.float32), equal_nan=True)
    assert normwise_err(got[fine], want[fine]) < BOUND


# strided maps of up to four positions, which the registers do not take: (N, C, HW, K, stride)
STRIDED = [(256, 64, 2, 128, 2), (256, 64, 4, 128, 2), (256, 64, 8, 128, 4)]


@pytest.mark.parametrize("t", STRIDED)
def test_strided_maps_of_few_positions_are_summed_in_short_chains(t):
    """Alone and beside long work on 4x4 planes, which leaves each layer few batch chunks.  The error of a chain of N additions of terms
    of one size grows as the square root of N: 2.0e-7 (2x2) and 1.4e-7 (4x4) in one of 256; the sparsified form's wavefronts add up
    a quarter of them or less: 1.0e-7 and 0.9e-7."""
    ds = [desc(t)] * 3 + [desc((t[0], 512, 4, 512, 1))]
    data = [rand_inputs(d, 90 + i) for i, d in enumerate(ds)]
    want = oracle.wgrad_approx(oracle_shape(ds[0]), *data[0])[0]
    for got in (run_approx(ds, data)[0] * 4, B.conv_wgrad_approx(ds[0], *map(to_gpu, data[0])).cpu().numpy()):
        assert np.linalg.norm(got - want) < 1.25e-7 * np.linalg.norm(want)


@pytest.mark.parametrize("t", [(6, 64, 2, 128, 2), (6, 64, 4, 128, 1), (6, 64, 4, 128, 2), (6, 64, 8, 128, 1), (6, 64, 8, 128, 2)])
def test_infinite_and_nan_map_sums(t):
    """A map whose sum is not finite makes NaNs of the padding's zeros that its patch sees, in runs and alone."""
    ds = [desc(t), desc((7, 64, 4, 128, 1))]
    data = [rand_inputs(d, 11) for d in ds]
    Y = data[0][1]
    Y[1, 3, 0, 0], Y[2, 40, -1, -1], Y[5, 127, 0, -1] = np.inf, -np.inf, np.nan
    with np.errstate(all="ignore"):
        want = oracle.wgrad_approx(oracle_shape(ds[0]), *data[0])[0]
    for got in (run_approx(ds, data)[0] * 4, B.conv_wgrad_approx(ds[0], *map(to_gpu, data[0])).cpu().numpy()):
        fine = np.isfinite(want)
        assert not fine.all() and np.array_equal(got[~fine], want[~fine].astype(np.float32), equal_nan=True)
        assert normwise_err(got[fine], want[fine]) < BOUND


@pytest.mark.parametrize("t, most, beside", [((16, 512, 4, 512, 1), 8, 0), ((128, 256, 4, 512, 1), 32, 1), ((33, 256, 8, 512, 1), 11, 3),
                                             ((64, 256, 8, 512, 1), 16, 0), ((128, 64, 4, 128, 1), 8, 1)])
def test_length_of_the_sums(t, most, beside):
    """The images of a batch chunk, read off a sum that starts with 2^24: the ones that follow it in its chain are lost, those of the
    other chunks are not."""
    d = desc(t)
    X, dY = np.ones((d.N, d.C, d.H, d.W), np.float32), np.zeros((d.N, d.K, d.Ho, d.Wo), np.float32)
    X[0] = 2.0 ** 24
    dY[:, :, 1, 1] = 1
    if beside:
        b = desc((d.N, 512, 4, 512, 1))
        got = run_approx([d] + [b] * beside, [(X, dY)] + [rand_inputs(b, 1)] * beside)[0] * 4
    else:
        got = B.conv_wgrad_approx(d, to_gpu(X), to_gpu(dY)).cpu().numpy()
    lost = d.N - 1 - (got - 2.0 ** 24)
    assert 0 <= lost.min() and lost.max() <= most               # (most - 1, and one where the sum is odd)


def test_fewer_chunks_only_where_fewer_additions_lie_in_a_row():
    """The gather cuts this layer into 16 chunks of three images: 19 additions between a product and the result.  In one chunk they would
    be 48 (1.18e-7 from 64 bits where the gather is at 1.13e-7)."""
    d, b = desc((48, 128, 8, 256, 1)), desc((48, 256, 8, 256, 1))
    X, dY = np.ones((d.N, d.C, d.H, d.W), np.float32), np.zeros((d.N, d.K, d.Ho, d.Wo), np.float32)
    X[0] = 2.0 ** 24
    dY[:, :, 1, 1] = 1
    got = run_approx([d] + [b] * 3, [(X, dY)] + [rand_inputs(b, 1)] * 3)[0] * 4
    lost = int((d.N - 1 - (got - 2.0 ** 24)).max())             # a chunk's images, or one less: the sum may be odd
    assert lost + -(-d.N // lost) <= 19


def test_infinite_and_nan_map_sums_on_2x2_planes():
    """Neither the registers (in the run) nor the plain product (alone) multiply the padding: the same NaNs, fewer than the definition's."""
    ds = [desc((6, 64, 2, 128, 1)), desc((7, 64, 4, 128, 1))]
    data = [rand_inputs(d, 11) for d in ds]
    Y = data[0][1]
    Y[1, 3, 0, 0], Y[2, 40, -1, -1], Y[5, 127, 0, -1] = np.inf, -np.inf, np.nan
    with np.errstate(all="ignore"):
        want = oracle.wgrad_approx(oracle_shape(ds[0]), *data[0])[0]
    run, alone = run_approx(ds, data)[0] * 4, B.conv_wgrad_approx(ds[0], *map(to_gpu, data[0])).cpu().numpy()
    assert np.array_equal(np.isnan(run), np.isnan(alone)) and not np.isfinite(run).all()
    assert np.array_equal(run[np.isinf(want)], want[np.isinf(want)].astype(np.float32))
    fine = np.isfinite(want)
    assert np.isfinite(run[fine]).all() and normwise_err(run[fine], want[fine]) < BOUND
