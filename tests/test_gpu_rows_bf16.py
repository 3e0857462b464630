"""bf16 layers row after row (4x4 to 32x32 planes): edges of its tiles, groups of images and batch chunks, in runs of several
layers and (approximated ones) alone, against the oracle on every dW entry."""
import numpy as np
import pytest

import oracle
from paper_1908_05460_amd import binding as B
from tests.gpu_util import TOL, normwise_err, oracle_shape, rand_inputs, to_gpu
from tests.test_run_forms import ROWS, SPARSE_ROWS, forms

pytestmark = pytest.mark.gpu

# (N, C, HW, K): a group is 32 / HW images and a tile 64 channels; a second tile of 1, 32, 33 or 36 channels, batches that end
# within a group, one image, and (with 64 channels on a side and many images) several chunks of several blocks each
SHAPES = [(1, 16, 4, 64), (9, 65, 4, 64), (67, 64, 4, 128), (300, 100, 4, 64),
          (1, 20, 8, 64), (6, 97, 8, 64), (43, 64, 8, 192), (150, 36, 8, 64),
          (1, 64, 16, 64), (5, 100, 16, 64), (38, 128, 16, 64), (90, 17, 16, 128),
          (1, 33, 32, 64), (4, 64, 32, 128), (21, 40, 32, 64), (60, 64, 32, 64)]


def desc(t):
    N, C, HW, K = t
    return B.desc(N, C, HW, HW, K, R=3, S=3, pad=1, dtype=B.BF16)


def run_layers(ds, Xs, dYs, method, scale=1.0):
    """The layers in one run, beside a layer of zeros that is work enough for this form to take the run."""
    import torch
    more = desc((320, 64, 16, 64))
    ds = ds + [more]
    Xs, dYs = Xs + [torch.zeros((320, 64, 16, 16), dtype=torch.bfloat16, device="cuda")], dYs + [torch.zeros((320, 64, 16, 16), dtype=torch.bfloat16, device="cuda")]
    assert forms([(method, "bf16", d.N, d.C, d.H, d.K, 1) for d in ds]) == [ROWS if method == B.EXACT else SPARSE_ROWS] * len(ds)
    out = [torch.full((d.K, d.C, 3, 3), float("nan"), device="cuda") for d in ds]
    S = B.Schedule(ds, Xs, dYs, out)
    mask = np.full(len(ds), method, np.uint8)
    S.run(mask, B.alloc_workspace(S.workspace_bytes(mask)), scale=scale)
    torch.cuda.synchronize()
    assert not out[-1].any()
    return out[:-1]


def run_exact(ds, data):
    return [o.cpu().numpy() for o in run_layers(ds, [to_gpu(x) for x, _ in data], [to_gpu(y) for _, y in data], B.EXACT)]


@pytest.mark.parametrize("hw", [4, 8, 16, 32])
def test_runs_match_the_oracle(hw):
    """All shapes of one plane size in one launch, two layers of the first."""
    shapes = [t for t in SHAPES if t[2] == hw]
    ds = [desc(t) for t in [shapes[0]] + shapes]
    data = [rand_inputs(d, 40 + i, "bf16") for i, d in enumerate(ds)]
    for d, (X, dY), got in zip(ds, data, run_exact(ds, data)):
        # fp32 sums of exact products
        assert normwise_err(got, oracle.wgrad_exact(oracle_shape(d), X, dY)) < TOL["fp32"] / 50


def test_short_batches_are_summed_in_short_chains():
    """A workgroup's few blocks have sums of their own.  With u = 2^-24 a chain of n additions costs about n / 2 u^2 of the squared error: of
    3 groups of images, 48 steps, in sums of 32 and 16 8.7e-8, in six of eight 6.2e-8."""
    ds = [desc((9, 128, 8, 128)), desc((9, 64, 8, 256)), desc((9, 256, 8, 64))]
    data = [rand_inputs(d, 60 + i, "bf16") for i, d in enumerate(ds)]
    for d, (X, dY), got in zip(ds, data, run_exact(ds, data)):
        want = oracle.wgrad_exact(oracle_shape(d), X, dY)
        assert np.linalg.norm(got - want) < 7.3e-8 * np.linalg.norm(want)


def test_alone_matches_the_oracle():
    """A long layer alone, which another form takes; the last batch chunk is shorter than the others."""
    d = desc((131, 128, 16, 128))
    X, dY = rand_inputs(d, 3, "bf16")
    got = B.conv_wgrad_exact(d, to_gpu(X), to_gpu(dY)).cpu().numpy()
    assert normwise_err(got, oracle.wgrad_exact(oracle_shape(d), X, dY)) < TOL["fp32"] / 50


@pytest.mark.parametrize("where", ["X", "dY"])
@pytest.mark.parametrize("bad", [0x7F80, 0xFF80, 0x7FC0])
def test_infinities_and_nans(where, bad):
    """Rows above and below a plane are not multiplied, and an infinity or a NaN of dY beside them makes NaNs of the
    padding's zeros all the same; one of X reaches only what sees it."""
    ds = [desc(t) for t in ((9, 33, 4, 64), (5, 33, 8, 64), (3, 33, 16, 64), (2, 33, 32, 64))]
    data = []
    for d in ds:
        X, dY = rand_inputs(d, 7, "bf16")
        a = X if where == "X" else dY
        for at in ((0, 0, 0, 0), (-1, -1, -1, -1), (0, 1, 0, a.shape[3] // 2), (-1, 2, a.shape[2] // 2, 0)):
            a[at] = bad
        data.append((X, dY))
    for d, (X, dY), got in zip(ds, data, run_exact(ds, data)):
        with np.errstate(all="ignore"):
            want = oracle.wgrad_exact(oracle_shape(d), X, dY)
        fine = np.isfinite(want)
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[~fine], want[~fine].astype(np.float32), equal_nan=True)
        assert normwise_err(got[fine], want[fine]) < TOL["fp32"] / 50


def rounded_sums(d, idx, sums):
    """dY as the approximated gradient contracts it: each map's sum, rounded to bf16 (to nearest even), at its position."""
    b = sums.astype(np.float32).view(np.uint32)
    out = np.zeros((d.N * d.K, d.Ho * d.Wo), np.uint16)
    out[np.arange(d.N * d.K), idx.ravel()] = ((b + 0x7FFF + ((b >> 16) & 1)) >> 16).astype(np.uint16).ravel()
    return out.reshape(d.N, d.K, d.Ho, d.Wo)


@pytest.mark.parametrize("t", [t for t in SHAPES if t[2] <= 16] + [(131, 128, 16, 128)])
def test_approximated_alone(t):
    import torch
    d = desc(t)
    X, dY = rand_inputs(d, 21, "bf16")
    idx = torch.full((d.N, d.K), -1, dtype=torch.int32, device="cuda")
    sums = torch.empty((d.N, d.K), device="cuda")
    got = B.conv_wgrad_approx(d, to_gpu(X), to_gpu(dY), scale=0.5, idx_out=idx, sum_out=sums).cpu().numpy()
    idx, sums = idx.cpu().numpy(), sums.cpu().numpy()
    assert np.array_equal(idx, oracle.select(oracle_shape(d), dY)[0])
    want = oracle.wgrad_exact(oracle_shape(d), X, rounded_sums(d, idx, sums)) * 0.5
    assert normwise_err(got, want) < TOL["fp32"] / 50       # fp32 sums of exact products, whichever form takes the shape


def test_approximated_runs():
    """All shapes in one launch; more groups than one carries."""
    ds = [desc(t) for t in SHAPES if t[2] <= 16]
    data = [rand_inputs(d, 80 + i, "bf16") for i, d in enumerate(ds)]
    out = run_layers(ds, [to_gpu(x) for x, _ in data], [to_gpu(y) for _, y in data], B.APPROX, scale=0.25)
    for d, (X, dY), got in zip(ds, data, out):
        idx, sums = B.conv_wgrad_select(d, to_gpu(dY))      # (a sum in 32 bits may round the other way than one in 64)
        assert np.array_equal(idx.cpu().numpy(), oracle.select(oracle_shape(d), dY)[0])
        want = oracle.wgrad_exact(oracle_shape(d), X, rounded_sums(d, idx.cpu().numpy(), sums.cpu().numpy())) * 0.25
        assert normwise_err(got.cpu().numpy(), want) < TOL["fp32"] / 50


def approximated(ds, data, alone):
    """-> [(dW, what the exact oracle makes of the rounded sums)]"""
    Xs, dYs = [to_gpu(x) for x, _ in data], [to_gpu(y) for _, y in data]
    out = [B.conv_wgrad_approx(d, x, y) for d, x, y in zip(ds, Xs, dYs)] if alone else run_layers(ds, Xs, dYs, B.APPROX)
    for d, (X, dY), y, got in zip(ds, data, dYs, out):
        idx, sums = (t.cpu().numpy() for t in B.conv_wgrad_select(d, y))
        with np.errstate(all="ignore"):
            yield got.cpu().numpy(), oracle.wgrad_exact(oracle_shape(d), X, rounded_sums(d, idx, sums))


@pytest.mark.parametrize("alone", [True, False])
@pytest.mark.parametrize("bad", [0x7F80, 0xFF80, 0x7FC0])
def test_approximated_infinite_and_nan_sums(bad, alone):
    """A map whose sum is not finite, kept in a first, a last and an inner row: NaNs of the padding's zeros as in the exact gradient of the
    sparsified map."""
    ds = [desc(t) for t in ((40, 33, 4, 64), (9, 33, 8, 64), (5, 33, 16, 64), (9, 100, 8, 128))]
    data = [rand_inputs(d, 7, "bf16") for d in ds]
    for d, (X, dY) in zip(ds, data):
        for at in ((0, 0, 0, 0), (-1, -1, -1, -1), (0, 1, 0, d.W // 2), (-1, 2, d.H // 2, 0), (2, 3, d.H - 1, 1), (1, 5, 1, d.W - 1)):
            dY[at] = bad
    for got, want in approximated(ds, data, alone):
        fine = np.isfinite(want)
        assert not fine.all() and np.array_equal(got[~fine], want[~fine].astype(np.float32), equal_nan=True)
        assert normwise_err(got[fine], want[fine]) < TOL["fp32"] / 50


@pytest.mark.parametrize("alone", [True, False])
def test_approximated_infinities_of_X(alone):
    """The operand's kept places of value zero make NaNs of an infinity that no position selected; other channels, and what is
    not a NaN, are as without it."""
    ds = [desc(t) for t in ((40, 33, 4, 64), (9, 33, 8, 64), (5, 33, 16, 64), (9, 100, 8, 128))]
    data = [rand_inputs(d, 8, "bf16") for d in ds]
    for d, (X, dY) in zip(ds, data):
        X[2, 3, d.H - 1, 0], X[4, 20, 0, d.W - 1] = 0x7F80, 0xFF80
    finite = [(np.where(X & 0x7F80 == 0x7F80, 0, X).astype(np.uint16), dY) for X, dY in data]
    for (got, _), (_, want), d, (X, dY) in zip(approximated(ds, data, alone), approximated(ds, finite, alone), ds, data):
        with np.errstate(all="ignore"):
            selected = oracle.wgrad_approx(oracle_shape(d), X, dY)[0]       # the definition: the selected patches only
        assert np.isfinite(np.delete(got, [3, 20], 1)).all() and np.isnan(got[np.isnan(selected)]).all()
        assert not np.isfinite(got[~np.isfinite(selected)]).any() and np.isfinite(got).any(axis=(0, 2, 3)).all()
        fine = np.isfinite(got)
        assert normwise_err(got[fine], want[fine]) < TOL["fp32"] / 50


def shifted(a, by):
    """The tensor `by` elements into an allocation."""
    import torch
    t = to_gpu(a)
    buf = torch.empty(t.numel() + by, dtype=t.dtype, device="cuda")
    buf[by:] = t.flatten()
    return buf[by:].view(t.shape)


@pytest.mark.parametrize("hw", [4, 8, 16])
@pytest.mark.parametrize("by", [4, 8])
def test_tensors_aligned_to_8_and_to_16_bytes(hw, by):
    """The kernels copy 16 bytes at a time; an X that begins between two multiples of 16 takes another form, alone and in runs."""
    import torch
    ds = [desc((38, 64, hw, 128)), desc((38, 128, hw, 64)), desc((38, 128, 8, 128))]
    data = [rand_inputs(d, 30 + i, "bf16") for i, d in enumerate(ds)]
    Xs, dYs = [shifted(x, by) for x, _ in data], [shifted(y, by) for _, y in data]
    assert all(x.data_ptr() % 16 == by * 2 % 16 for x in Xs)
    for method in (B.EXACT, B.APPROX):
        out = run_layers(ds, Xs, dYs, method)
        for d, X, dY, (x, y), run in zip(ds, Xs, dYs, data, out):
            if method == B.EXACT:
                alone, want = B.conv_wgrad_exact(d, X, dY), oracle.wgrad_exact(oracle_shape(d), x, y)
            else:
                idx = torch.empty((d.N, d.K), dtype=torch.int32, device="cuda")
                sums = torch.empty((d.N, d.K), device="cuda")
                alone = B.conv_wgrad_approx(d, X, dY, idx_out=idx, sum_out=sums)
                want = oracle.wgrad_exact(oracle_shape(d), x, rounded_sums(d, idx.cpu().numpy(), sums.cpu().numpy()))
            for got in (run, alone):
                assert normwise_err(got.cpu().numpy(), want) < TOL["fp32"] / 50
