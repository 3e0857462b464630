"""Approximated layers on planes of up to 256 positions in LDS: tiles of input and output channels with a remainder, planes of one and of
several positions a lane, the largest plane LDS holds, strides and paddings, batches that leave wavefronts without an image, alone
and in a run, against the oracle on every dW entry."""
import numpy as np
import pytest

import oracle
from paper_1908_05460_amd import binding as B
from tests.gpu_util import TOL, normwise_err, oracle_shape, rand_inputs, to_gpu
from tests.test_gpu_regs import run_approx

pytestmark = pytest.mark.gpu
BOUND = TOL["fp32"] / 50        # fp32 sums of a few products a wavefront, added in 64 bits

# (N, C, H, W, K, stride, padding)
SHAPES = [(100, 61, 5, 5, 65, 1, 1), (200, 41, 2, 3, 70, 1, 1), (21, 130, 7, 9, 129, 1, 1), (40, 66, 8, 8, 300, 2, 0), (160, 33, 13, 13, 71, 1, 1), (47, 131, 16, 16, 128, 1, 1),
          (92, 128, 16, 16, 64, 2, 1), (9, 300, 16, 16, 320, 1, 0), (30, 110, 4, 64, 256, 1, 1), (50, 125, 64, 4, 128, 1, 1), (70, 67, 15, 17, 70, 2, 0),
          (100, 67, 15, 17, 128, 2, 0), (60, 90, 7, 7, 90, 2, 0)]
OLDER = [SHAPES[3], SHAPES[10]]     # beside them, shapes that the LDS gather and the fused form keep (tests/test_run_forms.py)
BF16 = SHAPES[:5] + [(66, 128, 16, 16, 128, 2, 1)]


def desc(t, dtype="fp32"):
    N, C, H, W, K, stride, pad = t
    return B.desc(N, C, H, W, K, R=3, S=3, stride=stride, pad=pad, dtype=B.BF16 if dtype == "bf16" else B.F32)


# bf16: those that no matrix-core form takes
@pytest.mark.parametrize("t,dtype", [(t, "fp32") for t in SHAPES] + [(t, "bf16") for t in BF16])
def test_alone_matches_the_oracle(t, dtype):
    import torch
    d = desc(t, dtype)
    X, dY = rand_inputs(d, 31, dtype)
    want, want_idx, _ = oracle.wgrad_approx(oracle_shape(d), X, dY)
    idx = torch.full((d.N, d.K), -1, dtype=torch.int32, device="cuda")
    got = B.conv_wgrad_approx(d, to_gpu(X), to_gpu(dY), idx_out=idx).cpu().numpy()
    assert normwise_err(got, want) < BOUND
    assert np.array_equal(idx.cpu().numpy(), want_idx)


def test_run_matches_the_oracle():
    """More groups than a launch carries, layers of one shape, others in registers beside them; selections element by element and in pieces."""
    shapes = SHAPES[:10] + [SHAPES[5]] * 2 + [(5, 64, 8, 8, 128, 1, 1), (5, 64, 4, 4, 128, 1, 1)]
    dtypes = ["fp32"] * len(shapes) + ["bf16"] * 3
    shapes += [SHAPES[0], SHAPES[2], SHAPES[4]]
    ds = [desc(t, dtype) for t, dtype in zip(shapes, dtypes)]
    data = [rand_inputs(d, 50 + i, dtype) for i, (d, dtype) in enumerate(zip(ds, dtypes))]
    for d, (X, dY), got in zip(ds, data, run_approx(ds, data)):
        assert normwise_err(got * 4, oracle.wgrad_approx(oracle_shape(d), X, dY)[0]) < BOUND


def test_many_layers_in_a_run_are_not_summed_in_longer_rows():
    """24 layers share the chip's workgroups, N = 1000: the fused form, in chunks of its own, is 1.23e-7 of the result (2-norm) off, this one
    1.0e-7, with as many chunks as fill the chip alone 1.55e-7."""
    import torch
    d = desc((1000, 64, 8, 16, 64, 1, 1))
    X, dY = rand_inputs(d, 61)
    Xg, Yg = to_gpu(X), to_gpu(dY)
    out = [torch.full((d.K, d.C, 3, 3), float("nan"), device="cuda") for _ in range(24)]
    s = B.Schedule([d] * 24, [Xg] * 24, [Yg] * 24, out)
    m = [B.APPROX] * 24
    s.run(m, B.alloc_workspace(s.workspace_bytes(m)), scale=1.0)
    want = oracle.wgrad_approx(oracle_shape(d), X, dY)[0]
    for got in out:
        err = np.linalg.norm(got.cpu().numpy() - want) / np.linalg.norm(want)
        assert err < 1.35e-7, err


@pytest.mark.parametrize("where", ["X", "dY"])
@pytest.mark.parametrize("t", [SHAPES[0], SHAPES[5], SHAPES[6]])
def test_infinities_and_nans(t, where):
    """As in the definition: one of X reaches the taps that see it, a map's sum its patch, the padding's zeros among it."""
    d = desc(t)
    X, dY = rand_inputs(d, 33)
    A = X if where == "X" else dY
    A[3, 5, 0, 0], A[7, 11, -1, -1], A[8, 2, 1, 1] = np.inf, -np.inf, np.nan
    with np.errstate(all="ignore"):
        want = oracle.wgrad_approx(oracle_shape(d), X, dY)[0]
    got = B.conv_wgrad_approx(d, to_gpu(X), to_gpu(dY)).cpu().numpy()
    fine = np.isfinite(want)
    assert not fine.all() and np.array_equal(got[~fine], want[~fine].astype(np.float32), equal_nan=True)
    assert normwise_err(got[fine], want[fine]) < BOUND
