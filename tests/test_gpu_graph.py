"""A schedule run recorded into a HIP graph and replayed: every replay must reproduce the eager results bit for
bit (the library launches kernels only -- no memset nodes, no allocation, no synchronisation -- and its kernels
are deterministic), with eager work and synchronisations between the replays."""
import numpy as np
import pytest

import oracle
from paper_1908_05460_amd import binding as B, schedule as sch
from tests.gpu_util import TOL, normwise_err, oracle_shape, rand_inputs, to_gpu

pytestmark = pytest.mark.gpu

STACK = [  # (C, H, K, stride): fused, multi-shape exact, LDS-gather and 2x2-plane shapes, repeated shapes
    (3, 32, 16, 1), (16, 32, 16, 1), (16, 32, 16, 1), (16, 32, 32, 2), (32, 16, 32, 1), (32, 16, 32, 1),
    (64, 8, 128, 1), (128, 4, 256, 1), (128, 4, 256, 1), (64, 2, 128, 1), (64, 2, 128, 1),
]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_schedule_run_replays_from_a_graph(dtype):
    import torch
    N = 16
    descs = [B.desc(N, C, H, H, K, stride=st, dtype=B.BF16 if dtype == "bf16" else B.F32) for C, H, K, st in STACK]
    data = [rand_inputs(d, 40 + i, dtype) for i, d in enumerate(descs)]
    Xs = [to_gpu(x) for x, _ in data]
    dYs = [to_gpu(y) for _, y in data]
    dWs = [torch.zeros((d.K, d.C, 3, 3), device="cuda") for d in descs]
    s = B.Schedule(descs, Xs, dYs, dWs)
    rng = np.random.default_rng(5)
    masks = [np.full(len(descs), sch.EXACT, np.uint8), np.full(len(descs), sch.APPROX, np.uint8),
             rng.integers(0, 4, len(descs)).astype(np.uint8)]
    ws = B.alloc_workspace(max(s.workspace_bytes(m) for m in masks))
    for m in masks:
        kw = dict(scale=1 / 128, sigma=1 / 128, seed=9, offset=1000)
        s.run(m, ws, **kw)
        torch.cuda.synchronize()
        eager = [t.clone() for t in dWs]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            s.run(m, ws, **kw)
        for replay in range(3):
            for t in dWs:
                t.fill_(float("nan"))                    # eager work between the replays
            ws.fill_(replay + 1)                         # stale workspace contents must not matter
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for i, (a, b) in enumerate(zip(eager, dWs)):
                assert torch.equal(a, b), (replay, i, STACK[i], int(m[i]))


def test_topk_schedule_replays_from_a_graph():
    import torch
    N = 8
    descs = [B.desc(N, C, H, H, K, stride=st) for C, H, K, st in STACK]
    data = [rand_inputs(d, 90 + i) for i, d in enumerate(descs)]
    dWs = [torch.zeros((d.K, d.C, 3, 3), device="cuda") for d in descs]
    s = B.Schedule(descs, [to_gpu(x) for x, _ in data], [to_gpu(y) for _, y in data], dWs)
    m = np.array([sch.APPROX, sch.EXACT] * 5 + [sch.APPROX], np.uint8)
    ws = B.alloc_workspace(s.workspace_bytes_topk(m, 4))
    s.run_topk(m, 4, ws, scale=0.25)
    torch.cuda.synchronize()
    eager = [t.clone() for t in dWs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        s.run_topk(m, 4, ws, scale=0.25)
    for replay in range(3):
        for t in dWs:
            t.fill_(float("nan"))
        ws.fill_(replay + 7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(eager, dWs)):
            assert torch.equal(a, b), (replay, i, STACK[i], int(m[i]))


def test_run_of_mixed_types_and_forms_replays_from_a_graph():
    """fp32 and bf16 layers, exact and approximated, in one run: each form that takes several shapes in a launch of its own."""
    import torch
    from tests.test_run_forms import REGS, ROWS, SPARSE_ROWS, X3_RUN, forms
    E, A = B.EXACT, B.APPROX
    run = [(E, "bf16", 48, 64, 16, 128, 2), (E, "bf16", 48, 128, 8, 128, 1), (E, "bf16", 48, 128, 4, 128, 2),
           (A, "bf16", 48, 64, 16, 128, 2), (A, "bf16", 48, 128, 8, 128, 1), (A, "bf16", 48, 128, 4, 256, 2), (A, "bf16", 48, 64, 8, 64, 1),
           (A, "fp32", 48, 64, 8, 128, 1), (A, "fp32", 48, 128, 4, 128, 2), (A, "fp32", 48, 128, 2, 128, 1),
           (E, "fp32", 48, 16, 32, 16, 5), (E, "fp32", 48, 32, 16, 32, 5), (E, "fp32", 48, 3, 32, 16, 1)]
    assert forms(run) == [ROWS] * 3 + [SPARSE_ROWS] * 4 + [REGS] * 3 + [X3_RUN] * 2 + [0]
    descs, m = [], []
    for method, dtype, n, c, hw, k, count in run:
        descs += [B.desc(n, c, hw, hw, k, dtype=B.BF16 if dtype == "bf16" else B.F32)] * count
        m += [method] * count
    data = [rand_inputs(d, 60 + i, "bf16" if d.dtype == B.BF16 else "fp32") for i, d in enumerate(descs)]
    dWs = [torch.zeros((d.K, d.C, 3, 3), device="cuda") for d in descs]
    s = B.Schedule(descs, [to_gpu(x) for x, _ in data], [to_gpu(y) for _, y in data], dWs)
    m = np.array(m, np.uint8)
    ws = B.alloc_workspace(s.workspace_bytes(m))
    s.run(m, ws, scale=1.0)
    torch.cuda.synchronize()
    eager = [t.clone() for t in dWs]
    for d, method, (X, dY), got in zip(descs, m, data, eager):
        g, bf16 = oracle_shape(d), d.dtype == B.BF16
        want = oracle.wgrad_exact(g, X, dY) if method == E else oracle.wgrad_approx(g, X, dY)[0]
        assert normwise_err(got.cpu().numpy(), want) < TOL["bf16" if bf16 and method == A else "fp32"]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        s.run(m, ws, scale=1.0)
    for replay in range(3):
        for t in dWs:
            t.fill_(float("nan"))
        ws.fill_(replay + 3)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(eager, dWs)):
            assert torch.equal(a, b), (replay, i)
