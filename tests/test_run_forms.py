"""Which form the layers of a run take (host code of libwgrad): forms that pay only where enough work shares their launch, by runs
that were timed both ways."""
import ctypes as ct

import pytest

from paper_1908_05460_amd import binding as B, inputs

# bf16 layers row after row, exact and approximated; short fp32 layers in 16-bit pieces; approximated layers' planes in registers and in LDS
ROWS, SPARSE_ROWS, X3_RUN, REGS, LDS = 1, 2, 3, 4, 5
E, A = B.EXACT, B.APPROX


def flat(run):
    descs, methods, at = [], [], []
    for method, dtype, n, c, hw, k, count, *stride in run:
        at.append(len(descs))
        descs += [B.desc(n, c, hw, hw, k, stride=stride[0] if stride else 1, dtype=B.BF16 if dtype == "bf16" else B.F32)] * count
        methods += [method] * count
    return descs, methods, at


def forms(run):
    """run: [(method, type, N, C, H = W, K, layers[, stride])] -> the forms of its shapes"""
    descs, methods, at = flat(run)
    f = B.load()._ZN5wgrad14schedule_formsEPK15wgrad_conv_descPKhiPi
    f.argtypes = [ct.c_void_p, ct.c_void_p, ct.c_int, ct.c_void_p]
    n = len(descs)
    out = (ct.c_int * n)()
    assert f((B.ConvDesc * n)(*descs), (ct.c_uint8 * n)(*methods), n, out) == 0
    return [out[i] for i in at]


def stack(layers, method, dtype, n):
    return [(method(i) if callable(method) else method, dtype, n, l.C, l.H, l.K, 1) for i, l in enumerate(layers)]


# us before the form / with it
@pytest.mark.parametrize("run, taken", [
    ([(E, "bf16", 64, 512, 4, 512, 1), (E, "bf16", 64, 512, 2, 512, 1)], [0, 0]),                       # 18.1 / 35.4
    ([(E, "bf16", 512, 512, 4, 512, 1), (E, "bf16", 512, 16, 32, 16, 1)], [0, 0]),                      # 46.1 / 56.8
    ([(E, "bf16", 64, 128, 4, 128, 4), (E, "fp32", 64, 16, 16, 16, 1)], [0, 0]),                        # 22.6 / 33.0
    ([(E, "bf16", 200, 256, 8, 256, 1), (E, "bf16", 200, 128, 2, 128, 1)], [0, 0]),                     # 32.9 / 40.1
    ([(E, "bf16", 16, 512, 4, 512, 1), (E, "bf16", 16, 512, 8, 512, 1)], [0, 0]),                       # 18.7 / 25.6
    ([(E, "bf16", 64, 3, 32, 64, 1), (E, "bf16", 64, 64, 8, 64, 1)], [0, 0]),                           # 17.8 / 22.7
    ([(E, "bf16", 9, 256, 4, 256, 5), (E, "bf16", 9, 512, 4, 512, 1), (E, "bf16", 9, 64, 4, 64, 1)], [0, 0, 0]),   # too short
    ([(E, "bf16", 512, 512, 4, 512, 1), (E, "bf16", 512, 512, 8, 512, 1)], [ROWS, ROWS]),               # 203.7 / 142.2
    ([(E, "bf16", 200, 512, 4, 512, 4), (E, "bf16", 200, 512, 8, 512, 1)], [ROWS, ROWS]),               # 133.8 / 96.5
    ([(E, "bf16", 256, 64, 8, 64, 5), (E, "bf16", 256, 16, 32, 16, 7)], [ROWS, 0]),                     # (ResNet-20) 83.7 / 77.6
    ([(E, "bf16", 200, 512, 8, 512, 2)], [ROWS]),                                                       # 111.9 / 95.7
    ([(E, "bf16", 64, 512, 8, 512, 2)], [0]),                                                           # 44.5 / 45.2
    ([(E, "bf16", 16, 64, 32, 64, 2)], [0]),                                                            # 17.5 / 21.7
    ([(E, "bf16", 16, 512, 8, 512, 2), (E, "bf16", 16, 16, 32, 16, 1)], [0, 0]),                        # 29.9 / 37.1
    ([(E, "bf16", 272, 64, 8, 128, 2), (E, "bf16", 272, 3, 32, 64, 1)], [0, 0]),                        # 28.8 / 33.1
])
def test_exact_bf16_row_after_row(run, taken):
    assert forms(run) == taken


@pytest.mark.parametrize("n", [16, 64, 160, 512])
def test_exact_bf16_vgg19_goes_row_after_row(n):
    """All but the 2x2 planes and, in long batches, the first layer; also with every other layer approximated."""
    layers = inputs.vgg19_stack()
    for every in (1, 2):
        got = forms(stack(layers, lambda i: E if i % every == 0 else A, "bf16", n))
        assert [f == ROWS for f in got] == [i % every == 0 and l.H >= 4 and (l.C >= 16 or n < 512) for i, l in enumerate(layers)]


@pytest.mark.parametrize("run, taken", [
    ([(A, "bf16", 64, 128, 4, 128, 3)], [0]),                                                           # 11.6 / 22.2
    ([(A, "bf16", 16, 512, 4, 512, 1), (A, "bf16", 16, 512, 2, 512, 1)], [0, 0]),                       # 21.5 / 39.2
    ([(A, "bf16", 200, 128, 4, 128, 1), (A, "bf16", 200, 128, 2, 128, 1)], [0, 0]),                     # 25.3 / 38.3
    ([(A, "bf16", 16, 256, 8, 256, 3), (A, "bf16", 16, 64, 16, 64, 1)], [0, 0]),                        # 23.9 / 30.0
    ([(A, "bf16", 48, 512, 4, 512, 1), (A, "bf16", 48, 512, 2, 512, 1)], [0, 0]),                       # 26.3 / 41.0
    ([(A, "bf16", 512, 512, 4, 512, 1), (E, "bf16", 512, 64, 16, 64, 1)], [0, 0]),                      # one layer
    ([(A, "bf16", 512, 512, 4, 512, 3)], [SPARSE_ROWS]),                                                # 95.4 / 75.6
    ([(A, "bf16", 64, 64, 16, 64, 3)], [SPARSE_ROWS]),                                                  # 27.5 / 23.3
    ([(A, "bf16", 256, 64, 8, 64, 5), (A, "bf16", 256, 16, 32, 16, 7)], [SPARSE_ROWS, 0]),              # (ResNet-20) 72.2 / 65.2
    ([(A, "bf16", 64, 64, 8, 64, 4), (E, "bf16", 64, 64, 8, 64, 1)], [0, 0]),
    ([(A, "bf16", 256, 64, 8, 64, 4), (E, "bf16", 256, 64, 8, 64, 1)], [SPARSE_ROWS, 0]),               # (ResNet-20) 90.6 / 83.1
    ([(A, "bf16", 200, 128, 16, 128, 1), (A, "bf16", 200, 64, 16, 64, 1)], [SPARSE_ROWS, SPARSE_ROWS]),  # 56.7 / 37.1
    ([(A, "bf16", 200, 256, 8, 256, 2), (E, "bf16", 200, 64, 16, 64, 1)], [SPARSE_ROWS, 0]),            # 113.4 / 54.5
])
def test_approximated_bf16_row_after_row(run, taken):
    assert forms(run) == taken


@pytest.mark.parametrize("n", [16, 64, 160, 512])
def test_approximated_bf16_vgg19_goes_row_after_row(n):
    """All on 4x4 to 16x16 planes; also with every other layer exact."""
    layers = inputs.vgg19_stack()
    for every in (1, 2):
        got = forms(stack(layers, lambda i: A if i % every == every - 1 else E, "bf16", n))
        assert [f == SPARSE_ROWS for f in got] == [i % every == every - 1 and 4 <= l.H <= 16 for i, l in enumerate(layers)]


@pytest.mark.parametrize("run, taken", [
    ([(E, "fp32", 32, 32, 16, 32, 3), (E, "fp32", 32, 3, 32, 16, 1)], [0, 0]),                          # 18.8 / 26.5
    ([(E, "fp32", 64, 128, 4, 128, 6), (E, "fp32", 64, 16, 16, 16, 1)], [0, 0]),
    ([(E, "fp32", 128, 64, 4, 64, 6), (E, "fp32", 128, 3, 32, 16, 1)], [0, 0]),                         # 28.1 / 33.4
    ([(E, "fp32", 100, 16, 32, 16, 6), (E, "fp32", 100, 3, 32, 16, 1)], [X3_RUN, 0]),                   # 48.5 / 39.9
    ([(E, "fp32", 32, 32, 16, 32, 3), (E, "fp32", 32, 64, 16, 64, 1)], [X3_RUN, 0]),                    # 29.0 / 19.7 (with the longer one)
    ([(E, "fp32", 64, 32, 16, 32, 3), (E, "fp32", 64, 64, 8, 64, 2)], [X3_RUN, X3_RUN]),                # nothing else
    ([(E, "fp32", 64, 32, 16, 32, 3)], [0]),                                                            # (in a launch of its own)
])
def test_short_fp32_layers(run, taken):
    assert forms(run) == taken


@pytest.mark.parametrize("n, taken", [(16, False), (48, True), (80, True)])
def test_resnet20_in_the_three_piece_form(n, taken):
    got = forms(stack(inputs.resnet20_stack(), E, "fp32", n))
    assert (sum(f == X3_RUN for f in got) >= 10) == taken


@pytest.mark.parametrize("run, taken", [
    ([(A, "fp32", 256, 512, 2, 512, 2), (A, "fp32", 256, 64, 4, 128, 1)], [0, REGS]),                   # 67.6 / 83.6
    ([(A, "fp32", 128, 512, 2, 512, 2), (A, "fp32", 128, 64, 4, 128, 1)], [0, REGS]),                   # 47.5 / 48.8
    ([(A, "fp32", 64, 512, 2, 512, 2), (A, "fp32", 64, 64, 4, 128, 1)], [REGS, REGS]),                  # 36.3 / 29.3
    ([(A, "fp32", 256, 512, 2, 512, 4), (A, "fp32", 256, 512, 4, 512, 1)], [REGS, REGS]),               # 191.8 / 107.6
    ([(A, "fp32", 256, 128, 2, 128, 1), (A, "fp32", 256, 64, 4, 128, 1)], [REGS, REGS]),                # 46.8 / 22.6
    ([(A, "fp32", 128, 512, 2, 512, 4)], [0]),
    ([(A, "fp32", 128, 512, 2, 512, 4), (A, "fp32", 128, 256, 8, 256, 1)], [0, REGS]),
    ([(A, "fp32", 128, 512, 2, 512, 1), (E, "fp32", 128, 512, 4, 512, 1)], [0, 0]),
])
def test_planes_in_registers(run, taken):
    assert forms(run) == taken


def joins(run):
    """1: the shape is in the launch of 16-wide tiles because others are; 2: it is there in two fp16 pieces where three bf16 ones could be"""
    descs, methods, at = flat(run)
    f = B.load()._ZN5wgrad14schedule_joinsEPK15wgrad_conv_descPKhiPiS5_
    f.argtypes = [ct.c_void_p, ct.c_void_p, ct.c_int, ct.c_void_p, ct.c_void_p]
    n = len(descs)
    form, out = (ct.c_int * n)(), (ct.c_int * n)()
    assert f((B.ConvDesc * n)(*descs), (ct.c_uint8 * n)(*methods), n, form, out) == 0
    return [out[i] for i in at]


@pytest.mark.parametrize("n, taken", [(16, False), (32, True), (48, True), (80, True), (128, True)])
def test_resnet20_strided_and_first_layers_join_the_others(n, taken):
    """(44 / 53 / 76 / 100 us at N = 32 / 48 / 80 / 128 without, 30 / 38 / 57 / 80 with them)"""
    layers = inputs.resnet20_stack()
    got = joins([(E, "fp32", n, l.C, l.H, l.K, 1, l.stride) for l in layers])
    assert [f == 1 for f in got] == [taken and (l.stride == 2 or l.C == 3) for l in layers]


@pytest.mark.parametrize("n, taken", [(73, False), (74, True), (128, True)])                               # 89 us in bf16 pieces, 80 (N = 128)
def test_resnet20_long_rows_in_two_pieces(n, taken):
    layers = inputs.resnet20_stack()
    got = joins([(E, "fp32", n, l.C, l.H, l.K, 1, l.stride) for l in layers])
    assert [f == 2 for f in got] == [taken and l.stride == 1 and l.C >= 16 and l.H > 8 for l in layers]


def test_nothing_joins_without_a_host():
    assert joins([(E, "fp32", 64, 3, 32, 16, 1), (E, "fp32", 64, 16, 32, 32, 1, 2)]) == [0, 0]
    assert joins([(E, "fp32", 64, 3, 32, 16, 1), (E, "fp32", 64, 512, 4, 512, 2)]) == [0, 0]      # (no 16-wide tiles)


@pytest.mark.parametrize("n, taken", [(64, False), (96, True), (128, True)])                               # 129.7 / 130.9, 167.6 / 159.9
def test_vgg19_planes_in_lds(n, taken):
    layers = inputs.vgg19_stack()
    assert [f == LDS for f in forms(stack(layers, A, "fp32", n))] == [taken and l.H == 16 for l in layers]


def alone(d):
    f = B.load()._ZN5wgrad11approx_formEPK15wgrad_conv_desc
    f.argtypes = [ct.c_void_p]
    return f(ct.byref(d))


# us before the form / with it
@pytest.mark.parametrize("d, taken", [
    (B.desc(32, 128, 16, 16, 128), 0),                                          # 10.4 / 13.0
    (B.desc(48, 128, 16, 16, 128), LDS),                                        # 15.5 / 14.3
    (B.desc(48, 128, 16, 16, 128, stride=2, dtype=B.BF16), 0),                  # 12.9 / 14.0
    (B.desc(64, 128, 16, 16, 128, stride=2, dtype=B.BF16), LDS),                # 15.5 / 14.9
    (B.desc(35, 60, 9, 9, 150), 0),                                             # 14.1 / 14.9
    (B.desc(60, 60, 9, 9, 150), LDS),                                           # 15.3 / 13.6
    (B.desc(128, 128, 8, 8, 128), REGS),
])
def test_planes_in_lds_alone(d, taken):
    assert alone(d) == taken


def test_shapes_of_the_gpu_tests_take_planes_in_lds():
    from tests import test_gpu_planes as P
    for t in P.SHAPES:
        assert alone(P.desc(t)) == (0 if t in P.OLDER else LDS), t
    for t in P.BF16:
        assert alone(P.desc(t, "bf16")) == (0 if t in P.OLDER else LDS), t
