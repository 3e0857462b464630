"""Shapes chosen by the kernel variant that the planner gives them, and the planner itself (host code of libwgrad)."""
import ctypes as ct

from paper_1908_05460_amd import binding as B

# variant (numbered as in csrc/exact_x3_kernel.hpp): shape (N, C, H, W, K, R, S, stride_h, stride_w, pad_h, pad_w), dtype, whether
# the tiles are parts of rows.  The smallest found in which a workgroup has two or more tiles, not all workgroups the same
# number, and neither K nor C divides into whole tiles; 24 and 25 are the 4x4 and 2x2 planes.
PLANS = [
    (0, (91, 93, 6, 64, 119, 3, 3, 3, 1, 0, 1), "fp32", 0),
    (1, (26, 22, 11, 148, 122, 3, 3, 1, 1, 1, 1), "fp32", 1),
    (2, (279, 30, 4, 32, 118, 3, 3, 1, 1, 1, 3), "fp32", 1),
    (2, (266, 62, 28, 12, 26, 3, 3, 1, 1, 1, 0), "fp32", 0),
    (3, (205, 33, 15, 4, 65, 3, 3, 3, 1, 0, 1), "fp32", 0),
    (4, (14, 172, 30, 4, 65, 3, 3, 3, 1, 0, 3), "fp32", 1),
    (4, (277, 11, 37, 8, 33, 3, 3, 3, 1, 1, 0), "fp32", 0),
    (5, (43, 65, 21, 8, 65, 3, 3, 3, 2, 1, 1), "fp32", 0),
    (6, (224, 65, 8, 16, 9, 3, 3, 3, 2, 1, 3), "fp32", 1),
    (6, (115, 33, 7, 16, 33, 3, 3, 3, 2, 1, 3), "fp32", 0),
    (7, (49, 33, 36, 4, 33, 3, 3, 3, 1, 1, 1), "fp32", 0),
    (8, (37, 33, 18, 12, 33, 3, 3, 3, 1, 1, 0), "fp32", 1),
    (8, (25, 65, 35, 6, 33, 3, 3, 3, 1, 0, 0), "fp32", 0),
    (9, (16, 97, 71, 8, 159, 3, 3, 1, 1, 1, 1), "fp32", 0),
    (10, (57, 9, 25, 128, 40, 1, 3, 1, 1, 0, 3), "fp32", 1),
    (10, (107, 11, 51, 64, 13, 1, 3, 3, 1, 0, 0), "fp32", 0),
    (11, (112, 5, 37, 4, 65, 5, 5, 3, 1, 0, 3), "fp32", 1),
    (11, (125, 33, 25, 4, 33, 5, 5, 3, 1, 2, 2), "fp32", 0),
    (12, (72, 96, 32, 32, 97, 3, 3, 1, 1, 1, 1), "bf16", 0),
    (13, (37, 57, 24, 64, 33, 3, 3, 3, 1, 0, 1), "bf16", 1),
    (13, (169, 60, 24, 4, 54, 3, 3, 3, 1, 0, 1), "bf16", 0),
    (14, (286, 60, 4, 24, 65, 3, 3, 3, 1, 0, 3), "bf16", 1),
    (14, (137, 89, 12, 14, 65, 3, 3, 3, 1, 1, 1), "bf16", 0),
    (15, (107, 60, 34, 12, 33, 3, 3, 3, 1, 1, 1), "bf16", 0),
    (16, (47, 92, 27, 4, 33, 3, 3, 3, 1, 0, 3), "bf16", 1),
    (16, (269, 14, 54, 7, 33, 3, 3, 3, 1, 0, 1), "bf16", 0),
    (17, (61, 40, 37, 8, 33, 3, 3, 3, 2, 1, 1), "bf16", 0),
    (18, (116, 33, 7, 16, 40, 3, 3, 3, 2, 1, 3), "bf16", 1),
    (18, (131, 33, 16, 4, 33, 3, 3, 3, 2, 1, 3), "bf16", 0),
    (19, (194, 33, 14, 4, 33, 3, 3, 3, 1, 1, 1), "bf16", 0),
    (20, (37, 33, 11, 4, 33, 3, 3, 1, 1, 0, 3), "bf16", 1),
    (20, (125, 40, 15, 19, 10, 3, 3, 3, 1, 0, 0), "bf16", 0),
    (21, (139, 8, 43, 32, 65, 1, 3, 1, 1, 0, 1), "bf16", 0),
    (22, (92, 8, 15, 70, 40, 1, 3, 1, 1, 0, 3), "bf16", 1),
    (23, (218, 5, 15, 4, 65, 5, 5, 1, 1, 0, 3), "bf16", 1),
    (23, (106, 8, 20, 8, 65, 5, 5, 1, 1, 2, 0), "bf16", 0),
    (24, (74, 250, 4, 4, 450, 3, 3, 1, 1, 1, 1), "fp32", 0),
    (25, (162, 250, 2, 2, 450, 3, 3, 1, 1, 1, 1), "fp32", 0),
]
VARIANTS = 26

# layers that the older forms answer sooner (us of this form / of the older one)
OLDER = [
    ((53, 3, 64, 64, 128, 3, 3, 1, 1, 1, 1), "fp32"),       # 57 / 35
    ((164, 3, 64, 64, 128, 3, 3, 2, 2, 1, 1), "fp32"),      # 76 / 33
    ((190, 3, 12, 37, 161, 3, 3, 2, 2, 1, 1), "fp32"),      # 49 / 30
    ((37, 7, 64, 64, 97, 3, 3, 1, 1, 1, 1), "fp32"),        # 67 / 43
    ((58, 4, 30, 146, 126, 3, 3, 2, 2, 1, 1), "fp32"),      # 60 / 48
    ((8, 3, 112, 112, 128, 5, 5, 1, 1, 2, 2), "fp32"),      # 78 / 65
    ((44, 128, 8, 8, 512, 3, 3, 2, 2, 1, 1), "fp32"),       # 31 / 25
    ((145, 256, 7, 7, 256, 3, 3, 2, 2, 1, 1), "fp32"),      # 126 / 88
    ((125, 256, 17, 9, 128, 3, 3, 2, 2, 1, 1), "fp32"),     # 152 / 99
    ((23, 64, 56, 56, 64, 3, 3, 2, 2, 1, 1), "fp32"),       # 43 / 39
    ((249, 3, 56, 56, 128, 3, 3, 2, 2, 1, 1), "bf16"),      # 50 / 35
    ((12, 3, 112, 112, 128, 3, 3, 1, 1, 1, 1), "bf16"),     # 43 / 33
    ((67, 7, 112, 112, 32, 3, 3, 1, 1, 1, 1), "bf16"),      # 108 / 59
    ((100, 256, 4, 4, 256, 3, 3, 1, 1, 1, 1), "bf16"),      # 25 / 21
    ((40, 512, 4, 4, 512, 3, 3, 1, 1, 1, 1), "bf16"),       # 23 / 15
    ((28, 152, 16, 4, 512, 3, 3, 1, 1, 1, 1), "bf16"),      # 28 / 20
    ((82, 58, 16, 4, 512, 3, 3, 1, 1, 1, 1), "bf16"),       # 35 / 25
    ((90, 256, 4, 4, 512, 3, 3, 1, 1, 1, 1), "bf16"),       # 30 / 26
]


class _Geometry(ct.Structure):
    _fields_ = [(n, ct.c_int) for n in "N C H W K R S sh sw ph pw Ho Wo bf16".split()]


class _Plan(ct.Structure):
    _fields_ = [(n, ct.c_int) for n in "variant ktiles ctiles splits nti ht iht twc h_tiles w_tiles n_groups nch ch packed halo "
                                       "vlo xcol0 lds".split()]

    @property
    def tiles(self):
        return self.w_tiles * self.h_tiles * self.n_groups


def plan(t, dtype):
    """What csrc/exact_x3.hip plans for a shape, and whether a call takes it (0 no, 1 alone, 2 always, 3 in a run of
    several layers only)."""
    lib = B.load()
    one, whole = lib._ZN5wgrad13plan_exact_x3ERKNS_8GeometryERNS_6X3PlanE, lib._ZN5wgrad10plan_exactERKNS_8GeometryE
    one.restype, one.argtypes = ct.c_bool, [ct.c_void_p, ct.c_void_p]
    whole.restype, whole.argtypes = None, [ct.c_void_p, ct.c_void_p]          # (returned through a pointer)
    N, C, H, W, K, R, S, sh, sw, ph, pw = t
    g = _Geometry(N, C, H, W, K, R, S, sh, sw, ph, pw, (H + 2 * ph - R) // sh + 1, (W + 2 * pw - S) // sw + 1, dtype == "bf16")
    p, ex = _Plan(), (ct.c_int * 128)()
    assert one(ct.byref(g), ct.byref(p))
    whole(ct.byref(ex), ct.byref(g))
    at = 27                                            # ints of ExactPlan before the plan of this form
    if ex[at - 1]:
        assert list(ex[at:at + 18]) == [getattr(p, n) for n, _ in _Plan._fields_]
    return p, ex[at - 1]
