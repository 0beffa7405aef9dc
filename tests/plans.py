"""dn::frag_plan of the built library, for tests that depend on which GEMM kernel a shape takes."""

import ctypes as C

from paper_2511_06724_amd import dn

LINEAR, VT, CONV, FP8 = range(4)
CUS = 256  # compute units of the device the plans are checked for


class Plan(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("bm", "bn", "x5", "frag", "split", "tail_bands")]


_frag_plan = getattr(dn.lib, "_ZN2dn9frag_planEiiiiibNS_8PlanKindEb")
_frag_plan.argtypes = [C.c_int] * 5 + [C.c_bool, C.c_int, C.c_bool]
_frag_plan.restype = Plan


def plan(M, N, K, kind=LINEAR, geglu=False, fused_reduce=False, out_f32=False):
    return _frag_plan(M, N, K, int(geglu), CUS, fused_reduce, kind, out_f32)


_plan32 = getattr(dn.lib, "_ZN2dn9gemm_planIfEENS_8GemmPlanEiiiiibbbb")
_plan32.argtypes = [C.c_int] * 5 + [C.c_bool] * 4
_plan32.restype = Plan


def plan_fp32(M, N, K, geglu=False, conv=False):
    return _plan32(M, N, K, int(geglu), CUS, False, False, conv, False)


# One shape per tile and split the plans can choose, each with a ragged last row tile and a
# ragged last column tile: (kind, M, N, K, geglu, out_f32) -> (bm, bn, x5, split). Convolutions
# as (M = n H W, N, K = 9 Cin) with the images in CONV_IMAGES.
COVER = {
    (LINEAR, 33, 32, 64, False, True): (64, 128, 0, 1),
    (LINEAR, 33, 32, 1280, False, True): (64, 128, 0, 5),
    (LINEAR, 1000, 1248, 64, False, True): (64, 160, 0, 1),
    (LINEAR, 1900, 288, 1920, False, True): (64, 160, 0, 4),
    (LINEAR, 12000, 352, 64, False, True): (128, 128, 0, 1),
    (LINEAR, 6000, 32, 2560, False, True): (128, 128, 0, 5),
    (LINEAR, 2500, 1312, 64, False, True): (128, 160, 0, 1),
    (LINEAR, 5000, 1568, 64, False, False): (128, 160, 1, 1),
    (LINEAR, 3000, 288, 5120, False, True): (128, 160, 1, 5),
    (LINEAR, 12000, 480, 64, False, True): (128, 256, 0, 1),
    (LINEAR, 129, 3872, 10240, False, True): (128, 256, 0, 8),
    (LINEAR, 33, 64, 64, True, False): (128, 256, 0, 1),
    (VT, 66, 96, 64, False, False): (64, 128, 0, 1),
    (VT, 4000, 352, 64, False, False): (64, 160, 0, 1),
    (VT, 20000, 32, 960, False, False): (128, 128, 0, 1),
    (VT, 1900, 2528, 320, False, False): (128, 160, 0, 1),
    (VT, 20000, 672, 128, False, False): (128, 256, 0, 1),
    (CONV, 35, 32, 576, False, False): (64, 128, 0, 1),
    (CONV, 35, 32, 1728, False, False): (64, 128, 0, 6),
    (CONV, 20000, 288, 576, False, False): (128, 128, 0, 1),
    (CONV, 12000, 32, 2880, False, False): (128, 128, 0, 5),
    (CONV, 12000, 288, 576, False, False): (128, 160, 1, 1),
    (CONV, 3000, 288, 5760, False, False): (128, 160, 1, 5),
    (CONV, 5000, 1184, 576, False, False): (128, 256, 0, 1),
    (CONV, 1500, 1312, 2880, False, False): (128, 256, 0, 3),
    (FP8, 33, 32, 128, False, True): (128, 128, 0, 1),
    (FP8, 33, 32, 1280, False, True): (128, 128, 0, 5),
    (FP8, 8000, 608, 128, False, True): (128, 256, 0, 1),
    (FP8, 33, 64, 128, True, False): (128, 256, 0, 1),
    (FP8, 12000, 160, 10240, False, True): (128, 256, 0, 5),
}
CONV_IMAGES = {35: (1, 5, 7), 1500: (1, 30, 50), 3000: (2, 30, 50), 5000: (2, 50, 50), 12000: (3, 50, 80),
               20000: (2, 100, 100)}
