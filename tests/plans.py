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
