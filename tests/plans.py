"""How the library deals a call's rows to its attention kernels (a host function, no GPU needed)."""
import ctypes as C

import paper_2609_15810_amd as vc


def forward_plan(N, BH, qk_fmt=vc.QK_INT8, p_mode=vc.P_EXPCAST):
    """(n8, first4, n4, first1, n1) of csrc/vc_internal.hpp's ForwardPlan."""
    out = (C.c_int32 * 5)()
    f = vc.lib().vc_internal_forward_plan
    f.argtypes = [C.c_int32] * 4 + [C.POINTER(C.c_int32)]
    f.restype = None
    f(N, BH, qk_fmt, p_mode, out)
    return tuple(out)
