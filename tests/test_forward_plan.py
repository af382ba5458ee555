"""The rule that deals a call's rows to the attention kernels, on the host: every row exactly once, no key split
where there is nothing to split, and no second launch behind full rounds for a rest that they absorb."""
import pytest

import paper_2609_15810_amd as vc
from plans import forward_plan

FORMS = [(f, p) for f in (vc.QK_INT8, vc.QK_FP8, vc.QK_MXFP4) for p in (vc.P_EXPCAST, vc.P_EXP_THEN_CAST)]


@pytest.mark.parametrize("N", [1, 31, 32, 33, 127, 128, 129, 255, 256, 257, 300, 384, 385, 512, 1000, 1025, 1500, 2048,
                               4097, 5850, 13833, 16384, 16385, 32760, 75600, 131072])
def test_every_row_is_dealt_once(N):
    per = {q: -(-N // q) for q in (256, 128, 32)}

    def starts_at(pos, q):   # (head, query) of workgroup pos
        return pos // per[q], pos % per[q] * q

    for BH in (1, 2, 3, 5, 7, 12, 24, 40, 45, 55, 60, 100, 127, 128, 129, 200, 255, 256, 257, 300, 511, 640, 800):
        for form in FORMS:
            n8, first4, n4, first1, n1 = forward_plan(N, BH, *form)
            assert min(n8, n4, n1) >= 0 and (n4 == 0 or n1 == 0)
            if n4 or n1:   # the second kernel's first workgroup begins where the full rounds end
                q, first, n = (128, first4, n4) if n4 else (32, first1, n1)
                assert starts_at(first, q) == starts_at(n8, 256)
                assert first + n == BH * per[q]
                assert n8 % 256 == 0
            else:
                assert n8 == BH * per[256]


@pytest.mark.parametrize("N", [1, 64, 128, 129, 160, 192, 255, 256])
def test_no_key_split_up_to_two_tiles(N):
    for BH in (1, 2, 3, 8, 31, 32, 51, 64, 200, 300):
        for form in FORMS:
            assert forward_plan(N, BH, *form)[4] == 0


# calls whose rest was measured on each kernel: heads, tokens, score format, path, the kernel of the rest
@pytest.mark.parametrize("BH,N,fmt,p,queries", [
    (55, 1051, vc.QK_INT8, 0, 256), (103, 1051, vc.QK_INT8, 0, 256), (205, 1051, vc.QK_MXFP4, 0, 256),
    (205, 1051, vc.QK_FP8, 1, 256), (57, 2060, vc.QK_INT8, 0, 256), (229, 2060, vc.QK_INT8, 0, 256),
    (344, 1300, vc.QK_INT8, 0, 256), (208, 1152, vc.QK_INT8, 0, 256),
    (69, 1000, vc.QK_INT8, 0, 32), (34, 2000, vc.QK_INT8, 0, 32), (46, 1300, vc.QK_MXFP4, 0, 32),
    (59, 2060, vc.QK_FP8, 1, 32), (86, 6000, vc.QK_INT8, 0, 32), (12, 4096 * 2, vc.QK_INT8, 0, 128),
    (24, 5850, vc.QK_INT8, 0, 128), (7, 13833, vc.QK_FP8, 1, 128),
])
def test_rest_behind_full_rounds(BH, N, fmt, p, queries):
    n8, _, n4, _, n1 = forward_plan(N, BH, fmt, p)
    assert n8 >= 256 and (256 if n4 == n1 == 0 else 128 if n4 else 32) == queries
