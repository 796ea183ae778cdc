"""The short root, reciprocal and quotient of the step kernel (csrc/stq_round.h) are the correctly rounded ones over the whole
of their ranges: the functions themselves, compiled for the GPU and the host, against 64-bit arithmetic."""
import ctypes as C
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch  # before the library: one HIP runtime for both

NATIVE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native")


@pytest.fixture(scope="module")
def native():
    lib = os.path.join(NATIVE, "libshort_forms.so")
    if not os.path.exists(lib):
        from paper_2604_06836_amd.build import build_shared
        build_shared(os.path.join(NATIVE, "short_forms.hip"), lib)
    lib = C.CDLL(lib)
    lib.short_forms_check.argtypes = [C.c_int, C.c_uint32, C.c_uint32, C.POINTER(C.c_uint64), C.POINTER(C.c_uint32)]
    lib.short_forms_quotients.argtypes = [C.c_uint32, C.c_uint32, C.c_int, C.c_int, C.c_int, C.POINTER(C.c_uint64)]
    lib.short_forms_quotients.restype = C.c_uint64
    return lib


def on_gpu(native, which, a, b):
    assert torch.cuda.is_available()
    bad, first = C.c_uint64(), C.c_uint32()
    assert native.short_forms_check(which, a, b, C.byref(bad), C.byref(first)) == 0
    return bad.value, first.value


def bits(x):
    return int(np.float32(x).view(np.uint32))


@pytest.mark.gpu
def test_root_of_every_float_of_its_range(native):
    assert on_gpu(native, 0, 0, 0)[0] == 0
    bad, first = on_gpu(native, 0, bits(2.0 ** -96), bits(2.0 ** 96))
    assert bad == 0, hex(first)


@pytest.mark.gpu
def test_reciprocal_of_every_float_of_its_range(native):
    bad, first = on_gpu(native, 1, bits(2.0 ** -70), bits(2.0 ** 40))
    assert bad == 0, hex(first)


@pytest.mark.gpu
def test_quotients_over_the_range(native):
    bad, first = on_gpu(native, 2, 0, 1 << 30)
    assert bad == 0, first


@pytest.mark.gpu
def test_the_comparison_sees_a_wrong_result(native):
    """Out of range the forms are wrong, and the comparison says so: the root of a subnormal, the reciprocal of one too."""
    assert on_gpu(native, 0, 1, 1000)[0] > 900 and on_gpu(native, 1, 1, 1000)[0] > 900


# n and d at the ends of their ranges and between
@pytest.mark.parametrize("en,ed", [(0, 0), (-85, 39), (39, -70), (-85, -70)])
def test_quotients_next_to_a_rounding_boundary(native, en, ed):
    """Given the correctly rounded reciprocal y, the first quotient n*y is within 2 units in the last place and the last step
    multiplies its exact residual by y, 2^-24 off: the result can only be wrong where n/d lies within 2^-23 units of the middle
    between two floats, |R| / (2 D) <= 2^-23 with D < 2^24, so |R| < 4.  All of those, and |R| = 4."""
    edges = np.linspace(1 << 23, 1 << 24, 65).astype(int)

    def part(k):
        pairs = C.c_uint64()
        return native.short_forms_quotients(int(edges[k]), int(edges[k + 1]), 4, en, ed, C.byref(pairs)), pairs.value
    with ThreadPoolExecutor(8) as ex:
        got = list(ex.map(part, range(64)))
    assert sum(b for b, _ in got) == 0
    assert sum(n for _, n in got) > 2e7
