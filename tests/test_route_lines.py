"""Lines between routes that take the same call (the library's own rules, no device involved), at the calls measured on either side of them."""
import ctypes

import pytest

from paper_2311_05908_amd import fftconv

i64, flag = ctypes.c_int64, ctypes.c_bool


def rule(name, *types):
    f = fftconv.load()[name]
    f.argtypes, f.restype = types, ctypes.c_bool
    return f


@pytest.mark.parametrize("A,blocks,dtype,on_load,from_memory", [
    (16, 16, "16 bits", (15, 20, 40, 56, 97, 113, 160, 171, 256), (1, 14, 57, 64, 72, 85, 114, 128, 142)),
    (16, 16, "f32", (15, 20, 56, 97, 113, 128, 160, 171, 256), (1, 14, 57, 64, 72, 85, 92, 117)),
    (16, 12, "16 bits", (15, 56, 72, 113, 128, 256), (14, 57, 62)),
    (16, 12, "f32", (15, 56, 72, 118, 256), (14, 57, 62)),
    (16, 10, "16 bits", (15, 57, 114, 256), (14,)),
    (8, 8, "16 bits", (8, 16, 256), (1, 7)),
    (8, 8, "f32", (11, 16, 256), (1, 7, 8, 9)),              # (8 channels 12.9 -> 13.3 us)
    (16, 8, "f32", (6, 57, 256), (1, 4)),
    (8, 6, "f32", (8, 57, 256), (1, 7)),
    (4, 4, "f32", (1, 768), ()),
    (32, 4, "f32", (), (1, 768)),
])
def test_filters_formed_on_load(A, blocks, dtype, on_load, from_memory):
    """Channels whose filter transform forms its rows itself, and those where an outer pass is faster: a second round of few workgroups too."""
    f = rule("_ZN7fftconv14filter_on_loadElllb", i64, i64, i64, flag)
    assert [H for H in on_load + from_memory if f(A, blocks, H, dtype == "f32")] == list(on_load)
