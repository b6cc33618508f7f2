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
    (16, 16, "16 bits", (35, 40, 56, 97, 113, 160, 171, 256), (1, 15, 24, 32, 57, 64, 72, 85, 114, 128, 142)),
    (16, 16, "f32", (15, 20, 56, 97, 113, 122, 128, 160, 171, 256), (1, 14, 57, 64, 72, 85, 92, 117)),
    (16, 12, "16 bits", (21, 56, 72, 113, 128, 256), (14, 20, 57, 62)),
    (16, 12, "f32", (15, 56, 72, 114, 256), (14, 57, 62)),
    (16, 14, "f32", (15, 56, 97, 114, 256), (14, 57, 72)),
    (16, 10, "16 bits", (15, 57, 114, 256), (14,)),
    (8, 8, "16 bits", (22, 256), (1, 8, 16)),
    (16, 8, "16 bits", (12, 57, 256), (1, 11)),
    (8, 6, "16 bits", (8, 256), (1, 7)),
    (8, 8, "f32", (20, 256), (1, 8, 16)),              # (8 channels 12.9 -> 13.3 us)
    (16, 8, "f32", (6, 57, 256), (1, 4)),
    (8, 6, "f32", (8, 57, 256), (1, 7)),
    (4, 4, "f32", (1, 768), ()),
    (32, 4, "f32", (), (1, 768)),
])
def test_filters_formed_on_load(A, blocks, dtype, on_load, from_memory):
    """Channels whose filter transform forms its rows itself, and those where an outer pass is faster: a second round of few workgroups too."""
    f = rule("_ZN7fftconv14filter_on_loadElllb", i64, i64, i64, flag)
    assert [H for H in on_load + from_memory if f(A, blocks, H, dtype == "f32")] == list(on_load)


@pytest.mark.parametrize("A,blocks,gated,on_load,from_memory", [
    (8, 8, False, ((1, 12), (12, 1), (1, 256)), ((1, 1), (3, 1), (1, 11))),             # (B, H); a row 16.9 -> 17.9 us
    (8, 6, False, ((1, 1), (2, 256)), ()),
    (16, 8, False, ((1, 2), (2, 1), (4, 256), (4, 3), (3, 6), (27, 5)), ((1, 1), (3, 1), (3, 5), (5, 3), (23, 5))),      # (odd batches: 3.35e-7 of error, on load 3.40e-7)
    (16, 6, False, ((3, 5), (2, 4)), ((3, 4),)),
    (16, 6, True, ((5, 5), (8, 2)), ((5, 3), (9, 2))),
    (16, 4, False, ((3, 1), (5, 5)), ()),
    (4, 4, True, ((1, 12), (12, 1)), ((1, 1), (4, 2))),
    (4, 4, False, ((1, 1), (2, 300)), ()),
    (16, 4, True, ((1, 1), (2, 300)), ()),
    (8, 8, True, ((1, 36), (36, 1)), ((1, 35),)),
    (8, 6, True, ((1, 26), (26, 1)), ((1, 25),)),
    (16, 8, True, ((1, 56), (1, 64), (2, 29), (3, 19)), ((1, 14), (1, 57))),
    (16, 16, True, (), ((1, 256), (4, 256))),
    (16, 16, False, ((1, 16), (1, 24), (2, 15), (2, 28), (2, 32), (3, 20), (4, 16), (1, 90), (1, 114), (1, 200), (1, 256), (2, 57), (3, 57)),
     ((4, 14), (1, 20), (1, 57), (1, 64), (1, 171), (1, 190), (1, 228), (2, 29), (4, 15))),
    (16, 14, False, ((1, 15), (1, 74), (1, 114), (3, 20)), ((1, 57), (1, 64), (2, 29))),
    (16, 12, False, ((1, 57), (2, 29), (4, 15)), ((8, 14),)),
])
def test_fp32_rows_formed_on_load(A, blocks, gated, on_load, from_memory):
    """Batch rows and channels of fp32 convolutions whose kernel forms its rows itself, and those that take an outer pass."""
    f = rule("_ZN7fftconv12conv_on_loadEllllb", i64, i64, i64, i64, flag)
    assert [s for s in on_load + from_memory if f(A, blocks, *s, gated)] == list(on_load)


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("blocks", range(1, 17))
def test_fp32_rows_beside_a_workspace_without_pairs(blocks, gated):
    """The workspace of outer length 16 has no room for pairs of rows where two batch rows form theirs on load with and without a gate: larger
    batches then do, too."""
    f = rule("_ZN7fftconv12conv_on_loadEllllb", i64, i64, i64, i64, flag)
    for H in list(range(1, 70)) + [114, 256, 1000]:
        if f(16, blocks, 2, H, True) and f(16, blocks, 2, H, False):
            assert all(f(16, blocks, B, H, gated) for B in range(2, 200)), H


def test_rows_of_a_single_batch_row():
    """Rows as half as many points, or with zeros for imaginary parts (fp16 1 x 400 x 2048 7.6 us so, 8.2 in half the points)."""
    f = rule("_ZN7fftconv8row_loneEllb", i64, i64, flag)
    for f16, first in ((False, 257), (True, 513)):
        assert all(f(2048, H, f16) for H in (1, 256, 8192))
        assert [H for H in (1, 256, 257, 400, 512, 513, 768, 8192) if f(4096, H, f16)] == [H for H in (257, 400, 512, 513, 768, 8192) if H >= first]
        assert not any(f(M, H, f16) for M in (256, 512, 1024) for H in (1, 8192))


def test_rows_of_four_passes():
    """(N, H, B) of calls without gates in rows of four passes, and of those in three (fp32 2 x 1024 x 200 at fft 2048 7.7 us so, 8.0 in four)."""
    f = rule("_ZN7fftconv8row_quadElblll", i64, flag, i64, i64, i64)
    four = [(1024, 4, 2), (200, 768, 2), (1024, 1025, 1), (200, 640, 4), (200, 800, 4), (300, 1024, 4), (200, 2049, 2), (1024, 8192, 2), (1025, 900, 2), (2048, 768, 16),
            (1024, 1500, 64), (2048, 1, 1), (150, 1, 1), (150, 1, 1 << 24)]
    three = [(200, 769, 1), (1024, 1024, 2), (200, 512, 4), (256, 1793, 2), (200, 1024, 4), (256, 2048, 1),
             (2048, 1024, 16), (2047, 2048, 8), (1500, 768, 64), (1025, 1500, 32), (2048, 3, 1 << 31),      # (64 x 768 x 1500 188 us, 204 in four)
             (149, 1, 1), (8, 4, 2), (150, 1, (1 << 24) + 1), (1024, 3, 1 << 32)]                             # (8 samples: 5.6e-8 of error, 6.6e-8 in four)
    assert [c for c in four + three if f(2048, True, *c)] == four
    for M, f32, N, most in ((2048, False, 2048, 512), (2048, False, 1025, 512), (2048, False, 1024, 256), (2048, False, 100, 256),
                            (4096, True, 20, 256), (4096, True, 4096, 256), (4096, False, 1, 256), (4096, False, 4096, 256)):
        assert f(M, f32, N, most, 2) and not f(M, f32, N, most + 1, 2) and not f(M, f32, N, 1, 1 << 33)
    assert not f(4096, True, 19, 1, 1)


def test_gradients_formed_on_load():
    """Calls whose kernel forms its rows itself; with as many batch rows as 32 bits count, the last run's end would not fit."""
    f = rule("_ZN7fftconv12grad_on_loadEllll", i64, i64, i64, i64)
    on_load = [(8, 6, 26, 1), (8, 8, 36, 1), (8, 8, 1, 36), (16, 8, 20, 1), (16, 2, 1, 1), (4, 1, 1, 1), (4, 4, 43, 1), (16, 1, (1 << 31) - 514, 1)]
    from_memory = [(8, 6, 25, 1), (8, 8, 35, 1), (16, 8, 19, 1), (4, 4, 42, 1), (16, 9, 300, 300), (32, 1, 8, 8), (2, 1, 8, 8), (16, 1, (1 << 31) - 513, 1), (16, 1, 1 << 33, 1)]
    assert [c for c in on_load + from_memory if f(*c)] == on_load
