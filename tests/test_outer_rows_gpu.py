"""Transforms beyond 16384 points whose kernels form the rows of the outer factor from the samples themselves (outer_row.h): blocks of 8192
samples that end early, odd numbers of them, a single one, rows that fill the transform, and calls on either side of the lines to the
kernels that read them from memory.  Filter transform, convolution, both gates, both gradients against the same in fp64."""
import pytest
import torch

from paper_2311_05908_amd import fftconv, synth
from parity_util import TOL, parity_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("B,H,N,Nk,M", [
    (3, 11, 8191, 8191, 32768), (2, 9, 8192, 1, 32768), (2, 30, 8193, 8193, 32768),      # one block, two
    (2, 22, 32767, 32767, 32768), (1, 43, 16385, 100, 32768), (1, 42, 16385, 16384, 32768),    # 129 and 126 blocks: either side of the line
    (2, 13, 24577, 24577, 65536), (1, 26, 65536, 40000, 65536), (1, 3, 32768, 32768, 65536),   # of half a transform and of a whole one
    (5, 3, 65535, 65535, 131072), (5, 4, 65535, 65535, 131072), (1, 3, 65536, 65536, 131072),      # 135 blocks, 180, 27
    (1, 3, 131071, 131071, 131072), (2, 8, 81919, 8193, 131072),                         # sixteen blocks to a row, ten
    (1, 57, 100, 131072, 131072), (1, 97, 100, 131072, 131072),                          # filters in a second round of few workgroups, and of many
    (2, 29, 106501, 100, 131072), (1, 20, 122882, 100, 131072), (3, 1, 57345, 100, 65536),     # rows in a second round of few; too few rows
    (17, 1, 100, 100, 131072),                                                           # runs of one batch row; eighths of less than a row's blocks
    (150, 1, 9000, 9000, 32768),                                                         # runs of two, whose blocks lie across the dies' eighths
])
def test_rows_formed_on_load(dtype, B, H, N, Nk, M):
    g = torch.Generator().manual_seed(N + Nk)
    u, w, v, dy = (torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype]) for _ in range(4))
    k = torch.randn(H, Nk, generator=g) / Nk ** 0.5
    plan = fftconv.Plan(N, M, H, dtype, path="staged" if dtype == "f32" else "multipass")
    F = lambda x: torch.fft.rfft(x.double(), M)
    back = lambda X, n: torch.fft.irfft(X, M)[..., :n]

    def check(got, ref, tol, what, weight=None):
        err = parity_error(got.cpu().double().numpy(), ref.numpy(), tol, what, weight=weight)
        print("rows formed on load %s %s B=%d H=%d N=%d Nk=%d M=%d err=%.3e" % (what, dtype, B, H, N, Nk, M, err), flush=True)
        assert err <= tol

    nan = lambda x: torch.full_like(x, float("nan"), device="cuda")
    kf = plan.filter_fft(k.cuda())
    check(plan.forward(u.cuda(), kf, out=nan(u)), back(F(u) * F(k), N), TOL[dtype], "y")
    check(plan.forward_gated(u.cuda(), w.cuda(), v.cuda(), kf, out=nan(u)), v.double() * back(F(u.double() * w.double()) * F(k), N),
          TOL[dtype], "gated", v.double().numpy())           # (an element's rounding is relative to its gate)
    check(plan.backward_input(dy.cuda(), plan.filter_fft_adjoint(k.cuda()), out=nan(dy)), back(F(dy) * F(k).conj(), N), TOL[dtype], "du")
    check(plan.backward_filter(u.cuda(), dy.cuda(), Nk, out=nan(k)), back((F(u).conj() * F(dy)).sum(0), Nk), TOL["f32"], "dk")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_gradients_of_few_channels_keep_the_chip_busy(dtype):
    """As many samples in 2 channels and 128 batch rows as in 8 and 32: an eighth of each run's ten blocks to a die left three dies idle (f32 155 us
    beside 79)."""
    M = 65536
    best = {(128, 2): float("inf"), (32, 8): float("inf")}
    x, z = (torch.randn(256 * M, device="cuda").to(synth.TORCH_DTYPE[dtype]) for _ in range(2))
    plans = {s: fftconv.Plan(M, M, s[1], dtype, path="staged" if dtype == "f32" else "multipass") for s in best}
    for _ in range(10):
        for (B, H), plan in plans.items():
            u, dy, dk = x.view(B, H, M), z.view(B, H, M), torch.empty(H, M, device="cuda")
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            plan.backward_filter(u, dy, M, out=dk)
            t[0].record()
            for _ in range(20):
                plan.backward_filter(u, dy, M, out=dk)
            t[1].record()
            t[1].synchronize()
            best[B, H] = min(best[B, H], t[0].elapsed_time(t[1]) * 50)
    print("dk %s 128 x 2, 32 x 8: %.1f, %.1f us" % (dtype, best[128, 2], best[32, 8]), flush=True)
    assert best[128, 2] <= 1.3 * best[32, 8]
