"""The filter gradient of few channels and of transforms beyond 16384 points: the ways batch rows are cut into runs, channels into
trips and a batch into pieces.  Short rows in long transforms, so that the reference is a short linear correlation in fp64."""
import pytest
import torch

from paper_2311_05908_amd import fftconv, synth
from parity_util import TOL, parity_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("B,H,N,M", [
    (1, 2, 301, 32768),                  # one run
    (13, 1, 300, 65536),                 # a run for every batch row
    (33, 1, 77, 32768),                  # runs of two, the last one of one
    (40, 19, 200, 32768),                # two trips, of ten and nine channels
    (17, 1, 1000, 1 << 21),              # the workspace holds 15 batch rows: two pieces, in runs
    (16, 5, 130, 1 << 21),               # five trips of one channel, two pieces each
])
def test_runs_trips_and_pieces(dtype, B, H, N, M):
    g = torch.Generator().manual_seed(B * N)
    u, dy = (torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype]) for _ in range(2))
    plan = fftconv.Plan(N, M, H, dtype, path="staged" if dtype == "f32" else "multipass")
    dk = plan.backward_filter(u.cuda(), dy.cuda(), N).cpu().double()
    U, D = torch.fft.rfft(u.double(), 2 * N), torch.fft.rfft(dy.double(), 2 * N)
    ref = torch.fft.irfft((U.conj() * D).sum(0), 2 * N)[:, :N]
    err = parity_error(dk.numpy(), ref.numpy(), TOL["f32"], "dk")
    print("long gradient %s B=%d H=%d N=%d M=%d err=%.3e" % (dtype, B, H, N, M, err), flush=True)
    assert err <= TOL["f32"]             # fp32 sums whatever the I/O type


@pytest.mark.parametrize("dtype,B,H,N,M", [
    ("f16", 73, 1, 200, 65536),          # 37 runs of two, the last one of one: added up eight at a time, the last time four
    ("bf16", 4, 2, 120, 131072),         # four runs, the fewest that are added up by a kernel of their own
    ("f32", 9, 42, 60, 32768),           # four runs of 126 spectra
    ("f32", 6, 23, 60, 32768), ("f32", 14, 24, 60, 32768),      # six and seven runs of more than 64 spectra
    ("f32", 4, 16, 60, 32768), ("bf16", 11, 8, 60, 65536),               # a multiple of 8 spectra: each added up on its die
    ("f32", 4, 21, 60, 32768), ("f32", 4, 22, 60, 32768),                # on either side of 64 spectra
])
def test_many_runs(dtype, B, H, N, M):
    test_runs_trips_and_pieces(dtype, B, H, N, M)


@pytest.mark.parametrize("B,M", [(64, 32768), (256, 32768), (64, 65536)])
def test_many_runs_are_no_less_precise_than_one(B, M):
    """A channel alone goes in 64 runs or more, which are added up in pairs; the same rows in 128 channels go one after another in multiply-adds.
    (1.00 times the error; 1.04 to 1.06 when runs were added up in order.  2 %: five times what an error's norm over 32768 samples varies by.)"""
    g = torch.Generator(device="cuda").manual_seed(B)
    u, dy = (torch.randn(B, 1, M, generator=g, device="cuda") for _ in range(2))
    ref = sum(torch.fft.rfft(a.double()).conj() * torch.fft.rfft(b.double()) for a, b in zip(u, dy))
    ref = torch.fft.irfft(ref, M)

    def error(H):
        dk = fftconv.Plan(M, M, H, "f32").backward_filter(u.expand(B, H, M).contiguous(), dy.expand(B, H, M).contiguous(), M)
        return ((dk[:1].double() - ref).norm() / ref.norm()).item()

    many, one = error(1), error(128)
    print("dk of %d rows of %d: error %.3e in many runs, %.3e in one" % (B, M, many, one), flush=True)
    assert many <= 1.02 * one


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,H,N,M", [
    (64, 2, 128, 256), (70, 3, 120, 256),        # two runs of one input each; of an input and a ragged one
    (19, 1, 1000, 4096),                         # four transforms of 4096 points to an input: five inputs, five runs
    (13, 100, 4096, 8192), (6, 1, 4000, 8192),   # two runs, of three and four pairs; a run for every pair, ragged rows
    (16, 8, 4000, 8192), (256, 24, 200, 512),    # eight runs of a multiple of 8 channels: each channel added up on its die
    (5, 1, 8192, 16384), (27, 60, 5000, 16384),  # runs of one pair, the last without a partner; four runs, of three and four pairs
    (8, 1, 16384, 32768), (7, 90, 2000, 32768),
])
def test_runs_of_matrix_core_gradients(dtype, B, H, N, M):
    g = torch.Generator().manual_seed(B * N)
    u, dy = (torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype]) for _ in range(2))
    plan = fftconv.Plan(N, M, H, dtype, path="fused3")
    dk = plan.backward_filter(u.cuda(), dy.cuda(), N).cpu().double()
    U, D = torch.fft.rfft(u.double(), 2 * N), torch.fft.rfft(dy.double(), 2 * N)
    ref = torch.fft.irfft((U.conj() * D).sum(0), 2 * N)[:, :N]
    err = parity_error(dk.numpy(), ref.numpy(), TOL[dtype], "dk")
    print("gradient in runs %s B=%d H=%d N=%d M=%d err=%.3e" % (dtype, B, H, N, M, err), flush=True)
    assert err <= TOL[dtype]


@pytest.mark.parametrize("H,M,dtype", [(1, 8192, "bf16"), (100, 8192, "f16"), (300, 512, "bf16"), (7, 16384, "bf16"), (3, 32768, "f16")])
def test_workspace_of_a_larger_batch_of_a_matrix_core_plan(H, M, dtype):
    plan = fftconv.Plan(M // 2, M, H, dtype)
    assert plan.path == "fused3"
    sizes = [int(plan._lib.fftconv_workspace_bytes_backward_filter(plan._h, B)) for B in range(1, 80)]
    assert sizes[0] > 0
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("H,M", [(1, 32768), (40, 65536), (3, 1 << 21), (300, 1 << 17)])
def test_workspace_of_a_larger_batch(H, M):
    """A workspace asked for once, for the largest batch, holds every smaller one."""
    plan = fftconv.Plan(40, M, H, "f32")
    sizes = [int(plan._lib.fftconv_workspace_bytes_backward_filter(plan._h, B)) for B in range(1, 60)]
    assert sizes[0] > 0
    assert sizes == sorted(sizes)
