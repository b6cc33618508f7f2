"""The filter transform of fft 16384 and 32768 (a real row as half as many complex points, separated on the way out) at filters of one
tap to the whole transform, odd and even lengths (a pair across the end), with the padded half and without."""
import pytest
import torch

from paper_2311_05908_amd import fftconv, synth
from parity_util import TOL, parity_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M", [16384, 32768])
def test_filter_lengths(M, dtype):
    B, H, N = 2, 3, M // 2
    g = torch.Generator().manual_seed(M)
    u = torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype])
    plan = fftconv.Plan(N, M, H, dtype)
    assert plan.path == "fused3"
    U = torch.fft.rfft(u.double(), M)
    for Nk in (1, 2, 3, 301, M // 2 - 1, M // 2, M // 2 + 1, M - 1, M):
        k = torch.randn(H, Nk, generator=g) / Nk ** 0.5
        K = torch.fft.rfft(k.double(), M)
        for kf, ref in ((plan.filter_fft(k.cuda()), K), (plan.filter_fft_adjoint(k.cuda()), K.conj())):
            y = plan.forward(u.cuda(), kf).cpu().double()
            err = parity_error(y.numpy(), torch.fft.irfft(U * ref, M)[..., :N].numpy(), TOL[dtype], "Nk=%d" % Nk)
            print("filter %s M=%d Nk=%d err=%.3e" % (dtype, M, Nk, err), flush=True)
            assert err <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_filter_lengths_of_8192(dtype):
    """The same at fft 8192, with and without a mask of blocks (a bin and its mirror image masked differently count half)."""
    M, N, H = 8192, 4096, 5
    test_filter_lengths(M, dtype)
    g = torch.Generator().manual_seed(7)
    u, k = torch.randn(2, H, N, generator=g).to(synth.TORCH_DTYPE[dtype]), torch.randn(H, N, generator=g) / N ** 0.5
    keep = torch.randint(0, 2, (64,), generator=g)
    mask = keep.repeat_interleave(M // 64).double()
    weight = (mask + mask[-torch.arange(M) % M]) / 2
    plan = fftconv.Plan(N, M, H, dtype)
    y = plan.forward(u.cuda(), plan.filter_fft(k.cuda(), block_keep=keep.tolist())).cpu().double()
    ref = torch.fft.ifft(torch.fft.fft(u.double(), M) * torch.fft.fft(k.double(), M) * weight, dim=-1).real[..., :N]
    assert parity_error(y.numpy(), ref.numpy(), TOL[dtype], "masked") <= TOL[dtype]
