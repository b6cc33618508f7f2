"""Outer passes of the multi-pass plans at every outer length: rows of one sample, of odd lengths, short of and beyond half the transform, that
begin anywhere in memory; batches with and without a partner for the last row; nothing is read or written beyond."""
import pytest
import torch

from paper_2311_05908_amd import fftconv, synth
from parity_util import TOL, parity_error

pytestmark = pytest.mark.gpu


def conv(x, k, M, N):
    return torch.fft.irfft(torch.fft.rfft(x, M) * torch.fft.rfft(k, M), M)[..., :N]


def placed(t, shift):
    buf = torch.full((t.numel() + shift + 64,), float("nan"), dtype=t.dtype, device="cuda")
    buf[shift:shift + t.numel()] = t.flatten().cuda()
    return buf, buf[shift:shift + t.numel()].view(t.shape)


@pytest.mark.parametrize("B,H,n,shift", [
    (1, 2, 1, 1), (3, 2, 1, 0), (2, 1, 2, 1), (1, 1, -1, 3),       # negative: short of half the transform
    (3, 1, -3, 0), (2, 2, 0, 1), (1, 1, 0, 0), (3, 1, 0.63, 1),    # 0: half the transform; a fraction: that part of it, made odd
])
@pytest.mark.parametrize("M", [8192 << lg for lg in range(10)])
def test_outer_passes(M, B, H, n, shift):
    N = int(M * n) | 1 if isinstance(n, float) else M // 2 + n if n <= 0 else n
    # (a row of one sample in bf16: its spectrum is flat, and at 2^22 points fp16 intermediates of that size are subnormal, 2e-2)
    dtype = "bf16" if N == 1 or (M.bit_length() + B) % 2 else "f16"
    g = torch.Generator().manual_seed(N + B)
    u, w, v = (torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype]) for _ in range(3))
    k = torch.randn(H, N, generator=g) / N ** 0.5
    plan = fftconv.Plan(N, M, H, dtype)
    kf = plan.filter_fft(k.cuda())
    if plan.path != "multipass":
        shift = 0                                                  # the other paths take 16-byte aligned rows
    (_, cu), (_, cw), (_, cv) = (placed(t, shift) for t in (u, w, v))
    for name in ("y", "wv"):
        buf, out = placed(torch.zeros_like(u), shift)
        if name == "y":
            plan.forward(cu, kf, out=out)
            ref, weight = conv(u.double(), k.double(), M, N), None
        else:
            plan.forward_gated(cu, cw, cv, kf, out=out)
            ref, weight = conv(u.double() * w.double(), k.double(), M, N) * v.double(), v.double().abs().numpy()
        assert torch.isnan(buf[:shift]).all() and torch.isnan(buf[shift + u.numel():]).all()
        err = parity_error(out.cpu().double().numpy(), ref.numpy(), TOL[dtype], name, weight=weight)
        print("outer passes %s M=%d B=%d H=%d N=%d %s err=%.3e" % (dtype, M, B, H, N, name, err), flush=True)
        assert err <= TOL[dtype]
    if M >= 65536 and n != 1:
        # rows of u and dy of the filter gradient, fp32 sums: as the existing tests bound it
        dk = plan.backward_filter(cu, cw, N).cpu().double()
        ref = torch.fft.irfft((torch.fft.rfft(u.double(), M).conj() * torch.fft.rfft(w.double(), M)).sum(0), M)[..., :N]
        err = ((dk - ref).norm() / ref.norm()).item()
        print("outer passes M=%d N=%d dk err=%.3e" % (M, N, err), flush=True)
        assert err <= 2e-6
