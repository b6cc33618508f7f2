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


@pytest.mark.parametrize("B", [1, 2, 3])
@pytest.mark.parametrize("M", [8192 << lg for lg in range(10)])
def test_rows_of_one_fp16_sample(M, B):
    """The shortest rows in fp16 at every outer length.  Values within a quarter of 1, so that every row's bound is one number: some roundings
    of 2^-11 (input gate, k_f, intermediates, output), and, as fp16 k_f and its products are kept at boost / fft_size (boost = min(fft_size / 8192, 64))
    and are subnormal there from 2^20 points on, two roundings of 2^-25 fft_size / boost over the product's size, in a flat spectrum the same in every bin."""
    H = 5
    g = torch.Generator().manual_seed(M + B)

    def near_one(*shape):
        return (0.8 + 0.45 * torch.rand(*shape, generator=g)) * (1 - 2 * torch.randint(0, 2, shape, generator=g))

    u, w, v = (near_one(B, H, 1).to(torch.float16) for _ in range(3))
    k = near_one(H, 1)
    plan = fftconv.Plan(1, M, H, "f16")
    kf = plan.filter_fft(k.cuda())
    (_, cu), (_, cw), (_, cv) = (placed(t, 1) for t in (u, w, v))
    for name in ("y", "wv"):
        buf, out = placed(torch.zeros_like(u), 1)
        if name == "y":
            plan.forward(cu, kf, out=out)
            inner, ref = u.double() * k.double(), u.double() * k.double()
        else:
            plan.forward_gated(cu, cw, cv, kf, out=out)
            inner = u.double() * w.double() * k.double()
            ref = inner * v.double()
        assert torch.isnan(buf[:1]).all() and torch.isnan(buf[1 + u.numel():]).all()
        err = ((out.cpu().double() - ref).abs() / ref.abs()).max().item()
        bound = 2.0 ** -9 + 2 * 2.0 ** -25 * M / min(M // 8192, 64) / inner.abs().min().item()
        print("one sample f16 M=%d B=%d %s err=%.3e bound=%.3e" % (M, B, name, err, bound), flush=True)
        assert err <= bound


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,H,N,M", [
    (3, 128, 500, 65536),       # the last row of an odd batch with the pairs, at the line
    (3, 129, 500, 65536),       # ... and beyond, as a real row
    (5, 2, 4001, 1 << 22),      # outer length 512, the line again
    (3, 3, 4001, 1 << 22),
    (3, 700, 8190, 8192),       # outer length 1 has no passes of real rows
])
def test_the_last_row_of_an_odd_batch(dtype, B, H, N, M):
    g = torch.Generator().manual_seed(B * H)
    u = torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype])
    k = torch.randn(H, 300, generator=g) * 0.1
    plan = fftconv.Plan(N, M, H, dtype, path="multipass")
    y = plan.forward(u.cuda(), plan.filter_fft(k.cuda())).cpu().double()
    L = M if N + 299 > M else 2 * N             # the circular length, or one that no output reaches around
    ref = torch.fft.irfft(torch.fft.rfft(u.double(), L) * torch.fft.rfft(k.double(), L), L)[..., :N]
    assert parity_error(y.numpy(), ref.numpy(), TOL[dtype], "odd batch") <= TOL[dtype]


@pytest.mark.parametrize("dtype,B,H,N,M,gated", [
    ("bf16", 3, 33000, 101, 8192, False), ("f16", 3, 40000, 104, 8192, True),
    ("bf16", 3, 40000, 101, 16384, False), ("f16", 5, 30000, 104, 16384, True),
    ("bf16", 511, 256, 101, 32768, False), ("f16", 511, 256, 101, 32768, True),
    ("bf16", 4095, 32, 101, 65536, False),
])
def test_odd_batches_of_many_rows(dtype, B, H, N, M, gated):
    """The pairs and the lone rows fit into a launch's 65535 rows each, all pairs of the odd batch (65536 to 90000) do not."""
    assert B // 2 * H <= 65535 < (B + 1) // 2 * H
    g = torch.Generator().manual_seed(H)
    u = torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype])
    k = torch.randn(H, N, generator=g) / N ** 0.5
    plan = fftconv.Plan(N, M, H, dtype, path="multipass")
    kf, out = plan.filter_fft(k.cuda()), torch.full_like(u, float("nan"), device="cuda")
    x = u.double()
    if gated:
        w = torch.randn(B, H, N, generator=g).to(u.dtype)
        y, x = plan.forward_gated(u.cuda(), w.cuda(), None, kf, out=out), x * w.double()
    else:
        y = plan.forward(u.cuda(), kf, out=out)
    ref = conv(x, k.double(), 256, N).numpy()               # (no output reaches around 256 samples, either)
    assert parity_error(y.cpu().double().numpy(), ref, TOL[dtype], "y") <= TOL[dtype]
    if not gated:                                           # the gradient of u: the same passes on the conjugate spectrum
        du = plan.backward_input(u.cuda(), plan.filter_fft_adjoint(k.cuda()), out=out.fill_(float("nan")))
        ref = conv(x.flip(-1), k.double(), 256, N).flip(-1).numpy()
        assert parity_error(du.cpu().double().numpy(), ref, TOL[dtype], "du") <= TOL[dtype]
