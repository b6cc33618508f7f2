"""16-bit causal rows of lengths that are no multiple of 8, of transforms that run in a single kernel: rows that begin anywhere in
memory, the chunk across a row's end, batches with and without a partner for the last row; nothing is read or written beyond."""
import pytest
import torch

from paper_2311_05908_amd import fftconv, synth
from parity_util import TOL, parity_error

pytestmark = pytest.mark.gpu


def conv(x, k, N):
    n = 2 * N
    return torch.fft.irfft(torch.fft.rfft(x, n) * torch.fft.rfft(k, n), n)[..., :N]


def placed(t, shift):
    """The tensor on the GPU, its first element `shift` elements behind an allocation's start, NaN before and after it."""
    buf = torch.full((t.numel() + shift + 64,), float("nan"), dtype=t.dtype, device="cuda")
    buf[shift:shift + t.numel()] = t.flatten().cuda()
    return buf, buf[shift:shift + t.numel()].view(t.shape)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M", [16384, 32768])
@pytest.mark.parametrize("B,H,N,shift", [
    (1, 1, 9, 0), (2, 3, 15, 1), (3, 2, 4095, 3), (2, 1, 4100, 2), (5, 9, 5003, 0),
    (1, 2, -1, 5), (4, 1, -7, 0), (3, 300, 1001, 0),               # negative: short of half the transform
])
def test_odd_rows(dtype, M, B, H, N, shift):
    N = M // 2 + N if N < 0 else N
    g = torch.Generator().manual_seed(N + B)
    u, w, v = (torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype]) for _ in range(3))
    k = torch.randn(H, N, generator=g) / N ** 0.5
    plan = fftconv.Plan(N, M, H, dtype)
    assert plan.path == "multipass"
    kf, ka = plan.filter_fft(k.cuda()), plan.filter_fft_adjoint(k.cuda())
    (_, cu), (_, cw), (_, cv) = (placed(t, shift) for t in (u, w, v))
    ubuf, ux = placed(u, shift)
    for name in ("y", "w", "v", "wv", "du"):
        buf, out = placed(torch.zeros_like(u), shift)
        if name == "y":
            plan.forward(cu, kf, out=out)
        elif name == "du":
            plan.backward_input(cu, ka, out=out)
        else:
            plan.forward_gated(cu, cw if "w" in name else None, cv if "v" in name else None, kf, out=out)
        ud, kd = u.double(), k.double()
        if name == "du":
            ref = conv(ud.flip(-1), kd, N).flip(-1)
        else:
            ref = conv(ud * (w.double() if "w" in name else 1.0), kd, N)
        weight = None
        if name in ("v", "wv"):
            ref, weight = ref * v.double(), v.double().abs().numpy()
        assert torch.isnan(buf[:shift]).all() and torch.isnan(buf[shift + u.numel():]).all()
        err = parity_error(out.cpu().double().numpy(), ref.numpy(), TOL[dtype], name, weight=weight)
        print("odd rows %s M=%d B=%d H=%d N=%d %s err=%.3e" % (dtype, M, B, H, N, name, err), flush=True)
        assert err <= TOL[dtype]


@pytest.mark.parametrize("dtype,M,bound", [("bf16", 16384, 4.80e-3), ("bf16", 32768, 4.96e-3), ("f16", 16384, 6.56e-4), ("f16", 32768, 6.79e-4)])
def test_odd_rows_are_no_less_accurate_than_in_three_passes(dtype, M, bound):
    """Error (2-norm, fp64 reference, N(0, 1) rows and decaying filters that nearly fill half the transform) of the three-pass route on such rows; 2^20
    outputs, whose errors' norm scatters by well under 1 %."""
    g = torch.Generator().manual_seed(M)
    B, H, N = 4, 64, M // 2 - 1
    u = torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype])
    alpha = (4.0 / N) * 100.0 ** torch.rand(H, 1, generator=g)
    k = torch.randn(H, N, generator=g) * torch.exp(-alpha * torch.arange(N))
    plan = fftconv.Plan(N, M, H, dtype)
    y = plan.forward(u.cuda(), plan.filter_fft(k.cuda())).cpu().double()
    ref = conv(u.double(), k.double(), N)
    err = ((y - ref).norm() / ref.norm()).item()
    print("odd rows %s M=%d error %.4e bound %.4e" % (dtype, M, err, bound), flush=True)
    assert err <= 1.01 * bound


@pytest.mark.parametrize("M,norm,bound", [
    (16384, 1.0, 8.48e-4), (16384, 0.1, 2.149e-3), (16384, 0.05, 4.052e-3),
    (32768, 1.0, 8.63e-4), (32768, 0.1, 2.155e-3), (32768, 0.05, 4.071e-3),
])
def test_odd_rows_keep_the_bits_of_small_fp16_filters(M, norm, bound):
    """White filters of small norm, whose spectrum over fft_size is subnormal in fp16: the error (2-norm, fp64 reference) of the three-pass route on
    such rows, which keeps k_f at a power of two above that; 2^20 outputs, as above."""
    g = torch.Generator().manual_seed(M)
    B, H, N = 4, 64, M // 2 - 1
    u = torch.randn(B, H, N, generator=g).to(torch.float16)
    k = torch.randn(H, N, generator=g) * (norm / N ** 0.5)
    plan = fftconv.Plan(N, M, H, "f16")
    for kf, ref in ((plan.filter_fft(k.cuda()), conv(u.double(), k.double(), N)),
                    (plan.filter_fft_adjoint(k.cuda()), conv(u.double().flip(-1), k.double(), N).flip(-1))):
        y = plan.forward(u.cuda(), kf).cpu().double()
        err = ((y - ref).norm() / ref.norm()).item()
        print("odd rows f16 M=%d norm %g error %.4e bound %.4e" % (M, norm, err, bound), flush=True)
        assert err <= 1.01 * bound


@pytest.mark.parametrize("B,H", [(5, 30000), (6, 24000)])
def test_odd_rows_of_many_channels(B, H):
    """More pairs of rows than a launch of the three passes takes (90000 and 72000; 65535).  Those took the first shape, an odd batch's lone
    rows and its pairs being launches of their own.  (101 samples a row: the bound is the worst row's error over that row's norm, and of 150000 rows of 9
    samples one in some 10^4 has so small a norm that the roundings of its partial sums, 5e-3 of |u| |k| at any norm, are over it: 1.03e-2.)"""
    M, N = 16384, 101
    g = torch.Generator().manual_seed(H)
    u = torch.randn(B, H, N, generator=g).to(torch.bfloat16)
    k = torch.randn(H, N, generator=g) / N ** 0.5
    plan = fftconv.Plan(N, M, H, "bf16")
    y = plan.forward(u.cuda(), plan.filter_fft(k.cuda()), out=torch.full_like(u, float("nan"), device="cuda")).cpu()
    w = torch.randn(B, H, N, generator=g).to(torch.bfloat16)
    yg = plan.forward_gated(u.cuda(), w.cuda(), None, plan.filter_fft(k.cuda())).cpu()
    assert parity_error(y.double().numpy(), conv(u.double(), k.double(), N).numpy(), TOL["bf16"], "y") <= TOL["bf16"]
    assert parity_error(yg.double().numpy(), conv(u.double() * w.double(), k.double(), N).numpy(), TOL["bf16"], "w") <= TOL["bf16"]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M", [16384, 32768])
def test_odd_rows_with_masks(dtype, M):
    """Block masks and digit patterns of the plan's factorisation on such plans: Re(IDFT(mask K U)) whatever kernel runs them."""
    B, H, N = 3, 2, M // 2 - 5
    g = torch.Generator().manual_seed(M)
    u = torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype])
    k = torch.randn(H, N, generator=g) / N ** 0.5
    plan = fftconv.Plan(N, M, H, dtype)
    U, K = torch.fft.fft(u.double(), M), torch.fft.fft(k.double(), M)
    keep = [1 if j < 4 or j >= 28 else 0 for j in range(32)]
    y = plan.forward_freq_sparse(u.cuda(), plan.filter_fft(k.cuda(), block_keep=keep), keep)
    mask = torch.tensor(keep, dtype=torch.float64).repeat_interleave(M // 32)
    ref = torch.fft.ifft(mask * U * K).real[..., :N]
    assert parity_error(y.cpu().double().numpy(), ref.numpy(), TOL[dtype], "block") <= TOL[dtype]
    digits = [max(1, d // 2) for d in plan.factors]
    y = plan.forward_freq_sparse_digits(u.cuda(), plan.filter_fft_sparse_digits(k.cuda(), digits), digits)
    mask = torch.from_numpy(synth.digit_keep_mask(plan.factors, digits)).double()
    ref = torch.fft.ifft(mask * U * K).real[..., :N]
    assert parity_error(y.cpu().double().numpy(), ref.numpy(), TOL[dtype], "digits") <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M", [16384, 32768])
def test_odd_rows_need_no_workspace(dtype, M):
    """Nothing passes through memory: no workspace but that of a plan's calls of few rows, none missed by any entry point, and the static
    one's size bounds no batch."""
    B, H, N = 1031, 65, 101
    g = torch.Generator().manual_seed(M)
    u = torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype]).cuda()
    plan = fftconv.Plan(N, M, H, dtype)
    assert plan.workspace_bytes(B) == plan.workspace_bytes_gated(B) == 0
    kf = plan.filter_fft((torch.randn(H, N, generator=g) / N ** 0.5).cuda())
    y = plan.forward(u, kf)
    assert torch.equal(plan.forward_static(u, kf, torch.full_like(u, float("nan"))), y)
    keep, digits = [1] * 32, plan.factors
    assert torch.equal(plan.forward_freq_sparse(u, kf, keep), y)
    assert torch.equal(plan.forward_freq_sparse_digits(u, kf, digits), y)
    assert torch.equal(plan.forward_partial(u, kf, 100), y)
    assert torch.equal(plan.forward_gated(u, torch.ones_like(u), None, kf), y)
    for h in (1, 3, 33, 64):
        small = fftconv.Plan(N, M, h, dtype)
        sizes = [small.workspace_bytes(b) for b in range(1, 140)]
        assert sizes == sorted(sizes) and max(sizes) == (64 * M * 4 if M == 32768 else 0)
        assert sizes == [small.workspace_bytes_gated(b) for b in range(1, 140)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M", [16384, 32768])
@pytest.mark.parametrize("B,H,N,shift", [(3, 2, 9, 0), (2, 2, 4095, 1), (1, 2, 5003, 3), (5, 3, 8190, 1), (4, 2, 8188, 2)])
def test_odd_rows_in_three_passes(dtype, M, B, H, N, shift):
    """The family asked for by name runs its own passes on such rows, at both outer lengths; the single kernel is no less accurate.
    (Errors over all outputs; of the shortest rows, where a hundred of them scatter, only the bound.)"""
    g = torch.Generator().manual_seed(N + B + M)
    u, w, v = (torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype]) for _ in range(3))
    k = torch.randn(H, N, generator=g) / N ** 0.5
    (_, cu), (_, cw), (_, cv) = (placed(t, shift) for t in (u, w, v))
    one, three = fftconv.Plan(N, M, H, dtype), fftconv.Plan(N, M, H, dtype, path="multipass")
    assert three.path == one.path and three.factors == one.factors
    assert one.workspace_bytes(B) <= 64 * M * 4 and three.workspace_bytes(B) == (B + 1) // 2 * H * M * 4
    for gated in (False, True):
        ud = u.double() * (w.double() if gated else 1.0)
        ref = conv(ud, k.double(), N) * (v.double() if gated else 1.0)
        errs = []
        for plan in (one, three):
            kf = plan.filter_fft(k.cuda())
            buf, out = placed(torch.zeros_like(u), shift)
            plan.forward_gated(cu, cw if gated else None, cv if gated else None, kf, out=out)
            assert torch.isnan(buf[:shift]).all() and torch.isnan(buf[shift + u.numel():]).all()
            y = out.cpu().double()
            assert parity_error(y.numpy(), ref.numpy(), TOL[dtype], "y", weight=v.double().abs().numpy() if gated else None) <= TOL[dtype]
            errs.append(((y - ref).norm() / ref.norm()).item())
        print("odd rows %s M=%d B=%d H=%d N=%d gated=%d one kernel %.3e three passes %.3e" % (dtype, M, B, H, N, gated, *errs), flush=True)
        assert N < 1000 or errs[0] <= 1.02 * errs[1]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,H,gated", [
    (1, 1, False), (1, 40, False), (1, 41, False), (1, 64, True), (1, 65, True),       # the lines of a single row
    (2, 32, False), (2, 33, False), (64, 1, False), (66, 1, True), (2, 32, True), (8, 4, False), (3, 1, False), (3, 1, True),
])
@pytest.mark.parametrize("N,shift", [(9, 1), (10007, 3), (16382, 1)])
def test_calls_of_few_odd_rows(dtype, B, H, gated, N, shift):
    """On either side of the lines between the single kernel and the three passes, which read the single kernel's k_f: as accurate as the three
    passes on their own, masked filters and their skipped rows included."""
    M = 32768
    g = torch.Generator().manual_seed(N + 7 * B + H)
    u, w, v = (torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype]) for _ in range(3))
    k = torch.randn(H, N, generator=g) / N ** 0.5
    (_, cu), (_, cw), (_, cv) = (placed(t, shift) for t in (u, w, v))
    plan, three = fftconv.Plan(N, M, H, dtype), fftconv.Plan(N, M, H, dtype, path="multipass")
    ud = u.double() * (w.double() if gated else 1.0)
    ref, refd = conv(ud, k.double(), N) * (v.double() if gated else 1.0), conv(ud.flip(-1), k.double(), N).flip(-1)
    weight = v.double().abs().numpy() if gated else None
    errs = []
    for p in (plan, three):
        buf, out = placed(torch.zeros_like(u), shift)
        p.forward_gated(cu, cw if gated else None, cv if gated else None, p.filter_fft(k.cuda()), out=out)
        assert torch.isnan(buf[:shift]).all() and torch.isnan(buf[shift + u.numel():]).all()
        y = out.cpu().double()
        # (rows of 9 samples: the worst of a few hundred, see test_odd_rows_of_many_channels)
        parity_error(y.numpy(), ref.numpy(), TOL[dtype], "y", weight=weight)
        errs.append(((y - ref).norm() / ref.norm()).item())
        assert errs[-1] <= TOL[dtype]
    print("few odd rows %s B=%d H=%d N=%d gated=%d err=%.3e three passes %.3e" % (dtype, B, H, N, gated, *errs), flush=True)
    assert N < 1000 or errs[0] <= 1.02 * errs[1]
    if not gated:
        kf = plan.filter_fft(k.cuda())
        du = plan.backward_input(cu, plan.filter_fft_adjoint(k.cuda())).cpu().double()
        assert ((du - refd).norm() / refd.norm()).item() <= TOL[dtype]
        y = plan.forward(cu, kf)
        assert torch.equal(plan.forward_static(cu, kf, torch.full_like(y, float("nan"))), y)
        U, K = torch.fft.fft(u.double(), M), torch.fft.fft(k.double(), M)
        for digits in ([2, 16, 8, 16], [1, 32, 16, 16], [4, 32, 16, 3]):
            y = plan.forward_freq_sparse_digits(cu, plan.filter_fft_sparse_digits(k.cuda(), digits), digits).cpu().double()
            mask = torch.from_numpy(synth.digit_keep_mask(plan.factors, digits)).double()
            full = torch.fft.ifft(mask * U * K).real
            # a mask spreads a row over all of the transform: errors against its rms there; the norms over all rows, as above
            floor = full.pow(2).mean(-1).sqrt().numpy()
            parity_error(y.numpy(), full[..., :N].numpy(), TOL[dtype], "digits", floor_rms=floor)
            assert ((y - full[..., :N]).norm() / full[..., :N].norm()).item() <= TOL[dtype]
