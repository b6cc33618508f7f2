"""Gated convolution y = v . ((u . w) * k) through the C ABI against the CPU oracle:
the fused-gate 8192-point kernel, the row engine and the outer passes."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2311_05908_amd import fftconv, synth
from parity_util import TOL, batches, parity_error

pytestmark = pytest.mark.gpu
W = synth.WORKLOADS


def run_gated(w, use_w=True, use_v=True):
    u = synth.gen_u(w)
    gw = synth.gen_gate(w, "w") if use_w else None
    gv = synth.gen_gate(w, "v") if use_v else None
    k = synth.gen_k(w)
    plan = fftconv.Plan(w.N, w.fft_size, w.H, w.dtype)
    kf = plan.filter_fft(torch.from_numpy(k).cuda())
    y = plan.forward_gated(u.cuda(), None if gw is None else gw.cuda(), None if gv is None else gv.cuda(), kf)
    torch.cuda.synchronize()
    assert torch.isfinite(y.float()).all()
    return u, gw, gv, k, y.cpu(), plan, kf


def check_all(w, use_w=True, use_v=True):
    u, gw, gv, k, y, plan, kf = run_gated(w, use_w, use_v)
    v = None if gv is None else gv.double().numpy()
    ref = oracle.fftconv_gated(u.double().numpy(), None if gw is None else gw.double().numpy(), v, k, w.fft_size)
    err = parity_error(y.double().numpy(), ref, TOL[w.dtype], "gated", v)
    for rows in batches(plan, w.B)[1:]:
        y = plan.forward_gated(*[None if t is None else t[rows].cuda() for t in (u, gw, gv)], kf).cpu()
        err = max(err, parity_error(y.double().numpy(), ref[rows], TOL[w.dtype], "gated B=%d" % len(rows), None if v is None else v[rows]))
    return err, plan


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,H,N,use_w,use_v", [
    (2, 1, 4096, True, True),
    (3, 5, 4096, True, True),       # odd batch
    (8, 3, 4096, True, False),      # input gate only
    (8, 3, 4096, False, True),      # output gate only
    (2, 2, 1000, True, True),       # ragged N
    (1, 2, 2048, True, True),       # B = 1, N < fft/2
])
def test_gated_fused_fft8192(dtype, B, H, N, use_w, use_v):
    _gated_fused(dtype, B, H, N, 8192, use_w, use_v)


@pytest.mark.parametrize("dtype,B,H,N,M,use_w,use_v", [
    ("bf16", 5, 2, 2048, 4096, True, True),     # short transforms grouped on the 8192-point kernel: gates fused too
    ("f16", 16, 1, 1024, 2048, True, False),
    ("bf16", 9, 3, 200, 512, False, True),
])
def test_gated_fused_short_transforms(dtype, B, H, N, M, use_w, use_v):
    _gated_fused(dtype, B, H, N, M, use_w, use_v)


def _gated_fused(dtype, B, H, N, M, use_w, use_v):
    w = synth.scaled(W["cfg2"], B=B, H=H, N=N, fft_size=M, dtype=dtype)
    err, plan = check_all(w, use_w, use_v)
    print("gated fused %d %s B=%d H=%d N=%d w=%d v=%d path=%s err=%.3e" % (M, dtype, B, H, N, use_w, use_v, plan.path, err),
          flush=True)
    assert plan.path == "fused3" and plan.workspace_bytes_gated(B) == 0
    assert err <= TOL[dtype]


@pytest.mark.parametrize("dtype,B,H,N,M", [
    ("f32", 2, 3, 256, 512),        # short-transform kernel
    ("f32", 3, 2, 300, 1024),
    ("bf16", 2, 2, 204, 512),       # 16-bit I/O with N not a multiple of 8 stays on that kernel
    ("f32", 2, 2, 4096, 8192),      # staged path
])
def test_gated_other_plans(dtype, B, H, N, M):
    w = synth.scaled(W["cfg1"], B=B, H=H, N=N, fft_size=M, dtype=dtype, alpha=(1e-3, 1e-2))
    for use_w, use_v in ((True, True), (True, False), (False, True)):
        err, plan = check_all(w, use_w, use_v)
        print("gated %s B=%d H=%d N=%d M=%d w=%d v=%d path=%s err=%.3e" % (dtype, B, H, N, M, use_w, use_v, plan.path, err),
              flush=True)
        assert plan.workspace_bytes_gated(B) >= plan.workspace_bytes(B) + B * H * N * (4 if dtype == "f32" else 2)
        assert err <= TOL[dtype]


@pytest.mark.parametrize("dtype,B,H,N,M,shift", [
    ("bf16", 5, 3, 256, 256, 0),        # circular rows, words of two samples; odd batch
    ("bf16", 4, 3, 256, 256, 1),        # ... gates that start off a word
    ("f16", 3, 5, 255, 256, 0),         # odd rows: sample by sample
    ("bf16", 3, 2, 510, 512, 0),        # words, the last registers partly filled
    ("f16", 2, 9, 1024, 1024, 0),
    ("bf16", 3, 2, 1001, 2048, 0),
    ("f16", 1, 2, 2047, 2048, 0),       # N > M / 2, a row without a partner
    ("bf16", 2, 2, 4096, 4096, 0),
    ("f32", 3, 2, 130, 256, 0),
    ("f32", 2, 3, 4096, 4096, 0),
    ("f32", 3, 1, 8192, 8192, 0),
    ("f32", 3, 1, 5001, 16384, 0),
    ("f32", 1, 2, 16384, 16384, 0),
    ("f32", 3, 2, 9001, 32768, 0),      # rows of the outer factor formed on load: odd N, then N > M / 2
    ("f32", 2, 1, 20002, 32768, 0),
    ("f32", 2, 1, 9002, 65536, 1),      # ... gates that start off a pair of samples
    ("f32", 2, 1, 40002, 65536, 1),     # outer passes of real rows, of whose gates the same holds
    ("f32", 3, 1, 65538, 131072, 1),    # pairs of rows, the last one with zeros
    ("f32", 5, 1, 9001, 131072, 0),     # rows of the outer factor formed on load
    ("f32", 1, 2, 9002, 524288, 0),     # outer passes with a tile
])
def test_gates_on_the_row_engine(dtype, B, H, N, M, shift):
    w = synth.scaled(W["cfg1"], B=B, H=H, N=N, fft_size=M, dtype=dtype, alpha=(1e-3, 1e-2))
    u, gw, gv, k = synth.gen_u(w), synth.gen_gate(w, "w"), synth.gen_gate(w, "v"), synth.gen_k(w)
    plan = fftconv.Plan(N, M, H, dtype)
    kf = plan.filter_fft(torch.from_numpy(k).cuda())

    def placed(t):                      # `shift` elements behind an aligned address
        room = torch.empty(t.numel() + shift, dtype=t.dtype, device="cuda")
        room[shift:].copy_(t.flatten())
        return room[shift:].view(t.shape)

    for use_w, use_v in ((True, True), (True, False), (False, True)):
        y = plan.forward_gated(u.cuda(), placed(gw) if use_w else None, placed(gv) if use_v else None, kf).cpu()
        v = gv.double().numpy() if use_v else None
        ref = oracle.fftconv_gated(u.double().numpy(), gw.double().numpy() if use_w else None, v, k, M)
        assert parity_error(y.double().numpy(), ref, TOL[dtype], "gates %d%d" % (use_w, use_v), v) <= TOL[dtype]


@pytest.mark.parametrize("B,H,N,M", [
    (2, 1024, 16384, 32768), (2, 512, 65534, 65536), (2, 256, 131072, 131072),        # outer passes of pairs of fp32 rows
])
def test_an_output_gate_costs_no_more_than_a_kernel_of_its_own(B, H, N, M):
    """A gate inside the last kernel reads v; one of its own reads y and writes it again, a third of such a call (0.78 of the time with
    it at 2 x 256 x 131072, 1.15 when the kernel waited for its gates one after another)."""
    u, v = (torch.randn(B, H, N, device="cuda") for _ in range(2))
    plan = fftconv.Plan(N, M, H, "f32")
    kf = plan.filter_fft(torch.randn(H, N, device="cuda") / N ** 0.5)
    y, z = torch.empty_like(u), torch.empty_like(u)

    def apart():
        torch.mul(plan.forward(u, kf, out=y), v, out=z)

    def fused():
        plan.forward_gated(u, None, v, kf, out=y)

    def time(call):
        best = float("inf")
        for _ in range(10):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            call()
            t[1].record()
            t[1].synchronize()
            best = min(best, t[0].elapsed_time(t[1]))
        return best

    two, one = time(apart), time(fused)
    print("output gate %d x %d x %d: %.3f ms, of its own %.3f ms" % (B, H, N, one, two), flush=True)
    assert torch.equal(y, z)                # the same roundings, too
    assert one <= two


def test_gated_without_gates_is_forward_and_errors():
    w = synth.scaled(W["cfg2"], B=2, H=2)
    u = synth.gen_u(w).cuda()
    k = synth.gen_k(w)
    plan = fftconv.Plan(w.N, w.fft_size, w.H, w.dtype)
    kf = plan.filter_fft(torch.from_numpy(k).cuda())
    assert torch.equal(plan.forward_gated(u, None, None, kf), plan.forward(u, kf))
    y = torch.empty_like(u)
    lib = fftconv.load()
    rc = lib.fftconv_forward_gated(plan._h, u.data_ptr(), u.data_ptr(), y.data_ptr(), kf.data_ptr(), y.data_ptr(),
                                   2, 2, w.N, None, None)
    assert rc == -1                                     # v aliases y
    # a plan that needs workspace for the gated input refuses a NULL workspace
    w2 = synth.scaled(W["cfg1"], B=2, H=2, N=256, fft_size=512, dtype="f32")
    p2 = fftconv.Plan(w2.N, w2.fft_size, w2.H, w2.dtype)
    u2 = synth.gen_u(w2).cuda()
    kf2 = p2.filter_fft(torch.from_numpy(synth.gen_k(w2)).cuda())
    y2 = torch.empty_like(u2)
    rc = lib.fftconv_forward_gated(p2._h, u2.data_ptr(), u2.data_ptr(), None, kf2.data_ptr(), y2.data_ptr(),
                                   2, 2, w2.N, None, None)
    assert rc == -1


def test_gated_cfg2_full_size_sampled_sequences():
    w = W["cfg2"]
    u, gw, gv, k, y, plan, _ = run_gated(w)
    assert plan.path == "fused3"
    kext = oracle.extend_filter(k, w.fft_size)
    worst = 0.0
    for b, h in synth.sample_sequences(w, 28):
        ref = oracle.fftconv_gated(u[b, h].double().numpy()[None, None], gw[b, h].double().numpy()[None, None],
                                   gv[b, h].double().numpy()[None, None], kext[h][None])[0, 0]
        worst = max(worst, parity_error(y[b, h].double().numpy(), ref, TOL[w.dtype], "gated cfg2 b=%d h=%d" % (b, h),
                                             gv[b, h].double().numpy()))
    print("gated cfg2 full: worst sampled rel L2 = %.3e" % worst, flush=True)
    assert worst <= TOL[w.dtype]


@pytest.mark.parametrize("dtype,B,H,N,M", [
    ("bf16", 3, 2, 8192, 16384),    # fused 16384 kernel, odd batch
    ("f16", 4, 3, 8192, 16384),
    ("bf16", 2, 2, 4000, 16384),    # ragged N
    ("f16", 2, 2, 16384, 32768),    # fused 32768 kernel
    ("bf16", 3, 1, 16384, 32768),
    ("f16", 2, 1, 10000, 32768),
])
def test_gated_fused_16384_32768(dtype, B, H, N, M):
    w = synth.scaled(W["cfg1"], B=B, H=H, N=N, fft_size=M, dtype=dtype, alpha=(1e-3, 1e-2))
    for use_w, use_v in ((True, True), (True, False), (False, True)):
        err, plan = check_all(w, use_w, use_v)
        print("gated fused %d %s B=%d H=%d N=%d w=%d v=%d path=%s err=%.3e" % (M, dtype, B, H, N, use_w, use_v, plan.path, err),
              flush=True)
        assert plan.path == "fused3" and plan.workspace_bytes_gated(B) == 0
        assert err <= TOL[dtype]


@pytest.mark.parametrize("dtype,B,H,N,M", [
    ("bf16", 2, 1, 32768, 65536),   # gates fused into the outer passes of the multi-pass route
    ("f16", 3, 2, 20000, 65536),    # odd batch, ragged N (2-byte accesses)
    ("bf16", 2, 2, 8192, 8192),     # circular, no outer transform
    ("f16", 1, 1, 12002, 16384),    # N > fft/2, N not a multiple of 4
    ("bf16", 9, 256, 1321, 8192),   # many rows: blocks of the outer passes make 8, 4 and 2 trips
    ("f16", 8, 128, 3001, 16384),
    ("bf16", 7, 86, 9999, 32768),
])
def test_gated_multipass(dtype, B, H, N, M):
    w = synth.scaled(W["cfg1"], B=B, H=H, N=N, fft_size=M, dtype=dtype, alpha=(1e-3, 1e-2))
    for use_w, use_v in ((True, True), (True, False), (False, True)):
        err, plan = check_all(w, use_w, use_v)
        print("gated multipass %s B=%d H=%d N=%d M=%d w=%d v=%d path=%s err=%.3e" % (dtype, B, H, N, M, use_w, use_v, plan.path, err),
              flush=True)
        assert plan.path == "multipass"
        assert plan.workspace_bytes_gated(B) == plan.workspace_bytes(B)
        assert err <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_a_non_finite_gate_value_stays_in_its_own_element(dtype):
    """An infinity in the output gate, and a NaN in the input gate of ANOTHER sequence, reach exactly the elements
    they belong to: y is non-finite at the position of the infinite gate value and nowhere else in that sequence,
    every output of the sequence with the NaN input is NaN (it enters the transform), all other sequences are
    untouched."""
    w = synth.scaled(W["cfg2"], B=4, H=2, dtype=dtype)
    u, gw, gv = synth.gen_u(w), synth.gen_gate(w, "w"), synth.gen_gate(w, "v")
    gv[1, 0, 1001] = float("inf")
    gw[2, 1, 7] = float("nan")
    plan = fftconv.Plan(w.N, w.fft_size, w.H, w.dtype)
    kf = plan.filter_fft(torch.from_numpy(synth.gen_k(w)).cuda())
    y = plan.forward_gated(u.cuda(), gw.cuda(), gv.cuda(), kf).cpu().float()
    bad = ~torch.isfinite(y)
    assert bad[1, 0, 1001] and int(bad[1, 0].sum()) == 1
    # rows b = 2 and b = 3 share one complex transform: the NaN spreads over that pair of channel 1 and nowhere else
    assert bool(bad[2, 1].all())
    bad[2:4, 1] = False
    bad[1, 0, 1001] = False
    assert not bool(bad.any())
