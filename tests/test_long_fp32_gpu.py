"""fp32 convolutions of transforms beyond 16384 points at the edges of how their rows share launches: as real rows, formed on load or by an outer pass, or in
pairs, an odd batch's last row, several trips through the workspace and those of the static one.  Rows of up to 8 blocks of 8192 samples form theirs on
load at outer lengths 4 to 16, so that short rows serve for those; pairs of rows take longer ones."""
import pytest
import torch

from paper_2311_05908_amd import fftconv
from parity_util import TOL, parity_error

pytestmark = pytest.mark.gpu


def reference(u, k):
    N = u.shape[-1]
    return torch.fft.irfft(torch.fft.rfft(u.double(), 2 * N) * torch.fft.rfft(k.double(), 2 * N), 2 * N)[..., :N]


def data(B, H, N):
    g = torch.Generator().manual_seed(B * H + N)
    return torch.randn(B, H, N, generator=g), torch.randn(H, N, generator=g) / N ** 0.5


@pytest.mark.parametrize("B,H,N,M", [
    (1, 3, 100, 32768), (7, 73, 60, 32768), (7, 74, 61, 32768),     # formed on load: few rows, a round of the chip and more
    (2, 342, 50, 32768), (171, 3, 50, 32768),
    (5, 3, 1001, 65536), (86, 24, 40, 65536),                       # in one trip and in two
    (1, 2, 333, 131072), (7, 16, 50, 131072), (9, 16, 51, 131072),
    (16, 70, 30, 131072),                                           # in two trips, the second from within a batch row
    (3, 2, 777, 1 << 18), (35, 1, 20, 1 << 22),                     # an outer pass of real rows; pairs where there are no kernels for them
])
def test_rows_of_a_batch(B, H, N, M):
    u, k = data(B, H, N)
    plan = fftconv.Plan(N, M, H, "f32")
    assert plan.path == "staged"
    kf = plan.filter_fft(k.cuda())
    y = plan.forward(u.cuda(), kf, out=torch.full_like(u, float("nan"), device="cuda"))
    err = parity_error(y.cpu().double().numpy(), reference(u, k).numpy(), TOL["f32"], "y")
    print("fp32 rows B=%d H=%d N=%d M=%d err=%.3e" % (B, H, N, M, err), flush=True)
    assert err <= TOL["f32"]


@pytest.mark.parametrize("B,H,N,M", [(40, 32, 30, 131072), (300, 1, 20, 131072), (50, 4, 100, 1 << 20)])
def test_static_workspace_takes_any_batch(B, H, N, M):
    """H * M * 8 bytes fit into the static workspace: smaller trips than fftconv_forward's, the same results."""
    u, k = data(B, H, N)
    plan = fftconv.Plan(N, M, H, "f32")
    kf = plan.filter_fft(k.cuda())
    assert plan.workspace_bytes(B) > fftconv.STATIC_WORKSPACE_BYTES >= H * M * 8
    y = plan.forward_static(u.cuda(), kf, torch.full_like(u, float("nan"), device="cuda"))
    assert torch.equal(y, plan.forward(u.cuda(), kf))


@pytest.mark.parametrize("H,M", [(1, 32768), (40, 32768), (3, 65536), (2, 131072), (5, 1 << 18), (1, 1 << 22)])
def test_workspace_of_a_larger_batch(H, M):
    plan = fftconv.Plan(40, M, H, "f32")
    sizes = [plan.workspace_bytes(B) for B in range(1, 700)]
    assert sizes[0] > 0 and sizes == sorted(sizes)


@pytest.mark.parametrize("B,H,M", [
    (2, 85, 32768), (2, 86, 32768),              # formed on load: blocks in one round of the chip, in two
    (2, 160, 32768), (3, 100, 32768),
    (2, 320, 65536), (2, 321, 65536), (3, 214, 65536),
])
def test_rows_on_either_side_of_the_lines(B, H, M):
    N = 30
    u, k = data(B, H, N)
    plan = fftconv.Plan(N, M, H, "f32")
    y = plan.forward(u.cuda(), plan.filter_fft(k.cuda()), out=torch.full_like(u, float("nan"), device="cuda"))
    assert parity_error(y.cpu().double().numpy(), reference(u, k).numpy(), TOL["f32"], "y") <= TOL["f32"]
    sizes = [plan.workspace_bytes(b) for b in range(1, 40)]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("B,H,N", [
    (3, 8, 65537), (8, 1, 131072), (2, 14, 66000),      # pairs, an odd batch's last row with zeros for a partner; whole rows
    (9, 7, 65600), (9, 13, 65600),                      # the last row with the pairs, or after them, as a real row from an outer pass
    (1, 14, 70001), (2, 15, 70000), (3, 57, 65537),     # one batch row by an outer pass; from 15 channels on on load, without a gate
    (6, 180, 65537), (7, 180, 65537),                   # with a gate: pairs in two trips, the second from within a batch row; a last row after them
])
def test_pairs_of_long_rows(B, H, N, gated):
    """fft 131072, rows of more than 8 blocks, against the same in fp64."""
    M = 131072
    g = torch.Generator(device="cuda").manual_seed(B * H)
    u, w, v = (torch.randn(B, H, N, generator=g, device="cuda") for _ in range(3))
    k = torch.randn(H, N, generator=g, device="cuda") / N ** 0.5
    plan = fftconv.Plan(N, M, H, "f32")
    kf, out = plan.filter_fft(k), torch.full_like(u, float("nan"))
    y = plan.forward_gated(u, w, v, kf, out=out) if gated else plan.forward(u, kf, out=out)
    K = torch.fft.rfft(k.double(), M)
    for b in range(B):
        x = u[b].double() * w[b].double() if gated else u[b].double()
        ref = torch.fft.irfft(torch.fft.rfft(x, M) * K, M)[..., :N] * (v[b].double() if gated else 1)
        err = parity_error(y[b].cpu().double().numpy(), ref.cpu().numpy(), TOL["f32"], "y", v[b].cpu().double().numpy() if gated else None)
        assert err <= TOL["f32"], (b, err)


@pytest.mark.parametrize("B,H,N", [(13, 14, 65537), (8, 14, 131072)])
def test_pairs_of_long_rows_in_the_static_workspace(B, H, N):
    """A pair of batch rows a trip, and a last row; the workspace of the same call holds them at once."""
    g = torch.Generator(device="cuda").manual_seed(B)
    u, k = torch.randn(B, H, N, generator=g, device="cuda"), torch.randn(H, N, generator=g, device="cuda") / N ** 0.5
    plan = fftconv.Plan(N, 131072, H, "f32")
    kf = plan.filter_fft(k)
    assert torch.equal(plan.forward_static(u, kf, torch.full_like(u, float("nan"))), plan.forward(u, kf))
