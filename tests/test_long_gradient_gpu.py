"""The filter gradient of transforms beyond 16384 points: the ways its batch rows are cut into runs, its channels into trips and its
batch into pieces.  Short rows in long transforms, so that the reference is a short linear correlation in fp64."""
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


@pytest.mark.parametrize("H,M", [(1, 32768), (40, 65536), (3, 1 << 21), (300, 1 << 17)])
def test_workspace_of_a_larger_batch(H, M):
    """A workspace asked for once, for the largest batch, holds every smaller one."""
    plan = fftconv.Plan(40, M, H, "f32")
    sizes = [int(plan._lib.fftconv_workspace_bytes_backward_filter(plan._h, B)) for B in range(1, 60)]
    assert sizes[0] > 0
    assert sizes == sorted(sizes)
