"""How the streamed-table kernel (fft 16384 and 32768) shares out its pairs of rows: channels dealt to the dies, or all pairs in turn where
that leaves a die short; workgroups of one pair, of several, of unequal numbers."""
import pytest
import torch

from paper_2311_05908_amd import fftconv, synth
from parity_util import TOL, parity_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M", [16384, 32768])
@pytest.mark.parametrize("B,H", [
    (1, 1), (16, 1), (3, 9),                 # a die would have had all pairs
    (33, 17), (2, 300),                      # uneven: three channels on one die, two on the others; more than a round, not two
    (4, 128), (2, 1032),                     # even: one round; several, the last one short
])
def test_every_pair_once(B, H, M, dtype):
    N = 200
    g = torch.Generator().manual_seed(B * H)
    u, w = (torch.randn(B, H, N, generator=g).to(synth.TORCH_DTYPE[dtype]) for _ in range(2))
    k = torch.randn(H, N, generator=g) / N ** 0.5
    plan = fftconv.Plan(N, M, H, dtype)
    assert plan.path == "fused3"
    kf = plan.filter_fft(k.cuda())
    K = torch.fft.rfft(k.double(), 2 * N)
    for gate in (None, w):
        out = torch.full_like(u, float("nan"), device="cuda")
        y = plan.forward_gated(u.cuda(), None if gate is None else gate.cuda(), None, kf, out=out)
        x = u.double() * (1.0 if gate is None else gate.double())
        ref = torch.fft.irfft(torch.fft.rfft(x, 2 * N) * K, 2 * N)[..., :N]
        err = parity_error(y.cpu().double().numpy(), ref.numpy(), TOL[dtype], "y")
        print("split %s M=%d B=%d H=%d gate=%d err=%.3e" % (dtype, M, B, H, gate is not None, err), flush=True)
        assert err <= TOL[dtype]
