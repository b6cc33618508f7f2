"""The fp32 row kernels (one kernel per convolution, row_fft.h) at the edges of what they are dispatched for:
every row length, the shortest and longest rows, odd and even sample counts around fft/2 (16-bit rows of even length
move as words, the others element by element; the padded half is skipped up to fft/2), odd batches (a pair without
partner) and row counts that leave a workgroup partly empty."""
import pytest

from paper_2311_05908_amd import synth
from parity_util import TOL, check_all_sequences

pytestmark = pytest.mark.gpu
W = synth.WORKLOADS


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("M", [256, 512, 1024, 2048, 4096])
def test_row_convolution_edges(M, dtype):
    # B = 3: a pair and a lone row; H = 3: six pairs of rows, 2 .. 16 to a workgroup
    for N in (1, 2, 7, M // 2 - 1, M // 2 - 2, M // 2, M // 2 + 1, M // 2 + 2, M - 1, M):
        w = synth.scaled(W["cfg2"], B=3, H=3, N=N, fft_size=M, dtype=dtype, alpha=(1e-2, 1e-1))
        err, plan = check_all_sequences(w, path="small")
        print("rows %s M=%d N=%d err=%.3e" % (dtype, M, N, err), flush=True)
        assert err <= TOL[dtype]


@pytest.mark.parametrize("M", [8192, 16384])
def test_row_convolution_edges_long(M):
    for N in (1, 3, M // 2 - 1, M // 2, M // 2 + 1, M):
        w = synth.scaled(W["cfg2"], B=3, H=2, N=N, fft_size=M, dtype="f32", alpha=(1e-2, 1e-1))
        err, plan = check_all_sequences(w)
        print("rows f32 M=%d N=%d err=%.3e" % (M, N, err), flush=True)
        assert plan.path == "staged"
        assert err <= TOL["f32"]
