"""The work that users of this library have it do, as a list of cases with their inputs, one pass, its
unavoidable work and the error that its data types allow.

A case is one call, or one training step, on a plan:
  op       forward   y = conv(u, k) with the filter's spectrum k_f at hand (inference, evaluation)
           gated     y = v . ((u . w) * k), the gated form of the Hyena / H3 / M2 layers
           partial   forward with a filter of nk taps, much shorter than the sequence
           sparse    forward with a frequency-sparse filter, a quarter of 32 blocks kept
           train     one step: the filter changed, so filter transform, forward pass, adjoint filter
                     transform, gradient of the input and gradient of the filter
  b, h, n  the (batch, channels, samples) of u;  fft: the transform length (2 n padded up for a causal
           convolution, n for a circular one);  nk: taps of the filter;  dtype: I/O type of u and y.
"""
from __future__ import annotations

import math

import torch

from paper_2311_05908_amd import fftconv

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BLOCKS = 32                      # mask blocks of the frequency-sparse filters; 8 of them, nearest DC, are kept


def _case(op, dtype, b, h, n, fft, nk=None, name=None):
    c = {"op": op, "dtype": dtype, "b": b, "h": h, "n": n, "fft": fft, "nk": n if nk is None else nk}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a handful of short fp32 rows (a unit test, a debugging session, a tiny model)
        _case("forward", "f32", 2, 4, 1024, 2048, name="f32 fft 2048 tiny"),
        # one prompt through one gated layer: batch 1, where the time to the answer counts
        _case("gated", "bf16", 1, 768, 2048, 4096, name="bf16 fft 4096 gated batch 1"),
        # the headline shape: a batch of 4K sequences in a 768-channel layer
        _case("forward", "bf16", 64, 768, 4096, 8192, name="bf16 fft 8192"),
        # short sequences, circular: the paper's main table pads nothing
        _case("forward", "bf16", 64, 768, 1024, 1024, name="bf16 fft 1024 circular"),
        # a gated layer at 16K, fp16
        _case("gated", "f16", 16, 768, 16384, 32768, name="f16 fft 32768 gated"),
        # a filter that covers only the last 1024 samples of an 8K sequence
        _case("partial", "bf16", 32, 768, 8192, 16384, nk=1024, name="bf16 fft 16384 partial"),
        # a low-pass filter: 75 % of the frequency blocks dropped
        _case("sparse", "bf16", 32, 768, 8192, 16384, name="bf16 fft 16384 sparse"),
        # sequences of a length that nobody chose: odd, in an odd batch
        _case("forward", "bf16", 5, 256, 10007, 32768, name="bf16 fft 32768 ragged"),
        # very long sequences (a million samples), the multi-pass range
        _case("forward", "bf16", 1, 64, 1 << 20, 1 << 21, name="bf16 fft 2^21"),
        # training a layer at 4K in bf16
        _case("train", "bf16", 16, 768, 4096, 8192, name="bf16 fft 8192 train"),
        # training in fp32 (a reference run, a small model), a length that is no power of two
        _case("train", "f32", 8, 128, 3000, 8192, name="f32 fft 8192 train"),
        # training on 64K sequences, few rows at a time
        _case("train", "bf16", 2, 256, 65536, 131072, name="bf16 fft 131072 train"),
    ]


def _points(c):
    """Samples of u, weighted by the calls of a pass (a training step makes three passes over u-sized rows) and by
    the width of a sample: what keeps a drawn case no larger than the listed ones."""
    return c["b"] * c["h"] * c["n"] * (4 if c["op"] == "train" else 1) * (3 if c["dtype"] == "f32" else 1)


def draw(rng):
    """One more case of the ranges above: transforms of 256 .. 2^21 points, 2^13 .. 2^26 samples in 16 rows or more, every
    operation."""
    while True:
        op = rng.choice(["forward", "forward", "gated", "partial", "sparse", "train", "train"])
        dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
        lg = rng.randint(8, 21)
        fft = 1 << lg
        shape = rng.random()
        if op in ("partial", "sparse"):
            # the short-filter and low-pass forms are for long sequences with padded, 16-bit rows
            lg = rng.randint(14, 21)
            fft = 1 << lg
            dtype = rng.choice(["bf16", "f16"])
            n = fft // 2
        elif shape < 0.55:
            n = fft // 2                                                 # causal
        elif shape < 0.75:
            n = fft                                                      # circular
        else:
            n = max(1, int(fft // 2 * rng.uniform(0.51, 1.0)))           # any length, odd ones among them
        samples = 2 ** rng.uniform(13, 26)
        if op == "train" or dtype == "f32":
            samples /= 8
        rows = max(16, int(samples / n))
        b = max(1, min(rows, int(2 ** rng.uniform(0, 6.2))))
        h = min(768, rows // b)
        nk = rng.choice([128, 512, 1024, 2048]) if op == "partial" else n
        c = _case(op, dtype, b, h, n, fft, nk)
        if _points(c) <= 1 << 27:
            return c


def prepare(case, seed):
    """The plan, the inputs and, where the filter does not change from call to call, its spectrum."""
    c, dev = case, torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(int(seed))
    b, h, n, nk = c["b"], c["h"], c["n"], c["nk"]
    dtype = DTYPES[c["dtype"]]

    def rows():
        # normalised activations, gates and gradients: N(0, 1) rounded to the I/O type
        return torch.randn(b, h, n, generator=g, device=dev, dtype=torch.float32).to(dtype)

    # trained long filters decay: N(0, 1) exp(-alpha t), alpha per channel such that the filter fades within
    # 1/400 .. 1/4 of the sequence
    alpha = (4.0 / n) * 100.0 ** torch.rand(h, 1, generator=g, device=dev, dtype=torch.float32)
    t = torch.arange(nk, device=dev, dtype=torch.float32)
    k = torch.randn(h, nk, generator=g, device=dev, dtype=torch.float32) * torch.exp(-alpha * t)
    s = {"op": c["op"], "plan": fftconv.Plan(n, c["fft"], h, dtype), "k": k, "nk": nk, "u": rows()}
    if c["op"] == "gated":
        s["w"], s["v"] = rows(), rows()
    elif c["op"] == "train":
        s["dy"] = rows()
    if c["op"] == "sparse":
        half = BLOCKS // 8
        s["keep"] = [1 if j < half or j >= BLOCKS - half else 0 for j in range(BLOCKS)]
        s["kf"] = s["plan"].filter_fft(k, block_keep=s["keep"])
    elif c["op"] != "train":
        s["kf"] = s["plan"].filter_fft(k)
    return s


def run(state):
    s = state
    plan, op = s["plan"], s["op"]
    if op == "forward":
        return plan.forward(s["u"], s["kf"])
    if op == "gated":
        return plan.forward_gated(s["u"], s["w"], s["v"], s["kf"])
    if op == "partial":
        return plan.forward_partial(s["u"], s["kf"], s["nk"])
    if op == "sparse":
        return plan.forward_freq_sparse(s["u"], s["kf"], s["keep"])
    y = plan.forward(s["u"], plan.filter_fft(s["k"]))
    du = plan.backward_input(s["dy"], plan.filter_fft_adjoint(s["k"]))
    dk = plan.backward_filter(s["u"], s["dy"], s["nk"])
    return {"y": y, "du": du, "dk": dk}


def work(case):
    """Each input read once and each output written once; the filter counts as its taps where it is an input (train)
    and as its spectrum otherwise (real taps: fft / 2 complex values of the I/O type's width).  Operations: real
    transforms of fft points at 2.5 fft log2 fft each, one per row of an input and output, and the products between."""
    c = case
    size = 4 if c["dtype"] == "f32" else 2
    rows, fft = c["b"] * c["h"], c["fft"]
    tensor = rows * c["n"] * size
    transform = 2.5 * fft * math.log2(fft)
    if c["op"] == "train":
        # u, dy in; y, du out; k in, dk out (fp32).  Transforms: u, dy, y, du of every row, k and dk of every channel
        return {"bytes": 4 * tensor + 2 * c["h"] * c["nk"] * 4,
                "flops": rows * (4 * transform + 3 * 3 * fft) + 2 * c["h"] * transform}
    spectrum = c["h"] * fft * size
    if c["op"] == "sparse":
        spectrum //= 4
    elif c["op"] == "partial":
        spectrum = min(spectrum, c["h"] * c["nk"] * 4)
    tensors = 4 if c["op"] == "gated" else 2
    return {"bytes": tensors * tensor + spectrum, "flops": rows * (2 * transform + 3 * fft)}


def tolerance(case):
    """Against the same convolution in fp64 the outputs measure at most: fp32 5e-7 (2-norm) and 3e-6 (largest), fp16
    9e-4 and 1e-2, bf16 6.4e-3 and 7e-2; the larger values are those of 2^18-point transforms and of gated calls."""
    return {"f32": {"rel": 2e-6, "max": 1.2e-5}, "f16": {"rel": 2e-3, "max": 0.04},
            "bf16": {"rel": 1.2e-2, "max": 0.25}}[case["dtype"]]
