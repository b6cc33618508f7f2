// Filter gradient with fp32 arithmetic of rows that fit on chip, fft_size M in {256 .. 16384}, any I/O dtype, any
// N <= M (paper Section 3.1 "Kernel Fusion and Recomputation"):
//     dk_f[h] = sum_b conj(FFT(pad(u[b,h]))) . FFT(pad(dy[b,h])),      dk[h] = Re(iFFT(dk_f[h]))[0:Nk].
// Serves the plans without a matrix-core gradient kernel (fp32 I/O, circular and ragged shapes).
//
//  * The transforms are those of row_fft.h with exact twiddles, one of every row of u and of dy with zeros for an imaginary
//    part.  (Two rows in one complex transform, as in the convolution, would halve them; but dk is a real result of real
//    sequences, and half of the rounding errors of a real row's spectrum go with the imaginary part in the end: sharing
//    transforms costs a fifth in accuracy.)
//  * A row of threads owns a run of a channel's batch rows and adds their products up in registers.  A channel is cut into S
//    runs where channels alone would leave compute units idle (grad_splits); their sums meet in a second kernel, in a fixed
//    order, which also transforms back.  With S = 1 the first kernel does that itself and no sum leaves the registers.
//  * The sums go through memory in register order, [run][h][register pair][thread][2], as 16-byte accesses.
//  * Of the first pass' butterflies, on real samples, the half that is not a mirror image (dft_real(); the same bits).  us: fp32 8 x 256 x 4096 67.8 -> 63.4,
//    8 x 128 x 3000 43.9 -> 41.4, 4 x 128 x 8192 54.0 -> 52.4; bf16 8 x 4096 x 512 circular 48.5 -> 47.1; not at 256 points (64 x 768 x 128 31.3, 31.7) and not
//    at 4096, where it gains 1 to 3 % with many rows in fp32 but a launch of one to two rows to a compute unit loses (bf16 1 x 300 x 4095 11.4 -> 13.0, x 2047
//    10.6 -> 11.5, fp32 10.5 -> 10.7).
// Bound by the vector ALU and, at two waves per SIMD (the accumulator, a spectrum of u and the transform under way take
// 192 registers), by the latency of the exchanges between passes.  It replaces one
// kernel for every factor of either transform, batch row by batch row, with the row in memory between them.  A training step
// (filter transforms, forward pass, both gradients), us: fp32 8 x 128 x 3000 fft 8192 750 -> 124; bf16 circular
// 16 x 256 x 1024 699 -> 86, 8 x 256 x 8192 1005 -> 229; bf16 8 x 256 x 777 fft 2048 490 -> 78.  Few rows since (fp32 8 x 2 x 1024, fft 1024): 51 -> 38.
#include "fftconv_internal.h"
#include "row_io.h"

namespace fftconv {

namespace {

// Rows of the gradient.  Of 1024 points: radix-32 butterflies as 4 x 8 (FINE), as both passes are of radix 32 there and dk came out
// at 2.05e-7 of error (fp32, 4 x 64 rows of 512 samples), where a kernel for every factor had 1.97e-7; now 1.78e-7.
// (WIDE, with the radix-16 ones as 4 x 4: 1.73e-7.)  Same time: 64 x 768 rows of 512, 125 -> 117 us, of 1024, 158 - 161 -> 171, 16 x 256 37 -> 37.  Dividing 16 x 16 x 4 instead, 1.80e-7, costs
// a trip through LDS: 154, 177, 30.
template <int M, bool WIDE = false> using GradRow = rf::Row<M, true, M == 1024, WIDE>;

// waves per SIMD that the registers allow: 192 data registers with 32 points a thread (12 - 60 bytes spilled where N > M / 2, and at
// 1024 points), half of that with 16
template <int M, bool WIDE = false> constexpr int GRAD_WAVES = GradRow<M, WIDE>::P == 32 ? 2 : 3;

template <typename G>
__device__ __forceinline__ void store_dk(const float2 (&x)[G::P], float *__restrict__ dk, int64_t Nk, float scale, int tid)
{
#pragma unroll
    for (int m = 0; m < G::P; ++m) {
        const int n = tid + G::T * m;
        if (n < Nk) dk[n] = x[m].x * scale;
    }
}

// HALF: N <= M / 2.  Row t = h * S + s of threads: batch rows [s * per, (s + 1) * per) of channel h.
template <int M, typename IO, bool HALF, bool WIDE>
__global__ void __launch_bounds__(rf::threads_of(M), (GRAD_WAVES<M, WIDE>))
    k_row_corr(const IO *__restrict__ u, const IO *__restrict__ dy, float4 *__restrict__ part, float *__restrict__ dk,
               const float2 *__restrict__ tab, int B, int H, int N, int64_t Nk, int S, int per)
{
    using G = GradRow<M, WIDE>;
    constexpr int RW = rf::threads_of(M) / G::T;
    extern __shared__ float2 smem_rows[];
    const int row = threadIdx.x / G::T, tid = threadIdx.x % G::T, rows = H * S;
    const int t = min((int)blockIdx.x * RW + row, rows - 1);      // rows beyond the last one repeat it, unstored
    const bool live = (int)blockIdx.x * RW + row < rows;
    const int h = t / S, s = t - h * S;
    float2 *const Z = (float2 *)((char *)smem_rows + row * G::LDS_BYTES);
    const bool exact = N == (HALF ? G::R0 / 2 : G::R0) * G::T;
    const bool words = rf::word_rows<IO>(u, dy, N);

    float2 acc[G::P], zu[G::P];
#pragma unroll
    for (int p = 0; p < G::P; ++p) acc[p] = make_float2(0.f, 0.f);
    // one transform a step: a u row, then the dy row; the same count in every row of threads (shared barriers)
    float next[G::P];                                             // the dy row, fetched with the u row
#pragma unroll 1
    for (int i = 0; i < 2 * per; ++i) {
        const int b = s * per + i / 2;
        int j = tid;
        asm volatile("" : "+v"(j));                               // addresses, masks and twiddles of a step are not kept for the next
        float2 x[G::P];
        if (i & 1) {
#pragma unroll
            for (int m = 0; m < G::P; ++m) x[m] = make_float2(next[m], 0.f);
        } else {
            const int64_t at = ((int64_t)min(b, B - 1) * H + h) * N;          // past the channel's end: the last row, as zeros
            rf::load_pair<G, IO, HALF>(x, u + at, dy + at, N, j, exact, words, b < B, b < B);
#pragma unroll
            for (int m = 0; m < (HALF ? G::P / 2 : G::P); ++m) {
                next[m] = x[m].y;
                x[m].y = 0.f;
            }
        }
        rf::Tw1<G> tw1;
        tw1.load(tab, j);
        rf::row_barrier<G::T>();                                  // the slots are free
        rf::forward<G, HALF, M != 256 && M != 4096>(x, Z, tab, tw1, j, [] {});
        if (i & 1) {
#pragma unroll
            for (int p = 0; p < G::P; ++p) {                      // acc += conj(Z_u) Z_dy
                acc[p].x = __builtin_fmaf(zu[p].y, x[p].y, __builtin_fmaf(zu[p].x, x[p].x, acc[p].x));
                acc[p].y = __builtin_fmaf(-zu[p].y, x[p].x, __builtin_fmaf(zu[p].x, x[p].y, acc[p].y));
            }
        } else {
#pragma unroll
            for (int p = 0; p < G::P; ++p) zu[p] = x[p];
        }
    }
    if (S == 1) {
        rf::Tw1<G> tw1;
        tw1.load(tab, tid);
        rf::inverse<G>(acc, Z, tab, tw1, tid);
        if (live) store_dk<G>(acc, dk + (int64_t)h * Nk, Nk, 1.f / M, tid);
        return;
    }
    if (!live) return;
    float4 *const o = part + ((int64_t)s * H + h) * (M / 2) + tid;
#pragma unroll
    for (int q = 0; q < G::P / 2; ++q) o[q * G::T] = make_float4(acc[2 * q].x, acc[2 * q].y, acc[2 * q + 1].x, acc[2 * q + 1].y);
}

// dk[h] from the S sums of channel h
template <int M, bool WIDE>
__global__ void __launch_bounds__(rf::threads_of(M), (GRAD_WAVES<M, WIDE>))
    k_row_dk(const float4 *__restrict__ part, float *__restrict__ dk, const float2 *__restrict__ tab, int H, int64_t Nk, int S)
{
    using G = GradRow<M, WIDE>;
    constexpr int RW = rf::threads_of(M) / G::T;
    extern __shared__ float2 smem_rows[];
    const int row = threadIdx.x / G::T, tid = threadIdx.x % G::T;
    const int h = min((int)blockIdx.x * RW + row, H - 1);
    const bool live = (int)blockIdx.x * RW + row < H;
    float2 *const Z = (float2 *)((char *)smem_rows + row * G::LDS_BYTES);
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    float2 x[G::P];
    const float4 *in = part + (int64_t)h * (M / 2) + tid;
#pragma unroll
    for (int q = 0; q < G::P / 2; ++q) {
        const float4 v = in[q * G::T];
        x[2 * q] = make_float2(v.x, v.y);
        x[2 * q + 1] = make_float2(v.z, v.w);
    }
    for (int s = 1; s < S; ++s) {
        in += (int64_t)H * (M / 2);
        float4 v[G::P / 2];
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) v[q] = in[q * G::T];
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) {
            x[2 * q].x += v[q].x;
            x[2 * q].y += v[q].y;
            x[2 * q + 1].x += v[q].z;
            x[2 * q + 1].y += v[q].w;
        }
    }
    rf::inverse<G>(x, Z, tab, tw1, tid);
    if (live) store_dk<G>(x, dk + (int64_t)h * Nk, Nk, 1.f / M, tid);
}

// The sums of gradients' runs, two bins to a thread, n threads in all: part[r * apart + i] over r < runs, and acc[i] where there is one, to
// out[i] (in place, too).  Every compute unit takes part, where the kernels that transform them back have a workgroup to a channel or block and
// wait for a run after the other.  Eight runs are fetched at a time and added up in pairs: one after the other, more runs meant more error (dk of
// bf16 64 x 1 x 32768 in 64 runs 3.99e-7, in pairs 3.79e-7; in 32 runs, in order, 3.87e-7).
// rows: 0, or the workgroups to a spectrum, where one workgroup put out each run of it and the spectra are a multiple of 8.  Workgroup b then takes
// part of a spectrum whose number has b's remainder by 8: its runs are in that die's L2 (dk of fp32 4 x 16 x 16384 41.5 -> 37.7 us, 8 x 16 52.3 -> 47.3).
__global__ void __launch_bounds__(256) k_runs_add(const float4 *part, int64_t apart, int runs, const float4 *acc, float4 *out, int64_t n, int rows)
{
    const int b = blockIdx.x, at = rows ? (b / (8 * rows) * 8 + b % 8) * rows + b / 8 % rows : b;
    const int64_t i = (int64_t)at * 256 + threadIdx.x;
    if (i >= n) return;
    float4 x = acc ? acc[i] : part[i];
    constexpr int AT_ONCE = 8;
    for (int r = acc ? 0 : 1; r < runs; r += AT_ONCE) {
        float4 v[AT_ONCE];
#pragma unroll
        for (int j = 0; j < AT_ONCE; ++j) v[j] = part[min(r + j, runs - 1) * apart + i];
#pragma unroll
        for (int j = 0; j < AT_ONCE; ++j)
            if (r + j >= runs) v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int half = AT_ONCE / 2; half > 0; half /= 2)
#pragma unroll
            for (int j = 0; j < half; ++j) {
                v[j].x += v[j + half].x;
                v[j].y += v[j + half].y;
                v[j].z += v[j + half].z;
                v[j].w += v[j + half].w;
            }
        x.x += v[0].x;
        x.y += v[0].y;
        x.z += v[0].z;
        x.w += v[0].w;
    }
    out[i] = x;
}

// From how many runs on that kernel adds them up, and the most pairs of bins that it does so with.  A run costs k_row_dk 0.2 us at 256 points, 0.3 at 512, 0.35 to 4096,
// 0.75 at 8192, 1.5 at 16384; this kernel 3.5 us and little more (fp32, us: fft 512 16 x 1 rows 10.6, 14.2, 45 x 1 18.2, 14.1; 1024 16 x 1 14.2, 14.2, 45 x 1
// 24.5, 16.1; 4096 45 x 1 30.9, 18.7; 8192 8 x 16 28.4, 26.6, 4 x 100 33.1, 35.9; 256 40 x 100 25.1, 17.2), unless it waits for memory: 1024, 16 x 256 27.9, 29.5;
// four runs, which save least, from half of that on: 16384, 4 x 16 39.0 both, 4 x 32 40.3, 43.0.
template <int M> constexpr int64_t ADD_RUNS = M == 256 ? 21 : M == 512 ? 17 : M <= 4096 ? 13 : M == 8192 ? 7 : 4;
constexpr int64_t ADD_MOST = (int64_t)1 << 20;

// Runs per channel: as many as give every SIMD of 256 compute units two waves (16 points a thread: four), no more than
// the batch has rows, of equal length.  At 512 points, where adding up the runs of a few batch rows took longer than their transforms, up to 16 rows and 512
// channels: a wave to a SIMD, two beyond 256 channels, where few rows of threads would wait for one another's ends.  us, all runs, so: bf16 16 x 128 14.9, 11.8, 12 x 256
// 16.9, 12.5, 16 x 256 20.9, 14.3, 16 x 512 25.4, 19.1; fp32 16 x 256 20.7, 14.6; errors 1 to 3 % less.  (16 x 384 with a wave to a SIMD 20.4, with two 17.2.)
// most: the runs that no smaller batch exceeds (4 rows in runs of 1 are more than 5 in runs of 2): what the workspace holds.
struct Splits { int64_t S, per, most; };
Splits grad_splits(int64_t M, int64_t H, int64_t B)
{
    int64_t want = 1;
    (void)rf::with_row(M, [&](auto g) -> int {
        using G = GradRow<decltype(g)::M>;
        want = 256 * 4 * GRAD_WAVES<G::M> * 64 / G::T / H;
        return FFTCONV_OK;
    });
    if (const int64_t waves = H <= 256 ? 1024 : 2048; M == 512 && H <= 512 && B <= 16 && want * H > waves) want = waves / H;
    if (want > B) want = B;
    if (want < 1) want = 1;
    const int64_t per = (B + want - 1) / want;
    return Splits{(B + per - 1) / per, per, want};
}

template <int M, typename IO, bool HALF, bool WIDE>
int launch(const fftconv_plan *p, const void *u, const void *dy, float *dk, int64_t Nk, int64_t B, void *workspace, hipStream_t s)
{
    using G = GradRow<M, WIDE>;
    constexpr int NTHR = rf::threads_of(M), RW = NTHR / G::T, lds = RW * G::LDS_BYTES;
    const Splits sp = grad_splits(M, p->H, B);
    // rows of threads, and the threads of a launch (cut short without an error beyond 2^32), are 32-bit numbers
    if ((p->H * sp.S + RW) * G::T > UINT32_MAX || (sp.S == 1 && B >= ((int64_t)1 << 31))) {
        set_error("fftconv_backward_filter: too many sequences for the row kernel");
        return FFTCONV_EUNSUPPORTED;
    }
    FC_TRY(raise_dynamic_lds((const void *)k_row_corr<M, IO, HALF, WIDE>, lds));
    // so are batch rows: a longer batch goes out in pieces of whole runs, two or more in each
    const int64_t pieces = (sp.S * sp.per + (1 << 30) - 1) >> 30;
    for (int64_t i = 0; i < pieces; ++i) {
        const int64_t s0 = sp.S * i / pieces, ns = sp.S * (i + 1) / pieces - s0, b0 = s0 * sp.per, at = b0 * p->H * p->N;
        const int64_t nb = B - b0 < ns * sp.per ? B - b0 : ns * sp.per;
        hipLaunchKernelGGL((k_row_corr<M, IO, HALF, WIDE>), dim3((unsigned)((p->H * ns + RW - 1) / RW)), dim3(NTHR), lds, s, (const IO *)u + at,
                           (const IO *)dy + at, (float4 *)workspace + s0 * p->H * (M / 2), dk, rf::row_table<G>(p), (int)nb, (int)p->H,
                           (int)p->N, Nk, (int)ns, (int)sp.per);
        FC_HIP(hipGetLastError());
    }
    if (sp.S == 1) return FFTCONV_OK;
    int64_t left = sp.S;
    const int64_t apart = p->H * (M / 2);
    if (sp.S >= ADD_RUNS<M> && sp.S * apart <= (sp.S == 4 ? ADD_MOST / 2 : ADD_MOST)) {
        FC_TRY(runs_add(workspace, apart, sp.S, nullptr, workspace, apart, s));
        left = 1;
    }
    FC_TRY(raise_dynamic_lds((const void *)k_row_dk<M, WIDE>, lds));
    hipLaunchKernelGGL((k_row_dk<M, WIDE>), dim3((unsigned)((p->H + RW - 1) / RW)), dim3(NTHR), lds, s, (const float4 *)workspace, dk,
                       rf::row_table<G>(p), (int)p->H, Nk, (int)left);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

// WIDE rows (row_fft.h).  us, others, wide (and with fewer runs' sums, see above): fp32 fft 512 1 x 16 10.5, 8.0, 16 x 16 22.9, 11.7, 16 x 1024 32.0, 28.1, 64 x 768 68.8, 62.8,
// 2 x 4096 27.2, 26.7; fft 1024 1 x 16 11.0, 7.8, 16 x 16 25.4, 14.4, 32 x 256 39.3, 33.7, 16 x 1024 47.4, 49.5, 64 x 768 109, 123, 2 x 4096 22.8, 25.2.
// At 512 points the others only for many rows, fp32 ones up to M / 2 and 16-bit ones beyond, whose channels fill seven eighths of the rounds of 8192 that
// run at a time (two waves a SIMD): fp32 32 x 4096 x 256 142, 156, 13 x 8192 101.7, 105.7, 16 x 4096 74.7, 73.2, 98 x 2048 x 200 208, 237, but 32 x 5000 251, 192, 8 x 10000 112, 83, 8 x
// 12288 120, 98; bf16 32 x 4096 x 512 164, 178, 12 x 8192 102, 111, 12 x 4096 65.3, 66.1, but 16 x 7000 138, 134, 8 x 5000 69.8, 54.9, 258 x 256 99.7, 95.1; fp16 17 x 8192 x 401 149, 153, 8 x 8192
// 77.8, 76.1, 8 x 5000 74.2, 50.9.  Fewer channels, more of their rows: fp32 391 x 256 x 256 122, 115, 516 x 256 160, 167, fp16 516 x 256 x 401 173, 164, 1024 x 64 x 512 0.80, 4096 x 16 x 512 344, 247.
template <int M, typename IO, bool HALF> bool grad_wide(int64_t H, int64_t B, int64_t N)
{
    if (M == 1024) return H <= 1024 && H * B <= 8192;
    constexpr bool WORD = sizeof(IO) == 2;
    if (HALF == WORD || H <= 128 || H * B < (!WORD ? (H >= 1024 ? 3 << 15 : 1 << 17) : H < 512 ? 3 << 16 : N == M ? 3 << 14 : 1 << 17)) return true;
    const int64_t rows = H * grad_splits(M, H, B).S, at_once = (rows + 8191) / 8192 * 8192;
    return 8 * rows < 7 * at_once;
}

template <int M, typename IO, bool HALF>
int launch_rows(const fftconv_plan *p, const void *u, const void *dy, float *dk, int64_t Nk, int64_t B, void *workspace, hipStream_t s)
{
    if constexpr (rf::has_wide(M))
        if (grad_wide<M, IO, HALF>(p->H, B, p->N)) return launch<M, IO, HALF, true>(p, u, dy, dk, Nk, B, workspace, s);
    return launch<M, IO, HALF, false>(p, u, dy, dk, Nk, B, workspace, s);
}

template <int M, typename IO>
int launch_half(const fftconv_plan *p, const void *u, const void *dy, float *dk, int64_t Nk, int64_t B, void *workspace, hipStream_t s)
{
    return p->N <= M / 2 ? launch_rows<M, IO, true>(p, u, dy, dk, Nk, B, workspace, s)
                         : launch_rows<M, IO, false>(p, u, dy, dk, Nk, B, workspace, s);
}

}  // namespace

int runs_add(const void *part, int64_t apart, int64_t runs, const void *acc, void *out, int64_t pairs, hipStream_t s, int rows)
{
    hipLaunchKernelGGL(k_runs_add, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, s, (const float4 *)part, apart, (int)runs,
                       (const float4 *)acc, (float4 *)out, pairs, pairs % (8 * 256 * (int64_t)(rows ? rows : 1)) == 0 ? rows : 0);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

bool row_backward_filter_ok(const fftconv_plan *p) { return p->path != PATH_FUSED3 && p->M <= 16384; }

// Which gradients of matrix-core plans run on these rows: those of one batch row, where the other kernel sums a single product, and leaves it to a second one
// to transform it back, and of few at short lengths.  us, matrix cores, rows (bf16): 1 x 16 fft 256 11.5, 8.1, 512 13.4, 8.3, 1024 13.5, 8.4, 2048 15.0, 9.3,
// 4096 12.3, 9.4, 8192 14.1, 16.8; 1 x 768 25.8, 8.4, 29.5, 8.5, 28.6, 8.4, 35.5, 11.2, 28.0, 15.4; 2 x 64 11.8, 10.9, 13.6, 11.3, 13.8, 11.2, 16.1, 12.5, 12.5, 13.5;
// 8 x 16 11.5, 10.9, 13.3, 11.2, 13.6, 12.5, 14.9, 14.9; 8 x 64 12.0, 11.2, 13.9, 11.4, 14.1, 13.8; 8 x 256 13.8, 12.0, 15.9, 12.7, 16.1, 20.1; 16 x 16 11.4, 13.3,
// 13.4, 11.6, 13.5, 13.9; fft 512 16 x 96 13.7, 11.2, 16 x 256 16.2, 14.3, 16 x 512 23.6, 19.1, 16 x 768 31.1, 26.9.  The spectra of their runs, a batch row each at most, fit into the workspace for that kernel's 8192 slots a channel.
bool row_backward_filter_few(const fftconv_plan *p, int64_t B)
{
    if (B * p->H > 1 << 20) return false;                         // (far within the limits of a launch)
    switch (p->M) {
    case 256: return B <= 8;
    case 512: return B <= 16;
    case 1024: return B == 1 || (B <= 8 && B * p->H <= 512);
    case 2048: return B <= 4 && (B == 1 || B * p->H <= 512);
    case 4096: return B == 1;
    default: return false;
    }
}

// the sums of the runs; never 0 (the entry point refuses a missing workspace), and enough for every smaller batch
size_t row_backward_filter_bytes(const fftconv_plan *p, int64_t B)
{
    const Splits sp = grad_splits(p->M, p->H, B);
    return sp.most == 1 ? 256 : (size_t)(sp.most * p->H * p->M) * sizeof(float2);
}

// B >= 1
int row_backward_filter(const fftconv_plan *p, const void *u, const void *dy, float *dk, int64_t Nk, int64_t B, void *workspace,
                        hipStream_t s)
{
    return rf::with_row(p->M, [&](auto g) -> int {
        using G = decltype(g);
        if (p->dtype == FFTCONV_F32) return launch_half<G::M, float>(p, u, dy, dk, Nk, B, workspace, s);
        if (p->dtype == FFTCONV_F16) return launch_half<G::M, __half>(p, u, dy, dk, Nk, B, workspace, s);
        return launch_half<G::M, __hip_bfloat16>(p, u, dy, dk, Nk, B, workspace, s);
    });
}

}  // namespace fftconv
