// The two ends of the 8192-point matrix-core plans (fft_size 256 .. 8192) that are computed in fp32, on the row engine
// (row_fft.h): the filter transform, taps -> k_f, and the tail of the filter gradient, accumulated spectra -> dk.  One row
// of threads per channel, nothing in memory in between.
//
// The frequency digits of the kernels' slots are those of the engine's registers or multiples of them (8192: k1, k2, k3 are
// its digits 0, 1, 2), so both ends move slots in runs of 8 or 16 lanes straight between memory and registers.
// k_f has one 4-byte pair a bin, from which the convolution kernel makes its constants when it turns to a channel.  us, with 8-byte constants
// in as many copies as the kernel has groups (64 KB a channel) before: filter transform of 768 channels, fft 256 / 1024 / 2048 / 8192
// 12.5, 13.4, 21.9, 20 -> 7.5, 8.7, 8.8, 17.0 (the last one less again, see k_row_filter_8192); 8000 channels of fft 256 107 -> 8; convolutions of fft 8192, 64 x 768 x 4096 bf16 335 -> 323, f16
// 317 -> 295, 2 x 768 x 4096 20.7 -> 18.5.
// The gradient of plans below 8192 sums a spectrum for each of G = 8192 / fft_size groups (see build_tables() in fused3.hip): slot
// k1 of group g is g (32 / G) + k1'.  Up to 1024 points a row is part of one wave and most of the work is adding them up: there a
// workgroup takes one channel, and all of it moves the 64 KB, through an image of one group in LDS.
// Bound by the bytes.  Tail of the gradient, 768 channels of fft 8192: 46 -> 19 us (with every factor a trip through LDS and gathered
// twiddles before).
#include "fftconv_internal.h"
#include "lds_fft.h"
#include "row_io.h"

namespace fftconv {

namespace {

using rf::Row;

constexpr int SLOTS = 8192;                                       // of a channel, whatever the transform's length

// The gradient's tail.  One channel per workgroup, one group's slots in LDS: up to 1024 points, and where the runs of 2048 are added up (their
// slots lie scattered for a thread: 2.9 us for a run's spectrum, and those of two runs more than the second saved)
template <int M, bool RUNS> constexpr bool IMAGE = M <= 1024 || (RUNS && M == 2048);
template <int M, bool RUNS> constexpr int ROWS = IMAGE<M, RUNS> ? 1 : rf::threads_of(M) / Row<M>::T;      // channels per workgroup
// rows of the engine in a workgroup (2048 points: the second one repeats the first, unstored)
template <int M> constexpr int CHAINS = M <= 1024 ? 1 : rf::threads_of(M) / Row<M>::T;
template <int M, bool RUNS> constexpr int LDS_BYTES = CHAINS<M> * Row<M>::LDS_BYTES + (IMAGE<M, RUNS> ? 8 * M : 0);

// HALF: Nk <= M / 2.  conj_out: the conjugate spectrum, that of the circularly time-reversed taps, which are real.  k_f
// scaled by 1/M and by the frequency mask, one (re, im) pair of the I/O type a bin.
template <int M, bool F16, bool HALF>
__global__ void __launch_bounds__(rf::threads_of(M), 2)
    k_row_filter(const float *__restrict__ k, uint32_t *__restrict__ kf, const float2 *__restrict__ tab, int H, int64_t Nk, bool conj_out,
                 const uint8_t *__restrict__ keep, int64_t n_blocks, KfTag kf_tag)
{
    using G = Row<M>;
    set_tag(kf_tag);
    constexpr int RW = rf::threads_of(M) / G::T, MIN = HALF ? G::P / 2 : G::P;
    extern __shared__ float2 smem_rows[];
    const int row = threadIdx.x / G::T, tid = threadIdx.x % G::T;
    const int h = min((int)blockIdx.x * RW + row, H - 1);         // rows beyond the last one repeat it, unstored
    float2 *const Z = (float2 *)((char *)smem_rows + row * G::LDS_BYTES);
    uint32_t *const o = kf + (int64_t)h * M;
    float tap[MIN];
#pragma unroll
    for (int m = 0; m < MIN; ++m) {
        const int n = tid + G::T * m;
        tap[m] = k[h * Nk + (n < Nk ? n : 0)];
    }
#pragma unroll
    for (int m = 0; m < MIN; ++m) asm volatile("" ::"v"(tap[m]));   // the loads stay unconditional
    float2 x[G::P];
#pragma unroll
    for (int m = 0; m < MIN; ++m) x[m] = make_float2(tid + G::T * m < Nk ? tap[m] : 0.f, 0.f);
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    rf::forward<G, HALF>(x, Z, tab, tw1, tid, [] {});
    if ((int)blockIdx.x * RW + row >= H) return;
    // (one branch on the mask, not one for every bin)
    auto emit = [&](auto masked) {
        constexpr bool MASKED = decltype(masked)::value;
        auto constant = [&](int p) {
            const float sc = MASKED ? lds_mask_weight(keep, n_blocks, G::freq(tid, p), M) / M : 1.f / M;
            const float re = x[p].x * sc, im = (conj_out ? -x[p].y : x[p].y) * sc;
            return F16 ? f3::F16::pack(re, im) : f3::BF16::pack(re, im);
        };
#pragma unroll
        for (int p = 0; p < G::P; ++p) o[rf::slot_of<G>(tid, p)] = constant(p);
    };
    if (keep) emit(std::true_type());
    else emit(std::false_type());
}

// cos, sin of 2 pi 4 i / 8192
__device__ constexpr float COS4[8] = {1.f, 0.99999529380957617151f, 0.99998117528260110909f, 0.99995764455196389786f, 0.99992470183914450299f,
                                      0.99988234745421256111f, 0.99983058179582344007f, 0.99976940535121526662f};
__device__ constexpr float SIN4[8] = {0.f, 0.00306795676296597627f, 0.00613588464915447527f, 0.00920375478205981934f, 0.01227153828571992608f,
                                      0.01533920628498810015f, 0.01840672990580482092f, 0.02147408027546950739f};

// The same at 8192 points, where a row is most of a compute unit's registers: the taps are real, so it is transformed as 4096 points z[n] = k[2n] +
// i k[2n+1], Z goes back to the slots that the last pass read it from, and a lane forms the bins K[f], K[f + 4096] = E +- W_8192^f O of its f < 4096 from
// 2 E = Z[f] + conj Z[4096 - f] and 2 O = (Z[f] - conj Z[4096 - f]) / i.
// Half the transform for one more trip through LDS, and four workgroups to a compute unit instead of two; bound by its instructions, and by latency up to a
// workgroup or two to a unit.  us, rows of 8192 points -> so: 1 / 256 / 300 / 512 / 768 / 3000 channels 6.7, 7.2, 8.3, 9.3, 14.0, 42 -> 6.6, 6.5, 7.7, 8.7,
// 10.7, 28.5 (with a sine and a cosine for every k1 12.0 and 32.6).
// Of f = k1 + 32 k2 + 512 k3 the slot is (4 k1 + r) * 64 + 16 q + k2, where k3 = k3_at_index(4 q + r, 16) is 2 r + q / 2 for q = 0, 2 and 15 - (2 r + q / 2) for
// q = 1, 3: the bins f, f + 4096 of k3 = 2 r + s, s < 2, belong to q = 2 s of run 4 k1 + r and q = 3 - 2 s of run 4 k1 + 3 - r.  A wave takes two
// such runs, half its lanes the lower bins of either, and writes them whole in two stores.
template <bool F16, bool HALF>
__global__ void __launch_bounds__(256, 4)
    k_row_filter_8192(const float *__restrict__ k, uint32_t *__restrict__ kf, const float2 *__restrict__ tab, int64_t Nk, bool conj_out,
                      const uint8_t *__restrict__ keep, int64_t n_blocks, KfTag kf_tag)
{
    using G = Row<4096>;
    set_tag(kf_tag);
    constexpr int M = SLOTS, MIN = HALF ? G::P / 2 : G::P;
    static_assert(G::R0 == 16 && G::R1 == 16 && G::R2 == 16 && G::T == 256, "digits of a frequency, below");
    extern __shared__ float2 Z[];
    const int tid = threadIdx.x;
    const float *const row = k + blockIdx.x * Nk;
    {
        // (taps beyond Nk read tap 0 and are discarded)
        float2 x[G::P];
#pragma unroll
        for (int m = 0; m < MIN; ++m) {
            const int n = 2 * (tid + G::T * m);
            x[m].x = row[n < Nk ? n : 0];
            x[m].y = row[n + 1 < Nk ? n + 1 : 0];
        }
#pragma unroll
        for (int m = 0; m < MIN; ++m) asm volatile("" ::"v"(x[m].x), "v"(x[m].y));
#pragma unroll
        for (int m = 0; m < MIN; ++m) {
            const int n = 2 * (tid + G::T * m);
            x[m] = make_float2(n < Nk ? x[m].x : 0.f, n + 1 < Nk ? x[m].y : 0.f);
        }
        rf::Tw1<G> tw1;
        tw1.load(tab, tid);
        rf::forward<G, HALF>(x, Z, tab, tw1, tid, [] {});
#pragma unroll
        for (int i = 0; i < G::NBL; ++i) {
            float2 *const z = Z + G::slotl(tid + G::T * i);
#pragma unroll
            for (int r = 0; r < G::RL; ++r) z[r] = x[i * G::RL + r];
        }
    }
    __syncthreads();
    const int lane = tid & 63, up = lane >> 5, s = lane >> 4 & 1, k2 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t *const o = kf + blockIdx.x * (int64_t)M + k2;
    const float sgn = conj_out ? -1.f : 1.f;
    auto emit = [&](auto masked) {
        constexpr bool MASKED = decltype(masked)::value;
#pragma unroll
        for (int pair = 0; pair < 2; ++pair) {                    // runs r = pair (lanes 0 .. 31) and 3 - pair
            const int r = up ? 3 - pair : pair, k3 = 2 * r + s, fl = 32 * k2 + 512 * k3;
            const float rev = (float)(fl + wave) * (1.f / (float)M);          // exact: the sine and cosine take revolutions
            const float2 wl = make_float2(__builtin_amdgcn_cosf(rev), -__builtin_amdgcn_sinf(rev));
            // digits of f to base 16: d0 = k1 % 16, d1 = k1 / 16 + 2 (k2 % 8), d2 = k2 / 8 + 2 k3
            const int d1 = 2 * (k2 & 7), d2 = (k2 >> 3) + 2 * k3;
            const float2 *const za = Z + d1 * G::PAD + d2 + wave * G::PITCH, *const zm = Z + (15 - d1) * G::PAD + 15 - d2 - wave * G::PITCH;
            const int lo = wave * 256 + r * 64 + 32 * s, hi = wave * 256 + (3 - r) * 64 + 48 - 32 * s;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int top = i / 4, f = wave + 4 * i + fl;
                // the digits of 4096 - f: complements, plus one from the first that is not zero on
                const float2 a = za[4 * (i & 3) * G::PITCH + top * G::PAD];
                const float2 *m = zm + (16 - 4 * (i & 3)) * G::PITCH - top * G::PAD;
                if ((i & 3) == 0) {
                    const int e1 = d1 + top;
                    const float2 *const m0 = Z + ((16 - e1) & 15) * G::PAD + (e1 ? 15 - d2 : (16 - d2) & 15);
                    m = wave ? m : m0;
                }
                const float2 b = *m;
                const float2 w = i ? rf::mul(wl, make_float2(COS4[i], -SIN4[i])) : wl;
                const float2 e = make_float2(a.x + b.x, a.y - b.y);
                const float2 v = rf::mul(make_float2(a.y + b.y, b.x - a.x), w);
                const float s0 = MASKED ? lds_mask_weight(keep, n_blocks, f, M) * (0.5f / M) : 0.5f / M;
                const float s1 = MASKED ? lds_mask_weight(keep, n_blocks, f + M / 2, M) * (0.5f / M) : 0.5f / M;
                auto put = [&](int at, float re, float im) { o[1024 * i + at] = F16 ? f3::F16::pack(re, sgn * im) : f3::BF16::pack(re, sgn * im); };
                put(lo, (e.x + v.x) * s0, (e.y + v.y) * s0);
                put(hi, (e.x - v.x) * s1, (e.y - v.y) * s1);
            }
        }
    };
    if (keep) emit(std::true_type());
    else emit(std::false_type());
}

// dk[h][n] = Re(inverse transform)[n] / M, n < Nk, of the sum of the groups' spectra, and of the runs' (dkf[run][h]), added one
// after the other.  RUNS: more than one (the loop over them takes up to 45 registers, 1 - 2 us of 20 with many channels).
template <int M, bool RUNS>
__global__ void __launch_bounds__(rf::threads_of(M), 2)
    k_row_dk_finish(const float2 *__restrict__ dkf, float *__restrict__ dk, const float2 *__restrict__ tab, int H, int64_t Nk, int runs)
{
    using G = Row<M>;
    constexpr int RW = ROWS<M, RUNS>, NTHR = rf::threads_of(M);
    extern __shared__ float2 smem_rows[];
    const int row = CHAINS<M> == 1 ? 0 : threadIdx.x / G::T, tid = CHAINS<M> == 1 ? threadIdx.x : threadIdx.x % G::T;
    const int h = IMAGE<M, RUNS> ? (int)blockIdx.x : min((int)blockIdx.x * RW + row, H - 1);
    float2 *const Z = (float2 *)((char *)smem_rows + row * G::LDS_BYTES);
    float2 x[G::P];
    const float2 *in = dkf + (int64_t)h * SLOTS;
    if constexpr (IMAGE<M, RUNS>) {
        float2 *const image = (float2 *)((char *)smem_rows + CHAINS<M> * G::LDS_BYTES);
        constexpr int D = M / NTHR;
        static_assert(D * NTHR == M, "whole slots to a thread");
        float2 sum[D];
        auto add = [&](const float2 *spec, bool first) {           // all of a spectrum in flight at once
            float2 v[D][SLOTS / M];
#pragma unroll
            for (int d = 0; d < D; ++d)
#pragma unroll
                for (int g = 0; g < SLOTS / M; ++g) v[d][g] = spec[g * M + d * NTHR + threadIdx.x];
#pragma unroll
            for (int d = 0; d < D; ++d)
#pragma unroll
                for (int g = 0; g < SLOTS / M; ++g) {
                    sum[d].x = first && g == 0 ? v[d][g].x : sum[d].x + v[d][g].x;
                    sum[d].y = first && g == 0 ? v[d][g].y : sum[d].y + v[d][g].y;
                }
        };
        add(in, true);
#pragma unroll 1
        for (int i = 1; RUNS && i < runs; ++i) add(in + (int64_t)i * H * SLOTS, false);
#pragma unroll
        for (int d = 0; d < D; ++d) image[d * NTHR + threadIdx.x] = sum[d];
        __syncthreads();
        if (CHAINS<M> == 1 && tid >= G::T) return;
#pragma unroll
        for (int p = 0; p < G::P; ++p) x[p] = image[rf::slot_of<G>(tid, p)];
    } else {
        // (those of 2048 points, no base and immediates, are formed once: 6.8 us for few channels, 7.8 with each group's anew)
        int kept[M == 2048 ? G::P : 1];
        if constexpr (M == 2048) {
#pragma unroll
            for (int p = 0; p < G::P; ++p) {
                kept[p] = rf::slot_of<G>(tid, p);
                asm("" : "+v"(kept[p]));
            }
        }
        auto slot = [&](int p) {
            if constexpr (M == 2048) return kept[p];
            else return rf::slot_of<G>(tid, p);
        };
#pragma unroll
        for (int p = 0; p < G::P; ++p) x[p] = in[slot(p)];
        auto add = [&](const float2 *spec) {
            float2 v[G::P];
#pragma unroll
            for (int p = 0; p < G::P; ++p) v[p] = spec[slot(p)];
#pragma unroll
            for (int p = 0; p < G::P; ++p) {
                x[p].x += v[p].x;
                x[p].y += v[p].y;
            }
        };
#pragma unroll
        for (int g = 1; g < SLOTS / M; ++g) add(in + g * M);
#pragma unroll 1
        for (int i = SLOTS / M; RUNS && i < runs * (SLOTS / M); ++i) add(in + (int64_t)(i / (SLOTS / M)) * H * SLOTS + i % (SLOTS / M) * M);
    }
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    rf::inverse<G>(x, Z, tab, tw1, tid);
    if (IMAGE<M, RUNS> ? row > 0 : (int)blockIdx.x * RW + row >= H) return;
    float *const o = dk + (int64_t)h * Nk;
#pragma unroll
    for (int m = 0; m < G::P; ++m) {
        const int n = tid + G::T * m;
        if (n < Nk) o[n] = x[m].x * (1.f / M);
    }
}

// Factors of the fp64 filter transform's half-length rows: sixteens first, but 512 points as 8 . 8 . 8, as many passes as 16 . 16 . 2 and
// shorter ones (fft 1024, 257 / 3000 channels 12.0, 20.0 -> 10.6, 17.6 us; eights cost the other lengths a pass or more work: fft 8192,
// 128 channels 13.1, 14.5).
constexpr int filter64_factor(int L, int rest) { return L == 512 ? 8 : rest >= 16 ? 16 : rest; }
static FacList filter64_factors(int L)
{
    FacList fl{};
    for (int rest = L; rest > 1; rest /= fl.fac[fl.nf - 1]) fl.fac[fl.nf++] = filter64_factor(L, rest);
    return fl;
}
// lds_pos() for those factors.  The kernel asks for two of them a bin on its way out, and a loop over a list that it holds in memory took a
// quarter to a half of its time: fft 1024, 257 channels 10.6 -> 6.7 us, 3000 17.6 -> 12.4; 8192, 128 / 3000 13.1, 109 -> 11.5, 89; 16384, 2 / 3000
// 23.9, 313 -> 19.6, 268.
template <int L, int REST = L> __device__ __forceinline__ int filter64_pos(int f)
{
    if constexpr (REST == 1) {
        return 0;
    } else {
        constexpr int F = filter64_factor(L, REST);
        return (f & (F - 1)) * (REST / F) + filter64_pos<L, REST / F>(f / F);
    }
}

// ---- the filter transform of the plans that convolve on the row engine with k_f in fp32 (fft_size 256 .. 16384), in fp64:
// k_f[h] in the order of the engine's registers, [register pair][thread][2], scaled by 1/M and by the frequency mask.
// The taps are real, so a row is half as long: z[n] = k[2n] + i k[2n+1] is transformed in LDS (lds_fft.h, M/2 points: 139 KB at
// M = 16384), and with its even and odd parts E, O every bin is K[f] = E[f] + W_M^f O[f] on the way out.
// Bound by the latency of its passes.  Where a compute unit has one workgroup, which LDS makes it at 16384 points and up to 256
// channels at any length, M / 4 threads (at most 1024) shorten them most; with more channels than that, workgroups
// that fit beside one another do.  us, 4 / 256 / 3000 channels, one kernel for every row and one that permuted its spectrum (fft 16384: a
// kernel for every factor) -> half-length rows with few threads -> now: fft 1024 8.3, 14, 70 -> 12.3, 12.6, 21 -> 7.0, 7.6, 21;
// 4096 10.6, 46, 416 -> 13.2, 14.8, 60 -> 8.4, 10.2, 60; 8192 15, 53, 554 -> 15, 18, 112 -> 12, 15, 112; 16384 (4, 256, 1500) 26, 158, 966 ->
// 32, 37, 206 -> 25, 29, 150.  With positions known at compile time, 2 / 256 / 3000 channels: 6.5, 6.6, 12; 7.0, 8.5, 44;
// 10, 12, 89; 19.6, 24, 268.
template <int M, bool FEW> constexpr int FILTER64_THREADS = FEW ? (M >= 4096 ? 1024 : M / 4) : M >= 8192 ? 512 : M <= 1024 ? 64 : M / 16;
// SPLIT: gridDim.y workgroups a channel, each of which transforms the whole row and puts out its share of the bins, for channels that leave
// compute units idle: the way out is most of the time (fft 16384, 2 channels: 19.6 us, 11.5 without fifteen sixteenths of it).
template <int M, bool FEW, bool SPLIT>
__global__ void __launch_bounds__((FILTER64_THREADS<M, FEW>))
    k_row_filter64(const float *__restrict__ k, float2 *__restrict__ kf, const double2 *__restrict__ w, FacList fl, int64_t Nk,
                   bool conj_out, const uint8_t *__restrict__ keep, int64_t n_blocks)
{
    using G = Row<M>;
    constexpr int MH = M / 2, NTHR = FILTER64_THREADS<M, FEW>, PER = MH / NTHR < 8 ? MH / NTHR : 8;
    extern __shared__ double2 XD[];
    const float *row = k + blockIdx.x * Nk;
    for (int n0 = threadIdx.x; n0 < MH; n0 += PER * NTHR) {
        float a[PER], b[PER];                                     // (a tap beyond Nk reads tap 0 and is discarded)
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int n = 2 * (n0 + j * NTHR);
            a[j] = row[n < Nk ? n : 0];
            b[j] = row[n + 1 < Nk ? n + 1 : 0];
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) asm volatile("" ::"v"(a[j]), "v"(b[j]));
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int n = 2 * (n0 + j * NTHR);
            XD[lds_slot(n / 2)] = make_double2(n < Nk ? (double)a[j] : 0.0, n + 1 < Nk ? (double)b[j] : 0.0);
        }
    }
    __syncthreads();
    lds_forward(XD, w, fl, MH, 2);
    float2 *const o = kf + (int64_t)blockIdx.x * M;
    const int first = SPLIT ? blockIdx.y * NTHR + threadIdx.x : threadIdx.x, step = SPLIT ? gridDim.y * NTHR : NTHR;
#pragma unroll 4
    for (int d = first; d < M; d += step) {
        const int f = G::freq(d / 2 % G::T, d / (2 * G::T) * 2 + d % 2), fh = f & (MH - 1);
        const double2 z = XD[lds_slot(filter64_pos<MH>(fh))], m = XD[lds_slot(filter64_pos<MH>((MH - fh) & (MH - 1)))];
        const double2 e = make_double2(0.5 * (z.x + m.x), 0.5 * (z.y - m.y));          // (Z + conj Zm) / 2
        const double2 q = make_double2(0.5 * (z.y + m.y), -0.5 * (z.x - m.x));         // (Z - conj Zm) / (2i)
        const double2 v = cmul(q, w[f]);
        const double sc = (double)lds_mask_weight(keep, n_blocks, f, M) / (double)M;
        const double im = (e.y + v.y) * sc;
        o[d] = make_float2((float)((e.x + v.x) * sc), (float)(conj_out ? -im : im));
    }
}

}  // namespace

int row_filter64(const fftconv_plan *p, const float *k, int64_t Nk, bool conj_out, const uint8_t *keep_dev, int64_t n_blocks,
                 void *kf, hipStream_t s)
{
    return rf::with_row(p->M, [&](auto g) -> int {
        constexpr int M = decltype(g)::M;
        constexpr size_t lds = (size_t)(M / 2 + M / 32) * sizeof(double2);
        auto go = [&](auto few) -> int {
            constexpr bool FEW = decltype(few)::value;
            // Workgroups a channel: as many as the chip has compute units for, and a bin a thread at least.  us, one -> this rule, 2 / 16 / 64 / 128
            // channels: fft 4096 7.0, 7.3, 7.6, 8.0 -> 6.4, 6.7, 6.7, 7.5; 8192 10.1, 10.5, 10.9, 11.5 -> 7.1, 7.4, 8.5, 9.7; 16384 19.6,
            // 20.3, 21.1, 21.9 -> 11.5, 12.2, 14.4, 17.2.  Shorter rows are as fast without (fft 2048 6.5, 6.5).
            constexpr bool SPLIT = FEW && M >= 4096;
            int parts = 1;
            while (SPLIT && 2 * parts * p->H <= 256 && 2 * parts * FILTER64_THREADS<M, FEW> <= M) parts *= 2;
            const auto kernel = parts > 1 ? k_row_filter64<M, FEW, SPLIT> : k_row_filter64<M, FEW, false>;
            FC_TRY(raise_dynamic_lds((const void *)kernel, (int)lds));
            hipLaunchKernelGGL(kernel, dim3((unsigned)p->H, (unsigned)parts), dim3(FILTER64_THREADS<M, FEW>), lds, s, k, (float2 *)kf,
                               p->st.w64, filter64_factors(M / 2), Nk, conj_out, keep_dev, n_blocks);
            FC_HIP(hipGetLastError());
            return FFTCONV_OK;
        };
        if constexpr (M == 16384) return go(std::true_type());
        else return p->H <= 256 ? go(std::true_type()) : go(std::false_type());
    });
}

// k_f (H, Ms slots) of the 8192-point kernels for a transform of Ms = 256 .. 8192 points (min(fft_size, 8192): plans above
// keep the spectrum of a short filter this way)
int row_filter(const fftconv_plan *p, const float *k, int64_t Nk, int64_t Ms, bool conj_out, const uint8_t *keep_dev,
               int64_t n_blocks, uint32_t *kf, KfTag tag, hipStream_t s)
{
    return rf::with_row(Ms, [&](auto g) -> int {
        using G = decltype(g);
        if constexpr (G::M > SLOTS) {
            return FFTCONV_EUNSUPPORTED;
        } else if constexpr (G::M == SLOTS) {
            using R = Row<4096>;
            const bool f16 = p->dtype == FFTCONV_F16, half = 2 * Nk <= SLOTS;
            const auto kern = f16 ? (half ? k_row_filter_8192<true, true> : k_row_filter_8192<true, false>)
                                  : (half ? k_row_filter_8192<false, true> : k_row_filter_8192<false, false>);
            FC_TRY(raise_dynamic_lds((const void *)kern, R::LDS_BYTES));
            hipLaunchKernelGGL(kern, dim3((unsigned)p->H), dim3(R::T), R::LDS_BYTES, s, k, kf, rf::row_table<R>(p), Nk, conj_out, keep_dev,
                               n_blocks, tag);
            FC_HIP(hipGetLastError());
            return FFTCONV_OK;
        } else {
            constexpr int M = G::M, NTHR = rf::threads_of(M), RW = NTHR / G::T, lds = RW * G::LDS_BYTES;
            const bool f16 = p->dtype == FFTCONV_F16, half = 2 * Nk <= M;
            auto kern = f16 ? (half ? k_row_filter<M, true, true> : k_row_filter<M, true, false>)
                            : (half ? k_row_filter<M, false, true> : k_row_filter<M, false, false>);
            FC_TRY(raise_dynamic_lds((const void *)kern, lds));
            hipLaunchKernelGGL(kern, dim3((unsigned)((p->H + RW - 1) / RW)), dim3(NTHR), lds, s, k, kf, rf::row_table<G>(p), (int)p->H,
                               Nk, conj_out, keep_dev, n_blocks, tag);
            FC_HIP(hipGetLastError());
            return FFTCONV_OK;
        }
    });
}

// Runs from which they are added up by a kernel of its own (k_runs_add in row_grad.hip): a run costs the kernel above 1 us and more, that one 3.5 us in
// all.  us, bf16: fft 8192 16 x 1 rows (8 runs) 23.0, 17.2, 64 x 4 (16) 35.6, 22.3, 16 x 20 (8) 24.3, 21.4, 16 x 40 (6) 24.3, 27.5; 4096 32 x 1 (8) 22.3, 15.3, 64 x 30 (8)
// 30.8, 25.2; 2048 64 x 1 (8) 22.5, 17.5; 1024 200 x 1 (10) 25.3, 19.4.  Where channels are a multiple of 8, the workgroups of all runs of one, and the kernel
// above's, are on one die, whose L2 holds the sums: each is added up there.  Eight runs, the kernel above alone, with sums from any die, from their own: fft 8192 16 x 16
// 22.2, 20.2, 16.4, 16 x 32 24.9, 24.6, 19.7; 2048 64 x 32 24.4, 25.4, 20.6; 512 256 x 32 22.6, 24.0, 18.9; 256 512 x 32 20.9, 22.1, 17.1.
constexpr int64_t ADD_RUNS = 8;

// dkf: H * 8192 float2 in the kernels' slot order
int row_dk_finish(const fftconv_plan *p, void *dkf, int64_t runs, float *dk, int64_t Nk, hipStream_t s)
{
    if (runs >= ADD_RUNS) {
        FC_TRY(runs_add(dkf, p->H * (SLOTS / 2), runs, nullptr, dkf, p->H * (SLOTS / 2), s, SLOTS / 512));
        runs = 1;
    }
    return rf::with_row(p->M, [&](auto g) -> int {
        using G = decltype(g);
        if constexpr (G::M > SLOTS) {
            return FFTCONV_EUNSUPPORTED;
        } else {
            constexpr int NTHR = rf::threads_of(G::M);
            const auto kern = runs > 1 ? k_row_dk_finish<G::M, true> : k_row_dk_finish<G::M, false>;
            const int RW = runs > 1 ? ROWS<G::M, true> : ROWS<G::M, false>, lds = runs > 1 ? LDS_BYTES<G::M, true> : LDS_BYTES<G::M, false>;
            FC_TRY(raise_dynamic_lds((const void *)kern, lds));
            hipLaunchKernelGGL(kern, dim3((unsigned)((p->H + RW - 1) / RW)), dim3(NTHR), lds, s, (const float2 *)dkf,
                               dk, rf::row_table<G>(p), (int)p->H, Nk, (int)runs);
            FC_HIP(hipGetLastError());
            return FFTCONV_OK;
        }
    });
}

}  // namespace fftconv
