// fp32 transforms of rows too long for LDS (fft_size 16384 .. 2^22), two kernels per direction instead of one
// per factor: the decomposition of the generic path (Section 3.2, order-p Monarch form; decimation in
// frequency, position order out) with fft_size = A * 8192.
//   forward:  "columns" - the factors of A act at stride 8192: a workgroup takes C = 8192 / A adjacent columns
//             of the (A, 8192) view of a row into LDS (8192 points), runs those stages there with the twiddles
//             W_M^{k R r} of the full length and writes the tile back in place;
//             "blocks"  - the remaining factors act inside contiguous blocks of 8192 positions: one workgroup
//             per block, a transform of the row engine (row_fft.h) in registers and LDS.
//   inverse:  the same two kernels mirrored (blocks first, then columns).
// Users: the filter transform of the multi-pass plans (taps -> spectrum -> k_f, fp32 is ample for constants
// that are rounded to 16 bits) and the filter gradient of every plan from fft_size 16384 up that has no
// fused kernel (Section 3.1 "Kernel Fusion and Recomputation": dk = Re iFFT(sum_b conj(FFT(u_b)) FFT(dy_b))[0:Nk]).
// Two batch rows share one complex transform there, z = x_b + i x_{b+1}: conj(Z_u) Z_dy is the wanted sum plus
// i times a cross term that is itself the spectrum of a real sequence, so it ends up in the imaginary part of
// the inverse transform, which is dropped.
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include <cmath>
#include <type_traits>
#include <vector>

#include "fftconv_internal.h"
#include "lds_fft.h"
#include "outer_row.h"
#include "row_io.h"
#include "work_index.h"

namespace fftconv {

namespace {

constexpr int LB = 8192;                       // block length: what one workgroup holds in LDS
constexpr int LT = 512;                        // threads per workgroup
constexpr int OUTER_MOST = 16;                 // outer length up to which rows are formed on load
constexpr size_t L_LDS = (size_t)(LB + LB / 16) * sizeof(float2);

struct LongGeo {
    int A = 0, C = 0;                          // outer length, columns per tile (A * C = 8192)
    FacList flA, flB, fl;                      // factors of A, of 8192, and all of them (the position order)
};

LongGeo long_geo(int64_t M)
{
    LongGeo g;
    g.A = (int)(M / LB);
    g.C = LB / g.A;
    int nf = 0, rem = g.A;
    for (int i = 0; i < MAX_FACTORS; ++i) g.flA.fac[i] = g.flB.fac[i] = g.fl.fac[i] = 0;
    while (rem >= 16) {
        g.flA.fac[nf++] = 16;
        rem /= 16;
    }
    if (rem > 1) g.flA.fac[nf++] = rem;
    g.flA.nf = nf;
    g.flB = staged_factors_for(LB);
    g.fl.nf = g.flA.nf + g.flB.nf;
    for (int i = 0; i < g.flA.nf; ++i) g.fl.fac[i] = g.flA.fac[i];
    for (int i = 0; i < g.flB.nf; ++i) g.fl.fac[g.flA.nf + i] = g.flB.fac[i];
    return g;
}

__device__ __forceinline__ float ld_real(const float *p, int64_t i) { return p[i]; }
__device__ __forceinline__ float ld_real(const __half *p, int64_t i) { return __half2float(p[i]); }
__device__ __forceinline__ float ld_real(const __hip_bfloat16 *p, int64_t i) { return __bfloat162float(p[i]); }
__device__ __forceinline__ void st_real(float *p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void st_real(__half *p, int64_t i, float v) { p[i] = __float2half_rn(v); }
__device__ __forceinline__ void st_real(__hip_bfloat16 *p, int64_t i, float v) { p[i] = __float2bfloat16(v); }

// W_M^e of the full length as a product of two small tables, e = 2048 e_hi + e_lo: the exponents of the outer
// stages are spread over the whole range, and gathers from a table of M entries (16 MB at 2^21) miss every cache
struct LongTw {
    const float2 *lo, *hi;                     // W_M^t, t < 2048; W_M^{2048 t}, t < M / 2048
    __device__ __forceinline__ float2 operator()(int64_t e) const { return cmul(hi[e >> 11], lo[e & 2047]); }
};

// A thread's share of a tile of 8192 points: LPT points LT apart.  All loads of a thread are issued before the
// first value is used (a loop of load -> LDS write waits for every load in turn, and the round trip to HBM was most
// of these kernels' time); the launches use LT threads.
constexpr int LPT = LB / LT;
// column tile: slot i = a * C + c <- row[a * 8192 + col0 + c] (C a power of two)
__device__ __forceinline__ void load_cols(float2 *XL, const float2 *__restrict__ row, int C, int col0)
{
    const int lgC = __ffs(C) - 1;
    float2 v[LPT];
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        const int i = threadIdx.x + j * LT;
        v[j] = row[(int64_t)(i >> lgC) * LB + col0 + (i & (C - 1))];
    }
#pragma unroll
    for (int j = 0; j < LPT; ++j) XL[lds_slot(threadIdx.x + j * LT)] = v[j];
}

// One stage of the outer part on a tile X[a][c] (a < A, c < C, slot a * C + c): factor R_ along a at stride
// Sp, for every column; the twiddle exponent k Rj r uses the position r = rp * 8192 + (first column + c)
// inside the full-length stage.
template <int R_, bool INV>
__device__ inline void cols_stage(float2 *X, const LongTw &w, int A, int C, int Sp, int Rj, int col0)
{
    const int nb = (A / R_) * C;
    const int lgC = __ffs(C) - 1, lgSp = __ffs(Sp) - 1;          // powers of two
    for (int t = threadIdx.x; t < nb; t += blockDim.x) {
        const int c = t & (C - 1), q = t >> lgC;
        const int rp = q & (Sp - 1), prefix = q >> lgSp;
        const int a0 = prefix * R_ * Sp + rp;
        const int64_t rg = (int64_t)rp * LB + col0 + c;
        float2 x[R_], tw[R_];
        stage_twiddles<R_>(tw, w, (int64_t)Rj * rg);
#pragma unroll
        for (int n = 0; n < R_; ++n) {
            x[n] = X[lds_slot((a0 + n * Sp) * C + c)];
            if (INV) x[n] = cmul_conj(x[n], tw[n]);
        }
        dft_reg<R_, INV>(x);
#pragma unroll
        for (int k = 0; k < R_; ++k) X[lds_slot((a0 + k * Sp) * C + c)] = INV ? x[k] : cmul(x[k], tw[k]);
    }
}

template <bool INV>
__device__ inline void cols_stage_any(float2 *X, const LongTw &w, int A, int C, int Nj, int Sp, int Rj, int col0)
{
    switch (Nj) {
    case 2: cols_stage<2, INV>(X, w, A, C, Sp, Rj, col0); break;
    case 4: cols_stage<4, INV>(X, w, A, C, Sp, Rj, col0); break;
    case 8: cols_stage<8, INV>(X, w, A, C, Sp, Rj, col0); break;
    default: cols_stage<16, INV>(X, w, A, C, Sp, Rj, col0); break;
    }
}

// Forward, columns: rows of real input (re from src_re, im from src_im or zero; `len` valid samples, zeros
// beyond; reversed: position n holds sample (M - n) mod M) -> tmp (rows, M) after the factors of A.
// rows: where row i of the launch lies in its tensor (LongRows).
// half_rows (real input only, src_im == nullptr): only the blocks of the outer frequency digits ko <= A/2 are
// written; the others hold mirror images (see k_long_blocks_kf) and nobody reads them.
template <typename In>
__global__ void __launch_bounds__(LT) k_long_fwd_cols(const In *__restrict__ src_re, const In *__restrict__ src_im,
                                                     float2 *__restrict__ tmp, LongTw w, FacList flA, int A, int C, int64_t len,
                                                     bool reversed, bool half_rows, LongRows rows, const In *__restrict__ g_re,
                                                     const In *__restrict__ g_im)
{
    extern __shared__ float2 XL[];
    const int M = A * LB, N = (int)len;
    const int64_t row = blockIdx.y, first = rows.at(blockIdx.y) * len;
    const In *const re = src_re + first, *const im = src_im + first;
    const int col0 = blockIdx.x * C;
    const int lgC = __ffs(C) - 1;
    const bool two = src_im && rows.partner(blockIdx.y);
    // samples beyond `len` are zeros: their loads go to sample 0 instead and are discarded, so that every load of
    // the thread is unconditional and in flight at once (see load_block)
    float vr[LPT], vi[LPT];
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        const int i = threadIdx.x + j * LT;
        int n = (i >> lgC) * LB + col0 + (i & (C - 1));
        if (reversed && n != 0) n = M - n;
        vr[j] = ld_real(re, n < N ? n : 0);
        vi[j] = two ? ld_real(im, n < N ? n : 0) : 0.f;
    }
#pragma unroll
    for (int j = 0; j < LPT; ++j) asm volatile("" ::"v"(vr[j]), "v"(vi[j]));      // keeps the loads unconditional
    if (g_re) {                                               // the input gate (never with reversed)
        float gr[LPT], gi[LPT];
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            const int i = threadIdx.x + j * LT, n = (i >> lgC) * LB + col0 + (i & (C - 1));
            gr[j] = ld_real(g_re + first, n < N ? n : 0);
            gi[j] = two ? ld_real(g_im + first, n < N ? n : 0) : 0.f;
        }
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            vr[j] *= gr[j];
            vi[j] *= gi[j];
        }
    }
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        const int i = threadIdx.x + j * LT;
        int n = (i >> lgC) * LB + col0 + (i & (C - 1));
        if (reversed && n != 0) n = M - n;
        XL[lds_slot(i)] = n < N ? make_float2(vr[j], vi[j]) : make_float2(0.f, 0.f);
    }
    __syncthreads();
    int Sp = A, R = 1;
    for (int i = 0; i < flA.nf; ++i) {
        const int Nj = flA.fac[i];
        Sp /= Nj;
        cols_stage_any<false>(XL, w, A, C, Nj, Sp, R, col0);
        __syncthreads();
        R *= Nj;
    }
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        const int i = threadIdx.x + j * LT;
        const int ap = i >> lgC;                              // position of the block; its digit: lds_freq()
        if (!half_rows || 2 * lds_freq(ap, flA, A) <= A)
            (tmp + row * M)[ap * LB + col0 + (i & (C - 1))] = XL[lds_slot(i)];
    }
}

// ---- blocks of 8192 positions: whole rows of the row engine (row_fft.h), one to a workgroup of 256 threads, samples and
// results straight between HBM and registers.
using RB = rf::Row<LB>;
using RX = rf::Row<LB, true>;                  // exact twiddles: spectra that are kept in fp32
static_assert(RB::SLOTS == RX::SLOTS && RB::T == RX::T, "rows differ in their tables only");

template <typename G> __device__ __forceinline__ void load_row(float2 (&x)[G::P], const float2 *src, int tid)
{
#pragma unroll
    for (int m = 0; m < G::P; ++m) x[m] = src[tid + G::T * m];
}
template <typename G> __device__ __forceinline__ void store_row(const float2 (&x)[G::P], float2 *dst, int tid)
{
#pragma unroll
    for (int m = 0; m < G::P; ++m) dst[tid + G::T * m] = x[m];
}

// Filter transform: the block at position a' of a row holds the bins f = ko + A f' of one outer frequency digit ko (the
// digit reversal of a'), f' < 8192; they go straight to that digit's row of k_f, scaled by 1/M and by the frequency mask:
//   KF 0 / 1: bf16 / fp16 pairs [h][ko][slot of f' in the 8192-point kernel's per-lane order] (multi-pass plans; fp16
//             times the range boost, multipass_kf_boost);
//   KF 2:     fp32 pairs [h][position of ko][register order of the row engine] (fp32 I/O from fft_size 32768 up).
// The taps are real, so K[M - f] = conj K[f]: with f = ko + A f', M - f = (A - ko) + A (8191 - f') for ko >= 1.  Only the
// blocks of the digits ko <= A/2 are transformed (the kernel before wrote no others); a block with 0 < ko < A/2 also
// writes the row of the digit A - ko, bin g of which is the conjugate of this row's bin 8191 - g.  The rows ko = 0 and
// ko = A/2 are their own mirror images.
// natural: tmp holds the rows ko <= A/2 only, in the order of ko (A/2 + 1 blocks per channel: the output of
// k_filter_outer_real, multipass.hip) instead of all A blocks in position order.  conj_out: the conjugate spectrum
// (that of the circularly time-reversed taps, which are real).
// Bound by the memory traffic: the digits (k1, k2, k3) of f' are those of the row engine's registers (k1 = k0, k2 = digit 1,
// k3 = digit 2), so k_f needs no exchange through LDS.  128 channels of fft 131072 (142 MB): 54 us with stores of 16
// slots in a row, 41 with four lane groups transposed and runs of 64.
// fp32 pairs, 4 channels: fft 2^18 20.7 us with an LDS kernel, 22.5 with 8-byte stores and the last block fetched once more, 18.7
// now; 2^21 46.6, 50.8, 42.5; 768 channels of fft 32768 151, 134, 110; bf16, 768 channels of fft 65536 230, 163, 157.
// Workgroups are persistent, two to a compute unit, and fetch the next block ahead of the present one's transform: loads,
// transforms and stores of workgroups that all start together otherwise take turns on the whole chip.
// TAPS: src holds the taps themselves, and the rows ko are formed of them on the way in (outer_row.h).  Up to A = 16 most transforms go so: 256 channels of fft
// 131072 bf16 95 -> 61 us (of 65536 taps that stay in the caches; 76 each in a training step), 768 of 65536 151 -> 95, 768 of 32768 fp32 109 -> 51 (the times
// above are of rows from memory).
template <int KF, bool TAPS>
__global__ void __launch_bounds__(RB::T, 2) k_long_blocks_kf(const void *__restrict__ src, void *__restrict__ kf,
                                                             const float2 *__restrict__ tab, FacList flA, int A, int64_t h0, int blocks,
                                                             const uint8_t *__restrict__ keep, int64_t n_blocks, bool natural,
                                                             bool conj_out, KfTag kf_tag, const float2 *__restrict__ outer, int Nk)
{
    set_tag(kf_tag);
    using G = std::conditional_t<KF == 2, RX, RB>;
    extern __shared__ float2 XL[];
    const int M = A * LB, NR = A / 2 + 1;
    const float scale = (KF == 1 ? (float)multipass_kf_boost(true, A) : 1.f) / (float)M, sgn = conj_out ? -1.f : 1.f;
    auto source = [&](int blk) {                              // block blk = channel * (A / 2 + 1) + ko
        const int h = blk / NR, ko = blk % NR;
        return (const float2 *)src + (natural ? (int64_t)blk : (int64_t)h * A + lds_pos(ko, flA, A)) * LB;
    };
    using Taps = OuterRow<float, 32>;
    auto taps = [&](int blk) { return Taps{(const float *)src + (int64_t)(blk / NR) * Nk, Nk}; };
    // TAPS: a die takes an eighth of the blocks, so that the rows ko of a channel are formed from one L2
    const int each = TAPS ? (blocks + 7) / 8 : blocks, at0 = TAPS ? blockIdx.x % 8 * each : 0;
    const int end = at0 + each < blocks ? at0 + each : blocks, step = TAPS ? gridDim.x / 8 : gridDim.x;
    const int begin = TAPS ? at0 + blockIdx.x / 8 : blockIdx.x;
    if (TAPS && begin >= end) return;                         // (the others have no more workgroups than blocks)
    float2 next[TAPS ? 1 : G::P];
    Taps::Units word;
    if constexpr (TAPS) taps(begin).fetch(word, threadIdx.x);
    else load_row<G>(next, source(begin), threadIdx.x);
#pragma unroll 1
    for (int blk = begin; blk < end; blk += step) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));                         // nothing of a step's addresses and twiddles is kept for the next
        float2 x[G::P];
        rf::Tw1<G> tw1;
        if constexpr (TAPS) {
            const int ko = blk % NR;
            const float2 factor = outer[outer_tab_sums(A) + ko * OUTER_T + tid];
            taps(blk).sum(x, word, outer + ko * A * OUTER_M, taps(blk + step < end ? blk + step : blk), tid);
            tw1.load(tab, tid);
            rf::row_barrier<G::T>();                          // the slots are free
            rf::forward<G, false>(x, XL, tab, tw1, tid, [] {}, factor);
        } else {
#pragma unroll
            for (int p = 0; p < G::P; ++p) x[p] = next[p];
            if (blk + step < end) load_row<G>(next, source(blk + step), tid);
            tw1.load(tab, tid);
            rf::row_barrier<G::T>();                          // the slots are free
            rf::forward<G, false>(x, XL, tab, tw1, tid, [] {});
        }
        const int ko = blk % NR;
        const int64_t h = h0 + blk / NR;
        const bool mirror = ko > 0 && 2 * ko < A;
        const int km = mirror ? A - ko : ko;
        const int64_t row = (h * A + (KF == 2 ? lds_pos(ko, flA, A) : ko)) * LB;
        const int64_t row_m = (h * A + (KF == 2 ? lds_pos(km, flA, A) : km)) * LB;
        // (one branch on the mask, not one for every bin)
        auto emit = [&](auto masked) {
            constexpr bool MASKED = decltype(masked)::value;
            // weights of the bins of register p in this row and in the mirror row
            auto weight = [&](int p) { return MASKED ? lds_mask_weight(keep, n_blocks, ko + A * G::freq(tid, p), M) * scale : scale; };
            auto weight_m = [&](int p) {
                return MASKED ? lds_mask_weight(keep, n_blocks, km + A * (LB - 1 - G::freq(tid, p)), M) * scale : scale;
            };
            if constexpr (KF == 2) {
                // pairs of registers, as they lie in memory; bin 8191 - f' belongs to the thread and the register with all digits
                // complemented, T - 1 - tid and P - 1 - p
                float4 *const o = (float4 *)kf + row / 2 + tid, *const om = (float4 *)kf + row_m / 2 + (G::T - 1 - tid);
#pragma unroll
                for (int q = 0; q < G::P / 2; ++q) {
                    const float s0 = weight(2 * q), s1 = weight(2 * q + 1);
                    o[q * G::T] = make_float4(x[2 * q].x * s0, sgn * x[2 * q].y * s0, x[2 * q + 1].x * s1, sgn * x[2 * q + 1].y * s1);
                }
                if (mirror) {
#pragma unroll
                    for (int q = 0; q < G::P / 2; ++q) {
                        const int a = G::P - 1 - 2 * q, b = a - 1;
                        const float s0 = weight_m(a), s1 = weight_m(b);
                        om[q * G::T] = make_float4(x[a].x * s0, -sgn * x[a].y * s0, x[b].x * s1, -sgn * x[b].y * s1);
                    }
                }
            } else {
                // slots (k1 * 4 + r) * 64 + 16 (idx / 4) + k2, idx = k3_index(k3), r = idx % 4: lane group q holds k1 = 4 wave + q (+ 16 i),
                // k2 = its lane, and all k3 = p % 16 in registers; transposed, a store is a whole run of 64 slots
                auto pack = [](float re, float im) { return KF == 1 ? f3::F16::pack(re, im) : f3::BF16::pack(re, im); };
                const int lane = tid & 63, k1w = tid / 64 * 4;
                uint32_t *const o = (uint32_t *)kf + row + lane, *const om = (uint32_t *)kf + row_m + (lane & 48) + 15 - (lane & 15);
#pragma unroll
                for (int ir = 0; ir < 8; ++ir) {
                    const int i = ir / 4, r = ir % 4;
                    uint32_t v[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int p = 16 * i + k3_at_index(4 * c + r, 16);
                        const float sc = weight(p);
                        v[c] = pack(x[p].x * sc, sgn * x[p].y * sc);
                    }
                    rf::transpose_groups(v);
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[((k1w + j + 16 * i) * 4 + r) * 64] = v[j];
                    if (mirror) {                                     // bin 8191 - f': every digit is complemented
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const int p = 16 * i + 15 - k3_at_index(4 * c + r, 16);
                            const float scm = weight_m(p);
                            v[c] = pack(x[p].x * scm, -sgn * x[p].y * scm);
                        }
                        rf::transpose_groups(v);
#pragma unroll
                        for (int j = 0; j < 4; ++j) om[((31 - (k1w + j + 16 * i)) * 4 + r) * 64] = v[j];
                    }
                }
            }
        };
        if (keep) emit(std::true_type());
        else emit(std::false_type());
    }
}

// Filter gradient: sum over nb batch rows of conj(FFT(block of u)) . FFT(block of dy) for the blocks of a launch (grid:
// blocks of a channel, channels, runs of `per` batch rows; batch row b at a distance of b * stride), then back: acc holds the sum
// of earlier rows unless first, and takes it unless last, when the inverse transform goes to out (which may be a block of tu).
// The spectra and their sum stay in registers (one transform at a time: 192 data registers), where three kernels
// wrote and read them; the row of dy is fetched with that of u, in the registers that then take the spectrum of u.
// Several runs: a run's sum goes, in register order, where its first row of u was (nobody else reads that block), and
// k_long_blocks_sum adds them up.  Few channels leave the chip idle otherwise, and two launches per batch row and tensor ahead of
// this one: whole gradient, us, bf16 16 x 1 x 65536 307 -> 63, f16 73 x 1 x 20000 fft 65536 1317 -> 101, 16 x 1 x 2^20 467 -> 192, fp32
// 8 x 16 x 10000 fft 32768 170 -> 52; 16 x 64 x 16384 464 -> 231 (the first four less again, see ADD_RUNS); where the chip was full, bf16 2 x 256 x 65536, 414 -> 402.
__global__ void __launch_bounds__(RB::T, 2) k_long_blocks_corr(float2 *tu, const float2 *td, int64_t stride, int nb, int per,
                                                               float4 *acc, float2 *out, const float2 *__restrict__ tab, bool first,
                                                               bool last)
{
    using G = RB;
    extern __shared__ float2 XL[];
    const int64_t base = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * LB;
    const int tid = threadIdx.x, b0 = blockIdx.z * per, b1 = min(b0 + per, nb);
    const bool runs = gridDim.z > 1;
    float2 sum[G::P];
    if (first || runs) {
#pragma unroll
        for (int p = 0; p < G::P; ++p) sum[p] = make_float2(0.f, 0.f);
    } else {
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) {
            const float4 v = acc[base / 2 + tid + q * G::T];
            sum[2 * q] = make_float2(v.x, v.y);
            sum[2 * q + 1] = make_float2(v.z, v.w);
        }
    }
#pragma unroll 1
    for (int b = b0; b < b1; ++b) {
        float2 x[G::P], z[G::P];
        auto transform = [&](float2 (&v)[G::P], int j) {
            rf::Tw1<G> tw1;
            tw1.load(tab, j);
            rf::row_barrier<G::T>();                          // the slots are free
            rf::forward<G, false>(v, XL, tab, tw1, j, [] {});
        };
        int j = tid;
        asm volatile("" : "+v"(j));                           // nothing of a step's addresses and twiddles is kept for the next
        load_row<G>(z, tu + b * stride + base, j);
        load_row<G>(x, td + b * stride + base, j);
        transform(z, j);
        asm volatile("" : "+v"(j));
        transform(x, j);
#pragma unroll
        for (int p = 0; p < G::P; ++p) {                      // sum += conj(Z_u) Z_dy
            sum[p].x = __builtin_fmaf(z[p].y, x[p].y, __builtin_fmaf(z[p].x, x[p].x, sum[p].x));
            sum[p].y = __builtin_fmaf(-z[p].y, x[p].x, __builtin_fmaf(z[p].x, x[p].y, sum[p].y));
        }
    }
    if (runs || !last) {
        float4 *const o = (runs ? (float4 *)(tu + b0 * stride) : acc) + base / 2 + tid;
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) o[q * G::T] = make_float4(sum[2 * q].x, sum[2 * q].y, sum[2 * q + 1].x, sum[2 * q + 1].y);
        return;
    }
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    rf::inverse<G>(sum, XL, tab, tw1, tid);
    store_row<G>(sum, out + base, tid);
}

// The same from the rows of u and dy themselves (outer_row.h): block (ko, channel) of all batch rows of a run; part: the sums of the
// runs, `apart` pairs from one to the next, or out of one run, transformed back.
// ONE: one batch row to a run; no sum is held beside its transforms, and twice the samples are in flight.
template <typename IO, bool ONE>
__global__ void __launch_bounds__(RB::T, 2) k_long_rows_corr(const IO *__restrict__ u, const IO *__restrict__ dy, int N, int H, int A, int nb,
                                                             int per, int nruns, float2 *__restrict__ part, int64_t apart,
                                                             const float2 *__restrict__ tab, const float2 *__restrict__ outer)
{
    using G = RB;
    extern __shared__ float2 XL[];
    // A die takes an eighth of the blocks, those of a channel's runs one after another, so that the rows ko of a run are formed from one L2, and no die is left
    // without work where channels are few.  (An eighth of each run's blocks: three dies idle at 5 blocks, f32 300 x 1 x 65536 205.8 -> 84.9 us, 128 x 2 155 -> 80,
    // bf16 128 x 1 x 65536 fft 131072 127 -> 79; one run's blocks after another's: f32 8 x 8 x 32768 fft 65536 38.0 -> 35.8, 3 x 57 x 32768 49.2 -> 47.7.)
    const int NR = A / 2 + 1, total = H * NR * nruns, each = (total + 7) / 8, unit = blockIdx.x % 8 * each + blockIdx.x / 8;
    if (blockIdx.x / 8 >= each || unit >= total) return;
    const int h = unit / (NR * nruns), of_h = unit % (NR * nruns), run = of_h / NR, ko = of_h % NR, blk = h * NR + ko;
    const int tid = threadIdx.x, b0 = run * per, b1 = min(b0 + per, nb);
    const bool runs = nruns > 1;
    const float2 *const sums = outer + ko * A * OUTER_M, *const factors = outer + outer_tab_sums(A) + ko * OUTER_T;
    using Samples = OuterRow<IO, ONE ? 32 : 16>;
    auto row = [&](const IO *t, int b) { return Samples{t + ((int64_t)b * H + h) * N, N}; };
    float2 sum[G::P];
#pragma unroll
    for (int p = 0; p < G::P; ++p) sum[p] = make_float2(0.f, 0.f);
    auto add = [&](int b) {
        float2 x[G::P], z[G::P];
        typename Samples::Units word;
        auto transform = [&](float2 (&v)[G::P], int j) {
            rf::Tw1<G> tw1;
            tw1.load(tab, j);
            const float2 factor = factors[j];
            rf::row_barrier<G::T>();                          // the slots are free
            rf::forward<G, false>(v, XL, tab, tw1, j, [] {}, factor);
        };
        int j = tid;
        asm volatile("" : "+v"(j));                           // nothing of a step's addresses and twiddles is kept for the next
        row(u, b).fetch(word, j);
        row(u, b).sum(z, word, sums, row(dy, b), j);
        transform(z, j);
        asm volatile("" : "+v"(j));
        row(dy, b).sum(x, word, sums, Samples{dy, 0}, j);
        transform(x, j);
#pragma unroll
        for (int p = 0; p < G::P; ++p) {                      // sum += conj(Z_u) Z_dy
            sum[p].x = __builtin_fmaf(z[p].y, x[p].y, __builtin_fmaf(z[p].x, x[p].x, sum[p].x));
            sum[p].y = __builtin_fmaf(-z[p].y, x[p].x, __builtin_fmaf(z[p].x, x[p].y, sum[p].y));
        }
    };
    if constexpr (ONE) {
        add(b0);
    } else {
#pragma unroll 1
        for (int b = b0; b < b1; ++b) add(b);
    }
    float2 *const out = part + (int64_t)blk * LB;
    if (runs) {
        float4 *const o = (float4 *)(out + run * apart) + tid;
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) o[q * G::T] = make_float4(sum[2 * q].x, sum[2 * q].y, sum[2 * q + 1].x, sum[2 * q + 1].y);
        return;
    }
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    rf::inverse<G>(sum, XL, tab, tw1, tid);
    store_row<G>(sum, out, tid);
}

// The sums of the runs above, `apart` pairs from one to the next, added up in order; acc, first, last, out as there.
__global__ void __launch_bounds__(RB::T, 2) k_long_blocks_sum(const float2 *part, int64_t apart, int runs, float4 *acc, float2 *out,
                                                              const float2 *__restrict__ tab, bool first, bool last)
{
    using G = RB;
    extern __shared__ float2 XL[];
    const int64_t base = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * LB;
    const int tid = threadIdx.x;
    float2 x[G::P];
    auto add = [&](const float4 *in, bool set) {
        float4 v[G::P / 2];
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) v[q] = in[q * G::T];
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) asm volatile("" ::"v"(v[q].x));           // all loads of a run together
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) {
            x[2 * q].x = set ? v[q].x : x[2 * q].x + v[q].x;
            x[2 * q].y = set ? v[q].y : x[2 * q].y + v[q].y;
            x[2 * q + 1].x = set ? v[q].z : x[2 * q + 1].x + v[q].z;
            x[2 * q + 1].y = set ? v[q].w : x[2 * q + 1].y + v[q].w;
        }
    };
    const float4 *const in = (const float4 *)(part + base) + tid;
    add(first ? in : acc + base / 2 + tid, true);
    for (int r = first ? 1 : 0; r < runs; ++r) add(in + r * (apart / 2), false);
    if (!last) {
        float4 *const o = acc + base / 2 + tid;
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) o[q * G::T] = make_float4(x[2 * q].x, x[2 * q].y, x[2 * q + 1].x, x[2 * q + 1].y);
        return;
    }
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    rf::inverse<G>(x, XL, tab, tw1, tid);
    store_row<G>(x, out + base, tid);
}

// Inverse, columns: the factors of A, then real part times scale of the samples n < Nk -> dk (rows, Nk).
__global__ void __launch_bounds__(LT) k_long_inv_cols_dk(const float2 *__restrict__ tmp, float *__restrict__ dk, LongTw w,
                                                        FacList flA, int A, int C, int64_t Nk, float scale)
{
    extern __shared__ float2 XL[];
    const int64_t M = (int64_t)A * LB, row = blockIdx.y;
    const int col0 = blockIdx.x * C;
    if (col0 >= Nk) return;                                 // every sample of this tile is n >= col0 >= Nk
    load_cols(XL, tmp + row * M, C, col0);
    __syncthreads();
    int Sp = 1, R = A;
    for (int i = flA.nf - 1; i >= 0; --i) {
        const int Nj = flA.fac[i];
        R /= Nj;
        cols_stage_any<true>(XL, w, A, C, Nj, Sp, R, col0);
        __syncthreads();
        Sp *= Nj;
    }
    for (int i = threadIdx.x; i < LB; i += LT) {
        const int a = i >> (__ffs(C) - 1), c = i & (C - 1);
        const int64_t n = (int64_t)a * LB + col0 + c;
        if (n < Nk) dk[row * Nk + n] = XL[lds_slot(i)].x * scale;
    }
}

// ---- The convolution itself in fp32 (plans with fp32 I/O from fft_size 32768 up; shorter rows: row_conv.hip):
// y = iFFT(FFT(pad(u)) . k_f)[0:N] with k_f as fp32 pairs in position order, already scaled by 1 / fft_size.  Two batch
// rows share a complex transform (re = row b, im = row b + 1; k is real, so the two convolutions come back as re and im).
//
// Middle kernel: a block of 8192 positions forward, times its piece of k_f, and back, in place in tmp.
// natural: tmp holds the rows ko <= A/2 of real sequences in the order of ko (A/2 + 1 blocks per row, the output
// of k_filter_outer_real); the k_f of digit ko sits at that digit's position among the A blocks of the channel.  Row i of the
// launch belongs to channel (h0 + i) mod H.
__global__ void __launch_bounds__(RB::T, 2) k_long_conv_blocks(float2 *__restrict__ tmp, const float4 *__restrict__ kf,
                                                               const float2 *__restrict__ tab, FacList flA, int A, bool natural, int h0,
                                                               int H)
{
    using G = RB;
    extern __shared__ float2 XL[];
    const int64_t base = natural ? ((int64_t)blockIdx.y * (A / 2 + 1) + blockIdx.x) * LB
                                 : ((int64_t)blockIdx.y * A + blockIdx.x) * LB;
    const int64_t kbase = ((int64_t)((h0 + (int)blockIdx.y) % H) * A + (natural ? lds_pos(blockIdx.x, flA, A) : (int)blockIdx.x)) * LB;
    const int tid = threadIdx.x;
    float2 x[G::P];
    load_row<G>(x, tmp + base, tid);
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    float4 kv[G::P / 2];
    const float4 *const kr = kf + kbase / 2 + tid;
    rf::forward<G, false>(x, XL, tab, tw1, tid, [&] {
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) kv[q] = kr[q * G::T];
    });
#pragma unroll
    for (int q = 0; q < G::P / 2; ++q) {
        x[2 * q] = rf::mul(x[2 * q], make_float2(kv[q].x, kv[q].y));
        x[2 * q + 1] = rf::mul(x[2 * q + 1], make_float2(kv[q].z, kv[q].w));
    }
    rf::inverse<G>(x, XL, tab, tw1, tid);
    store_row<G>(x, tmp + base, tid);
}

// The same from rows of u (outer_row.h), fp32: row i of the `rows` of u belongs to channel (h0 + i) mod H, and its blocks ko <= A/2 go to
// tmp.  Whole batch rows (nb of them, else nb = 1): a channel's rows one after another, so that its k_f is fetched once.
template <bool GATED>
__global__ void __launch_bounds__(RB::T, 2) k_long_conv_rows(const float *__restrict__ u, const float *__restrict__ gate, int N,
                                                             float2 *__restrict__ tmp,
                                                             const float4 *__restrict__ kf, const float2 *__restrict__ tab,
                                                             const float2 *__restrict__ outer, FacList flA, int A, int rows, int nb, int h0,
                                                             int H)
{
    using G = RB;
    extern __shared__ float2 XL[];
    const int NR = A / 2 + 1, blocks = rows * NR, each = (blocks + 7) / 8, blk = blockIdx.x % 8 * each + blockIdx.x / 8;
    if (blockIdx.x / 8 >= each || blk >= blocks) return;
    const int ko = blk % NR, i = blk / NR, row = i % nb * (rows / nb) + i / nb;
    const int64_t kbase = ((int64_t)((h0 + row) % H) * A + lds_pos(ko, flA, A)) * LB;
    const int tid = threadIdx.x;
    float2 x[G::P];
    using Samples = OuterRow<float, GATED ? 16 : 32, GATED>;
    {
        const Samples from{u + (int64_t)row * N, N, gate + (GATED ? (int64_t)row * N : 0)};
        typename Samples::Units word;
        from.fetch(word, tid);
        from.sum(x, word, outer + ko * A * OUTER_M, Samples{u, 0, gate}, tid);
    }
    const float2 factor = outer[outer_tab_sums(A) + ko * OUTER_T + tid];
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    float4 kv[G::P / 2];
    const float4 *const kr = kf + kbase / 2 + tid;
    rf::forward<G, false>(x, XL, tab, tw1, tid, [&] {
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) kv[q] = kr[q * G::T];
    }, factor);
#pragma unroll
    for (int q = 0; q < G::P / 2; ++q) {
        x[2 * q] = rf::mul(x[2 * q], make_float2(kv[q].x, kv[q].y));
        x[2 * q + 1] = rf::mul(x[2 * q + 1], make_float2(kv[q].z, kv[q].w));
    }
    rf::inverse<G>(x, XL, tab, tw1, tid);
    store_row<G>(x, tmp + ((int64_t)row * NR + ko) * LB, tid);
}

// Longer rows, last kernel: the outer factors back, real part -> row of y_re, imaginary part -> row of y_im
// (nullptr: no second row), the first N samples.
// GATED: times the rows of g_re and g_im.  A thread asks for all its gates at once, and ahead of the transforms: a workgroup has its compute
// unit to itself (70 KB, 131 registers), so nothing else covers a load that is waited for.  us, output gate, sample by sample behind them -> so (with a
// kernel of its own): 2 x 256 x 131072 circular 641 -> 435 (552), 2 x 1024 x 16384 fft 32768 494 -> 408 (446).
template <typename IO, bool GATED>
__global__ void __launch_bounds__(LT) k_long_inv_cols_y(const float2 *__restrict__ tmp, IO *__restrict__ y_re,
                                                       IO *__restrict__ y_im, LongTw w, FacList flA, int A, int C, int64_t N,
                                                       LongRows rows, const IO *__restrict__ g_re, const IO *__restrict__ g_im)
{
    extern __shared__ float2 XL[];
    const int64_t M = (int64_t)A * LB, row = blockIdx.y, first = rows.at(blockIdx.y) * N;
    IO *const re = y_re + first, *const im = y_im + first;
    const int col0 = blockIdx.x * C;
    if (col0 >= N) return;
    const bool two = y_im && rows.partner(blockIdx.y);
    const int lgC = __ffs(C) - 1;
    float gr[GATED ? LPT : 1], gi[GATED ? LPT : 1];
    if constexpr (GATED) {
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            const int i = threadIdx.x + j * LT, n = (i >> lgC) * LB + col0 + (i & (C - 1));
            gr[j] = ld_real(g_re + first, n < N ? n : 0);
            gi[j] = two ? ld_real(g_im + first, n < N ? n : 0) : 0.f;
        }
    }
    load_cols(XL, tmp + row * M, C, col0);
    __syncthreads();
    int Sp = 1, R = A;
    for (int i = flA.nf - 1; i >= 0; --i) {
        const int Nj = flA.fac[i];
        R /= Nj;
        cols_stage_any<true>(XL, w, A, C, Nj, Sp, R, col0);
        __syncthreads();
        Sp *= Nj;
    }
    if constexpr (GATED) {
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            const int i = threadIdx.x + j * LT, n = (i >> lgC) * LB + col0 + (i & (C - 1));
            if (n < N) {
                const float2 v = XL[lds_slot(i)];
                st_real(re, n, v.x * gr[j]);
                if (two) st_real(im, n, v.y * gi[j]);
            }
        }
    } else {
        for (int i = threadIdx.x; i < LB; i += LT) {
            const int n = (i >> lgC) * LB + col0 + (i & (C - 1));
            if (n < N) {
                const float2 v = XL[lds_slot(i)];
                st_real(re, n, v.x);
                if (two) st_real(im, n, v.y);
            }
        }
    }
}

__global__ void k_zero_dk(float *x, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0.f;
}

LongTw long_tw(const fftconv_plan *p)
{
    LongTw t;
    t.lo = p->long_tw;
    t.hi = t.lo + 2048;
    return t;
}

int raise_lds(const void *kern) { return raise_dynamic_lds(kern, (int)L_LDS); }

template <typename In>
int launch_fwd_cols(const LongGeo &g, const In *re, const In *im, float2 *tmp, const LongTw &w, int64_t rows, int64_t len,
                    bool reversed, hipStream_t s, bool half_rows = false, LongRows where = long_rows(0), const In *g_re = nullptr,
                    const In *g_im = nullptr)
{
    const int rc = raise_lds((const void *)k_long_fwd_cols<In>);
    if (rc) return rc;
    hipLaunchKernelGGL(k_long_fwd_cols<In>, dim3((unsigned)g.A, (unsigned)rows), dim3(LT), L_LDS, s, re, im, tmp, w, g.flA,
                       g.A, g.C, len, reversed, half_rows && im == nullptr, where, g_re, g_im);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

// outer lengths whose rows the block kernels form themselves
bool outer_on_load(int64_t A) { return A >= 4 && A <= OUTER_MOST; }
const float2 *outer_table(const fftconv_plan *p) { return p->long_tw + 2048 + p->M / 2048; }

// rows of the block kernels' launches: their LDS and the plan's table
constexpr int B_LDS = RB::LDS_BYTES;

// Filter gradient of real rows: pairs of transformed rows of u and dy in a trip through the workspace, as many as it holds, up to 2 GiB.  us
// with trips of 128, 256, 768 MiB, all at once: bf16 64 rows of 2^20, two batch rows 1664, 1434, 1385, 1350, one 908, 807, 800, 783; fp32 64 rows of
// 2^19, two batch rows 771, 752, 726, 713; bf16 2 x 256 x 65536 367, 376, 367, 369; launches too short for the chip cost more than the
// memory-side cache returns.  The workspace: three spectra of a batch row, and no less than 256 MiB (fp32 16 x 64 x 16384 fft 32768 with
// 64, 128, 256 MiB, all at once 510, 325, 246, 246).
constexpr int64_t GRAD_TRIP = (int64_t)1 << 28, GRAD_LEAST = (int64_t)1 << 25;

// Four runs or more are added up by k_runs_add (row_grad.hip) first, on every compute unit, and cost less, up to 64 spectra; beyond those the next
// kernel has that many workgroups of its own to fetch them, and six runs are needed.  (Where a trip's sums are not transformed back, that kernel is left
// out, at any number.)  Whole gradient, us, with the other kernel alone: bf16 16 x 1 x 65536 59.7 -> 40.5, 30 x 2 x 131072 105 -> 87, f16 73 x 1 x 20000 fft 65536
// 97.8 -> 60.9 (64.7 with no more runs than before), fp32 fft 32768, 3 spectra a channel, 4 x 1 x 16384 28.9 -> 26.2, 4 x 16 38.2 -> 37.7, 4 x 20 43.0, 43.4, 8 x 20 61.0 -> 56.5,
// 4 x 24 43.6, 45.3, 4 x 30 49.1, 52.0, 8 x 42 85, 89, but six and seven runs 7 x 24 58.1 -> 54.5, 14 x 24 88.7 -> 85.3, 14 x 26 91.7, 91.4; two trips, 32 x 30 244 -> 221.
constexpr int64_t ADD_RUNS = 4, ADD_MOST = 64, ADD_MANY = 6;

// nh channels of `blocks` blocks each; runs of batch rows where channels alone leave compute units idle: as many as fill the
// chip (two workgroups to a unit), and no more than pay for adding them up (a run's sum takes about a sixteenth of the time of
// a batch row's two transforms, one after another; a quarter of that from ADD_RUNS up)
int launch_corr(const fftconv_plan *p, int blocks, int64_t nh, float2 *tu, const float2 *td, int64_t stride, int64_t nb, float2 *acc,
                float2 *out, bool first, bool last, hipStream_t s)
{
    FC_TRY(raise_dynamic_lds((const void *)k_long_blocks_corr, B_LDS));
    int64_t runs = 512 / (blocks * nh);
    if (runs > nb) runs = nb;
    while (runs > 1 && runs * runs > (runs >= ADD_RUNS ? 64 : 16) * nb) --runs;
    if (runs < 1) runs = 1;
    const int64_t per = (nb + runs - 1) / runs;
    runs = (nb + per - 1) / per;
    const float2 *tab = rf::row_table<RB>(p);
    hipLaunchKernelGGL(k_long_blocks_corr, dim3((unsigned)blocks, (unsigned)nh, (unsigned)runs), dim3(RB::T), B_LDS, s, tu, td, stride,
                       (int)nb, (int)per, (float4 *)acc, out, tab, first, last);
    FC_HIP(hipGetLastError());
    if (runs == 1) return FFTCONV_OK;
    if (runs >= ADD_RUNS && (!last || blocks * nh <= ADD_MOST || runs >= ADD_MANY)) {
        FC_TRY(runs_add(tu, per * stride / 2, runs, first ? nullptr : acc, last ? tu : acc, blocks * nh * (LB / 2), s, LB / 512));
        if (!last) return FFTCONV_OK;
        first = true;
        runs = 1;
    }
    FC_TRY(raise_dynamic_lds((const void *)k_long_blocks_sum, B_LDS));
    hipLaunchKernelGGL(k_long_blocks_sum, dim3((unsigned)blocks, (unsigned)nh), dim3(RB::T), B_LDS, s, tu, per * stride, (int)runs,
                       (float4 *)acc, out, tab, first, last);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

// Gradients whose kernel forms its rows itself (outer_row.h): where the chip has enough of them, or a row has few blocks to add up, one after
// another.  Whole gradient, us, from an outer pass -> so: bf16 2 x 256 x 65536 364 -> 280, 1 x 256 204 -> 169, 2 x 256 x 32768 194 -> 121, f32 2 x 256 x 65536
// 404 -> 302, 20 x 100 x 16384 431 -> 252, 1 x 1 x 16384 20.1 -> 19.2, bf16 16 x 1 x 65536 39.4 -> 37.7; one row of 65536 samples 23.7 -> 26.2, one of
// 32768 21.3 -> 21.5, 2 x 8 x 32768 30.0 -> 31.0; with other kernels between, 7 and 8 blocks: bf16 1 x 26 x 65536 28.7 -> 30.1, 4 x 8 34.8 -> 36.0, fft 131072 16 x 1
// 35.1 -> 36.4, from 176 spectra on none slower; sixteen blocks, 2 x 256 x 131072 400 -> 405, f32 5 x 3 40.4 -> 46.6.  A few calls of 7 and 8 blocks just beyond the line lose as well (1 x 40 x 65536 f32 33.6 -> 36.0, bf16
// 1 x 48 34.4 -> 36.4, 3 x 20 fft 131072 59.1 -> 60.4; 1 x 57 1.06 times as fast).  dk of fft 131072 4.33e-7 -> 3.67e-7.
// (Batch rows are counted in 32 bits, in up to 512 runs that end less than a row each beyond the last one.)
}  // namespace
bool grad_on_load(int64_t A, int64_t n, int64_t B, int64_t H)
{
    return outer_on_load(A) && B < INT32_MAX - 512 && (n <= 2 || (n <= 8 && B * H * (A / 2 + 1) >= (n <= 6 ? 128 : 176)));
}
namespace {


// The same from u and dy (k_long_rows_corr): the inverse transforms' rows of all channels -> out, which holds `fit` rows of A/2 + 1 blocks
template <typename IO>
int launch_rows_corr(const fftconv_plan *p, const IO *u, const IO *dy, int64_t nb, float2 *out, int64_t fit, hipStream_t s)
{
    const int64_t A = p->M / LB, blocks = p->H * (A / 2 + 1);
    int64_t runs = 512 / blocks;
    if (runs > nb) runs = nb;
    if (runs > fit / p->H) runs = fit / p->H;
    while (runs > 1 && runs * runs > (runs >= ADD_RUNS ? 64 : 16) * nb) --runs;
    if (runs < 1) runs = 1;
    const int64_t per = (nb + runs - 1) / runs, apart = blocks * LB;
    runs = (nb + per - 1) / per;
    const float2 *tab = rf::row_table<RB>(p);
    const auto kern = per == 1 ? k_long_rows_corr<IO, true> : k_long_rows_corr<IO, false>;
    FC_TRY(raise_dynamic_lds((const void *)kern, B_LDS));
    hipLaunchKernelGGL(kern, dim3((unsigned)((blocks * runs + 7) / 8 * 8)), dim3(RB::T), B_LDS, s, u, dy, (int)p->N, (int)p->H, (int)A,
                       (int)nb, (int)per, (int)runs, out, apart, tab, outer_table(p));
    FC_HIP(hipGetLastError());
    if (runs == 1) return FFTCONV_OK;
    if (runs >= ADD_RUNS && (blocks <= ADD_MOST || runs >= ADD_MANY)) {
        FC_TRY(runs_add(out, apart / 2, runs, nullptr, out, blocks * (LB / 2), s, LB / 512));
        runs = 1;
    }
    FC_TRY(raise_dynamic_lds((const void *)k_long_blocks_sum, B_LDS));
    hipLaunchKernelGGL(k_long_blocks_sum, dim3((unsigned)(A / 2 + 1), (unsigned)p->H), dim3(RB::T), B_LDS, s, out, apart, (int)runs,
                       (float4 *)nullptr, out, tab, true, true);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

// Rows of a batch row's channel (A/2 + 1 blocks of 8192 pairs) that the workspace of the real pipeline below holds at most
int64_t grad_rows(const fftconv_plan *p)
{
    const int64_t row = (p->M / LB / 2 + 1) * LB, all = 3 * p->H * p->M;
    return (all > GRAD_LEAST ? all : GRAD_LEAST) / row;
}

template <typename IO>
int long_backward_filter_t(const fftconv_plan *p, const IO *u, const IO *dy, float *dk, int64_t Nk, int64_t B,
                           void *workspace, hipStream_t s)
{
    const LongGeo g = long_geo(p->M);
    const LongTw tw = long_tw(p);
    const int64_t M = p->M, N = p->N, H = p->H;
    if (B == 0) {
        const int bs = 256;
        hipLaunchKernelGGL(k_zero_dk, dim3((unsigned)((H * Nk + bs - 1) / bs)), dim3(bs), 0, s, dk, H * Nk);
        FC_HIP(hipGetLastError());
        return FFTCONV_OK;
    }
    if (grad_on_load(M / LB, (N + LB - 1) / LB, B, H)) {
        FC_TRY(launch_rows_corr(p, u, dy, B, (float2 *)workspace, grad_rows(p), s));
        return multipass_dk_outer_inv(p, workspace, dk, Nk, H, 1.0f / (float)M, s);
    }
    if (multipass_filter_outer_ok(p)) {
        // Outer lengths with a register kernel for real rows (multipass.hip): every row of u and dy is transformed
        // as a real sequence -- outer pass on the rows ko <= A/2 only, 8192-point block transforms of those rows,
        // acc (+)= conj(U) DY on them -- and the sum, the spectrum of a real sequence again, goes back through the
        // inverse block transforms and the real inverse outer pass: half the intermediate traffic of the complex
        // pipeline below, and a row without a partner costs no more than half a pair.
        // The channels go in trips of at most GRAD_TRIP pairs of transformed rows of u and dy, with all batch rows where they fit,
        // else in pieces with the sum so far behind them.
        const int NR = g.A / 2 + 1;
        const int64_t row = NR * (int64_t)LB, fit = grad_rows(p);
        const int64_t trip = fit < GRAD_TRIP / row ? fit : GRAD_TRIP / row;
        int64_t nh = H;
        if (2 * B * H > trip) nh = trip / (2 * B);
        if (nh > 16384 / B) nh = 16384 / B;                       // rows of a launch
        if (nh < 1) nh = 1;
        // (of up to a third fewer channels, the number whose blocks leave least of a round of the chip empty: bf16 2 x 256 x 65536 in
        // three trips, of 86, 113 + 113 + 30: 402, 393 us)
        auto full = [&](int64_t n) { return (double)(n * NR) / (double)((n * NR + 511) / 512); };
        for (int64_t n = nh - 1, most = nh; nh < H && 3 * n >= 2 * most; --n)
            if (full(n) > full(nh)) nh = n;
        const bool once = 2 * B * nh <= fit && 2 * B * nh <= 65535;
        int64_t nb = once ? B : (fit - 1) / 2;                    // (nh is 1 then)
        if (nb > 32767) nb = 32767;
        for (int64_t h0 = 0; h0 < H; h0 += nh) {
            const int64_t n_h = H - h0 < nh ? H - h0 : nh, stride = n_h * row;
            for (int64_t b = 0; b < B; b += nb) {
                const int64_t n = B - b < nb ? B - b : nb;
                float2 *const tu = (float2 *)workspace, *const td = tu + n * stride, *const acc = tu + (fit - 1) * row;
                const int64_t o = (b * H + h0) * N;
                FC_TRY(multipass_filter_outer(p, OuterRows{u + o, dy + o, (int)(n * n_h), (int)n_h, (int)H}, p->dtype, N, 2 * n * n_h, tu, s));
                FC_TRY(launch_corr(p, NR, n_h, tu, td, stride, n, acc, tu, b == 0, b + n == B, s));
            }
            FC_TRY(multipass_dk_outer_inv(p, workspace, dk + h0 * Nk, Nk, n_h, 1.0f / (float)M, s));
        }
        return FFTCONV_OK;
    }
    float2 *acc = (float2 *)workspace, *tu = acc + H * M, *td = tu + H * M;
    for (int64_t b = 0; b < B; b += 2) {                      // rows b and b + 1 share a transform
        const IO *u0 = u + b * H * N, *u1 = b + 1 < B ? u0 + H * N : nullptr;
        const IO *d0 = dy + b * H * N, *d1 = b + 1 < B ? d0 + H * N : nullptr;
        FC_TRY(launch_fwd_cols<IO>(g, u0, u1, tu, tw, H, N, false, s));
        FC_TRY(launch_fwd_cols<IO>(g, d0, d1, td, tw, H, N, false, s));
        FC_TRY(launch_corr(p, g.A, H, tu, td, 0, 1, acc, tu, b == 0, b + 2 >= B, s));
    }
    FC_TRY(raise_lds((const void *)k_long_inv_cols_dk));
    hipLaunchKernelGGL(k_long_inv_cols_dk, dim3((unsigned)g.A, (unsigned)H), dim3(LT), L_LDS, s, tu, dk, tw, g.flA,
                       g.A, g.C, Nk, 1.0f / (float)M);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

template <int KF>
int launch_kf(const fftconv_plan *p, const LongGeo &g, int64_t nh, const float2 *tmp, void *kf, int64_t h0, const uint8_t *keep_dev,
              int64_t n_blocks, bool natural, bool conj_out, KfTag tag, hipStream_t s)
{
    FC_TRY(raise_dynamic_lds((const void *)k_long_blocks_kf<KF, false>, B_LDS));
    const float2 *tab = KF == 2 ? rf::row_table<RX>(p) : rf::row_table<RB>(p);
    const int64_t blocks = nh * (g.A / 2 + 1);                // at most 2^16 channels of 257
    hipLaunchKernelGGL((k_long_blocks_kf<KF, false>), dim3((unsigned)(blocks < 512 ? blocks : 512)), dim3(RB::T), B_LDS, s, tmp, kf, tab,
                       g.flA, g.A, h0, (int)blocks, keep_dev, n_blocks, natural, conj_out, tag, nullptr, 0);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

// from the taps themselves (outer_row.h)
template <int KF>
int launch_kf_taps(const fftconv_plan *p, const float *k, int64_t Nk, bool conj_out, const uint8_t *keep_dev, int64_t n_blocks, void *kf,
                   KfTag tag, hipStream_t s)
{
    const LongGeo g = long_geo(p->M);
    FC_TRY(raise_dynamic_lds((const void *)k_long_blocks_kf<KF, true>, B_LDS));
    const float2 *tab = KF == 2 ? rf::row_table<RX>(p) : rf::row_table<RB>(p);
    const int64_t blocks = p->H * (g.A / 2 + 1), grid = blocks < 512 ? (blocks + 7) / 8 * 8 : 512;
    hipLaunchKernelGGL((k_long_blocks_kf<KF, true>), dim3((unsigned)grid), dim3(RB::T), B_LDS, s, k, kf, tab, g.flA, g.A, (int64_t)0,
                       (int)blocks, keep_dev, n_blocks, true, conj_out, tag, outer_table(p), (int)Nk);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

// ---- the forward pass: rows of the whole batch go through the workspace in trips (one pair of batch rows at a time, three launches each,
// left the chip idle where channels are few: 30 x 1 x 65536 fft 65536 348 -> 28 us, 7 x 2 x 2^19 gated 219 -> 79, 8 x 16 x 131072 fft 2^18
// 281 -> 169, 16 x 64 x 16384 fft 32768 262 -> 177).
// Rows go one at a time as real sequences (the rows ko <= A/2 of the outer transform, their blocks (forward, k_f, inverse), real
// inverse outer pass; k_f is the spectrum of real taps, so the product is the spectrum of a real sequence again) where outer
// lengths have register kernels for real rows (multipass.hip), else in pairs of batch rows.  Real rows are half the blocks of a complex transform
// per row (3 for 2 at A = 4), with cheaper outer kernels (2.8 against 3.3 ms for 2^27 samples at fft 2^18); up to A = 16 the blocks' kernel forms its rows ko
// itself (outer_row.h), for the trip that this saves.  Pairs -> real rows so formed, us, fp32: A = 4, 8 x 256 x 16384 363 -> 299, 4 x 64 51.5 -> 40.4; A = 8,
// 4 x 256 x 32768 364 -> 274, 2 x 16 26.3 -> 21.0 (real rows from an outer pass before); A = 16, 4 x 256 x 65536 693 -> 542, 2 x 256 x 131072 394 -> 353; errors
// 3.29e-7 -> 2.79e-7, 3.54e-7 -> 2.98e-7, 3.45e-7 -> 3.15e-7.
// Rows of more than 8 blocks (4 with an input gate, which doubles the loads) are not formed so by a few workgroups, which add the blocks up one
// after another (1 x 1 x 131072 19.9 -> 22.2 us; gated 1 x 1 x 65536 19.5 -> 21.3, 4 x 64 200 -> 179), nor are those of 7 and 8 by fewer still (fft 65536, 1, 2, 4, 6 rows of
// 65536 16.9 -> 17.9, 17.2 -> 18.2, 17.7 -> 18.1, 18.4 -> 18.3, of 6 and 12 with other kernels between 19.6 -> 20.7 and 20.4 -> 21.1; gated, four blocks of fft 32768, 1 and 12 rows 16.1 -> 16.4, 19.4 -> 18.9), and not those of more than 8 with a gate
// (2 x 256 x 131072 442 -> 455).  They take an outer pass, at A = 16 in pairs: real rows from an outer pass are a tenth less accurate there (3.45e-7,
// 3.80e-7); a row without a partner goes as a real one, or, where the chip has room, with the pairs and zeros for a partner.
// Rounds of 512 workgroups, as with the filters (filter_on_load()): a second one of few does not pay from 13 blocks on, 1 x 57 x 131072 51 -> 57, 1 x 90 1.03 times as
// fast, 2 x 29 53 -> 55, 2 x 32 59 -> 58, 4 x 15 55.5 -> 57; odd batches, whose last row has no partner, gain all the same (3 x 20 1.29 times), and so do more
// rounds but for one batch row of more than 14 blocks (1 x 114 1.08 times, 1 x 190 145 -> 149, 1 x 200 159 -> 152, 1 x 228 176 -> 178, 1 x 256 196 -> 190), and in the
// first round 17 to 23 channels of it (16 30.3 -> 28.0, 20 31.5 -> 32.5, 24 1.02 times).
// An odd batch whose last row can go with the pairs does, where the filter takes an outer pass: on load it would be less accurate (3 x 3 x 65536 at fft 131072
// 3.35e-7 -> 3.40e-7, though 3 x 2 19.7 us instead of 27.2; with the filter on load, too, it is more accurate: 3 x 6 3.35e-7 -> 3.14e-7, 36.9 -> 24.8 us).
bool lone_in_pairs(int64_t A, int64_t B, int64_t H) { return B > 1 && A == 16 && (B + 1) / 2 * H * 16 <= 1024; }
}  // namespace
bool conv_on_load(int64_t A, int64_t n, int64_t B, int64_t H, bool gated)
{
    if (!outer_on_load(A) || (gated && n > 8)) return false;
    if (A == 16 && B > 1 && B % 2 == 1 && lone_in_pairs(A, B, H) && !filter_on_load(A, n, H, true)) return false;
    const int64_t blocks = B * H * (A / 2 + 1);
    if (n <= 3 || (n <= 6 && !gated)) return true;
    if (n == 4) return A != 4 || blocks >= 36;
    if (!gated && n <= 8) return blocks >= (A == 8 ? 60 : 18);
    if ((gated ? B : 1) * H * (A / 2 + 1) < (gated && n > 6 ? 176 : 128)) return false;
    const int64_t rounds = (blocks + 511) / 512, last = blocks - 512 * (rounds - 1), turns = (n + 1) / 2;
    if (gated) return A != 16 || n < 8 || B > 1 || rounds != 2 || last >= 64;
    if (turns < 7) return true;
    if (rounds == 1) return B > 1 || turns < 8 || blocks <= 144 || blocks >= 216;
    if (rounds > 2) return B > 1 || turns < 8 || rounds == 3 || rounds > 5 || last >= 200;
    return B == 1 ? last >= 149 * (turns - 6) : B % 2 == 1 || last >= 64;
}
namespace {

bool conv_on_load(const fftconv_plan *p, int64_t B, bool gated)
{
    return fftconv::conv_on_load(p->M / LB, (p->N + LB - 1) / LB, B, p->H, gated);
}
bool conv_real(const fftconv_plan *p, int64_t B, bool gated)
{
    return multipass_filter_outer_ok(p) && (p->M / LB != 16 || conv_on_load(p, B, gated));
}
int64_t real_row(const fftconv_plan *p) { return (p->M / LB / 2 + 1) * LB; }

// pairs of fp32 values in the workspace of a trip: 512 MiB, or a row where that is more.  us with 64, 128, 256, 512 MiB: 4 x 8 x 2^20 fft
// 2^21 390, 368, 350, 344; 16 x 256 x 16384 fft 32768 751, 703, 719, 681; 16 x 256 x 32768 1572, 1419, 1443, 1378
constexpr int64_t CONV_TRIP = (int64_t)1 << 26;
// the workspace that the static entry point was sized for: a pair of batch rows of as many channels as 512 MiB hold
int64_t conv_least(const fftconv_plan *p)
{
    const int64_t c = ((int64_t)512 << 20) / (p->M * (int64_t)sizeof(float2));
    return (c < 1 ? 1 : c < p->H ? c : p->H) * p->M;
}
// no more for a smaller batch
int64_t conv_pairs(const fftconv_plan *p, int64_t B)
{
    auto pairs = [](int64_t units, int64_t unit) {
        const int64_t fit = CONV_TRIP / unit < 1 ? 1 : CONV_TRIP / unit;
        return (units < fit ? units : fit) * unit;
    };
    const int64_t rows = multipass_filter_outer_ok(p) ? pairs(B * p->H, real_row(p)) : 0;
    // (whether any batch goes in pairs, with gates or without)
    const int64_t two = conv_real(p, 2, true) && conv_real(p, 2, false) ? 0 : pairs((B + 1) / 2 * p->H, p->M);
    return rows > two ? rows : two;
}

// cap: pairs that the workspace holds (at least a row's)
template <typename IO>
int long_forward_t(const fftconv_plan *p, const IO *u, const float2 *kf, IO *y, int64_t B, void *workspace, int64_t cap, hipStream_t s,
                   const IO *wg, const IO *vg)
{
    const int64_t M = p->M, N = p->N, H = p->H;
    const LongGeo g = long_geo(M);
    const LongTw tw = long_tw(p);
    float2 *tmp = (float2 *)workspace;
    FC_TRY(raise_dynamic_lds((const void *)k_long_conv_blocks, B_LDS));
    const auto inv_cols = vg ? k_long_inv_cols_y<IO, true> : k_long_inv_cols_y<IO, false>;
    FC_TRY(raise_lds((const void *)inv_cols));
    auto blocks = [&](int per_row, int64_t first, int64_t n, bool natural) -> int {
        hipLaunchKernelGGL(k_long_conv_blocks, dim3((unsigned)per_row, (unsigned)n), dim3(RB::T), B_LDS, s, tmp, (const float4 *)kf,
                           rf::row_table<RB>(p), g.flA, g.A, natural, (int)(first % H), (int)H);
        FC_HIP(hipGetLastError());
        return FFTCONV_OK;
    };
    // trips of n of `units` units from `first` on, of about equal size; 65535: the grid's second dimension
    auto trips = [&](int64_t units, int64_t unit, auto trip) -> int {
        int64_t fit = cap / unit < 1 ? 1 : cap / unit;
        if (fit > 65535) fit = 65535;
        const int64_t count = (units + fit - 1) / fit;
        for (int64_t i = 0; i < count; ++i) FC_TRY(trip(units * i / count, units * (i + 1) / count - units * i / count));
        return FFTCONV_OK;
    };
    auto as_real = [&](int64_t row0, int64_t rows) -> int {
        return trips(rows, real_row(p), [&](int64_t first, int64_t n) -> int {
            const int64_t o = (row0 + first) * N;
            if (conv_on_load(p, B, wg != nullptr)) {
                const auto kern = wg ? k_long_conv_rows<true> : k_long_conv_rows<false>;
                FC_TRY(raise_dynamic_lds((const void *)kern, B_LDS));
                hipLaunchKernelGGL(kern, dim3((unsigned)(n * (g.A / 2 + 1) + 7) / 8 * 8), dim3(RB::T), B_LDS, s, (const float *)(u + o),
                                   (const float *)(wg ? wg + o : nullptr), (int)N, tmp, (const float4 *)kf, rf::row_table<RB>(p),
                                   outer_table(p), g.flA, g.A, (int)n, n % H ? 1 : (int)(n / H), (int)((row0 + first) % H), (int)H);
                FC_HIP(hipGetLastError());
            } else {
                FC_TRY(multipass_filter_outer(p, outer_rows(u + o), FFTCONV_F32, N, n, tmp, s, wg ? wg + o : nullptr));
                FC_TRY(blocks(g.A / 2 + 1, row0 + first, n, true));
            }
            return multipass_dk_outer_inv(p, tmp, (float *)(y + o), N, n, 1.0f, s, vg ? vg + o : nullptr);
        });
    };
    auto as_complex = [&](int64_t b, int64_t units, bool pairs) -> int {
        return trips(units, M, [&](int64_t first, int64_t n) -> int {
            const LongRows where = pairs ? long_row_pairs(first, H, (B - b) * H) : long_rows(first);
            const IO *u0 = u + b * H * N, *w0 = wg ? wg + b * H * N : nullptr, *v0 = vg ? vg + b * H * N : nullptr;
            IO *y0 = y + b * H * N;
            FC_TRY(launch_fwd_cols<IO>(g, u0, pairs ? u0 + H * N : nullptr, tmp, tw, n, N, false, s, false, where, w0,
                                       wg && pairs ? w0 + H * N : nullptr));
            FC_TRY(blocks(g.A, first, n, false));
            hipLaunchKernelGGL(inv_cols, dim3((unsigned)g.A, (unsigned)n), dim3(LT), L_LDS, s, (const float2 *)tmp, y0,
                               pairs ? y0 + H * N : nullptr, tw, g.flA, g.A, g.C, N, where, v0, vg && pairs ? v0 + H * N : nullptr);
            FC_HIP(hipGetLastError());
            return FFTCONV_OK;
        });
    };
    if (conv_real(p, B, wg != nullptr)) return as_real(0, B * H);
    if (lone_in_pairs(M / LB, B, H)) return as_complex(0, (B + 1) / 2 * H, true);
    if (B > 1) FC_TRY(as_complex(0, B / 2 * H, true));
    if (B % 2 == 0) return FFTCONV_OK;
    return multipass_filter_outer_ok(p) ? as_real((B - 1) * H, H) : as_complex(B - 1, H, false);
}

}  // namespace

// The filter transform and the filter gradient: rows of fft_size = A * 8192, A = 2 .. 512; a channel must fit the grid's second
// dimension (the forward pass goes in chunks of channels and takes any number)
bool long_fft_supported(const fftconv_plan *p) { return p->M >= 2 * LB && p->M <= 512 * (int64_t)LB && p->H <= 65535; }

int long_fft_init(fftconv_plan *p)
{
    const int64_t M = p->M, nhi = M / 2048;
    const int A = (int)(M / LB);
    std::vector<float2> t((size_t)(2048 + nhi + (outer_on_load(A) ? outer_tab_size(A) : 0)));
    const double two_pi = 6.283185307179586476925286766559;
    auto wpow = [&](double num, double den) {
        const double a = two_pi * num / den;
        return make_float2((float)std::cos(a), (float)-std::sin(a));
    };
    for (int64_t i = 0; i < 2048; ++i) t[(size_t)i] = wpow((double)i, (double)M);
    for (int64_t i = 0; i < nhi; ++i) t[(size_t)(2048 + i)] = wpow((double)i, (double)nhi);
    if (outer_on_load(A)) {
        float2 *to = t.data() + 2048 + nhi;
        std::vector<float2> w((size_t)(OUTER_M * A));
        for (int i = 0; i < OUTER_M * A; ++i) w[(size_t)i] = wpow(i, OUTER_M * A);
        for (int ko = 0; ko <= A / 2; ++ko)
            for (int i = 0; i < OUTER_M * A; ++i) *to++ = w[(size_t)(ko * i % (OUTER_M * A))];
        for (int ko = 0; ko <= A / 2; ++ko)
            for (int j = 0; j < OUTER_T; ++j) *to++ = wpow((double)(ko * j), (double)M);
    }
    FC_HIP(hipMalloc((void **)&p->long_tw, t.size() * sizeof(float2)));
    FC_HIP(hipMemcpy(p->long_tw, t.data(), t.size() * sizeof(float2), hipMemcpyHostToDevice));
    return FFTCONV_OK;
}

void long_fft_destroy(fftconv_plan *p)
{
    if (p->long_tw) (void)hipFree(p->long_tw);
    p->long_tw = nullptr;
}

// The filter transform of channels [h0, h0 + nh) of a multi-pass plan: taps (nh, Nk) -> their rows of k_f; tmp holds
// nh * (A/2 + 1) * 8192 float2 with multipass_filter_outer_ok(p) (the chunks of the caller count on it), else nh * M.  adjoint: the spectrum of the circularly time-reversed filter (the conjugate spectrum).
int long_filter_transform(const fftconv_plan *p, const float *k, int64_t Nk, int64_t h0, int64_t nh, bool adjoint,
                          const uint8_t *keep_dev, int64_t n_blocks, float2 *tmp, void *kf, KfTag tag, hipStream_t s)
{
    const LongGeo g = long_geo(p->M);
    const LongTw tw = long_tw(p);
    // outer factor: the register kernel of the multi-pass route where it exists for this outer length (rows ko <= A/2
    // in natural order; the adjoint spectrum is then the conjugate, taken on the way out), else the generic column kernel
    const bool natural = multipass_filter_outer_ok(p);
    int rc = natural ? multipass_filter_outer(p, outer_rows(k), FFTCONV_F32, Nk, nh, tmp, s)
                     : launch_fwd_cols<float>(g, k, nullptr, tmp, tw, nh, Nk, adjoint, s, true);
    if (rc) return rc;
    return p->dtype == FFTCONV_F16 ? launch_kf<1>(p, g, nh, tmp, kf, h0, keep_dev, n_blocks, natural, natural && adjoint, tag, s)
                                   : launch_kf<0>(p, g, nh, tmp, kf, h0, keep_dev, n_blocks, natural, natural && adjoint, tag, s);
}

// The filter transform of all channels of a plan with A = M / 8192 = 4, 8 or 16, whatever its I/O type: one kernel from the taps to k_f (filter_on_load())
int long_filter_taps(const fftconv_plan *p, const float *k, int64_t Nk, bool adjoint, const uint8_t *keep_dev, int64_t n_blocks, void *kf,
                     KfTag tag, hipStream_t s)
{
    switch (p->dtype) {
    case FFTCONV_F32: return launch_kf_taps<2>(p, k, Nk, adjoint, keep_dev, n_blocks, kf, KfTag{}, s);
    case FFTCONV_F16: return launch_kf_taps<1>(p, k, Nk, adjoint, keep_dev, n_blocks, kf, tag, s);
    default: return launch_kf_taps<0>(p, k, Nk, adjoint, keep_dev, n_blocks, kf, tag, s);
    }
}
// Filters of n blocks of taps that take it.  Where few workgroups would add many blocks up, one after another, an outer pass is faster, us from an outer pass -> so:
// one channel of 65536 taps, fp32 12.2 -> 12.9, bf16 11.8 -> 11.7, 8 of fft 65536 fp32 12.9 -> 13.3, bf16 13.9 -> 13.8; of 131072, fft 131072, 12.6 -> 15.2; 10 of
// 65536 14.6 -> 12.5, 20 of 131072 19.8 -> 16.9, 40 fp32 26.7 -> 24.9, 256 of 65536 bf16 95 -> 61; 768 of 32768 151 -> 95, 768 of 16384 fp32 109 -> 51.
// Those are calls one after another; in a training step other kernels have put the sums' constants out of the L2s, and each block waits for its own: 131072 taps,
// with 96 MB copied between calls, bf16 15 / 24 / 32 / 40 channels 0.84, 0.92, 1.00, 1.04 times as fast as an outer pass (98304 taps 0.95, 1.04, 1.11; fft 65536 8 / 16 /
// 24 of 65536 0.95, 0.96, 1.04), a training step of 1 x 16 x 131072 104.6 -> 108.9.  The lines of 16-bit plans are those of such steps; fp32 plans keep the
// earlier one beyond 8 blocks (15 of 131072 0.87), as their convolutions go on load from there on, and with a spectrum from an outer pass an odd batch of those
// would be 3 % less accurate than in pairs (3.90e-7, 3.79e-7).
// The workgroups take the same number of blocks each, 512 a round, and beyond 10 blocks of taps a second or third round of few costs more than the pass: 131072 taps,
// bf16, 56 channels 26.6 -> 24.0, 57 29.0 -> 36.7, 85 36.5 -> 39.1, 97 41.9 -> 39.6, 128 51.0 -> 55.7, 160 65.3 -> 59.5, fp32 57 33.8 -> 42.9, 117 58 -> 62, 125 66 -> 62; 98304
// taps 57 28.4 -> 33.7, 72 33.2 -> 32.1, fp32 114 55.2 -> 53.7; 81920 57 30.0 -> 29.3.
bool filter_on_load(int64_t A, int64_t n, int64_t H, bool f32)
{
    const int64_t blocks = H * (A / 2 + 1), rounds = (blocks + 511) / 512, last = blocks - 512 * (rounds - 1), turns = (n + 1) / 2;
    if (!outer_on_load(A)) return false;
    if (n <= 4) return true;
    if (n <= 6) return blocks >= 40;
    if (n <= 8) return blocks >= (!f32 ? 108 : A == 8 ? 100 : 54);
    if (blocks < (f32 ? 128 : 128 + 60 * (turns - 5))) return false;
    return n <= 10 || rounds == 1 || rounds > 3 || last >= (rounds == 2 ? 120 * (turns - 5) : f32 ? 70 * (turns - 7) : 110 * (turns - 5));
}
bool long_filter_on_load(const fftconv_plan *p, int64_t Nk)
{
    return filter_on_load(p->M / LB, (Nk + LB - 1) / LB, p->H, p->dtype == FFTCONV_F32);
}

// The filter transform of channels [h0, h0 + nh) of a plan that keeps k_f as fp32 pairs (fp32 I/O, fft_size 32768 .. 2^21): the real outer pass and the block
// transforms of the rows ko <= A/2.  tmp holds nh * (A/2 + 1) * 8192 float2.  Needs multipass_filter_outer_ok(p).
int long_filter_transform_f32(const fftconv_plan *p, const float *k, int64_t Nk, int64_t h0, int64_t nh, bool adjoint,
                              const uint8_t *keep_dev, int64_t n_blocks, float2 *tmp, void *kf, hipStream_t s)
{
    const LongGeo g = long_geo(p->M);
    FC_TRY(multipass_filter_outer(p, outer_rows(k), FFTCONV_F32, Nk, nh, tmp, s));
    return launch_kf<2>(p, g, nh, tmp, kf, h0, keep_dev, n_blocks, true, adjoint, KfTag{}, s);
}

// The position order of the spectra of these transforms (k_f of the fp32 plans from fft_size 32768 up is stored in it)
FacList long_fft_factor_list(int64_t M) { return long_geo(M).fl; }

size_t long_forward_workspace_bytes(const fftconv_plan *p, int64_t B, bool least)
{
    return p->M <= 2 * LB ? 0 : (size_t)(least ? conv_least(p) : conv_pairs(p, B)) * sizeof(float2);
}

// forward pass of the fp32 plans from fft_size 32768 up; kf: (H, fft_size) fp32 pairs in position order; least: the workspace
// holds only long_forward_workspace_bytes(p, B, true)
int long_forward(const fftconv_plan *p, const void *u, const void *kf, void *y, int64_t B, void *workspace, bool least, hipStream_t s,
                 const void *wg, const void *vg)
{
    return long_forward_t<float>(p, (const float *)u, (const float2 *)kf, (float *)y, B, workspace,
                                 least ? conv_least(p) : conv_pairs(p, B), s, (const float *)wg, (const float *)vg);
}

// enough for every smaller batch
size_t long_backward_filter_bytes(const fftconv_plan *p, int64_t B)
{
    if (!multipass_filter_outer_ok(p)) return (size_t)(3 * p->H * p->M) * sizeof(float2);
    const int64_t row = (p->M / LB / 2 + 1) * LB, fit = grad_rows(p);
    return (size_t)(2 * B < fit / p->H ? 2 * B * p->H * row : fit * row) * sizeof(float2);
}

int long_backward_filter(const fftconv_plan *p, const void *u, const void *dy, float *dk, int64_t Nk, int64_t B,
                         void *workspace, hipStream_t s)
{
    switch (p->dtype) {
    case FFTCONV_F32: return long_backward_filter_t<float>(p, (const float *)u, (const float *)dy, dk, Nk, B, workspace, s);
    case FFTCONV_F16:
        return long_backward_filter_t<__half>(p, (const __half *)u, (const __half *)dy, dk, Nk, B, workspace, s);
    default:
        return long_backward_filter_t<__hip_bfloat16>(p, (const __hip_bfloat16 *)u, (const __hip_bfloat16 *)dy, dk, Nk, B,
                                                      workspace, s);
    }
}

}  // namespace fftconv
