// One row ko of the outer factor of a transform of fft_size = A * 8192 points, formed in the registers of the row engine
// while its samples are loaded: what a kernel for the outer factor would write for all rows, and the block kernel read again.
//
// Samples n = 8192 no + r of a real row, r = j + 256 m as thread j of a row of 8192 points holds them in register m:
//   X_ko[r] = W_M^{r ko} sum_no x[8192 no + r] W_A^{no ko} = W_M^{j ko} sum_no x[8192 no + r] W_{32 A}^{ko (32 no + m)}.
// The constants of the sum are the same in all threads (scalar registers), each correct to its own rounding; the factor in front is the
// same in all registers of a thread and rides on the twiddles of its first pass (rf::twiddle_times()).  That is two multiply-adds for a
// real sample and row ko, where a transform for all rows at once takes a few for a point, but the samples of a row reach the A/2 + 1 workgroups of
// its rows ko from one L2 (they are on one die), and the rows, of fp32 pairs, are neither written nor read: a filter transform of 256 channels of fft 131072
// moves 0.2 GB instead of 0.5 (95 -> 61 us, 76 in a training step), a gradient of 2 x 256 x 65536 bf16 samples 0.5 instead of 1.7 (364 -> 280 us; vector instructions at four
// cycles each are 220 of them now).  Fewer roundings, too: the gradient's error 4.33e-7 -> 3.67e-7.  At A = 32 the sums cost what the trip does (filter 128
// channels of fft 2^18 bf16 105 -> 88 us, but 64 fp32 60 -> 62, gradient 205 -> 229), at 64 twice that.
#pragma once

#include <hip/hip_runtime.h>

#include "row_io.h"

namespace fftconv {

// Tables of a plan (long_fft_init()): sum constants [ko][no][m] of the rows ko <= A/2, no < A, m < 32, then the factors
// W_M^{j ko}, [ko][j], j < 256.
constexpr int OUTER_M = 32, OUTER_T = 256, OUTER_LB = 8192;
__host__ __device__ constexpr int outer_tab_sums(int A) { return (A / 2 + 1) * A * OUTER_M; }
__host__ __device__ constexpr int outer_tab_size(int A) { return outer_tab_sums(A) + (A / 2 + 1) * OUTER_T; }

// A real row of `len` samples.  They come in units of U registers m of a block no (U = 32: a whole block), two units in flight; samples at
// and beyond len read as zeros (the buffer's bounds check: no load behind a branch).
// GATED (fp32): times the samples of `gate`, which lies alike.
template <typename IO, int U, bool GATED = false> struct OuterRow {
    static_assert(!GATED || sizeof(IO) == 4, "gates of 16-bit rows are rounded");
    static constexpr int PARTS = OUTER_M / U, SIZE = sizeof(IO);
    const IO *row;
    int len;
    const IO *gate = nullptr;
    struct Units { uint32_t a[U], b[U], ga[GATED ? U : 1], gb[GATED ? U : 1]; };

    __device__ __forceinline__ int blocks() const { return (len + OUTER_LB - 1) / OUTER_LB; }
    // (the descriptor of a block, not an offset from the row's: no register offset takes part in the bounds check)
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t block(const IO *row, int no) const
    {
        const int first = no * OUTER_LB, left = len > first ? len - first : 0;
        return __builtin_amdgcn_make_buffer_rsrc((void *)(row + (left ? first : 0)), 0, left * SIZE, 0x00020000);
    }
    __device__ __forceinline__ void fetch(uint32_t (&w)[U], const IO *row, int unit, int at) const
    {
        at += unit % PARTS * U * OUTER_T * SIZE;
        const auto r = block(row, unit / PARTS);
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int o = at + i * OUTER_T * SIZE;
            if constexpr (SIZE == 4) w[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0);
            else w[i] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, o, 0, 0);
        }
    }
    __device__ __forceinline__ void fetch(Units &w, int tid) const
    {
        fetch(w.a, row, 0, tid * SIZE);
        if constexpr (GATED) fetch(w.ga, gate, 0, tid * SIZE);
        fetch(w.b, row, 1, tid * SIZE);
        if constexpr (GATED) fetch(w.gb, gate, 1, tid * SIZE);
    }
    // x[m0 + m] += a unit's samples times its constants, m < U
    static __device__ __forceinline__ void add(float2 (&x)[OUTER_M], const uint32_t (&w)[U], const uint32_t (&g)[GATED ? U : 1], int m0,
                                               const float2 *c)
    {
#pragma unroll
        for (int m = 0; m < U; ++m) {
            float v;
            if constexpr (SIZE == 4) v = __uint_as_float(w[m]);
            else v = rf::unpack<IO>(w[m]).x;
            if constexpr (GATED) v *= __uint_as_float(g[m]);
            x[m0 + m].x = __builtin_fmaf(v, c[m].x, x[m0 + m].x);
            x[m0 + m].y = __builtin_fmaf(v, c[m].y, x[m0 + m].y);
        }
    }
    // x[m] = the sum over no, its first two units in w; sums: the constants of row ko.  On return w holds the first two of `next`.
    // A unit is asked for when the one in its registers has been used (the fences; else the compiler asks first, into
    // others, and waits for all of them at the end of a turn to move them).
    __device__ __forceinline__ void sum(float2 (&x)[OUTER_M], Units &w, const float2 *__restrict__ sums, const OuterRow &next, int tid) const
    {
        int at = tid * SIZE;
        auto fence = [&](int m0) {
#pragma unroll
            for (int m = 0; m < U; ++m) asm volatile("" : "+v"(at) : "v"(x[m0 + m].x), "v"(x[m0 + m].y));
        };
#pragma unroll
        for (int m = 0; m < OUTER_M; ++m) x[m] = make_float2(0.f, 0.f);
        const int turns = PARTS == 2 ? blocks() : (blocks() + 1) / 2;       // (an odd last block's partner is zeros)
#pragma unroll 1
        for (int i = 0; i < turns; ++i) {
            const bool more = i + 1 < turns;
            const OuterRow from = more ? *this : next;
            const int unit = more ? 2 * i + 2 : 0;
            const float2 *const c = sums + i * 2 * U;
            add(x, w.a, w.ga, 0, c);
            fence(0);
            from.fetch(w.a, from.row, unit, at);
            if constexpr (GATED) from.fetch(w.ga, from.gate, unit, at);
            constexpr int m1 = PARTS == 2 ? U : 0;
            add(x, w.b, w.gb, m1, c + U);
            fence(m1);
            from.fetch(w.b, from.row, unit + 1, at);
            if constexpr (GATED) from.fetch(w.gb, from.gate, unit + 1, at);
        }
    }
};

}  // namespace fftconv
