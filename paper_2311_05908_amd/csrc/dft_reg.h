// In-register DFTs of power-of-two length <= 32 on the vector ALUs, shared by the outer passes of the
// multi-pass path, the small-transform kernel (fp32) and the generic per-stage kernels (fp32, fp64).
#pragma once

#include <hip/hip_runtime.h>

namespace fftconv {

// cos / sin of 2 pi j / 32: every twiddle of the transforms below
__device__ constexpr float C32[32] = {1.000000000f, 0.980785280f, 0.923879533f, 0.831469612f, 0.707106781f, 0.555570233f, 0.382683432f, 0.195090322f, 0.000000000f, -0.195090322f, -0.382683432f, -0.555570233f, -0.707106781f, -0.831469612f, -0.923879533f, -0.980785280f, -1.000000000f, -0.980785280f, -0.923879533f, -0.831469612f, -0.707106781f, -0.555570233f, -0.382683432f, -0.195090322f, -0.000000000f, 0.195090322f, 0.382683432f, 0.555570233f, 0.707106781f, 0.831469612f, 0.923879533f, 0.980785280f};
__device__ constexpr float S32[32] = {0.000000000f, 0.195090322f, 0.382683432f, 0.555570233f, 0.707106781f, 0.831469612f, 0.923879533f, 0.980785280f, 1.000000000f, 0.980785280f, 0.923879533f, 0.831469612f, 0.707106781f, 0.555570233f, 0.382683432f, 0.195090322f, 0.000000000f, -0.195090322f, -0.382683432f, -0.555570233f, -0.707106781f, -0.831469612f, -0.923879533f, -0.980785280f, -1.000000000f, -0.980785280f, -0.923879533f, -0.831469612f, -0.707106781f, -0.555570233f, -0.382683432f, -0.195090322f};

// the first half in double precision, for the fp64 filter transform
__device__ constexpr double C32D[16] = {1.0, 0.9807852804032304, 0.9238795325112867, 0.8314696123025452, 0.7071067811865476, 0.5555702330196023, 0.38268343236508984, 0.19509032201612833, 0.0, -0.1950903220161282, -0.3826834323650897, -0.555570233019602, -0.7071067811865475, -0.8314696123025453, -0.9238795325112867, -0.9807852804032304};
__device__ constexpr double S32D[16] = {0.0, 0.19509032201612825, 0.3826834323650898, 0.5555702330196022, 0.7071067811865475, 0.8314696123025452, 0.9238795325112867, 0.9807852804032304, 1.0, 0.9807852804032304, 0.9238795325112867, 0.8314696123025455, 0.7071067811865476, 0.5555702330196022, 0.3826834323650899, 0.1950903220161286};

constexpr int bitrev(int v, int bits)
{
    int r = 0;
    for (int i = 0; i < bits; ++i) r |= ((v >> i) & 1) << (bits - 1 - i);
    return r;
}
constexpr int ilog2(int v) { return v <= 1 ? 0 : 1 + ilog2(v / 2); }

// In-register DFT of length R (power of two <= 32), natural order in and out, unnormalised;
// INV conjugates the kernel.  Radix-2 decimation in time, fully unrolled so every index and
// twiddle is a compile-time constant.  A butterfly with a twiddle is eight fused operations, a + w b and
// a - w b as two chained multiply-adds per part each; SIX: six, the difference as 2 a - (a + w b), which carries the
// rounding of the sum (4 % more error of a transform); PRODUCT: eight, w b first, then sum and difference in the place of its
// operands (for kernels that are out of registers).  Those with w = 1 or -+i are four additions, those with odd powers of W_8,
// c (+-1 +-i), two additions and four multiply-adds, whichever the form (SIX has no more itself).  HALFIN: the inputs x[R/2 ..] are zero (the padding of a
// causal convolution) and are not read; the first level of butterflies then only copies.
enum Butterfly { EIGHT, SIX, PRODUCT };
template <int R, bool INV, bool HALFIN = false, Butterfly FORM = EIGHT> __device__ __forceinline__ void dft_reg(float2 (&x)[R])
{
    constexpr int LG = ilog2(R);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int j = bitrev(i, LG);
        if (j > i) {
            const float2 t = x[i];
            x[i] = x[j];
            x[j] = t;
        }
    }
    if constexpr (HALFIN && R >= 2) {
#pragma unroll
        for (int blk = 0; blk < R; blk += 2) x[blk + 1] = x[blk];
    }
#pragma unroll
    for (int len = HALFIN ? 4 : 2; len <= R; len *= 2) {
#pragma unroll
        for (int blk = 0; blk < R; blk += len) {
#pragma unroll
            for (int j = 0; j < len / 2; ++j) {
                const int q = j * (32 / len);                  // twiddle W_32^q, 0 <= q < 16
                const float2 a = x[blk + j], b = x[blk + j + len / 2];
                if ((q == 4 || q == 12) && FORM != SIX) {
                    // W_8^1, W_8^3: (forward) c (b.x + b.y), c (b.y - b.x) with c = cos(pi/4), and the first of them negative at W_8^3
                    const float s = INV ? b.x - b.y : b.x + b.y, d = INV ? b.x + b.y : b.y - b.x;
                    const float cs = C32[4];
                    const float2 t = q == 4 ? make_float2(s, d) : INV ? make_float2(-d, s) : make_float2(d, -s);
                    x[blk + j] = make_float2(__builtin_fmaf(cs, t.x, a.x), __builtin_fmaf(cs, t.y, a.y));
                    x[blk + j + len / 2] = make_float2(__builtin_fmaf(-cs, t.x, a.x), __builtin_fmaf(-cs, t.y, a.y));
                } else if (q == 0 || q == 8 || FORM == PRODUCT) {     // 1; -i forward, +i inverse
                    const float wr = C32[q], wi = INV ? S32[q] : -S32[q];
                    const float2 t = q == 0   ? b
                                     : q == 8 ? (INV ? make_float2(-b.y, b.x) : make_float2(b.y, -b.x))
                                              : make_float2(b.x * wr - b.y * wi, b.x * wi + b.y * wr);
                    x[blk + j] = make_float2(a.x + t.x, a.y + t.y);
                    x[blk + j + len / 2] = make_float2(a.x - t.x, a.y - t.y);
                } else {
                    const float wr = C32[q];
                    const float wi = INV ? S32[q] : -S32[q];
                    const float sx = __builtin_fmaf(-b.y, wi, __builtin_fmaf(b.x, wr, a.x));
                    const float sy = __builtin_fmaf(b.y, wr, __builtin_fmaf(b.x, wi, a.y));
                    const float dx = FORM == SIX ? __builtin_fmaf(2.f, a.x, -sx) : __builtin_fmaf(b.y, wi, __builtin_fmaf(-b.x, wr, a.x));
                    const float dy = FORM == SIX ? __builtin_fmaf(2.f, a.y, -sy) : __builtin_fmaf(-b.y, wr, __builtin_fmaf(-b.x, wi, a.y));
                    x[blk + j] = make_float2(sx, sy);
                    x[blk + j + len / 2] = make_float2(dx, dy);
                }
            }
        }
    }
}

// The forward transform of real inputs, the imaginary parts of x, which are not read.  The halves that a level puts together are spectra of real
// sequences, x[len - k] = conj x[k]: of its butterflies (of eight operations) a quarter's worth and one are worked out, the others are mirror images, the same
// values to the bit.  32 points with zeros in the upper half: 170 operations instead of 370.
// (a level to an instance: as a loop over them the compiler gives up on unrolling it)
template <int R, int LEN> __device__ __forceinline__ void dft_real_level(float2 (&x)[R])
{
    constexpr int h = LEN / 2;
#pragma unroll
    for (int blk = 0; blk < R; blk += LEN) {
#pragma unroll
        for (int j = 0; j <= LEN / 4; ++j) {
            const int q = j * (32 / LEN);                      // twiddle W_32^q, q <= 8
            const float2 a = x[blk + j], b = x[blk + j + h];
            if (q == 0) {
                x[blk] = make_float2(a.x + b.x, 0.f);
                x[blk + h] = make_float2(a.x - b.x, 0.f);
            } else if (q == 8) {
                x[blk + j] = make_float2(a.x, -b.x);
                x[blk + j + h] = make_float2(a.x, b.x);
            } else {
                float2 p, m;
                if (q == 4) {
                    const float cs = C32[4], tx = b.x + b.y, ty = b.y - b.x;
                    p = make_float2(__builtin_fmaf(cs, tx, a.x), __builtin_fmaf(cs, ty, a.y));
                    m = make_float2(__builtin_fmaf(-cs, tx, a.x), __builtin_fmaf(-cs, ty, a.y));
                } else {
                    const float wr = C32[q], wi = -S32[q];
                    p = make_float2(__builtin_fmaf(-b.y, wi, __builtin_fmaf(b.x, wr, a.x)), __builtin_fmaf(b.y, wr, __builtin_fmaf(b.x, wi, a.y)));
                    m = make_float2(__builtin_fmaf(b.y, wi, __builtin_fmaf(-b.x, wr, a.x)), __builtin_fmaf(-b.y, wr, __builtin_fmaf(-b.x, wi, a.y)));
                }
                x[blk + j] = p;
                x[blk + h + j] = m;
                x[blk + LEN - j] = make_float2(p.x, -p.y);
                x[blk + h - j] = make_float2(m.x, -m.y);
            }
        }
    }
    if constexpr (LEN < R) dft_real_level<R, 2 * LEN>(x);
}
template <int R, bool HALFIN = false> __device__ __forceinline__ void dft_real(float2 (&x)[R])
{
    constexpr int LG = ilog2(R);
    static_assert(R >= 4, "a quarter");
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int j = bitrev(i, LG);
        if (j > i) {
            const float t = x[i].x;
            x[i].x = x[j].x;
            x[j].x = t;
        }
    }
#pragma unroll
    for (int blk = 0; blk < R; blk += 2) {
        const float a = x[blk].x, b = x[blk + 1].x;
        x[blk] = make_float2(HALFIN ? a : a + b, 0.f);
        x[blk + 1] = make_float2(HALFIN ? a : a - b, 0.f);
    }
    dft_real_level<R, 4>(x);
}

// The transform of 32 points as 4 x 8, or of 16 as 4 x 4, the twiddles W_R^{j k} between the two products of their own: x[j + R/4 a] over a,
// times W_R^{j k}, then over j; frequency k + 4 m.  As many operations as the radix-2 form above with eight a butterfly, and half
// as many roundings on a path (32 points: 1.2 levels of products instead of 2.1).
template <int R, bool INV, bool HALFIN> __device__ __forceinline__ void dft_4xn(float2 (&x)[R])
{
    constexpr int Q = R / 4;
    float2 t[4][Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        float2 v[4] = {x[j], x[j + Q], x[j + 2 * Q], x[j + 3 * Q]};
        dft_reg<4, INV, HALFIN>(v);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int q = j * k * (32 / R);                    // 0 .. 21
            const float wr = C32[q], wi = INV ? S32[q] : -S32[q];
            if (q == 0) t[k][j] = v[k];
            else if (q == 8) t[k][j] = INV ? make_float2(-v[k].y, v[k].x) : make_float2(v[k].y, -v[k].x);
            else t[k][j] = make_float2(__builtin_fmaf(-v[k].y, wi, v[k].x * wr), __builtin_fmaf(v[k].y, wr, v[k].x * wi));
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        dft_reg<Q, INV>(t[k]);
#pragma unroll
        for (int m = 0; m < Q; ++m) x[k + 4 * m] = t[k][m];
    }
}

// The same transform in double precision.
template <int R, bool INV> __device__ __forceinline__ void dft_reg(double2 (&x)[R])
{
    constexpr int LG = ilog2(R);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int j = bitrev(i, LG);
        if (j > i) {
            const double2 t = x[i];
            x[i] = x[j];
            x[j] = t;
        }
    }
#pragma unroll
    for (int len = 2; len <= R; len *= 2) {
#pragma unroll
        for (int blk = 0; blk < R; blk += len) {
#pragma unroll
            for (int j = 0; j < len / 2; ++j) {
                const int q = j * (32 / len);                  // twiddle W_32^q, 0 <= q < 16
                const double2 a = x[blk + j], b = x[blk + j + len / 2];
                if (q == 4 || q == 12) {
                    const double s = INV ? b.x - b.y : b.x + b.y, d = INV ? b.x + b.y : b.y - b.x;
                    const double cs = C32D[4];
                    const double2 t = q == 4 ? make_double2(s, d) : INV ? make_double2(-d, s) : make_double2(d, -s);
                    x[blk + j] = make_double2(__builtin_fma(cs, t.x, a.x), __builtin_fma(cs, t.y, a.y));
                    x[blk + j + len / 2] = make_double2(__builtin_fma(-cs, t.x, a.x), __builtin_fma(-cs, t.y, a.y));
                    continue;
                }
                double2 t;
                if (q == 0) {
                    t = b;
                } else if (q == 8) {                           // -i forward, +i inverse
                    t = INV ? make_double2(-b.y, b.x) : make_double2(b.y, -b.x);
                } else {
                    const double wr = C32D[q];
                    const double wi = INV ? S32D[q] : -S32D[q];
                    t = make_double2(b.x * wr - b.y * wi, b.x * wi + b.y * wr);
                }
                x[blk + j] = make_double2(a.x + t.x, a.y + t.y);
                x[blk + j + len / 2] = make_double2(a.x - t.x, a.y - t.y);
            }
        }
    }
}

}  // namespace fftconv
