// fp32 transforms of whole rows of M = 256 .. 16384 complex points, two or three passes of in-register
// butterflies (dft_reg.h) with one exchange through LDS between passes: the engine of the kernels that compute
// in fp32 (short and fp32 convolutions, filter transforms, filter gradients).
//
// M = R0 R1 R2 (R2 = 1: two passes).  T = M / R0 threads hold a row, R0 points each; time n = j + (M / R0) m:
//   pass 0: thread j < T transforms m (radix R0, stride T) straight from where its caller loaded the samples,
//           times W_M^{j k0};
//   pass 1: in every block k0 of L1 = T positions, radix R1 at stride S1 = L1 / R1, times W_L1^{j1 k1}, j1 < S1;
//   pass 2: radix R2 over adjacent positions, no twiddles.
// The last pass leaves frequency f = k0 + R0 k1 + R0 R1 k2 in registers (freq() below names it), where the caller
// multiplies, stores or accumulates; the inverse runs the mirrored passes (conjugate twiddles before the
// butterflies) and returns sample j + T m in x[m].  A complete convolution therefore makes four trips through LDS
// (two with two passes) and touches every sample and every bin once in registers.  Every position is written by
// the thread that read it last, so one barrier per exchange suffices; rows of up to 64 threads live inside one wave
// and need none (LDS operations of a wave complete in order).
//
// What bounds these kernels is the vector ALU (about 110 operations per point and convolution at M = 8192), so
//  * radices 32 and 16 (fewest twiddle products and exchanges that 64 data registers allow);
//  * twiddles come from tables in thread order, [factor][thread] (gathers from a table of W_M^t, one cache line per lane,
//    bounded the kernels that this file replaces).
// FINE: radix-32 butterflies as 4 x 8, radix-16 ones as 4 x 4 (dft_4xn()), see row_grad.hip.
// Two kinds of row.  EXACT: all R - 1 twiddles of a butterfly come from the table, each correct to its own rounding, and the
// in-register butterflies take eight operations.  Otherwise the table holds those for 1, 2, 3 and the multiples of 4, the
// others are products of them, and butterflies take six: a tenth more error of a transform, and at fft 1024 68 us
// instead of 79 for 201 MB of rows.  Exact are convolutions with fp32 I/O up to fft 4096 and filter gradients up to 16384 that run
// on whole rows (row_grad.hip), so that they are no less accurate than kernels with a gather for every twiddle.  The others are
// not, and still no less accurate than what they replace: 16-bit results, and dk accumulated from 16-bit operands, do not show
// the difference (the same error to four digits); fp32 convolutions of 8192 and 16384 points measure 5 - 12 % below the four and more
// passes before, those beyond 3 - 12 %, filter gradients beyond 16384 points 2 - 8 % (fft 131072: dk 4.70e-7 -> 4.39e-7).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "dft_reg.h"
#include "fused3_common.h"

namespace fftconv {
namespace rf {

template <int M, bool WIDE = false> struct Radix;
template <> struct Radix<256> { static constexpr int R0 = 16, R1 = 16, R2 = 1; };
template <> struct Radix<512> { static constexpr int R0 = 32, R1 = 16, R2 = 1; };
template <> struct Radix<1024> { static constexpr int R0 = 32, R1 = 32, R2 = 1; };
template <> struct Radix<2048> { static constexpr int R0 = 16, R1 = 16, R2 = 8; };
template <> struct Radix<4096> { static constexpr int R0 = 16, R1 = 16, R2 = 16; };
template <> struct Radix<8192> { static constexpr int R0 = 32, R1 = 16, R2 = 16; };
template <> struct Radix<16384> { static constexpr int R0 = 32, R1 = 32, R2 = 16; };
// WIDE rows: a wave each, 8 or 16 points a thread and a trip through LDS more, for calls of few rows: the instructions of a thread one after the
// other are the time there (16 pairs of rows: fp32 fft 512 7.4 -> 5.0 us, 1024 8.0 -> 5.4; 16 . 8 . 8 instead, 5.7).
template <> struct Radix<512, true> { static constexpr int R0 = 8, R1 = 8, R2 = 8; };
template <> struct Radix<1024, true> { static constexpr int R0 = 16, R1 = 4, R2 = 16; };

// number of twiddles of a radix-R pass that come from the table, all or 1, 2, 3, 4, 8, 12, .., and their powers
constexpr int tw_count(int R, bool exact) { return exact ? R - 1 : R / 4 + 2; }
constexpr int tw_power(int i, bool exact) { return exact || i < 3 ? i + 1 : 4 * (i - 2); }

template <int M_, bool EXACT_ = false, bool FINE_ = false, bool WIDE_ = false> struct Row {
    static constexpr int M = M_;
    static constexpr bool EXACT = EXACT_, FINE = FINE_, WIDE = WIDE_;
    static constexpr int R0 = Radix<M, WIDE>::R0, R1 = Radix<M, WIDE>::R1, R2 = Radix<M, WIDE>::R2;
    static constexpr int P = R0;                           // points per thread
    static constexpr int T = M / R0;                       // threads per row
    static constexpr bool THREE = R2 > 1;
    static constexpr int RL = THREE ? R2 : R1;             // radix of the last pass
    static constexpr int S1 = R2;                          // stride of pass 1 (three passes)
    static constexpr int NB1 = P / R1, NBL = P / RL;       // butterflies per thread of pass 1, of the last pass
    static constexpr int TW0 = tw_count(R0, EXACT), TW1 = THREE ? tw_count(R1, EXACT) : 0;
    static constexpr int TABLE = TW0 * T + (THREE ? TW1 * S1 : 0);         // entries of the twiddle table
    // LDS slot of position blk * T + sub * RL + r (r < RL, sub < T / RL): one word pair of padding per RL positions
    // spreads the last pass (lanes RL positions apart) over the banks; where blocks of T positions would still start
    // at the same bank, 16 more per block.
    static constexpr int PAD = RL + 1;                     // distance of two runs of RL positions
    static constexpr int PITCH = T / RL * PAD + ((THREE && (T / RL * PAD * 2) % 64 == 0) ? 16 : 0);   // ... of two blocks
    // rows of up to 64 threads: real and imaginary parts go through LDS one after the other, in half the space
    static constexpr bool SPLIT = !THREE && T <= 64;
    static constexpr int SLOTS = R0 * PITCH + (SPLIT && R0 * PITCH % 64 == 32 && T == 16 ? 16 : 0);
    static constexpr int LDS_BYTES = SLOTS * (SPLIT ? 4 : 8);
    static_assert(T % RL == 0, "blocks hold whole runs");
    static __device__ __forceinline__ int slot0(int j) { return j / RL * PAD + j % RL; }              // position j < T
    // first slot of butterfly bi of pass 1 (its points are PAD slots apart) and of the last pass (adjacent slots)
    static __device__ __forceinline__ int slot1(int bi) { return bi / S1 * PITCH + bi % S1; }
    static __device__ __forceinline__ int slotl(int bi) { return bi / (T / RL) * PITCH + bi % (T / RL) * PAD; }
    // frequency held in register p = i * RL + r after forward() (butterfly i of the last pass, digit r)
    static __host__ __device__ __forceinline__ int freq(int tid, int p)
    {
        const int bi = tid + T * (p / RL), r = p % RL;
        if constexpr (THREE) return bi / R1 + R0 * (bi % R1) + R0 * R1 * r;
        else return bi + R0 * r;
    }
    // place of frequency f in register order, [register pair][thread][2]
    static __host__ __device__ __forceinline__ int index(int f)
    {
        const int bi = THREE ? f % R0 * R1 + f / R0 % R1 : f % R0, r = THREE ? f / (R0 * R1) : f / R0, p = bi / T * RL + r;
        return (p / 2 * T + bi % T) * 2 + p % 2;
    }
};

__device__ __forceinline__ float2 mul(float2 a, float2 b)
{
    return make_float2(__builtin_fmaf(-a.y, b.y, a.x * b.x), __builtin_fmaf(a.y, b.x, a.x * b.y));
}
__device__ __forceinline__ float2 mul_conj(float2 a, float2 b)     // a * conj(b)
{
    return make_float2(__builtin_fmaf(a.y, b.y, a.x * b.x), __builtin_fmaf(a.y, b.x, -(a.x * b.y)));
}

// x[k] *= W^k (CONJ: its conjugate), k < R, from the products of the tw_count(R) table entries t
template <int R, bool CONJ> __device__ __forceinline__ void twiddle(float2 (&x)[R], const float2 (&t)[tw_count(R, false)])
{
#pragma unroll
    for (int k = 1; k < R; ++k) {
        const int a = k / 4, b = k % 4;
        const float2 w = a == 0 ? t[b - 1] : b == 0 ? t[a + 2] : mul(t[a + 2], t[b - 1]);
        x[k] = CONJ ? mul_conj(x[k], w) : mul(x[k], w);
    }
}
// x[k] *= w W^k, k < R: the factor rides on the products of the table's entries
template <int R> __device__ __forceinline__ void twiddle_times(float2 (&x)[R], const float2 (&t)[tw_count(R, false)], float2 w)
{
#pragma unroll
    for (int a = 0; a < R / 4; ++a) {
        const float2 wa = a == 0 ? w : mul(t[a + 2], w);
        x[4 * a] = mul(x[4 * a], wa);
#pragma unroll
        for (int b = 1; b < 4; ++b) x[4 * a + b] = mul(x[4 * a + b], mul(wa, t[b - 1]));
    }
}
// x[k] *= W^k, W^k = tab[(k - 1) * stride], at most 16 of them in registers at a time
template <int R, bool CONJ> __device__ __forceinline__ void twiddle_exact(float2 (&x)[R], const float2 *tab, int stride)
{
#pragma unroll
    for (int k0 = 0; k0 < R; k0 += 16) {
        if (k0 > 0) asm volatile("" : "+v"(tab) : "v"(x[k0 - 1].x), "v"(x[k0 - 1].y));
        float2 t[16];
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (k0 + k > 0 && k0 + k < R) t[k] = tab[(k0 + k - 1) * stride];
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (k0 + k > 0 && k0 + k < R) x[k0 + k] = CONJ ? mul_conj(x[k0 + k], t[k]) : mul(x[k0 + k], t[k]);
    }
}

// The exchanges of a row whose threads span several waves meet at a workgroup barrier; a row inside one wave
// only has to keep the compiler from moving LDS accesses across.
template <int T> __device__ __forceinline__ void row_barrier()
{
    if constexpr (T > 64) f3::lds_barrier();
    else asm volatile("" ::: "memory");
}

// The twiddles of pass 1, the same for every butterfly of a thread (its position inside a block does not change):
// in registers, or where to read them.
template <typename G> struct Tw1 {
    float2 t[G::THREE && !G::EXACT ? G::TW1 : 1];
    const float2 *p;
    __device__ __forceinline__ void load(const float2 *__restrict__ tab, int tid)
    {
        p = tab + G::TW0 * G::T + tid % G::S1;
        if constexpr (G::THREE && !G::EXACT) {
#pragma unroll
            for (int i = 0; i < G::TW1; ++i) t[i] = p[i * G::S1];
        }
    }
    template <bool CONJ> __device__ __forceinline__ void apply(float2 (&v)[G::R1]) const
    {
        if constexpr (G::EXACT) twiddle_exact<G::R1, CONJ>(v, p, G::S1);
        else twiddle<G::R1, CONJ>(v, t);
    }
};
// The twiddles of pass 0, ready to use: requested by load(), or read by apply() where they are too many to hold
template <typename G> struct Tw0 {
    float2 t[G::EXACT ? 1 : G::TW0];
    const float2 *p;
    __device__ __forceinline__ void load(const float2 *__restrict__ tab, int tid)
    {
        p = tab + tid;
        if constexpr (!G::EXACT) {
#pragma unroll
            for (int i = 0; i < G::TW0; ++i) t[i] = p[i * G::T];
        }
    }
    template <bool CONJ> __device__ __forceinline__ void apply(float2 (&x)[G::R0]) const
    {
        if constexpr (G::EXACT) twiddle_exact<G::R0, CONJ>(x, p, G::T);
        else twiddle<G::R0, CONJ>(x, t);
    }
    // times w, too
    __device__ __forceinline__ void apply_times(float2 (&x)[G::R0], float2 w) const
    {
        if constexpr (G::EXACT) {
            twiddle_exact<G::R0, false>(x, p, G::T);
#pragma unroll
            for (int k = 0; k < G::R0; ++k) x[k] = mul(x[k], w);
        } else {
            twiddle_times<G::R0>(x, t, w);
        }
    }
};
struct NoFactor {};                                           // of forward()

// The exchange of a two-pass row inside one wave: x[k] of column tid <-> x[i * RL + r] of the butterflies of the last pass
// (FWD: first to last pass), one part at a time.
template <typename G, bool FWD> __device__ __forceinline__ void exchange(float2 (&x)[G::P], float *Z, int tid)
{
    float *const z0 = Z + G::slot0(tid);
    auto at = [&](int p) { return Z + G::slotl(tid + G::T * (p / G::RL)) + p % G::RL; };
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
        for (int p = 0; p < G::P; ++p) *(FWD ? z0 + p * G::PITCH : at(p)) = part ? x[p].y : x[p].x;
        row_barrier<G::T>();
#pragma unroll
        for (int p = 0; p < G::P; ++p) (part ? x[p].y : x[p].x) = *(FWD ? at(p) : z0 + p * G::PITCH);
        row_barrier<G::T>();
    }
}

// a butterfly of the row's passes
template <typename G, int R, bool INV, bool HALFIN = false> __device__ __forceinline__ void butterfly(float2 (&x)[R])
{
    if constexpr (G::FINE && R >= 16) dft_4xn<R, INV, HALFIN>(x);
    else dft_reg<R, INV, HALFIN, G::EXACT ? EIGHT : SIX>(x);
}

// Forward transform of the row whose samples j + T m the thread j = tid holds in x[m]; Z: the row's Row<M>::SLOTS
// slots of LDS, free (the caller's barrier lies before).  HALF: x[m] = 0 for m >= R0 / 2.  On return x[p] holds
// frequency freq(tid, p).  before_last() runs ahead of the last pass (loads that whoever uses the result needs).
// factor: every sample of the thread is multiplied by it (a float2; rows of three passes).  REAL: the samples are real, the imaginary parts of x are not read.
template <typename G, bool HALF, bool REAL = false, typename F, typename W = NoFactor>
__device__ __forceinline__ void forward(float2 (&x)[G::P], float2 *Z, const float2 *__restrict__ tab, const Tw1<G> &tw1, int tid,
                                        F before_last, W factor = W())
{
    {
        Tw0<G> t;
        t.load(tab, tid);
        if constexpr (REAL && !(G::FINE && G::R0 >= 16)) dft_real<G::R0, HALF>(x);
        else butterfly<G, G::R0, false, HALF>(x);
        if constexpr (std::is_same<W, NoFactor>::value) t.template apply<false>(x);
        else t.apply_times(x, factor);
    }
    if constexpr (G::SPLIT) {
        before_last();
        exchange<G, true>(x, (float *)Z, tid);
#pragma unroll
        for (int i = 0; i < G::NBL; ++i) {
            float2 v[G::RL];
#pragma unroll
            for (int r = 0; r < G::RL; ++r) v[r] = x[i * G::RL + r];
            butterfly<G, G::RL, false>(v);
#pragma unroll
            for (int r = 0; r < G::RL; ++r) x[i * G::RL + r] = v[r];
        }
        return;
    }
    float2 *const z0 = Z + G::slot0(tid);
#pragma unroll
    for (int k = 0; k < G::R0; ++k) z0[k * G::PITCH] = x[k];
    row_barrier<G::T>();
    if constexpr (G::THREE) {
#pragma unroll
        for (int i = 0; i < G::NB1; ++i) {
            float2 *const z = Z + G::slot1(tid + G::T * i);
            float2 v[G::R1];
#pragma unroll
            for (int m = 0; m < G::R1; ++m) v[m] = z[m * G::PAD];
            butterfly<G, G::R1, false>(v);
            tw1.template apply<false>(v);
#pragma unroll
            for (int k = 0; k < G::R1; ++k) z[k * G::PAD] = v[k];
        }
        before_last();
        row_barrier<G::T>();
    } else {
        before_last();
    }
#pragma unroll
    for (int i = 0; i < G::NBL; ++i) {
        float2 *const z = Z + G::slotl(tid + G::T * i);
        float2 v[G::RL];
#pragma unroll
        for (int r = 0; r < G::RL; ++r) v[r] = z[r];
        butterfly<G, G::RL, false>(v);
#pragma unroll
        for (int r = 0; r < G::RL; ++r) x[i * G::RL + r] = v[r];
    }
}

// Unnormalised inverse of forward(), in the slots that forward() left (no barrier needed between the two).
template <typename G>
__device__ __forceinline__ void inverse(float2 (&x)[G::P], float2 *Z, const float2 *__restrict__ tab, const Tw1<G> &tw1, int tid)
{
#pragma unroll
    for (int i = 0; i < G::NBL; ++i) {
        float2 v[G::RL];
#pragma unroll
        for (int r = 0; r < G::RL; ++r) v[r] = x[i * G::RL + r];
        butterfly<G, G::RL, true>(v);
        if constexpr (G::SPLIT) {
#pragma unroll
            for (int r = 0; r < G::RL; ++r) x[i * G::RL + r] = v[r];
        } else {
            float2 *const z = Z + G::slotl(tid + G::T * i);
#pragma unroll
            for (int r = 0; r < G::RL; ++r) z[r] = v[r];
        }
    }
    if constexpr (G::SPLIT) {
        exchange<G, false>(x, (float *)Z, tid);
        Tw0<G> t;
        t.load(tab, tid);
        t.template apply<true>(x);
        butterfly<G, G::R0, true>(x);
        return;
    }
    row_barrier<G::T>();
    if constexpr (G::THREE) {
#pragma unroll
        for (int i = 0; i < G::NB1; ++i) {
            float2 *const z = Z + G::slot1(tid + G::T * i);
            float2 v[G::R1];
#pragma unroll
            for (int k = 0; k < G::R1; ++k) v[k] = z[k * G::PAD];
            tw1.template apply<true>(v);
            butterfly<G, G::R1, true>(v);
#pragma unroll
            for (int m = 0; m < G::R1; ++m) z[m * G::PAD] = v[m];
        }
        row_barrier<G::T>();
    }
    Tw0<G> t;
    t.load(tab, tid);
    const float2 *const z0 = Z + G::slot0(tid);
#pragma unroll
    for (int k = 0; k < G::R0; ++k) x[k] = z0[k * G::PITCH];
    t.template apply<true>(x);
    butterfly<G, G::R0, true>(x);
}

// Rows of 2048 and 4096 points for calls of few: 8 points a thread, four passes (8 . 8 . 8 . 4 and 8 . 8 . 8 . 8), exact twiddles.  As with wide rows above, the
// instructions of a thread one after the other are the time there, and half as many of them are worth a trip through LDS more each way.  Position p < M
// lies in slot p + p / 8.  Only the first exchange is between waves: the blocks of 8 S1 positions that pass 1 works in, and those of 8 S2 of
// pass 2, belong to as many threads one after another, S1 <= 64 of them.  Frequency f = k0 + 8 k1 + 64 k2 + 512 k3.
template <int M_> struct Quad {
    static constexpr int M = M_, P = 8, R0 = 8, T = M / 8, S1 = T / 8, S2 = S1 / 8, R3 = S2, NB3 = P / R3;
    static_assert(S1 <= 64 && (R3 == 4 || R3 == 8), "2048 or 4096 points");
    static constexpr int TABLE = 7 * (T + S1 + S2), SLOTS = M + M / 8, LDS_BYTES = 8 * SLOTS;
    static __host__ __device__ __forceinline__ int freq(int tid, int p)
    {
        const int b = tid * NB3 + p / R3;
        return b / 64 + 8 * (b / 8 % 8) + 64 * (b % 8) + 512 * (p % R3);
    }
};
// x[k] *= tab[(k - 1) * stride], 0 < k < 8 (CONJ: its conjugate)
template <bool CONJ> __device__ __forceinline__ void twiddle8(float2 (&x)[8], const float2 (&t)[7])
{
#pragma unroll
    for (int k = 1; k < 8; ++k) x[k] = CONJ ? mul_conj(x[k], t[k - 1]) : mul(x[k], t[k - 1]);
}
// The twiddles of a thread's three passes, asked for together
template <typename Q> struct QuadTw {
    float2 t0[7], t1[7], t2[7];
    __device__ __forceinline__ void load(const float2 *__restrict__ tab, int tid)
    {
#pragma unroll
        for (int k = 0; k < 7; ++k) t0[k] = tab[k * Q::T + tid];
#pragma unroll
        for (int k = 0; k < 7; ++k) t1[k] = tab[7 * Q::T + k * Q::S1 + tid % Q::S1];
#pragma unroll
        for (int k = 0; k < 7; ++k) t2[k] = tab[7 * (Q::T + Q::S1) + k * Q::S2 + tid % Q::S2];
    }
};
template <typename Q> struct QuadSlots {                          // first slots of a thread in passes 0 .. 3
    float2 *z0, *z1, *z2, *z3;
    __device__ __forceinline__ QuadSlots(float2 *Z, int tid)
        : z0(Z + tid + tid / 8), z1(Z + 9 * Q::S1 * (tid / Q::S1) + tid % Q::S1 + tid % Q::S1 / 8),
          z2(Z + 9 * Q::S2 * (tid / Q::S2) + tid % Q::S2), z3(Z + 9 * tid) {}
    static constexpr int at(int stride, int m) { return stride * m + stride * m / 8; }
};
// forward() and inverse() of such rows
template <typename Q, bool HALF> __device__ __forceinline__ void quad_forward(float2 (&x)[8], const QuadSlots<Q> &z, const QuadTw<Q> &tw)
{
    using S = QuadSlots<Q>;
    dft_reg<8, false, HALF>(x);
    twiddle8<false>(x, tw.t0);
#pragma unroll
    for (int k = 0; k < 8; ++k) z.z0[S::at(Q::T, k)] = x[k];
    row_barrier<Q::T>();
#pragma unroll
    for (int m = 0; m < 8; ++m) x[m] = z.z1[S::at(Q::S1, m)];
    dft_reg<8, false>(x);
    twiddle8<false>(x, tw.t1);
#pragma unroll
    for (int k = 0; k < 8; ++k) z.z1[S::at(Q::S1, k)] = x[k];
    row_barrier<64>();
#pragma unroll
    for (int m = 0; m < 8; ++m) x[m] = z.z2[S::at(Q::S2, m)];
    dft_reg<8, false>(x);
    twiddle8<false>(x, tw.t2);
#pragma unroll
    for (int k = 0; k < 8; ++k) z.z2[S::at(Q::S2, k)] = x[k];
    row_barrier<64>();
#pragma unroll
    for (int i = 0; i < Q::NB3; ++i) {
        float2 v[Q::R3];
#pragma unroll
        for (int r = 0; r < Q::R3; ++r) v[r] = z.z3[i * Q::R3 + r];
        dft_reg<Q::R3, false>(v);
#pragma unroll
        for (int r = 0; r < Q::R3; ++r) x[i * Q::R3 + r] = v[r];
    }
}
template <typename Q> __device__ __forceinline__ void quad_inverse(float2 (&x)[8], const QuadSlots<Q> &z, const QuadTw<Q> &tw)
{
    using S = QuadSlots<Q>;
#pragma unroll
    for (int i = 0; i < Q::NB3; ++i) {
        float2 v[Q::R3];
#pragma unroll
        for (int r = 0; r < Q::R3; ++r) v[r] = x[i * Q::R3 + r];
        dft_reg<Q::R3, true>(v);
#pragma unroll
        for (int r = 0; r < Q::R3; ++r) z.z3[i * Q::R3 + r] = v[r];
    }
    row_barrier<64>();
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = z.z2[S::at(Q::S2, k)];
    twiddle8<true>(x, tw.t2);
    dft_reg<8, true>(x);
#pragma unroll
    for (int m = 0; m < 8; ++m) z.z2[S::at(Q::S2, m)] = x[m];
    row_barrier<64>();
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = z.z1[S::at(Q::S1, k)];
    twiddle8<true>(x, tw.t1);
    dft_reg<8, true>(x);
#pragma unroll
    for (int m = 0; m < 8; ++m) z.z1[S::at(Q::S1, m)] = x[m];
    row_barrier<Q::T>();
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = z.z0[S::at(Q::T, k)];
    twiddle8<true>(x, tw.t0);
    dft_reg<8, true>(x);
}
template <typename Q, typename W> inline void fill_quad_table(float2 *tab, W w)
{
    auto put = [&](int k, int j, int den) {
        const double2 v = w(k * j % den, den);
        *tab++ = make_float2((float)v.x, (float)v.y);
    };
    for (int k = 1; k < 8; ++k)
        for (int j = 0; j < Q::T; ++j) put(k, j, Q::M);
    for (int k = 1; k < 8; ++k)
        for (int j = 0; j < Q::S1; ++j) put(k, j, Q::T);
    for (int k = 1; k < 8; ++k)
        for (int j = 0; j < Q::S2; ++j) put(k, j, Q::S1);
}

// Host side: the twiddle table of Row<M>, rounded once; w(num, den) = exp(-2 pi i num / den) in fp64, num < den.
template <typename G, typename W> inline void fill_table(float2 *tab, W w)
{
    auto put = [&](float2 *at, int num, int den) {
        const double2 v = w(num % den, den);
        *at = make_float2((float)v.x, (float)v.y);
    };
    for (int i = 0; i < G::TW0; ++i)
        for (int j = 0; j < G::T; ++j) put(tab + i * G::T + j, tw_power(i, G::EXACT) * j, G::M);
    if (G::THREE)
        for (int i = 0; i < G::TW1; ++i)
            for (int j = 0; j < G::S1; ++j) put(tab + G::TW0 * G::T + i * G::S1 + j, tw_power(i, G::EXACT) * j, G::T);
}

}  // namespace rf
}  // namespace fftconv
