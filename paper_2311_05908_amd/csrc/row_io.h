// Samples of the row kernels (row_fft.h): pairs of batch rows of any I/O dtype into the registers of the first pass.
#pragma once

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include <type_traits>

#include "fftconv_internal.h"
#include "row_fft.h"

namespace fftconv {
namespace rf {

template <typename IO> __device__ __forceinline__ float ld(const IO *p, int64_t i)
{
    if constexpr (std::is_same<IO, float>::value) return p[i];
    else if constexpr (std::is_same<IO, __half>::value) return __half2float(p[i]);
    else return __bfloat162float(p[i]);
}
template <typename IO> __device__ __forceinline__ void st(IO *p, int64_t i, float v)
{
    if constexpr (std::is_same<IO, float>::value) p[i] = v;
    else if constexpr (std::is_same<IO, __half>::value) p[i] = __float2half_rn(v);
    else p[i] = __float2bfloat16(v);
}
// a packed pair of 16-bit values <-> fp32
template <typename IO> __device__ __forceinline__ float2 unpack(uint32_t w)
{
    if constexpr (std::is_same<IO, __half>::value) {
        const f3::f16x2 h = __builtin_bit_cast(f3::f16x2, w);
        return make_float2((float)h[0], (float)h[1]);
    } else {
        return make_float2(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
    }
}
template <typename IO> __device__ __forceinline__ uint32_t pack(float lo, float hi)
{
    if constexpr (std::is_same<IO, __half>::value) return f3::F16::pack(lo, hi);
    else return f3::BF16::pack(lo, hi);
}
// the nearest values of the 16-bit type
template <typename IO> __device__ __forceinline__ float2 rounded(float lo, float hi) { return unpack<IO>(pack<IO>(lo, hi)); }
// the word of the neighbouring lane (lane ^ 1)
__device__ __forceinline__ uint32_t neighbour(uint32_t w)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xf, 0xf, true);
}

constexpr int threads_of(int M) { return M <= 8192 ? 256 : 512; }

// 16-bit rows of N samples at a and b whose words are aligned: lane pair (2i, 2i+1) can move the words of samples (2i, 2i+1)
template <typename IO> __device__ __forceinline__ bool word_rows(const void *a, const void *b, int N)
{
    return sizeof(IO) == 2 && N % 2 == 0 && ((((uintptr_t)a | (uintptr_t)b) & 3) == 0);
}

// x[m] = sample tid + T m of the rows r0 (real part) and r1 (imaginary part), zero from N on; a row that is not there
// (has0, has1 false; its pointer still leads to N samples) is zero.  HALF: only m < R0 / 2.  exact: N fills them all.
// Every load is issued before the first is used.
template <typename G, typename IO, bool HALF>
__device__ __forceinline__ void load_pair(float2 (&x)[G::P], const IO *__restrict__ r0, const IO *__restrict__ r1, int N, int tid,
                                          bool exact, bool words, bool has0, bool has1)
{
    constexpr int MIN = HALF ? G::R0 / 2 : G::R0;                 // registers that can hold samples
    if (words) {
        const int odd = tid & 1;
        const IO *const wrow = (odd ? r1 : r0) - odd;             // the lane's row, so that element wrow + n starts its word
        const uint32_t sel = odd ? 0x03020706u : 0x05040100u;     // even: own.lo, other.lo; odd: other.hi, own.hi
        const uint32_t keep = (has0 ? 0xffffu : 0u) | (has1 ? 0xffff0000u : 0u);
        uint32_t wd[MIN];
        if (exact) {
#pragma unroll
            for (int m = 0; m < MIN; ++m) wd[m] = *(const uint32_t *)(wrow + tid + G::T * m);
        } else {
#pragma unroll
            for (int m = 0; m < MIN; ++m) {
                const int n = tid + G::T * m;
                wd[m] = *(const uint32_t *)(wrow + (n < N ? n : odd));
            }
#pragma unroll
            for (int m = 0; m < MIN; ++m) asm volatile("" ::"v"(wd[m]));      // the loads stay unconditional
#pragma unroll
            for (int m = 0; m < MIN; ++m)
                if (tid + G::T * m >= N) wd[m] = 0;
        }
#pragma unroll
        for (int m = 0; m < MIN; ++m) x[m] = unpack<IO>(__builtin_amdgcn_perm(neighbour(wd[m]), wd[m], sel) & keep);
    } else {
        float a[MIN], b[MIN];
#pragma unroll
        for (int m = 0; m < MIN; ++m) {
            const int n = tid + G::T * m, at = n < N ? n : 0;
            a[m] = ld(r0, at);
            b[m] = ld(r1, at);
        }
#pragma unroll
        for (int m = 0; m < MIN; ++m) asm volatile("" ::"v"(a[m]), "v"(b[m]));
#pragma unroll
        for (int m = 0; m < MIN; ++m) {
            const bool in = exact || tid + G::T * m < N;
            x[m] = make_float2(in && has0 ? a[m] : 0.f, in && has1 ? b[m] : 0.f);
        }
    }
}

// The way back: x[m].x -> sample tid + T m of row r0, x[m].y -> r1 (two), below N.
template <typename G, typename IO, bool HALF>
__device__ __forceinline__ void store_pair(const float2 (&x)[G::P], IO *__restrict__ r0, IO *__restrict__ r1, int N, int tid,
                                           bool exact, bool words, bool two)
{
    constexpr int MIN = HALF ? G::R0 / 2 : G::R0;
    if (words) {
        const int odd = tid & 1;
        IO *const wrow = (odd ? r1 : r0) - odd;
        const uint32_t sel = odd ? 0x03020706u : 0x05040100u;     // even: own.re, other.re; odd: other.im, own.im
        const bool put = two || !odd;
#pragma unroll
        for (int m = 0; m < MIN; ++m) {
            const uint32_t z = pack<IO>(x[m].x, x[m].y);
            const uint32_t o = __builtin_amdgcn_perm(neighbour(z), z, sel);
            if (put && (exact || tid + G::T * m < N)) *(uint32_t *)(wrow + tid + G::T * m) = o;
        }
    } else {
#pragma unroll
        for (int m = 0; m < MIN; ++m) {
            const int n = tid + G::T * m;
            if (exact || n < N) {
                st(r0, n, x[m].x);
                if (two) st(r1, n, x[m].y);
            }
        }
    }
}

// a . b of two packed pairs, each product rounded to the I/O type (the fp32 product of 16-bit values is exact)
template <typename IO> __device__ __forceinline__ uint32_t mul_words(uint32_t a, uint32_t b)
{
    if constexpr (std::is_same<IO, __half>::value) {
        return __builtin_bit_cast(uint32_t, __builtin_bit_cast(f3::f16x2, a) * __builtin_bit_cast(f3::f16x2, b));
    } else {
        const float2 x = unpack<IO>(a), y = unpack<IO>(b);
        return pack<IO>(x.x * y.x, x.y * y.y);
    }
}
template <typename IO> __device__ __forceinline__ float mul_io(float a, float b)
{
    if constexpr (sizeof(IO) == 2) return rounded<IO>(a * b, 0.f).x;
    float v = a * b;
    asm("" : "+v"(v));                                            // (rounded: not part of a multiply-add)
    return v;
}

// The samples of load_pair() in two steps, for kernels that multiply by gates: fetch() only asks for them, so that those of a row and of its
// gates are in flight together, and value() multiplies and unpacks.  Words are multiplied as they are, before the neighbours of a
// pair of lanes swap halves.
template <typename G, typename IO, bool HALF> struct RawPair {
    static constexpr int MIN = HALF ? G::R0 / 2 : G::R0;
    uint32_t a[MIN], b[MIN];                                      // words (b unused), or a sample of either row
    // (16-bit samples: a behind b.  The compiler makes one store of the last ones of both branches below, and where those are of a and of b
    // the arrays stay in memory for it)

    __device__ __forceinline__ void fetch(const IO *__restrict__ r0, const IO *__restrict__ r1, int N, int tid, bool words)
    {
        if (words) {
            const int odd = tid & 1;
            const IO *const wrow = (odd ? r1 : r0) - odd;
#pragma unroll
            for (int m = 0; m < MIN; ++m) {
                const int n = tid + G::T * m;
                a[m] = *(const uint32_t *)(wrow + (n < N ? n : odd));
            }
        } else {
#pragma unroll
            for (int m = 0; m < MIN; ++m) {
                const int n = tid + G::T * m, at = n < N ? n : 0;
                if constexpr (sizeof(IO) == 4) {
                    a[m] = ((const uint32_t *)r0)[at];
                    b[m] = ((const uint32_t *)r1)[at];
                } else {
                    b[m] = ((const uint16_t *)r1)[at];
                    a[m] = ((const uint16_t *)r0)[at];
                }
            }
        }
    }
    static __device__ __forceinline__ float one(uint32_t w)
    {
        if constexpr (sizeof(IO) == 4) return __uint_as_float(w);
        else return unpack<IO>(w).x;
    }
    // sample m of both rows, times the gate's where there is one (on); zero from N on, and the second where it is not there
    __device__ __forceinline__ float2 value(int m, int N, int tid, bool words, bool has1, const RawPair &g, bool on) const
    {
        const bool in = tid + G::T * m < N;
        if (words) {
            const uint32_t sel = tid & 1 ? 0x03020706u : 0x05040100u;
            uint32_t w = on ? mul_words<IO>(a[m], g.a[m]) : a[m];
            w = in ? w : 0;
            return unpack<IO>(__builtin_amdgcn_perm(neighbour(w), w, sel) & (has1 ? 0xffffffffu : 0xffffu));
        }
        float2 x = make_float2(one(a[m]), one(b[m]));
        if (on) x = make_float2(mul_io<IO>(x.x, one(g.a[m])), mul_io<IO>(x.y, one(g.b[m])));
        return make_float2(in ? x.x : 0.f, in && has1 ? x.y : 0.f);
    }
    // x[m], rounded to the I/O type, times this gate where there is one (on) -> the rows r0, r1 as in store_pair()
    __device__ __forceinline__ void store(const float2 (&x)[G::P], IO *__restrict__ r0, IO *__restrict__ r1, int N, int tid, bool words,
                                          bool two, bool on) const
    {
        if (words) {
            const int odd = tid & 1;
            IO *const wrow = (odd ? r1 : r0) - odd;
            const uint32_t sel = odd ? 0x03020706u : 0x05040100u;
            const bool put = two || !odd;
#pragma unroll
            for (int m = 0; m < MIN; ++m) {
                const uint32_t z = pack<IO>(x[m].x, x[m].y);
                uint32_t o = __builtin_amdgcn_perm(neighbour(z), z, sel);
                if (on) o = mul_words<IO>(o, a[m]);
                if (put && tid + G::T * m < N) *(uint32_t *)(wrow + tid + G::T * m) = o;
            }
        } else {
#pragma unroll
            for (int m = 0; m < MIN; ++m) {
                const int n = tid + G::T * m;
                float2 c = x[m];
                if (on) {
                    if constexpr (sizeof(IO) == 2) c = rounded<IO>(c.x, c.y);
                    c = make_float2(c.x * one(a[m]), c.y * one(b[m]));
                }
                if (n < N) {
                    st(r0, n, c.x);
                    if (two) st(r1, n, c.y);
                }
            }
        }
    }
};

// calls f(Row<M>()) for the row length of the plan
template <typename F> int with_row(int64_t M, F f)
{
    switch (M) {
    case 256: return f(Row<256>());
    case 512: return f(Row<512>());
    case 1024: return f(Row<1024>());
    case 2048: return f(Row<2048>());
    case 4096: return f(Row<4096>());
    case 8192: return f(Row<8192>());
    case 16384: return f(Row<16384>());
    default:
        set_error("row kernels: no instance for rows of %lld points", (long long)M);
        return FFTCONV_EUNSUPPORTED;
    }
}


// 4 x 4 transpose between the registers v[0 .. 3] and the four groups of 16 lanes of a wave: lane group g of v[j] gets what
// lane group j of v[g] held.
__device__ __forceinline__ void transpose_groups(uint32_t (&v)[4])
{
#pragma unroll
    for (int c = 0; c < 2; ++c) {                                 // upper 32 lanes of v[c] <-> lower 32 of v[c + 2]
        const auto t = __builtin_amdgcn_permlane32_swap(v[c], v[c + 2], false, false);
        v[c] = t[0];
        v[c + 2] = t[1];
    }
#pragma unroll
    for (int c = 0; c < 4; c += 2) {                              // odd groups of v[c] <-> even groups of v[c + 1]
        const auto t = __builtin_amdgcn_permlane16_swap(v[c], v[c + 1], false, false);
        v[c] = t[0];
        v[c + 1] = t[1];
    }
}

// kernel_slot() of the frequency in register p of thread tid.  Every digit of a slot depends on the thread alone or the register alone, but at
// 2048 points and in wide rows of 512 (bit 5 of a frequency is a thread's there, the other bits of its digit k3 a register's), whose slots are worked
// out in full.  Otherwise the slots of a thread lie a constant apart: one address and immediates, where digit by digit they were 1700 of the 3000 vector
// instructions of the gradient's tail at 8192 points (k_row_dk_finish, 768 channels 25.1 -> 19.8 us; the few-row kernel, 1 x 768 x 2048 gated 13.5 -> 10.5).
template <typename G> __device__ __forceinline__ int slot_of(int tid, int p)
{
    if constexpr (G::M == 2048 || (G::M == 512 && G::WIDE)) return kernel_slot<G::M>(G::freq(tid, p));
    else return kernel_slot<G::M>(G::freq(tid, 0)) + (kernel_slot<G::M>(G::freq(0, p)) - kernel_slot<G::M>(G::freq(0, 0)));
}

// lengths with rows of four passes, and their table, behind all others
constexpr bool has_quad(int M) { return M == 2048 || M == 4096; }
template <int M> inline const float2 *quad_table(const fftconv_plan *p)
{
    constexpr int HALF = M == 2048 ? Row<1024, false, false, true>::TABLE : Row<2048>::TABLE;
    return p->row_tw + Row<M, false>::TABLE + Row<M, true>::TABLE + HALF;
}

// lengths with WIDE rows
constexpr bool has_wide(int M) { return M == 512 || M == 1024; }

// The tables of a plan, behind its table of W_M^t: rows of min(M, 8192) points, fast and exact, then those of 16384 where M is
// that or 32768, and of wide rows where M has them; beyond 1024 points, last, those of fast rows of half
// the length, or of 4096 points (rows of 1024 wide).
template <typename G> inline const float2 *row_table(const fftconv_plan *p)
{
    size_t at = G::M == 16384 ? Row<8192, false>::TABLE + Row<8192, true>::TABLE : 0;
    if constexpr (G::WIDE) at = Row<G::M, false>::TABLE + Row<G::M, true>::TABLE;
    if constexpr (!G::EXACT && (G::M == 4096 || G::M == 2048 || G::WIDE)) {
        if (G::M < p->M) {
            if (G::M == 1024) at = Row<2048, false>::TABLE + Row<2048, true>::TABLE;
            if (G::M == 2048) at = Row<4096, false>::TABLE + Row<4096, true>::TABLE;
            if (G::M == 4096) at = Row<8192, false>::TABLE + Row<8192, true>::TABLE;
            if (p->M == 16384 || p->M == 32768) at += Row<16384, false>::TABLE + Row<16384, true>::TABLE;
        }
    }
    return p->row_tw + at + (G::EXACT ? Row<G::M, false, false, G::WIDE>::TABLE : 0);
}

}  // namespace rf
}  // namespace fftconv
