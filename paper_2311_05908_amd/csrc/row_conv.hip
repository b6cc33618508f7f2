// Fused FFT convolution with fp32 arithmetic of rows that fit on chip: fft_size M in {256 .. 16384}, any I/O
// dtype, any N <= M (paper Section 2.1, Eq. 1; the fused single-kernel path of Section 3.1).  Serves the short
// transforms that the matrix-core kernels do not take (fp32 I/O, circular and ragged shapes).
//
// At these lengths there are O(log M) butterflies per point and the work is not reshaped into matrix products:
// radix-16 / 32 passes on the vector ALUs in fp32 (row_fft.h), the samples straight from HBM into the registers of
// the first pass and from those of the last pass back, two (fft <= 1024) or four trips through LDS in between.
//  * Two batch rows of a channel share one complex transform, z = u[b] + i u[b+1] (real filter).
//  * M / R0 threads hold a row (16 .. 512), a workgroup of 256 threads as many rows as fit; rows of one channel are
//    neighbours, and a die (workgroups go to the 8 dies in turn) takes a contiguous range of them, so that k_f is
//    fetched into one L2 only.
//  * k_f is stored in the order of the last pass' registers, [h][register pair][thread][2], so that it streams
//    as 16-byte accesses; it is requested before the last forward pass.
//  * 16-bit rows move as 32-bit words of two adjacent samples: of two neighbouring lanes one fetches the word of row
//    b, the other that of row b + 1, and they swap halves (half the memory instructions of one sample each).
// What bounds it: the vector ALU (about 80 operations per point and convolution at fft 1024, 100 at 4096), close to
// the copy of its bytes.  201 MB of rows (a copy takes 41 us): bf16 circular 50 / 54 / 57 / 67 / 70 us at fft 256 / 512 /
// 1024 / 2048 / 4096 (57 / 100 / 121 / 99 / 123 us with the samples staged through LDS, an exchange for every pass and
// the twiddles gathered from a table in LDS), fp32 causal 47 / 55 / 57 / 70 / 76 us with
// exact twiddles (91 / 114 / 130 / 100 / 122 before; 41 / 47 / 51 / 60 / 61 with products of them, see row_fft.h).
#include "fftconv_internal.h"
#include "row_io.h"

namespace fftconv {

namespace {

using rf::Row;

// waves per SIMD the register budget is held to: what LDS allows (8.5 KB a wave, 17 KB where 32 points of a thread go
// through it as pairs) and the registers can be had for (GATED: one less, for the gates); nothing is spilled
constexpr int waves_of(int M, bool gated = false) { return (M == 256 ? 5 : M == 2048 || M == 4096 ? 4 : 2) - (gated && M <= 4096 && M != 512 && M != 1024 ? 1 : 0); }

template <int M, typename IO, bool WIDE = false> using ConvRow = Row<M, std::is_same<IO, float>::value && M <= 4096, false, WIDE>;

// 16-bit rows of 256 points, which lie 512 bytes or less from those of the next channel: beyond the 256 MB memory-side cache the
// order of the rows in memory counts for more than that of k_f (2 KB a channel), and neighbours are the channels of a pair,
// t = pair * nh + h, and so are workgroups on different dies.  682 x 768 x 256 bf16: 189 us with the pairs of a channel as neighbours, 171 so; 16384 channels 199, 176.  Within the
// cache 36 against 37 (170 x 768), and at 512 points either is up to 20 % faster, depending on H.
template <int M, typename IO> constexpr bool BY_PAIR = M == 256 && sizeof(IO) == 2;

// kf: see the head of this file, scaled by 1/M.  HALF: N <= M / 2.  total: pairs of rows, t = h * npairs + pair, or, with nh > 0
// channels (BY_PAIR), t = pair * nh + h.
// GATED: y = v . ((u . w) * k), either gate may be null; roundings as below (k_row_conv_few).  With an elementwise kernel for each gate
// instead, us: f16 circular 42 x 768 x 512 69 -> 36, bf16 circular 64 x 256 x 256 23 -> 11, 16 x 256 x 2048 41 -> 23, odd rows 16 x 256 x 1001
// (fft 2048) 28 -> 19; fp32 8 x 128 x 4096 (fft 8192) 35 -> 20, 8 x 64 x 16384 circular 55 -> 31, 16 x 64 x 1024 (fft 2048) 16 -> 8.
template <int M, typename IO, bool HALF, bool GATED, bool WIDE>
__global__ void __launch_bounds__(rf::threads_of(M), WIDE ? (GATED ? 3 : 4) : waves_of(M, GATED))
    k_row_conv(const IO *__restrict__ u, IO *__restrict__ y, const float4 *__restrict__ kf, const float2 *__restrict__ tab, int B,
               int H, int N, int npairs, int total, int per_die, int nh, const IO *__restrict__ wg, const IO *__restrict__ vg)
{
    using G = ConvRow<M, IO, WIDE>;
    constexpr int RW = rf::threads_of(M) / G::T;                  // rows (pairs) per workgroup
    extern __shared__ float2 smem_rows[];
    const bool by_pair = BY_PAIR<M, IO> && nh > 0;
    const int group = by_pair ? (int)blockIdx.x : (blockIdx.x & 7) * per_die + (blockIdx.x >> 3);
    if ((int64_t)group * RW >= total) return;
    const int row = threadIdx.x / G::T, tid = threadIdx.x % G::T;
    const int t = min(group * RW + row, total - 1);               // rows beyond the last one repeat it, unstored
    const bool live = group * RW + row < total;
    const int major = t / (by_pair ? nh : npairs), minor = t - major * (by_pair ? nh : npairs);
    const int h = by_pair ? minor : major, pair = by_pair ? major : minor;
    const bool two = 2 * pair + 1 < B;
    const int64_t r0 = ((int64_t)(2 * pair) * H + h) * N, r1 = two ? r0 + (int64_t)H * N : r0;
    float2 *const Z = (float2 *)((char *)smem_rows + row * G::LDS_BYTES);
    const bool exact = N == (HALF ? G::R0 / 2 : G::R0) * G::T;    // every sample of the registers exists
    const bool words = rf::word_rows<IO>(u, y, N) && (!GATED || rf::word_rows<IO>(wg, vg, N));

    float2 x[G::P];
    if constexpr (GATED) {
        using Raw = rf::RawPair<G, IO, HALF>;
        Raw ru, rw;
        ru.fetch(u + r0, u + r1, N, tid, words);
        if (wg) rw.fetch(wg + r0, wg + r1, N, tid, words);
#pragma unroll
        for (int m = 0; m < Raw::MIN; ++m) x[m] = ru.value(m, N, tid, words, two, rw, wg);
    } else {
        rf::load_pair<G, IO, HALF>(x, u + r0, u + r1, N, tid, exact, words, true, two);
    }
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    // k_f of this thread's bins: requested ahead of the last pass as far as the registers go
    if constexpr (WIDE) {                                         // (it lies in the order of the other rows' registers)
        using G0 = ConvRow<M, IO>;
        float2 kv[G::P];
        const float2 *const kr = (const float2 *)kf + (int64_t)h * M + G0::index(G::freq(tid, 0));
        rf::forward<G, HALF>(x, Z, tab, tw1, tid, [&] {
#pragma unroll
            for (int p = 0; p < G::P; ++p) kv[p] = kr[G0::index(G::freq(0, p))];
        });
#pragma unroll
        for (int p = 0; p < G::P; ++p) x[p] = rf::mul(x[p], kv[p]);
    } else {
        constexpr int EARLY = M == 16384 ? G::P / 4 : G::P / 2;
        float4 kv[G::P / 2];
        const float4 *kr = kf + (int64_t)h * (M / 2) + tid;
        rf::forward<G, HALF>(x, Z, tab, tw1, tid, [&] {
#pragma unroll
            for (int q = 0; q < EARLY; ++q) kv[q] = kr[q * G::T];
        });
#pragma unroll
        for (int q = EARLY; q < G::P / 2; ++q) kv[q] = kr[q * G::T];
#pragma unroll
        for (int q = 0; q < G::P / 2; ++q) {
            x[2 * q] = rf::mul(x[2 * q], make_float2(kv[q].x, kv[q].y));
            x[2 * q + 1] = rf::mul(x[2 * q + 1], make_float2(kv[q].z, kv[q].w));
        }
    }
    if constexpr (GATED) {
        using Raw = rf::RawPair<G, IO, HALF>;
        // the output gate asked for ahead of the inverse transform, as registers allow (kept from there, nineteen of fp32 512 were spilled:
        // 3 x 16384 x 512, output gate, 132 -> 81 us)
        constexpr bool AHEAD = HALF ? M <= 8192 : M <= 4096 && !(M == 512 && sizeof(IO) == 4) && !(M == 256 && std::is_same<IO, __hip_bfloat16>::value);
        Raw rv;
        int j = tid;
        if (!HALF) asm volatile("" : "+v"(j));                    // (neither addresses nor masks of the samples are kept from the input to here)
        if (AHEAD && vg) rv.fetch(vg + r0, vg + r1, N, j, words);
        rf::inverse<G>(x, Z, tab, tw1, tid);
        asm volatile("" : "+v"(j));
        if (!AHEAD && vg) rv.fetch(vg + r0, vg + r1, N, j, words);
        if (live) rv.store(x, y + r0, y + r1, N, j, words, two, vg);
    } else {
        rf::inverse<G>(x, Z, tab, tw1, tid);
        // real part -> row b, imaginary part -> row b + 1
        if (live) rf::store_pair<G, IO, HALF>(x, y + r0, y + r1, N, tid, exact, words, two);
    }
}

// The same without gates, one pair of rows to a workgroup of rows of four passes (row_fft.h), for calls of few pairs.
template <int M, typename IO, bool HALF>
__global__ void __launch_bounds__(rf::Quad<M>::T)
    k_row_conv_quad(const IO *__restrict__ u, IO *__restrict__ y, const float2 *__restrict__ kf, const float2 *__restrict__ tab, int B,
                    int H, int N, int npairs, int total, int per_die)
{
    using Q = rf::Quad<M>;
    using G0 = ConvRow<M, IO>;
    extern __shared__ float2 smem_rows[];
    const int tid = threadIdx.x, t = (blockIdx.x & 7) * per_die + (blockIdx.x >> 3);
    if (t >= total) return;
    const int h = t / npairs, pair = t - h * npairs;
    const bool two = 2 * pair + 1 < B;
    const int64_t r0 = ((int64_t)(2 * pair) * H + h) * N, r1 = two ? r0 + (int64_t)H * N : r0;
    const bool exact = N == (HALF ? M / 2 : M), words = rf::word_rows<IO>(u, y, N);
    rf::QuadTw<Q> tw;
    tw.load(tab, tid);
    float2 x[Q::P], kv[Q::P];
    rf::load_pair<Q, IO, HALF>(x, u + r0, u + r1, N, tid, exact, words, true, two);
    const float2 *const kr = kf + (int64_t)h * M + G0::index(Q::freq(tid, 0));          // (in the order of the other rows' registers)
#pragma unroll
    for (int p = 0; p < Q::P; ++p) kv[p] = kr[G0::index(Q::freq(0, p))];
    const rf::QuadSlots<Q> z(smem_rows, tid);
    rf::quad_forward<Q, HALF>(x, z, tw);
#pragma unroll
    for (int p = 0; p < Q::P; ++p) x[p] = rf::mul(x[p], kv[p]);
    rf::quad_inverse<Q>(x, z, tw);
    rf::store_pair<Q, IO, HALF>(x, y + r0, y + r1, N, tid, exact, words, two);
}

// The same convolution for the plans of the matrix-core kernels (16-bit I/O, N <= fft/2 a multiple of 8, 16-byte aligned rows),
// with their k_f: 16-bit (re, im) pairs in the slot order of those kernels (kernel_slot), and with their gates (GATE bit 0:
// wg multiplies u, bit 1: vg multiplies y).  The transforms and the product with k_f are fp32; u . w is rounded to the I/O type,
// as is the convolution before it meets the output gate: the same values as without a fused gate, whichever kernel a call
// takes.  For calls of few rows: see row_forward_few().
template <int M, typename IO, int GATE, bool WIDE, bool WORDS>
__global__ void __launch_bounds__(rf::threads_of(M), WIDE ? 4 : waves_of(M))
    k_row_conv_few(const IO *__restrict__ u, IO *__restrict__ y, const uint32_t *__restrict__ kf, const float2 *__restrict__ tab,
                   const IO *__restrict__ wg, const IO *__restrict__ vg, int B, int H, int N, int npairs, int total)
{
    using G = Row<M, false, false, WIDE>;
    constexpr int RW = rf::threads_of(M) / G::T;
    extern __shared__ float2 smem_rows[];
    const int row = threadIdx.x / G::T, tid = threadIdx.x % G::T;
    const int t = min((int)blockIdx.x * RW + row, total - 1);
    const bool live = (int)blockIdx.x * RW + row < total;
    const int h = t / npairs, pair = t - h * npairs;
    const bool two = 2 * pair + 1 < B;
    const int64_t r0 = ((int64_t)(2 * pair) * H + h) * N, r1 = two ? r0 + (int64_t)H * N : r0;
    float2 *const Z = (float2 *)((char *)smem_rows + row * G::LDS_BYTES);
    const bool exact = N == M / 2;
    // WORDS: the gates as words, in flight with what they multiply.  Otherwise as fp32, one after the other (but bf16 input gates, which are the faster ones
    // as words).
    constexpr bool WORDS_IN = WORDS || std::is_same<IO, __hip_bfloat16>::value;
    using Raw = rf::RawPair<G, IO, true>;
    float2 x[G::P], g[G::P];
    Raw rv;
    if constexpr ((GATE & 1) && WORDS_IN) {
        Raw ru, rw;
        ru.fetch(u + r0, u + r1, N, tid, true);
        rw.fetch(wg + r0, wg + r1, N, tid, true);
#pragma unroll
        for (int m = 0; m < Raw::MIN; ++m) x[m] = ru.value(m, N, tid, true, two, rw, true);
    } else {
        rf::load_pair<G, IO, true>(x, u + r0, u + r1, N, tid, exact, true, true, two);
        if constexpr (GATE & 1) {
            rf::load_pair<G, IO, true>(g, wg + r0, wg + r1, N, tid, exact, true, true, two);
#pragma unroll
            for (int m = 0; m < G::P / 2; ++m) x[m] = rf::rounded<IO>(x[m].x * g[m].x, x[m].y * g[m].y);
        }
    }
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    uint32_t kv[G::P];
    const uint32_t *kr = kf + (int64_t)h * M;
    rf::forward<G, true>(x, Z, tab, tw1, tid, [&] {
#pragma unroll
        for (int p = 0; p < G::P; ++p) kv[p] = kr[rf::slot_of<G>(tid, p)];
    });
#pragma unroll
    for (int p = 0; p < G::P; ++p) x[p] = rf::mul(x[p], rf::unpack<IO>(kv[p]));
    if constexpr ((GATE & 2) && WORDS) rv.fetch(vg + r0, vg + r1, N, tid, true);
    rf::inverse<G>(x, Z, tab, tw1, tid);
    if constexpr ((GATE & 2) && WORDS) {
        if (live) rv.store(x, y + r0, y + r1, N, tid, true, two, true);
        return;
    }
    if constexpr ((GATE & 2) && !WORDS) {
        rf::load_pair<G, IO, true>(g, vg + r0, vg + r1, N, tid, exact, true, true, two);
#pragma unroll
        for (int m = 0; m < G::P / 2; ++m) {
            const float2 c = rf::rounded<IO>(x[m].x, x[m].y);
            x[m] = make_float2(c.x * g[m].x, c.y * g[m].y);
        }
    }
    if (live) rf::store_pair<G, IO, true>(x, y + r0, y + r1, N, tid, exact, true, two);
}

// The same for calls of one batch row, whose rows have no partners: M / 2 points z[n] = a[2n] + i a[2n+1], a word of samples each (no halves to swap), instead
// of M with zeros for imaginary parts.  With Z = FFT(z), E and O the spectra of the even and odd samples, W = W_M^f, and K0, K1 the bins f and f + M/2 of
// k_f, the result's transform is
//   Z'[f] = Z S + D (W O + i conj(W) E),  S, D = (K0 +- K1) / 2,  2 E = Z[f] + conj Z[M/2 - f],  2 O = (Z[f] - conj Z[M/2 - f]) / i,
// so that a thread needs the mirror images of its bins only: one trip through LDS more, of half the points, and half the waves.
// Bound by the latency of a row up to three of them to a compute unit, by its instructions beyond.  us, rows with zeros -> so, on inputs that stay in the caches: both
// gates, bf16 1 x 768 x 2048 (fft 4096) 10.4 -> 8.3 (10.4 -> 9.5 on new inputs each call; the kernel alone 11.1 -> 8.8 traced), 1 x 8192 80 -> 57, 1 x 8192 x 1024 (fft 2048) 56 -> 33; without 1 x 768 x 2048 9.4 -> 7.8, 1 x 4096 x 1024
// 28.8 -> 17.9, 1 x 64 7.3 -> 5.8.  k_f asked for with the samples, ahead of the transform: 9.5 instead of 8.8.
template <int M> constexpr bool LONE_STAGED = M == 2048;
template <int M> using LoneRow = Row<M / 2, false, false, M / 2 == 1024>;
template <int M, typename IO, int GATE>
__global__ void __launch_bounds__(LoneRow<M>::T, 2)
    k_row_conv_lone(const IO *__restrict__ u, IO *__restrict__ y, const uint32_t *__restrict__ kf, const float2 *__restrict__ tab,
                    const IO *__restrict__ wg, const IO *__restrict__ vg, int N)
{
    using G = LoneRow<M>;
    static_assert(G::THREE && G::T / G::RL == G::R1, "slots of the mirror images, below");
    constexpr int MIN = G::P / 2;
    extern __shared__ float2 Z[];
    const int tid = threadIdx.x, words = N / 2;
    const int64_t first = blockIdx.x * (int64_t)words;
    auto fetch = [&](uint32_t (&w)[MIN], const IO *t) {
        const uint32_t *const r = (const uint32_t *)t + first;
#pragma unroll
        for (int m = 0; m < MIN; ++m) {
            const int n = tid + G::T * m;
            w[m] = r[n < words ? n : 0];
        }
    };
    float2 x[G::P];
    {
        uint32_t a[MIN], g[MIN];
        fetch(a, u);
        if constexpr (GATE & 1) fetch(g, wg);
#pragma unroll
        for (int m = 0; m < MIN; ++m) asm volatile("" ::"v"(a[m]));       // the loads stay unconditional
#pragma unroll
        for (int m = 0; m < MIN; ++m) {
            uint32_t w = a[m];
            if constexpr (GATE & 1) w = rf::mul_words<IO>(w, g[m]);
            x[m] = rf::unpack<IO>(tid + G::T * m < words ? w : 0);
        }
    }
    rf::Tw1<G> tw1;
    tw1.load(tab, tid);
    // k_f: the digits of a slot depend on the thread alone or the register alone.  Rows of 4096 points ask for their bins ahead of the last pass; those of
    // 2048, of one wave, whose lanes lie scattered in it, take it whole into LDS, asked for with the samples (1 x 8192 x 1024 both gates 43.5 -> 33.1 us; 4096 points so:
    // 57 -> 71), with 16 words of padding behind 256.
    constexpr bool STAGED = LONE_STAGED<M>;
    typedef uint32_t Four __attribute__((ext_vector_type(4)));
    constexpr int KQ = STAGED ? M / (4 * G::T) : 1;
    auto padded = [](int slot) { return STAGED ? slot + slot / 256 * 16 : slot; };
    auto lower = [&](int p) { return padded(kernel_slot<M>(G::freq(0, p)) - kernel_slot<M>(0)); };
    auto upper = [&](int p) { return padded(kernel_slot<M>(G::freq(0, p) + M / 2) - kernel_slot<M>(0)); };
    uint32_t *const KL = (uint32_t *)(Z + G::SLOTS);
    const int slot = padded(kernel_slot<M>(G::freq(tid, 0)));
    Four kq[KQ];
    uint32_t k0[STAGED ? 1 : G::P], k1[STAGED ? 1 : G::P];
    if constexpr (STAGED) {
#pragma unroll
        for (int i = 0; i < KQ; ++i) kq[i] = ((const Four *)kf)[(int64_t)blockIdx.x * (M / 4) + tid + G::T * i];
    }
    rf::forward<G, true>(x, Z, tab, tw1, tid, [&] {
        if constexpr (STAGED) {
#pragma unroll
            for (int i = 0; i < KQ; ++i) *(Four *)(KL + padded(4 * (tid + G::T * i))) = kq[i];
        } else {
            const uint32_t *const kr = kf + (int64_t)blockIdx.x * M + slot;
#pragma unroll
            for (int p = 0; p < G::P; ++p) {
                k0[p] = kr[lower(p)];
                k1[p] = kr[upper(p)];
            }
        }
    });
#pragma unroll
    for (int i = 0; i < G::NBL; ++i) {
        float2 *const z = Z + G::slotl(tid + G::T * i);
#pragma unroll
        for (int r = 0; r < G::RL; ++r) z[r] = x[i * G::RL + r];
    }
    rf::row_barrier<G::T>();
    const float rev = (float)G::freq(tid, 0) * (1.f / (float)M);          // exact: the sine and cosine take revolutions
    const float2 w0 = make_float2(__builtin_amdgcn_cosf(rev), -__builtin_amdgcn_sinf(rev));
    uint32_t v[MIN];
    if constexpr (GATE & 2) fetch(v, vg);
    float2 mirror[G::P];
#pragma unroll
    for (int i = 0; i < G::NBL; ++i) {
        // digits of M/2 - f: complements, plus one from the first that is not zero on
        const int bi = tid + G::T * i, d0 = bi / G::R1, d1 = bi % G::R1;
        const float2 *const z = Z + (d0 ? (G::R0 - d0) * G::PITCH + (G::R1 - 1 - d1) * G::PAD + G::RL - 1 : d1 ? (G::R1 - d1) * G::PAD + G::RL - 1 : G::RL);
#pragma unroll
        for (int r = 0; r < G::RL; ++r) mirror[i * G::RL + r] = *(r == 0 && bi == 0 ? Z : z - r);
    }
#pragma unroll
    for (int p = 0; p < G::P; ++p) {
        constexpr float TWO_PI = 6.283185307179586f;
        const float2 z = x[p], m = mirror[p];
        const float2 w = p ? rf::mul(w0, make_float2(__builtin_cosf(TWO_PI / M * G::freq(0, p)), -__builtin_sinf(TWO_PI / M * G::freq(0, p)))) : w0;
        const float2 e = make_float2(z.x + m.x, z.y - m.y), o = make_float2(z.y + m.y, m.x - z.x);             // 2 E, 2 O
        uint32_t ka, kb;
        if constexpr (STAGED) ka = KL[slot + lower(p)], kb = KL[slot + upper(p)];
        else ka = k0[p], kb = k1[p];
        const float2 a = rf::unpack<IO>(ka), b = rf::unpack<IO>(kb);
        const float2 s = make_float2(a.x + b.x, a.y + b.y), d = make_float2(0.5f * (a.x - b.x), 0.5f * (a.y - b.y));     // (k_f is scaled by 1 / M)
        const float2 c = rf::mul_conj(e, w), t = rf::mul(o, w);
        const float2 q = rf::mul(make_float2(t.x - c.y, t.y + c.x), d), h = rf::mul(z, s);
        x[p] = make_float2(h.x + q.x, h.y + q.y);
    }
    rf::row_barrier<G::T>();                                      // the mirror images have been read
    rf::inverse<G>(x, Z, tab, tw1, tid);
    uint32_t *const out = (uint32_t *)y + first;
#pragma unroll
    for (int m = 0; m < MIN; ++m) {
        uint32_t w = rf::pack<IO>(x[m].x, x[m].y);
        if constexpr (GATE & 2) w = rf::mul_words<IO>(w, v[m]);
        if (tid + G::T * m < words) out[tid + G::T * m] = w;
    }
}

template <int M, typename IO, bool HALF, bool GATED, bool WIDE>
int launch(const fftconv_plan *p, const void *u, const void *kf, void *y, int64_t B, const void *wg, const void *vg, hipStream_t s)
{
    using G = ConvRow<M, IO, WIDE>;
    constexpr int NTHR = rf::threads_of(M), RW = NTHR / G::T;
    constexpr int lds = RW * G::LDS_BYTES;
    FC_TRY(raise_dynamic_lds((const void *)k_row_conv<M, IO, HALF, GATED, WIDE>, lds));
    // A launch holds less than 2^32 threads, and the kernel counts rows in 32 bits: longer calls go out in pieces of MOST
    // pairs, whole channels where the batch allows it.
    constexpr int64_t MOST = ((int64_t)1 << 31) / G::T;
    const int64_t H = p->H, N = p->N, npairs = (B + 1) / 2;
    const bool by_pair = BY_PAIR<M, IO> && N % 2 == 0 && 2 * B * H * N * (int64_t)sizeof(IO) > ((int64_t)1 << 28);
    for (int64_t p0 = 0; p0 < npairs; p0 += MOST) {
        const int64_t np = npairs - p0 < MOST ? npairs - p0 : MOST, nb = B - 2 * p0 < 2 * np ? B - 2 * p0 : 2 * np, nh = MOST / np;
        for (int64_t h0 = 0; h0 < H; h0 += nh) {
            const int64_t hs = H - h0 < nh ? H - h0 : nh, total = hs * np, groups = (total + RW - 1) / RW, per_die = (groups + 7) / 8;
            const int64_t at = (2 * p0 * H + h0) * N;
            hipLaunchKernelGGL((k_row_conv<M, IO, HALF, GATED, WIDE>), dim3((unsigned)(8 * per_die)), dim3(NTHR), lds, s, (const IO *)u + at,
                               (IO *)y + at, (const float4 *)kf + h0 * (M / 2), rf::row_table<G>(p), (int)nb, (int)H, (int)N, (int)np,
                               (int)total, (int)per_die, by_pair ? (int)hs : 0, wg ? (const IO *)wg + at : nullptr,
                               vg ? (const IO *)vg + at : nullptr);
            FC_HIP(hipGetLastError());
        }
    }
    return FFTCONV_OK;
}

// Pairs of rows up to which they are WIDE.  us, others, wide: fp32 causal fft 512, 512 pairs 7.9, 5.3, 2048 8.3, 6.1, 3072 8.6, 8.1, 4096 8.8, 10.1; 1024, 512 8.6,
// 6.1, 2048 9.5, 8.3, 3072 13.4, 13.1, 3584 13.0, 14.6; fp16 circular 512, 3072 9.2, 7.8, 4096 9.4, 9.5; bf16 circular 1024, 3072 13.7, 13.3, 3584 13.5, 14.6 (256 channels;
// 3584 of a pair each 17.5, 16.7 in circular fp32, 13.5, 14.0 in bf16).  Both gates: 512,
// fp32 6144 18.3, 17.4, 8192 21.1, 22.2, bf16 circular 19.3, 18.0 and 21.4, 22.6; 1024 always, fp32 8192 36.8, 34.1, 32768 160, 156, bf16 circular 8192
// 40.5, 37.2, fp16 32768 171, 171.  Calls of few rows (k_row_conv_few): 512 bf16 3072 7.9, 7.1, 4096 8.0, 8.2; 1024, 1024 8.0, 6.9, 1536 8.1, 8.9.
template <int M> constexpr int64_t wide_most(bool gated) { return !gated ? 3072 : M == 512 ? 6144 : INT64_MAX; }
template <int M> constexpr int64_t FEW_WIDE = M == 512 ? 3072 : 1024;

// The same of four passes; row_quad() holds what one launch does
template <int M, typename IO>
int launch_quad(const fftconv_plan *p, const void *u, const void *kf, void *y, int64_t B, hipStream_t s)
{
    using Q = rf::Quad<M>;
    const auto kern = p->N <= M / 2 ? k_row_conv_quad<M, IO, true> : k_row_conv_quad<M, IO, false>;
    FC_TRY(raise_dynamic_lds((const void *)kern, Q::LDS_BYTES));
    const int64_t npairs = (B + 1) / 2, total = p->H * npairs, per_die = (total + 7) / 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)(8 * per_die)), dim3(Q::T), Q::LDS_BYTES, s, (const IO *)u, (IO *)y, (const float2 *)kf,
                       rf::quad_table<M>(p), (int)B, (int)p->H, (int)p->N, (int)npairs, (int)total, (int)per_die);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

template <int M, typename IO>
int launch_row(const fftconv_plan *p, const void *u, const void *kf, void *y, int64_t B, const void *wg, const void *vg, hipStream_t s)
{
    const bool half = p->N <= M / 2, gated = wg || vg;
    if constexpr (rf::has_wide(M)) {
        if (p->H * ((B + 1) / 2) <= wide_most<M>(gated)) {
            if (gated) return half ? launch<M, IO, true, true, true>(p, u, kf, y, B, wg, vg, s) : launch<M, IO, false, true, true>(p, u, kf, y, B, wg, vg, s);
            return half ? launch<M, IO, true, false, true>(p, u, kf, y, B, wg, vg, s) : launch<M, IO, false, false, true>(p, u, kf, y, B, wg, vg, s);
        }
    }
    if constexpr (rf::has_quad(M))
        if (!gated && row_quad(M, std::is_same<IO, float>::value, p->N, p->H, B)) return launch_quad<M, IO>(p, u, kf, y, B, s);
    if constexpr (M != 1024)
        if (gated) return half ? launch<M, IO, true, true, false>(p, u, kf, y, B, wg, vg, s) : launch<M, IO, false, true, false>(p, u, kf, y, B, wg, vg, s);
    return half ? launch<M, IO, true, false, false>(p, u, kf, y, B, wg, vg, s) : launch<M, IO, false, false, false>(p, u, kf, y, B, wg, vg, s);
}

}  // namespace

// Calls without gates whose rows take four passes (a launch holds 2^23 pairs): while the pairs have a compute unit each, or, where rows are full, two of them one, and fp32 rows of 2048
// points at nearly any number.  us, three passes, four: fp32 causal fft 2048, 4 pairs 6.6, 4.5 (the kernels alone, traced), 256 6.7, 6.1, 768 8.6, 7.7,
// 2048 17.1, 15.2, 16384 107, 103, circular 1024 12.8, 10.6; bf16 circular 256 6.9, 6.5, 512 7.2, 6.9, 768 8.7, 8.7, 1024 9.0, 10.0, 500 samples 257 to 512 pairs
// 6.15, 6.3; fft 4096 fp32
// 4 6.6, 5.9 and 256 7.6, 6.9 (traced), 300 8.5, 8.9, 384 8.8, 9.2, bf16 circular 256 7.4, 7.2, 300 9.2, 9.9.  Errors of fp32: fft 2048 1.42e-7 -> 1.34e-7, 4096 1.58e-7 -> 1.38e-7;
// rows so short that the first pass of three, of 16 points, has a sample or two to add up are more accurate there (fft 2048, 8 samples 5.6e-8, 6.6e-8 in four, 128 7.95e-8, 8.28e-8,
// 150 8.47e-8, 8.37e-8, 200 9.5e-8, 8.7e-8; 4096, 16 6.2e-8, 6.8e-8, 20 6.8e-8, 6.8e-8, 64 8.9e-8, 7.2e-8).
// fp32 rows of 2048 points that are more than half full, once u and y exceed the memory-side cache: three passes are faster (8 x 1024 x 2048 128 MB 1.20 times as
// fast in four, 16 x 768 192 MB 1.15, 16 x 1024 256 MB 0.98, 64 x 768 384 MB 0.96, 64 x 768 x 1500 562 MB 0.92); half-empty rows are no slower in four there
// (64 x 1500 x 1024 750 MB 1.01, 256 x 2048 x 256 1 GB 1.03).
// fp32 rows of 2048 points that are half zeros: three passes are as fast or faster with 769 to 1024 pairs, and short rows with 1793 to 2048, where the memory's
// time does not count: 1024 pairs of 100 samples 7.6, 7.9, of 1024 8.9, 8.9, 1536 of 100 10.1, 10.1, 1600 11.6, 11.2, 2048 11.8, 12.4, of 512 13.2, 13.4, of 1024
// 17.1, 15.2; between those lines a few calls of 1536 to 2048 pairs are up to 3 % slower so (2 x 1536 x 400 10.3, 10.7; 2 x 2048 x 400 14.9, 13.4).
// fp32 rows of 4096 beyond 256 pairs: full rows of 700 to 1700 pairs are up to a tenth faster so, as are those of half as many samples in two batch rows, but short
// rows, and many batch rows, up to a tenth slower (2 x 768 x 2048 13.7, 13.2, 4 x 384 x 2048 12.0, 12.8, 2 x 1024 x 100 12.3, 13.7): three passes.
bool row_quad(int64_t M, bool f32, int64_t N, int64_t H, int64_t B)
{
    const int64_t npairs = (B + 1) / 2;
    const bool half = N <= M / 2;
    if (npairs > (1 << 23) / H || (f32 && N < (M == 2048 ? 150 : 20))) return false;
    const int64_t pairs = H * npairs;
    if (M == 4096) return pairs <= 256;
    if (!f32) return pairs <= (half ? 256 : 512);
    if (!half) return B * H * N <= (int64_t)28 << 20;             // 224 MB of u and y
    return pairs <= 768 || (pairs > 1024 && (pairs <= 1792 || pairs > 2048 || N > M / 8));
}

// The twiddle tables of the row kernels for a plan of M points (see row_table()), from w[t] = W_M^t
std::vector<float2> row_tables(int64_t M, const double2 *w)
{
    std::vector<float2> t;
    auto add = [&](auto g) {
        using G = decltype(g);
        t.resize(t.size() + G::TABLE);
        rf::fill_table<G>(t.data() + t.size() - G::TABLE, [&](int num, int den) { return w[num * (M / den)]; });
    };
    auto add_length = [&](int64_t L) {
        (void)rf::with_row(L, [&](auto g) -> int {
            using G = decltype(g);
            add(Row<G::M, false>());
            add(Row<G::M, true>());
            return FFTCONV_OK;
        });
    };
    add_length(M < 8192 ? M : 8192);
    if (M == 16384 || M == 32768) add_length(16384);
    if (M == 512) add(Row<512, false, false, true>()), add(Row<512, true, false, true>());
    if (M == 1024) add(Row<1024, false, false, true>()), add(Row<1024, true, false, true>());
    if (M == 2048) add(Row<1024, false, false, true>());
    if (M == 4096) add(Row<2048>());
    if (M > 4096) add(Row<4096>());
    auto add_quad = [&](auto q) {
        using Q = decltype(q);
        t.resize(t.size() + Q::TABLE);
        rf::fill_quad_table<Q>(t.data() + t.size() - Q::TABLE, [&](int num, int den) { return w[num * (M / den)]; });
    };
    if (M == 2048) add_quad(rf::Quad<2048>());
    if (M == 4096) add_quad(rf::Quad<4096>());
    return t;
}

int row_forward(const fftconv_plan *p, const void *u, const void *kf, void *y, int64_t B, hipStream_t s, const void *wg, const void *vg)
{
    return rf::with_row(p->M, [&](auto g) -> int {
        using G = decltype(g);
        if (p->dtype == FFTCONV_F32) return launch_row<G::M, float>(p, u, kf, y, B, wg, vg, s);
        if constexpr (G::M <= 4096) {                             // longer 16-bit rows run on the matrix cores
            if (p->dtype == FFTCONV_F16) return launch_row<G::M, __half>(p, u, kf, y, B, wg, vg, s);
            return launch_row<G::M, __hip_bfloat16>(p, u, kf, y, B, wg, vg, s);
        }
        set_error("row kernels: no 16-bit instance for rows of %lld points", (long long)p->M);
        return FFTCONV_EUNSUPPORTED;
    });
}

// Few rows: which calls of a matrix-core plan up to fft 4096 the row kernel takes.  Both kernels' times are staircases.  The
// matrix-core kernel runs its work items (8192 / fft pairs of rows of one channel, however few there are) in rounds of one per
// compute unit: 7.0 - 7.9, 10.7, 14.1, 17.2 us for 1, 2, 3, 4 of them (bf16; fp16 with both gates 7.3 - 8.2, 11.5, 16.1, 19).  The row kernel runs workgroups of
// `rows` pairs.  us, rows, matrix cores (bf16, or fp16 with both gates where two pairs are given):
//   fft 4096: as many workgroups as one a compute unit for each round: 1 x 64 6.1, 7.3, 1 x 768 9.3, 13.0, 1 x 2048 20.5, 26.6, 1 x 8192 77, 87; twice as many
//     would be slower (4 x 256 7.8, 7.7; 9.3, 8.2; 3 x 1024 21.4, 17.5);
//   fft 2048: as many, beyond six rounds half as many: 1 x 512 7.6, 10.2, 3 x 1024 15.9, 16.2, 3 x 2048 28.9, 26.8, 1 x 8192 51, 85 (in the first round
//     either: 3 x 64 7.6, 7.5, 8 x 128 7.8, 7.2);
//   fft 1024: half as many, and not in the first round (16 x 256 8.3, 7.8): 1 x 768 6.7, 12.6, 1 x 8192 17.9, 84.6;
//   fft 512: half as many, and only if items are not full: 1 x 64 5.2, 7.2, 1 x 2048 5.5, 24.8; 32 x 256 8.0, 7.9 (8.6, 8.2);
//   fft 256: 40 Ki pairs + 56 a channel.  B x 768 channels, bf16, matrix cores, rows: B = 64 16.9, 13.0 us, 128 27, 23, 256 42, 40; 8192
//     channels: B = 33 98, 51, fp16 64 106, 116.
// (A line that rose without bound at fft 256 sent all calls here: 191 -> 258 us at B = 1365, and gated
// calls in the first round at fft 2048 took up to 13.0 against 10.0 us.)
// At 512, 1024 and 4096 these are the lines of a slower row kernel.  Today's would also be the faster one for full items of few rows at 512 (32 x 16 5.5, 6.9),
// in the first round of few at 1024 (16 x 16 6.7, 7.0) and for half as many workgroups again at 4096 (4 x 384 9.7, 10.6; 11.3, 11.9).  Those calls keep the
// kernel and the last bits that they have had; tests/test_planner.py holds shapes of either side.
// At 8192 points the row kernel is not the faster one (16 channels: 8.8 and more against 7.5).
// The kernel counts rows and threads (at most 64, or M / 16, to a pair of rows) in 32 bits: calls beyond that are not few rows.
bool row_few(int64_t M, int64_t H, int64_t B)
{
    const int64_t npairs = (B + 1) / 2;
    if (M > 4096 || npairs > INT32_MAX / (H * (M / 16))) return false;
    const int64_t pairs = H * npairs;
    if (M == 256) return pairs < 40 * 1024 + 56 * H;
    constexpr int CUS = 256;
    const int64_t full = 8192 / M, items = H * ((npairs + full - 1) / full), rounds = (items + CUS - 1) / CUS;
    const int64_t rows = M == 512 ? 16 : M == 1024 ? 8 : M == 2048 ? 2 : 1, groups = (pairs + rows - 1) / rows;
    if (M >= 2048) return groups <= CUS * rounds && (M == 4096 || rounds <= 6 || 2 * groups <= CUS * rounds);
    if (M == 1024) return rounds > 1 && groups <= CUS * ((rounds + 1) / 2);
    return pairs < full * items && 2 * groups <= CUS * (rounds + 1);
}

// Calls of one batch row whose rows go as half as many points.  At 4096 points, one row to a compute unit takes as long either way, the other kernel having twice
// the threads for it, and fp16 rows, whose samples take conversions, up to two longer: 1 x 257 / 400 / 512 / 513 / 768 x 2048, us, rows with zeros -> so,
// fp16 6.9, 7.6, 7.8, 8.7, 9.6 -> 7.6, 8.2, 8.3, 8.3, 8.5, bf16 7.0, 7.5, 7.6, 8.5, 9.3 -> 7.0, 7.4, 7.5, 7.6, 7.9.
bool row_lone(int64_t M, int64_t H, bool f16) { return M == 2048 || (M == 4096 && H > (f16 ? 512 : 256)); }

// for calls that row_few() takes
int row_forward_few(const fftconv_plan *p, const void *u, const void *kf, void *y, int64_t B, const void *wg, const void *vg,
                    hipStream_t s)
{
    return rf::with_row(p->M, [&](auto g) -> int {
        constexpr int M = decltype(g)::M;
        if constexpr (M > 4096) {
            return FFTCONV_EUNSUPPORTED;
        } else {
            auto lone = [&](auto io) -> int {                     // N is even, and rows lie at whole words
                if constexpr (M >= 2048) {
                    using IO = decltype(io);
                    using G = LoneRow<M>;
                    const auto kern = wg ? (vg ? k_row_conv_lone<M, IO, 3> : k_row_conv_lone<M, IO, 1>)
                                         : (vg ? k_row_conv_lone<M, IO, 2> : k_row_conv_lone<M, IO, 0>);
                    constexpr int lds = G::LDS_BYTES + (LONE_STAGED<M> ? 4 * (M + M / 16) : 0);
                    FC_TRY(raise_dynamic_lds((const void *)kern, lds));
                    hipLaunchKernelGGL(kern, dim3((unsigned)p->H), dim3(G::T), lds, s, (const IO *)u, (IO *)y, (const uint32_t *)kf,
                                       rf::row_table<G>(p), (const IO *)wg, (const IO *)vg, (int)p->N);
                    FC_HIP(hipGetLastError());
                }
                return FFTCONV_OK;
            };
            if (B == 1 && row_lone(M, p->H, p->dtype == FFTCONV_F16)) return p->dtype == FFTCONV_F16 ? lone(__half()) : lone(__hip_bfloat16());
            auto form = [&](auto io, auto w) -> int {
                using IO = decltype(io);
                constexpr bool WIDE = decltype(w)::value;
                using G = Row<M, false, false, WIDE>;
                constexpr int NTHR = rf::threads_of(M), RW = NTHR / G::T, lds = RW * G::LDS_BYTES;
                const int64_t npairs = (B + 1) / 2, total = p->H * npairs;
                auto kern = wg ? (vg ? k_row_conv_few<M, IO, 3, WIDE, true> : k_row_conv_few<M, IO, 1, WIDE, true>)
                               : (vg ? k_row_conv_few<M, IO, 2, WIDE, true> : k_row_conv_few<M, IO, 0, WIDE, true>);
                // At 256 points, 8 samples a thread, the masks of the words, which rows that fill their registers do without otherwise, are most of what the
                // loads in flight save.  us, words, not: input gate fp16 2 x 256 x 128 4.77, 4.55, 16 x 768 x 128 6.09, 6.78, 2 x 256 x 64 4.73, 4.88, 16 x 768 x 64 5.80,
                // 6.72; output gate 2 x 256 x 128 4.74, 4.59, 16 x 768 x 128 6.66, 6.35, 2 x 256 x 64 4.62, 4.86, fp16 24 x 768 x 120 8.70, 8.29, bf16 16 x 768 x 64 6.05, 6.32; both 16 x 768 x 128
                // 6.62, 6.48, 16 x 768 x 64 6.19, 6.83.
                if constexpr (M == 256)
                    if (wg && vg ? p->N == M / 2 : wg ? p->N == M / 2 && total <= 4096 : vg && (p->N == M / 2 || (std::is_same<IO, __half>::value && total > 4096)))
                        kern = wg ? (vg ? k_row_conv_few<M, IO, 3, WIDE, false> : k_row_conv_few<M, IO, 1, WIDE, false>)
                                  : k_row_conv_few<M, IO, 2, WIDE, false>;
                FC_TRY(raise_dynamic_lds((const void *)kern, lds));
                hipLaunchKernelGGL(kern, dim3((unsigned)((total + RW - 1) / RW)), dim3(NTHR), lds, s, (const IO *)u, (IO *)y,
                                   (const uint32_t *)kf, rf::row_table<G>(p), (const IO *)wg, (const IO *)vg, (int)B, (int)p->H,
                                   (int)p->N, (int)npairs, (int)total);
                FC_HIP(hipGetLastError());
                return FFTCONV_OK;
            };
            auto go = [&](auto io) -> int {
                if constexpr (rf::has_wide(M))
                    if (p->H * ((B + 1) / 2) <= FEW_WIDE<M>) return form(io, std::true_type());
                return form(io, std::false_type());
            };
            return p->dtype == FFTCONV_F16 ? go(__half()) : go(__hip_bfloat16());
        }
    });
}

FacList small_factor_list(int64_t M)
{
    FacList fl{};
    (void)rf::with_row(M, [&](auto g) -> int {
        using G = decltype(g);
        fl = FacList{G::THREE ? 3 : 2, {G::R0, G::R1, G::R2}};
        return FFTCONV_OK;
    });
    return fl;
}

bool small_supported(int64_t N, int64_t M, int dtype)
{
    (void)dtype;
    return M >= 256 && M <= 4096 && N <= M;
}

int small_init(fftconv_plan *p)
{
    const FacList fl = small_factor_list(p->M);
    p->f3.N1 = fl.fac[0];
    p->f3.N2 = fl.fac[1];
    p->f3.N3 = fl.fac[2];
    return FFTCONV_OK;
}

size_t small_kf_bytes(const fftconv_plan *p) { return (size_t)(p->H * p->M) * sizeof(float2); }

}  // namespace fftconv
