// Multi-pass causal FFT convolution for transforms too long to keep on chip
// (paper Algorithm 4 and Section 3.1 "Kernel Fusion": the outermost matrix
// operation of the forward and of the inverse transform takes one trip through
// HBM each, everything inside stays fused).  16-bit I/O, fft_size M = No * Mi with
// Mi = 8192 (the fused inner transform) and No = M / Mi in [1, 512].  Causal shapes (N <= M/2)
// of the sizes the single-kernel paths do not take, and every shape with N > M/2 (circular
// convolution, Section 2.1: the input fills the transform) from M = 8192 up: the kernels are
// instantiated with and without the implicit zero half (FULLN).  No = 1 has no outer transform:
// pass A only packs a pair of rows into a complex row, pass C unpacks it.
//
// Index maps: time n = no*Mi + r, frequency f = ko + No*f'.  Then
//   W_M^{n f} = W_No^{no ko} * W_M^{r ko} * W_Mi^{r f'},
// so, with z = u[b] + i*u[b+1] (two batch rows share one complex transform because the
// filter is real),
//   pass A:  S[ko, r] = W_M^{r ko} * sum_{no < No/2} z[no*Mi + r] W_No^{no ko}     (zeros for no >= No/2
//            are implicit; the listing in the paper omits the twiddle, its prose names it)
//   pass B:  every row S[ko, :] is circularly convolved (length Mi, complex in / complex out,
//            fused kernel) with the spectrum row k_f[ko + No*f'] / M
//   pass C:  y[no*Mi + r] = sum_{ko} conj(W_M^{r ko} W_No^{no ko}) S[ko, r] / boost,  no < No/2;
//            real part -> row b, imaginary part -> row b+1.
// S lives in the caller's workspace as 16-bit (re, im) pairs, M per pair of rows, and is
// rewritten in place by pass B.  The outer DFT of length No is itself split in two
// (No = Ra * Rb, Ra = min(16, No)) inside one workgroup: in-register radix-2 butterflies on the
// vector ALUs in fp32, one thread per column, so HBM sees rows of consecutive columns.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "dft_reg.h"
#include "fftconv_internal.h"
#include "fused3_common.h"

#include <mutex>

namespace fftconv {

// ---- workspace for callers that cannot allocate (fftconv_forward_static): one array per GPU, part of the
// library's device image, held until the process ends.  Host code never uses the array's name as an
// address: static_workspace_init() asks the runtime for the array's device address once per device and
// every later use goes through that pointer.
static __device__ __align__(256) unsigned char scratch[FFTCONV_STATIC_WORKSPACE_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
void *g_scratch_ptr[MAX_DEVICES] = {};          // device address of `scratch` on each device, nullptr = not asked yet
std::mutex g_scratch_mu;
}  // namespace

// with `device` current; called from plan creation
int static_workspace_init(int device)
{
    if (device < 0 || device >= MAX_DEVICES) {
        set_error("static workspace: device index %d out of range", device);
        return FFTCONV_EUNSUPPORTED;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return FFTCONV_OK;
    void *ptr = nullptr;
    FC_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    g_scratch_ptr[device] = ptr;
    return FFTCONV_OK;
}

void *static_workspace(int device)
{
    if (device < 0 || device >= MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return g_scratch_ptr[device];
}

namespace {

constexpr int MI = 8192;
constexpr int TB = 512;          // threads per block of the outer passes

__device__ __forceinline__ float2 cmulf(float2 a, float2 b)
{
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cmulcf(float2 a, float2 b)      // a * conj(b)
{
    return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
// exp(-2 pi i rev), 0 <= rev < 1.  The exponents of W_M, M <= 2^22, are exact in fp32 revolutions, products of them included, and go
// straight to the hardware sine and cosine, which take their argument in revolutions (two quarter-rate instructions
// instead of the ~25 of the library routine).  Their absolute error over every e / 2^22 measures 1.3e-7, far
// below the 16-bit roundings of the values these twiddles multiply.
__device__ __forceinline__ float2 wrev(float rev)
{
    return make_float2(__builtin_amdgcn_cosf(rev), -__builtin_amdgcn_sinf(rev));
}

template <bool F16> __device__ __forceinline__ uint16_t cv16(float v)
{
    if constexpr (F16) {
        __half hv = __float2half_rn(v);
        return *(uint16_t *)&hv;
    } else {
        __hip_bfloat16 bv = __float2bfloat16(v);
        return *(uint16_t *)&bv;
    }
}
template <bool F16> __device__ __forceinline__ float2 unpack2(uint32_t w)
{
    if constexpr (F16) {
        __half2 hv = *(__half2 *)&w;
        return make_float2(__low2float(hv), __high2float(hv));
    } else {
        return make_float2(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
    }
}

// half v (0, 1) of a packed pair
template <bool F16> __device__ __forceinline__ float half_of(uint32_t w, int v)
{
    if constexpr (F16) return __half2float(__builtin_bit_cast(__half, (uint16_t)(v ? w >> 16 : w)));
    else return __uint_as_float(v ? w & 0xffff0000u : w << 16);
}
template <bool F16> __device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    if constexpr (F16) return (uint32_t)cv16<true>(lo) | ((uint32_t)cv16<true>(hi) << 16);
    else return f3::BF16::pack(lo, hi);
}

// An access `bytes` beyond an address that is the same for every thread: a 32-bit offset of the load or store, where an index into the
// array costs two 64-bit operations for each (rows of these passes are fewer than 2^31 bytes).
template <typename T> __device__ __forceinline__ T ld_at(const void *base, uint32_t bytes) { return *(const T *)((const char *)base + bytes); }
// Two 16-bit samples n, n + 1 of a row of N >= 2, wherever the row lies (a 4-byte access needs 2-byte alignment here); what lies
// beyond its end reads as zeros, and nothing beyond it is touched: there the row's last pair is fetched, unconditionally, so that
// a thread's loads go out back to back, and pair_of() moves its second half down or drops it.  (A row of one sample: that in the second half.)
struct __attribute__((packed, aligned(2))) Word { uint32_t w; };
__device__ __forceinline__ uint32_t ld_pair(const uint16_t *row, int n, int N) { return ld_at<Word>(row, 2u * (uint32_t)min(n, N - 2)).w; }
__device__ __forceinline__ uint32_t pair_of(uint32_t w, int n, int N) { return n >= N ? 0 : n == N - 1 ? w >> 16 : w; }
template <typename T> __device__ __forceinline__ void st_at(void *base, uint32_t bytes, T v) { *(T *)((char *)base + bytes) = v; }

// elementwise product of two packed pairs of 16-bit values, each product rounded to the I/O dtype (the
// gates of the gated form, Section 3.1: the rounded product is what the transform consumes / what is stored)
template <bool F16> __device__ __forceinline__ uint32_t mul_pair16(uint32_t a, uint32_t b)
{
    const float2 x = unpack2<F16>(a), g = unpack2<F16>(b);
    return pack2<F16>(x.x * g.x, x.y * g.y);
}

// columns per block of the passes with a tile, No = RA RB > 16: an fp32 tile T[No][.] of 64 KiB (two blocks per compute unit), at least 32
template <int RA, int RB> constexpr int TILE_COLS = MI / (RA * RB) < 32 ? 32 : MI / (RA * RB);

struct OuterGeo {
    int No, Ra, Rb, CT;          // outer length, its two factors, columns per block
    // of the passes over real rows: column pairs per block (the same tile), and the tile's bytes
    int pairs() const { return Rb == 1 ? CT / 2 : CT; }
    size_t lds() const { return Rb == 1 ? 0 : sizeof(float2) * ((size_t)No + (size_t)No * CT); }
};

// ---- pass A: zero-padded pair of real rows -> outer forward DFT (No = RA * RB) -> twiddle -> S.
// One block = CT consecutive columns r of one (pair, channel); one thread = CV adjacent columns of
// one butterfly, so that 16-bit input moves as 2*CV-byte and S as 4*CV-byte accesses.
// Step 1: for every b2 < RB the length-RA transform over a (unless FULLN, inputs a >= RA/2 are the
// implicit zeros), times W_No^{ka b2}, into the fp32 LDS tile T[ka*RB + b2][c].  Step 2: for every ka the
// length-RB transform over b2, times W_M^{r ko} (ko = ka + RA kb, by recurrence over kb), to S.
// RB == 1 (No <= 16; all six outer kernels): a thread reads every outer row of its two columns, transforms them in registers
// and writes every row; no tile, no barrier, 8 or 16 loads of a thread in flight instead of one per trip of a loop.  Bound by
// the copy of the bytes.  Same operations on the same values as through the tile.  us, before and after: fft 131072, 2 x 256 x 65536
// bf16: pass A 54 -> 40 (201 MB), pass C 67 -> 52 (40 with fewer threads, see there), gradient: rows of u and dy 39 -> 36 each, last pass 56 -> 37; fft 32768,
// 5 x 256 x 10007: A 29 -> 21, C 30 -> 17, lone row 13 -> 9 and 13 -> 8.
// RB > 1: bound by the vector ALU, whose instructions a wave issues every four clocks: 924 of a thread took 112 us of 2^21 points, 64 rows.
// Hence constant tile shapes (LDS and row offsets are immediates or scalars), twiddle angles as exact products in fp32, pairs packed by one
// conversion, no masks where nothing is masked: 690.  us: bf16 2^21, 1 x 64 rows 390 -> 366; circular 2 x 128 x 2^19 402 -> 358,
// 2 x 256 x 2^18 420 -> 383, 1 x 256 x 2^17 (fft 2^18) 218 -> 195.
// N odd, or rows that start off a 4-byte boundary: pairs are fetched and stored as unaligned words (ld_pair()); a load behind a branch for
// every sample before: gated 2 x 64 x 400001 639 -> 444 us, 3 x 64 x 200001 330 -> 262, 2 x 64 x 100001 104 -> 84.
// EXACT (all four outer kernels): N is even and equals the input length the instantiation is for (M/2, or M
// with FULLN), so every load of u and store of y is in range, 4-byte aligned and unconditional: the compiler
// can then issue a thread's loads back to back instead of one guarded load at a time.
// RB > 1: butterflies with the product first.  As chained multiply-adds they cost the passes of full-length rows their last
// registers (28 - 40 bytes of scratch; 2 x 192 x 2^18 circular bf16 333 -> 352 us, 334 so; 2 x 48 x 2^20 334 - 342 -> 362, 342).
template <bool F16, int RA, int RB, int CV, bool FULLN, bool GATED, bool EXACT>
__global__ void __launch_bounds__(TB, 4) k_outer_fwd(const uint16_t *__restrict__ u, uint32_t *__restrict__ S, int ct,
                                                 int B, int H, int N, int ko_lo, int ko_hi,
                                                 const uint16_t *__restrict__ wg, LaunchGate gate)
{
    extern __shared__ float2 sm[];
    if (gate_closed(gate)) return;
    constexpr int No = RA * RB;
    constexpr Butterfly FORM = RB > 1 ? PRODUCT : EIGHT;
    constexpr int RAIN = FULLN ? RA : RA / 2;      // outer rows that can hold input
    float2 *wno = sm;                              // W_No^j, j < No
    float2 *T = sm + No;                           // [No][CT]
    const int CT = RB > 1 ? TILE_COLS<RA, RB> : ct;
    const int tid = threadIdx.x;
    const int r0 = blockIdx.x * CT;
    const int ph = blockIdx.y;                     // pair * H + h
    const int pair = ph / H, h = ph % H;
    const int b0 = 2 * pair;
    const bool two = b0 + 1 < B;
    const uint16_t *row0 = u + ((size_t)b0 * H + h) * N;
    const uint16_t *row1 = u + ((size_t)(b0 + (two ? 1 : 0)) * H + h) * N;
    // input gate of the gated form (same shape as u), multiplied in as the samples arrive; nullptr = none
    const uint16_t *g0 = GATED ? wg + ((size_t)b0 * H + h) * N : nullptr;
    const uint16_t *g1 = GATED ? wg + ((size_t)(b0 + (two ? 1 : 0)) * H + h) * N : nullptr;
    auto load = [&](const uint16_t *row, int n) -> uint32_t {
        if constexpr (CV == 1) return ld_at<uint16_t>(row, EXACT || n < N ? 2 * n : 0);
        else if constexpr (EXACT) return ld_at<uint32_t>(row, 2 * n);
        else return ld_pair(row, n, N);
    };
    auto kept = [&](uint32_t w, int n) -> uint32_t {
        if constexpr (EXACT) return w;
        else if constexpr (CV == 1) return n < N ? w : 0;
        else return pair_of(w, n, N);
    };
    const int CG = CT / CV;                        // column groups, a power of two
    const int lgCG = 31 - __builtin_clz(CG);
    if constexpr (RB > 1) {
        for (int j = tid; j < No; j += TB) wno[j] = wrev((float)j * (1.0f / (float)No));
        __syncthreads();
    }
    constexpr float im = 1.0f / (float)((int64_t)No * MI);       // exact, and so are r ko / M (r < 8192, ko < 512)
#pragma unroll 1
    for (int e = tid; e < RB * CG; e += TB) {
        const int c = (e & (CG - 1)) * CV, b2 = e >> lgCG;
        uint32_t in0[RAIN], in1[RAIN];             // CV 16-bit values of row b / row b+1
        uint32_t gt0[GATED ? RAIN : 1], gt1[GATED ? RAIN : 1];
        // (a missing row b+1 reads row b)
        if (EXACT || CV == 1 || N > 1) {
#pragma unroll
            for (int a = 0; a < RAIN; ++a) {
                const int n = (a * RB + b2) * MI + r0 + c;
                in0[a] = load(row0, n);
                in1[a] = load(row1, n);
                if constexpr (GATED) {
                    gt0[a] = load(g0, n);
                    gt1[a] = load(g1, n);
                }
            }
        } else {
#pragma unroll
            for (int a = 0; a < RAIN; ++a) {
                in0[a] = (uint32_t)row0[0] << 16;
                in1[a] = (uint32_t)row1[0] << 16;
                if constexpr (GATED) {
                    gt0[a] = (uint32_t)g0[0] << 16;
                    gt1[a] = (uint32_t)g1[0] << 16;
                }
            }
        }
#pragma unroll
        for (int a = 0; a < RAIN; ++a) {
            asm volatile("" ::"v"(in0[a]), "v"(in1[a]));                 // keeps the loads unconditional
            if constexpr (GATED) asm volatile("" ::"v"(gt0[a]), "v"(gt1[a]));
        }
#pragma unroll
        for (int a = 0; a < RAIN; ++a) {
            const int n = (a * RB + b2) * MI + r0 + c;
            in0[a] = kept(in0[a], n);
            in1[a] = two ? kept(in1[a], n) : 0;
            if constexpr (GATED) {                                        // (0 times a discarded gate must stay 0)
                gt0[a] = kept(gt0[a], n);
                gt1[a] = two ? kept(gt1[a], n) : 0;
            }
        }
        if constexpr (GATED) {
#pragma unroll
            for (int a = 0; a < RAIN; ++a) {
                in0[a] = mul_pair16<F16>(in0[a], gt0[a]);
                in1[a] = mul_pair16<F16>(in1[a], gt1[a]);
            }
        }
        if constexpr (RB == 1) {
            uint32_t o[RA][CV];
#pragma unroll
            for (int v = 0; v < CV; ++v) {
                float2 x[RA];
#pragma unroll
                for (int a = 0; a < RA; ++a) {
                    x[a] = make_float2(0.f, 0.f);
                    if (a < RAIN) x[a] = make_float2(half_of<F16>(in0[a], v), half_of<F16>(in1[a], v));
                }
                dft_reg<RA, false, !FULLN, FORM>(x);
                const float rf = (float)(r0 + c + v);
#pragma unroll
                for (int ka = 0; ka < RA; ++ka) {
                    const float2 t = cmulf(x[ka], wrev(rf * ((float)ka * im)));
                    o[ka][v] = pack2<F16>(t.x, t.y);
                }
            }
            const uint32_t at = 4u * (uint32_t)multipass_row_slot(r0 + c, multipass_quarter_rows(No));
#pragma unroll
            for (int ka = 0; ka < RA; ++ka)
                if (ko_lo >= ko_hi || ka < ko_lo || ka >= ko_hi) {        // (a zeroed part of the spectrum is never used)
                    uint32_t *const dst = S + ((size_t)ph * No + ka) * MI;
                    if constexpr (CV == 2) st_at(dst, at, make_uint2(o[ka][0], o[ka][1]));
                    else st_at(dst, at, o[ka][0]);
                }
            continue;
        }
        float2 o[RA][CV];
#pragma unroll
        for (int v = 0; v < CV; ++v) {
            float2 x[RA];
#pragma unroll
            for (int a = 0; a < RA; ++a) {
                x[a] = make_float2(0.f, 0.f);
                if (a < RAIN)                                        // (row b, row b+1) = (re, im)
                    x[a] = make_float2(half_of<F16>(in0[a], v), half_of<F16>(in1[a], v));
            }
            dft_reg<RA, false, !FULLN, FORM>(x);
#pragma unroll
            for (int ka = 0; ka < RA; ++ka) o[ka][v] = cmulf(x[ka], wno[ka * b2]);
        }
#pragma unroll
        for (int ka = 0; ka < RA; ++ka) {
            float2 *dst = &T[(ka * RB + b2) * CT + c];
            if constexpr (CV == 2)
                *(float4 *)dst = make_float4(o[ka][0].x, o[ka][0].y, o[ka][1].x, o[ka][1].y);
            else
                *dst = o[ka][0];
        }
    }
    if constexpr (RB == 1) return;
    __syncthreads();
#pragma unroll 1
    for (int e = tid; e < RA * CG; e += TB) {
        const int c = (e & (CG - 1)) * CV, ka = e >> lgCG;
        uint32_t o[RB][CV];
#pragma unroll
        for (int v = 0; v < CV; ++v) {
            float2 x[RB];
#pragma unroll
            for (int b2 = 0; b2 < RB; ++b2) x[b2] = T[(ka * RB + b2) * CT + c + v];
            dft_reg<RB, false, false, FORM>(x);
            const float rf = (float)(r0 + c + v);
            float2 w = wrev(rf * ((float)ka * im));                 // W_M^{r ka}
            const float2 step = wrev(rf * ((float)RA * im));        // W_M^{r RA}
#pragma unroll
            for (int kb = 0; kb < RB; ++kb) {
                const float2 t = cmulf(x[kb], w);
                o[kb][v] = pack2<F16>(t.x, t.y);
                w = cmulf(w, step);
            }
        }
        const uint32_t at = 4u * (uint32_t)(ka * MI + multipass_row_slot(r0 + c, multipass_quarter_rows(No)));
        auto put = [&](int kb) {
            uint32_t *const dst = S + ((size_t)ph * No + RA * kb) * MI;
            if constexpr (CV == 2) st_at(dst, at, make_uint2(o[kb][0], o[kb][1]));
            else st_at(dst, at, o[kb][0]);
        };
        if (ko_lo >= ko_hi) {                             // dense: unconditional stores, back to back
#pragma unroll
            for (int kb = 0; kb < RB; ++kb) put(kb);
        } else {
            // frequency-sparse filter: rows of a zeroed part of the spectrum are never used
#pragma unroll
            for (int kb = 0; kb < RB; ++kb) {
                const int ko = ka + RA * kb;
                if (ko < ko_lo || ko >= ko_hi) put(kb);
            }
        }
    }
}

// ---- pass C: S -> conjugate twiddle -> outer inverse DFT -> the two real rows of the pair
// No = 8 and 16: 16 rows of two columns, their transform and the packed results do not fit into the 128 registers of four waves per SIMD,
// and blocks of half the threads can be three: bf16 2 x 256 x 65536 (fft 131072) 157 -> 145 us, 8 x 64 x 30001 157 -> 137 (as many
// threads less at 128 registers: no difference).  Shorter ones fit, and smaller blocks cost them: 8 x 512 x 1321 (fft 8192) 66 -> 71.
template <int RA, int RB> constexpr int INV_TB = RB == 1 && RA >= 8 ? TB / 2 : TB;
template <int RA, int RB> constexpr int INV_WAVES = RB == 1 && RA >= 8 ? 3 : 4;
template <bool F16, int RA, int RB, int CV, bool FULLN, bool GATED, bool MIRROR, bool EXACT>
__global__ void __launch_bounds__((INV_TB<RA, RB>), (INV_WAVES<RA, RB>)) k_outer_inv(const uint32_t *__restrict__ S, uint16_t *__restrict__ y, int ct,
                                                 int B, int H, int N, int ko_lo, int ko_hi,
                                                 const uint16_t *__restrict__ vg, LaunchGate gate)
{
    extern __shared__ float2 sm[];
    if (gate_closed(gate)) return;
    constexpr int No = RA * RB;
    constexpr Butterfly FORM = RB > 1 ? PRODUCT : EIGHT;
    constexpr int RAIN = FULLN ? RA : RA / 2;      // outer rows that are kept
    float2 *wno = sm;
    float2 *T = sm + No;                           // [No][CT]
    const int CT = RB > 1 ? TILE_COLS<RA, RB> : ct;
    const int tid = threadIdx.x;
    const int r0 = blockIdx.x * CT;
    const int ph = blockIdx.y;
    const int pair = ph / H, h = ph % H;
    const int b0 = 2 * pair;
    const bool two = b0 + 1 < B;
    const int CG = CT / CV;
    const int lgCG = 31 - __builtin_clz(CG);
    if constexpr (RB > 1) {
        for (int j = tid; j < No; j += INV_TB<RA, RB>) wno[j] = wrev((float)j * (1.0f / (float)No));
        __syncthreads();
    }
    constexpr float im = 1.0f / (float)((int64_t)No * MI);       // exact, and so are r ko / M (r < 8192, ko < 512)
    // step 1: T[ka*RB + b2] = conj(W_No^{ka b2}) * sum_{kb} conj(W_RB^{b2 kb}) conj(W_M^{r ko}) S[ko], ko = ka + RA kb
    // MIRROR: rows ko > No/2 were never computed (a lone real row, see multipass_forward): before the
    // twiddle row ko is the complex conjugate of row ko' = No - ko, i.e.
    //   conj(W_M^{r ko}) S[ko] = conj(conj(W_M^{r ko'}) S[ko']),   W_M^{r ko'} = W_Mi^{r} conj(W_M^{r ko}),
    // so the value that enters the inverse is conj(S[ko']) conj(conj(W_Mi^{r}) W_M^{r ko}): the mirror row is
    // read and conjugated (a sign flip on the packed word), and from the first mirrored row on the twiddle of the
    // recurrence carries the extra factor conj(W_Mi^{r}).
#pragma unroll 1
    for (int e = tid; RB > 1 && e < RA * CG; e += INV_TB<RA, RB>) {
        const int c = (e & (CG - 1)) * CV, ka = e >> lgCG;
        // the row that holds ko: itself, or with MIRROR from ko > No/2 on row No - ko, which the thread decides only at kb == RB/2;
        // `up` or `down` beyond a row that is the same for every thread
        const uint32_t slot = 4u * (uint32_t)multipass_row_slot(r0 + c, multipass_quarter_rows(No));
        const uint32_t up = 4u * (uint32_t)(ka * MI) + slot, down = 4u * (uint32_t)((RA - ka) * MI) + slot;
        const uint32_t *const src = S + (size_t)ph * No * MI;
        auto get = [&](uint32_t (&w)[CV], const uint32_t *base, uint32_t at) {
            if constexpr (CV == 2) {
                const uint2 t = ld_at<uint2>(base, at);
                w[0] = t.x;
                w[1] = t.y;
            } else {
                w[0] = ld_at<uint32_t>(base, at);
            }
        };
        uint32_t in[RB][CV];
        if (ko_lo >= ko_hi || ko_lo >= No) {
#pragma unroll
            for (int kb = 0; kb < RB; ++kb) {
                if (MIRROR && kb >= RB / 2) get(in[kb], src + (kb > RB / 2 ? RB - 1 - kb : RB / 2 - 1) * RA * MI, down);
                else get(in[kb], src + kb * RA * MI, up);
            }
        } else {
            // zeroed part of the spectrum (never with MIRROR): the row counts as zero and was never written.  The load stays
            // unconditional (of row 0 instead, its value discarded), so that a thread's loads go out back to
            // back: behind a branch each of them would be waited for before the next is issued.
            auto dead = [&](int kb) { return ka + RA * kb >= ko_lo && ka + RA * kb < ko_hi; };
#pragma unroll
            for (int kb = 0; kb < RB; ++kb) get(in[kb], src, dead(kb) ? slot : up + 4u * (uint32_t)(kb * RA * MI));
            // (an empty statement that reads the loaded words: without it the compiler moves each load back under its
            //  condition)
#pragma unroll
            for (int kb = 0; kb < RB; ++kb)
#pragma unroll
                for (int v = 0; v < CV; ++v) asm volatile("" ::"v"(in[kb][v]));
#pragma unroll
            for (int kb = 0; kb < RB; ++kb)
#pragma unroll
                for (int v = 0; v < CV; ++v)
                    if (dead(kb)) in[kb][v] = 0;
        }
        if constexpr (MIRROR) {                               // conjugate: the imaginary part is the upper half
#pragma unroll
            for (int kb = RB / 2; kb < RB; ++kb)
                if (kb > RB / 2 || ka > 0) {
#pragma unroll
                    for (int v = 0; v < CV; ++v) in[kb][v] ^= 0x80000000u;
                }
        }
        float2 o[RB][CV];
#pragma unroll
        for (int v = 0; v < CV; ++v) {
            const float rf = (float)(r0 + c + v);
            float2 w = wrev(rf * ((float)ka * im));
            const float2 step = wrev(rf * ((float)RA * im));
            constexpr float unboost = 1.0f / (float)multipass_kf_boost(F16, No);     // exact: a power of two
            w.x *= unboost;
            w.y *= unboost;
            float2 x[RB];
#pragma unroll
            for (int kb = 0; kb < RB; ++kb) {
                // the first mirrored row of this thread: kb = RB/2 (ka > 0) or RB/2 + 1 (ka == 0)
                const bool first_mirrored = RB == 1 ? ka > RA / 2
                                                    : ((kb == RB / 2 && ka > 0) || (kb == RB / 2 + 1 && ka == 0));
                if (MIRROR && first_mirrored)
                    w = cmulcf(w, wrev(rf * (1.0f / (float)MI)));        // times conj(W_Mi^{r}), once
                x[kb] = cmulcf(unpack2<F16>(in[kb][v]), w);
                w = cmulf(w, step);
            }
            dft_reg<RB, true, false, FORM>(x);
#pragma unroll
            for (int b2 = 0; b2 < RB; ++b2) o[b2][v] = cmulcf(x[b2], wno[ka * b2]);
        }
#pragma unroll
        for (int b2 = 0; b2 < RB; ++b2) {
            float2 *dst = &T[(ka * RB + b2) * CT + c];
            if constexpr (CV == 2)
                *(float4 *)dst = make_float4(o[b2][0].x, o[b2][0].y, o[b2][1].x, o[b2][1].y);
            else
                *dst = o[b2][0];
        }
    }
    if constexpr (RB > 1) __syncthreads();
    // step 2: z[a*RB + b2] = sum_{ka} conj(W_RA^{a ka}) T[ka*RB + b2], kept for a < RAIN (n < M/2 unless FULLN)
    uint16_t *row0 = y + ((size_t)b0 * H + h) * N;
    uint16_t *row1 = y + ((size_t)(b0 + (two ? 1 : 0)) * H + h) * N;
    // output gate of the gated form: multiplies the result after its rounding to the I/O dtype; nullptr = none
    const uint16_t *g0 = GATED ? vg + ((size_t)b0 * H + h) * N : nullptr;
    const uint16_t *g1 = GATED ? vg + ((size_t)(b0 + (two ? 1 : 0)) * H + h) * N : nullptr;
#pragma unroll 1
    for (int e = tid; e < RB * CG; e += INV_TB<RA, RB>) {
        const int c = (e & (CG - 1)) * CV, b2 = e >> lgCG;
        // RB == 1: a thread reads all rows of its columns and no tile lies in between
        uint32_t in[RB == 1 ? RA : 1][CV];
        if constexpr (RB == 1) {
            auto mirrored = [](int ka) { return MIRROR && ka > RA / 2; };
            auto dead = [&](int ka) { return ka >= ko_lo && ka < ko_hi; };
#pragma unroll
            for (int ka = 0; ka < RA; ++ka) {
                const uint32_t *src = &S[((size_t)ph * No + (dead(ka) ? 0 : (mirrored(ka) ? No - ka : ka))) * MI +
                                         multipass_row_slot(r0 + c, multipass_quarter_rows(No))];
                if constexpr (CV == 2) {
                    const uint2 t = *(const uint2 *)src;
                    in[ka][0] = t.x;
                    in[ka][1] = t.y;
                } else {
                    in[ka][0] = *src;
                }
            }
#pragma unroll
            for (int ka = 0; ka < RA; ++ka)
#pragma unroll
                for (int v = 0; v < CV; ++v) asm volatile("" ::"v"(in[ka][v]));
#pragma unroll
            for (int ka = 0; ka < RA; ++ka)
#pragma unroll
                for (int v = 0; v < CV; ++v) {
                    if (dead(ka)) in[ka][v] = 0;
                    if (mirrored(ka)) in[ka][v] ^= 0x80000000u;
                }
        }
        uint32_t o0[RAIN], o1[RAIN];
        float2 left[CV == 2 ? RAIN : 1];           // the even column's results, until the odd one's are there
#pragma unroll
        for (int v = 0; v < CV; ++v) {
            float2 x[RA];
#pragma unroll
            for (int ka = 0; ka < RA; ++ka) {
                if constexpr (RB == 1) {
                    constexpr float unboost = 1.0f / (float)multipass_kf_boost(F16, No);     // exact: a power of two
                    const float rf = (float)(r0 + c + v);
                    float2 w = wrev(rf * ((float)ka * im));
                    w.x *= unboost;
                    w.y *= unboost;
                    if (MIRROR && ka > RA / 2) w = cmulcf(w, wrev(rf * (1.0f / (float)MI)));
                    x[ka] = cmulcf(unpack2<F16>(in[ka][v]), w);
                } else {
                    x[ka] = T[(ka * RB + b2) * CT + c + v];
                }
            }
            dft_reg<RA, true, false, FORM>(x);
#pragma unroll
            for (int a = 0; a < RAIN; ++a) {
                if (v == CV - 1) {
                    o0[a] = CV == 2 ? pack2<F16>(left[CV == 2 ? a : 0].x, x[a].x) : (uint32_t)cv16<F16>(x[a].x);
                    o1[a] = CV == 2 ? pack2<F16>(left[CV == 2 ? a : 0].y, x[a].y) : (uint32_t)cv16<F16>(x[a].y);
                } else {
                    left[a] = x[a];
                }
            }
        }
#pragma unroll
        for (int a = 0; a < RAIN; ++a) {
            const int n = (a * RB + b2) * MI + r0 + c;
            const uint32_t at = 2 * n;
            if (CV == 2 && (EXACT || n + 1 < N)) {
                if constexpr (GATED) {
                    o0[a] = mul_pair16<F16>(o0[a], ld_at<Word>(g0, at).w);
                    if (two) o1[a] = mul_pair16<F16>(o1[a], ld_at<Word>(g1, at).w);
                }
                st_at(row0, at, Word{o0[a]});
                if (two) st_at(row1, at, Word{o1[a]});
            } else if (EXACT || n < N) {                                  // one column, or the last sample of an odd row
                if constexpr (GATED) {
                    o0[a] = mul_pair16<F16>(o0[a], ld_at<uint16_t>(g0, at));
                    if (two) o1[a] = mul_pair16<F16>(o1[a], ld_at<uint16_t>(g1, at));
                }
                st_at(row0, at, (uint16_t)o0[a]);
                if (two) st_at(row1, at, (uint16_t)o1[a]);
            }
        }
    }
}

// ---- the outer passes of a LONE real row (B = 1, or the last row of an odd batch): two adjacent columns of
// the real row share one complex outer transform, z[no] = x[no, c] + i x[no, c+1] (Appendix A.1's point that a
// real transform costs half a complex one, taken on the column pairs of the outer factor), and only the
// outer frequencies ko <= No/2 are kept (the others are their conjugates, see multipass_forward).
//   pass A:  Z = DFT_No(z);  X_c[ko] = (Z[ko] + conj Z[No-ko]) / 2,  X_{c+1}[ko] = (Z[ko] - conj Z[No-ko]) / (2i);
//            S[ko, r] = W_M^{r ko} X_r[ko] for ko <= No/2.
//   pass C:  U_r[ko] = conj(W_M^{r ko}) S[ko, r] (ko <= No/2), U_r[ko] = conj(U_r[No-ko]) (ko > No/2);
//            z = IDFT_No(U_c + i U_{c+1}): its real part is column c of y, its imaginary part column c+1.
// One block = 2 CG consecutive columns of one channel, T[No][CG] in LDS; a 16-bit pair of adjacent samples
// is one 32-bit word, so a wave moves whole 128-byte lines of u and y.
template <bool F16, int RA, int RB, bool FULLN, bool GATED, bool EXACT>
__global__ void __launch_bounds__(TB, 4) k_outer_fwd_real(const uint16_t *__restrict__ u, uint32_t *__restrict__ S, int cgs,
                                                      int H, int N, int ko_lo, const uint16_t *__restrict__ wg,
                                                      LaunchGate gate)
{
    extern __shared__ float2 sm[];
    if (gate_closed(gate)) return;
    constexpr int No = RA * RB;
    constexpr int RAIN = FULLN ? RA : RA / 2;      // outer rows that can hold input
    float2 *wno = sm;                              // W_No^j, j < No
    float2 *T = sm + No;                           // [No][CG]
    const int CG = RB > 1 ? TILE_COLS<RA, RB> : cgs;
    const int tid = threadIdx.x;
    const int r0 = blockIdx.x * 2 * CG;
    const int lgCG = 31 - __builtin_clz(CG);       // CG is a power of two
    const int h = blockIdx.y;
    const uint16_t *row0 = u + (size_t)h * N;
    const uint16_t *g0 = GATED ? wg + (size_t)h * N : nullptr;
    if constexpr (RB > 1) {
        for (int j = tid; j < No; j += TB) wno[j] = wrev((float)j * (1.0f / (float)No));
        __syncthreads();
    }
    constexpr float im = 1.0f / (float)((int64_t)No * MI);       // exact, and so are r ko / M (r < 8192, ko < 512)
    // step 1: length-RA transforms over a, times W_No^{ka b2}
#pragma unroll 1
    for (int e = tid; e < RB * CG; e += TB) {
        const int cg = e & (CG - 1), b2 = e >> lgCG;
        float2 x[RA];
        uint32_t wd[RAIN], gt[GATED ? RAIN : 1];
        if (EXACT || N > 1) {
#pragma unroll
            for (int a = 0; a < RAIN; ++a) {
                const int n = (a * RB + b2) * MI + r0 + 2 * cg;
                wd[a] = EXACT ? ld_at<uint32_t>(row0, 2 * n) : ld_pair(row0, n, N);
                if constexpr (GATED) gt[a] = EXACT ? ld_at<uint32_t>(g0, 2 * n) : ld_pair(g0, n, N);
            }
        } else {
#pragma unroll
            for (int a = 0; a < RAIN; ++a) {
                wd[a] = (uint32_t)row0[0] << 16;
                if constexpr (GATED) gt[a] = (uint32_t)g0[0] << 16;
            }
        }
        if constexpr (!EXACT) {
#pragma unroll
            for (int a = 0; a < RAIN; ++a) {
                asm volatile("" ::"v"(wd[a]));                           // keeps the loads unconditional
                if constexpr (GATED) asm volatile("" ::"v"(gt[a]));
            }
#pragma unroll
            for (int a = 0; a < RAIN; ++a) {
                const int n = (a * RB + b2) * MI + r0 + 2 * cg;
                wd[a] = pair_of(wd[a], n, N);
                if constexpr (GATED) gt[a] = pair_of(gt[a], n, N);       // (0 times a discarded gate must stay 0)
            }
        }
#pragma unroll
        for (int a = 0; a < RA; ++a) {
            x[a] = make_float2(0.f, 0.f);
            if (a < RAIN) {
                if constexpr (GATED) wd[a] = mul_pair16<F16>(wd[a], gt[a]);
                x[a] = unpack2<F16>(wd[a]);        // (column c, column c+1) = (re, im)
            }
        }
        dft_reg<RA, false, !FULLN>(x);
        if constexpr (RB == 1) {                   // Z[ko] and its mirror row are both at hand
            const int r = r0 + 2 * cg;
            const float rf = (float)r;
#pragma unroll
            for (int ko = 0; ko <= No / 2; ++ko) {
                const float2 z = x[ko], zm = x[(No - ko) % No];
                const float2 xa = make_float2(0.5f * (z.x + zm.x), 0.5f * (z.y - zm.y));
                const float2 xb = make_float2(0.5f * (z.y + zm.y), -0.5f * (z.x - zm.x));
                const float2 ta = cmulf(xa, wrev(rf * ((float)ko * im))), tb = cmulf(xb, wrev((rf + 1.f) * ((float)ko * im)));
                if (ko < ko_lo)
                    *(uint2 *)&S[((size_t)h * No + ko) * MI + multipass_row_slot(r, multipass_quarter_rows(No))] =
                        make_uint2(pack2<F16>(ta.x, ta.y),
                                   pack2<F16>(tb.x, tb.y));
            }
            continue;
        }
#pragma unroll
        for (int ka = 0; ka < RA; ++ka) T[(ka * RB + b2) * CG + cg] = cmulf(x[ka], wno[ka * b2]);
    }
    if constexpr (RB == 1) return;
    __syncthreads();
    // step 2: length-RB transforms over b2, in place: slot ka*RB + kb then holds Z[ko], ko = ka + RA kb
#pragma unroll 1
    for (int e = tid; e < RA * CG; e += TB) {
        const int cg = e & (CG - 1), ka = e >> lgCG;
        float2 x[RB];
#pragma unroll
        for (int b2 = 0; b2 < RB; ++b2) x[b2] = T[(ka * RB + b2) * CG + cg];
        dft_reg<RB, false>(x);
#pragma unroll
        for (int kb = 0; kb < RB; ++kb) T[(ka * RB + kb) * CG + cg] = x[kb];
    }
    __syncthreads();
    // step 3: split the two columns, twiddle (by recurrence over kb), store the rows ko <= No/2 and below ko_lo (from there on
    // they only meet zeroed bins of a sparse filter)
    const int end = ko_lo < No / 2 + 1 ? ko_lo : No / 2 + 1;
#pragma unroll 1
    for (int e = tid; e < RA * CG; e += TB) {
        const int cg = e & (CG - 1), ka = e >> lgCG;
        const int r = r0 + 2 * cg;
        const float rf = (float)r;
        float2 z[RB / 2 + 1], zm[RB / 2 + 1];                      // ko = ka + RA kb <= No/2 needs kb <= RB/2
#pragma unroll
        for (int kb = 0; kb <= RB / 2; ++kb) {
            // row (No - ko) % No: kb' = RB - 1 - kb of ka' = RA - ka, or (RB - kb) % RB of ka' = 0
            const float2 *const m = T + (ka ? ((RA - ka) * RB + RB - 1 - kb) * CG : (RB - kb) % RB * CG);
            z[kb] = T[(ka * RB + kb) * CG + cg];
            zm[kb] = m[cg];
        }
        float2 w0 = wrev(rf * ((float)ka * im)), w1 = wrev((rf + 1.f) * ((float)ka * im));
        const float2 s0 = wrev(rf * ((float)RA * im)), s1 = wrev((rf + 1.f) * ((float)RA * im));
        w0.x *= 0.5f, w0.y *= 0.5f, w1.x *= 0.5f, w1.y *= 0.5f;
        uint32_t *const dst = S + (size_t)h * No * MI;
        const uint32_t at = 4u * (uint32_t)(ka * MI + multipass_row_slot(r, multipass_quarter_rows(No)));
#pragma unroll
        for (int kb = 0; kb <= RB / 2; ++kb) {
            if (ka + RA * kb < end) {
                const float2 xa = make_float2(z[kb].x + zm[kb].x, z[kb].y - zm[kb].y);        // Z + conj Zm (halved by the twiddle)
                const float2 xb = make_float2(z[kb].y + zm[kb].y, zm[kb].x - z[kb].x);        // (Z - conj Zm) / i
                const float2 ta = cmulf(xa, w0), tb = cmulf(xb, w1);
                st_at(dst + RA * kb * MI, at, make_uint2(pack2<F16>(ta.x, ta.y), pack2<F16>(tb.x, tb.y)));
            }
            w0 = cmulf(w0, s0);
            w1 = cmulf(w1, s1);
        }
    }
}

template <bool F16, int RA, int RB, bool FULLN, bool GATED, bool EXACT>
__global__ void __launch_bounds__(TB, 4) k_outer_inv_real(const uint32_t *__restrict__ S, uint16_t *__restrict__ y, int cgs,
                                                      int H, int N, int ko_lo, const uint16_t *__restrict__ vg,
                                                      LaunchGate gate)
{
    extern __shared__ float2 sm[];
    if (gate_closed(gate)) return;
    constexpr int No = RA * RB;
    constexpr int RAIN = FULLN ? RA : RA / 2;      // outer rows that are kept
    float2 *wno = sm;
    float2 *T = sm + No;                           // [No][CG]
    const int CG = RB > 1 ? TILE_COLS<RA, RB> : cgs;
    const int tid = threadIdx.x;
    const int r0 = blockIdx.x * 2 * CG;
    const int lgCG = 31 - __builtin_clz(CG);       // CG is a power of two
    const int h = blockIdx.y;
    if constexpr (RB > 1) {
        for (int j = tid; j < No; j += TB) wno[j] = wrev((float)j * (1.0f / (float)No));
        __syncthreads();
    }
    constexpr float im = 1.0f / (float)((int64_t)No * MI);       // exact, and so are r ko / M (r < 8192, ko < 512)
    constexpr float unboost = 1.0f / (float)multipass_kf_boost(F16, No);     // exact: a power of two
    // step 1: untwiddle both columns, complete the rows ko > No/2 from their mirror rows, combine the columns
    // into one complex sequence, length-RB inverse over kb, times conj(W_No^{ka b2})
#pragma unroll 1
    for (int e = tid; RB > 1 && e < RA * CG; e += TB) {
        const int cg = e & (CG - 1), ka = e >> lgCG;
        const int r = r0 + 2 * cg;
        const float rf = (float)r;
        // Row ko is held by itself or, beyond No/2, by its mirror row kr = No - ko; which of the two depends on the thread only at kb ==
        // RB/2.  Either lies `up` or `down` beyond a row that is the same for every thread.
        const uint32_t slot = 4u * (uint32_t)multipass_row_slot(r, multipass_quarter_rows(No));
        const uint32_t up = 4u * (uint32_t)(ka * MI) + slot, down = 4u * (uint32_t)((RA - ka) * MI) + slot;
        const uint32_t *const src = S + (size_t)h * No * MI;
        auto base = [&](int kb) { return src + (kb < RB / 2 ? kb : kb > RB / 2 ? RB - 1 - kb : RB / 2 - 1) * RA * MI; };
        uint2 in[RB];
        if (ko_lo > No / 2) {
#pragma unroll
            for (int kb = 0; kb < RB; ++kb) in[kb] = ld_at<uint2>(base(kb), kb < RB / 2 ? up : down);
        } else {
            // rows from ko_lo on: zeroed bins of a sparse filter, never written; they count as zero (the load stays
            // unconditional, of row 0 instead, see k_outer_inv)
            auto dead = [&](int kb) { return (kb < RB / 2 ? ka + RA * kb : RA * (RB - kb) - ka) >= ko_lo; };
#pragma unroll
            for (int kb = 0; kb < RB; ++kb) in[kb] = ld_at<uint2>(dead(kb) ? src : base(kb), dead(kb) ? slot : kb < RB / 2 ? up : down);
            // (an empty statement that reads the loaded words: without it the compiler moves each load back under its
            //  condition)
#pragma unroll
            for (int kb = 0; kb < RB; ++kb) asm volatile("" ::"v"(in[kb].x), "v"(in[kb].y));
#pragma unroll
            for (int kb = 0; kb < RB; ++kb)
                if (dead(kb)) in[kb] = make_uint2(0, 0);
        }
#pragma unroll
        for (int kb = RB / 2; kb < RB; ++kb)
            if (kb > RB / 2 || ka > 0) {                      // conjugate: the imaginary part is the upper half
                in[kb].x ^= 0x80000000u;
                in[kb].y ^= 0x80000000u;
            }
        float2 w0 = wrev(rf * ((float)ka * im)), w1 = wrev((rf + 1.f) * ((float)ka * im));
        const float2 s0 = wrev(rf * ((float)RA * im)), s1 = wrev((rf + 1.f) * ((float)RA * im));
        w0.x *= unboost, w0.y *= unboost, w1.x *= unboost, w1.y *= unboost;
        float2 x[RB];
#pragma unroll
        for (int kb = 0; kb < RB; ++kb) {
            // from the first mirrored row on the twiddle carries the extra factor conj(W_Mi^{r}) (see k_outer_inv)
            if ((kb == RB / 2 && ka > 0) || (kb == RB / 2 + 1 && ka == 0)) {
                w0 = cmulcf(w0, wrev(rf * (1.0f / (float)MI)));
                w1 = cmulcf(w1, wrev((rf + 1.f) * (1.0f / (float)MI)));
            }
            const float2 ua = cmulcf(unpack2<F16>(in[kb].x), w0), ub = cmulcf(unpack2<F16>(in[kb].y), w1);
            x[kb] = make_float2(ua.x - ub.y, ua.y + ub.x);               // U_c + i U_{c+1}
            w0 = cmulf(w0, s0);
            w1 = cmulf(w1, s1);
        }
        dft_reg<RB, true>(x);
#pragma unroll
        for (int b2 = 0; b2 < RB; ++b2) T[(ka * RB + b2) * CG + cg] = cmulcf(x[b2], wno[ka * b2]);
    }
    if constexpr (RB > 1) __syncthreads();
    // step 2: length-RA inverse over ka; real part -> column c, imaginary part -> column c+1
    uint16_t *row0 = y + (size_t)h * N;
    const uint16_t *g0 = GATED ? vg + (size_t)h * N : nullptr;
#pragma unroll 1
    for (int e = tid; e < RB * CG; e += TB) {
        const int cg = e & (CG - 1), b2 = e >> lgCG;
        float2 x[RA];
        if constexpr (RB == 1) {                   // every row <= No/2 is read once and serves its mirror row too
            const int r = r0 + 2 * cg;
            const float rf = (float)r;
            uint2 in[No / 2 + 1];
#pragma unroll
            for (int ko = 0; ko <= No / 2; ++ko)
                in[ko] = *(const uint2 *)&S[((size_t)h * No + (ko < ko_lo ? ko : 0)) * MI + multipass_row_slot(r, multipass_quarter_rows(No))];
#pragma unroll
            for (int ko = 0; ko <= No / 2; ++ko) asm volatile("" ::"v"(in[ko].x), "v"(in[ko].y));
            const float2 m0 = wrev(rf * (1.0f / (float)MI)), m1 = wrev((rf + 1.f) * (1.0f / (float)MI));
#pragma unroll
            for (int ka = 0; ka < RA; ++ka) {
                const bool mir = ka > RA / 2;
                const int kr = mir ? No - ka : ka;
                uint2 v = kr < ko_lo ? in[kr] : make_uint2(0, 0);
                if (mir) {
                    v.x ^= 0x80000000u;
                    v.y ^= 0x80000000u;
                }
                float2 w0 = wrev(rf * ((float)ka * im)), w1 = wrev((rf + 1.f) * ((float)ka * im));
                w0.x *= unboost, w0.y *= unboost, w1.x *= unboost, w1.y *= unboost;
                if (mir) {
                    w0 = cmulcf(w0, m0);
                    w1 = cmulcf(w1, m1);
                }
                const float2 ua = cmulcf(unpack2<F16>(v.x), w0), ub = cmulcf(unpack2<F16>(v.y), w1);
                x[ka] = make_float2(ua.x - ub.y, ua.y + ub.x);           // U_c + i U_{c+1}
            }
        } else {
#pragma unroll
            for (int ka = 0; ka < RA; ++ka) x[ka] = T[(ka * RB + b2) * CG + cg];
        }
        dft_reg<RA, true>(x);
#pragma unroll
        for (int a = 0; a < RAIN; ++a) {
            const int n = (a * RB + b2) * MI + r0 + 2 * cg;
            uint32_t o = pack2<F16>(x[a].x, x[a].y);
            if (EXACT || n + 1 < N) {
                if constexpr (GATED) o = mul_pair16<F16>(o, ld_at<Word>(g0, 2 * n).w);
                st_at(row0, 2 * n, Word{o});
            } else if (n < N) {                                           // the last sample of an odd row
                if constexpr (GATED) o = mul_pair16<F16>(o, ld_at<uint16_t>(g0, 2 * n));
                st_at(row0, 2 * n, (uint16_t)o);
            }
        }
    }
}

// ---- the outer pass of the FILTER transform of a multi-pass plan (fftconv_filter_fft: taps -> k_f): pass A of a
// lone real row (k_outer_fwd_real above) with fp32 taps in and fp32 rows out.  k_f holds 16-bit constants, so
// its transform runs in fp32 throughout: this kernel, then the 8192-point transform of every row in LDS
// (k_long_blocks_kf, long_fft.hip).  Rows ko <= No/2 only, T2[h][ko][r] (No/2 + 1 rows of 8192 fp32 pairs per
// channel): the taps are real, the other rows are mirror images that the second kernel writes from these.
// Taps at and beyond Nk are zeros (their loads read tap 0 and are discarded: no load sits behind a branch).
// The filter gradient of these plans (long_fft.hip) transforms its rows of u and dy the same way: IN = 0: fp32
// rows, 1: fp16, 2: bf16; row i of the launch is row rows.at(i) of its source, Nk elements each.
// GATED (fp32 convolutions; IN = 0): the rows are multiplied by those of gate, which lie alike.  As a kernel of its own that took as long as this pass:
// 7 x 2 x 2^19 circular fp32, both gates, 74 -> 53 us; 4 x 16 x 65536 fft 131072 70 -> 63.
template <int IN, int RA, int RB, bool FULLN, bool GATED>
__global__ void __launch_bounds__(TB, 4) k_filter_outer_real(OuterRows rows, float2 *__restrict__ T2, int cgs,
                                                         int64_t Nk, bool wide, const float *__restrict__ gate)
{
    extern __shared__ float2 sm[];
    constexpr int No = RA * RB, NR = No / 2 + 1;
    constexpr int RAIN = FULLN ? RA : RA / 2;      // outer rows that can hold taps
    float2 *wno = sm;                              // W_No^j, j < No
    float2 *T = sm + No;                           // [No][CG]
    const int CG = RB > 1 ? TILE_COLS<RA, RB> : cgs;
    const int tid = threadIdx.x;
    const int r0 = blockIdx.x * 2 * CG;
    const int lgCG = 31 - __builtin_clz(CG);       // CG is a power of two
    const int64_t h = blockIdx.y;
    const bool second = (int)blockIdx.y >= rows.split;
    const int at = (int)blockIdx.y - (second ? rows.split : 0);
    const void *const src = second ? rows.src2 : rows.src;
    const int64_t first = ((int64_t)(at / rows.nh) * rows.H + at % rows.nh) * Nk;
    const float *row0 = (const float *)src + first;                // IN == 0
    const uint16_t *row16 = (const uint16_t *)src + first;         // IN != 0
    if constexpr (RB > 1) {
        for (int j = tid; j < No; j += TB) wno[j] = wrev((float)j * (1.0f / (float)No));
        __syncthreads();
    }
    constexpr float im = 1.0f / (float)((int64_t)No * MI);       // exact, and so are r ko / M (r < 8192, ko < 512)
    // step 1: length-RA transforms over a, times W_No^{ka b2}; (column c, column c+1) = (re, im)
#pragma unroll 1
    for (int e = tid; e < RB * CG; e += TB) {
        const int cg = e & (CG - 1), b2 = e >> lgCG;
        float2 x[RA];
#pragma unroll
        for (int a = 0; a < RA; ++a) x[a] = make_float2(0.f, 0.f);
#pragma unroll
        for (int a = 0; a < RAIN; ++a) {
            const int n = (a * RB + b2) * MI + r0 + 2 * cg;
            if constexpr (IN == 0) {
                if (wide) {                        // Nk even, rows 8-byte aligned: a pair is inside or outside as a whole
                    // (from four rows to a thread's second factor up with 64-bit addresses: 64 channels of fft 2^21 425 -> 385 us the
                    // filter transform, 2^20 202 -> 184; below, 16 x 100001 of fft 2^18, the offsets are the faster ones: 24.9, 25.4)
                    x[a] = RB >= 4 ? *(const float2 *)(row0 + (int64_t)(n < Nk ? n : 0)) : ld_at<float2>(row0, n < Nk ? 4 * n : 0);
                } else {
                    x[a].x = row0[n < Nk ? n : 0];
                    x[a].y = row0[n + 1 < Nk ? n + 1 : 0];
                }
            } else {
                uint32_t wd;
                if (wide) wd = ld_pair(row16, n, (int)Nk);                // two samples or more
                else wd = (uint32_t)row16[0] << 16;
                x[a] = unpack2<IN == 1>(pair_of(wd, n, (int)Nk));
            }
        }
        float2 gt[GATED ? RAIN : 1];
        if constexpr (GATED) {
            const float *const row = gate + first;
#pragma unroll
            for (int a = 0; a < RAIN; ++a) {
                const int n = (a * RB + b2) * MI + r0 + 2 * cg;
                if (wide) {
                    gt[a] = RB >= 4 ? *(const float2 *)(row + (int64_t)(n < Nk ? n : 0)) : ld_at<float2>(row, n < Nk ? 4 * n : 0);
                } else {
                    gt[a].x = row[n < Nk ? n : 0];
                    gt[a].y = row[n + 1 < Nk ? n + 1 : 0];
                }
            }
        }
#pragma unroll
        for (int a = 0; a < RAIN; ++a) asm volatile("" ::"v"(x[a].x), "v"(x[a].y));      // keeps the loads unconditional
        if constexpr (GATED) {
#pragma unroll
            for (int a = 0; a < RAIN; ++a) {
                x[a].x *= gt[a].x;
                x[a].y *= gt[a].y;
                asm("" : "+v"(x[a].x), "+v"(x[a].y));             // (rounded: not part of a multiply-add)
            }
        }
#pragma unroll
        for (int a = 0; a < RAIN; ++a) {
            const int n = (a * RB + b2) * MI + r0 + 2 * cg;
            if (n >= Nk) x[a].x = 0.f;
            if (n + 1 >= Nk) x[a].y = 0.f;
        }
        dft_reg<RA, false, !FULLN>(x);
        if constexpr (RB == 1) {                   // Z[ko] and its mirror row are both at hand
            const int r = r0 + 2 * cg;
            const float rf = (float)r;
#pragma unroll
            for (int ko = 0; ko <= No / 2; ++ko) {
                const float2 z = x[ko], zm = x[(No - ko) % No];
                const float2 xa = make_float2(0.5f * (z.x + zm.x), 0.5f * (z.y - zm.y));
                const float2 xb = make_float2(0.5f * (z.y + zm.y), -0.5f * (z.x - zm.x));
                const float2 ta = cmulf(xa, wrev(rf * ((float)ko * im))), tb = cmulf(xb, wrev((rf + 1.f) * ((float)ko * im)));
                st_at(T2 + ((size_t)h * NR + ko) * MI, 8u * (uint32_t)r, make_float4(ta.x, ta.y, tb.x, tb.y));
            }
            continue;
        }
#pragma unroll
        for (int ka = 0; ka < RA; ++ka) T[(ka * RB + b2) * CG + cg] = cmulf(x[ka], wno[ka * b2]);
    }
    if constexpr (RB == 1) return;
    __syncthreads();
    // step 2: length-RB transforms over b2, in place: slot ka*RB + kb then holds Z[ko], ko = ka + RA kb
#pragma unroll 1
    for (int e = tid; e < RA * CG; e += TB) {
        const int cg = e & (CG - 1), ka = e >> lgCG;
        float2 x[RB];
#pragma unroll
        for (int b2 = 0; b2 < RB; ++b2) x[b2] = T[(ka * RB + b2) * CG + cg];
        dft_reg<RB, false>(x);
#pragma unroll
        for (int kb = 0; kb < RB; ++kb) T[(ka * RB + kb) * CG + cg] = x[kb];
    }
    __syncthreads();
    // step 3: split the two columns, twiddle (by recurrence over kb), store the rows ko <= No/2
#pragma unroll 1
    for (int e = tid; e < RA * CG; e += TB) {
        const int cg = e & (CG - 1), ka = e >> lgCG;
        const int r = r0 + 2 * cg;
        const float rf = (float)r;
        float2 z[RB / 2 + 1], zm[RB / 2 + 1];                      // ko = ka + RA kb <= No/2 needs kb <= RB/2
#pragma unroll
        for (int kb = 0; kb <= RB / 2; ++kb) {
            // row (No - ko) % No, see k_outer_fwd_real
            const float2 *const m = T + (ka ? ((RA - ka) * RB + RB - 1 - kb) * CG : (RB - kb) % RB * CG);
            z[kb] = T[(ka * RB + kb) * CG + cg];
            zm[kb] = m[cg];
        }
        float2 w0 = wrev(rf * ((float)ka * im)), w1 = wrev((rf + 1.f) * ((float)ka * im));
        const float2 s0 = wrev(rf * ((float)RA * im)), s1 = wrev((rf + 1.f) * ((float)RA * im));
        w0.x *= 0.5f, w0.y *= 0.5f, w1.x *= 0.5f, w1.y *= 0.5f;
        float2 *const dst = T2 + (size_t)h * NR * MI;
        const uint32_t at = 8u * (uint32_t)(ka * MI + r);
#pragma unroll
        for (int kb = 0; kb <= RB / 2; ++kb) {
            if (kb < RB / 2 || ka == 0) {
                const float2 xa = make_float2(z[kb].x + zm[kb].x, z[kb].y - zm[kb].y);        // Z + conj Zm (halved by the twiddle)
                const float2 xb = make_float2(z[kb].y + zm[kb].y, zm[kb].x - z[kb].x);        // (Z - conj Zm) / i
                const float2 ta = cmulf(xa, w0), tb = cmulf(xb, w1);
                st_at(dst + RA * kb * MI, at, make_float4(ta.x, ta.y, tb.x, tb.y));
            }
            w0 = cmulf(w0, s0);
            w1 = cmulf(w1, s1);
        }
    }
}

// ---- the last pass of the filter gradient of a multi-pass plan: pass C of a lone real row (k_outer_inv_real)
// with fp32 rows in and fp32 samples out.  T2[h][ko][r], ko <= No/2, holds the rows of sum_b conj(FFT u_b) FFT dy_b
// after their inverse 8192-point transforms (unnormalised); the spectrum is that of a real sequence, so the rows
// ko > No/2 are the mirror images described at k_outer_inv.  dk[h][n] = scale * (the inverse outer transform),
// n < Nk.
// GATED (fp32 convolutions): times the rows of gate, which lie like those of dk.
template <int RA, int RB, bool FULLN, bool GATED>
__global__ void __launch_bounds__(TB, 4) k_dk_outer_inv_real(const float2 *__restrict__ T2, float *__restrict__ dk, int cgs,
                                                         int64_t Nk, float scale, const float *__restrict__ gate)
{
    extern __shared__ float2 sm[];
    constexpr int No = RA * RB, NR = No / 2 + 1;
    constexpr int RAIN = FULLN ? RA : RA / 2;      // outer rows that are kept
    constexpr int KBC = RB < 8 ? RB : 8;           // rows loaded at a time (16 bytes each per thread)
    float2 *wno = sm;
    float2 *T = sm + No;                           // [No][CG]
    const int CG = RB > 1 ? TILE_COLS<RA, RB> : cgs;
    const int tid = threadIdx.x;
    const int r0 = blockIdx.x * 2 * CG;
    const int lgCG = 31 - __builtin_clz(CG);       // CG is a power of two
    const int64_t h = blockIdx.y;
    if constexpr (RB > 1) {
        for (int j = tid; j < No; j += TB) wno[j] = wrev((float)j * (1.0f / (float)No));
        __syncthreads();
    }
    constexpr float im = 1.0f / (float)((int64_t)No * MI);       // exact, and so are r ko / M (r < 8192, ko < 512)
    // step 1: untwiddle both columns, complete the rows ko > No/2 from their mirror rows, combine the columns
    // into one complex sequence, length-RB inverse over kb, times conj(W_No^{ka b2})
#pragma unroll 1
    for (int e = tid; RB > 1 && e < RA * CG; e += TB) {
        const int cg = e & (CG - 1), ka = e >> lgCG;
        const int r = r0 + 2 * cg;
        const float rf = (float)r;
        float2 w0 = wrev(rf * ((float)ka * im)), w1 = wrev((rf + 1.f) * ((float)ka * im));
        const float2 s0 = wrev(rf * ((float)RA * im)), s1 = wrev((rf + 1.f) * ((float)RA * im));
        w0.x *= scale, w0.y *= scale, w1.x *= scale, w1.y *= scale;
        // (see k_outer_inv_real)
        const uint32_t up = 8u * (uint32_t)(ka * MI + r), down = 8u * (uint32_t)((RA - ka) * MI + r);
        const float2 *const src = T2 + (size_t)h * NR * MI;
        auto base = [&](int kb) { return src + (kb < RB / 2 ? kb : kb > RB / 2 ? RB - 1 - kb : RB / 2 - 1) * RA * MI; };
        float2 x[RB];
#pragma unroll
        for (int kb0 = 0; kb0 < RB; kb0 += KBC) {
            float4 in[KBC];
#pragma unroll
            for (int kk = 0; kk < KBC; ++kk) {
                const int kb = kb0 + kk;
                in[kk] = ld_at<float4>(base(kb), kb < RB / 2 ? up : down);
            }
#pragma unroll
            for (int kk = 0; kk < KBC; ++kk) {
                const int kb = kb0 + kk;
                const bool mir = kb > RB / 2 || (kb == RB / 2 && ka > 0);
                // from the first mirrored row on the twiddle carries the extra factor conj(W_Mi^{r}) (see k_outer_inv)
                if ((kb == RB / 2 && ka > 0) || (kb == RB / 2 + 1 && ka == 0)) {
                    w0 = cmulcf(w0, wrev(rf * (1.0f / (float)MI)));
                    w1 = cmulcf(w1, wrev((rf + 1.f) * (1.0f / (float)MI)));
                }
                const float2 sa = make_float2(in[kk].x, mir ? -in[kk].y : in[kk].y);
                const float2 sb = make_float2(in[kk].z, mir ? -in[kk].w : in[kk].w);
                const float2 ua = cmulcf(sa, w0), ub = cmulcf(sb, w1);
                x[kb] = make_float2(ua.x - ub.y, ua.y + ub.x);               // U_c + i U_{c+1}
                w0 = cmulf(w0, s0);
                w1 = cmulf(w1, s1);
            }
        }
        dft_reg<RB, true>(x);
#pragma unroll
        for (int b2 = 0; b2 < RB; ++b2) T[(ka * RB + b2) * CG + cg] = cmulcf(x[b2], wno[ka * b2]);
    }
    if constexpr (RB > 1) __syncthreads();
    // step 2: length-RA inverse over ka; real part -> column c, imaginary part -> column c+1
    float *row0 = dk + h * Nk;
    const bool wide = Nk % 2 == 0 && (((uintptr_t)dk | (uintptr_t)(GATED ? gate : nullptr)) & 7) == 0;
#pragma unroll 1
    for (int e = tid; e < RB * CG; e += TB) {
        const int cg = e & (CG - 1), b2 = e >> lgCG;
        float2 x[RA];
        if constexpr (RB == 1) {                   // every row is read once and serves its mirror row too
            const int r = r0 + 2 * cg;
            const float rf = (float)r;
            float4 in[NR];
#pragma unroll
            for (int ko = 0; ko < NR; ++ko) in[ko] = ld_at<float4>(T2 + ((size_t)h * NR + ko) * MI, 8u * (uint32_t)r);
            const float2 m0 = wrev(rf * (1.0f / (float)MI)), m1 = wrev((rf + 1.f) * (1.0f / (float)MI));
#pragma unroll
            for (int ka = 0; ka < RA; ++ka) {
                const bool mir = ka > RA / 2;
                const float4 v = in[mir ? No - ka : ka];
                float2 w0 = wrev(rf * ((float)ka * im)), w1 = wrev((rf + 1.f) * ((float)ka * im));
                w0.x *= scale, w0.y *= scale, w1.x *= scale, w1.y *= scale;
                if (mir) {
                    w0 = cmulcf(w0, m0);
                    w1 = cmulcf(w1, m1);
                }
                const float2 ua = cmulcf(make_float2(v.x, mir ? -v.y : v.y), w0), ub = cmulcf(make_float2(v.z, mir ? -v.w : v.w), w1);
                x[ka] = make_float2(ua.x - ub.y, ua.y + ub.x);           // U_c + i U_{c+1}
            }
        } else {
#pragma unroll
            for (int ka = 0; ka < RA; ++ka) x[ka] = T[(ka * RB + b2) * CG + cg];
        }
        dft_reg<RA, true>(x);
        if constexpr (GATED) {                     // (samples beyond Nk read the row's first gate and are not stored)
            const float *const g = gate + h * Nk;
            constexpr int CH = RAIN < 8 ? RAIN : 8;                  // at a time
#pragma unroll
            for (int a0 = 0; a0 < RAIN; a0 += CH) {
                float2 gt[CH];
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const int n = ((a0 + i) * RB + b2) * MI + r0 + 2 * cg;
                    if (wide) {
                        gt[i] = ld_at<float2>(g, n < Nk ? 4 * n : 0);
                    } else {
                        gt[i].x = g[n < Nk ? n : 0];
                        gt[i].y = g[n + 1 < Nk ? n + 1 : 0];
                    }
                }
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    x[a0 + i].x *= gt[i].x;
                    x[a0 + i].y *= gt[i].y;
                    asm volatile("" : "+v"(x[a0 + i].x), "+v"(x[a0 + i].y));
                }
            }
        }
#pragma unroll
        for (int a = 0; a < RAIN; ++a) {
            const int n = (a * RB + b2) * MI + r0 + 2 * cg;
            if (wide) {
                if (n < Nk) st_at(row0, 4 * n, x[a]);
            } else {
                if (n < Nk) row0[n] = x[a].x;
                if (n + 1 < Nk) row0[n + 1] = x[a].y;
            }
        }
    }
}

template <int RA, int RB>
int launch_dk_outer_inv(const OuterGeo &g, const float2 *T2, float *dk, int64_t Nk, int64_t M, int64_t nh, float scale,
                        const float *gate, hipStream_t s)
{
    auto kern = Nk > M / 2 ? (gate ? k_dk_outer_inv_real<RA, RB, true, true> : k_dk_outer_inv_real<RA, RB, true, false>)
                           : (gate ? k_dk_outer_inv_real<RA, RB, false, true> : k_dk_outer_inv_real<RA, RB, false, false>);
    FC_TRY(raise_dynamic_lds((const void *)kern, 160 * 1024));
    hipLaunchKernelGGL(kern, dim3((unsigned)(MI / (2 * g.pairs())), (unsigned)nh), dim3(TB), g.lds(), s, T2, dk, g.pairs(), Nk, scale, gate);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

template <int IN, int RA, int RB, bool GATED>
int launch_filter_outer_in(const OuterGeo &g, const OuterRows &rows, float2 *T2, int64_t Nk, int64_t M, int64_t nh, const float *gate,
                           hipStream_t s)
{
    const bool wide = IN == 0 ? Nk % 2 == 0 && (((uintptr_t)rows.src | (uintptr_t)rows.src2 | (uintptr_t)gate) & 7) == 0 : Nk > 1;
    auto kern = Nk > M / 2 ? k_filter_outer_real<IN, RA, RB, true, GATED> : k_filter_outer_real<IN, RA, RB, false, GATED>;
    FC_TRY(raise_dynamic_lds((const void *)kern, 160 * 1024));
    hipLaunchKernelGGL(kern, dim3((unsigned)(MI / (2 * g.pairs())), (unsigned)nh), dim3(TB), g.lds(), s, rows, T2, g.pairs(), Nk, wide, gate);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}
// dtype: FFTCONV_F32 / F16 / BF16 of the rows; gate: fp32 rows only
template <int RA, int RB>
int launch_filter_outer(const OuterGeo &g, const OuterRows &rows, int dtype, float2 *T2, int64_t Nk, int64_t M, int64_t nh,
                        const float *gate, hipStream_t s)
{
    if (dtype == FFTCONV_F32)
        return gate ? launch_filter_outer_in<0, RA, RB, true>(g, rows, T2, Nk, M, nh, gate, s)
                    : launch_filter_outer_in<0, RA, RB, false>(g, rows, T2, Nk, M, nh, nullptr, s);
    if (dtype == FFTCONV_F16) return launch_filter_outer_in<1, RA, RB, false>(g, rows, T2, Nk, M, nh, nullptr, s);
    return launch_filter_outer_in<2, RA, RB, false>(g, rows, T2, Nk, M, nh, nullptr, s);
}

// k_f for the multi-pass path: [h][ko][inner order of f'] 16-bit (re, im) pairs, f = ko + No*f', scaled 1/M
// (fp16: boost/M, see multipass_kf_boost; pass C takes the boost out again).
template <bool F16>
__global__ void k_pack_multipass(const double2 *spec, uint32_t *kf, FacList fl, int64_t M, int No, int64_t h0,
                                 int64_t nh, const uint8_t *keep, int64_t n_blocks)
{
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= nh * M) return;
    const int64_t h = idx / M, f = idx % M;
    const int ko = (int)(f % No);
    const int64_t fi = f / No;
    const double2 v = spec[h * M + freq_to_pos(f, fl, M)];
    const double sc = mask_weight(keep, n_blocks, f, M) * (double)multipass_kf_boost(F16, No) / (double)M;
    kf[((h0 + h) * No + ko) * (int64_t)MI + fused3_kf_slot_8192(fi)] =
        (uint32_t)cv16<F16>((float)(v.x * sc)) | ((uint32_t)cv16<F16>((float)(v.y * sc)) << 16);
}

// rows: pairs of rows of a launch of the paired passes
OuterGeo outer_geo(int64_t M, int64_t rows = 0)
{
    OuterGeo g;
    g.No = (int)(M / MI);
    g.Ra = g.No < 16 ? g.No : 16;
    g.Rb = g.No / g.Ra;
    // No > 16: an fp32 tile T[No][CT] of 64 KiB (two blocks per compute unit), at least 32 columns.  Up to 16 a thread
    // transforms a pair of columns in registers and there is no tile: two columns for every thread of a block, and up to No = 4
    // several times that (of 8192 points, as above) where 1024 blocks or more remain: a block's start and its one trip to
    // memory are most of its time there.  us, 8 x 1268 x 1321 bf16, fft 8192, plain / gated: 220 / 258 in blocks of 8192 columns with a
    // tile, 225 / 361 with 1024, 150 / 196 with 8192; 2 x 16 x 8192 gated: 22, 14, 19 (1024 columns: 14); fft 16384, 8 x 512 x 1321: 158 / 169,
    // 136 / 153, 111 / 116; fft 32768, 8 x 512 x 1321: 343 / 408, 251 / 300, 239 / 280.
    g.CT = g.Rb == 1 ? 2 * TB : MI / g.No < 32 ? 32 : MI / g.No;
    while (g.Rb == 1 && g.CT * g.No < MI && rows * (MI / (2 * g.CT)) >= 1024) g.CT *= 2;
    return g;
}

template <bool F16, int RA, int RB, bool FULLN, bool GATED, bool EXACT>
int launch_outer_t(bool inverse, const OuterGeo &g, dim3 grid, const void *src, void *dst, int B, int H, int N,
                   hipStream_t s, int ko_lo, int ko_hi, bool mirror, const void *gate)
{
    // two columns per thread while the registers allow and while that still leaves an entry for every thread
    // (at No = 256 a block has 32 columns: 16 x 32 / 2 entries would keep half of its 512 threads idle)
    constexpr int CV = (RB <= 16 && RA * TILE_COLS<RA, RB> / 2 >= TB) ? 2 : 1;
    const size_t lds = g.lds();
    const int ct_inv = g.CT / (TB / INV_TB<RA, RB>);              // columns of a block of INV_TB threads
    const dim3 grid_inv(grid.x * (unsigned)(g.CT / ct_inv), grid.y);
    FC_TRY(raise_dynamic_lds((const void *)k_outer_fwd<F16, RA, RB, CV, FULLN, GATED, EXACT>, 160 * 1024));
    FC_TRY(raise_dynamic_lds((const void *)k_outer_inv<F16, RA, RB, CV, FULLN, GATED, false, EXACT>, 160 * 1024));
    FC_TRY(raise_dynamic_lds((const void *)k_outer_inv<F16, RA, RB, CV, FULLN, GATED, true, EXACT>, 160 * 1024));
    if (!inverse)
        hipLaunchKernelGGL((k_outer_fwd<F16, RA, RB, CV, FULLN, GATED, EXACT>), grid, dim3(TB), lds, s, (const uint16_t *)src,
                           (uint32_t *)dst, g.CT, B, H, N, ko_lo, ko_hi, (const uint16_t *)gate, launch_gate());
    else if (mirror)
        hipLaunchKernelGGL((k_outer_inv<F16, RA, RB, CV, FULLN, GATED, true, EXACT>), grid_inv, dim3(INV_TB<RA, RB>), lds, s, (const uint32_t *)src,
                           (uint16_t *)dst, ct_inv, B, H, N, ko_lo, ko_hi, (const uint16_t *)gate, launch_gate());
    else
        hipLaunchKernelGGL((k_outer_inv<F16, RA, RB, CV, FULLN, GATED, false, EXACT>), grid_inv, dim3(INV_TB<RA, RB>), lds, s, (const uint32_t *)src,
                           (uint16_t *)dst, ct_inv, B, H, N, ko_lo, ko_hi, (const uint16_t *)gate, launch_gate());
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

// the half-input instantiation needs an outer transform (No >= 2) and N <= M/2; EXACT: N is even and fills its
// half (or, FULLN, the whole transform), so that no load or store needs a range check (ungated calls only)
template <bool F16, int RA, int RB>
int launch_outer(bool inverse, const OuterGeo &g, dim3 grid, const void *src, void *dst, int B, int H, int N, int64_t M,
                 hipStream_t s, int ko_lo, int ko_hi, bool mirror, const void *gate)
{
#define FFTCONV_OUTER(FULLN, GATED, EXACT) \
    launch_outer_t<F16, RA, RB, FULLN, GATED, EXACT>(inverse, g, grid, src, dst, B, H, N, s, ko_lo, ko_hi, mirror, gate)
    if constexpr (RA >= 2) {
        if ((int64_t)N <= M / 2) {
            if (gate) return FFTCONV_OUTER(false, true, false);
            return (int64_t)N == M / 2 && N % 2 == 0 ? FFTCONV_OUTER(false, false, true) : FFTCONV_OUTER(false, false, false);
        }
    }
    if (gate) return FFTCONV_OUTER(true, true, false);
    return (int64_t)N == M && N % 2 == 0 ? FFTCONV_OUTER(true, false, true) : FFTCONV_OUTER(true, false, false);
#undef FFTCONV_OUTER
}

template <bool F16>
int dispatch_outer(bool inverse, const OuterGeo &g, dim3 grid, const void *src, void *dst, int B, int H, int N,
                   int64_t M, hipStream_t s, int ko_lo, int ko_hi, bool mirror, const void *gate)
{
    switch (g.No) {
    case 1: return launch_outer<F16, 1, 1>(inverse, g, grid, src, dst, B, H, N, M, s, ko_lo, ko_hi, mirror, gate);
    case 2: return launch_outer<F16, 2, 1>(inverse, g, grid, src, dst, B, H, N, M, s, ko_lo, ko_hi, mirror, gate);
    case 4: return launch_outer<F16, 4, 1>(inverse, g, grid, src, dst, B, H, N, M, s, ko_lo, ko_hi, mirror, gate);
    case 8: return launch_outer<F16, 8, 1>(inverse, g, grid, src, dst, B, H, N, M, s, ko_lo, ko_hi, mirror, gate);
    case 16: return launch_outer<F16, 16, 1>(inverse, g, grid, src, dst, B, H, N, M, s, ko_lo, ko_hi, mirror, gate);
    case 32: return launch_outer<F16, 16, 2>(inverse, g, grid, src, dst, B, H, N, M, s, ko_lo, ko_hi, mirror, gate);
    case 64: return launch_outer<F16, 16, 4>(inverse, g, grid, src, dst, B, H, N, M, s, ko_lo, ko_hi, mirror, gate);
    case 128: return launch_outer<F16, 16, 8>(inverse, g, grid, src, dst, B, H, N, M, s, ko_lo, ko_hi, mirror, gate);
    case 256: return launch_outer<F16, 16, 16>(inverse, g, grid, src, dst, B, H, N, M, s, ko_lo, ko_hi, mirror, gate);
    case 512: return launch_outer<F16, 16, 32>(inverse, g, grid, src, dst, B, H, N, M, s, ko_lo, ko_hi, mirror, gate);
    default:
        set_error("multipass: unsupported outer length %d", g.No);
        return FFTCONV_EUNSUPPORTED;
    }
}

template <bool F16, int RA, int RB>
int launch_outer_real(bool inverse, const OuterGeo &g, const void *src, void *dst, int H, int N, int64_t M, hipStream_t s,
                      int ko_lo, const void *gate)
{
    const size_t lds = g.lds();
    const dim3 grid((unsigned)(MI / (2 * g.pairs())), (unsigned)H);
    const bool fulln = (int64_t)N > M / 2;
#define FFTCONV_REAL_LAUNCH(FULLN, GATED, EXACT)                                                                                  \
    do {                                                                                                                    \
        if (!inverse) {                                                                                                     \
            FC_TRY(raise_dynamic_lds((const void *)k_outer_fwd_real<F16, RA, RB, FULLN, GATED, EXACT>, 160 * 1024));               \
            hipLaunchKernelGGL((k_outer_fwd_real<F16, RA, RB, FULLN, GATED, EXACT>), grid, dim3(TB), lds, s, (const uint16_t *)src, \
                               (uint32_t *)dst, g.pairs(), H, N, ko_lo, (const uint16_t *)gate, launch_gate());               \
        } else {                                                                                                            \
            FC_TRY(raise_dynamic_lds((const void *)k_outer_inv_real<F16, RA, RB, FULLN, GATED, EXACT>, 160 * 1024));               \
            hipLaunchKernelGGL((k_outer_inv_real<F16, RA, RB, FULLN, GATED, EXACT>), grid, dim3(TB), lds, s, (const uint32_t *)src, \
                               (uint16_t *)dst, g.pairs(), H, N, ko_lo, (const uint16_t *)gate, launch_gate());               \
        }                                                                                                                   \
    } while (0)
    // exact: N is even and fills its half (or the whole transform): no range checks (ungated calls only)
    const bool exact = N % 2 == 0 && (int64_t)N == (fulln ? M : M / 2);
    if (fulln) {
        if (gate) FFTCONV_REAL_LAUNCH(true, true, false);
        else if (exact) FFTCONV_REAL_LAUNCH(true, false, true);
        else FFTCONV_REAL_LAUNCH(true, false, false);
    } else {
        if (gate) FFTCONV_REAL_LAUNCH(false, true, false);
        else if (exact) FFTCONV_REAL_LAUNCH(false, false, true);
        else FFTCONV_REAL_LAUNCH(false, false, false);
    }
#undef FFTCONV_REAL_LAUNCH
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

// outer lengths the packed real-row passes exist for
bool outer_real_ok(int No) { return No >= 4 && No <= 256; }

template <bool F16>
int dispatch_outer_real(bool inverse, const OuterGeo &g, const void *src, void *dst, int H, int N, int64_t M, hipStream_t s,
                        int ko_lo, const void *gate)
{
    switch (g.No) {
    case 4: return launch_outer_real<F16, 4, 1>(inverse, g, src, dst, H, N, M, s, ko_lo, gate);
    case 8: return launch_outer_real<F16, 8, 1>(inverse, g, src, dst, H, N, M, s, ko_lo, gate);
    case 16: return launch_outer_real<F16, 16, 1>(inverse, g, src, dst, H, N, M, s, ko_lo, gate);
    case 32: return launch_outer_real<F16, 16, 2>(inverse, g, src, dst, H, N, M, s, ko_lo, gate);
    case 64: return launch_outer_real<F16, 16, 4>(inverse, g, src, dst, H, N, M, s, ko_lo, gate);
    case 128: return launch_outer_real<F16, 16, 8>(inverse, g, src, dst, H, N, M, s, ko_lo, gate);
    case 256: return launch_outer_real<F16, 16, 16>(inverse, g, src, dst, H, N, M, s, ko_lo, gate);
    default:
        set_error("multipass: no real-row outer pass for outer length %d", g.No);
        return FFTCONV_EUNSUPPORTED;
    }
}

}  // namespace

bool multipass_supported(int64_t N, int64_t M, int dtype)
{
    if (dtype != FFTCONV_F16 && dtype != FFTCONV_BF16) return false;
    if (M < MI || M > 512 * (int64_t)MI) return false;
    return N >= 1 && N <= M;
}

int multipass_init(fftconv_plan *p, bool forced)
{
    p->f3.odd = !forced && fused3_odd_rows(p);
    int rc = fused3_init_inner(p);
    if (rc) return rc;
    return fused3_init_short(p);      // short filters run as overlapping 8192-point segments (fused3.hip)
}

size_t multipass_kf_bytes(const fftconv_plan *p)
{
    return (size_t)(p->H * p->M) * sizeof(uint32_t) + fused3_short_kf_bytes(p);
}

size_t multipass_workspace_bytes(const fftconv_plan *p, int64_t B)
{
    int64_t rows = (B + 1) / 2 * p->H;
    // (a larger batch that needs none: enough for a smaller one that does)
    if (p->f3.odd && rows > fused3_odd_few_rows(p)) rows = fused3_odd_few_rows(p);
    return (size_t)(rows * p->M) * sizeof(uint32_t);
}

int multipass_pack_kf(const fftconv_plan *p, const double2 *spec, int64_t h0, int64_t nh, const uint8_t *keep_dev,
                      int64_t n_blocks, void *kf, hipStream_t s)
{
    const int bs = 256;
    const unsigned grid = (unsigned)((nh * p->M + bs - 1) / bs);
    if (p->dtype == FFTCONV_F16)
        hipLaunchKernelGGL(k_pack_multipass<true>, dim3(grid), dim3(bs), 0, s, spec, (uint32_t *)kf, staged_fac_list(p),
                           p->M, (int)(p->M / MI), h0, nh, keep_dev, n_blocks);
    else
        hipLaunchKernelGGL(k_pack_multipass<false>, dim3(grid), dim3(bs), 0, s, spec, (uint32_t *)kf, staged_fac_list(p),
                           p->M, (int)(p->M / MI), h0, nh, keep_dev, n_blocks);
    FC_HIP(hipGetLastError());
    return FFTCONV_OK;
}

// Outer pass of the transform of nh real rows of Nk samples each (see k_filter_outer_real, OuterRows; dtype: FFTCONV_F32 / F16 /
// BF16 of the rows); T2 takes nh * (No/2 + 1) * 8192 fp32 pairs.  multipass_filter_outer_ok(): false = no such kernel
// for this outer length (the caller takes the generic column kernel instead).
bool multipass_filter_outer_ok(const fftconv_plan *p) { return outer_real_ok((int)(p->M / MI)); }

int multipass_filter_outer(const fftconv_plan *p, const OuterRows &rows, int dtype, int64_t Nk, int64_t nh, void *T2, hipStream_t s,
                           const float *gate)
{
    const OuterGeo g = outer_geo(p->M);
    if (nh > 65535) {
        set_error("multipass: %lld rows per launch of the real outer pass exceed the grid limit", (long long)nh);
        return FFTCONV_EUNSUPPORTED;
    }
    float2 *t = (float2 *)T2;
    switch (g.No) {
    case 4: return launch_filter_outer<4, 1>(g, rows, dtype, t, Nk, p->M, nh, gate, s);
    case 8: return launch_filter_outer<8, 1>(g, rows, dtype, t, Nk, p->M, nh, gate, s);
    case 16: return launch_filter_outer<16, 1>(g, rows, dtype, t, Nk, p->M, nh, gate, s);
    case 32: return launch_filter_outer<16, 2>(g, rows, dtype, t, Nk, p->M, nh, gate, s);
    case 64: return launch_filter_outer<16, 4>(g, rows, dtype, t, Nk, p->M, nh, gate, s);
    case 128: return launch_filter_outer<16, 8>(g, rows, dtype, t, Nk, p->M, nh, gate, s);
    case 256: return launch_filter_outer<16, 16>(g, rows, dtype, t, Nk, p->M, nh, gate, s);
    default:
        set_error("multipass: no real outer pass for outer length %d", g.No);
        return FFTCONV_EUNSUPPORTED;
    }
}

// Last pass of the filter gradient, and of the fp32 forward pass of long plans (see k_dk_outer_inv_real): T2 holds
// nh * (No/2 + 1) rows; dk (nh, Nk) = scale * the real inverse outer transform.
int multipass_dk_outer_inv(const fftconv_plan *p, const void *T2, float *dk, int64_t Nk, int64_t nh, float scale, hipStream_t s,
                           const float *gate)
{
    const OuterGeo g = outer_geo(p->M);
    if (nh > 65535) {
        set_error("multipass: %lld rows per launch of the real outer pass exceed the grid limit", (long long)nh);
        return FFTCONV_EUNSUPPORTED;
    }
    const float2 *t = (const float2 *)T2;
    switch (g.No) {
    case 4: return launch_dk_outer_inv<4, 1>(g, t, dk, Nk, p->M, nh, scale, gate, s);
    case 8: return launch_dk_outer_inv<8, 1>(g, t, dk, Nk, p->M, nh, scale, gate, s);
    case 16: return launch_dk_outer_inv<16, 1>(g, t, dk, Nk, p->M, nh, scale, gate, s);
    case 32: return launch_dk_outer_inv<16, 2>(g, t, dk, Nk, p->M, nh, scale, gate, s);
    case 64: return launch_dk_outer_inv<16, 4>(g, t, dk, Nk, p->M, nh, scale, gate, s);
    case 128: return launch_dk_outer_inv<16, 8>(g, t, dk, Nk, p->M, nh, scale, gate, s);
    case 256: return launch_dk_outer_inv<16, 16>(g, t, dk, Nk, p->M, nh, scale, gate, s);
    default:
        set_error("multipass: no real outer pass for outer length %d", g.No);
        return FFTCONV_EUNSUPPORTED;
    }
}

constexpr int64_t MOST_ROWS = 65535;          // second dimension of a launch's grid

// One set of the three passes over rows [0, B) of u.  ko_lo, ko_hi: outer frequency digits ko in [ko_lo, ko_hi)
// only meet zeroed bins of k_f (frequency-sparse filters); their rows of the workspace are skipped by all three
// passes.  ko_lo >= ko_hi: none.  wg, vg: input / output gate of the gated form, fused into passes A and C.
// lone: B == 1 and the row is transformed as a REAL sequence (Appendix A.1's point -- a real input needs half
// of a complex transform -- taken at the outer factor): before the twiddle, row No - ko of the outer transform
// of a real sequence is the conjugate of row ko, its spectrum is the mirror image of row ko's, and since the
// filter is real the same holds after the inner convolutions.  So only the rows ko <= No/2 are written by pass A,
// convolved by pass B (which then reads only those rows of k_f) and read by pass C, which forms the others as
// conjugates: half of the workspace traffic, of the k_f traffic and of the inner transforms.
static int multipass_passes(const fftconv_plan *p, const void *u, const void *kf, void *y, int64_t B, uint32_t *S,
                            hipStream_t s, int ko_lo, int ko_hi, const void *wg, const void *vg, bool lone)
{
    const int64_t npairs = (B + 1) / 2;
    const int64_t rows = npairs * p->H;
    const bool packed = lone && outer_real_ok((int)(p->M / MI));
    const OuterGeo g = outer_geo(p->M, packed ? 0 : rows);
    if (rows > MOST_ROWS) {
        set_error("fftconv_forward: ceil(B/2) * H = %lld exceeds the multi-pass grid limit %lld", (long long)rows, (long long)MOST_ROWS);
        return FFTCONV_EUNSUPPORTED;
    }
    const bool f16 = p->dtype == FFTCONV_F16;
    const dim3 grid((unsigned)(MI / g.CT), (unsigned)rows);
    if (ko_lo >= ko_hi) ko_lo = ko_hi = g.No;            // nothing skipped
    // rows that passes A and B leave out, rows that pass C takes as zero, rows that pass C mirrors
    int ab_lo = ko_lo, ab_hi = ko_hi, c_lo = ko_lo, c_hi = ko_hi;
    bool mirror = false;
    if (packed) {
        // a sparse filter keeps ko < ko_lo and ko >= ko_hi = No - (ko_lo - 1), mirror images of each other: of the rows
        // ko <= No/2 those below ko_lo are live
        ab_lo = ko_lo < g.No / 2 + 1 ? ko_lo : g.No / 2 + 1;
        ab_hi = g.No;
    } else if (lone && g.No >= 4 && ko_lo >= ko_hi) {     // outer length 512: paired kernels, pass C mirrors the rows
        mirror = true;
        ab_lo = g.No / 2 + 1;
        ab_hi = g.No;
    }
    // the lone row's outer passes pack two columns into one complex transform where such kernels exist
    // (outer lengths 4 .. 256); at 512 the paired kernels run with the missing partner and pass C mirrors the rows
    int rc;
    if (packed)
        rc = f16 ? dispatch_outer_real<true>(false, g, u, S, (int)p->H, (int)p->N, p->M, s, ab_lo, wg)
                 : dispatch_outer_real<false>(false, g, u, S, (int)p->H, (int)p->N, p->M, s, ab_lo, wg);
    else
        rc = f16 ? dispatch_outer<true>(false, g, grid, u, S, (int)B, (int)p->H, (int)p->N, p->M, s, ab_lo, ab_hi, false, wg)
                 : dispatch_outer<false>(false, g, grid, u, S, (int)B, (int)p->H, (int)p->N, p->M, s, ab_lo, ab_hi, false, wg);
    if (rc) return rc;
    rc = fused3_inner_rows(p, S, kf, npairs, p->H * g.No, s, g.No, ab_lo, ab_hi, multipass_quarter_rows(g.No));
    if (rc) return rc;
    if (packed)
        return f16 ? dispatch_outer_real<true>(true, g, S, y, (int)p->H, (int)p->N, p->M, s, ab_lo, vg)
                   : dispatch_outer_real<false>(true, g, S, y, (int)p->H, (int)p->N, p->M, s, ab_lo, vg);
    return f16 ? dispatch_outer<true>(true, g, grid, S, y, (int)B, (int)p->H, (int)p->N, p->M, s, c_lo, c_hi, mirror, vg)
               : dispatch_outer<false>(true, g, grid, S, y, (int)B, (int)p->H, (int)p->N, p->M, s, c_lo, c_hi, mirror, vg);
}

// Whether the last row of an odd batch goes with the pairs and zeros for a partner.  On its own it has half the work, and three launches:
// 15 us where the chip has room for it beside the pairs.  us, on its own, with the pairs (outer length x H; B = 3): 16 11 x 1 x 65536 fp16 35.0, 19.3; 256
// 3 x 16 x 65536 43.9, 34.4; 512 54.5, 45.7; 1024 75.5, 69.8, outer length 8 71.2, 66.7, 256 91.8, 85.8, 512 113, 103; 33 x 64 x 65536 561, 554; 1536
// 112, 113; 2048 152, 170.  Outer lengths 1 and 2 have no passes for a row on its own: 9 x 400 x 8190 circular 90, 73.  Its error is that of the
// other rows, a fifth to a quarter below that of a real row.  Only where a launch holds them all: pairs and lone rows may be MOST_ROWS each.
static bool lone_in_pairs(const fftconv_plan *p, int64_t B)
{
    return (B + 1) / 2 * p->H <= MOST_ROWS && (p->M <= 2 * MI || p->H * (p->M / MI) <= 1024);
}

// Batch rows are transformed two at a time (one complex transform per pair, the filter being real); a row left
// over (odd B, B = 1) goes with them, or through a set of passes of its own as a real sequence (see above).
int multipass_forward(const fftconv_plan *p, const void *u, const void *kf, void *y, int64_t B, void *workspace,
                      hipStream_t s, int ko_lo, int ko_hi, const void *wg, const void *vg)
{
    uint32_t *S = (uint32_t *)workspace;
    if (p->f3.odd && !fused3_odd_few(p, B, wg || vg)) return f3::fused3_big_forward_odd(p, u, wg, vg, kf, y, B, s);
    // fft_size 8192 (outer length 1: a circular or ragged shape the causal kernel does not take): the inner kernel
    // reads u and writes y itself, nothing passes through the workspace.  Gated calls and N not a multiple of 4
    // (rows that start off an 8-byte boundary) keep the three passes.
    if (p->M == MI && p->N % 4 == 0 && !wg && !vg) return fused3_inner_whole(p, u, kf, y, B, s);
    const int64_t Be = B > 1 && lone_in_pairs(p, B) ? B : B - B % 2;      // rows in pairs
    if (Be > 0) {
        const int rc = multipass_passes(p, u, kf, y, Be, S, s, ko_lo, ko_hi, wg, vg, false);
        if (rc) return rc;
    }
    if (Be == B) return FFTCONV_OK;
    const size_t ofs = (size_t)Be * (size_t)p->H * (size_t)p->N;             // elements before the last row
    auto at = [&](const void *base) { return base ? (const void *)((const uint16_t *)base + ofs) : nullptr; };
    return multipass_passes(p, at(u), kf, (uint16_t *)y + ofs, 1, S + (size_t)(Be / 2) * p->H * p->M, s, ko_lo, ko_hi,
                            at(wg), at(vg), true);
}

}  // namespace fftconv
