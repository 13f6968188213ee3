// Token-wise FP8 (E4M3) activation quantizer, with the optional LoRC left
// factor T = X.U computed in the same sweep (paper Section 3: token-wise
// activation quantization, LoRC; Appendix A).  The normalisation whose output
// the quantizer sees (Section 3 names the layer normalisation in front of the
// quantized linear layers; LLaMA uses the RMS form) can run in the same sweep.
//
// One workgroup of 256 threads per token (1024 for a handful of tokens).  The row is read once with 16-byte
// loads (8 bf16 per lane), kept in registers across the absmax reduction
// (rows up to 8192 elements; longer rows are re-read, from L2), scaled,
// converted with the hardware FP8 conversion (round to nearest even) after an
// explicit clamp to +-448, and written with 8-byte stores.  HBM-bound: 2 B read
// and 1 B written per element.
#include "zqfp_internal.h"

namespace zqfp {
namespace {

constexpr int kRegChunks = 4;  // 16-byte chunks per thread kept in registers

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

__device__ inline float half_bits_to_float(uint32_t h) { return half_bits_to_f32((uint16_t)h); }

// RP consecutive ranks of a row of U (binary16), and their products with x; a row past the end counts as zeros
template <int RP>
struct alignas(2 * RP < 16 ? 2 * RP : 16) Ranks {
    uint32_t w[RP / 2];
};
template <int RP>
__device__ inline void add_ranks(float (&acc)[RP], float x, const Ranks<RP>& u, bool live)
{
#pragma unroll
    for (int q = 0; q < RP / 2; ++q) {
        const uint32_t w = live ? u.w[q] : 0u;
        acc[2 * q] = fmaf(x, half_bits_to_float(w & 0xFFFFu), acc[2 * q]);
        acc[2 * q + 1] = fmaf(x, half_bits_to_float(w >> 16), acc[2 * q + 1]);
    }
}

// acc[j] += sum_i x_i * U[k_i][j] for the 8 elements (x_i, k_i = kbase + 64 i) that a lane picked up
// from its wave's 512-element slice: consecutive lanes own consecutive k, so a wave's load of U
// rows is one contiguous run (r = 8: 1 KB per instruction) instead of 64 scattered 16-byte pieces.
// U points to the first of this workgroup's `rb` <= RP ranks, rows lie r elements apart.
// How a row of U is read: as r allows, whole blocks in vector loads, or one rank after the other.
enum class Rows { kAny, kWhole, kSingle };
template <int RP, Rows ROWS>
__device__ inline void lorc_accumulate(float (&acc)[RP], const float (&x)[8], const uint16_t* U, int64_t kbase, int64_t K, int r, int rb)
{
    // K is a multiple of 128, not of 512: elements past the row's end are zero and meet a zeroed row of U
    if (ROWS == Rows::kWhole || (ROWS == Rows::kAny && (r & (RP < 8 ? RP - 1 : 7)) == 0)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bool live = kbase + 64 * i < K;
            const Ranks<RP> u = *reinterpret_cast<const Ranks<RP>*>(U + (live ? kbase + 64 * i : 0) * r);
            add_ranks<RP>(acc, x[i], u, live);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < RP; ++j)
                if (j < rb && kbase + 64 * i < K) acc[j] = fmaf(x[i], half_bits_to_float(U[(kbase + 64 * i) * r + j]), acc[j]);
    }
}

// two binary32 values -> two bf16 in one dword (round to nearest even): the packed hardware conversion
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pack_bf16_rne(float lo, float hi)
{
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}


// 8 bf16 -> 8 bf16: (x * rstd) * g, each product one binary32 operation, rounded to bf16
__device__ inline uint4 normalize8(uint4 v, uint4 g, float rstd)
{
    uint32_t w[4] = {v.x, v.y, v.z, v.w}, gw[4] = {g.x, g.y, g.z, g.w}, o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float lo = (bf16_lo(w[i]) * rstd) * bf16_lo(gw[i]);
        const float hi = (bf16_hi(w[i]) * rstd) * bf16_hi(gw[i]);
        o[i] = pack_bf16_rne(lo, hi);
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
}

// 8 bf16 -> 8 bf16: ((x - mu) * rstd) * g + b, four separately rounded binary32 operations (the
// product and the sum must not fuse into one), rounded to bf16
__device__ inline uint4 normalize8_affine(uint4 v, uint4 g, uint4 b, float mu, float rstd)
{
#pragma clang fp contract(off)
    uint32_t w[4] = {v.x, v.y, v.z, v.w}, gw[4] = {g.x, g.y, g.z, g.w}, bw[4] = {b.x, b.y, b.z, b.w}, o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float dl = bf16_lo(w[i]) - mu, dh = bf16_hi(w[i]) - mu;
        const float al = dl * rstd, ah = dh * rstd;
        const float cl = al * bf16_lo(gw[i]), ch = ah * bf16_hi(gw[i]);
        const float lo = cl + bf16_lo(bw[i]), hi = ch + bf16_hi(bw[i]);
        o[i] = pack_bf16_rne(lo, hi);
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
}

// 8 bf16 + 8 bf16 -> 8 bf16: one binary32 addition each, rounded to bf16
__device__ inline uint4 add8(uint4 x, uint4 r)
{
    uint32_t xw[4] = {x.x, x.y, x.z, x.w}, rw[4] = {r.x, r.y, r.z, r.w}, o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        o[i] = pack_bf16_rne(bf16_lo(xw[i]) + bf16_lo(rw[i]), bf16_hi(xw[i]) + bf16_hi(rw[i]));
    return make_uint4(o[0], o[1], o[2], o[3]);
}

// ReLU on 8 bf16: a value passes unmodified if it is greater than zero, anything else becomes +0
__device__ inline uint4 relu8(uint4 x)
{
    uint32_t w[4] = {x.x, x.y, x.z, x.w}, o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        o[i] = (bf16_lo(w[i]) > 0.0f ? (w[i] & 0xFFFFu) : 0u) | (bf16_hi(w[i]) > 0.0f ? (w[i] & 0xFFFF0000u) : 0u);
    return make_uint4(o[0], o[1], o[2], o[3]);
}

// silu(g) * u = g / (1 + exp(-g)) * u as the binary32 value whose rounding to bf16 (nearest even) equals
// that of the expression evaluated in binary64 and rounded to binary32 first.
// Fast path, binary32 throughout: for 2^-30 <= |g| <= 32 and 2^-30 <= |u| <= 2^30 every intermediate
// is a normal number (exp(-g) in 2^+-47, the quotient above 2^-77, the product in 2^-107 .. 2^35), so
// the relative error is bounded by that of exp (below, taken as 4 ulp), of the hardware
// reciprocal (1 ulp) and three roundings: 13 * 2^-24 in all, at most 13 binary32 ulps of the result.
// The bf16 rounding of the true value and of the
// binary64 evaluation (which is within half a binary32 ulp of it after its own rounding) is therefore
// the one of this value whenever its low 16 bits are more than 32 ulps away from the half-way pattern
// 0x8000.  Anything else (1 value in 1000, and inputs outside the ranges) is evaluated in binary64.
//
// exp(-g) = 2^(-g L) e^(-g c) with L = 47274 / 2^15, log2 e to 16 bits, and c = 1 - L ln 2.  g has 8 bits, so -g L is exact and the
// hardware's power of two (1 ulp) is of the number meant; |g c| <= 2^-12.6, so 1 - g c is e^(-g c) within a quarter ulp.
//
// The vector units are the bound: a row of 28672 values on its one compute unit, and from some hundred rows on all of them.  Hence no
// general expf, and the conditions in 16-bit arithmetic on pairs (what a saturating difference leaves of a value outside a
// range is not zero), not in comparisons of each value: about 21 issue slots a value in place of 33.  Graph-timed, before -> after: 4 x 28672
// 10.2 -> 9.2 us, 16 x 8192 5.0 -> 4.7, 333 x 4096 6.4 -> 5.7, 1500 x 4096 17.7 -> 15.1, 2048 x 8192 rank 8 43.7 -> 37.8, 4096 x 11008
// 64.0 -> 60.6.  (All loads of the second operand ahead of the evaluations lose: 64 x 28672 11.7 -> 12.1, 4096 x 11008 64 -> 101.)
__device__ inline uint32_t outside(uint32_t pair, uint16_t lo, uint16_t hi)  // a half of the result is 0 where lo <= pair's half <= hi
{
    const u16x2_t v = __builtin_bit_cast(u16x2_t, pair), l = {lo, lo}, h = {hi, hi};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(l, v)) | __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(v, h));
}

__device__ inline uint4 swiglu8(uint4 g, uint4 u)
{
    constexpr float L = 47274.0f / 32768.0f, c = 0x1.480fb6p-18f;
    const uint32_t gw[4] = {g.x, g.y, g.z, g.w}, uw[4] = {u.x, u.y, u.z, u.w};
    uint32_t o[4], open[4];
    auto fast = [&](float gf, float uf) __attribute__((always_inline)) {
        const float e = __builtin_amdgcn_exp2f(gf * -L);
        return gf * __builtin_amdgcn_rcpf(1.0f + fmaf(e, gf * -c, e)) * uf;
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float y0 = fast(bf16_lo(gw[i]), bf16_lo(uw[i])), y1 = fast(bf16_hi(gw[i]), bf16_hi(uw[i]));
        o[i] = pack_bf16_rne(y0, y1);
        const u16x2_t low = __builtin_bit_cast(u16x2_t, __builtin_amdgcn_perm(__float_as_uint(y1), __float_as_uint(y0), 0x05040100u));
        const u16x2_t first = {0x8000 - 32, 0x8000 - 32}, count = {65, 65};
        open[i] = outside(gw[i] & 0x7FFF7FFFu, 0x3080, 0x4200) | outside(uw[i] & 0x7FFF7FFFu, 0x3080, 0x4E80) |
                  __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(count, (u16x2_t)(low - first)));
    }
    if ((open[0] | open[1] | open[2] | open[3]) != 0) {
        uint32_t redo = 0;  // a bit per value
#pragma unroll
        for (int i = 0; i < 4; ++i) redo |= ((open[i] & 0xFFFFu) != 0 ? 1u << 2 * i : 0u) | (open[i] >> 16 != 0 ? 2u << 2 * i : 0u);
        // every lane takes its own next value: one turn where a branch at each place would make one per place that any lane has open
        do {
            const int b = __builtin_ctz(redo);
            redo &= redo - 1;
            uint32_t gb = gw[0], ub = uw[0];
#pragma unroll
            for (int i = 1; i < 4; ++i) {
                gb = (b >> 1) == i ? gw[i] : gb;
                ub = (b >> 1) == i ? uw[i] : ub;
            }
            asm volatile("" : "+v"(gb), "+v"(ub));  // the conversions' halves need not live across turns
            const double gd = (double)((b & 1) ? bf16_hi(gb) : bf16_lo(gb)), ud = (double)((b & 1) ? bf16_hi(ub) : bf16_lo(ub));
            const float y = (float)(gd / (1.0 + exp(-gd)) * ud);
            const uint32_t half = (b & 1) ? 0xFFFF0000u : 0xFFFFu, bits = pack_bf16_rne(y, y) & half;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = (b >> 1) == i ? (o[i] & ~half) | bits : o[i];
        } while (redo != 0);
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
}

__device__ inline double sum_values(double acc, uint4 v)
{
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc += (double)bf16_lo(w[i]);
        acc += (double)bf16_hi(w[i]);
    }
    return acc;
}

// statistics of a row from its two binary64 sums: 1 / sqrt(second moment or variance + eps) in binary32
// arithmetic (IEEE add, square root, division), and for layer normalisation the mean rounded to binary32
template <int NORM>
__device__ inline void row_statistics(double s1, double ss, int64_t K, float eps, float& mu, float& rstd)
{
#pragma clang fp contract(off)
    double second = ss / (double)K;
    mu = 0.0f;
    if constexpr (NORM == 2) {
        const double mean = s1 / (double)K;
        second = fmax(second - mean * mean, 0.0);  // variance, never negative
        mu = (float)mean;
    }
    rstd = 1.0f / sqrtf((float)second + eps);
}

__device__ inline double sum_squares(double acc, uint4 v)
{
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double lo = (double)bf16_lo(w[i]), hi = (double)bf16_hi(w[i]);
        acc += lo * lo;  // each square is exact in binary64
        acc += hi * hi;
    }
    return acc;
}

// NORM (the producer fused in front): 0 plain quantizer, 1 RMS normalisation (gain), 2 layer normalisation
// (gain, bias), 3 ReLU, 4 gated SiLU (X is the gate, `other` the second operand).  With 1 and 2 a non-null
// `other` is a residual added to X first; the sum, rounded to bf16, also goes to H.  Every thread reads an
// element of `other` before it writes the same element of H, and nothing else touches it: H may be `other`.
// NT threads per token: 256 when there are tokens enough to fill the chip, 1024 for a handful of
// tokens (decode), where one row's latency chain is all there is.  The gated unit in 1024 threads is held to 64 registers, so that two
// tokens share a compute unit (4096 x 11008: 81 -> 61 us; the four that do not fit are the binary64 loop's).
// With sixteen sums for a left factor and 256 threads a token is four waves, one a SIMD, so the waves a SIMD holds are the rounds of
// 256 tokens a launch takes at once: the instances that miss one by a few registers are held to it, none of them spills
// (five in 96 registers, the gated unit seven in 72; left alone four and five.  1166 x 384, RMS normalisation, rank 15: 26.1 -> 17.4 us;
// 1268 x 640 with a residual, rank 9: 24.7 -> 17.0; gated, 1489 x 4736, rank 14: 96.2 -> 76.2).
constexpr int waves_per_simd(int rp, int nt, int norm)
{
    if (nt == 1024) return norm == 4 && rp == 0 ? 8 : 1;
    if (norm == 4) return rp == 16 ? 7 : 1;
    return rp == 16 && norm != 2 ? 5 : 1;
}
template <int RP, int NT, int NORM, Rows ROWS = Rows::kAny>
__global__ __launch_bounds__(NT, waves_per_simd(RP, NT, NORM)) void k_quantize_act(const uint16_t* __restrict__ X, int64_t K, int64_t ldx,
                                                         uint8_t* __restrict__ Xq, float* __restrict__ sx,
                                                         const uint16_t* __restrict__ U, int r, float* __restrict__ T,
                                                         Producer pr)
{
    const uint16_t* __restrict__ gain = pr.gain;
    const uint16_t* __restrict__ bias = pr.bias;
    const float eps = pr.eps;
    constexpr int kThreads = NT, kWaves = NT / 64;
    __shared__ uint32_t s_amax[kWaves];
    __shared__ float s_t[kWaves][RP > 0 ? RP : 1];
    __shared__ __attribute__((aligned(16))) uint16_t s_x[RP > 0 ? kWaves : 1][512];  // per wave: its current 512-element slice
    const int64_t row = blockIdx.x;
    const int tid = threadIdx.x;
    const uint4* xrow = reinterpret_cast<const uint4*>(X + row * ldx);
    uint2* qrow = reinterpret_cast<uint2*>(Xq + row * K);
    const int nchunk = (int)(K / 8);
    // More than 8 ranks and few tokens: a workgroup per 8 (or 4) of them, each of which forms the row for itself (one workgroup with all
    // sums in its threads waits for up to eight loads of U in turn, and spills: 4 x 4096, RMS normalisation, rank 16 / 40: 11.7 / 43.5
    // -> 8.6 / 8.7 us; 64 x 20224 plain, rank 40: 74 -> 29).  The first one writes what is not T.
    const bool first_block = RP == 0 || blockIdx.y == 0;
    const int rb = RP == 0 ? 0 : min(r - RP * (int)blockIdx.y, RP);
    if constexpr (RP > 0) U += RP * blockIdx.y;

    uint4 v[kRegChunks];
#pragma unroll
    for (int c = 0; c < kRegChunks; ++c) {
        int idx = tid + c * kThreads;
        v[c] = make_uint4(0, 0, 0, 0);
        if (idx < nchunk) v[c] = xrow[idx];
    }
    // Eight ranks behind the RMS normalisation: the rows of U that meet the thread's first chunk are loaded here, not behind the
    // normalisation whose result they are multiplied with (300 x 5120: 10.4 -> 8.7 us, 800 x 4096: 12.0 -> 11.1, 16 x 8192:
    // 9.1 -> 8.9; behind the other producers it cost 1 to 4 %).  A row past the end is read as row 0 and zeroed at its use.
    // In 1024 threads (few tokens, or rows beyond 8192 elements) only where it gains: a thread with several chunks of the row, and
    // of the residual, ahead of its sums waits for these loads as well (1 x 11008 with a residual: 10.1 us with them, 9.4 without;
    // 128 x 20480: 13.3, 12.4; 300 x 11008, no residual: 18.5, 17.7; the other way round at 300 x 20480 with one: 26.3, 28.9).
    constexpr bool EARLY_U = RP > 0 && RP <= 8 && NORM == 1;
    Ranks<EARLY_U ? RP : 8> u0[EARLY_U ? 8 : 1];
    const int64_t k0 = (int64_t)(tid & ~63) * 8 + (tid & 63);
    const bool early = EARLY_U && (r & (RP < 8 ? RP - 1 : 7)) == 0 &&
                       (NT != 1024 || (K > 4096 && K <= 8192) || (pr.other == nullptr ? K > 12288 : K > 16384 && gridDim.x > 256));
    if constexpr (EARLY_U) {
        if (early && (tid & ~63) < nchunk) {
#pragma unroll
            for (int i = 0; i < 8; ++i) u0[i] = *reinterpret_cast<const Ranks<RP>*>(U + (k0 + 64 * i < K ? ((uint32_t)k0 + 64u * i) * (uint32_t)r : 0u));  // K <= 32768
        }
    }
    if constexpr (NORM != 0) {  // the whole row sits in registers (the launcher guarantees K <= 8 * kRegChunks * NT)
        if (pr.other != nullptr || NORM == 4) {
            const uint4* orow = reinterpret_cast<const uint4*>(pr.other + row * pr.ld_other);
            uint4* hrow = reinterpret_cast<uint4*>(pr.H + row * K);
#pragma unroll
            for (int c = 0; c < kRegChunks; ++c) {
                const int idx = tid + c * kThreads;
                if (idx < nchunk) {
                    if constexpr (NORM == 4) {
                        v[c] = swiglu8(v[c], orow[idx]);
                        if (pr.H != nullptr && first_block) hrow[idx] = v[c];
                    } else {
                        v[c] = add8(v[c], orow[idx]);
                        if (first_block) hrow[idx] = v[c];
                    }
                }
            }
        }
        if constexpr (NORM == 3) {
#pragma unroll
            for (int c = 0; c < kRegChunks; ++c) v[c] = relu8(v[c]);
        }
    }
    if constexpr (NORM == 1 || NORM == 2) {
        // the whole row sits in registers (the launcher guarantees K <= 8 * kRegChunks * NT): sum of
        // squares (and of the values, for layer normalisation) in binary64, waves meet in LDS and
        // every thread adds the partial sums in the same order; then the normalised row replaces the row
        __shared__ double s_ss[kWaves], s_s1[NORM == 2 ? kWaves : 1];
        const uint4* grow = reinterpret_cast<const uint4*>(gain);
        const uint4* brow = reinterpret_cast<const uint4*>(bias);
        uint4 g[kRegChunks], b[NORM == 2 ? kRegChunks : 1];
        double ss = 0.0, s1 = 0.0;
#pragma unroll
        for (int c = 0; c < kRegChunks; ++c) {
            int idx = tid + c * kThreads;
            g[c] = make_uint4(0, 0, 0, 0);
            if (idx < nchunk) g[c] = grow[idx];
            if constexpr (NORM == 2) {
                b[c] = make_uint4(0, 0, 0, 0);
                if (idx < nchunk) b[c] = brow[idx];
                s1 = sum_values(s1, v[c]);
            }
            ss = sum_squares(ss, v[c]);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            ss += __shfl_xor(ss, off);
            if constexpr (NORM == 2) s1 += __shfl_xor(s1, off);
        }
        if ((tid & 63) == 0) {
            s_ss[tid >> 6] = ss;
            if constexpr (NORM == 2) s_s1[tid >> 6] = s1;
        }
        __syncthreads();
        ss = s_ss[0];
        if constexpr (NORM == 2) s1 = s_s1[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            ss += s_ss[w];
            if constexpr (NORM == 2) s1 += s_s1[w];
        }
        float mu, rstd;
        row_statistics<NORM>(s1, ss, K, eps, mu, rstd);
#pragma unroll
        for (int c = 0; c < kRegChunks; ++c) {
            if constexpr (NORM == 2) {
                // chunks past the row's end stay zero: the bias must not leak into the absmax
                if (tid + c * kThreads < nchunk) v[c] = normalize8_affine(v[c], g[c], b[c], mu, rstd);
            } else {
                v[c] = normalize8(v[c], g[c], rstd);
            }
        }
    }
    uint32_t am = 0;
#pragma unroll
    for (int c = 0; c < kRegChunks; ++c) am = absmax_bits(am, v[c]);
    if constexpr (NORM == 0)
        for (int idx = tid + kRegChunks * kThreads; idx < nchunk; idx += kThreads) am = absmax_bits(am, xrow[idx]);

    // LoRC left factor first: its loads of U overlap the row's own loads and the absmax reduction.
    // A lane holds 8 consecutive elements; for the product with U it trades them, through a
    // wave-private LDS slice, for the 8 elements lane, lane + 64, ... of the wave's 512.
    float acc[RP > 0 ? RP : 1];
    if constexpr (RP > 0) {
        const int wave = tid >> 6, lane = tid & 63;
#pragma unroll
        for (int j = 0; j < RP; ++j) acc[j] = 0.0f;
        auto one_chunk = [&](uint4 vc, int idx, bool first = false) {
            *reinterpret_cast<uint4*>(&s_x[wave][lane * 8]) = vc;  // same wave writes and reads: no barrier
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = __uint_as_float((uint32_t)s_x[wave][lane + 64 * i] << 16);
            if constexpr (EARLY_U)
                if (first && early) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        add_ranks<RP>(acc, x[i], u0[i], k0 + 64 * i < K);
                    }
                    return;
                }
            lorc_accumulate<RP, ROWS>(acc, x, U, (int64_t)(idx - lane) * 8 + lane, K, r, rb);
        };
#pragma unroll
        for (int c = 0; c < kRegChunks; ++c) {
            int idx = tid + c * kThreads;
            if (idx - lane < nchunk) one_chunk(idx < nchunk ? v[c] : make_uint4(0, 0, 0, 0), idx, c == 0);
        }
        if constexpr (NORM == 0)
            for (int idx = tid + kRegChunks * kThreads; idx - lane < nchunk; idx += kThreads)
                one_chunk(idx < nchunk ? xrow[idx] : make_uint4(0, 0, 0, 0), idx);
    }

#pragma unroll
    for (int off = 32; off > 0; off >>= 1) am = max(am, (uint32_t)__shfl_xor((int)am, off));
    if ((tid & 63) == 0) s_amax[tid >> 6] = am;
    __syncthreads();
    am = s_amax[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) am = max(am, s_amax[w]);

    const float amax = __uint_as_float(am << 16);
    float scale = 1.0f, inv = 0.0f;  // all-zero (or vanishing) token: signed-zero codes, scale 1
    if (amax >= 0x1p-96f) {
        scale = amax / 448.0f;  // IEEE binary32 division
        inv = 448.0f / amax;    // IEEE binary32 division
    }
    if (tid == 0 && first_block) sx[row] = scale;

#pragma unroll
    for (int c = 0; c < kRegChunks; ++c) {
        int idx = tid + c * kThreads;
        if (idx < nchunk && first_block) qrow[idx] = encode8(v[c], inv);
    }
    if constexpr (NORM == 0)
        for (int idx = tid + kRegChunks * kThreads; idx < nchunk && first_block; idx += kThreads) qrow[idx] = encode8(xrow[idx], inv);

    if constexpr (RP > 0) {
#pragma unroll
        for (int j = 0; j < RP; ++j) {
            float a = acc[j];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off);
            if ((tid & 63) == 0) s_t[tid >> 6][j] = a;
        }
        __syncthreads();
        if (tid < rb) {  // fixed order: pairs of waves, then the pairs in sequence
            float t = 0.0f;
#pragma unroll
            for (int w = 0; w < kWaves; w += 2) t += s_t[w][tid] + s_t[w + 1][tid];
            T[row * r + RP * blockIdx.y + tid] = t;
        }
    }
}

// ---------------------------------------------------------------------------
// Wave-per-token form for many tokens without the LoRC factor: a row of up to 8 * 64 * MAXC
// elements sits in one wave's registers (16 B per lane per load, 1 KB contiguous per instruction),
// the reductions are wave shuffles only, and no barrier or LDS is involved; 16 waves per compute
// unit keep 8 * MAXC KB of loads in flight each.
// ---------------------------------------------------------------------------
// LORC: the rank-8 left factor T = y . U rides along.  The workgroup then has eight waves (eight tokens) and keeps
// the whole of U (K x 8 binary16 values, 16 bytes per row, at most 128 KB) in LDS: the loads of U are issued ahead of
// the row's own, so that they are the first to land, and the multiply-adds of a chunk start as soon as that chunk
// of the row has arrived, while the rest of the row is still on its way -- there is no barrier and no further load
// in the loop.
template <int MAXC, int NORM, bool LORC>
__global__ __launch_bounds__(LORC ? 512 : 256) void k_quantize_rows(const uint16_t* __restrict__ X, int64_t M, int64_t K, int64_t ldx,
                                                     uint8_t* __restrict__ Xq, float* __restrict__ sx,
                                                     const uint16_t* __restrict__ U, float* __restrict__ T, Producer pr)
{
    const uint16_t* __restrict__ gain = pr.gain;
    const uint16_t* __restrict__ bias = pr.bias;
    const float eps = pr.eps;
    const int lane = threadIdx.x & 63;
    constexpr int kRowsPerWg = LORC ? 8 : 4;
    int64_t row = (int64_t)blockIdx.x * kRowsPerWg + (threadIdx.x >> 6);
    bool live = true;  // LORC: the waves stage U together, so a wave past the last token stays, repeats that token and stores nothing
    if (row >= M) {
        if constexpr (!LORC) return;  // whole waves leave; nothing below synchronises across waves
        live = false;
        row = M - 1;
    }
    const uint4* xrow = reinterpret_cast<const uint4*>(X + row * ldx);
    uint2* qrow = reinterpret_cast<uint2*>(Xq + row * K);
    const int nchunk = (int)(K / 8);

    // LORC: row k of U is 8 binary16 values, one uint4.  Thread t fetches row 512 c + t of every 512-row chunk c
    // (past K: the last row; the row's elements are zero there) and stores it at slot 64 i + (l ^ 2 i) of the
    // chunk, i = t % 8, l = t / 8: lane l, which holds elements 8 l .. 8 l + 7 of the chunk, then finds the row of
    // its i-th element at slot 64 i + (l ^ 2 i) -- for a fixed i the 64 lanes read 64 consecutive slots in a
    // permuted order (conflict-free 16-byte reads, no exchange of elements), and the sixteen lanes that store
    // together (two values of l, all eight i) hit sixteen different slots of a 16-slot block (without the XOR
    // they would hit two, eight lanes each).
    // Every load of this form is unconditional (indices past the end are clamped into the row, what they fetch is
    // replaced by zeros afterwards): with loads inside branches the compiler can no longer count the outstanding ones
    // and waits for all of them at the first use of any.
    extern __shared__ __attribute__((aligned(16))) uint4 s_u[];  // LORC: MAXC * 512 slots
    uint4 ureg[LORC ? MAXC : 1];
    if constexpr (LORC) {
        const uint4* u4 = reinterpret_cast<const uint4*>(U);
#pragma unroll
        for (int c = 0; c < MAXC; ++c) {
            const int64_t k = (int64_t)c * 512 + threadIdx.x;
            ureg[c] = u4[k < K ? k : K - 1];
        }
    }
    uint4 v[MAXC];
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        const int idx = c * 64 + lane;
        if constexpr (LORC) {
            v[c] = xrow[idx < nchunk ? idx : nchunk - 1];
        } else {
            v[c] = make_uint4(0, 0, 0, 0);
            if (idx < nchunk) v[c] = xrow[idx];
        }
    }
    if constexpr (LORC) {  // needs the loads of U only: the row's are younger
        const int slot = (threadIdx.x & 7) * 64 + ((threadIdx.x >> 3) ^ (2 * (threadIdx.x & 7)));
#pragma unroll
        for (int c = 0; c < MAXC; ++c) s_u[c * 512 + slot] = ureg[c];
        __syncthreads();
    }
    auto zero_past_end = [&](int c) {  // LORC: what the clamped loads fetched past the row's end
        if (c * 64 + lane >= nchunk) v[c] = make_uint4(0, 0, 0, 0);
    };
    if constexpr (LORC && NORM != 0) {
#pragma unroll
        for (int c = 0; c < MAXC; ++c) zero_past_end(c);
    }
    if constexpr (NORM != 0) {
        if (pr.other != nullptr || NORM == 4) {
            const uint4* orow = reinterpret_cast<const uint4*>(pr.other + row * pr.ld_other);
            uint4* hrow = reinterpret_cast<uint4*>(pr.H + row * K);
#pragma unroll
            for (int c = 0; c < MAXC; ++c) {
                const int idx = c * 64 + lane;
                if (idx < nchunk) {
                    if constexpr (NORM == 4) {
                        v[c] = swiglu8(v[c], orow[idx]);
                        if (pr.H != nullptr && live) hrow[idx] = v[c];
                    } else {
                        v[c] = add8(v[c], orow[idx]);
                        if (live) hrow[idx] = v[c];
                    }
                }
            }
        }
        if constexpr (NORM == 3) {
#pragma unroll
            for (int c = 0; c < MAXC; ++c) v[c] = relu8(v[c]);
        }
    }
    if constexpr (NORM == 1 || NORM == 2) {
        double ss = 0.0, s1 = 0.0;
#pragma unroll
        for (int c = 0; c < MAXC; ++c) {
            ss = sum_squares(ss, v[c]);
            if constexpr (NORM == 2) s1 = sum_values(s1, v[c]);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {  // every lane ends with the same sums
            ss += __shfl_xor(ss, off);
            if constexpr (NORM == 2) s1 += __shfl_xor(s1, off);
        }
        float mu, rstd;
        row_statistics<NORM>(s1, ss, K, eps, mu, rstd);
        const uint4* grow = reinterpret_cast<const uint4*>(gain);
        const uint4* brow = reinterpret_cast<const uint4*>(bias);
#pragma unroll
        for (int c = 0; c < MAXC; ++c) {
            const int idx = c * 64 + lane;
            if (idx < nchunk) {
                if constexpr (NORM == 2) v[c] = normalize8_affine(v[c], grow[idx], brow[idx], mu, rstd);
                else v[c] = normalize8(v[c], grow[idx], rstd);
            }
        }
    }
    float acc[8];
    if constexpr (LORC) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
#pragma unroll
        for (int c = 0; c < MAXC; ++c) {
            if constexpr (NORM == 0) zero_past_end(c);  // here, so that chunk c waits for its own load only
            if (c * 64 < nchunk) {  // the same for the whole workgroup; lanes past the row's end hold zeros
                const uint32_t xw[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float x = __uint_as_float((i & 1) ? (xw[i >> 1] & 0xffff0000u) : (xw[i >> 1] << 16));
                    const uint4 u = s_u[c * 512 + 64 * i + (lane ^ (2 * i))];
                    const uint32_t uw[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        // binary16 halves of a dword, widened inside the multiply-add (mixed-precision FMA: the same
                        // exact widening and one binary32 rounding as convert-then-fma, without the conversions)
                        const half2_t p = __builtin_bit_cast(half2_t, uw[q]);
                        acc[2 * q] = fmaf(x, (float)p[0], acc[2 * q]);
                        acc[2 * q + 1] = fmaf(x, (float)p[1], acc[2 * q + 1]);
                    }
                }
            }
        }
    }
    uint32_t am = 0;
#pragma unroll
    for (int c = 0; c < MAXC; ++c) am = absmax_bits(am, v[c]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) am = max(am, (uint32_t)__shfl_xor((int)am, off));
    const float amax = __uint_as_float(am << 16);
    float scale = 1.0f, inv = 0.0f;  // all-zero (or vanishing) token: signed-zero codes, scale 1
    if (amax >= 0x1p-96f) {
        scale = amax / 448.0f;  // IEEE binary32 division
        inv = 448.0f / amax;    // IEEE binary32 division
    }
    if (lane == 0 && live) sx[row] = scale;
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        const int idx = c * 64 + lane;
        if (idx < nchunk && live) qrow[idx] = encode8(v[c], inv);
    }
    if constexpr (LORC) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float a = acc[j];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off);
            if (lane == 0 && live) T[row * 8 + j] = a;
        }
    }
}

// The same with a helper wave per token (plain and ReLU forms, rows of at most 5120 elements): 2048 tokens are only
// eight waves per compute unit, and a lone chain of K x 8 multiply-adds per token is what the call then waits for
// (one or two waves per SIMD issue a vector instruction every 12 or 6 cycles).  Sixteen waves per workgroup: wave
// w < 8 owns token w as before but multiplies only the first H chunks of its row; wave w + 8 fetches the other
// chunks of the same row (the requests of the token wave for them, issued behind the staging barrier, then hit in
// L2), multiplies them and hands its eight partial sums over through LDS.  Both kinds issue the same number of
// loads ahead of the barrier, in the same straight-line code, so the compiler's load counts stay exact.
template <int MAXC, int NORM>
__global__ __launch_bounds__(1024) void k_quantize_rows_helped(const uint16_t* __restrict__ X, int64_t M, int64_t K, int64_t ldx,
                                                             uint8_t* __restrict__ Xq, float* __restrict__ sx,
                                                             const uint16_t* __restrict__ U, float* __restrict__ T)
{
    static_assert(NORM == 0 || NORM == 3, "element-wise producers only: a helper has half a row");
    constexpr int H = (MAXC + 1) / 2, R = MAXC - H;  // chunks multiplied by the token wave / by its helper
    extern __shared__ __attribute__((aligned(16))) uint4 s_u[];  // MAXC * 512 slots, as in k_quantize_rows
    __shared__ float s_part[8][8];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const bool helper = w >= 8;  // wave-uniform
    int64_t row = (int64_t)blockIdx.x * 8 + (w & 7);
    const bool live = row < M;
    if (!live) row = M - 1;  // stays for the barriers, repeats the last token, stores nothing
    const uint4* xrow = reinterpret_cast<const uint4*>(X + row * ldx);
    uint2* qrow = reinterpret_cast<uint2*>(Xq + row * K);
    const int nchunk = (int)(K / 8);
    const int base = helper ? H : 0;  // first chunk of this wave's share

    // U: the 512 threads of each half of the workgroup take the chunks of one parity (a chunk past the last is the
    // last again: the same rows to the same slots)
    uint4 ureg[H];
    const int st = threadIdx.x & 511, par = threadIdx.x >> 9;
    const uint4* u4 = reinterpret_cast<const uint4*>(U);
#pragma unroll
    for (int j = 0; j < H; ++j) {
        const int c = min(2 * j + par, MAXC - 1);
        const int64_t k = (int64_t)c * 512 + st;
        ureg[j] = u4[k < K ? k : K - 1];
    }
    uint4 f[H];  // this wave's share of the row (a helper with one chunk less fetches its last one twice)
#pragma unroll
    for (int c = 0; c < H; ++c) {
        const int idx = min(base + c, MAXC - 1) * 64 + lane;
        f[c] = xrow[idx < nchunk ? idx : nchunk - 1];
    }
    {
        const int slot = (st & 7) * 64 + ((st >> 3) ^ (2 * (st & 7)));
#pragma unroll
        for (int j = 0; j < H; ++j) s_u[min(2 * j + par, MAXC - 1) * 512 + slot] = ureg[j];
    }
    __syncthreads();
    // the rest of the row, which the token wave needs for the maximum and the codes (its helper asked for the same
    // lines ahead of the barrier).  Issued by both kinds of wave, so that no load sits in a branch.
    uint4 g[R > 0 ? R : 1];
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const int idx = (H + c) * 64 + lane;
        g[c] = xrow[idx < nchunk ? idx : nchunk - 1];
    }
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
#pragma unroll
    for (int c = 0; c < H; ++c) {
        const int ch = base + c;  // the chunk in f[c]; a helper's repeated last chunk counts for nothing
        if (ch * 64 + lane >= nchunk || ch >= MAXC) f[c] = make_uint4(0, 0, 0, 0);
        if constexpr (NORM == 3) f[c] = relu8(f[c]);
        if (ch * 64 < nchunk && ch < MAXC) {  // wave-uniform
            const uint32_t xw[4] = {f[c].x, f[c].y, f[c].z, f[c].w};
            const uint4* su = s_u + ch * 512;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float x = __uint_as_float((i & 1) ? (xw[i >> 1] & 0xffff0000u) : (xw[i >> 1] << 16));
                const uint4 u = su[64 * i + (lane ^ (2 * i))];
                const uint32_t uw[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const half2_t p = __builtin_bit_cast(half2_t, uw[q]);  // widened inside the multiply-add, as above
                    acc[2 * q] = fmaf(x, (float)p[0], acc[2 * q]);
                    acc[2 * q + 1] = fmaf(x, (float)p[1], acc[2 * q + 1]);
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc[j] += __shfl_xor(acc[j], off);
    }
    float mine = acc[0];  // every lane holds all eight sums: lane j keeps the j-th
#pragma unroll
    for (int j = 1; j < 8; ++j) mine = lane == j ? acc[j] : mine;
    if (helper) {
        if (lane < 8) s_part[w - 8][lane] = mine;
        __syncthreads();
        return;
    }
    uint32_t am = 0;
#pragma unroll
    for (int c = 0; c < H; ++c) am = absmax_bits(am, f[c]);
#pragma unroll
    for (int c = 0; c < R; ++c) {
        if ((H + c) * 64 + lane >= nchunk) g[c] = make_uint4(0, 0, 0, 0);
        if constexpr (NORM == 3) g[c] = relu8(g[c]);
        am = absmax_bits(am, g[c]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) am = max(am, (uint32_t)__shfl_xor((int)am, off));
    float scale, inv;
    token_scale(am, scale, inv);
    if (lane == 0 && live) sx[row] = scale;
#pragma unroll
    for (int c = 0; c < H; ++c) {
        const int idx = c * 64 + lane;
        if (idx < nchunk && live) qrow[idx] = encode8(f[c], inv);
    }
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const int idx = (H + c) * 64 + lane;
        if (idx < nchunk && live) qrow[idx] = encode8(g[c], inv);
    }
    __syncthreads();  // the helper's sums are in LDS
    if (lane < 8 && live) T[row * 8 + lane] = mine + s_part[w][lane];  // first half of the row plus second half: a fixed order
}

// ---------------------------------------------------------------------------
// The left factor alone, T = y . U, for many tokens with more than 8 ranks: a launch of its own behind the quantizer without
// one.  On the float32 matrix cores (v_mfma_f32_16x16x4_f32; in bfloat16, with U as the sum of two, the products are exact as
// well but the unit drops bits of a run of eight: 4.4e-7 against 1e-7 relative error at 20224 elements).  A workgroup takes
// 16 tokens and 16 * NB ranks, its eight waves split K.  A wave takes 64 elements at a time, a line of every row, PF such units ahead;
// which element of its eight a lane feeds to an instruction is free as long as U's rows follow, so both operands are used as
// they come, and U goes through the wave's own slice of LDS, which turns it round (a row of U is sixteen ranks, the operand
// wants one of eight rows per lane).  The sums of 16 elements are added to the total with its rounding compensated, which keeps
// the error at that of the other forms' trees (9e-8 at 4096 elements, 9e-8 against 1.25e-7 at 20224).  Bound by the matrix cores and
// the scattered 16-byte pieces of X and U, about a microsecond per unit and wave.  With the quantizer, before -> now: 4000 x 4096
// plain, rank 16 / 40: 50 -> 22.5 / 257 -> 37 us; 1000 x 11008 RMS normalisation, rank 40: 304 -> 64; 4000 x 2048, rank 64: 328 -> 39.
// NORM as above, but a residual has been added already (X is then H).  Row statistics are formed again, in another order of
// the same binary64 sums.
// ---------------------------------------------------------------------------
typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int NORM, int NB>
__global__ __launch_bounds__(512) void k_lorc_left(const uint16_t* __restrict__ X, int64_t M, int64_t K, int64_t ldx,
                                                   const uint16_t* __restrict__ U, int r, float* __restrict__ T, Producer pr)
{
    constexpr int kSlice = 32 * 16 + 3 * 16;  // binary16 values of 32 rows x 16 ranks; 16 more behind every 8 rows spread the reads over all banks
    constexpr int kWaveBytes = NB * kSlice * 2 > NB * 1024 ? NB * kSlice * 2 : NB * 1024;
    __shared__ __attribute__((aligned(16))) uint8_t s_mem[8 * kWaveBytes];  // slices of U, then the waves' sums
    __shared__ float s_stat[NORM == 1 || NORM == 2 ? 16 : 1][2];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t m0 = (int64_t)blockIdx.x * 16;
    const int q0 = (int)blockIdx.y * (16 * NB);  // first rank of the workgroup

    if constexpr (NORM == 1 || NORM == 2) {
        const int nchunk = (int)(K / 8);
        for (int rr = 0; rr < 2; ++rr) {
            const uint4* x = reinterpret_cast<const uint4*>(X + min(m0 + 2 * wave + rr, M - 1) * ldx);
            double ss = 0.0, s1 = 0.0;
            for (int i0 = lane; i0 < nchunk; i0 += 256) {
                uint4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = x[min(i0 + 64 * u, nchunk - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (i0 + 64 * u < nchunk) {
                        ss = sum_squares(ss, v[u]);
                        if constexpr (NORM == 2) s1 = sum_values(s1, v[u]);
                    }
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                ss += __shfl_xor(ss, off);
                if constexpr (NORM == 2) s1 += __shfl_xor(s1, off);
            }
            float mu, rstd;
            row_statistics<NORM>(s1, ss, K, pr.eps, mu, rstd);
            if (lane == 0) {
                s_stat[2 * wave + rr][0] = mu;
                s_stat[2 * wave + rr][1] = rstd;
            }
        }
        __syncthreads();
    }
    const int row = lane & 15, lb = lane >> 4;
    float mu = 0.0f, rstd = 0.0f;
    if constexpr (NORM == 1 || NORM == 2) {
        mu = s_stat[row][0];
        rstd = s_stat[row][1];
    }
    // operand A: lane (row, lb) holds y[row][8 lb + [0, 8)] of a step of 32; two steps are a line of every row
    const int64_t mrow = min(m0 + row, M - 1);  // a row past the end repeats the last one and is not stored
    const uint16_t* xp = X + mrow * ldx + 8 * lb;
    const uint16_t* op = NORM == 4 ? pr.other + mrow * pr.ld_other + 8 * lb : nullptr;
    // U: lane l fetches ranks 8 (l % 2) + [0, 8) of row l / 2 of a step; ranks past the last are zeroed in the slice
    const int uk = lane >> 1, un = q0 + 8 * (lane & 1);
    const bool whole = (r & 7) == 0;  // eight ranks lie on 16 bytes
    uint16_t* slice = reinterpret_cast<uint16_t*>(s_mem + wave * kWaveBytes);
    uint16_t* const put = slice + uk * 16 + (uk >> 3) * 16 + 8 * (lane & 1);
    const uint16_t* const get = slice + lb * (8 * 16 + 16) + row;

    struct Fetched {
        uint4 x[2], o[NORM == 4 ? 2 : 1], g[NORM == 1 || NORM == 2 ? 2 : 1], b[NORM == 2 ? 2 : 1], u[2][NB];
    };
    const int units = (int)(K / 64);
    auto fetch = [&](Fetched& f, int unit) __attribute__((always_inline)) {
        const int64_t k = (int64_t)min(unit, units - 1) * 64;  // past the end: the last again, unused
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            f.x[s] = *reinterpret_cast<const uint4*>(xp + k + 32 * s);
            if constexpr (NORM == 4) f.o[s] = *reinterpret_cast<const uint4*>(op + k + 32 * s);
            if constexpr (NORM == 1 || NORM == 2) f.g[s] = *reinterpret_cast<const uint4*>(pr.gain + k + 32 * s + 8 * lb);
            if constexpr (NORM == 2) f.b[s] = *reinterpret_cast<const uint4*>(pr.bias + k + 32 * s + 8 * lb);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int n = un + 16 * nb;
                const uint16_t* p = U + (k + 32 * s + uk) * r;
                if (whole) {
                    f.u[s][nb] = *reinterpret_cast<const uint4*>(p + (n < r ? n : 0));
                } else {
                    uint32_t w[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) w[j] = p[min(n + j, r - 1)];
                    f.u[s][nb] = make_uint4(w[0] | w[1] << 16, w[2] | w[3] << 16, w[4] | w[5] << 16, w[6] | w[7] << 16);
                }
            }
        }
    };
    f32x4_t acc[NB], lost[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = lost[nb] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    bool live[NB];  // this lane's rank (its operand column) exists
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) live[nb] = q0 + 16 * nb + row < r;
    auto multiply = [&](const Fetched& f) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            uint4 y = f.x[s];
            if constexpr (NORM == 1) y = normalize8(y, f.g[s], rstd);
            if constexpr (NORM == 2) y = normalize8_affine(y, f.g[s], f.b[s], mu, rstd);
            if constexpr (NORM == 3) y = relu8(y);
            if constexpr (NORM == 4) y = swiglu8(y, f.o[s]);
            const uint32_t yw[4] = {y.x, y.y, y.z, y.w};
            __builtin_amdgcn_wave_barrier();  // behind the reads of the step before
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<uint4*>(put + nb * kSlice) = f.u[s][nb];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            uint16_t h[NB][8];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int i = 0; i < 8; ++i) h[nb][i] = get[nb * kSlice + 16 * i];
            f32x4_t part[NB][2];  // even and odd elements
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) part[nb][0] = part[nb][1] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float a = (i & 1) ? bf16_hi(yw[i >> 1]) : bf16_lo(yw[i >> 1]);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    part[nb][i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, live[nb] ? half_bits_to_f32(h[nb][i]) : 0.0f, part[nb][i & 1], 0, 0, 0);
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {  // compensated: what the total's rounding drops is added to the next sum
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4_t add = part[nb][h] - lost[nb], total = acc[nb] + add;
#pragma unroll
                    for (int i = 0; i < 4; ++i) lost[nb][i] = fabsf(total[i]) <= 0x1.fffffep127f ? (total[i] - acc[nb][i]) - add[i] : 0.0f;  // an infinity stays one
                    acc[nb] = total;
                }
            }
        }
    };
    constexpr int PF = NB == 1 ? 4 : NB == 2 ? 3 : 2;
    {
        Fetched f[PF];
#pragma unroll
        for (int i = 0; i < PF - 1; ++i) fetch(f[i], wave + 8 * i);
        for (int u = wave; u < units;) {
#pragma unroll
            for (int i = 0; i < PF; ++i) {
                fetch(f[(i + PF - 1) % PF], u + 8 * (PF - 1));
                __builtin_amdgcn_sched_barrier(0);
                multiply(f[i]);
                __builtin_amdgcn_sched_barrier(0);
                u += 8;
                if (u >= units) break;
            }
        }
    }
    __syncthreads();  // the waves' slices become their sums
    float* part = reinterpret_cast<float*>(s_mem);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<f32x4_t*>(part + ((wave * NB + nb) * 64 + lane) * 4) = acc[nb];
    __syncthreads();
    // D[row][col] sits in lane 16 (row / 4) + col, register row % 4; the waves' sums in order
    for (int o = tid; o < NB * 256; o += 512) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) t += part[w * NB * 256 + o];
        const int nb = o >> 8, ln = (o >> 2) & 63;
        const int64_t m = m0 + 4 * (ln >> 4) + (o & 3);
        const int q = q0 + 16 * nb + (ln & 15);
        if (m < M && q < r) T[m * r + q] = t;
    }
}

template <int KIND>
hipError_t launch_lorc_left(const uint16_t* X, int64_t M, int64_t K, int64_t ldx, const uint16_t* U, int r, float* T,
                            const Producer& pr, hipStream_t s)
{
    // sixteen ranks per workgroup while that leaves the chip idle, all of them where it would read the activations again for nothing
    const unsigned gm = (unsigned)((M + 15) / 16), blocks = (unsigned)((r + 15) / 16);
    const dim3 wg(512);
    if (blocks == 1 || (int64_t)gm * blocks <= 2 * compute_units()) hipLaunchKernelGGL((k_lorc_left<KIND, 1>), dim3(gm, blocks), wg, 0, s, X, M, K, ldx, U, r, T, pr);
    else if (blocks == 3) hipLaunchKernelGGL((k_lorc_left<KIND, 3>), dim3(gm, 1), wg, 0, s, X, M, K, ldx, U, r, T, pr);
    else hipLaunchKernelGGL((k_lorc_left<KIND, 2>), dim3(gm, blocks / 2), wg, 0, s, X, M, K, ldx, U, r, T, pr);  // 2 or 4 blocks; four at once spill
    return hipGetLastError();
}

// The plain quantizer's blocks of eight ranks have an instance for each way to read U: with both in one, its registers leave room for
// four waves per SIMD (97 of them) in place of five and seven, which a launch of 1025 to 1280 tokens pays with a second round
// (1100 x 4096, rank 6: 26.6 -> 19.8 us; 1100 x 28672, rank 8: 50.0 -> 43.5).  Held to five waves in one instance, the loads of U no longer run
// ahead of their sums (2048 x 28672, rank 8: 102, 69.7 now).
template <int RP, int NT>
void launch_plain(dim3 grid, hipStream_t s, const uint16_t* X, int64_t K, int64_t ldx, uint8_t* Xq, float* sx, const uint16_t* U, int r, float* T,
                  const Producer& pr)
{
    if constexpr (RP == 8 && NT == 256) {
        if (r % 8 == 0) hipLaunchKernelGGL((k_quantize_act<RP, NT, 0, Rows::kWhole>), grid, dim3(NT), 0, s, X, K, ldx, Xq, sx, U, r, T, pr);
        else hipLaunchKernelGGL((k_quantize_act<RP, NT, 0, Rows::kSingle>), grid, dim3(NT), 0, s, X, K, ldx, Xq, sx, U, r, T, pr);
    } else {
        hipLaunchKernelGGL((k_quantize_act<RP, NT, 0>), grid, dim3(NT), 0, s, X, K, ldx, Xq, sx, U, r, T, pr);
    }
}

// whether the bytes of two strided [M, K] bf16 matrices can meet
bool overlap(const void* a, int64_t lda, const void* b, int64_t ldb, int64_t M, int64_t K)
{
    if (a == nullptr || b == nullptr) return false;
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return a0 < b0 + 2 * (uintptr_t)((M - 1) * ldb + K) && b0 < a0 + 2 * (uintptr_t)((M - 1) * lda + K);
}

// the wave-per-token kernel with the rank-8 factor: eight tokens per workgroup, all of U in dynamic LDS
template <int MAXC, int KIND>
hipError_t launch_rows_lorc(const uint16_t* X, int64_t M, int64_t K, int64_t ldx, uint8_t* Xq, float* sx, const uint16_t* U,
                            float* T, const Producer& pr, hipStream_t s)
{
    const size_t smem = (size_t)MAXC * 512 * sizeof(uint4);
    static OnceStatus attr;  // raising the dynamic LDS limit is a per-function, per-process setting
    // A helper wave per token while every compute unit gets at most one workgroup (its 16 waves leave 128 registers
    // each, hence rows of at most 5120 elements): 2048 x 5120 12.1 -> 11.0 us, 1024 x 5120 11.1 -> 9.9.  With more
    // tokens the waves of later workgroups fill the SIMDs anyway and the helpers' second fetch of half of every row
    // only costs (4096 x 4096: 16.6 -> 19.3 us), so the plain form stays.
    if constexpr ((KIND == 0 || KIND == 3) && MAXC <= 10) {
        if ((M + 7) / 8 <= compute_units()) {
            auto kern = k_quantize_rows_helped<MAXC, KIND>;
            static OnceStatus attr_helped;
            if (hipError_t e = run_once(attr_helped, [&] {
                    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
                }); e != hipSuccess)
                return e;
            hipLaunchKernelGGL(kern, dim3((unsigned)((M + 7) / 8)), dim3(1024), smem, s, X, M, K, ldx, Xq, sx, U, T);
            return hipGetLastError();
        }
    }
    auto kern = k_quantize_rows<MAXC, KIND, true>;
    if (hipError_t e = run_once(attr, [&] {
            return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        }); e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)((M + 7) / 8)), dim3(512), smem, s, X, M, K, ldx, Xq, sx, U, T, pr);
    return hipGetLastError();
}

}  // namespace

// In microseconds, graph-timed; b = blocks of 8 ranks.  Blocks cost about M b rows, kApart is flat up to 2000 tokens and then follows
// the activations, so the line between them is one in M b^2: plain, 4096 elements, rank 40, 64 / 128 / 300 / 800 tokens: 13.6 / 12.0 / 20.8
// / 44.4 in blocks, 13.2 / 13.1 / 13.4 / 14.4 apart; rank 24, 300 / 800: 11.0 / 21.9, 13.3 / 14.0.  Behind a normalisation kApart reads
// the rows twice (rank 40, 128 / 300 / 800 tokens: 13.3 / 21.5 / 46.9, 19.6 / 20.1 / 21.8; 11008 elements: 38 / 76 / 184, 40 / 47 / 59), behind
// the gated unit it evaluates it again (300 / 800: 22 / 46, 34 / 37; 11008: 72 / 178, 76 / 86).
//
// Up to 16 ranks there is one workgroup with all sums as well, which reads the row once.  The lines are set where neither side is slower than
// that one by more than 4 % (7000 timings: the seven producers and sums, 13 row lengths, 24 token counts, ranks 9, 12, 15 and 16).  Blocks win
// while both launches take as many rounds of workgroups: a row beyond 8192 elements behind a producer takes 1024 threads, one to a
// compute unit, so up to 128 tokens (layer normalisation with a residual, 14336 elements, rank 16: 128 tokens 13.9 in blocks, 15.9; 256 tokens 25.0, 17.7); else up to 512 (RMS normalisation, 512 x 4096, rank 16: 10.9, 11.8),
// the plain quantizer with ranks one at a time, whose seven waves a SIMD take 896 tokens at once, up to 768.  kApart pays off the sooner
// the longer the sums take: sixteen ranks come in one vector load, fewer one by one (plain, 1024 x 8192, rank 16: 18.7, 27.9 apart;
// rank 12: 58.5, 39.9).  Behind a normalisation its second reading of the rows counts (layer normalisation, 1400 x 8192, rank 16: 28.1, 52.6
// apart; 4096 x 2048: 34.8, 22.7), behind the gated unit its second evaluation (4000 x 4096: 52.7, 56.3).
LeftForm left_form(int64_t M, int64_t K, int r, int kind, bool in_place)
{
    if (r <= 8) return LeftForm::kBlocks;
    if (r <= 16) {
        const bool plain = kind == 0, whole = r == 16;
        const int64_t blocks = !plain && K > 8192 ? 128 : plain && !whole && K <= 8192 ? 768 : 512;
        if (!in_place && M <= blocks) return LeftForm::kBlocks;
        bool apart;
        if (plain || kind == 3) apart = whole ? M >= 1300 : plain || M >= 800;
        else if (kind == 4) apart = false;
        else apart = !whole ? M >= 1400 : K > 8192 ? M >= 1800 : M >= 1400 && M >= K;
        return apart ? LeftForm::kApart : LeftForm::kOne;
    }
    // with H over X or the second operand a row cannot be formed twice
    if (in_place) return LeftForm::kApart;
    const int64_t b = (r + 7) / 8, bound = kind == 0 || kind == 3 ? 3200 : kind == 4 ? (K > 8192 ? 6500 : 14000) : K > 8192 ? 3200 : 6000;
    return M * b * b > bound ? LeftForm::kApart : LeftForm::kBlocks;
}

hipError_t launch_quantize_act(const uint16_t* X, int64_t M, int64_t K, int64_t ldx, uint8_t* Xq, float* sx,
                               const uint16_t* U, int r, float* T, const Producer& pr, hipStream_t s)
{
    if (M == 0) return hipSuccess;
    const int kind = pr.kind;
    const bool in_place = overlap(pr.H, K, X, ldx, M, K) || overlap(pr.H, K, pr.other, pr.ld_other, M, K);
    const LeftForm form = left_form(M, K, r, kind, in_place);
    if (form == LeftForm::kApart) {
        if (hipError_t e = launch_quantize_act(X, M, K, ldx, Xq, sx, nullptr, 0, nullptr, pr, s); e != hipSuccess) return e;
        // behind the quantizer the sum with a residual, or the gated product, is read from H where there is one
        const bool from_h = pr.H != nullptr;
        const uint16_t* Y = from_h ? pr.H : X;
        const int64_t ldy = from_h ? K : ldx;
        switch (kind) {
        case 1: return launch_lorc_left<1>(Y, M, K, ldy, U, r, T, pr, s);
        case 2: return launch_lorc_left<2>(Y, M, K, ldy, U, r, T, pr, s);
        case 3: return launch_lorc_left<3>(Y, M, K, ldy, U, r, T, pr, s);
        case 4: if (!from_h) return launch_lorc_left<4>(Y, M, K, ldy, U, r, T, pr, s);
        }
        return launch_lorc_left<0>(Y, M, K, ldy, U, r, T, pr, s);
    }
    // many tokens: one wave per token, without the LoRC factor or with the rank-8 one (U in LDS)
    if (M >= 1024 && K <= 8192 && (r == 0 || r == 8)) {
        const dim3 g4((unsigned)((M + 3) / 4));
#define ZQ_ROWS_N(MAXC, KIND)                                                                                               \
    do {                                                                                                                    \
        if (r == 8) {  /* every chunk's load of U and of the row is issued: a tight chunk count wastes none */                 \
            constexpr int C1 = MAXC == 16 ? 10 : MAXC == 8 ? 6 : MAXC, C2 = MAXC == 16 ? 12 : MAXC;                              \
            hipError_t e = K <= 512 * C1   ? launch_rows_lorc<C1, KIND>(X, M, K, ldx, Xq, sx, U, T, pr, s)                       \
                           : K <= 512 * C2 ? launch_rows_lorc<C2, KIND>(X, M, K, ldx, Xq, sx, U, T, pr, s)                       \
                                           : launch_rows_lorc<MAXC, KIND>(X, M, K, ldx, Xq, sx, U, T, pr, s);                   \
            if (e != hipSuccess) return e;                                                                                      \
        } else {                                                                                                                \
            hipLaunchKernelGGL((k_quantize_rows<MAXC, KIND, false>), g4, dim3(256), 0, s, X, M, K, ldx, Xq, sx, U, T, pr);        \
        }                                                                                                                       \
    } while (0)
#define ZQ_ROWS(MAXC)                          \
    do {                                       \
        switch (kind) {                        \
        case 1: ZQ_ROWS_N(MAXC, 1); break;     \
        case 2: ZQ_ROWS_N(MAXC, 2); break;     \
        case 3: ZQ_ROWS_N(MAXC, 3); break;     \
        case 4: ZQ_ROWS_N(MAXC, 4); break;     \
        default: ZQ_ROWS_N(MAXC, 0); break;    \
        }                                      \
    } while (0)
        if (K <= 2048) ZQ_ROWS(4);
        else if (K <= 4096) ZQ_ROWS(8);
        else ZQ_ROWS(16);
#undef ZQ_ROWS
#undef ZQ_ROWS_N
        return hipGetLastError();
    }
    const bool wide_sums = r > 8 && form == LeftForm::kOne;
    // Four ranks per workgroup while that still gives every one a compute unit: half the loads of U and half the sums (16 x 8192, RMS
    // normalisation, rank 8 / 16: 9.6 -> 8.3 / 9.7 -> 8.5 us; 64 x 4096, rank 16: 9.0 -> 8.2; twice the units lose, rank 40: 18.0 -> 23.3;
    // so do ten workgroups over a long row of U, 16 x 20224, rank 40: 14.9 -> 16.4).  Two ranks gain 0.1 to 0.5 more, or lose.
    const bool spread = r % 4 == 0 && !in_place && M * (r / 4) <= 256 && (K <= 8192 || r <= 16);
    const int per = spread || r == 4 ? 4 : 8;
    const dim3 grid((unsigned)M, (unsigned)(r > 0 && !wide_sums ? (r + per - 1) / per : 1));
    // 1024 threads per token for a handful of tokens, and for rows with a producer too long for 256 threads' registers
    const bool wide = (M <= 64 && K >= 2048) || (kind != 0 && K > 8 * kRegChunks * 256);
#define ZQ_QUANT_N(RP, NT, KIND) \
    hipLaunchKernelGGL((k_quantize_act<RP, NT, KIND>), grid, dim3(NT), 0, s, X, K, ldx, Xq, sx, U, r, T, pr)
#define ZQ_QUANT_K(RP, NT)                        \
    do {                                          \
        switch (kind) {                           \
        case 1: ZQ_QUANT_N(RP, NT, 1); break;     \
        case 2: ZQ_QUANT_N(RP, NT, 2); break;     \
        case 3: ZQ_QUANT_N(RP, NT, 3); break;     \
        case 4: ZQ_QUANT_N(RP, NT, 4); break;     \
        default: launch_plain<RP, NT>(grid, s, X, K, ldx, Xq, sx, U, r, T, pr); break; \
        }                                         \
    } while (0)
#define ZQ_QUANT(RP)                    \
    do {                                \
        if (wide) ZQ_QUANT_K(RP, 1024); \
        else ZQ_QUANT_K(RP, 256);       \
    } while (0)
    if (r == 0) ZQ_QUANT(0);
    else if (wide_sums) ZQ_QUANT(16);
    else if (per == 4) ZQ_QUANT(4);
    else ZQ_QUANT(8);
#undef ZQ_QUANT
#undef ZQ_QUANT_K
#undef ZQ_QUANT_N
    return hipGetLastError();
}

}  // namespace zqfp
