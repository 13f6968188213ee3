// LoRC factorisation (paper Section 3: singular value decomposition of the error matrix
// E = W - W^, original minus quantized weight; the two low-rank matrices are made from its r
// leading singular triplets).  Offline step, once per layer.
//
// E is K x N with K, N in the thousands and r around 8 (Appendix A: 8 for LLaMA, 16..56 for OPT),
// so the leading triplets come from a subspace iteration instead of a full decomposition:
//   Y = E Omega (Omega: N x l Gaussian, l = r + 8, supplied by the caller), Y <- orth(Y);
//   q times:  Z = E^T Y, Z <- orth(Z), Y = E Z, Y <- orth(Y);
//   B^T = E^T Y (N x l);  B B^T = P L P^T (l x l symmetric eigenproblem, Jacobi rotations);
//   s_i = sqrt(L_i), left vectors Y P, right vectors B^T P / s;
//   U = (Y P)_r diag(s_r)^(1/2),  V = diag(s_r)^(-1/2) (B^T P)_r^T      (singular values shared evenly).
//
// E is never stored: every pass reads W and the packed codes (2.5 bytes per weight, which also fits the last-level
// cache for ordinary layers, where E in float32 does not) and forms its elements in registers as the operand of a
// float32 matrix instruction -- one FP4 conversion per two weights, one multiply-subtract per weight.  Both passes sum
// in float32; K or N is split over workgroups and the kernel behind adds the partial sums in a fixed order.
// 4096 x 12288, r = 8, two power iterations: 2190 -> 335 us, of which the six passes take 175 (30 and 28 us each, 4.3 TB/s; 64
// and 197 us when they read E), the eigenproblem 63, the orthonormalisations 82 and the first and last kernels 10.
//
// The K x l and N x l matrices ("panels") are kept as [R / 16][lp][16] float32, lp = l rounded up to 16: 64
// consecutive bytes of a column, so that all their readers load 16 bytes per lane.  Rows and columns beyond
// the matrix hold zeros.
//
// The l x l work runs in float64: Gram matrices on the float64 matrix cores, a Cholesky factor with its inverse by
// elimination, redundantly in every workgroup of the kernel that applies it, Jacobi rotations l / 2 at a time.
#include "zqfp_internal.h"

namespace zqfp {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef double v4d __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kLMax = 72;      // r <= 64 plus 8 columns of oversampling
constexpr int kGramParts = 32;  // workgroups of the Gram kernel

// 8 or 4 bfloat16 of a row of W, which may start at any even address
struct __attribute__((packed, aligned(2))) Row8 { u32x4 v; };
struct __attribute__((packed, aligned(2))) Row4 { u32x2 v; };

// CW (8 or 4) weights of a row from column n on, in one load; a window that would pass the end of the row is moved back to end
// with it (N >= 9 here)
template <int CW>
__device__ __forceinline__ void load_row(uint32_t (&w)[CW / 2], const uint16_t* row, int64_t n, int64_t N)
{
    n = n < N - CW ? n : N - CW;
    if constexpr (CW == 8) {
        const u32x4 v = reinterpret_cast<const Row8*>(row + n)->v;
#pragma unroll
        for (int d = 0; d < 4; ++d) w[d] = v[d];
    } else {
        const u32x2 v = reinterpret_cast<const Row4*>(row + n)->v;
        w[0] = v[0];
        w[1] = v[1];
    }
}

// undoes the moving: the first weight is column n's again, zeros follow the last
template <int CW>
__device__ __forceinline__ void realign_row(uint32_t (&w)[CW / 2], int64_t n, int64_t N)
{
    const int64_t d64 = n - (N - CW);
    const int d = d64 < 0 ? 0 : d64 > CW ? CW : (int)d64;
#pragma unroll
    for (int step = CW / 2; step >= 1; step >>= 1)
        if (d & (2 * step)) {
#pragma unroll
            for (int k = 0; k < CW / 2; ++k) w[k] = k + step < CW / 2 ? w[k + step] : 0u;
        }
    if (d & 1) {
#pragma unroll
        for (int k = 0; k < CW / 2; ++k) w[k] = (w[k] >> 16) | (k + 1 < CW / 2 ? w[k + 1] << 16 : 0u);
    }
}

// 1 / x and 1 / sqrt(x) for positive normal x: the hardware's start and two Newton steps, correct to an ulp or two
__device__ __forceinline__ double recip(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ double recip_sqrt(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    y = fma(fma(-x * y, y, 1.0), 0.5 * y, y);
    return fma(fma(-x * y, y, 1.0), 0.5 * y, y);
}

// Omega [N][l] row-major -> panel
__global__ __launch_bounds__(256) void k_lorc_start(const float* __restrict__ Omega, int64_t N, int64_t Rp, int l, int lp, float* __restrict__ P)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= Rp * lp) return;
    const int64_t n = idx / (16 * lp) * 16 + (idx & 15);
    const int j = (int)(idx / 16 % lp);
    P[idx] = n < N && j < l ? Omega[n * l + j] : 0.0f;
}

// Y = E Z: part[s] = the share of slice s of the columns.  A workgroup owns 32 rows; its four waves take the
// slice's chunks of 64 columns in turn and add up at the end.  Lane (i = l % 16, b = l / 16) loads rows 2i, 2i + 1 of
// columns 16 b ... 16 b + 15 -- whole 128-byte lines per row -- and matrix instruction q sums over column q of the
// four strips.  The codes come as the blob has them (16 bytes: column i, 32 rows) and change places inside the wave
// through LDS: a byte holds rows 2i, 2i + 1.
// Bound by HBM or the last-level cache: 2.5 bytes per weight; the matrix cores need 10 us of a pass over 4096 x 12288
// for l = 16.
template <int NJ>
__global__ __launch_bounds__(256, NJ == 1 ? 4 : 2) void k_lorc_rows(const uint16_t* __restrict__ W, int64_t ldw, const uint8_t* __restrict__ blob,
                                                                    BlobLayout L, const float* __restrict__ Z, float* __restrict__ part)
{
    constexpr int LP = 16 * NJ;
    constexpr int STRIP = 16 * 16 + 16;  // bytes of a strip's codes in LDS; the pad sets the four strips on different banks
    __shared__ __attribute__((aligned(16))) uint8_t s_code[4][4 * STRIP];
    __shared__ __attribute__((aligned(16))) float s_scale[4][64];
    __shared__ __attribute__((aligned(16))) float s_sum[4][32 * LP];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, b = lane >> 4;
    const int64_t kb = blockIdx.x, kt = kb >> 2;
    const int64_t nch = (L.N + 63) / 64;
    const int64_t c0 = nch * blockIdx.y / gridDim.y, c1 = nch * (blockIdx.y + 1) / gridDim.y;
    const uint32_t* exps = reinterpret_cast<const uint32_t*>(blob + L.off_exps);
    const float* colscale = reinterpret_cast<const float*>(blob + L.off_colscale);
    const int64_t sg = kb * 32 / L.Gs;  // a stored group is at least 32 rows
    const uint16_t* row = W + (kb * 32 + 2 * i) * ldw;

    struct Chunk {
        uint32_t w[2][2][4];
        u32x4 code;
        uint32_t e;
        float cs;
    };
    auto load = [&](Chunk& c, int64_t ch) __attribute__((always_inline)) {
        if (ch >= c1) ch = c1 - 1;  // past the end: the last one again, unused
        const int64_t n = 64 * ch + 16 * b;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int g = 0; g < 2; ++g) load_row<8>(c.w[h][g], row + h * ldw, n + 8 * g, L.N);
        const int64_t strip = 4 * ch + b < L.nstrips ? 4 * ch + b : L.nstrips - 1;
        c.code = *reinterpret_cast<const u32x4*>(blob + L.off_codes + ((size_t)(strip * L.nkt + kt) * 64 + (kb & 3) * 16 + i) * 16);
        c.e = exps[(size_t)(strip * L.ngq + (sg >> 2)) * 16 + i];
        c.cs = colscale[strip * 16 + i];
    };
    v4f acc[2][NJ];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) acc[h][jt] = (v4f){0.f, 0.f, 0.f, 0.f};
    uint8_t* lcode = s_code[wave];
    float* lscale = s_scale[wave];
    auto multiply = [&](Chunk& c, int64_t ch) __attribute__((always_inline)) {
        if (64 * ch + 64 > L.N) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < 2; ++g) realign_row<8>(c.w[h][g], 64 * ch + 16 * b + 8 * g, L.N);
        }
        v4f z[NJ][4];
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                z[jt][q] = *reinterpret_cast<const v4f*>(Z + ((4 * ch + b) * LP + 16 * jt + i) * 16 + 4 * q);
        *reinterpret_cast<u32x4*>(lcode + b * STRIP + i * 16) = c.code;
        // both scales of the column in one factor (a power of two times the column scale)
        lscale[lane] = c.cs * __uint_as_float((c.e >> (8 * (int)(sg & 3)) & 0xFFu) << 23);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        uint32_t byte[16];
        v4f m[4];
#pragma unroll
        for (int q = 0; q < 16; ++q) byte[q] = lcode[b * STRIP + q * 16 + i];
#pragma unroll
        for (int q = 0; q < 4; ++q) m[q] = *reinterpret_cast<const v4f*>(lscale + 16 * b + 4 * q);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const v2f v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(byte[q], 1.0f, 0);
            const uint32_t w0 = c.w[0][q >> 3][(q >> 1) & 3], w1 = c.w[1][q >> 3][(q >> 1) & 3];
            const float e0 = fmaf(-v[0], m[q >> 2][q & 3], (q & 1) ? bf16_hi(w0) : bf16_lo(w0));
            const float e1 = fmaf(-v[1], m[q >> 2][q & 3], (q & 1) ? bf16_hi(w1) : bf16_lo(w1));
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) {
                acc[0][jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(e0, z[jt][q >> 2][q & 3], acc[0][jt], 0, 0, 0);
                acc[1][jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(e1, z[jt][q >> 2][q & 3], acc[1][jt], 0, 0, 0);
            }
        }
    };
    if (c0 + wave < c1) {
        Chunk x, y;
        load(x, c0 + wave);
        for (int64_t ch = c0 + wave; ch < c1; ch += 8) {
            load(y, ch + 4);
            multiply(x, ch);
            if (ch + 4 >= c1) break;
            load(x, ch + 8);
            multiply(y, ch + 4);
        }
    }
    // accumulator h, element r of lane (i, b): row 8 b + 2 r + h of the 32, column i
#pragma unroll
    for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float* d = &s_sum[wave][((b >> 1) * LP + 16 * jt + i) * 16 + 8 * (b & 1) + 2 * r];
            d[0] = acc[0][jt][r];
            d[1] = acc[1][jt][r];
        }
    __syncthreads();
    float* out = part + ((int64_t)blockIdx.y * L.K + 32 * kb) * LP;
    for (int idx = tid; idx < 32 * LP; idx += 256) out[idx] = (s_sum[0][idx] + s_sum[1][idx]) + (s_sum[2][idx] + s_sum[3][idx]);
}

// Z = E^T Y: part[s] = the share of slice s of the rows.  A workgroup owns 16 CW columns; its four waves take the slice's
// k-tiles in turn.  Lane (i, b) holds columns CW i ... CW i + CW - 1 of the 32 rows of block b of the k-tile: their codes are
// 16 CW consecutive bytes of the blob, a row of W comes in whole lines, and matrix instruction t of step p sums
// over row p of the four blocks.  CW = 8 up to l = 32, 4 beyond, where the accumulators take the registers.
// The bounds are those of k_lorc_rows.
template <int NJ, int CW>
__global__ __launch_bounds__(256, NJ == 1 ? 3 : 2) void k_lorc_cols(const uint16_t* __restrict__ W, int64_t ldw, const uint8_t* __restrict__ blob,
                                                                    BlobLayout L, int64_t Rp, const float* __restrict__ Y, float* __restrict__ part)
{
    constexpr int LP = 16 * NJ;
    __shared__ __attribute__((aligned(16))) float s_sum[4][256 * CW];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, b = lane >> 4;
    const int64_t n0 = (int64_t)blockIdx.x * 16 * CW, n = n0 + CW * i;
    const bool full = n0 + 16 * CW <= L.N;
    const int64_t kt0 = L.nkt * blockIdx.y / gridDim.y, kt1 = L.nkt * (blockIdx.y + 1) / gridDim.y;
    const int64_t strip = (n >> 4) < L.nstrips ? n >> 4 : L.nstrips - 1;
    const int c0 = (CW * i) & 15;
    const uint8_t* codes = blob + L.off_codes + ((size_t)(strip * L.nkt) * 64 + b * 16 + c0) * 16;
    const uint8_t* exps = blob + L.off_exps + ((size_t)(strip * L.ngq) * 16 + c0) * 4;
    float cs[CW];
#pragma unroll
    for (int t = 0; t < CW; ++t) cs[t] = reinterpret_cast<const float*>(blob + L.off_colscale)[strip * 16 + c0 + t];

    v4f acc[NJ][CW];
#pragma unroll
    for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
        for (int t = 0; t < CW; ++t) acc[jt][t] = (v4f){0.f, 0.f, 0.f, 0.f};
    struct Rows {
        uint32_t w[4][CW / 2];
    };
    u32x4 code[CW];
    float m[CW];
    // rows 4 g ... 4 g + 3 of every block of k-tile kt
    auto load = [&](Rows& x, int64_t kt, int g) __attribute__((always_inline)) {
        if (kt >= kt1) return;
        const uint16_t* row = W + (kt * 128 + 32 * b + 4 * g) * ldw;
#pragma unroll
        for (int p = 0; p < 4; ++p) load_row<CW>(x.w[p], row + p * ldw, n, L.N);
    };
    auto multiply = [&](Rows& x, int64_t kt, int g) __attribute__((always_inline)) {
        if (!full) {
#pragma unroll
            for (int p = 0; p < 4; ++p) realign_row<CW>(x.w[p], n, L.N);
        }
        v4f y[NJ];
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) y[jt] = *reinterpret_cast<const v4f*>(Y + ((8 * kt + 2 * b + (g >> 2)) * LP + 16 * jt + i) * 16 + 4 * (g & 3));
        auto pair = [&](const v2f (&v)[CW], int p) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int t = 0; t < CW; ++t) {
                    const uint32_t w = x.w[p + h][t >> 1];
                    const float e = fmaf(-v[t][h], m[t], (t & 1) ? bf16_hi(w) : bf16_lo(w));
#pragma unroll
                    for (int jt = 0; jt < NJ; ++jt)
                        acc[jt][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(e, y[jt][p + h], acc[jt][t], 0, 0, 0);
                }
        };
        v2f v[CW];
#define ZQ_PAIR(B)                                                                                                                \
    _Pragma("unroll") for (int t = 0; t < CW; ++t) v[t] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(code[t][g >> 1], 1.0f, B); \
    pair(v, 2 * (B & 1))
        if (g & 1) {
            ZQ_PAIR(2);
            ZQ_PAIR(3);
        } else {
            ZQ_PAIR(0);
            ZQ_PAIR(1);
        }
#undef ZQ_PAIR
    };
    Rows x, y;
    load(x, kt0 + wave, 0);
    for (int64_t kt = kt0 + wave; kt < kt1; kt += 4) {
        const int64_t sg = (kt * 128 + 32 * b) / L.Gs;
        const uint32_t* eq = reinterpret_cast<const uint32_t*>(exps + (size_t)(sg >> 2) * 64);
#pragma unroll
        for (int t = 0; t < CW; ++t) {
            code[t] = *reinterpret_cast<const u32x4*>(codes + (size_t)kt * 1024 + 16 * t);
            m[t] = cs[t] * __uint_as_float((eq[t] >> (8 * (int)(sg & 3)) & 0xFFu) << 23);
        }
#pragma unroll
        for (int g = 0; g < 8; g += 2) {
            load(y, kt, g + 1);
            multiply(x, kt, g);
            if (g < 6) load(x, kt, g + 2);
            else load(x, kt + 4, 0);
            multiply(y, kt, g + 1);
        }
    }
    // accumulator t, element r of lane (i, b): column 4 CW b + CW r + t of the workgroup's, column i of Y
    float* out = part + (int64_t)blockIdx.y * Rp * LP;
#pragma unroll
    for (int jt = 0; jt < NJ; ++jt) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < CW; ++t) {
                const int c = 4 * CW * b + CW * r + t;
                s_sum[wave][(c >> 4) * 256 + i * 16 + (c & 15)] = acc[jt][t][r];
            }
        __syncthreads();
        for (int idx = tid; idx < 256 * CW; idx += 256) {
            const int64_t blk = (n0 >> 4) + (idx >> 8), nn = 16 * blk + (idx & 15);
            const float s = (s_sum[0][idx] + s_sum[1][idx]) + (s_sum[2][idx] + s_sum[3][idx]);
            if (16 * blk < Rp) out[(blk * LP + 16 * jt) * 16 + (idx & 255)] = nn < L.N ? s : 0.0f;
        }
        __syncthreads();
    }
}

// A = the sum of a pass's partial panels (in slice order), and partial Gram matrices of A in float64: workgroup w's share
// goes to gram[w] ([lp][lp]).  A wave takes a block of 16 rows; a lane's four rows of a column feed both operands of the
// matrix instruction.  A single slice may be A itself.
template <int NJ>
__global__ __launch_bounds__(512) void k_lorc_gram(const float* part, int slices, int64_t blocks, float* A, double* __restrict__ gram)
{
    constexpr int LP = 16 * NJ;
    __shared__ double s_tile[8][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, b = lane >> 4;
    v4d g[NJ][NJ];
#pragma unroll
    for (int p = 0; p < NJ; ++p)
#pragma unroll
        for (int q = p; q < NJ; ++q) g[p][q] = (v4d){0.0, 0.0, 0.0, 0.0};
    for (int64_t blk = (int64_t)blockIdx.x * 8 + wave; blk < blocks; blk += 8 * (int64_t)gridDim.x) {
        v4f a[NJ];
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) {
            const int64_t at = (blk * LP + 16 * jt + i) * 16 + 4 * b;
            v4f t = *reinterpret_cast<const v4f*>(part + at);
#pragma unroll 8
            for (int s = 1; s < slices; ++s) t += *reinterpret_cast<const v4f*>(part + s * blocks * 16 * LP + at);
            a[jt] = t;
            *reinterpret_cast<v4f*>(A + at) = t;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int p = 0; p < NJ; ++p)
#pragma unroll
                for (int q = p; q < NJ; ++q)
                    g[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[p][r], (double)a[q][r], g[p][q], 0, 0, 0);
    }
    double* out = gram + (int64_t)blockIdx.x * LP * LP;
#pragma unroll
    for (int p = 0; p < NJ; ++p)
#pragma unroll
        for (int q = p; q < NJ; ++q) {
#pragma unroll
            for (int r = 0; r < 4; ++r) s_tile[wave][(b + 4 * r) * 16 + i] = g[p][q][r];  // element r: row b + 4 r, column i
            __syncthreads();
            if (tid < 256) {
                double t = 0.0;
#pragma unroll
                for (int w = 0; w < 8; ++w) t += s_tile[w][tid];
                out[(16 * p + (tid >> 4)) * LP + 16 * q + (tid & 15)] = t;
                out[(16 * q + (tid & 15)) * LP + 16 * p + (tid >> 4)] = t;
            }
            __syncthreads();
        }
}

// A <- A C^-T with C C^T = the summed Gram matrix (Cholesky).  Every workgroup eliminates the matrix and, beside it, the
// identity, which leaves C^-1; thread t holds elements t, t + 256, ... of both in registers and a step costs one barrier.
// Then a wave takes blocks of 16 rows through the float64 matrix cores.
// A column that depends on the ones before it (E of lower rank than l, or singular values that fall by 2^-22 and more within l
// columns) has a pivot of nothing but rounding: what float32 left of the column, (2^-24)^2 of its squared norm, and
// l 2^-53 from the sums.  Dividing by such a pivot, however it is bounded from below, blows up the later rows step by step
// until they overflow, so a column with a pivot below 2^-44 of its squared norm is dropped: zeros, here and in all that follows
// from it.  What it could add lies below 2^-22 of what is kept, the factors' binary16 is 2^-11.
template <int NJ>
__global__ __launch_bounds__(256) void k_lorc_orth(float* __restrict__ A, int64_t blocks, int l, const double* __restrict__ gram, int nparts)
{
    constexpr int LP = 16 * NJ, NE = NJ * NJ, LDT = LP + 2;  // the pad sets 16 rows on different banks
    __shared__ double s_t[LP * LDT];   // C^-1, row by row as the elimination finishes them
    __shared__ double s_col[2][LP], s_d[LP], s_diag[LP];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, b = lane >> 4;
    double g[NE], w[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int idx = tid + 256 * e, i = idx / LP, k = idx % LP;
        double t = 0.0;
#pragma unroll 16
        for (int p = 0; p < nparts; ++p) t += gram[(int64_t)p * LP * LP + idx];
        g[e] = t;
        w[e] = i == k ? 1.0 : 0.0;
        if (i == k) s_diag[i] = t;
    }
    for (int idx = tid; idx < LP * LDT; idx += 256) s_t[idx] = 0.0;
    __syncthreads();
    for (int j = 0; j < l; ++j) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int idx = tid + 256 * e, i = idx / LP, k = idx % LP;
            if (k == j) s_col[j & 1][i] = g[e];
            if (i == j) s_t[j * LDT + k] = w[e];
        }
        __syncthreads();
        const double d = s_col[j & 1][j];
        const bool drop = d <= 0x1p-44 * s_diag[j];  // false for NaN, which goes on to the results
        const double inv = drop ? 0.0 : recip(d);
        if (tid == 0) s_d[j] = drop ? 0.0 : recip_sqrt(d);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int idx = tid + 256 * e, i = idx / LP, k = idx % LP;
            if (i > j && i < l && !drop) {
                const double f = s_col[j & 1][i] * inv;
                g[e] -= f * s_col[j & 1][k];
                w[e] -= f * s_t[j * LDT + k];
            }
        }
    }
    __syncthreads();
    for (int idx = tid; idx < l * LP; idx += 256) s_t[idx / LP * LDT + idx % LP] *= s_d[idx / LP];
    __syncthreads();
    for (int64_t blk = (int64_t)blockIdx.x * 4 + wave; blk < blocks; blk += 4 * (int64_t)gridDim.x) {
        float* a = A + blk * LP * 16;
#pragma unroll
        for (int jt = NJ - 1; jt >= 0; --jt) {  // columns from the last: column j needs those up to j as they were
            v4d x = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int it = 0; it <= jt; ++it)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    x = __builtin_amdgcn_mfma_f64_16x16x4f64(s_t[(16 * jt + i16) * LDT + 16 * it + 4 * q + b],
                                                             (double)a[(16 * it + 4 * q + b) * 16 + i16], x, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) a[(16 * jt + b + 4 * r) * 16 + i16] = (float)x[r];
        }
    }
}

// Pair `a` (a < mm / 2, mm = l made even) of step T = sweep * l + tau of the Jacobi rotations.  The rotations are those of the
// row-cyclic order (0,1), (0,2), ... (1,2), ..., which also settles the signs of the vectors, but every step takes all
// pairs with p + q = T mod l: they are disjoint, each comes behind all earlier ones that share an index with it, and the next
// sweep (p + q = T - l) follows into the places that the last (p + q = T) leaves.  False: nothing to rotate -- indices that
// are their own partners, taken together or with the row of zeros that makes l even; before the first sweep, the others too.
__device__ __forceinline__ bool jacobi_pair(int a, int tau, int l, int half, bool first, int& p, int& q)
{
    const int c1 = (tau + 1) / 2, c2 = (tau + l + 1) / 2 - tau - 1;
    if (a < c1) {
        p = a;
        q = tau - a;
        return true;
    }
    if (a < c1 + c2) {
        p = tau + 1 + a - c1;
        q = tau + l - p;
        return !first;
    }
    p = (tau & 1) ? (tau + l) / 2 : tau / 2;
    q = (l & 1) ? l : p + half;
    return false;
}

// the rotation that annihilates apq: t = sgn(theta) / (|theta| + sqrt(theta^2 + 1)), theta = d / (2 apq), d = aqq - app
__device__ __forceinline__ void jacobi_rotation(bool live, double apq, double d, double& c, double& s)
{
    const double y = fma(d, d, 4.0 * apq * apq);
    const double t = copysign(2.0 * fabs(apq) * recip(fabs(d) + y * recip_sqrt(y)), d == 0.0 ? 1.0 : d * apq);
    live = live && apq != 0.0 && y >= 1e-300;
    c = live ? recip_sqrt(fma(t, t, 1.0)) : 1.0;
    s = live ? t * c : 0.0;
}

// Eigen-decomposition of M = Zb^T Zb (summed from its partial Gram matrices) by cyclic Jacobi rotations,
// descending order, and the two l x r coefficient matrices of the factors:
// CU = P_r diag(s_r)^(1/2),  CV = P_r diag(s_r)^(-1/2).  One workgroup: a serial chain of l steps per sweep and about seven
// sweeps.  SMALL (l <= 16): after the sums a single wave goes on alone, a 2 x 2 block per lane, and every lane finds
// the rotation of its columns by itself; what counts there is the number of instructions of the one wave, 1000 cycles a step (63 us; 622 us
// with one rotation at a time).  Otherwise a thread per rotation leaves it in LDS for the others.
template <bool SMALL>
__global__ __launch_bounds__(256) void k_lorc_eig(const double* __restrict__ gram, int nparts, int l, int lp, int r,
                                                  double* __restrict__ CU, double* __restrict__ CV, float* __restrict__ sigma)
{
    constexpr int MAX = SMALL ? 16 : kLMax, NT = SMALL ? 64 : 256, SIDE = SMALL ? 8 : 16;
    __shared__ double M[MAX * (MAX + 1)], P[MAX * (MAX + 1)];
    __shared__ double s_c[MAX / 2], s_s[MAX / 2], s_red[2][4];
    __shared__ int s_p[MAX / 2], s_q[MAX / 2], s_order[MAX], s_pair[SMALL ? MAX : 1][MAX / 2];
    const int tid = threadIdx.x;
    const int mm = (l + 1) & ~1, half = mm / 2, ld = mm + 1;
    for (int idx = tid; idx < mm * mm; idx += 256) {
        const int i = idx / mm, j = idx % mm;
        double t = 0.0;
        if (i < l && j < l) {
#pragma unroll 16
            for (int p = 0; p < nparts; ++p) t += gram[(int64_t)p * lp * lp + i * lp + j];
        }
        M[i * ld + j] = t;
        P[i * ld + j] = i == j ? 1.0 : 0.0;
    }
    if constexpr (SMALL)
        for (int idx = tid; idx < l * half; idx += 256) {  // the pairs of every step; bits 16, 17: rotated, also in the first sweep
            int p, q;
            const int tau = idx / half, a = idx % half;
            const int later = jacobi_pair(a, tau, l, half, false, p, q), first = jacobi_pair(a, tau, l, half, true, p, q);
            s_pair[tau][a] = p | q << 8 | later << 16 | first << 17;
        }
    __syncthreads();
    if (tid >= NT) return;
    // a barrier for those that go on: none that waves which have left would have to reach
    auto sync = []() __attribute__((always_inline)) {
        if constexpr (SMALL) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            __syncthreads();
        }
    };
    const int ty = tid / SIDE, tx = tid % SIDE;  // threads as a square
    for (int sweep = 0; sweep < 31; ++sweep) {
        double off = 0.0, diag = 0.0;
        for (int i = ty; i < mm; i += SIDE)
            for (int j = tx; j < mm; j += SIDE) {
                const double v = M[i * ld + j] * M[i * ld + j];
                if (i == j) diag += v;
                else off += v;
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            off += __shfl_xor(off, o);
            diag += __shfl_xor(diag, o);
        }
        if ((tid & 63) == 0) {
            s_red[0][tid >> 6] = off;
            s_red[1][tid >> 6] = diag;
        }
        sync();
        off = diag = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) {
            off += s_red[0][w];
            diag += s_red[1][w];
        }
        if (off <= 1e-30 * diag) break;  // the same for every thread: read from LDS behind a barrier
        for (int tau = 0; tau < l; ++tau) {
            // rows of pair (p, q), columns of pair (u, v); `zero`: the same pair, annihilated
            auto rotate_block = [&](int p, int q, int u, int v, double ca, double sa, double cb, double sb, bool zero) __attribute__((always_inline)) {
                const double pu = M[p * ld + u], pv = M[p * ld + v], qu = M[q * ld + u], qv = M[q * ld + v];
                const double pu1 = cb * pu - sb * pv, pv1 = sb * pu + cb * pv;
                const double qu1 = cb * qu - sb * qv, qv1 = sb * qu + cb * qv;
                M[p * ld + u] = ca * pu1 - sa * qu1;
                M[q * ld + v] = sa * pv1 + ca * qv1;
                M[p * ld + v] = zero ? 0.0 : ca * pv1 - sa * qv1;
                M[q * ld + u] = zero ? 0.0 : sa * pu1 + ca * qu1;
            };
            auto rotate_vectors = [&](int u, int v, double cb, double sb) __attribute__((always_inline)) {
                for (int row = ty; row < mm; row += SIDE) {
                    const double x = P[row * ld + u], y = P[row * ld + v];
                    P[row * ld + u] = cb * x - sb * y;
                    P[row * ld + v] = sb * x + cb * y;
                }
            };
            if constexpr (SMALL) {
                if (tx < half) {  // all eight ty: the vectors have mm rows, of which ty < half alone would leave some out
                    const int pb = s_pair[tau][tx], u = pb & 255, v = pb >> 8 & 255;
                    double cb, sb;
                    jacobi_rotation(pb >> (sweep == 0 ? 17 : 16) & 1, M[u * ld + v], M[v * ld + v] - M[u * ld + u], cb, sb);
                    const double ca = __shfl(cb, ty), sa = __shfl(sb, ty);  // lane ty has tx = ty; unused where ty >= half
                    if (ty < half) {
                        const int pa = s_pair[tau][ty];
                        rotate_block(pa & 255, pa >> 8 & 255, u, v, ca, sa, cb, sb, tx == ty && sb != 0.0);
                    }
                    rotate_vectors(u, v, cb, sb);
                }
            } else {
                if (tid < half) {
                    int p, q;
                    const bool live = jacobi_pair(tid, tau, l, half, sweep == 0, p, q);
                    jacobi_rotation(live, M[p * ld + q], M[q * ld + q] - M[p * ld + p], s_c[tid], s_s[tid]);
                    s_p[tid] = p;
                    s_q[tid] = q;
                }
                sync();
                for (int b = tx; b < half; b += SIDE) {
                    for (int a = ty; a < half; a += SIDE)
                        rotate_block(s_p[a], s_q[a], s_p[b], s_q[b], s_c[a], s_s[a], s_c[b], s_s[b], a == b && s_s[b] != 0.0);
                    rotate_vectors(s_p[b], s_q[b], s_c[b], s_s[b]);
                }
            }
            sync();
        }
    }
    if (tid < l) {  // place of the eigenvalue, largest first
        int place = 0;
        const double d = M[tid * ld + tid];
        for (int j = 0; j < l; ++j) {
            const double o = M[j * ld + j];
            place += o > d || (o == d && j < tid) ? 1 : 0;
        }
        s_order[place] = tid;
    }
    sync();
    for (int idx = tid; idx < l * r; idx += NT) {
        const int j = idx / r, i = idx % r;
        const int col = s_order[i];
        const double sv = sqrt(fmax(M[col * ld + col], 0.0));
        const double root = sqrt(sv);
        CU[idx] = P[j * ld + col] * root;
        CV[idx] = root > 0.0 ? P[j * ld + col] / root : 0.0;
        if (j == 0) sigma[i] = (float)sv;
    }
}

// U[k][i] = sum_j Y[k][j] CU[j][i] and V[i][n] = sum_j Z[n][j] CV[j][i], as binary16
__global__ __launch_bounds__(256) void k_lorc_emit(const float* __restrict__ Y, int64_t K, const double* __restrict__ CU, uint16_t* __restrict__ U,
                                                   const float* __restrict__ Z, int64_t N, const double* __restrict__ CV, uint16_t* __restrict__ V,
                                                   int l, int lp, int r)
{
    int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool left = idx < K * r;
    if (!left) idx -= K * r;
    if (!left && idx >= N * r) return;
    const int64_t row = left ? idx / r : idx % N;
    const int i = (int)(left ? idx % r : idx / N);
    const float* a = (left ? Y : Z) + (row >> 4) * lp * 16 + (row & 15);
    const double* c = (left ? CU : CV) + i;
    double t = 0.0;
#pragma unroll 8
    for (int j = 0; j < l; ++j) t += (double)a[j * 16] * c[j * r];
    (left ? U : V)[idx] = __builtin_bit_cast(uint16_t, (_Float16)(float)t);
}

// Column and row slices: enough workgroups for four (rows pass) or three (columns pass) on each of 256 compute units, which is
// what their registers allow at l = 16, as long as every wave keeps a chunk or k-tile of its own.
int64_t rows_slices(int64_t K, int64_t N)
{
    const int64_t most = ((N + 63) / 64 + 3) / 4, want = 1024 / ((K + 31) / 32);
    return want < 1 ? 1 : want < most ? want : most;
}
int64_t cols_width(int nj) { return nj <= 2 ? 128 : 64; }
int64_t cols_slices(int64_t K, int64_t N, int nj)
{
    const int64_t w = cols_width(nj), most = (K / 128 + 3) / 4, want = 768 / ((N + w - 1) / w);
    return want < 1 ? 1 : want < most ? want : most;
}

struct Workspace {
    int nj, lp;
    int64_t Rp;            // N rounded up to the 64 columns of a chunk
    int64_t srows, scols;  // slices of the two passes
    size_t part, ya, za, cu, gram;
    Workspace(int64_t K, int64_t N, int r)
    {
        const int l = r + 8;
        nj = (l + 15) / 16;
        lp = 16 * nj;
        Rp = (N + 63) / 64 * 64;
        srows = rows_slices(K, N);
        scols = cols_slices(K, N, nj);
        auto up = [](size_t b) { return (b + 255) / 256 * 256; };
        const size_t pr = (size_t)srows * K * lp * 4, pc = (size_t)scols * Rp * lp * 4;
        part = up(pr > pc ? pr : pc);
        ya = up((size_t)K * lp * 4);
        za = up((size_t)Rp * lp * 4);
        cu = up((size_t)l * r * 8);
        gram = up((size_t)kGramParts * lp * lp * 8);
    }
    size_t total() const { return part + ya + za + 2 * cu + gram; }
};

template <int NJ>
hipError_t factorize(const uint16_t* W, int64_t ldw, const uint8_t* blob, const BlobLayout& L, int r, const float* Omega,
                     int power_iters, uint16_t* U, uint16_t* V, float* sigma, void* workspace, hipStream_t s)
{
    constexpr int LP = 16 * NJ, CW = NJ <= 2 ? 8 : 4;
    const int64_t K = L.K, N = L.N;
    const int l = r + 8;
    const Workspace ws(K, N, r);
    uint8_t* p = static_cast<uint8_t*>(workspace);
    float* part = reinterpret_cast<float*>(p);
    float* Ya = reinterpret_cast<float*>(p += ws.part);
    float* Za = reinterpret_cast<float*>(p += ws.ya);
    double* CU = reinterpret_cast<double*>(p += ws.za);
    double* CV = reinterpret_cast<double*>(p += ws.cu);
    double* gram = reinterpret_cast<double*>(p += ws.cu);
    const int64_t yb = K / 16, zb = ws.Rp / 16;

    auto rows = [&]() {
        hipLaunchKernelGGL(k_lorc_rows<NJ>, dim3((unsigned)(K / 32), (unsigned)ws.srows), dim3(256), 0, s, W, ldw, blob, L, Za, part);
    };
    auto cols = [&]() {
        hipLaunchKernelGGL((k_lorc_cols<NJ, CW>), dim3((unsigned)((N + 16 * CW - 1) / (16 * CW)), (unsigned)ws.scols), dim3(256), 0, s, W, ldw, blob, L,
                           ws.Rp, Ya, part);
    };
    auto parts = [&](int64_t blocks) { return (int)((blocks + 7) / 8 < kGramParts ? (blocks + 7) / 8 : kGramParts); };
    auto sum = [&](const float* from, int64_t slices, int64_t blocks, float* A) {
        hipLaunchKernelGGL(k_lorc_gram<NJ>, dim3(parts(blocks)), dim3(512), 0, s, from, (int)slices, blocks, A, gram);
    };
    auto orth = [&](float* A, int64_t blocks) {
        const int64_t wgs = (blocks + 3) / 4 < 256 ? (blocks + 3) / 4 : 256;
        hipLaunchKernelGGL(k_lorc_orth<NJ>, dim3((unsigned)wgs), dim3(256), 0, s, A, blocks, l, gram, parts(blocks));
    };

    hipLaunchKernelGGL(k_lorc_start, dim3((unsigned)((ws.Rp * LP + 255) / 256)), dim3(256), 0, s, Omega, N, ws.Rp, l, LP, Za);
    rows();
    sum(part, ws.srows, yb, Ya);
    orth(Ya, yb);
    for (int it = 0; it < power_iters; ++it) {
        cols();
        sum(part, ws.scols, zb, Za);
        orth(Za, zb);
        rows();
        sum(part, ws.srows, yb, Ya);
        orth(Ya, yb);
    }
    // Between passes one Cholesky QR is enough (six in place of ten at two power iterations): it keeps the span, which is all the
    // next pass uses, and leaves the basis well conditioned.  The last basis, whose orthonormality the singular values rest on, goes
    // through a second, which removes what rounding left of the first.  Against two everywhere: the same singular values and
    // residuals on 256 combinations of spectrum, rank and iteration count, wherever two passes gave finite ones.
    sum(Ya, 1, yb, Ya);
    orth(Ya, yb);
    cols();  // B^T = E^T Y
    sum(part, ws.scols, zb, Za);
    hipLaunchKernelGGL(k_lorc_eig<NJ == 1>, dim3(1), dim3(256), 0, s, gram, parts(zb), l, LP, r, CU, CV, sigma);
    hipLaunchKernelGGL(k_lorc_emit, dim3((unsigned)(((K + N) * r + 255) / 256)), dim3(256), 0, s, Ya, K, CU, U, Za, N, CV, V, l, LP, r);
    return hipGetLastError();
}

}  // namespace

// the slices' partial panels, the two panels [K] and [N], CU and CV [l][r] float64, partial Gram matrices
size_t lorc_workspace_bytes(int64_t K, int64_t N, int r) { return Workspace(K, N, r).total(); }

hipError_t launch_lorc_factorize(const uint16_t* W, int64_t ldw, const uint8_t* blob, const BlobLayout& L, int r,
                                 const float* Omega, int power_iters, uint16_t* U, uint16_t* V, float* sigma,
                                 void* workspace, hipStream_t s)
{
    switch ((r + 8 + 15) / 16) {
    case 1: return factorize<1>(W, ldw, blob, L, r, Omega, power_iters, U, V, sigma, workspace, s);
    case 2: return factorize<2>(W, ldw, blob, L, r, Omega, power_iters, U, V, sigma, workspace, s);
    case 3: return factorize<3>(W, ldw, blob, L, r, Omega, power_iters, U, V, sigma, workspace, s);
    case 4: return factorize<4>(W, ldw, blob, L, r, Omega, power_iters, U, V, sigma, workspace, s);
    default: return factorize<5>(W, ldw, blob, L, r, Omega, power_iters, U, V, sigma, workspace, s);
    }
}

}  // namespace zqfp
