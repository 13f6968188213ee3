// Group-wise FP4 (E2M1) weight quantizer with power-of-two group scales
// (paper Section 3: fine-grained quantization; "Casting the FP4 to FP8",
// methods M1 and M2) and its inverse view.
//
// A workgroup takes 64 output channels (one 128-byte line of a row of W) and one "unit" of input channels: the
// least stretch of whole groups and whole k-tiles, 128 rows for groups of 32, 64 and 128.  Thread (c, q) holds the
// 32 weights of column c and 32-block q in registers -- exactly the 16 bytes of codes that lane 16 (q % 4) + c % 16
// of a fragment owns, so that no transpose is needed and a wave stores four runs of 256 bytes -- and the blocks of a
// group agree on its absmax in LDS.  Bound by HBM (2 B read, 0.5 B written per weight).  With W in its natural
// order the loads are 2 bytes per lane, 128 bytes per instruction and 32 of them in flight per thread, which also
// serves rows of any alignment; the vector work is about four operations per weight because the code and the division
// by the power-of-two scale are one hardware conversion per pair (v_cvt_scalef32_pk_fp4: round to nearest, ties to the even
// code, saturating at 6, sign kept -- compared on all 2^32 binary32 values, and on every bfloat16 value under every scale).  4096 x 12288, G = 128,
// M1: 249 -> 25 us (a workgroup per 16 columns before: 32-byte pieces of lines that four L2s fetched, the whole K in
// sequence, a compare chain per code).
#include "zqfp_internal.h"

namespace zqfp {
namespace {

constexpr int kThreads = 256;
constexpr int kCols = 64;  // output channels per workgroup

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// largest group magnitude a power-of-two scale maps onto: 6 (E2M1) or 448 (E4M3)
__device__ inline float format_max(const BlobLayout& L) { return L.wbits == 8 ? 448.0f : 6.0f; }

// M2's column scale, absmax / format maximum (1 for an all-zero column, 0 for padding columns), into the blob; where one
// group spans a column, its exponent byte too.
// One workgroup per 64 columns walks the whole K: 128 bytes of a row per wave, eight rows in flight per wave.
__global__ __launch_bounds__(1024) void k_column_scale(const uint16_t* __restrict__ W, int64_t ldw, BlobLayout L, int mode,
                                                       uint8_t* __restrict__ blob)
{
    __shared__ float s_max[16][kCols];
    const int c = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t n = (int64_t)blockIdx.x * kCols + c;
    const uint16_t* w = W + (n < L.N ? n : L.N - 1);
    float m = 0.0f;
    for (int64_t k = wave; k < L.K; k += 128) {  // K is a multiple of 128: eight rows per wave and step
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = bf16_bits_to_f32(w[(k + 16 * i) * ldw]);
#pragma unroll
        for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(v[i]));
    }
    s_max[wave][c] = m;
    __syncthreads();
    if (wave == 0 && n < L.Np) {
#pragma unroll
        for (int i = 1; i < 16; ++i) m = fmaxf(m, s_max[i][c]);
        reinterpret_cast<float*>(blob + L.off_colscale)[n] = n >= L.N ? 0.0f : mode != 1 && m != 0.0f ? m / format_max(L) : 1.0f;  // IEEE binary32 division
        if (L.G == L.K) {  // one stored group, one dword per column
            const int e = mode != 1 ? -m2_shift(m, m) : L.wbits == 8 ? m1_exponent_e4m3(m) : m1_exponent(m);
            reinterpret_cast<uint32_t*>(blob + L.off_exps)[n] = 0x7F7F7F00u | (uint32_t)(n < L.N ? e + 127 : 127);
        }
    }
}

// The codes of one 32-block: x holds 32 bfloat16 weights (pairs of consecutive k), e the group's exponent.
template <int WBITS>
__device__ inline void encode_block(const uint32_t (&x)[16], int mode, int e, float cs, uint8_t* __restrict__ frag, int q, int col)
{
    const float scale = ldexpf(1.0f, e);
    if constexpr (WBITS == 4) {
        u32x4 o;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t word = 0;
            if (mode == 1) {  // exact division by 2^e
                word = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(word, __builtin_bit_cast(bf16x2, x[4 * d]), scale, 0);
                word = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(word, __builtin_bit_cast(bf16x2, x[4 * d + 1]), scale, 1);
                word = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(word, __builtin_bit_cast(bf16x2, x[4 * d + 2]), scale, 2);
                word = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(word, __builtin_bit_cast(bf16x2, x[4 * d + 3]), scale, 3);
            } else {  // IEEE division by the column scale, then the exact shift
                word = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, bf16_lo(x[4 * d]) / cs, bf16_hi(x[4 * d]) / cs, scale, 0);
                word = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, bf16_lo(x[4 * d + 1]) / cs, bf16_hi(x[4 * d + 1]) / cs, scale, 1);
                word = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, bf16_lo(x[4 * d + 2]) / cs, bf16_hi(x[4 * d + 2]) / cs, scale, 2);
                word = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, bf16_lo(x[4 * d + 3]) / cs, bf16_hi(x[4 * d + 3]) / cs, scale, 3);
            }
            o[d] = word;
        }
        *reinterpret_cast<u32x4*>(frag + (q * 16 + col) * 16) = o;
    } else {
        // E4M3 codes: same encoder as the activations' (clamp to +-448, then the hardware conversion, round to
        // nearest even, sign kept); block q is two runs of 16 bytes of half q / 2 of the fragment
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 o;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                float y[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t p = x[8 * h + 2 * d + (i >> 1)];
                    const float w = (i & 1) ? bf16_hi(p) : bf16_lo(p);
                    y[i] = clamp448(ldexpf(mode == 1 ? w : w / cs, -e));
                }
                int pk = __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], 0, false);
                o[d] = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], pk, true);
            }
            *reinterpret_cast<u32x4*>(frag + (q >> 1) * 1024 + (((q & 1) * 2 + h) * 16 + col) * 16) = o;
        }
    }
}

// TILES: k-tiles of a unit, kept in registers between the absmax and the codes (1 or 2); 0: a unit of any length,
// walked four k-tiles at a time by 1024 threads and read a second time for the codes (from L2 where it fits).
// WHOLE: one group spans a column and k_column_scale has written its scale and exponent; the k-tiles are independent.
template <int TILES, int WBITS, bool WHOLE = false>
__global__ __launch_bounds__(TILES == 0 ? 1024 : 256) void k_pack_weight(const uint16_t* __restrict__ W, int64_t ldw, BlobLayout L,
                                                                         int mode, int unit_tiles, uint8_t* __restrict__ blob)
{
    constexpr int PAR = TILES == 0 ? 4 : 1;  // k-tiles worked on at once
    __shared__ uint32_t s_gmax[4][kCols];    // a unit holds one, two or four groups, or one group spans it
    const int tid = threadIdx.x, c = tid & 63, q = (tid >> 6) & 3, par = tid >> 8;
    const int64_t n = (int64_t)blockIdx.x * kCols + c;
    const bool live = n < L.N, in_blob = n < L.Np;
    const uint16_t* wcol = W + (live ? n : L.N - 1);
    const int64_t kt0 = (int64_t)blockIdx.y * unit_tiles;
    float* colscale = reinterpret_cast<float*>(blob + L.off_colscale);
    const int blocks_per_group = L.G / 32;

    auto load_block = [&](int64_t kt, uint32_t (&x)[16]) __attribute__((always_inline)) {
        const uint16_t* p = wcol + (kt * 128 + 32 * q) * ldw;
        uint16_t v[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = p[i * ldw];
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = live ? (uint32_t)v[2 * i] | ((uint32_t)v[2 * i + 1] << 16) : 0u;  // padding columns: +0
    };
    auto group_max = [&](int t, const uint32_t (&x)[16]) __attribute__((always_inline)) {
        float m = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) m = fmaxf(m, fmaxf(fabsf(bf16_lo(x[i])), fabsf(bf16_hi(x[i]))));
        // a maximum of non-negative floats is the maximum of their bit patterns, in any order
        atomicMax(&s_gmax[(t * 4 + q) / blocks_per_group][c], __float_as_uint(m));
    };

    if constexpr (!WHOLE) {
        s_gmax[tid >> 6 & 3][c] = 0u;
        __syncthreads();
    }
    uint32_t x[TILES == 0 ? 1 : TILES][16];
    if constexpr (WHOLE) {
        load_block(kt0, x[0]);
    } else if constexpr (TILES == 0) {
        for (int t = par; t < unit_tiles; t += PAR) {
            load_block(kt0 + t, x[0]);
            group_max(t, x[0]);
        }
    } else {
#pragma unroll
        for (int t = 0; t < TILES; ++t) load_block(kt0 + t, x[t]);
#pragma unroll
        for (int t = 0; t < TILES; ++t) group_max(t, x[t]);
    }
    float cs = 1.0f, cmax = 0.0f;
    if (mode != 1 && live) {  // padding columns: +0 over 1
        cs = colscale[n];
        // the column's absmax is a bfloat16 value and cs is it over the format maximum, correctly rounded: the
        // product is within 2^-23 of it, relatively (2^-9 where cs is subnormal: an absmax below 2^-117, with 448), and
        // rounds back to it (an all-zero column has no use for it)
        cmax = bf16_bits_to_f32(f32_to_bf16_bits(cs * format_max(L)));
    }
    if constexpr (!WHOLE) __syncthreads();
    if (!in_blob) return;  // no barrier below

    auto finish_tile = [&](int t, const uint32_t (&xt)[16]) __attribute__((always_inline)) {
        int e;
        if constexpr (WHOLE) {
            e = (int)(reinterpret_cast<const uint32_t*>(blob + L.off_exps)[n] & 0xFFu) - 127;
        } else {
            const float amax = __uint_as_float(s_gmax[(t * 4 + q) / blocks_per_group][c]);
            e = mode == 1 ? (WBITS == 8 ? m1_exponent_e4m3(amax) : m1_exponent(amax)) : -m2_shift(cmax, amax);
        }
        const int64_t kt = kt0 + t, strip = n >> 4;
        const int col = c & 15;
        encode_block<WBITS>(xt, mode, e, cs, blob + L.off_codes + (size_t)(strip * L.nkt + kt) * (256 * WBITS), q, col);
        if constexpr (WHOLE) return;
        // exponent bytes, [strip][quad][column][4], one per stored group; the last dword is filled up with 127
        const int64_t k = kt * 128 + 32 * q;
        if (k % L.Gs == 0) {
            const int64_t sg = k / L.Gs;
            uint8_t* p = blob + L.off_exps + ((size_t)(strip * L.ngq + (sg >> 2)) * 16 + col) * 4;
            p[sg & 3] = (uint8_t)(live ? e + 127 : 127);
            if (sg == L.ngs - 1)
                for (int b = (int)(sg & 3) + 1; b < 4; ++b) p[b] = 127;
        }
    };
    if constexpr (TILES == 0) {
        for (int t = par; t < unit_tiles; t += PAR) {
            load_block(kt0 + t, x[0]);
            finish_tile(t, x[0]);
        }
    } else {
#pragma unroll
        for (int t = 0; t < TILES; ++t) finish_tile(t, x[t]);
    }
    if (!WHOLE && mode == 1 && blockIdx.y == 0 && tid < kCols) colscale[n] = live ? 1.0f : 0.0f;
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {
        BlobHeader h;
        h.magic = kBlobMagic; h.version = kBlobVersion;
        h.K = L.K; h.N = L.N; h.Np = L.Np;
        h.G = L.G; h.Gs = L.Gs; h.mode = mode; h.ngs = L.ngs; h.ngq = L.ngq; h.wbits = WBITS;
        h.off_codes = L.off_codes; h.off_exps = L.off_exps; h.off_colscale = L.off_colscale; h.total = L.total;
        *reinterpret_cast<BlobHeader*>(blob) = h;
    }
}

__global__ __launch_bounds__(kThreads) void k_unpack(const uint8_t* __restrict__ blob, BlobLayout L,
                                                   uint8_t* __restrict__ codes, uint8_t* __restrict__ exps,
                                                   float* __restrict__ colscale)
{
    const int64_t total = L.K * L.N;
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < total) {
        const int64_t k = i / L.N, n = i % L.N;
        const int64_t strip = n >> 4, kt = k >> 7;
        const int c = (int)(n & 15), kk = (int)(k & 127), lb = kk >> 5, p = kk & 31;
        if (L.wbits == 8) {
            const int half = kk >> 6, lb8 = (kk >> 4) & 3;
            codes[i] = blob[L.off_codes + (size_t)(strip * L.nkt + kt) * 2048 + half * 1024 + (lb8 * 16 + c) * 16 + (kk & 15)];
        } else {
            const uint8_t byte = blob[L.off_codes + ((size_t)(strip * L.nkt + kt) * 64 + (lb * 16 + c)) * 16 + (p >> 1)];
            codes[i] = (p & 1) ? (byte >> 4) : (byte & 15);
        }
    }
    const int64_t ng = L.K / L.G;
    if (i < ng * L.N) {
        const int64_t g = i / L.N, n = i % L.N;
        const int64_t sg = g * L.G / L.Gs;
        exps[i] = blob[L.off_exps + ((size_t)((n >> 4) * L.ngq + (sg >> 2)) * 16 + (n & 15)) * 4 + (sg & 3)];
    }
    if (i < L.N) colscale[i] = reinterpret_cast<const float*>(blob + L.off_colscale)[i];
}

}  // namespace

hipError_t launch_pack_weight(const uint16_t* W, int64_t ldw, const BlobLayout& L, int mode, uint8_t* blob,
                              hipStream_t s)
{
    if (L.nstrips == 0) return hipSuccess;
    // a unit: whole groups and whole k-tiles.  G is a multiple of 32, so it is G or 128 rows where one divides the
    // other and two or four groups otherwise (G = 320: 640 rows).
    const int64_t unit = (int64_t)L.G / gcd_int(L.G, 128) * 128;
    const int tiles = (int)(unit / 128);
    const unsigned gx = (unsigned)((L.Np + kCols - 1) / kCols);
    // One group per column and more than its registers hold: where the absmax takes a launch anyway (M2), or from 1024 rows on, the
    // exponent comes with it and the codes from as many workgroups as there are k-tiles, instead of one workgroup for the
    // whole column twice over (FP8, 1024 columns, M2: 384 rows 10.8 -> 7.0 us, 4096 rows 63.2 -> 16.2; M1, 4096 rows 53.5 -> 16.3;
    // FP4, 512 rows: M1 6.6 in one launch, M2 7.0 in these two).
    const bool whole = tiles > 2 && L.G == L.K && (mode != 1 || tiles >= 8);
    const dim3 grid(gx, (unsigned)(whole ? L.nkt : L.K / unit));
    if (mode != 1 || whole) hipLaunchKernelGGL(k_column_scale, dim3(gx), dim3(1024), 0, s, W, ldw, L, mode, blob);
#define ZQ_PACK(TILES, WB, ...) \
    hipLaunchKernelGGL((k_pack_weight<TILES, WB, ##__VA_ARGS__>), grid, dim3(TILES == 0 ? 1024 : 256), 0, s, W, ldw, L, mode, \
                       whole ? 1 : tiles, blob)
    if (L.wbits == 8) {
        if (whole) ZQ_PACK(1, 8, true); else if (tiles == 1) ZQ_PACK(1, 8); else if (tiles == 2) ZQ_PACK(2, 8); else ZQ_PACK(0, 8);
    } else {
        if (whole) ZQ_PACK(1, 4, true); else if (tiles == 1) ZQ_PACK(1, 4); else if (tiles == 2) ZQ_PACK(2, 4); else ZQ_PACK(0, 4);
    }
#undef ZQ_PACK
    return hipGetLastError();
}

hipError_t launch_unpack(const uint8_t* blob, const BlobLayout& L, uint8_t* codes, uint8_t* exps, float* colscale,
                         hipStream_t s)
{
    int64_t total = L.K * L.N;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_unpack, dim3((unsigned)((total + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, blob, L,
                       codes, exps, colscale);
    return hipGetLastError();
}

}  // namespace zqfp
