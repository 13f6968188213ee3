// W4A8 / W8A8 GEMM for a few dozen tokens (small serving batches, verification of drafts).
//
//   Y[m,n] = (sx[m] c[n]) * sum_k a[m,k] * q[k,n] * 2^e[g(k),n]   (+ T.V, LoRC)
//
// (paper Sections 1 and 3.)  Neither the matrix cores nor HBM bound these sizes but the latency of a workgroup's
// first loads and the number of compute units that get work at all: 64 tokens x 12288 channels are 96 tiles of the
// tiled kernel for 256 compute units.  Here a workgroup takes S strips of 16 channels, S chosen so that the strips
// come out in whole rounds of compute units, and up to 64 tokens; its eight waves split K.  A wave therefore needs
// every activation byte of its k-tiles exactly once, so operands go from memory straight into registers, NB k-tiles
// ahead, with no barrier before the partial tiles meet in LDS at the end (fixed order, no atomics, no second launch).
// What is left at 64 tokens is the 64 * K bytes of activations that every compute unit fetches (4096 x 12288: 5.3 of 14.7 us
// against 16 tokens; 9.4 of 17.5 before a row's line was loaded by eight lanes).
#include <type_traits>

#include "zqfp_internal.h"

namespace zqfp {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;

// MT: blocks of 16 tokens, S: strips of 16 channels, NB: k-tiles in flight per wave, WB: weight bits
template <int MT, int S, int NB, bool EXACT, int WB>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_mid(
    const uint8_t* __restrict__ Xq, const float* __restrict__ sx, int64_t M, const uint8_t* __restrict__ blob, BlobLayout L,
    Lorc lorc, void* __restrict__ Y, int64_t ldy, int out_dtype, int mblocks)
{
    extern __shared__ __attribute__((aligned(16))) float s_part[];  // [S * MT][kWaves][64][4]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, lb = lane >> 4;
    const int nkt = (int)L.nkt;
    // Consecutive workgroup ids sit on consecutive XCDs: each XCD gets a contiguous run of units, so that its L2 merges
    // the parts of a line of Y and serves the strips of one group to all its token blocks.
    const int units = (int)gridDim.x, xcd = (int)blockIdx.x & 7;
    const int unit = xcd * (units >> 3) + min(xcd, units & 7) + ((int)blockIdx.x >> 3);
    const int group = unit / mblocks;
    const int64_t m_base = (int64_t)(unit - group * mblocks) * (16 * MT);
    const int64_t strip0 = (int64_t)group * S;

    const uint8_t* codes = blob + L.off_codes;
    const uint32_t* exq = reinterpret_cast<const uint32_t*>(blob + L.off_exps);

    // A operand: lane (row = lane % 16, lb) needs the bytes k = 16 lb + [0, 16) and 64 + 16 lb + [0, 16) of a k-tile.
    // Loaded like that every lane of an instruction touches a line of its own (16 B a clock and compute unit), so
    // eight lanes load a row's 128 bytes instead and the wave's own slice of LDS turns them round (chunk c of row r at
    // slot c ^ (r % 8), which keeps both sides free of bank conflicts; a wave's LDS operations stay in order).  A row past M
    // repeats row M - 1, a strip past the last one repeats it: neither is stored.
    const uint8_t* xbase = Xq + m_base * L.K;
    uint32_t arow[2 * MT];
#pragma unroll
    for (int j = 0; j < 2 * MT; ++j) arow[j] = (uint32_t)(min((int64_t)(j * 8 + (lane >> 3)), M - 1 - m_base) * L.K) + 16u * (uint32_t)(lane & 7);
    uint8_t* turn = reinterpret_cast<uint8_t*>(s_part) + wave * (MT * 2048);
    uint8_t* turn_w = turn + (lane >> 3) * 128 + ((lane & 7) ^ (lane >> 3)) * 16;
    const uint8_t* turn_r0 = turn + col * 128 + (lb ^ (col & 7)) * 16;
    const uint8_t* turn_r1 = turn + col * 128 + ((lb + 4) ^ (col & 7)) * 16;
    int64_t strip[S];
#pragma unroll
    for (int s = 0; s < S; ++s) strip[s] = min(strip0 + s, L.nstrips - 1);

    u32x4 a[NB][2 * MT], b[NB][S], bh[WB == 8 ? NB : 1][S];
    uint32_t e[NB][S];
    int esh[NB];
    auto issue = [&](int buf, int kt_unclamped) {
        const int kt = min(kt_unclamped, nkt - 1);  // past the end: loaded again, never used
        const int blk = kt * 4 + lb;
        const int sg = L.gsb_shift >= 0 ? blk >> L.gsb_shift : blk / L.gsb;
        esh[buf] = 8 * (sg & 3);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const u32x4* f = reinterpret_cast<const u32x4*>(codes + ((strip[s] * nkt + kt) << (WB == 8 ? 11 : 10)));
            b[buf][s] = f[lane];
            if constexpr (WB == 8) bh[buf][s] = f[64 + lane];
            e[buf][s] = (exq + strip[s] * L.ngq * 16)[(sg >> 2) * 16 + col];
        }
        const uint8_t* x = xbase + (int64_t)kt * 128;
#pragma unroll
        for (int j = 0; j < 2 * MT; ++j) a[buf][j] = *reinterpret_cast<const u32x4*>(x + arow[j]);
    };

    v4f acc[S][MT];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[s][t] = (v4f){0.f, 0.f, 0.f, 0.f};

    auto multiply = [&](int buf) {
        __builtin_amdgcn_wave_barrier();  // behind the reads of the k-tile before
#pragma unroll
        for (int j = 0; j < 2 * MT; ++j) *reinterpret_cast<u32x4*>(turn_w + j * 1024) = a[buf][j];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const u32x4 a0 = *reinterpret_cast<const u32x4*>(turn_r0 + t * 2048), a1 = *reinterpret_cast<const u32x4*>(turn_r1 + t * 2048);
            const v8i av = {(int)a0[0], (int)a0[1], (int)a0[2], (int)a0[3], (int)a1[0], (int)a1[1], (int)a1[2], (int)a1[3]};
            v8i hi = av, lo = av;
            if constexpr (EXACT) split_exponent_bands(av, hi, lo);
            constexpr int BLGP = WB == 8 ? 0 : 4;  // B is E4M3 or E2M1; A is E4M3 with scale byte 127 = 2^0
#pragma unroll
            for (int band = 0; band < (EXACT ? 2 : 1); ++band)
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    v8i bv = {(int)b[buf][s][0], (int)b[buf][s][1], (int)b[buf][s][2], (int)b[buf][s][3], 0, 0, 0, 0};
                    if constexpr (WB == 8) {
                        bv[4] = (int)bh[buf][s][0]; bv[5] = (int)bh[buf][s][1]; bv[6] = (int)bh[buf][s][2]; bv[7] = (int)bh[buf][s][3];
                    }
                    acc[s][t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(band ? lo : hi, bv, acc[s][t], 0, BLGP, 0, 127, 0,
                                                                                (int)(e[buf][s] >> esh[buf]));
                }
        }
    };

    // k-tiles wave, wave + 8, ...; the loop is unrolled by NB so that the buffers are addressed statically.  At most one of them
    // (K up to 1024): nothing to run ahead of, and nothing but it is loaded (1024 x 16, 17 tokens: 3.39 -> 2.85 us).
    if (nkt - wave <= kWaves) {
        if (wave < nkt) {
            issue(0, wave);
            multiply(0);
        }
    } else {
#pragma unroll
        for (int i = 0; i < NB; ++i) issue(i, wave + kWaves * i);
        for (int kt = wave; kt < nkt;) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                multiply(i);
                issue(i, kt + kWaves * NB);
                __builtin_amdgcn_sched_barrier(0);
                kt += kWaves;
                if (kt >= nkt) break;
            }
        }
    }

    __syncthreads();  // the waves' slices of LDS become the partial tiles
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int t = 0; t < MT; ++t) *reinterpret_cast<v4f*>(s_part + (((s * MT + t) * kWaves + wave) * 64 + lane) * 4) = acc[s][t];
    __syncthreads();

    // D[row][col] sits in lane 16 * (row / 4) + col, register row % 4: a thread adds up the four rows of one lane
    const float* colscale = reinterpret_cast<const float*>(blob + L.off_colscale);
    for (int o = tid; o < S * MT * 64; o += 64 * kWaves) {
        const int tile = o >> 6, ln = o & 63;
        const int s = tile / MT, t = tile - s * MT;
        const int64_t n = (strip0 + s) * 16 + (ln & 15), m0 = m_base + t * 16 + 4 * (ln >> 4);
        if (n >= L.N) continue;
        v4f sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += *reinterpret_cast<const v4f*>(s_part + ((tile * kWaves + w) * 64 + ln) * 4);
        const float cs = colscale[n];
        float y[4];
        const float* tr[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t m = min(m0 + i, M - 1);
            y[i] = (sx[m] * cs) * sum[i];
            tr[i] = lorc.T + m * lorc.r;
        }
        // ranks eight and then four at a time, every load ahead of the sums (clamped to the last rank): one after the other they
        // cost 0.2 us each
        auto ranks = [&](auto count, int j0) __attribute__((always_inline)) {
            constexpr int C = decltype(count)::value;
            float v[C], tv[4][C];
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const int j = min(j0 + q, lorc.r - 1);
                v[q] = half_bits_to_f32(lorc.V[(int64_t)j * L.N + n]);
#pragma unroll
                for (int i = 0; i < 4; ++i) tv[i][q] = tr[i][j];
            }
#pragma unroll
            for (int q = 0; q < C; ++q)
                if (j0 + q < lorc.r) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) y[i] = fmaf(tv[i][q], v[q], y[i]);
                }
        };
        int j0 = 0;
        for (; j0 + 8 <= lorc.r; j0 += 8) ranks(std::integral_constant<int, 8>{}, j0);
        for (; j0 < lorc.r; j0 += 4) ranks(std::integral_constant<int, 4>{}, j0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (m0 + i >= M) break;
            if (out_dtype == 0) reinterpret_cast<float*>(Y)[(m0 + i) * ldy + n] = y[i];
            else reinterpret_cast<uint16_t*>(Y)[(m0 + i) * ldy + n] = f32_to_bf16_bits(y[i]);
        }
    }
}

template <int MT, int S, bool EXACT, int WB>
hipError_t launch_cfg(int mblocks, const uint8_t* Xq, const float* sx, int64_t M, const uint8_t* blob, const BlobLayout& L,
                      Lorc lorc, void* Y, int64_t ldy, int out_dtype, hipStream_t s)
{
    // FP8 weights, 64 tokens and four strips in one pass: a second k-tile in flight does not fit the registers (12288 x 16384, 64
    // tokens: 57.2 us with 20 bytes a lane spilled, 45.2 with one; 28672 x 8192, 128 tokens: 82.3 -> 70.9)
    constexpr int NB = MT == 1 ? 4 : MT == 2 ? 3 : WB == 8 && !EXACT && MT * S == 16 ? 1 : 2;
    constexpr size_t smem = (size_t)(S > 2 ? S : 2) * MT * kWaves * 1024;  // partial tiles, the waves' slices before them
    auto kern = k_gemm_mid<MT, S, NB, EXACT, WB>;
    if constexpr (smem > 65536) {  // above the default limit of dynamic LDS, which is a per-function setting
        static OnceStatus attr;
        if (hipError_t e = run_once(attr, [&] {
                return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
            }); e != hipSuccess)
            return e;
    }
    const unsigned grid = (unsigned)((L.nstrips + S - 1) / S * mblocks);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kWaves), smem, s, Xq, sx, M, blob, L, lorc, Y, ldy, out_dtype, mblocks);
    return hipGetLastError();
}

}  // namespace

namespace {

// Token blocks per workgroup (16 each), workgroups along the tokens and strips per workgroup of a launch, with its time in
// microseconds: whole rounds of compute units, each a fixed part, the partial tiles and the k-tiles (fitted to 600 timings:
// ten weight shapes with 8 ... 224 k-tiles, 4 ... 256 tokens; within 11 % on average, and its choice of S was the fastest one
// at every point).
struct MidShape {
    int mt, mblocks, S;
    float us;
};

MidShape mid_shape(int64_t M, const BlobLayout& L)
{
    const int blocks = (int)((M + 15) / 16), mblocks64 = (blocks + 3) / 4;
    const float nkt = (float)L.nkt;
    MidShape best{0, 0, 0, 0.0f};
    // Up to 64 tokens each, except where a few strips are all there is: then fewer, so that more workgroups start at once
    // (512 x 48, 300 tokens: 4.24 -> 2.94 us; 4096 tokens: 4.51 -> 3.40).
    for (int mt = L.N < 64 ? 1 : (blocks + mblocks64 - 1) / mblocks64; mt <= 4; ++mt) {
        const int mblocks = (blocks + mt - 1) / mt;
        for (int S = 1; S <= 4; ++S) {
            const float rounds = (float)(((L.nstrips + S - 1) / S * mblocks + 255) / 256), m = (float)mt, s = (float)S;
            const float us = rounds * (L.wbits == 8 ? 3.3f + 0.159f * s * m + nkt * (0.034f + 0.0223f * m + 0.0482f * s)
                                                    : 3.1f + 0.163f * s * m + nkt * (0.003f + 0.0335f * m + 0.0242f * s));
            if (best.S == 0 || us < best.us) best = MidShape{mt, mblocks, S, us};
        }
        if (L.N >= 64) break;
    }
    return best;
}

// The tiled kernel's time with 2 x 2 waves per tile and wave group, in microseconds, for the line below: a launch is
// 3 + t (e + s k-tiles), t = the most tiles any compute unit gets, or the K slices that the workspace query plans (then `split`).
float two_by_two_us(int64_t M, const BlobLayout& L, bool& split)
{
    static constexpr struct { int bm, bn, kg; float e, s; } kinds[] = {
        {64, 128, 2, 3.8f, 0.368f}, {64, 192, 2, 6.0f, 0.477f}, {64, 256, 2, 6.8f, 0.584f}, {64, 128, 1, 2.1f, 0.368f}, {64, 192, 1, 3.3f, 0.464f},
        {64, 256, 1, 4.5f, 0.549f}, {128, 128, 1, 4.3f, 0.632f}, {128, 192, 1, 6.6f, 0.778f}, {128, 256, 1, 8.6f, 0.928f}, {256, 256, 1, 12.4f, 2.009f}};
    float us = plan_slices(M, L.Np, L.nkt).us;
    split = us > 0.0f;
    if (split) return us;
    for (const auto& k : kinds) {
        const int64_t t = ((M + k.bm - 1) / k.bm) * ((L.Np + k.bn - 1) / k.bn);
        if ((k.kg == 2 && (t > 256 || (L.nkt & 1))) || (k.bm > 64 && M <= 64)) continue;
        const float one = 3.0f + (float)((t + 255) / 256) * (k.e + k.s * (float)L.nkt) * (t <= 256 && k.kg == 1 && k.bm < 256 ? 1.3f : 1.0f);
        if (us == 0.0f || one < us) us = one;
    }
    return us;
}

}  // namespace

// Where this form is the faster one (graph-timed, weights beyond the last-level cache, exact mode, before -> after in us).
bool gemm_mid_wins(int64_t M, const BlobLayout& L, int r, int accum, bool workspace)
{
    const bool fast = accum != 0;
    if (M <= 16) {
        // E4M3 weights: K beyond the registers of the persistent kernel, which left it to the streaming one (11008 x 4096,
        // 16 tokens: 15.2 -> 13.7; 16384 x 12288, 1 token: 45.1 -> 40.5).  Up to 11 tokens and two strips per compute
        // unit: two of the streaming kernel's workgroups share a unit and are ahead (9216 x 8192, 8 / 9 tokens: 17.2 against 18.3 /
        // 17.7 against 18.6; 12 tokens: 17.8 against 17.8), up to rank 8: its epilogue takes one rank after the other (9 tokens, rank
        // 9 / 16 / 40: 19.3 / 21.2 / 27.6 us, here 18.4 / 18.7 / 20.9).
        if (L.wbits == 8) return L.nkt > 40 && (M > 11 || r > 8 || L.nstrips <= 256 || (L.nstrips > 512 && L.nstrips <= 768));
        // K in one piece instead of chunks and a second launch (11008 x 4096, 4 tokens: 11.6 -> 9.5; 28672 x 8192: 28.8 -> 26.4;
        // 16384 x 12288, 16 tokens: 28.8 -> 25.1).  Beyond one round of compute units the persistent kernel's stream wins,
        // as it does where 16 tokens' activations would outweigh a single strip's weights for long (28672 x 4096: 19.5 against 21.2).
        if (L.nkt > 64)
            return L.nstrips <= 768 && !(M > 8 && L.nkt > 128 && L.nstrips <= 256 && L.nstrips * plan_decode(L.nkt).chunks >= 1024);
        // A strip per compute unit: the persistent kernel's prologue serves no second one (8192 x 1024, 16 tokens:
        // 8.2 -> 6.2; 5120 x 4096: 7.1 -> 6.6).  With few tokens it is as short (8192 x 2048, 1 token: 6.2 against 6.7).
        // In one pass it holds the factors of five tokens and ranks up to 8 as well (5120 x 4000, 5 tokens: 5.8 against 6.1).
        return M > (fast && r > 4 && r <= 8 ? 5 : 4) && L.nkt > 32 && L.nstrips <= 256;
    }
    // More tokens: against the tiled kernel's estimate.
    const TilePlan p = effective_tile_plan(M, L.Np, L.nkt, accum, L.wbits, workspace);
    if (p.forced) return false;
    const MidShape ms = mid_shape(M, L);
    // Every L2 fetches the activations of its workgroups, all M x K bytes once several groups of strips are about: beyond what the
    // rest of the time hides that costs 1 us per 8 MB (11008 x 64: 17.6 us up to 1024 tokens, 22.3 at 2048, 33.7 at 4096, 180 MB).
    const int64_t groups = (L.nstrips + ms.S - 1) / ms.S;
    const float fetched = 1e-6f * (float)(groups < 8 ? groups : 8) * (float)M * (float)L.K;
    const float excess = fetched - (18.0f + 0.003f * (float)L.K), extra = excess > 0.0f ? 0.127f * excess : 0.0f;
    const float us = ms.us;
    if (L.wbits == 8) {
        if (M <= 32 && L.nstrips <= 256) {
            // The streaming kernel, a strip per compute unit as here and no LDS on the way of the activations: short K (1024 x 1024,
            // 24 tokens: 3.8 against 4.3; 2048 x 4096, 17 tokens: 5.2 against 5.6), and in the one-pass mode, where it waits for
            // memory only, while its stream fills the chip (4096 x 4096, 24 tokens: 7.3 against 7.8; 3072 x 3072: 5.7
            // against 5.5).  From rank 8 on its epilogue, one rank after the other, decides (4096 x 4096, rank 8: 9.1 against 8.3),
            // with a single k-tile per wave from rank 11 on (1024 x 4096, 24 tokens, rank 16: 6.0 against 5.3; 512 x 1040, rank 9: 3.97
            // against 4.08).
            if ((L.nkt < 16 && r <= 10) || (r < (L.nstrips < 32 ? 9 : 8) && L.nkt <= 20 && M < 24)) return false;
            if (fast && r < 8 && L.nkt <= 40 && L.nstrips >= 192 && (L.nkt * L.nstrips >= 5120 || L.nstrips > 224)) return false;
        }
        if (L.N < 64) return true;  // the tiled kernel has no such tile
        // 64 x 128 tiles in two wave groups, one per compute unit, no K-split: fitted when these took k-tiles in pairs only (6.9 + 0.434 a k-tile by the
        // tiled kernel's present fit) (4096 x 12288, 64 tokens: 24.4 -> 18.8; 28672 x 8192:
        // 111 -> 64.7; 14336 x 2048, 300 tokens: 57.0 -> 32.5).  Near 256 tiles the tiled kernel is 6 to 13 % above its estimate and
        // this one, bound by HBM or in a second round, 10 to 25 % (12288 x 16384, 96 tokens: 57.9 against 65.8 us; 28672 x 8192, 256 tokens:
        // 119 against 140; 8192 x 28672, 32 tokens: 49.3 against 53.3).
        // Many tokens on few channels, one pass: the tiled kernel reads the activations once per 128 channels (11008 x 512,
        // 2048 tokens: 32.4 against 38.7; in two passes 44.6 against 41.8).
        const int64_t tiles = (M + 63) / 64 * ((L.Np + 127) / 128);
        return tiles <= 256 && us < 7.0f + 0.465f * (float)L.nkt && !(fast && extra > 8.0f);
    }
    if (L.N < 64) return true;
    if (M > 64 && M < 1024) {
        // Both sides' estimates, this one's fitted to the exact mode, on 21 weight shapes, both modes and ranks 0, 8 and 40: the lines below
        // give away 0.7 % against always taking the faster one (2304 x 6912, 96 tokens: 8.9, tiled 9.4; 4096 x 12288: 22.1, 16.5; 4096 x
        // 4096, 163 tokens: 13.0, 11.9; 11008 x 1024, 512 tokens: 20.9, 25.4).  One pass takes 4 % off this kernel, which waits for memory;
        // a rank costs both much the same up to 16, beyond that the tiled kernel, whose factors lie in LDS, less.
        // K slices take longer than their estimate where they are short (11008 x 1024, 96 tokens: 13.6 here, 15.7 in slices; one pass, 11008 x
        // 256, 200 tokens: 11.7, 12.3; but 20352 x 1713, 128 tokens: 29.1, 19.8).
        if (p.ksplit > 1) return us + extra < p.us * (fast ? 1.6f : 1.13f);
        return us + extra < p.us * (fast ? 1.12f : r == 0 ? 0.95f : r <= 16 ? 1.05f : 0.92f);
    }
    // Up to 64 tokens, and where very many meet few channels, against the time of 2 x 2 waves a tile, the tiled kernel's only form when
    // this line was fitted; four wave groups are ahead of that, but in a block of 64 tokens by less than 10 % (4096 x 12288: 15.3 here, 13.9;
    // 8192 x 28672, 24 tokens: 35.4, 34.6).  In the exact mode; one pass takes an un-split tiled launch down by 13 to 20 %, this one, which
    // waits for memory, by 3 to 5 (8192 x 28672, 32 tokens: 29.8 against 33.9; 6144 x 24576, 24 tokens: 22.1 against 24.1), and the
    // low-rank correction costs the tiled kernel half as much (3072 x 20000, 32 tokens, rank 8: 18.7 against 19.1).  Beyond 16384 rows this
    // kernel is slower than its estimate (28672 x 8192, 32 tokens: 37.3 against 38.2 us; one pass 33.3 against 37.7).  Many tokens on
    // few channels go to the tiled kernel by the activations they fetch (11008 x 128, 2048 tokens: 19.2 against 34.2).
    bool split;
    float bar = two_by_two_us(M, L, split);
    if (L.nkt > 128) bar *= fast ? 0.87f : 0.97f;
    else if (!split) bar *= fast ? 0.87f : r > 0 ? 0.95f : 1.0f;
    else if (fast && extra > 0.0f) bar *= 0.93f;  // 11008 x 1024, 1024 tokens: 22.6 against 24.4
    return us + extra < bar;
}

hipError_t launch_gemm_mid(const uint8_t* Xq, const float* sx, int64_t M, const uint8_t* blob, const BlobLayout& L,
                           Lorc lorc, void* Y, int64_t ldy, int out_dtype, int accum, hipStream_t s)
{
    if (M == 0 || L.N == 0) return hipSuccess;
    const MidShape ms = mid_shape(M, L);
    const int mblocks = ms.mblocks, mt = ms.mt, S = ms.S;
#define ZQ_MID(MT_, S_) \
    if (mt == MT_ && S == S_) { \
        if (L.wbits == 8) return accum == 0 ? launch_cfg<MT_, S_, true, 8>(mblocks, Xq, sx, M, blob, L, lorc, Y, ldy, out_dtype, s) \
                                            : launch_cfg<MT_, S_, false, 8>(mblocks, Xq, sx, M, blob, L, lorc, Y, ldy, out_dtype, s); \
        return accum == 0 ? launch_cfg<MT_, S_, true, 4>(mblocks, Xq, sx, M, blob, L, lorc, Y, ldy, out_dtype, s) \
                          : launch_cfg<MT_, S_, false, 4>(mblocks, Xq, sx, M, blob, L, lorc, Y, ldy, out_dtype, s); \
    }
#define ZQ_MID_ALL(MT_) ZQ_MID(MT_, 1) ZQ_MID(MT_, 2) ZQ_MID(MT_, 3) ZQ_MID(MT_, 4)
    ZQ_MID_ALL(1) ZQ_MID_ALL(2) ZQ_MID_ALL(3) ZQ_MID_ALL(4)
#undef ZQ_MID_ALL
#undef ZQ_MID
    return hipErrorInvalidValue;
}

}  // namespace zqfp
