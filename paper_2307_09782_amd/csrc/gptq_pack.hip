// GPTQ on the E2M1 grid with power-of-two group scales (the weight quantizer the paper runs: Section 3,
// Appendix A; scales as in "Casting the FP4 to FP8", methods M1 / M2).  Offline step; its output is the same
// packed blob zqfp_pack_weight_fp4 makes.
//
// Input channels (rows of the K x N weight) are quantized in order; the scaled error of channel k is pushed
// onto the channels behind it with row k of U, the upper Cholesky factor of the inverse Hessian:
//     q_k = S e2m1(w_k / S);  err = (w_k - q_k) / U[k][k];  w_j -= U[k][j] err   (j > k).
// Output channels never interact, so ONE launch does everything: a workgroup owns C = 16 ... 64 output channels for
// the whole of K and never waits for another.  It takes the rows in panels of 128.  A panel is first brought up to
// date with all earlier channels,
//     w[i][n] -= sum_{k < i0} U[k][i] err[k][n],
// a float32 matrix product with the errors the workgroup itself has left in its part of the workspace, and is then
// quantized in sub-blocks of 16 rows: one wave runs the serial chain with the 16 x C values in registers (lane =
// channel), while three others push the previous sub-block's errors onto the rows further down, on the matrix cores,
// out of LDS.
//
// The product and the chain are each about half of the work, and one leaves idle what the other needs: the chain is one
// wave's latency (0.24 us a row), the product is the matrix cores' time.  So twelve waves run side by side, three
// to a SIMD: waves 0 .. 3 quantize panel p while waves 4 .. 11 already form the sums of panel p + 1 over all the
// errors there are, 0 .. p - 1, spread over the intervals between the others' barriers; when panel p is done only its own
// 128 errors are left to add.  Eight waves for the sums (two halves of the panel's rows, four quarters of k; 64 x C values
// of a wave in registers on v_mfma_f32_16x16x4_f32, operands straight from L2, 16 bytes per lane, with the rows and
// columns dealt to the instructions such that a lane's four consecutive floats feed four instructions) were
// within 5 % of four at 4096 x 12288 and 12 % better at 4096 x 4096.  Groups of 256 need both of their panels before the first
// is quantized, so their sums are formed in between, as one after the other.
//
// K^2 N / 2 multiply-adds are the bound: 1.34 ms at the 154 TFLOP/s that a large float32 product reaches, for
// 4096 x 12288; K^2 / 2 floats of U per workgroup come from L2.  Measured, G = 128, M1, one after the other -> side by side:
// 4096 x 12288 3670 -> 2272 us, 4096 x 4096 2019 -> 1077, 4096 x 16384 4305 -> 2913, 6144 x 12288 7903 -> 4683, 1024 x 12288
// 381 -> 288; G = 256, 4096 x 12288 3953 -> 2576 (there by the eight waves alone).  With the sums in registers for every width, where
// 48 and 64 channels had 80 and 144 bytes a lane of them in scratch memory: 4096 x 12288 2272 -> 2165, 4096 x 16384 2920 -> 2623, 4096 x
// 4096 (16 channels) unchanged, G = 256, 4096 x 12288 2573 -> 2430, 2048 x 16384 1023 -> 915.  The matrix cores are then 62 % busy over
// the whole run; U's reads hit L2 at 226 cycles and hold nothing up.  C is the least that lets every workgroup have a
// compute unit of its own, so that N = 4096 runs on all of them as N = 12288 does.
#include "zqfp_internal.h"

namespace zqfp {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

constexpr int kPanel = 128;  // rows brought up to date at once
constexpr int kSub = 16;     // rows quantized by one serial chain

// NT floats in a row, 4-byte aligned (one load of 4 NT bytes)
template <int NT>
struct __attribute__((packed, aligned(4))) Floats {
    float v[NT];
};
// four of the caller's floats, which may start at any of them
struct __attribute__((packed, aligned(4))) Row4 { v4f v; };

// acc[r][t] += sum_{k in [ka, kb)} U[k][i0 + row] err[k][col], this wave's quarter of the k (16 in a row, dealt in
// turn; kb - ka is a multiple of 128), for 64 rows of the panel.  Instruction (r, t) holds rows 4 i + r (i = 0..15) and columns
// NT j + t (j = 0..15): a lane's 16 bytes of a row of U are the A operands of four instructions.  The chunks go by one
// at a time, the next ones loaded meanwhile, as many as the caller asks for.
template <int NT>
struct PanelSum {
    static constexpr int C = 16 * NT;
    static constexpr int S = 4;  // steps of 4 k in a chunk
    static constexpr int PF = NT == 4 ? 2 : 3;  // 168 registers a lane; chunks in registers: the one multiplied and PF - 1 on their way
    struct Chunk {
        v4f a[S];
        float b[S][NT];
    };
    v4f acc[4][NT];
    Chunk c[PF];
    const char *u, *e;       // the wave's first row of U and of err (uniform: scalar registers), and the lane's offset from it
    uint32_t u_lane, e_lane;
    int64_t ldu;
    int n, done;             // chunks of this wave, and how many are done

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[r][t] = (v4f){0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void load(Chunk& c, int i)
    {
        const int64_t k0 = 16 * S * (int64_t)min(i, n - 1);  // past the end: the last one again, unused
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const char* p = u + (k0 + 4 * s) * ldu * 4;
            c.a[s] = reinterpret_cast<const Row4*>(p + u_lane)->v;
            const Floats<NT> f = *reinterpret_cast<const Floats<NT>*>(e + (k0 + 4 * s) * (4 * C) + e_lane);
#pragma unroll
            for (int t = 0; t < NT; ++t) c.b[s][t] = f.v[t];
        }
    }
    __device__ __forceinline__ void multiply(const Chunk& c)
    {
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(c.a[s][r], c.b[s][t], acc[r][t], 0, 0, 0);
    }
    // the sum over [ka, kb) for rows 64 * half + [0, 64) of panel i0 begins; `wave` of four
    __device__ __forceinline__ void begin(const float* U, int64_t K, int64_t i0, const float* err, int64_t ka, int64_t kb, int wave, int half, int lane)
    {
        const int j = lane & 15, lb = lane >> 4;
        n = (int)((kb - ka) / (16 * S));
        done = 0;
        ldu = K;
        u = reinterpret_cast<const char*>(U + (ka + 4 * S * wave) * K + i0 + 64 * half);
        e = reinterpret_cast<const char*>(err + (ka + 4 * S * wave) * C);
        u_lane = 4u * ((uint32_t)lb * (uint32_t)K + 4u * (uint32_t)j);
        e_lane = 4u * (uint32_t)(lb * C + NT * j);
        if (n > 0) {
#pragma unroll
            for (int i = 0; i < PF - 1; ++i) load(c[i], i);
        }
    }
    // chunks up to the one given; the registers move on by copies, in the shadow of the matrix instructions
    __device__ __forceinline__ void advance(int upto)
    {
        for (; done < upto; ++done) {
            load(c[PF - 1], done + PF - 1);
            multiply(c[0]);
#pragma unroll
            for (int i = 0; i < PF - 1; ++i)
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    c[i].a[s] = c[i + 1].a[s];
#pragma unroll
                    for (int t = 0; t < NT; ++t) c[i].b[s][t] = c[i + 1].b[s][t];
                }
        }
    }
};

template <int NT, int MODE>
__global__ __launch_bounds__(768) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_gptq(const uint16_t* __restrict__ W, int64_t ldw, const float* __restrict__ U, BlobLayout L,
                                                 float* ws_err, float* ws_held, uint8_t* __restrict__ blob)
{
    constexpr int C = 16 * NT, mode = MODE;  // 1: M1, 2: M2
    constexpr int LDW = C + 4;    // slab row: the four row groups of a 16 x 16 tile fall on disjoint banks
    constexpr int LDE = C + 16;   // error row, for the same reason
    constexpr int LDU = kPanel + 16;
    __shared__ __attribute__((aligned(16))) float s_w[kPanel][LDW];       // the panel's weights as they stand
    __shared__ __attribute__((aligned(16))) float s_u[2][kSub][LDU];      // a sub-block's rows of U / 2^x, columns of the panel
    __shared__ v2f s_rdiag[2][kSub];                                      // 1 / (U[k][k] / 2^x), and x (an int's bits)
    __shared__ float s_err[2][kSub][LDE];                                 // a sub-block's errors times 2^x, negated
    __shared__ float s_amax[4][C];
    extern __shared__ __attribute__((aligned(16))) uint16_t s_next[];     // [kPanel][C]: the next panel's weights as they came

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j16 = lane & 15, lb = lane >> 4;
    const bool summing = wave >= 4;  // waves 4 .. 11 form the panels' sums, waves 0 .. 3 quantize
    const int64_t n0 = (int64_t)blockIdx.x * C;
    const int64_t K = L.K;
    float* err = ws_err + (int64_t)blockIdx.x * K * C;            // [K][C], this workgroup's own
    float* held = ws_held + (int64_t)blockIdx.x * kPanel * C;     // [128][C]: groups of 256 only
    float* colscale = reinterpret_cast<float*>(blob + L.off_colscale);

    // the channel of this lane where a wave's lanes are channels
    const int64_t n = n0 + lane;
    const bool chan = lane < C && n < L.Np, live = lane < C && n < L.N;

    // ---- column scales (M2: from the original column) and header
    float cmax = 0.0f, cs = 1.0f;
    if (mode != 1) {
        float m = 0.0f;
        if (live && !summing)
            for (int64_t k = wave; k < K; k += 32) {  // K is a multiple of 128
                float v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = bf16_bits_to_f32(W[(k + 4 * i) * ldw + n]);
#pragma unroll
                for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(v[i]));
            }
        if (lane < C && !summing) s_amax[wave][lane] = m;
        __syncthreads();
        if (lane < C) cmax = fmaxf(fmaxf(s_amax[0][lane], s_amax[1][lane]), fmaxf(s_amax[2][lane], s_amax[3][lane]));
        if (cmax != 0.0f) cs = cmax / 6.0f;  // IEEE binary32 division
        __syncthreads();
    }
    if (wave == 0 && chan) colscale[n] = live ? cs : 0.0f;
    // w / c in the chain below: lifted by 2^60 in columns so small that its residuals would leave the normal range
    const float lift = cs < 0x1p-60f ? 0x1p60f : 1.0f, lcs = cs * lift, rcs = 1.0f / lcs;
    if (blockIdx.x == 0 && tid == 0) {
        BlobHeader h;
        h.magic = kBlobMagic; h.version = kBlobVersion;
        h.K = L.K; h.N = L.N; h.Np = L.Np;
        h.G = L.G; h.Gs = L.Gs; h.mode = mode; h.ngs = L.ngs; h.ngq = L.ngq; h.wbits = 4;
        h.off_codes = L.off_codes; h.off_exps = L.off_exps; h.off_colscale = L.off_colscale; h.total = L.total;
        *reinterpret_cast<BlobHeader*>(blob) = h;
    }

    const bool ahead = L.G != 256;  // a group of 256 needs both of its panels at once

    // ================================================================ waves 4 .. 11: the panels' sums
    // Every barrier of the other waves has its counterpart here, in the same order.
    if (summing) {
        PanelSum<NT> sum;
        const int half = (wave - 4) >> 2;  // rows 64 * half + [0, 64); the four waves of a half split k
        // The four waves of a half take their sums off s_w in four rounds, a quarter of its rows each, so that all work: a fixed order.
        auto take_off = [&]() __attribute__((always_inline)) {
            for (int round = 0; round < 4; ++round) {
                __syncthreads();  // s_w holds the weights / the round before is done
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (((wave + round) & 3) == q) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            float* w = &s_w[64 * half + 16 * lb + 4 * i + q][NT * j16];
#pragma unroll
                            for (int t = 0; t < NT; ++t) w[t] -= sum.acc[q][t][i];
                        }
                        asm volatile("" ::"n"(q));  // keeps the four apart: folded into one with a run-time q they would put the sums in scratch memory
                    }
            }
            __syncthreads();
        };
        auto all_of = [&](int64_t i0, int64_t ka, int64_t kb) __attribute__((always_inline)) {
            sum.begin(U, K, i0, err, ka, kb, wave & 3, half, lane);
            sum.advance(sum.n);
        };
        if (ahead) __syncthreads();  // the first panel: nothing to take off
        for (int64_t i0 = 0; i0 < K; i0 += kPanel) {
            if (!ahead) {
                const bool first = (i0 & 255) == 0;
                if (first) {
                    sum.clear();
                    all_of(i0 + kPanel, 0, i0);
                    take_off();
                    __syncthreads();  // held
                }
                sum.clear();
                all_of(i0, first ? 0 : i0 - kPanel, i0);
                take_off();
            }
            __syncthreads();  // rows of U
            // The next panel's sums over all errors but this panel's, spread over the intervals between the barriers of the other waves:
            // three parts where the chain runs, one where its errors are pushed on.  Plain barriers, which leave loads in flight.
            const bool more = ahead && i0 + kPanel < K;
            constexpr int kIntervals = 2 * (kPanel / kSub) - 1, kParts = 4 * (kPanel / kSub) - 1;
            if (more) {
                sum.clear();
                if (i0 == 0) sum.begin(U, K, kPanel, err, 0, 0, wave & 3, half, lane);  // else begun below, a panel ago
            }
            for (int iv = 0; iv < kIntervals - 1; ++iv) {
                const int t = iv >> 1;
                const bool push = (iv & 1) != 0;
                if (more) sum.advance(sum.n * (4 * t + (push ? 4 : 3)) / kParts);
                __builtin_amdgcn_s_barrier();
                if (push && ((i0 + kSub * (t + 1)) % L.G) == 0) __builtin_amdgcn_s_barrier();
            }
            if (more) sum.advance(sum.n);
            __syncthreads();  // this panel's errors are out
            if (more) {
                all_of(i0 + kPanel, i0, i0 + kPanel);
                if (i0 + 2 * kPanel < K) sum.begin(U, K, i0 + 2 * kPanel, err, 0, i0 + kPanel, wave & 3, half, lane);  // its first loads
                take_off();
            } else if (!ahead) {
                __syncthreads();
            }
        }
        return;
    }

    // ================================================================ waves 0 .. 3: the chain and what it pushes on
    __builtin_amdgcn_s_setprio(3);  // a wave of the others shares the SIMD: its matrix instructions can wait, the chain cannot
    auto taken_off = [&]() __attribute__((always_inline)) {
        for (int round = 0; round < 5; ++round) __syncthreads();
    };
    // tid, but not as a value known before: the addresses of a copy of a whole panel, the same for every panel, would be formed ahead of
    // all panels, and kept in scratch memory
    auto here = [](int i) __attribute__((always_inline)) {
        asm volatile("" : "+v"(i));
        return i;
    };
    // the panel's weights, or what has been held of it, into s_w, from which the sums are taken off then
    auto fill = [&](int64_t i0, bool from_held) __attribute__((always_inline)) {
        for (int idx = here(tid); idx < kPanel * C; idx += 256) {
            const int r = idx / C, c = idx % C;
            s_w[r][c] = from_held ? held[idx] : n0 + c < L.N ? bf16_bits_to_f32(W[(i0 + r) * ldw + n0 + c]) : 0.0f;
        }
    };
    // absmax of `rows` rows of s_w from row r0 on, per channel, over all four waves; combined by combined_max()
    auto partial_max = [&](int r0, int rows, float m) __attribute__((always_inline)) {
        if (lane < C) {
            for (int r = wave; r < rows; r += 4) m = fmaxf(m, fabsf(s_w[r0 + r][lane]));
            s_amax[wave][lane] = m;
        }
        return m;
    };
    // rows of U of the sub-block at row k0 = i0 + 16 t, columns i0 + [0, 128): thread -> 8 floats of row tid / 16, that row's
    // diagonal, and the diagonal of row tid % 16
    auto fetch_u = [&](v4f (&u)[2], float& d, float& dr, int64_t k0, int64_t i0) __attribute__((always_inline)) {
        const float* p = U + (k0 + (tid >> 4)) * K + i0 + 8 * (tid & 15);
        u[0] = reinterpret_cast<const Row4*>(p)->v;
        u[1] = reinterpret_cast<const Row4*>(p + 4)->v;
        d = U[(k0 + (tid & 15)) * K + k0 + (tid & 15)];
        dr = U[(k0 + (tid >> 4)) * K + k0 + (tid >> 4)];
    };
    // A row of U and its error times the inverse power of two are the same row: every row is held over the 2^x that brings
    // its diagonal into [1/2, 1), so that neither the reciprocal nor the residual below leaves the normal range.
    auto store_u = [&](const v4f (&u)[2], float d, float dr, int buf) __attribute__((always_inline)) {
        const int x = __builtin_amdgcn_frexp_expf(dr);
        float* p = &s_u[buf][tid >> 4][8 * (tid & 15)];
        v4f a, b;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = ldexpf(u[0][i], -x);
            b[i] = ldexpf(u[1][i], -x);
        }
        *reinterpret_cast<v4f*>(p) = a;
        *reinterpret_cast<v4f*>(p + 4) = b;
        if (tid < kSub)  // IEEE binary32 division: correctly rounded
            s_rdiag[buf][tid] = (v2f){1.0f / __builtin_amdgcn_frexp_mantf(d), __int_as_float(__builtin_amdgcn_frexp_expf(d))};
    };
    // 16 x 16 tile (row block rb of the panel, column block cb) -= its share of a sub-block's errors
    auto push_tile = [&](int rb, int cb, int buf) __attribute__((always_inline)) {
        v4f a;
        float* w = &s_w[16 * rb + 4 * lb][16 * cb + j16];
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] = w[q * LDW];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            a = __builtin_amdgcn_mfma_f32_16x16x4f32(s_u[buf][4 * s + lb][16 * rb + j16], s_err[buf][4 * s + lb][16 * cb + j16], a, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q * LDW] = a[q];
    };

    int e = 0;                     // the current group's exponent (wave 0's lanes)
    uint32_t ebytes = 0x7F7F7F7Fu;  // and the dword of exponent bytes being filled
    const int64_t strip = n >> 4;
    v4f u[2];
    float d, dr;
    auto first_rows = [&](int64_t i0) __attribute__((always_inline)) {
        fetch_u(u, d, dr, i0, i0);
        store_u(u, d, dr, 0);
        fetch_u(u, d, dr, i0 + kSub, i0);
    };
    if (ahead) {
        fill(0, false);
        first_rows(0);
        __syncthreads();
    }
    for (int64_t i0 = 0; i0 < K; i0 += kPanel) {
        // ---- the panel (up to date already, or brought up to date now), and the absmax of a group that begins with it
        if (ahead) {
            partial_max(0, L.G, 0.0f);
        } else if ((i0 & 255) == 0) {  // the group's second panel comes first and waits in the workspace
            fill(i0 + kPanel, false);
            taken_off();
            const float m = partial_max(0, kPanel, 0.0f);
            for (int idx = here(tid); idx < kPanel * C; idx += 256) held[idx] = s_w[idx / C][idx % C];
            __syncthreads();
            fill(i0, false);
            taken_off();
            partial_max(0, kPanel, m);
        } else {
            fill(i0, true);
            taken_off();
        }
        const bool more = ahead && i0 + kPanel < K;  // the next panel is formed meanwhile
        if (!ahead) first_rows(i0);
        __syncthreads();

        for (int t = 0; t < kPanel / kSub; ++t) {
            const int buf = t & 1;
            const int64_t k0 = i0 + kSub * t;
            if (wave == 0) {
                // ---- the serial chain of sub-block t, lane = channel
                if (lane < C) {
                    if (k0 % L.G == 0) {  // a new group: its scale from the weights as they stand now
                        const float amax = fmaxf(fmaxf(s_amax[0][lane], s_amax[1][lane]), fmaxf(s_amax[2][lane], s_amax[3][lane]));
                        e = mode == 1 ? m1_exponent(amax) : -m2_shift(cmax, amax);
                        const int64_t sg = k0 / L.Gs;  // G is 32, 64, 128 or 256 here: stored groups are the groups
                        const int b = (int)(sg & 3);
                        if (b == 0) ebytes = 0x7F7F7F7Fu;
                        ebytes = (ebytes & ~(0xFFu << (8 * b))) | ((uint32_t)(live ? e + 127 : 127) << (8 * b));
                        if (chan && (b == 3 || sg == L.ngs - 1))
                            reinterpret_cast<uint32_t*>(blob + L.off_exps)[(size_t)(strip * L.ngq + (sg >> 2)) * 16 + (lane & 15)] = ebytes;
                    }
                    const float scale = ldexpf(1.0f, e);
                    // what four rows' steps read, ahead of them: an LDS read among the steps is waited for there
                    float w[kSub], ur[kSub][kSub];
                    v2f rd16[kSub];
#pragma unroll
                    for (int r = 0; r < kSub; ++r) w[r] = s_w[kSub * t + r][lane];
                    auto rows_of_u = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
                        for (int r = r0; r < r0 + 4; ++r) {
                            rd16[r] = s_rdiag[buf][r];
#pragma unroll
                            for (int q = r / 4; q < 4; ++q) {
                                const v4f v = *reinterpret_cast<const v4f*>(&s_u[buf][r][kSub * t + 4 * q]);
#pragma unroll
                                for (int i = 0; i < 4; ++i) ur[r][4 * q + i] = v[i];
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    rows_of_u(0);
                    uint32_t code[2] = {0u, 0u};
#pragma unroll
                    for (int r = 0; r < kSub; ++r) {
                        // code of w / S and its value, by the hardware conversions (exact: see pack_weight.hip);
                        // under M2 w / c first, rounded correctly: two residual corrections of w times the
                        // correctly rounded reciprocal (the second one starts within one ulp, as Markstein's theorem asks)
                        if (r > 0 && r % 4 == 0) rows_of_u(r);
                        float x = w[r];
                        if (mode != 1) {
                            x *= lift;
                            float y = x * rcs;
                            y = fmaf(fmaf(-y, lcs, x), rcs, y);
                            x = fmaf(fmaf(-y, lcs, x), rcs, y);
                        }
                        const uint32_t c4 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, x, 0.0f, scale, 0);
                        const v2f q2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c4, scale, 0);
                        const float q = mode == 1 ? q2[0] : q2[0] * cs;
                        code[r >> 3] |= (c4 & 15u) << (4 * (r & 7));
                        // (w - q) / U[k][k], times 2^x.  One residual correction of the product with the correctly rounded
                        // reciprocal rounds correctly: it is within 1.5 * 2^-24 ulp of the quotient before its last rounding, and
                        // quotients that near the middle of two floats leave remainders of a few units; the 2.6e8 mantissa pairs
                        // that do (every divisor, up to 9 units) all come out as the IEEE division has them.
                        const v2f rdx = rd16[r];
                        const float diff = w[r] - q, diag = ur[r][r], rd = rdx[0];
                        const float y = diff * rd;
                        const float ev = fmaf(fmaf(-y, diag, diff), rd, y);
#pragma unroll
                        for (int s = r + 1; s < kSub; ++s) w[s] = fmaf(-ur[r][s], ev, w[s]);
                        s_err[buf][r][lane] = -ev;
                        err[(k0 + r) * C + lane] = ldexpf(ev, -__float_as_int(rdx[1]));
                    }
                    if (chan) {
                        const int kk = (int)(k0 & 127);
                        *reinterpret_cast<uint2*>(blob + L.off_codes + ((size_t)(strip * L.nkt + (k0 >> 7)) * 64 + (kk >> 5) * 16 + (lane & 15)) * 16 +
                                                  ((kk >> 4) & 1) * 8) = live ? make_uint2(code[0], code[1]) : make_uint2(0u, 0u);
                    }
                }
            } else if (t > 0 && (k0 % L.G) != 0) {
                // ---- meanwhile: the previous sub-block's errors onto the rows beyond this one
                const int tiles = (kPanel / kSub - 1 - t) * NT;
                for (int i = wave - 1; i < tiles; i += 3) push_tile(t + 1 + i / NT, i % NT, buf ^ 1);
            } else if (t == 0 && more) {
                // ---- or fetch the next panel's weights
                for (int idx = tid - 64; idx < kPanel * C; idx += 8 * 192) {
                    uint16_t v[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const int at = min(idx + 192 * q, kPanel * C - 1), r = at / C, c = at - r * C;
                        v[q] = W[(i0 + kPanel + r) * ldw + min(n0 + c, L.N - 1)];
                        if (n0 + c >= L.N) v[q] = 0;
                    }
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        if (idx + 192 * q < kPanel * C) s_next[idx + 192 * q] = v[q];
                }
            }
            __syncthreads();
            if (t + 1 == kPanel / kSub) break;
            // ---- the errors onto the next sub-block's rows; onto all rows further down where a group begins with it
            const bool starts_group = ((k0 + kSub) % L.G) == 0;
            const int tiles = starts_group ? (kPanel / kSub - 1 - t) * NT : NT;
            for (int i = wave; i < tiles; i += 4) push_tile(t + 1 + i / NT, i % NT, buf);
            store_u(u, d, dr, buf ^ 1);
            if (t + 2 < kPanel / kSub) fetch_u(u, d, dr, k0 + 2 * kSub, i0);
            __syncthreads();
            if (starts_group) {
                partial_max(kSub * (t + 1), L.G, 0.0f);
                __syncthreads();
            }
        }
        if (more) {
            for (int idx = here(tid); idx < kPanel * C; idx += 256) s_w[idx / C][idx % C] = bf16_bits_to_f32(s_next[idx]);
            first_rows(i0 + kPanel);
            taken_off();
        } else if (!ahead) {
            __syncthreads();  // nobody fills s_w with the next panel before the chain has left it
        }
    }
}

template <int NT, int MODE>
hipError_t launch_nt(unsigned wgs, const uint16_t* W, int64_t ldw, const float* U, const BlobLayout& L, float* err, float* held, uint8_t* blob,
                     hipStream_t s)
{
    constexpr size_t smem = (size_t)kPanel * 16 * NT * sizeof(uint16_t);  // with the static part above the default limit of 64 KB
    static OnceStatus attr;
    if (hipError_t e = run_once(attr, [] {
            return hipFuncSetAttribute(reinterpret_cast<const void*>(k_gptq<NT, MODE>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        }); e != hipSuccess)
        return e;
    hipLaunchKernelGGL((k_gptq<NT, MODE>), dim3(wgs), dim3(768), smem, s, W, ldw, U, L, err, held, blob);
    return hipGetLastError();
}

// output channels per workgroup: the least multiple of 16 that leaves every workgroup a compute unit, at most 64
int gptq_tiles(int64_t Np)
{
    const int64_t cus = compute_units();
    for (int nt = 1; nt < 4; ++nt)
        if ((Np + 16 * nt - 1) / (16 * nt) <= cus) return nt;
    return 4;
}

}  // namespace

// the errors of every workgroup, [K][C] float32, and (groups of 256) a panel held back, [128][C]; C divides the
// channel count rounded up to whole workgroups, which is less than N + 64
size_t gptq_workspace_bytes(int64_t K, int64_t N, int G)
{
    const int64_t B = G > 128 ? G : 128;
    auto up = [](size_t b) { return (b + 255) / 256 * 256; };
    return up((size_t)K * (N + 63) * 4) + up((size_t)B * (N + 63) * 4);
}

hipError_t launch_gptq_pack(const uint16_t* W, int64_t ldw, const BlobLayout& L, int mode, const float* U, uint8_t* blob,
                            void* workspace, hipStream_t s)
{
    const int nt = gptq_tiles(L.Np);
    const int64_t wgs = (L.Np + 16 * nt - 1) / (16 * nt);
    float* err = static_cast<float*>(workspace);
    float* held = err + ((size_t)L.K * (wgs * 16 * nt) * 4 + 255) / 256 * 64;
#define ZQ_GPTQ(NT) \
    return mode == 1 ? launch_nt<NT, 1>((unsigned)wgs, W, ldw, U, L, err, held, blob, s) : launch_nt<NT, 2>((unsigned)wgs, W, ldw, U, L, err, held, blob, s)
    if (nt == 1) ZQ_GPTQ(1);
    if (nt == 2) ZQ_GPTQ(2);
    if (nt == 3) ZQ_GPTQ(3);
    ZQ_GPTQ(4);
#undef ZQ_GPTQ
}

}  // namespace zqfp
