// Projection kernels of the decode path: y = W x for up to 8 rows sharing one sweep over W, with the
// epilogues of the layer (store, residual + next RMSNorm inputs, SwiGLU, exit / final head partials of
// Eq. 2), on the vector ALUs and on the matrix cores; the tile packing of the weights; the head
// evaluation whose scratch area is a static device array.  As everywhere in this library, a row's
// value never depends on how many rows share the launch.
#include "kernels.h"
#include "device_utils.h"

#include <math.h>
#include <mutex>
#include <type_traits>

namespace sb {

// What the kernels read of GemvArgs.  The host writes a launch's arguments across the bus: 32 / 168 / 328 bytes take 2.11 / 2.26 / 2.32 us of it in a
// process beside the GPU and 2.7 / 3.3 / 4.0 in one on the far socket, and a chain of small launches is bound by that.
struct HeadOut { float* partials; float* logits; float T; };
template <int EPI> struct ValuOut { float* y; int32_t ldy; };
template <> struct ValuOut<EPI_HEAD> : HeadOut {};
template <int EPI> struct MfmaOut;
template <> struct MfmaOut<EPI_STORE> { float* y; int32_t ldy; };
template <> struct MfmaOut<EPI_SWIGLU> { float* y; uint16_t* ys; int32_t ldy; };
template <> struct MfmaOut<EPI_RESID> { float* y; const float* gainA; uint16_t* nxA; const float* gainB; uint16_t* nxB; float* ssq_out; float* ssq_out2; int32_t ldy; };
template <> struct MfmaOut<EPI_HEAD> : HeadOut {};
template <int EPI> struct ValuArgs {
    const void* W; const float* x; const float* norm_gain;
    int32_t N, K;
    float eps;
    ValuOut<EPI> out;
};
template <int EPI> struct MfmaArgs {
    const void* W; const void* x;   // (x: float rows or their parts)
    int32_t N, K, M;
    uint32_t row_mask;
    const float* ssq_in;
    int32_t ssq_nb, ssq_ld;
    float eps;
    MfmaOut<EPI> out;
};
static HeadOut head_out(const HeadArgs& h) { return {h.partials, h.logits, h.T}; }
template <int EPI>
static ValuArgs<EPI> valu_args(const GemvArgs& a) {
    ValuArgs<EPI> v{a.W, a.x, a.norm_gain, a.N, a.K, a.eps, {}};
    if constexpr (EPI == EPI_HEAD) static_cast<HeadOut&>(v.out) = head_out(a.head);
    else v.out = {a.y, a.ldy};
    return v;
}
template <int EPI, bool RAW>
static MfmaArgs<EPI> mfma_args(const GemvArgs& a) {
    MfmaArgs<EPI> v{a.W, RAW ? (const void*)a.x : (const void*)a.xs, a.N, a.K, a.M, a.row_mask, a.ssq_in, a.ssq_nb, a.ssq_ld, a.eps, {}};
    if constexpr (EPI == EPI_HEAD) static_cast<HeadOut&>(v.out) = head_out(a.head);
    else if constexpr (EPI == EPI_STORE) v.out = {a.y, a.ldy};
    else if constexpr (EPI == EPI_SWIGLU) v.out = {a.y, a.ys, a.ldy};
    else v.out = {a.y, a.gainA, a.nxA, a.gainB, a.nxB, a.ssq_out, a.ssq_out2, a.ldy};
    return v;
}

// Partial (max, arg max, sum exp) of the block's logits zs[i][m], i < ROWS: thread (m, i) holds one
// logit, the ROWS lanes of a row are reduced with a fixed shuffle tree (ties: the lower index).
// Every thread of the block calls it (blocks have at least 8 * ROWS threads).
template <int ROWS>
__device__ __forceinline__ void head_partial(const HeadOut& h, float (*zs)[SB_MAX_W], uint32_t rows, int n0, int N, int nb) {
    static_assert(ROWS == 16 || ROWS == 32, "a row's lanes lie in one wave");
    const int tid = threadIdx.x;
    if (tid >= SB_MAX_W * ROWS) return;   // (whole waves: 8 * ROWS is a multiple of 64)
    const int m = tid / ROWS, i = tid % ROWS, n = n0 + i;
    const bool live = n < N;
    const float z = live ? zs[i][m] : -SB_INF;
    const bool row_on = (rows >> m) & 1u;
    if (h.logits && live && row_on) h.logits[(size_t)m * N + n] = z;
    float mx = z;
    int idx = live ? n : 0x7fffffff;
    lanes_argmax<ROWS / 2>(mx, idx);
    const float sum = lanes_sum<ROWS / 2>(live ? expf((z - mx) / h.T) : 0.f);
    if (i == 0 && row_on) {
        float* p = h.partials + ((size_t)m * nb + blockIdx.x) * 4;
        p[0] = mx;
        p[1] = __int_as_float(idx);
        p[2] = sum;
    }
}

// ---------------------------------------------------------------- GEMV, vector ALU
// y[m][n] = sum_k W[n][k] x[m][k] for M rows sharing one sweep over W.  One wave
// owns one, two or four weight rows (launch_gemv_valu_m); lanes stride the K dimension in 16-byte pieces (128-bit
// loads), partial sums are combined with a fixed shuffle tree.  x is staged in
// LDS in chunks.  The order in which a row's products are added is a function of
// K alone.
//
// SHORT (K <= SB_VALU_NORM_K, one 16-byte piece of a row per thread): the whole matrix is one round trip, so the weights are
// requested before the rows are staged, and the rows are normalised while they are staged where the caller asks for it: a
// small model is bound by its number of launches (4.2 us each in a chain of them), and the sum of squares costs
// a block two barriers (same order of additions as rmsnorm_kernel).  Longer rows would be read twice by every
// block, and registers that hold weights through the staging are waves the stream misses: [11008 x 4096] bf16, 8 rows, 52.7 us
// with the weights first and 24.6 without ([1024 x 1024] fp32, one row, 3.4 us with them first, 4.0 in a loop of load and store).
template <typename WT, int M, int EPI, bool SHORT, int R>
__global__ __launch_bounds__(256) void gemv_valu_kernel(ValuArgs<EPI> a) {
    static_assert(EPI != EPI_HEAD || R == 4, "a head's partial is taken over 16 logits");
    constexpr int KC = SHORT ? SB_VALU_NORM_K : (M <= 4) ? 2048 : 1024;
    constexpr int RO = (EPI == EPI_SWIGLU) ? R / 2 : R;   // outputs per wave
    __shared__ __attribute__((aligned(16))) float xs[M][KC];
    __shared__ float zs[16][SB_MAX_W];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const WT* __restrict__ W = reinterpret_cast<const WT*>(a.W);
    const int N = a.N, K = a.K;
    const int n0 = blockIdx.x * 4 * RO;
    const int total_rows = (EPI == EPI_SWIGLU) ? 2 * N : N;

    int outn[R];
    const WT* wrow[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int n, row;
        if (EPI == EPI_SWIGLU) {
            n = n0 + wave * RO + r % RO;
            row = (r < RO) ? n : N + n;
        } else {
            n = n0 + wave * R + r;
            row = n;
        }
        outn[r] = n;
        if (row > total_rows - 1) row = total_rows - 1;  // loads stay inside W; the result is dropped
        wrow[r] = W + (size_t)row * K;
    }

    float acc[R][M];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int m = 0; m < M; ++m) acc[r][m] = 0.f;

    auto madd = [&](const float (&w)[R][8], int kk) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            float4 xa = *reinterpret_cast<const float4*>(&xs[m][kk]);
            float4 xb = *reinterpret_cast<const float4*>(&xs[m][kk + 4]);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float s = acc[r][m];
                s = fmaf(w[r][0], xa.x, s); s = fmaf(w[r][1], xa.y, s);
                s = fmaf(w[r][2], xa.z, s); s = fmaf(w[r][3], xa.w, s);
                s = fmaf(w[r][4], xb.x, s); s = fmaf(w[r][5], xb.y, s);
                s = fmaf(w[r][6], xb.z, s); s = fmaf(w[r][7], xb.w, s);
                acc[r][m] = s;
            }
        }
    };
    // (the residual's element is requested with the first weights, not after the last)
    float pre_y = 0.f;
    if constexpr (EPI == EPI_RESID)
        if (lane < R * M && n0 + wave * R + lane / M < N) pre_y = a.out.y[(size_t)(lane % M) * a.out.ldy + n0 + wave * R + lane / M];
    for (int k0 = 0; k0 < K; k0 += KC) {   // (SHORT: one chunk)
        const int kc = (K - k0 < KC) ? (K - k0) : KC;
        Piece8<WT> w0[R], w1[R];   // (SHORT)
        const bool live0 = lane * 8 < kc, live1 = lane * 8 + 512 < kc;
        // rows: all loads before the first store (a loop of load and store would be one round trip after the other)
        float4 v[M][KC / 1024];
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int i = 0; i < KC / 1024; ++i) {
                const int kk = i * 1024 + tid * 4;
                v[m][i] = kk < kc ? *reinterpret_cast<const float4*>(a.x + (size_t)m * K + k0 + kk) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        if (SHORT) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (live0) w0[r].load(wrow[r] + lane * 8);
                if (live1) w1[r].load(wrow[r] + lane * 8 + 512);
            }
        }
        if (SHORT && a.norm_gain) {
            const float4 g = tid * 4 < K ? *reinterpret_cast<const float4*>(a.norm_gain + tid * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const float4 q = v[m][0];
                const float ss = wave_sum((q.x * q.x + q.y * q.y) + (q.z * q.z + q.w * q.w));
                if (lane == 0) zs[wave][m] = ss;
            }
            __syncthreads();
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const float inv = 1.0f / sqrtf((((zs[0][m] + zs[1][m]) + zs[2][m]) + zs[3][m]) / (float)K + a.eps);
                const float4 q = v[m][0];
                v[m][0] = make_float4(q.x * inv * g.x, q.y * inv * g.y, q.z * inv * g.z, q.w * inv * g.w);
            }
        }
        if (!SHORT) __syncthreads();   // (the last chunk's rows have been read)
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int i = 0; i < KC / 1024; ++i) {
                const int kk = i * 1024 + tid * 4;
                if (kk < kc) *reinterpret_cast<float4*>(&xs[m][kk]) = v[m][i];
            }
        __syncthreads();
        if (SHORT) {
            float w[R][8];
            if (live0) {
#pragma unroll
                for (int r = 0; r < R; ++r) w0[r].unpack(w[r]);
                madd(w, lane * 8);
            }
            if (live1) {
#pragma unroll
                for (int r = 0; r < R; ++r) w1[r].unpack(w[r]);
                madd(w, lane * 8 + 512);
            }
        } else {
#pragma unroll 2
            for (int kk = lane * 8; kk < kc; kk += 512) {
                float w[R][8];
#pragma unroll
                for (int r = 0; r < R; ++r) load8(wrow[r] + k0 + kk, w[r]);
                madd(w, kk);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int m = 0; m < M; ++m) acc[r][m] = wave_sum(acc[r][m]);

    if constexpr (EPI == EPI_STORE || EPI == EPI_RESID) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (lane == r * M + m && outn[r] < N) {
                    float* yp = a.out.y + (size_t)m * a.out.ldy + outn[r];
                    *yp = (EPI == EPI_RESID) ? (pre_y + acc[r][m]) : acc[r][m];
                }
    } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
        for (int j = 0; j < RO; ++j)
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (lane == j * M + m && outn[j] < N)
                    a.out.y[(size_t)m * a.out.ldy + outn[j]] = silu_mul(acc[j][m], acc[RO + j][m]);
    } else {  // EPI_HEAD
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (lane == r * M + m) zs[wave * R + r][m] = acc[r][m];
        __syncthreads();
        head_partial<16>(a.out, zs, (1u << M) - 1u, n0, N, gridDim.x);
    }
}

int head_blocks_valu(int32_t N) { return (N + 15) / 16; }

// Weight rows per wave: one (gate / up: a pair), so that a small matrix has four (two) times the blocks, or four, so that a block's rows
// are staged for four times the weights.  One while four would leave CUs without a block, and beyond that while a block
// stages no more bytes than it reads of the weights, up to four blocks a CU where K is long enough for more blocks to pay and two
// else (gate / up, whose waves keep a pair, gains at K = 256 as well: [2 * 8000 x 256] bf16, one row, 1.07x).
// Four / one, in us: fp32 [256 x 688], one row 3.7 / 2.5, four 6.2 / 3.5, eight 9.6 / 4.0; bf16 [4000 x 4096], eight 17.4 / 16.9;
// one row, bf16 [6144 x 4096] 12.7 / 11.7, [12288 x 4096] 21.4 / 20.4, [6144 x 256] 1.07x, fp32 [12288 x 1024] 10.8 / 10.1, [16000 x 4096]
// 51.4 / 46.2, four 54.6 / 46.5; but bf16 [6144 x 4096], eight 19.7 / 24.7, [12288 x 4096], four 25.0 / 28.5, and one row of
// [12288 x 256] bf16 4.0 / 4.3, fp32 5.0 / 5.3.  A row's sums are the same either way.
template <typename WT, int M, bool SHORT>
static hipError_t launch_gemv_valu_m(const GemvArgs& a, hipStream_t st) {
    const int n = a.epi == EPI_SWIGLU ? 2 * a.N : a.N;
    const bool few = n < 16 * 256 || (M <= (int)sizeof(WT) && n < 16 * (a.K >= 1024 || a.epi == EPI_SWIGLU ? 1024 : 512));
    const auto go = [&](auto epi_c, auto r_c) {   // (r: weight rows of a wave)
        constexpr int EPI = decltype(epi_c)::value, R = decltype(r_c)::value, RB = 4 * (EPI == EPI_SWIGLU ? R / 2 : R);
        return launch(&gemv_valu_kernel<WT, M, EPI, SHORT, R>, dim3((a.N + RB - 1) / RB), 256, st, valu_args<EPI>(a));
    };
    using std::integral_constant;
    using Four = integral_constant<int, 4>;
    switch (a.epi) {
        case EPI_STORE: return few ? go(integral_constant<int, EPI_STORE>{}, integral_constant<int, 1>{}) : go(integral_constant<int, EPI_STORE>{}, Four{});
        case EPI_RESID: return few ? go(integral_constant<int, EPI_RESID>{}, integral_constant<int, 1>{}) : go(integral_constant<int, EPI_RESID>{}, Four{});
        case EPI_SWIGLU: return few ? go(integral_constant<int, EPI_SWIGLU>{}, integral_constant<int, 2>{}) : go(integral_constant<int, EPI_SWIGLU>{}, Four{});
        case EPI_HEAD: {
            const hipError_t e = go(integral_constant<int, EPI_HEAD>{}, Four{});
            return e != hipSuccess ? e : launch_head_merge(a.head, M, head_blocks_valu(a.N), st);
        }
        default: return hipErrorInvalidValue;
    }
}
template <typename WT>
static hipError_t launch_gemv_valu_t(const GemvArgs& a, hipStream_t st) {
    switch (a.M) {
        case 1: return a.K <= SB_VALU_NORM_K ? launch_gemv_valu_m<WT, 1, true>(a, st) : launch_gemv_valu_m<WT, 1, false>(a, st);
        case 2: return a.K <= SB_VALU_NORM_K ? launch_gemv_valu_m<WT, 2, true>(a, st) : launch_gemv_valu_m<WT, 2, false>(a, st);
        case 3: return a.K <= SB_VALU_NORM_K ? launch_gemv_valu_m<WT, 3, true>(a, st) : launch_gemv_valu_m<WT, 3, false>(a, st);
        case 4: return a.K <= SB_VALU_NORM_K ? launch_gemv_valu_m<WT, 4, true>(a, st) : launch_gemv_valu_m<WT, 4, false>(a, st);
        case 5: return a.K <= SB_VALU_NORM_K ? launch_gemv_valu_m<WT, 5, true>(a, st) : launch_gemv_valu_m<WT, 5, false>(a, st);
        case 6: return a.K <= SB_VALU_NORM_K ? launch_gemv_valu_m<WT, 6, true>(a, st) : launch_gemv_valu_m<WT, 6, false>(a, st);
        case 7: return a.K <= SB_VALU_NORM_K ? launch_gemv_valu_m<WT, 7, true>(a, st) : launch_gemv_valu_m<WT, 7, false>(a, st);
        case 8: return a.K <= SB_VALU_NORM_K ? launch_gemv_valu_m<WT, 8, true>(a, st) : launch_gemv_valu_m<WT, 8, false>(a, st);
        default: return hipErrorInvalidValue;
    }
}
hipError_t launch_gemv_valu(const GemvArgs& a, hipStream_t st) {
    if (a.K % 8 != 0 || a.N < 1 || (a.norm_gain && a.K > SB_VALU_NORM_K)) return hipErrorInvalidValue;
    return a.w_dtype == SB_BF16 ? launch_gemv_valu_t<uint16_t>(a, st) : launch_gemv_valu_t<float>(a, st);
}

// ---------------------------------------------------------------- GEMV, MFMA tiles
// bf16 weights only.  The M <= 8 activation rows are given as two bf16 parts each
// (x ~= hi + lo, 16 bits of mantissa), laid out as the 16 columns of one
// 16x16x32 MFMA B operand: columns 0-7 high parts, 8-15 low parts.  A 16-row
// tile of W is the A operand, read straight from HBM with 128-bit loads: the four
// lanes (i, q = 0..3) of row i read 64 contiguous bytes per instruction, 256 bytes
// per 128-wide k block.
// The four waves of a block take k blocks round-robin and are summed through LDS
// in wave order.  Products of bf16 values are exact in fp32, so the only rounding
// is fp32 accumulation.  Columns never mix, hence row results do not depend on M.
//
// PACKED: the weights were re-laid out once (repack_kernel) so that what a wave
// loads is contiguous: per 16-row tile and 128-wide k block one 4 KB unit, in it
// 1 KB per MFMA step holding lane l's 16 bytes at l * 16.  Every load instruction
// then reads 1 KB of consecutive memory (whole cache lines, so a streaming hint is
// safe) and a block walks one contiguous slab.  Same values in the same MFMA slots
// as the row-major path: results are bit-identical.
// Element offset of lane group lq's share of MFMA step u inside a 128-wide k block:
// one load instruction then covers 64 contiguous bytes of each of the 16 rows (the
// k order inside a block is free as long as A and B use the same one).
#define SB_KOFF(lq, u) ((u) * 32 + (lq) * 8)
// W [N][K] row-major -> packed tiles (N % 16 == 0, K % 128 == 0); one thread moves 16 bytes.
__global__ __launch_bounds__(256) void repack_kernel(const uint16_t* __restrict__ W, uint16_t* __restrict__ P, int N,
                                                     int K) {
    const int KB = K >> 7;
    const size_t unit = (size_t)blockIdx.x * 256 + threadIdx.x;  // 16-byte unit of the packed array
    const size_t n_units = (size_t)N * K / 8;
    if (unit >= n_units) return;
    const int l = (int)(unit & 63), u = (int)((unit >> 6) & 3);
    const size_t blk = unit >> 8;  // (tile, k block)
    const int kb = (int)(blk % KB);
    const size_t tile = blk / KB;
    const int i = l & 15, q = l >> 4;
    const uint4 v = *reinterpret_cast<const uint4*>(W + (tile * 16 + i) * (size_t)K + (size_t)kb * 128 + SB_KOFF(q, u));
    *reinterpret_cast<uint4*>(P + unit * 8) = v;
}
hipError_t launch_repack(const void* W, void* P, int32_t N, int32_t K, hipStream_t st) {
    if (N % 16 || K % 128 || N < 16 || K < 128) return hipErrorInvalidValue;
    const size_t n_units = (size_t)N * K / 8;
    return launch(&repack_kernel, dim3((unsigned)((n_units + 255) / 256)), 256, st, (const uint16_t*)W, (uint16_t*)P, N, K);
}

// RAW: the rows come as floats and every block makes the two bf16 parts of what it multiplies by itself: the same
// bytes through L2 and the same registers (the lanes of a row's high and low column load four of its eight floats each
// and exchange parts), some 80 vector instructions per k block, and no launch before this one.
// [6144 x 4096], one row: 13.6 -> 10.6 us with the launch it saves, [27648 x 5120], six rows: 49.4 -> 48.5.
template <int RT, int EPI, int WPB, int DEPTH, bool PACKED, bool RAW>
__global__ __launch_bounds__(64 * WPB) void gemv_mfma_kernel(MfmaArgs<EPI> a) {
    constexpr int NT = 64 * WPB;
    static_assert(NT >= (EPI == EPI_SWIGLU ? RT / 2 : RT) * 128, "the tails take one element per thread");
    __shared__ __attribute__((aligned(16))) float red[WPB][RT][64][4];
    __shared__ float cs[RT][16][17];
    __shared__ float zs[16 * RT][SB_MAX_W];
    __shared__ float s_inv[SB_MAX_W];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lq = lane >> 4;
    const uint16_t* __restrict__ W = reinterpret_cast<const uint16_t*>(a.W);
    const int N = a.N, K = a.K, M = a.M;
    const int KB = K >> 7;  // k blocks of 128
    constexpr int OT = (EPI == EPI_SWIGLU) ? RT / 2 : RT;   // 16-output tiles of the block (gate / up: the gate tiles, then their up tiles)
    const int n0 = blockIdx.x * 16 * OT;

    const uint16_t* wp[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        int row0 = (EPI == EPI_SWIGLU) ? (t < OT ? n0 + t * 16 : N + n0 + (t - OT) * 16) : (n0 + t * 16);  // first row of the tile
        int total = (EPI == EPI_SWIGLU) ? 2 * N : N;
        if (PACKED) {
            if (row0 > total - 16) row0 = total - 16;
            wp[t] = W + (size_t)(row0 >> 4) * KB * 2048 + lane * 8;
        } else {
            int row = row0 + li;
            if (row > total - 1) row = total - 1;
            wp[t] = W + (size_t)row * K;
        }
    }
    // Rows of this launch: the first M slots, or (passes that gather the rows of several
    // sequences) the slots of a bit mask.  Lanes whose column is a row that is not there load nothing.
    const uint32_t rows = a.row_mask ? a.row_mask : ((1u << M) - 1u);
    const bool bact = (rows >> (li & 7)) & 1u;
    const uint16_t* bp = reinterpret_cast<const uint16_t*>(a.x) + (size_t)li * K;
    const float* xp = reinterpret_cast<const float*>(a.x) + (size_t)(li & 7) * K + (li >> 3) * 4;   // (RAW)

    f32x4 acc[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // Ring of DEPTH register buffers, DEPTH - 1 k blocks in flight per wave.  The
    // stage loop is fully unrolled, so every buffer index is a compile-time constant.
    uint4 wbuf[DEPTH][RT][4], bbuf[DEPTH][4];
    // k block index is clamped instead of tested: what the ring's first loads ask for past the end of a short K
    // is the last block again (unused).
    auto load_block = [&](uint4 (&wr)[RT][4], uint4 (&br)[4], int kb) {
        const int kc = kb < KB ? kb : KB - 1;
        const size_t off = (size_t)kc * 128;
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                wr[t][u] = PACKED ? ld_weights_packed(wp[t] + (size_t)kc * 2048 + u * 512)
                                  : *reinterpret_cast<const uint4*>(wp[t] + off + SB_KOFF(lq, u));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (RAW) br[u] = bact ? *reinterpret_cast<const uint4*>(xp + off + SB_KOFF(lq, u)) : make_uint4(0, 0, 0, 0);
            else br[u] = bact ? *reinterpret_cast<const uint4*>(bp + off + SB_KOFF(lq, u)) : make_uint4(0, 0, 0, 0);
        }
    };
    auto mma_block = [&](const uint4 (&wr)[RT][4], const uint4 (&br)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bf16x8 bv = __builtin_bit_cast(bf16x8, br[u]);
            if (RAW) {   // columns 0-7: high parts, floats 0-3 here, 4-7 in the lane 8 further; columns 8-15: low parts
                uint32_t h0, h1, l0, l1, r0, r1, t;
                split_pair(br[u].x, br[u].y, h0, l0);
                split_pair(br[u].z, br[u].w, h1, l1);
                const bool low = li >= 8;
                lane_pair<8>(low ? h0 : l0, t, r0);
                lane_pair<8>(low ? h1 : l1, t, r1);
                bv = __builtin_bit_cast(bf16x8, make_uint4(low ? r0 : h0, low ? r1 : h1, low ? l0 : r0, low ? l1 : r1));
            }
#pragma unroll
            for (int t = 0; t < RT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr[t][u]), bv, acc[t],
                                                                 0, 0, 0);
        }
    };
    const int kb0 = wave;
    const int nkb = KB > wave ? (KB - wave + WPB - 1) / WPB : 0;  // k blocks of this wave
    // The rows' partial sums of squares are requested before the weights: loads come back in order, and behind them these were waited for with
    // the ring's first two blocks of every wave, 25 MB at the 7B shape's QKV, before the next was asked for ([12288 x 4096], one / six rows 18.25 / 20.3 -> 17.25 / 19.7 us,
    // [22016 x 4096] gate and up 28.0 / 30.7 -> 27.6 / 30.0, [6144 x 4096] one row 11.6 -> 11.2).
    constexpr int SQ_ROWS = SB_MAX_W / WPB, SQ_U = 8;   // rows per wave; values per lane up to K = 8192
    float sq[SQ_ROWS][SQ_U];
    const auto sq_row = [&](int i) { return wave + i * WPB; };
    if (a.ssq_in)
#pragma unroll
        for (int i = 0; i < SQ_ROWS; ++i)
            if ((rows >> sq_row(i)) & 1u) {   // (wave-uniform, as the bounds below)
                const float* const p = a.ssq_in + (size_t)sq_row(i) * a.ssq_ld;
#pragma unroll
                for (int u = 0; u < SQ_U; ++u)
                    if (u * 64 < a.ssq_nb) sq[i][u] = p[u * 64 + lane < a.ssq_nb ? u * 64 + lane : 0];
            }
#pragma unroll
    for (int s = 0; s < DEPTH - 1; ++s) load_block(wbuf[s], bbuf[s], kb0 + s * WPB);
    // What the residual tail needs from memory (the element this thread finishes, its norm gains)
    // is requested now, behind the first weight loads, instead of at the end of the k loop.
    float pre_y = 0.f, pre_gA = 0.f, pre_gB = 0.f;
    if constexpr (EPI == EPI_RESID) {
        if (tid < RT * 16 * 8) {
            const int t = tid >> 7, m = (tid >> 4) & 7, i = tid & 15, n = n0 + t * 16 + i;
            if (((rows >> m) & 1u) && n < N) {
                pre_y = a.out.y[(size_t)m * a.out.ldy + n];
                if (a.out.nxA) pre_gA = a.out.gainA[n];
                if (a.out.nxB) pre_gB = a.out.gainB[n];
            }
        }
    }
    // RMSNorm scale of each row from the partial sums of squares its producer left
    // (added in index order; the first weight loads are in flight)
    if (a.ssq_in) {
#pragma unroll
        for (int i = 0; i < SQ_ROWS; ++i) {
            const int m = sq_row(i);
            if (!((rows >> m) & 1u)) continue;
            float t = 0.f;
#pragma unroll
            for (int u = 0; u < SQ_U; ++u)
                if (u * 64 < a.ssq_nb) t += u * 64 + lane < a.ssq_nb ? sq[i][u] : 0.f;
            for (int b = lane + SQ_U * 64; b < a.ssq_nb; b += 64) t += a.ssq_in[(size_t)m * a.ssq_ld + b];
            t = wave_sum(t);
            if (lane == 0) s_inv[m] = 1.0f / sqrtf(t / (float)K + a.eps);
        }
    } else if (tid < SB_MAX_W) {
        s_inv[tid] = 1.0f;
    }
    int it = 0;
    for (; it + 2 * DEPTH - 1 <= nkb; it += DEPTH) {  // steady state: before it, buf[s] holds block it + s (s < DEPTH-1)
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            load_block(wbuf[(s + DEPTH - 1) % DEPTH], bbuf[(s + DEPTH - 1) % DEPTH], kb0 + (it + s + DEPTH - 1) * WPB);
            mma_block(wbuf[s], bbuf[s]);
        }
    }
    // The last blocks, at most 2 DEPTH - 2, a form for each count: nothing is requested past the end, and every wait is exact.  One round more, with the
    // last block read again for those that are not there, cost one or two blocks of a wave's four to thirty: [4096 x 4096] one / six rows
    // 7.6 / 9.7 -> 7.3 / 9.1 us, [15360 x 5120] four 27.5 -> 26.4, [27648 x 5120] gate and up 44.9 -> 43.2, [5120 x 13824] 28.1 -> 27.1.
    const auto finish = [&](auto left) {
        constexpr int L = decltype(left)::value;
#pragma unroll
        for (int s = 0; s < L; ++s) {
            if (s + DEPTH - 1 < L) load_block(wbuf[(s + DEPTH - 1) % DEPTH], bbuf[(s + DEPTH - 1) % DEPTH], kb0 + (it + s + DEPTH - 1) * WPB);
            mma_block(wbuf[s % DEPTH], bbuf[s % DEPTH]);
        }
    };
    using std::integral_constant;
    switch (nkb - it) {
        case 1: finish(integral_constant<int, 1>{}); break;
        case 2: finish(integral_constant<int, 2>{}); break;
        case 3: if constexpr (DEPTH > 2) finish(integral_constant<int, 3>{}); break;
        case 4: if constexpr (DEPTH > 2) finish(integral_constant<int, 4>{}); break;
        default: break;
    }
    static_assert(DEPTH == 2 || DEPTH == 3, "two or four blocks are left at most");
#pragma unroll
    for (int t = 0; t < RT; ++t) *reinterpret_cast<f32x4*>(&red[wave][t][lane][0]) = acc[t];
    __syncthreads();
    // C layout of the 16x16 tile: lane (j = l%16, g = l/16), register r -> row 4g + r, column j.
    for (int e = tid; e < RT * 256; e += NT) {
        int t = e >> 8, l = (e >> 2) & 63, r = e & 3;
        float v = red[0][t][l][r];
#pragma unroll
        for (int w = 1; w < WPB; ++w) v += red[w][t][l][r];
        cs[t][4 * (l >> 4) + r][l & 15] = v;
    }
    __syncthreads();

    if constexpr (EPI == EPI_STORE || EPI == EPI_RESID) {
        for (int e = tid; e < RT * 16 * 8; e += NT) {
            int t = e >> 7, m = (e >> 4) & 7, i = e & 15;
            int n = n0 + t * 16 + i;
            float sq = 0.f;
            if (((rows >> m) & 1u) && n < N) {
                float v = (cs[t][i][m] + cs[t][i][m + 8]) * s_inv[m];
                float* yp = a.out.y + (size_t)m * a.out.ldy + n;
                if (EPI == EPI_RESID) v += pre_y;   // (e == tid: a block has at least RT * 128 threads)
                *yp = v;
                if constexpr (EPI == EPI_RESID) {
                    if (a.out.nxA) split_store(a.out.nxA, a.out.ldy, m, n, v * pre_gA);
                    if (a.out.nxB) split_store(a.out.nxB, a.out.ldy, m, n, v * pre_gB);
                    sq = v * v;
                }
            }
            if (EPI == EPI_RESID) zs[t * 16 + i][m] = sq;
        }
        if constexpr (EPI == EPI_RESID) {
            if (a.out.ssq_out) {  // sum of squares of each 16-row tile, rows in index order
                __syncthreads();
                if (tid < RT * 8) {
                    int t = tid >> 3, m = tid & 7;
                    if (((rows >> m) & 1u) && n0 + t * 16 < N) {
                        float sum = 0.f;
                        for (int i = 0; i < 16; ++i) sum += zs[t * 16 + i][m];
                        a.out.ssq_out[(size_t)m * a.ssq_ld + blockIdx.x * RT + t] = sum;
                        if (a.out.ssq_out2) a.out.ssq_out2[(size_t)m * a.ssq_ld + blockIdx.x * RT + t] = sum;
                    }
                }
            }
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
        if (tid < OT * 128) {
            int t = tid >> 7, m = (tid >> 4) & 7, i = tid & 15;
            int n = n0 + t * 16 + i;
            if (((rows >> m) & 1u) && n < N) {
                float g = (cs[t][i][m] + cs[t][i][m + 8]) * s_inv[m];
                float u = (cs[OT + t][i][m] + cs[OT + t][i][m + 8]) * s_inv[m];
                float v = silu_mul(g, u);
                if (a.out.y) a.out.y[(size_t)m * a.out.ldy + n] = v;
                if (a.out.ys) split_store(a.out.ys, a.out.ldy, m, n, v);
            }
        }
    } else if constexpr (EPI == EPI_HEAD) {
        for (int e = tid; e < RT * 16 * 8; e += NT) {
            int t = e >> 7, m = (e >> 4) & 7, i = e & 15;
            zs[t * 16 + i][m] = (cs[t][i][m] + cs[t][i][m + 8]) * (((rows >> m) & 1u) ? s_inv[m] : 0.f);
        }
        __syncthreads();
        head_partial<16 * RT>(a.out, zs, rows, n0, N, gridDim.x);
    }
}

// Row tiles and waves of a block.  The waves (the order in which a row's products are added) are fixed by the number of output rows
// alone: eight up to 4096, four above.  The tiles follow the rows too.  What counts first is that no CU has more tiles than the others
// (256 CUs):
//   up to 256 tiles   a tile per block, eight waves splitting K, a ring of two (a deeper one only costs occupancy)
//   up to 512         a CU with two tiles sets the time; as one block they read the rows once, not twice, which pays with several rows, fewer
//                     of them where only some CUs have a second tile, and a K long enough for the start. One / two tiles per block at
//                     three, four and eight rows: [5120 x 5120] 13.5 / 12.7, 14.3 / 12.8 and 17.5 / 14.1 us, [6144 x 4096] 1.02, 1.07 and 1.18x,
//                     [5120 x 2048] 1.02, 1.04 and 1.15x, [5120 x 1024] 0.96, 0.98 and 1.03x; [8192 x 4096] 0.97, 1.00 and 1.13x, [8192 x 8192]
//                     22.0 / 23.3, 22.6 / 22.7 and 26.2 / 22.9. One row: [5120 x 13824] 29.8 / 28.2, [5120 x 10240] 22.5 / 21.9, [4224 x 6144]
//                     14.5 / 15.0, [8192 x 5120] 14.7 / 15.7, row-major [5120 x 5120] 16.9 / 18.1. (Row-major
//                     [8192 x 8192], rows 16 KB apart, is slower at five rows, 29.7 / 34.8; 8192 x 4224, 5120 and 13824 gain.) Eight waves on two tiles would take 10.5 /
//                     11.6 / 13.3 at one, four and eight rows of [5120 x 5120], 26.2 / 29.8 / 35.4 of [5120 x 13824], in another order of additions
//   up to 768         a tile per block, three blocks per CU ([12288 x 4096], four rows: 18.6, two tiles 23.8)
//   more              two tiles (row-major weights, few rows and short K: one, [13312 x 4096] 24.2 and 25.9)
struct MfmaShape { int rt, wpb; };
static int mfma_rows(const GemvArgs& a) { return a.row_mask ? __builtin_popcount(a.row_mask) : a.M; }
static MfmaShape mfma_shape(const GemvArgs& a) {
    const int rows = mfma_rows(a);
    if (a.N <= 4096) return {1, 8};
    if (a.N <= 6144) return {(rows >= 3 && a.K >= 2048) || (a.packed && a.K > 8192) ? 2 : 1, 4};
    if (a.N <= 8192) return {rows >= 5 && a.K >= 2048 ? 2 : 1, 4};
    if (a.N <= 12288) return {1, 4};
    return {a.K > 4096 || a.packed || rows >= 3 ? 2 : 1, 4};
}
// Heads, and gate / up with its pair of tiles, keep four waves: [32000 x 4096] 46.7 us, with eight 49.6; [2 * 11008 x 4096] 30.3 and 31.9.
static int mfma_row_tiles(int32_t N) { return N >= 15000 ? 2 : 1; }   // (heads)
static int mfma_waves(int32_t N) { return N <= 4096 ? 8 : 4; }
int head_blocks_mfma(int32_t N) { return (N + 16 * mfma_row_tiles(N) - 1) / (16 * mfma_row_tiles(N)); }

template <int EPI, bool PACKED, bool RAW = false>
static hipError_t launch_gemv_mfma_e(const GemvArgs& a, hipStream_t st) {
    if constexpr (!RAW && EPI != EPI_RESID)
        if (!a.xs) return launch_gemv_mfma_e<EPI, PACKED, true>(a, st);
    const MfmaArgs<EPI> m = mfma_args<EPI, RAW>(a);
    if constexpr (EPI == EPI_SWIGLU) {
        const int pairs = a.N / 16;
        // Four tiles (two pairs) read the rows half as often; two blocks of them fit on a CU, so up to 1024 pairs, and only where
        // one pair per block would give a CU more than three, with K long enough and three rows or more. Two / four tiles at K = 5120:
        // 688 pairs, six rows 39.9 / 46.0 us; 769, three / six / eight rows 45.1 / 43.2, 46.9 / 44.6, 49.1 / 45.6; 816 47.5 / 45.5, 49.4 /
        // 47.0, 51.6 / 48.2; 864 49.2 / 45.6, 50.6 / 46.5, 52.8 / 47.5, one row 45.5 and 46.4; 1024 52.8 / 52.3, 54.4 / 53.5, 56.5 / 52.8;
        // 1040, six rows 61.0 / 65.5. K = 4096: 896 pairs, three rows 38.9 and 39.5, row-major weights 47.4 and 50.4.
        if constexpr (PACKED)
            if (a.K > 4096 && mfma_rows(a) >= 3 && pairs > 768 && pairs <= 1024)
                return launch(&gemv_mfma_kernel<4, EPI, 4, 2, PACKED, RAW>, dim3((pairs + 1) / 2), 256, st, m);
        return launch(&gemv_mfma_kernel<2, EPI, 4, 3, PACKED, RAW>, dim3(pairs), 256, st, m);
    } else {
        const MfmaShape sh = EPI == EPI_HEAD ? MfmaShape{mfma_row_tiles(a.N), mfma_waves(a.N)} : mfma_shape(a);
        const int one = a.N / 16, two = (a.N + 31) / 32;
        if (sh.rt == 1 && sh.wpb == 8) return launch(&gemv_mfma_kernel<1, EPI, 8, 2, PACKED, RAW>, dim3(one), 512, st, m);
        if (sh.rt == 1) return launch(&gemv_mfma_kernel<1, EPI, 4, 3, PACKED, RAW>, dim3(one), 256, st, m);
        return launch(&gemv_mfma_kernel<2, EPI, 4, 3, PACKED, RAW>, dim3(two), 256, st, m);
    }
}

hipError_t launch_gemv_mfma(const GemvArgs& a, hipStream_t st) {
    if (a.w_dtype != SB_BF16 || a.K % 128 != 0 || a.N % 16 != 0 || a.M < 1 || a.M > 8 || (!a.xs && (!a.x || a.epi == EPI_RESID)))
        return hipErrorInvalidValue;
    switch (a.epi) {
        case EPI_STORE: return a.packed ? launch_gemv_mfma_e<EPI_STORE, true>(a, st) : launch_gemv_mfma_e<EPI_STORE, false>(a, st);
        case EPI_RESID: return a.packed ? launch_gemv_mfma_e<EPI_RESID, true>(a, st) : launch_gemv_mfma_e<EPI_RESID, false>(a, st);
        case EPI_SWIGLU: return a.packed ? launch_gemv_mfma_e<EPI_SWIGLU, true>(a, st) : launch_gemv_mfma_e<EPI_SWIGLU, false>(a, st);
        case EPI_HEAD: {
            const hipError_t e = a.packed ? launch_gemv_mfma_e<EPI_HEAD, true>(a, st) : launch_gemv_mfma_e<EPI_HEAD, false>(a, st);
            if (e != hipSuccess || a.head.skip_merge) return e;
            return launch_head_merge(a.head, a.M, head_blocks_mfma(a.N), st);
        }
        default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------- head evaluation without a workspace
// For callers that cannot allocate device memory (code under graph capture, tight serving
// loops): the head partials of a single head evaluation live in a file-scope device array instead of a caller's scratch buffer.  Each GPU holds its own copy
// of the array at its own address, looked up once per device; every call on a GPU shares it,
// so calls that overlap on one GPU race.  Nothing in it has to start at zero: every element a
// launch reads was written by that launch sequence (partials of all blocks of rows < M).
static __device__ __align__(256) unsigned char scratch[SB_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each GPU, once looked up
std::mutex g_scratch_mu;
}  // namespace

hipError_t static_scratch(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // the array's address on the current device
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace sb
