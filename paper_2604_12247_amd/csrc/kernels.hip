// gfx950 kernels of the bounded self-speculative decode step: embedding, RMSNorm, operand split, the
// merge stage of a head evaluation, sampling-mode acceptance, bandwidth yardsticks.  The projections
// are in gemv.hip, attention in attention.hip, the prompt pass in prefill.hip.
//
// Every kernel here is written so that the value computed for one token row
// depends only on that row's inputs, its absolute position and the operand
// shapes -- never on how many other rows share the launch.  That is what makes a
// row verified in a pass of M rows bit-identical to the same row decoded alone,
// and hence speculative output identical to greedy decoding by the same library
// (the exactness property of Sec. 3.3).
#include "kernels.h"
#include "device_utils.h"

#include <math.h>
#include <mutex>

namespace sb {

// ---------------------------------------------------------------- embedding
// Row r of the hidden cache := embedding of token `tok` (+ what the first layer's projection
// needs: bf16 parts of gain * h and the row's sum of squares).  Executed by the first 256
// threads of a block, which all reach the barrier inside; the same code serves the embedding
// kernel and the head merge that embeds the token it has just drafted, so a row's values do
// not depend on which of the two wrote it.
template <typename WT>
__device__ __forceinline__ void embed_row(const WT* __restrict__ E, int vocab, int d, float* __restrict__ H, int tok, int r,
                                          EmbedNorm en, float* red /*[4] shared*/) {
    constexpr int VMAX = 4;  // 8-element groups a thread keeps in registers (covers d <= 8192)
    const int tid = threadIdx.x;
    const bool act = tid < 256;
    if (tok < 0 || tok >= vocab) tok = 0;  // never index outside the table
    const WT* e = E + (size_t)tok * d;
    const int ngrp = d >> 3;
    float ss = 0.f;
    if (act) {
        float v[VMAX][8], gn[VMAX][8];
#pragma unroll
        for (int j = 0; j < VMAX; ++j) {
            const int gi = tid + j * 256;
            if (gi < ngrp) {
                load8(e + gi * 8, v[j]);
                if (en.nx) load8(en.gain + gi * 8, gn[j]);
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) v[j][k] = 0.f;
            }
        }
#pragma unroll
        for (int j = 0; j < VMAX; ++j) {
            const int gi = tid + j * 256;
            if (gi < ngrp) {
                store8_split(v[j], gn[j], H + (size_t)r * d + gi * 8, en.nx, (size_t)r * d + gi * 8, (size_t)(8 + r) * d + gi * 8);
#pragma unroll
                for (int k = 0; k < 8; ++k) ss += v[j][k] * v[j][k];
            }
        }
        for (int i = VMAX * 2048 + tid; i < d; i += 256) {  // d > 8192
            float x = ldf(e + i);
            H[(size_t)r * d + i] = x;
            ss += x * x;
            if (en.nx) split_store(en.nx, d, r, i, x * en.gain[i]);
        }
    }
    if (en.ssq_out) {  // the row's sum of squares, as a single partial
        ss = wave_sum(ss);
        if (act && (tid & 63) == 0) red[tid >> 6] = ss;
        __syncthreads();
        if (tid == 0) en.ssq_out[(size_t)r * en.ssq_ld] = ((red[0] + red[1]) + red[2]) + red[3];
    }
}

template <typename WT>
__global__ __launch_bounds__(256) void embed_kernel(const WT* __restrict__ E, int vocab, int d, float* __restrict__ H,
                                                    RowToks toks, const int32_t* __restrict__ slot_tok,
                                                    int32_t* clear_flag, EmbedNorm en) {
    __shared__ float red[4];
    int r = blockIdx.x, tid = threadIdx.x;
    int tok = toks.tok[r];
    if (tok < 0) tok = slot_tok[r];
    if (clear_flag && r == 0 && tid == 0) *clear_flag = 0;
    embed_row<WT>(E, vocab, d, H, tok, r, en, red);
}

hipError_t launch_embed(const void* E, int32_t w_dtype, int32_t vocab, int32_t d, float* H, int32_t M,
                        RowToks toks, const int32_t* slot_tok, int32_t* clear_flag, EmbedNorm en, hipStream_t st) {
    if (w_dtype == SB_BF16) return launch(&embed_kernel<uint16_t>, dim3(M), 256, st, (const uint16_t*)E, vocab, d, H, toks, slot_tok, clear_flag, en);
    return launch(&embed_kernel<float>, dim3(M), 256, st, (const float*)E, vocab, d, H, toks, slot_tok, clear_flag, en);
}

// The same for one row each of n sequences.
template <typename WT>
__global__ __launch_bounds__(256) void embed_batch_kernel(const WT* __restrict__ E, int vocab, int d, EmbedBatch eb) {
    __shared__ float red[4];
    const EmbedRow r = eb.row[blockIdx.x];
    const int tok = r.tok < 0 ? *r.slot_tok : r.tok;
    if (r.exit_flag_to_clear && threadIdx.x == 0) *r.exit_flag_to_clear = 0;
    embed_row<WT>(E, vocab, d, r.H, tok, 0, r.en, red);
}
hipError_t launch_embed_batch(const void* E, int32_t w_dtype, int32_t vocab, int32_t d, const EmbedBatch& eb, int32_t n, hipStream_t st) {
    if (n < 1 || n > SB_MAX_W) return hipErrorInvalidValue;
    if (w_dtype == SB_BF16) return launch(&embed_batch_kernel<uint16_t>, dim3(n), 256, st, (const uint16_t*)E, vocab, d, eb);
    return launch(&embed_batch_kernel<float>, dim3(n), 256, st, (const float*)E, vocab, d, eb);
}

// ---------------------------------------------------------------- RMSNorm
// out = x / sqrt(mean(x^2) + eps) * gain, one block per row.
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* __restrict__ x, const float* __restrict__ gain,
                                                      float* __restrict__ out, uint16_t* __restrict__ outs, int lds,
                                                      int d, float eps) {
    constexpr int VMAX = 8;  // float4 values a thread keeps in registers (covers d <= 8192)
    __shared__ float red[4];
    const int r = blockIdx.x, tid = threadIdx.x;
    const int nvec = d >> 2;
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)r * d);
    const float4* g4 = reinterpret_cast<const float4*>(gain);
    float4 v[VMAX], g[VMAX];
    // all loads are issued before the first use: one memory round trip, not d/256
#pragma unroll
    for (int j = 0; j < VMAX; ++j) {
        int idx = tid + j * 256;
        v[j] = idx < nvec ? xr[idx] : make_float4(0.f, 0.f, 0.f, 0.f);
        g[j] = idx < nvec ? g4[idx] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < VMAX; ++j) ss += (v[j].x * v[j].x + v[j].y * v[j].y) + (v[j].z * v[j].z + v[j].w * v[j].w);
    for (int idx = tid + VMAX * 256; idx < nvec; idx += 256) {
        float4 t = xr[idx];
        ss += (t.x * t.x + t.y * t.y) + (t.z * t.z + t.w * t.w);
    }
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    const float tot = ((red[0] + red[1]) + red[2]) + red[3];
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
    auto emit = [&](int idx, float4 t, float4 gg) {
        float4 o = make_float4(t.x * inv * gg.x, t.y * inv * gg.y, t.z * inv * gg.z, t.w * inv * gg.w);
        if (out) reinterpret_cast<float4*>(out + (size_t)r * d)[idx] = o;
        if (outs) {
            uint16_t h0 = f2bf(o.x), h1 = f2bf(o.y), h2 = f2bf(o.z), h3 = f2bf(o.w);
            uint16_t l0 = f2bf(o.x - bf2f(h0)), l1 = f2bf(o.y - bf2f(h1)), l2 = f2bf(o.z - bf2f(h2)),
                     l3 = f2bf(o.w - bf2f(h3));
            uint2 hi = make_uint2((uint32_t)h0 | ((uint32_t)h1 << 16), (uint32_t)h2 | ((uint32_t)h3 << 16));
            uint2 lo = make_uint2((uint32_t)l0 | ((uint32_t)l1 << 16), (uint32_t)l2 | ((uint32_t)l3 << 16));
            *reinterpret_cast<uint2*>(outs + (size_t)r * lds + idx * 4) = hi;
            *reinterpret_cast<uint2*>(outs + (size_t)(8 + r) * lds + idx * 4) = lo;
        }
    };
#pragma unroll
    for (int j = 0; j < VMAX; ++j) {
        int idx = tid + j * 256;
        if (idx < nvec) emit(idx, v[j], g[j]);
    }
    for (int idx = tid + VMAX * 256; idx < nvec; idx += 256) emit(idx, xr[idx], g4[idx]);
}

hipError_t launch_rmsnorm(const float* x, const float* gain, float* out, uint16_t* out_split, int32_t ld_split,
                          int32_t M, int32_t d, float eps, hipStream_t st) {
    return launch(&rmsnorm_kernel, dim3(M), 256, st, x, gain, out, out_split, ld_split, d, eps);
}

__global__ void split_kernel(const float* __restrict__ x, uint16_t* __restrict__ xs, int K) {
    int m = blockIdx.y;
    int i = blockIdx.x * 256 + threadIdx.x;
    if (i < K) split_store(xs, K, m, i, x[(size_t)m * K + i]);
}
hipError_t launch_split(const float* x, uint16_t* xs, int32_t M, int32_t K, hipStream_t st) {
    return launch(&split_kernel, dim3((K + 255) / 256, M), 256, st, x, xs, K);
}

__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}
hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t st) {
    if (n == 0) return hipSuccess;
    fill_u32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(p, n, v);
    return hipGetLastError();
}

// ---------------------------------------------------------------- bandwidth yardsticks
__global__ __launch_bounds__(256) void copy_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src, size_t n) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * 256;
    for (; i < n; i += stride) dst[i] = src[i];
}
hipError_t launch_copy(void* dst, const void* src, size_t nbytes, hipStream_t st) {
    size_t n = nbytes / 16;
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    copy_kernel<<<(unsigned)blocks, 256, 0, st>>>((uint4*)dst, (const uint4*)src, n);
    return hipGetLastError();
}
__global__ __launch_bounds__(256) void read_kernel(const uint4* __restrict__ src, size_t n, float* sink) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * 256;
    uint32_t acc = 0;
    for (; i + 3 * stride < n; i += 4 * stride) {
        uint4 a = src[i], b = src[i + stride], c = src[i + 2 * stride], d = src[i + 3 * stride];
        acc ^= a.x ^ a.y ^ a.z ^ a.w ^ b.x ^ b.y ^ b.z ^ b.w ^ c.x ^ c.y ^ c.z ^ c.w ^ d.x ^ d.y ^ d.z ^ d.w;
    }
    for (; i < n; i += stride) { uint4 a = src[i]; acc ^= a.x ^ a.y ^ a.z ^ a.w; }
    if (acc == 0x9e3779b9u) *sink = 1.0f;  // practically never: keeps the loads alive
}
hipError_t launch_read(const void* src, size_t nbytes, float* sink, hipStream_t st) {
    size_t n = nbytes / 16;
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 1023) / 1024;
    if (blocks > 256 * 16) blocks = 256 * 16;
    read_kernel<<<(unsigned)blocks, 256, 0, st>>>((const uint4*)src, n, sink);
    return hipGetLastError();
}

// ---------------------------------------------------------------- head reduction
// Second stage of a head evaluation: one block merges the per-block partials
// (max, arg max, sum of exp((z - max)/T)) of every row in a fixed order -- so the
// result does not depend on block scheduling -- and carries out the exit test
// (Eq. 2) or the acceptance rule.  When a draft
// exits, the block also embeds the drafted token as the next row (the next draft step
// then starts at its first layer).  It is a kernel of its own: publishing the
// partials inside the projection kernel would need a device-wide fence per
// block, which on this chip writes back and invalidates a whole L2, or stores past it
// and a counter (one row of [1024 x 256] 5.6 -> 6.1 us, of [4096 x 256] 6.2 -> 8.6).
constexpr int MERGE_T = 1024;   // threads

// TPR threads a row, MERGE_T / TPR rows side by side; a thread holds U partials in registers from the
// search for the maximum to the sum, those past TPR * U are read again.  Every partial's sum is scaled once, from its own
// maximum to the row's, whatever either is: a NaN in a partial reaches the confidence, and so does a row without a
// finite logit.  A row's order of additions depends on nb alone.
template <int TPR, int U>
__device__ __forceinline__ void merge_rows(const HeadArgs& h, const int M, const int nb, int* s_am, float* s_cf) {
    constexpr int NW = TPR / 64, SIDE = MERGE_T / TPR;   // waves per row, rows side by side
    __shared__ float r_max[SB_MAX_W][NW], r_sum[SB_MAX_W][NW];
    __shared__ int r_idx[SB_MAX_W][NW];
    const int tid = threadIdx.x, lane = tid & 63, t = tid % TPR, w = t >> 6, side = tid / TPR;
    for (int r0 = 0; r0 < M; r0 += SIDE) {
        const int row = r0 + side;
        const bool on = row < M;   // (whole waves)
        const float4* p = reinterpret_cast<const float4*>(h.partials) + (size_t)(h.row0 + row) * nb;
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = (on && t + TPR * u < nb) ? p[t + TPR * u] : make_float4(-SB_INF, __int_as_float(0x7fffffff), 0.f, 0.f);
        float mx = -SB_INF;
        int idx = 0x7fffffff;
        auto take = [&](float z, int i) {
            if (z > mx || (z == mx && i < idx)) { mx = z; idx = i; }
        };
        if (on) {
#pragma unroll
            for (int u = 0; u < U; ++u) take(v[u].x, __float_as_int(v[u].y));
#pragma unroll 4
            for (int b = t + TPR * U; b < nb; b += TPR) take(p[b].x, __float_as_int(p[b].y));
            lanes_argmax<32>(mx, idx);
            if (lane == 0) { r_max[row][w] = mx; r_idx[row][w] = idx; }
        }
        __syncthreads();
        if (on) {
            mx = r_max[row][0];
            idx = r_idx[row][0];
#pragma unroll
            for (int i = 1; i < NW; ++i) take(r_max[row][i], r_idx[row][i]);
            if (t == 0) s_am[row] = idx == 0x7fffffff ? 0 : idx;
            float sum = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (t + TPR * u < nb) sum += v[u].z * expf((v[u].x - mx) / h.T);
#pragma unroll 4
            for (int b = t + TPR * U; b < nb; b += TPR) sum += p[b].z * expf((p[b].x - mx) / h.T);
            sum = wave_sum(sum);
            if (lane == 0) r_sum[row][w] = sum;
        }
    }
    __syncthreads();
    if (tid < M) {
        float sum = r_sum[tid][0];
#pragma unroll
        for (int i = 1; i < NW; ++i) sum += r_sum[tid][i];
        s_cf[tid] = 1.0f / sum;
    }
}

__device__ __forceinline__ void head_merge_body(const HeadArgs& h, const int M, const int nb) {
    __shared__ int s_am[SB_MAX_W];
    __shared__ float s_cf[SB_MAX_W];
    __shared__ int s_embed_tok;
    __shared__ float e_red[4];
    const int tid = threadIdx.x;
    // What bounds it is one trip to memory that blocks on other XCDs wrote, then what one CU pulls.  As many rows side by
    // side as leave a row's partials in registers: eight with 128 threads each, four with 256, two with 512.  All
    // 1024 threads on two rows at a time, head calls of 1 and 8 rows: [32000 x 4096] 44.7 and 59.3 us against 44.1 and
    // 46.8, [128256 x 1024] 47.3 and 65.4 against 47.8 and 61.0.
    if (nb <= 1024) merge_rows<128, 8>(h, M, nb, s_am, s_cf);
    else if (nb <= 4096) merge_rows<256, 16>(h, M, nb, s_am, s_cf);
    else merge_rows<512, 16>(h, M, nb, s_am, s_cf);
    if (tid == 0) s_embed_tok = -1;
    __syncthreads();
    if (tid == 0) {
        for (int r = 0; r < M; ++r) {
            if (h.argmax_out) h.argmax_out[r] = s_am[r];
            if (h.conf_out) h.conf_out[r] = s_cf[r];
        }
        if (h.post == POST_EXIT) {
            // Early exit at the first layer whose confidence reaches the threshold
            // (Sec. 3.2), or exactly at the forced layer.
            DevRound* R = h.round;
            int s = h.slot;
            float cf = s_cf[0];
            int am = s_am[0];
            R->conf[s] = cf;
            R->head_argmax[s] = am;
            bool ex = h.forced_exit >= 0 ? (h.layer == h.forced_exit) : (cf >= h.threshold);
            R->exit_flag = ex ? 1 : 0;
            int tok = -1;
            if (ex) {
                tok = h.forced_draft >= 0 ? h.forced_draft : am;
                R->drafts[s] = tok;
                R->slot_tok[s + 1] = tok;
                R->exit_layer[s] = h.layer;
                if (h.embed_E) s_embed_tok = tok;
            }
            if (h.note) {   // the decision for the host, the sequence number last (system-scope release)
                h.note[1] = ex ? 1 : 0;
                h.note[2] = tok;
                h.note[3] = __float_as_int(cf);
                h.note[4] = am;
                __hip_atomic_store(&h.note[0], h.note_seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        } else if (h.post == POST_ACCEPT) {
            // Keep the longest prefix of drafts equal to the greedy tokens; the row
            // after it yields one more token: min(m + 1, M) >= 1 are emitted.
            DevRound* R = h.round;
            int mt = 0;
            for (int r = 0; r < M; ++r) { R->g[r] = s_am[r]; R->gconf[r] = s_cf[r]; }
            while (mt < h.n_drafts && mt < M && R->drafts[mt] == s_am[mt]) ++mt;
            R->n_matched = mt;
            R->n_emit = mt + 1 < M ? mt + 1 : M;
        }
    }
    if (h.post == POST_EXIT && h.embed_E) {   // (uniform for the block)
        __syncthreads();
        const int tok = s_embed_tok;
        if (tok >= 0) {   // the drafted token becomes the next row of the round
            if (h.embed_dtype == SB_BF16) embed_row<uint16_t>((const uint16_t*)h.embed_E, h.embed_vocab, h.embed_d, h.embed_H, tok, 0, h.embed_en, e_red);
            else embed_row<float>((const float*)h.embed_E, h.embed_vocab, h.embed_d, h.embed_H, tok, 0, h.embed_en, e_red);
        }
    }
}

__global__ __launch_bounds__(MERGE_T) void head_merge_kernel(HeadArgs h, int M, int nb) { head_merge_body(h, M, nb); }

// The merges of several sequences after one shared head sweep (batch > 1): block b is the
// single-sequence merge on sequence b's arguments.
__global__ __launch_bounds__(MERGE_T) void head_merge_batch_kernel(HeadMergeBatch hb, int nb) {
    const HeadArgs h = hb.h[blockIdx.x];
    head_merge_body(h, hb.M[blockIdx.x], nb);
}

hipError_t launch_head_merge(const HeadArgs& h, int32_t M, int32_t nb, hipStream_t st) {
    return launch(&head_merge_kernel, dim3(1), MERGE_T, st, h, M, nb);
}

hipError_t launch_head_merge_batch(const HeadMergeBatch& hb, int32_t n, int32_t nb, hipStream_t st) {
    if (n < 1 || n > SB_MAX_W) return hipErrorInvalidValue;
    if (n == 1) return launch_head_merge(hb.h[0], hb.M[0], nb, st);
    return launch(&head_merge_batch_kernel, dim3(n), MERGE_T, st, hb, nb);
}

// ---------------------------------------------------------------- sampling-mode acceptance
// Verification when the output is sampled (Sec. 4.3, "sampling strategies": temperature and
// top-p; the paper gives no rule, the one taken is that of speculative sampling for a draft
// proposed deterministically): with P the distribution the full model samples from after a row
// -- softmax(z / temp), cut to its nucleus of mass top_p and renormalised -- the row's draft x is
// accepted with probability P(x); at the first rejection the token is drawn from P without x;
// when every draft is accepted and one more row exists its token is drawn from P.  Each emitted
// token is then distributed exactly as the full model's own sample.  Works on unnormalised weights
// e_j = exp((z_j - max)/temp).
//
// The nucleus' edge -- the largest weight value `cut` such that the weights >= cut hold a share top_p of the
// sum (so equal weights at its edge stay together) -- is found by three histograms of the weights' mass over
// ten bits of their bit pattern each (monotone in the value of a positive float).  Mass is counted in units of
// 2^-40 of the largest weight, in 64-bit integers: exact in any order, finer than a float sum of as many
// terms.  All rows and all of the vocabulary go through each stage side by side; whether a row is reached at
// all is decided in the last one.  What bounds it: the launches (six of 4.5 to 9 us).  One block that searched the
// edge by bisection, row after row, took 345 us a row at V = 128256 and 100 us at 32000.
constexpr int SMP_T = 1024, SMP_PER = 4, SMP_TOK = SMP_T * SMP_PER;   // threads, tokens per thread, tokens per block
constexpr int SMP_BINS = 1024;
constexpr float SMP_UNIT = 1099511627776.0f;   // 2^40

int sample_blocks(int32_t V) { return (V + SMP_TOK - 1) / SMP_TOK; }
// Scratch of SB_MAX_W rows: weights, histograms, what is known of the edge, per block the mass without the draft and the last token.
struct SampleRow { float* w; unsigned long long* hist; SampleEdge* edge; float* bsum; int* blast; };
size_t sample_scratch_bytes(int32_t V) {
    return (size_t)SB_MAX_W * (3 * SMP_BINS * 8 + sizeof(SampleEdge) + (size_t)V * 4 + (size_t)sample_blocks(V) * 8);
}
__host__ __device__ __forceinline__ SampleRow sample_row(void* scratch, int V, int nb, int row) {
    SampleRow r;
    char* p = (char*)scratch;
    r.hist = (unsigned long long*)p + (size_t)row * 3 * SMP_BINS;
    p += (size_t)SB_MAX_W * 3 * SMP_BINS * 8;
    r.edge = (SampleEdge*)p + row;
    p += SB_MAX_W * sizeof(SampleEdge);
    r.w = (float*)p + (size_t)row * V;
    p += (size_t)SB_MAX_W * V * 4;
    r.bsum = (float*)p + (size_t)row * nb;
    p += (size_t)SB_MAX_W * nb * 4;
    r.blast = (int*)p + (size_t)row * nb;
    return r;
}

// Largest bin whose mass, with that of all bins above and `above`, reaches `need`: {bin, mass above it}.
// 1024 threads, one bin each; every thread gets the result.
__device__ __forceinline__ void find_bin(const unsigned long long* hist, unsigned long long above, unsigned long long need, int& bin, unsigned long long& mass_above) {
    __shared__ unsigned long long wsum[16];
    __shared__ unsigned long long s_above;
    __shared__ int s_bin;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = SMP_BINS - 1 - tid;   // from the top
    unsigned long long own = hist[b], v = own;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    if (lane == 63) wsum[wave] = v;
    if (tid == 0) { s_bin = 0; s_above = above; }
    __syncthreads();
    unsigned long long base = above;
    for (int w = 0; w < wave; ++w) base += wsum[w];
    const unsigned long long upto = base + v, before = upto - own;   // mass of the bins >= b; > b
    if (upto >= need && before < need) { s_bin = b; s_above = before; }
    __syncthreads();
    bin = s_bin;
    mass_above = s_above;
    __syncthreads();
}

// grid (blocks of the vocabulary, rows).  Level 0 makes the weights, counts all of them by their bits 29..20 and is
// told by the head's arg max where the maximum is; level 1 and 2 first finish the level before (every block for
// itself, block 0 leaves it for the next launch), then count the weights that agree with it so far.
template <int LEVEL>
__global__ __launch_bounds__(SMP_T) void sample_hist_kernel(SampleArgs a) {
    __shared__ unsigned long long h[SMP_BINS];
    const int tid = threadIdx.x, row = blockIdx.y, V = a.V;
    const SampleRow r = sample_row(a.scratch, V, gridDim.x, a.row0 + row);
    h[tid] = 0;
    uint32_t prefix = 0;
    if (LEVEL > 0) {
        unsigned long long above = 0, need;
        if (LEVEL == 1) {
            unsigned long long total;
            int bin;
            __shared__ unsigned long long tsum[16];
            unsigned long long v = r.hist[tid];
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            if ((tid & 63) == 0) tsum[tid >> 6] = v;
            __syncthreads();
            total = 0;
            for (int w = 0; w < 16; ++w) total += tsum[w];
            need = (unsigned long long)((double)a.top_p * (double)total);
            if (need < 1) need = 1;   // (the largest weight alone)
            find_bin(r.hist, 0, need, bin, above);
            prefix = (uint32_t)bin;
        } else {
            int bin;
            need = r.edge[0].need;
            find_bin(r.hist + SMP_BINS, r.edge[0].above1, need, bin, above);
            prefix = (r.edge[0].bin1 << 10) | (uint32_t)bin;
        }
        if (blockIdx.x == 0 && tid == 0) {
            if (LEVEL == 1) { r.edge[0].need = need; r.edge[0].above1 = above; r.edge[0].bin1 = prefix; }
            else { r.edge[0].above2 = above; r.edge[0].bin2 = prefix; }
        }
    }
    __syncthreads();
    const float* z = a.logits + (size_t)row * V;
    const float mx = LEVEL == 0 ? z[a.round->g[row]] : 0.f;
    for (int i = 0; i < SMP_PER; ++i) {
        const int j = blockIdx.x * SMP_TOK + i * SMP_T + tid;
        if (j >= V) break;
        float e;
        if (LEVEL == 0) {
            e = expf((z[j] - mx) / a.temp);
            r.w[j] = e;
        } else {
            e = r.w[j];
        }
        const uint32_t bits = __float_as_uint(e);
        if (!(e > 0.f) || (LEVEL > 0 && (bits >> (30 - 10 * LEVEL)) != prefix)) continue;
        const uint32_t bin = LEVEL == 0 ? bits >> 20 : (bits >> (20 - 10 * LEVEL)) & (SMP_BINS - 1);
        atomicAdd(&h[bin < SMP_BINS ? bin : SMP_BINS - 1], (unsigned long long)(e * SMP_UNIT + 0.5f));
    }
    __syncthreads();
    if (h[tid]) atomicAdd(&r.hist[LEVEL * SMP_BINS + tid], h[tid]);
}

// grid (blocks of the vocabulary, rows): the edge, the mass it keeps, and per block what is left to draw from.
__global__ __launch_bounds__(SMP_T) void sample_mass_kernel(SampleArgs a) {
    __shared__ float ws[16];
    __shared__ int wl[16];
    const int tid = threadIdx.x, row = blockIdx.y, V = a.V;
    const SampleRow r = sample_row(a.scratch, V, gridDim.x, a.row0 + row);
    float cut = 0.f;
    unsigned long long kept = 0;
    if (a.top_p < 1.0f) {
        int bin;
        unsigned long long above;
        find_bin(r.hist + 2 * SMP_BINS, r.edge[0].above2, r.edge[0].need, bin, above);
        cut = __uint_as_float((r.edge[0].bin2 << 10) | (uint32_t)bin);
        kept = above + r.hist[2 * SMP_BINS + bin];
    } else {   // everything is kept
        unsigned long long v = r.hist[tid];
        __shared__ unsigned long long tsum[16];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((tid & 63) == 0) tsum[tid >> 6] = v;
        __syncthreads();
        for (int w = 0; w < 16; ++w) kept += tsum[w];
    }
    if (blockIdx.x == 0 && tid == 0) {
        r.edge[0].cut = cut;
        r.edge[0].keep = (float)((double)kept * (1.0 / (double)SMP_UNIT));
    }
    const int x = row < a.n_drafts ? a.round->drafts[row] : -1;
    const int j0 = blockIdx.x * SMP_TOK + tid * SMP_PER;
    float s = 0.f;
    int last = -1;
#pragma unroll
    for (int i = 0; i < SMP_PER; ++i) {
        const int j = j0 + i;
        const float e = j < V ? r.w[j] : 0.f;
        if (j < V && e >= cut && j != x) { s += e; last = j; }
    }
    s = wave_sum(s);
    for (int o = 32; o > 0; o >>= 1) { const int v = __shfl_xor(last, o, 64); last = v > last ? v : last; }
    if ((tid & 63) == 0) { ws[tid >> 6] = s; wl[tid >> 6] = last; }
    __syncthreads();
    if (tid == 0) {
        float t = 0.f;
        int l = -1;
        for (int w = 0; w < 16; ++w) { t += ws[w]; l = wl[w] > l ? wl[w] : l; }
        r.bsum[blockIdx.x] = t;
        r.blast[blockIdx.x] = l;
    }
}

// One block: the rows in order, until one is not accepted.
__global__ __launch_bounds__(SMP_T) void sample_accept_kernel(SampleArgs a, int nb) {
    __shared__ float wtot[16], s_bs[SMP_T], s_cut[SB_MAX_W], s_keep[SB_MAX_W], s_ex[SB_MAX_W];
    __shared__ int s_bl[SMP_T], s_x[SB_MAX_W];
    __shared__ float s_base;
    __shared__ int s_blk, s_tok;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, V = a.V;
    DevRound* R = a.round;
    if (tid < a.M) {   // every row's edge, draft and weight of the draft
        const SampleRow r = sample_row(a.scratch, V, nb, a.row0 + tid);
        const int x = tid < a.n_drafts ? R->drafts[tid] : -1;
        const float cut = r.edge[0].cut, e = x >= 0 && x < V ? r.w[x] : 0.f;
        s_cut[tid] = cut;
        s_keep[tid] = r.edge[0].keep;
        s_x[tid] = x;
        s_ex[tid] = e < cut ? 0.f : e;
    }
    __syncthreads();
    int m = 0;       // accepted drafts so far (uniform)
    int drawn = -1;  // row at which a token was drawn
    for (int row = 0; row < a.M; ++row) {
        const SampleRow r = sample_row(a.scratch, V, nb, a.row0 + row);
        const float cut = s_cut[row], keep = s_keep[row], ex = s_ex[row];
        const int x = s_x[row];
        if (tid == 0) R->gconf[row] = ex / keep;   // P(x): the row's acceptance probability
        if (row < a.n_drafts && a.ua[row] * keep < ex) {  // accepted
            if (tid == 0) R->g[row] = x;
            ++m;
            continue;
        }
        // draw from P without x: inverse CDF over the tokens in index order, first the block, then the token
        const float target = a.ur[row] * (keep - ex);
        if (tid == 0) { s_blk = -1; s_base = 0.f; s_tok = -1; }
        for (int t0 = 0; t0 < nb; t0 += SMP_T) {
            __syncthreads();
            if (s_blk >= 0) break;
            s_bs[tid] = t0 + tid < nb ? r.bsum[t0 + tid] : 0.f;
            s_bl[tid] = t0 + tid < nb ? r.blast[t0 + tid] : -1;
            __syncthreads();
            if (tid == 0) {
                const int n = nb - t0 < SMP_T ? nb - t0 : SMP_T;
                float c = s_base;
                int last = s_tok;   // (rounding at the upper end: the last token that has mass)
                for (int t = 0; t < n; ++t) {
                    if (c + s_bs[t] > target) { s_blk = t0 + t; break; }
                    c += s_bs[t];
                    last = s_bl[t] >= 0 ? s_bl[t] : last;
                }
                s_base = c;
                s_tok = s_blk >= 0 ? 0x7fffffff : last;
            }
        }
        __syncthreads();
        const int blk = s_blk;
        if (blk >= 0) {
            const int j0 = blk * SMP_TOK + tid * SMP_PER;
            float e[SMP_PER], s = 0.f;
#pragma unroll
            for (int i = 0; i < SMP_PER; ++i) {
                const int j = j0 + i;
                e[i] = j < V ? r.w[j] : 0.f;
                if (!(j < V && e[i] >= cut && j != x)) e[i] = 0.f;
                s += e[i];
            }
            float v = s;   // inclusive scan over the block's threads
            for (int o = 1; o < 64; o <<= 1) {
                const float u = __shfl_up(v, o, 64);
                if (lane >= o) v += u;
            }
            if (lane == 63) wtot[wave] = v;
            __syncthreads();
            float c = s_base;
            for (int w = 0; w < wave; ++w) c += wtot[w];
            c += v - s;
            int tok = 0x7fffffff;
#pragma unroll
            for (int i = 0; i < SMP_PER; ++i) {
                c += e[i];
                if (tok == 0x7fffffff && e[i] > 0.f && c > target) tok = j0 + i;
            }
            if (tok != 0x7fffffff) atomicMin(&s_tok, tok);
            __syncthreads();
            if (tid == 0 && s_tok == 0x7fffffff) s_tok = r.blast[blk];
        }
        if (tid == 0) R->g[row] = s_tok;
        drawn = row;
        break;
    }
    if (tid == 0) {
        for (int row = (drawn >= 0 ? drawn : a.M - 1) + 1; row < a.M; ++row) { R->g[row] = -1; R->gconf[row] = 0.f; }
        R->n_matched = m;
        R->n_emit = m + 1 < a.M ? m + 1 : a.M;
    }
}

hipError_t launch_sample_accept(const SampleArgs& a, hipStream_t st) {
    if (!a.logits || !a.round || !a.scratch || ((uintptr_t)a.scratch & 7) || a.V < 1 || a.V > (1 << 24) || a.M < 1 || a.row0 < 0 ||
        a.row0 + a.M > SB_MAX_W || !(a.temp > 0.f) || !(a.top_p > 0.f))
        return hipErrorInvalidValue;
    const int nb = sample_blocks(a.V);
    const dim3 grid(nb, a.M);
    const SampleRow r = sample_row(a.scratch, a.V, nb, a.row0);
    hipError_t e = launch_fill_u32((uint32_t*)r.hist, (size_t)a.M * 3 * SMP_BINS * 2, 0u, st);
    if (e != hipSuccess) return e;
    sample_hist_kernel<0><<<grid, SMP_T, 0, st>>>(a);
    if (a.top_p < 1.0f) {
        sample_hist_kernel<1><<<grid, SMP_T, 0, st>>>(a);
        sample_hist_kernel<2><<<grid, SMP_T, 0, st>>>(a);
    }
    sample_mass_kernel<<<grid, SMP_T, 0, st>>>(a);
    sample_accept_kernel<<<1, SMP_T, 0, st>>>(a, nb);
    return hipGetLastError();
}

}  // namespace sb
