// Attention of the decode path over the paged KV cache: rotary embedding and cache append of the new
// rows, partial soft-max attention per 128-key chunk (vector ALUs for an fp32 cache, matrix cores for
// a bf16 cache), the merge of the chunks, and the same for several sequences in one launch pair.
#include "kernels.h"
#include "device_utils.h"

#include <math.h>
#include <type_traits>

namespace sb {

// ---------------------------------------------------------------- RoPE + KV append + attention
// M causal query rows at positions pos0..pos0+M-1 against keys 0..pos of the
// paged cache.  qkv holds the rows' raw projections (q heads, k heads, v heads).
// The key range is cut into fixed chunks of absolute positions; one block handles
// one (kv head, chunk, group of <= 16 queries) and writes a partial (max, sum,
// weighted V) per query; a second kernel merges the chunks in ascending order.
//
// The work inside a block is latency, not bandwidth, so everything is laid out for
// few dependent steps: K and V go from the cache straight into registers (no LDS
// tile), each in the mapping its consumer needs, all loads issued up front.
//   scores   four lanes per key, each with every fourth piece of 16 bytes: two exchanges add them up
//   softmax  wave per query over the chunk's keys
//   values   thread = (16-byte group of dims, key slot): a few keys each, then a fixed
//            tree over the key slots of a wave
// Whatever the cache holds in the slots of the new rows (they are loaded with the rest, without
// a condition) is replaced: the block rotates their keys (half-split pairing, table built on the
// host in double and held in float) and rounds keys and values from qkv exactly as they are
// stored, and the block of query group 0 also writes them into the cache (KV append).  A row's result depends on its own
// position and keys only.
// Four values of an fp32 cache.
__device__ __forceinline__ void unpack4(uint4 v, float* f) {
    f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
}
__device__ __forceinline__ uint4 pack4(const float* f) {
    return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
}

// A value as the cache holds it.
template <typename KVT>
__device__ __forceinline__ KVT kv_round(float f) {
    if constexpr (sizeof(KVT) == 2) return f2bf(f);
    else return f;
}

// A rotated pair, x cos - y sin and y cos + x sin, with the product that is rounded by itself spelled out: the compiler's choice
// between the two follows the code around it, and a stored key's last bit would change with that.
__device__ __forceinline__ float rope_lo(float x, float y, float c, float sn) { return fmaf(x, c, -(y * sn)); }
__device__ __forceinline__ float rope_hi(float x, float y, float c, float sn) { return fmaf(x, sn, y * c); }

// A finished value of row r, as the merge stage leaves it.
__device__ __forceinline__ void attn_finish(const AttnArgs& a, int r, int col, int ld, float v) {
    if (a.out) a.out[(size_t)r * ld + col] = v;
    if (a.out_split) split_store_rows(a.out_split, ld, a.split_rows, r, col, v);
}

// N neighbouring floats: one load where the operands are 16-byte aligned (VEC), else N.
template <int N, bool VEC>
__device__ __forceinline__ void load_near(const float* p, float (&v)[N]) {
    typedef float vec_t __attribute__((ext_vector_type(N == 1 ? 2 : N)));
    if constexpr (N > 1 && VEC) {
        const vec_t t = *reinterpret_cast<const vec_t*>(p);
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = t[i];
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = p[i];
    }
}
// N neighbouring values into LDS at a multiple of their size
template <int N, typename T>
__device__ __forceinline__ void store_near(T* p, const T (&v)[N]) {
    if constexpr (N == 1) {
        p[0] = v[0];
    } else {
        typedef T vec_t __attribute__((ext_vector_type(N)));
        vec_t t;
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = v[i];
        *reinterpret_cast<vec_t*>(p) = t;
    }
}

// Row of a kv head's query qq (row-major over the head's group), qq / G.  VEC: by a multiplication with 2^32 / G rounded up, exact while
// qq (G - 1) < 2^32, as attn_fast sees to; a division by a number that only the launch knows is some forty instructions, here in
// front of the query loads.
template <bool VEC>
__device__ __forceinline__ int attn_row(const AttnArgs& a, int qq) {
    if constexpr (VEC) return a.g_inv ? (int)__umulhi((uint32_t)qq, a.g_inv) : qq;   // (0: one query per row and kv head)
    else return qq / a.group;
}

// The queries of a block with their rotary factors, four pairs per thread.  VEC: four loads of 16 bytes each instead of sixteen.
template <int HD, bool VEC>
struct QueryRows {
    static constexpr int HALF = HD / 2, TPQ = HALF / 4;   // threads per query
    float x[4], y[4], c[4], sn[4];
    bool live;
    static __device__ __forceinline__ int query() { return threadIdx.x / TPQ; }
    static __device__ __forceinline__ int dim() { return threadIdx.x % TPQ * 4; }
    // queries q0 .. q0 + nq - 1 of kv head g; the others read the first one and count as zeros
    __device__ __forceinline__ void load(const AttnArgs& a, int g, int q0, int nq) {
        const int G = a.group, qi = query(), j = dim();
        live = qi < nq;
        const int qq = q0 + (live ? qi : 0), r = attn_row<VEC>(a, qq), gi = qq - r * G;
        const float* qp = a.q + (size_t)r * a.qkv_rows + (size_t)(g * G + gi) * HD + j;
        const size_t rope = (size_t)(a.pos0 + r) * HALF + j;
        load_near<sizeof(x) / 4, VEC>(qp, x);
        load_near<sizeof(y) / 4, VEC>(qp + HALF, y);
        load_near<sizeof(c) / 4, VEC>(a.rope_cos + rope, c);
        load_near<sizeof(sn) / 4, VEC>(a.rope_sin + rope, sn);
    }
    // rotated: dims j .. j + 3 and, HALF further, their partners
    __device__ __forceinline__ void rotate(float (&lo)[4], float (&hi)[4]) const {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float u = x[e] * c[e] - y[e] * sn[e], v = y[e] * c[e] + x[e] * sn[e];
            lo[e] = live ? u : 0.f;
            hi[e] = live ? v : 0.f;
        }
    }
};

// The new rows' keys and values of kv head g (at most SB_MAX_W rows), HD / 64 pairs and HD / 32 values per thread: loaded with everything
// else a block reads, rotated and rounded once, and left in LDS for the lanes whose keys they are.
template <int HD, bool VEC>
struct NewRows {
    static constexpr int HALF = HD / 2, NP = HALF / 32, NV = HD / 32;
    float x[NP], y[NP], c[NP], sn[NP], v[NV];
    __device__ __forceinline__ void load(const AttnArgs& a, int g) {
        const int r = threadIdx.x >> 5, i = threadIdx.x & 31;   // 32 threads per row
        const float* kp = a.q + (size_t)(r < a.M ? r : 0) * a.qkv_rows + (size_t)(a.n_heads + g) * HD;
        const size_t rope = (size_t)(a.pos0 + (r < a.M ? r : 0)) * HALF + i * NP;
        load_near<sizeof(x) / 4, VEC>(kp + i * NP, x);
        load_near<sizeof(y) / 4, VEC>(kp + i * NP + HALF, y);
        load_near<sizeof(c) / 4, VEC>(a.rope_cos + rope, c);
        load_near<sizeof(sn) / 4, VEC>(a.rope_sin + rope, sn);
        load_near<sizeof(v) / 4, VEC>(kp + (size_t)a.kv.n_kv_heads * HD + i * NV, v);
    }
    // V_BY_DIM: the values by dim, 16 keys each from key pos0 & ~7 on, else by row
    template <typename KVT, int LDK, bool V_BY_DIM>
    __device__ __forceinline__ void store(const AttnArgs& a, KVT* k_s, KVT* v_s) const {
        const int r = threadIdx.x >> 5, i = threadIdx.x & 31;
        if (r >= a.M) return;
        KVT lo[NP], hi[NP], w[NV];
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            lo[k] = kv_round<KVT>(rope_lo(x[k], y[k], c[k], sn[k]));
            hi[k] = kv_round<KVT>(rope_hi(x[k], y[k], c[k], sn[k]));
        }
#pragma unroll
        for (int k = 0; k < NV; ++k) w[k] = kv_round<KVT>(v[k]);
        store_near(k_s + r * LDK + i * NP, lo);
        store_near(k_s + r * LDK + i * NP + HALF, hi);
        if constexpr (V_BY_DIM) {
#pragma unroll
            for (int k = 0; k < NV; ++k) v_s[(i * NV + k) * 16 + (a.pos0 & 7) + r] = w[k];
        } else {
            store_near(v_s + r * HD + i * NV, w);
        }
    }
};

// Four blocks per CU (one wave of each per SIMD).  MANY: passes of more than SB_MAX_W rows, whose chunks are full of new rows: each thread
// prepares its own.  Else the new rows go through LDS.  VEC: as in QueryRows.
// What bounds it: few keys the instructions of one wave in a row, of which each is some six cycles, behind two round trips (page table,
// operands) and an empty launch's 1.7 us; many keys the memory.  So what a wave can do without is left to a branch of the whole wave (new rows,
// slots past the last key, dims of dead queries), a query is finished by the lanes of one key slot after the loop over queries, not by all
// inside it, and four lanes share a key: a load covers 64 bytes of each of 16 keys (a lane with half a key for itself touched 64 lines with
// each load), and a query's dims come out of LDS once for two keys.  Before and after: 4 heads x 64 behind 60 keys, one / four / eight rows
// 5.0 / 7.3 / 10.8 -> 3.7 / 4.7 / 6.5 us; 32 heads x 128, one row behind 300 / 2000 / 9000 keys 8.9 / 16.8 / 62.8 -> 8.1 / 16.3 / 62.5, six behind 2000
// 20.3 -> 19.3; 128 rows of 32 heads x 128 behind none / 4000 31 / 280 -> 20.5 / 259.
template <int HD, bool MANY, bool VEC>
__global__ __launch_bounds__(256, 4) void attn_kernel(AttnArgs a) {
    constexpr int CH = HD <= 64 ? 128 : 64;                   // keys per chunk
    constexpr int EPV = 4;                                    // elements per 16 bytes
    constexpr int QG = 16;                                    // queries per block
    constexpr int HALF = HD / 2;
    // scores mapping: a wave takes CH / 4 keys, a page at a time; four lanes per key, each with every fourth piece of 16 bytes
    constexpr int KT = CH / 4 / SB_KV_BLOCK;                  // pages per wave
    constexpr int NKV = HD / EPV / 4;                         // pieces per key and lane
    // values mapping: each wave owns HD/4 dims and sees every key of the chunk, so the
    // sum over keys ends inside the wave (no cross-wave stage, no LDS buffer for it)
    constexpr int DGW = HD / 4 / EPV;                         // 16-byte dim groups per wave
    constexpr int KS = 64 / DGW;                              // key slots (lanes per dim group)
    constexpr int KPT = CH / KS;                              // keys per value thread
    // (head_dim 128: the values are requested behind the keys' first use.  32 heads, one row behind 300 / 2000 / 9000 keys 8.0 / 16.2 / 62.5 us, together 7.8 /
    // 16.9 / 62.3)
    constexpr bool LATE_V = HD > 64;
    static_assert(KT >= 1 && NKV % 2 == 0, "a wave's keys are whole pages; a lane has both parts of its rotary pairs");
    static_assert(DGW >= 1 && KS * KPT == CH && KPT % 4 == 0 && SB_KV_BLOCK % KS == 0, "value mapping: a load's keys lie in one page");
    __shared__ __attribute__((aligned(16))) float qs[QG * HD];
    __shared__ __attribute__((aligned(16))) float sp[QG * CH];  // scores by key, then probabilities by key slot
    __shared__ float s_m[QG], s_l[QG];
    constexpr int NR = MANY ? 1 : SB_MAX_W;
    __shared__ __attribute__((aligned(16))) float nk_s[NR * HD], nv_s[NR * HD];   // (!MANY) the new rows' keys and values

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (the chunk with the new rows, the longest to prepare, first)
    const int g = blockIdx.x, chunk = gridDim.y - 1 - blockIdx.y, qg = blockIdx.z;
    const int Hq = a.n_heads, Hkv = a.kv.n_kv_heads, G = a.group;
    const int nq_total = a.M * G, q0 = qg * QG;
    const int nq = (nq_total - q0 < QG) ? (nq_total - q0) : QG;
    const int key0 = chunk * CH, n_total = a.pos0 + a.M;
    const float scale = 1.0f / sqrtf((float)HD);
    const size_t page_elems = (size_t)Hkv * SB_KV_BLOCK * HD;
    float* const kbase = reinterpret_cast<float*>(a.kv.pool) + (size_t)(a.layer * 2 + 0) * a.kv.n_pages * page_elems;
    float* const vbase = reinterpret_cast<float*>(a.kv.pool) + (size_t)(a.layer * 2 + 1) * a.kv.n_pages * page_elems;

    // ---- page-table entries, all in flight at once; a key past the end takes the last page (what its slot holds is not used)
    const bool has_new = key0 + CH > a.pos0;
    const uint32_t last = (uint32_t)(n_total - 1) / SB_KV_BLOCK;
    auto page_at = [&](int key) {   // (key: the same in all lanes, so through the scalar cache)
        const uint32_t p = (uint32_t)key / SB_KV_BLOCK;
        return a.kv.table[p < last ? p : last];
    };
    const int kw = key0 + wave * (CH / 4);                     // the wave's first key
    const int kslot = lane >> 2, kd0 = (lane & 3) * EPV;       // scores: key kw + 16 t + kslot, dims kd0 + 4 EPV i ..
    const int vd0 = wave * (HD / 4) + (lane % DGW) * EPV, vks = lane / DGW;   // values: dims vd0 .., keys vks + KS * i
    int kpage[KT], vpage[KPT];
#pragma unroll
    for (int t = 0; t < KT; ++t) kpage[t] = page_at(kw + t * SB_KV_BLOCK);
#pragma unroll
    for (int i = 0; i < KPT; ++i) vpage[i] = page_at(key0 + KS * i);
    // ---- the other loads: q (+ its rotary factors), the new rows, K, V
    QueryRows<HD, VEC> qr;
    qr.load(a, g, q0, nq);
    NewRows<HD, VEC> nr;
    if (!MANY && has_new) nr.load(a, g);
    uint4 kreg[KT][NKV];   // (of a wave without keys: unset and unused)
    const uint32_t koff = (uint32_t)((g * SB_KV_BLOCK + kslot) * HD + kd0);
    if (kw < n_total)
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int i = 0; i < NKV; ++i) kreg[t][i] = *reinterpret_cast<const uint4*>(kbase + (size_t)kpage[t] * page_elems + koff + i * 4 * EPV);
    uint4 vreg[KPT];
    auto vaddr = [&](int i) { return (size_t)vpage[i] * page_elems + (uint32_t)((g * SB_KV_BLOCK + ((vks + KS * i) % SB_KV_BLOCK)) * HD + vd0); };
    auto load_v = [&]() {
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            vreg[i] = make_uint4(0, 0, 0, 0);   // (slots past the last key: 0 x stale bits that read as NaN is not 0)
            if (key0 + KS * i < n_total) vreg[i] = *reinterpret_cast<const uint4*>(vbase + vaddr(i));
        }
    };
    if (!LATE_V) load_v();
    // ---- rotated queries -> LDS, and the new rows' keys and values as they are stored
    if (qr.live) {
        float lo[4], hi[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {   // (one rounding for all forms: a row's bits do not depend on the rows beside it)
            lo[e] = rope_lo(qr.x[e], qr.y[e], qr.c[e], qr.sn[e]);
            hi[e] = rope_hi(qr.x[e], qr.y[e], qr.c[e], qr.sn[e]);
        }
        store_near(qs + qr.query() * HD + qr.dim(), lo);
        store_near(qs + qr.query() * HD + qr.dim() + HALF, hi);
    }
    if (!MANY && has_new) nr.template store<float, HD, false>(a, nk_s, nv_s);
    __syncthreads();
    if (LATE_V) {
        __builtin_amdgcn_sched_barrier(0);
        load_v();
    }
    // ---- keys (and, below, values) of the new rows take the place of what the cache held, appended by query group 0
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        const int k0 = kw + t * SB_KV_BLOCK, key = k0 + kslot;
        if (k0 + SB_KV_BLOCK <= a.pos0 || k0 >= n_total) continue;
        if (key >= a.pos0 && key < n_total) {
            if constexpr (MANY) {
                const float* kp = a.q + (size_t)(key - a.pos0) * a.qkv_rows + (size_t)(Hq + g) * HD;
#pragma unroll
                for (int i = 0; i < NKV / 2; ++i) {
                    const int j = kd0 + i * 4 * EPV;
                    float x[EPV], y[EPV], c[EPV], sn[EPV], lo[EPV], hi[EPV];
                    load_near<EPV, VEC>(kp + j, x);
                    load_near<EPV, VEC>(kp + j + HALF, y);
                    load_near<EPV, VEC>(a.rope_cos + (size_t)key * HALF + j, c);
                    load_near<EPV, VEC>(a.rope_sin + (size_t)key * HALF + j, sn);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) {
                        lo[e] = rope_lo(x[e], y[e], c[e], sn[e]);
                        hi[e] = rope_hi(x[e], y[e], c[e], sn[e]);
                    }
                    kreg[t][i] = pack4(lo);
                    kreg[t][i + NKV / 2] = pack4(hi);
                }
            } else {
#pragma unroll
                for (int i = 0; i < NKV; ++i) kreg[t][i] = *reinterpret_cast<const uint4*>(&nk_s[(key - a.pos0) * HD + kd0 + i * 4 * EPV]);
            }
            if (qg == 0)
#pragma unroll
                for (int i = 0; i < NKV; ++i) *reinterpret_cast<uint4*>(kbase + (size_t)kpage[t] * page_elems + koff + i * 4 * EPV) = kreg[t][i];
        }
    }
    auto new_values = [&]() {
        if (!has_new) return;
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            const int k0 = key0 + KS * i, key = k0 + vks;
            if (k0 + KS <= a.pos0 || k0 >= n_total) continue;
            if (key >= a.pos0) {
                vreg[i] = make_uint4(0, 0, 0, 0);
                if (key < n_total) {
                    if constexpr (MANY) {
                        float f[EPV];
                        load_near<EPV, VEC>(a.q + (size_t)(key - a.pos0) * a.qkv_rows + (size_t)(Hq + Hkv + g) * HD + vd0, f);
                        vreg[i] = pack4(f);
                    } else {
                        vreg[i] = *reinterpret_cast<const uint4*>(&nv_s[(key - a.pos0) * HD + vd0]);
                    }
                    if (qg == 0) *reinterpret_cast<uint4*>(vbase + vaddr(i)) = vreg[i];
                }
            }
        }
    };
    if (!LATE_V) new_values();

    // ---- scores of this wave's keys against every live query
    if (kw < n_total) {
        float kf[KT][NKV][EPV];
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int i = 0; i < NKV; ++i) unpack4(kreg[t][i], kf[t][i]);
        for (int qi = 0; qi < nq; ++qi) {
            float4 qv[NKV * EPV / 4];   // (all requested before the first is used: one wait, not one per piece)
#pragma unroll
            for (int i = 0; i < NKV; ++i)
#pragma unroll
                for (int e = 0; e < EPV; e += 4) qv[(i * EPV + e) / 4] = *reinterpret_cast<const float4*>(&qs[qi * HD + kd0 + i * 4 * EPV + e]);
            __builtin_amdgcn_sched_barrier(0);
            float s[KT];
#pragma unroll
            for (int t = 0; t < KT; ++t) s[t] = 0.f;
#pragma unroll
            for (int i = 0; i < NKV; ++i)
#pragma unroll
                for (int e = 0; e < EPV; e += 4) {
                    const float4 v = qv[(i * EPV + e) / 4];
#pragma unroll
                    for (int t = 0; t < KT; ++t) s[t] = fmaf(v.x, kf[t][i][e], s[t]);
#pragma unroll
                    for (int t = 0; t < KT; ++t) s[t] = fmaf(v.y, kf[t][i][e + 1], s[t]);
#pragma unroll
                    for (int t = 0; t < KT; ++t) s[t] = fmaf(v.z, kf[t][i][e + 2], s[t]);
#pragma unroll
                    for (int t = 0; t < KT; ++t) s[t] = fmaf(v.w, kf[t][i][e + 3], s[t]);
                }
#pragma unroll
            for (int t = 0; t < KT; ++t) sp[qi * CH + wave * (CH / 4) + t * SB_KV_BLOCK + kslot] = lanes_sum<2>(s[t]);
        }
    }
    __syncthreads();
    // ---- softmax partial of each live query over the chunk (one wave per query)
    for (int qi = wave; qi < nq; qi += 4) {
        const int r = attn_row<VEC>(a, q0 + qi);
        float sc[CH / 64];
        float mx = -SB_INF;
#pragma unroll
        for (int h = 0; h < CH / 64; ++h) {
            const int t = lane + 64 * h;
            sc[h] = (key0 + t <= a.pos0 + r) ? sp[qi * CH + t] * scale : -SB_INF;
            mx = fmaxf(mx, sc[h]);
        }
        mx = wave_max(mx);
        float l = 0.f;
#pragma unroll
        for (int h = 0; h < CH / 64; ++h) {
            float p = (mx == -SB_INF) ? 0.f : expf(sc[h] - mx);
            sc[h] = p;
            l += p;
        }
        l = wave_sum(l);
#pragma unroll
        for (int h = 0; h < CH / 64; ++h) {
            const int t = lane + 64 * h;
            sp[qi * CH + (t % KS) * KPT + t / KS] = sc[h];
        }
        if (lane == 0) { s_m[qi] = mx; s_l[qi] = l; }
    }
    __syncthreads();
    if (LATE_V) new_values();
    // ---- weighted values; the lanes of key slot s finish query q1 + s
    {
        float vf[KPT][EPV];
#pragma unroll
        for (int i = 0; i < KPT; ++i) unpack4(vreg[i], vf[i]);
        for (int q1 = 0; q1 < nq; q1 += KS) {
            float res[EPV];
#pragma unroll
            for (int e = 0; e < EPV; ++e) res[e] = 0.f;
            const int nk = nq - q1 < KS ? nq - q1 : KS;
            for (int z = 0; z < nk; ++z) {
                float p[KPT], o[EPV];
#pragma unroll
                for (int i = 0; i < KPT; i += 4) {
                    const float4 v = *reinterpret_cast<const float4*>(&sp[(q1 + z) * CH + vks * KPT + i]);
                    p[i] = v.x; p[i + 1] = v.y; p[i + 2] = v.z; p[i + 3] = v.w;
                }
#pragma unroll
                for (int e = 0; e < EPV; ++e) o[e] = 0.f;
#pragma unroll
                for (int i = 0; i < KPT; ++i)
#pragma unroll
                    for (int e = 0; e < EPV; ++e) o[e] = fmaf(p[i], vf[i][e], o[e]);
                // sum over the key slots: fixed tree inside the wave
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float t = lanes_sum<32, DGW>(o[e]);
                    res[e] = vks == z ? t : res[e];
                }
            }
            const int qi = q1 + vks, qq = q0 + qi, r = attn_row<VEC>(a, qq), gi = qq - r * G;
            if (vks < nk && key0 <= a.pos0 + r) {  // (a chunk with no visible key leaves no partial)
                if (a.direct) {
#pragma unroll
                    for (int e = 0; e < EPV; ++e) res[e] /= s_l[qi];
                    if (a.out)
#pragma unroll
                        for (int e = 0; e < EPV; ++e) a.out[(size_t)r * Hq * HD + (g * G + gi) * HD + vd0 + e] = res[e];
                    if (a.out_split)
#pragma unroll
                        for (int e = 0; e < EPV; ++e) split_store_rows(a.out_split, Hq * HD, a.split_rows, r, (g * G + gi) * HD + vd0 + e, res[e]);
                } else {
                    float* dst = a.partials + ((size_t)(r * Hq + g * G + gi) * a.max_chunks + chunk) * (HD + 2);
#pragma unroll
                    for (int e = 0; e < EPV; ++e) dst[2 + vd0 + e] = res[e];
                    if (vd0 == 0) { dst[0] = s_m[qi]; dst[1] = s_l[qi]; }
                }
            }
        }
    }
}

// The same step for a bf16 cache, with both contractions on the matrix cores.
//   scores   S = Q K^T: A operand = rotated queries (16 rows; fp32 carried as a bf16
//            hi + lo pair, two MFMAs), B operand = keys straight from the cache (a lane's
//            8 consecutive dims of one key are one 16-byte load); a wave takes 32 keys
//   softmax  wave per query over the chunk's keys, probabilities left in LDS as hi + lo
//   values   O = P V: A operand = probabilities, B operand = values.  A lane needs 8
//            consecutive keys of one dim, so the V pages of a bf16 cache are stored
//            transposed, [kv head][dim][16 keys]: the operand is again one 16-byte load
//            and a wave's loads cover whole pages.  A wave owns HD/4 output dims.
// Every output row of an MFMA depends on its own operand row only, so a query's
// partial does not depend on which other queries share the block.
// What bounds it: the chain page table -> operands -> scores -> soft-max -> values of a block, of which four per CU cover for each
// other (126 registers at head_dim 128, 98 at 64, 26 and 22 KB of LDS).  The chunk with the new rows is the longest: it is started first, and its new keys and values come with the other operands
// and through LDS (a load and a wait for each element, as lanes picked them from the projections, cost 3 us at six rows).
// Both kernels in a graph of launches, 32 heads x 128, one row behind 520 / 1000 keys 8.5 / 9.4 -> 7.75 / 8.7 us, six behind 520 / 2000 / 4200 9.70 / 12.7 /
// 20.9 -> 8.75 / 12.2 / 20.3; 32 heads over 8 x 128, one / four rows behind 700 8.55 / 9.9 -> 7.5 / 8.1; one row of 32 behind 20 keys (the first stage alone)
// 5.4 -> 4.6.  What that took: the queries in wide loads, a query's row by a multiplication, the group's size from the host, new rows looked for only
// where a tile has one and taken under a branch, up to sixteen queries' soft-max side by side with their probabilities split in pairs, nothing
// written for queries that are not there, a partial's maximum and sum stored where they are found, its address in 32 bits.  Of some
// 8500 cycles of a block's chain (one row) the page table takes 500, the operands 3000, the new rows 1400, the queries 850, scores 500,
// soft-max 850, values and stores 1000.
// LDS of one block of the matrix-core attention kernels.
template <int HD>
struct AttnLds {
    static constexpr int CH = 128, QG = 16, QS = HD + 8, PS = CH + 8, SS = CH + 4;   // padded row strides
    __attribute__((aligned(16))) uint16_t q_hi[QG * QS], q_lo[QG * QS];
    __attribute__((aligned(16))) uint16_t p_hi[QG * PS], p_lo[QG * PS];
    __attribute__((aligned(16))) float s_s[QG * SS];
    float s_l[QG];
};

// A block's work -- (kv head g, key chunk, slice zb of the query groups) -- in two steps: load() requests everything that it
// reads from memory (the first query group with its rotary factors, the chunk's K and V operands) into registers, compute() does the rest.
template <int HD, bool VEC>
struct AttnItem {
    static constexpr int CH = 128, QG = 16, HALF = HD / 2;
    static constexpr int KSQ = HD / 32;      // k steps (of 32 dims) of the score product
    static constexpr int KSV = CH / 32;      // k steps (of 32 keys) of the value product
    static constexpr int DT = HD / 64;       // 16-dim output tiles per wave
    static constexpr int QS = HD + 8, PS = CH + 8, SS = CH + 4;
    int g, chunk, zb;
    QueryRows<HD, VEC> qr;
    uint4 kreg[2][KSQ];
    int kpage[2];
    uint4 vreg[DT][KSV];
    int vpg[KSV];       // page of this lane's keys of a step
    NewRows<HD, VEC> nr;

    __device__ __forceinline__ void load_q(const AttnArgs& a, int qg) {
        const int nq_total = a.M * a.group, q0 = qg * QG;
        qr.load(a, g, q0, nq_total - q0 < QG ? nq_total - q0 : QG);
    }

    __device__ __forceinline__ void load(const AttnArgs& a, int g_, int chunk_, int zb_) {
        g = g_; chunk = chunk_; zb = zb_;
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        const int li = lane & 15, lq = lane >> 4;
        const int key0 = chunk * CH, n_total = a.pos0 + a.M;
        const size_t page_elems = (size_t)a.kv.n_kv_heads * SB_KV_BLOCK * HD;
        const uint16_t* const kbase = reinterpret_cast<const uint16_t*>(a.kv.pool) + (size_t)(a.layer * 2 + 0) * a.kv.n_pages * page_elems;
        const uint16_t* const vbase = reinterpret_cast<const uint16_t*>(a.kv.pool) + (size_t)(a.layer * 2 + 1) * a.kv.n_pages * page_elems;
        // ---- page-table entries of the chunk, all in flight at once, through the scalar cache; a page past the end is the
        // last one (what its slots hold is masked or replaced)
        const int last_page = (n_total - 1) / SB_KV_BLOCK;
        int vpage[2 * KSV];
    #pragma unroll
        for (int i = 0; i < 2 * KSV; ++i) {
            const int p = key0 / SB_KV_BLOCK + i;
            vpage[i] = a.kv.table[p < last_page ? p : last_page];
        }
    #pragma unroll
        for (int t = 0; t < 2; ++t) {   // (a tile is one page)
            const int p = __builtin_amdgcn_readfirstlane(key0 / SB_KV_BLOCK + wave * 2 + t);
            kpage[t] = a.kv.table[p < last_page ? p : last_page];
        }
        // ---- every other load of the item: q (+ its rotary factors) of the first group, the new rows, K, V
        load_q(a, zb * a.qg_per_block);
        if (key0 + CH > a.pos0) nr.load(a, g);   // (the chunk holds keys of the new rows)
        // K operands: tile t of this wave = keys key0 + wave*32 + t*16 + li (one page), dims ks*32 + lq*8 ..
    #pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint16_t* kp = kbase + (size_t)kpage[t] * page_elems + (uint32_t)((g * SB_KV_BLOCK + li) * HD + lq * 8);
    #pragma unroll
            for (int ks = 0; ks < KSQ; ++ks) kreg[t][ks] = *reinterpret_cast<const uint4*>(kp + ks * 32);
        }
        // V operands: dim (wave*DT + dt)*16 + li, keys key0 + ks*32 + lq*8 .. +8 (half a page row); the 32 keys of a step lie
        // in two pages (lq 0-1, lq 2-3)
        const uint32_t voff = (uint32_t)((g * HD + wave * DT * 16 + li) * SB_KV_BLOCK + (lq & 1) * 8);
    #pragma unroll
        for (int ks = 0; ks < KSV; ++ks) {
            vpg[ks] = vpage[2 * ks] + ((vpage[2 * ks + 1] - vpage[2 * ks]) & -(lq >> 1));   // (a choice in registers, not of addresses)
            const uint16_t* vp = vbase + (size_t)vpg[ks] * page_elems + voff;
    #pragma unroll
            for (int dt = 0; dt < DT; ++dt) vreg[dt][ks] = *reinterpret_cast<const uint4*>(vp + dt * 16 * SB_KV_BLOCK);
        }
    }

    __device__ __forceinline__ void compute(const AttnArgs& a, AttnLds<HD>& lds) {
        const int Hq = a.n_heads, G = a.group;
        const int nq_total = a.M * G;
        // this block's query groups (16 queries each), handled one after the other with the
        // chunk's K and V held in registers
        const int n_qg = (nq_total + QG - 1) / QG;
        const int qg_first = zb * a.qg_per_block;
        const int qg_last = (qg_first + a.qg_per_block < n_qg) ? qg_first + a.qg_per_block : n_qg;
        const int key0 = chunk * CH, n_total = a.pos0 + a.M;
        const float scale = 1.0f / sqrtf((float)HD);
        const size_t page_elems = (size_t)a.kv.n_kv_heads * SB_KV_BLOCK * HD;
        uint16_t* const kbase = reinterpret_cast<uint16_t*>(a.kv.pool) + (size_t)(a.layer * 2 + 0) * a.kv.n_pages * page_elems;
        uint16_t* const vbase = reinterpret_cast<uint16_t*>(a.kv.pool) + (size_t)(a.layer * 2 + 1) * a.kv.n_pages * page_elems;
        const bool has_new = key0 + CH > a.pos0;  // the chunk holds keys of the new rows
        uint16_t* const q_hi = lds.q_hi; uint16_t* const q_lo = lds.q_lo;
        uint16_t* const p_hi = lds.p_hi; uint16_t* const p_lo = lds.p_lo;
        float* const s_s = lds.s_s; float* const s_l = lds.s_l;
        // (the new rows lie where the probabilities come later)
        uint16_t* const nk_s = lds.p_hi; uint16_t* const nv_s = lds.p_lo;
        static_assert(SB_MAX_W * QS <= QG * PS && HD * 16 <= QG * PS && SB_MAX_W <= 8, "the new rows fit");
        if (has_new) nr.template store<uint16_t, QS, true>(a, nk_s, nv_s);
        for (int qg = qg_first; qg < qg_last; ++qg) {
        // (the thread's number anew for every group: the addresses that follow from it, some hundred instructions and
        // as many registers, would otherwise be worked out ahead of the loop, which most launches go round once)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int li = lane & 15, lq = lane >> 4;
        const int q0 = qg * QG;
        const int nq = (nq_total - q0 < QG) ? (nq_total - q0) : QG;
        // ---- rotated queries -> LDS as hi + lo
        if (qr.query() < QG) {
            float lo[4], hi[4];
            qr.rotate(lo, hi);
            const int at = qr.query() * QS + qr.dim();
    #pragma unroll
            for (int o = 0; o < 2; ++o) {
                const float (&u)[4] = o ? hi : lo;
                uint32_t h[2], l[2];
                split_pair(__float_as_uint(u[0]), __float_as_uint(u[1]), h[0], l[0]);
                split_pair(__float_as_uint(u[2]), __float_as_uint(u[3]), h[1], l[1]);
                *reinterpret_cast<uint2*>(q_hi + at + o * HALF) = make_uint2(h[0], h[1]);
                *reinterpret_cast<uint2*>(q_lo + at + o * HALF) = make_uint2(l[0], l[1]);
            }
        }
        if (qg + 1 < qg_last) load_q(a, qg + 1);  // (in flight during this group's products)
        __syncthreads();
        // ---- keys and values of the new rows take the place of what the cache held, appended by query group 0; values of
        // slots past the last key become zero (0 x stale bits that read as NaN is not 0; their scores are masked): in a step
        // with new rows by masks, in a later one all at once
        if (has_new && qg == qg_first) {
    #pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int kt0 = key0 + wave * 32 + t * 16, key = kt0 + li;
                if (kt0 + 16 <= a.pos0 || kt0 >= n_total) continue;   // (wave-uniform: no new key in this tile)
                if (key >= a.pos0 && key < n_total) {
                    uint16_t* const at = kbase + (size_t)kpage[t] * page_elems + (uint32_t)((g * SB_KV_BLOCK + li) * HD + lq * 8);
    #pragma unroll
                    for (int ks = 0; ks < KSQ; ++ks) {
                        kreg[t][ks] = *reinterpret_cast<const uint4*>(nk_s + (key - a.pos0) * QS + lq * 8 + ks * 32);
                        if (zb == 0) *reinterpret_cast<uint4*>(at + ks * 32) = kreg[t][ks];
                    }
                }
            }
    #pragma unroll
            for (int ks = 0; ks < KSV; ++ks) {
                const int kf = key0 + ks * 32 + lq * 8;
                // (block-uniform: no new row in this step, or no row at all)
                if (key0 + ks * 32 + 32 <= a.pos0) continue;
                if (key0 + ks * 32 >= n_total) {
    #pragma unroll
                    for (int dt = 0; dt < DT; ++dt) vreg[dt][ks] = make_uint4(0, 0, 0, 0);
                    continue;
                }
                // of this lane's eight keys: which are new (or past the last key), which exist
                uint32_t fresh[4], keep[4];
    #pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = kf + 2 * e;
                    fresh[e] = (k >= a.pos0 ? 0xffffu : 0u) | (k + 1 >= a.pos0 ? 0xffff0000u : 0u);
                    keep[e] = (k < n_total ? 0xffffu : 0u) | (k + 1 < n_total ? 0xffff0000u : 0u);
                }
                const int at = kf - (a.pos0 & ~7);   // (a multiple of 8; the slots are 0 and 8)
    #pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const uint4 v = *reinterpret_cast<const uint4*>(nv_s + ((wave * DT + dt) * 16 + li) * 16 + (at == 8 ? 8 : 0));
                    uint4& w = vreg[dt][ks];
                    w = make_uint4(((w.x & ~fresh[0]) | (v.x & fresh[0])) & keep[0], ((w.y & ~fresh[1]) | (v.y & fresh[1])) & keep[1],
                                   ((w.z & ~fresh[2]) | (v.z & fresh[2])) & keep[2], ((w.w & ~fresh[3]) | (v.w & fresh[3])) & keep[3]);
                }
                if (zb == 0 && kf + 8 > a.pos0 && kf < n_total)
    #pragma unroll
                    for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<uint4*>(vbase + (size_t)vpg[ks] * page_elems + (uint32_t)((g * HD + (wave * DT + dt) * 16 + li) * SB_KV_BLOCK + (lq & 1) * 8)) = vreg[dt][ks];
            }
        }

        // ---- scores of this wave's 32 keys against the 16 query rows
        {
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    #pragma unroll
            for (int ks = 0; ks < KSQ; ++ks) {
                const bf16x8 ah = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&q_hi[li * QS + ks * 32 + lq * 8]));
                const bf16x8 al = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&q_lo[li * QS + ks * 32 + lq * 8]));
    #pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const bf16x8 kb = __builtin_bit_cast(bf16x8, kreg[t][ks]);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, kb, acc[t], 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, kb, acc[t], 0, 0, 0);
                }
            }
            // result register r of lane (li, lq): query 4*lq + r, key li of the tile
    #pragma unroll
            for (int t = 0; t < 2; ++t)
    #pragma unroll
                for (int r = 0; r < 4; ++r) s_s[(4 * lq + r) * SS + wave * 32 + t * 16 + li] = acc[t][r];
        }
        __syncthreads();
        // ---- softmax partial of each query over the chunk: up to four queries a wave each, with more all sixteen at once, 16 lanes
        // each with keys t0, t0 + 16, ..; either way a query's sum is taken over key bits 6, 5, .. 0 in this order
        // (what lies in the operand rows of queries that are not there reaches their own result rows only)
        const auto put_pair = [&](int at, int step, float x, float y) {   // two probabilities as high and low parts
            uint32_t h, l;
            split_pair(__float_as_uint(x), __float_as_uint(y), h, l);
            p_hi[at] = (uint16_t)h; p_hi[at + step] = (uint16_t)(h >> 16);
            p_lo[at] = (uint16_t)l; p_lo[at + step] = (uint16_t)(l >> 16);
        };
        const auto partial = [&](int qq, int r) {   // of query qq, a query of row r (the head's number is g G + qq - r G)
            const uint32_t at = (uint32_t)(r * (Hq - G) + g * G + qq) * (uint32_t)a.max_chunks + (uint32_t)chunk;
            return a.partials + (size_t)at * (HD + 2);
        };
        const auto put_sum = [&](int qi, int r, float mx, float l) {
            if (a.direct) s_l[qi] = l;
            else if (key0 <= a.pos0 + r) *reinterpret_cast<float2*>(partial(q0 + qi, r)) = make_float2(mx, l);
        };
        if (nq <= 4) {
            const int qi = wave;
            if (qi < nq) {
                const int r = attn_row<VEC>(a, q0 + qi);
                float sc[2], mx = -SB_INF;
    #pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int t = lane + 64 * h;
                    sc[h] = (key0 + t <= a.pos0 + r) ? s_s[qi * SS + t] * scale : -SB_INF;
                    mx = fmaxf(mx, sc[h]);
                }
                mx = wave_max(mx);
                float p[2];
    #pragma unroll
                for (int h = 0; h < 2; ++h) p[h] = (mx == -SB_INF) ? 0.f : expf(sc[h] - mx);
                put_pair(qi * PS + lane, 64, p[0], p[1]);
                const float l = wave_sum(p[0] + p[1]);
                if (lane == 0) put_sum(qi, r, mx, l);
            }
        } else {
            const int qi = tid >> 4, t0 = tid & 15;
            const bool live = qi < nq;   // (unused operand rows: defined values)
            const int r = attn_row<VEC>(a, q0 + qi), vis = a.pos0 + r - key0 - t0;
            float sc[8], p[8], mx = -SB_INF;
    #pragma unroll
            for (int k = 0; k < 8; ++k) {
                sc[k] = 16 * k <= vis ? s_s[qi * SS + t0 + 16 * k] * scale : -SB_INF;
                mx = fmaxf(mx, sc[k]);
            }
            mx = lanes_max<8>(mx);
    #pragma unroll
            for (int k = 0; k < 8; ++k) p[k] = !live || mx == -SB_INF ? 0.f : expf(sc[k] - mx);
    #pragma unroll
            for (int k = 0; k < 8; k += 2) put_pair(qi * PS + t0 + 16 * k, 16, p[k], p[k + 1]);
    #pragma unroll
            for (int d = 4; d > 0; d >>= 1)
    #pragma unroll
                for (int k = 0; k < d; ++k) p[k] += p[k + d];
            const float l = lanes_sum<8>(p[0]);
            if (t0 == 0 && live) put_sum(qi, r, mx, l);
        }
        __syncthreads();
        // ---- weighted values: this wave's DT tiles of 16 dims, all keys of the chunk
        {
            f32x4 o[DT];
    #pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    #pragma unroll
            for (int ks = 0; ks < KSV; ++ks) {
                const bf16x8 ah = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&p_hi[li * PS + ks * 32 + lq * 8]));
                const bf16x8 al = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&p_lo[li * PS + ks * 32 + lq * 8]));
    #pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const bf16x8 vb = __builtin_bit_cast(bf16x8, vreg[dt][ks]);
                    o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, vb, o[dt], 0, 0, 0);
                    o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, vb, o[dt], 0, 0, 0);
                }
            }
    #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int qi = 4 * lq + r;
                if (qi >= nq) continue;
                const int rr = attn_row<VEC>(a, q0 + qi);
                if (key0 > a.pos0 + rr) continue;  // (a chunk with no visible key leaves no partial)
                if (a.direct) {
                    const int gi = q0 + qi - rr * G;
    #pragma unroll
                    for (int dt = 0; dt < DT; ++dt) attn_finish(a, rr, (g * G + gi) * HD + (wave * DT + dt) * 16 + li, Hq * HD, o[dt][r] / s_l[qi]);
                    continue;
                }
                float* const p = partial(q0 + qi, rr) + 2 + wave * DT * 16 + li;
    #pragma unroll
                for (int dt = 0; dt < DT; ++dt) p[dt * 16] = o[dt][r];
            }
        }
        __syncthreads();  // the next group overwrites the LDS arrays
        }
    }
};

template <int HD, bool VEC>
__device__ __forceinline__ void attn_mfma_body(const AttnArgs& a, const int g, const int chunk, const int zb) {
    __shared__ AttnLds<HD> lds;
    AttnItem<HD, VEC> it;
    it.load(a, g, chunk, zb);
    it.compute(a, lds);
}

template <int HD, bool VEC>
__global__ __launch_bounds__(256, 3) void attn_mfma_kernel(AttnArgs a) {
    attn_mfma_body<HD, VEC>(a, blockIdx.x, gridDim.y - 1 - blockIdx.y, blockIdx.z);   // (the chunk with the new rows first)
}

// Several sequences' passes in one launch (batch > 1): grid.z = sequence x query-group slice, grid.y
// = the longest sequence's chunks; a block outside its sequence's range leaves at once.  A block
// inside runs the code above on its sequence's arguments, so every value is the one the
// sequence's own launch computes.
template <int HD>
__global__ __launch_bounds__(256, 3) void attn_mfma_batch_kernel(AttnBatchArgs ab) {
    const int sq = blockIdx.z / ab.zdim, zb = blockIdx.z - sq * ab.zdim;
    const AttnArgs a = ab.seq[sq];
    const int n_chunks = (a.pos0 + a.M + 127) / 128;
    const int n_qg = (a.M * (a.n_heads / a.kv.n_kv_heads) + 15) / 16;
    if ((int)blockIdx.y >= n_chunks || zb * a.qg_per_block >= n_qg) return;
    attn_mfma_body<HD, true>(a, blockIdx.x, n_chunks - 1 - blockIdx.y, zb);
}

// Second stage: one block per (row, query head) merges that row's chunk partials
// (online-softmax rule against the row's overall maximum).  A thread owns two dims;
// the chunks are dealt round-robin to the block's thread groups so that all loads
// of a short context are in flight at once, each group adds its chunks in ascending
// order and the groups are added in index order.  The order depends on the row's
// position only.
template <int HD, int CH>
__device__ __forceinline__ void attn_merge_body(const AttnArgs& a, const int hq, const int r) {
    constexpr int MAXC = 512;
    constexpr int TPG = HD / 2;       // threads per group
    constexpr int NG = 256 / TPG;     // chunk groups
    constexpr int U = 8;              // loads in flight per thread
    __shared__ float sm[MAXC], sl[MAXC];
    __shared__ float red[4];
    __shared__ __attribute__((aligned(8))) float go[NG][HD];
    __shared__ float gl[NG];
    const int tid = threadIdx.x;
    const int grp = tid / TPG, dp = tid % TPG;
    const int Hq = a.n_heads, stride = HD + 2;
    const int nc = (a.pos0 + r) / CH + 1;
    const float* p = a.partials + (size_t)(r * Hq + hq) * a.max_chunks * stride;
    // this thread's first U chunks' values are requested before anything else
    float2 av[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int c = grp + NG * u;
        av[u] = make_float2(0.f, 0.f);
        if (c < nc) av[u] = *reinterpret_cast<const float2*>(p + (size_t)c * stride + 2 + 2 * dp);
    }
    float mx = -SB_INF;
    for (int c = tid; c < nc; c += 256) {
        const float2 ml = *reinterpret_cast<const float2*>(p + (size_t)c * stride);
        sm[c] = ml.x;
        sl[c] = ml.y;
        mx = fmaxf(mx, ml.x);
    }
    mx = wave_max(mx);
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    float L = 0.f, O0 = 0.f, O1 = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int c = grp + NG * u;
        if (c < nc) {
            const float w = expf(sm[c] - mx);
            L += sl[c] * w; O0 += av[u].x * w; O1 += av[u].y * w;
        }
    }
    for (int c0 = grp + NG * U; c0 < nc; c0 += NG * U) {  // long contexts: further rounds of U loads
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + NG * u;
            av[u] = make_float2(0.f, 0.f);
            if (c < nc) av[u] = *reinterpret_cast<const float2*>(p + (size_t)c * stride + 2 + 2 * dp);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + NG * u;
            if (c < nc) {
                const float w = expf(sm[c] - mx);
                L += sl[c] * w; O0 += av[u].x * w; O1 += av[u].y * w;
            }
        }
    }
    go[grp][2 * dp] = O0;
    go[grp][2 * dp + 1] = O1;
    if (dp == 0) gl[grp] = L;
    __syncthreads();
    if (tid < HD) {
        float Ls = 0.f, Os = 0.f;
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) { Ls += gl[gi]; Os += go[gi][tid]; }
        attn_finish(a, r, hq * HD + tid, Hq * HD, Os / Ls);
    }
}

template <int HD, int CH>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a) {
    attn_merge_body<HD, CH>(a, blockIdx.x, blockIdx.y);
}

template <int HD, int CH>
__global__ __launch_bounds__(256) void attn_merge_batch_kernel(AttnBatchArgs ab) {
    const AttnArgs a = ab.seq[blockIdx.z];
    if ((int)blockIdx.y >= a.M) return;
    attn_merge_body<HD, CH>(a, blockIdx.x, blockIdx.y);
}

int attn_chunk_keys(int32_t head_dim, int32_t kv_dtype) {
    return (head_dim * (kv_dtype == SB_BF16 ? 2 : 4) <= 256) ? 128 : 64;
}

// Checks one pass's arguments and gives its launch shape: chunks, query groups, groups per block.
static bool attn_shape(const AttnArgs& a, int* n_chunks, int* n_qg, int* qpb) {
    const int hd = a.kv.head_dim;
    if ((hd != 64 && hd != 128) || a.M < 1 || a.M > SB_PREFILL_ROWS || a.n_heads % a.kv.n_kv_heads) return false;
    if (a.out_split && a.split_rows < a.M) return false;
    if (!a.rope_cos || !a.rope_sin) return false;
    const int ch = attn_chunk_keys(hd, a.kv.kv_dtype);
    *n_chunks = (a.pos0 + a.M + ch - 1) / ch;
    if (*n_chunks > a.max_chunks || *n_chunks > 512) return false;
    const int G = a.n_heads / a.kv.n_kv_heads;
    // Query groups of 16: one block each while the launch is small; in a large launch (a prompt
    // pass over a long context) a block takes several groups in turn on one load of its K/V
    // chunk.  A query's result does not depend on the grouping.
    *n_qg = (a.M * G + 15) / 16;
    *qpb = (int)(((long)a.kv.n_kv_heads * *n_chunks * *n_qg + 1023) / 1024);
    if (*qpb > *n_qg) *qpb = *n_qg;
    return true;
}

// The fast form of the matrix-core kernel: rows and tables that 16-byte loads may read (their rows are whole multiples of that), and rows found by
// a multiplication (at most 8 G queries and 15 unused ones: 8 G G < 2^32).
static bool attn_fast(const AttnArgs& a) {
    return (((uintptr_t)a.q | (uintptr_t)a.rope_cos | (uintptr_t)a.rope_sin) & 15) == 0 && a.qkv_rows % 4 == 0 && a.n_heads / a.kv.n_kv_heads <= 16384;
}
static uint32_t attn_g_inv(const AttnArgs& a) {
    const uint64_t G = a.n_heads / a.kv.n_kv_heads;
    return G == 1 ? 0u : (uint32_t)(((1ull << 32) + G - 1) / G);
}

hipError_t launch_attention(const AttnArgs& a, hipStream_t st) {
    const int hd = a.kv.head_dim;
    int n_chunks, n_qg, qpb;
    if (!attn_shape(a, &n_chunks, &n_qg, &qpb)) return hipErrorInvalidValue;
    AttnArgs b = a;
    b.qg_per_block = qpb;
    b.group = a.n_heads / a.kv.n_kv_heads;
    b.g_inv = attn_g_inv(a);
    // With a single chunk the merge would multiply by exp(0) and add zeros: the first stage divides and
    // stores by itself (the same bits), a launch less.  An output over the input has to wait for the end of the first stage.
    b.direct = n_chunks == 1 && !attn_out_over_input(a);
    dim3 grid(a.kv.n_kv_heads, n_chunks, (n_qg + qpb - 1) / qpb);
    dim3 grid1(a.kv.n_kv_heads, n_chunks, n_qg);
    dim3 mgrid(a.n_heads, a.M);
    const auto go = [&](auto hd_c) {
        constexpr int HD = decltype(hd_c)::value, CH32 = HD == 128 ? 64 : 128;   // (keys per chunk of an fp32 cache)
        const bool fast = attn_fast(a);
        hipError_t e;
        if (a.kv.kv_dtype == SB_BF16) {
            if (a.M > SB_MAX_W) return hipErrorInvalidValue;   // (more rows: launch_prefill_attention)
            e = launch(fast ? &attn_mfma_kernel<HD, true> : &attn_mfma_kernel<HD, false>, grid, 256, st, b);
        } else if (a.M > SB_MAX_W) {
            e = launch(&attn_kernel<HD, true, false>, grid1, 256, st, b);
        } else {
            e = launch(fast ? &attn_kernel<HD, false, true> : &attn_kernel<HD, false, false>, grid1, 256, st, b);
        }
        if (b.direct || e != hipSuccess) return e;
        return launch(a.kv.kv_dtype == SB_BF16 ? &attn_merge_kernel<HD, 128> : &attn_merge_kernel<HD, CH32>, mgrid, 256, st, a);
    };
    return hd == 128 ? go(std::integral_constant<int, 128>{}) : go(std::integral_constant<int, 64>{});
}

hipError_t launch_attention_batch(const AttnArgs* seqs, int n, hipStream_t st) {
    if (n < 1 || n > SB_MAX_W) return hipErrorInvalidValue;
    bool one_shape = seqs[0].kv.kv_dtype == SB_BF16;
    for (int i = 1; i < n; ++i)
        one_shape = one_shape && seqs[i].kv.kv_dtype == SB_BF16 && seqs[i].kv.head_dim == seqs[0].kv.head_dim &&
                    seqs[i].kv.n_kv_heads == seqs[0].kv.n_kv_heads && seqs[i].n_heads == seqs[0].n_heads;
    for (int i = 0; i < n; ++i) one_shape = one_shape && attn_fast(seqs[i]);
    if (n == 1 || !one_shape) {  // (an fp32 cache takes the vector-ALU kernel, a launch per sequence)
        for (int i = 0; i < n; ++i) {
            hipError_t e = launch_attention(seqs[i], st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    AttnBatchArgs ab{};
    int max_chunks = 0, max_m = 0;
    ab.zdim = 1;
    for (int i = 0; i < n; ++i) {
        int n_chunks, n_qg, qpb;
        if (!attn_shape(seqs[i], &n_chunks, &n_qg, &qpb) || seqs[i].M > SB_MAX_W) return hipErrorInvalidValue;
        ab.seq[i] = seqs[i];
        ab.seq[i].qg_per_block = qpb;
        ab.seq[i].group = seqs[i].n_heads / seqs[i].kv.n_kv_heads;
        ab.seq[i].g_inv = attn_g_inv(seqs[i]);
        const int z = (n_qg + qpb - 1) / qpb;
        if (z > ab.zdim) ab.zdim = z;
        if (n_chunks > max_chunks) max_chunks = n_chunks;
        if (seqs[i].M > max_m) max_m = seqs[i].M;
    }
    for (int i = 0; i < n; ++i) ab.seq[i].direct = max_chunks == 1;   // (the sessions' own buffers: no output over an input)
    dim3 grid(seqs[0].kv.n_kv_heads, max_chunks, n * ab.zdim);
    dim3 mgrid(seqs[0].n_heads, max_m, n);
    const auto go = [&](auto hd_c) {
        constexpr int HD = decltype(hd_c)::value;
        const hipError_t e = launch(&attn_mfma_batch_kernel<HD>, grid, 256, st, ab);
        return max_chunks == 1 || e != hipSuccess ? e : launch(&attn_merge_batch_kernel<HD, 128>, mgrid, 256, st, ab);
    };
    return seqs[0].kv.head_dim == 128 ? go(std::integral_constant<int, 128>{}) : go(std::integral_constant<int, 64>{});
}

}  // namespace sb
