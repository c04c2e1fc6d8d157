// gfx950 kernels of the prompt passes: the same decoder layer as a decode pass, for
// up to SB_PREFILL_ROWS rows at once, so that the weights are streamed once per 128
// prompt tokens instead of once per 8 (prefill is the base model's own, Sec. 4.3;
// only its cost matters, not its schedule).
//
// A projection is two kernels.  prefill_gemm_kernel streams the tile-packed bf16
// weights (A operand, straight from HBM into registers, as in the decode path) against
// the rows' activations, which every wave of the block needs and which are therefore
// staged through LDS (B operand; bf16 high and low parts, two MFMAs per weight tile,
// so a product keeps about 16 bits of the activation's mantissa as in the decode
// path).  The work is cut evenly across thread blocks, also along k, so a row of the
// result is left as a few partial sums.  prefill_epilogue_kernel adds them in index
// order, applies the RMSNorm scale and the projection's tail (store, residual + next
// input, SwiGLU).
#include <type_traits>
#include "kernels.h"
#include "device_utils.h"

namespace sb {

namespace {
constexpr int PM = SB_PREFILL_ROWS;
constexpr int WPB = 8;                     // waves per thread block, one thread block per CU
constexpr int ROWB = 288;                  // LDS bytes per staged row: 128 bf16 + 32 bytes of padding (16-byte operand
                                           // reads at rows 272 bytes apart measure as 2-way bank conflicts, at 288 as none)
constexpr int stage_bytes(int ct) { return 2 * ct * 16 * ROWB; }            // one k block of both planes
constexpr int lds_bytes(int ct) { return 2 * stage_bytes(ct) + PM * 4; }    // two stages + the rows' scales
}  // namespace

// Work decomposition: the rows of the super-pass are cut into equal passes of at most PM rows
// (whole 16-row column tiles), the weight rows into row blocks (8 waves x rt tiles of 16).  Per pass,
// the (row block, k block) pairs are numbered row block first and cut into equal contiguous
// ranges, one per thread block, so that every block streams the same number of weight bytes
// whatever the shape (a plain k split leaves a ragged last round of blocks on 256 CUs).  A range
// may end in the middle of a row block: each thread block that touches a row block leaves one
// partial sum for it, in slot (range index - first range of that row block).  rt, q and grid depend on
// the weights' shape and the number of passes only, so a row's sums do not depend on the rows beside
// it within a launch of as many passes.
struct GemmPlan {
    int rt;          // 16-row weight tiles per wave
    int block_rows;  // weight rows of a row block
    int nb;          // row blocks
    int q;           // (row block, k block) pairs per thread block
    int grid;        // thread blocks per pass
    int smax;        // most partial sums a row block can get
};
static GemmPlan gemm_plan_rt(int32_t rows, int32_t K, int32_t n_pass, int rt) {
    GemmPlan p;
    const int KB = K >> 7;
    p.rt = rt;
    p.block_rows = WPB * rt * 16;
    p.nb = (rows + p.block_rows - 1) / p.block_rows;
    const long total = (long)p.nb * KB;
    // resident thread blocks: one per CU (LDS), shared out among the passes of the launch --
    // every pass gets the same cut, so the blocks of different passes that work on the same
    // weights are neighbours in the grid and run at the same time
    int slots = 256 / n_pass;
    if (slots < 1) slots = 1;
    p.q = (int)((total + slots - 1) / slots);
    if (p.q < 2 && KB >= 2) p.q = 2;          // (never one partial per k block)
    p.grid = (int)((total + p.q - 1) / p.q);  // per pass
    p.smax = (KB + p.q - 1) / p.q + 1;
    if (p.smax > KB) p.smax = KB;
    return p;
}
// Tiles per wave.  A wave reads the pass's activations from LDS once per tile set: with two tiles these reads
// alone keep the LDS as busy as the matrix cores are, with four half as busy ([28672 x 4096] at 1999 rows: 821
// and 739 us), but twice the weight rows per thread block leave twice the partial sums: four where
// a thread block still gets half a row block's k range or more (measured about even below it: [12288 x 4096] at
// 512 rows 120 and 126 us with their epilogues, [4096 x 11008] at 1024 rows 183 and 196).  A single pass is bound
// by the weight stream: small matrices take one tile, so that a thread block's range is long and its partial
// sums few.  Calls that split their rows first, with one / two tiles at 16, 64 and 128 rows: [12288 x 4096] (q = 12) 24.8 / 28.8, 32.5 / 38.6,
// 46.3 / 53.8 us; [16384 x 4096] (16) 35.0 / 38.8, 39.9 / 47.5, 53.4 / 58.7; [5120 x 13824] (17) 31.6 / 31.6, 42.4 / 42.0,
// 69.9 / 57.5; [15360 x 5120] (19) 33.2 / 33.5, 44.8 / 41.7, 61.3 / 58.4.
static GemmPlan gemm_plan(int32_t rows, int32_t K, int32_t n_pass, bool gate_up) {
    const int KB = K >> 7;
    if (n_pass == 1) {
        const GemmPlan p = gemm_plan_rt(rows, K, 1, 1);
        return p.q <= 16 && !gate_up ? p : gemm_plan_rt(rows, K, 1, 2);   // (gate and up tiles meet in one wave)
    }
    const GemmPlan p = gemm_plan_rt(rows, K, n_pass, 4);
    return 2 * p.q >= KB ? p : gemm_plan_rt(rows, K, n_pass, 2);
}
int gemm_splits(int32_t rows, int32_t K, int32_t n_pass, bool gate_up) { return gemm_plan(rows, K, n_pass, gate_up).smax; }
// Rows of a pass: the super-pass in n_pass equal parts, rounded up to whole column tiles.
static int gemm_pass_rows(int32_t M, int32_t n_pass) { return ((M + n_pass - 1) / n_pass + 15) / 16 * 16; }

// The sum of the n values at p (16-byte aligned, readable up to the next multiple of four), added in index order: the first 4 U are requested
// together (a loop of load and add would be a round trip for each, single values four times the requests), and added
// up where the caller has other loads on their way as well.
template <int U>
struct IndexSum {
    float4 q[U];
    __device__ __forceinline__ void load(const float* p, int n, int j0 = 0) {
#pragma unroll
        for (int k = 0; k < U; ++k) q[k] = *reinterpret_cast<const float4*>(p + (j0 + 4 * k < n ? j0 + 4 * k : 0));
    }
    __device__ __forceinline__ float sum(const float* p, int n) {
        float t = 0.f;
        for (int j0 = 0;;) {
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int j = j0 + 4 * k;
                t += j < n ? q[k].x : 0.f;
                t += j + 1 < n ? q[k].y : 0.f;
                t += j + 2 < n ? q[k].z : 0.f;
                t += j + 3 < n ? q[k].w : 0.f;
            }
            j0 += 4 * U;
            if (j0 >= n) return t;   // (the same for all lanes)
            load(p, n, j0);
        }
    }
};

// ---- pieces of the GEMM kernel (all inlined; register arrays are passed by reference) ----
struct GemmCtx {
    int KB, n_tiles, it1, wr;          // wr: the wave's row group
    int Mp, cid, pass, row0;           // live rows of this pass, range index, pass, its first row
    int n_out_tiles;                   // fused gate/up: 16-column groups of the output (gate tile j pairs with up tile n_out_tiles + j)
};

// Weight tile t of this wave in row block b; -1 past the end.  Gate/up with the fused tail: the
// wave's tiles are the gate tiles of RT / 2 groups of 16 outputs, then their up tiles.
template <int RT, bool SWI>
__device__ __forceinline__ int gemm_tile(const GemmCtx& c, int b, int t) {
    if (SWI) {
        const int j = (b * WPB + c.wr) * (RT / 2) + t % (RT / 2);
        return j < c.n_out_tiles ? (t < RT / 2 ? j : c.n_out_tiles + j) : -1;
    }
    const int tile = (b * WPB + c.wr) * RT + t;
    return tile < c.n_tiles ? tile : -1;
}

// Where the weights of a (row block, k block) pair begin, one pointer per tile of the wave: wave-uniform
// (scalar registers).  Past the block's range it stays on the last pair: a re-read keeps the
// steady-state loop free of conditional loads.
template <int RT, bool SWI>
struct GemmWeights {
    const char* p[RT];
    int it, b, kb;
    __device__ __forceinline__ void base(const GemmCtx& c, const void* W) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            int tile = gemm_tile<RT, SWI>(c, b, t);
            if (tile < 0) tile = c.n_tiles - 1;  // a tile past the end re-reads the last one (not stored)
            p[t] = reinterpret_cast<const char*>(W) + ((size_t)tile * c.KB + kb) * 4096;
        }
    }
    __device__ __forceinline__ void init(const GemmCtx& c, const void* W, int it_) {
        it = it_;
        b = it / c.KB;
        kb = it - b * c.KB;
        base(c, W);
    }
    __device__ __forceinline__ void next(const GemmCtx& c, const void* W) {
        if (it + 1 >= c.it1) return;
        ++it;
        if (++kb == c.KB) {
            kb = 0;
            ++b;
            base(c, W);
        } else {
#pragma unroll
            for (int t = 0; t < RT; ++t) p[t] += 4096;
        }
    }
};
// MFMA step u (32 k) of every tile.  STREAM: the weights are read once by this launch (a single pass),
// so the loads carry the streaming hint; with several passes the other passes' blocks read the same
// lines and they are left to the caches.
template <int RT, bool STREAM, bool SWI>
__device__ __forceinline__ void gemm_load_a(uint4 (&ar)[RT], const GemmWeights<RT, SWI>& w, int u, uint32_t lane_off) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const uint16_t* wp = reinterpret_cast<const uint16_t*>(w.p[t] + u * 1024 + lane_off);
        ar[t] = STREAM ? ld_weights_packed(wp) : *reinterpret_cast<const uint4*>(wp);
    }
}

// Staging map: 2 planes x 16 CT rows x 16 segments of 16 bytes, CT per thread; unit i of a thread
// lies 32 rows below unit i - 1 (same segment), first in the high plane, then in the low plane.
// Rows past the live ones are read too, from the planes' unused rows: whatever they hold only
// reaches result columns that are never stored.
template <int CT, bool RAW>
struct GemmStage {
    static constexpr int N = CT, FIRST = CT > 4 ? (CT + 1) / 2 : CT;   // 16-byte registers of a k block; requested at its start, the rest half way
    const char* base;      // the pass's first row in the high plane
    uint32_t off;          // this thread's byte offset at unit 0
    size_t off_mid;        // ... at the unit that holds the last rows of the high and the first of the low plane (odd CT)
    int row_bytes, lo_off, dst;
    __device__ __forceinline__ void init(const GemmArgs& a, const GemmCtx& c, int tid) {
        row_bytes = a.K * 2;
        lo_off = a.plane_rows;
        base = reinterpret_cast<const char*>(a.xs + (size_t)c.row0 * a.K);
        const int r = tid >> 4, seg = (tid & 15) * 16;
        off = (uint32_t)(r * row_bytes + seg);
        const int rm = (CT / 2) * 32 + r;
        off_mid = (size_t)(rm < CT * 16 ? rm : lo_off + rm - CT * 16) * row_bytes + seg;
        dst = r * ROWB + seg;
    }
    template <int I0, int I1, int NR>
    __device__ __forceinline__ void load(u32x4 (&br)[NR], int kb) const {
        const char* p = base + (size_t)kb * 256;
#pragma unroll
        for (int i = I0; i < I1; ++i) {
            if (CT % 2 && i == CT / 2) {
                br[i - I0] = *reinterpret_cast<const u32x4*>(p + off_mid);
            } else {
                const int row = i * 32 < CT * 16 ? i * 32 : lo_off + i * 32 - CT * 16;  // high plane, then low plane
                br[i - I0] = *reinterpret_cast<const u32x4*>(p + (size_t)row * row_bytes + off);
            }
        }
    }
    template <int I0, int I1, int NR>
    __device__ __forceinline__ void store(unsigned char* stage, const u32x4 (&br)[NR]) const {
#pragma unroll
        for (int i = I0; i < I1; ++i) *reinterpret_cast<u32x4*>(stage + dst + i * 32 * ROWB) = br[i - I0];
    }
};
// The same from float rows (a single pass): a thread loads eight floats of a row, registers 2 i and 2 i + 1 of the rows 32 i below its first, and
// makes both parts of them on the way to LDS: the bytes are the same, and a launch that splits the rows first is saved ([15360 x 5120] at
// 45 rows, whole call 38.7 us, with it 36.0; at 128 rows 55.2 and 48.4, [4096 x 4096] 27.0 and 22.5).  Rows past the live ones read the
// last of them; it has no others.
template <int CT>
struct GemmStage<CT, true> {
    static constexpr int U = (CT + 1) / 2, N = 2 * U, FIRST = CT > 4 ? (U + 1) / 2 * 2 : N;
    const char* base;
    uint32_t off[U];
    int dst;
    bool half;             // of the last unit of an odd CT, whose rows are 16: this thread has one
    __device__ __forceinline__ void init(const GemmArgs& a, const GemmCtx& c, int tid) {
        base = reinterpret_cast<const char*>(a.x);
        const int r = tid >> 4, seg = tid & 15;
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int row = i * 32 + r < c.Mp ? i * 32 + r : c.Mp - 1;
            off[i] = (uint32_t)row * (uint32_t)(a.K * 4) + seg * 32;
        }
        dst = r * ROWB + seg * 16;
        half = r < 16;
    }
    template <int I0, int I1, int NR>
    __device__ __forceinline__ void load(u32x4 (&br)[NR], int kb) const {
        const char* p = base + (size_t)kb * 512;
#pragma unroll
        for (int i = I0; i < I1; ++i) br[i - I0] = *reinterpret_cast<const u32x4*>(p + off[i / 2] + (i & 1) * 16);
    }
    template <int I0, int I1, int NR>
    __device__ __forceinline__ void store(unsigned char* stage, const u32x4 (&br)[NR]) const {
#pragma unroll
        for (int i = I0; i < I1; i += 2) {
            const u32x4 x = br[i - I0], y = br[i - I0 + 1];
            uint32_t h[4], l[4];
            split_pair(x[0], x[1], h[0], l[0]);
            split_pair(x[2], x[3], h[1], l[1]);
            split_pair(y[0], y[1], h[2], l[2]);
            split_pair(y[2], y[3], h[3], l[3]);
            unsigned char* const d = stage + dst + (i / 2) * 32 * ROWB;
            if (CT % 2 == 0 || i / 2 < U - 1 || half) {
                *reinterpret_cast<u32x4*>(d) = u32x4{h[0], h[1], h[2], h[3]};
                *reinterpret_cast<u32x4*>(d + CT * 16 * ROWB) = u32x4{l[0], l[1], l[2], l[3]};
            }
        }
    }
};

// Four outputs silu(g inv) (u inv) as their two bf16 parts, {high, low} of two neighbours each.  The low part is what the unrounded product has
// beyond the high one, spelled out: left to the compiler it is that only where the product is at hand, and a row's bits would depend on the form.
__device__ __forceinline__ uint4 silu_parts4(f32x4 g, f32x4 u, float inv) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float x = g[i] * inv, y = u[i] * inv, s = x / (1.0f + expf(-x));
        h[i] = f2bf(s * y);
        l[i] = f2bf(fmaf(s, y, -bf2f((uint16_t)h[i])));
    }
    return make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), l[0] | (l[1] << 16), l[2] | (l[3] << 16));
}
__device__ __forceinline__ void store_parts4(uint16_t* xs, int ld, int lo_rows, int m, int n, uint4 p) {
    *reinterpret_cast<uint2*>(xs + (size_t)m * ld + n) = make_uint2(p.x, p.y);
    *reinterpret_cast<uint2*>(xs + (size_t)(lo_rows + m) * ld + n) = make_uint2(p.z, p.w);
}

// Where columns 4 quad .. 4 quad + 3 of a row lie in a piece (in floats): row by row, or as the registers hold it.
__device__ __forceinline__ int piece_offset(int row, int quad, bool by_row) { return by_row ? row * 16 + quad * 4 : (quad * 16 + row) * 4; }

// Partial sum of row block b, or the finished tail where the row block's whole k range was this thread
// block's; then zero for the next row block.  C layout: register r of lane l is weight row 4 (l / 16) + r
// of the tile, activation row l % 16.  A partial sum is left in 1 KB pieces, one per weight tile and column tile: of several passes as the registers
// hold it, lane l's four values at 16 l (as rows of the result, 64 bytes of each of 16 rows per store, the launches took 4 to 6 % longer:
// [22016 x 4096] at 512 rows 154 us, now 144; without any partial sums 132); of a single pass row by row, so that four rows of
// it are 256 bytes in one place for the epilogue (13B shape, three layers at 45 / 64 rows 596 / 641 us as the registers hold it, 588 / 628 so;
// at 200 / 512 rows, two and four passes, 1078 / 1985 and 1089 / 1990).  Of a column tile that is not full only the live rows are left, 64
// neighbouring bytes each ([28672 x 4096] at 17 rows 42.6 us, with all 32 rows 44.9, with the live lanes at 16 l 43.8).
template <int RT, int CT, bool SWI>
__device__ __forceinline__ void gemm_flush(f32x4 (&acc)[RT][CT], const GemmArgs& a, const GemmCtx& c, int b, int q,
                                           const float* s_inv, int lane) {
    const int first = (b * c.KB) / q;
    const bool whole = first == ((b + 1) * c.KB - 1) / q;
    // (the lane's number anew: the addresses that follow from it, forty registers and some spilled, would otherwise be worked out
    // ahead of the main loop and kept from its operands)
    asm volatile("" : "+v"(lane));
    const int li = lane & 15, sub = 4 * (lane >> 4);
    if (SWI && whole) {
#pragma unroll
        for (int t = 0; t < RT / 2; ++t) {
            const int j = gemm_tile<RT, SWI>(c, b, t);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int m = ct * 16 + li;
                if (j >= 0 && m < c.Mp) {
                    const float inv = s_inv[m];
                    const f32x4 g = acc[t][ct], u = acc[RT / 2 + t][ct];
                    store_parts4(a.ys, a.N, a.plane_rows, c.row0 + m, j * 16 + sub, silu_parts4(g, u, inv));
                }
            }
        }
    } else if (!SWI && a.fused && whole) {
        float* const y = a.y + (size_t)c.row0 * a.ldy;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int tile = gemm_tile<RT, SWI>(c, b, t);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int m = ct * 16 + li;
                if (tile >= 0 && m < c.Mp) {
                    const float f = s_inv[m];
                    const f32x4 v = acc[t][ct];
                    *reinterpret_cast<float4*>(y + (size_t)m * a.ldy + tile * 16 + sub) = make_float4(v[0] * f, v[1] * f, v[2] * f, v[3] * f);
                }
            }
        }
    } else {
        float* const p = a.part + (size_t)(c.pass * a.S + c.cid - first) * a.pass_rows * a.rows;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int tile = gemm_tile<RT, SWI>(c, b, t);
            if (tile < 0) continue;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                if (ct * 16 + li < c.Mp)
                    *reinterpret_cast<f32x4*>(p + ((size_t)tile * CT + ct) * 256 + piece_offset(li, lane >> 4, a.n_pass == 1 || c.Mp - ct * 16 < 16)) = acc[t][ct];
        }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[t][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// 512 threads; a wave multiplies its RT weight tiles (16 rows each, registers) with all CT column
// tiles (16 of the pass's rows, bf16 high and low parts, LDS): a 16 RT x 16 CT tile of the result.
//   weights      a ring of D register stages, 32 k each, requested D - 1 steps ahead (WHOLE: the four of a k block together, four to seven ahead)
//   activations  a k block (128 k) ahead through registers into the other LDS stage; one barrier per k block
//   operands     read from LDS PD column tiles before the MFMAs that take them
// What bounds it: a long prompt the power the card gives the matrix cores (random operands: an MFMA-only loop
// reaches 1.81 PFLOP/s, this kernel 1.27 on [28672 x 4096] at 1999 rows; with zeros it reaches 1.69 and the loop
// 2.25), a short one the weight stream.  Operand reads that wait right before their MFMAs, and two tiles per wave
// throughout, took 819 us there against 739; multiplying all 128 rows of a pass whatever it holds took 82 us on
// [27648 x 5120] at 45 rows against 55 (5.1 TB/s) with only the live column tiles.  32 x 32 x 16 MFMAs, which the
// MFMA-only loop prefers by 4 %, were 5 % slower here.
template <int RT, int CT, int D, int PD, bool STREAM, bool SWI, bool WHOLE, bool RAW>
__global__ __launch_bounds__(64 * WPB) void prefill_gemm_kernel(GemmArgs a, int q, int xa) {
    constexpr int STAGE = stage_bytes(CT), UB = D / 4;   // UB: k blocks per turn of the ring
    using Stage = GemmStage<CT, RAW>;
    constexpr int H0 = Stage::FIRST, HN = Stage::N, H1 = HN > H0 ? HN - H0 : 1;
    static_assert(D == 4 || D == 8, "the ring turns over in whole k blocks");
    static_assert(!WHOLE || D == 8, "one k block multiplied, the next requested");
    constexpr int AHEAD = WHOLE ? 4 : D - 1;   // steps requested before the first is multiplied
    static_assert(!SWI || RT % 2 == 0, "gate and up tiles in one wave");
    extern __shared__ __attribute__((aligned(16))) unsigned char bt[];  // [2][STAGE], then PM floats: the rows' RMSNorm scales (fused tails)
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t lane_off = lane * 16;
    GemmCtx c;
    c.wr = __builtin_amdgcn_readfirstlane(tid >> 6);
    c.KB = a.K >> 7; c.n_tiles = a.rows >> 4;
    c.n_out_tiles = SWI ? a.N >> 4 : 0;
    const int nb = (c.n_tiles + WPB * RT - 1) / (WPB * RT);
    const int total = nb * c.KB;  // (checked on the host to fit an int)
    // Thread blocks go to the 8 XCDs round-robin by index.  The blocks that share a range of the
    // weights (same range index, different passes) are given indices of one residue mod 8, so that
    // they meet in one L2 and each L2 fetches an eighth of the layer's weights instead of all of them.
    // Here the 8 XCDs form an xa x (8 / xa) array: range indices are dealt to its rows, passes to its
    // columns, so the weights of a range are fetched by 8 / xa of the L2s and the activations of a
    // pass by xa of them (xa is chosen on the host).
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int xb = 8 / xa, npb = (a.n_pass + xb - 1) / xb;
    c.pass = (j % npb) * xb + xcd / xa;
    c.cid = (j / npb) * xa + xcd % xa;
    if (c.pass >= a.n_pass) return;
    c.row0 = c.pass * a.pass_rows;
    c.Mp = a.M - c.row0 < a.pass_rows ? a.M - c.row0 : a.pass_rows;
    const int it0 = c.cid * q;
    c.it1 = it0 + q < total ? it0 + q : total;
    if (it0 >= c.it1) return;
    f32x4 acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[t][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint4 ar[D][RT];
    Stage sg;
    sg.init(a, c, tid);
    GemmWeights<RT, SWI> w;  // the pair whose last step (WHOLE: all steps) is requested at the first step of a k block; then the pair after it
    w.init(c, a.Wp, it0);
    int b = w.b, kb = w.kb;  // the pair being multiplied
    {
        u32x4 br[HN];
        sg.template load<0, HN>(br, kb);
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            gemm_load_a<RT, STREAM, SWI>(ar[s], w, s & 3, lane_off);
            if ((s & 3) == 3) w.next(c, a.Wp);
        }
        sg.template store<0, HN>(bt, br);
    }
    float* const s_inv = reinterpret_cast<float*>(bt + 2 * STAGE);
    if (a.fused) {  // 1 / rms of this pass's input rows, from the partial sums of squares their producer left
        const int m = tid >> 2, part = tid & 3;
        float t = 0.f;
        if (a.ssq_in && m < c.Mp) {
            const float* const p = a.ssq_in + (size_t)(c.row0 + m) * a.ssq_ld;
            for (int i0 = part; i0 < a.ssq_nb; i0 += 20) {   // (five loads in flight: all of them up to K = 5120)
                float x[5];
#pragma unroll
                for (int k = 0; k < 5; ++k) x[k] = p[i0 + 4 * k < a.ssq_nb ? i0 + 4 * k : 0];
#pragma unroll
                for (int k = 0; k < 5; ++k) t += i0 + 4 * k < a.ssq_nb ? x[k] : 0.f;
            }
        }
        t += __shfl_xor(t, 1, 64);
        t += __shfl_xor(t, 2, 64);
        if (part == 0) s_inv[m] = a.ssq_in ? 1.0f / sqrtf(t / (float)a.K + a.eps) : 1.0f;
    }
    __syncthreads();
    const unsigned char* const rd0 = bt + (lane & 15) * ROWB + (lane >> 4) * 16;
    int buf = 0;  // LDS stage that holds the current k block's activations

    auto k_block = [&](auto phase, int it) {
        constexpr int P = decltype(phase)::value * 4;   // ring position of the k block's first step
        const unsigned char* const src = rd0 + buf * STAGE;
        unsigned char* const dst = bt + (buf ^ 1) * STAGE;
        int kbn = kb + 1 < c.KB ? kb + 1 : 0;            // k block of the next pair (re-read past the range)
        u32x4 br0[H0], br1[H1];
        bf16x8 bh[PD + 1], bl[PD + 1];
        auto read = [&](int n) {                         // operands of column tile n % CT of step n / CT
            const unsigned char* rp = src + (n % CT) * 16 * ROWB + (n / CT) * 64;
            bh[n % (PD + 1)] = *reinterpret_cast<const bf16x8*>(rp);
            bl[n % (PD + 1)] = *reinterpret_cast<const bf16x8*>(rp + CT * 16 * ROWB);
        };
#pragma unroll
        for (int n = 0; n < PD; ++n) read(n);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u == 0) sg.template load<0, H0>(br0, kbn);
            if (HN > H0 && u == 2) {
                sg.template store<0, H0>(dst, br0);
                sg.template load<H0, HN>(br1, kbn);
            }
            if (WHOLE) {
                if (u == 0) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) gemm_load_a<RT, STREAM, SWI>(ar[(P + 4 + s) % D], w, s, lane_off);
                    w.next(c, a.Wp);
                }
            } else {
                gemm_load_a<RT, STREAM, SWI>(ar[(P + u + D - 1) % D], w, (u + 3) & 3, lane_off);
                if (u == 0) w.next(c, a.Wp);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int n = u * CT; n < (u + 1) * CT; ++n) {
                const int ct = n % CT;
                if (n + PD < 4 * CT) read(n + PD);
                const bf16x8 xh = bh[n % (PD + 1)], xl = bl[n % (PD + 1)];
#pragma unroll
                for (int t = 0; t < RT; ++t)
                    acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ar[(P + u) % D][t]), xh, acc[t][ct], 0, 0, 0);
#pragma unroll
                for (int t = 0; t < RT; ++t)
                    acc[t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ar[(P + u) % D][t]), xl, acc[t][ct], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (it + 1 >= c.it1 || kb + 1 == c.KB) gemm_flush<RT, CT, SWI>(acc, a, c, b, q, s_inv, lane);
        if (HN > H0) sg.template store<H0, HN>(dst, br1);
        else sg.template store<0, H0>(dst, br0);
        if (++kb == c.KB) { kb = 0; ++b; }
        buf ^= 1;
        __syncthreads();
    };
    int it = it0;
    for (; it + UB <= c.it1; it += UB) {
        k_block(std::integral_constant<int, 0>{}, it);
        if constexpr (UB > 1) k_block(std::integral_constant<int, 1>{}, it + 1);
    }
    if constexpr (UB > 1) if (it < c.it1) k_block(std::integral_constant<int, 0>{}, it);
}

template <int RT, int CT, int D, int PD, bool STREAM, bool SWI, bool WHOLE, bool RAW>
static hipError_t launch_gemm_t(const GemmArgs& a, int q, int xa, int grid, hipStream_t st) {
    constexpr int LDS = lds_bytes(CT);
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&prefill_gemm_kernel<RT, CT, D, PD, STREAM, SWI, WHOLE, RAW>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    prefill_gemm_kernel<RT, CT, D, PD, STREAM, SWI, WHOLE, RAW><<<grid, 64 * WPB, LDS, st>>>(a, q, xa);
    return hipGetLastError();
}
// D and PD by measurement (45 and 128 rows, 7B to 13B shapes): one tile per wave keeps seven steps in flight
// ([4096 x 4096], 45 rows: 9.6 us), two or four tiles three; reading two operands ahead instead of one
// takes [22016 x 4096] at 512 rows from 200 to 173 us with two tiles, four operands or seven steps no further.  Four tiles take two
// operands as well (three: 4 % slower) since the flush's addresses stay out of the main loop's registers: 1999 rows of the 8B shape, four layers,
// 6.28 -> 6.13 ms, of which 0.03 are the operands.
// A single pass with two tiles and a range of an odd number of k blocks, nine or more, requests the weights a whole k block at a time,
// 4 KB of a tile in one go: thread blocks start their ranges that many 4 KB pieces apart, and an odd distance keeps their
// bursts off each other's channels. Three shapes for each q from 9 to 24 at 16, 45 and 112 rows, step by step / whole: odd q 0.98 to
// 1.07x, 1.03 on the average ([27648 x 5120], q = 17, 45 rows 67.1 -> 63.6 us, [20480 x 6784] 66.0 -> 62.8, [24144 x 3584], q = 11, 1.06x), even
// q 0.96 to 1.02x, 0.99 ([20480 x 8192], q = 20, 45 rows 76.1 and 78.5, [16384 x 8192], q = 16, 62.1 and 64.0). Below nine only gate / up takes two
// tiles, and a range has hardly more than the start, which is longer this way.
template <int RT, int CT, bool STREAM>
static hipError_t launch_gemm_ct(const GemmArgs& a, int q, int xa, int grid, hipStream_t st) {
    constexpr int D = RT == 1 ? 8 : 4, PD = 2;
    if constexpr (STREAM) {
        const bool whole = RT == 2 && q >= 9 && q % 2;
        if (a.x) {
            if constexpr (RT == 2)
                if (whole) return launch_gemm_t<RT, CT, 8, PD, STREAM, false, true, true>(a, q, xa, grid, st);
            return launch_gemm_t<RT, CT, D, PD, STREAM, false, false, true>(a, q, xa, grid, st);
        }
        if constexpr (RT == 2)
            if (whole) return a.fused == 1 + EPI_SWIGLU ? launch_gemm_t<RT, CT, 8, PD, STREAM, true, true, false>(a, q, xa, grid, st)
                                                        : launch_gemm_t<RT, CT, 8, PD, STREAM, false, true, false>(a, q, xa, grid, st);
    }
    if constexpr (RT > 1)
        if (a.fused == 1 + EPI_SWIGLU) return launch_gemm_t<RT, CT, D, PD, STREAM, true, false, false>(a, q, xa, grid, st);
    return launch_gemm_t<RT, CT, D, PD, STREAM, false, false, false>(a, q, xa, grid, st);
}

hipError_t launch_prefill_gemm(const GemmArgs& a_, hipStream_t st) {
    GemmArgs a = a_;
    if (a.rows < 16 || a.rows % 16 || a.K < 128 || a.K % 128 || a.M < 1 || a.n_pass < 1 || a.n_pass > SB_PREFILL_PASSES ||
        a.n_pass != (a.M + PM - 1) / PM || a.plane_rows < a.n_pass * PM)
        return hipErrorInvalidValue;
    if (a.x ? (a.n_pass != 1 || a.fused == 1 + EPI_SWIGLU || ((uintptr_t)a.x & 15) || (size_t)a.M * a.K >= 1u << 30) : !a.xs) return hipErrorInvalidValue;
    const GemmPlan p = gemm_plan(a.rows, a.K, a.n_pass, a.fused == 1 + EPI_SWIGLU);
    a.pass_rows = gemm_pass_rows(a.M, a.n_pass);
    if (a.S != p.smax || (long)p.nb * (a.K >> 7) > 0x3fffffffL) return hipErrorInvalidValue;
    if (a.fused != 0 && a.fused != 1 + EPI_STORE && a.fused != 1 + EPI_SWIGLU) return hipErrorInvalidValue;
    if (a.fused == 1 + EPI_SWIGLU && (a.rows != 2 * a.N || a.N % 16 || !a.ys)) return hipErrorInvalidValue;
    if (a.fused == 1 + EPI_STORE && (a.rows != a.N || !a.y || a.ldy < a.N || a.ldy % 4)) return hipErrorInvalidValue;
    if (a.fused && a.ssq_in && (a.ssq_nb < 1 || a.ssq_ld < a.ssq_nb || a.ssq_ld % 4 || ((uintptr_t)a.ssq_in & 15))) return hipErrorInvalidValue;
    // XCD array shape, by measurement at the 7B shapes: with few passes the weights dominate what the
    // L2s fetch (one L2 per range: 8 % faster than every L2 fetching everything at 4 passes); with many
    // passes the activations weigh as much and 2 x 4 is 2 % ahead of both 8 x 1 and 1 x 8
    const int xa = a.n_pass >= 8 ? 2 : (a.n_pass >= 5 ? 4 : 8);
    const int xb = 8 / xa;
    const int grid = 8 * ((a.n_pass + xb - 1) / xb) * ((p.grid + xa - 1) / xa);
    const int ct = a.pass_rows / 16;
    if (a.n_pass == 1) {
        switch (ct * 4 + p.rt) {
#define SB_GEMM_CASE(CT) \
    case CT * 4 + 1: return launch_gemm_ct<1, CT, true>(a, p.q, xa, grid, st); \
    case CT * 4 + 2: return launch_gemm_ct<2, CT, true>(a, p.q, xa, grid, st);
            SB_GEMM_CASE(1) SB_GEMM_CASE(2) SB_GEMM_CASE(3) SB_GEMM_CASE(4) SB_GEMM_CASE(5) SB_GEMM_CASE(6) SB_GEMM_CASE(7) SB_GEMM_CASE(8)
#undef SB_GEMM_CASE
        }
    } else {
        switch (ct * 8 + p.rt) {   // (more than PM / 2 rows per pass)
#define SB_GEMM_CASE(CT) \
    case CT * 8 + 2: return launch_gemm_ct<2, CT, false>(a, p.q, xa, grid, st); \
    case CT * 8 + 4: return launch_gemm_ct<4, CT, false>(a, p.q, xa, grid, st);
            SB_GEMM_CASE(5) SB_GEMM_CASE(6) SB_GEMM_CASE(7) SB_GEMM_CASE(8)
#undef SB_GEMM_CASE
        }
    }
    return hipErrorInvalidValue;
}

// Partial sums that row block b received: thread blocks first..last of the plan.
struct GemmSplitMap { int rows_per_block, KB, q, pass_rows; };
__device__ __forceinline__ int splits_of(const GemmSplitMap& mp, int n) {
    const uint32_t b = (uint32_t)n / (uint32_t)mp.rows_per_block;   // (pairs are checked on the host to fit an int)
    return (int)(((b + 1) * mp.KB - 1) / (uint32_t)mp.q - b * mp.KB / (uint32_t)mp.q) + 1;
}

// This lane's four values of TN neighbouring weight tiles, one column tile (16 rows): the partial sums added in slot order, U
// slots in flight at a time.  p: the first tile's piece in slot 0, tile_stride and plane in floats.
template <int TN, int U>
__device__ __forceinline__ void sum_splits(f32x4 (&v)[TN], const float* p, size_t tile_stride, size_t plane, int n_splits) {
#pragma unroll
    for (int t = 0; t < TN; ++t) v[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < n_splits; s0 += U) {
        f32x4 x[U][TN];
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                x[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (s0 + i < n_splits) x[i][t] = *reinterpret_cast<const f32x4*>(p + (size_t)(s0 + i) * plane + t * tile_stride);   // (uniform)
            }
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
            for (int t = 0; t < TN; ++t) v[t] += x[i][t];
    }
}
// grid (ceil(N / 256), column tiles of all passes, of FEW quarters of them), 256 threads: a block takes 256 columns of 16 rows, or, FEW, of four, a
// wave four weight tiles of them.  The sums are read as the GEMM left them, a 1 KB piece per load (FEW: 256 bytes of each of four), and what is
// loaded and stored besides is whole cache lines: 16 rows are turned in LDS so that a wave has a row's 256 columns, of
// four rows a wave has 64 neighbouring columns each (1999 rows, N = 6144: launch and GEMM 179 -> 169 us, of which 24 -> 20 here, with rows
// of float4 read from row-major partial sums before).  The residual turns four rows as well: its sums of squares are per 256 columns.
// A row's scale is the same in both forms: its partial sums of squares are added in index order.
template <int EPI, bool FEW>
__global__ __launch_bounds__(256) void prefill_epilogue_kernel(GemmEpiArgs a, GemmSplitMap mp) {
    constexpr int ROWS = FEW ? 4 : 16, TN = FEW ? 1 : 4;   // rows of a block, weight tiles of a lane
    constexpr int LD = 260, U = FEW ? 8 : 2;               // (LDS rows four banks apart)
    constexpr bool TURN = !FEW || EPI == EPI_RESID;
    __shared__ __attribute__((aligned(16))) float turn[TURN ? ROWS * LD : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int CT = mp.pass_rows / 16, tile = FEW ? blockIdx.y >> 2 : blockIdx.y, pass = tile / CT, ct = tile - pass * CT;
    const int r1 = FEW ? (blockIdx.y & 3) * 4 : 0;  // the block's first row in the column tile
    const int m0 = pass * mp.pass_rows + ct * 16;   // the tile's first row, in the super-pass
    const int live = a.M - m0, rows = live - r1;    // live rows from there (a pass before the last is full)
    if (rows <= 0) return;
    const bool fused = (EPI == EPI_SWIGLU || EPI == EPI_STORE) && a.fused;
    const int nb0 = blockIdx.x * 256, nw = nb0 + wave * 64;   // the block's first column, this wave's (its tiles lie in one row block)
    // this lane's row of the block, quad of columns and (FEW: a lane has one of the wave's tiles) first column
    const bool by_row = a.n_pass == 1;              // (a lane's place in a full piece follows the piece's order)
    const int li = (by_row ? lane >> 2 : lane) & (ROWS - 1), lq = (by_row ? lane : FEW ? lane >> 2 : lane >> 4) & 3, nt = FEW ? nw + (lane >> 4) * 16 : nw;
    const bool skip = nt >= a.N || (fused && splits_of(mp, nw) == 1);   // (past the end, or finished by the GEMM)
    // ([28672 x 4096] at 1999 rows, where the GEMM finishes six row blocks in seven, took 46 us with every wave adding up its rows' sums
    // of squares first, 29 without)
    if (fused && __syncthreads_and(skip)) return;
    // Scale of the lane's row, requested before the sums and added up behind them.
    const float* const ssp = a.ssq_in + (size_t)(m0 + r1 + (li < rows ? li : 0)) * a.ssq_ld;
    IndexSum<5> ss;
    if (a.ssq_in) ss.load(ssp, a.ssq_nb);
    f32x4 v[TN], u[TN];
    if (!skip && li < rows) {
        const size_t plane = (size_t)mp.pass_rows * a.rows, tstride = (size_t)CT * 256;
        const float* const p0 = a.part + (size_t)pass * a.S * plane + piece_offset(r1 + li, lq, by_row || live < 16);
        const int sp = splits_of(mp, nw);
        const bool full = nt + TN * 16 <= a.N;
        const auto sum = [&](f32x4 (&x)[TN], int c0, int splits) {
            const float* p = p0 + ((size_t)(c0 / 16) * CT + ct) * 256;
            // (the last wave of a row may have fewer tiles: the first again, not stored)
            sum_splits<TN, U>(x, p, full ? tstride : 0, plane, splits);
            if (TN > 1 && !full)
#pragma unroll
                for (int t = 1; t < TN; ++t)
                    if (nt + t * 16 < a.N) {
                        f32x4 one[1];
                        sum_splits<1, 4>(one, p + t * tstride, 0, plane, splits);
                        x[t] = one[0];
                    }
        };
        // (a row block holds gate and up tiles side by side)
        if constexpr (EPI == EPI_SWIGLU && FEW) {
            f32x4 x[2];
            sum_splits<2, 4>(x, p0 + ((size_t)(nt / 16) * CT + ct) * 256, (size_t)(a.N / 16) * CT * 256, plane, sp);
            v[0] = x[0];
            u[0] = x[1];
        } else {
            sum(v, nt, sp);
            if (EPI == EPI_SWIGLU) sum(u, a.N + nt, sp);
        }
    }
    float inv = 1.0f;
    if (a.ssq_in) inv = 1.0f / sqrtf(ss.sum(ssp, a.ssq_nb) / (float)a.K + a.eps);
    if constexpr (!TURN) {
        if (skip || li >= rows) return;
        const int m = m0 + r1 + li, n = nt + lq * 4;
        if (EPI == EPI_SWIGLU)
            store_parts4(a.ys, a.N, a.plane_rows, m, n, silu_parts4(v[0], u[0], inv));
        else
            *reinterpret_cast<float4*>(a.y + (size_t)m * a.ldy + n) = make_float4(v[0][0] * inv, v[0][1] * inv, v[0][2] * inv, v[0][3] * inv);
        return;
    }
    // this thread's four columns, the same for all of its TN rows (a wave takes a row's 256); what the residual needs of them is on its way while
    // the block turns its tiles
    const int c4 = lane * 4, n = nb0 + c4, m1 = m0 + r1;
    const bool mine = n < a.N && !(fused && splits_of(mp, n) == 1);
    float4 gn = make_float4(0.f, 0.f, 0.f, 0.f), y0[TN];
    if (EPI == EPI_RESID && mine) {
        if (a.nx) gn = *reinterpret_cast<const float4*>(a.gain + n);
#pragma unroll
        for (int k = 0; k < TN; ++k) {
            const int r = wave + k * 4;
            y0[k] = *reinterpret_cast<const float4*>(a.y + (size_t)(m1 + (r < rows ? r : 0)) * a.ldy + n);
        }
    }
    if (!skip) {
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            f32x4 x;   // (gate / up: the parts, so that they are made of the same unrounded products as in the other forms)
            if constexpr (EPI == EPI_SWIGLU) x = __builtin_bit_cast(f32x4, silu_parts4(v[t], u[t], inv));
            else x = v[t] * inv;
            *reinterpret_cast<f32x4*>(turn + li * LD + nt - nb0 + t * 16 + lq * 4) = x;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TN; ++k) {
        const int r = wave + k * 4, m = m1 + r;
        float sq = 0.f;
        if (mine && r < rows) {
            float4 x = *reinterpret_cast<const float4*>(turn + r * LD + c4);
            if (EPI == EPI_SWIGLU) {
                store_parts4(a.ys, a.N, a.plane_rows, m, n, __builtin_bit_cast(uint4, x));
            } else {
                if (EPI == EPI_RESID) {
                    x.x += y0[k].x; x.y += y0[k].y; x.z += y0[k].z; x.w += y0[k].w;
                    if (a.nx) split_store4(a.nx, a.N, a.plane_rows, m, n, make_float4(x.x * gn.x, x.y * gn.y, x.z * gn.z, x.w * gn.w));
                    sq = (x.x * x.x + x.y * x.y) + (x.z * x.z + x.w * x.w);
                }
                *reinterpret_cast<float4*>(a.y + (size_t)m * a.ldy + n) = x;
            }
        }
        if (EPI == EPI_RESID && a.ssq_out) {
            static_assert(SB_PREFILL_SSQ == 256, "a wave of four columns each");
            sq = wave_sum(sq);
            if (lane == 0 && r < rows) a.ssq_out[(size_t)m * a.ssq_ld + blockIdx.x] = sq;
        }
    }
}
template <int EPI, bool FEW>
static void launch_epilogue_t(const GemmEpiArgs& a, const GemmSplitMap& mp, hipStream_t st) {
    const dim3 grid((a.N + 255) / 256, a.n_pass * (mp.pass_rows / 16) * (FEW ? 4 : 1));
    prefill_epilogue_kernel<EPI, FEW><<<grid, 256, 0, st>>>(a, mp);
}

hipError_t launch_prefill_epilogue(const GemmEpiArgs& a, hipStream_t st) {
    if (a.M < 1 || a.N < 1 || a.S < 1 || a.n_pass != (a.M + PM - 1) / PM || a.plane_rows < a.M) return hipErrorInvalidValue;
    if (a.epi == EPI_SWIGLU ? (!a.ys || a.rows != 2 * a.N) : (!a.y || a.rows != a.N)) return hipErrorInvalidValue;
    if (a.ssq_out && (a.N + SB_PREFILL_SSQ - 1) / SB_PREFILL_SSQ > a.ssq_ld) return hipErrorInvalidValue;
    if (a.N % 16 || a.ldy % 4) return hipErrorInvalidValue;
    if (a.ssq_in && (a.ssq_nb < 1 || a.ssq_ld < a.ssq_nb || a.ssq_ld % 4 || ((uintptr_t)a.ssq_in & 15))) return hipErrorInvalidValue;
    const GemmPlan pl = gemm_plan(a.rows, a.K, a.n_pass, a.fused == 1 + EPI_SWIGLU);
    if (a.S != pl.smax) return hipErrorInvalidValue;
    if ((a.fused && a.fused != 1 + a.epi) || (a.epi == EPI_SWIGLU && !a.fused)) return hipErrorInvalidValue;
    const GemmSplitMap mp{a.epi == EPI_SWIGLU ? pl.block_rows / 2 : pl.block_rows, a.K >> 7, pl.q,
                          gemm_pass_rows(a.M, a.n_pass)};
    if (a.epi != EPI_STORE && a.epi != EPI_RESID && a.epi != EPI_SWIGLU) return hipErrorInvalidValue;
    // Blocks of 16 rows read whole pieces and have four tiles' loads on their way in a lane; of four rows there are four times as many, which a
    // launch of few needs.  Several passes leave pieces as the registers hold them, of which four rows are half lines, so the line is lower
    // there.  Four rows / 16, us: GEMM and epilogue [4096 x 4096] at 45 rows (48 blocks of 16) 13.8 / 15.2, [5120 x 13824] 31.2 / 33.4, [22016 x 4096] at
    // 64 rows (344) 44.4 / 45.6, [27648 x 5120] (432) 63.5 / 63.9, [32000 x 1024] at 64 / 128 rows (500 / 1000) 25.2 / 24.4, 36.2 / 33.8; three layers, whole prompt, 8B
    // shape at 17 / 45 / 90 rows (residual 32 / 48 / 96 blocks) 541 / 566, 597 / 617, 724 / 735, 200 (208) 919 / 921, 13B at 200 / 300 / 512 (260 / 420 / 640) 1101 / 1084,
    // 2067 / 2052, 2091 / 2006.
    const long wide_blocks = (long)((a.N + 255) / 256) * a.n_pass * (mp.pass_rows / 16);
    const bool few = wide_blocks < (a.n_pass == 1 ? 512 : 256);
    if (a.epi == EPI_RESID) few ? launch_epilogue_t<EPI_RESID, true>(a, mp, st) : launch_epilogue_t<EPI_RESID, false>(a, mp, st);
    else if (a.epi == EPI_STORE) few ? launch_epilogue_t<EPI_STORE, true>(a, mp, st) : launch_epilogue_t<EPI_STORE, false>(a, mp, st);
    else few ? launch_epilogue_t<EPI_SWIGLU, true>(a, mp, st) : launch_epilogue_t<EPI_SWIGLU, false>(a, mp, st);
    return hipGetLastError();
}

// grid (ceil(d / 2048), M), d % 8 == 0: a thread takes eight neighbouring columns, the 32 lanes of half a wave the 256
// columns of one partial sum of squares (16-byte stores throughout: 1999 rows of 4096 took 37 us with two-byte ones)
template <typename WT>
__global__ __launch_bounds__(256) void prefill_embed_kernel(const WT* __restrict__ E, int vocab, int d,
                                                            const int32_t* __restrict__ tokens, float* __restrict__ H,
                                                            const float* __restrict__ gain, uint16_t* __restrict__ nx,
                                                            int plane_rows, float* __restrict__ ssq_out, int ssq_ld) {
    const int tid = threadIdx.x, m = blockIdx.y, n = blockIdx.x * 2048 + tid * 8;
    int tok = tokens[m];
    if (tok < 0 || tok >= vocab) tok = 0;  // never index outside the table
    float sq = 0.f;
    if (n < d) {
        float v[8], g[8];
        load8(E + (size_t)tok * d + n, v);
        if (nx) load8(gain + n, g);
        store8_split(v, g, H + (size_t)m * d + n, nx, (size_t)m * d + n, (size_t)(plane_rows + m) * d + n);
#pragma unroll
        for (int k = 0; k < 8; ++k) sq += v[k] * v[k];
    }
    if (ssq_out) {
        static_assert(SB_PREFILL_SSQ == 256, "32 lanes of eight columns");
        sq = lanes_sum<16>(sq);
        if ((tid & 31) == 0 && n < d) ssq_out[(size_t)m * ssq_ld + n / SB_PREFILL_SSQ] = sq;
    }
}

hipError_t launch_prefill_embed(const void* E, int32_t w_dtype, int32_t vocab, int32_t d, const int32_t* tokens,
                                int32_t M, float* H, const float* gain, uint16_t* nx, int32_t plane_rows,
                                float* ssq_out, int32_t ssq_ld, hipStream_t st) {
    if (M < 1 || plane_rows < M || d % 8 || (ssq_out && (d + SB_PREFILL_SSQ - 1) / SB_PREFILL_SSQ > ssq_ld)) return hipErrorInvalidValue;
    dim3 grid((d + 2047) / 2048, M);
    if (w_dtype == SB_BF16)
        prefill_embed_kernel<uint16_t><<<grid, 256, 0, st>>>((const uint16_t*)E, vocab, d, tokens, H, gain, nx, plane_rows,
                                                              ssq_out, ssq_ld);
    else
        prefill_embed_kernel<float><<<grid, 256, 0, st>>>((const float*)E, vocab, d, tokens, H, gain, nx, plane_rows,
                                                           ssq_out, ssq_ld);
    return hipGetLastError();
}

__global__ void prefill_split_kernel(const float* __restrict__ x, uint16_t* __restrict__ xs, int plane_rows, int K) {
    const int m = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
    if (i < K) split_store_rows(xs, K, plane_rows, m, i, x[(size_t)m * K + i]);
}
hipError_t launch_prefill_split(const float* x, uint16_t* xs, int32_t plane_rows, int32_t M, int32_t K, hipStream_t st) {
    if (M < 1 || plane_rows < M) return hipErrorInvalidValue;
    prefill_split_kernel<<<dim3((K + 255) / 256, M), 256, 0, st>>>(x, xs, plane_rows, K);
    return hipGetLastError();
}

// ---------------------------------------------------------------- prompt attention
typedef float f32x16 __attribute__((ext_vector_type(16)));
// The prompt's attention for a bf16 cache: first the keys and values of all rows of the
// super-pass go into the cache (rotary embedding on the keys, both rounded to bf16; V
// transposed per page, as everywhere), then one launch computes every row's attention with
// the running-softmax scheme: a wave owns 32 queries of one kv head (rows x the heads of
// its group), walks the keys up to its last row's position and keeps a reference point of the
// exponentials, their sum and the weighted values of each query in registers -- no
// partials in memory, no merge pass.  Both products run on the matrix cores with hi + lo pairs
// for the fp32 side (queries, probabilities) like the decode kernel; a query's result depends
// only on its own column of the accumulators, not on the other queries of the block (three forms of the kernel, chosen in
// launch_prefill_attention from the heads and the number of passes).
//
// grid (pages touched, n_kv_heads), 256 threads: a block writes one head's part of one page --
// K as 16-byte pieces (8 dims of a key), V transposed as 16-byte pieces (8 keys of a dim);
// where the rows cover a page only partly, the V pieces go out key by key.  The eight values of a V piece are loaded without a
// condition, so that they are one round trip and not eight (a condition each was a wait each): 512 rows of 32 heads x 128
// 8.2 -> 6.4 us, 1999 of 8 heads 10.5 -> 8.2.
template <int HD>
__global__ __launch_bounds__(256) void prefill_kv_append_kernel(AttnArgs a) {
    constexpr int HALF = HD / 2, PPK = HD / 8;
    const int g = blockIdx.y, tid = threadIdx.x;
    const int Hq = a.n_heads, Hkv = a.kv.n_kv_heads;
    const int n_total = a.pos0 + a.M;
    const int lpage = a.pos0 / SB_KV_BLOCK + blockIdx.x;
    const int key_lo = lpage * SB_KV_BLOCK > a.pos0 ? lpage * SB_KV_BLOCK : a.pos0;
    const int key_hi = (lpage + 1) * SB_KV_BLOCK < n_total ? (lpage + 1) * SB_KV_BLOCK : n_total;  // keys key_lo .. key_hi - 1
    const size_t page_elems = (size_t)Hkv * SB_KV_BLOCK * HD;
    const size_t page = (size_t)a.kv.table[lpage] * page_elems;
    uint16_t* const kdst = reinterpret_cast<uint16_t*>(a.kv.pool) + (size_t)(a.layer * 2 + 0) * a.kv.n_pages * page_elems + page + (size_t)g * SB_KV_BLOCK * HD;
    uint16_t* const vdst = reinterpret_cast<uint16_t*>(a.kv.pool) + (size_t)(a.layer * 2 + 1) * a.kv.n_pages * page_elems + page + (size_t)g * SB_KV_BLOCK * HD;
    for (int idx = tid; idx < SB_KV_BLOCK * PPK; idx += 256) {
        const int t = idx / PPK, d0 = (idx - t * PPK) * 8;
        const int key = lpage * SB_KV_BLOCK + t;
        if (key < key_lo || key >= key_hi) continue;
        const bool lower = d0 < HALF;
        const int j0 = lower ? d0 : d0 - HALF;
        const float* kp = a.q + (size_t)(key - a.pos0) * a.qkv_rows + (size_t)(Hq + g) * HD;
        const float* cp = a.rope_cos + (size_t)key * HALF + j0;
        const float* sp = a.rope_sin + (size_t)key * HALF + j0;
        uint32_t w[4];
#pragma unroll
        for (int e4 = 0; e4 < 8; e4 += 4) {
            const float4 x = *reinterpret_cast<const float4*>(kp + j0 + e4);
            const float4 y = *reinterpret_cast<const float4*>(kp + j0 + HALF + e4);
            const float4 c = *reinterpret_cast<const float4*>(cp + e4);
            const float4 sn = *reinterpret_cast<const float4*>(sp + e4);
            const float u0 = lower ? x.x * c.x - y.x * sn.x : y.x * c.x + x.x * sn.x;
            const float u1 = lower ? x.y * c.y - y.y * sn.y : y.y * c.y + x.y * sn.y;
            const float u2 = lower ? x.z * c.z - y.z * sn.z : y.z * c.z + x.z * sn.z;
            const float u3 = lower ? x.w * c.w - y.w * sn.w : y.w * c.w + x.w * sn.w;
            w[e4 / 2] = (uint32_t)f2bf(u0) | ((uint32_t)f2bf(u1) << 16);
            w[e4 / 2 + 1] = (uint32_t)f2bf(u2) | ((uint32_t)f2bf(u3) << 16);
        }
        *reinterpret_cast<uint4*>(kdst + (size_t)t * HD + d0) = make_uint4(w[0], w[1], w[2], w[3]);
    }
    for (int idx = tid; idx < HD * 2; idx += 256) {
        const int dim = idx >> 1, t0 = (idx & 1) * 8;
        const int key0 = lpage * SB_KV_BLOCK + t0;
        const float* vp = a.q + (size_t)(Hq + Hkv + g) * HD + dim;
        float f[8];
        uint16_t b[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const int key = key0 + x < key_lo ? key_lo : key0 + x < key_hi ? key0 + x : key_hi - 1;   // (no condition, so the eight go out together)
            f[x] = vp[(size_t)(key - a.pos0) * a.qkv_rows];
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) b[x] = f2bf(f[x]);
        uint16_t* dst = vdst + (size_t)dim * SB_KV_BLOCK + t0;
        if (key0 >= key_lo && key0 + 8 <= key_hi) {
            *reinterpret_cast<uint4*>(dst) = make_uint4(b[0] | ((uint32_t)b[1] << 16), b[2] | ((uint32_t)b[3] << 16), b[4] | ((uint32_t)b[5] << 16), b[6] | ((uint32_t)b[7] << 16));
        } else {
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (key0 + x >= key_lo && key0 + x < key_hi) dst[x] = b[x];
        }
    }
}

// ---- pieces of the prompt attention kernels
// The query (row x head of kv head g's group) of this lane; past the end: zeros, nothing masked, never stored.
struct AttnQuery { int row, head, pos; bool valid; };
__device__ __forceinline__ AttnQuery attn_query(const AttnArgs& a, int g, int qq, int nq_total) {
    const int G = a.n_heads / a.kv.n_kv_heads;
    AttnQuery q;
    q.valid = qq < nq_total;
    q.row = q.valid ? qq / G : 0;
    q.head = g * G + (q.valid ? qq - q.row * G : 0);
    q.pos = q.valid ? a.pos0 + q.row : 0x7fffffff;
    return q;
}
// Its rotated values as hi + lo B operands, scores in units of log 2: this lane has dims 16 ks + 8 lh ..; steps
// ks and ks + HD / 32 are the two ends of the rotation's pairs.
template <int HD>
__device__ __forceinline__ void attn_load_query(const AttnArgs& a, const AttnQuery& qi, int lh, bf16x8 (&qh)[HD / 16], bf16x8 (&ql)[HD / 16]) {
    constexpr int HALF = HD / 2, KS = HD / 16;
    const float* qp = a.q + (size_t)qi.row * a.qkv_rows + (size_t)qi.head * HD + lh * 8;
    const float* cp = a.rope_cos + (size_t)(a.pos0 + qi.row) * HALF + lh * 8;
    const float* sp = a.rope_sin + (size_t)(a.pos0 + qi.row) * HALF + lh * 8;
    const float c2 = 1.4426950408889634f / sqrtf((float)HD);
#pragma unroll
    for (int ks = 0; ks < KS / 2; ++ks) {
        uint32_t h[2][4], l[2][4];
#pragma unroll
        for (int e4 = 0; e4 < 8; e4 += 4) {
            const float4 x = *reinterpret_cast<const float4*>(qp + ks * 16 + e4);
            const float4 y = *reinterpret_cast<const float4*>(qp + ks * 16 + HALF + e4);
            const float4 c = *reinterpret_cast<const float4*>(cp + ks * 16 + e4);
            const float4 sn = *reinterpret_cast<const float4*>(sp + ks * 16 + e4);
            const float xs4[4] = {x.x, x.y, x.z, x.w}, ys4[4] = {y.x, y.y, y.z, y.w};
            const float cs4[4] = {c.x, c.y, c.z, c.w}, sn4[4] = {sn.x, sn.y, sn.z, sn.w};
            float u[2][4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float ua = (xs4[e] * cs4[e] - ys4[e] * sn4[e]) * c2, ub = (ys4[e] * cs4[e] + xs4[e] * sn4[e]) * c2;
                u[0][e] = qi.valid ? ua : 0.f;
                u[1][e] = qi.valid ? ub : 0.f;
            }
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    const uint32_t hp = pack_bf16(u[o][e], u[o][e + 1]);
                    h[o][(e4 + e) / 2] = hp;
                    l[o][(e4 + e) / 2] = pack_bf16(u[o][e] - __uint_as_float(hp << 16), u[o][e + 1] - __uint_as_float(hp & 0xffff0000u));
                }
        }
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            qh[ks + o * (KS / 2)] = __builtin_bit_cast(bf16x8, make_uint4(h[o][0], h[o][1], h[o][2], h[o][3]));
            ql[ks + o * (KS / 2)] = __builtin_bit_cast(bf16x8, make_uint4(l[o][0], l[o][1], l[o][2], l[o][3]));
        }
    }
}
// Running soft-max over KT key tiles of this lane's query (masked scores are -inf): exponentials as hi + lo B
// operands, a page's 16 keys each, this lane's part of their sum, the output rescaled where needed.
// The reference point follows the maximum only when that has grown by more than 2^8: until then the
// exponentials stay below 2^8 and nothing has to be rescaled (any reference point gives the same
// quotient; sums and products are float, the bf16 pairs relative).
template <int KT, int DT>
__device__ __forceinline__ void attn_softmax(const f32x16 (&st)[KT], f32x16 (&o)[DT], float& m_run, float& l_run, bf16x8 (&ph)[2 * KT], bf16x8 (&pl)[2 * KT]) {
    float mx = -__builtin_inff();
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, st[kt][r]);
    mx = lanes_max<32, 32>(mx);
    const float m_new = mx > m_run + 8.0f ? mx : m_run;
    if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
        const float alpha = m_new == m_run ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
        l_run *= alpha;
        m_run = m_new;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
    }
    const float ref = m_new == -__builtin_inff() ? 0.f : m_new;   // (a tile none of whose keys the query sees, before any it does)
    float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
    for (int s = 0; s < KT * 2; ++s) {   // the 16 keys of a page: 8 of them in this lane
        uint32_t hw[4], lw[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float p0 = __builtin_amdgcn_exp2f(st[s >> 1][(s & 1) * 8 + 2 * e] - ref);
            const float p1 = __builtin_amdgcn_exp2f(st[s >> 1][(s & 1) * 8 + 2 * e + 1] - ref);
            sum0 += p0;
            sum1 += p1;
            hw[e] = pack_bf16(p0, p1);
            lw[e] = pack_bf16(p0 - __uint_as_float(hw[e] << 16), p1 - __uint_as_float(hw[e] & 0xffff0000u));
        }
        ph[s] = __builtin_bit_cast(bf16x8, make_uint4(hw[0], hw[1], hw[2], hw[3]));
        pl[s] = __builtin_bit_cast(bf16x8, make_uint4(lw[0], lw[1], lw[2], lw[3]));
    }
    l_run += sum0 + sum1;
}

// grid (n_kv_heads, ceil(M G / 128)), 256 threads.  A wave owns 32 queries and is independent of the
// other waves but for the K/V chunk (64 keys) the block stages in LDS.  Scores are computed transposed,
// S^T = K Q^T in 32 x 32 tiles, so a lane holds, for ONE query (its column), 16 keys of every key tile: the
// running maximum, sum and rescaling are per-lane scalars, completed across the two halves of the wave
// only.  The rows of a key tile are taken in the order (bits 2 and 3 of the key swapped) that leaves a lane
// the exponentials of 8 neighbouring keys in neighbouring registers: they are the B operand of
// O^T += V^T P^T as they stand, and the A operand is one 16-byte piece of the transposed V page.
//
// What bounds it: the matrix cores and, beside them, about 300 vector instructions and 32 quarter-rate
// exponentials per 64 MFMAs; two waves per SIMD cover for each other.  2048 rows behind 2048, 32 heads x 128:
// 189 us, 1.09 PFLOP/s of MFMAs; 300 us as 16 x 16 x 32 tiles of two query tiles per wave, whose operand reads
// were waited for one by one, with 480 vector instructions per chunk and spills.
constexpr int ATTN_CH = 64;   // keys per chunk

template <int HD>
__global__ __launch_bounds__(256, 2) void prefill_attn_kernel(AttnArgs a) {
    constexpr int CH = ATTN_CH, NT = 256, BQ = 128;   // keys of a chunk, threads, queries of a block
    constexpr int KT = CH / 32;              // key tiles of a chunk
    constexpr int KS = HD / 16;              // k steps (16 dims) of the score product
    constexpr int DT = HD / 32;              // 32-dim tiles of the output
    constexpr int PPK = HD / 8;              // 16-byte pieces of a key
    constexpr int SLAB = SB_KV_BLOCK * HD;   // one head's part of a page
    constexpr int NPG = CH / SB_KV_BLOCK;    // pages of a chunk
    constexpr int NL = NPG * SLAB / (NT * 8);  // 16-byte pieces per thread, operand and chunk
    constexpr int PD = 4;                    // operands are read from LDS PD key / dim tiles ahead of their MFMAs
    // Two chunks in LDS, filled by direct global -> LDS loads (lane l of a wave lands 16 l bytes
    // after the wave's base).  Which piece lands where is chosen so that operand reads are free of
    // bank conflicts: a K piece (key, p) sits at piece p ^ f(key) of its key's row; the two
    // halves (8 keys each) of a V row change places in every second group of 8 dims.
    __shared__ __attribute__((aligned(16))) uint16_t k_s[2][CH * HD];
    __shared__ __attribute__((aligned(16))) uint16_t v_s[2][NPG * SLAB];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lh = lane >> 5;
    const int g = blockIdx.x;
    // The longest blocks (last rows) start first; where all blocks are resident at once (two per CU), the second
    // half goes shortest first, so that a CU's two blocks are a long and a short one.
    const int first = (256 + gridDim.x - 1) / gridDim.x, ny = gridDim.y;
    const int qtile = ny <= 2 * first && (int)blockIdx.y >= first ? (int)blockIdx.y - first : ny - 1 - (int)blockIdx.y;
    const int Hq = a.n_heads, Hkv = a.kv.n_kv_heads, G = Hq / Hkv;
    const int nq_total = a.M * G, q0 = qtile * BQ;
    const int n_total = a.pos0 + a.M;
    const int q_last = (q0 + BQ < nq_total ? q0 + BQ : nq_total) - 1;
    const int n_chunks = (a.pos0 + q_last / G) / CH + 1;  // chunks with a key the block's last row sees
    const int wq0 = q0 + wave * 32;                        // the wave's queries: wq0 .. wq1
    const int wq1 = (wq0 + 31 < nq_total - 1) ? wq0 + 31 : nq_total - 1;
    const bool wave_live = wq0 < nq_total;
    const int wpos_min = a.pos0 + wq0 / G, wpos_max = a.pos0 + wq1 / G;
    const size_t page_elems = (size_t)Hkv * SLAB;
    const uint16_t* const kbase = reinterpret_cast<const uint16_t*>(a.kv.pool) + (size_t)(a.layer * 2 + 0) * a.kv.n_pages * page_elems + (size_t)g * SLAB;
    const uint16_t* const vbase = reinterpret_cast<const uint16_t*>(a.kv.pool) + (size_t)(a.layer * 2 + 1) * a.kv.n_pages * page_elems + (size_t)g * SLAB;

    // ---- staging of a chunk: thread -> 16-byte pieces of the chunk's pages (K and V slabs of head g).  A wave's 64
    // pieces lie in one page, so the page is a scalar; lane i < NPG of `pg` holds the i-th page of the chunk
    // issued next (-1: no key there), read one chunk ahead of the issue.
    int pg;
    auto lookup = [&](int chunk) {
        const int page = chunk * NPG + (lane & (NPG - 1));
        pg = (page * SB_KV_BLOCK < n_total) ? a.kv.table[page] : -1;
    };
    auto issue = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int slot0 = i * NT + wave * 64, slot = slot0 + lane;   // the piece's place in LDS
            const int page = __builtin_amdgcn_readlane(pg, slot0 / (SB_KV_BLOCK * PPK));
            const int key = slot / PPK, pp = slot % PPK;
            const int piece = pp ^ (PPK == 16 ? (key & 15) : ((key >> 1) & 7));
            uint16_t* kw = &k_s[buf][slot0 * 8];   // the wave's 64 pieces
            uint16_t* vw = &v_s[buf][slot0 * 8];
            if (page >= 0) {
                const size_t base = (size_t)page * page_elems;
                __builtin_amdgcn_global_load_lds(kbase + base + (uint32_t)((key % SB_KV_BLOCK) * HD + piece * 8), kw, 16, 0, 0);
                __builtin_amdgcn_global_load_lds(vbase + base + (uint32_t)(((slot ^ ((slot >> 4) & 1)) * 8) % SLAB), vw, 16, 0, 0);
            } else {  // past the last key: zeros
                *reinterpret_cast<u32x4*>(kw + lane * 8) = u32x4{0u, 0u, 0u, 0u};
                *reinterpret_cast<u32x4*>(vw + lane * 8) = u32x4{0u, 0u, 0u, 0u};
            }
        }
    };
    lookup(0);
    issue(0);
    lookup(1);

    const AttnQuery qi = attn_query(a, g, wq0 + li, nq_total);
    bf16x8 qh[KS], ql[KS];
    attn_load_query<HD>(a, qi, lh, qh, ql);

    f32x16 o[DT];  // O^T: register r of lane (li, lh) is dim 32 dt + 8 (r / 4) + 4 lh + r % 4 of query li
    float m_run = -__builtin_inff(), l_run = 0.f;  // reference point of the exponentials (log-2 units); this lane's part of the sum
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;

    // row li of a key tile is key (bits 2 and 3 of li swapped)
    const int krow = (li & 19) | ((li & 4) << 1) | ((li & 8) >> 1);
    const int kswz = PPK == 16 ? (krow & 15) : ((krow >> 1) & 7);   // f(key) of this lane's key

    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    for (int chunk = 0; chunk < n_chunks; ++chunk) {
        const int key0 = chunk * CH, buf = chunk & 1;
        if (chunk + 1 < n_chunks) {
            issue(buf ^ 1);
            lookup(chunk + 2);
        }
        if (key0 + CH > n_total) {
            // The last page has slots past the last key; what V holds there would meet a zero
            // probability, and 0 x (stale bits that read as NaN) is not 0: zeros instead.  (K needs
            // nothing: those scores are masked.)  Once per block at most.
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                const int slot = i * NT + tid;
                const int vk = key0 + (slot / (SB_KV_BLOCK * PPK)) * SB_KV_BLOCK + ((slot ^ (slot >> 4)) & 1) * 8;  // keys vk .. vk+7 of one dim
                if (vk < n_total && vk + 8 > n_total) {
                    u32x4 vv = *reinterpret_cast<u32x4*>(&v_s[buf][slot * 8]);
#pragma unroll
                    for (int x = 0; x < 8; ++x)
                        if (vk + x >= n_total) vv[x >> 1] &= (x & 1) ? 0x0000ffffu : 0xffff0000u;
                    *reinterpret_cast<u32x4*>(&v_s[buf][slot * 8]) = vv;
                } else if (vk >= n_total && vk < (n_total + SB_KV_BLOCK - 1) / SB_KV_BLOCK * SB_KV_BLOCK) {
                    *reinterpret_cast<u32x4*>(&v_s[buf][slot * 8]) = u32x4{0u, 0u, 0u, 0u};
                }
            }
            __syncthreads();
        }
        if (wave_live && key0 <= wpos_max) {
            // ---- S^T = K Q^T for the key tiles
            f32x16 st[KT];
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) st[kt][r] = 0.f;
            bf16x8 op[PD];
            auto read_k = [&](int n) {   // step n / KT of key tile n % KT
                op[n % PD] = *reinterpret_cast<const bf16x8*>(&k_s[buf][(((n % KT) * 32 + krow) * PPK + (((n / KT) * 2 + lh) ^ kswz)) * 8]);
            };
#pragma unroll
            for (int n = 0; n < PD; ++n) read_k(n);
#pragma unroll
            for (int n = 0; n < KT * KS; n += KT) {
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) st[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[(n + kt) % PD], qh[n / KT], st[kt], 0, 0, 0);
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) st[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[(n + kt) % PD], ql[n / KT], st[kt], 0, 0, 0);
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
                    if (n + kt + PD < KT * KS) read_k(n + kt + PD);
                __builtin_amdgcn_sched_barrier(0);
            }
            // ---- running soft-max of the query (register r of tile kt: key key0 + 32 kt + 16 (r / 8) + 8 lh + r % 8)
            if (key0 + CH - 1 > wpos_min) {
                const int vis = qi.pos - key0 - 8 * lh;   // last visible key, from this lane's first one
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (kt * 32 + (r >> 3) * 16 + (r & 7) > vis) st[kt][r] = -__builtin_inff();
            }
            auto read_v = [&](int n) {   // page n / DT, dims 32 (n % DT) + li, keys 8 lh ..
                const int slot = ((n % DT) * 32 + li) * 2 + lh;
                op[n % PD] = *reinterpret_cast<const bf16x8*>(&v_s[buf][(n / DT) * SLAB + (slot ^ ((slot >> 4) & 1)) * 8]);
            };
#pragma unroll
            for (int n = 0; n < PD; ++n) read_v(n);
            bf16x8 ph[KT * 2], pl[KT * 2];
            attn_softmax<KT, DT>(st, o, m_run, l_run, ph, pl);
            // ---- O^T += V^T P^T: k step s = page s of the chunk
#pragma unroll
            for (int n = 0; n < KT * 2 * DT; n += 2) {
#pragma unroll
                for (int x = 0; x < 2; ++x) o[(n + x) % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[(n + x) % PD], ph[n / DT], o[(n + x) % DT], 0, 0, 0);
#pragma unroll
                for (int x = 0; x < 2; ++x) o[(n + x) % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[(n + x) % PD], pl[n / DT], o[(n + x) % DT], 0, 0, 0);
#pragma unroll
                for (int x = 0; x < 2; ++x)
                    if (n + x + PD < KT * 2 * DT) read_v(n + x + PD);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_s_waitcnt(0);  // this wave's pieces of the next chunk have landed
        __syncthreads();                // ... and everybody's; every wave is done with this chunk
    }
    // ---- normalise; a lane has 4 neighbouring dims in 4 neighbouring registers
    const float inv_l = 1.0f / lanes_sum<32, 32>(l_run);
    if (!qi.valid) return;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
            const int col = qi.head * HD + dt * 32 + 2 * r + 4 * lh;
            const float4 val = make_float4(o[dt][r] * inv_l, o[dt][r + 1] * inv_l, o[dt][r + 2] * inv_l, o[dt][r + 3] * inv_l);
            if (a.out) *reinterpret_cast<float4*>(a.out + (size_t)qi.row * Hq * HD + col) = val;
            else split_store4(a.out_split, Hq * HD, a.split_rows, qi.row, col, val);
        }
}

// The same for launches that the form above would leave short of blocks: a block owns 32 queries, its W waves
// take the 32-key tiles in turn (tile t to wave t mod W) with a running soft-max each, and the waves'
// results are added in wave order through LDS at the end.  Operands come straight from the cache into
// registers, a tile ahead: the next tile's keys are requested when this tile's scores are done, its values
// when this tile's products are.  grid (n_kv_heads, ceil(M G / 32)).  What bounds it: the chain page
// table -> keys -> scores -> products of a wave's few tiles.  32 heads x 128: 512 rows 15.5 us, 64 rows 6.5 us;
// as blocks of 64 queries that walk all keys 23.7 and 8.4 us.  With the queries loaded without conditions, and the append launch:
// 512 rows 26.2 -> 22.7 us, 64 rows 11.5 -> 9.1, 100 rows of 8 heads x 64 behind 2000 19.7 -> 17.7.
template <int HD, int W>
__global__ __launch_bounds__(64 * W, W == 4 ? 2 : 1) void prefill_attn_split_kernel(AttnArgs a) {
    constexpr int KS = HD / 16, DT = HD / 32, SLAB = SB_KV_BLOCK * HD, NS = DT * 4;
    __shared__ __attribute__((aligned(16))) float o_s[W][NS][64][4];
    __shared__ float m_s[W][32], l_s[W][32];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lh = lane >> 5;
    const int g = blockIdx.x, qtile = gridDim.y - 1 - blockIdx.y;   // (the longest blocks start first)
    const int Hq = a.n_heads, Hkv = a.kv.n_kv_heads, G = Hq / Hkv;
    const int nq_total = a.M * G, q0 = qtile * 32, n_total = a.pos0 + a.M;
    const int q_last = (q0 + 32 < nq_total ? q0 + 32 : nq_total) - 1;
    const int n_tiles = (a.pos0 + q_last / G) / 32 + 1;   // tiles with a key the block's last row sees
    const int pos_min = a.pos0 + q0 / G;
    const size_t page_elems = (size_t)Hkv * SLAB;
    const uint16_t* const kbase = reinterpret_cast<const uint16_t*>(a.kv.pool) + (size_t)(a.layer * 2 + 0) * a.kv.n_pages * page_elems + (size_t)g * SLAB;
    const uint16_t* const vbase = reinterpret_cast<const uint16_t*>(a.kv.pool) + (size_t)(a.layer * 2 + 1) * a.kv.n_pages * page_elems + (size_t)g * SLAB;
    const int krow = (li & 19) | ((li & 4) << 1) | ((li & 8) >> 1);   // row li of a tile is key krow of it
    const uint32_t koff = (uint32_t)((krow & 15) * HD + lh * 8), voff = (uint32_t)(li * SB_KV_BLOCK + lh * 8);
    uint4 kr[KS], vr[2][DT];
    // the two pages of the tile whose operands are requested next; where the second holds no key, the first twice (its
    // scores are masked, its values zeroed).  (Scalars: an array here would be put into LDS.)
    int pg0 = 0, pg1 = 0;
    auto lookup = [&](int t) {
        pg0 = a.kv.table[t * 2];
        pg1 = (t * 2 + 1) * SB_KV_BLOCK < n_total ? a.kv.table[t * 2 + 1] : pg0;
    };
    auto load_k = [&]() {
        const uint16_t* p = kbase + (size_t)((li & 16) ? pg1 : pg0) * page_elems + koff;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kr[ks] = *reinterpret_cast<const uint4*>(p + ks * 16);
    };
    auto load_v = [&](int p0, int p1) {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const uint16_t* p = vbase + (size_t)(x ? p1 : p0) * page_elems + voff;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) vr[x][dt] = *reinterpret_cast<const uint4*>(p + dt * 32 * SB_KV_BLOCK);
        }
    };
    int t = wave;
    const bool any = t < n_tiles;
    if (any) {
        lookup(t);
        load_k();
        load_v(pg0, pg1);
        if (t + W < n_tiles) lookup(t + W);
    }
    // ---- the block's rotated queries, hi + lo in LDS once for all waves (a wave that rotated them by itself would
    // spend longer on that than on a tile), then as B operands in registers
    const AttnQuery qi = attn_query(a, g, q0 + li, nq_total);
    bf16x8 qh[KS], ql[KS];
    {
        constexpr int QS = HD + 8, HALF = HD / 2, TPQ = 2 * W < HALF / 4 ? 2 * W : HALF / 4;   // row stride; threads per query
        uint16_t* const q_hi = reinterpret_cast<uint16_t*>(&o_s[0][0][0][0]);
        uint16_t* const q_lo = q_hi + 32 * QS;
        static_assert(2 * 32 * QS * 2 <= (int)sizeof(o_s), "the queries fit where the results go later");
        const int r = tid / TPQ;
        const AttnQuery qr = attn_query(a, g, q0 + r, nq_total);
        const float* qp = a.q + (size_t)qr.row * a.qkv_rows + (size_t)qr.head * HD;
        const float* cp = a.rope_cos + (size_t)(a.pos0 + qr.row) * HALF;
        const float* sp = a.rope_sin + (size_t)(a.pos0 + qr.row) * HALF;
        const float c2 = 1.4426950408889634f / sqrtf((float)HD);   // scores in units of log 2
        // (all loads first, and a query past the end reads row 0's first head and is blanked afterwards: no load under a condition,
        // which would be a wait each)
        constexpr int NQ = HALF / (4 * TPQ);
        const uint32_t keep = qr.valid ? 0xffffffffu : 0u;
        float4 x[NQ], y[NQ], c[NQ], sn[NQ];
        if (r < 32) {
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                const int j = (i * TPQ + tid % TPQ) * 4;
                x[i] = *reinterpret_cast<const float4*>(qp + j); y[i] = *reinterpret_cast<const float4*>(qp + j + HALF);
                c[i] = *reinterpret_cast<const float4*>(cp + j); sn[i] = *reinterpret_cast<const float4*>(sp + j);
            }
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                const int j = (i * TPQ + tid % TPQ) * 4;
                const float xs4[4] = {x[i].x, x[i].y, x[i].z, x[i].w}, ys4[4] = {y[i].x, y[i].y, y[i].z, y[i].w};
                const float cs4[4] = {c[i].x, c[i].y, c[i].z, c[i].w}, sn4[4] = {sn[i].x, sn[i].y, sn[i].z, sn[i].w};
                float u[2][4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    u[0][e] = (xs4[e] * cs4[e] - ys4[e] * sn4[e]) * c2;
                    u[1][e] = (ys4[e] * cs4[e] + xs4[e] * sn4[e]) * c2;
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    uint32_t h[2], l[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        // (the low part is the remainder of the value, not of the product that it was rounded from)
#pragma clang fp contract(off)
                        h[e] = pack_bf16(u[k][2 * e], u[k][2 * e + 1]);
                        l[e] = pack_bf16(u[k][2 * e] - __uint_as_float(h[e] << 16), u[k][2 * e + 1] - __uint_as_float(h[e] & 0xffff0000u));
                    }
                    *reinterpret_cast<uint2*>(q_hi + r * QS + j + k * HALF) = make_uint2(h[0] & keep, h[1] & keep);
                    *reinterpret_cast<uint2*>(q_lo + r * QS + j + k * HALF) = make_uint2(l[0] & keep, l[1] & keep);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qh[ks] = *reinterpret_cast<const bf16x8*>(q_hi + li * QS + ks * 16 + lh * 8);
            ql[ks] = *reinterpret_cast<const bf16x8*>(q_lo + li * QS + ks * 16 + lh * 8);
        }
    }
    f32x16 o[DT];
    float m_run = -__builtin_inff(), l_run = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    for (; t < n_tiles; t += W) {
        const int key0 = t * 32;
        f32x16 st[1];
#pragma unroll
        for (int r = 0; r < 16; ++r) st[0][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            st[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kr[ks]), qh[ks], st[0], 0, 0, 0);
            st[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kr[ks]), ql[ks], st[0], 0, 0, 0);
        }
        const bool more = t + W < n_tiles;
        const int vp0 = pg0, vp1 = pg1;
        if (more) {
            load_k();
            if (t + 2 * W < n_tiles) lookup(t + 2 * W);
        }
        if (key0 + 31 > pos_min) {
            const int vis = qi.pos - key0 - 8 * lh;   // last visible key, from this lane's first one
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if ((r >> 3) * 16 + (r & 7) > vis) st[0][r] = -__builtin_inff();
        }
        if (key0 + 32 > n_total) {   // slots past the last key: 0 x (stale bits that read as NaN) is not 0
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int live = n_total - key0 - 16 * x - 8 * lh;   // keys of this lane's 8 that exist
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    uint32_t w[4] = {vr[x][dt].x, vr[x][dt].y, vr[x][dt].z, vr[x][dt].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] = 2 * e + 1 < live ? w[e] : (2 * e < live ? w[e] & 0xffffu : 0u);
                    vr[x][dt] = make_uint4(w[0], w[1], w[2], w[3]);
                }
            }
        }
        bf16x8 ph[2], pl[2];
        attn_softmax<1, DT>(st, o, m_run, l_run, ph, pl);
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vr[x][dt]), ph[x], o[dt], 0, 0, 0);
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vr[x][dt]), pl[x], o[dt], 0, 0, 0);
            }
        if (more) load_v(vp0, vp1);
    }
    // ---- the waves' results, brought to one reference point and added in wave order
    l_run = lanes_sum<32, 32>(l_run);
    if (lh == 0) { m_s[wave][li] = m_run; l_s[wave][li] = l_run; }
    __syncthreads();
    float mx = m_s[0][li];   // finite: wave 0 has key 0
#pragma unroll
    for (int w = 1; w < W; ++w) mx = fmaxf(mx, m_s[w][li]);
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) l += l_s[w][li] * __builtin_amdgcn_exp2f(m_s[w][li] - mx);
    if (any) {
        const float f = __builtin_amdgcn_exp2f(m_run - mx);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; r += 4)
                *reinterpret_cast<f32x4*>(o_s[wave][dt * 4 + r / 4][lane]) = f32x4{o[dt][r] * f, o[dt][r + 1] * f, o[dt][r + 2] * f, o[dt][r + 3] * f};
    }
    __syncthreads();
    if (!qi.valid) return;
    const float inv_l = 1.0f / l;
    const int nw = n_tiles < W ? n_tiles : W;   // waves that had a tile
    for (int s = wave; s < NS; s += W) {        // (a lane finishes its own query: slot s holds dims 32 (s / 4) + 8 (s % 4) + 4 lh ..)
        f32x4 v = *reinterpret_cast<const f32x4*>(o_s[0][s][lane]);
        for (int w = 1; w < nw; ++w) {
            const f32x4 u = *reinterpret_cast<const f32x4*>(o_s[w][s][lane]);
            v[0] += u[0]; v[1] += u[1]; v[2] += u[2]; v[3] += u[3];
        }
        const int col = qi.head * HD + (s >> 2) * 32 + (s & 3) * 8 + 4 * lh;
        const float4 val = make_float4(v[0] * inv_l, v[1] * inv_l, v[2] * inv_l, v[3] * inv_l);
        if (a.out) *reinterpret_cast<float4*>(a.out + (size_t)qi.row * Hq * HD + col) = val;
        else split_store4(a.out_split, Hq * HD, a.split_rows, qi.row, col, val);
    }
}

// Four waves of 32 queries share a staged chunk; a launch that this leaves with hardly a block per CU takes the
// key tiles apart instead.  The forms add a query's keys up in different orders, so the choice is made from the heads and
// the number of 128-row passes alone, as the projections' plans are: a row's result does not depend on the rows beside it
// within a launch of as many passes.  Measured with the append launch, apart / shared: 256 blocks of 128 queries 51 / 57 us,
// 320 70 / 72 (99 / 101 behind 700 keys), 384 85 / 82 (124 / 114).  Apart eight / four ways, up to 64 such blocks: head_dim 64
// 53 / 68 us (64 rows behind 8000), 19 / 22 (behind 2048), 12.2 / 12.4 (128 rows behind 300), but 22.8 / 20.9 for 128
// blocks; head_dim 128, where the LDS of eight leaves one block per CU, 37.3 / 36.8 (64 rows behind 2048), 18.5 / 17.9
// (256 rows): four throughout.
enum AttnForm { ATTN_SHARED, ATTN_APART8, ATTN_APART4 };
static AttnForm attn_form(int32_t n_heads, int32_t head_dim, int32_t M) {
    const int64_t blocks = (int64_t)n_heads * ((M + PM - 1) / PM);   // blocks of 128 queries in full passes
    return blocks >= 320 ? ATTN_SHARED : head_dim == 64 && blocks <= 64 ? ATTN_APART8 : ATTN_APART4;
}
int prefill_attention_block_queries(int32_t n_heads, int32_t head_dim, int32_t M) {
    return attn_form(n_heads, head_dim, M) == ATTN_SHARED ? 128 : 32;
}

// M rows at positions pos0.. (bf16 cache): append their K/V, then attention of all rows,
// output as floats (out) or as bf16 planes (out_split / split_rows as in launch_attention).
hipError_t launch_prefill_attention(const AttnArgs& a, hipStream_t st) {
    const int hd = a.kv.head_dim;
    if ((hd != 64 && hd != 128) || a.kv.kv_dtype != SB_BF16 || a.M < 1 || a.n_heads % a.kv.n_kv_heads ||
        (!a.out && (!a.out_split || a.split_rows < a.M)) || !a.rope_cos || !a.rope_sin)
        return hipErrorInvalidValue;
    const int G = a.n_heads / a.kv.n_kv_heads, nq = a.M * G;
    // An output over the input: a block reads its queries before any wave of it stores a result, so the form with the
    // larger blocks takes what those blocks keep apart (one row, or one kv head with up to 128 queries).
    const AttnForm form = attn_out_over_input(a) ? ATTN_SHARED : attn_form(a.n_heads, hd, a.M);
    const bool wide = form == ATTN_SHARED;
    const dim3 agrid((a.pos0 + a.M - 1) / SB_KV_BLOCK - a.pos0 / SB_KV_BLOCK + 1, a.kv.n_kv_heads);
    const dim3 grid(a.kv.n_kv_heads, wide ? (nq + 127) / 128 : (nq + 31) / 32);
    if (hd == 128) {
        prefill_kv_append_kernel<128><<<agrid, 256, 0, st>>>(a);
        if (wide) prefill_attn_kernel<128><<<grid, 256, 0, st>>>(a);
        else prefill_attn_split_kernel<128, 4><<<grid, 256, 0, st>>>(a);
    } else {
        prefill_kv_append_kernel<64><<<agrid, 256, 0, st>>>(a);
        if (wide) prefill_attn_kernel<64><<<grid, 256, 0, st>>>(a);
        else if (form == ATTN_APART8) prefill_attn_split_kernel<64, 8><<<grid, 512, 0, st>>>(a);
        else prefill_attn_split_kernel<64, 4><<<grid, 256, 0, st>>>(a);
    }
    return hipGetLastError();
}

}  // namespace sb
