// Small device helpers shared by the kernel files.
#ifndef SB_DEVICE_UTILS_H
#define SB_DEVICE_UTILS_H

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace sb {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

#define SB_INF __builtin_inff()

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
// float -> bf16, round to nearest even (finite inputs)
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
// two floats -> a packed bf16 pair, round to nearest even (the hardware's conversion)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{a, b}, bf16x2v));
}
// the high and the low bf16 parts of two floats (given as bits), packed; the values split_store leaves
__device__ __forceinline__ void split_pair(uint32_t f0, uint32_t f1, uint32_t& h, uint32_t& l) {
    const float a = __uint_as_float(f0), b = __uint_as_float(f1);
    h = pack_bf16(a, b);
    l = pack_bf16(a - __uint_as_float(h << 16), b - __uint_as_float(h & 0xffff0000u));
}
__device__ __forceinline__ float ldf(const float* p) { return *p; }
__device__ __forceinline__ float ldf(const uint16_t* p) { return bf2f(*p); }

// {v, the value of the lane whose number differs in bit O}: the exchange of a reduction tree, on the vector ALU
// (data-parallel moves inside a row of 16 lanes, row and half-wave swaps across) instead of a round trip
// through the LDS crossbar per step.  For O >= 16 both lanes of a pair get the two values in the same order,
// so what is made of them has to be symmetric.  All lanes of the wave are active.
template <int O>
__device__ __forceinline__ void lane_pair(uint32_t v, uint32_t& x, uint32_t& y) {
    static_assert(O == 1 || O == 2 || O == 4 || O == 8 || O == 16 || O == 32, "one bit of the lane number");
    if constexpr (O >= 16) {
        if constexpr (O == 32) {
            const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
            x = s[0]; y = s[1];
        } else {
            const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
            x = s[0]; y = s[1];
        }
    } else {
        x = v;
        if constexpr (O == 1) y = __builtin_amdgcn_update_dpp(0u, v, 0xB1, 0xf, 0xf, true);        // quad_perm [1,0,3,2]
        else if constexpr (O == 2) y = __builtin_amdgcn_update_dpp(0u, v, 0x4E, 0xf, 0xf, true);   // quad_perm [2,3,0,1]
        else if constexpr (O == 8) y = __builtin_amdgcn_update_dpp(0u, v, 0x128, 0xf, 0xf, true);  // row_ror 8
        else y = __builtin_amdgcn_update_dpp(0u, (uint32_t)__builtin_amdgcn_update_dpp(0u, v, 0x1B, 0xf, 0xf, true), 0x141, 0xf, 0xf, true);  // quads reversed, then row_half_mirror
    }
}
template <int O>
__device__ __forceinline__ void lane_pair(float v, float& x, float& y) {
    uint32_t a, b;
    lane_pair<O>(__float_as_uint(v), a, b);
    x = __uint_as_float(a); y = __uint_as_float(b);
}
// sum / maximum over the lanes whose numbers agree in all bits but HI .. LO, in that order of steps
template <int HI, int LO = 1>
__device__ __forceinline__ float lanes_sum(float v) {
    float x, y;
    lane_pair<HI>(v, x, y);
    if constexpr (HI > LO) return lanes_sum<HI / 2, LO>(x + y);
    else return x + y;
}
template <int HI, int LO = 1>
__device__ __forceinline__ float lanes_max(float v) {
    float x, y;
    lane_pair<HI>(v, x, y);
    if constexpr (HI > LO) return lanes_max<HI / 2, LO>(fmaxf(x, y));
    else return fmaxf(x, y);
}
__device__ __forceinline__ float wave_sum(float v) { return lanes_sum<32>(v); }
__device__ __forceinline__ float wave_max(float v) { return lanes_max<32>(v); }
// maximum with the index that goes with it (ties: the lower index)
template <int HI>
__device__ __forceinline__ void lanes_argmax(float& v, int& i) {
    float x, y;
    uint32_t a, b;
    lane_pair<HI>(v, x, y);
    lane_pair<HI>((uint32_t)i, a, b);
    const bool second = y > x || (y == x && (int)b < (int)a);
    v = second ? y : x;
    i = second ? (int)b : (int)a;
    if constexpr (HI > 1) lanes_argmax<HI / 2>(v, i);
}

// value v of row m, column i -> the two bf16 parts used by the MFMA path:
// rows 0..7 hold the high parts, rows 8..15 the low parts (v ~= hi + lo).
__device__ __forceinline__ void split_store(uint16_t* xs, int ld, int m, int i, float v) {
    uint16_t hi = f2bf(v);
    uint16_t lo = f2bf(v - bf2f(hi));
    xs[(size_t)m * ld + i] = hi;
    xs[(size_t)(8 + m) * ld + i] = lo;
}
// the same with the low parts `lo_rows` rows after the high parts (prompt passes keep more rows)
__device__ __forceinline__ void split_store_rows(uint16_t* xs, int ld, int lo_rows, int m, int i, float v) {
    uint16_t hi = f2bf(v);
    uint16_t lo = f2bf(v - bf2f(hi));
    xs[(size_t)m * ld + i] = hi;
    xs[(size_t)(lo_rows + m) * ld + i] = lo;
}

// four values of row m, columns n..n+3 -> the two bf16 planes (8-byte stores)
__device__ __forceinline__ void split_store4(uint16_t* xs, int ld, int lo_rows, int m, int n, float4 v) {
    const uint16_t h0 = f2bf(v.x), h1 = f2bf(v.y), h2 = f2bf(v.z), h3 = f2bf(v.w);
    const uint16_t l0 = f2bf(v.x - bf2f(h0)), l1 = f2bf(v.y - bf2f(h1)), l2 = f2bf(v.z - bf2f(h2)), l3 = f2bf(v.w - bf2f(h3));
    *reinterpret_cast<uint2*>(xs + (size_t)m * ld + n) = make_uint2((uint32_t)h0 | ((uint32_t)h1 << 16), (uint32_t)h2 | ((uint32_t)h3 << 16));
    *reinterpret_cast<uint2*>(xs + (size_t)(lo_rows + m) * ld + n) =
        make_uint2((uint32_t)l0 | ((uint32_t)l1 << 16), (uint32_t)l2 | ((uint32_t)l3 << 16));
}

__device__ __forceinline__ void unpack8(uint4 v, float (&w)[8]) {
    w[0] = __uint_as_float(v.x << 16); w[1] = __uint_as_float(v.x & 0xffff0000u);
    w[2] = __uint_as_float(v.y << 16); w[3] = __uint_as_float(v.y & 0xffff0000u);
    w[4] = __uint_as_float(v.z << 16); w[5] = __uint_as_float(v.z & 0xffff0000u);
    w[6] = __uint_as_float(v.w << 16); w[7] = __uint_as_float(v.w & 0xffff0000u);
}
__device__ __forceinline__ void load8(const uint16_t* p, float (&w)[8]) {
    uint4 v = *reinterpret_cast<const uint4*>(p);
    w[0] = __uint_as_float(v.x << 16); w[1] = __uint_as_float(v.x & 0xffff0000u);
    w[2] = __uint_as_float(v.y << 16); w[3] = __uint_as_float(v.y & 0xffff0000u);
    w[4] = __uint_as_float(v.z << 16); w[5] = __uint_as_float(v.z & 0xffff0000u);
    w[6] = __uint_as_float(v.w << 16); w[7] = __uint_as_float(v.w & 0xffff0000u);
}
__device__ __forceinline__ void load8(const float* p, float (&w)[8]) {
    float4 a = *reinterpret_cast<const float4*>(p);
    float4 b = *reinterpret_cast<const float4*>(p + 4);
    w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
    w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
}

// eight weights as loaded, to be made floats where they are used
template <typename WT>
struct Piece8 {
    uint4 v[sizeof(WT) / 2];
    __device__ __forceinline__ void load(const WT* p) {
#pragma unroll
        for (int i = 0; i < (int)sizeof(WT) / 2; ++i) v[i] = reinterpret_cast<const uint4*>(p)[i];
    }
    __device__ __forceinline__ void unpack(float (&w)[8]) const {
        const uint32_t u[4] = {v[0].x, v[0].y, v[0].z, v[0].w};
        if constexpr (sizeof(WT) == 2) {
#pragma unroll
            for (int i = 0; i < 4; ++i) { w[2 * i] = __uint_as_float(u[i] << 16); w[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u); }
        } else {
            const uint32_t h[4] = {v[1].x, v[1].y, v[1].z, v[1].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) { w[i] = __uint_as_float(u[i]); w[4 + i] = __uint_as_float(h[i]); }
        }
    }
};

// eight values of a hidden row and, where nx is given, the bf16 parts of gain * value (16-byte stores; the places
// are multiples of 8 elements)
__device__ __forceinline__ void store8_split(const float (&v)[8], const float (&gain)[8], float* h, uint16_t* nx, size_t hi, size_t lo) {
    *reinterpret_cast<float4*>(h) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(h + 4) = make_float4(v[4], v[5], v[6], v[7]);
    if (!nx) return;
    uint32_t a[4], b[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) split_pair(__float_as_uint(v[2 * k] * gain[2 * k]), __float_as_uint(v[2 * k + 1] * gain[2 * k + 1]), a[k], b[k]);
    *reinterpret_cast<uint4*>(nx + hi) = make_uint4(a[0], a[1], a[2], a[3]);
    *reinterpret_cast<uint4*>(nx + lo) = make_uint4(b[0], b[1], b[2], b[3]);
}

__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.0f + expf(-g)) * u; }

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// streaming (non-temporal) 128-bit load: weights are read once per launch
__device__ __forceinline__ uint4 ld_weights_packed(const uint16_t* p) {
    u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

}  // namespace sb
#endif
