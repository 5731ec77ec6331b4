// Shared device helpers for the MoC FFN kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moc {

typedef uint16_t bf16_t;  // raw bfloat16 bits in memory

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// Round to nearest, ties to even, with the gfx950 conversion instruction (v_cvt_pk_bf16_f32: two
// values per instruction; the bit arithmetic it replaces took about six).
typedef __bf16 hw_bf16x2_t __attribute__((ext_vector_type(2)));
typedef float hw_f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const hw_f32x2_t f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, hw_bf16x2_t));
}

__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)(pack_bf16x2(f, 0.0f) & 0xFFFFu); }

template <class E> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float load(const float* p) { return *p; }
    static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
    static __device__ __forceinline__ float round(float v) { return v; }
};
template <> struct Elem<bf16_t> {
    static __device__ __forceinline__ float load(const bf16_t* p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void store(bf16_t* p, float v) { *p = f32_to_bf16(v); }
    static __device__ __forceinline__ float round(float v) { return bf16_to_f32(f32_to_bf16(v)); }
};

// SiLU(x) = x / (1 + exp(-x))  (paper Eq. 3) and the logistic function it is built from.
__device__ __forceinline__ float sigmoid_f32(float x) { return 1.0f / (1.0f + expf(-x)); }
__device__ __forceinline__ float silu_f32(float x) { return x * sigmoid_f32(x); }
// What a dense row of SiLU(g) holds on channels that are not selected: SiLU is never below -0.279 (and NaN at -inf).
constexpr float kNotSelected = -1.0f;

// Given the stored g and u of one selected channel and the incoming dz' (Eqs. bp-2, bp-3):
//   s = SiLU(g), z' = s u, du = s dz', dg = u dz' SiLU'(g), SiLU'(g) = sig (1 + g (1 - sig)).
__device__ __forceinline__ void moc_bwd_pointwise(float g, float u, float dz, float& z, float& dg, float& du) {
    float sg = sigmoid_f32(g);
    float s = g * sg;
    z = s * u;
    du = s * dz;
    dg = u * dz * (sg * (1.0f + g * (1.0f - sg)));
}

// Order-preserving map float -> uint32: a > b  <=>  key(a) > key(b); -0.0 and +0.0 share a key.
// Branch-free: flip all bits of negative values and the sign bit of the others; -0.0 lands on
// 0x7FFFFFFF, one below the key of +0.0 and the image of no other value, and is bumped up.
__device__ __forceinline__ uint32_t float_key(float f) {
    const uint32_t u = __float_as_uint(f);
    const uint32_t k = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
    return k + (k == 0x7FFFFFFFu ? 1u : 0u);
}
__device__ __forceinline__ float key_float(uint32_t k) {
    uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    return __uint_as_float(u);
}

// Towards zero; values outside the integer range give its nearest end, NaN gives 0 (a cast leaves both undefined).
__device__ __forceinline__ int cvt_i32(float f) {
    int r;
    asm("v_cvt_i32_f32 %0, %1" : "=v"(r) : "v"(f));
    return r;
}

// min(max(x, lo), hi) for lo <= hi in one instruction; hi uniform.
__device__ __forceinline__ int clamp_i32(int x, int lo, int hi) {
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(lo), "s"(hi));
    return r;
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Number of set bits of `mask` below this lane.
__device__ __forceinline__ int mbcnt(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// Wavefront reductions: lanes l and l ^ 32, then ^ 16, 8, 4, 2, 1 are combined; every lane gets the result.  The exchanges are register
// moves (gfx950's half- and quarter-wavefront swaps, then rotations inside 16 lanes, which reach the xor partner because the values
// repeat with the period of the step before); the same reduction through __shfl_xor costs six trips to LDS.
template <int CTRL> __device__ __forceinline__ float dpp_move(float v) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(v), __float_as_uint(v), CTRL, 0xF, 0xF, false));
}
template <class Op> __device__ __forceinline__ float wave_reduce(float v, const Op& op) {
    {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    v = op(v, dpp_move<0x128>(v));      // row_ror:8
    v = op(v, dpp_move<0x124>(v));      // row_ror:4
    v = op(v, dpp_move<0x122>(v));      // row_ror:2
    v = op(v, dpp_move<0x121>(v));      // row_ror:1
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
    return wave_reduce(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
    return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float wave_min(float v) {
    return wave_reduce(v, [](float a, float b) { return fminf(a, b); });
}

// Reductions whose result only the last lane holds: six instructions instead of about twelve.  Not the order of wave_reduce.
template <int CTRL, int ROWS> __device__ __forceinline__ int dpp_or(int v, int identity) {
    return __builtin_amdgcn_update_dpp(identity, v, CTRL, ROWS, 0xF, false);
}
template <class Op> __device__ __forceinline__ int wave_reduce_last(int v, int identity, const Op& op) {
    v = op(v, dpp_or<0x111, 0xF>(v, identity));      // row_shr:1, 2, 4, 8: the last lane of every 16 has its row's result
    v = op(v, dpp_or<0x112, 0xF>(v, identity));
    v = op(v, dpp_or<0x114, 0xF>(v, identity));
    v = op(v, dpp_or<0x118, 0xF>(v, identity));
    v = op(v, dpp_or<0x142, 0xA>(v, identity));      // row_bcast:15 into rows 1 and 3
    return op(v, dpp_or<0x143, 0xC>(v, identity));   // row_bcast:31 into rows 2 and 3
}

// Inclusive prefix sum over the lanes of a wavefront.
__device__ __forceinline__ int wave_inclusive_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);      // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);      // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);      // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);      // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);      // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);      // row_bcast:31 into rows 2 and 3
    return v;
}

inline int round_up(int v, int m) { return (v + m - 1) / m * m; }
inline size_t round_up_sz(size_t v, size_t m) { return (v + m - 1) / m * m; }

}  // namespace moc
