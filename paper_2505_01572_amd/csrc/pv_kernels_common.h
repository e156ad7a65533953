// Device helpers and launcher declarations shared by the kernel files.
#pragma once
#include "pv_internal.h"

// storage-type access: float, or bfloat16 kept as raw uint16_t bit patterns
__device__ inline float pv_bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ inline uint16_t pv_f32_to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }     // round to nearest, ties to even (v_cvt_pk_bf16_f32)
__device__ inline float pv_ld(const float *p, size_t i) { return p[i]; }
__device__ inline float pv_ld(const uint16_t *p, size_t i) { return pv_bf16_to_f32(p[i]); }
__device__ inline void pv_st(float *p, size_t i, float v) { p[i] = v; }
__device__ inline void pv_st(uint16_t *p, size_t i, float v) { p[i] = pv_f32_to_bf16(v); }

// The other lane's value combined with the own one, for lanes 16 or 32 apart, or n apart within a row of 16 (a rotation): vector instructions, where a shuffle goes through LDS (some
// 120 cycles each, and they come in chains).
template <typename F> __device__ inline float with_lane32(float v, F op)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <typename F> __device__ inline float with_lane16(float v, F op)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int N, typename F> __device__ inline float with_rotated(float v, F op) { return op(v, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x120 + N, 0xF, 0xF, true))); }
template <typename F> __device__ inline float over_wave(float v, F op)
{
    v = with_rotated<1>(v, op); v = with_rotated<2>(v, op); v = with_rotated<4>(v, op); v = with_rotated<8>(v, op);
    return with_lane32(with_lane16(v, op), op);
}
__device__ inline float op_max(float a, float b) { return fmaxf(a, b); }
__device__ inline float op_add(float a, float b) { return a + b; }
// the value of the lane 16 further on (even rows of 16 lanes) or 16 back (odd ones)
__device__ inline float of_lane16(float v, bool odd)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(odd ? r[0] : r[1]);
}

pv_kv_geom pv_geom(const pv_cache *c);
int pv_k_begin(pv_cache *c, int rows_pad, hipStream_t s);
int pv_k_finish(pv_cache *c, int rows, const float *pmax_val, const int32_t *pmax_idx, int strips, hipStream_t s);
int pv_k_tree_compact(pv_cache *c, hipStream_t s);
int pv_k_set_state(pv_cache *c, int len, int pending, hipStream_t s);
int pv_k_export(pv_cache *c, size_t e0, size_t n, void *d_out, hipStream_t s);
