// Pieces shared by the matrix-core kernel files: MFMA wrapper, split-bf16 operand writers.
#pragma once
#include "pv_kernels_common.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// D(16x16, fp32) += A(16x32, bf16) * B(32x16, bf16).  Lane l holds A[l%16][8*(l/16)..+7],
// B[8*(l/16)..+7][l%16] and D[4*(l/16)+r][l%16], r = 0..3.
__device__ inline f32x4 mfma16(uint4 a, uint4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Loads of data that a kernel reads once (the weight stream): marked non-temporal, so that these lines do not
// push the activation tiles, which every workgroup reads again, out of the L2.  Measured on whole steps: 8B shape
// 3.49 -> 3.30 ms, 70B shape 24.3 -> 22.2 ms.
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
__device__ inline uint4 load_once(const uint4 *p)
{
    const u32x4 v = __builtin_nontemporal_load((const u32x4 *)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ inline uint2 load_once(const uint2 *p)
{
    const u32x2 v = __builtin_nontemporal_load((const u32x2 *)p);
    return make_uint2(v.x, v.y);
}

// A store that goes through to memory at once (sc1), for the partial sums of the shared-tile kernels' K-slices, which workgroups of other XCDs read in the next kernel.  Left dirty in the L2 they are written back
// when the kernel ends, and the next one waits for that: 4 MiB of sums (256 strips, 32 rows, eight slices), K = 4096, projection and sum 12.6 -> 12.0 us, K = 14336 25.3 -> 24.8; 64 rows 16.6 ->
// 15.8 and 30.9 -> 30.3.  Four layers of the 8B shape, 4-bit, 32 rows, 472 -> 458 us
// a step.  One MiB (16 rows, four slices) 10.2 and 10.4: there plain stores, and in k_gemm_wide.  The s_nop: an instruction right behind a store of more than 8 bytes must not write the registers it reads, and the
// compiler, which sees to that for stores of its own, does not look into assembly.
__device__ inline void store_through(float4 *p, f32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(p), "v"(v) : "memory");
}

// One 1 KiB operand tile (64 lanes x 16 bytes) from global memory straight into LDS.  Written in assembly (there is
// no vector output register) because the compiler otherwise waits for every copy in flight before any LDS read; the
// kernels wait for the copies by count (pre_wait).  src is uniform, voff the lane's byte offset behind it.  m0 is put back:
// the compiler may hold a value of its own in it, and a clobber list does not tell it otherwise (m0 is a reserved register there: it
// warns, and reuses the value all the same).  0.3 % of a prompt's time (8B shape, 2048 tokens: 6.68 -> 6.70 ms); 0.9 % with an s_nop behind
// it, which only an instruction that reads m0 next would need: tests/test_lds_copies.py sees to it that there is none, and that no vector instruction writes the scalar registers of src
// in the five states before the copy reads them.
__device__ inline void dma_tile(uint32_t lds, const void *src, uint32_t voff)
{
    uint32_t m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
                 : "=&s"(m0) : "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(voff), "s"(src) : "memory");
}

// N of them in a row, on both sides (the offset in the instruction counts for the LDS address as well): N KiB
template <int N> __device__ inline void dma_tiles(uint32_t lds, const void *src, uint32_t voff)
{
    static_assert(N == 1 || N == 2 || N == 4, "");
    uint32_t m0;
    if constexpr (N == 1) { dma_tile(lds, src, voff); return; }
    else if constexpr (N == 2)
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\tglobal_load_lds_dwordx4 %2, %3 offset:1024\n\ts_mov_b32 m0, %0"
                     : "=&s"(m0) : "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(voff), "s"(src) : "memory");
    else
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\tglobal_load_lds_dwordx4 %2, %3 offset:1024\n\t"
                     "global_load_lds_dwordx4 %2, %3 offset:2048\n\tglobal_load_lds_dwordx4 %2, %3 offset:3072\n\ts_mov_b32 m0, %0"
                     : "=&s"(m0) : "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(voff), "s"(src) : "memory");
}

__device__ inline uint32_t lds_addr(const void *p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p; }

template <typename T> __device__ inline const T *uniform_ptr(const T *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));   // (the builtin returns a signed int)
    return (const T *)((uint64_t)hi << 32 | lo);
}

// ------------------------------------------------------------------------------------------
// Operand writers.  Element (row j, K-index k) of an activation lives at
//   arr[(k/32)*512 + (j%16 + 16*((k%32)/8))*8 + k%8]            (NB == 2: rows in column tiles of 16, tile j/16 has a hi
//   array and behind it a lo array of (K/32)*512 elements each)
//   arr[(k/32)*64*R + (col + 2*R*((k%32)/8))*8 + k%8],  col = j (hi) / j + R (lo)      (NB == 1: a block of R <= 8 rows)
// A packed tile holds the columns of its R rows and nothing else: R lines of 128 bytes.  What every workgroup reads again
// from L2 beside its weights is then in proportion to the rows (with half tiles up to 4 rows and whole ones from 5 on, one row read 4 lines and
// five read 8): one row of the 1B shape (8 layers) 459 -> 449 us a step, five rows of the 7B shape (4 layers) 414 -> 402.
// ------------------------------------------------------------------------------------------
__device__ inline uint16_t bf16_rne(float f) { return pv_f32_to_bf16(f); }

// two numbers as bf16 hi parts, and what is left of them as bf16 lo parts: one conversion instruction per pair
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ inline uint32_t pack_bf16(float a, float b) { const f32x2 v = {a, b}; return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2)); }
__device__ inline void split2(float a, float b, uint32_t &hi, uint32_t &lo)
{
    hi = pack_bf16(a, b);
    lo = pack_bf16(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xFFFF0000u));
}

// four consecutive k (k0 % 4 == 0) of row j; R: rows of the block (packed rows)
template <int NB>
__device__ inline void store_operand4(uint16_t *xop, int K, int j, int k0, const float y[4], int R = 0)
{
    const int tile_elems = NB == 1 ? 64 * R : 512, cols = NB == 1 ? 2 * R : 16;
    const size_t tile = (size_t)(k0 >> 5) * tile_elems, in = (size_t)(((k0 & 31) >> 3) * cols) * 8 + (k0 & 7);
    uint2 vh, vl;
    split2(y[0], y[1], vh.x, vl.x);
    split2(y[2], y[3], vh.y, vl.y);
    if (NB == 1) {
        *(uint2 *)(xop + tile + in + (size_t)j * 8) = vh;
        *(uint2 *)(xop + tile + in + (size_t)(j + R) * 8) = vl;
    } else {
        const size_t arr = (size_t)(K / 32) * 512;
        uint16_t *base = xop + (size_t)(j >> 4) * 2 * arr + tile + in + (size_t)(j & 15) * 8;
        *(uint2 *)base = vh;
        *(uint2 *)(base + arr) = vl;
    }
}

// Where feature e (of hd) of row j (of rows) of query head h lies in the queries' hi and lo arrays: [head][8 features][row][8].  A lane of the attention reads 8 features of one
// row, its neighbours the next rows: 256 bytes for 16 lanes.  With each row's features in one piece every lane had a line of its own, and the address path, which takes a cycle a line and 16
// lanes, a third of k_attn's time (eight rows, groups of four heads).
__device__ inline size_t q_at(int h, int j, int e, int hd, int rows) { return (((size_t)h * (hd >> 3) + (e >> 3)) * rows + j) * 8 + (e & 7); }
