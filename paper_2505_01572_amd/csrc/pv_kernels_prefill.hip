// Long prompts on the matrix path: up to PV_PRE_ROWS rows in one pass over the weights.
//
// The kernels for blocks of up to 64 rows stream every weight once per block, so a prompt in
// 64-row blocks is bound by the weight stream (8B-shaped layer: 0.16 ms per 64 rows, 180
// TFLOP/s).  Here a block has up to 2048 rows and the matrix cores are the bound: the operands
// of a GEMM are as before (16-bit weights in MFMA tile order, activations as bf16 hi + lo pairs,
// fp32 accumulators), but a workgroup owns a rectangle of 128 rows x 128 to 256 features, and both operands
// pass through LDS, loaded by direct global -> LDS copies.  2048 tokens through four 8B-shaped layers:
// 20.7 -> 6.7 ms; the gate/up GEMM then takes 0.73 ms, 1310 TFLOP/s of MFMAs (hi and lo counted).
#include "pv_gemm_epilogue.h"
#include "pv_prefill.h"
#include <algorithm>
#include <type_traits>

// all but the newest N copies of this wave have landed, its LDS reads are done, and so it is for every wave of the workgroup
template <int N> __device__ inline void pre_wait()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// workgroup number -> position in the work list: the 8 XCDs take workgroups in turn, so each gets a contiguous run of the list (its
// workgroups then share operand tiles in that XCD's L2)
__device__ inline int xcd_order(int bid, int total)
{
    const int q = total >> 3, r = total & 7, x = bid & 7;
    return x * q + min(x, r) + (bid >> 3);
}

// tiles of a stage: activations (hi, lo), weights, rounded up so that every wave copies the same number (what is beyond is a strip more, not used)
constexpr int pre_stage_tiles(int br, int bf) { return (2 * br + bf + 7) / 8 * 8; }

// K-tiles added up in one accumulator before it is added to the total.  An accumulator that ran over the whole K would carry
// a rounding error of the size of the operands' own.  Blocks of 64 rows cut K over workgroups when strips are few, into up to 16 runs
// of 8 tiles or more; a prompt's values must not be further off than theirs were without a second level: runs of 8 where those were shorter
// than 16.  Keys and values of a first layer that are not the rounded 64-bit result, 1000 tokens, runs of 16 / runs of 8 / blocks of 64 rows (their
// run): K = 2048 2.16 / 1.76 / 1.76e-4 (8), K = 2080 2.19 / 1.82 / 1.85e-4 (8), K = 4096 2.41 / 1.97 / 2.68e-4 (22), K = 8192 2.62 / 2.05 /
// 4.34e-4 (64).  Runs of 8 take 2 % more time (8B shape, 2048 tokens: 6.60 -> 6.73 ms), hence only where they are needed.
static inline int pre_run(int ktiles, int strips)
{
    const int groups = (strips + 7) / 8, runs = std::min(16, (256 + groups - 1) / groups);
    return ktiles < 16 * runs ? 8 : 16;
}

struct pre_gemm_args {
    const float *rscale;        // RMSNorm scale of each row (QKV, SWIGLU)
    float4 *part;               // K-slice partial sums [slice][strip][row tile][64], or null: one slice
    int mtiles;                 // 16-row tiles of the block
    int rb, fb;                 // rectangles along the rows and the features
    int kps;                    // K-tiles per slice
    int run;                    // K-tiles per accumulator (pre_run): a multiple of 4
    int rows, len;              // rows of the block, and the position of the first
    const float *rowsum; int rsum_rows;   // 4-bit weights: -24 x the operand's row sums, [K-tile][rsum_rows]
    const float *rinv;          // 16-bit float operand: what its rows' sums have to be multiplied with (null: nothing)
};

// What the epilogue of a strip needs from memory.  Length and the row's page are known here (epi_prefetch reads them
// from the step's state in memory, which the stores of the previous strip might have changed, for all the compiler knows).
template <int EPI>
__device__ inline void pre_fetch(const gemm_args &a, const pre_gemm_args &p, int strip, int lane, int ct, int phys, float rj, epi_pre &e)
{
    const int j = ct * 16 + (lane & 15), g = lane >> 4, jr = min(j, p.rows - 1);
    e.rows = p.rows; e.rj = rj; e.pos = p.len + j; e.phys = phys;
    if (EPI == EPI_RESID) {
        const int n = strip * 16 + 4 * g;
        e.xo = *(const float4 *)(a.x + (size_t)jr * a.d + n);
        e.gn = *(const uint2 *)(a.gain_next + n);
    }
    if (EPI == EPI_QKV) {
        const int tt = strip % (a.geom.head_dim >> 4), i = tt * 8 + 4 * (g >> 1);
        const float4 *q = (const float4 *)(a.rope + (size_t)jr * (a.geom.head_dim >> 1) + i);     // (used by q and k strips only)
        const float4 c0 = q[0], c1 = q[1];
        e.cs[0] = make_float2(c0.x, c0.y); e.cs[1] = make_float2(c0.z, c0.w); e.cs[2] = make_float2(c1.x, c1.y); e.cs[3] = make_float2(c1.z, c1.w);
    }
}

template <int EPI>
__device__ inline int pre_page(const gemm_args &a, const pre_gemm_args &p, int lane, int ct)
{
    return EPI == EPI_QKV ? a.page_table[(p.len + min(ct * 16 + (lane & 15), p.rows - 1)) >> a.geom.page_shift] : 0;
}

// SwiGLU of two neighbouring strips at once: the lanes of a pair (16 apart) hold the gate and the up features of both, so
// one takes the first strip and the other the second, instead of both computing the same (expf and the
// division are most of this epilogue).
__device__ inline void pre_swiglu2(const gemm_args &a, const pre_gemm_args &p, int strip, int lane, int ct, float rj, f32x4 v0, f32x4 v1)
{
    const int j = ct * 16 + (lane & 15), g = lane >> 4;
    const bool odd = g & 1;
    float act[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float mine = (odd ? v1[r] : v0[r]) * rj, other = __shfl_xor((odd ? v0[r] : v1[r]) * rj, 16, 64);
        const float gate = odd ? other : mine, up = odd ? mine : other;
        act[r] = gate / (1.0f + expf(-gate)) * up;
    }
    if (j < p.rows) store_operand4<2>(a.xop_act, a.F, j, (strip + odd) * 8 + 4 * (g >> 1), act);
}

// factor of this lane's row: its RMSNorm scale, and what takes the scaling of a 16-bit float operand back
template <int EPI>
__device__ inline float pre_rowfactor(const pre_gemm_args &p, int lane, int ct)
{
    const int j = min(ct * 16 + (lane & 15), p.rows - 1);
    float v = (EPI == EPI_QKV || EPI == EPI_SWIGLU) ? p.rscale[j] : 1.f;
    if (p.rinv != nullptr) v *= p.rinv[j];
    return v;
}

// Epilogue of one row tile of a wave, whose nf accumulators (strip0 ...) lie in the wave's own piece of LDS (`mine`, at this lane): the loop
// over the strips need not be unrolled then (unrolled, the rotary epilogue of 16 accumulator tiles does not fit the registers).
template <int EPI, int FT>
__device__ inline void pre_epilogue(const gemm_args &a, const pre_gemm_args &p, int slice, int ct, int strip0, int nf, int lane, const f32x4 *mine)
{
    if (p.part != nullptr) {
        for (int f = 0; f < nf; ++f) ((f32x4 *)p.part)[(((size_t)slice * a.nstrips + strip0 + f) * p.mtiles + ct) * 64 + lane] = mine[f * 64];
        return;
    }
    const float rj = pre_rowfactor<EPI>(p, lane, ct);
    const int phys = pre_page<EPI>(a, p, lane, ct);
    if constexpr (EPI == EPI_SWIGLU) {
        int f = 0;
        for (; f + 2 <= nf; f += 2) pre_swiglu2(a, p, strip0 + f, lane, ct, rj, mine[f * 64], mine[(f + 1) * 64]);
        if (f < nf) { epi_pre e; pre_fetch<EPI>(a, p, strip0 + f, lane, ct, phys, rj, e); epi_apply<2, EPI>(a, strip0 + f, lane, mine[f * 64], e, ct); }
    } else {
        constexpr int G = EPI == EPI_RESID ? FT : FT < 4 ? FT : 4;          // the loads of G strips go out together
        for (int f = 0; f < nf; f += G) {
            epi_pre e[G];
#pragma unroll
            for (int u = 0; u < G; ++u) pre_fetch<EPI>(a, p, min(strip0 + f + u, a.nstrips - 1), lane, ct, phys, rj, e[u]);
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (f + u < nf) epi_apply<2, EPI>(a, strip0 + f + u, lane, EPI == EPI_RESID ? mine[(f + u) * 64] * rj : mine[(f + u) * 64], e[u], ct);
        }
    }
}

// ------------------------------------------------------------------------------------------
// The GEMM.  WR x WF waves of a workgroup, each RT row tiles x FT strips: per K-tile a wave
// reads 2 RT + FT operand tiles from LDS for 2 RT FT MFMAs, a workgroup copies 2 WR RT + WF FT
// tiles into it.  NST stages of one K-tile each; the barrier of stage k + 1 sits in front of the last
// row tile's MFMAs of stage k, whose operands are in registers, so the matrix cores have work while
// the next stage's first operands come out of LDS.  One barrier per K-tile.
// 256 x 256 rectangles (half the operand traffic) were 4 % faster where they fill the CUs, but leave no registers
// for the second level of accumulators (pre_run).
// ------------------------------------------------------------------------------------------
template <int WR, int WF, int RT, int FT, int NST, int EPI>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_pre_gemm(const gemm_args a, const pre_gemm_args p)
{
    static_assert(WR * WF == 8 && RT % 2 == 0, "8 waves; row tiles alternate between two operand buffers");
    constexpr int BR = WR * RT, BF = WF * FT, TPS = pre_stage_tiles(BR, BF), NLD = TPS / 8;
    static_assert((2 * BR) % 8 == 0, "a wave's i-th tile is an activation tile in every wave or in none");
    extern __shared__ uint4 pre_lds[];                 // [NST][TPS][64]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wr = wave / WF, wf = wave % WF;
    const int L = xcd_order(blockIdx.x, gridDim.x), per = p.rb * p.fb, slice = L / per, rest = L - slice * per;
    const int ct0 = (rest % p.rb) * BR, fs0 = (rest / p.rb) * BF;           // rows vary fastest
    const int KT = a.ktiles, kt0 = slice * p.kps, n = min(KT - kt0, p.kps); // this slice's K-tiles (not empty: the launch sees to it)
    const size_t arr = (size_t)KT * 64;
    // the tiles this wave copies: activation tiles (row tile, hi | lo) first, then weight tiles; past the end of either the last one again
    const uint4 *src[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int t = wave + 8 * i;
        const uint4 *q = i < 2 * BR / 8 ? a.xop + (size_t)(2 * min(ct0 + (t >> 1), p.mtiles - 1) + (t & 1)) * arr
                                        : a.W + (size_t)min(fs0 + t - 2 * BR, a.nstrips - 1) * arr;
        src[i] = uniform_ptr(q + (size_t)kt0 * 64);
    }
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(pre_lds)) + wave * 1024;
    // tiles [i0, i1) of this wave's share of stage s (K-tile kt0 + s; past the end the last one again: the counts of copies in flight stay constant) into buffer buf
    auto copy = [&](int s, int buf, int i0, int i1) {
        const uint32_t vo = (uint32_t)lane * 16 + (uint32_t)min(s, n - 1) * 1024;
#pragma unroll
        for (int i = 0; i < NLD; ++i) if (i >= i0 && i < i1) dma_tile(lds0 + (uint32_t)(buf * TPS + 8 * i) * 1024, src[i], vo);
    };
    f32x4 acc[RT][FT], tot[RT][FT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int f = 0; f < FT; ++f) acc[r][f] = tot[r][f] = (f32x4){0.f, 0.f, 0.f, 0.f};

    uint4 wa[FT], wb[FT], xh[2], xl[2];
    const uint4 *Lx = pre_lds + (wr * RT * 2) * 64 + lane, *Lw = pre_lds + (2 * BR + wf * FT) * 64 + lane;
    auto read_w = [&](uint4 (&w)[FT], int buf) {
#pragma unroll
        for (int f = 0; f < FT; ++f) w[f] = Lw[buf * TPS * 64 + f * 64];
    };
    auto read_x = [&](int r, int buf) { xh[r & 1] = Lx[buf * TPS * 64 + 2 * r * 64]; xl[r & 1] = Lx[buf * TPS * 64 + (2 * r + 1) * 64]; };
    int buf = 0, fill = NST - 1;                       // buffers of the stage in use and of the one being copied
    auto step = [&](int s, const uint4 (&w)[FT], uint4 (&wn)[FT]) {      // on entry: w and row tile 0 of stage s are in registers (or on their way)
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if (r + 1 < RT) read_x(r + 1, buf);
            else {
                pre_wait<(NST - 2) * NLD>();           // stage s + 1 is there
                fill = buf;
                buf = buf + 1 == NST ? 0 : buf + 1;
                read_w(wn, buf);
                read_x(0, buf);
            }
            // The copies of stage s + NST - 1 go out a few at a time among the MFMAs: issued together behind the barrier they
            // hold up the waves (the address path takes 16 cycles for each of the workgroup's copies).
            constexpr int PER = (NLD + RT - 2) / (RT - 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < FT; ++f) acc[r][f] = mfma16(w[f], xh[r & 1], acc[r][f]);
            __builtin_amdgcn_sched_barrier(0);
            if (r + 1 < RT) copy(s + NST - 1, fill, r * PER, r * PER + (PER + 1) / 2);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < FT; ++f) acc[r][f] = mfma16(w[f], xl[r & 1], acc[r][f]);
            __builtin_amdgcn_sched_barrier(0);
            if (r + 1 < RT) copy(s + NST - 1, fill, r * PER + (PER + 1) / 2, (r + 1) * PER);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) copy(s, s, 0, NLD);
    pre_wait<(NST - 2) * NLD>();
    read_w(wa, 0);
    read_x(0, 0);
    for (int s = 0; s < n;) {
        const int e = min(s + p.run, n);
        for (; s + 2 <= e; s += 2) { step(s, wa, wb); step(s + 1, wb, wa); }
        if (s < e) { step(s, wa, wb); ++s; }
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int f = 0; f < FT; ++f) { tot[r][f] += acc[r][f]; acc[r][f] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
    }

    pre_wait<0>();                                     // every wave is done with the stages, and no copy is on its way
    f32x4 *mine = (f32x4 *)pre_lds + wave * FT * 64 + lane;
    const int strip0 = fs0 + wf * FT, nf = min(FT, a.nstrips - strip0);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int ct = ct0 + wr * RT + r;
        if (ct >= p.mtiles) break;
#pragma unroll
        for (int f = 0; f < FT; ++f) mine[f * 64] = tot[r][f];
        pre_epilogue<EPI, FT>(a, p, slice, ct, strip0, nf, lane, mine);
    }
}

// ------------------------------------------------------------------------------------------
// The same for 4-bit weights (of matrices with scales that k_pre_gemm_h4 below does not hold): 128 rows x 64 FT features, 2 x 4 waves, each 4
// row tiles x FT strips.
// Arithmetic as in k_gemm_q4 (codes enter as 16 + c on top of -24 x the row sums, product taken
// transposed, scaled per K-tile); the row sums of the operand come from k_pre_rowsum.  Per K-tile a
// wave expands FT code tiles (9 vector instructions each) and scales 4 FT products (4 each) beside 8 FT MFMAs: the
// vector ALU is busy 80 % of the time that the matrix cores need, so the products are scaled one group of strips
// behind the MFMAs, and the two waves of a SIMD fill each other's gaps.  1000 tokens through two 70B-shaped layers:
// 11.5 ms in blocks of 64 rows, 7.0 here; gate/up 1.82 ms, 1030 TFLOP/s of MFMAs (FT = 8, without the second level of accumulators: the same).
// In LDS: activation stages of one K-tile, and two buffers of a batch of 4 K-tiles of codes, scales and row sums.
// ------------------------------------------------------------------------------------------
template <int FT> struct pre_q4_shape {
    static constexpr int BR = 8, BF = 4 * FT, NST = 4;
    static constexpr int XT = 2 * BR, CT = BF, ST = BF / 8, RT = 2;        // KiB of a stage's activations; of a batch's codes, scales, row sums
    static constexpr int BT = CT + ST + RT;
    static constexpr int lds = (NST * XT + 2 * BT) * 1024;
};

template <int FT, int EPI>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_pre_gemm_q4(const gemm_args a, const pre_gemm_args p)
{
    using S = pre_q4_shape<FT>;
    constexpr int RT = 4, WF = 4, NST = S::NST, NX = S::XT / 8, NC = S::CT / 8, BC = NC + 1;    // copies of a wave: NX a stage, BC a batch
    static_assert(S::ST + S::RT <= 8 && FT % 2 == 0, "one scale or row-sum tile a wave");
    extern __shared__ uint4 pre_lds[];                 // [NST][XT][64], then [2][BT][64]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, fl = lane & 15;
    const int wr = wave / WF, wf = wave % WF;
    const int L = xcd_order(blockIdx.x, gridDim.x), per = p.rb * p.fb, slice = L / per, rest = L - slice * per;
    const int ct0 = (rest % p.rb) * S::BR, fs0 = (rest / p.rb) * S::BF;
    const int KT = a.ktiles, kt0 = slice * p.kps, n = min(KT - kt0, p.kps), nb = n >> 2;        // K-tiles and batches of this slice (whole batches, not empty)
    const size_t arr = (size_t)KT * 64, qstrip = (size_t)(KT >> 2) * PV_Q4_BATCH;
    const char *W = (const char *)a.W + (size_t)(kt0 >> 2) * PV_Q4_BATCH;
    const uint4 *xsrc[NX];
    const char *csrc[NC];
#pragma unroll
    for (int i = 0; i < NX; ++i) { const int t = wave + 8 * i; xsrc[i] = uniform_ptr(a.xop + (size_t)(2 * min(ct0 + (t >> 1), p.mtiles - 1) + (t & 1)) * arr + (size_t)kt0 * 64); }
#pragma unroll
    for (int i = 0; i < NC; ++i) csrc[i] = uniform_ptr(W + (size_t)min(fs0 + wave + 8 * i, a.nstrips - 1) * qstrip);
    // the wave's scale tile (8 strips x 128 bytes) or row-sum tile (2 K-tiles x 128 rows); the waves that are left over repeat the first
    const int small = wave < S::ST + S::RT ? wave : 0;
    const char *ssrc; uint32_t soff, sstep;
    if (small < S::ST) {
        ssrc = W + (size_t)fs0 * qstrip; sstep = PV_Q4_BATCH;
        soff = (uint32_t)((min(fs0 + small * 8 + (lane >> 3), a.nstrips - 1) - fs0) * qstrip) + 1024 + (lane & 7) * 16;
    } else {
        ssrc = (const char *)(p.rowsum + (size_t)kt0 * p.rsum_rows + ct0 * 16); sstep = 4 * p.rsum_rows * 4;
        soff = (uint32_t)(((small - S::ST) * 2 + (lane >> 5)) * p.rsum_rows * 4 + (lane & 31) * 16);
    }
    ssrc = uniform_ptr(ssrc);
    const uint32_t ldsx = __builtin_amdgcn_readfirstlane(lds_addr(pre_lds)) + wave * 1024, ldsb = ldsx + NST * S::XT * 1024;
    auto copy_x = [&](int s, int buf) {
        const uint32_t vo = (uint32_t)lane * 16 + (uint32_t)min(s, n - 1) * 1024;
#pragma unroll
        for (int i = 0; i < NX; ++i) dma_tile(ldsx + (uint32_t)(buf * S::XT + 8 * i) * 1024, xsrc[i], vo);
    };
    auto copy_b = [&](int b, int i0, int i1) {         // copies i0 .. i1 - 1 of batch b (past the end: the last one again)
        const uint32_t bt = min(b, nb - 1), base = ldsb + (uint32_t)((b & 1) * S::BT) * 1024;
#pragma unroll
        for (int i = 0; i < NC; ++i) if (i >= i0 && i < i1) dma_tile(base + 8 * i * 1024, csrc[i], (uint32_t)lane * 16 + bt * PV_Q4_BATCH);
        if (NC >= i0 && NC < i1) dma_tile(base + (uint32_t)(S::CT + small - wave) * 1024, ssrc, soff + bt * sstep);
    };
    f32x4 acc[RT][FT], tot[RT][FT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int f = 0; f < FT; ++f) acc[r][f] = tot[r][f] = (f32x4){0.f, 0.f, 0.f, 0.f};

    uint4 w[FT], xh[2], xl[2];
    f32x4 t0[2];
    uint2 cd[FT]; uint32_t sp[FT];                     // codes and scales of two K-tiles
    float sc[FT];
    const uint4 *Lx = pre_lds + (wr * RT * 2) * 64 + lane;
    const char *Lb = (const char *)(pre_lds + NST * S::XT * 64);
    auto read_x = [&](int r, int buf, int bb, int u) {
        xh[r & 1] = Lx[buf * S::XT * 64 + 2 * r * 64]; xl[r & 1] = Lx[buf * S::XT * 64 + (2 * r + 1) * 64];
        t0[r & 1] = *(const f32x4 *)(Lb + (bb * S::BT + S::CT + S::ST) * 1024 + u * 512 + ((wr * RT + r) * 16 + 4 * g) * 4);
    };
    auto read_c = [&](int bb, int h) {
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            const int st = wf * FT + f;
            cd[f] = *(const uint2 *)(Lb + (bb * S::BT + st) * 1024 + lane * 16 + h * 8);
            sp[f] = *(const uint32_t *)(Lb + (bb * S::BT + S::CT) * 1024 + st * 128 + fl * 8 + h * 4);
        }
    };
    int buf = 0, fill = NST - 1;
    constexpr int G = 2, NG = FT / G;                  // strips whose products are in flight together (more do not fit the registers)
    auto step = [&](int b, auto uc) {                  // K-tile 4 b + u; on entry its row tile 0 and codes are in registers (or on their way)
        constexpr int u = decltype(uc)::value;
        const int s = 4 * b + u, bb = b & 1;
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            const uint32_t c = (u & 1) ? cd[f].y : cd[f].x;
            w[f] = make_uint4(((c << 3) & 0x00780078u) | 0x41804180u, ((c >> 1) & 0x00780078u) | 0x41804180u,
                              ((c >> 5) & 0x00780078u) | 0x41804180u, ((c >> 9) & 0x00780078u) | 0x41804180u);
            sc[f] = __uint_as_float((u & 1) ? (sp[f] & 0xFFFF0000u) : (sp[f] << 16));
        }
        f32x4 T[2][G];
        auto scale = [&](int r, int h, const f32x4 (&t)[G]) {
#pragma unroll
            for (int f = 0; f < G; ++f)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[r][h * G + f][q] = fmaf(sc[h * G + f], t[f][q], acc[r][h * G + f][q]);
        };
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if (r + 1 < RT) read_x(r + 1, buf, bb, u);
            else {
                if (u == 3) pre_wait<(NST - 2) * NX>(); else pre_wait<(NST - 2) * NX + BC>();   // stage s + 1 is there (and with u = 3 the next batch)
                fill = buf;
                buf = buf + 1 == NST ? 0 : buf + 1;
                read_x(0, buf, u == 3 ? bb ^ 1 : bb, (u + 1) & 3);
                if (u & 1) read_c(u == 3 ? bb ^ 1 : bb, u == 3 ? 0 : 1);
            }
#pragma unroll
            for (int h = 0; h < NG; ++h) {
                const int k = (r * NG + h) & 1;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int f = 0; f < G; ++f) T[k][f] = mfma16(xh[r & 1], w[h * G + f], t0[r & 1]);
#pragma unroll
                for (int f = 0; f < G; ++f) T[k][f] = mfma16(xl[r & 1], w[h * G + f], T[k][f]);
                __builtin_amdgcn_sched_barrier(0);
                if (r + h > 0) scale(h ? r : r - 1, h ? h - 1 : NG - 1, T[k ^ 1]);      // the group before this one
                __builtin_amdgcn_sched_barrier(0);
                if (r == 0 && h == 0) copy_x(s + NST - 1, fill);
                if (u == 0 && r == 1 && h < 2) copy_b(b + 1, h ? (BC + 2) / 3 : 0, h ? 2 * ((BC + 2) / 3) : (BC + 2) / 3);
                if (u == 0 && r == 2 && h == 0) copy_b(b + 1, 2 * ((BC + 2) / 3), BC);
            }
        }
        scale(RT - 1, NG - 1, T[(RT * NG - 1) & 1]);
    };
    copy_b(0, 0, BC);
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) copy_x(s, s);
    pre_wait<(NST - 2) * NX>();
    read_c(0, 0);
    read_x(0, 0, 0, 0);
    for (int b = 0, left = p.run >> 2; b < nb; ++b) {
        step(b, std::integral_constant<int, 0>()); step(b, std::integral_constant<int, 1>());
        step(b, std::integral_constant<int, 2>()); step(b, std::integral_constant<int, 3>());
        if (--left == 0 || b + 1 == nb) {
            left = p.run >> 2;
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int f = 0; f < FT; ++f) { tot[r][f] += acc[r][f]; acc[r][f] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
        }
    }
    pre_wait<0>();
    // an accumulator is (row 4 g + r, feature fl) of lane (g, fl); the epilogue takes (feature 4 g' + r', row j) from lane (g', j): turned on the way through LDS
    float *turn = (float *)((f32x4 *)pre_lds + wave * FT * 64);
    const int strip0 = fs0 + wf * FT, nf = min(FT, a.nstrips - strip0);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int ct = ct0 + wr * RT + r;
        if (ct >= p.mtiles) break;
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int q = 0; q < 4; ++q) turn[f * 256 + ((fl >> 2) * 16 + 4 * g + q) * 4 + (fl & 3)] = tot[r][f][q];
        pre_epilogue<EPI, FT>(a, p, slice, ct, strip0, nf, lane, (const f32x4 *)turn + lane);
    }
}

// -24 x the sum over the 32 features of each (K-tile, row) of an operand, [K-tile][rows of all row tiles].  One wave per K-tile and row tile.
__global__ void __launch_bounds__(256)
k_pre_rowsum(const uint4 *xop, int ktiles, float *rowsum, int rsum_rows)
{
    const int lane = threadIdx.x & 63, kt = blockIdx.x * 4 + (threadIdx.x >> 6), ct = blockIdx.y;
    if (kt >= ktiles) return;
    const uint4 *q = xop + ((size_t)2 * ct * ktiles + kt) * 64 + lane;
    const uint4 hi = q[0], lo = q[(size_t)ktiles * 64];
    auto sum2 = [](uint32_t v) { return __uint_as_float(v << 16) + __uint_as_float(v & 0xFFFF0000u); };
    float v = ((sum2(hi.x) + sum2(hi.y)) + (sum2(hi.z) + sum2(hi.w))) + ((sum2(lo.x) + sum2(lo.y)) + (sum2(lo.z) + sum2(lo.w)));
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (lane < 16) rowsum[(size_t)kt * rsum_rows + ct * 16 + lane] = -24.f * v;
}

// ------------------------------------------------------------------------------------------
// 4-bit weights as 16-bit floats.  (c - 8) x scale has at most 11 significant bits (3 of the code, 8 of the bf16
// scale), which is what f16 holds, so for scales inside f16's range the weight itself enters the matrix core, exactly,
// and nothing is left to do per product: the vector ALU, which bounds k_pre_gemm_q4 (scaling every product), only
// expands the codes.  The activations become f16 hi + lo pairs of rows that are scaled by a power of two so that a
// row's largest value lies in [2^14, 2^15); the rows' sums are scaled back in the epilogue.  Such a pair holds the 16 bits of the bf16
// pair it is made from exactly down to 2^-22 of the row's largest value; smaller elements are off by up to 2^-39 of that value (the
// step of f16's subnormals is 2^-24), which is 2^22 times less than the largest element's own rounding to 16 bits.  128
// rows x 64 FT features, 2 x 4 waves of 4 row tiles x FT strips; the codes of K-tile k + 1 are expanded, one strip per row tile,
// among the MFMAs of K-tile k.  70B-shaped gate/up, 1000 rows: 1.82 -> 1.71 ms (16-bit weights: 1.45), and fewer K/V
// values off by a rounding step against 64 bits (1.43 % for 1.66 %, 1.62 % in blocks of 64 rows).
// ------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;

__device__ inline f32x4 mfma16h(uint4 a, uint4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

template <int FT> struct pre_h4_shape {
    static constexpr int BR = 8, BF = 4 * FT, NST = 4;
    static constexpr int XT = 2 * BR, CT = 16, ST = 2, BT = CT + ST;           // KiB of a stage's activations; of a batch's codes and scales (of 16 strips, also where fewer are used)
    static constexpr int lds = (NST * XT + 2 * BT) * 1024;
};

template <int FT, int EPI>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_pre_gemm_h4(const gemm_args a, const pre_gemm_args p)
{
    using S = pre_h4_shape<FT>;
    constexpr int RT = 4, WF = 4, NST = S::NST, NX = S::XT / 8, NC = S::CT / 8, BC = NC + 1;    // copies of a wave: NX a stage, BC a batch
    static_assert(FT <= RT && S::BF <= S::CT, "a strip is expanded beside each row tile");
    extern __shared__ uint4 pre_lds[];                 // [NST][XT][64], then [2][BT][64]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, fl = lane & 15;
    const int wr = wave / WF, wf = wave % WF;
    const int L = xcd_order(blockIdx.x, gridDim.x), per = p.rb * p.fb, slice = L / per, rest = L - slice * per;
    const int ct0 = (rest % p.rb) * S::BR, fs0 = (rest / p.rb) * S::BF;
    const int KT = a.ktiles, kt0 = slice * p.kps, n = min(KT - kt0, p.kps), nb = n >> 2;        // K-tiles and batches of this slice (whole batches, not empty)
    const size_t arr = (size_t)KT * 64, qstrip = (size_t)(KT >> 2) * PV_Q4_BATCH;
    const char *W = (const char *)a.W + (size_t)(kt0 >> 2) * PV_Q4_BATCH;
    const uint4 *xsrc[NX];
    const char *csrc[NC];
#pragma unroll
    for (int i = 0; i < NX; ++i) { const int t = wave + 8 * i; xsrc[i] = uniform_ptr(a.xop + (size_t)(2 * min(ct0 + (t >> 1), p.mtiles - 1) + (t & 1)) * arr + (size_t)kt0 * 64); }
#pragma unroll
    for (int i = 0; i < NC; ++i) csrc[i] = uniform_ptr(W + (size_t)min(fs0 + wave + 8 * i, a.nstrips - 1) * qstrip);
    const int small = wave < S::ST ? wave : 0;         // the wave's scale tile (8 strips x 128 bytes); the waves that are left over repeat the first
    const char *ssrc = uniform_ptr(W + (size_t)fs0 * qstrip);
    const uint32_t soff = (uint32_t)((min(fs0 + small * 8 + (lane >> 3), a.nstrips - 1) - fs0) * qstrip) + 1024 + (lane & 7) * 16;
    const uint32_t ldsx = __builtin_amdgcn_readfirstlane(lds_addr(pre_lds)) + wave * 1024, ldsb = ldsx + NST * S::XT * 1024;
    auto copy_x = [&](int s, int buf) {
        const uint32_t vo = (uint32_t)lane * 16 + (uint32_t)min(s, n - 1) * 1024;
#pragma unroll
        for (int i = 0; i < NX; ++i) dma_tile(ldsx + (uint32_t)(buf * S::XT + 8 * i) * 1024, xsrc[i], vo);
    };
    auto copy_b = [&](int b, int i0, int i1) {         // copies i0 .. i1 - 1 of batch b (past the end: the last one again)
        const uint32_t bt = min(b, nb - 1), base = ldsb + (uint32_t)((b & 1) * S::BT) * 1024;
#pragma unroll
        for (int i = 0; i < NC; ++i) if (i >= i0 && i < i1) dma_tile(base + 8 * i * 1024, csrc[i], (uint32_t)lane * 16 + bt * PV_Q4_BATCH);
        if (NC >= i0 && NC < i1) dma_tile(base + (uint32_t)(S::CT + small - wave) * 1024, ssrc, soff + bt * PV_Q4_BATCH);
    };
    f32x4 acc[RT][FT], tot[RT][FT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int f = 0; f < FT; ++f) acc[r][f] = tot[r][f] = (f32x4){0.f, 0.f, 0.f, 0.f};

    uint4 wa[FT], wb[FT], xh[2], xl[2];
    uint2 cd[FT]; uint32_t sp[FT];                     // codes and scales of two K-tiles
    const uint4 *Lx = pre_lds + (wr * RT * 2) * 64 + lane;
    const char *Lb = (const char *)(pre_lds + NST * S::XT * 64);
    auto read_x = [&](int r, int buf) { xh[r & 1] = Lx[buf * S::XT * 64 + 2 * r * 64]; xl[r & 1] = Lx[buf * S::XT * 64 + (2 * r + 1) * 64]; };
    auto read_c = [&](int bb, int h) {
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            const int st = wf * FT + f;
            cd[f] = *(const uint2 *)(Lb + (bb * S::BT + st) * 1024 + lane * 16 + h * 8);
            sp[f] = *(const uint32_t *)(Lb + (bb * S::BT + S::CT) * 1024 + st * 128 + fl * 8 + h * 4);
        }
    };
    // the codes of one strip and K-tile (the odd or the even one of the pair) as weights.  A nibble OR-ed into 1024.0 (0x6400) counts ones in the lowest
    // mantissa bits and sixteens in the next: 1024 + c and 1024 + 16 c; less 1032 or 1152 that is c - 8 or 16 (c - 8), exactly (integers to
    // floats without a conversion instruction, as in Y. J. Kim et al., "Who Says Elephants Can't Run", arXiv 2211.10017, for 8- and 4-bit weights)
    auto expand = [&](int f, bool odd) {
        const uint32_t c = odd ? cd[f].y : cd[f].x, c8 = c >> 8;
        const float sc = __uint_as_float(odd ? (sp[f] & 0xFFFF0000u) : (sp[f] << 16));
        const f16x2 s1 = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(sc, sc)), s16 = s1 * (f16x2){(_Float16)0.0625f, (_Float16)0.0625f};
        const f16x2 one = {(_Float16)-1032.f, (_Float16)-1032.f}, sixteen = {(_Float16)-1152.f, (_Float16)-1152.f};
        auto low = [&](uint32_t v) { return __builtin_bit_cast(uint32_t, (__builtin_bit_cast(f16x2, (v & 0x000F000Fu) | 0x64006400u) + one) * s1); };
        auto high = [&](uint32_t v) { return __builtin_bit_cast(uint32_t, (__builtin_bit_cast(f16x2, (v & 0x00F000F0u) | 0x64006400u) + sixteen) * s16); };
        return make_uint4(low(c), high(c), low(c8), high(c8));
    };
    int buf = 0, fill = NST - 1;
    auto step = [&](int b, auto uc, const uint4 (&w)[FT], uint4 (&wn)[FT]) {   // K-tile 4 b + u; on entry its weights are expanded and row tile 0 is in registers (or on its way)
        constexpr int u = decltype(uc)::value;
        const int s = 4 * b + u, bb = b & 1;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if (r + 1 < RT) read_x(r + 1, buf);
            else {
                if (u >= 2) pre_wait<(NST - 2) * NX>(); else pre_wait<(NST - 2) * NX + BC>();   // stage s + 1 is there; from u = 2 on the next batch is, too
                fill = buf;
                buf = buf + 1 == NST ? 0 : buf + 1;
                read_x(0, buf);
            }
            if (r == 0 && (u & 1)) read_c(u == 3 ? bb ^ 1 : bb, u == 3 ? 0 : 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < FT; ++f) acc[r][f] = mfma16h(w[f], xh[r & 1], acc[r][f]);
            __builtin_amdgcn_sched_barrier(0);
            if (r == 0) copy_x(s + NST - 1, fill);
            if (u == 0 && r == 1) copy_b(b + 1, 0, 1);
            if (u == 0 && r == 2) copy_b(b + 1, 1, BC);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < FT; ++f) acc[r][f] = mfma16h(w[f], xl[r & 1], acc[r][f]);
            if (r < FT) wn[r] = expand(r, !(u & 1));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    copy_b(0, 0, BC);
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) copy_x(s, s);
    pre_wait<(NST - 2) * NX>();
    read_c(0, 0);
    read_x(0, 0);
#pragma unroll
    for (int f = 0; f < FT; ++f) wa[f] = expand(f, false);
    for (int b = 0, left = p.run >> 2; b < nb; ++b) {
        step(b, std::integral_constant<int, 0>(), wa, wb); step(b, std::integral_constant<int, 1>(), wb, wa);
        step(b, std::integral_constant<int, 2>(), wa, wb); step(b, std::integral_constant<int, 3>(), wb, wa);
        if (--left == 0 || b + 1 == nb) {
            left = p.run >> 2;
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int f = 0; f < FT; ++f) { tot[r][f] += acc[r][f]; acc[r][f] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
        }
    }
    pre_wait<0>();
    f32x4 *mine = (f32x4 *)pre_lds + wave * FT * 64 + lane;
    const int strip0 = fs0 + wf * FT, nf = min(FT, a.nstrips - strip0);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int ct = ct0 + wr * RT + r;
        if (ct >= p.mtiles) break;
#pragma unroll
        for (int f = 0; f < FT; ++f) mine[f * 64] = tot[r][f];
        pre_epilogue<EPI, FT>(a, p, slice, ct, strip0, nf, lane, mine);
    }
}

// RMSNorm scales of a row tile from the per-strip sums of squares ([row tile][strips][16]): once per row instead of once per workgroup of the GEMM that follows.  One workgroup of NT threads: thread
// t adds the strips t / 16, t / 16 + NT / 16, ... of row t % 16, eight loads at a time.  Bound by its chain, so few trips to
// memory (256 strips 5.5 -> 4.7 us between other kernels, 2.5 of them the start); with 4-bit weights k_pre_rowmax does it beside its own work.  Prompts, three or four layers: 8B shape, 100 tokens 1219 -> 1190
// us, 4-bit, 349 tokens 2100 -> 2052; 231 tokens of a 2080-wide model 741 -> 723; 2048 tokens 6383 -> 6363.
template <int NT>
__device__ inline void pre_rscale(const float *ssq, float *rscale, int ct, int strips, float inv_d, float eps)
{
    __shared__ float s[NT / 64][16];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const float *q = ssq + (size_t)ct * strips * 16 + threadIdx.x;
    float v = 0.f;
    for (int i0 = threadIdx.x >> 4; i0 < strips; i0 += NT / 2) {
        float p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = q[(size_t)(i0 - (threadIdx.x >> 4) + (i0 + u * (NT / 16) < strips ? u * (NT / 16) : 0)) * 16];
#pragma unroll
        for (int u = 0; u < 8; ++u) if (i0 + u * (NT / 16) < strips) v += p[u];
    }
    v = with_lane32(with_lane16(v, op_add), op_add);
    if (lane < 16) s[wave][lane] = v;
    __syncthreads();
    if (threadIdx.x < 16) {
        v = s[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) v += s[w][threadIdx.x];
        rscale[ct * 16 + threadIdx.x] = 1.0f / sqrtf(v * inv_d + eps);
    }
}

__global__ void __launch_bounds__(1024)
k_pre_rscale(const float *ssq, float *rscale, int strips, float inv_d, float eps) { pre_rscale<1024>(ssq, rscale, blockIdx.x, strips, inv_d, eps); }

// An operand's rows as scaled f16 pairs, in place.  First the largest |hi| of each row, PRE_MAX_PARTS pieces of K side by side (and beside them, where an RMSNorm scales the rows, that); then the conversion.
#define PRE_MAX_PARTS 16
__global__ void __launch_bounds__(256)
k_pre_rowmax(const uint4 *xop, int ktiles, float *part, int part_rows, const float *ssq, float *rscale, int strips, float inv_d, float eps)
{
    if (blockIdx.x == PRE_MAX_PARTS) { pre_rscale<256>(ssq, rscale, blockIdx.y, strips, inv_d, eps); return; }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ct = blockIdx.y;
    const int per = (ktiles + PRE_MAX_PARTS - 1) / PRE_MAX_PARTS, t0 = blockIdx.x * per, t1 = min(ktiles, t0 + per);
    const uint4 *q = xop + (size_t)2 * ct * ktiles * 64 + lane;
    uint32_t m = 0;                                    // as the bits of |hi| (NaN and infinity largest)
    auto take = [&](uint32_t v) { m = max(m, max(v & 0x7FFFu, (v >> 16) & 0x7FFFu)); };
#pragma unroll 4
    for (int t = t0 + wave; t < t1; t += 4) { const uint4 v = q[(size_t)t * 64]; take(v.x); take(v.y); take(v.z); take(v.w); }
    m = max(m, (uint32_t)__shfl_xor((int)m, 16, 64));
    m = max(m, (uint32_t)__shfl_xor((int)m, 32, 64));
    __shared__ uint32_t s[4][16];
    if (lane < 16) s[wave][lane] = m;
    __syncthreads();
    if (threadIdx.x < 16) part[(size_t)blockIdx.x * part_rows + ct * 16 + threadIdx.x] = __uint_as_float(max(max(s[0][threadIdx.x], s[1][threadIdx.x]), max(s[2][threadIdx.x], s[3][threadIdx.x])) << 16);
}

__global__ void __launch_bounds__(256)
k_pre_to_f16(uint4 *xop, int ktiles, const float *part, int part_rows, float *rinv)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ct = blockIdx.y, row = ct * 16 + (lane & 15);
    const int t = blockIdx.x * 4 + wave;
    uint4 *q = xop + ((size_t)2 * ct * ktiles + min(t, ktiles - 1)) * 64 + lane;
    uint4 *ql = q + (size_t)ktiles * 64;
    const uint4 hi = *q, lo = *ql;                     // (with the maxima: one trip to memory)
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < PRE_MAX_PARTS; ++i) m = max(m, __float_as_uint(part[(size_t)i * part_rows + row]));
    // 2^e <= the row's largest value < 2^(e + 1); a row of zeros or with something not finite stays as it is
    const int e = (int)(m >> 23) - 127, up = m == 0 || e == 128 ? 0 : 14 - max(e, -100);
    const float f = __uint_as_float((uint32_t)(127 + up) << 23), inv = __uint_as_float((uint32_t)(127 - up) << 23);
    if (blockIdx.x == 0 && threadIdx.x < 16) rinv[row] = inv;
    if (t >= ktiles) return;
    uint4 oh, ol;
    auto conv = [&](uint32_t h, uint32_t l, uint32_t &rh, uint32_t &rl) {
        const float x0 = (__uint_as_float(h << 16) + __uint_as_float(l << 16)) * f, x1 = (__uint_as_float(h & 0xFFFF0000u) + __uint_as_float(l & 0xFFFF0000u)) * f;
        const f16x2 a = {(_Float16)x0, (_Float16)x1};
        const f16x2 b = {(_Float16)(x0 - (float)a.x), (_Float16)(x1 - (float)a.y)};
        rh = __builtin_bit_cast(uint32_t, a); rl = __builtin_bit_cast(uint32_t, b);
    };
    conv(hi.x, lo.x, oh.x, ol.x); conv(hi.y, lo.y, oh.y, ol.y); conv(hi.z, lo.z, oh.z, ol.z); conv(hi.w, lo.w, oh.w, ol.w);
    *q = oh; *ql = ol;
}

// Adds the K-slices' partial sums in slice order and runs the epilogue: one wave per (strip, row tile).
template <int EPI>
__global__ void __launch_bounds__(256)
k_pre_sum(const gemm_args a, const pre_gemm_args p, int slices)
{
    const int lane = threadIdx.x & 63, strip = blockIdx.x * 4 + (threadIdx.x >> 6), ct = blockIdx.y;
    if (strip >= a.nstrips) return;
    const float4 *q = p.part + ((size_t)strip * p.mtiles + ct) * 64 + lane;
    const size_t step = (size_t)a.nstrips * p.mtiles * 64;
    epi_pre pre;
    const float rj = pre_rowfactor<EPI>(p, lane, ct);
    pre_fetch<EPI>(a, p, strip, lane, ct, pre_page<EPI>(a, p, lane, ct), rj, pre);
    float4 v = q[0];
    for (int y = 1; y < slices; ++y) { const float4 u = q[y * step]; v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w; }
    f32x4 sum = {v.x, v.y, v.z, v.w};
    if (EPI == EPI_RESID) sum *= rj;
    epi_apply<2, EPI>(a, strip, lane, sum, pre, ct);
}

// ------------------------------------------------------------------------------------------
// Block set-up.  The token ids come from pinned host memory in one read.  The cache's state only changes when the block is
// committed; until then rows and length are kernel arguments (the launches are not recorded).
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(1024)
k_pre_tokens(const int32_t *host_tokens, int32_t *tokens, int rows)
{
    for (int i = threadIdx.x; i < rows; i += 1024) tokens[i] = host_tokens[i];
}

__global__ void __launch_bounds__(64)
k_pre_embed(int rows, int len, const int32_t *tokens, const uint16_t *embed, const uint16_t *gain, const double *inv_freq,
            float *x, float *ssq, uint16_t *xop, float2 *rope, int d, int half)
{
    const int lane = threadIdx.x, ct = blockIdx.y, j = ct * 16 + (lane & 15), g = lane >> 4, strip = blockIdx.x;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (j < rows) {
        const uint16_t *e = embed + (size_t)tokens[j] * d + strip * 16 + 4 * g;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = pv_bf16_to_f32(e[r]);
    }
    emit_x<2>(lane, rows, strip, d, v, *(const uint2 *)(gain + strip * 16 + 4 * g), x, ssq, xop, ct, 8);
    // rotary table: every workgroup takes its share
    for (int idx = (ct * gridDim.x + strip) * 64 + lane; idx < rows * half; idx += gridDim.x * gridDim.y * 64) {
        const int jj = idx / half, i = idx - jj * half;
        double sn, cs;
        sincos((double)(len + jj) * inv_freq[i], &sn, &cs);
        rope[idx] = make_float2((float)cs, (float)sn);
    }
}

// The block's rows are part of the cache, but for its last `keep` rows, which become the cache's running block: the
// head and k_finish commit those as they do for a block of at most 64 rows.
__global__ void k_pre_commit(pv_dev_state *st, int rows, int keep)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    st->len += rows - keep;
    if (rows > keep) st->pending = -1;
    if (keep) { st->gamma = keep; st->mode = PV_MODE_PREFILL_LAST; st->blk.seq[0].gamma = keep; }
}

// ------------------------------------------------------------------------------------------
// Causal attention of the whole block.  A workgroup of 4 waves owns 128 query rows of one kv
// head (row m = token * group + head in group, so a workgroup's tokens are neighbours), a wave
// two 16-row tiles; Q (hi + lo) and the running output stay in registers while the keys go by 64
// at a time through LDS (two buffers, copied a step ahead).  Products, operand orders and splits are those
// of attn_chunk (pv_attention_body.h); the softmax is kept running (maximum and sum per row).
// The matrix cores add up the 64 keys of a step only: the step's P x V and its sum of weights are added to the running totals on the
// vector ALU (by the multiply-add that also rescales them), one feature tile behind the matrix cores.  In one accumulator over all
// keys the rounding errors grew with the context: a prompt of one repeated token, whose exact output is the same at any length, was
// off by 1.1 - 1.3e-6 of the logits' rms at 300 keys and 1.8 - 2.5e-6 at 12000; now 1.2 - 1.4e-6 at 12000.  The additions cost 1 - 4 %
// (8B shape, passes of 12000 tokens: 443 -> 447 us a layer; 2048 tokens, 7B shape: 115 -> 119 us), 5 - 8 % without the lag and
// with the exponent's difference and product as two instructions.
// Every query row reads K and V once per workgroup from L2 instead of once per 32 rows as partial
// results: at 2048 keys the chunked kernel with its merge took 26 us per 64 rows of an 8B-shaped layer.
// ------------------------------------------------------------------------------------------
struct pre_attn_args {
    int rows, len;
    const int32_t *page_table;
    const uint16_t *q_hi, *q_lo;
    const uint16_t *pool;
    pv_kv_geom geom;
    int layer, n_q_heads, group, qtiles, paired;
    float scale2;               // log2(e) / sqrt(head_dim)
    uint16_t *xop_o;
};

template <int HD>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_pre_attn(const pre_attn_args a)
{
    constexpr int KS = HD / 32, ET = HD / 16, RT = 2, TB = 2 * KS;          // TB: KiB of one 16-key group (K and V)
    extern __shared__ uint4 pre_lds[];                                       // [2][4 groups][K | V][KS][64]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, jl = lane & 15, g = lane >> 4;
    // The longest first.  Two workgroups fit on a CU: where all of them start at once, the second half comes
    // shortest first, so that a CU's two add up to about the same everywhere.
    const int kvh = blockIdx.x % a.geom.n_kv_heads, o = blockIdx.x / a.geom.n_kv_heads, half = (a.qtiles + 1) >> 1;
    const int qt = (a.paired && o >= half) ? o - half : a.qtiles - 1 - o;
    const int len = a.len, nrows = a.rows * a.group;
    const int m0 = qt * 128;
    const int jmin = m0 / a.group, jmax = min(m0 + 127, nrows - 1) / a.group;
    const int nkeys = len + jmax + 1, nsteps = (nkeys + 63) >> 6;
    const int sub_shift = a.geom.page_shift - 4, sub_mask = (1 << sub_shift) - 1;
    const int last_grp = (nkeys - 1) >> 4;
    // group 4 s + wave of step s: copied by this wave.  Page table entries are fetched one step ahead.
    const __attribute__((address_space(4))) int32_t *pt = (const __attribute__((address_space(4))) int32_t *)(uintptr_t)uniform_ptr(a.page_table);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(pre_lds)) + wave * TB * 1024;
    auto page_of = [&](int s) { return pt[min(4 * s + wave, last_grp) >> sub_shift]; };
    auto copy = [&](int s, int phys, int buf) {
        const int grp = min(4 * s + wave, last_grp);
        const char *kb = (const char *)(a.pool + pv_kv_block(a.geom, a.layer, phys, kvh, 0) + (size_t)(grp & sub_mask) * 16 * HD);
        const char *vb = (const char *)(a.pool + pv_kv_block(a.geom, a.layer, phys, kvh, 1) + (size_t)(grp & sub_mask) * 16 * HD);
        kb = uniform_ptr(kb); vb = uniform_ptr(vb);
#pragma unroll
        for (int i = 0; i < KS; ++i) dma_tile(lds0 + (uint32_t)(buf * 4 * TB + i) * 1024, kb + i * 1024, lane * 16);
#pragma unroll
        for (int i = 0; i < KS; ++i) dma_tile(lds0 + (uint32_t)(buf * 4 * TB + KS + i) * 1024, vb + i * 1024, lane * 16);
    };
    copy(0, page_of(0), 0);
    int ph_next = page_of(1);

    // this lane's query rows (a row past the end reads the last one and is not stored)
    int j[RT], al[RT];
    uint4 qh[RT][KS], ql[RT][KS];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int m = min(m0 + wave * 32 + t * 16 + jl, nrows - 1);
        j[t] = m / a.group; al[t] = m - j[t] * a.group;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const size_t qo = q_at(kvh * a.group + al[t], j[t], ks * 32 + g * 8, HD, a.rows);
            qh[t][ks] = *(const uint4 *)(a.q_hi + qo); ql[t][ks] = *(const uint4 *)(a.q_lo + qo);
        }
    }
    // Q is here before the loop starts: a wait for it inside would also wait for the copies of the next step
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    f32x4 O[RT][ET];
    float mx[RT], mxs[RT], sum[RT];                    // maximum (as it is, and times scale2), sum
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        mx[t] = mxs[t] = -INFINITY; sum[t] = 0.f;
#pragma unroll
        for (int e = 0; e < ET; ++e) O[t][e] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    for (int s = 0; s < nsteps; ++s) {
        const int buf = s & 1;
        pre_wait<0>();                                 // step s has landed for every wave, and every wave is done with the other buffer
        if (s + 1 < nsteps) { copy(s + 1, ph_next, buf ^ 1); ph_next = page_of(s + 2); }
        const uint4 *Lk = pre_lds + (size_t)buf * 4 * TB * 64 + lane;
        const char *Lv = (const char *)(pre_lds + (size_t)buf * 4 * TB * 64) + KS * 1024 + jl * 32 + g * 8;
        f32x4 S[RT][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int t = 0; t < RT; ++t) S[t][q] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const uint4 k = Lk[(q * TB + ks) * 64];
#pragma unroll
                for (int t = 0; t < RT; ++t) { S[t][q] = mfma16(k, qh[t][ks], S[t][q]); S[t][q] = mfma16(k, ql[t][ks], S[t][q]); }
            }
        }
        const bool edge = s * 64 + 63 > len + jmin;    // some row of the workgroup may not see some key of the step
        uint32_t P[RT][4][4];                          // per group: keys 4 g .. + 3 as hi (2 dwords), lo (2 dwords)
        float f[RT];                                   // what the earlier steps' sums are worth under the new maximum
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            if (edge) {
                const int lim = len + j[t] - s * 64 - 4 * g;
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int r = 0; r < 4; ++r) if (16 * q + r > lim) S[t][q][r] = -INFINITY;
            }
            float m = mx[t];
#pragma unroll
            for (int q = 0; q < 4; ++q) m = fmaxf(fmaxf(m, fmaxf(S[t][q][0], S[t][q][1])), fmaxf(S[t][q][2], S[t][q][3]));
            m = fmaxf(m, __shfl_xor(m, 16, 64));
            m = fmaxf(m, __shfl_xor(m, 32, 64));
            const float ms = m * a.scale2;             // (key 0 is visible to every row: the maximum is finite from the first step on)
            f[t] = __builtin_amdgcn_exp2f(mxs[t] - ms);
            mx[t] = m; mxs[t] = ms;
            float ps = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float p[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) { p[r] = __builtin_amdgcn_exp2f(fmaf(S[t][q][r], a.scale2, -ms)); ps += p[r]; }
                split2(p[0], p[1], P[t][q][0], P[t][q][2]);
                split2(p[2], p[3], P[t][q][1], P[t][q][3]);
            }
            sum[t] = fmaf(sum[t], f[t], ps);
        }
        f32x4 T[2][RT];                                // (added to the totals one feature tile behind the matrix cores)
        auto add = [&](int e) {
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) O[t][e][r] = fmaf(O[t][e][r], f[t], T[e & 1][t][r]);
        };
#pragma unroll
        for (int e = 0; e < ET; ++e) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < RT; ++t) T[e & 1][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int hq = 0; hq < 2; ++hq) {
                const uint2 v0 = *(const uint2 *)(Lv + (2 * hq) * TB * 1024 + e * 512), v1 = *(const uint2 *)(Lv + (2 * hq + 1) * TB * 1024 + e * 512);
                const uint4 v = make_uint4(v0.x, v0.y, v1.x, v1.y);
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    const uint4 ph = make_uint4(P[t][2 * hq][0], P[t][2 * hq][1], P[t][2 * hq + 1][0], P[t][2 * hq + 1][1]);
                    const uint4 pl = make_uint4(P[t][2 * hq][2], P[t][2 * hq][3], P[t][2 * hq + 1][2], P[t][2 * hq + 1][3]);
                    T[e & 1][t] = mfma16(v, ph, T[e & 1][t]);
                    T[e & 1][t] = mfma16(v, pl, T[e & 1][t]);
                }
            }
            if (e > 0) add(e - 1);
        }
        add(ET - 1);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        float l = sum[t];
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        const float inv = 1.0f / l;
        if (m0 + wave * 32 + t * 16 + jl < nrows) {
#pragma unroll
            for (int e = 0; e < ET; ++e) {
                const float y[4] = {O[t][e][0] * inv, O[t][e][1] * inv, O[t][e][2] * inv, O[t][e][3] * inv};
                store_operand4<2>(a.xop_o, a.n_q_heads * HD, j[t], (kvh * a.group + al[t]) * HD + e * 16 + 4 * g, y, 8);
            }
        }
    }
}

// ------------------------------- host side ----------------------------------------

struct pre_ws {
    int32_t *tokens;
    float2 *rope;
    float *x, *ssq, *rscale;
    uint16_t *xop;              // QKV and gate/up input (K = d)
    uint16_t *xop_d;            // down input (K = F); before that the queries and the O input (K = qd)
    uint16_t *q_hi, *q_lo, *xop_o;
    float *rowsum;              // 4-bit weights: see pre_layout
    float *part; size_t part_floats;   // K-slices' partial sums
};

static size_t pre_layout(const pv_model *m, int rows, char *base, pre_ws *w)
{
    const pv_model_config &f = m->cfg;
    const size_t R = rows, d = f.d_model, qd = (size_t)f.n_q_heads * f.head_dim;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) / 256 * 256; return base ? base + o : (char *)nullptr; };
    char *p;
    p = take(4 * R); if (w) w->tokens = (int32_t *)p;
    p = take(sizeof(float2) * R * (f.head_dim / 2)); if (w) w->rope = (float2 *)p;
    p = take(4 * R * d); if (w) w->x = (float *)p;
    p = take(4 * R * (d / 16)); if (w) w->ssq = (float *)p;
    p = take(4 * R); if (w) w->rscale = (float *)p;
    p = take(4 * R * d); if (w) w->xop = (uint16_t *)p;
    p = take(std::max((size_t)4 * R * f.ffn_dim, 8 * R * qd));
    if (w) { w->xop_d = (uint16_t *)p; w->q_hi = w->xop_d; w->q_lo = w->q_hi + R * qd; w->xop_o = w->q_lo + R * qd; }
    // row sums [K / 32][rows], or the rows' factors and PRE_MAX_PARTS maxima of each
    if (m->wbits == 4) { p = take(4 * std::max(std::max(std::max(d, qd), (size_t)f.ffn_dim) / 32, (size_t)PRE_MAX_PARTS + 1) * ((R + 127) / 128 * 128)); if (w) w->rowsum = (float *)p; }
    // a GEMM is cut along K only where it has fewer rectangles than the chip has CUs: 256 x 128 KiB
    const size_t pf = std::min((size_t)8 << 20, 8 * R * d);
    p = take(4 * pf); if (w) { w->part = (float *)p; w->part_floats = pf; }
    return off;
}

size_t pv_pre_bytes(const pv_model *m, int rows)
{
    return m->path >= PV_PATH_MATRIX && rows > PV_PRE_MIN ? pre_layout(m, rows, nullptr, nullptr) : 0;
}

template <int WR, int WF, int RT, int FT, int NST>
struct pre_shape {
    static constexpr int BR = WR * RT, BF = WF * FT;
    static constexpr int lds = NST * pre_stage_tiles(BR, BF) * 1024;
    template <int EPI> static int allow()
    {
        PV_HIP(hipFuncSetAttribute((const void *)k_pre_gemm<WR, WF, RT, FT, NST, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        return PV_OK;
    }
    static int allow_all()
    {
        int rc;
        if ((rc = allow<EPI_QKV>()) != PV_OK || (rc = allow<EPI_RESID>()) != PV_OK) return rc;
        return allow<EPI_SWIGLU>();
    }
    template <int EPI> static int run(const gemm_args &ga, pre_gemm_args pa, int slices, hipStream_t s)
    {
        pa.rb = (pa.mtiles + BR - 1) / BR; pa.fb = (ga.nstrips + BF - 1) / BF;
        pa.kps = (ga.ktiles + slices - 1) / slices;
        slices = (ga.ktiles + pa.kps - 1) / pa.kps;
        if (slices == 1) pa.part = nullptr;
        k_pre_gemm<WR, WF, RT, FT, NST, EPI><<<pa.rb * pa.fb * slices, 512, lds, s>>>(ga, pa);
        PV_HIP(hipGetLastError());
        if (slices > 1) { k_pre_sum<EPI><<<dim3((ga.nstrips + 3) / 4, pa.mtiles), 256, 0, s>>>(ga, pa, slices); PV_HIP(hipGetLastError()); }
        return PV_OK;
    }
};
using pre_wide = pre_shape<2, 4, 4, 4, 4>;     // 128 rows x 256 features
using pre_mid = pre_shape<2, 4, 4, 3, 5>;      // 128 x 192
using pre_small = pre_shape<2, 4, 4, 2, 6>;    // 128 x 128

template <int FT>
struct pre_q4 {
    using S = pre_q4_shape<FT>;
    template <int EPI> static int allow()
    {
        PV_HIP(hipFuncSetAttribute((const void *)k_pre_gemm_q4<FT, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, S::lds));
        return PV_OK;
    }
    static int allow_all()
    {
        int rc;
        if ((rc = allow<EPI_QKV>()) != PV_OK || (rc = allow<EPI_RESID>()) != PV_OK) return rc;
        return allow<EPI_SWIGLU>();
    }
    template <int EPI> static int run(const gemm_args &ga, pre_gemm_args pa, int slices, hipStream_t s)
    {
        pa.rb = (pa.mtiles + S::BR - 1) / S::BR; pa.fb = (ga.nstrips + S::BF - 1) / S::BF;
        pa.kps = (ga.ktiles / 4 + slices - 1) / slices * 4;
        slices = (ga.ktiles + pa.kps - 1) / pa.kps;
        if (slices == 1) pa.part = nullptr;
        k_pre_gemm_q4<FT, EPI><<<pa.rb * pa.fb * slices, 512, S::lds, s>>>(ga, pa);
        PV_HIP(hipGetLastError());
        if (slices > 1) { k_pre_sum<EPI><<<dim3((ga.nstrips + 3) / 4, pa.mtiles), 256, 0, s>>>(ga, pa, slices); PV_HIP(hipGetLastError()); }
        return PV_OK;
    }
};

template <int FT>
struct pre_h4 {
    using S = pre_h4_shape<FT>;
    template <int EPI> static int allow()
    {
        PV_HIP(hipFuncSetAttribute((const void *)k_pre_gemm_h4<FT, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, S::lds));
        return PV_OK;
    }
    static int allow_all()
    {
        int rc;
        if ((rc = allow<EPI_QKV>()) != PV_OK || (rc = allow<EPI_RESID>()) != PV_OK) return rc;
        return allow<EPI_SWIGLU>();
    }
    template <int EPI> static int run(const gemm_args &ga, pre_gemm_args pa, int slices, hipStream_t s)
    {
        pa.rb = (pa.mtiles + S::BR - 1) / S::BR; pa.fb = (ga.nstrips + S::BF - 1) / S::BF;
        pa.kps = (ga.ktiles / 4 + slices - 1) / slices * 4;
        slices = (ga.ktiles + pa.kps - 1) / pa.kps;
        if (slices == 1) pa.part = nullptr;
        k_pre_gemm_h4<FT, EPI><<<pa.rb * pa.fb * slices, 512, S::lds, s>>>(ga, pa);
        PV_HIP(hipGetLastError());
        if (slices > 1) { k_pre_sum<EPI><<<dim3((ga.nstrips + 3) / 4, pa.mtiles), 256, 0, s>>>(ga, pa, slices); PV_HIP(hipGetLastError()); }
        return PV_OK;
    }
};

int pv_pre_init(const pv_model *m)
{
    int rc;
    if (m->wbits == 4) { if ((rc = pre_q4<4>::allow_all()) != PV_OK) return rc; if ((rc = pre_h4<4>::allow_all()) != PV_OK) return rc; return pre_h4<3>::allow_all(); }
    if ((rc = pre_mid::allow_all()) != PV_OK || (rc = pre_wide::allow_all()) != PV_OK || (rc = pre_small::allow_all()) != PV_OK) return rc;
    return PV_OK;
}

template <int EPI>
static int pre_gemm(const pv_model *m, const gemm_args &g, bool wide, int strips, float *rscale, float *rowsum, int rows, int len, size_t part_floats, hipStream_t s)
{
    const int mtiles = (rows + 15) / 16;
    gemm_args ga = g;
    ga.nstrips = strips;
    pre_gemm_args pa = {};
    pa.rscale = rscale; pa.part = (float4 *)g.tile_part; pa.mtiles = mtiles; pa.run = pre_run(g.ktiles, strips); pa.rows = rows; pa.len = len;
    const bool h4 = m->wbits == 4 && !wide;            // every scale of the GEMM's matrices fits the f16 form of its weights
    if (h4) {
        float *rinv = rowsum, *part = rowsum + (mtiles + 7) / 8 * 128;       // (in the place of the row sums)
        pa.rinv = rinv;
        k_pre_rowmax<<<dim3(PRE_MAX_PARTS + (rscale != nullptr), mtiles), 256, 0, s>>>(g.xop, g.ktiles, part, mtiles * 16, g.ssq, rscale, g.ssq_parts, g.inv_d, g.eps);
        PV_HIP(hipGetLastError());
        k_pre_to_f16<<<dim3((g.ktiles + 3) / 4, mtiles), 256, 0, s>>>((uint4 *)g.xop, g.ktiles, part, mtiles * 16, rinv);
        PV_HIP(hipGetLastError());
    } else if (m->wbits == 4) {
        pa.rowsum = rowsum; pa.rsum_rows = (mtiles + 7) / 8 * 128;
        k_pre_rowsum<<<dim3((g.ktiles + 3) / 4, mtiles), 256, 0, s>>>(g.xop, g.ktiles, rowsum, pa.rsum_rows);
        PV_HIP(hipGetLastError());
    }
    // The rectangle and the number of K-slices with the smallest estimated time, in units of 3.85 ns.  The constants stand for 0.53, 0.41 and 0.30 us a K-tile of a 128 x 256, 128 x 192 and 128 x 128 rectangle,
    // 4-bit weights 0.79 and 0.61, on top of 13, 11 and 9.5 us for the start, the epilogue and the end; partial sums: 3 us and 0.2 ns for
    // each 16 x 16 of them.  Where more workgroups than CUs come out, they run in rounds.  Measured with 4096 x 4096 and 4096 x 14336 weights:
    // 0.58, 0.51 and 0.38 us on 64 to 128 CUs, 0.63, 0.56 and 0.47 us on twice as many, on top of 16 to 18, 13 and 10 to 11 us; 4-bit
    // weights on 128 and 176 CUs 0.81 and 0.66 us, and 0.88 us in k_pre_gemm_q4, on top of 16 to 20 us.
    struct rect { int br, bf; double cost; };
    static const rect R16[3] = {{8, 16, 1.07}, {8, 12, 1.12}, {8, 8, 1.22}}, R4[2] = {{8, 16, 1.6}, {8, 12, 1.65}};
    const rect *R = m->wbits == 4 ? R4 : R16;
    const int kinds = h4 ? 2 : m->wbits == 4 ? 1 : 3;
    double best = 1e30; int shape = 0, cut = 1;
    for (int i = 0; i < kinds; ++i) {
        const int blocks = ((mtiles + R[i].br - 1) / R[i].br) * ((strips + R[i].bf - 1) / R[i].bf);
        for (int sl = 1; sl <= 16; ++sl) {
            if (sl > 1 && (g.ktiles / sl < 8 || (size_t)sl * strips * mtiles * 256 > part_floats || g.tile_part == nullptr)) break;
            const int rounds = (blocks * sl + m->n_cus - 1) / m->n_cus;
            const double t = rounds * ((g.ktiles + sl - 1) / sl * R[i].br * R[i].bf * R[i].cost + 1500.0 + 15.0 * R[i].br * R[i].bf)
                           + (sl > 1 ? 800.0 + 0.05 * sl * strips * mtiles : 0.0);
            if (t < best) { best = t; shape = i; cut = sl; }
        }
    }
    if (h4) return shape == 0 ? pre_h4<4>::run<EPI>(ga, pa, cut, s) : pre_h4<3>::run<EPI>(ga, pa, cut, s);
    if (m->wbits == 4) return pre_q4<4>::run<EPI>(ga, pa, cut, s);
    if (shape == 0) return pre_wide::run<EPI>(ga, pa, cut, s);
    if (shape == 1) return pre_mid::run<EPI>(ga, pa, cut, s);
    return pre_small::run<EPI>(ga, pa, cut, s);
}

template <int HD>
static int pre_attention(const pre_attn_args &a, int kv_heads, hipStream_t s)
{
    k_pre_attn<HD><<<a.qtiles * kv_heads, 256, 2 * 4 * 2 * (HD / 32) * 1024, s>>>(a);
    PV_HIP(hipGetLastError());
    return PV_OK;
}

int pv_pre_block(pv_cache *c, const int32_t *d_host_tokens, int rows, int keep, pv_pre_out *out, hipStream_t s)
{
    const pv_model *m = c->m;
    const pv_model_config &f = m->cfg;
    const int d = f.d_model, hd = f.head_dim, qd = f.n_q_heads * hd, kvd = f.n_kv_heads * hd, F = f.ffn_dim, mtiles = (rows + 15) / 16, len = c->len;
    const char *Wb = m->d_weights;
    auto gainp = [&](int kind, int l) { return (const uint16_t *)(Wb + pv_tref(m, kind, l).off); };
    auto wide = [&](int kind, int l) { return pv_tref(m, kind, l).wide != 0; };
    pre_ws w = {};
    pre_layout(m, m->pre_rows, m->pre_base, &w);

    k_pre_tokens<<<1, 1024, 0, s>>>(d_host_tokens, w.tokens, rows);
    PV_HIP(hipGetLastError());
    k_pre_embed<<<dim3(d / 16, mtiles), 64, 0, s>>>(rows, len, w.tokens, (const uint16_t *)(Wb + m->global[PV_T_EMBED].off), gainp(PV_T_ATTN_NORM, 0),
                                                    (const double *)(Wb + m->inv_freq_off), w.x, w.ssq, w.xop, w.rope, d, hd / 2);
    PV_HIP(hipGetLastError());

    gemm_args g = {};
    g.st = c->ws.state; g.inv_d = 1.0f / (float)d; g.eps = (float)f.rms_eps; g.ssq_parts = d / 16;
    g.q_hi = w.q_hi; g.q_lo = w.q_lo; g.q_rows = rows; g.pool = (uint16_t *)c->d_pool; g.page_table = c->ws.page_table; g.rope = w.rope; g.geom = pv_geom(c);
    g.n_q_heads = f.n_q_heads; g.q_strips = qd / 16; g.k_strips = kvd / 16;
    g.x = w.x; g.d = d; g.xop_act = w.xop_d; g.F = F; g.tile_part = w.part; g.ssq = w.ssq; g.ssq_out = w.ssq; g.xop_out = w.xop;

    pre_attn_args at = {};
    at.rows = rows; at.len = len; at.page_table = c->ws.page_table; at.q_hi = w.q_hi; at.q_lo = w.q_lo; at.pool = (const uint16_t *)c->d_pool; at.geom = g.geom;
    at.n_q_heads = f.n_q_heads; at.group = f.n_q_heads / f.n_kv_heads; at.qtiles = (rows * at.group + 127) / 128;
    at.paired = at.qtiles * f.n_kv_heads <= 2 * m->n_cus;
    at.scale2 = 1.44269504088896340736f / sqrtf((float)hd); at.xop_o = w.xop_o;

    int rc;
    auto rscale = [&](bool wide_w) -> int {
        if (m->wbits == 4 && !wide_w) return PV_OK;         // (k_pre_rowmax does it)
        k_pre_rscale<<<mtiles, 1024, 0, s>>>(w.ssq, w.rscale, d / 16, g.inv_d, g.eps);
        PV_HIP(hipGetLastError());
        return PV_OK;
    };
    for (int l = 0; l < f.n_layers; ++l) {
        const bool wide_qkv = wide(PV_T_WQ, l) || wide(PV_T_WK, l) || wide(PV_T_WV, l), wide_gu = wide(PV_T_WG, l) || wide(PV_T_WU, l);
        if ((rc = rscale(wide_qkv)) != PV_OK) return rc;
        g.W = (const uint4 *)(Wb + pv_tref(m, PV_T_WQ, l).off); g.xop = (const uint4 *)w.xop; g.ktiles = d / 32; g.layer = l;
        if ((rc = pv_prof_mark(c, PV_PROF_QKV, l, 0, s)) != PV_OK) return rc;
        if ((rc = pre_gemm<EPI_QKV>(m, g, wide_qkv, (qd + 2 * kvd) / 16, w.rscale, w.rowsum, rows, len, w.part_floats, s)) != PV_OK) return rc;
        if ((rc = pv_prof_mark(c, PV_PROF_QKV, l, 1, s)) != PV_OK) return rc;
        at.layer = l;
        if ((rc = pv_prof_mark(c, PV_PROF_ATTENTION, l, 0, s)) != PV_OK) return rc;
        rc = hd == 128 ? pre_attention<128>(at, f.n_kv_heads, s) : hd == 64 ? pre_attention<64>(at, f.n_kv_heads, s) : pre_attention<32>(at, f.n_kv_heads, s);
        if (rc != PV_OK) return rc;
        if ((rc = pv_prof_mark(c, PV_PROF_ATTENTION, l, 1, s)) != PV_OK) return rc;
        g.W = (const uint4 *)(Wb + pv_tref(m, PV_T_WO, l).off); g.xop = (const uint4 *)w.xop_o; g.ktiles = qd / 32; g.gain_next = gainp(PV_T_FFN_NORM, l);
        if ((rc = pv_prof_mark(c, PV_PROF_OPROJ, l, 0, s)) != PV_OK) return rc;
        if ((rc = pre_gemm<EPI_RESID>(m, g, wide(PV_T_WO, l), d / 16, nullptr, w.rowsum, rows, len, w.part_floats, s)) != PV_OK) return rc;
        if ((rc = pv_prof_mark(c, PV_PROF_OPROJ, l, 1, s)) != PV_OK) return rc;
        if ((rc = rscale(wide_gu)) != PV_OK) return rc;
        g.W = (const uint4 *)(Wb + pv_tref(m, PV_T_WG, l).off); g.xop = (const uint4 *)w.xop; g.ktiles = d / 32;
        if ((rc = pv_prof_mark(c, PV_PROF_GATEUP, l, 0, s)) != PV_OK) return rc;
        if ((rc = pre_gemm<EPI_SWIGLU>(m, g, wide_gu, F / 8, w.rscale, w.rowsum, rows, len, w.part_floats, s)) != PV_OK) return rc;
        if ((rc = pv_prof_mark(c, PV_PROF_GATEUP, l, 1, s)) != PV_OK) return rc;
        g.W = (const uint4 *)(Wb + pv_tref(m, PV_T_WD, l).off); g.xop = (const uint4 *)w.xop_d; g.ktiles = F / 32;
        g.gain_next = (l + 1 < f.n_layers) ? gainp(PV_T_ATTN_NORM, l + 1) : (const uint16_t *)(Wb + m->global[PV_T_FINAL_NORM].off);
        if ((rc = pv_prof_mark(c, PV_PROF_DOWN, l, 0, s)) != PV_OK) return rc;
        if ((rc = pre_gemm<EPI_RESID>(m, g, wide(PV_T_WD, l), d / 16, nullptr, w.rowsum, rows, len, w.part_floats, s)) != PV_OK) return rc;
        if ((rc = pv_prof_mark(c, PV_PROF_DOWN, l, 1, s)) != PV_OK) return rc;
    }
    k_pre_commit<<<1, 64, 0, s>>>(c->ws.state, rows, keep);
    PV_HIP(hipGetLastError());
    const int ct = (rows - keep) / 16;                  // (the kept rows start on a row tile)
    out->xop = w.xop + (size_t)ct * 2 * (d / 32) * 512;
    out->ssq = w.ssq + (size_t)ct * d;
    return PV_OK;
}
