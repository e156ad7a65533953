// Causal grouped-query attention over the paged bf16 KV cache on the matrix cores.
//
// Work unit: one workgroup of 8 wavefronts = (kv head, chunk of keys, group of <= 32 query
// rows).  The query rows of a kv head are its `group` query heads x gamma block rows, packed
// densely (row m = head_in_group * gamma + j).  Two shapes of the unit:
//   TILES = 1: up to 16 rows, 256 keys; every wave takes 32 keys of the one 16-row tile;
//   TILES = 2: 17..32 rows, 128 keys; wave w takes row tile w / 4 and 32 keys (w % 4).
// A wave makes one pass (in a short context the workgroup goes through all chunks, one pass each).  The waves of a row tile are merged through LDS (every
// wave writes its rescaled partial, then all threads add them in wave order) into one partial
// (max, sum, output) per chunk; a small merge kernel combines the chunks and writes the
// attention output directly as the output projection's split-bf16 operand.
//
// Everything is computed transposed so that no register shuffling is needed:
//   S^T (keys x rows) = K (keys x hd) * Q^T (hd x rows)      A = K tile, B = Q^T
//   O^T (hd x rows)   = V^T (hd x keys) * P^T (keys x rows)   A = V^T tile, B = P^T
// A 16-key page group stored as [hd/32][lane][8] is exactly the A operand of the first
// product.  The accumulator of S^T holds, per lane, 4 consecutive keys of row lane%16 — and
// that is, for two key groups side by side, the B operand of the second product when the 32
// keys of a step are taken in the order (group0 keys 4g..4g+3, group1 keys 4g..4g+3); V^T is
// read in that same order (8-byte loads from the [hd][16] page layout).  Softmax statistics
// of row lane%16 then sit in the same lane as that row's output accumulators.
//
// Q and P are carried as bf16 hi + lo pairs (two MFMAs each), K and V are the stored bf16.
// Softmax weights use the hardware exponential (__expf, relative error ~1e-6 at these
// arguments): they are rounded to 16 mantissa bits for the second product anyway.
// Q arrives already split (the QKV projection's epilogue writes the two bf16 arrays).
// The causal part only touches keys >= len: block row j sees the block slots its mask names (a chain:
// keys up to len + j; a draft tree: its ancestors' slots and its own).
#pragma once
#include "pv_matrix_common.h"

struct attn_args {
    const pv_dev_state *st;
    const int32_t *page_table;
    const uint16_t *q_hi, *q_lo; // [n_q_heads][hd / 8][rows][8] each (q_at), rotary already applied: q = hi + lo
    const uint16_t *pool;
    pv_kv_geom geom;
    int layer, n_q_heads, group, max_chunks;
    int chunk_shift;            // log2 of the keys per chunk of the partials (8 with one row tile, 7 with two)
    float scale;
    float *part_o;              // [n_kv_heads][MP][max_chunks][32][hd]
    float *part_ml;             // [n_kv_heads][MP][max_chunks][32][2]  (max, sum)
    uint16_t *xop_o;            // merge output: operand of the output projection, K = n_q_heads*hd
    int n_pages;                // entries of the page table
    int chunks;                 // chunks launched: the host's bound of a step's keys, at most max_chunks
    size_t page_bytes, block_bytes;    // one page in one layer (all kv heads, K and V), and a kv head's K or V of it
    int rows, batched;          // rows of the block; several sequences in it (their rows, lengths and pages are in the state's description).  Arguments, so
                                // that what depends on them only is asked for at once, not a memory round trip later
};

__device__ inline void split8(const float v[8], uint4 &hi, uint4 &lo)
{
    uint32_t h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) split2(v[2 * i], v[2 * i + 1], h[i], l[i]);
    hi = make_uint4(h[0], h[1], h[2], h[3]); lo = make_uint4(l[0], l[1], l[2], l[3]);
}

template <int HD>
__host__ __device__ constexpr int attn_smem_floats() { return 8 * 16 * (HD + 4) + 2 * 8 * 16; }

// A wave's running result for its 16 query rows: lane (g, jl) has row jl's maximum and sum and its features 16 e + 4 g .. + 3.
template <int HD> struct attn_acc { f32x4 O[HD / 16]; float m, l; };

// 32 keys (two groups of 16, from p0 on) of one wave; p0 and the groups' places in memory (K; V lies a block behind) are the same for the whole wave.  Called with Q on its way, so
// that Q, K and V are one memory round trip.  MORE: the accumulator holds earlier keys.  V goes through LDS (vs: the wave's own 64 HD bytes): a lane needs 8 bytes here and 8 there of it, and
// straight from memory the address path takes four cycles for every line of that.
template <int HD, bool MORE, typename VIS>
__device__ inline void attn_keys(const attn_args &a, const char *kb0, const char *kb1, int p0, int len,
                                 const uint4 (&qh)[HD / 32], const uint4 (&ql)[HD / 32], VIS visible, attn_acc<HD> &A, const char *vs)
{
    constexpr int KS = HD / 32, ET = HD / 16;
    const int lane = threadIdx.x & 63, jl = lane & 15, g = lane >> 4;
    uint4 kt[2][KS];
    const uint32_t vl = lds_addr(vs);
    if (MORE) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (the earlier keys' V has been read)
    dma_tiles<KS>(vl, uniform_ptr(kb0 + a.block_bytes), lane * 16);
    dma_tiles<KS>(vl + KS * 1024, uniform_ptr(kb1 + a.block_bytes), lane * 16);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) { kt[0][ks] = ((const uint4 *)kb0)[ks * 64 + lane]; kt[1][ks] = ((const uint4 *)kb1)[ks * 64 + lane]; }
    // every load above is in flight before the first use: one memory round trip, not one per operand
    asm volatile("" ::: "memory");

    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        s0 = mfma16(kt[0][ks], qh[ks], s0); s1 = mfma16(kt[1][ks], qh[ks], s1);
        s0 = mfma16(kt[0][ks], ql[ks], s0); s1 = mfma16(kt[1][ks], ql[ks], s1);
    }
    float sv[8];
    float mx = MORE ? A.m : -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) { sv[r] = s0[r] * a.scale; sv[4 + r] = s1[r] * a.scale; }
    if (p0 + 32 > len) {                               // (keys below: committed, every row sees them)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int pa = p0 + 4 * g + r, pb = pa + 16;
            if (!visible(pa)) sv[r] = -INFINITY;
            if (!visible(pb)) sv[4 + r] = -INFINITY;
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) mx = fmaxf(mx, fmaxf(sv[r], sv[4 + r]));
    mx = with_lane32(with_lane16(mx, op_max), op_max);
    const bool none = mx == -INFINITY;                 // no visible key for this row so far
    const float keep = MORE ? (A.m == -INFINITY ? 0.f : __expf(A.m - mx)) : 0.f;
    float pr[8], ps = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) { pr[i] = none ? 0.f : __expf(sv[i] - mx); ps += pr[i]; }
    ps = with_lane32(with_lane16(ps, op_add), op_add);
    A.l = MORE ? A.l * keep + ps : ps;
    A.m = mx;
    uint4 ph, pl;
    split8(pr, ph, pl);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // V is there (K went out behind it and has been used)
    const char *vr = vs + jl * 32 + g * 8;
#pragma unroll
    for (int et = 0; et < ET; ++et) {
        const uint2 v0 = *(const uint2 *)(vr + et * 512), v1 = *(const uint2 *)(vr + KS * 1024 + et * 512);
        const uint4 va = make_uint4(v0.x, v0.y, v1.x, v1.y);
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        if (MORE) { const f32x4 b = A.O[et]; o = (f32x4){b[0] * keep, b[1] * keep, b[2] * keep, b[3] * keep}; }
        o = mfma16(va, ph, o);
        o = mfma16(va, pl, o);
        A.O[et] = o;
    }
}

// One (kv head, chunk, 32-row group) unit, executed by the 8 wavefronts of the workgroup (all
// 512 threads must call).  TILES as above; chunk c covers keys c * (256 / TILES) ... .
// NB = 0: the chunk's partial result is left for the merge kernel.  NB = 1, 2: the workgroup goes through all the chunks
// one after the other and writes the output projection's operand (of that layout) itself.
// smem: attn_smem_floats<HD>() floats of LDS (more than 64 KiB for HD = 128: dynamic).
// Bound by latency: per wave one chain of some 600 instructions with one trip to memory in it, two waves a SIMD.  So: places in memory from scalars, a row's head by a float multiplication,
// no masks on committed keys, reductions across lanes on the vector ALU, one barrier.  8 rows, 2048 keys, 8B shape, inside the kernel 5.7 -> 4.4 us (loads on their way after 3.0 -> 1.5 us of it), the
// merge behind it 2.5 -> 1.9; 16384 keys, 4 rows 14.2 -> 12.1.
template <int HD, int TILES, int NB>
__device__ inline void attn_chunk(const attn_args &a, int c, int kvh, int z, int n_units, float *smem)
{
    constexpr int KS = HD / 32, ET = HD / 16, OS = HD + 4, NWM = 8 / TILES, CK = 256 / TILES;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, jl = lane & 15, g = lane >> 4;
    const int rt = wave / NWM, kq = wave % NWM;
    const int sub_shift = a.geom.page_shift - 4, sub_mask = (1 << sub_shift) - 1;
    // this wave's 32 keys: two groups of 16.  Which pages they sit in does not depend on the cache
    // length, so the page-table entries are fetched beside the length, not behind it (an entry past
    // the table's end is clamped; such keys are past the length as well and never used).
    int p0 = c * CK + kq * 32;
    typedef const __attribute__((address_space(4))) int32_t *table;            // (read by scalar loads)
    table pt = (table)(uintptr_t)a.page_table;
    int npages = a.n_pages;
    int ph0 = pt[min((p0 >> 4) >> sub_shift, npages - 1)], ph1 = pt[min(((p0 >> 4) + 1) >> sub_shift, npages - 1)];
    int len = a.st->len, gamma = a.rows, row0 = 0, mp = z;
    const char *pool = (const char *)a.pool;
    if (a.batched) {
        // batched step: unit z belongs to the sequence with the largest unit0 <= z; its rows, length and pages
        const int nseq = a.st->blk.n_seq;
        int sidx = 0;
        for (int k = 1; k < nseq; ++k) if (z >= a.st->blk.seq[k].unit0) sidx = k;
        const pv_seq_ref &sq = a.st->blk.seq[sidx];
        len = sq.st->len; gamma = sq.gamma; row0 = sq.row0; mp = z - sq.unit0;
        pool = (const char *)sq.pool;
        pt = (table)(uintptr_t)sq.page_table; npages = sq.n_pages;
        ph0 = pt[min((p0 >> 4) >> sub_shift, npages - 1)]; ph1 = pt[min(((p0 >> 4) + 1) >> sub_shift, npages - 1)];
    }
    len = __builtin_amdgcn_readfirstlane(len); gamma = __builtin_amdgcn_readfirstlane(gamma);
    const int nkeys = len + gamma;
    if (c * CK >= nkeys) return;
    const int nrows = a.group * gamma;
    if (mp * 32 >= nrows) return;                      // (a unit beyond the sequence's rows: the grid is sized for the largest)
    pool += ((size_t)a.layer * npages) * a.page_bytes + (size_t)(2 * kvh) * a.block_bytes;
    auto group_at = [&](int grp, int phys) { return uniform_ptr(pool + (size_t)phys * a.page_bytes + (size_t)(grp & sub_mask) * (32 * HD)); };
    // this lane's query row: row lane%16 of the wave's 16-row tile.  A lane past the rows takes row 0 of the first head: its results are not used
    const int m = mp * 32 + rt * 16 + jl;
    const int al0 = (int)(((float)m + 0.5f) * __builtin_amdgcn_rcpf((float)gamma));     // m / gamma: up to m = 2^21 (the grid's 65536 units) the rounding errors are under 0.5 / gamma
    const bool live = m < nrows;
    const int al = live ? al0 : 0, j = live ? m - al0 * gamma : 0;
    // which keys the row may see: every committed position, and of the block's own slots (len + q) those its
    // mask names (a chain: up to its own; a draft tree: its ancestors and itself)
    uint64_t vmask = 0;
    if (NB != 0 || p0 + 32 > len) vmask = a.st->rowmask[row0 + j];
    auto visible = [&](int p) { const int q = p - len; return q < 0 || (q < 64 && ((vmask >> q) & 1ull)); };
    attn_acc<HD> A;
    A.m = -INFINITY; A.l = 0.f;
#pragma unroll
    for (int et = 0; et < ET; ++et) A.O[et] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float2 (*sh_ml)[16] = (float2 (*)[16])smem;                               // [8][16]: a wave's maximum and sum for its rows
    float (*sh_o)[16][OS] = (float (*)[16][OS])(smem + 2 * 8 * 16);           // [8][16][OS]
    if (p0 < nkeys) {
        uint4 qh[KS], ql[KS];
        // (the group's first head from scalars, 64-bit; a lane's place behind it is under 2^29 bytes)
        const size_t qb = q_at(kvh * a.group, 0, 0, HD, a.rows) * 2;
        const uint32_t qo = (uint32_t)(q_at(al, row0 + j, 8 * g, HD, a.rows) * 2), qs = (uint32_t)a.rows * 64;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qh[ks] = *(const uint4 *)((const char *)a.q_hi + qb + ks * qs + qo);
            ql[ks] = *(const uint4 *)((const char *)a.q_lo + qb + ks * qs + qo);
        }
        const char *vs = (const char *)sh_o[wave];     // (V, and then the wave's partial result)
        const char *kb0 = group_at(p0 >> 4, ph0);      // a second group past the end re-reads the first one (it is masked)
        attn_keys<HD, false>(a, kb0, p0 + 16 < nkeys ? group_at((p0 >> 4) + 1, ph1) : kb0, p0, len, qh, ql, visible, A, vs);
        if (NB != 0) {
            for (p0 += CK; p0 < nkeys; p0 += CK) {
                ph0 = pt[(p0 >> 4) >> sub_shift]; ph1 = pt[min(((p0 >> 4) + 1) >> sub_shift, npages - 1)];
                kb0 = group_at(p0 >> 4, ph0);
                attn_keys<HD, true>(a, kb0, p0 + 16 < nkeys ? group_at((p0 >> 4) + 1, ph1) : kb0, p0, len, qh, ql, visible, A, vs);
            }
        }
    }

    // merge the NWM waves of each row tile: every wave parks its partial result, all threads scale them to the tile's maximum and add them in wave order
#pragma unroll
    for (int et = 0; et < ET; ++et) *(float4 *)&sh_o[wave][jl][et * 16 + 4 * g] = make_float4(A.O[et][0], A.O[et][1], A.O[et][2], A.O[et][3]);
    if (g == 0) sh_ml[wave][jl] = make_float2(A.m, A.l);
    __syncthreads();
    const size_t unit = ((size_t)kvh * n_units + z) * a.max_chunks + c;
    float *po = a.part_o + unit * 32 * HD;
#pragma unroll
    for (int i0 = 0; i0 < TILES * 16 * (HD / 4); i0 += 512) {
        const int i = i0 + threadIdx.x;
        if (TILES * 16 * (HD / 4) < 512 && i >= TILES * 16 * (HD / 4)) break;
        const int row = i / (HD / 4), c4 = i - row * (HD / 4), t = row >> 4, r = row & 15;
        float2 ml[NWM];
        float4 o[NWM];
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < NWM; ++w) { ml[w] = sh_ml[t * NWM + w][r]; o[w] = *(const float4 *)&sh_o[t * NWM + w][r][4 * c4]; M = fmaxf(M, ml[w].x); }
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < NWM; ++w) {
            const float f = (ml[w].x == -INFINITY) ? 0.f : __expf(ml[w].x - M);
            acc.x = fmaf(f, o[w].x, acc.x); acc.y = fmaf(f, o[w].y, acc.y); acc.z = fmaf(f, o[w].z, acc.z); acc.w = fmaf(f, o[w].w, acc.w);
            L = fmaf(f, ml[w].y, L);
        }
        if constexpr (NB == 0) {
            *(float4 *)(po + (size_t)row * HD + 4 * c4) = acc;
            if (c4 == 0) *(float2 *)(a.part_ml + (unit * 32 + row) * 2) = make_float2(M, L);
        } else {
            const int mr = mp * 32 + row;
            if (mr >= nrows) continue;
            const float inv = 1.0f / L, y[4] = {acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv};
            const int alr = mr / gamma, jr = mr - alr * gamma;
            store_operand4<(NB == 1 ? 1 : 2)>(a.xop_o, a.n_q_heads * HD, row0 + jr, (kvh * a.group + alr) * HD + 4 * c4, y, a.rows);
        }
    }
}

// Combine the chunk partials of one (block row, query head) and emit the operand of the
// output projection.  One thread per 4 consecutive features.
// (block row j, query head aq) unit, executed by NT threads (tid = 0..NT-1, all must call).
// smem: NT + (NT / 64) * (HD / 4) * 8 floats.
template <int NB, int HD, int NT>
__device__ inline void attn_merge_unit(const attn_args &a, int r, int aq, int n_units, int tid, float *smem)
{
    static_assert(NT % 64 == 0 && HD / 4 <= 32, "");
    constexpr int TPC = HD / 4;            // threads per chunk: 4 consecutive features each
    constexpr int NG = NT / TPC;           // chunk groups working side by side
    // block row r: its sequence's rows, length and first unit (a plain step: the cache itself)
    int gamma = a.rows, len = a.st->len, row0 = 0, unit_s = 0;
    if (a.batched) {
        const pv_seq_ref &sq = a.st->blk.seq[max((a.st->rowphys[r] >> PV_SEQ_TAG_SHIFT) - 1, 0)];      // (a batch of one carries no tag)
        gamma = sq.gamma; len = sq.st->len; row0 = sq.row0; unit_s = sq.unit0;
    }
    const int j = r - row0;
    const int kvh = aq / a.group, al = aq - kvh * a.group, m = al * gamma + j, mp = m >> 5, row = m & 31;
    const size_t unit0 = ((size_t)kvh * n_units + unit_s + mp) * a.max_chunks;
    float *sh_m = smem;                                              // [NT]
    float (*sh_acc)[TPC][8] = (float (*)[TPC][8])(smem + NT);        // [waves][TPC][8]
    const int t = tid % TPC, cg = tid / TPC;
    float acc[4] = {0.f, 0.f, 0.f, 0.f}, L = 0.f;
    // Up to 256 chunks: lane c of every wave holds (max, sum) of the chunks c, c + 64, ...; the global max, the
    // weights and the total come from wave shuffles (every wave redundantly, no barrier), and
    // the partial outputs are fetched eight chunks at a time with nothing depending on them.  Statistics and the first outputs go out beside the
    // length, for as many chunks as were launched, whatever the length turns out to be: one memory round trip instead of three
    // (with the rows as an argument 3462 -> 3442 us for 8 steps of four 8B-shaped layers; the kernel stays at the 4.6 us that any small kernel takes here).
    // Not for as many as the cache has room for: 1000 of 32768 tokens, 64 rows, two layers, 70B shape 975 -> 924 us, 8B shape 369 -> 342 a step.
    // More than 64 chunks, or 32 (128 features), were a loop of round trips before: 65 chunks 6.4 -> 4.7 us, 94 chunks 7.5 -> 5.8.
    constexpr int SL = 4, FL = 8;
    const int lane = tid & 63;
    // (a row of a unit: places known to the whole workgroup, its up to 256 chunks 32-bit offsets behind them)
    const char *pm = (const char *)uniform_ptr(a.part_ml + (unit0 * 32 + row) * 2), *po = (const char *)uniform_ptr(a.part_o + (unit0 * 32 + row) * HD);
    float2 ml[SL];
#pragma unroll
    for (int q = 0; q < SL; ++q) {
        ml[q] = make_float2(-INFINITY, 0.f);
        if (q == 0 || 64 * q < a.chunks) ml[q] = *(const float2 *)(pm + (uint32_t)min(64 * q + lane, a.chunks - 1) * 256u);
    }
    float4 o[FL];
    auto fetch = [&](int base) {
#pragma unroll
        for (int u = 0; u < FL; ++u)
            if (u == 0 || base + u * NG < a.chunks) o[u] = *(const float4 *)(po + ((uint32_t)min(base + cg + u * NG, a.chunks - 1) * (128u * HD) + 16 * t));
    };
    fetch(0);
    asm volatile("" ::: "memory");
    const int nchunks = (len + gamma + (1 << a.chunk_shift) - 1) >> a.chunk_shift;
    if (nchunks <= 64 * SL) {
        float M = -INFINITY, wl[SL];
#pragma unroll
        for (int q = 0; q < SL; ++q) { if (64 * q + lane >= nchunks) ml[q] = make_float2(-INFINITY, 0.f); M = fmaxf(M, ml[q].x); }
        M = over_wave(M, op_max);
#pragma unroll
        for (int q = 0; q < SL; ++q) { wl[q] = (ml[q].x == -INFINITY) ? 0.f : expf(ml[q].x - M); L += ml[q].y * wl[q]; }
        L = over_wave(L, op_add);
        for (int base = 0; base < nchunks; base += FL * NG) {     // same trip count in every lane: the shuffles below need all lanes
            if (base > 0) fetch(base);
#pragma unroll
            for (int u = 0; u < FL; ++u) {
                const int c0 = base + u * NG, c = c0 + cg;        // (NG divides 64: c0 / 64 = c / 64)
                if (c0 >= nchunks) break;
                const float v = c0 < 64 ? wl[0] : c0 < 128 ? wl[1] : c0 < 192 ? wl[2] : wl[3];
                const float w = __shfl(v, c & 63, 64);
                if (c < nchunks) { acc[0] += w * o[u].x; acc[1] += w * o[u].y; acc[2] += w * o[u].z; acc[3] += w * o[u].w; }      // (others were never written this step: anything)
            }
        }
        if (cg != 0) L = 0.f;                     // the total is added up over the chunk groups below: count it once
    } else {
        // more: each thread looks at chunks tid, tid+NT, ... and a tree in LDS finishes the max
        float M = -INFINITY;
        for (int c = tid; c < nchunks; c += NT) M = fmaxf(M, a.part_ml[((unit0 + c) * 32 + row) * 2]);
        sh_m[tid] = M;
        __syncthreads();
        for (int s2 = NT / 2; s2 > 0; s2 >>= 1) {
            if ((int)tid < s2) sh_m[tid] = fmaxf(sh_m[tid], sh_m[tid + s2]);
            __syncthreads();
        }
        M = sh_m[0];
        for (int c = cg; c < nchunks; c += NG) {
            const float *pm = a.part_ml + ((unit0 + c) * 32 + row) * 2;
            const float w = (pm[0] == -INFINITY) ? 0.f : expf(pm[0] - M);
            L += pm[1] * w;
            const float4 oc = *(const float4 *)(a.part_o + ((unit0 + c) * 32 + row) * HD + 4 * t);
            acc[0] += w * oc.x; acc[1] += w * oc.y; acc[2] += w * oc.z; acc[3] += w * oc.w;
        }
    }
    // the chunk groups of a wave first (TPC lanes apart), then the waves
    float v[5] = {acc[0], acc[1], acc[2], acc[3], L};
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        v[i] = with_lane32(v[i], op_add);
        if (TPC <= 16) v[i] = with_lane16(v[i], op_add);
        if (TPC <= 8) v[i] = with_rotated<8>(v[i], op_add);
    }
    const int w = tid >> 6;
    if ((tid & 63) < TPC) {
        *(float4 *)sh_acc[w][t] = make_float4(v[0], v[1], v[2], v[3]);
        sh_acc[w][t][4] = v[4];
    }
    __syncthreads();
    if (tid >= TPC) return;
    L = 0.f;
    acc[0] = acc[1] = acc[2] = acc[3] = 0.f;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) {
        const float4 p = *(const float4 *)sh_acc[k][t];
        acc[0] += p.x; acc[1] += p.y; acc[2] += p.z; acc[3] += p.w; L += sh_acc[k][t][4];
    }
    const float inv = 1.0f / L;
    const float y[4] = {acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
    store_operand4<NB>(a.xop_o, a.n_q_heads * HD, r, aq * HD + 4 * t, y, a.rows);
}

