// Matrix-core kernel family for bf16 models.
//
// Skinny GEMMs y[rows<=64][N] = x[rows][K] W^T stream W once from HBM.  W is stored pre-tiled
// in MFMA operand order: strips of 16 output features, each strip a run of K/32 tiles of
// 16x32 bf16 (1 KiB), a tile laid out [lane 0..63][8 bf16] so that one 16-byte load per lane
// is exactly the A operand of v_mfma_f32_16x16x32_bf16.  Up to 16 rows (k_gemm): a workgroup
// owns one or a few strips, its wavefronts split K, accumulate in fp32, and are summed in wave
// order through LDS, so the owner sees complete outputs and the whole epilogue (RMSNorm scale,
// rotary embedding + KV append, SwiGLU, residual add, vocabulary arg-max) is fused into the
// GEMM.  Many strips, where whole rounds of CUs come out of them (k_gemm_wide): the same with one workgroup per CU;
// 4-bit weights and up to 16 rows: k_gemm_q4.  Else, from 17 rows on (k_gemm_tile; with 4-bit weights k_gemm_tile_q4): the waves
// of a workgroup own different strips, walk K together and share the activation tiles through LDS.
//
// Activations enter as the B operand.  To keep fp32-grade accuracy with bf16 matrix cores an
// activation a is carried as two bf16 numbers hi = bf16(a), lo = bf16(a - hi) (16 mantissa
// bits).  A block of R <= 8 rows is packed: a tile of 2 R columns holds hi of row j in column j and lo in column
// R + j (store_operand4; packed_lane puts them where one MFMA does both and the epilogue adds the two halves);
// for more rows hi and lo are separate operands and two MFMAs accumulate into the same registers.
//
// RMSNorm is folded in: the producer of x writes (gain * x) as the next operand plus per-strip
// partial sums of x^2; the consumer multiplies its outputs by rsqrt(mean + eps), which
// commutes with the contraction.  Rows of W_q/W_k are permuted inside each head so that the two
// members of a rotary pair sit in the same half of a strip, 4 rows apart (lanes l and l^16 of
// the accumulator; either 8-row half of a strip holds 4 whole pairs); gate and up rows are
// interleaved the same way for SwiGLU (4 gate + 4 up features per half strip).
#include <stdio.h>
#include <stdlib.h>
#include <type_traits>
#include "pv_gemm_epilogue.h"
#include "pv_prefill.h"



struct mat_ws {                 // carved out of pv_ws::part
    uint16_t *xop_a, *xop_o, *xop_f, *xop_d;   // operands: QKV in (K=d), O in (K=qd), gate/up in (K=d), down in (K=F)
    float *ssq0, *ssq1;                         // [column tile][d/16][16] partial sums of x^2
    float *pmax_val; int32_t *pmax_idx;         // [row][vocab/16] per-strip arg-max candidates, row-major
    float *attn_part;                           // attention chunk partials
    float *tile_part;                           // K-slice partial sums of the wide-block GEMMs (TILE_PART_FLOATS)
};

static inline size_t xop_elems(int K) { return (size_t)2 * (K / 32) * 512; }   // hi and lo arrays of one 16-row column tile
static inline int col_tiles(int rows) { return rows <= 16 ? 1 : rows <= 32 ? 2 : 4; }
// K-slice partial sums of the shared-tile GEMMs: slices x strips x column tiles KiB.  The launches cut a GEMM into at most 16
// slices and 256 workgroups in all (512 for 4-bit weights and up to 32 rows), which bounds slices x strips by 16 x 512 (16 strips per
// workgroup; fewer with 8), i.e. 2 Mi floats per column tile; 24 MiB in all, which the launches stay under.
static const size_t TILE_PART_FLOATS = (size_t)6 << 20;
static inline size_t tile_part_floats(int col_tiles) { return std::min(TILE_PART_FLOATS, (size_t)col_tiles << 21); }
// blocks that use those kernels: more than 16 rows, or any block with 4-bit weights
static inline bool tile_part_needed(const pv_model *m, int col_tiles) { return col_tiles >= 2 || m->wbits == 4; }
// 16-bit weights and up to 16 rows, where O and down projections are cut (cut_slices): at most a group of four strips and a slice per CU
static inline size_t cut_part_floats(const pv_model *m) { return (size_t)m->n_cus * 4 * 256; }

// slices: with room for the sums of cut projections in a layout of up to 16 rows; without it (have: the floats that there are) these projections stay whole
static size_t mat_ws_layout(const pv_model *m, int rows_cap, int units_cap, int max_tokens, bool slices, float *base, mat_ws *w, size_t have = 0)
{
    const pv_model_config &f = m->cfg;
    const int qd = f.n_q_heads * f.head_dim;
    const size_t ctc = col_tiles(rows_cap);          // every per-row piece is sized for the widest block
    size_t off = 0;   // in floats, every piece a multiple of 64 floats (256 B)
    auto take = [&](size_t floats) { size_t o = off; off += (floats + 63) / 64 * 64; return base ? base + o : (float *)nullptr; };
    float *p;
    p = take(ctc * xop_elems(f.d_model) / 2); if (w) w->xop_a = (uint16_t *)p;
    p = take(ctc * xop_elems(qd) / 2); if (w) w->xop_o = (uint16_t *)p;
    p = take(ctc * xop_elems(f.d_model) / 2); if (w) w->xop_f = (uint16_t *)p;
    p = take(ctc * xop_elems(f.ffn_dim) / 2); if (w) w->xop_d = (uint16_t *)p;
    p = take(ctc * (size_t)f.d_model); if (w) w->ssq0 = p;
    p = take(ctc * (size_t)f.d_model); if (w) w->ssq1 = p;
    p = take(ctc * (size_t)f.vocab); if (w) w->pmax_val = p;
    p = take(ctc * (size_t)f.vocab); if (w) w->pmax_idx = (int32_t *)p;
    p = take(pv_attn_part_floats(m, units_cap, max_tokens)); if (w) w->attn_part = p;
    const size_t tp = tile_part_needed(m, (int)ctc) ? tile_part_floats((int)ctc) : slices ? cut_part_floats(m) : 0;
    p = take(tp); if (w) w->tile_part = tp && off <= have ? p : nullptr;  // (none: the launches then do not slice)
    return off;
}

size_t pv_mat_part_floats(const pv_model *m, int rows_cap, int units_cap, int max_tokens, bool slices) { return mat_ws_layout(m, rows_cap, units_cap, max_tokens, slices, nullptr, nullptr); }

// ------------------------------------------------------------------------------------------
// Weight repack: rows [row_begin, row_begin+row_count) of one tensor, row-major in staging,
// into the tiled region.  One thread moves 8 consecutive K elements (16 bytes).
// ------------------------------------------------------------------------------------------
enum { PERM_NONE = 0, PERM_ROPE = 1, PERM_GATEUP = 2 };

__global__ void k_repack(const uint4 *src, uint4 *dst, int64_t row_begin, int64_t row_count, int K,
                         int perm, int head_dim, int strip_mul, int strip_add)
{
    const int kg = K / 8;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= row_count * kg) return;
    const int64_t n = row_begin + idx / kg;
    const int kb = (int)(idx % kg);                 // group of 8 along K
    int64_t strip; int i;
    if (perm == PERM_ROPE) {
        const int half = head_dim / 2, e = (int)(n % head_dim);
        const int64_t h = n / head_dim;
        const int side = e >= half, p = e - side * half;
        strip = h * (head_dim / 16) + p / 8; i = (p & 3) + 4 * side + 8 * ((p >> 2) & 1);
    } else if (perm == PERM_GATEUP) {
        strip = n / 8; i = (int)(n & 3) + 4 * strip_add + 8 * (int)((n >> 2) & 1);   // strip_add: 0 = gate, 1 = up
    } else {
        strip = (n / 16) * strip_mul + strip_add; i = (int)(n & 15);
    }
    const int kt = kb / 4, lane = i + 16 * (kb & 3);
    dst[((size_t)strip * (K / 32) + kt) * 64 + lane] = src[idx];
}

int pv_mat_repack(const pv_model *m, const pv_tensor_ref &t, int kind, int64_t row_begin, int64_t row_count, hipStream_t s)
{
    int perm = PERM_NONE, mul = 1, add = 0;
    if (kind == PV_T_WQ || kind == PV_T_WK) perm = PERM_ROPE;
    else if (kind == PV_T_WG || kind == PV_T_WU) { perm = PERM_GATEUP; add = t.strip_add; }
    const int64_t n = row_count * (t.cols / 8);
    k_repack<<<(unsigned)((n + 255) / 256), 256, 0, s>>>((const uint4 *)m->d_staging, (uint4 *)(m->d_weights + t.off),
                                                         row_begin, row_count, (int)t.cols, perm, m->cfg.head_dim, mul, add);
    PV_HIP(hipGetLastError());
    return PV_OK;
}

// Rows of a 4-bit matrix, row-major in staging (codes: K/8 dwords per row, a dword = 8 consecutive
// k, low nibble first; scales: K/32 bf16 per row), into the batched strip layout (pv_internal.h).
// One thread moves one dword of codes; the thread of a tile's first dword also moves its scale.
__global__ void k_repack_q4(const uint32_t *codes, const uint16_t *scales, char *dst, int64_t row_begin, int64_t row_count,
                            int K, int perm, int head_dim, int strip_mul, int strip_add, uint32_t *wide)
{
    const int kd = K / 8, nb4 = K / 128;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= row_count * kd) return;
    const int64_t nl = idx / kd, n = row_begin + nl;
    const int w = (int)(idx % kd), kt = w >> 2, q = w & 3;      // tile, feature-of-k group
    int64_t strip; int i;
    if (perm == PERM_ROPE) {
        const int half = head_dim / 2, e = (int)(n % head_dim);
        const int64_t h = n / head_dim;
        const int side = e >= half, p = e - side * half;
        strip = h * (head_dim / 16) + p / 8; i = (p & 3) + 4 * side + 8 * ((p >> 2) & 1);
    } else if (perm == PERM_GATEUP) {
        strip = n / 8; i = (int)(n & 3) + 4 * strip_add + 8 * (int)((n >> 2) & 1);
    } else {
        strip = (n / 16) * strip_mul + strip_add; i = (int)(n & 15);
    }
    char *batch = dst + ((size_t)strip * nb4 + (kt >> 2)) * PV_Q4_BATCH;
    const int u = kt & 3;
    // the lane's 8 codes c0..c7 (source: c0 in the lowest nibble) are stored as
    // (c0 | c2 << 4 | c4 << 8 | c6 << 12) | (c1 | c3 << 4 | c5 << 8 | c7 << 12) << 16,
    // so that one shift and one mask give the bf16 pair (k = 2t, 2t + 1) of operand dword t
    const uint32_t src = codes[idx];
    uint32_t even = 0, odd = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) { even |= ((src >> (8 * t)) & 0xFu) << (4 * t); odd |= ((src >> (8 * t + 4)) & 0xFu) << (4 * t); }
    ((uint32_t *)batch)[(i + 16 * q) * 4 + u] = even | (odd << 16);
    if (q == 0) {
        const uint16_t sc = scales[nl * (K / 32) + kt];
        ((uint16_t *)(batch + 1024))[i * 4 + u] = sc;
        // (c - 8) x scale and scale / 16 are exact in f16 for scales of 0 and of 2^-13 .. 2^12
        const int e = (sc >> 7) & 0xFF;
        if ((sc & 0x7FFF) != 0 && (e < 114 || e > 138)) *wide = 1;
    }
}

int pv_mat_repack_q4(const pv_model *m, const pv_tensor_ref &t, int kind, int64_t row_begin, int64_t row_count, size_t scales_off, uint32_t *wide, hipStream_t s)
{
    int perm = PERM_NONE, mul = 1, add = 0;
    if (kind == PV_T_WQ || kind == PV_T_WK) perm = PERM_ROPE;
    else if (kind == PV_T_WG || kind == PV_T_WU) { perm = PERM_GATEUP; add = t.strip_add; }
    const int64_t n = row_count * (t.cols / 8);
    k_repack_q4<<<(unsigned)((n + 255) / 256), 256, 0, s>>>((const uint32_t *)m->d_staging, (const uint16_t *)(m->d_staging + scales_off),
                                                            m->d_weights + t.off, row_begin, row_count, (int)t.cols, perm, m->cfg.head_dim, mul, add, wide);
    PV_HIP(hipGetLastError());
    return PV_OK;
}

// Block set-up on the matrix path: embedding rows -> x, first operand, first sum of squares;
// rotary table for positions len .. len+rows-1.  The draft ids come straight from the cache's
// pinned host mailbox; one workgroup copies them, the row count and the mode into the
// device state for the kernels that follow.
template <int NB>
__global__ void __launch_bounds__(64)
k_mat_begin(pv_dev_state *st, const int32_t *mailbox, int rows, int mode, const uint16_t *embed, const uint16_t *gain, const double *inv_freq,
            float *x, float *ssq, uint16_t *xop, float2 *rope, int d, int half, const int32_t *page_table, int page_shift)
{
    const int lane = threadIdx.x, ct = blockIdx.y, j = ct * 16 + (lane & 15), g = lane >> 4, strip = blockIdx.x;
    const int nseq = st->blk.n_seq;
    const bool tree = mode == PV_MODE_TREE, writes_rows = blockIdx.x == gridDim.x - 1 && ct == 0;
    // The token ids come over the bus, the longest trip of all: asked for first, the rotary table meanwhile.  (The last workgroup along the strips writes the rows' state, the first ones
    // the table.  8B shape, 8 rows, inside the kernel 4.5 -> 3.6 us.)
    const int tok = j < rows ? mailbox[j] : 0, own = writes_rows && lane < rows ? mailbox[lane] : 0;
    const uint2 gn = *(const uint2 *)(gain + strip * 16 + 4 * g);
    __shared__ int parent[PV_MAX_ROWS];               // draft tree: the parents follow the draft ids in the mailbox; one read each, then walked in LDS
    if (tree) { parent[lane] = lane < rows ? mailbox[PV_MAX_ROWS + lane] : -1; __syncthreads(); }
    // Cache slot of block row r: the cache's length + r, or in a batched step the length of the row's
    // sequence + the row's index inside that sequence's block.  Its rotary position is the same, except in a
    // draft tree, where a row sits at (length + its depth) whatever slot it is stored in.
    auto seq_of = [&](int r) { int sidx = 0; for (int k = 1; k < nseq; ++k) if (r >= st->blk.seq[k].row0) sidx = k; return sidx; };
    auto slot_of = [&](int r) { if (nseq <= 1) return st->len + r; const pv_seq_ref &sq = st->blk.seq[seq_of(r)]; return sq.st->len + r - sq.row0; };
    auto depth_of = [&](int r) { int dpt = 0; for (int q = parent[r]; q >= 0 && dpt < PV_MAX_ROWS; q = parent[q]) ++dpt; return dpt; };
    if (ct == 0)
        for (int idx = blockIdx.x * 64 + lane; idx < rows * half; idx += gridDim.x * 64) {
            const int jj = idx / half, i = idx - jj * half;
            double sn, cs;
            sincos((double)(tree ? st->len + depth_of(jj) : slot_of(jj)) * inv_freq[i], &sn, &cs);
            rope[idx] = make_float2((float)cs, (float)sn);
        }
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (j < rows) {
        const uint2 e = *(const uint2 *)(embed + (size_t)tok * d + strip * 16 + 4 * g);
        v[0] = pv_bf16_to_f32((uint16_t)(e.x & 0xffffu)); v[1] = pv_bf16_to_f32((uint16_t)(e.x >> 16));
        v[2] = pv_bf16_to_f32((uint16_t)(e.y & 0xffffu)); v[3] = pv_bf16_to_f32((uint16_t)(e.y >> 16));
    }
    emit_x<NB>(lane, rows, strip, d, v, gn, x, ssq, xop, ct, rows);
    if (writes_rows) {
        if (const int i = lane; i < rows) {           // (at most 64 rows)
            const int pos = slot_of(i);
            st->draft[i] = own; st->rowpos[i] = pos;
            if (nseq <= 1) st->rowphys[i] = page_table[pos >> page_shift];
            else { const int sidx = seq_of(i); st->rowphys[i] = st->blk.seq[sidx].page_table[pos >> page_shift] | (sidx + 1) << PV_SEQ_TAG_SHIFT; }
            uint64_t m;
            if (tree) { m = 1ull << i; for (int q = parent[i], k = 0; q >= 0 && k < PV_MAX_ROWS; q = parent[q], ++k) m |= 1ull << q; st->parent[i] = parent[i]; }
            else { const int jj = i - (nseq <= 1 ? 0 : st->blk.seq[seq_of(i)].row0); m = jj >= 63 ? ~0ull : (2ull << jj) - 1; }
            st->rowmask[i] = m;
        }
        if (lane == 0) { st->gamma = rows; st->mode = mode; if (nseq <= 1) st->blk.seq[0].gamma = rows; }
    }
}

// A wave's K walk with DEPTH register buffers: while one batch is used, the loads of the next
// DEPTH - 1 are in flight.  issue(q, k) starts the loads of the wave's k-th batch into q,
// consume(q, k) uses it; between() runs once behind the first loads (work that may wait on older,
// shorter loads).  Buffers rotate by name, so the steady state is unrolled DEPTH times and every
// issue in it is unconditional: the wait before a consume then only covers that batch's loads.
template <int DEPTH, typename Q, typename FI, typename FC, typename FB>
__device__ inline void k_walk(int cnt, Q &q0, Q &q1, Q &q2, FI issue, FC consume, FB between)
{
    if (cnt > 0) issue(q0, 0);
    if (DEPTH == 3 && cnt > 1) issue(q1, 1);
    between();
    int i = 0;
    if constexpr (DEPTH == 3) {
        for (; i + 4 < cnt; i += 3) {                // q0 and q1 hold batches i and i + 1, in flight or landed
            issue(q2, i + 2); consume(q0, i);
            issue(q0, i + 3); consume(q1, i + 1);
            issue(q1, i + 4); consume(q2, i + 2);
        }
        if (i + 2 < cnt) issue(q2, i + 2);            // at most four batches are left
        if (i < cnt) consume(q0, i);
        if (i + 3 < cnt) issue(q0, i + 3);
        if (i + 1 < cnt) consume(q1, i + 1);
        if (i + 2 < cnt) consume(q2, i + 2);
        if (i + 3 < cnt) consume(q0, i + 3);
    } else {
        for (; i + 2 < cnt; i += 2) {                // q0 holds batch i
            issue(q1, i + 1); consume(q0, i);
            issue(q0, i + 2); consume(q1, i + 1);
        }
        if (i + 1 < cnt) issue(q1, i + 1);            // at most two batches are left
        if (i < cnt) consume(q0, i);
        if (i + 1 < cnt) consume(q1, i + 1);
    }
}

// Loads through buffer descriptors: the lane's offset in a register, the wave's in a scalar, zeros (and no traffic) past the end.
__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, bytes, 0x00020000); }
#define BUFFER_END 0xC0000000u                     // past the end of every buffer, and no sum with an offset inside one wraps: k_gemm_wide up to wide_fits, k_gemm_q4 up to pv_offsets_fit
template <int AUX> __device__ inline uint4 buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t base)
{
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, off, base, AUX));
}
template <int AUX> __device__ inline uint2 buffer_load8(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t base)
{
    return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, off, base, AUX));
}
#define LOAD_ONCE 2                                // the non-temporal bit (see load_once)

// Where lane l of the B operand reads inside a packed tile of R rows, in uint4s: its columns 0..7 are the rows' hi parts, 8..15 their
// lo parts (R <= 8; the columns in between read the last row again: no further line, and their results are never used).
__device__ inline int packed_lane(int lane, int R)
{
    const int col = lane & 15;
    return (lane >> 4) * 2 * R + (col < 8 ? min(col, R - 1) : R + min(col - 8, R - 1));
}

// The attention's chunks of a small block, merged by every workgroup of the output projection for itself, into operand tiles in LDS.  A thread takes
// IT (row, four features) items at a time, all their up to MG chunks in flight at once, beside the first weights.  Arithmetic of
// attn_merge_unit.  A chunk beyond the keys has left nothing: its weight is 0 and its values are not used.
constexpr int merge_items(int mg) { return 8 / mg; }
template <int MG, int NT>
__device__ inline void merge_chunks(const gemm_args &a, uint16_t *dst)
{
    constexpr int IT = merge_items(MG);
    const int R = a.rows, hd = a.geom.head_dim, K = a.ktiles * 32, group = a.n_q_heads / a.geom.n_kv_heads, items = R * (K >> 2);
    const int len = a.st->len;
    for (int i0 = threadIdx.x; i0 < items; i0 += NT * IT) {
        float2 ml[IT][MG];
        float4 o[IT][MG];
#pragma unroll
        for (int v = 0; v < IT; ++v) {
            const int i = min(i0 + v * NT, items - 1), j = i / (K >> 2), k = (i - j * (K >> 2)) * 4, aq = k / hd, kvh = aq / group, m = (aq - kvh * group) * R + j;
            const size_t unit0 = ((size_t)kvh * a.units + (m >> 5)) * a.max_chunks;
#pragma unroll
            for (int c = 0; c < MG; ++c) {
                const size_t at = (unit0 + min(c, a.chunks - 1)) * 32 + (m & 31);
                ml[v][c] = *(const float2 *)(a.part_ml + at * 2);
                o[v][c] = *(const float4 *)(a.part_o + at * hd + (k - aq * hd));
            }
        }
        const int n = (len + R + (1 << a.chunk_shift) - 1) >> a.chunk_shift;
#pragma unroll
        for (int v = 0; v < IT; ++v) {
            const int i = i0 + v * NT, j = i / (K >> 2), k = (i - j * (K >> 2)) * 4;
            if (i >= items) break;
            float M = ml[v][0].x;
#pragma unroll
            for (int c = 1; c < MG; ++c) if (c < n) M = fmaxf(M, ml[v][c].x);
            float L = 0.f, y[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < MG; ++c)
                if (c < n) {
                    const float w = (ml[v][c].x == -INFINITY) ? 0.f : expf(ml[v][c].x - M);
                    L += ml[v][c].y * w;
                    y[0] += w * o[v][c].x; y[1] += w * o[v][c].y; y[2] += w * o[v][c].z; y[3] += w * o[v][c].w;
                }
            const float inv = 1.0f / L;
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] *= inv;
            store_operand4<1>(dst, K, j, k, y, R);
        }
    }
}

// ------------------------------------------------------------------------------------------
// The streaming GEMM: a workgroup owns S adjacent strips, its NW waves split K in batches of U
// tiles.
//
// Rows: NB == 1 packs up to 8 rows (hi and lo halves in one operand; CT == 1).  NB == 2 takes
// the rows in CT column tiles of 16, each with a hi and a lo operand, and keeps S x CT
// accumulators: every operand tile fetched from L2 is used for S strips from registers, which
// keeps the operand traffic (2 CT tiles per batch tile) from outgrowing the weight stream
// (S tiles) in the CU's load path.  (CT > 1 is only used for a K too short for k_gemm_tile.)
//
// K assignment: contiguous runs of batches per wave, or batch b to wave b % NW (the workgroup
// then reads its strips as advancing windows).
// ------------------------------------------------------------------------------------------
//
// DP > 1 (one column tile): the wave keeps DP batches in registers and loads
// ahead (k_walk): bytes in flight come from depth per wave rather than from the number of
// resident waves.  HF: the last of the S strips is an 8-feature half (see below).
//
template <int NB, int CT, int S, int EPI, int NW, int DP = 1, bool HF = false, int MG = 0>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu((NB == 1 && S == 1 && DP == 1) ? 6 : (S * CT >= 16) ? 2 : 4)))   // packed bf16 rows, one strip, a short K: latency is hidden by resident waves (three workgroups per CU at <= 80 VGPRs); 16 accumulator tiles (wide blocks with a short K): more than 128
k_gemm(const gemm_args a)
{
    static_assert(NB == 2 || CT == 1, "packed rows come in one tile");
    static_assert(S <= NW, "one epilogue wave per strip");
    static_assert(!HF || DP > 1, "half strips: walked batches");
    static_assert(MG == 0 || (NB == 1 && DP > 1 && EPI == EPI_RESID), "merged operand: packed rows, output projection");
    constexpr int U = (S * CT >= 16) ? 1 : (S * CT >= 4) ? 2 : (DP > 1 && (S >= 2 || NB == 2)) ? 2 : 4;   // tiles per batch
    constexpr bool NORM = (EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_LMHEAD);
    constexpr bool PARK = (CT == 1);                 // epilogue inputs fetched early (by the wave that will run the strip's epilogue) and parked in LDS
    // HF: the workgroup owns S - 1 whole strips and one 8-feature half of a strip it shares with
    // its neighbour (strips a.half_base ...), so that a GEMM with (k + 1/2) x 256 strips puts the
    // same bytes on every CU; the lanes of the other half duplicate the owned half's loads for
    // that slot and their rows of the product are not stored.
    // Two strips a workgroup and a short K: many workgroups with little to do each.  All arguments are asked for at once; left alone, the compiler asks for the weights' only
    // behind the first loads, one more trip to memory a workgroup (13 rows, gate/up, us: K = 512, 1376 strips 8.9 -> 8.4, 1536 strips 9.2 -> 9.0; K = 1024, 11.8 -> 11.5, 13.2 -> 13.0).
    // Elsewhere no difference or, with one strip, up to 0.1 us more.
    if constexpr (NB == 2 && CT == 1 && S == 2 && DP == 1) asm volatile("" :: "s"(a.W), "s"(a.xop), "s"(a.ktiles), "s"(a.interleave), "s"(a.nstrips), "s"(a.rows), "s"(a.ssq), "s"(a.ssq_parts));
    const int strip0 = blockIdx.x * (HF ? S - 1 : S), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int hstrip = HF ? a.half_base + ((int)blockIdx.x >> 1) : 0, hsel = blockIdx.x & 1;
    const int hl = HF ? ((lane & ~8) | (hsel << 3)) - lane : 0;    // half slot: the lanes of the other half read the owned half's lines again (no further bytes)
    const int KT = a.ktiles, nbat = KT / U;        // whole batches of U tiles; a ragged rest goes to the last wave
    const size_t arr = (size_t)KT * 64;             // tiles of one strip = elements of one operand array, in uint4
    const uint4 *A = a.W + (size_t)strip0 * arr + lane;
    // tile ct: hi at B + (2 ct) arr, lo at B + (2 ct + 1) arr   (NB == 2)
    const uint4 *B = a.xop + lane;
    const uint32_t xs = NB == 1 ? 128u * (uint32_t)a.rows : 1024u, xl = (NB == 1 ? packed_lane(lane, a.rows) : lane) * 16;   // bytes of an operand tile, the lane's place in it
    const __amdgpu_buffer_rsrc_t P = buffer_of(a.xop, NB * (uint32_t)KT * xs);
    auto operand = [&](int t) { return buffer_load16<0>(P, xl, (uint32_t)t * xs); };        // one column tile: K-tile t, the lo halves of a 16-row tile at KT + t (the same t for the whole wave)
    // a ragged last workgroup re-reads its first strip for the missing ones and drops the result
    size_t so[S];
#pragma unroll
    for (int si = 0; si < S; ++si) so[si] = (HF && si == S - 1) ? (size_t)(hstrip - strip0) * arr : (strip0 + si < a.nstrips) ? (size_t)si * arr : 0;
    f32x4 acc[S][CT];
#pragma unroll
    for (int si = 0; si < S; ++si)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[si][ct] = (f32x4){0.f, 0.f, 0.f, 0.f};

    __shared__ f32x4 red[NW][S][CT][64];
    __shared__ float ssq_s[NW][CT][16];
    __shared__ epi_pre pre_s[PARK ? S : 1][PARK ? 64 : 1];
    extern __shared__ uint4 merged[];               // MG > 0: the operand's packed tiles

    // RMSNorm of the input rows: every wave takes its share of the per-strip sums of squares; the
    // loads go out ahead of the weight stream and are folded in behind its first batch
    ssq_loads<2> sl[CT];
    if (NORM) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) ssq_issue(a.ssq + (size_t)ct * a.ssq_parts * 16, a.ssq_parts, threadIdx.x, NW * 64, sl[ct]);
    }

    if constexpr (DP > 1) {
        static_assert(CT == 1, "deep variant: one column tile");
        struct wbatch { uint4 w[S][U], x[U], xl[NB == 2 ? U : 1]; };     // xl: the lo halves of a 16-row tile
        int first, cnt, bstride;
        if (a.interleave) { first = wave; bstride = NW; cnt = wave < nbat ? (nbat - wave + NW - 1) / NW : 0; }
        else { const int per = (nbat + NW - 1) / NW; first = min(nbat, wave * per); cnt = min(nbat, first + per) - first; bstride = 1; }
        auto issue = [&](wbatch &q, int k) {
            const size_t o = (size_t)(first + k * bstride) * U * 64;
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int si = 0; si < S; ++si) q.w[si][u] = load_once(&A[so[si] + o + u * 64 + ((HF && si == S - 1) ? hl : 0)]);
                if (MG == 0) q.x[u] = operand((first + k * bstride) * U + u);
                if (NB == 2) q.xl[NB == 2 ? u : 0] = operand(KT + (first + k * bstride) * U + u);
            }
            asm volatile("" ::: "memory");
        };
        auto consume = [&](const wbatch &q, int k) {
            (void)k;
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int si = 0; si < S; ++si) {
                    acc[si][0] = mfma16(q.w[si][u], MG > 0 ? merged[((first + k * bstride) * U + u) * (xs >> 4) + (xl >> 4)] : q.x[u], acc[si][0]);
                    if (NB == 2) acc[si][0] = mfma16(q.w[si][u], q.xl[NB == 2 ? u : 0], acc[si][0]);
                }
        };
        wbatch q0, q1, q2;
        k_walk<DP>(cnt, q0, q1, q2, issue, consume, [&]() {
            if constexpr (MG > 0) { merge_chunks<MG, NW * 64>(a, (uint16_t *)merged); __syncthreads(); }      // (every wave comes here once)
            if (NORM) {
                const float4 s4 = ssq_finish(a.ssq, a.ssq_parts, threadIdx.x, NW * 64, sl[0]);
                if (lane < 4) *(float4 *)&ssq_s[wave][0][4 * lane] = s4;
            }
            if (PARK && wave < S) {
                epi_pre pre;
                epi_prefetch<EPI>(a, (HF && wave == S - 1) ? hstrip : min(strip0 + wave, a.nstrips - 1), lane, pre, 0);
                epi_park<EPI>(&pre_s[wave][lane], pre);
            }
        });
        if (wave == NW - 1) {
            for (int t = nbat * U; t < KT; ++t) {
                const uint4 x = MG > 0 ? merged[t * (xs >> 4) + (xl >> 4)] : operand(t);
                uint4 xl = x;
                if (NB == 2) xl = operand(KT + t);
#pragma unroll
                for (int si = 0; si < S; ++si) {
                    const uint4 w = load_once(&A[so[si] + (size_t)t * 64 + ((HF && si == S - 1) ? hl : 0)]);
                    acc[si][0] = mfma16(w, x, acc[si][0]);
                    if (NB == 2) acc[si][0] = mfma16(w, xl, acc[si][0]);
                }
            }
        }
    } else {
    int b, bend, bstep;
    if (a.interleave) { b = wave; bend = nbat; bstep = NW; }
    else { const int per = (nbat + NW - 1) / NW; b = min(nbat, wave * per); bend = min(nbat, b + per); bstep = 1; }
    uint4 ra[S][U], rb[CT][U], rc[CT][U];
    auto load_batch = [&](int t) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t o = (size_t)(t + u) * 64;
#pragma unroll
            for (int si = 0; si < S; ++si) ra[si][u] = load_once(&A[so[si] + o]);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                rb[ct][u] = NB == 1 ? operand(t + u) : B[(size_t)(2 * ct) * arr + o];
                if (NB == 2) rc[ct][u] = B[(size_t)(2 * ct + 1) * arr + o];
            }
        }
    };
    auto use_batch = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int si = 0; si < S; ++si)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    acc[si][ct] = mfma16(ra[si][u], rb[ct][u], acc[si][ct]);
                    if (NB == 2) acc[si][ct] = mfma16(ra[si][u], rc[ct][u], acc[si][ct]);
                }
    };

    // Few registers on purpose (NB == 1): latency is hidden by many resident waves per CU.
    {   // first batch peeled: the sums of squares are folded in while its loads are in flight
        const bool first = b < bend;
        if (first) load_batch(b * U);
        if (NORM) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const float4 s4 = ssq_finish(a.ssq + (size_t)ct * a.ssq_parts * 16, a.ssq_parts, threadIdx.x, NW * 64, sl[ct]);
                if (lane < 4) *(float4 *)&ssq_s[wave][ct][4 * lane] = s4;
            }
        }
        if (PARK && wave < S) {                     // behind the first batch's loads, ahead of its use
            epi_pre pre;
            epi_prefetch<EPI>(a, min(strip0 + wave, a.nstrips - 1), lane, pre, 0);
            epi_park<EPI>(&pre_s[wave][lane], pre);
        }
        if (first) { use_batch(); b += bstep; }
    }
    for (; b < bend; b += bstep) {
        load_batch(b * U);
        use_batch();
    }
    if (wave == NW - 1) {

        for (int t = nbat * U; t < KT; ++t) {
            const size_t o = (size_t)t * 64;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const uint4 bh = NB == 1 ? operand(t) : B[(size_t)(2 * ct) * arr + o];
                uint4 bl = bh;
                if (NB == 2) bl = B[(size_t)(2 * ct + 1) * arr + o];
#pragma unroll
                for (int si = 0; si < S; ++si) {
                    const uint4 wa = load_once(&A[so[si] + o]);
                    acc[si][ct] = mfma16(wa, bh, acc[si][ct]);
                    if (NB == 2) acc[si][ct] = mfma16(wa, bl, acc[si][ct]);
                }
            }
        }
    }
    }

    // sum the NW K-slices (and the NW shares of the sums of squares) in wave order; wave si runs
    // the epilogue of strip strip0 + si
#pragma unroll
    for (int si = 0; si < S; ++si)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) red[wave][si][ct][lane] = acc[si][ct];
    __syncthreads();
    const bool hslot = HF && wave == S - 1;
    if (wave >= S || (!hslot && strip0 + wave >= a.nstrips)) return;
    const int strip = hslot ? hstrip : strip0 + wave;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        f32x4 sum = red[0][wave][ct][lane];
        for (int w = 1; w < NW; ++w) { const f32x4 p = red[w][wave][ct][lane]; sum[0] += p[0]; sum[1] += p[1]; sum[2] += p[2]; sum[3] += p[3]; }
        epi_pre pre;
        if (PARK) epi_unpark<EPI>(&pre_s[wave][lane], pre);
        else epi_prefetch<EPI>(a, strip, lane, pre, ct);
        if (NORM) {
            auto col = [&](int w) { return NB == 1 ? ssq_s[w][ct][lane & 7] + ssq_s[w][ct][8 + (lane & 7)] : ssq_s[w][ct][lane & 15]; };   // (two halves of a strip: emit_x)
            float tot = col(0);
#pragma unroll
            for (int w = 1; w < NW; ++w) tot += col(w);
            pre.rj = 1.0f / sqrtf(tot * a.inv_d + a.eps);
        }
        if (hslot && (lane >> 5) != hsel) pre.rows = 0;           // features 4 (lane / 16) .. + 3 of the other half: nothing to store
        epi_apply<NB, EPI>(a, strip, lane, sum, pre, ct, hslot ? hsel : -1);
    }
}

// ------------------------------------------------------------------------------------------
// Projections with three or more strips a CU (gate/up, the vocabulary, the QKV projection without shared heads; others cut along K), 9..64 rows (NB = 2: CT column
// tiles of 16 rows, a hi and a lo operand each; which of them: wide_strips), and up to 8 (NB = 1) with more than four and up to seven strips a CU (packed_wide): one workgroup per CU owns S strips and its NW waves split K, so
// that each activation tile enters the CU once, for S strips, and straight into the registers of the one wave
// that uses it: no LDS and no barrier before the final sum over the waves.
// A CU has some 32 KiB of loads in flight (its L1's size: 56 GB/s of HBM latency, 130 GB/s of L2 latency, whatever the waves ask for), so what counts is
// bytes per CU times their latency: S + 2 CT tiles per K-tile here, 8 + 2 CT with the same CU count short of 12 % in k_gemm_tile (224 groups of eight
// for 1792 strips).  Two K-tiles per wave (one used, one on its way) are enough for that; three or four measured the same.
// 8B-shaped gate/up, 235 MB, us: 16 rows 45.6 (two strips a workgroup) -> 37.5, 32 rows 43.8 (k_gemm_tile) -> 41.0, 48 rows 52.2 -> 46.8 (three
// column tiles instead of four; 64 rows 53.2 -> 50.3); 1024-strip vocabulary 26.1 -> 24.0, 34.2 -> 26.5, 39.0 -> 31.1, 39.8 -> 37.8.
// Output and down projections of up to half as many groups of four strips as CUs are cut along K over blockIdx.y (EPI_PART: the sums go to `part` and k_tile_finish adds them in slice order): cut_slices.
// Their stores are plain ones: half as many sums as k_gemm_tile's, and through to memory (store_through) they were no faster (us a step, plain / through, 17, 32, 48 and 64 rows: four layers of the 8B
// shape 453 / 455, 460 / 461, 518 / 518, 571 / 569; eight layers, 256 strips, K = 4096 571 / 571, 585 / 586, 640 / 645, 715 / 720; 64 strips, K = 8192 443 / 446, 464 / 466, 533 / 533, 593 / 591).
// Loads go through buffer descriptors: a K-tile past the end of the slice gets an offset past the buffer's end,
// for which zeros come back and nothing is fetched, so every load of the loop is unconditional.
// ------------------------------------------------------------------------------------------

constexpr int wide_waves(int ct, int s) { return ct <= 2 || s <= 4 ? 8 : 4; }              // (what the registers of one workgroup per CU hold)
constexpr int wide_lds(int ct, int s) { return wide_waves(ct, s) * s * ct * 1024; }       // dynamic: the waves' sums
constexpr int wide_ssq_lds(int ct, int s) { return wide_waves(ct, s) * ct * 64; }         // static: the waves' shares of the rows' sums of squares
static inline bool wide_fits(int ktiles) { return ktiles <= (1 << 16); }                   // the largest buffer: 8 arrays of K-tiles of 1 KiB = 0.5 GiB

template <int NB, int CT, int S, int EPI>
__global__ void __launch_bounds__(wide_waves(CT, S) * 64) __attribute__((amdgpu_waves_per_eu(wide_waves(CT, S) / 4, wide_waves(CT, S) / 4)))
k_gemm_wide(const gemm_args a, int tps, float4 *part)
{
    static_assert(NB == 2 || CT == 1, "packed rows come in one tile");
    constexpr bool CUT = (EPI == EPI_PART);                     // blockIdx.y: a slice of tps K-tiles, its sums go to `part`
    constexpr int NW = wide_waves(CT, S), NX = NB == 1 ? 1 : 2 * CT;
    constexpr bool NORM = (EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_LMHEAD);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int KT = a.ktiles, t0 = CUT ? blockIdx.y * tps : 0, t1 = CUT ? min(KT, t0 + tps) : KT;
    const int nst = (t1 - t0 + NW - 1) / NW;                    // K-tiles of a wave: wave, wave + NW, ... (some waves' last one is past the end)
    const int rot = (int)((blockIdx.x * 5u + (CUT ? blockIdx.y * 3u : 0u)) % (unsigned)nst);   // workgroups start at different ones, or all would stream from addresses a power of two apart
    const int strip0 = blockIdx.x * S;
    extern __shared__ f32x4 wide_red[];                         // [NW][S * CT][64]
    __shared__ float ssq_s[NW][CT][16];
    static_assert(sizeof(ssq_s) == wide_ssq_lds(CT, S), "the launches count it");

    ssq_loads<CT == 4 ? 4 : 32 / NW> sl[CT];
    if (NORM) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) ssq_issue(a.ssq + (size_t)ct * a.ssq_parts * 16, a.ssq_parts, threadIdx.x, NW * 64, sl[ct]);
    }
    const uint32_t tb = (uint32_t)KT * 1024;                    // bytes of a strip, and of an operand array
    const int mine = min(S, a.nstrips - strip0);                // (strips past the end re-read the last one; dropped below)
    const __amdgpu_buffer_rsrc_t W = buffer_of((const char *)a.W + (size_t)strip0 * tb, (uint32_t)mine * tb);
    const uint32_t xs = NB == 1 ? 128u * (uint32_t)a.rows : 1024u, xl = (NB == 1 ? packed_lane(lane, a.rows) : lane) * 16;   // as in k_gemm
    const __amdgpu_buffer_rsrc_t X = buffer_of(a.xop, NX * (uint32_t)KT * xs);
    uint32_t wo[S];
#pragma unroll
    for (int si = 0; si < S; ++si) wo[si] = (uint32_t)min(si, mine - 1) * tb;

    // 17 rows and more: an accumulator takes 8 K-tiles, then it is added to the total (the reason and its figures: k_gemm_tile).  Up to 16
    // rows the waves' accumulators are as long as in k_gemm
    constexpr bool TWO = CT >= 2;
    f32x4 acc[S][CT], tot[S][CT];
#pragma unroll
    for (int si = 0; si < S; ++si)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[si][ct] = tot[si][ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
    struct stage { uint4 w[S], x[NX]; };
    auto issue = [&](stage &q, int i) {
        const int k = i + rot, t = t0 + (k < nst ? k : k - nst) * NW + wave;
        const bool in = i < nst && t < t1;
        const uint32_t off = lane * 16 + (in ? (uint32_t)t * 1024 : BUFFER_END), offx = xl + (in ? (uint32_t)t * xs : BUFFER_END);
#pragma unroll
        for (int si = 0; si < S; ++si) q.w[si] = buffer_load16<LOAD_ONCE>(W, off, wo[si]);
#pragma unroll
        for (int r = 0; r < NX; ++r) q.x[r] = buffer_load16<0>(X, offx, r * tb);
        asm volatile("" ::: "memory");
    };
    auto use = [&](const stage &q) {
#pragma unroll
        for (int r = 0; r < NX; ++r)
#pragma unroll
            for (int si = 0; si < S; ++si) acc[si][r >> 1] = mfma16(q.w[si], q.x[r], acc[si][r >> 1]);
    };
    stage q0, q1;
    issue(q0, 0);
    issue(q1, 1);
    if (NORM) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const float4 s4 = ssq_finish(a.ssq + (size_t)ct * a.ssq_parts * 16, a.ssq_parts, threadIdx.x, NW * 64, sl[ct]);
            if (lane < 4) *(float4 *)&ssq_s[wave][ct][4 * lane] = s4;
        }
    }
    for (int i = 0; i < nst;) {
        const int e = min(i + 8, nst);
        for (; i < e; i += 2) {
            use(q0); issue(q0, i + 2);
            if (i + 1 < e) use(q1);
            issue(q1, i + 3);
        }
        if (TWO) {
#pragma unroll
            for (int si = 0; si < S; ++si)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) { tot[si][ct] += acc[si][ct]; acc[si][ct] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
        }
    }
#pragma unroll
    for (int si = 0; si < S; ++si)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) wide_red[(wave * S * CT + si * CT + ct) * 64 + lane] = TWO ? tot[si][ct] : acc[si][ct];
    __syncthreads();
    for (int u = wave; u < mine * CT; u += NW) {                // the waves' sums in wave order; a wave finishes every NW-th (strip, column tile)
        const int si = u / CT, ct = u - si * CT;
        f32x4 v = wide_red[u * 64 + lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += wide_red[(w * S * CT + u) * 64 + lane];
        if constexpr (CUT) {
            const size_t at = ((size_t)blockIdx.y * a.nstrips + strip0 + si) * CT + ct;
            if (NB == 1) {                                      // hi and lo columns together: half a KiB a strip
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = with_rotated<8>(v[r], op_add);
                if (!(lane & 8)) part[at * 32 + (lane >> 4) * 8 + (lane & 7)] = make_float4(v[0], v[1], v[2], v[3]);
            } else part[at * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
        } else {
        epi_pre pre;
        epi_prefetch<EPI>(a, strip0 + si, lane, pre, ct);
        if (NORM) {
            auto col = [&](int w) { return NB == 1 ? ssq_s[w][ct][lane & 7] + ssq_s[w][ct][8 + (lane & 7)] : ssq_s[w][ct][lane & 15]; };   // (two halves of a strip: emit_x)
            float s = col(0);
#pragma unroll
            for (int w = 1; w < NW; ++w) s += col(w);
            pre.rj = 1.0f / sqrtf(s * a.inv_d + a.eps);
        }
        epi_apply<NB, EPI>(a, strip0 + si, lane, v, pre, ct);
        }
    }
}

// ------------------------------------------------------------------------------------------
// 4-bit weights, up to 16 rows: a workgroup owns S strips and reads the operand once for them; its NW waves split the batches of a strip (4 K-tiles of
// codes and bf16 group scales, one scale per output feature and K-tile).  A code c enters the matrix core as the bf16 number
// 16 + c (the nibble OR-ed into the top mantissa bits of 16.0 = 0x4180: exact).  Per K-tile the accumulator is started by the product of
// the activation tile with an all -24 operand (= -24 x row sums, shared by the S strips), so that the codes' product on top of it is
// sum_k (c_k - 8) * x_k; the vector ALU only multiplies that by the tile's scale and adds.  The product is taken transposed (activation rows x
// features) so that a lane's four results share one feature, hence one scale; the accumulators are turned back on their way through LDS.
// A wave goes through a batch in two halves, two K-tiles of every strip each, and loads every piece for its next batch as soon as it is dead: two K-tiles of the operand and the scales
// behind the first half, a strip's codes behind its last tile, the other two K-tiles at the end.  So there are loads in flight while it multiplies; with a batch loaded, used up and loaded again
// they drained once a batch (70B-shaped gate/up, 264 MB, 8 rows, inside the kernel 50.0 -> 43.1 us; without the products and the operand 37.0, 7.1 TB/s; 8B shape, 13 rows, 17.4 -> 14.7).
// The scales of up to eight strips come in one load and go through LDS to the lanes of their features: as a load a strip (8 bytes of 16 lanes) they took 6 of the 50 us.
// A product is scaled and added while the next one runs.  128 registers hold seven strips, two workgroups of eight waves a CU, as 16-row tiles too (all 128 of them).  Where the strips take
// several rounds that is what covers a workgroup's start and end: 13 rows, 2560 strips, K = 4096, four layers, one workgroup a CU / two 293 / 285 us a step, 3584 strips 320 / 312, 70B shape, two layers 308 / 301; one
// round (1376 and 1792 strips) 217 / 216 and 233 / 233.  The multiply-adds are pinned behind their products: left alone, the compiler moves all of them to the end
// of the batch and holds every product.
// One or two strips (the 70B-shaped output projection, 12.0 us, 4.5 of which a kernel takes in any case): the L2 -> CU path, 262 KB of operand beside 147 KB of codes per CU at 54 GB/s.  Where that
// is much more operand than codes, K-slices (q4_slices).
// Against k_gemm_tile_q4 and the sum of its K-slices, 13 rows, us, before the loads went out early: 8B shape QKV 15.0 -> 9.1, O 11.2 -> 7.2, gate/up 24.6 -> 18.9; 70B shape 23.1 -> 17.5, 18.4 -> 14.4, 65.5 -> 56.4.
// ------------------------------------------------------------------------------------------
template <int NB, int S, int EPI, int NW = 8>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_gemm_q4(const gemm_args a, int bps, float4 *part)
{
    static_assert(S <= NW, "one epilogue wave per strip");
    constexpr bool NORM = (EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_LMHEAD);
    constexpr bool EARLY = S <= 4;                              // the epilogue's inputs are fetched beside the first batch (more strips: no registers for them)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    constexpr bool CUT = EPI == EPI_RESID;                      // (may be cut along K: blockIdx.y; the sums then go to part, for k_tile_finish)
    const int KT = a.ktiles, nb4 = KT >> 2, b0 = CUT ? (int)blockIdx.y * bps : 0, b1 = CUT ? min(nb4, b0 + bps) : nb4;      // this slice's batches (not none: the launch sees to it)
    const int nst = (b1 - b0 + NW - 1) / NW;                    // batches of a wave: wave, wave + NW, ... (some waves' last one is past the end)
    const int rot = (int)((blockIdx.x * 5u) % (unsigned)nst);   // workgroups start at different ones, or all would stream from addresses a power of two apart
    const int strip0 = blockIdx.x * S, mine = min(S, a.nstrips - strip0);   // (strips past the end re-read the last one; dropped below)
    __shared__ f32x4 red[NW][S][64];
    __shared__ float ssq_s[NW][16];

    ssq_loads<32 / NW> sl;                                      // d up to 8192 without a serial tail of loads
    if (NORM) ssq_issue(a.ssq, a.ssq_parts, threadIdx.x, NW * 64, sl);
    const uint32_t qs = (uint32_t)nb4 * PV_Q4_BATCH;            // bytes of a strip
    const uint32_t xs = NB == 1 ? 128u * (uint32_t)a.rows : 1024u, xl = (NB == 1 ? packed_lane(lane, a.rows) : lane) * 16;   // as in k_gemm
    const __amdgpu_buffer_rsrc_t W = buffer_of((const char *)a.W + (size_t)strip0 * qs, (uint32_t)mine * qs), X = buffer_of(a.xop, NB * (uint32_t)KT * xs);
    f32x4 acc[S];
#pragma unroll
    for (int si = 0; si < S; ++si) acc[si] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // The wave's batch: codes and scales of its strips, the operand's four K-tiles.  Each piece is loaded again for the next batch as soon as it is dead.
    uint4 c[S], h[4], l[NB == 2 ? 4 : 1], sv;
    uint4 *scs = (uint4 *)red[wave][0];                         // the wave's scales of the batch in use: [strip][feature][K-tile], in its own piece of the sums' place
    struct place { uint32_t off, offx, offs; };
    const uint32_t sl8 = (uint32_t)min(lane >> 3, mine - 1) * qs + 1024 + (lane & 7) * 16;
    auto place_of = [&](int i) {
        const int k = i + rot, t = b0 + (k < nst ? k : k - nst) * NW + wave;
        const bool in = t < b1;                                 // (past the end: codes, scales and activations of zero, nothing fetched)
        return place{in ? (uint32_t)t * PV_Q4_BATCH : BUFFER_END, xl + (in ? (uint32_t)t * 4 * xs : BUFFER_END), in ? (uint32_t)t * PV_Q4_BATCH + sl8 : BUFFER_END};
    };
    auto load_strip = [&](place p, int si) {
        c[si] = buffer_load16<LOAD_ONCE>(W, p.off + lane * 16, (uint32_t)min(si, mine - 1) * qs);
        asm volatile("" ::: "memory");
    };
    auto load_scales = [&](place p) { sv = buffer_load16<LOAD_ONCE>(W, p.offs, 0); asm volatile("" ::: "memory"); };       // of up to eight strips at once
    auto load_x = [&](place p, int half) {
#pragma unroll
        for (int u = 2 * half; u < 2 * half + 2; ++u) {
            h[u] = buffer_load16<0>(X, p.offx, u * xs);
            if (NB == 2) l[NB == 2 ? u : 0] = buffer_load16<0>(X, p.offx, (uint32_t)(KT + u) * xs);
        }
        asm volatile("" ::: "memory");
    };
    const uint4 neg24 = make_uint4(0xC1C0C1C0u, 0xC1C0C1C0u, 0xC1C0C1C0u, 0xC1C0C1C0u);
    uint32_t sixteen = 0x41804180u, nibble = 0x00780078u;       // (kept in registers, so that mask-and-merge is one instruction)
    asm volatile("" : "+v"(sixteen), "+s"(nibble));
    // Half a batch: two K-tiles of every strip.  A product is scaled and added one product later, when it is there.
    auto use_half = [&](auto hc, auto more, place next) {
        constexpr int half = decltype(hc)::value;
        f32x4 T0[2], T, P;
        float sp = 0.f;
        const uint32_t *sr = (const uint32_t *)scs + (lane & 15) * 2 + half;
        uint32_t sw = sr[0], sn = S > 1 ? sr[32] : 0;           // (one strip ahead)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int u = 2 * half + v;
            T0[v] = mfma16(h[u], neg24, (f32x4){0.f, 0.f, 0.f, 0.f});
            if (NB == 2) T0[v] = mfma16(l[NB == 2 ? u : 0], neg24, T0[v]);
        }
#pragma unroll
        for (int j = 0; j <= 2 * S; ++j) {
            const int si = j >> 1, u = 2 * half + (j & 1);
            float s1 = 0.f;
            if (j < 2 * S) {
                const uint32_t cw = half == 0 ? ((j & 1) ? c[si].y : c[si].x) : ((j & 1) ? c[si].w : c[si].z);
                s1 = __uint_as_float((j & 1) ? (sw & 0xFFFF0000u) : (sw << 16));
                // operand dword t = bf16 pair (16 + c_2t, 16 + c_2t+1): nibble t of each half into the top mantissa bits of 16.0
                const uint4 wa = make_uint4(((cw << 3) & nibble) | sixteen, ((cw >> 1) & nibble) | sixteen, ((cw >> 5) & nibble) | sixteen, ((cw >> 9) & nibble) | sixteen);
                T = mfma16(h[u], wa, T0[j & 1]);
                if (NB == 2) T = mfma16(l[NB == 2 ? u : 0], wa, T);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (j > 0) {
                const int sj = (j - 1) >> 1;
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[sj][r] = fmaf(sp, P[r], acc[sj][r]);
                asm volatile("" : "+v"(acc[sj]));               // the multiply-adds stay here
            }
            P = T; sp = s1;
            if ((j & 1) && j < 2 * S) { sw = sn; if (si + 2 < S) sn = sr[(si + 2) * 32]; }
            if (half == 1 && decltype(more)::value && (j & 1) && j < 2 * S) load_strip(next, si);
        }
    };
    auto use = [&](auto more, place next) {
        scs[lane] = sv;                                   // (a wave's LDS traffic stays in order: no barrier)
        use_half(std::integral_constant<int, 0>(), more, next);
        if (decltype(more)::value) { load_x(next, 0); load_scales(next); }
        use_half(std::integral_constant<int, 1>(), more, next);
        if (decltype(more)::value) load_x(next, 1);
    };
    const place first = place_of(0);
    load_x(first, 0);
    load_scales(first);
#pragma unroll
    for (int si = 0; si < S; ++si) load_strip(first, si);
    load_x(first, 1);
    epi_pre pre;
    if (EARLY && wave < mine) epi_prefetch<EPI>(a, strip0 + wave, lane, pre, 0);
    if (NORM) {
        const float4 s4 = ssq_finish(a.ssq, a.ssq_parts, threadIdx.x, NW * 64, sl);
        if (lane < 4) *(float4 *)&ssq_s[wave][4 * lane] = s4;
    }
    for (int i = 1; i < nst; ++i) use(std::true_type(), place_of(i));
    use(std::false_type(), first);
    {   // acc is (row 4 g + r, feature f) for lane (g, f); the sum below and the epilogues take (feature 4 g' + r', row j) from lane (g', j): store transposed
        const int g = lane >> 4, f = lane & 15;
#pragma unroll
        for (int si = 0; si < S; ++si)
#pragma unroll
            for (int r = 0; r < 4; ++r) ((float *)red[wave][si])[((f >> 2) * 16 + 4 * g + r) * 4 + (f & 3)] = acc[si][r];
    }
    __syncthreads();
    if (wave >= mine) return;
    f32x4 v = red[0][wave][lane];                               // the waves' sums in wave order
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w][wave][lane];
    if (CUT && part != nullptr) {
        const size_t at = (size_t)blockIdx.y * a.nstrips + strip0 + wave;
        if (NB == 1) {                                          // hi and lo columns together: half a KiB a strip
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = with_rotated<8>(v[r], op_add);
            if (!(lane & 8)) part[at * 32 + (lane >> 4) * 8 + (lane & 7)] = make_float4(v[0], v[1], v[2], v[3]);
        } else part[at * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
        return;
    }
    if (!EARLY) epi_prefetch<EPI>(a, strip0 + wave, lane, pre, 0);
    if (NORM) {
        auto col = [&](int w) { return NB == 1 ? ssq_s[w][lane & 7] + ssq_s[w][8 + (lane & 7)] : ssq_s[w][lane & 15]; };   // (two halves of a strip: emit_x)
        float t = col(0);
#pragma unroll
        for (int w = 1; w < NW; ++w) t += col(w);
        pre.rj = 1.0f / sqrtf(t * a.inv_d + a.eps);
    }
    epi_apply<NB, EPI>(a, strip0 + wave, lane, v, pre, 0);
}

// ------------------------------------------------------------------------------------------
// Blocks of 17..64 rows (CT = 2, 3 or 4 column tiles of 16 rows, a hi and a lo operand each): 2 CT
// activation tiles go with every weight tile.  Fetched per wave they outgrow the weight stream
// in the CU's load path, so here the 8 waves of a workgroup walk the same K range in step, each
// with its own S strips, and every activation tile is fetched once per workgroup and shared
// through LDS (two buffers, one barrier per step of U K-tiles).  Weights and activation tiles
// are loaded D steps ahead into registers; the activation tiles pass through LDS on use.
// A GEMM with few strips is cut along K as well (blockIdx.y): the slices' partial sums go to
// `part` and k_tile_finish adds them in slice order and runs the epilogue; with one slice the
// epilogue runs here.  Workgroups start their K walk at different steps so that they do not
// all stream from addresses a power of two apart.
// ------------------------------------------------------------------------------------------
template <int CT, int S, int EPI>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
k_gemm_tile(const gemm_args a, int tps, float4 *part)
{
    constexpr int NW = 8, U = 2, D = 4, TPS = U * CT * 2;                    // TPS activation tiles per step: wave w brings in tiles w and w + 8, where there are as many
    static_assert(TPS >= NW && TPS <= 2 * NW, "a wave loads one or two tiles of the step");
    constexpr bool NORM = (EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_LMHEAD);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int KT = a.ktiles, t0 = blockIdx.y * tps, t1 = min(KT, t0 + tps);  // this slice's K-tiles (not empty: the launch sees to it)
    const int nsteps = (t1 - t0 + U - 1) / U;
    const int rot = (int)((blockIdx.x * 5u + blockIdx.y * 3u) % (unsigned)nsteps);
    const size_t arr = (size_t)KT * 64;
    const int sw = (blockIdx.x * NW + wave) * S;                              // the wave's first strip
    size_t so[S];                                                             // strips past the end re-read the last one; dropped below
#pragma unroll
    for (int si = 0; si < S; ++si) so[si] = (size_t)min(sw + si, a.nstrips - 1) * arr;
    const uint4 *A = a.W + lane, *B = a.xop + lane;
    __shared__ uint4 sa[2][TPS][64];
    __shared__ float ssq_s[NW][CT][16];

    ssq_loads<2> sl[CT];
    if (NORM && part == nullptr) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) ssq_issue(a.ssq + (size_t)ct * a.ssq_parts * 16, a.ssq_parts, threadIdx.x, NW * 64, sl[ct]);
    }
    f32x4 acc[S][CT], tot[S][CT];
#pragma unroll
    for (int si = 0; si < S; ++si)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[si][ct] = tot[si][ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // An accumulator takes 8 K-tiles, then it is added to the total: over a whole slice of up to 448 it would carry a rounding error
    // of the size of the operands' own.  Keys and values of a first layer that are not the rounded 64-bit result, runs of 16 / runs of 8: K =
    // 3072 2.39 / 1.85e-4 (slices of 14 tiles without runs: 2.23e-4), K = 4096 2.22 / 1.83e-4; 48 nodes or 4 x 8 rows, 8B shape: no slower.
    auto add_up = [&]() {
#pragma unroll
        for (int si = 0; si < S; ++si)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) { tot[si][ct] += acc[si][ct]; acc[si][ct] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
    };

    struct slot { uint4 x0, x1, w[S][U]; };           // one step in flight: the wave's one or two activation tiles, its weight tiles
    auto first_tile = [&](int step) { int k = step + rot; if (k >= nsteps) k -= nsteps; return t0 + k * U; };
    auto issue = [&](slot &q, int step) {             // loads of (rotated) step `step`; a tile past the slice's end re-reads its last one
        const int tb = first_tile(step);
        auto tile = [&](int t) { return B[(size_t)(t % (CT * 2)) * arr + (size_t)min(tb + t / (CT * 2), t1 - 1) * 64]; };   // K-tile t / (2 CT) of the step, operand array t % (2 CT)
        q.x0 = tile(wave);
        if (TPS > NW) q.x1 = tile(min(wave + NW, TPS - 1));     // (CT = 3: 12 tiles, the last four waves read the last one again)
#pragma unroll
        for (int si = 0; si < S; ++si)
#pragma unroll
            for (int u = 0; u < U; ++u) q.w[si][u] = load_once(&A[so[si] + (size_t)min(tb + u, t1 - 1) * 64]);
        asm volatile("" ::: "memory");
    };
    auto use = [&](const slot &q, int buf, int step) {   // q holds step `step`: share its activation tiles through sa[buf], multiply
        sa[buf][wave][lane] = make_uint4(q.x0.x, q.x0.y, q.x0.z, q.x0.w);
        if (TPS > NW && wave + NW < TPS) sa[buf][wave + NW][lane] = make_uint4(q.x1.x, q.x1.y, q.x1.z, q.x1.w);
        __syncthreads();
        const int tb = first_tile(step);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (tb + u < t1) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const uint4 hi = sa[buf][u * CT * 2 + 2 * ct][lane], lo = sa[buf][u * CT * 2 + 2 * ct + 1][lane];
#pragma unroll
                    for (int si = 0; si < S; ++si) {
                        acc[si][ct] = mfma16(q.w[si][u], hi, acc[si][ct]);
                        acc[si][ct] = mfma16(q.w[si][u], lo, acc[si][ct]);
                    }
                }
            }
        }
    };
    static_assert(D == 4, "slots are spelled out");
    slot q0, q1, q2, q3;
    issue(q0, 0);
    issue(q1, min(1, nsteps - 1));
    issue(q2, min(2, nsteps - 1));
    issue(q3, min(3, nsteps - 1));
    if (NORM && part == nullptr) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const float4 s4 = ssq_finish(a.ssq + (size_t)ct * a.ssq_parts * 16, a.ssq_parts, threadIdx.x, NW * 64, sl[ct]);
            if (lane < 4) *(float4 *)&ssq_s[wave][ct][4 * lane] = s4;
        }
    }
    int s0 = 0;
    for (; s0 + D <= nsteps; s0 += D) {               // every wave of the workgroup takes the same steps: the barriers match
        use(q0, 0, s0);     issue(q0, min(s0 + 4, nsteps - 1));
        use(q1, 1, s0 + 1); issue(q1, min(s0 + 5, nsteps - 1));
        use(q2, 0, s0 + 2); issue(q2, min(s0 + 6, nsteps - 1));
        use(q3, 1, s0 + 3); issue(q3, min(s0 + 7, nsteps - 1));
        add_up();
    }
    if (s0 < nsteps) use(q0, 0, s0);
    if (s0 + 1 < nsteps) use(q1, 1, s0 + 1);
    if (s0 + 2 < nsteps) use(q2, 0, s0 + 2);
    add_up();

    if (part != nullptr) {
#pragma unroll
        for (int si = 0; si < S; ++si)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                if (sw + si < a.nstrips) store_through(&part[(((size_t)blockIdx.y * a.nstrips + sw + si) * CT + ct) * 64 + lane], tot[si][ct]);
        return;
    }
    __syncthreads();                                  // (ssq_s of every wave; also covers a slice of a single step)
#pragma unroll
    for (int si = 0; si < S; ++si) {
        const int strip = sw + si;
        if (strip >= a.nstrips) continue;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            epi_pre pre;
            epi_prefetch<EPI>(a, strip, lane, pre, ct);
            if (NORM) {
                float tot = ssq_s[0][ct][lane & 15];
#pragma unroll
                for (int w = 1; w < NW; ++w) tot += ssq_s[w][ct][lane & 15];
                pre.rj = 1.0f / sqrtf(tot * a.inv_d + a.eps);
            }
            epi_apply<2, EPI>(a, strip, lane, tot[si][ct], pre, ct);
        }
    }
}

// ------------------------------------------------------------------------------------------
// The same for 4-bit weights (17..64 rows, and 9..16 where k_gemm_q4 is not faster; CT = 1, 2 or 4): the 8 waves of a workgroup own two strips each and walk
// the strips' batches (4 K-tiles of codes + scales, 1152 bytes) in step; the 8 CT activation tiles of
// a step are fetched once per workgroup and shared through LDS (two buffers, one barrier per step).
// Per weight byte a 4-bit strip needs 3.6 times the activation bytes of a 16-bit one, on the L2 -> CU
// path as well as out of LDS: hence two strips per wave.  A step is long (72 MFMAs at 64 rows), so the
// weights are loaded two steps ahead and the activation tiles one (their registers are free once they sit in LDS).
// Arithmetic as in k_gemm_q4: a code c enters as the bf16 number 16 + c, the product is taken
// transposed (activation rows x features) on top of -24 x (row sums), scaled per K-tile; the row sums
// are the same for every strip and are taken once per workgroup by the wave that brings the tile in.
// The accumulators are turned back through LDS before the epilogue (or before they are stored as a
// K-slice's partial sums for k_tile_finish).
// ------------------------------------------------------------------------------------------
template <int CT, int EPI>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(CT <= 2 ? 4 : 2)))
k_gemm_tile_q4(const gemm_args a, int bps, float4 *part)
{
    constexpr int NW = 8, S = 2, U = 4, P = U * CT, TPS = P * 2;            // P (K-tile, column tile) pairs = TPS activation tiles per step
    static_assert(CT == 1 || CT == 2 || CT == 4, "a wave brings in pair `wave` (if there is one) and, with 16 pairs, pair `wave + 8`");
    constexpr bool NORM = (EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_LMHEAD);
    extern __shared__ uint4 tile_lds[];                         // [2][TPS][64]
    uint4 (*sa)[TPS][64] = (uint4 (*)[TPS][64])tile_lds;
    __shared__ float ssq_s[NW][CT][16];
    __shared__ f32x4 rs[2][TPS / 2][4];                         // per (K-tile, column tile) of a step: -24 x its rows' sums, rows 4 g .. 4 g + 3 at [g]
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int NBAT = a.ktiles >> 2;                             // batches of a strip
    const int b0 = blockIdx.y * bps, b1 = min(NBAT, b0 + bps), nsteps = b1 - b0;   // this slice (not empty: the launch sees to it)
    const int rot = (int)((blockIdx.x * 5u + blockIdx.y * 3u) % (unsigned)nsteps);
    const size_t arr = (size_t)a.ktiles * 64;
    const int sw = (blockIdx.x * NW + wave) * S;                // the wave's first strip; strips past the end: the last one again, dropped below
    const char *Aq0 = (const char *)a.W + (size_t)min(sw, a.nstrips - 1) * (size_t)NBAT * PV_Q4_BATCH;
    const char *Aq1 = (const char *)a.W + (size_t)min(sw + 1, a.nstrips - 1) * (size_t)NBAT * PV_Q4_BATCH;
    const uint4 *B = a.xop + lane;

    ssq_loads<2> sl[CT];
    if (NORM && part == nullptr) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) ssq_issue(a.ssq + (size_t)ct * a.ssq_parts * 16, a.ssq_parts, threadIdx.x, NW * 64, sl[ct]);
    }
    f32x4 acc0[CT], acc1[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc0[ct] = acc1[ct] = (f32x4){0.f, 0.f, 0.f, 0.f};

    struct wslot { uint4 c0, c1; uint2 s0, s1; };               // a batch of either strip
    struct xslot { uint4 a, b, c, d; };                         // (named members: an array here ends up in scratch memory)
    const bool loads = wave < P;                                // (CT = 1: four pairs a step, the other four waves bring in none)
    auto batch_of = [&](int step) { int k = min(step, nsteps - 1) + rot; if (k >= nsteps) k -= nsteps; return b0 + k; };   // (a step past the end re-reads the last one)
    auto issue_w = [&](wslot &q, int step) {
        const size_t o = (size_t)batch_of(step) * PV_Q4_BATCH;
        q.c0 = load_once((const uint4 *)(Aq0 + o + lane * 16));
        q.c1 = load_once((const uint4 *)(Aq1 + o + lane * 16));
        q.s0 = load_once((const uint2 *)(Aq0 + o + 1024 + (lane & 15) * 8));
        q.s1 = load_once((const uint2 *)(Aq1 + o + 1024 + (lane & 15) * 8));
        asm volatile("" ::: "memory");
    };
    auto issue_x = [&](xslot &q, int step) {                    // pair p = wave (+ 8) of the step: K-tile p / CT of the batch, column tile p % CT, hi and lo
        const int bt = batch_of(step);
        auto tile = [&](int p, int half) { const int u = p / CT, ct = p % CT; return B[(size_t)(2 * ct + half) * arr + (size_t)(bt * 4 + u) * 64]; };
        if (loads) { q.a = tile(wave, 0); q.b = tile(wave, 1); }
        if (P > NW) { q.c = tile(wave + NW, 0); q.d = tile(wave + NW, 1); }
        asm volatile("" ::: "memory");
    };
    const uint4 neg24 = make_uint4(0xC1C0C1C0u, 0xC1C0C1C0u, 0xC1C0C1C0u, 0xC1C0C1C0u);
    auto stage = [&](const xslot &x, int buf) {                 // the wave's tiles of the step into LDS, with -24 x the row sums of each hi + lo pair
        const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
        if (loads) {
            sa[buf][2 * wave][lane] = x.a; sa[buf][2 * wave + 1][lane] = x.b;
            const f32x4 ra = mfma16(x.b, neg24, mfma16(x.a, neg24, zero4));
            if ((lane & 15) == 0) rs[buf][wave][lane >> 4] = ra;
        }
        if (P > NW) {
            sa[buf][2 * (wave + NW)][lane] = x.c; sa[buf][2 * (wave + NW) + 1][lane] = x.d;
            const f32x4 rc = mfma16(x.d, neg24, mfma16(x.c, neg24, zero4));
            if ((lane & 15) == 0) rs[buf][wave + NW][lane >> 4] = rc;
        }
    };
    uint32_t sixteen = 0x41804180u;                             // (in a vector register, so that mask-and-merge is one instruction)
    asm volatile("" : "+v"(sixteen));
    auto codes = [&](uint32_t cw) {                             // 8 codes of a dword as the bf16 numbers 16 + c, in operand order
        auto pick = [&](uint32_t v) { uint32_t r; asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "s"(0x00780078u), "v"(sixteen)); return r; };
        return make_uint4(pick(cw << 3), pick(cw >> 1), pick(cw >> 5), pick(cw >> 9));
    };
    auto scale = [](uint2 s2, int u) { const uint32_t w = (u & 2) ? s2.y : s2.x; return __uint_as_float((u & 1) ? (w & 0xFFFF0000u) : (w << 16)); };
    // One (K-tile, column tile) pair after the other, software-pipelined by hand: the LDS reads of the next pair go out,
    // then the four MFMAs of this pair, then the scaling of the previous pair's products (whose MFMAs are done by then);
    // the scheduling fences keep that order, which the compiler would otherwise serialise (read, wait, multiply, wait, scale).
    auto compute = [&](const wslot &w, int buf) {
        uint4 hiN = sa[buf][0][lane], loN = sa[buf][1][lane], wa0, wa1;
        f32x4 t0N = rs[buf][0][lane >> 4], pa, pb;
        float sc0 = 0.f, sc1 = 0.f, ps0 = 0.f, ps1 = 0.f;
#pragma unroll
        for (int p = 0; p < U * CT; ++p) {
            const int u = p / CT, ct = p % CT;
            const uint4 hi = hiN, lo = loN;
            const f32x4 T0 = t0N;
            if (ct == 0) {
                wa0 = codes(u == 0 ? w.c0.x : u == 1 ? w.c0.y : u == 2 ? w.c0.z : w.c0.w);
                wa1 = codes(u == 0 ? w.c1.x : u == 1 ? w.c1.y : u == 2 ? w.c1.z : w.c1.w);
                sc0 = scale(w.s0, u); sc1 = scale(w.s1, u);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (p + 1 < U * CT) { hiN = sa[buf][2 * p + 2][lane]; loN = sa[buf][2 * p + 3][lane]; t0N = rs[buf][p + 1][lane >> 4]; }
            __builtin_amdgcn_sched_barrier(0);
            f32x4 Ta = mfma16(hi, wa0, T0), Tb = mfma16(hi, wa1, T0);
            Ta = mfma16(lo, wa0, Ta); Tb = mfma16(lo, wa1, Tb);
            __builtin_amdgcn_sched_barrier(0);
            if (p > 0) {
                const int pc = (p - 1) % CT;
#pragma unroll
                for (int r = 0; r < 4; ++r) { acc0[pc][r] = fmaf(ps0, pa[r], acc0[pc][r]); acc1[pc][r] = fmaf(ps1, pb[r], acc1[pc][r]); }
            }
            pa = Ta; pb = Tb; ps0 = sc0; ps1 = sc1;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) { acc0[CT - 1][r] = fmaf(ps0, pa[r], acc0[CT - 1][r]); acc1[CT - 1][r] = fmaf(ps1, pb[r], acc1[CT - 1][r]); }
    };
    wslot wA, wB;
    xslot x = {};
    issue_w(wA, 0); issue_w(wB, 1);
    if (NORM && part == nullptr) {                              // (their loads went out before the weights': no wait for those; the
#pragma unroll                                                  //  registers are free again before the activation slot fills)
        for (int ct = 0; ct < CT; ++ct) {
            const float4 s4 = ssq_finish(a.ssq + (size_t)ct * a.ssq_parts * 16, a.ssq_parts, threadIdx.x, NW * 64, sl[ct]);
            if (lane < 4) *(float4 *)&ssq_s[wave][ct][4 * lane] = s4;
        }
    }
    issue_x(x, 0);
    // every wave of the workgroup takes the same steps: the barriers match.  Buffer i & 1 is rewritten at step i + 2,
    // behind the barrier of step i + 1, which every wave reaches with its reads of step i done.
#define PV_Q4_STEP(W, I)                                                                     \
    if (s0 + (I) < nsteps) { stage(x, (I) & 1); issue_x(x, s0 + (I) + 1); __syncthreads(); compute(W, (I) & 1); issue_w(W, s0 + (I) + 2); }
    for (int s0 = 0; s0 < nsteps; s0 += 2) { PV_Q4_STEP(wA, 0) PV_Q4_STEP(wB, 1) }
#undef PV_Q4_STEP
    __syncthreads();                                            // the last step's tiles have been read; ssq_s of every wave
    // an accumulator is (row 4 g + r, feature f) for lane (g, f); the epilogues take (feature 4 g' + r', row j) from
    // lane (g', j): turned through the wave's own KiB of the tile buffer
    float *rf = (float *)&sa[0][wave][0];
    const int g = lane >> 4, f = lane & 15;
    auto turn = [&](f32x4 &v) {
#pragma unroll
        for (int r = 0; r < 4; ++r) rf[((f >> 2) * 16 + 4 * g + r) * 4 + (f & 3)] = v[r];
        const f32x4 t = ((const f32x4 *)rf)[lane];              // (a wave's LDS traffic stays in order: no barrier inside the wave)
        v = t;
    };
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) { turn(acc0[ct]); turn(acc1[ct]); }
#pragma unroll
    for (int si = 0; si < S; ++si) {
        const int strip = sw + si;
        if (strip >= a.nstrips) continue;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const f32x4 v = si == 0 ? acc0[ct] : acc1[ct];
            if (part != nullptr) {
                store_through(&part[(((size_t)blockIdx.y * a.nstrips + strip) * CT + ct) * 64 + lane], v);
                continue;
            }
            epi_pre pre;
            epi_prefetch<EPI>(a, strip, lane, pre, ct);
            if (NORM) {
                float tot = ssq_s[0][ct][lane & 15];
#pragma unroll
                for (int w = 1; w < NW; ++w) tot += ssq_s[w][ct][lane & 15];
                pre.rj = 1.0f / sqrtf(tot * a.inv_d + a.eps);
            }
            epi_apply<2, EPI>(a, strip, lane, v, pre, ct);
        }
    }
}

// Adds the K-slices' partial sums of k_gemm_tile in slice order and runs the epilogue: one wave
// per (strip, column tile), the four waves of a workgroup take four strips of column tile
// blockIdx.y.  At most TILE_MAX_SLICES slices: their loads go out together.
#define TILE_MAX_SLICES 16
template <int CT, int EPI, int NB = 2>
__global__ void __launch_bounds__(256)
k_tile_finish(const gemm_args a, const float4 *part, int slices)
{
    constexpr int NW = 4;
    constexpr bool NORM = (EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_LMHEAD);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, ct = blockIdx.y;
    const int strip = min((int)blockIdx.x * NW + wave, a.nstrips - 1);           // a wave past the end repeats the last strip's loads and stores nothing
    const bool mine = (int)blockIdx.x * NW + wave < a.nstrips;
    __shared__ float ssq_s[NW][16];
    ssq_loads<4> sl;
    if (NORM) ssq_issue(a.ssq + (size_t)ct * a.ssq_parts * 16, a.ssq_parts, threadIdx.x, NW * 64, sl);
    float4 p[TILE_MAX_SLICES];
    // (packed rows: hi and lo columns have been added up, 32 lanes a strip)
    const float4 *q = NB == 1 ? part + (size_t)strip * 32 + (lane >> 4) * 8 + (lane & 7) : part + ((size_t)strip * CT + ct) * 64 + lane;
    const size_t step = (size_t)a.nstrips * (NB == 1 ? 32 : CT * 64);
    auto fetch = [&](int y0, int y1) {
#pragma unroll
        for (int y = 0; y < TILE_MAX_SLICES; ++y) if (y >= y0 && y < y1) p[y] = q[(size_t)(y < slices ? y : 0) * step];
    };
    fetch(0, 4);
    if (slices > 4) fetch(4, 8);
    if (slices > 8) fetch(8, TILE_MAX_SLICES);
    epi_pre pre;
    epi_prefetch<EPI>(a, strip, lane, pre, ct);
    if (NORM) {
        const float4 s4 = ssq_finish(a.ssq + (size_t)ct * a.ssq_parts * 16, a.ssq_parts, threadIdx.x, NW * 64, sl);
        if (lane < 4) *(float4 *)&ssq_s[wave][4 * lane] = s4;
        __syncthreads();
        float tot = ssq_s[0][lane & 15];
#pragma unroll
        for (int w = 1; w < NW; ++w) tot += ssq_s[w][lane & 15];
        pre.rj = 1.0f / sqrtf(tot * a.inv_d + a.eps);
    }
    float4 v = p[0];
#pragma unroll
    for (int y = 1; y < TILE_MAX_SLICES; ++y)
        if (y < slices) { v.x += p[y].x; v.y += p[y].y; v.z += p[y].z; v.w += p[y].w; }
    if (NB == 1 && (lane & 8)) v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (mine) epi_apply<NB, EPI>(a, strip, lane, (f32x4){v.x, v.y, v.z, v.w}, pre, ct);   // (wave-uniform; no barrier inside)
}

// ------------------------------- host side ----------------------------------------



static constexpr size_t tile_q4_lds(int ct) { return (size_t)2 * 4 * ct * 2 * 64 * sizeof(uint4); }   // two buffers of 8 ct activation tiles

template <int CT, int EPI>
static int allow_tile_q4_lds()
{
    PV_HIP(hipFuncSetAttribute((const void *)k_gemm_tile_q4<CT, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)tile_q4_lds(CT)));
    return PV_OK;
}

// Strips a workgroup of k_gemm_wide, 0: the GEMM goes elsewhere.  Workgroups run in rounds of one per CU; per K-tile a CU takes in S weight tiles and 2 CT
// activation tiles, and one of those costs about 0.3 of a weight tile (L2 against HBM latency).  Strips a workgroup for 1376 strips, 16 / 32 / 48 rows: six (230
// workgroups) 30.8 / 34.4 / 40.8 us, seven (197) 32.3 / 36.3 / 44.2.
// Up to 16 rows the alternative is k_gemm: K = 2048, 1024 strips 14.5 there, 15.8 here; K = 4096 26.1 and 24.0.
// More rows: k_gemm_tile, a workgroup of eight strips on every CU or, up to four strips a CU, two or more that share a CU's strips along K.  What decides is how many
// strips the CU with the most of them goes through, S a round here and 8 a round there (gate/up and vocabulary, us, there / here):
//  - up to four strips a CU the slices leave no CU idle and cost one more kernel: K = 4096, 1024 strips, 32 / 48 / 64 rows 34.6 / 31.3, 37.1 / 36.3, 39.9 / 39.6;
//    K = 5120 37.0 / 34.7, 40.9 / 40.4, 44.9 / 45.7; K = 8192 54.3 / 54.3, 56.6 / 62.2, 61.0 / 69.6.  Below 2 3/4 strips a CU (640 strips, K = 5120) 28.8 / 30.3, 31.5 / 34.7, 34.7 / 38.3;
//  - three quarters of the strips or less: always (K = 4096, 1376 strips 40.8 / 37.2, 47.4 / 43.5, 52.0 / 47.5; 2560 strips 80.7 / 67.8, 87.6 / 82.8, 94.0 / 91.1);
//  - seven eighths: up to 32 rows (K = 4096, 3584 strips 87.2 / 82.0, 5120 strips 125.7 / 119.4), in one round with more rows as well (1792 strips 50.8 / 49.2 and 55.1 / 53.1),
//    in several up to 48 rows from K = 5120 on (3584 strips, K = 4096 96.9 / 99.0, K = 8192 174.7 / 171.0), and with 64 rows in one round up to K = 6656 (K = 8192 97.5 / 99.4);
//  - as many or more: never (K = 4096, 2000 strips 50.9 / 55.0, 52.8 / 66.7, 56.7 / 73.8; 8016 strips 184 / 192, 200 / 229, 212 / 249).
static int wide_strips(const pv_model *m, int strips, int ktiles, int ct)
{
    const int cus = m->n_cus;
    if (!wide_fits(ktiles) || ktiles < (ct == 1 ? 128 : 16) || 4 * strips < 11 * cus) return 0;
    int best = 0, through = 0;
    double least = 1e30;
    for (int S : {7, 6, 4, 3}) {
        const int rounds = ((strips + S - 1) / S + cus - 1) / cus;
        const double t = rounds * (S + 0.6 * ct);
        if (t < least) { least = t; best = S; through = rounds * S; }
    }
    if (ct == 1) return best;
    const int there = ((strips + 7) / 8 + cus - 1) / cus * 8;
    if (strips <= 4 * cus) return ktiles <= 160 ? best : 0;
    if (4 * through <= 3 * there) return best;
    if (8 * through > 7 * there) return 0;
    if (ct == 2 || (ct == 3 && (there == 8 || ktiles >= 160)) || (ct == 4 && there == 8 && ktiles <= 208)) return best;
    return 0;
}

// How evenly workgroups, one per CU a round, fill their rounds
static double even(const pv_model *m, int wgs) { const int rounds = (wgs + m->n_cus - 1) / m->n_cus; return (double)wgs / ((double)rounds * m->n_cus); }

// Packed rows in k_gemm_wide: more than four and up to seven strips a CU, in one round of six or seven each, so that the operand enters a CU once.  us, K = 4096 / 5120 / 8192, one
// strip a workgroup there against here: 1088 strips, one row 25.6 / 31.5 / 48.2 against 24.9 / 29.1 / 45.7, 8 rows 28.6 / 36.0 / 55.6 against 25.5 / 29.8 / 47.0; 1600 strips, 8 rows
// 39.4 / 49.7 / 77.5 against 33.6 / 40.8 / 63.0.  Elsewhere, since whole rounds of smaller workgroups leave nothing to gain by it and these overlap their starts and ends:
//  - up to four strips a CU (1024 strips in four each 24.3 / 27.7 / 44.2, in two each 22.8 / 27.1 / 43.5);
//  - one strip a workgroup in even rounds, up to 4 rows and K = 4608 (K = 4096, 1280 strips 27.4 / 28.5, K = 4608 29.5 / 30.2, but K = 5120 33.0 / 33.1; 1792 strips 36.7 / 37.6);
//  - two in even rounds, up to K = 7168 (one row, K = 5120, 1536 strips 38.5 / 39.9, K = 7168 53.3 / 54.1, but K = 8192, 1440 strips 59.3 / 58.0); how even goes with the operand:
//    K = 4096, 1376 strips, one row 30.0 / 31.2, 8 rows 31.1 / 30.6, 1440 strips 31.5 / 31.4; K = 5120, 1376 strips, one row 35.5 / 35.8, 1440 strips 36.6 / 37.3, 8 rows 38.1 / 36.8,
//    1536 strips, 5 rows 38.5 / 39.8;
//  - half strips in even rounds, from there up to K = 7168 (1792 strips of gate/up, one row and 8: K = 4096 38.8 / 37.6 and 38.4 / 37.5, K = 4608 40.7 / 42.8 and 40.5 / 41.8, K = 5120
//    45.2 / 46.0 and 45.2 / 45.5, K = 7168 61.6 / 63.0 and 61.6 / 62.2, K = 8192 71.1 / 70.5 and 71.0 / 69.8).
static bool one_strip_even(const pv_model *m, int strips, int ktiles, int rows) { return rows <= 4 && ktiles <= 144 && strips <= 7 * m->n_cus && even(m, strips) >= 15. / 16; }
static bool half_strips_even(int strips) { return (2 * strips) % 7 == 0 && (2 * strips / 7) % 256 == 0; }
static bool packed_wide(const pv_model *m, int strips, int ktiles, int rows, bool gate_up)
{
    if (strips <= 4 * m->n_cus || strips > 7 * m->n_cus || one_strip_even(m, strips, ktiles, rows)) return false;
    const double line = ktiles <= 128 ? (rows <= 4 ? 0.88 : 0.935) : (rows <= 4 ? 0.935 : 0.965);
    if (ktiles <= 224 && even(m, (strips + 1) / 2) >= line) return false;
    return !(gate_up && half_strips_even(strips) && ktiles > 128 && ktiles <= 224);
}

template <int NB, int CT, int S, int EPI>
static int allow_wide_lds()
{
    if (wide_lds(CT, S) + wide_ssq_lds(CT, S) > 65536) PV_HIP(hipFuncSetAttribute((const void *)k_gemm_wide<NB, CT, S, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds(CT, S)));
    return PV_OK;
}
template <int NB, int CT, int EPI>
static int allow_wide_all()
{
    int rc;
    if constexpr (NB == 2) if ((rc = allow_wide_lds<NB, CT, 3, EPI>()) != PV_OK || (rc = allow_wide_lds<NB, CT, 4, EPI>()) != PV_OK) return rc;
    if ((rc = allow_wide_lds<NB, CT, 6, EPI>()) != PV_OK) return rc;
    return allow_wide_lds<NB, CT, 7, EPI>();
}

template <int NB, int CT, int EPI, int S>
static int launch_wide_s(const gemm_args &ga, int strips, hipStream_t s)
{
    k_gemm_wide<NB, CT, S, EPI><<<(strips + S - 1) / S, wide_waves(CT, S) * 64, wide_lds(CT, S), s>>>(ga, ga.ktiles, nullptr);
    PV_HIP(hipGetLastError());
    return PV_OK;
}
template <int NB, int CT, int EPI>
static int launch_wide(const gemm_args &ga, int strips, int ws, hipStream_t s)
{
    if constexpr (NB == 2) if (ws <= 4) return ws == 3 ? launch_wide_s<NB, CT, EPI, 3>(ga, strips, s) : launch_wide_s<NB, CT, EPI, 4>(ga, strips, s);      // (packed rows: packed_wide)
    return ws == 6 ? launch_wide_s<NB, CT, EPI, 6>(ga, strips, s) : launch_wide_s<NB, CT, EPI, 7>(ga, strips, s);
}

// once per device before the first launch (and outside any stream capture): kernels that use more dynamic LDS than the default limit
template <int NB, int CT> static int allow_wide() { int rc; if ((rc = allow_wide_all<NB, CT, EPI_QKV>()) != PV_OK || (rc = allow_wide_all<NB, CT, EPI_SWIGLU>()) != PV_OK) return rc; return allow_wide_all<NB, CT, EPI_LMHEAD>(); }
template <int CT> static int allow_tile_q4()
{
    int rc;
    if ((rc = allow_tile_q4_lds<CT, EPI_QKV>()) != PV_OK || (rc = allow_tile_q4_lds<CT, EPI_RESID>()) != PV_OK || (rc = allow_tile_q4_lds<CT, EPI_SWIGLU>()) != PV_OK) return rc;
    return allow_tile_q4_lds<CT, EPI_LMHEAD>();
}
int pv_mat_gemm_init(int wbits)
{
    int rc;
    if (wbits == 4) {
        if ((rc = allow_tile_q4<1>()) != PV_OK || (rc = allow_tile_q4<2>()) != PV_OK) return rc;
        return allow_tile_q4<4>();
    }
    if ((rc = allow_wide_lds<1, 1, 4, EPI_PART>()) != PV_OK || (rc = allow_wide_lds<2, 1, 4, EPI_PART>()) != PV_OK || (rc = allow_wide_lds<2, 2, 4, EPI_PART>()) != PV_OK ||
        (rc = allow_wide_lds<2, 3, 4, EPI_PART>()) != PV_OK || (rc = allow_wide_lds<2, 4, 4, EPI_PART>()) != PV_OK) return rc;
    if ((rc = allow_wide<1, 1>()) != PV_OK || (rc = allow_wide<2, 1>()) != PV_OK || (rc = allow_wide<2, 2>()) != PV_OK || (rc = allow_wide<2, 3>()) != PV_OK) return rc;
    return allow_wide<2, 4>();
}

// Strips a workgroup of k_gemm_q4, in rounds of one workgroup per CU: a round takes as long as its strips and the operand, which costs an eighth of a strip a row (the
// packed tiles hold the rows and nothing else), two strips as 16-row tiles.  Without that, 13 rows, 1376 strips: three strips and two rounds, K = 4096 / 8192 20.4 / 34.4 us,
// seven and one 19.0 / 30.5; 8 rows, K = 8192 28.7 and 27.2; 1 row, K = 4096 16.8 and 17.5.  Below K = 2048 an operand of any size is there by the time the codes are
// (K = 1024, three strips and seven, 8 rows 9.1 and 9.6, 13 rows 10.0 and 10.3).  One or two strips: in one round only.
struct q4_split { int S, rounds; };
static q4_split q4_strips(const pv_model *m, int strips, int ktiles, int rows, bool seven)
{
    const double operand = ktiles < 64 ? 0.4 : rows <= 8 ? 0.125 * rows : 2.0;
    q4_split best = {1, 1};
    double least = 1e30;
    for (int S : {7, 4, 3, 2, 1}) {
        const int rounds = ((strips + S - 1) / S + m->n_cus - 1) / m->n_cus;
        if ((S <= 2 && rounds > 1) || (S == 7 && !seven)) continue;
        const double t = rounds * (S + operand);
        if (t < least) { least = t; best = {S, rounds}; }
    }
    return best;
}
template <int NB, int EPI> static constexpr bool q4_seven() { return NB == 1 || EPI != EPI_LMHEAD; }       // (the vocabulary's epilogue is two registers short)

// 9..16 rows: whether k_gemm_q4 is ahead of k_gemm_tile_q4, whose slices leave no CU idle whatever the strips but cost one more kernel.  13 rows, us, there / here:
//  - up to two strips a CU: up to K = 12800 (256 strips, K = 4096 10.8 / 7.7, K = 12288 18.3 / 18.8, K = 14336 18.2 / 18.8; 512 strips, K = 12288 27.5 / 24.8, K = 28672 36.8 / 47.2);
//  - more: what a round of the operand costs grows with K, so fewer rounds the longer it is: one up to K = 16384 (1024 strips 44.2 / 41.2; K = 28672 58.9 / 65.6), two up to
//    8192 (2048 strips 42.6 / 40.5; K = 12288 55.7 / 57.6), three (2560 strips, K = 4096 32.6 / 30.9, K = 6144 41.4 / 43.6, K = 8192 50.7 / 55.7), four (3584 strips, K = 4096
//    40.1 / 40.0, K = 5120 46.3 / 48.7, K = 8192 65.0 / 73.0); with seven strips at any K where the shared tiles' CUs get as many eighths (3584 strips, K = 8192 65.3 / 57.8, K = 16384 115.7 / 104.0);
//  - past fourteen strips a CU only gate/up and QKV would gain, and only in part (K = 4096, 4352 strips 54.5 / 42.8, 7168 strips 59.3 / 56.5, 8016 strips 61.1 / 66.8;
//    vocabulary 55.1 / 48.9, 59.4 / 70.8, 61.5 / 78.3): not taken.
static bool q4_unshared(const pv_model *m, int strips, int ktiles, q4_split q)
{
    if (strips > 14 * m->n_cus || !pv_offsets_fit(ktiles)) return false;
    if (strips <= 2 * m->n_cus) return ktiles <= 400;
    if (q.rounds * ktiles <= 512) return true;
    const int groups = (strips + 15) / 16, slices = max(1, min(TILE_MAX_SLICES, 2 * m->n_cus / groups)), there = (groups * slices + m->n_cus - 1) / m->n_cus * 16;      // (strips a CU, times the slices)
    return q.S == 7 && 8 * q.S * q.rounds * slices <= 7 * there;
}

// Output and down projections: K-slices for k_gemm_q4, four strips a workgroup and one workgroup a CU, or 1.  Uncut, a CU reads the whole operand (4 bytes a row and feature, 64 as
// 16-row tiles) for one or two strips of codes (9 bytes a strip and feature); cut, its share of it for four, and k_tile_finish follows, some 3.5 us in all.  So what counts is the operand that a CU
// no longer reads, few rows as 18 bytes a feature (their waves have few bytes in flight).  us, uncut / cut, 256 strips: 8 rows, K = 4096 5.8 / 6.9, 8192 8.8 / 8.3, 14336 13.4 / 11.4, 28672
// 24.0 / 16.0; 13 rows, K = 2048 5.0 / 7.0, 4096 7.4 / 7.2, 8192 12.0 / 9.1, 14336 19.2 / 12.9, 28672 35.4 / 19.4; 1 row, 8192 7.5 / 7.8, 14336 11.0 / 10.9, 28672 19.1 / 14.8; 512 strips: 8 rows,
// 8192 10.9 / 11.3, 14336 16.9 / 16.2, 28672 30.9 / 26.8; 13 rows, 4096 8.7 / 9.1, 8192 14.8 / 13.2, 28672 44.0 / 33.5; 1 row, 14336 14.5 / 15.0, 28672 26.2 / 24.4.  Where the
// groups are no multiple of eight, cut ones take 0.6 us more (200 strips, 8 rows, K = 8192 8.7 / 9.0; 65 strips, 13 rows, K = 4096 6.9 / 7.4; 400 strips, 13 rows, K = 8192 14.4 / 12.9).
// These are chains of one projection; between a step's other kernels the sum takes another us (four 8B-shaped layers, one row, uncut / cut 229 / 233 us a step), hence lines a little further out.
// Steps of four layers, us: 8B shape, 13 rows 296 -> 290, 8 rows 257 -> 253, 70B shape, 8 rows 514 -> 501.
static int q4_slices(const pv_model *m, int strips, int ktiles, int rows, const float *part)
{
    const int groups = (strips + 3) / 4;
    if (part == nullptr || !pv_offsets_fit(ktiles) || 2 * groups > m->n_cus) return 1;
    const int slices = min(min(TILE_MAX_SLICES, m->n_cus / groups), ktiles / 32);       // (a batch for each of eight waves)
    if (slices < 2) return 1;
    const double operand = 32.0 * ktiles * (rows <= 8 ? max(4 * rows, 18) : 64);
    return operand * (slices - 1) / slices >= (groups % 8 == 0 ? 280e3 : 340e3) ? slices : 1;
}

// Output and down projections, 16-bit weights: K-slices for k_gemm_wide, four strips a workgroup and at most one workgroup a CU, or 1.
// Up to 16 rows: whole, a CU reads all of the operand for each of its strips, and with 257 strips some CUs go through two; cut, its share of it once for four strips, and k_tile_finish
// follows.  Both sides of 250 sizes (32 to 516 strips, K = 2048 to 28672, 1, 4, 8 and 13 rows) lie within some 6 % of 2.7 us (cut, with the sum: 5.3) plus the larger of what the busiest CU takes
// in at 59 GB/s, strips and operand, and the weights of all 256 CUs at 7.64 TB/s, with a smooth step between them (both).  us, whole / cut: 256 strips, 13 rows, K = 4096 9.7 / 9.8, 8192 16.9 /
// 14.5, 14336 27.8 / 22.0, 28672 52.9 / 39.9, 8 rows, 14336 21.6 / 21.4, 28672 40.9 / 38.0; 128 strips, 13 rows, 4096 8.7 / 7.3, 8192 15.4 / 9.6, 8 rows, 8192 10.3 / 9.6, 14336 16.2 / 13.2; 320
// strips, 13 rows, 4096 15.5 / 11.3, 8 rows, 8192 21.8 / 17.4; 512 strips, 13 rows, 14336 41.1 / 41.1, 28672 80.2 / 74.5; one row, 256 strips, 14336 18.9 / 21.6, 64 strips 12.6 / 9.3.
// These are chains of one projection; between a step's other kernels the sum takes another 1.2 us, and the line leaves as much again.  Steps of four layers, us: 8B shape, 13 rows 472 -> 453,
// 7B shape 411 -> 401, 70B shape (two layers) 636 -> 628; 1B shape, 12 rows, eight layers 560 -> 525.
static int cut_slices(const pv_model *m, int strips, int ktiles, int rows, const float *part)
{
    const int cus = m->n_cus, groups = (strips + 3) / 4;
    if (part == nullptr || !wide_fits(ktiles) || 2 * groups > cus) return 1;
    const int slices = min(TILE_MAX_SLICES, cus / groups);
    const double K = 32.0 * ktiles, operand = rows > 8 ? 64.0 : rows > 2 ? 4.0 * rows : 10.5;       // bytes a feature (one and two rows: the waves have few bytes in flight)
    const bool halves = rows <= 8 && ktiles >= 64 && 2 * strips <= cus, two = strips >= 512;
    const int wgs = halves ? 2 * strips : two ? (strips + 1) / 2 : strips, rounds = (wgs + cus - 1) / cus;
    const double hbm = strips * 32.0 * K / 7.64e6;
    auto both = [&](double load) { return pow(pow(load / 59.2e3, 2.73) + pow(hbm, 2.73), 1 / 2.73); };
    const double whole = both(rounds * ((halves ? 16 : two ? 64 : 32) + operand) * K), cut = both((128 + operand) * K / slices);
    return whole - cut > 2.6 + 2.1 ? slices : 1;
}

// 17..64 rows: against k_gemm_tile, whose workgroups take eight strips and half as long slices, so that twice as many sums are written and read (4 MiB with 32 rows and 256 strips), but half
// as much of the operand: up to 1024 features a slice, a multiple of eight groups.  us, there / here, 32 and 64 rows: 256 strips, K = 2048 10.0 / 8.4, 13.4 / 10.1, 4096 12.0 / 10.9, 15.9 / 14.0, 8192
// 16.6 / 16.8, 20.1 / 22.2; 128 strips, 8192 12.1 / 10.9, 15.9 / 14.1, 14336 15.9 / 16.0, 20.1 / 21.9; 64 strips, 14336 13.1 / 11.0, 16.0 / 14.7; 512 strips, 2048 14.8 / 12.1, 18.0 / 14.6, 4096
// 18.0 / 17.8, 21.3 / 22.9; 25 groups, 2048 8.0 / 8.2, 9.8 / 10.8, 33 groups, 4096 9.5 / 10.0, 12.4 / 13.1.  Four layers of the 8B shape, us a step: 4 x 8 rows 542 -> 533, 48
// nodes 593 -> 579.  From K = 512 on: below it k_gemm takes the projection whole, and the sum is a kernel for nothing (steps of eight layers with two such projections each, us, 17 / 64 rows, there / here: 32 strips,
// K = 256 248 / 283, 298 / 335, 480 270 / 293, 317 / 342, 512 296 / 297, 351 / 351; 256 strips, 256 292 / 326, 360 / 407, 480 317 / 346, 383 / 430, 512 352 / 346, 433 / 432; 48 rows go to
// k_gemm_tile there, K = 256 306 / 306 and 366 / 372, 384 324 / 317 and 387 / 381).
static int cut_slices_shared(const pv_model *m, int strips, int ktiles, const float *part)
{
    const int groups = (strips + 3) / 4;
    if (part == nullptr || ktiles < 16 || !wide_fits(ktiles) || groups % 8 != 0 || 2 * groups > m->n_cus) return 1;
    const int slices = min(TILE_MAX_SLICES, m->n_cus / groups);
    return ktiles <= 32 * slices ? slices : 1;
}

template <int NB, int CT, int EPI>
static int launch_cut(const gemm_args &ga, int strips, int slices, hipStream_t s)
{
    const int tps = (ga.ktiles + slices - 1) / slices, groups = (strips + 3) / 4;
    slices = (ga.ktiles + tps - 1) / tps;                        // (none empty)
    float4 *part = (float4 *)ga.tile_part;
    k_gemm_wide<NB, CT, 4, EPI_PART><<<dim3(groups, slices), wide_waves(CT, 4) * 64, wide_lds(CT, 4), s>>>(ga, tps, part);
    PV_HIP(hipGetLastError());
    k_tile_finish<CT, EPI, NB><<<dim3(groups, CT), 256, 0, s>>>(ga, part, slices);
    PV_HIP(hipGetLastError());
    return PV_OK;
}

// Eight waves, two workgroups a CU where there are that many.  Sixteen waves and one or two strips up to 4 rows, whose operand is small (K = 14336, 256 strips 16.4 -> 13.8; 8
// rows 16.8 and 16.5), but not below K = 2048, where sixteen waves have no batch each: 4 rows, K = 512, 256 strips 7.4 against
// 6.7, 512 strips 8.2 against 7.3, K = 1024 7.4 and 8.3 against 6.8 and 7.4, K = 2048 7.7 and 8.5 against 7.7 and 8.7.
template <int NB, int EPI>
static int launch_q4(const gemm_args &ga, int strips, q4_split q, hipStream_t s)
{
    const int groups = (strips + q.S - 1) / q.S;
    bool done = false;
    if constexpr (NB == 1) {
        if (q.S <= 2 && ga.rows <= 4 && ga.ktiles >= 64) {
            if (q.S == 1) k_gemm_q4<NB, 1, EPI, 16><<<groups, 1024, 0, s>>>(ga, ga.ktiles >> 2, nullptr);
            else k_gemm_q4<NB, 2, EPI, 16><<<groups, 1024, 0, s>>>(ga, ga.ktiles >> 2, nullptr);
            done = true;
        }
    }
    if (done) ;
    else if (q.S == 1) k_gemm_q4<NB, 1, EPI><<<groups, 512, 0, s>>>(ga, ga.ktiles >> 2, nullptr);
    else if (q.S == 2) k_gemm_q4<NB, 2, EPI><<<groups, 512, 0, s>>>(ga, ga.ktiles >> 2, nullptr);
    else if (q.S == 3) k_gemm_q4<NB, 3, EPI><<<groups, 512, 0, s>>>(ga, ga.ktiles >> 2, nullptr);
    else if (q.S == 4) k_gemm_q4<NB, 4, EPI><<<groups, 512, 0, s>>>(ga, ga.ktiles >> 2, nullptr);
    else if constexpr (q4_seven<NB, EPI>()) k_gemm_q4<NB, 7, EPI><<<groups, 512, 0, s>>>(ga, ga.ktiles >> 2, nullptr);
    PV_HIP(hipGetLastError());
    return PV_OK;
}

template <int NB, int CT, int EPI>
static int launch_gemm(const pv_model *m, const gemm_args &g, int strips, hipStream_t s)
{
    gemm_args ga = g;
    ga.nstrips = strips;
    // long strips: measured 0.3 % faster per step, short ones 0.3 % slower; a whole vocabulary (8016 strips, K = 4096) 176 -> 172 us: there the contiguous
    // runs of many workgroups, a power of two apart, advance in step
    ga.interleave = g.ktiles > 128 || (NB == 1 && EPI == EPI_LMHEAD && strips >= 2048);
    if (m->wbits == 4) {
        if constexpr (CT == 1) {
            if constexpr (EPI == EPI_RESID) {
                const int cut = q4_slices(m, strips, g.ktiles, NB == 1 ? g.rows : 16, g.tile_part);
                if (cut > 1) {
                    const int nb4 = g.ktiles >> 2, bps = (nb4 + cut - 1) / cut, slices = (nb4 + bps - 1) / bps;
                    float4 *part = (float4 *)g.tile_part;
                    k_gemm_q4<NB, 4, EPI><<<dim3((strips + 3) / 4, slices), 512, 0, s>>>(ga, bps, part);
                    PV_HIP(hipGetLastError());
                    k_tile_finish<1, EPI, NB><<<dim3((strips + 3) / 4, 1), 256, 0, s>>>(ga, part, slices);
                    PV_HIP(hipGetLastError());
                    return PV_OK;
                }
            }
            const q4_split q = q4_strips(m, strips, g.ktiles, NB == 1 ? g.rows : 16, q4_seven<NB, EPI>());
            if (NB == 1 || q4_unshared(m, strips, g.ktiles, q)) return launch_q4<NB, EPI>(ga, strips, q, s);
        }
        if constexpr (NB == 1) {
            return PV_EINVAL;                                  // (not reached)
        } else if constexpr (CT == 3) {
            pv_set_error("4-bit weights have no kernel for three column tiles");       // (their blocks of 33..48 rows run as four)
            return PV_EINVAL;
        } else {
            // Activation tiles shared through LDS, two strips per wave.  Few strips: cut along K.  Up to 32 rows two
            // workgroups fit on a CU (120 registers): at most 512 of them in one round (8B shape, 4 layers, 24 rows: 483 -> 442 us a
            // step against 256 and one per CU); more rows: one per CU, at most 256 (K = 4096, 48 rows, us for a projection and its
            // sum, one slice / two: 129 groups of 16 strips 77.6 / 85.5, 172 groups 78.1 / 88.5, 224 groups 83 / 79)
            const int nbat = g.ktiles / 4, ngroups = (strips + 15) / 16;
            int slices = g.tile_part == nullptr ? 1 : max(1, min(TILE_MAX_SLICES, (CT <= 2 ? 512 : 256) / ngroups));
            int bps = max(CT <= 2 ? 2 : 4, (nbat + slices - 1) / slices);
            slices = (nbat + bps - 1) / bps;
            while (slices > 1 && (size_t)slices * strips * CT * 256 > tile_part_floats(CT)) { bps += 1; slices = (nbat + bps - 1) / bps; }
            float4 *part = slices > 1 ? (float4 *)g.tile_part : nullptr;
            k_gemm_tile_q4<CT, EPI><<<dim3(ngroups, slices), 512, tile_q4_lds(CT), s>>>(ga, bps, part);
            PV_HIP(hipGetLastError());
            if (slices > 1) { k_tile_finish<CT, EPI><<<dim3((strips + 3) / 4, CT), 256, 0, s>>>(ga, part, slices); PV_HIP(hipGetLastError()); }
            return PV_OK;
        }
    } else if constexpr (NB == 2) {
        // Strips per workgroup: with enough strips to fill the machine anyway, the 2 CT operand
        // tiles per batch tile are matched by as many weight tiles (S = 2 or 4); a GEMM with few
        // strips keeps one strip per workgroup and more waves instead.
        constexpr int S = CT == 1 ? 2 : 4, NW = CT == 1 ? 8 : 4;
        if constexpr (EPI != EPI_RESID) {
            const int ws = wide_strips(m, strips, g.ktiles, CT);
            if (ws) return launch_wide<NB, CT, EPI>(ga, strips, ws, s);
        }
        if constexpr (EPI == EPI_RESID) {
            const int cut = CT == 1 ? cut_slices(m, strips, g.ktiles, 16, g.tile_part) : cut_slices_shared(m, strips, g.ktiles, g.tile_part);
            if (cut > 1) return launch_cut<NB, CT, EPI>(ga, strips, cut, s);
        }
        if constexpr (CT >= 2) {
            // Activation tiles shared through LDS; few strips: cut along K, into at most 256 workgroups, one a CU: with a few more (288 for the
            // 8B-shaped QKV projection) some CUs have two and the others wait for them (4 layers, us a step: 32 rows 542 -> 528, 48 rows 632 -> 614;
            // up to 512 workgroups: 570, 663).  From 129 groups of eight strips on that is one slice (K = 4096, us for a projection
            // and its sum with 24 / 48 rows, one slice / two: 129 groups 38.5 / 46.4 and 50.6 / 55.3, 224 groups 47.0 / 57.2 and 55.1 / 67.0).
            // Three column tiles for 33..48 rows instead of four, 48 rows, 8B shape, us: QKV 16.9 -> 15.0, O 12.7 -> 11.2, down 28.3 -> 25.5.
            if (CT == 3 || g.ktiles >= 16) {
                const int ngroups = (strips + 7) / 8;
                int slices = g.tile_part == nullptr ? 1 : max(1, min(TILE_MAX_SLICES, 256 / ngroups));
                int tps = (g.ktiles + slices - 1) / slices;
                tps = max(8, (tps + 1) & ~1);                        // whole steps, at least four per slice
                slices = (g.ktiles + tps - 1) / tps;
                while (slices > 1 && (size_t)slices * strips * CT * 256 > tile_part_floats(CT)) { tps += 2; slices = (g.ktiles + tps - 1) / tps; }
                float4 *part = slices > 1 ? (float4 *)g.tile_part : nullptr;
                k_gemm_tile<CT, 1, EPI><<<dim3(ngroups, slices), 512, 0, s>>>(ga, tps, part);
                PV_HIP(hipGetLastError());
                if (slices > 1) { k_tile_finish<CT, EPI><<<dim3((strips + 3) / 4, CT), 256, 0, s>>>(ga, part, slices); PV_HIP(hipGetLastError()); }
                return PV_OK;
            }
        }
        if constexpr (CT == 1) {
            // one column tile: batches walked several deep, like the packed rows (measured 2 - 3 % per step)
            if (g.ktiles >= 64 && pv_offsets_fit(g.ktiles)) {
                bool done = false;
                if constexpr (EPI == EPI_QKV) {       // (k + 1/2) x 256 strips: half strips as for the packed rows
                    if (strips % 256 == 128 && strips / 256 >= 1 && strips / 256 <= 2) {
                        ga.half_base = (strips / 256) * 256;
                        if (strips / 256 == 1) k_gemm<NB, CT, 2, EPI, 8, 3, true><<<256, 512, 0, s>>>(ga);
                        else k_gemm<NB, CT, 3, EPI, 8, 2, true><<<256, 512, 0, s>>>(ga);
                        done = true;
                    }
                }
                if (done) ;
                else if (strips >= 512) k_gemm<NB, CT, 2, EPI, 8, 2><<<(strips + 1) / 2, 512, 0, s>>>(ga);
                else k_gemm<NB, CT, 1, EPI, 8, 3><<<strips, 512, 0, s>>>(ga);
                PV_HIP(hipGetLastError());
                return PV_OK;
            }
        }
        if constexpr (CT != 3) {           // a short K, or (one column tile) one past the buffers' offsets
            if (strips >= 256 * S) k_gemm<NB, CT, S, EPI, NW><<<(strips + S - 1) / S, NW * 64, 0, s>>>(ga);
            else k_gemm<NB, CT, 1, EPI, 8><<<strips, 512, 0, s>>>(ga);
        }
    } else {
        // Eight waves, each three batches deep (two workgroups per CU at <= 128 registers): measured
        // 1 - 8 % faster per GEMM than sixteen waves that load and use one batch at a time; a short K
        // has too few batches per wave for that
        // Two strips per workgroup share every activation tile; taken where the halved number of
        // workgroups fills the 256 CUs as evenly as the full one (measured, 70B shapes: gate/up
        // 165 -> 156 us, down 79 -> 75 us, vocabulary projection 97 -> 92 us; where it would leave
        // CUs unevenly loaded, e.g. 640 or 1792 strips, one strip per workgroup is 3 - 10 % faster)
        // (k + 1/2) x 256 strips (the fused QKV projection of both benchmark shapes): k whole strips
        // and half of a shared one per workgroup, 256 workgroups
        if constexpr (EPI == EPI_QKV) {
            if (g.ktiles >= 64 && strips % 256 == 128 && strips / 256 >= 1 && strips / 256 <= 2) {
                ga.half_base = (strips / 256) * 256;
                if (strips / 256 == 1) k_gemm<NB, CT, 2, EPI, 8, 3, true><<<256, 512, 0, s>>>(ga);
                else k_gemm<NB, CT, 3, EPI, 8, 2, true><<<256, 512, 0, s>>>(ga);
                PV_HIP(hipGetLastError());
                return PV_OK;
            }
        }
        if constexpr (EPI != EPI_RESID) {
            // (more rounds than one: no better, or worse, than workgroups that start as others end: K = 8192, 3584 strips 137.5 both; K = 4096, 8016 strips 175 / 179)
            if (packed_wide(m, strips, g.ktiles, g.rows, EPI == EPI_SWIGLU))
                if (const int ws = wide_strips(m, strips, g.ktiles, 1)) return launch_wide<NB, CT, EPI>(ga, strips, ws, s);
        }
        if constexpr (EPI == EPI_SWIGLU) {
            // 3.5 x G strips, G a multiple of the CUs: three whole strips and a half per workgroup, so that every CU holds
            // the same number of equal workgroups from start to end (70B-shaped gate/up: 156.5 -> 153.7 us)
            if (g.ktiles >= 128 && half_strips_even(strips) && !one_strip_even(m, strips, g.ktiles, g.rows)) {
                const int G = 2 * strips / 7;
                ga.half_base = 3 * G;
                k_gemm<NB, CT, 4, EPI, 8, 2, true><<<G, 512, 0, s>>>(ga);
                PV_HIP(hipGetLastError());
                return PV_OK;
            }
        }
        if constexpr (EPI == EPI_RESID) {
            // at most half as many strips as CUs: a workgroup per 8-feature half (every CU works, on half the weights: 128 strips, one row,
            // K = 2048 and 8192 together 14.9 -> 13.6 us)
            if (ga.chunks > 0) {                                 // (merges_in_oproj)
                const int lds = ga.rows * g.ktiles * 128;
                const bool half = 2 * strips <= m->n_cus;
                ga.half_base = 0;
                auto go = [&](auto mg) {
                    if (half) k_gemm<NB, CT, 1, EPI, 8, 3, true, mg.value><<<2 * strips, 512, lds, s>>>(ga);
                    else k_gemm<NB, CT, 1, EPI, 8, 3, false, mg.value><<<strips, 512, lds, s>>>(ga);
                };
                if (ga.chunks <= 4) go(std::integral_constant<int, 4>());
                else go(std::integral_constant<int, 8>());
                PV_HIP(hipGetLastError());
                return PV_OK;
            }
            const int cut = cut_slices(m, strips, g.ktiles, g.rows, g.tile_part);
            if (cut > 1) return launch_cut<NB, CT, EPI>(ga, strips, cut, s);
            if (g.ktiles >= 64 && 2 * strips <= m->n_cus) {
                ga.half_base = 0;
                k_gemm<NB, CT, 1, EPI, 8, 3, true><<<2 * strips, 512, 0, s>>>(ga);
                PV_HIP(hipGetLastError());
                return PV_OK;
            }
        }
        const bool two = strips >= 512 && even(m, (strips + 1) / 2) >= even(m, strips);
        // (three batches deep, us: K = 2048, 1024 strips of gate/up 13.2 -> 12.8, 8016 of the vocabulary 83.0 -> 80.7; K = 4096, 4096 strips with one row
        // 86.2 -> 87.9, K = 5120 96.7 -> 96.8, K = 8192 162.1 -> 164.2, 1376 strips 56.4 -> 58.1; 512 with the residual 23.4 -> 24.3)
        // Their waves' batches interleaved from K = 4096 on, us: gate/up, 8 rows, 2000 strips 45.3 -> 41.5, 4096 strips 86.4 -> 79.8 (one strip a workgroup, vocabulary, 768 strips:
        // 21.4 -> 21.9; two below K = 4096: no difference)
        if (two) ga.interleave |= g.ktiles >= 128;
        bool done = false;
        if constexpr (EPI != EPI_RESID) {
            if (g.ktiles >= 64 && g.ktiles < 128 && two) { k_gemm<NB, CT, 2, EPI, 8, 3><<<(strips + 1) / 2, 512, 0, s>>>(ga); done = true; }
        }
        if (done) ;
        else if (g.ktiles >= 64 && two) k_gemm<NB, CT, 2, EPI, 8, 2><<<(strips + 1) / 2, 512, 0, s>>>(ga);
        else if (g.ktiles >= 64) k_gemm<NB, CT, 1, EPI, 8, 3><<<strips, 512, 0, s>>>(ga);
        else k_gemm<NB, CT, 1, EPI, 8><<<strips, 512, 0, s>>>(ga);
    }
    PV_HIP(hipGetLastError());
    return PV_OK;
}

// Whether the output projection of a block merges the attention's chunks itself, so that a layer has five kernels instead of six.  Every workgroup of it then reads
// the chunks of all heads, rows x K x chunks x 4 bytes, which pays while its threads have them in flight all at once: attention's
// merge and output projection, us: 1B shape, one row, 5 chunks 8.7 -> 6.5, two rows, 4 chunks 9.3 -> 7.4; 8B shape, one row, 4 chunks 11.9 -> 10.1; but in two rounds
// (8 chunks; two rows, 3 chunks) 12.0 -> 11.7 and 11.9 -> 12.1.  Up to two chunks the attention needs no merge.
// (Packed rows: the caller sees to it.)
static bool merges_in_oproj(const pv_cache *c, int rows, const pv_attn_split_info &sp)
{
    const pv_model_config &f = c->m->cfg;
    const int qd = f.n_q_heads * f.head_dim;
    if (c->blk_units != 0 || c->m->wbits != 16 || sp.chunks < 3 || sp.chunks > 8) return false;
    return qd >= 64 * 32 && f.d_model / 16 < 512 && rows * qd <= 4 * 512 * merge_items(sp.chunks <= 4 ? 4 : 8);      // (and the operand is at most 16 KiB)
}

template <int NB, int CT>
static int run_block(pv_cache *c, hipStream_t s)
{
    const pv_model *m = c->m;
    const pv_model_config &f = m->cfg;
    const int rows = c->last_rows, d = f.d_model, hd = f.head_dim, qd = f.n_q_heads * hd, kvd = f.n_kv_heads * hd, F = f.ffn_dim;
    mat_ws mw;
    mat_ws_layout(m, c->rows_cap, c->units_cap, c->n_pages * f.page_tokens, true, c->ws.part, &mw, c->ws.part_floats);
    const char *Wb = m->d_weights;
    auto gainp = [&](int kind, int l) { return (const uint16_t *)(Wb + pv_tref(m, kind, l).off); };

    k_mat_begin<NB><<<dim3(d / 16, CT), 64, 0, s>>>(c->ws.state, c->d_io->draft, rows, c->io->hdr[3], (const uint16_t *)(Wb + m->global[PV_T_EMBED].off), gainp(PV_T_ATTN_NORM, 0),
                                           (const double *)(Wb + m->inv_freq_off), c->ws.x, mw.ssq0, mw.xop_a, c->ws.rope, d, hd / 2, c->ws.page_table, pv_geom(c).page_shift);
    PV_HIP(hipGetLastError());

    gemm_args g = {};
    int prc;
    g.st = c->ws.state; g.rows = rows; g.inv_d = 1.0f / (float)d; g.eps = (float)f.rms_eps; g.ssq_parts = d / 16;
    g.q_hi = (uint16_t *)c->ws.q; g.q_lo = g.q_hi + (size_t)c->rows_cap * qd; g.q_rows = rows; g.pool = (uint16_t *)c->d_pool; g.rope = c->ws.rope; g.geom = pv_geom(c);
    g.n_q_heads = f.n_q_heads; g.q_strips = qd / 16; g.k_strips = kvd / 16;
    g.x = c->ws.x; g.d = d; g.xop_act = mw.xop_d; g.F = F;
    g.logits = c->ws.logits; g.pmax_val = mw.pmax_val; g.pmax_idx = mw.pmax_idx; g.vocab = f.vocab;
    g.tile_part = mw.tile_part;
    const pv_attn_split_info sp = pv_attn_split(c, rows, mw.attn_part);
    const bool fused = NB == 1 && merges_in_oproj(c, rows, sp);
    g.part_o = sp.part_o; g.part_ml = sp.part_ml; g.max_chunks = sp.max_chunks; g.chunk_shift = sp.chunk_shift; g.units = sp.units;

    for (int l = 0; l < f.n_layers; ++l) {
        // fused QKV projection: RMSNorm scale, rotary embedding, KV append
        g.W = (const uint4 *)(Wb + pv_tref(m, PV_T_WQ, l).off); g.xop = (const uint4 *)mw.xop_a; g.ktiles = d / 32;
        g.ssq = mw.ssq0; g.layer = l;
        if ((prc = pv_prof_mark(c, PV_PROF_QKV, l, 0, s)) != PV_OK) return prc;
        if ((prc = launch_gemm<NB, CT, EPI_QKV>(m, g, (qd + 2 * kvd) / 16, s)) != PV_OK) return prc;
        if ((prc = pv_prof_mark(c, PV_PROF_QKV, l, 1, s)) != PV_OK) return prc;
        // attention over the paged cache -> operand of the output projection
        if ((prc = pv_prof_mark(c, PV_PROF_ATTENTION, l, 0, s)) != PV_OK) return prc;
        int rc = pv_mat_attention(c, l, rows, mw.attn_part, mw.xop_o, !fused, s);
        if (rc != PV_OK) return rc;
        if ((prc = pv_prof_mark(c, PV_PROF_ATTENTION, l, 1, s)) != PV_OK) return prc;
        // output projection + residual; emits the FFN operand and sum of squares
        g.W = (const uint4 *)(Wb + pv_tref(m, PV_T_WO, l).off); g.xop = (const uint4 *)mw.xop_o; g.ktiles = qd / 32;
        g.gain_next = gainp(PV_T_FFN_NORM, l); g.ssq_out = mw.ssq1; g.xop_out = mw.xop_f; g.chunks = fused ? sp.chunks : 0;
        if ((prc = pv_prof_mark(c, PV_PROF_OPROJ, l, 0, s)) != PV_OK) return prc;
        if ((prc = launch_gemm<NB, CT, EPI_RESID>(m, g, d / 16, s)) != PV_OK) return prc;
        if ((prc = pv_prof_mark(c, PV_PROF_OPROJ, l, 1, s)) != PV_OK) return prc;
        g.chunks = 0;
        // gate/up projection + SwiGLU
        g.W = (const uint4 *)(Wb + pv_tref(m, PV_T_WG, l).off); g.xop = (const uint4 *)mw.xop_f; g.ktiles = d / 32;
        g.ssq = mw.ssq1;
        if ((prc = pv_prof_mark(c, PV_PROF_GATEUP, l, 0, s)) != PV_OK) return prc;
        if ((prc = launch_gemm<NB, CT, EPI_SWIGLU>(m, g, F / 8, s)) != PV_OK) return prc;
        if ((prc = pv_prof_mark(c, PV_PROF_GATEUP, l, 1, s)) != PV_OK) return prc;
        // down projection + residual; emits the next layer's (or the head's) operand
        g.W = (const uint4 *)(Wb + pv_tref(m, PV_T_WD, l).off); g.xop = (const uint4 *)mw.xop_d; g.ktiles = F / 32;
        g.gain_next = (l + 1 < f.n_layers) ? gainp(PV_T_ATTN_NORM, l + 1) : (const uint16_t *)(Wb + m->global[PV_T_FINAL_NORM].off);
        g.ssq_out = mw.ssq0; g.xop_out = mw.xop_a;
        if ((prc = pv_prof_mark(c, PV_PROF_DOWN, l, 0, s)) != PV_OK) return prc;
        if ((prc = launch_gemm<NB, CT, EPI_RESID>(m, g, d / 16, s)) != PV_OK) return prc;
        if ((prc = pv_prof_mark(c, PV_PROF_DOWN, l, 1, s)) != PV_OK) return prc;
    }
    const bool head = c->io->hdr[3] != PV_MODE_PREFILL_MID;
    if (head) {
        g.W = (const uint4 *)(Wb + m->global[PV_T_LM_HEAD].off); g.xop = (const uint4 *)mw.xop_a; g.ktiles = d / 32; g.ssq = mw.ssq0;
        if ((prc = pv_prof_mark(c, PV_PROF_LMHEAD, 0, 0, s)) != PV_OK) return prc;
        if ((prc = launch_gemm<NB, CT, EPI_LMHEAD>(m, g, f.vocab / 16, s)) != PV_OK) return prc;
        if ((prc = pv_prof_mark(c, PV_PROF_LMHEAD, 0, 1, s)) != PV_OK) return prc;
    }
    return pv_k_finish(c, rows, mw.pmax_val, mw.pmax_idx, f.vocab / 16, s);
}

int pv_mat_run_block(pv_cache *c, hipStream_t s)
{
    const int rows = c->last_rows;
    if (rows > 64) { pv_set_error("matrix path handles at most 64 rows per block"); return PV_ERANGE; }
    if (pv_packs_rows(c->m, rows)) return run_block<1, 1>(c, s);
    if (rows <= 16) return run_block<2, 1>(c, s);
    if (rows <= 32) return run_block<2, 2>(c, s);
    if (rows <= 48 && c->m->wbits == 16) return run_block<2, 3>(c, s);
    return run_block<2, 4>(c, s);
}

int pv_mat_run_prompt(pv_cache *c, int rows, int keep, hipStream_t s)
{
    const pv_model *m = c->m;
    const pv_model_config &f = m->cfg;
    mat_ws mw;
    mat_ws_layout(m, c->rows_cap, c->units_cap, c->n_pages * f.page_tokens, true, c->ws.part, &mw, c->ws.part_floats);
    pv_pre_out out;
    int rc = pv_pre_block(c, c->d_io->prompt, rows, keep, &out, s);
    if (rc != PV_OK || keep == 0) return rc;
    // the head of the kept rows (whatever their number, as column tiles of 16 rows: the layout of the prompt's operand)
    gemm_args g = {};
    g.st = c->ws.state; g.rows = keep; g.inv_d = 1.0f / (float)f.d_model; g.eps = (float)f.rms_eps; g.ssq_parts = f.d_model / 16;
    g.logits = c->ws.logits; g.pmax_val = mw.pmax_val; g.pmax_idx = mw.pmax_idx; g.vocab = f.vocab; g.tile_part = mw.tile_part;
    g.W = (const uint4 *)(m->d_weights + m->global[PV_T_LM_HEAD].off); g.xop = (const uint4 *)out.xop; g.ktiles = f.d_model / 32; g.ssq = out.ssq;
    if ((rc = pv_prof_mark(c, PV_PROF_LMHEAD, 0, 0, s)) != PV_OK) return rc;
    const int ct = col_tiles(keep);
    rc = ct == 1 ? launch_gemm<2, 1, EPI_LMHEAD>(m, g, f.vocab / 16, s) : ct == 2 ? launch_gemm<2, 2, EPI_LMHEAD>(m, g, f.vocab / 16, s) : launch_gemm<2, 4, EPI_LMHEAD>(m, g, f.vocab / 16, s);
    if (rc != PV_OK) return rc;
    if ((rc = pv_prof_mark(c, PV_PROF_LMHEAD, 0, 1, s)) != PV_OK) return rc;
    return pv_k_finish(c, keep, mw.pmax_val, mw.pmax_idx, f.vocab / 16, s);
}
