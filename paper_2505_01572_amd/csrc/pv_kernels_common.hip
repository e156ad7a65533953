// Small kernels both kernel families use: block set-up (embedding gather + rotary table), the end of
// a step (arg-max over the candidates, acceptance rule), KV export.
// None of them is bandwidth relevant; they are written for clarity and determinism.
#include "pv_kernels_common.h"

// ---------------------------------------------------------------------------------------
// Block set-up: x[j,:] = E[draft[j],:] and the rotary table of positions len .. len+gamma-1.
// Angles are formed in double (pos * base^(-2i/head_dim)) so that large positions lose no
// precision before sin/cos; the table is stored as float2 (cos, sin).
// ---------------------------------------------------------------------------------------
// The draft ids are read straight from the cache's pinned host mailbox; block 0 copies them, the
// row count and the mode into the device state for the kernels that follow.
template <typename ST>
__global__ void __launch_bounds__(256)
k_begin(pv_dev_state *st, const int32_t *mailbox, int gamma, int mode, const ST *embed, const double *inv_freq, float *x, float2 *rope, int d, int half)
{
    const int j = blockIdx.x;
    if (j == 0) {
        if ((int)threadIdx.x < gamma) st->draft[threadIdx.x] = mailbox[threadIdx.x];
        if (threadIdx.x == 0) { st->gamma = gamma; st->mode = mode; st->blk.seq[0].gamma = gamma; }
    }
    float *xr = x + (size_t)j * d;
    if (j >= gamma) {                        // padding rows: keep them finite
        for (int i = threadIdx.x; i < d; i += 256) xr[i] = 0.f;
        for (int i = threadIdx.x; i < half; i += 256) rope[(size_t)j * half + i] = make_float2(1.f, 0.f);
        return;
    }
    const ST *e = embed + (size_t)mailbox[j] * d;
    for (int i = threadIdx.x; i < d; i += 256) xr[i] = pv_ld(e, i);
    const double pos = (double)(st->len + j);
    for (int i = threadIdx.x; i < half; i += 256) {
        double s, c;
        sincos(pos * inv_freq[i], &s, &c);
        rope[(size_t)j * half + i] = make_float2((float)c, (float)s);
    }
}

// order of the arg-max: value descending, index ascending
__device__ inline bool pv_better(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }

// The best candidate of the wave, in every lane.
__device__ inline void pv_wave_argmax(float &bv, int &bi)
{
    auto take = [&](uint32_t ov, uint32_t oi) { const float v = __uint_as_float(ov); if (pv_better(v, (int)oi, bv, bi)) { bv = v; bi = (int)oi; } };
#define PV_ROTATED(N) take(__builtin_amdgcn_update_dpp(0u, __float_as_uint(bv), 0x120 + N, 0xF, 0xF, true), __builtin_amdgcn_update_dpp(0u, (uint32_t)bi, 0x120 + N, 0xF, 0xF, true))
    PV_ROTATED(1); PV_ROTATED(2); PV_ROTATED(4); PV_ROTATED(8);
#undef PV_ROTATED
    auto pair = [&](auto v, auto i) { take(v[0], i[0]); take(v[1], i[1]); };       // (one of the two is the lane's own)
    pair(__builtin_amdgcn_permlane16_swap(__float_as_uint(bv), __float_as_uint(bv), false, false), __builtin_amdgcn_permlane16_swap((uint32_t)bi, (uint32_t)bi, false, false));
    pair(__builtin_amdgcn_permlane32_swap(__float_as_uint(bv), __float_as_uint(bv), false, false), __builtin_amdgcn_permlane32_swap((uint32_t)bi, (uint32_t)bi, false, false));
}

// The arg-max of one row, ahead of k_finish, where the candidates of all rows are more than its one workgroup reads quickly.
__global__ void __launch_bounds__(256)
k_row_argmax(pv_dev_state *st, const float *pv, const int32_t *pi, int strips)
{
    const float *rv = pv + (size_t)blockIdx.x * strips; const int32_t *ri = pi + (size_t)blockIdx.x * strips;
    float bv = -INFINITY; int bi = 0x7fffffff;
    for (int s0 = threadIdx.x; s0 < strips; s0 += 256 * 4) {
        float v[4]; int i[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) { const int s = s0 + 256 * u, sc = s < strips ? s : s0; v[u] = rv[sc]; i[u] = ri[sc]; }
#pragma unroll
        for (int u = 0; u < 4; ++u) if (pv_better(v[u], i[u], bv, bi)) { bv = v[u]; bi = i[u]; }      // (a candidate taken twice changes nothing)
    }
    pv_wave_argmax(bv, bi);
    __shared__ float wv[4];
    __shared__ int wi[4];
    if ((threadIdx.x & 63) == 0) { wv[threadIdx.x >> 6] = bv; wi[threadIdx.x >> 6] = bi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) if (pv_better(wv[w], wi[w], bv, bi)) { bv = wv[w]; bi = wi[w]; }
        st->pred[blockIdx.x] = (bv == -INFINITY) ? -1 : bi;                  // no finite logit in the row: no arg-max
    }
}

// ---------------------------------------------------------------------------------------
// End of a step in one launch: vocabulary arg-max of every row from the candidates that the
// vocabulary projection left (one per strip and row; NaN counted as -inf), the acceptance rule
// (Algorithm 1, verify branch: longest draft prefix that equals the stage's own greedy tokens,
// one correction token) and the in-step rollback (length, pending).  The two results and an
// error flag go straight to the cache's pinned host mailbox.
// One workgroup of 16 waves: a row is scanned by 16 / (rows rounded up to a power of two) waves
// (one wave takes up to four rows when there are more than 16), sixteen candidates per lane in
// flight; after the barrier one thread per sequence of the block applies the rule.
// ---------------------------------------------------------------------------------------
// What the rule needs from memory (the sequences, their pending tokens, the drafts) is asked for beside the candidates and ahead of the reductions, which stay on the
// vector ALU: one trip to memory and a half instead of four in a row (with the set-up kernel: two layers, 4 rows, 16384 keys 237.5 -> 235.6 us a step, four sequences 545 -> 541, the fp32 configuration 79.1 -> 78.2).
__global__ void __launch_bounds__(1024)
k_finish(pv_dev_state *st, int32_t *result, const float *pv, const int32_t *pi, int strips, int gamma, int mode, int vocab)
{
    __shared__ float wv[16];
    __shared__ int wi[16];
    __shared__ int pred_s[PV_MAX_ROWS], draft_s[PV_MAX_ROWS], parent_s[PV_MAX_ROWS];
    __shared__ int err_s;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, tid = threadIdx.x;
    int nseq = 0, draft = 0, parent = 0, pending = 0, len = 0;
    pv_seq_ref sq = {};
    if (wave == 0) {
        nseq = st->blk.n_seq;
        if (tid < PV_MAX_SEQ) sq = st->blk.seq[tid];            // (those past the block's own are not looked at)
        draft = st->draft[tid];
        if (mode == PV_MODE_TREE) parent = st->parent[tid];
    }
    auto own_state = [&]() { if (tid < nseq) { pending = sq.st->pending; len = sq.st->len; } };
    if (pv != nullptr && mode != PV_MODE_PREFILL_MID) {
        int wpr = 16;                                 // waves per row
        while (wpr > 1 && gamma * wpr > 16) wpr >>= 1;
        for (int j0 = 0; j0 < gamma; j0 += 16 / wpr) {           // one pass unless there are more than 16 rows
            const int j = j0 + wave / wpr, part = wave % wpr;
            float bv = -INFINITY; int bi = 0x7fffffff;
            if (j < gamma) {
                const float *rv = pv + (size_t)j * strips; const int32_t *ri = pi + (size_t)j * strips;
                for (int s0 = part * 64 + lane; s0 < strips; s0 += 64 * wpr * 16) {
                    float v[16]; int i[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) { const int s = s0 + 64 * wpr * u, sc = s < strips ? s : s0; v[u] = rv[sc]; i[u] = ri[sc]; }
#pragma unroll
                    for (int u = 0; u < 16; ++u)
                        if (s0 + 64 * wpr * u < strips && pv_better(v[u], i[u], bv, bi)) { bv = v[u]; bi = i[u]; }
                }
            }
            if (j0 == 0) own_state();
            pv_wave_argmax(bv, bi);
            if (lane == 0) { wv[wave] = bv; wi[wave] = bi; }
            __syncthreads();
            if (tid < 16 / wpr && j0 + tid < gamma) {
                float fv = wv[tid * wpr]; int fi = wi[tid * wpr];
                for (int w = 1; w < wpr; ++w) if (pv_better(wv[tid * wpr + w], wi[tid * wpr + w], fv, fi)) { fv = wv[tid * wpr + w]; fi = wi[tid * wpr + w]; }
                pred_s[j0 + tid] = (fv == -INFINITY) ? -1 : fi;     // no finite logit in the row: no arg-max
            }
            __syncthreads();
        }
    } else {
        own_state();
        if (tid < gamma) pred_s[tid] = st->pred[tid];
    }
    if (wave == 0) { draft_s[tid] = draft; parent_s[tid] = parent; }
    if (tid == 0) err_s = 0;
    __syncthreads();
    // the rule, one thread per sequence of the block (a plain step has one: the cache itself)
    if (tid < nseq) {
        pv_dev_state *ps = sq.st;                    // the sequence's own state
        const int g = sq.gamma, r0 = sq.row0;
        int n, next, err = 0;
        if (mode == PV_MODE_PREFILL_MID) { n = g; next = -1; }
        else {
            // a row without a finite logit has no arg-max: the step reports an error and commits nothing
            for (int j = 0; j < g; ++j) { if (pred_s[r0 + j] < 0 || pred_s[r0 + j] >= vocab) err = 1; st->pred[r0 + j] = pred_s[r0 + j]; }
            if (err) { n = 0; next = pending; }
            else if (mode == PV_MODE_PREFILL_LAST) { n = g; next = pred_s[r0 + g - 1]; }
            else if (mode == PV_MODE_TREE) {
                // Greedy walk down the draft tree: at every step the child (lowest row first) whose token is the one
                // the stage itself predicts next is taken; its own prediction is then what its children must match.
                // The rows of the path are left in st->path for the compaction of their keys and values.
                int cur = -1, expected = pending;
                n = 0;
                for (;;) {
                    int pick = -1;
                    for (int r = cur + 1; r < g && pick < 0; ++r)
                        if (parent_s[r] == cur && (expected < 0 ? true : draft_s[r] == expected)) pick = r;     // (pending unknown: the first root is trusted)
                    if (pick < 0) break;
                    st->path[n++] = pick;
                    cur = pick; expected = pred_s[pick];
                }
                next = (n >= 1) ? pred_s[cur] : pending;
            }
            else {
                n = 0;
                while (n < g) {
                    const int expected = (n == 0) ? (pending >= 0 ? pending : draft_s[r0]) : pred_s[r0 + n - 1];
                    if (draft_s[r0 + n] != expected) break;
                    ++n;
                }
                next = (n >= 1) ? pred_s[r0 + n - 1] : pending;
            }
        }
        result[2 * tid] = n; result[2 * tid + 1] = next;
        ps->accepted = n;
        ps->next_token = next;
        ps->pending = next;
        ps->len = len + n;
        if (err) err_s = 1;
    }
    __syncthreads();
    if (tid == 0) result[PV_RESULT_ERR] = err_s;
}

// ---------------------------------------------------------------------------------------
// After a draft-tree step: the accepted path's rows sit in the slots of their row numbers
// (old length + path[d]); move their keys and values to the positions they now hold
// (old length + d).  path[] is increasing and path[d] >= d, so going through d in order never
// overwrites a row that is still to be moved.  One thread per (layer, K|V, kv head, feature).
// ---------------------------------------------------------------------------------------
template <typename ST>
__global__ void __launch_bounds__(256)
k_tree_compact(const pv_dev_state *st, const int32_t *page_table, ST *pool, pv_kv_geom g, int n_layers)
{
    const int kvd = g.n_kv_heads * g.head_dim;
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (size_t)n_layers * 2 * kvd) return;
    const int c = (int)(idx % kvd), which = (int)((idx / kvd) & 1), layer = (int)(idx / kvd / 2);
    const int h = c / g.head_dim, e = c - h * g.head_dim;
    const int n = st->accepted, len0 = st->len - n;          // (the finishing kernel has added n already)
    for (int d = 0; d < n; ++d) {
        const int src = len0 + st->path[d], dst = len0 + d;
        if (src == dst) continue;
        const ST *sb = pool + pv_kv_block(g, layer, page_table[src >> g.page_shift], h, which);
        ST *db = pool + pv_kv_block(g, layer, page_table[dst >> g.page_shift], h, which);
        const int ts = src & (g.page_tokens - 1), td = dst & (g.page_tokens - 1);
        db[which ? pv_v_off(g, td, e) : pv_k_off(g, td, e)] = sb[which ? pv_v_off(g, ts, e) : pv_k_off(g, ts, e)];
    }
}

__global__ void k_set_state(pv_dev_state *st, int len, int pending)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) { st->len = len; st->pending = pending; }
}

// ---------------------------------------------------------------------------------------
// Gather logical K/V elements [e0, e0+n) of the layout [layer][2][len][kv_dim] into out.
// ---------------------------------------------------------------------------------------
template <typename ST>
__global__ void k_export(const ST *pool, const int32_t *page_table, pv_kv_geom g, int len, size_t e0, size_t n, ST *out)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const size_t e = e0 + i;
    const int kvd = g.n_kv_heads * g.head_dim;
    const int c = (int)(e % kvd);
    const size_t r = e / kvd;
    const int pos = (int)(r % len);
    const size_t lw = r / len;
    const int which = (int)(lw & 1), layer = (int)(lw >> 1);
    const int h = c / g.head_dim, d = c - h * g.head_dim;
    const int phys = page_table[pos >> g.page_shift], tok = pos & (g.page_tokens - 1);
    const ST *b = pool + pv_kv_block(g, layer, phys, h, which);
    out[i] = which ? b[pv_v_off(g, tok, d)] : b[pv_k_off(g, tok, d)];
}

// ------------------------------- host launchers ----------------------------------------

pv_kv_geom pv_geom(const pv_cache *c)
{
    pv_kv_geom g;
    g.n_pages = c->n_pages; g.n_kv_heads = c->m->cfg.n_kv_heads; g.page_tokens = c->m->cfg.page_tokens;
    g.head_dim = c->m->cfg.head_dim;
    g.tiled = c->m->path >= PV_PATH_MATRIX;
    g.page_shift = 0;
    while ((1 << g.page_shift) < g.page_tokens) ++g.page_shift;
    return g;
}

int pv_k_begin(pv_cache *c, int rows_pad, hipStream_t s)
{
    const pv_model *m = c->m;
    const double *inv = (const double *)(m->d_weights + m->inv_freq_off);
    const void *emb = m->d_weights + m->global[PV_T_EMBED].off;
    const int rows = c->last_rows, mode = c->io->hdr[3];
    if (m->cfg.dtype == PV_BF16)
        k_begin<uint16_t><<<rows_pad, 256, 0, s>>>(c->ws.state, c->d_io->draft, rows, mode, (const uint16_t *)emb, inv, c->ws.x, c->ws.rope, m->cfg.d_model, m->cfg.head_dim / 2);
    else
        k_begin<float><<<rows_pad, 256, 0, s>>>(c->ws.state, c->d_io->draft, rows, mode, (const float *)emb, inv, c->ws.x, c->ws.rope, m->cfg.d_model, m->cfg.head_dim / 2);
    PV_HIP(hipGetLastError());
    return PV_OK;
}

// pmax_val / pmax_idx: per-strip arg-max candidates [rows][strips] (null: none, a prompt's middle)
int pv_k_finish(pv_cache *c, int rows, const float *pmax_val, const int32_t *pmax_idx, int strips, hipStream_t s)
{
    // The finishing kernel is one workgroup, and a CU reads some 50 GB/s: above 32768 candidates the rows' arg-max is a kernel of its own
    // (48 rows x 1024 strips: 18.4 us in one, 4.6 + 8.8 in two; 32 x 1024: 8.8 and 4.6 + 5.0)
    if (pmax_val != nullptr && c->io->hdr[3] != PV_MODE_PREFILL_MID && (size_t)rows * strips > 32768) {
        k_row_argmax<<<rows, 256, 0, s>>>(c->ws.state, pmax_val, pmax_idx, strips);
        PV_HIP(hipGetLastError());
        pmax_val = nullptr;
    }
    k_finish<<<1, 1024, 0, s>>>(c->ws.state, c->d_io->result, pmax_val, pmax_idx, strips, rows, c->io->hdr[3], c->m->cfg.vocab);
    PV_HIP(hipGetLastError());
    return PV_OK;
}

int pv_k_tree_compact(pv_cache *c, hipStream_t s)
{
    const pv_kv_geom g = pv_geom(c);
    const size_t n = (size_t)c->m->cfg.n_layers * 2 * g.n_kv_heads * g.head_dim;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (c->m->cfg.dtype == PV_BF16)
        k_tree_compact<uint16_t><<<blocks, 256, 0, s>>>(c->ws.state, c->ws.page_table, (uint16_t *)c->d_pool, g, c->m->cfg.n_layers);
    else
        k_tree_compact<float><<<blocks, 256, 0, s>>>(c->ws.state, c->ws.page_table, (float *)c->d_pool, g, c->m->cfg.n_layers);
    PV_HIP(hipGetLastError());
    return PV_OK;
}

int pv_k_set_state(pv_cache *c, int len, int pending, hipStream_t s)
{
    k_set_state<<<1, 64, 0, s>>>(c->ws.state, len, pending);
    PV_HIP(hipGetLastError());
    return PV_OK;
}

int pv_k_export(pv_cache *c, size_t e0, size_t n, void *d_out, hipStream_t s)
{
    const pv_kv_geom g = pv_geom(c);
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (c->m->cfg.dtype == PV_BF16)
        k_export<uint16_t><<<blocks, 256, 0, s>>>((const uint16_t *)c->d_pool, c->ws.page_table, g, c->len, e0, n, (uint16_t *)d_out);
    else
        k_export<float><<<blocks, 256, 0, s>>>((const float *)c->d_pool, c->ws.page_table, g, c->len, e0, n, (float *)d_out);
    PV_HIP(hipGetLastError());
    return PV_OK;
}
