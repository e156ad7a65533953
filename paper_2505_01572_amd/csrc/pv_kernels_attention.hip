// Kernel wrappers of the attention units (pv_attention_body.h) for the per-kernel step sequence.
#include "pv_attention_body.h"

// NB = 0: one chunk a workgroup, partial results (k_attn_merge follows); NB = 1, 2: all chunks, the operand itself
template <int HD, int TILES, int NB>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 4)))
k_attn(const attn_args a)
{
    extern __shared__ float4 smem4[];               // attn_smem_floats<HD>() floats: above the static limit for HD = 128
    attn_chunk<HD, TILES, NB>(a, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.z, (float *)smem4);
}

template <int NB, int HD>
__global__ void __launch_bounds__(256)
k_attn_merge(const attn_args a, int n_units)
{
    __shared__ float4 smem4[64 + 4 * (HD / 4) * 2];
    attn_merge_unit<NB, HD, 256>(a, blockIdx.x, blockIdx.y, n_units, threadIdx.x, (float *)smem4);
}

// ------------------------------- host side ----------------------------------------

// Row-group units (32 query rows of one kv head) of one sequence with `rows` block rows
int pv_attn_units(const pv_model *m, int rows)
{
    const int group = m->cfg.n_q_heads / m->cfg.n_kv_heads;
    return (group * rows + 31) / 32;
}

size_t pv_attn_part_floats(const pv_model *m, int units_cap, int max_tokens)
{
    const pv_model_config &f = m->cfg;
    const int chunks = (max_tokens + 127) / 128;   // the finer of the two chunkings
    return (size_t)f.n_kv_heads * units_cap * chunks * 32 * (f.head_dim + 2);
}

// Keys the launch has to cover (the host's bound, not the whole cache), cut into chunks of 256 (up to 16 query rows per kv head) or 128
pv_attn_split_info pv_attn_split(const pv_cache *c, int rows, const float *part)
{
    const pv_model_config &f = c->m->cfg;
    const int nrows = f.n_q_heads / f.n_kv_heads * rows, keys = c->attn_keys > 0 && c->attn_keys < c->max_tokens ? c->attn_keys : c->max_tokens;
    pv_attn_split_info i;
    i.chunk_shift = nrows <= 16 ? 8 : 7;
    i.chunks = (keys + (1 << i.chunk_shift) - 1) >> i.chunk_shift;
    i.max_chunks = (c->max_tokens + (1 << i.chunk_shift) - 1) >> i.chunk_shift;
    i.units = (nrows + 31) / 32;
    i.part_o = part; i.part_ml = part + (size_t)f.n_kv_heads * c->units_cap * ((c->max_tokens + 127) / 128) * 32 * f.head_dim;
    return i;
}

// rows: rows of the block; a batched step also gives its unit count and the most rows any one sequence has
template <int NB, int HD>
static int launch(pv_cache *c, attn_args &a, int rows, bool merge, hipStream_t s)
{
    const pv_model_config &f = c->m->cfg;
    const int seq_rows = c->blk_units ? c->blk_seq_rows : rows;
    const int nrows = a.group * seq_rows, units = c->blk_units ? c->blk_units : (nrows + 31) / 32;
    // up to 16 query rows per kv head: 256-key chunks, eight waves of 32 keys each; more rows:
    // 128-key chunks, the waves split into two 16-row tiles x four 32-key groups
    constexpr size_t lds = attn_smem_floats<HD>() * sizeof(float);
    // chunks to launch: enough for the keys this step can reach (the host's bound), not for the whole cache
    const int keys = c->attn_keys > 0 && c->attn_keys < c->max_tokens ? c->attn_keys : c->max_tokens;
    // Up to two chunks: one workgroup per kv head and row group goes through them and there is nothing to merge.  Measured per layer
    // against chunks and merge (8B and 1B shapes): one chunk -3.5 us, two -2 us, four +3 us, eight +10 us (a chunk costs its
    // workgroup 2 us, mostly latency; loading the next keys ahead did not help).
    if (merge && keys <= (nrows <= 16 ? 512 : 256)) {
        if (nrows <= 16) k_attn<HD, 1, NB><<<dim3(1, f.n_kv_heads, units), 512, lds, s>>>(a);
        else k_attn<HD, 2, NB><<<dim3(1, f.n_kv_heads, units), 512, lds, s>>>(a);
        PV_HIP(hipGetLastError());
        return PV_OK;
    }
    if (nrows <= 16) {
        a.chunk_shift = 8; a.max_chunks = (c->max_tokens + 255) / 256; a.chunks = (keys + 255) / 256;
        k_attn<HD, 1, 0><<<dim3(a.chunks, f.n_kv_heads, units), 512, lds, s>>>(a);
    } else {
        a.chunk_shift = 7; a.max_chunks = (c->max_tokens + 127) / 128; a.chunks = (keys + 127) / 128;
        k_attn<HD, 2, 0><<<dim3(a.chunks, f.n_kv_heads, units), 512, lds, s>>>(a);
    }
    PV_HIP(hipGetLastError());
    if (!merge) return PV_OK;
    k_attn_merge<NB, HD><<<dim3(rows, f.n_q_heads), 256, 0, s>>>(a, units);
    PV_HIP(hipGetLastError());
    return PV_OK;
}

template <int HD>
static int allow_lds()
{
    constexpr int lds = attn_smem_floats<HD>() * (int)sizeof(float);
    auto allow = [&](const void *k) { return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lds); };
    PV_HIP(allow((const void *)k_attn<HD, 1, 0>)); PV_HIP(allow((const void *)k_attn<HD, 1, 1>)); PV_HIP(allow((const void *)k_attn<HD, 1, 2>));
    PV_HIP(allow((const void *)k_attn<HD, 2, 0>)); PV_HIP(allow((const void *)k_attn<HD, 2, 1>)); PV_HIP(allow((const void *)k_attn<HD, 2, 2>));
    return PV_OK;
}

// once per device before the first launch (and outside any stream capture): the attention
// kernels use more dynamic LDS than the default limit
int pv_mat_attention_init(int head_dim)
{
    switch (head_dim) {
    case 32: return allow_lds<32>();
    case 64: return allow_lds<64>();
    case 128: return allow_lds<128>();
    default: pv_set_error("matrix path: unsupported head_dim %d", head_dim); return PV_EINVAL;
    }
}

// q (bf16 hi + lo, rotated) -> xop_o; part = scratch of pv_attn_part_floats floats
int pv_mat_attention(pv_cache *c, int layer, int rows, float *part, uint16_t *xop_o, bool merge, hipStream_t s)
{
    const pv_model_config &f = c->m->cfg;
    attn_args a;
    a.st = c->ws.state; a.page_table = c->ws.page_table; a.q_hi = (const uint16_t *)c->ws.q; a.q_lo = a.q_hi + (size_t)c->rows_cap * f.n_q_heads * f.head_dim; a.pool = (const uint16_t *)c->d_pool;
    a.geom = pv_geom(c); a.layer = layer; a.n_q_heads = f.n_q_heads; a.group = f.n_q_heads / f.n_kv_heads;
    a.max_chunks = (c->max_tokens + 127) / 128;        // sizes the partial arrays; the launch sets the chunking in use
    a.chunk_shift = 7; a.chunks = a.max_chunks;
    a.scale = 1.0f / sqrtf((float)f.head_dim); a.block_bytes = (size_t)f.page_tokens * f.head_dim * 2; a.page_bytes = (size_t)(2 * f.n_kv_heads) * a.block_bytes;
    a.part_o = part;
    a.part_ml = part + (size_t)f.n_kv_heads * c->units_cap * a.max_chunks * 32 * f.head_dim;
    a.xop_o = xop_o; a.n_pages = c->n_pages; a.rows = rows; a.batched = c->blk_units != 0;
    const bool nb1 = pv_packs_rows(c->m, rows);
    switch (f.head_dim) {
    case 32: return nb1 ? launch<1, 32>(c, a, rows, merge, s) : launch<2, 32>(c, a, rows, merge, s);
    case 64: return nb1 ? launch<1, 64>(c, a, rows, merge, s) : launch<2, 64>(c, a, rows, merge, s);
    case 128: return nb1 ? launch<1, 128>(c, a, rows, merge, s) : launch<2, 128>(c, a, rows, merge, s);
    default: pv_set_error("matrix path: unsupported head_dim %d", f.head_dim); return PV_EINVAL;
    }
}
