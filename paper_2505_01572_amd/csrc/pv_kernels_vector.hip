// Vector-ALU kernel family: row-major weights of any storage type, fp32 arithmetic.
// This is the path of fp32 models (the tiny parity configuration) and a second, structurally
// different GPU implementation that the matrix-core path can be cross-checked against.
// Every reduction has a fixed order, so repeated runs give identical bits.
#include <algorithm>
#include <type_traits>
#include "pv_kernels_common.h"

__device__ inline float wave_sum(float v) { return over_wave(v, op_add); }

// The totals over the wave of N values (1, 4, 8 or 16); lane l is left with that of value l / (64 / N).  Two values share a register from the first exchange on, so 16 of them take some 50
// vector instructions (six shuffles through LDS each before: 96, in chains of some 120 cycles a link).
template <int N> __device__ inline float fold(const float (&v)[N], int lane)
{
    static_assert(N == 1 || N == 4 || N == 8 || N == 16, "");
    auto both = [](const auto r) { return __uint_as_float(r[0]) + __uint_as_float(r[1]); };
    auto two32 = [&](float a, float b) { return both(__builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false)); };
    auto two16 = [&](float a, float b) { return both(__builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false)); };
    auto select = [](bool c, float x, float y) { asm("" : "+v"(x), "+v"(y)); return c ? x : y; };      // (or the compiler makes an indexed load of it, from LDS)
#define PV_PLUS_DPP(A, CTRL) ((A) + __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(A), CTRL, 0xF, 0xF, true)))      // row_ror:8 0x128, row_half_mirror 0x141, quad_perm [1,0,3,2] 0xB1 and [2,3,0,1] 0x4E
    float a[N < 4 ? 1 : N / 2];
    if constexpr (N == 1) a[0] = two16(two32(v[0], v[0]), two32(v[0], v[0]));
    else {
#pragma unroll
        for (int i = 0; i < N / 2; ++i) a[i] = two32(v[i], v[i + N / 2]);
#pragma unroll
        for (int i = 0; i < N / 4; ++i) a[i] = two16(a[i], a[i + N / 4]);
    }
#pragma unroll
    for (int i = 0; i < (N < 4 ? 1 : N / 4); ++i) a[i] = PV_PLUS_DPP(a[i], 0x128);
    if constexpr (N >= 8) {
#pragma unroll
        for (int i = 0; i < N / 8; ++i) a[i] = select(lane & 8, a[i + N / 8], a[i]);
    }
#pragma unroll
    for (int i = 0; i < (N < 8 ? 1 : N / 8); ++i) a[i] = PV_PLUS_DPP(a[i], 0x141);
    if constexpr (N == 16) a[0] = select(lane & 4, a[1], a[0]);
    a[0] = PV_PLUS_DPP(a[0], 0xB1);
    return PV_PLUS_DPP(a[0], 0x4E);
#undef PV_PLUS_DPP
}
// which value that is, and whether the lane is the first one that has it
template <int N> __device__ inline int fold_row(int lane) { return lane / (64 / N); }
template <int N> __device__ inline bool fold_first(int lane) { return lane % (64 / N) == 0; }

// four consecutive stored elements
__device__ inline float4 ld4(const float *p, size_t i) { return *(const float4 *)(p + i); }
__device__ inline float4 ld4(const uint16_t *p, size_t i)
{
    const uint2 v = *(const uint2 *)(p + i);
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xFFFF0000u));
}

// ---- reductions over a workgroup of four waves, fixed order; red: 4 floats of LDS ----
__device__ inline float block_sum(float v, float *red)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return v;
}

__device__ inline float block_max(float v, float *red)
{
    v = over_wave(v, op_max);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    return v;
}

// The small models of this path are bound by launches and memory round trips, not bytes: a step of the tiny
// configuration took 158 us in 28 kernels of 2..5 us (attention 27 us), with some 4 us between dependent ones.
// (now 70 us in 13, 16 rows 80, 64 rows 96; before the totals stayed on the vector ALU, the loads of a row went out at once and more than 16 rows came in one launch 79, 125 and 375).  RMSNorm, the rotary embedding and the page writes, SwiGLU and the vocabulary arg-max ride in the
// projections: a wave that multiplies a weight row with the input rows passes over the whole rows
// anyway and adds up their squares beside it (the norm's scale commutes with the dot product).

// Pieces of 256 features whose loads go out together: one trip to memory for rows of up to 1024 features where the registers hold that (688 features were three)
template <int G> constexpr int pieces() { return G <= 4 ? 4 : G <= 8 ? 2 : 1; }

// Dot products of G input rows x (times the gain) with M weight rows, and the rows' sums of squares, over one wavefront: of row
// fold_row<G>(lane) on return.
template <typename ST, int G, int M>
__device__ inline void norm_dots(const ST *const (&w)[M], const ST *gain, const float *x, int K, int lane, float (&dot)[M], float &sq)
{
    constexpr int U = pieces<G>();
    float acc[M][G], ss[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        ss[g] = 0.f;
#pragma unroll
        for (int m = 0; m < M; ++m) acc[m][g] = 0.f;
    }
    for (int k0 = lane * 4; k0 < K; k0 += 256 * U) {
        float4 wv[U][M], gn[U], v[U][G];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + 256 * u;
            if (u == 0 || k < K) {
                gn[u] = ld4(gain, k);
#pragma unroll
                for (int m = 0; m < M; ++m) wv[u][m] = ld4(w[m], k);
#pragma unroll
                for (int g = 0; g < G; ++g) v[u][g] = *(const float4 *)(x + (size_t)g * K + k);
            }
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u > 0 && k0 + 256 * u >= K) break;
#pragma unroll
            for (int m = 0; m < M; ++m) wv[u][m] = make_float4(wv[u][m].x * gn[u].x, wv[u][m].y * gn[u].y, wv[u][m].z * gn[u].z, wv[u][m].w * gn[u].w);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float4 y = v[u][g];
                ss[g] += (y.x * y.x + y.y * y.y) + (y.z * y.z + y.w * y.w);
#pragma unroll
                for (int m = 0; m < M; ++m) acc[m][g] += y.x * wv[u][m].x + y.y * wv[u][m].y + y.z * wv[u][m].z + y.w * wv[u][m].w;
            }
        }
    }
    sq = fold<G>(ss, lane);
#pragma unroll
    for (int m = 0; m < M; ++m) dot[m] = fold<G>(acc[m], lane);
}

struct vec_norm { const void *gain; const float *x; int K, rows; float eps; };       // rows: of the whole block; a workgroup takes G of them, from G * blockIdx.y on (the buffers hold whole groups of 16)


// RMSNorm + q, k, v projections + rotary embedding + append to the pages.  One wavefront per pair of outputs (i, i + head_dim / 2)
// of a head; the first lane that has a row's totals finishes it.  K page block: [token][head_dim]; V: [head_dim][token].
template <typename ST, int G>
__global__ void __launch_bounds__(256)
k_vec_qkv(const vec_norm a, const ST *Wq, const ST *Wk, const ST *Wv, const pv_dev_state *st, const int32_t *page_table, const float2 *rope,
          float *q, ST *pool, pv_kv_geom g, int layer, int n_q_heads)
{
    const int lane = threadIdx.x & 63, hd = g.head_dim, half = hd >> 1;
    const int unit = blockIdx.x * 4 + (threadIdx.x >> 6), h = unit / half, i = unit - h * half;       // head (q heads, then k, then v), pair
    if (h >= n_q_heads + 2 * g.n_kv_heads) return;
    const int kind = h < n_q_heads ? 0 : h < n_q_heads + g.n_kv_heads ? 1 : 2, hh = kind == 0 ? h : kind == 1 ? h - n_q_heads : h - n_q_heads - g.n_kv_heads;
    const ST *W = (kind == 0 ? Wq : kind == 1 ? Wk : Wv) + ((size_t)hh * hd + i) * a.K;
    const ST *const w[2] = {W, W + (size_t)half * a.K};
    const int row0 = blockIdx.y * G, j = row0 + fold_row<G>(lane);
    const bool mine = fold_first<G>(lane) && j < a.rows;
    int pos = 0, phys = 0;
    float2 cs = make_float2(1.f, 0.f);
    if (mine) {                               // on their way while the dot products are taken
        pos = st->len + j;
        if (kind != 0) phys = page_table[pos >> g.page_shift];
        if (kind != 2) cs = rope[(size_t)j * half + i];
    }
    float dot[2], sq;
    norm_dots<ST, G, 2>(w, (const ST *)a.gain, a.x + (size_t)row0 * a.K, a.K, lane, dot, sq);
    if (!mine) return;
    const float r = 1.0f / sqrtf(sq / (float)a.K + a.eps);
    const float u = dot[0] * r, v = dot[1] * r;
    const float ru = u * cs.x - v * cs.y, rv = v * cs.x + u * cs.y;
    const int tok = pos & (g.page_tokens - 1);
    if (kind == 0) {
        float *o = q + ((size_t)j * n_q_heads + hh) * hd;
        o[i] = ru; o[i + half] = rv;
    } else if (kind == 1) {
        ST *kb = pool + pv_kv_block(g, layer, phys, hh, 0);
        pv_st(kb, pv_k_off(g, tok, i), ru); pv_st(kb, pv_k_off(g, tok, i + half), rv);
    } else {
        ST *vb = pool + pv_kv_block(g, layer, phys, hh, 1);
        pv_st(vb, pv_v_off(g, tok, i), u); pv_st(vb, pv_v_off(g, tok, i + half), v);
    }
}

// RMSNorm + gate and up projections + SwiGLU.  One wavefront per feature.
template <typename ST, int G>
__global__ void __launch_bounds__(256)
k_vec_gateup(const vec_norm a, const ST *Wg, const ST *Wu, float *act, int F)
{
    const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= F) return;
    const ST *const w[2] = {Wg + (size_t)n * a.K, Wu + (size_t)n * a.K};
    float dot[2], sq;
    const int row0 = blockIdx.y * G, row = row0 + fold_row<G>(lane);
    norm_dots<ST, G, 2>(w, (const ST *)a.gain, a.x + (size_t)row0 * a.K, a.K, lane, dot, sq);
    if (!fold_first<G>(lane) || row >= a.rows) return;
    const float r = 1.0f / sqrtf(sq / (float)a.K + a.eps), z = dot[0] * r;
    act[(size_t)row * F + n] = z / (1.0f + expf(-z)) * (dot[1] * r);
}

// Final RMSNorm + vocabulary projection; a workgroup takes the outputs 4 b + wave, 4 (b + gridDim.x) + wave, ... and leaves
// the best of each row (value descending, index ascending; NaN counts as -inf) as a candidate for k_finish.
template <typename ST, int G>
__global__ void __launch_bounds__(256)
k_vec_head(const vec_norm a, const ST *W, float *logits, int N, float *cand_val, int32_t *cand_idx)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row0 = blockIdx.y * G, in = fold_row<G>(lane), row = row0 + in;
    const bool mine = fold_first<G>(lane) && row < a.rows;
    float bv = -INFINITY; int bi = 0x7fffffff;
    for (int n = blockIdx.x * 4 + wave; n < N; n += gridDim.x * 4) {
        const ST *const w[1] = {W + (size_t)n * a.K};
        float dot[1], sq;
        norm_dots<ST, G, 1>(w, (const ST *)a.gain, a.x + (size_t)row0 * a.K, a.K, lane, dot, sq);
        if (mine) {
            const float r = 1.0f / sqrtf(sq / (float)a.K + a.eps);
            float v = dot[0] * r;
            logits[(size_t)row * N + n] = v;
            v = (v == v) ? v : -INFINITY;
            if (v > bv || (v == bv && n < bi)) { bv = v; bi = n; }
        }
    }
    __shared__ float sv[4][16];
    __shared__ int si[4][16];
    if (fold_first<G>(lane)) { sv[wave][in] = bv; si[wave][in] = bi; }
    __syncthreads();
    if ((int)threadIdx.x < min(G, a.rows - row0)) {
        bv = sv[0][threadIdx.x]; bi = si[0][threadIdx.x];
        for (int w = 1; w < 4; ++w) {
            const float v = sv[w][threadIdx.x]; const int i = si[w][threadIdx.x];
            if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
        }
        const size_t at = (size_t)(row0 + threadIdx.x) * gridDim.x + blockIdx.x;
        cand_val[at] = bv; cand_idx[at] = bi;
    }
}

// y[g][n] = res[g][n] + sum_k x[g][k] * W[n][k]   for g < G rows; one wavefront per n.
// K must be a multiple of 4.  Rows >= `rows` are computed from padding and not stored.
template <typename ST, int G>
__global__ void __launch_bounds__(256)
k_linear(const ST *W, const float *x, const float *res, float *y, int N, int K, int rows)
{
    const int lane = threadIdx.x & 63;
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= N) return;
    const ST *w = W + (size_t)n * K;
    constexpr int U = pieces<G>();
    const int row0 = blockIdx.y * G, row = row0 + fold_row<G>(lane);
    x += (size_t)row0 * K;
    const bool mine = fold_first<G>(lane) && row < rows;
    float before = 0.f;
    if (mine) before = res[(size_t)row * N + n];       // (on its way while the dot products are taken)
    float acc[G];
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = 0.f;
    for (int k0 = lane * 4; k0 < K; k0 += 256 * U) {
        float4 wv[U], v[U][G];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + 256 * u;
            if (u == 0 || k < K) {
                wv[u] = ld4(w, k);
#pragma unroll
                for (int g = 0; g < G; ++g) v[u][g] = *(const float4 *)(x + (size_t)g * K + k);
            }
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u > 0 && k0 + 256 * u >= K) break;
#pragma unroll
            for (int g = 0; g < G; ++g) acc[g] += v[u][g].x * wv[u].x + v[u][g].y * wv[u].y + v[u][g].z * wv[u].z + v[u][g].w * wv[u].w;
        }
    }
    const float total = fold<G>(acc, lane);
    if (mine) y[(size_t)row * N + n] = before + total;
}

// Causal attention for one (query head, row): keys 0 .. len+j, 128 at a time, streaming softmax.  K/V come from the paged pool.  Bound by latency: so the pages of 1024 keys
// are looked up at once, a pass has all its keys and values in flight together (four lanes share a key, 16 bytes a load; along a
// value row 4 tokens a load, split over 256 / HD groups), and it takes one barrier: behind the scores, whose maximum, weights and sum every wave works out for itself.
// 104 keys, four heads of 64: 9.0 -> 5.2 us.  Passes of 1024 keys (k_attention_any) are behind at every length: a step of two layers with 4 rows and 8 heads of 32 / 64 / 128, us,
// 30 keys 79 / 81 / 85 -> 76 / 77 / 83, 1000 keys 124 / 164 / 266 -> 99 / 113 / 144, 8200 keys 554 / 937 / 1673 -> 303 / 416 / 614.
template <typename ST, int HD>
__global__ void __launch_bounds__(256)
k_attention(const pv_dev_state *st, const int32_t *page_table, const float *q, const ST *pool, float *out,
            pv_kv_geom g, int layer, int n_q_heads)
{
    constexpr int NK = HD / 16, GR = 256 / HD, NQ = 32 / GR;        // float4s of a key per lane; groups along the values, and their quads of tokens a pass
    const int j = blockIdx.y, a = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, kvh = a / (n_q_heads / g.n_kv_heads);
    const int key = tid >> 2, sub = tid & 3, grp = tid / HD, e0 = tid % HD;
    __shared__ float sc[2][128], pw[4][128], red[256];
    __shared__ int pg[1024];
    float4 qv[NK];
#pragma unroll
    for (int i = 0; i < NK; ++i) qv[i] = *(const float4 *)(q + ((size_t)j * n_q_heads + a) * HD + 16 * i + 4 * sub);
    const int nkeys = st->len + j + 1, tmask = g.page_tokens - 1;
    const float scale = 1.0f / sqrtf((float)HD);
    float m = -INFINITY, l = 0.f, o = 0.f;
    for (int c0 = 0; c0 < nkeys; c0 += 128) {
        if ((c0 & 1023) == 0) {                        // the next 1024 keys' pages (a page lies in one or more such stretches)
            const int p0 = c0 >> g.page_shift, np = ((min(c0 + 1024, nkeys) - 1) >> g.page_shift) - p0 + 1;
            for (int i = tid; i < np; i += 256) pg[i] = page_table[p0 + i];
            __syncthreads();
        }
        const int pbase = (c0 & ~1023) >> g.page_shift;
        auto block = [&](int t, int which) { return pool + pv_kv_block(g, layer, pg[(t >> g.page_shift) - pbase], kvh, which); };
        float4 kv[2][NK], vv[NQ];
#pragma unroll
        for (int h = 0; h < 2; ++h) {                  // (a key past the end: the last one again, masked)
            const int t = min(c0 + 64 * h + key, nkeys - 1);
            const ST *kb = block(t, 0);
#pragma unroll
            for (int i = 0; i < NK; ++i) kv[h][i] = ld4(kb, pv_k_off(g, t & tmask, 16 * i + 4 * sub));
        }
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int t = c0 + 4 * (grp + GR * i), tc = t < nkeys ? t : c0;
            vv[i] = ld4(block(tc, 1), pv_v_off(g, tc & tmask, e0));
        }
        float *s = sc[(c0 >> 7) & 1];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float d = 0.f;
#pragma unroll
            for (int i = 0; i < NK; ++i) d += (kv[h][i].x * qv[i].x + kv[h][i].y * qv[i].y) + (kv[h][i].z * qv[i].z + kv[h][i].w * qv[i].w);
            d += __shfl_xor(d, 1, 64);
            d += __shfl_xor(d, 2, 64);
            if (sub == 0) s[64 * h + key] = c0 + 64 * h + key < nkeys ? d * scale : -INFINITY;
        }
        __syncthreads();
        const float s0 = s[lane], s1 = s[64 + lane];
        float mn = fmaxf(m, fmaxf(s0, s1));
        mn = over_wave(mn, op_max);
        const float w0 = expf(s0 - mn), w1 = expf(s1 - mn), resc = expf(m - mn);
        pw[wave][lane] = w0; pw[wave][64 + lane] = w1;               // (the wave's own copy: no barrier)
        l = l * resc + wave_sum(w0 + w1);
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int t = 4 * (grp + GR * i);
            const float4 p = *(const float4 *)&pw[wave][t];
            const int left = nkeys - c0 - t;           // tokens past the end: their slots of the page may hold anything
            acc += ((left > 0 ? p.x * vv[i].x : 0.f) + (left > 1 ? p.y * vv[i].y : 0.f)) + ((left > 2 ? p.z * vv[i].z : 0.f) + (left > 3 ? p.w * vv[i].w : 0.f));
        }
        o = o * resc + acc;
        m = mn;
    }
    red[tid] = o;                                      // the groups' sums, added in group order
    __syncthreads();
    if (grp == 0) {
#pragma unroll
        for (int k = 1; k < GR; ++k) o += red[k * HD + e0];
        out[((size_t)j * n_q_heads + a) * HD + e0] = o / l;
    }
}

// The same for other head sizes and for pages of fewer than 4 tokens: streaming softmax over chunks
// of 1024 keys.  K/V come from the paged pool.  The chunk's pages are looked up once, ahead of everything else; four lanes
// share a key's score, and the value sum is split over 256 / head_dim groups of keys (27 -> 8 us at 104 keys: the
// time was a chain of page look-ups and loads, one per key).
template <typename ST>
__global__ void __launch_bounds__(256)
k_attention_any(const pv_dev_state *st, const int32_t *page_table, const float *q, const ST *pool, float *out,
            pv_kv_geom g, int layer, int n_q_heads)
{
    const int j = blockIdx.y, a = blockIdx.x, tid = threadIdx.x;
    const int hd = g.head_dim, kvh = a / (n_q_heads / g.n_kv_heads);
    __shared__ float qs[256], sc[1024], red[256];
    __shared__ int pg[1024];
    const int nkeys = st->len + j + 1;
    if (j >= st->gamma) return;
    if (tid < hd) qs[tid] = q[((size_t)j * n_q_heads + a) * hd + tid];
    const float scale = 1.0f / sqrtf((float)hd);
    int lanes = 1;                                     // threads that go along a value row: head_dim rounded up to a power of two
    while (lanes < hd) lanes <<= 1;
    const int groups = 256 / lanes, grp = tid / lanes, e0 = tid - grp * lanes;
    float m = -INFINITY, l = 0.f, o = 0.f;
    for (int c0 = 0; c0 < nkeys; c0 += 1024) {
        const int cn = min(1024, nkeys - c0), p0 = c0 >> g.page_shift, np = ((c0 + cn - 1) >> g.page_shift) - p0 + 1;
        for (int i = tid; i < np; i += 256) pg[i] = page_table[p0 + i];
        __syncthreads();
        float lm = -INFINITY;
        const int sub = tid & 3;
        for (int t0 = 0; t0 < cn; t0 += 64) {          // 64 keys at a time, four lanes each
            const int t = t0 + (tid >> 2), tc = min(t, cn - 1), p = c0 + tc;
            const ST *kb = pool + pv_kv_block(g, layer, pg[(p >> g.page_shift) - p0], kvh, 0);
            const int tk = p & (g.page_tokens - 1);
            float s = 0.f;
#pragma unroll 8
            for (int e = sub; e < hd; e += 4) s += qs[e] * pv_ld(kb, pv_k_off(g, tk, e));
            s += __shfl_xor(s, 1, 64);
            s += __shfl_xor(s, 2, 64);
            s *= scale;
            if (t < cn) { if (sub == 0) sc[t] = s; lm = fmaxf(lm, s); }
        }
        const float m_new = fmaxf(m, block_max(lm, red));
        float ls = 0.f;
        for (int t = tid; t < cn; t += 256) { const float w = expf(sc[t] - m_new); sc[t] = w; ls += w; }
        const float cs = block_sum(ls, red);          // also orders the sc[] writes before the reads below
        const float resc = expf(m - m_new);
        l = l * resc + cs;
        float acc = 0.f;
        if (e0 < hd) {
#pragma unroll 8
            for (int t = grp; t < cn; t += groups) {
                const int p = c0 + t;
                const ST *vb = pool + pv_kv_block(g, layer, pg[(p >> g.page_shift) - p0], kvh, 1);
                acc += sc[t] * pv_ld(vb, pv_v_off(g, p & (g.page_tokens - 1), e0));
            }
        }
        o = o * resc + acc;
        m = m_new;
        __syncthreads();
    }
    red[tid] = o;                                      // the groups' sums, added in group order
    __syncthreads();
    if (grp == 0 && e0 < hd) {
        for (int k = 1; k < groups; ++k) o += red[k * lanes + e0];
        out[((size_t)j * n_q_heads + a) * hd + e0] = o / l;
    }
}

// ------------------------------- host side ----------------------------------------

// calls f(G, groups) once: G the smallest of 1, 4, 8, 16 that holds the rows, more than 16 as groups of 16 in one launch (one after the other, 40 rows: 147 -> 92 us a step of the tiny configuration)
template <typename F>
static int row_groups(int rows, F f)
{
    if (rows <= 1) f(std::integral_constant<int, 1>(), 1u);
    else if (rows <= 4) f(std::integral_constant<int, 4>(), 1u);
    else if (rows <= 8) f(std::integral_constant<int, 8>(), 1u);
    else f(std::integral_constant<int, 16>(), (unsigned)((rows + 15) / 16));
    PV_HIP(hipGetLastError());
    return PV_OK;
}

template <typename ST>
static int launch_linear(const pv_model *m, const pv_tensor_ref &t, const float *x, const float *res, float *y,
                         int rows, hipStream_t s)
{
    const ST *W = (const ST *)(m->d_weights + t.off);
    const int N = (int)t.rows, K = (int)t.cols;
    return row_groups(rows, [&](auto G, unsigned groups) { k_linear<ST, G.value><<<dim3((unsigned)((N + 3) / 4), groups), 256, 0, s>>>(W, x, res, y, N, K, rows); });
}

template <typename ST>
static int run_block(pv_cache *c, hipStream_t s)
{
    const pv_model *m = c->m;
    const pv_model_config &f = m->cfg;
    const int rows = c->last_rows, rows_pad = (rows + PV_ROW_PAD - 1) / PV_ROW_PAD * PV_ROW_PAD;
    const int d = f.d_model, F = f.ffn_dim, V = f.vocab;
    const pv_kv_geom g = pv_geom(c);
    pv_ws &w = c->ws;
    auto wt = [&](int kind, int l) { return (const ST *)(m->d_weights + pv_tref(m, kind, l).off); };
    auto normed = [&](const ST *gain) { return vec_norm{gain, w.x, d, rows, (float)f.rms_eps}; };
    int rc;
    if ((rc = pv_k_begin(c, rows_pad, s)) != PV_OK) return rc;
    for (int l = 0; l < f.n_layers; ++l) {
        const int units = (f.n_q_heads + 2 * f.n_kv_heads) * (f.head_dim / 2);
        rc = row_groups(rows, [&](auto G, unsigned groups) {
            k_vec_qkv<ST, G.value><<<dim3((units + 3) / 4, groups), 256, 0, s>>>(normed(wt(PV_T_ATTN_NORM, l)), wt(PV_T_WQ, l), wt(PV_T_WK, l), wt(PV_T_WV, l), w.state,
                                                                   w.page_table, w.rope, w.q, (ST *)c->d_pool, g, l, f.n_q_heads);
        });
        if (rc != PV_OK) return rc;
        auto attention = [&](auto k) { k<<<dim3(f.n_q_heads, rows), 256, 0, s>>>(w.state, w.page_table, w.q, (const ST *)c->d_pool, w.attn, g, l, f.n_q_heads); };
        const int hd = f.page_tokens < 4 ? 0 : f.head_dim;            // (k_attention loads 4 tokens of a page at a time)
        if (hd == 64) attention(k_attention<ST, 64>);
        else if (hd == 128) attention(k_attention<ST, 128>);
        else if (hd == 32) attention(k_attention<ST, 32>);
        else attention(k_attention_any<ST>);
        PV_HIP(hipGetLastError());
        if ((rc = launch_linear<ST>(m, pv_tref(m, PV_T_WO, l), w.attn, w.x, w.x, rows, s)) != PV_OK) return rc;
        rc = row_groups(rows, [&](auto G, unsigned groups) {
            k_vec_gateup<ST, G.value><<<dim3((F + 3) / 4, groups), 256, 0, s>>>(normed(wt(PV_T_FFN_NORM, l)), wt(PV_T_WG, l), wt(PV_T_WU, l), w.gate, F);
        });
        if (rc != PV_OK) return rc;
        if ((rc = launch_linear<ST>(m, pv_tref(m, PV_T_WD, l), w.gate, w.x, w.x, rows, s)) != PV_OK) return rc;
    }
    if (c->io->hdr[3] == PV_MODE_PREFILL_MID) return pv_k_finish(c, rows, nullptr, nullptr, 0, s);
    // the candidates ([row][strips]) go where gate and up were
    const int strips = std::min((V + 3) / 4, F);
    rc = row_groups(rows, [&](auto G, unsigned groups) {
        k_vec_head<ST, G.value><<<dim3(strips, groups), 256, 0, s>>>(normed((const ST *)(m->d_weights + m->global[PV_T_FINAL_NORM].off)), (const ST *)(m->d_weights + m->global[PV_T_LM_HEAD].off),
                                                       w.logits, V, w.gate, (int32_t *)w.up);
    });
    if (rc != PV_OK) return rc;
    return pv_k_finish(c, rows, w.gate, (const int32_t *)w.up, strips, s);
}

int pv_vec_run_block(pv_cache *c, hipStream_t s)
{
    return c->m->cfg.dtype == PV_BF16 ? run_block<uint16_t>(c, s) : run_block<float>(c, s);
}
