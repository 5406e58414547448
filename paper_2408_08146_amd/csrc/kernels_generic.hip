// The bookkeeping steps of the draft-then-verify iteration that both model dtypes share, and the small fp32 kernels
// (start of a pass, norm, top-k) beside the fp32 projections and attention.
#include "koala_pass.h"

namespace {

// ------------------------------------------------------------------ first kernel of a pass, fp32
// grid (rows, ceil(width / 256)), 64 threads x 4 columns; the first workgroup of a row writes its metadata as well
__global__ __launch_bounds__(64) void k_pass_in(PassArgs a, const float *E, float *x, int H) {
    const int r = blockIdx.x, W = a.mode == 0 ? H : 2 * H, j = (blockIdx.y * 64 + threadIdx.x) * 4;
    const float *f;
    const size_t t = (size_t)pass_token(a, r, H, f);
    if (j < W) *(float4 *)(x + (size_t)r * W + j) = j < H ? *(const float4 *)(E + t * H + j) : *(const float4 *)(f + j - H);
    if (blockIdx.y == 0) pass_meta(a, r);
}

// ------------------------------------------------------------------ RMSNorm
__global__ __launch_bounds__(256) void k_rmsnorm(const float *x, const float *g, float *out, int H, float eps) {
    __shared__ float red[4];
    const int r = blockIdx.x;
    const float *xr = x + (size_t)r * H;
    float ss = 0.f;
    for (int j = threadIdx.x; j < H; j += 256) { const float v = xr[j]; ss += v * v; }
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float tot = red[0] + red[1] + red[2] + red[3];
    const float inv = 1.0f / sqrtf(tot / (float)H + eps);
    for (int j = threadIdx.x; j < H; j += 256) out[(size_t)r * H + j] = xr[j] * inv * g[j];
}

__global__ void k_resblock(float *x, const float *y, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float v = y[i];
    x[i] += v / (1.0f + __expf(-v));
}

// ------------------------------------------------------------------ top-k of each row (k <= 16)
// Descending value, equal values ordered by ascending index; one workgroup per row.  A thread holds its first TR values in
// registers (rows up to 4096 are read once).
__device__ __forceinline__ bool topk_better(float v, int i, float bv, int bi) {   // index 0x7fffffff: nothing yet
    return i != 0x7fffffff && (bi == 0x7fffffff || v > bv || (v == bv && i < bi));
}
__global__ __launch_bounds__(256) void k_topk(const float *logits, int ld, int V, int k, int32_t *idx, float *val,
                                              ChildFill fill) {
    constexpr int TR = 16;
    __shared__ float bv[2][4];
    __shared__ int bi[2][4];
    __shared__ int chosen[KOALA_TOPK_MAX];
    __shared__ float chosen_val[KOALA_TOPK_MAX];
    const int r = blockIdx.x, tid = threadIdx.x;
    const float *row = logits + (size_t)r * ld;
    float w[TR];
    unsigned taken = 0;
#pragma unroll
    for (int u = 0; u < TR; ++u) w[u] = tid + 256 * u < V ? row[tid + 256 * u] : 0.f;
    for (int it = 0; it < k; ++it) {
        float best = -INFINITY;
        int besti = 0x7fffffff;
#pragma unroll
        for (int u = 0; u < TR; ++u) {
            const int j = tid + 256 * u;
            if (j < V && !((taken >> u) & 1u) && topk_better(w[u], j, best, besti)) { best = w[u]; besti = j; }
        }
        for (int j = tid + 256 * TR; j < V; j += 256) {
            bool was = false;
            for (int c = 0; c < it; ++c) was |= (chosen[c] == j);
            const float v = row[j];
            if (!was && topk_better(v, j, best, besti)) { best = v; besti = j; }
        }
        for (int o = 32; o > 0; o >>= 1) {
            const float v2 = __shfl_xor(best, o);
            const int i2 = __shfl_xor(besti, o);
            if (topk_better(v2, i2, best, besti)) { best = v2; besti = i2; }
        }
        if ((tid & 63) == 0) { bv[it & 1][tid >> 6] = best; bi[it & 1][tid >> 6] = besti; }
        __syncthreads();
        // from the waves' first lanes alone: a not-a-number leaves the lanes of a wave with different winners, and all threads
        // have to agree on which token is taken
        best = bv[it & 1][0];
        besti = bi[it & 1][0];
#pragma unroll
        for (int u = 1; u < 4; ++u)
            if (topk_better(bv[it & 1][u], bi[it & 1][u], best, besti)) { best = bv[it & 1][u]; besti = bi[it & 1][u]; }
        if (besti % 256 == tid && besti < 256 * TR) taken |= 1u << (besti / 256);
        if (tid == 0) {
            chosen[it] = besti;
            chosen_val[it] = best;
            if (idx) idx[(size_t)r * k + it] = besti;
            if (val) val[(size_t)r * k + it] = best;
        }
        if (V > 256 * TR) __syncthreads();   // the next round reads `chosen`
    }
    if (fill.tree_tokens) {
        __syncthreads();
        fill_children(fill, r, chosen, chosen_val);
    }
}

// ------------------------------------------------------------------ draft bookkeeping
__global__ void k_gather_last(const float *x, float *dst, size_t dst_stride, int m, int H) {
    const int b = blockIdx.x;
    for (int j = threadIdx.x; j < H; j += blockDim.x)
        dst[(size_t)b * dst_stride + j] = x[((size_t)b * m + m - 1) * H + j];
}

__global__ void k_store_fhat(const float *x, float *fhat, const int32_t *level_nodes, int n_level, int T, int H) {
    const int r = blockIdx.x, b = r / n_level, u = level_nodes[r % n_level];
    for (int j = threadIdx.x; j < H; j += blockDim.x)
        fhat[((size_t)b * T + u) * H + j] = x[(size_t)r * H + j];
}

__global__ void k_set_root(const int32_t *tok_in, int m, int32_t *tree_tokens, float *scores, int batch, int T) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= batch) return;
    tree_tokens[b * T] = tok_in[b * m + m - 1];
    if (scores) scores[b * T] = 0.f;
}

// ------------------------------------------------------------------ acceptance
// The greedy walk of one sequence, by a wave that holds one node a lane (its parent, token and greedy token): lane j gets
// the j-th node of the path.  Returns the accepted length.  A node's next is the lowest-numbered child whose token is its
// greedy token, found by a ballot.
__device__ __forceinline__ int accept_walk(int parent, int tok, int greedy, int T, int D, int &path, int &last) {
    const int l = threadIdx.x & 63;
    int cur = 0, a = 0;
    path = l == 0 ? 0 : -1;
    while (a < D) {
        const int g = __builtin_amdgcn_readlane(greedy, cur);
        const unsigned long long hit = __ballot(l < T && parent == cur && tok == g);
        if (!hit) break;
        cur = __ffsll((long long)hit) - 1;
        ++a;
        if (l == a) path = cur;
    }
    last = cur;
    return a;
}
__device__ __forceinline__ int accept_load(const TreeTables &tt, int T, int D, int b, const int32_t *tree_tokens,
                                           const int32_t *greedy, int &path, int &next) {
    const int l = threadIdx.x & 63;
    const int parent = l < T ? tt.parent[l] : -2;
    const int tok = l < T ? tree_tokens[(size_t)b * T + l] : 0, g = l < T ? greedy[(size_t)b * T + l] : 0;
    int last;
    const int a = accept_walk(parent, tok, g, T, D, path, last);
    next = __builtin_amdgcn_readlane(g, last);
    return a;
}
// path of at most D + 1 <= 64 entries, -1 past the accepted ones
__device__ __forceinline__ void accept_store(int b, int D, int a, int path, int next, int32_t *accept_len, int32_t *accept_path,
                                             int32_t *next_token) {
    const int l = threadIdx.x & 63;
    if (l <= D) accept_path[(size_t)b * (D + 1) + l] = path;
    if (l == 0) {
        accept_len[b] = a;
        next_token[b] = next;
    }
}

__global__ __launch_bounds__(64) void k_accept(TreeTables tt, int T, int D, const int32_t *tree_tokens, const int32_t *greedy,
                                               int32_t *accept_len, int32_t *accept_path, int32_t *next_token) {
    int path, next;
    const int a = accept_load(tt, T, D, blockIdx.x, tree_tokens, greedy, path, next);
    accept_store(blockIdx.x, D, a, path, next, accept_len, accept_path, next_token);
}

// The walk (every wave for itself) and the move of the accepted nodes' rows to slots C .. C + a: path node j is number j or
// higher, so no slot is written before it has been read, and the rows are fetched four at a time.
// grid (layers, batch, heads), head_dim threads
template <typename CT>
__global__ void k_accept_commit(TreeTables tt, int T, int D, const int32_t *tree_tokens, const int32_t *greedy, CT *kc, CT *vc,
                                const int32_t *ctx_len, int32_t *accept_len, int32_t *accept_path, int32_t *next_token,
                                int max_batch, int n_heads, int cap, int DH) {
    const int l = blockIdx.x, b = blockIdx.y, h = blockIdx.z, d = threadIdx.x;
    int path, next;
    const int C = ctx_len[b], a = accept_load(tt, T, D, b, tree_tokens, greedy, path, next);
    if (l == 0 && h == 0 && d < 64) accept_store(b, D, a, path, next, accept_len, accept_path, next_token);
    const size_t base = ((((size_t)l * max_batch + b) * n_heads + h) * cap) * DH + d;
    for (int j0 = 1; j0 <= a; j0 += 4) {
        CT k[4], v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int node = __builtin_amdgcn_readlane(path, min(j0 + q, a));
            k[q] = kc[base + (size_t)(C + node) * DH];
            v[q] = vc[base + (size_t)(C + node) * DH];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (j0 + q > a) continue;
            kc[base + (size_t)(C + j0 + q) * DH] = k[q];
            vc[base + (size_t)(C + j0 + q) * DH] = v[q];
        }
    }
}

// Move the accepted nodes' rows to slots C..C+a.  Each thread owns one element column and
// walks the path in order, so a slot is always read before a later step overwrites it.
template <typename CT>
__global__ void k_kv_commit(CT *kc, CT *vc, const int32_t *ctx_len, const int32_t *accept_len,
                            const int32_t *accept_path, int D, int max_batch, int n_heads, int cap, int DH) {
    const int l = blockIdx.x, b = blockIdx.y, h = blockIdx.z, d = threadIdx.x;
    const int C = ctx_len[b], a = accept_len[b];
    const size_t base = ((((size_t)l * max_batch + b) * n_heads + h) * cap) * DH + d;
    for (int j = 1; j <= a; ++j) {
        const int node = accept_path[(size_t)b * (D + 1) + j];
        if (node == j) continue;
        kc[base + (size_t)(C + j) * DH] = kc[base + (size_t)(C + node) * DH];
        vc[base + (size_t)(C + j) * DH] = vc[base + (size_t)(C + node) * DH];
    }
}

__global__ void k_advance(int32_t *ctx_len, const int32_t *accept_len, int batch) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < batch) ctx_len[b] += accept_len[b] + 1;
}

// Inputs of the next draft step from one accepted path (one sequence): block i <= a copies the
// feature of path node i to row i and sets tok_next[i] to the token that follows it (the next
// path node's token, or the target's own token after the last accepted node); the same tokens are
// appended to out_tokens[n_done + i] while that index is below max_new.  grid D+1 blocks.
__global__ void k_gen_next(const float *feat_out, const int32_t *tree_tokens, const int32_t *accept_len,
                           const int32_t *accept_path, const int32_t *next_token, int T, int H, float *feat_next,
                           int32_t *tok_next, int32_t *out_tokens, int n_done, int max_new) {
    const int i = blockIdx.x, a = accept_len[0];
    if (i > a) return;
    const int node = accept_path[i];
    if (node < 0 || node >= T) return;   // never for a path the accept scan wrote
    const float *src = feat_out + (size_t)node * H;
    float *dst = feat_next + (size_t)i * H;
    for (int j = threadIdx.x; j < H; j += blockDim.x) dst[j] = src[j];
    if (threadIdx.x == 0) {
        int32_t tok = next_token[0];
        if (i < a) {
            const int nx = accept_path[i + 1];
            if (nx >= 0 && nx < T) tok = tree_tokens[nx];
        }
        tok_next[i] = tok;
        if (n_done + i < max_new) out_tokens[n_done + i] = tok;
    }
}

// Streaming read of n 16-byte words (measurement aid): every thread xors what it reads; the result is
// stored only to keep the loads alive.
typedef __attribute__((ext_vector_type(4))) unsigned int rd_u32x4;
__global__ __launch_bounds__(256) void k_stream_read(const rd_u32x4 *src, size_t n, unsigned *sink) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    rd_u32x4 acc = {0u, 0u, 0u, 0u};
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n; i += 4 * stride) {
        const rd_u32x4 a = __builtin_nontemporal_load(src + i), b = __builtin_nontemporal_load(src + i + stride);
        const rd_u32x4 c = __builtin_nontemporal_load(src + i + 2 * stride);
        const rd_u32x4 d = __builtin_nontemporal_load(src + i + 3 * stride);
        acc ^= a ^ b ^ c ^ d;
    }
    for (; i < n; i += stride) acc ^= __builtin_nontemporal_load(src + i);
    const unsigned r = acc.x ^ acc.y ^ acc.z ^ acc.w;
    if (r == 0x9e3779b9u) sink[0] = r;
}

inline int cdiv(size_t a, size_t b) { return (int)((a + b - 1) / b); }

}  // namespace

// =====================================================================================================
namespace kg {

PassArgs pass_args(const koala_ctx *c, int mode, int rows_per_seq, int m, int d) {
    PassArgs a{};
    a.mode = mode;
    a.ctx_len = c->kv.ctx_len;
    a.tt = c->tt;
    a.meta = c->meta;
    a.T = c->T; a.rows_per_seq = rows_per_seq; a.m = m; a.d = d; a.n_exp = c->n_exp;
    a.half = c->shape.head_dim / 2;
    a.inv_freq = (const double *)(c->ws);  // first table of the workspace
    return a;
}

void pass_in(hipStream_t s, const PassArgs &a, const void *E, float *x, int rows, int H) {
    k_pass_in<<<dim3(rows, ((a.mode == 0 ? H : 2 * H) + 255) / 256), 64, 0, s>>>(a, (const float *)E, x, H);
}

void rmsnorm(hipStream_t s, const float *x, const void *g, float *out, int rows, int H, float eps) {
    k_rmsnorm<<<rows, 256, 0, s>>>(x, (const float *)g, out, H, eps);
}

void resblock_update(hipStream_t s, float *x, const float *y, int n) {
    k_resblock<<<cdiv(n, 256), 256, 0, s>>>(x, y, (size_t)n);
}

void topk_rows(hipStream_t s, const float *logits, int ld, int rows, int V, int k, int32_t *idx, float *val,
               const ChildFill &fill) {
    k_topk<<<rows, 256, 0, s>>>(logits, ld, V, k, idx, val, fill);
}

void store_fhat(hipStream_t s, const float *x, float *fhat, const int32_t *level_nodes, int batch, int n_level,
                int T, int H) {
    k_store_fhat<<<batch * n_level, 256, 0, s>>>(x, fhat, level_nodes, n_level, T, H);
}

void set_root(hipStream_t s, const int32_t *tok_in, int m, int32_t *tree_tokens, float *scores, int batch, int T) {
    k_set_root<<<cdiv(batch, 64), 64, 0, s>>>(tok_in, m, tree_tokens, scores, batch, T);
}

void accept_scan(hipStream_t s, const TreeTables &tt, int T, int D, const int32_t *tree_tokens,
                 const int32_t *greedy, int32_t *accept_len, int32_t *accept_path, int32_t *next_token, int batch) {
    k_accept<<<batch, 64, 0, s>>>(tt, T, D, tree_tokens, greedy, accept_len, accept_path, next_token);
}

void accept_commit(hipStream_t s, bool bf16, const TreeTables &tt, int T, int D, const int32_t *tree_tokens, const int32_t *greedy,
                   void *kcache, void *vcache, const int32_t *ctx_len, int32_t *accept_len, int32_t *accept_path,
                   int32_t *next_token, int n_layers, int max_batch, int batch, int n_heads, int capacity, int head_dim) {
    const dim3 grid(n_layers, batch, n_heads);
    if (bf16)
        k_accept_commit<bf16_t><<<grid, head_dim, 0, s>>>(tt, T, D, tree_tokens, greedy, (bf16_t *)kcache, (bf16_t *)vcache,
                                                          ctx_len, accept_len, accept_path, next_token, max_batch, n_heads,
                                                          capacity, head_dim);
    else
        k_accept_commit<float><<<grid, head_dim, 0, s>>>(tt, T, D, tree_tokens, greedy, (float *)kcache, (float *)vcache,
                                                         ctx_len, accept_len, accept_path, next_token, max_batch, n_heads,
                                                         capacity, head_dim);
}

void kv_commit(hipStream_t s, bool bf16, void *kcache, void *vcache, const int32_t *ctx_len,
               const int32_t *accept_len, const int32_t *accept_path, int D, int n_layers, int max_batch,
               int batch, int n_heads, int capacity, int head_dim) {
    const dim3 grid(n_layers, batch, n_heads);
    if (bf16)
        k_kv_commit<bf16_t><<<grid, head_dim, 0, s>>>((bf16_t *)kcache, (bf16_t *)vcache, ctx_len, accept_len,
                                                      accept_path, D, max_batch, n_heads, capacity, head_dim);
    else
        k_kv_commit<float><<<grid, head_dim, 0, s>>>((float *)kcache, (float *)vcache, ctx_len, accept_len,
                                                     accept_path, D, max_batch, n_heads, capacity, head_dim);
}

void advance_ctx(hipStream_t s, int32_t *ctx_len, const int32_t *accept_len, int batch) {
    k_advance<<<cdiv(batch, 64), 64, 0, s>>>(ctx_len, accept_len, batch);
}

// dst[b * dst_stride + j] = x[(b*m + m-1) * H + j]: the newest row of every sequence
void gather_last_rows(hipStream_t s, const float *x, float *dst, size_t dst_stride, int batch, int m, int H) {
    k_gather_last<<<batch, 256, 0, s>>>(x, dst, dst_stride, m, H);
}

void stream_read(hipStream_t s, const void *src, size_t bytes, unsigned *sink) {
    k_stream_read<<<2048, 256, 0, s>>>((const rd_u32x4 *)src, bytes / 16, sink);
}

void gen_next(hipStream_t s, const float *feat_out, const int32_t *tree_tokens, const int32_t *accept_len,
              const int32_t *accept_path, const int32_t *next_token, int T, int D, int H, float *feat_next,
              int32_t *tok_next, int32_t *out_tokens, int n_done, int max_new) {
    k_gen_next<<<D + 1, 256, 0, s>>>(feat_out, tree_tokens, accept_len, accept_path, next_token, T, H, feat_next,
                                     tok_next, out_tokens, n_done, max_new);
}

}  // namespace kg
