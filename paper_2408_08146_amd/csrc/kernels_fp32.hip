// fp32 model path: projections and tree attention on the fp32 matrix pipe (16x16x4 MFMA, fp32 operands and sums).
//
// A call of the fp32 configuration (hidden 256) moves little; what it costs is its launches and the chain of memory round
// trips inside each.  A decoder layer is five launches, each of which requests everything it needs before its first wait:
//   QKV projection with RMSNorm in front and rotary embedding and cache append behind, attention, O projection added to
//   the residual stream, gate/up projection with RMSNorm in front and SwiGLU behind, down projection added to the stream
// (ten launches with norm, rotary embedding, split merge and SwiGLU as kernels of their own, which ran one output column
// per wave on the vector unit and attention rows by the thread: iteration of the 4-layer model 515 us, so 224 us).
//
// Operand layout: the contraction order is free as long as both operands use the same, so lane (i = l%16, g = l/16) loads
// four consecutive k, 16 bytes, and element e of every lane forms the MFMA's k step {4g + e}: sixteen k per load.
#include "koala_internal.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

enum { F32_STORE = 0, F32_ADD = 1, F32_SWIGLU = 2, F32_QKV = 3 };
constexpr int NW = 8;   // waves per workgroup

struct F32Epi {
    const float *gain;   // RMSNorm of the input rows (nullptr: none): x * gain goes in, the row scale is applied to the sums
    float eps;
    float *Y;            // STORE, ADD: [M][ldy]; SWIGLU: [M][N/2]
    int ldy;
    RowMeta meta;        // QKV
    float *qrot, *kc, *vc;
    int H, n_heads, DH, cap;
};

// Y = epilogue(X[M,K] W[N,K]^T).  One workgroup owns U groups of 16 output columns (QKV: the two halves of a rotary group,
// dimensions 16t.. and 16t.. + head_dim/2 of one head) and MT * 16 rows; its waves take the 16-k groups in turn, two
// in flight each, and their sums meet in LDS in wave order.  grid (column groups, row blocks).
template <int U, int MT, int EPI>
__global__ __launch_bounds__(64 * NW) void k_gemm_f32(const float *__restrict__ W, const float *__restrict__ X, int ldx, int M,
                                                      int N, int K, F32Epi e) {
    __shared__ f32x4 red[NW][U][MT][64];
    __shared__ float sq[NW][MT * 16];
    const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, li = l & 15, lg = l >> 4;
    const int m0 = blockIdx.y * MT * 16;
    int n0[U], which = 0, head = 0, t = 0;
    if (EPI == F32_QKV) {
        const int gh = e.DH / 32, gm = e.H / 32;
        which = blockIdx.x / gm;
        head = blockIdx.x % gm / gh;
        t = blockIdx.x % gh;
        n0[0] = which * e.H + head * e.DH + 16 * t;
        n0[U - 1] = n0[0] + e.DH / 2;
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) n0[u] = (blockIdx.x * U + u) * 16;
    }
    const float *w[U], *x[MT];
#pragma unroll
    for (int u = 0; u < U; ++u) w[u] = W + (size_t)min(n0[u] + li, N - 1) * K + 4 * lg;
#pragma unroll
    for (int m = 0; m < MT; ++m) x[m] = X + (size_t)min(m0 + m * 16 + li, M - 1) * ldx + 4 * lg;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    // one accumulator per k step of a load, added pairwise at the end: shorter chains, both of waiting and of rounding
    f32x4 acc[4][U][MT];
    float ss[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        ss[m] = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q][u][m] = zero;
    }
    constexpr int PF = 2;
    f32x4 wr[PF][U], xr[PF][MT], gr[PF];
    auto load = [&](int k, int p) {   // K is a multiple of four: a lane's four k are all inside or all past the end
        const bool in = k + 4 * lg < K;
#pragma unroll
        for (int u = 0; u < U; ++u) wr[p][u] = in ? *(const f32x4 *)(w[u] + k) : zero;
#pragma unroll
        for (int m = 0; m < MT; ++m) xr[p][m] = in ? *(const f32x4 *)(x[m] + k) : zero;
        if (e.gain) gr[p] = in ? *(const f32x4 *)(e.gain + k + 4 * lg) : zero;
    };
    const int step = 16 * NW;
    int k = 16 * wave;
#pragma unroll
    for (int p = 0; p < PF; ++p)
        if (k + p * step < K) load(k + p * step, p);
    for (; k < K; k += PF * step) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            if (k + p * step >= K) continue;
            f32x4 wv[U], xv[MT];
#pragma unroll
            for (int u = 0; u < U; ++u) wv[u] = wr[p][u];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                xv[m] = xr[p][m];
                if (e.gain) {
                    ss[m] += xv[m][0] * xv[m][0] + xv[m][1] * xv[m][1] + xv[m][2] * xv[m][2] + xv[m][3] * xv[m][3];
                    xv[m] *= gr[p];
                }
            }
            if (k + (p + PF) * step < K) load(k + (p + PF) * step, p);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[q][u][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[u][q], xv[m][q], acc[q][u][m], 0, 0, 0);
        }
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) {
#pragma unroll
        for (int u = 0; u < U; ++u) red[wave][u][m][l] = (acc[0][u][m] + acc[1][u][m]) + (acc[2][u][m] + acc[3][u][m]);
        if (e.gain) {
            ss[m] += __shfl_xor(ss[m], 16);
            ss[m] += __shfl_xor(ss[m], 32);
            if (lg == 0) sq[wave][m * 16 + li] = ss[m];
        }
    }
    __syncthreads();
    // wave m finishes row tile m: lane (li, lg) has columns n0 + 4 lg .. + 3 of row m0 + 16 m + li
    if (wave >= MT) return;
    const int m = wave, row = m0 + m * 16 + li;
    f32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        f32x4 t[NW];
#pragma unroll
        for (int q = 0; q < NW; ++q) t[q] = red[q][u][m][l];
        v[u] = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    }
    if (e.gain) {
        float tot = 0.f;
#pragma unroll
        for (int q = 0; q < NW; ++q) tot += sq[q][m * 16 + li];
        const float inv = 1.0f / sqrtf(tot / (float)K + e.eps);
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] *= inv;
    }
    if (row >= M) return;
    if (EPI == F32_QKV) {
        const int half = e.DH / 2, d = 16 * t + 4 * lg;
        const f32x4 a = v[0], b = v[U - 1];
        const size_t o = which == 0 ? (size_t)row * e.H + head * e.DH
                                    : (((size_t)e.meta.row_b[row] * e.n_heads + head) * e.cap + e.meta.row_slot[row]) * e.DH;
        float *dst = (which == 0 ? e.qrot : which == 1 ? e.kc : e.vc) + o + d;
        if (which == 2) {
            *(f32x4 *)dst = a;
            *(f32x4 *)(dst + half) = b;
        } else {
            const f32x4 c = *(const f32x4 *)(e.meta.rope_cos + (size_t)row * half + d);
            const f32x4 s = *(const f32x4 *)(e.meta.rope_sin + (size_t)row * half + d);
            *(f32x4 *)dst = a * c - b * s;
            *(f32x4 *)(dst + half) = b * c + a * s;
        }
        return;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int n = n0[u] + 4 * lg;
        if (EPI == F32_SWIGLU) {   // columns interleave gate and up; N is a multiple of four
            if (n >= N) continue;
            float *y = e.Y + (size_t)row * (N / 2) + n / 2;
            y[0] = v[u][0] / (1.0f + __expf(-v[u][0])) * v[u][1];
            y[1] = v[u][2] / (1.0f + __expf(-v[u][2])) * v[u][3];
            continue;
        }
        float *y = e.Y + (size_t)row * e.ldy + n;
        if (n + 4 <= N && e.ldy % 4 == 0) {
            *(f32x4 *)y = EPI == F32_ADD ? *(const f32x4 *)y + v[u] : v[u];
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (n + q < N) y[q] = EPI == F32_ADD ? y[q] + v[u][q] : v[u][q];
        }
    }
}

template <int U, int EPI>
void launch_gemm(hipStream_t st, const float *W, const float *X, int ldx, int groups, int M, int N, int K, const F32Epi &e) {
    if (M <= 16) k_gemm_f32<U, 1, EPI><<<dim3(groups, 1), 64 * NW, 0, st>>>(W, X, ldx, M, N, K, e);
    else k_gemm_f32<U, 2, EPI><<<dim3(groups, (M + 31) / 32), 64 * NW, 0, st>>>(W, X, ldx, M, N, K, e);
}

// ---------------------------------------------------------------------------------------------
// Tree-masked attention, fp32.  grid (batch * row groups of 16, n_heads, key splits; the first dimension alone holds
// any batch), eight waves that take the 16-key
// steps of the split's share in turn (step = split + splits * (wave + 8 k)), online softmax per wave, merged through LDS.
//   S^T[key][row] = K Q^T    A = K rows straight from the cache, B = the queries, in registers
//   O^T[d][row] += V^T P^T   B = the probabilities where the S^T tile left them (k step r: keys 4g + r), A = V, 16 consecutive
//                            dimensions per lane group
// One split: the rows go out finished; more: partial results for k_attn_combine.
// ---------------------------------------------------------------------------------------------
template <int DH>
__global__ __launch_bounds__(64 * NW) void k_attn_f32(const float *qrot, RowMeta meta, const float *kc, const float *vc,
                                                      float *o_part, float *ml, float *out, int rows_per_seq, int n_heads,
                                                      int cap, int nsplit, int ngroups) {
    constexpr int C = DH / 16;
    extern __shared__ __attribute__((aligned(16))) f32x4 mo[];   // [NW][C][64]
    __shared__ float mm[NW][16][2];
    const int s = blockIdx.z, h = blockIdx.y, b = blockIdx.x / ngroups, r0 = blockIdx.x % ngroups * 16;
    const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, li = l & 15, lg = l >> 4;
    const int kv_end = meta.kv_end[b];
    const bool ok = r0 + li < rows_per_seq;
    const int r = b * rows_per_seq + (ok ? r0 + li : 0), H = n_heads * DH;
    const float scale = rsqrtf((float)DH);
    f32x4 q[C], acc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        q[c] = *(const f32x4 *)(qrot + (size_t)r * H + h * DH + 16 * c + 4 * lg) * scale;
        acc[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    const int nvis = ok ? meta.row_nvis[r] : 0, base = ok ? meta.row_base[r] : 0;
    const uint64_t mask = ok ? meta.row_mask[r] : 0ull;
    const float *kb = kc + ((size_t)b * n_heads + h) * cap * DH, *vb = vc + ((size_t)b * n_heads + h) * cap * DH;
    const int nsteps = (kv_end + 15) / 16, stride = nsplit * NW;
    float m_run = -INFINITY, l_run = 0.f;
    for (int stp = s + nsplit * wave; stp < nsteps; stp += stride) {
        const int k0 = stp * 16;
        const float *kr = kb + (size_t)min(k0 + li, cap - 1) * DH + 4 * lg;
        f32x4 kf[C];
        float vf[4][C];
#pragma unroll
        for (int c = 0; c < C; ++c) kf[c] = *(const f32x4 *)(kr + 16 * c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float *vr = vb + (size_t)min(k0 + 4 * lg + e, cap - 1) * DH + li;
#pragma unroll
            for (int c = 0; c < C; ++c) vf[e][c] = vr[16 * c];
        }
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        f32x4 part[4] = {zero, zero, zero, zero};   // four chains, added at the end
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], q[c][e], part[e], 0, 0, 0);
        const f32x4 sc = (part[0] + part[1]) + (part[2] + part[3]);
        float tmax = -INFINITY, p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int key = k0 + 4 * lg + e;
            const unsigned rel = (unsigned)(key - base);   // negative differences wrap to >= 64
            const bool vis = key < kv_end && (key < nvis || (rel < 64u && ((mask >> (rel & 63u)) & 1ull)));
            p[e] = vis ? sc[e] : -INFINITY;
            tmax = fmaxf(tmax, p[e]);
        }
        tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
        const float m_new = fmaxf(m_run, tmax);
        const float alpha = m_run == -INFINITY ? 0.f : __expf(m_run - m_new);
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p[e] = p[e] == -INFINITY ? 0.f : __expf(p[e] - m_new);
            sum += p[e];
        }
        l_run = l_run * alpha + sum;
        m_run = m_new;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            acc[c] *= alpha;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = k0 + 4 * lg + e < kv_end ? vf[e][c] : 0.f;   // rows past the end: exact zeros
                acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, p[e], acc[c], 0, 0, 0);
            }
        }
    }
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
#pragma unroll
    for (int c = 0; c < C; ++c) mo[((size_t)wave * C + c) * 64 + l] = acc[c];
    if (lg == 0) {
        mm[wave][li][0] = m_run;   // -inf, 0 and zeros from a wave without a step
        mm[wave][li][1] = l_run;
    }
    __syncthreads();
    if (wave >= C || !ok) return;
    const int c = wave;   // this wave merges dimensions 16 c .. 16 c + 15
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, mm[w][li][0]);
    f32x4 O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float mw = mm[w][li][0], a = mw == -INFINITY ? 0.f : __expf(mw - M);
        L += a * mm[w][li][1];
        O += a * mo[((size_t)w * C + c) * 64 + l];
    }
    const int d = 16 * c + 4 * lg;
    if (nsplit == 1) {
        *(f32x4 *)(out + (size_t)r * H + h * DH + d) = O * (1.0f / L);
    } else {
        *(f32x4 *)(o_part + (((size_t)r * n_heads + h) * nsplit + s) * DH + d) = O;
        if (c == 0 && lg == 0) {
            ml[(((size_t)r * n_heads + h) * nsplit + s) * 2] = M;
            ml[(((size_t)r * n_heads + h) * nsplit + s) * 2 + 1] = L;
        }
    }
}

// merge the per-split partial results: grid (rows, n_heads), DH threads
__global__ void k_attn_combine(const float *o_part, const float *ml, float *out, int n_heads, int nsplit, int DH, int H) {
    const int r = blockIdx.x, h = blockIdx.y, d = threadIdx.x;
    const float *p = ml + ((size_t)r * n_heads + h) * nsplit * 2;
    float M = -INFINITY;
    for (int s = 0; s < nsplit; ++s) M = fmaxf(M, p[2 * s]);
    float num = 0.f, den = 0.f;
    for (int s = 0; s < nsplit; ++s) {
        const float ms = p[2 * s];
        if (ms == -INFINITY) continue;
        const float w = __expf(ms - M);
        num += w * o_part[(((size_t)r * n_heads + h) * nsplit + s) * DH + d];
        den += w * p[2 * s + 1];
    }
    out[(size_t)r * H + h * DH + d] = num / den;
}

}  // namespace

namespace kf {

void gemm(hipStream_t st, const float *X, int ldx, const void *W, float *Y, int ldy, int M, int N, int K, bool add) {
    F32Epi e{};
    e.Y = Y; e.ldy = ldy;
    const int groups = (N + 15) / 16;
    if (add) launch_gemm<1, F32_ADD>(st, (const float *)W, X, ldx, groups, M, N, K, e);
    else launch_gemm<1, F32_STORE>(st, (const float *)W, X, ldx, groups, M, N, K, e);
}

void norm_qkv(hipStream_t st, const float *X, const void *gain, float eps, const void *W, const RowMeta &meta, float *qrot,
              void *kc, void *vc, int rows, int H, int n_heads, int head_dim, int cap) {
    F32Epi e{};
    e.gain = (const float *)gain; e.eps = eps;
    e.meta = meta; e.qrot = qrot; e.kc = (float *)kc; e.vc = (float *)vc;
    e.H = H; e.n_heads = n_heads; e.DH = head_dim; e.cap = cap;
    launch_gemm<2, F32_QKV>(st, (const float *)W, X, H, 3 * H / 32, rows, 3 * H, H, e);
}

void norm_swiglu(hipStream_t st, const float *X, const void *gain, float eps, const void *W, float *act, int rows, int F, int H) {
    F32Epi e{};
    e.gain = (const float *)gain; e.eps = eps;
    e.Y = act;
    launch_gemm<1, F32_SWIGLU>(st, (const float *)W, X, H, (2 * F + 15) / 16, rows, 2 * F, H, e);
}

void attention(hipStream_t st, const float *qrot, const RowMeta &meta, const void *kc, const void *vc, float *o_part, float *ml,
               float *out, int batch, int rows_per_seq, int n_heads, int head_dim, int cap, int max_split) {
    // four steps of a full cache for each of a workgroup's waves
    const int nsplit = std::max(1, std::min(max_split, ((cap + 15) / 16 + 4 * NW - 1) / (4 * NW)));
    const int ngroups = (rows_per_seq + 15) / 16;
    const dim3 grid(batch * ngroups, n_heads, nsplit);
    const size_t sm = (size_t)NW * (head_dim / 16) * 64 * 16;
    if (head_dim == 128) {
        static OncePerDevice once;
        allow_lds(once, (const void *)k_attn_f32<128>, sm);
        k_attn_f32<128><<<grid, 64 * NW, sm, st>>>(qrot, meta, (const float *)kc, (const float *)vc, o_part, ml, out,
                                                   rows_per_seq, n_heads, cap, nsplit, ngroups);
    } else {
        k_attn_f32<64><<<grid, 64 * NW, sm, st>>>(qrot, meta, (const float *)kc, (const float *)vc, o_part, ml, out,
                                                  rows_per_seq, n_heads, cap, nsplit, ngroups);
    }
    if (nsplit > 1)
        k_attn_combine<<<dim3(batch * rows_per_seq, n_heads), head_dim, 0, st>>>(o_part, ml, out, n_heads, nsplit, head_dim,
                                                                                 n_heads * head_dim);
}

}  // namespace kf
