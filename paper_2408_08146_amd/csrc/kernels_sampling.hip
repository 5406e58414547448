// Non-greedy (temperature) drafting and acceptance, section 2.2:
//   * children of a tree node are draws without replacement from softmax(draft logits / temperature);
//   * the acceptance walk keeps child x with probability min(1, q(x)/d(x)); after a rejection the target
//     distribution becomes norm(max(0, q - d)), the rejected token leaves the draft distribution, and the
//     next child (in draw order) is tried; where the walk stops, one token is drawn from what q has become.
// Every uniform random number is an input.  One workgroup of 1024 threads per row, sequence or node.
//
// A draw is an inverse CDF over ascending token id: the first id at which the running sum of the weights
// exceeds u * total.  The vocabulary is cut into segments of 256 consecutive ids; a wave sums a segment
// with lane l holding ids 4l..4l+3 (fp64, fixed shuffle order), the segment sums are added up in a fixed order, and
// inside the chosen segment a wave-wide inclusive scan in lane order finds the id.  All orders are fixed,
// so a draw does not depend on scheduling.
//
// Two forms.  Up to 32768 tokens a workgroup holds its rows in registers (32 values of a row per thread): a row is read
// once, every later pass over it is arithmetic, and the draws of a row exchange one number each through LDS.  Larger
// vocabularies keep their rows in memory and read them again in every pass.  Acceptance for eight sequences of 60 nodes and
// 32000 tokens: 35 us with the nodes side by side in registers, 81 us with a workgroup a sequence that takes them in turn (94
// with shuffles through LDS in its reductions), 278 us in the memory form.  Draws (the children of 208 nodes, a 64-node
// Medusa-style tree for eight sequences): 33 us where the memory form takes 427 us.
#include "koala_internal.h"

namespace {

constexpr int NT = 1024;         // threads per workgroup
constexpr int NW = NT / 64;      // waves per workgroup
constexpr int SEG = 256;          // ids per segment
constexpr int MAX_SEG = 1024;     // vocabularies up to 262144
constexpr int UNR = 4;            // independent loads in flight per thread in the vocabulary-wide passes

struct Shared {
    double seg[MAX_SEG];
    double red[NW];
    float fmax_[NW];
    double total, base, target;
    int sidx, idx, fallback;
    int kids[64];
    int nk;
};

__device__ __forceinline__ double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// every thread gets the sum of v over the workgroup (waves added in order)
__device__ __forceinline__ double block_sum(double v, Shared &sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    for (int k = 0; k < NW; ++k) t += sh.red[k];
    return t;
}

__device__ __forceinline__ float block_max(float v, Shared &sh) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.fmax_[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = sh.fmax_[0];
    for (int k = 1; k < NW; ++k) t = fmaxf(t, sh.fmax_[k]);
    return t;
}

// the four weights of lane l in segment s (zero past V)
__device__ __forceinline__ void seg_load(const float *w, int V, int s, int l, float *x) {
    const int i = s * SEG + 4 * l;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = i + e < V ? w[i + e] : 0.f;
}

__device__ __forceinline__ double seg_lane_sum(const float *x) {
    return (((double)x[0] + (double)x[1]) + (double)x[2]) + (double)x[3];
}

// sh.seg[s] = sum of w over segment s, for all segments (wave k takes segments k, k+NW, ...)
__device__ void segment_sums(const float *w, int V, Shared &sh) {
    const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, nseg = (V + SEG - 1) / SEG;
    __syncthreads();
    for (int s0 = wave; s0 < nseg; s0 += 4 * NW) {   // four segments' loads in flight per wave
        float x[4][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) seg_load(w, V, s0 + NW * k, l, x[k]);   // past the last segment: zeros
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double t = wave_sum(seg_lane_sum(x[k]));
            if (l == 0 && s0 + NW * k < nseg) sh.seg[s0 + NW * k] = t;
        }
    }
    __syncthreads();
}

// Index of the first id at which the running sum of w exceeds u * sum(w); the last positive id if rounding
// leaves none; 0 if nothing is positive.  sh.seg must hold the segment sums of w.  Every thread gets it.
__device__ int block_inverse_cdf(const float *w, int V, double u, Shared &sh) {
    const int tid = threadIdx.x, nseg = (V + SEG - 1) / SEG;
    __syncthreads();
    if (tid == 0) {
        double total = 0.0;
        for (int s = 0; s < nseg; ++s) total += sh.seg[s];
        const double target = u * total;
        double run = 0.0;
        int t = -1;
        for (int s = 0; s < nseg; ++s) {
            if (run + sh.seg[s] > target) { t = s; break; }
            run += sh.seg[s];
        }
        sh.fallback = 0;
        if (t < 0) {   // rounding: the last segment that holds anything
            sh.fallback = 1;
            for (int s = nseg - 1; s >= 0; --s)
                if (sh.seg[s] > 0.0) { t = s; break; }
        }
        sh.sidx = t;
        sh.base = run;
        sh.target = target;
        sh.idx = 0;
    }
    __syncthreads();
    if (tid < 64 && sh.sidx >= 0) {   // wave 0 resolves the id inside the segment
        const int s = sh.sidx, l = tid;
        float x[4];
        seg_load(w, V, s, l, x);
        const double own = seg_lane_sum(x);
        double incl = own;
        for (int o = 1; o < 64; o <<= 1) {
            const double t = __shfl_up(incl, o);
            if (l >= o) incl += t;
        }
        const double lo = sh.base + (incl - own), hi = sh.base + incl;
        int pick = -1, lastpos = -1;
        double run = lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (x[e] > 0.f) {
                lastpos = s * SEG + 4 * l + e;
                run += (double)x[e];
                if (pick < 0 && run > sh.target) pick = lastpos;
            }
        }
        const bool mine = !sh.fallback && lo <= sh.target && hi > sh.target && pick >= 0;
        // the first lane that claims the id wins; otherwise the last positive id of the segment
        const unsigned long long claims = __ballot(mine);
        int last_all = lastpos;
        for (int o = 32; o > 0; o >>= 1) last_all = max(last_all, __shfl_xor(last_all, o));
        if (claims) {
            const int first = __ffsll((long long)claims) - 1;
            const int got = __shfl(pick, first);
            if (l == 0) sh.idx = got;
        } else if (l == 0) {
            sh.idx = last_all < 0 ? 0 : last_all;
        }
    }
    __syncthreads();
    return sh.idx;
}

// children of node p in draw order (ascending rank, then node id) into sh.kids
__device__ void list_children(const TreeTables &tt, int T, int p, Shared &sh) {
    __syncthreads();
    if (threadIdx.x == 0) {
        int n = 0;
        for (int c = 0; c < T && n < 64; ++c) {
            if (tt.parent[c] != p) continue;
            int j = n++;
            while (j > 0 && tt.rank[sh.kids[j - 1]] > tt.rank[c]) { sh.kids[j] = sh.kids[j - 1]; --j; }
            sh.kids[j] = c;
        }
        sh.nk = n;
    }
    __syncthreads();
}

// w[i] = exp((z[i] - max z) / tau); returns sum(w).  z and w may alias.  copy: optional copy of z.
__device__ double softmax_weights(const float *z, float *w, float *copy, int V, float inv_tau, Shared &sh) {
    const int tid = threadIdx.x;
    float m = -INFINITY;
    for (int i0 = tid; i0 < V; i0 += NT * UNR) {
        float v[UNR];
#pragma unroll
        for (int k = 0; k < UNR; ++k) v[k] = i0 + k * NT < V ? z[i0 + k * NT] : -INFINITY;
#pragma unroll
        for (int k = 0; k < UNR; ++k) {
            m = fmaxf(m, v[k]);
            if (copy && i0 + k * NT < V) copy[i0 + k * NT] = v[k];
        }
    }
    m = block_max(m, sh);
    double s = 0.0;
    for (int i0 = tid; i0 < V; i0 += NT * UNR) {
        float v[UNR];
#pragma unroll
        for (int k = 0; k < UNR; ++k) v[k] = i0 + k * NT < V ? z[i0 + k * NT] : -INFINITY;
#pragma unroll
        for (int k = 0; k < UNR; ++k) {
            if (i0 + k * NT < V) {
                const float e = expf((v[k] - m) * inv_tau);
                w[i0 + k * NT] = e;
                s += (double)e;
            }
        }
    }
    return block_sum(s, sh);
}

// w[i] /= total over the vocabulary
__device__ void scale_by(float *w, int V, double total) {
    for (int i0 = threadIdx.x; i0 < V; i0 += NT * UNR) {
        float v[UNR];
#pragma unroll
        for (int k = 0; k < UNR; ++k) v[k] = i0 + k * NT < V ? w[i0 + k * NT] : 0.f;
#pragma unroll
        for (int k = 0; k < UNR; ++k)
            if (i0 + k * NT < V) w[i0 + k * NT] = (float)((double)v[k] / total);
    }
}

// One workgroup per sequence and listed node.  The node's logits are row (stride_by_depth: depth * batch + sequence, the
// heads of a Medusa-style draft; else the workgroup's own number) of src; z: [workgroup][V] scratch, may be src.
__global__ __launch_bounds__(NT) void k_sample_children(const float *src, float *z, ks::NodeList nodes, int by_depth,
                                                         int batch, TreeTables tt, int T, int V, float inv_tau,
                                                         const float *u_draw, int32_t *tree_tokens,
                                                         float *draft_logits) {
    __shared__ Shared sh;
    const int row = blockIdx.x, b = row / nodes.n, p = nodes.node[row % nodes.n], tid = threadIdx.x;
    list_children(tt, T, p, sh);
    float *zr = z + (size_t)row * V;
    src += (size_t)(by_depth ? nodes.depth[row % nodes.n] * batch + b : row) * V;
    (void)softmax_weights(src, zr, draft_logits + ((size_t)b * T + p) * V, V, inv_tau, sh);
    segment_sums(zr, V, sh);
    for (int j = 0; j < sh.nk; ++j) {
        const int c = sh.kids[j];
        const int idx = block_inverse_cdf(zr, V, (double)u_draw[(size_t)b * T + c], sh);
        if (tid == 0) {
            tree_tokens[(size_t)b * T + c] = idx;
            zr[idx] = 0.f;   // drawn without replacement
        }
        __syncthreads();
        if (tid < 64) {      // wave 0 refreshes the sum of the segment that lost the token
            const int s = idx / SEG;
            float x[4];
            seg_load(zr, V, s, tid, x);
            const double t = wave_sum(seg_lane_sum(x));
            if (tid == 0) sh.seg[s] = t;
        }
        __syncthreads();
    }
}

// grid: batch.  qv, dv: [batch][V] scratch.
__global__ __launch_bounds__(NT) void k_accept_sample(TreeTables tt, int T, int D, int V, float inv_tau,
                                                       const int32_t *tree_tokens, const float *target_logits,
                                                       const float *draft_logits, const float *u_accept,
                                                       const float *u_resample, float *qv_all, float *dv_all,
                                                       int32_t *accept_len, int32_t *accept_path,
                                                       int32_t *next_token) {
    __shared__ Shared sh;
    const int b = blockIdx.x, tid = threadIdx.x;
    float *qv = qv_all + (size_t)b * V, *dv = dv_all + (size_t)b * V;
    const int32_t *tok = tree_tokens + (size_t)b * T;
    int32_t *path = accept_path + (size_t)b * (D + 1);
    int cur = 0, a = 0;
    if (tid == 0) path[0] = 0;
    for (;;) {
        // q = softmax(target logits at cur)
        double tot = softmax_weights(target_logits + ((size_t)b * T + cur) * V, qv, nullptr, V, inv_tau, sh);
        scale_by(qv, V, tot);
        list_children(tt, T, cur, sh);
        const int nk = a < D ? sh.nk : 0;
        bool moved = false;
        if (nk > 0) {
            tot = softmax_weights(draft_logits + ((size_t)b * T + cur) * V, dv, nullptr, V, inv_tau, sh);
            scale_by(dv, V, tot);
            __syncthreads();
            for (int j = 0; j < nk; ++j) {
                const int c = sh.kids[j];
                int x = tok[c];
                x = x < 0 ? 0 : x >= V ? V - 1 : x;
                const double qx = (double)qv[x], dx = (double)dv[x];
                const double ratio = dx > 0.0 ? fmin(1.0, qx / dx) : 0.0;
                if (dx > 0.0 && (double)u_accept[(size_t)b * T + c] < ratio) {
                    cur = c;
                    ++a;
                    if (tid == 0) path[a] = c;
                    moved = true;
                    break;
                }
                // rejected: q <- norm(max(0, q - d)) (kept if that is all zero); d loses x and is renormalised
                double rs = 0.0, ds = 0.0;
                for (int i0 = tid; i0 < V; i0 += NT * UNR) {
                    float qa[UNR], da[UNR];
#pragma unroll
                    for (int k = 0; k < UNR; ++k) {
                        const bool in = i0 + k * NT < V;
                        qa[k] = in ? qv[i0 + k * NT] : 0.f;
                        da[k] = in ? dv[i0 + k * NT] : 0.f;
                    }
#pragma unroll
                    for (int k = 0; k < UNR; ++k) {
                        rs += (double)fmaxf(0.f, qa[k] - da[k]);
                        if (i0 + k * NT != x) ds += (double)da[k];
                    }
                }
                const double R = block_sum(rs, sh);
                const double Dn = block_sum(ds, sh);
                for (int i0 = tid; i0 < V; i0 += NT * UNR) {
                    float qa[UNR], da[UNR];
#pragma unroll
                    for (int k = 0; k < UNR; ++k) {
                        const bool in = i0 + k * NT < V;
                        qa[k] = in ? qv[i0 + k * NT] : 0.f;
                        da[k] = in ? dv[i0 + k * NT] : 0.f;
                    }
#pragma unroll
                    for (int k = 0; k < UNR; ++k) {
                        const int i = i0 + k * NT;
                        if (i < V) {
                            if (R > 0.0) qv[i] = (float)((double)fmaxf(0.f, qa[k] - da[k]) / R);
                            dv[i] = (i == x) ? 0.f : (Dn > 0.0 ? (float)((double)da[k] / Dn) : da[k]);
                        }
                    }
                }
                __syncthreads();
            }
        }
        if (!moved) {
            segment_sums(qv, V, sh);
            const int idx = block_inverse_cdf(qv, V, (double)u_resample[(size_t)b * T + cur], sh);
            if (tid == 0) {
                next_token[b] = idx;
                accept_len[b] = a;
                for (int j = a + 1; j <= D; ++j) path[j] = -1;
            }
            return;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------
// Register form.  Thread t holds ids (u * 1024 + t) * 4 + e, u < NQ, e < 4, of a row: group u of wave w is segment
// u * 16 + w, lane l of it ids 4l..4l+3 of the segment.
// ---------------------------------------------------------------------------------------------
constexpr int REG_SEG = 128;                 // segments of a row held in registers, at most
constexpr int REG_V = REG_SEG * SEG;         // vocabularies of the register form: up to 32768
typedef __attribute__((ext_vector_type(4))) float f32q;
struct __attribute__((packed, aligned(4))) f4_any { float v[4]; };   // 16 bytes at a 4-byte aligned address

struct RegShared {
    double seg[REG_SEG];
    double red[2][NW];
    float mx[2][NW];
    double news[2];        // the sum a draw leaves its segment with, by parity of the draw
    float qx[2], dx[2];    // probabilities of the child to be tried, by parity
};

template <int NQ>
__device__ __forceinline__ void row_load(const float *row, int V, float (&w)[NQ][4]) {
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int i = (u * NT + (int)threadIdx.x) * 4;
        if (i + 4 <= V) {
            const f4_any x = *(const f4_any *)(row + i);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[u][e] = x.v[e];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) w[u][e] = i + e < V ? row[i + e] : -INFINITY;
        }
    }
}
template <int NQ>
__device__ __forceinline__ float row_max(const float (&w)[NQ][4]) {
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < NQ; ++u) m = fmaxf(m, fmaxf(fmaxf(w[u][0], w[u][1]), fmaxf(w[u][2], w[u][3])));
    return m;
}
// w <- exp((w - m) / tau), past the vocabulary zero (by index: at an infinite temperature the exponent of the -inf there
// is no number); returns this thread's sum
template <int NQ>
__device__ __forceinline__ double row_exp(float (&w)[NQ][4], int V, float m, float inv_tau) {
    asm volatile("" : "+s"(V));   // compared anew: no masks kept from the loads
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[u][e] = expf((w[u][e] - m) * inv_tau);
        if (V < (u + 1) * NT * 4)   // the same for all threads
#pragma unroll
            for (int e = 0; e < 4; ++e) w[u][e] = (int)threadIdx.x * 4 < V - u * NT * 4 - e ? w[u][e] : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) s += (double)w[u][e];
        __builtin_amdgcn_sched_barrier(0);
    }
    return s;
}
template <int NQ>
__device__ __forceinline__ void row_scale(float (&w)[NQ][4], double f) {
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            asm volatile("" : "+v"(w[u][e]));   // widened again here: a row of doubles from the sums would not fit
            w[u][e] = (float)((double)w[u][e] * f);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}
// Reductions over the wave without LDS: a shuffle goes through LDS (two trips for a double, about 120 cycles each), the swap
// and row instructions below stay in the vector unit.  A butterfly by 32, 16, 8, 4, 2, 1: the swap of a value with itself
// leaves a lane's own and its partner's value in the two results; a rotation by o within sixteen lanes is the exchange with
// lane ^ o once the lanes 2 o apart hold the same value (by 8 it is that exchange itself).
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t dpp32(uint32_t v) {   // lanes without a source, and rows not named, get zero
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, true);
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp64(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, (uint64_t)dpp32<CTRL, ROWS>((uint32_t)(b >> 32)) << 32 | dpp32<CTRL, ROWS>((uint32_t)b));
}
enum { DPP_ROR = 0x120, DPP_SHR = 0x110, DPP_WAVE_SHR1 = 0x138, DPP_BCAST15 = 0x142, DPP_BCAST31 = 0x143 };
__device__ __forceinline__ double swap_sum(double v, bool by32) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
    const auto p = by32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false) : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto q = by32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false) : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __builtin_bit_cast(double, (uint64_t)q[0] << 32 | p[0]) + __builtin_bit_cast(double, (uint64_t)q[1] << 32 | p[1]);
}
__device__ __forceinline__ float swap_max(float v, bool by32) {
    const uint32_t b = __float_as_uint(v);
    const auto p = by32 ? __builtin_amdgcn_permlane32_swap(b, b, false, false) : __builtin_amdgcn_permlane16_swap(b, b, false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
__device__ __forceinline__ double row16_sum(double v) {   // over sixteen lanes, in each of them
    v += dpp64<DPP_ROR + 8>(v);
    v += dpp64<DPP_ROR + 4>(v);
    v += dpp64<DPP_ROR + 2>(v);
    return v + dpp64<DPP_ROR + 1>(v);
}
__device__ __forceinline__ float row16_max(float v) {
    v = fmaxf(v, __uint_as_float(dpp32<DPP_ROR + 8>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(dpp32<DPP_ROR + 4>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(dpp32<DPP_ROR + 2>(__float_as_uint(v))));
    return fmaxf(v, __uint_as_float(dpp32<DPP_ROR + 1>(__float_as_uint(v))));
}
__device__ __forceinline__ double wave_total(double v) { return row16_sum(swap_sum(swap_sum(v, true), false)); }
__device__ __forceinline__ double lane_value(double v, int lane) {   // of a lane that is the same for all
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), lane));
}
__device__ __forceinline__ double wave_scan(double v) {   // inclusive, in lane order
    v += dpp64<DPP_SHR + 1>(v);
    v += dpp64<DPP_SHR + 2>(v);
    v += dpp64<DPP_SHR + 4>(v);
    v += dpp64<DPP_SHR + 8>(v);
    v += dpp64<DPP_BCAST15, 0xa>(v);   // the sums of rows 0 and 2 to rows 1 and 3
    return v + dpp64<DPP_BCAST31, 0xc>(v);
}
// maxima / sums of two values over the workgroup; nobody may still be reading the arrays of an earlier call
__device__ __forceinline__ void block_max2(float &a, float &b, RegShared &sh) {
    a = row16_max(swap_max(swap_max(a, true), false));
    b = row16_max(swap_max(swap_max(b, true), false));
    if ((threadIdx.x & 63) == 0) { sh.mx[0][threadIdx.x >> 6] = a; sh.mx[1][threadIdx.x >> 6] = b; }
    __syncthreads();
    const int l = threadIdx.x & 63;   // sixteen lanes a value
    const float v = row16_max(sh.mx[(l >> 4) & 1][l & 15]);
    a = lane_value(v, 0);
    b = lane_value(v, 16);
}
__device__ __forceinline__ void block_sum2(double &a, double &b, RegShared &sh) {
    a = wave_total(a);
    b = wave_total(b);
    if ((threadIdx.x & 63) == 0) { sh.red[0][threadIdx.x >> 6] = a; sh.red[1][threadIdx.x >> 6] = b; }
    __syncthreads();
    const int l = threadIdx.x & 63;
    const double v = row16_sum(sh.red[(l >> 4) & 1][l & 15]);
    a = lane_value(v, 0);
    b = lane_value(v, 16);
}

// The sums of segments 2l and 2l + 1 in lane l of every wave
struct SegPair { double a, b; };
template <int NQ>
__device__ __forceinline__ SegPair segment_pairs(const float (&w)[NQ][4], int wave, RegShared &sh) {
    const int l = threadIdx.x & 63;
    double t[NQ];
#pragma unroll
    for (int u = 0; u < NQ; ++u) t[u] = wave_total(seg_lane_sum(w[u]));
    if (l == 0) {
#pragma unroll
        for (int u = 0; u < NQ; ++u) sh.seg[u * NW + wave] = t[u];
    }
    __syncthreads();
    SegPair p;
    p.a = 2 * l < NQ * NW ? sh.seg[2 * l] : 0.0;
    p.b = 2 * l + 1 < NQ * NW ? sh.seg[2 * l + 1] : 0.0;
    return p;
}
struct SegPick { int s; bool rounding; double base, target; };   // s: the segment that holds the id, -1 if nothing is positive
// The first segment with anything in it at which the running sum exceeds u * total; the last one with anything if
// rounding leaves none.  The same in every wave.
__device__ __forceinline__ SegPick pick_segment(const SegPair &p, double u) {
    const double incl = wave_scan(p.a + p.b);
    const double excl = dpp64<DPP_WAVE_SHR1>(incl);   // zero in lane 0
    SegPick r;
    r.target = u * lane_value(incl, 63);
    const bool first = p.a > 0.0 && excl + p.a > r.target, second = p.b > 0.0 && incl > r.target;
    const unsigned long long hit = __ballot(first || second);
    const double base = first ? excl : excl + p.a;
    r.rounding = hit == 0;
    r.base = 0.0;
    if (hit) {
        const int at = __ffsll((long long)hit) - 1;
        r.s = 2 * at + ((__ballot(first) >> at) & 1 ? 0 : 1);
        r.base = lane_value(base, at);
    } else {
        const unsigned long long any = __ballot(p.a > 0.0 || p.b > 0.0);
        if (any == 0) { r.s = -1; return r; }
        const int at = 63 - __clzll((long long)any);
        r.s = 2 * at + ((__ballot(p.b > 0.0) >> at) & 1 ? 1 : 0);
    }
    return r;
}
// The id inside the picked segment, by the wave that holds it in group x (every lane gets it)
__device__ __forceinline__ int pick_in_segment(const float (&x)[4], const SegPick &r) {
    const int l = threadIdx.x & 63;
    const double own = seg_lane_sum(x), incl = wave_scan(own);
    const double lo = r.base + (incl - own), hi = r.base + incl;
    int pick = -1, last = -1;
    double run = lo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (x[e] > 0.f) {
            last = r.s * SEG + 4 * l + e;
            run += (double)x[e];
            if (pick < 0 && run > r.target) pick = last;
        }
    }
    const unsigned long long claims = __ballot(!r.rounding && lo <= r.target && hi > r.target && pick >= 0);
    if (claims) return __builtin_amdgcn_readlane(pick, __ffsll((long long)claims) - 1);
    for (int o = 32; o > 0; o >>= 1) last = max(last, __shfl_xor(last, o));
    return max(last, 0);
}

// The children of node p as bits, from the tree held one node a lane, and the child of the j-th lowest rank (lowest id
// among equal ranks, as the other form lists them)
__device__ __forceinline__ unsigned long long children_of(int parent_of_lane, int p) { return __ballot(parent_of_lane == p); }
__device__ __forceinline__ int child_order(unsigned long long kids, int rank_of_lane) {   // place of the lane's node among them
    const int l = threadIdx.x & 63;
    int place = 0;
    for (unsigned long long m = kids; m; m &= m - 1) {
        const int j = __ffsll((long long)m) - 1, rj = __builtin_amdgcn_readlane(rank_of_lane, j);
        place += rj < rank_of_lane || (rj == rank_of_lane && j < l) ? 1 : 0;
    }
    return (kids >> l) & 1 ? place : -1;
}
__device__ __forceinline__ int child_at(int place_of_lane, int j) { return __ffsll((long long)__ballot(place_of_lane == j)) - 1; }

template <int NQ>
__global__ __launch_bounds__(NT) void k_sample_children_r(const float *src, ks::NodeList nodes, int by_depth, int batch,
                                                          TreeTables tt, int T, int V, float inv_tau, const float *u_draw,
                                                          int32_t *tree_tokens, float *draft_logits) {
    __shared__ RegShared sh;
    const int row = blockIdx.x, b = row / nodes.n, p = nodes.node[row % nodes.n];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    float w[NQ][4];
    row_load<NQ>(src + (size_t)(by_depth ? nodes.depth[row % nodes.n] * batch + b : row) * V, V, w);
    const int par = l < T ? tt.parent[l] : -2, rank = l < T ? tt.rank[l] : 0;
    const float u_lane = l < T ? u_draw[(size_t)b * T + l] : 0.f;
    const unsigned long long kids = children_of(par, p);
    const int nk = __popcll(kids), place = child_order(kids, rank);
    float *copy = draft_logits + ((size_t)b * T + p) * V;
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int i = (u * NT + (int)threadIdx.x) * 4;
        if (i + 4 <= V) {
            f4_any x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x.v[e] = w[u][e];
            *(f4_any *)(copy + i) = x;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e < V) copy[i + e] = w[u][e];
        }
    }
    float m = row_max<NQ>(w), unused = 0.f;
    block_max2(m, unused, sh);
    (void)row_exp<NQ>(w, V, m, inv_tau);
    SegPair seg = segment_pairs<NQ>(w, wave, sh);
    for (int j = 0; j < nk; ++j) {
        const int c = child_at(place, j);
        const SegPick r = pick_segment(seg, (double)lane_value(u_lane, c));
        if (r.s < 0) {   // nothing left to draw from, here and for the children that follow
            if (threadIdx.x == 0) tree_tokens[(size_t)b * T + c] = 0;
            continue;
        }
        if ((r.s & (NW - 1)) == wave) {
            float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < NQ; ++u)
                if (u == r.s / NW)
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = w[u][e];
            const int idx = pick_in_segment(x, r);
#pragma unroll
            for (int u = 0; u < NQ; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e)   // drawn without replacement
                    if (idx - (int)threadIdx.x * 4 == u * NT * 4 + e) w[u][e] = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (r.s * SEG + 4 * l + e == idx) x[e] = 0.f;
            const double left = wave_total(seg_lane_sum(x));
            if (l == 0) {
                tree_tokens[(size_t)b * T + c] = idx;
                sh.news[j & 1] = left;
            }
        }
        __syncthreads();
        if (l == r.s / 2) { if (r.s & 1) seg.b = sh.news[j & 1]; else seg.a = sh.news[j & 1]; }
    }
}

// What acceptance asks of a sequence's nodes, and the tree held one node a lane in every wave
struct WalkShared {
    RegShared r;
    float ua[KOALA_MAX_NODES], ur[KOALA_MAX_NODES];   // in LDS: the rows fill the registers
    int tok[KOALA_MAX_NODES];
    int off;                                          // found, on the way, not to be on the path
};
struct WalkArgs {
    const int32_t *tree_tokens;
    const float *target_logits, *draft_logits, *u_accept, *u_resample;
    int32_t *accept_len, *accept_path, *next_token;
};
// the accepted child or, 0, where the walk stops: then token, in the wave that says mine; -1: not on the path
struct NodeEnd { int child, token; bool mine; };
// Nodes side by side: those that their parent has turned down, one bit each, and the bits of a node and its ancestors
struct Branch {
    unsigned long long *dead, line;
    __device__ __forceinline__ void turn_down(unsigned long long kids) const {
        if (threadIdx.x == 0) __hip_atomic_fetch_or(dead, kids, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ unsigned long long told() const {
        return __hip_atomic_load(dead, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

__device__ __forceinline__ void walk_inputs(const WalkArgs &g, int b, int T, int V, WalkShared &sh) {   // read behind the first barrier
    const int tid = threadIdx.x;
    if (tid < T) {
        const int x = g.tree_tokens[(size_t)b * T + tid];
        sh.tok[tid] = x < 0 ? 0 : x >= V ? V - 1 : x;
        sh.ua[tid] = g.u_accept[(size_t)b * T + tid];
        sh.ur[tid] = g.u_resample[(size_t)b * T + tid];
    }
}

__device__ __forceinline__ void written_through() {   // this lane's atomics have been performed (see k_accept_nodes)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
}

// What happens at node `cur` of sequence b, which depends on nothing that came before: its children are tried in draw order,
// and where none is accepted a token is drawn.  The draft's row is in registers and the target's in LDS, where a thread only
// ever touches its own 16-byte pieces (no barriers, no bank conflicts): both in registers with 512 threads spilled.  Both are
// divided by their sums only once a child has been rejected or a token is drawn; the first child needs two quotients.
// SIDE: other nodes are under way; they are told of every child turned down, and what they tell ends this one.
template <int NQ, bool SIDE>
__device__ __forceinline__ NodeEnd walk_node(const WalkArgs &g, int b, int cur, int T, int V, float inv_tau, int par, int rank,
                                             f32q *ql, WalkShared &sh, const Branch &br) {
    constexpr bool LOOK = SIDE && NQ >= 4;   // passes over rows of up to 4096 tokens are too short to cover the look (13 -> 15 us)
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned long long kids = children_of(par, cur);
    const int nk = __popcll(kids), place = child_order(kids, rank);
    float d[NQ][4], mq, md = 0.f;
    int Vi = V;
    asm volatile("" : "+s"(Vi));   // the row's bounds are worked out anew for each node
    double sq, sd = 1.0;
    {
        float q[NQ][4];
        row_load<NQ>(g.target_logits + ((size_t)b * T + cur) * V, Vi, q);
        if (nk > 0) row_load<NQ>(g.draft_logits + ((size_t)b * T + cur) * V, Vi, d);
        mq = row_max<NQ>(q);
        if (nk > 0) md = row_max<NQ>(d);
        block_max2(mq, md, sh.r);
        sq = row_exp<NQ>(q, Vi, mq, inv_tau);
        if (nk > 0) sd = row_exp<NQ>(d, Vi, md, inv_tau);
        block_sum2(sq, sd, sh.r);
        if (nk == 0) row_scale<NQ>(q, 1.0 / sq);
#pragma unroll
        for (int u = 0; u < NQ; ++u) ql[u * NT] = (f32q){q[u][0], q[u][1], q[u][2], q[u][3]};
    }
    for (int j = 0; j < nk; ++j) {
        const int c = child_at(place, j), x = sh.tok[c], xo = x - tid * 4;
        if (xo >= 0 && xo % (NT * 4) < 4) {   // this thread has the probabilities of the child's token
            float dx = 0.f, qx = ((const float *)(ql + xo / (NT * 4) * NT))[xo % 4];
#pragma unroll
            for (int u = 0; u < NQ; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) dx = xo == u * NT * 4 + e ? d[u][e] : dx;
            if (j == 0) { qx = (float)((double)qx * (1.0 / sq)); dx = (float)((double)dx * (1.0 / sd)); }
            sh.r.dx[j & 1] = dx;
            sh.r.qx[j & 1] = qx;
        }
        __syncthreads();
        const double qx = (double)sh.r.qx[j & 1], dx = (double)sh.r.dx[j & 1];
        const double ratio = dx > 0.0 ? fmin(1.0, qx / dx) : 0.0;
        if (dx > 0.0 && (double)sh.ua[c] < ratio) {
            if (SIDE) br.turn_down(kids & ~(1ull << c));
            return NodeEnd{c, 0, wave == 0};
        }
        if (SIDE) br.turn_down(1ull << c);
        const unsigned long long told = LOOK && tid == 0 ? br.told() : 0;   // on its way while the distributions are passed over
        // rejected: q <- norm(max(0, q - d)) (kept if that is all zero); d loses x and is renormalised
        double rs = 0.0, ds = 0.0;
        int xd = xo;
        asm volatile("" : "+v"(xd));   // compared anew: no 32 masks kept from above
        if (j == 0) {
            const double fq = 1.0 / sq;
#pragma unroll
            for (int u = 0; u < NQ; ++u) {
                f32q q = ql[u * NT];
#pragma unroll
                for (int e = 0; e < 4; ++e) q[e] = (float)((double)q[e] * fq);
                ql[u * NT] = q;
                __builtin_amdgcn_sched_barrier(0);
            }
            row_scale<NQ>(d, 1.0 / sd);
        }
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const f32q q = ql[u * NT];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                rs += (double)fmaxf(0.f, q[e] - d[u][e]);
                d[u][e] = xd == u * NT * 4 + e ? 0.f : d[u][e];
                ds += (double)d[u][e];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (LOOK && tid == 0) sh.off = (told & br.line) != 0;
        block_sum2(rs, ds, sh.r);
        if (LOOK && sh.off) return NodeEnd{-1, 0, wave == 0};
        const bool keep = !(rs > 0.0);
        const double fr = keep ? 1.0 : 1.0 / rs, fd = ds > 0.0 ? 1.0 / ds : 1.0;
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            f32q q = ql[u * NT];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                asm volatile("" : "+v"(d[u][e]));   // as in row_scale
                const float t = fmaxf(0.f, q[e] - d[u][e]);
                q[e] = (float)((double)(keep ? q[e] : t) * fr);
                d[u][e] = (float)((double)d[u][e] * fd);
            }
            ql[u * NT] = q;
            __builtin_amdgcn_sched_barrier(0);
        }
        if (xo >= 0 && xo % (NT * 4) < 4) {   // d has lost x by now: q there once more, from the values tried above
            const float qo = sh.r.qx[j & 1], t = fmaxf(0.f, qo - sh.r.dx[j & 1]);
            ((float *)(ql + xo / (NT * 4) * NT))[xo % 4] = (float)((double)(keep ? qo : t) * fr);
        }
    }
    float q[NQ][4];
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const f32q x = ql[u * NT];
#pragma unroll
        for (int e = 0; e < 4; ++e) q[u][e] = x[e];
    }
    if (SIDE && wave == 0) written_through();   // what it has told the others, before the barrier behind which any wave may count
    const SegPair seg = segment_pairs<NQ>(q, wave, sh.r);
    const SegPick r = pick_segment(seg, (double)sh.ur[cur]);
    const bool mine = r.s < 0 ? wave == 0 : (r.s & (NW - 1)) == wave;
    int idx = 0;
    if (mine && r.s >= 0) {
        float y[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < NQ; ++u)
            if (u == r.s / NW)
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = q[u][e];
        idx = pick_in_segment(y, r);
    }
    return NodeEnd{0, idx, mine};
}

// One workgroup per sequence follows the path from the root.
template <int NQ>
__global__ __launch_bounds__(NT) void k_accept_walk(TreeTables tt, int T, int D, int V, float inv_tau, WalkArgs g) {
    extern __shared__ __attribute__((aligned(16))) f32q walk_q[];   // [NQ][NT]
    __shared__ WalkShared sh;
    const int b = blockIdx.x, tid = threadIdx.x, l = tid & 63;
    int32_t *path = g.accept_path + (size_t)b * (D + 1);
    const int par = l < T ? tt.parent[l] : -2, rank = l < T ? tt.rank[l] : 0;
    walk_inputs(g, b, T, V, sh);
    int cur = 0, a = 0;
    if (tid == 0) path[0] = 0;
    for (;;) {
        const NodeEnd e = walk_node<NQ, false>(g, b, cur, T, V, inv_tau, par, rank, walk_q + tid, sh, Branch{});
        if (e.child > 0) {
            cur = e.child;
            ++a;
            if (tid == 0) path[a] = cur;
            continue;
        }
        if (e.mine && l == 0) g.next_token[b] = e.token;
        if (tid == 0) {
            g.accept_len[b] = a;
            for (int j = a + 1; j <= D; ++j) path[j] = -1;
        }
        return;
    }
}

// All nodes at once, one workgroup each: the path is a chain of nodes that each take a row's way through the compute unit
// (about 13 us), but what happens at a node does not depend on the path to it.  Nodes are dealt out from the root down, the
// sequences in turn.  A node tells the others of every child it turns down (the rejected, one by one, and the siblings of an
// accepted one); a workgroup that does not start with the first ones looks whether its branch has been, and is done if so, and
// longer rows look again with every rejection of their own.
// state [sequence][STATE], whole numbers: what became of each node (0: not known, the child taken, or -1 - the token drawn), a
// count of finished workgroups, and a bit for every node turned down.  The last workgroup of a sequence follows the path and
// leaves zeros.  Nobody waits for anybody.
// State is read and written by agent-scope atomics only.  Those go past the caches that are not coherent between dies (the sc1
// bit of their instructions: loads miss them, stores and read-modify-writes are performed behind them), and the count of memory
// operations that s_waitcnt waits for covers them until then; so a wave that has waited has its results where every other
// workgroup's atomics look, and no cache has to be written back or dropped, which a fence of agent scope would do.
enum { STATE = 80, DONE = 64, DEAD = 66 };
static_assert((int)STATE == (int)ks::ACCEPT_STATE && (int)DONE >= KOALA_MAX_NODES && STATE % 2 == 0 && DEAD % 2 == 0 && DEAD + 2 <= STATE,
              "room for every node, the bits at a multiple of eight bytes");
template <int NQ>
__global__ __launch_bounds__(NT) void k_accept_nodes(TreeTables tt, int T, int D, int V, float inv_tau, WalkArgs g, int batch,
                                                     int n_first, int *state) {
    extern __shared__ __attribute__((aligned(16))) f32q walk_q[];   // [NQ][NT]
    __shared__ WalkShared sh;
    const int b = blockIdx.x % batch, cur = blockIdx.x / batch, tid = threadIdx.x, l = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int *mine = state + (size_t)b * STATE;
    auto known = [&]() { return l < T ? __hip_atomic_load(mine + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0; };
    const int par = l < T ? tt.parent[l] : -2, rank = l < T ? tt.rank[l] : 0;
    NodeEnd e{0, 0, wave == 0};
    Branch br{(unsigned long long *)(mine + DEAD), 0};
    if (wave == 0)
        for (int x = cur; x != 0; x = __builtin_amdgcn_readlane(par, x)) br.line |= 1ull << x;
    bool off = false;
    if ((int)blockIdx.x >= n_first) {   // the waves may find different things out: the first one's decide
        if (tid == 0) sh.off = (br.told() & br.line) != 0;
        __syncthreads();
        off = sh.off != 0;
        __syncthreads();
    }
    if (!off) {
        walk_inputs(g, b, T, V, sh);
        e = walk_node<NQ, true>(g, b, cur, T, V, inv_tau, par, rank, walk_q + tid, sh, br);
        off = e.child < 0;
    }
    if (!e.mine) return;
    // one wave is left: the result is written through before the count moves
    int n = 0;
    if (l == 0) {
        if (!off) __hip_atomic_store(mine + cur, e.child > 0 ? e.child : -1 - e.token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        written_through();
        n = __hip_atomic_fetch_add(mine + DONE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (__builtin_amdgcn_readfirstlane(n) != T - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const int st = known();
    int at = 0, a = 0, on = l == 0 ? 0 : -1;   // lane l: the path's node at depth l
    for (int s = __builtin_amdgcn_readlane(st, 0); s > 0; s = __builtin_amdgcn_readlane(st, at)) {
        at = s;
        ++a;
        if (l == a) on = at;
    }
    if (l <= D) g.accept_path[(size_t)b * (D + 1) + l] = on;
    if (l == 0) {
        g.next_token[b] = -1 - __builtin_amdgcn_readlane(st, at);
        g.accept_len[b] = a;
        __hip_atomic_store(mine + DONE, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(br.dead, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (l < T) __hip_atomic_store(mine + l, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

namespace ks {

int max_vocab() { return MAX_SEG * SEG; }
int register_vocab() { return REG_V; }

void sample_children(hipStream_t st, const float *src, float *scratch, const NodeList &nodes, bool by_depth,
                     const TreeTables &tt, int T, int V, float temperature, const float *u_draw, int32_t *tree_tokens,
                     float *draft_logits, int batch) {
    const float it = 1.0f / temperature;
    const int grid = batch * nodes.n;
#define KOALA_DRAW(NQ) k_sample_children_r<NQ><<<grid, NT, 0, st>>>(src, nodes, by_depth, batch, tt, T, V, it, u_draw, tree_tokens, draft_logits)
    if (V <= REG_V / 8) KOALA_DRAW(1);
    else if (V <= REG_V / 2) KOALA_DRAW(4);
    else if (V <= REG_V) KOALA_DRAW(8);
    else k_sample_children<<<grid, NT, 0, st>>>(src, scratch, nodes, by_depth, batch, tt, T, V, it, u_draw, tree_tokens, draft_logits);
#undef KOALA_DRAW
}

void accept_sample(hipStream_t st, const TreeTables &tt, int T, int D, int V, float temperature,
                   const int32_t *tree_tokens, const float *target_logits, const float *draft_logits,
                   const float *u_accept, const float *u_resample, float *qv, float *dv, int *state, int n_cu, int32_t *accept_len,
                   int32_t *accept_path, int32_t *next_token, int batch) {
    const float it = 1.0f / temperature;
    const WalkArgs g{tree_tokens, target_logits, draft_logits, u_accept, u_resample, accept_len, accept_path, next_token};
    // Up to eight nodes a compute unit.  60 nodes of 32000 tokens, one workgroup a node against one a sequence, us at 1 / 8 / 16 /
    // 32 / 64 sequences: 21 / 35 / 49 / 58 / 74 against 81 / 81 / 94 / 98 / 100 where a target is near its draft, 38 / 45 / 45 /
    // 46 / 62 against 37 / 38 / 38 / 38 / 38 where every child of the root is turned down; 4000 tokens 10 / 14 / 15 / 19 / 25
    // against 21 / 29 / 29 / 29 / 29 and 14 / 17 / 18 / 20 / 25 against 13.  Beyond, nodes that the path leaves out cost a path
    // that ends at once more than they gain a long one.
    const bool nodes = T > 1 && (long)batch * T <= 8L * n_cu;
#define KOALA_WALK(NQ)                                                                                                  \
    {                                                                                                                  \
        static OncePerDevice once[2];                                                                                  \
        if (nodes) {                                                                                                   \
            allow_lds(once[0], (const void *)k_accept_nodes<NQ>, NQ * NT * 16);                                        \
            k_accept_nodes<NQ><<<batch * T, NT, NQ * NT * 16, st>>>(tt, T, D, V, it, g, batch, n_cu, state);           \
        } else {                                                                                                       \
            allow_lds(once[1], (const void *)k_accept_walk<NQ>, NQ * NT * 16);                                         \
            k_accept_walk<NQ><<<batch, NT, NQ * NT * 16, st>>>(tt, T, D, V, it, g);                                    \
        }                                                                                                              \
    }
    if (V <= REG_V / 8) KOALA_WALK(1)
    else if (V <= REG_V / 2) KOALA_WALK(4)
    else if (V <= REG_V) KOALA_WALK(8)
    else k_accept_sample<<<batch, NT, 0, st>>>(tt, T, D, V, it, tree_tokens, target_logits, draft_logits, u_accept, u_resample,
                                               qv, dv, accept_len, accept_path, next_token);
#undef KOALA_WALK
}

}  // namespace ks
