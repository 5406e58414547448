// Internal declarations shared by the library's translation units (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <stddef.h>
#include <atomic>
#include <string>
#include <vector>

#include "koala.h"

typedef uint16_t bf16_t;  // raw bfloat16 bit pattern

enum { KOALA_NSPLIT_MAX = 16, KOALA_TOPK_MAX = 16 };

// Per-row metadata of one pass (verify, draft catch-up, or one draft tree level).
// Row r of the pass belongs to sequence row_b[r]; its key/value go to cache slot
// row_slot[r]; it has rotary position row_pos[r]; it attends to cache slots
// [0, row_nvis[r]) and to slot row_base[r] + j for every set bit j of row_mask[r].
struct RowMeta {
    int32_t *row_b, *row_pos, *row_slot, *row_nvis, *row_base;
    uint64_t *row_mask;
    int32_t *kv_end;   // [batch]: one past the last slot any row of the sequence may see
    float *rope_cos, *rope_sin;  // [rows][head_dim/2]
};

// Device tables describing the static tree (uploaded at bind).
struct TreeTables {
    int32_t *parent, *depth, *rank;   // [T]
    uint64_t *anc_mask;               // [T] bit j: j is the node or one of its ancestors
    int32_t *exp_index;               // [T] index among expanded non-root nodes, or -1
    uint64_t *draft_mask;             // [T] bit e: expanded non-root ancestor-or-self with index e
    int32_t *level_nodes;             // [D][64] expanded nodes of each depth (-1 padded)
};

struct koala_ctx {
    koala_shape shape;
    koala_draft_shape draft;
    int T, D, max_batch, max_rows;  // max_rows = max_batch * max(T, max_m)
    std::vector<int32_t> parent, rank, topk, depth, exp_index;
    std::vector<uint64_t> anc_mask, draft_mask;
    std::vector<std::vector<int32_t>> level_exp;  // expanded nodes per depth
    int n_exp;                                    // expanded non-root nodes
    std::string err;

    bool bound;
    koala_weights w;
    std::vector<const void *> layer_w, draft_w;
    koala_kv kv;
    char *ws;
    size_t ws_bytes;

    // workspace carve-up (device pointers)
    TreeTables tt;
    RowMeta meta;
    float *x, *qrot, *o_part, *ml, *logits, *fhat;
    float *act, *attn_out, *block_y;                     // fp32: fc input or SwiGLU output, attention output, a Medusa block's product
    // generation loop state of sequence 0 (koala_generate)
    float *gen_dlogits, *gen_tlogits;                    // [T][V] draft / target logits of the non-greedy loop
    float *gen_feat, *gen_feat_in;                       // [T][H] verify features; [max(D+1, max_m)][H] next draft inputs
    int32_t *gen_tree, *gen_greedy, *gen_acc, *gen_path, *gen_next, *gen_tok_in;
    int n_cu;                      // compute units of the device the context is bound on
    int attn_ns;                   // key splits of the attention kernels (fixed at create)
    float *med_logits;                                   // [D * max_batch][V] per-depth logits of Medusa-style heads (sampled drafting)
    int *acc_state;                                      // [max_batch][ks::ACCEPT_STATE] cleared by koala_bind, left clear by every call
    float *acc_q, *acc_d;                                // [max_batch][V] distributions of the stochastic acceptance walk (rows in memory)
    // bf16 path: GEMM input as fp16 MFMA fragments, and the split-K partial sums
    void *xf, *xf2;   // xf2: input of the down projection (written by the gate/up projection's epilogue)
    float *part;
    size_t xf_bytes, part_bytes;
    void *qf;          // query fragments of the bf16 attention (in the buffer of qrot)
    int *attn_cnt;     // arrival counters of the attention kernel's split merge
    size_t opart_bytes, ml_bytes;
    float *cand_val;   // [rows][ceil(V/1024)][16] top-k candidates of the LM-head epilogue
    int *cand_idx;
    float *row_sums;   // [64 chunks][rows] sums of squares per 512-column chunk (RMSNorm row scale)
    int pend_S, pend_ld, pend_mode;  // partial sums waiting to be folded into x (0 = none)
    bool frags_ready;                // the next layer's input fragments and row sums are in place already

    // optional event timing of the GEMM launches (koala_profile_begin / _end)
    std::vector<hipEvent_t> prof_ev;
    int prof_used;
    double prof_bytes;
    bool prof_on;
};

// Which of a process's devices something has been done on.  Devices past the 64th are always new.
struct OncePerDevice {
    std::atomic<uint64_t> done{0};
    bool needed(int dev) const { return dev < 0 || dev >= 64 || !((done.load(std::memory_order_relaxed) >> dev) & 1u); }
    void mark(int dev) {
        if (dev >= 0 && dev < 64) done.fetch_or(1ull << dev, std::memory_order_relaxed);
    }
};
// Allows a kernel its dynamic LDS on the current device: a function's attribute is set per device.  A failure shows at
// the launch.
inline void allow_lds(OncePerDevice &once, const void *kernel, size_t bytes) {
    static const int n_devices = [] { int n = 0; return hipGetDeviceCount(&n) == hipSuccess ? n : 0; }();
    int dev = 0;   // a process that sees one device is spared the question with every launch (0.1 us each)
    if ((n_devices != 1 && hipGetDevice(&dev) != hipSuccess) || !once.needed(dev)) return;
    (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    once.mark(dev);
}

#define KOALA_CHECK_LAUNCH(ctx)                                              \
    do {                                                                     \
        hipError_t e__ = hipGetLastError();                                  \
        if (e__ != hipSuccess) {                                             \
            (ctx)->err = std::string("kernel launch failed: ") + hipGetErrorString(e__); \
            return KOALA_E_DEVICE;                                           \
        }                                                                    \
    } while (0)

struct PassArgs;   // koala_pass.h: what the first kernel of a pass works from

// Where the winners of a top-k go (tree_tokens null: nowhere): see fill_children in koala_pass.h
struct ChildFill {
    TreeTables tt;
    int n_level, d, batch, T;
    int32_t *tree_tokens;
    float *scores;
};

// ---------------------------------------------------------------------------------------------
// launchers implemented in kernels_generic.hip: bookkeeping shared by both model dtypes
// ---------------------------------------------------------------------------------------------
namespace kg {

PassArgs pass_args(const koala_ctx *c, int mode, int rows_per_seq, int m, int d);
// fp32 form of the first kernel of a pass: row metadata and rotary tables, and the embedded rows (mode 0: x [rows][H]) or the
// fc input [embedding ; feature] (modes 1, 2: x [rows][2H])
void pass_in(hipStream_t s, const PassArgs &a, const void *E, float *x, int rows, int H);
// fp32 features after the final norm
void rmsnorm(hipStream_t s, const float *x, const void *g, float *out, int rows, int H, float eps);
void resblock_update(hipStream_t s, float *x, const float *y, int n);
// k largest of each row, to idx / val (may be null) and to the nodes `fill` names
void topk_rows(hipStream_t s, const float *logits, int ld, int rows, int V, int k, int32_t *idx, float *val,
               const ChildFill &fill);

// draft bookkeeping
void gather_last_rows(hipStream_t s, const float *x, float *dst, size_t dst_stride, int batch, int m, int H);
void store_fhat(hipStream_t s, const float *x, float *fhat, const int32_t *level_nodes, int batch,
                int n_level, int T, int H);
void set_root(hipStream_t s, const int32_t *tok_in, int m, int32_t *tree_tokens, float *scores, int batch, int T);

void accept_scan(hipStream_t s, const TreeTables &tt, int T, int D, const int32_t *tree_tokens,
                 const int32_t *greedy, int32_t *accept_len, int32_t *accept_path, int32_t *next_token,
                 int batch);
// accept_scan and kv_commit in one launch
void accept_commit(hipStream_t s, bool bf16, const TreeTables &tt, int T, int D, const int32_t *tree_tokens, const int32_t *greedy,
                   void *kcache, void *vcache, const int32_t *ctx_len, int32_t *accept_len, int32_t *accept_path,
                   int32_t *next_token, int n_layers, int max_batch, int batch, int n_heads, int capacity, int head_dim);
void kv_commit(hipStream_t s, bool bf16, void *kcache, void *vcache, const int32_t *ctx_len,
               const int32_t *accept_len, const int32_t *accept_path, int D, int n_layers,
               int max_batch, int batch, int n_heads, int capacity, int head_dim);
void advance_ctx(hipStream_t s, int32_t *ctx_len, const int32_t *accept_len, int batch);
// measurement aid: read `bytes` (multiple of 16) once with streaming loads
void stream_read(hipStream_t s, const void *src, size_t bytes, unsigned *sink);
// generation loop: next draft inputs (rows 0..a) and emitted tokens from the accepted path of sequence 0
void gen_next(hipStream_t s, const float *feat_out, const int32_t *tree_tokens, const int32_t *accept_len,
              const int32_t *accept_path, const int32_t *next_token, int T, int D, int H, float *feat_next,
              int32_t *tok_next, int32_t *out_tokens, int n_done, int max_new);

}  // namespace kg

// ---------------------------------------------------------------------------------------------
// launchers implemented in kernels_fp32.hip (fp32 model: row-major weights and caches)
// ---------------------------------------------------------------------------------------------
namespace kf {

// Y[M,N] (ldy) = or += X[M,K] (ldx) * W[N,K]^T
void gemm(hipStream_t st, const float *X, int ldx, const void *W, float *Y, int ldy, int M, int N, int K, bool add);
// QKV projection of RMSNorm(X): rotated queries to qrot [rows][H], keys and values to their cache slots
void norm_qkv(hipStream_t st, const float *X, const void *gain, float eps, const void *W, const RowMeta &meta, float *qrot,
              void *kc, void *vc, int rows, int H, int n_heads, int head_dim, int cap);
// act[rows][F] = SiLU(gate) * up of RMSNorm(X)
void norm_swiglu(hipStream_t st, const float *X, const void *gain, float eps, const void *W, float *act, int rows, int F, int H);
void attention(hipStream_t st, const float *qrot, const RowMeta &meta, const void *kc, const void *vc, float *o_part, float *ml,
               float *out, int batch, int rows_per_seq, int n_heads, int head_dim, int cap, int max_split);

}  // namespace kf

// ---------------------------------------------------------------------------------------------
// launchers implemented in kernels_sampling.hip (non-greedy drafting and acceptance, section 2.2)
// ---------------------------------------------------------------------------------------------
namespace ks {

enum { ACCEPT_STATE = 80 };   // whole numbers of state a sequence, see accept_sample
int max_vocab();        // largest vocabulary the sampling kernels handle
int register_vocab();   // and the largest whose rows they hold in registers: beyond, they need scratch

// the nodes whose children are drawn in one launch, handed over by value
struct NodeList {
    int n;
    uint8_t node[KOALA_MAX_NODES], depth[KOALA_MAX_NODES];
};
// Children of the listed nodes get draws without replacement from softmax(logits / temperature); the logits are copied to
// draft_logits[b][node].  src: the logits, row depth * batch + b (by_depth) or b * n + index in the list.  scratch:
// [batch * n][V], may be src unless by_depth (used for vocabularies above 32768 only).
void sample_children(hipStream_t st, const float *src, float *scratch, const NodeList &nodes, bool by_depth,
                     const TreeTables &tt, int T, int V, float temperature, const float *u_draw, int32_t *tree_tokens,
                     float *draft_logits, int batch);
// state: [batch][ACCEPT_STATE], zero before the first call and zero again after each.  qv, dv: [batch][V], used for vocabularies above 32768.
void accept_sample(hipStream_t st, const TreeTables &tt, int T, int D, int V, float temperature,
                   const int32_t *tree_tokens, const float *target_logits, const float *draft_logits,
                   const float *u_accept, const float *u_resample, float *qv, float *dv, int *state, int n_cu,
                   int32_t *accept_len, int32_t *accept_path, int32_t *next_token, int batch);

}  // namespace ks

// ---------------------------------------------------------------------------------------------
// launchers implemented in kernels_bf16.hip (fragment-major weights and activations in fp16)
// ---------------------------------------------------------------------------------------------
namespace kb {

enum { GEMM_HEADS = 8 };   // matrices of one gemm_rows_heads launch, at most
// number of 16-row activation tiles used for `rows` rows: 1, 2 or a multiple of 4
inline int mt_of(int rows) { return rows <= 16 ? 1 : rows <= 32 ? 2 : 4 * ((rows + 63) / 64); }
inline int pad64(int n) { return (n + 63) / 64 * 64; }

inline size_t xf_bytes(int K, int MT) { return (size_t)(K / 32) * MT * 1024; }
// a packed bf16 weight matrix of n_elements values (a multiple of 8) to the fp16 the GEMMs multiply with, in place
void weights_to_f16(hipStream_t st, void *w, size_t n_elements);

// Pending RMSNorm row scale: 1/sqrt(sum_c sums[c][row] / K + eps); sums == nullptr means scale 1.
struct NormScale {
    const float *sums;
    int nparts, srows, K;
    float eps;
};

int gemm_splits(int Npad, int K, int MTT = 0);       // split count of gemm_packed; MTT: activation tiles of the call (0: at most four)
int rows_splits(int Npad, int K, int n_heads = 1);   // split count of gemm_rows_partial / _heads
// P[S][MTT*16][Npad] = partial sums of X * W^T, X given as fp16 fragments [K/32][MTT][64] x 16 B
// ev_start/ev_stop (either may be null) are attached to the dispatch: they take the kernel's own begin and end times
void gemm_packed(hipStream_t st, const void *Wp, const void *Xf, float *P, int Npad, int K, int MTT, int S,
                 hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
// Row-group GEMM (one workgroup per few 16-row groups of the weights and K range, waves take 64-k tiles in
// turn; n_cu = compute units of the device, which sets the groups per workgroup), MTT = 1, 2 or 4:
// _partial: P[S][MTT*16][Npad] partial sums, like gemm_packed;  _qkv (S = 1): row scale, rotary embedding,
// queries as attention fragments qf, keys/values into their cache slots (W_q, W_k rows pair-interleaved);  _swiglu (S = 1): row
// scale, SiLU(gate) * up as fragments Xo of the down projection's input
void gemm_rows_partial(hipStream_t st, const void *Wp, const void *Xf, float *P, int Npad, int K, int MTT, int S,
                       hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
// Up to 64 rows against a matrix of which a workgroup takes eight row groups and finishes them (one split, so P holds finished
// sums), where that is one round of compute units and at least five eighths of one: an LM head of 20481 to 32768 tokens.
// Measured at 4096 columns, with the top-k behind it, us at 1 / 26 / 64 rows, against gemm_packed: 16000 tokens 32 / 36 / 47
// against 30 / 35 / 42, 20000 34 / 38 / 47 against 35 / 40 / 48, 24000 36 / 39 / 49 against 40 / 45 / 54, 28600 41 / 44 / 53
// against 49 / 54 / 64, 32768 46 / 49 / 57 against 52 / 57 / 68, 33000 (two rounds) 64 / 70 / 87 against 53 / 60 / 69.
bool rows_wide(int Npad, int n_cu);
void gemm_rows_wide(hipStream_t st, const void *Wp, const void *Xf, float *P, int Npad, int K, int MTT, hipEvent_t ev_start = nullptr,
                    hipEvent_t ev_stop = nullptr);
// n matrices W[h] of one shape on the same input: P[n][S][MTT*16][Npad]
void gemm_rows_heads(hipStream_t st, const void *const *W, int n, const void *Xf, float *P, int Npad, int K, int MTT, int S,
                     hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
void gemm_rows_qkv(hipStream_t st, const void *Wp, const void *Xf, int K, int MTT, const NormScale &ns, int rows,
                   int rows_per_seq, const RowMeta &meta, void *qf, void *kc, void *vc, int H, int n_heads, int head_dim,
                   int cap, int n_cu, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
void gemm_rows_swiglu(hipStream_t st, const void *Wp, const void *Xf, int K, int MTT, const NormScale &ns, int rows,
                      void *Xo, int F, int n_cu, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
// GEMM for many activation rows (MTT >= 8 tiles): P[S][MTT*16][Npad] partial sums; big_shape picks the launch
struct BigShape { int n_mt, n_pm, mtw, U, S, n_full; };
BigShape big_shape(int Npad, int K, int rows, int n_cu, bool epilogue = false, size_t room = 0, int n_cnt = 0);
void gemm_big(hipStream_t st, const void *Wp, const void *Xf, float *P, int Npad, int K, int MTT, const BigShape &b,
              hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
void gemm_big_qkv(hipStream_t st, const void *Wp, const void *Xf, int K, int MTT, const BigShape &b, const NormScale &ns,
                  int rows, int rows_per_seq, const RowMeta &meta, void *qf, void *kc, void *vc, int H, int n_heads,
                  int head_dim, int cap, float *scratch, size_t room, int *counters, hipEvent_t ev_start = nullptr,
                  hipEvent_t ev_stop = nullptr);
void gemm_big_swiglu(hipStream_t st, const void *Wp, const void *Xf, int K, int MTT, const BigShape &b,
                     const NormScale &ns, int rows, void *Xo, int F, float *scratch, size_t room, int *counters,
                     hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
// The LM head of V tokens with its logits finished in the GEMM (gemm_rows_logits up to 64 rows, gemm_big_logits for MTT >= 8):
// logits (may be null) [rows][V], and per row and workgroup (rows_logits_groups or big_groups of them) the largest logit and its
// token to cand_val / cand_idx (may be null), which best_logit merges.  rows_logits_groups is 0 where the vocabulary is more
// than one round of compute units with eight row groups each (32768 tokens on 256).
int rows_logits_groups(int Npad, int n_cu);
int big_groups(int Npad, const BigShape &b);
void gemm_rows_logits(hipStream_t st, const void *Wp, const void *Xf, int K, int MTT, const NormScale &ns, int rows,
                      float *logits, int V, float *cand_val, int *cand_idx, int n_cu, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
void gemm_big_logits(hipStream_t st, const void *Wp, const void *Xf, int K, int MTT, const BigShape &b, const NormScale &ns,
                     int rows, float *logits, int V, float *cand_val, int *cand_idx, float *scratch, size_t room, int *counters,
                     hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
// v = (mode 1: x +) sum of partials (mode 0: x as is); x <- v for modes 1, 2; Xf (may be NULL) receives the
// fragments of gain * v (gain NULL: v); sums (may be NULL) the sums of squares of v per 512-column chunk
void fold(hipStream_t st, float *x, int ldx, const float *P, int S, int Mp, int ldp, int mode, int M, int N,
          const void *gain, void *Xf, int MT, float *sums, int srows);
// qf: query fragments [batch][n_heads][ceil(rows_per_seq/16)][head_dim/32][hi, lo][64 lanes] x 16 B, times
// 1/sqrt(head_dim)
void rope_append(hipStream_t st, const float *P, int S, int Mp, int ldp, const NormScale &ns, const RowMeta &meta,
                 void *qf, void *kc, void *vc, int rows, int H, int n_heads, int head_dim, int cap, int rows_per_seq);
// tree-masked attention over the cache, key splits merged in the kernel, rows written as fragments Xf of the
// O projection's input; counters: max_batch * n_heads * 4 ints, zero before the first launch
void attention_tree(hipStream_t st, const void *qf, const RowMeta &meta, const void *kc, const void *vc, float *o_part,
                    size_t opart_bytes, float *ml, size_t ml_bytes, int *counters, void *Xf, int MT_out, int batch,
                    int rows_per_seq, int n_heads, int head_dim, int cap, int nsplit);
void silu_frag(hipStream_t st, const float *P, int S, int Mp, int ldp, const NormScale &ns, void *Xf, int MT, int M,
               int F);
// First kernel of a pass: row metadata and rotary tables, and mode 0: the embedded rows x, fragments of gain * x and chunk
// sums of squares; modes 1, 2: fragments of the fc input [embedding ; feature]
void pass_in(hipStream_t st, const PassArgs &a, const void *E, const void *gain, float *x, void *Xf, float *sums, int srows,
             int rows, int H, int MT);
// Last kernel of a draft pass: x + pending partials -> fhat, and their fragments.  Level pass: every row b * n_level + li to
// fhat[b][node]; catch-up pass (level_nodes null): row b * m + m - 1 to fhat[b][0]
void head_out(hipStream_t st, const float *x, const float *P, int S, int Mp, float *fhat, const int32_t *level_nodes, int n_level,
              int m, int T, void *Xf, int MT, int rows_out, int H);
// rows of x and their fragments: the newest feature of sequence row % batch; and each sequence's root
void medusa_in(hipStream_t st, const float *feat, const int32_t *tok_in, float *x, void *Xf, int batch, int m, int rows, int H,
               int MT, int T, int32_t *root_tok, float *root_score);
// x[r] += SiLU(partials of row r - p0) and (Xf not null) the fragments of the new x, r = r0 .. r0 + rows - 1;
// P[head][S][Mp][H], batch rows a head
void resblock_p(hipStream_t st, float *x, void *Xf, const float *P, int S, int Mp, int batch, int r0, int p0, int rows, int H,
                int MT);
// the k largest logits of each row (k = 0: none, the logits are only written) to idx / val (may be null) and to the nodes
// `fill` names; feat (may be null): the rows after the final norm
struct FeatOut { const float *x; const void *gain; float *feat; int H; };
void logits_topk(hipStream_t st, const float *P, int S, int Mp, int ldp, const NormScale &ns, float *logits, int ldl,
                 int rows, int V, int k, float *cand_val, int *cand_idx, int32_t *idx, float *val, const ChildFill &fill,
                 const FeatOut &fo);
// the best of a row's n_cand <= 1024 candidates to idx, and the rows after the final norm
void best_logit(hipStream_t st, const float *cand_val, const int *cand_idx, int n_cand, int rows, int32_t *idx,
                const NormScale &ns, const FeatOut &fo);

}  // namespace kb
