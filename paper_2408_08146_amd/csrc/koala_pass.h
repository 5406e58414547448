// Device code shared by the first kernel of a pass (fp32 and bf16 form) and by the kernels that hand out drafted tokens.
#pragma once

#include "koala_internal.h"

// What the first kernel of a pass works from.  mode 0: verification rows (node i of sequence b); mode 1: draft catch-up
// rows; mode 2: one draft tree level.
struct PassArgs {
    int mode;
    const int32_t *ctx_len;
    TreeTables tt;
    RowMeta meta;
    int T, rows_per_seq, m, d, n_exp, half;
    const double *inv_freq;
    const int32_t *tok;     // mode 0: [rows] node tokens; mode 1: [batch][m]; mode 2: [batch][T] node tokens
    const float *feat;      // mode 1: [batch][m][H] target features; mode 2: [batch][T][H] predicted features
    int32_t *root_tok;      // mode 1: [batch][T], entry 0 of a sequence receives its newest token
    float *root_score;      // mode 1: as root_tok, receives 0 (may be null)
};

// token of row r and, for the draft, the feature row beside it
__device__ __forceinline__ int pass_token(const PassArgs &a, int r, int H, const float *&f) {
    if (a.mode != 2) {
        f = a.mode == 1 ? a.feat + (size_t)r * H : nullptr;
        return a.tok[r];
    }
    const int b = r / a.rows_per_seq, u = a.tt.level_nodes[a.d * 64 + r % a.rows_per_seq];
    f = a.feat + ((size_t)b * a.T + a.tt.parent[u]) * H;
    return a.tok[b * a.T + u];
}

// metadata and rotary angles of row r, by one workgroup of at least 64 threads
__device__ __forceinline__ void pass_meta(const PassArgs &a, int r) {
    const int b = r / a.rows_per_seq, i = r % a.rows_per_seq;
    const int C = a.ctx_len[b];
    int pos, slot, nvis, base, kv_end;
    uint64_t mask;
    if (a.mode == 0) {
        pos = C + a.tt.depth[i]; slot = C + i; nvis = C; base = C; mask = a.tt.anc_mask[i]; kv_end = C + a.T;
    } else if (a.mode == 1) {
        pos = C - a.m + i; slot = pos; nvis = pos + 1; base = 0; mask = 0; kv_end = C;
    } else {
        const int u = a.tt.level_nodes[a.d * 64 + i];
        pos = C - 1 + a.d; slot = C + a.tt.exp_index[u]; nvis = C; base = C; mask = a.tt.draft_mask[u];
        kv_end = C + a.n_exp;
    }
    if (threadIdx.x == 0) {
        a.meta.row_b[r] = b; a.meta.row_pos[r] = pos; a.meta.row_slot[r] = slot; a.meta.row_nvis[r] = nvis;
        a.meta.row_base[r] = base; a.meta.row_mask[r] = mask;
        if (i == 0) a.meta.kv_end[b] = kv_end;
        if (a.mode == 1 && i == a.m - 1) {
            a.root_tok[b * a.T] = a.tok[r];
            if (a.root_score) a.root_score[b * a.T] = 0.f;
        }
    }
    for (int j = threadIdx.x; j < a.half; j += blockDim.x) {
        const double ang = (double)pos * a.inv_freq[j];
        a.meta.rope_cos[(size_t)r * a.half + j] = (float)cos(ang);
        a.meta.rope_sin[(size_t)r * a.half + j] = (float)sin(ang);
    }
}

// Row r of a top-k result hands its tokens to the children it decides, by their rank: EAGLE-style level d, row b * n_level +
// li, the children of that node; Medusa-style (n_level 0), row j * batch + b, all nodes of depth j + 1.  best / val hold the
// row's k winners in order.
__device__ __forceinline__ void fill_children(const ChildFill &f, int r, const int *best, const float *val) {
    for (int c = threadIdx.x; c < f.T; c += blockDim.x) {
        const int b = f.n_level ? r / f.n_level : r % f.batch;
        if (f.n_level ? f.tt.parent[c] != f.tt.level_nodes[f.d * 64 + r % f.n_level] : f.tt.depth[c] != r / f.batch + 1) continue;
        f.tree_tokens[b * f.T + c] = best[f.tt.rank[c]];
        if (f.scores) f.scores[b * f.T + c] = val[f.tt.rank[c]];
    }
}
