// Adversarial training step of a draft head (section 3.2, Algorithm 1, Eq. 5 and 6) in fp32: the
// discriminator's forward and backward passes with its gradient-descent update, the draft-head loss and its
// gradient at the logits, and the forward pass / backward pass / update of a Medusa-style head.  Dense
// products run on the matrix pipe with fp32 operands cut into three bfloat16 pieces; the rest is small row-wise kernels.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "koala_internal.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
struct __attribute__((packed, aligned(4))) f32x4_any { float x, y, z, w; };   // 16 bytes at a 4-byte aligned address
typedef float __attribute__((ext_vector_type(4), aligned(4))) f32x4_a4;   // as vectors: loaded, kept and used as one
typedef float __attribute__((ext_vector_type(2), aligned(4))) f32x2_a4;

// ---------------------------------------------------------------------------------------------
// fp32 products on the 16-bit matrix pipe: C[M,N] = sum_k Q(m,k) P(n,k).
//
// A float is the exact sum of three bfloat16 values (round to nearest, subtract, twice: the rest has 16, then eight
// significant bits, so every subtraction and the last piece are exact), so a product of two floats is the sum of nine
// bfloat16 products, each exact in the fp32 accumulator of the MFMA.  Six of them are kept; the other three come to at most
// 2^-24 of the product, with either sign, and to 2^-27 root mean square (pieces cut off instead of rounded cost as much but
// leave up to 2^-21, always towards zero).  The products of two first pieces have an accumulator of their own, rounded once
// per 32 terms; the others are 2^-8 of them and meet it once, at the end.  Error of a sum of K random terms, measured, as a
// multiple of the same sum in fp32 MFMAs (which round with every term): 1.03 at one term, 0.85 at two, 0.5 at eight,
// 0.35 at 64, 0.33 at 1024.
// Six 16x16x32 MFMAs (16 cycles each) do the work of eight 16x16x4 fp32 MFMAs (32 cycles each), so the pipe is 2.7 times
// as fast as in fp32.
//
// Workgroup of 256 threads on a tile of 64 n x BM m; K in chunks of 32.  Both operands of a chunk go from memory to
// registers (up to 64 rows four chunks ahead, else two), are cut into their three planes there and put into LDS as MFMA
// fragments, double-buffered with one barrier a chunk.  P is the MFMA's row operand: a lane then holds four consecutive n of
// one m, a 16-byte piece of a row of C.
//   k-contiguous (KS false; Q is): element (i, k) at i * ld + k;  8 threads x 16 B cover 128 B of a row
//   k-strided    (KS true):        element (i, k) at k * ld + i;  a thread takes 8 consecutive k of one i, the eight values
//                                  of a fragment lane
// LDS plane of a 16-row tile: 64 slots of 16 B, lane (i, g = k/8) in slot (i ^ 4 g) + 16 g: the 8-byte stores of 32 lanes of
// the k-contiguous form (four rows, all g) then fall into different banks.
// Rows past the end re-read the last one (never stored); k past the end is zero in both operands.  Where pieces do not stand
// for an operand of the tile (an infinity, or all of it below 2^-102: the MFMA takes pieces below 2^-126 as zero) the tile is
// summed again on the fp32 pipe, so that it comes out as it does there.  Values below 2^-102 beside larger ones
// are off by up to 2^-125.  In input gradients (KS) Q is taken times 2^24 instead, and pieces stand for all of its values: the
// gradients of a discriminator that no longer errs are such, and summing again took 109 us instead of 28 (40 x 32000 from K = 1024).
// Sums that overflow for it are summed again.
// grid: x = n tiles x m blocks, the m blocks of an n tile on one die (indices 8 apart), y = K splits.  A
// split's sums go to out[split][M][N], for k_sum_parts where there are several.
// Its products are the small ones, of few chunks or few tiles (gemm_weights), and what bounds them is latency: a start, and a
// round trip a chunk.  The others are k_stream_x3's, the updates k_update_x3's and k_update_rows' (all below).
// Registers for four workgroups a compute unit up to 32 rows (room for three is as fast: forward pass of a head of 512 x 4000 at 20
// rows 20.6 us and 20.4), two beyond (three spill with 128 rows: 256 x 1000 at 100 rows 21 -> 36 us).
// ---------------------------------------------------------------------------------------------
enum { X3_BN = 64, X3_BK = 32 };

// The mapped hidden state z[p][v] joined to a logits row: u[p] = z + la[p] and, with lb, u[n + p] = z + lb[p], nV elements on.
struct Join { const float *la, *lb; long nV; };
// elements lo .. hi - 1 of the four at `at` of an output; vec: they are 16-byte aligned in every matrix
__device__ __forceinline__ void put4(float *out, const Join &j, long at, f32x4 v, int lo, int hi, bool vec) {
    if (vec && lo <= 0 && hi >= 4) {
        if (!j.la) { *(f32x4 *)(out + at) = v; return; }
        *(f32x4 *)(out + at) = v + *(const f32x4 *)(j.la + at);
        if (j.lb) *(f32x4 *)(out + j.nV + at) = v + *(const f32x4 *)(j.lb + at);
        return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (r >= lo && r < hi) {
            out[at + r] = j.la ? v[r] + j.la[at + r] : v[r];
            if (j.lb) out[j.nV + at + r] = v[r] + j.lb[at + r];
        }
}
bool join_aligned(const Join &j) { return (((uintptr_t)j.la | (uintptr_t)j.lb) & 15) == 0 && j.nV % 4 == 0; }

// a and b as pairs of pieces; top: the largest magnitude so far
__device__ __forceinline__ void split3(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l, float &top) {
    auto round2 = [](float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x, y}, bf16x2)); };
    auto low = [](uint32_t p) { return __uint_as_float(p << 16); };
    auto high = [](uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); };
    h = round2(a, b);
    const float ra = a - low(h), rb = b - high(h);
    m = round2(ra, rb);
    l = round2(ra - low(m), rb - high(m));
    top = fmaxf(fmaxf(fabsf(a), fabsf(b)), top);
}
// whether pieces stand for an operand of this largest magnitude: not where one is infinite or rounds to infinity in bfloat16,
// nor where all are so small (but not zero) that their last pieces are below 2^-126, which the MFMA takes as zero.  Not-a-numbers
// pass: their pieces are some as well.
// up: of the operand times 2^24.  Every float is then a multiple of 2^-125, and so are its pieces: none is below the smallest
// normal bfloat16.
constexpr float x3_up(bool up) { return up ? 0x1p24f : 1.f; }
constexpr float x3_down(bool up) { return up ? 0x1p-24f : 1.f; }
__device__ __forceinline__ bool pieces_hold(float top, bool up) { return top < 0x1.ffp127f && (up || top >= 0x1p-102f || top == 0.f); }

// One operand's share of a chunk in a thread's registers, and its way into LDS.  T rows (32, 64 or 128).
template <int T, bool KS, int DEPTH, bool UP>
struct X3Loader {
    static_assert(!KS || T == 64, "k-strided: a wave per eight k");
    static constexpr int PER = T * X3_BK / 256;              // floats per thread
    static constexpr int TILE = 64;                          // 16-byte units of a plane of one 16-row tile
    const float *p;
    long ld;
    int rows, i0, K;
    float v[DEPTH][PER];

    __device__ __forceinline__ void init(const float *base, long ld_, int rows_, int i0_, int K_) {
        p = base; ld = ld_; rows = rows_; i0 = i0_; K = K_;
    }
    template <int SLOT>
    __device__ __forceinline__ void load(int k0) {
        const int t = threadIdx.x;
        float *d = v[SLOT];
        if (!KS) {
            const int k = k0 + 4 * (t & 7);
#pragma unroll
            for (int q = 0; q < T / 32; ++q) {
                const float *src = p + (long)min(i0 + (t >> 3) + 32 * q, rows - 1) * ld + k;
                if (k0 + X3_BK <= K) {
                    const f32x4_any w = *(const f32x4_any *)src;
                    d[4 * q] = w.x; d[4 * q + 1] = w.y; d[4 * q + 2] = w.z; d[4 * q + 3] = w.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) d[4 * q + e] = k + e < K ? src[e] : 0.f;
                }
            }
        } else {
            const int g = t >> 6, i = min(i0 + (t & 63), rows - 1);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = k0 + 8 * g + e;
                const float x = p[(long)min(k, K - 1) * ld + i];
                d[e] = k < K ? x : 0.f;
            }
        }
    }
    template <int SLOT>
    __device__ __forceinline__ void store(u32x4 *lds, float &top) const {   // planes [3][T/16][64]
        const int t = threadIdx.x;
        const float *d = v[SLOT];
        if (!KS) {
            const int g = (t & 7) >> 1;
#pragma unroll
            for (int q = 0; q < T / 32; ++q) {
                const int i = (t >> 3) + 32 * q;
                uint32_t h[2], m[2], l[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) split3(x3_up(UP) * d[4 * q + 2 * e], x3_up(UP) * d[4 * q + 2 * e + 1], h[e], m[e], l[e], top);
                unsigned char *dst = (unsigned char *)(lds + (i >> 4) * TILE + ((i & 15) ^ (4 * g)) + 16 * g) + 8 * (t & 1);
                constexpr int PL = (T / 16) * TILE * 16;
                *(u32x2 *)dst = (u32x2){h[0], h[1]};
                *(u32x2 *)(dst + PL) = (u32x2){m[0], m[1]};
                *(u32x2 *)(dst + 2 * PL) = (u32x2){l[0], l[1]};
            }
        } else {
            const int g = t >> 6, i = t & 63;
            uint32_t h[4], m[4], l[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) split3(d[2 * e], d[2 * e + 1], h[e], m[e], l[e], top);
            u32x4 *dst = lds + (i >> 4) * TILE + ((i & 15) ^ (4 * g)) + 16 * g;
            dst[0] = (u32x4){h[0], h[1], h[2], h[3]};
            dst[(T / 16) * TILE] = (u32x4){m[0], m[1], m[2], m[3]};
            dst[2 * (T / 16) * TILE] = (u32x4){l[0], l[1], l[2], l[3]};
        }
    }
};

template <int BM, bool PKS, int DEPTH>
__global__ __launch_bounds__(256, BM == 32 ? 4 : 2) void k_gemm_x3(const float *__restrict__ P, long ldp, const float *__restrict__ Q,
                                                    long ldq, float *out, int M, int N, int K, int vec, Join join) {
    constexpr int WN = BM == 32 ? 4 : 2, WM = 4 / WN;        // waves along n and m
    constexpr int TN = X3_BN / 16 / WN, TM = BM / 16 / WM;   // accumulator tiles of a wave
    constexpr int PU = 3 * (X3_BN / 16) * 64, QU = 3 * (BM / 16) * 64;   // 16-byte units of a chunk's planes
    extern __shared__ __attribute__((aligned(16))) u32x4 x3_lds[];   // [2][PU + QU]
    const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, li = l & 15, lg = l >> 4;
    const int wn = wave % WN, wm = wave / WN;
    const int nmb = (M + BM - 1) / BM, ntile = (N + X3_BN - 1) / X3_BN;
    const int die = blockIdx.x & 7, rnd = blockIdx.x >> 3;
    const int nt = (rnd / nmb) * 8 + die, mb = rnd % nmb;
    if (nt >= ntile) return;                                 // the grid is padded to whole rounds of eight
    const int n0 = nt * X3_BN, m0 = mb * BM;
    const int nch = (K + X3_BK - 1) / X3_BK, S = gridDim.y;
    const int c0 = (int)((unsigned)(blockIdx.y * nch) / (unsigned)S), c1 = (int)((unsigned)((blockIdx.y + 1) * nch) / (unsigned)S);
    X3Loader<X3_BN, PKS, DEPTH, false> lp;
    X3Loader<BM, false, DEPTH, PKS> lq;
    lp.init(P, ldp, N, n0, K);
    lq.init(Q, ldq, M, m0, K);
    // the products of the first pieces, and all the others, which are 2^-8 of them: small as they are, the second sum's
    // roundings are lost in the first one's, which is rounded once a chunk
    f32x4 acc[TN][TM], low[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = low[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](int c, auto sc) __attribute__((always_inline)) {
        constexpr int B = decltype(sc)::value;
        if (c < c1) { lp.template load<B>(c * X3_BK); lq.template load<B>(c * X3_BK); }
    };
    fetch(c0, std::integral_constant<int, 0>{});
    fetch(c0 + 1, std::integral_constant<int, 1>{});
    if constexpr (DEPTH == 4) {
        fetch(c0 + 2, std::integral_constant<int, 2>{});
        fetch(c0 + 3, std::integral_constant<int, 3>{});
    }
    const int slot = (li ^ (4 * lg)) + 16 * lg;
    float ptop = 0.f, qtop = 0.f;   // largest magnitudes
    auto chunk = [&](int c, auto sc) __attribute__((always_inline)) {
        constexpr int B = decltype(sc)::value;
        u32x4 *lds = x3_lds + (B & 1) * (PU + QU);
        lp.template store<B>(lds, ptop);
        lq.template store<B>(lds + PU, qtop);
        fetch(c + DEPTH, sc);
        // a bare barrier behind this wave's LDS writes: the fence of __syncthreads would wait for the loads too
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        bf16x8 a[3][TN];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
#pragma unroll
            for (int i = 0; i < TN; ++i)
                a[pl][i] = __builtin_bit_cast(bf16x8, lds[(pl * (X3_BN / 16) + wn * TN + i) * 64 + slot]);
        // small terms first.  Up to 32 rows one row tile's fragments at a time, which leaves registers for four workgroups a
        // compute unit; else all of them, whose reads are then over before the first MFMA
        constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0}, JT = BM == 32 ? 1 : TM;
#pragma unroll
        for (int j0 = 0; j0 < TM; j0 += JT) {
            bf16x8 b[3][JT];
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int j = 0; j < JT; ++j)
                    b[pl][j] = __builtin_bit_cast(bf16x8, lds[PU + (pl * (BM / 16) + wm * TM + j0 + j) * 64 + slot]);
#pragma unroll
            for (int z = 0; z < 6; ++z)
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int j = 0; j < JT; ++j) {
                        f32x4 &sum = z == 5 ? acc[i][j0 + j] : low[i][j0 + j];
                        sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[PA[z]][i], b[PB[z]][j], sum, 0, 0, 0);
                    }
        }
    };
    static_assert(DEPTH == 2 || DEPTH == 4, "a chunk's registers and its LDS buffer go by the chunk number");
    for (int c = c0; c < c1; c += DEPTH) {
        chunk(c, std::integral_constant<int, 0>{});
        if (c + 1 < c1) chunk(c + 1, std::integral_constant<int, 1>{});
        if constexpr (DEPTH == 4) {
            if (c + 2 < c1) chunk(c + 2, std::integral_constant<int, 2>{});
            if (c + 3 < c1) chunk(c + 3, std::integral_constant<int, 3>{});
        }
    }
    bool finite = true;   // PKS: every sum
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                f32x4 &sum = acc[i][j];
                if (PKS) {   // one that has overflowed is taken anew below, whatever the small terms make of it
                    sum[r] = (sum[r] + low[i][j][r]) * x3_down(PKS);
                    finite &= fabsf(sum[r]) < INFINITY;
                } else         // it stays as it is: the small terms may be of the other sign
                    sum[r] += fabsf(sum[r]) < INFINITY ? low[i][j][r] : 0.f;
            }
    // every thread has cut up its share of both operands: the tile's largest magnitudes
    __shared__ float tops[2][4];
    for (int o = 32; o > 0; o >>= 1) { ptop = fmaxf(ptop, __shfl_xor(ptop, o)); qtop = fmaxf(qtop, __shfl_xor(qtop, o)); }
    if (l == 0) { tops[0][wave] = ptop; tops[1][wave] = qtop; }
    __syncthreads();
    ptop = fmaxf(fmaxf(tops[0][0], tops[0][1]), fmaxf(tops[0][2], tops[0][3]));
    qtop = fmaxf(fmaxf(tops[1][0], tops[1][1]), fmaxf(tops[1][2], tops[1][3]));
    if (!pieces_hold(ptop, false) || !pieces_hold(qtop, PKS) || !__all(finite)) {
        // the tile once more on the fp32 matrix pipe (16x16x4: lane (i, g) holds k = g of row i), sixteen k a step
        const int kend = min(K, c1 * X3_BK);
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int k0 = c0 * X3_BK; k0 < kend; k0 += 16) {
            float pv[4][TN], qv[4][TM];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = k0 + 4 * e + lg;
                const long kc = min(k, kend - 1);
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    const long n = min(n0 + (wn * TN + i) * 16 + li, N - 1);
                    const float x = P[PKS ? kc * ldp + n : n * ldp + kc];
                    pv[e][i] = k < kend ? x : 0.f;
                }
#pragma unroll
                for (int j = 0; j < TM; ++j) {
                    const long m = min(m0 + (wm * TM + j) * 16 + li, M - 1);
                    const float x = Q[m * ldq + kc];
                    qv[e][j] = k < kend ? x : 0.f;
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int j = 0; j < TM; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[e][i], qv[e][j], acc[i][j], 0, 0, 0);
        }
    }
    out += (long)blockIdx.y * M * N;
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            const int m = m0 + (wm * TM + j) * 16 + li, n = n0 + (wn * TN + i) * 16 + 4 * lg;
            if (m < M) put4(out, join, (long)m * N + n, acc[i][j], 0, N - n, vec);
        }
}

// ---------------------------------------------------------------------------------------------
// The same products for a weight matrix that streams past the activations, the forward and backward passes' form:
// C[M,N] = sum_k Q(m,k) P(n,k), Q k-contiguous, P k-contiguous (KS false) or k-strided (KS true).
//
// Workgroup of eight waves on 128 n x up to 128 m (MT row tiles), K in stages of 64: waves 0..3 take the first 32 k of every
// stage, waves 4..7 the others, each wave 32 n.  A weight goes from memory straight to the wave that multiplies with it: a
// lane loads the eight k of a fragment lane (two 16-byte pieces of its row; KS: two neighbouring n of eight k) and cuts them
// in registers, PF stages ahead.  The activations of a stage are loaded, cut and put into LDS by all threads, double-buffered
// with one barrier a stage.  Waves 0..3 do their cutting at the start of a stage and waves 4..7 at its end, so that of the two
// waves of a SIMD one has matrix work while the other cuts.  The two halves' sums meet in LDS.
// k of fragment lane (i, g): element e < 4 is 4 g + e, the others 16 + 4 g + e - 4, so that the 16-byte pieces of the four
// lanes of a row are 64 contiguous bytes.  The order of k within a fragment is free as long as both operands agree.
// No load is conditional or bounded, so that the compiler can count those under way: a wave's n and the last stage's k are
// moved back to where the matrix ends (columns that are another wave's are not stored, k that were another stage's are zero
// in Q; where a weight there is infinite the tile is summed anew below), stages past the last re-read it.
// grid: x = n tiles x m blocks, the m blocks of an n tile on one die, y = K splits.
// N >= 32, K >= 64, ldp and ldq < 2^23 (32-bit offsets).
// Measured within training steps, by kernel trace, against the form above (both operands through LDS): 20 x 32000 from K = 4096
// 115 (in two splits, joined by a further launch) -> 97 us (5.4 TB/s), where the step before has just updated that matrix
// 137 -> 127 (4.1 TB/s), with three models in turn 172 -> 153; 40 x 1024 from K = 32000 53 -> 41; 40 x 32000 from K = 1024 (KS)
// 54 -> 34; 128 x 32000 from K = 4096 273 -> 181 (six products of pieces: 1.11 PFLOP/s in bfloat16, what a large product reaches
// here); 128 x 4096 from K = 32000 (KS) 299 -> 186.
// The stream bounds up to 64 rows (without its MFMAs the kernel takes as long), the matrix pipe beyond.
// ---------------------------------------------------------------------------------------------
template <int MT, bool KS, bool KT>
__global__ __launch_bounds__(512, 2) void k_stream_x3(const float *__restrict__ P, long ldp, const float *__restrict__ Q, long ldq,
                                                      float *out, int M, int N, int K, int vec, Join join) {
    constexpr int TN = 2, NQ = (MT + 1) / 2;                        // n tiles of a wave, rows of Q a thread
    constexpr int PF = MT >= 6 ? 2 : MT == 2 ? 4 : 3, QF = MT >= 6 ? 1 : PF;   // stages of P and of Q under way
    constexpr int PL = 2 * NQ * 64, ST = 2 * 3 * PL;                // 16-byte units of a plane of 32 k, of a stage
    extern __shared__ __attribute__((aligned(16))) u32x4 x3s[];     // [2][ST]
    __shared__ float tops[8];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, li = l & 15, lg = l >> 4;
    const int kg = wave >> 2, wn = wave & 3;
    const int nmb = (M + MT * 16 - 1) / (MT * 16), ntile = (N + 127) / 128;
    const int die = blockIdx.x & 7, rnd = blockIdx.x >> 3;
    const int nt = (rnd / nmb) * 8 + die, m0 = rnd % nmb * (MT * 16);
    if (nt >= ntile) return;                                 // the grid is padded to whole rounds of eight
    const int nown = nt * 128 + wn * 32, n0 = min(nown, N - 32);   // this wave's columns start at nown
    const int nst = (K + 63) / 64, S = gridDim.y;
    const int s0 = (int)((unsigned)(blockIdx.y * nst) / (unsigned)S), s1 = (int)((unsigned)((blockIdx.y + 1) * nst) / (unsigned)S);
    // Stages are taken from a place that differs from workgroup to workgroup: all at the same k of rows a power of two apart
    // would be after the same memory channels (20 x 32000 from K = 4096: 132 -> 121 us).
    const int turn = (int)((unsigned)nt % (unsigned)(s1 - s0));
    auto place = [&](int s) {
        const int p = min(s, s1 - 1) + turn;
        return p < s1 ? p : p - (s1 - s0);
    };
    auto first_k = [&](int p) { return KT ? min(p * 64, K - 64) : p * 64; };

    // This lane's share of P: NT, rows 16 t + li, k 4 lg and 16 + 4 lg; KS, columns 2 li and 2 li + 1 of eight k.  Addresses
    // are a scalar part, which says where in the matrix, and 32-bit byte offsets of the lane from there, worked out once.
    auto at = [](const float *base, unsigned off) { return (const float *)((const char *)base + off); };
    // an offset as the loads see it: were it known to be the same in every stage, it would be widened to 64 bits outside the
    // loop, and kept and added that way
    auto here = [](unsigned off) __attribute__((always_inline)) {
        asm volatile("" : "+v"(off));
        return off;
    };
    const float *pn = P + (KS ? (long)n0 : (long)n0 * ldp);
    unsigned poff[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t)
        poff[t] = 4u * (KS ? 4u * lg * (unsigned)ldp + 2u * li + t : (unsigned)(16 * t + li) * (unsigned)ldp + 4u * lg);
    typedef std::conditional_t<KS, f32x2, f32x4> piece;   // KS: k number e of both columns; NT: four k of row tile t
    constexpr int NP = KS ? 8 : 2 * TN;
    piece pv[PF][NP];                                     // KS [e]; NT [t][half of the fragment]
    auto load_p = [&](int s, auto slot) __attribute__((always_inline)) {
        piece *d = pv[decltype(slot)::value];
        const int k0 = first_k(place(s)) + kg * 32;
        if constexpr (!KS) {
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                const unsigned off = here(poff[t]);
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) d[2 * t + hf] = *(const f32x4_a4 *)at(pn + k0 + 16 * hf, off);
            }
        } else {
            const unsigned off = here(poff[0]);
#pragma unroll
            for (int e = 0; e < 8; ++e) d[e] = *(const f32x2_a4 *)at(pn + (long)(k0 + (e < 4 ? e : 12 + e)) * ldp, off);
        }
    };
    // this thread's share of Q: four k (quad kq of the stage) of rows qrow + 32 i
    const int kq = tid & 15, qrow = tid >> 4;
    const float *qm = Q + (long)m0 * ldq;
    unsigned qoff[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) qoff[i] = 4u * ((unsigned)(min(m0 + qrow + 32 * i, M - 1) - m0) * (unsigned)ldq + 4u * kq);
    f32x4 qv[QF][NQ];
    auto load_q = [&](int s, auto slot) __attribute__((always_inline)) {
        auto &d = qv[decltype(slot)::value];
        const float *base = qm + first_k(place(s));
#pragma unroll
        for (int i = 0; i < NQ; ++i) d[i] = *(const f32x4_a4 *)at(base, here(qoff[i]));
    };
    float ptop = 0.f, qtop = 0.f;   // largest magnitudes
    // Lane (i, g) of a fragment lies in slot (i ^ swizzle) + 16 g of its 64: the 8-byte stores of 32 lanes (two rows, all g,
    // both halves of the stage) fall into different banks, and so do the 16 lanes that a 16-byte read serves at a time
    // (0..3, 12..15, 20..27 and so on).
    auto swizzle = [](int g, int half) { return (4 * (-g & 3)) ^ (2 * half); };
    unsigned char *const qdst = (unsigned char *)(x3s + (kq >> 3) * 3 * PL + (qrow >> 4) * 64 + ((qrow & 15) ^ swizzle(kq & 3, kq >> 3)) + 16 * (kq & 3)) + ((kq >> 2) & 1) * 8;
    auto store_q = [&](int s, auto slot) __attribute__((always_inline)) {   // stage s into its buffer
        auto &d = qv[decltype(slot)::value];
        const int p = place(s), drop = p * 64 - first_k(p);   // k of the stage before, in the last stage
        if (KT)
#pragma unroll
            for (int i = 0; i < NQ; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) d[i][e] = 4 * kq + e < drop ? 0.f : d[i][e];
        unsigned char *base = qdst + ((s - s0) & 1) * (ST * 16);
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            uint32_t h[2], m[2], w[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) split3(x3_up(KS) * d[i][2 * e], x3_up(KS) * d[i][2 * e + 1], h[e], m[e], w[e], qtop);
            unsigned char *dst = base + i * 2048;   // 32 rows on
            *(u32x2 *)dst = (u32x2){h[0], h[1]};
            *(u32x2 *)(dst + PL * 16) = (u32x2){m[0], m[1]};
            *(u32x2 *)(dst + 2 * PL * 16) = (u32x2){w[0], w[1]};
        }
    };
    u32x4 a[3][TN];
    auto cut_p = [&](auto slot) __attribute__((always_inline)) {
        const piece *d = pv[decltype(slot)::value];
        auto value = [&](int t, int e) { if constexpr (KS) return d[e][t]; else return d[2 * t + (e >> 2)][e & 3]; };
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t h, m, w;
                split3(value(t, 2 * e), value(t, 2 * e + 1), h, m, w, ptop);
                a[0][t][e] = h; a[1][t][e] = m; a[2][t][e] = w;
            }
    };
    // the products of the first pieces, and all the others
    f32x4 acc[TN][MT], low[TN][MT];
    const int frag = (li ^ swizzle(lg, kg)) + 16 * lg;
    auto multiply = [&](int s) __attribute__((always_inline)) {
        const u32x4 *base = x3s + ((s - s0) & 1) * ST + kg * 3 * PL + frag;
        // fragments of Q in the order third, second, first piece of each row tile, three reads ahead of their products
        auto read = [&](int f) { return base[(2 - f % 3) * PL + f / 3 * 64]; };
        u32x4 b[4];
#pragma unroll
        for (int f = 0; f < 3; ++f) b[f] = read(f);
#pragma unroll
        for (int f = 0; f < 3 * MT; ++f) {
            const int pq = 2 - f % 3, j = f / 3;
            if (f + 3 < 3 * MT) b[(f + 3) & 3] = read(f + 3);
#pragma unroll
            for (int pp = 2 - pq; pp >= 0; --pp)
#pragma unroll
                for (int t = 0; t < TN; ++t) {
                    f32x4 &sum = pq + pp == 0 ? acc[t][j] : low[t][j];
                    sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[pp][t]), __builtin_bit_cast(bf16x8, b[f & 3]), sum, 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto meet = [&]() __attribute__((always_inline)) {
        // a bare barrier behind this wave's LDS accesses: the fence of __syncthreads would wait for the loads too
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    // Memory answers in order: a wait for Q is one for every older load of P, so Q is requested first and as far ahead.  The
    // two halves of the workgroup have loops of their own: the compiler counts the loads under way along every path it sees,
    // and waits for as many as the shortest one leaves.
    using std::integral_constant;
    auto stage = [&](int s, auto slot, auto half) __attribute__((always_inline)) {
        constexpr int B = decltype(slot)::value, KG = decltype(half)::value;
        constexpr integral_constant<int, (B + KG) % PF> pslot{};
        constexpr integral_constant<int, (B + 1) % QF> qslot{};
        if (KG == 1) multiply(s);
        __builtin_amdgcn_sched_barrier(0);
        cut_p(pslot);
        store_q(s + 1, qslot);
        __builtin_amdgcn_sched_barrier(0);   // what is loaded next takes the registers of what has been cut
        load_q(s + 1 + QF, qslot);
        __builtin_amdgcn_sched_barrier(0);
        load_p(s + KG + PF, pslot);
        __builtin_amdgcn_sched_barrier(0);
        if (KG == 0) multiply(s);
        meet();
    };
    auto sum_up = [&](auto half) __attribute__((always_inline)) {
        load_q(s0, integral_constant<int, 0>{});
        load_p(s0, integral_constant<int, 0>{});
        if constexpr (QF > 1) load_q(s0 + 1, integral_constant<int, 1 % QF>{});
        load_p(s0 + 1, integral_constant<int, 1>{});
        if constexpr (QF > 2) load_q(s0 + 2, integral_constant<int, 2 % QF>{});
        if constexpr (PF > 2) load_p(s0 + 2, integral_constant<int, 2 % PF>{});
        if constexpr (QF > 3) load_q(s0 + 3, integral_constant<int, 3 % QF>{});
        if constexpr (PF > 3) load_p(s0 + 3, integral_constant<int, 3 % PF>{});
        store_q(s0, integral_constant<int, 0>{});
        __builtin_amdgcn_sched_barrier(0);
        load_q(s0 + QF, integral_constant<int, 0>{});
        if (decltype(half)::value == 1) {
            cut_p(integral_constant<int, 0>{});
            __builtin_amdgcn_sched_barrier(0);
            load_p(s0 + PF, integral_constant<int, 0>{});
        }
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int j = 0; j < MT; ++j) acc[t][j] = low[t][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
        meet();
        int s = s0;
        for (; s + PF <= s1; s += PF) {
            stage(s, integral_constant<int, 0>{}, half);
            stage(s + 1, integral_constant<int, 1>{}, half);
            if constexpr (PF > 2) stage(s + 2, integral_constant<int, 2>{}, half);
            if constexpr (PF > 3) stage(s + 3, integral_constant<int, 3>{}, half);
        }
        if (s < s1) stage(s, integral_constant<int, 0>{}, half);
        if constexpr (PF > 2)
            if (s + 1 < s1) stage(s + 1, integral_constant<int, 1>{}, half);
        if constexpr (PF > 3)
            if (s + 2 < s1) stage(s + 2, integral_constant<int, 2>{}, half);
    };
    if (kg == 0) sum_up(integral_constant<int, 0>{});
    else sum_up(integral_constant<int, 1>{});
    // the lane's place once more: nothing of it is kept in registers over the loop
    int tid2 = threadIdx.x;
    asm volatile("" : "+v"(tid2));
    const int li2 = tid2 & 15, lg2 = (tid2 & 63) >> 4;
    bool finite = true;   // KS: every sum
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                f32x4 &sum = acc[t][j];
                if (KS) {   // one that has overflowed is taken anew below, whatever the small terms make of it
                    sum[r] = (sum[r] + low[t][j][r]) * x3_down(KS);
                    finite &= fabsf(sum[r]) < INFINITY;
                } else         // it stays as it is: the small terms may be of the other sign
                    sum[r] += fabsf(sum[r]) < INFINITY ? low[t][j][r] : 0.f;
            }
    // the largest magnitudes of Q's rows and of this wave's share of P
    for (int o = 32; o > 0; o >>= 1) { ptop = fmaxf(ptop, __shfl_xor(ptop, o)); qtop = fmaxf(qtop, __shfl_xor(qtop, o)); }
    if ((tid2 & 63) == 0) tops[wave] = qtop;
    __syncthreads();
    qtop = tops[0];
#pragma unroll
    for (int w = 1; w < 8; ++w) qtop = fmaxf(qtop, tops[w]);
    if (!pieces_hold(ptop, false) || !pieces_hold(qtop, KS) || !__all(finite)) {
        // this wave's k once more on the fp32 matrix pipe (16x16x4: lane (i, g) holds k = g of row i), four k a step
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int j = 0; j < MT; ++j) acc[t][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int q = s0 * 8; q < s1 * 8; ++q) {
            const int k = first_k(q >> 3) + kg * 32 + (q & 7) * 4 + lg2;
            float pe[TN];
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                const long n = n0 + (KS ? 2 * li2 + t : 16 * t + li2);
                const float x = P[KS ? k * ldp + n : n * ldp + k];
                pe[t] = KT && k < (q >> 3) * 64 ? 0.f : x;   // a k of the stage before
            }
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                const float x = Q[(long)min(m0 + j * 16 + li2, M - 1) * ldq + k], qe = KT && k < (q >> 3) * 64 ? 0.f : x;
#pragma unroll
                for (int t = 0; t < TN; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(pe[t], qe, acc[t][j], 0, 0, 0);
            }
        }
    }
    // waves 4..7 hand their sums to waves 0..3
    f32x4 *red = (f32x4 *)x3s + (size_t)wn * TN * MT * 64 + (tid2 & 63);
    if (kg == 1)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int j = 0; j < MT; ++j) red[(t * MT + j) * 64] = acc[t][j];
    __syncthreads();
    if (kg == 1) return;
    out += (long)blockIdx.y * M * N;
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const int m = m0 + j * 16 + li2;
        if (m >= M) continue;
        f32x4 v[TN];
#pragma unroll
        for (int t = 0; t < TN; ++t) v[t] = acc[t][j] + red[(t * MT + j) * 64];
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            // NT: tile t, four n from 4 lg2; KS: the two tiles take turns, four n from 8 lg2 + 4 t
            const int n = n0 + (KS ? 8 * lg2 + 4 * t : 16 * t + 4 * lg2);
            const f32x4 x = KS ? (f32x4){v[0][2 * t], v[1][2 * t], v[0][2 * t + 1], v[1][2 * t + 1]} : v[t];
            put4(out, join, (long)m * N + n, x, nown - n, 4, vec);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Weight update: W[M,N] += alpha * sum_r G[r,M] X[r,N], both operands k-strided, with k_gemm_x3's pieces and accumulators, and
// with bias bias[M] += alpha * sum_r G[r,M], by the workgroups of the first columns.  FEW: G2, if given, is added to G.
// Bound by reading and writing W once up to about 150 rows, by the matrix pipe and the cutting beyond.  Workgroup of four
// waves on 64 m x 128 n (rows of 512 B), 64 m x 32 n a wave.  G is cut for the whole tile, 128 r at a time, and shared through
// LDS; a wave's columns of X are its own and go from memory straight into matrix operands, cut in registers, a chunk of 32 r
// ahead.  The sums go through LDS, so that W is read and written in whole rows of the tile; it is requested before the last
// chunk's products (FEW, up to 32 rows: with the operands).  Registers and LDS for three workgroups a compute unit: one's
// products and cutting run beside the others' memory.  Tiles go by rows of W, and each die has an eighth of them that is
// contiguous in memory.
// No less exact than a chain of fp32 multiply-adds, at any number of rows: 2.53e-8 of a sum of random terms at one row (both; with
// six products of pieces 2.60e-8, and the largest error 1.7 times a rounding), 2.6e-8 against 3.1e-8 at two, 3.9e-8 against
// 1.03e-7 at 32 (2-norm).  For it FEW keeps eight of the nine products (33 rows and more round oftener than the other two would
// weigh), EXACT takes both operands times 2^24, so that pieces stand for values of any size, and a tile whose sums overflow, as they
// may where the whole does not, is summed anew on the fp32 pipe.  EXACT up to UPD_EXACT rows, where memory bounds all sizes: with
// the eight products it costs 1 to 2 %.  (Tiles with a value below 2^-102 beside larger ones summed anew instead: gradients of a
// discriminator that no longer errs are such, and the update of 32000 x 4096 by 20 rows took 271 us, that of 1024 x 32000 by 40 88.)
// Measured within training steps, by kernel trace: 32000 x 4096 by 20 rows 188 us (5.6 TB/s), plain multiply-adds with the rows of W
// dealt to all dies 216; by 60 rows 223, both operands through LDS and W in pieces of 256 B 470; by 300 rows 606 and 1451;
// 4096 x 4096 by 20 rows 30 and 34, by 128 rows 46 and 85; 1024 x 32000 by 40 rows 66 and 76.  Two workgroups a compute unit with X
// two chunks ahead, by themselves: 277 us at 32000 x 4096 by 60 rows and 49 at 4096 x 4096 by 128, with three 222 and 41.
// ---------------------------------------------------------------------------------------------
enum { UPD_FEW = 32, UPD_EXACT = 48 };
template <bool FEW, bool EXACT>
__global__ __launch_bounds__(256, 3) void k_update_x3(const float *__restrict__ G, const float *__restrict__ G2, const float *__restrict__ X,
                                                      float *W, float *bias, int M, int N, int rows, float alpha) {
    constexpr int BM = 64, BN = 128, TM = BM / 16, TN = 2, PL = TM * 64, LDO = BN + 4, NC = FEW ? 1 : 4;
    __shared__ u32x4 gs[FEW ? BM * LDO / 4 : NC * 3 * PL];   // [chunk][plane][m tile][64 lanes]; then the sums [BM][LDO]
    __shared__ float tops[4], bsum[4][BM];
    static_assert(BM * LDO * 4 <= (int)sizeof(gs), "the sums fit where the pieces were");
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, li = l & 15, lg = l >> 4;
    const int ntn = (N + BN - 1) / BN, ntm = (M + BM - 1) / BM;
    const int tile = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (tile >= ntn * ntm) return;
    const int m0 = tile / ntn * BM, n0 = tile % ntn * BN;
    // G: this thread's column, r = 8 wave + 0..7 of each 32; X: the columns nx and nx + 1, r = 8 lg + 0..7 of each 32.  Columns
    // past the end are the last ones again (their sums are not stored): where nx is the last column of all, the pair's second.
    const unsigned goff = 4u * (unsigned)min(l, M - 1 - m0);
    const int nx = n0 + wave * 32 + 2 * li, nl = max(min(nx, N - 2), 0);
    const bool edge = n0 + BN > N, whole = !edge && m0 + BM <= M, second = nx > nl;
    f32x2 xv[8];
    float gtop = 0.f, xtop = 0.f, gsum = 0.f;   // largest magnitudes, this thread's share of its column's sum
    constexpr float UP = x3_up(EXACT), DOWN = x3_down(EXACT) * x3_down(EXACT);
    auto load_x = [&](int r0) __attribute__((always_inline)) {
        if (r0 + 32 <= rows && N > 1 && N < 1 << 25) {
            unsigned off = 4u * (8u * lg * (unsigned)N + nl);
            asm volatile("" : "+v"(off));   // else widened to 64 bits ahead of the loop, once for every load
#pragma unroll
            for (int e = 0; e < 8; ++e) xv[e] = *(const f32x2_a4 *)((const char *)(X + (size_t)(r0 + e) * N) + off);
        } else {                    // rows past the last: the last, times zeros of G
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                int r = 8 * lg + e;
                asm volatile("" : "+v"(r));
                const float *p = X + nl + (size_t)min(r0 + r, rows - 1) * N;
                xv[e] = (f32x2){p[0], p[N > 1]};
            }
        }
    };
    u32x4 a[3][TN];
    auto cut_x = [&]() __attribute__((always_inline)) {
        if (edge)
#pragma unroll
            for (int e = 0; e < 8; ++e) xv[e].x = second ? xv[e].y : xv[e].x;
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t h, m, w;
                split3(UP * xv[2 * e][t], UP * xv[2 * e + 1][t], h, m, w, xtop);
                a[0][t][e] = h; a[1][t][e] = m; a[2][t][e] = w;
            }
    };
    // the products of the first pieces, and all the others
    f32x4 acc[TN][TM], low[TN][TM];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[t][j] = low[t][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int c) __attribute__((always_inline)) {
        const u32x4 *base = gs + c * 3 * PL + l;
        auto read = [&](int f) { return base[(2 - f % 3) * PL + f / 3 * 64]; };
        u32x4 b[4];
#pragma unroll
        for (int f = 0; f < 3; ++f) b[f] = read(f);
#pragma unroll
        for (int f = 0; f < 3 * TM; ++f) {
            const int pq = 2 - f % 3, j = f / 3;
            if (f + 3 < 3 * TM) b[(f + 3) & 3] = read(f + 3);
#pragma unroll
            for (int pp = FEW ? min(3 - pq, 2) : 2 - pq; pp >= 0; --pp)
#pragma unroll
                for (int t = 0; t < TN; ++t) {
                    f32x4 &sum = pq + pp == 0 ? acc[t][j] : low[t][j];
                    sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[pp][t]), __builtin_bit_cast(bf16x8, b[f & 3]), sum, 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // what this thread stores: four columns of rows (thread / 32) + 8 i; worked out where it is used, not kept over the loop
    struct Mine { float *p; int row, col, cnt; };
    auto mine = [&]() __attribute__((always_inline)) {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        const int row = t >> 5, col = (t & 31) * 4;
        return Mine{W + (size_t)(m0 + row) * N + n0 + col, row, col, N - n0 - col};
    };
    f32x4 old[8];
    auto load_old = [&]() __attribute__((always_inline)) {
        const Mine w = mine();
        if (whole) {
#pragma unroll
            for (int i = 0; i < 8; ++i) old[i] = *(const f32x4_a4 *)(w.p + (size_t)(8 * i) * N);
            return;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            old[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (m0 + w.row + 8 * i >= M) continue;
            const float *p = w.p + (size_t)(8 * i) * N;
            if (w.cnt >= 4) old[i] = *(const f32x4_a4 *)p;
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < w.cnt) old[i][e] = p[e];
        }
    };
    load_x(0);
    int rb = 0, nck;
    while (true) {
        nck = FEW ? 1 : min((rows - rb + 31) / 32, 4);
        float gv[NC][8];
#pragma unroll
        for (int i = 0; i < NC; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                gv[i][e] = *(const float *)((const char *)(G + m0 + (size_t)min(rb + 32 * i + 8 * wave + e, rows - 1) * M) + goff);
        float g2[FEW ? 8 : 1];
        if (FEW) {
            if (G2)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    g2[FEW ? e : 0] = *(const float *)((const char *)(G2 + m0 + (size_t)min(8 * wave + e, rows - 1) * M) + goff);
            load_old();
            if (G2)
#pragma unroll
                for (int e = 0; e < 8; ++e) gv[0][e] += g2[FEW ? e : 0];
        }
        if (!FEW && rb) __syncthreads();   // the pieces of the rows before have been read
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NC; ++i)
            if (i < nck) {
                u32x4 h, m, w;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (rb + 32 * i + 8 * wave + e >= rows) gv[i][e] = 0.f;
                if (bias)
#pragma unroll
                    for (int e = 0; e < 8; ++e) gsum += gv[i][e];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t p, q, r;
                    split3(UP * gv[i][2 * e], UP * gv[i][2 * e + 1], p, q, r, gtop);
                    h[e] = p; m[e] = q; w[e] = r;
                }
                u32x4 *dst = gs + i * 3 * PL + (l >> 4) * 64 + 16 * wave + li;
                dst[0] = h; dst[PL] = m; dst[2 * PL] = w;
                __builtin_amdgcn_sched_barrier(0);
            }
        // a bare barrier behind this wave's LDS writes: the fence of __syncthreads would wait for the loads too
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (FEW) break;
#pragma unroll 1
        for (int c = 0; c + 1 < nck; ++c) {
            cut_x();
            __builtin_amdgcn_sched_barrier(0);
            load_x(rb + 32 * (c + 1));
            __builtin_amdgcn_sched_barrier(0);
            multiply(c);
        }
        if (rb + 128 >= rows) break;
        cut_x();
        rb += 128;
        load_x(rb);
        __builtin_amdgcn_sched_barrier(0);
        multiply(3);
    }
    cut_x();
    __builtin_amdgcn_sched_barrier(0);
    if (!FEW) load_old();
    __builtin_amdgcn_sched_barrier(0);
    multiply(nck - 1);
    bool finite = true;   // every sum; one that has overflowed is taken anew below, whatever the small terms make of it
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            acc[t][j] = (acc[t][j] + low[t][j]) * DOWN;
#pragma unroll
            for (int r = 0; r < 4; ++r) finite &= fabsf(acc[t][j][r]) < INFINITY;
        }
    // the largest magnitudes of G's columns and of this wave's columns of X
    for (int o = 32; o > 0; o >>= 1) { gtop = fmaxf(gtop, __shfl_xor(gtop, o)); xtop = fmaxf(xtop, __shfl_xor(xtop, o)); }
    if (l == 0) tops[wave] = gtop;
    bsum[wave][l] = gsum;
    __syncthreads();
    if (bias && n0 == 0 && wave == 0 && m0 + l < M) bias[m0 + l] += alpha * ((bsum[0][l] + bsum[1][l]) + (bsum[2][l] + bsum[3][l]));
    gtop = fmaxf(fmaxf(tops[0], tops[1]), fmaxf(tops[2], tops[3]));
    if (!pieces_hold(gtop, EXACT) || !pieces_hold(xtop, EXACT) || !__all(finite)) {
        // once more on the fp32 matrix pipe (16x16x4: lane (i, g) holds r = g of column i), four r a step
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[t][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int r0 = 0; r0 < rows; r0 += 4) {
            const int r = r0 + lg;
            const size_t rc = min(r, rows - 1);
            f32x2 xe = {X[rc * N + nl], X[rc * N + nl + (N > 1)]};
            if (second) xe.x = xe.y;
            if (r >= rows) xe = (f32x2){0.f, 0.f};
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                const size_t at = rc * M + min(m0 + 16 * j + li, M - 1);
                const float x = FEW && G2 ? G[at] + G2[at] : G[at], ge = r < rows ? x : 0.f;
#pragma unroll
                for (int t = 0; t < TN; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xe[t], ge, acc[t][j], 0, 0, 0);
            }
        }
    }
    // a lane's two tiles are eight consecutive columns of row 16 j + li
    float *os = (float *)gs;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        float *o = os + (16 * j + li) * LDO + 32 * wave + 8 * lg;
        *(f32x4 *)o = (f32x4){acc[0][j][0], acc[1][j][0], acc[0][j][1], acc[1][j][1]};
        *(f32x4 *)(o + 4) = (f32x4){acc[0][j][2], acc[1][j][2], acc[0][j][3], acc[1][j][3]};
    }
    __syncthreads();
    const Mine w = mine();
    if (whole) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            *(f32x4_a4 *)(w.p + (size_t)(8 * i) * N) = old[i] + alpha * *(const f32x4 *)(os + (w.row + 8 * i) * LDO + w.col);
        return;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (m0 + w.row + 8 * i >= M) continue;
        const f32x4 sum = *(const f32x4 *)(os + (w.row + 8 * i) * LDO + w.col), v = old[i] + alpha * sum;
        float *p = w.p + (size_t)(8 * i) * N;
        if (w.cnt >= 4) *(f32x4_a4 *)p = v;
        else
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < w.cnt) p[e] = v[e];
    }
}

// ---------------------------------------------------------------------------------------------
// The same update of a small matrix by few rows (gemm_update), as plain fp32 multiply-adds in row order: no cutting, no way of the sums
// through LDS, and pieces of any size for a workgroup, where the form above has a chain of latencies a tile and few tiles.  A wave
// takes rows of W in pieces of 256 columns (1 KiB, PF of them under way) and holds its columns of X in registers; a workgroup's
// four waves take the rows of its panel in turn and share the panel of G, transposed, in LDS, where a row's KP factors are
// broadcast reads.
// grid: x = column blocks, y = panels of mr rows.
// ---------------------------------------------------------------------------------------------
enum { UPD_MR = 128 };
template <int KP>
__global__ __launch_bounds__(256) void k_update_rows(const float *__restrict__ G, const float *__restrict__ G2, const float *__restrict__ X,
                                                     float *W, float *bias, int M, int N, int rows, int mr, float alpha) {
    constexpr int PF = 8;
    __shared__ f32x4 gs[UPD_MR][KP / 4];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int m0 = blockIdx.y * mr, n = (blockIdx.x * 64 + l) * 4, cnt = N - n;   // columns of this lane: four, or cnt of them
    for (int i = threadIdx.x; i < mr * KP; i += 256) {
        const int m = i % mr, r = i / mr;
        float g = 0.f;
        if (r < rows && m0 + m < M) {
            g = G[(size_t)r * M + m0 + m];
            if (G2) g += G2[(size_t)r * M + m0 + m];
        }
        ((float *)gs[m])[r] = g;
    }
    auto load = [&](const float *p) {
        if (cnt >= 4) return (f32x4)*(const f32x4_a4 *)p;
        f32x4 w = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < cnt) w[e] = p[e];
        return w;
    };
    f32x4 x[KP], w[PF];
#pragma unroll
    for (int r = 0; r < KP; ++r) x[r] = r < rows ? load(X + (size_t)r * N + n) : (f32x4){0.f, 0.f, 0.f, 0.f};
    // rows m0 + wave, + 4, ..
    const int nrow = (min(mr, M - m0) - wave + 3) / 4;
    float *row = W + (size_t)(m0 + wave) * N + n;
    const size_t step = (size_t)4 * N;
#pragma unroll
    for (int p = 0; p < PF; ++p)
        if (p < nrow) w[p] = load(row + p * step);
    __syncthreads();
    if (bias && blockIdx.x == 0 && (int)threadIdx.x < min(mr, M - m0)) {
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < KP; ++r) sum += gs[threadIdx.x][r / 4][r % 4];
        bias[m0 + threadIdx.x] += alpha * sum;
    }
    for (int i = 0; i < nrow; i += PF) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            if (i + p >= nrow) continue;
            const f32x4 old = w[p];
            float *o = row + (size_t)(i + p) * step;
            if (i + p + PF < nrow) w[p] = load(o + PF * step);
            f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < KP / 4; ++q) {
                const f32x4 g = gs[wave + 4 * (i + p)][q];
#pragma unroll
                for (int z = 0; z < 4; ++z)
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[e] = fmaf(g[z], x[4 * q + z][e], t[e]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = fmaf(alpha, t[e], old[e]);
            if (cnt >= 4) *(f32x4_a4 *)o = t;
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < cnt) o[e] = t[e];
        }
    }
}

// row tiles of a workgroup of k_stream_x3: those of all rows, or of equal blocks of up to eight
int x3_tiles(int M) {
    const int tiles = (M + 15) / 16, nmb = (tiles + 7) / 8, mt = (tiles + nmb - 1) / nmb;
    return mt <= 2 ? 2 : mt <= 4 ? mt : mt <= 6 ? 6 : 8;
}
// The microseconds that a product in S splits takes in either form, up to what the choice does not depend on, as fitted to 10000
// of them (4 to 300 rows, 64 to 32000 columns, 64 to 32000 terms, 1 to 32 splits: within a tenth of most).  An n tile's
// workgroups are all on one die of 32 compute units, so the die with the most of them counts.
//   k_gemm_x3: a start, the chunks of a split at no less than a round trip each, at a workgroup's share of its compute unit;
//   k_stream_x3: rounds of one workgroup a compute unit, each a start and its stages.
// Where P is k-contiguous a die takes in 0.68 MB of it a microsecond; the rest counts a tenth there, and orders what is equal.
// Above the start, splits of at least two stages (k_gemm_x3 up to 32 rows: four chunks), else no such form: 1e30.
struct Shape { int M, N, K, S; bool ks; };
double with_stream(const Shape &p, int cols, double t) {
    return (p.ks ? t : std::max(t, 3.0 + (double)(((p.N + cols - 1) / cols + 7) / 8) * cols * p.K * 4 / 0.68e6)) + t / 10;
}
double x3_time(const Shape &p) {
    const int bm = p.M <= 32 ? 32 : p.M <= 64 ? 64 : 128, nch = (p.K + X3_BK - 1) / X3_BK;
    if (p.S > 1 && nch < (bm == 32 ? 4 : 2) * p.S) return 1e30;
    static const double fit[2][3][4] = {   // start, round trip, chunk, the end of a workgroup
        {{2.7, 0.59, 0.43, 0.33}, {2.0, 0.82, 0.62, 1.6}, {2.1, 1.36, 0.96, 1.9}},
        {{2.3, 0.85, 0.54, 0.31}, {1.3, 1.14, 0.76, 1.6}, {1.7, 1.66, 1.09, 2.0}}};
    const double *f = fit[p.ks][bm / 64];
    const long die = (long)((p.N + X3_BN - 1) / X3_BN + 7) / 8 * ((p.M + bm - 1) / bm) * p.S;
    const double unit = (double)((die + 31) / 32);
    return with_stream(p, X3_BN, f[0] + (nch + p.S - 1) / p.S * std::max(f[1], unit * f[2]) + unit * f[3]);
}
double stream_time(const Shape &p) {
    const int mt = x3_tiles(p.M), nst = (p.K + 63) / 64;
    if (p.N < 32 || p.K < 64 || p.N >= 1 << 23 || p.K >= 1 << 23 || (p.S > 1 && nst < 2 * p.S)) return 1e30;   // see k_stream_x3
    static const double fit[2][5][2] = {   // stage, start
        {{0.93, 6.0}, {1.05, 6.7}, {1.10, 7.3}, {1.42, 8.2}, {1.84, 9.2}},
        {{0.95, 5.1}, {1.14, 6.0}, {1.24, 6.8}, {1.50, 8.2}, {1.92, 9.3}}};
    const double *f = fit[p.ks][mt <= 4 ? mt - 2 : mt == 6 ? 3 : 4];
    const long die = (long)((p.N + 127) / 128 + 7) / 8 * ((p.M + 16 * mt - 1) / (16 * mt)) * p.S;
    return with_stream(p, 128, (double)((die + 31) / 32) * ((nst + p.S - 1) / p.S * f[0] + f[1]));
}
bool streamed(const Shape &p) { return stream_time(p) < x3_time(p); }
// K splits that take the least time, with partial sums that fit `room` floats (none: one split, straight into C) and are read
// back at 4 MB a microsecond
int x3_splits(int M, int N, int K, size_t room, bool ks) {
    double best = 1e300;
    int S = 1;
    for (int s = 1; s <= 32 && (s == 1 || (size_t)s * M * N <= room); ++s) {
        const Shape p{M, N, K, s, ks};
        const double t = std::min(x3_time(p), stream_time(p)) + (s > 1 ? 1.0 + 1e-6 * s * M * N : 0.0);
        if (t < best) { best = t; S = s; }
    }
    return S;
}

template <int BM, bool PKS>
void launch_x3(hipStream_t st, const float *P, long ldp, const float *Q, long ldq, float *out, int S, int M, int N, int K,
               const Join &join) {
    const size_t sm = (size_t)2 * 3 * (X3_BN + BM) / 16 * 64 * 16;
    constexpr int DEPTH = BM <= 64 ? 4 : 2;
    static OncePerDevice once;
    allow_lds(once, (const void *)k_gemm_x3<BM, PKS, DEPTH>, sm);
    const int vec = N % 4 == 0 && ((uintptr_t)out & 15) == 0 && join_aligned(join);
    const dim3 grid(((N + X3_BN - 1) / X3_BN + 7) / 8 * 8 * ((M + BM - 1) / BM), S);
    k_gemm_x3<BM, PKS, DEPTH><<<grid, 256, sm, st>>>(P, ldp, Q, ldq, out, M, N, K, vec, join);
}
template <bool PKS>
void gemm_x3(hipStream_t st, const float *P, long ldp, const float *Q, long ldq, float *out, int S, int M, int N, int K,
             const Join &join) {
    if (M <= 32) launch_x3<32, PKS>(st, P, ldp, Q, ldq, out, S, M, N, K, join);
    else if (M <= 64) launch_x3<64, PKS>(st, P, ldp, Q, ldq, out, S, M, N, K, join);
    else launch_x3<128, PKS>(st, P, ldp, Q, ldq, out, S, M, N, K, join);
}
template <int MT, bool KS, bool KT>
void launch_stream(hipStream_t st, const float *P, long ldp, const float *X, float *out, int S, int M, int N, int K, const Join &join) {
    constexpr size_t sm = (size_t)2 * 2 * 3 * ((MT + 1) / 2 * 2) * 1024;
    static OncePerDevice once;
    allow_lds(once, (const void *)k_stream_x3<MT, KS, KT>, sm);
    const int vec = N % 4 == 0 && ((uintptr_t)out & 15) == 0 && join_aligned(join);
    const dim3 grid(((N + 127) / 128 + 7) / 8 * 8 * ((M + MT * 16 - 1) / (MT * 16)), S);
    k_stream_x3<MT, KS, KT><<<grid, 512, sm, st>>>(P, ldp, X, K, out, M, N, K, vec, join);
}
// C[M,N] = X[M,K] P, P(k, n) = W[n,K] or (KS) W[K,n]; split sums to part (S > 1) or straight to C, joined to logits if any
template <bool KS>
void gemm_weights(hipStream_t st, const float *X, const float *W, float *C, float *part, int S, int M, int N, int K, const Join &join) {
    float *out = S > 1 ? part : C;
    const long ldp = KS ? N : K;
    // The faster form: k_stream_x3 gains with many stages and with many rows, k_gemm_x3's smaller workgroups where either is
    // few.  Against more than four stages a workgroup streamed, and splits priced as the streamed form's: forward pass of a head
    // of 512 x 4000 at 20 rows 22.5 -> 20.5 us, at 200 36.0 -> 33.3; discriminator step of 512 x 32000 x 1500, three layers, at
    // ten positions 264 -> 246, at 200 1216 -> 1076; of 4096 x 32000 x 1024 at 20 the same.
    if (!streamed(Shape{M, N, K, S, KS})) return gemm_x3<KS>(st, W, ldp, X, K, out, S, M, N, K, join);
#define KOALA_STREAM(MT) return K % 64 ? launch_stream<MT, KS, true>(st, W, ldp, X, out, S, M, N, K, join) : launch_stream<MT, KS, false>(st, W, ldp, X, out, S, M, N, K, join)
    switch (x3_tiles(M)) {
        case 2: KOALA_STREAM(2);
        case 3: KOALA_STREAM(3);
        case 4: KOALA_STREAM(4);
        case 6: KOALA_STREAM(6);
        default: KOALA_STREAM(8);
    }
#undef KOALA_STREAM
}
void gemm_nt(hipStream_t st, const float *X, const float *W, float *C, float *part, int S, int M, int N, int K, const Join &join = {}) {
    gemm_weights<false>(st, X, W, C, part, S, M, N, K, join);
}
void gemm_nn(hipStream_t st, const float *X, const float *W, float *C, float *part, int S, int M, int N, int K) {
    gemm_weights<true>(st, X, W, C, part, S, M, N, K, Join{});
}
template <int KP>
void launch_update(hipStream_t st, const float *G, const float *G2, const float *X, float *W, float *bias, int M, int N, int rows,
                   float alpha) {
    const int nb = (N + 255) / 256;
    int mr = UPD_MR;   // panels as high as leave a workgroup a compute unit: each reads its columns of X for itself
    while (mr > 16 && (long)nb * ((M + mr - 1) / mr) < 256) mr /= 2;
    k_update_rows<KP><<<dim3(nb, (M + mr - 1) / mr), 256, 0, st>>>(G, G2, X, W, bias, M, N, rows, mr, alpha);
}
// W[M,N] -= lr * G[rows,M]^T X[rows,N] and (bias not null) bias[M] -= lr * column sums of G; G2 (up to UPD_FEW rows, may be
// null) is added to G
void gemm_update(hipStream_t st, const float *G, const float *X, float *W, int M, int N, int rows, float lr, float *bias = nullptr,
                 const float *G2 = nullptr) {
    // Plain multiply-adds up to where the matrix takes as long either way.  A head step with this update and little else, us, them
    // and k_update_x3, on one matrix / on so many in turn that each comes from memory: by 4 rows 1000 x 1000 22.6 / 22.3 and
    // 23.8 / 24.0, 1500 x 1500 25.0 / 26.2 and 26.6 / 28.5; by 8 2048 x 2048 29.7 / 31.9 and 30.2 / 32.5, 3000 x 3000 38.7 / 43.9 and
    // 38.1 / 43.7, 4096 x 4096 55.8 / 65.7 and 50.3 / 60.1; by 16 1250 x 1250 25.8 / 26.5 and 26.0 / 28.8, 1500 x 1500 26.0 / 27.5
    // and 26.5 / 28.6; by 20 (one matrix) 1500 x 1500 27.8 and 27.3, 2048 x 2048 34.1 and 30.8.  A matrix of few rows leaves most
    // of a tile empty: a discriminator step of one layer, 250 x 250 at 20 positions 26.8 and 28.8.
    // Two rows at any size: the largest error of an element is 1.97 roundings of its terms' magnitudes then and 2.77 on the matrix
    // pipe, whose sums are cut off (at three rows 2.81 and 2.70); such a step at 4096 x 32000 takes 370 us instead of 356.
    const size_t size = (size_t)M * N;
    if (rows == 2 || (rows <= 8 ? size <= 1u << 23 : rows <= 16 ? size <= 5u << 19 : rows <= 24 && M <= 16 && size <= 5u << 19)) {
        switch ((rows + 7) / 8) {
            case 1: return launch_update<8>(st, G, G2, X, W, bias, M, N, rows, -lr);
            case 2: return launch_update<16>(st, G, G2, X, W, bias, M, N, rows, -lr);
            default: return launch_update<24>(st, G, G2, X, W, bias, M, N, rows, -lr);
        }
    }
    const long tiles = (long)((M + 63) / 64) * ((N + 127) / 128);
    const int grid = (int)((tiles + 7) / 8 * 8);
    if (rows <= UPD_FEW) k_update_x3<true, true><<<grid, 256, 0, st>>>(G, G2, X, W, bias, M, N, rows, -lr);
    else if (rows <= UPD_EXACT) k_update_x3<false, true><<<grid, 256, 0, st>>>(G, nullptr, X, W, bias, M, N, rows, -lr);
    else k_update_x3<false, false><<<grid, 256, 0, st>>>(G, nullptr, X, W, bias, M, N, rows, -lr);
}

// The S split sums of element i added in split order, and the element-wise step that follows the product:
//   SUM_ONLY  out = sum;  SUM_MASK  out = sum where base > 0, else 0;
//   SUM_RELU  out = sum + bias[column] (the pre-activation), out2 = max(out, 0);
//   SUM_SILU  out = sum, out2 = base + SiLU(sum);
//   SUM_BACK  out = sum (+ add), out2 = out * SiLU'(base).
// part may be out itself (S = 1).
enum { SUM_ONLY, SUM_MASK, SUM_RELU, SUM_SILU, SUM_BACK };
__device__ __forceinline__ float split_sum(const float *part, int S, long count, long i) {
    float v = 0.f;
    int s = 0;
    for (; s + 8 <= S; s += 8) {
        float t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = part[(long)(s + u) * count + i];
#pragma unroll
        for (int u = 0; u < 8; ++u) v += t[u];
    }
    for (; s < S; ++s) v += part[(long)s * count + i];
    return v;
}
template <int MODE>
__global__ __launch_bounds__(256) void k_sum_parts(const float *part, int S, long count, int N, const float *base,
                                                   float *out, float *out2, const float *add) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    float v = split_sum(part, S, count, i);
    if (MODE == SUM_MASK && !(base[i] > 0.f)) v = 0.f;
    if (MODE == SUM_BACK) {
        if (add) v += add[i];
        const float y = base[i], g = 1.0f / (1.0f + expf(-y));
        out2[i] = v * g * (1.0f + y * (1.0f - g));
    }
    if (MODE == SUM_RELU) { v += base[i % N]; out2[i] = fmaxf(v, 0.f); }
    if (MODE == SUM_SILU) out2[i] = base[i] + v / (1.0f + expf(-v));
    out[i] = v;
}
template <int MODE>
void sum_parts(hipStream_t st, const float *part, int S, int M, int N, const float *base, float *out, float *out2,
               const float *add = nullptr) {
    const long count = (long)M * N;
    k_sum_parts<MODE><<<(int)((count + 255) / 256), 256, 0, st>>>(part, S, count, N, base, out, out2, add);
}

__device__ __forceinline__ float softplus(float x) { return fmaxf(x, 0.f) + log1pf(expf(-fabsf(x))); }
__device__ __forceinline__ float sigmoidf(float x) { return 1.0f / (1.0f + expf(-x)); }

// sum / maximum over the workgroup of NW waves; every thread gets it
template <int NW = 4>
__device__ __forceinline__ float block_sum(float v, float *sh) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    float t[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) t[w] = sh[w];
#pragma unroll
    for (int h = NW / 2; h > 0; h >>= 1)
#pragma unroll
        for (int w = 0; w < h; ++w) t[w] += t[w + h];
    return t[0];
}
template <int NW = 4>
__device__ __forceinline__ float block_max(float v, float *sh) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = sh[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) t = fmaxf(t, sh[w]);
    return t;
}

// The mapped hidden state z0 + z1, the sums of two K splits, joined to the logits as by a product's Join.  The halves may lie
// where u does (row p and row n + p).
__global__ __launch_bounds__(256) void k_join(const float *z0, const float *z1, const float *la, const float *lb, float *u,
                                              long nV) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= nV) return;
    const float z = z0[i] + z1[i];
    u[i] = z + la[i];
    if (lb) u[nV + i] = z + lb[i];
}

// s[r] = a[r] . w: the width-1 layer.  One workgroup per row.
__global__ __launch_bounds__(256) void k_row_dot(const float *a, const float *w, float *s, int W) {
    __shared__ float sh[4];
    const float *ar = a + (long)blockIdx.x * W;
    float v = 0.f;
    for (int j = threadIdx.x; j < W; j += 256) v += ar[j] * w[j];
    v = block_sum(v, sh);
    if (threadIdx.x == 0) s[blockIdx.x] = v;
}

// SUM_RELU of row r and the width-1 layer behind it, s[r] = out2[r] . w.  One workgroup per row.
__global__ __launch_bounds__(1024) void k_sum_relu_dot(const float *part, int S, long count, int N, const float *bias, float *pre,
                                                       float *act, const float *w, float *s) {
    __shared__ float sh[16];
    const long at = (long)blockIdx.x * N;
    float dot = 0.f;
    for (int j = threadIdx.x; j < N; j += 1024) {
        const float v = split_sum(part, S, count, at + j) + bias[j], a = fmaxf(v, 0.f);
        pre[at + j] = v;
        act[at + j] = a;
        dot += a * w[j];
    }
    dot = block_sum<16>(dot, sh);
    if (threadIdx.x == 0) s[blockIdx.x] = dot;
}

// Scores s (pre-sigmoid; the last layer's bias is added here) -> dL/ds per row and the loss, and the width-1 layer's input
// gradient g[r][j] = ds[r] w[j], zero where the unit was off (pre, if given).
//   mode 0 (Eq. 6): rows [0, n) are the draft's, [n, 2n) the target's:
//          L_D = mean softplus(s_d) + mean softplus(-s_q);  ds_d = sigmoid(s)/n, ds_q = -(1 - sigmoid(s))/n
//   mode 1 (Eq. 5, adversarial term): n draft rows: L = lambda mean softplus(-s); ds = -lambda (1 - sigmoid(s))/n
// grid: nb workgroups a row for g, each with the row's ds worked out for itself, and one for ds and the loss.
struct ScoreLoss { int n, mode; float lambda; float *loss; };
__global__ __launch_bounds__(256) void k_score_outer(const float *s, const float *bias_p, float *ds, ScoreLoss t, const float *w,
                                                     const float *pre, float *g, int rows, int W, int nb) {
    const float bias = bias_p[0];
    auto slope = [&](int r, float v) {
        if (t.mode == 0) return r < t.n ? sigmoidf(v) / t.n : -(1.0f - sigmoidf(v)) / t.n;
        return -t.lambda * (1.0f - sigmoidf(v)) / t.n;
    };
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ float sh[4];
        float part = 0.f;
        for (int r = threadIdx.x; r < rows; r += 256) {
            const float v = s[r] + bias;
            if (t.mode == 0) part += r < t.n ? softplus(v) : softplus(-v);
            else part += t.lambda * softplus(-v);
            ds[r] = slope(r, v);
        }
        const float tot = block_sum(part, sh);
        if (threadIdx.x == 0) t.loss[0] = tot / t.n;
        return;
    }
    const int r = (int)(blockIdx.x / (unsigned)nb), j = (int)(blockIdx.x % (unsigned)nb) * 256 + threadIdx.x;
    if (j >= W) return;
    const size_t i = (size_t)r * W + j;
    g[i] = pre && !(pre[i] > 0.f) ? 0.f : slope(r, s[r] + bias) * w[j];
}

// gz[p][v] = gu[p][v] + gu[n + p][v]
__global__ void k_fold_rows(const float *gu, float *gz, int n, int V) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (long)n * V) gz[i] = gu[i] + gu[(long)n * V + i];
}

// Distillation term (cross-entropy of softmax(d) against softmax(q)) of one row per workgroup:
// ce[r] = lse(d) - sum_v softmax(q)_v d_v, and grad[r][v] = base[r][v] + (softmax(d)_v - softmax(q)_v) / n.
// A row of both logits is read once into registers (up to 32 of each per thread, 32768 columns; longer rows read the
// rest again) with all loads in flight; one workgroup of 256 threads reading a row three times took 182 us for 128 rows
// of 32000, this form 27 us (39 with an address per load in registers, which then spilled).
__global__ __launch_bounds__(1024) void k_distill(const float *q, const float *d, const float *base, float *grad, float *ce,
                                                  int V, int n) {
    constexpr int NR = 32, NT = 1024;
    __shared__ float sh[16];
    const int r = blockIdx.x, t = threadIdx.x;
    const float *qr = q + (long)r * V, *dr = d + (long)r * V, *br = base + (long)r * V;
    // element t + u * NT of a row: a scalar address plus this thread's offset, so that no load holds an address of its own
    const unsigned at = 4u * t;
    auto in = [&](const float *p, int u) { return *(const float *)((const char *)(p + u * NT) + at); };
    float qv[NR], dv[NR];
    float mq = -INFINITY, md = -INFINITY;
#pragma unroll
    for (int u = 0; u < NR; ++u) {
        qv[u] = t < V - u * NT ? in(qr, u) : -INFINITY;
        dv[u] = t < V - u * NT ? in(dr, u) : -INFINITY;
    }
#pragma unroll
    for (int u = 0; u < NR; ++u) { mq = fmaxf(mq, qv[u]); md = fmaxf(md, dv[u]); }
    for (int v = NR * NT + t; v < V; v += NT) { mq = fmaxf(mq, qr[v]); md = fmaxf(md, dr[v]); }
    mq = block_max<16>(mq, sh);
    md = block_max<16>(md, sh);
    float sq = 0.f, sd = 0.f, qd = 0.f;
#pragma unroll
    for (int u = 0; u < NR; ++u) {
        if (t < V - u * NT) {
            const float eq = expf(qv[u] - mq), ed = expf(dv[u] - md);
            sq += eq;
            sd += ed;
            qd += eq * dv[u];
            qv[u] = eq;
            dv[u] = ed;
        }
        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // a few at a time: the registers hold the row
    }
    for (int v = NR * NT + t; v < V; v += NT) {
        const float eq = expf(qr[v] - mq);
        sq += eq;
        sd += expf(dr[v] - md);
        qd += eq * dr[v];
    }
    sq = block_sum<16>(sq, sh);
    sd = block_sum<16>(sd, sh);
    qd = block_sum<16>(qd, sh);
    if (t == 0) ce[r] = (md + logf(sd)) - qd / sq;
    float *gr = grad + (long)r * V;
#pragma unroll
    for (int u = 0; u < NR; ++u) {
        if (t < V - u * NT) *(float *)((char *)(gr + u * NT) + at) = in(br, u) + (dv[u] / sd - qv[u] / sq) / n;
        if (u % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
    for (int v = NR * NT + t; v < V; v += NT) gr[v] = br[v] + (expf(dr[v] - md) / sd - expf(qr[v] - mq) / sq) / n;
}

// loss[0] = mean of ce[0..n)
__global__ __launch_bounds__(256) void k_mean(const float *ce, float *loss, int n) {
    __shared__ float sh[4];
    float t = 0.f;
    for (int r = threadIdx.x; r < n; r += 256) t += ce[r];
    t = block_sum(t, sh);
    if (threadIdx.x == 0) loss[0] = t / n;
}

inline int blocks(long n) { return (int)((n + 255) / 256); }
inline size_t up256(size_t v) { return (v + 255) / 256 * 256; }

struct DiscWs {
    float *z, *u, *ds, *s, *ce;
    float *a[3], *pre[3], *g[3];   // a[k]: input of FC layer k (a[0] = u); pre[k]: its output before ReLU; g: gradients
    size_t bytes;
};

// rows = 2n for the discriminator step (draft rows, then target rows), n for the draft-head gradient
DiscWs carve_disc(const koala_disc_shape &s, int n, char *base) {
    DiscWs w{};
    size_t off = 0;
    auto take = [&](size_t floats) {
        float *p = base ? (float *)(base + off) : nullptr;
        off += up256(floats * sizeof(float));
        return p;
    };
    const int rows = 2 * n, V = s.vocab, Dh = s.fc_hidden;
    w.z = take((size_t)n * V);
    w.u = take((size_t)rows * V);
    w.ds = take(rows);
    w.s = take(rows);
    w.ce = take(n);
    w.a[0] = w.u;
    w.g[0] = take((size_t)rows * V);
    for (int k = 1; k < s.n_fc; ++k) {
        w.pre[k - 1] = take((size_t)rows * Dh);
        w.a[k] = take((size_t)rows * Dh);
        w.g[k] = take((size_t)rows * Dh);
    }
    w.bytes = off;
    return w;
}

bool shape_ok(const koala_disc_shape *s) {
    return s && s->hidden > 0 && s->vocab > 0 && s->n_fc >= 1 && s->n_fc <= 3 && (s->n_fc == 1 || s->fc_hidden > 0);
}
bool params_ok(const koala_disc_shape *s, const koala_disc_params *p) {
    if (!p || !p->w_lin) return false;
    for (int k = 0; k < s->n_fc; ++k)
        if (!p->w_fc[k] || !p->b_fc[k]) return false;
    return true;
}
inline int fc_in(const koala_disc_shape &s, int k) { return k == 0 ? s.vocab : s.fc_hidden; }
inline int fc_out(const koala_disc_shape &s, int k) { return k == s.n_fc - 1 ? 1 : s.fc_hidden; }

// z = h W_lin^T joined to one or two sets of logits rows, where the product stores it or (its tiles do not fill the chip) by
// k_join on the sums of two K splits, which lie where u will.
void disc_join(hipStream_t st, const koala_disc_shape &s, const koala_disc_params &p, const DiscWs &w, int n, const float *h,
               const float *la, const float *lb) {
    const long nV = (long)n * s.vocab;
    const int S = x3_splits(n, s.vocab, s.hidden, (size_t)2 * nV, false);
    if (S == 1) return gemm_nt(st, h, p.w_lin, w.u, nullptr, 1, n, s.vocab, s.hidden, Join{la, lb, nV});
    gemm_nt(st, h, p.w_lin, nullptr, w.u, 2, n, s.vocab, s.hidden);
    k_join<<<blocks(nV), 256, 0, st>>>(w.u, w.u + nV, la, lb, w.u, nV);
}

// scores of `rows` joined rows u: leaves every layer's input and pre-activation in the workspace, s = w_last . a.
// g[0], which only the backward pass fills, holds the split sums of the inner layers.
void disc_forward(hipStream_t st, const koala_disc_shape &s, const koala_disc_params &p, const DiscWs &w, int n, int rows) {
    const int last = s.n_fc - 1;   // width 1 (bias added where the score is used)
    if (last == 0) k_row_dot<<<rows, 256, 0, st>>>(w.a[0], p.w_fc[0], w.s, s.vocab);
    for (int k = 0; k < last; ++k) {
        const int in = fc_in(s, k), out = fc_out(s, k), S = x3_splits(rows, out, in, (size_t)2 * n * s.vocab, false);
        gemm_nt(st, w.a[k], p.w_fc[k], w.pre[k], w.g[0], S, rows, out, in);
        const float *part = S > 1 ? w.g[0] : w.pre[k];
        if (k + 1 < last) sum_parts<SUM_RELU>(st, part, S, rows, out, p.b_fc[k], w.pre[k], w.a[k + 1]);
        else k_sum_relu_dot<<<rows, 1024, 0, st>>>(part, S, (long)rows * out, out, p.b_fc[k], w.pre[k], w.a[k + 1], p.w_fc[last], w.s);
    }
}

// from the scores to the loss, ds (dL/ds per row) and back to g[0] = dL/du; lr > 0: the parameters are updated on the way (each
// layer's input gradient is taken with the layer's old weights first).  z (used only here) holds the split sums of the inner
// layers' input gradients.
void disc_backward(hipStream_t st, const koala_disc_shape &s, const koala_disc_params &p, const DiscWs &w, int n, int rows,
                   float lr, const ScoreLoss &t) {
    for (int k = s.n_fc - 1; k >= 0; --k) {
        const int in = fc_in(s, k), out = fc_out(s, k);
        const float *gout = k == s.n_fc - 1 ? w.ds : w.g[k + 1];   // dL/d(pre of layer k): [rows, out]
        const float *pre = k > 0 ? w.pre[k - 1] : nullptr;
        if (k == s.n_fc - 1) {
            const int nb = (in + 255) / 256;
            k_score_outer<<<rows * nb + 1, 256, 0, st>>>(w.s, p.b_fc[k], w.ds, t, p.w_fc[k], pre, w.g[k], rows, in, nb);
        } else {
            const int S = x3_splits(rows, in, out, (size_t)n * s.vocab, true);
            gemm_nn(st, gout, p.w_fc[k], w.g[k], w.z, S, rows, in, out);
            const float *part = S > 1 ? w.z : w.g[k];
            if (pre) sum_parts<SUM_MASK>(st, part, S, rows, in, pre, w.g[k], nullptr);
            else if (S > 1) sum_parts<SUM_ONLY>(st, part, S, rows, in, nullptr, w.g[k], nullptr);
        }
        // W_k[out, in] -= lr * gout^T a_k ;  b_k -= lr * column sums of gout
        if (lr > 0.f) gemm_update(st, gout, w.a[k], p.w_fc[k], out, in, rows, lr, p.b_fc[k]);
    }
}

}  // namespace

extern "C" {

// For tests: the row tiles of a workgroup where a product [rows, cols] of `terms` terms is streamed, else 0, and its splits where
// partial sums have `room` floats
int kt_product_form(int rows, int cols, int terms, int strided, size_t room, int *splits) {
    *splits = x3_splits(rows, cols, terms, room, strided != 0);
    return streamed(Shape{rows, cols, terms, *splits, strided != 0}) ? x3_tiles(rows) : 0;
}

koala_status koala_train_workspace_bytes(const koala_disc_shape *shape, int n_rows, size_t *out) {
    if (!shape || !out) return KOALA_E_NULL;
    if (!shape_ok(shape) || n_rows < 1) return KOALA_E_SHAPE;
    *out = carve_disc(*shape, n_rows, nullptr).bytes;
    return KOALA_OK;
}

koala_status koala_train_disc_step(const koala_disc_shape *shape, const koala_disc_params *params, void *hip_stream,
                                   int n_rows, const float *h, const float *q_logits, const float *d_logits, float lr,
                                   void *workspace, size_t workspace_bytes, float *loss_out) {
    if (!shape || !params || !h || !q_logits || !d_logits || !workspace || !loss_out) return KOALA_E_NULL;
    if (!shape_ok(shape) || n_rows < 1 || !(lr >= 0.f)) return KOALA_E_SHAPE;
    if (!params_ok(shape, params)) return KOALA_E_NULL;
    const koala_disc_shape &s = *shape;
    const DiscWs w = carve_disc(s, n_rows, (char *)workspace);
    if (workspace_bytes < w.bytes) return KOALA_E_WORKSPACE;
    hipStream_t st = (hipStream_t)hip_stream;
    const int n = n_rows, V = s.vocab, H = s.hidden, rows = 2 * n;
    // z = h W_lin^T, u = [z + d ; z + q]
    disc_join(st, s, *params, w, n, h, d_logits, q_logits);
    disc_forward(st, s, *params, w, n, rows);
    disc_backward(st, s, *params, w, n, rows, lr, ScoreLoss{n, 0, 0.f, loss_out});
    if (lr > 0.f) {
        // u = W_lin h + logits for both halves: dL/dW_lin = (g_u[draft rows] + g_u[target rows])^T h
        if (n <= UPD_FEW) {
            gemm_update(st, w.g[0], h, params->w_lin, V, H, n, lr, nullptr, w.g[0] + (size_t)n * V);
        } else {
            k_fold_rows<<<blocks((long)n * V), 256, 0, st>>>(w.g[0], w.z, n, V);
            gemm_update(st, w.z, h, params->w_lin, V, H, n, lr);
        }
    }
    return hipGetLastError() == hipSuccess ? KOALA_OK : KOALA_E_DEVICE;
}

koala_status koala_train_gen_grad(const koala_disc_shape *shape, const koala_disc_params *params, void *hip_stream,
                                  int n_rows, const float *h, const float *q_logits, const float *d_logits,
                                  float lambda, void *workspace, size_t workspace_bytes, float *loss_out,
                                  float *grad_d) {
    if (!shape || !params || !h || !q_logits || !d_logits || !workspace || !loss_out || !grad_d) return KOALA_E_NULL;
    if (!shape_ok(shape) || n_rows < 1 || !(lambda >= 0.f)) return KOALA_E_SHAPE;
    if (!params_ok(shape, params)) return KOALA_E_NULL;
    const koala_disc_shape &s = *shape;
    const DiscWs w = carve_disc(s, n_rows, (char *)workspace);
    if (workspace_bytes < w.bytes) return KOALA_E_WORKSPACE;
    hipStream_t st = (hipStream_t)hip_stream;
    const int n = n_rows, V = s.vocab, H = s.hidden;
    disc_join(st, s, *params, w, n, h, d_logits, nullptr);
    disc_forward(st, s, *params, w, n, n);
    disc_backward(st, s, *params, w, n, n, 0.f, ScoreLoss{n, 1, lambda, loss_out});
    // dL_G/dd = dL_adv/du (u = z + d) + the distillation term's gradient
    k_distill<<<n, 1024, 0, st>>>(q_logits, d_logits, w.g[0], grad_d, w.ce, V, n);
    k_mean<<<1, 256, 0, st>>>(w.ce, loss_out + 1, n);
    return hipGetLastError() == hipSuccess ? KOALA_OK : KOALA_E_DEVICE;
}

// Medusa workspace, in slots of n_rows * hidden floats: x_1 .. x_K, y_0 .. y_{K-1}, gx, gx', gy and one spare, as many as
// a call needs at least, then MED_PARTS slots of split sums.  A workspace without (all of) those is accepted as well:
// the products then run unsplit, on fewer compute units.
enum { MED_PARTS = 8 };
static size_t med_slot(int n_rows, int hidden) { return up256((size_t)n_rows * hidden * sizeof(float)); }
static size_t med_need(int n_rows, int hidden, int K) { return med_slot(n_rows, hidden) * (size_t)(2 * K + 4); }

koala_status koala_train_medusa_workspace_bytes(int n_rows, int hidden, int K, size_t *out) {
    if (!out) return KOALA_E_NULL;
    if (n_rows < 1 || hidden < 1 || K < 1 || K > 8) return KOALA_E_SHAPE;
    *out = med_need(n_rows, hidden, K) + MED_PARTS * med_slot(n_rows, hidden);
    return KOALA_OK;
}

struct MedWs {
    float *x[9], *y[8], *gx, *gx2, *gy, *part;
    size_t room;   // floats at part
};
static MedWs med_carve(int n, int H, int K, const float *h, void *workspace, size_t bytes) {
    const size_t slot = med_slot(n, H) / sizeof(float);
    MedWs w{};
    float *p = (float *)workspace;
    w.x[0] = const_cast<float *>(h);
    for (int k = 1; k <= K; ++k) w.x[k] = p + slot * k;
    for (int k = 0; k < K; ++k) w.y[k] = p + slot * (K + 1 + k);
    w.gx = p + slot * (2 * K + 1);
    w.gx2 = w.gx + slot;
    w.gy = w.gx2 + slot;
    w.part = w.gy + slot;
    // all of the split area or none, however much larger the workspace is: the split count, and with it the last bits of a
    // result, goes by the shapes alone
    const size_t parts = MED_PARTS * med_slot(n, H);
    w.room = bytes - med_need(n, H, K) >= parts ? parts / sizeof(float) : 0;
    return w;
}

static void medusa_forward(hipStream_t st, int n, int H, int K, float *const *blocks_w, const MedWs &w) {
    const int S = x3_splits(n, H, H, w.room, false);
    for (int k = 0; k < K; ++k) {
        gemm_nt(st, w.x[k], blocks_w[k], w.y[k], w.part, S, n, H, H);
        sum_parts<SUM_SILU>(st, S > 1 ? w.part : w.y[k], S, n, H, w.x[k], w.y[k], w.x[k + 1]);
    }
}

static koala_status med_check(int n_rows, int hidden, int vocab, int K, float *const *blocks_w, size_t workspace_bytes,
                              float lr) {
    if (n_rows < 1 || hidden < 1 || K < 1 || K > 8 || vocab < 1 || !(lr >= 0.f)) return KOALA_E_SHAPE;
    if (workspace_bytes < med_need(n_rows, hidden, K)) return KOALA_E_WORKSPACE;
    for (int k = 0; k < K; ++k)
        if (!blocks_w[k]) return KOALA_E_NULL;
    return KOALA_OK;
}

koala_status koala_train_medusa_head_forward(void *hip_stream, int n_rows, int hidden, int vocab, int K,
                                             float *const *blocks_w, const float *w_lm, const float *h,
                                             void *workspace, size_t workspace_bytes, float *d_logits) {
    if (!blocks_w || !w_lm || !h || !workspace || !d_logits) return KOALA_E_NULL;
    const koala_status rc = med_check(n_rows, hidden, vocab, K, blocks_w, workspace_bytes, 0.f);
    if (rc != KOALA_OK) return rc;
    hipStream_t st = (hipStream_t)hip_stream;
    const MedWs w = med_carve(n_rows, hidden, K, h, workspace, workspace_bytes);
    medusa_forward(st, n_rows, hidden, K, blocks_w, w);
    const int S = x3_splits(n_rows, vocab, hidden, w.room, false);
    gemm_nt(st, w.x[K], w_lm, d_logits, w.part, S, n_rows, vocab, hidden);
    if (S > 1) sum_parts<SUM_ONLY>(st, w.part, S, n_rows, vocab, nullptr, d_logits, nullptr);
    return hipGetLastError() == hipSuccess ? KOALA_OK : KOALA_E_DEVICE;
}

koala_status koala_train_medusa_head_step(void *hip_stream, int n_rows, int hidden, int vocab, int K,
                                          float *const *blocks_w, const float *w_lm, const float *h,
                                          const float *grad_d, float lr, void *workspace, size_t workspace_bytes) {
    if (!blocks_w || !w_lm || !h || !grad_d || !workspace) return KOALA_E_NULL;
    const koala_status rc = med_check(n_rows, hidden, vocab, K, blocks_w, workspace_bytes, lr);
    if (rc != KOALA_OK) return rc;
    hipStream_t st = (hipStream_t)hip_stream;
    const int n = n_rows, H = hidden, V = vocab;
    MedWs w = med_carve(n, H, K, h, workspace, workspace_bytes);
    medusa_forward(st, n, H, K, blocks_w, w);
    const int Sv = x3_splits(n, H, V, w.room, true), Sh = x3_splits(n, H, H, w.room, true);
    gemm_nn(st, grad_d, w_lm, w.gx, w.part, Sv, n, H, V);                 // gx = grad_d W_lm, gy = gx * SiLU'(y)
    sum_parts<SUM_BACK>(st, Sv > 1 ? w.part : w.gx, Sv, n, H, w.y[K - 1], w.gx, w.gy);
    for (int k = K - 1; k >= 0; --k) {
        // gx <- gx + gy W_k with the block's old weights, and gy for the block below
        if (k > 0) gemm_nn(st, w.gy, blocks_w[k], w.gx2, w.part, Sh, n, H, H);
        gemm_update(st, w.gy, w.x[k], blocks_w[k], H, H, n, lr);             // W_k -= lr * gy^T x_k
        if (k > 0) {
            sum_parts<SUM_BACK>(st, Sh > 1 ? w.part : w.gx2, Sh, n, H, w.y[k - 1], w.gx2, w.gy, w.gx);
            std::swap(w.gx, w.gx2);
        }
    }
    return hipGetLastError() == hipSuccess ? KOALA_OK : KOALA_E_DEVICE;
}

}  // extern "C"
