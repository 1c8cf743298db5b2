// Argument block and launchers of the many-row bf16 GEMM (see gemm256.hip).
#pragma once
#include "gemmco.h"

struct Gemm256Args {
    const bf16_t* W;       // fused matrix in fragment order
    int32_t K, NT;         // inputs (multiple of 256), n-tiles
    const bf16_t* AF;      // activations as bf16 hi + lo B-fragments [row tile][k-tile][hi|lo][64 lanes][8]
    int32_t planes;        // 3 = fragments of three parts (fc_split3; LM head only); any other value: hi + lo
    int32_t M;             // rows
    float* out;            // RESID: residual stream (+=); SWIGLU: hidden [M][F]; QKV: q [M][H*128]; LMHEAD: logits or NULL
    int32_t ldo;
    const int32_t* n_state; const float* cosT; const float* sinT;
    bf16_t* kc; bf16_t* vc;
    int32_t layer, H, Hkv, B, S, Wn, kvp, kvq;
    RowMap rm;             // QKV: which sequence and slot a row is (dense when rm.rowb is NULL)
    float* amax_val; int32_t* amax_idx;   // LM head: winners per column block [ncb][amax_stride]
    int32_t amax_stride;
    int32_t sk;            // K slices (RESID only when > 1: partial tiles to `part`, then added in slice order)
    float* part;           // [sk][M][NT*16] fp32
    int32_t ncb;           // column blocks (set by fc_gemm256 from its plan)
    // Activations that arrive without their RMSNorm row scale (fragments written by a residual GEMM, see rf_AF,
    // or by fc_embed_split): ssq [nssq][row tiles * 16] partial row sums of squares; the epilogue multiplies row m by
    // 1 / sqrt(sum_c ssq[c][m] / K + eps) before anything else.  NULL = the fragments are final.
    const float* ssq; int32_t nssq; float eps;
    // SWIGLU: also (or, with out == NULL, only) write the hidden activations as hi + lo fragments for the
    // down projection, [row tile][F / 32][hi|lo][64][8]
    bf16_t* hfrag;
    // RESID: also the new residual rows times rf_gain (the next norm's gain) as hi + lo fragments to rf_AF and their
    // partial sums of squares to rf_ssq [fc_gemm256_nssq][row tiles * 16] (needed with sk > 1, else rf_AF may be NULL)
    bf16_t* rf_AF; const float* rf_gain; float* rf_ssq;
};
#define FC_GEMM256_MAX_SK 8
struct Gemm256Plan { int ksplit, cw, rt, ncb; };   // two k-groups, column tiles per wave, row tiles per block, column blocks (see gemm256.hip)
Gemm256Plan fc_gemm256_plan(int M, int NT, int sk, int planes);
int fc_gemm256_sk(int M, int K, int NT);   // slices that fill the chip for a matrix with few columns
// partial sums per row that a residual GEMM of these sizes leaves in rf_ssq; never more than NT
static inline int fc_gemm256_nssq(int M, int NT, int sk) { return sk > 1 ? NT / 16 : fc_gemm256_plan(M, NT, 1, 2).ncb; }

// X [M][ldx] fp32 -> AF, three parts
hipError_t fc_split3(const float* X, int ldx, int M, int K, bf16_t* AF, hipStream_t st);
static inline size_t fc_split_bytes(int M, int K, int planes = 2) { return (size_t)((M + 15) / 16) * 16 * K * 2 * planes; }
// embedding rows of the pass, with the fragments (times gain) and row sums of squares [d / 256][row tiles * 16] of the first GEMM
hipError_t fc_embed_split(const void* emb, const int32_t* win, float* x, int M, int d, int V, RowMap rm, int W, const float* gain,
                          bf16_t* AF, float* ssq, hipStream_t st);
hipError_t fc_gemm256(int epi, const Gemm256Args& a, hipStream_t st);
