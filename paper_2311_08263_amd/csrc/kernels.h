// Host-side launchers of all kernels (each enqueues on `st` and returns the hipGetLastError code).
#pragma once
#include "common.h"

// text of the last failure of a context-less call (what fastcot_last_error(NULL) returns)
void fc_set_error(const char* msg);

// ---- plain kernels (fp32 arithmetic without matrix cores; used for fp32 models and as the on-device cross-check)
// x[m] = embedding of win[m] (dense), or of win[rowb[m] * W + rowj[m]] with a row map
hipError_t fc_embed(const void* emb, int dt, const int32_t* win, float* x, int M, int d, int V, hipStream_t st,
                    RowMap rm = RowMap{nullptr, nullptr, nullptr}, int W = 0);
// argument block of the plain GEMM (a norm in front where gain is given; the QKV fields only for fc_qkv_plain)
struct PlainGemm {
    const void* W; int32_t K, NP, N;       // fused matrix: K inputs, N of NP columns
    const float* X; int32_t ldx;
    float* Y; int32_t ldy, M;
    const float* gain; float eps;
    const float* emb; const int32_t* tok; int32_t V;   // emb not NULL: row m of the residual stream is still the embedding of token tok[m]
                                                       // (< V): the inputs X of a product with a norm in front, what an adding one adds to
    KernelDims kd; int32_t layer;
    float* qrot; const int32_t* n_state; const float* cosT; const float* sinT; void* kc; void* vc;
};
// residual rows that no launch has written yet: the fp32 embeddings of tokens tok[m] (all NULL / 0: the rows are in memory)
struct TokenRows { const float* emb; const int32_t* tok; int32_t V; };
hipError_t fc_gemm_plain(const void* W, int dt, int K, int NP, int N, const float* X, int ldx, float* Y, int ldy,
                         int M, int accumulate, hipStream_t st, const float* gain = nullptr, float eps = 0.f, TokenRows tr = TokenRows{nullptr, nullptr, 0});
// QKV product of the normed rows, rotary embedding and cache write; qkv keeps the product as it was before the rotation
hipError_t fc_qkv_plain(const void* W, int dt, const KernelDims& kd, int layer, const float* X, const float* gain, float* qkv, float* qrot,
                        const int32_t* n_state, const float* cosT, const float* sinT, void* kc, void* vc, hipStream_t st,
                        TokenRows tr = TokenRows{nullptr, nullptr, 0});
// committed lengths from n_state[b], or n_host for every sequence where that is NULL
hipError_t fc_attn_plain(const float* q, int ldq, const void* kc, const void* vc, int dt, const KernelDims& kd,
                         int layer, const int32_t* n_state, int n_host, float* out, hipStream_t st);
// gate/up product of the normed rows and SwiGLU: h [M][F]
hipError_t fc_swiglu_plain(const void* W, int dt, int K, int F, const float* X, int ldx, float* h, int M, const float* gain,
                           float eps, hipStream_t st);
hipError_t fc_argmax_plain(const float* logits, int M, int V, int32_t* ids, float* top, hipStream_t st);

// ---- decoding-state kernels
hipError_t fc_prefill_window(int32_t* state, const StateMap& sm, int B, int R, int S, int p0, hipStream_t st);
hipError_t fc_prefill_advance(int32_t* state, const StateMap& sm, int B, int W, int S, int p1, int last,
                              hipStream_t st);
hipError_t fc_rewindow(int32_t* state, const StateMap& sm, int B, int W, int S, hipStream_t st);
hipError_t fc_accept_commit(int32_t* state, const StateMap& sm, int B, int W, int S, hipStream_t st);
// g[B], done[B], flags[2] to pinned host memory
hipError_t fc_report(const int32_t* state, const StateMap& sm, int B, int32_t* host, hipStream_t st);
// argmax of a step's rows and the accept step in one launch, where fc_tail_fits (rows M, logits per row or partial winners per row)
bool fc_tail_fits(int B, int W, int M, int V_or_parts, bool winners);
hipError_t fc_tail_logits(const float* logits, int M, int V, float* top, int32_t* state, const StateMap& sm, int B, int W, int S, hipStream_t st);
hipError_t fc_tail_winners(const float* val, const int32_t* idx, int nparts, int stride, int M, float* top, RowMap rm, int32_t* state,
                           const StateMap& sm, int B, int W, int S, hipStream_t st);
// sequences b1 and b2 trade slots: state entries and K/V cache (seq_bytes per sequence and layer, layers layer_stride_bytes apart)
hipError_t fc_swap_sequences(int32_t* state, const StateMap& sm, int b1, int b2, int W, int S, void* kc, void* vc,
                             size_t seq_bytes, int layers, size_t layer_stride_bytes, hipStream_t st);

// ---- weight packing
hipError_t fc_pack(const void* src, int dt, int rows, int cols, void* dst_base, const FusedMat& fm, int col_off,
                   int mode /*0 natural, 1 gate, 2 up, 3 + Dh: q/k heads of Dh*/, hipStream_t st, void* stamp = nullptr /*of the packed model, bf16*/, int tensor = 0 /*its own part of it*/);
// the coded copy at C of a matrix of K inputs and NT n-tiles
hipError_t fc_code(const void* W, void* C, int K, int NT, hipStream_t st);
// the record of coded copies takes a packed model's stamp over (made = 0: there are no copies); whether they differ, to host memory
hipError_t fc_stamp_keep(const void* stamp, void* record, int made, hipStream_t st);
hipError_t fc_stamp_look(const void* stamp, const void* record, int* host, hipStream_t st);
hipError_t fc_fill_f32(float* dst, size_t n, float v, hipStream_t st);
hipError_t fc_copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t st);
hipError_t fc_kv_scatter(const void* k, const void* v, int S_in, int Hkv, int Dh, int S, int dt, void* kc, void* vc,
                         hipStream_t st);
