// MFMA (matrix-core) forward path for bf16 models: launch plan and entry points.
#pragma once
#include "common.h"

#define FC_MAX_COUNTERS 8192
#define FC_MAX_ATTN_SPLITS 16 // largest split of the key range across workgroups

struct FastPlan {
    int32_t attn_splits;
    int32_t attn_cut;  // units past the last full round of CUs may run in key splits (fc_attn16_rest); 0: every unit in attn_splits splits, as asked for
    int32_t attn_bpw;  // key blocks of 32 per attention workgroup (decides at run time how many of the splits work)
    int32_t attn_many; // many-row attention kernel (attnp.hip): 0 never, 1 where it gives half of the CUs a workgroup, 2 for every pass of more than 32 rows per sequence
    int32_t co_single; // column-owner GEMM: pairs of k-tiles under way per wave for every GEMM as co_sb below; 2 = per GEMM (co_sb)
    int32_t co_sb[2][5];   // ... for up to 16 rows [0] and 17..32 rows [1]: 0 two, 1 one, 2 by the n-tiles a workgroup owns
    int32_t co_rot[2][5];  // per GEMM: walk the pairs in an order rotated by workgroup and wave: 0 no, 1 yes, 2 plain tiles of up to eight n-tiles per workgroup
    int32_t ks[5];     // column-owner GEMM: K slices per owner (residual GEMMs only; 1 elsewhere)
    int32_t nw2[5], ks2[5];   // the same for passes of 17..32 rows (two row tiles per workgroup)
    int32_t nw[5];     // column-owner GEMM: workgroups for QKV, O, gate/up, down, LM head
    int32_t ks_rule[5];   // K slices a rule over sizes chose where a workgroup count set later may go with half as many; 0: as they are
};
struct FastArgs {
    KernelDims kd;     // kd.M = rows of this pass
    int Bact, lmhead;
    int ctx_len = 0;   // positions of the longest sequence with this pass's rows, as far as the host knows (a lower bound)
    const ModelMap* mm;
    const WorkspaceMap* wm;
    const char* weights;
    char* ws;
    float* dbg_logits;
    const FastPlan* plan;
    hipStream_t st;
    void* prof;
    hipError_t (*prof_mark)(void*, int);
    RowMap rm = RowMap{nullptr, nullptr, nullptr};   // packed rows of a step with per-sequence windows (kd.M = their sum, kd.W = the largest)
    bool accept = false;   // the pass is a Jacobi step: the accept step follows the argmax, in the same launch where that pays ...
    bool* accepted = nullptr;   // ... and *accepted says whether it did
    bool coded = false;    // the coded copies of the weights have been made
    int dbg_stop;      // debug: number of stages to run (5 per layer), < 0 = all
};

// true when the MFMA path covers this shape (else the caller uses the plain kernels)
bool fc_fast_supported(const KernelDims& kd, int rows);
void fc_fast_scratch_sizes(const KernelDims& kd, size_t* gemm_part_bytes, size_t* attn_part_bytes);
void fc_fast_plan(const KernelDims& kd, FastPlan* plan);
hipError_t fc_fast_forward(const FastArgs& a);
// true: a pass of kd.W rows per sequence runs its attention as workgroups of one query tile, with *splits key splits
bool fc_attn_one_tile(const KernelDims& kd, int Bact, const FastPlan& plan, int ctx_len, int* splits);
// which of the attention launch's forms such a pass takes (one query tile, cut last units, many rows): a captured step stays valid while this is the same
int fc_attn_form(const KernelDims& kd, int Bact, const FastPlan& plan, int ctx_len);
// isolation launchers (same kernels as the step)
size_t fc_attn_iso_scratch_bytes(int W, int H, int Dh);
hipError_t fc_attn_iso(const float* q, const void* kc, const void* vc, int n, int W, int H, int Hkv, int Dh, int S,
                       int dt, float* out, void* scratch, hipStream_t st);
size_t fc_lmhead_iso_scratch_bytes(int M, int d, int V);
hipError_t fc_lmhead_iso(const float* act, const void* packed, int M, int d, int V, int32_t* ids, float* top, float* top2,
                         float* logits, void* scratch, hipStream_t st);
