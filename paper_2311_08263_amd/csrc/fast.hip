// MFMA forward path for bf16 models: per layer five launches (QKV+RoPE+cache write, attention,
// O-proj+residual, gate/up+SwiGLU, down+residual), then the LM head with fused argmax.
#include <string.h>
#include "kernels.h"
#include "attn16.h"
#include "gemmco.h"
#include "gemm256.h"

enum { KK_EMBED = 0, KK_QKV = 2, KK_ATTN = 4, KK_O = 5, KK_GU = 6, KK_DOWN = 8, KK_LM = 9, KK_ARGMAX = 10 };

bool fc_fast_supported(const KernelDims& kd, int rows) {
    return kd.esz == 2 && kd.Dh == 128 && rows >= 1 && kd.d % 256 == 0 && kd.F % 256 == 0 &&
           (kd.H * kd.Dh) % 256 == 0 && kd.S % 32 == 0 && kd.V % 16 == 0;
}

void fc_fast_plan(const KernelDims& kd, FastPlan* p) {
    memset(p, 0, sizeof(*p));
    // at most 8 key splits: the last workgroup to arrive folds up to 8 partial results in one round of loads
    // (measured at 2050 positions, 32 heads: 8 splits 24 us, 12 splits 32 us; at 350 positions 6 splits of 2
    // key blocks 12.7 us, 3 splits of 4 blocks 14.9 us)
    int nb = (kd.S + 31) / 32, sp = (nb + 1) / 2;
    if (sp > 8) sp = 8;
    // and no more workgroups than CUs: the kernel's register budget allows one workgroup per CU, a second
    // round costs more than the split saves (measured: 64 heads, 600 positions: 4 splits 20.6 us, 8 splits
    // 24.3 us; batch 8 x 40 heads: 1 split 75 us, 2 splits 102 us)
    while (sp > 1 && kd.B * kd.H * sp > fc_num_cus()) --sp;
    p->attn_splits = sp < 1 ? 1 : sp;
    p->attn_cut = 1;
    p->attn_bpw = 2;
    p->attn_many = 1;
    // column-owner kernel: workgroups per GEMM (one per CU where the matrix allows)
    const int nts[5] = {kd.qkvN / 16, kd.d / 16, 2 * kd.F / 16, kd.d / 16, kd.V / 16};
    // measured on the 7B shape: one workgroup per CU
    for (int i = 0; i < 5; ++i) { p->nw[i] = fc_gemmco_grid(nts[i], 8, i != 1 && i != 3); p->ks[i] = 1; }
    // K slices per owner cut the activations a workgroup reads and cost a meeting of the slices in memory.  (Contexts of one plan differ by up
    // to 1 % with where their copies lie, at some widths by 5: the lines are drawn where several shapes agree, not at the best of each.)
    if (nts[1] <= 512) {                 // O projection with at most two n-tiles per CU
        // two K slices per owner, four from 4096 inputs on.  Steps with one / two / four slices, us, 16 rows: eight 4096-wide layers 736 / 729 /
        // 720, with grouped K/V heads 806 / 796 / 776, four 6144-wide 594 / 592 / 581, six 5120-wide 723 / 705 / 716, two 8192-wide 561 / 552 /
        // 551, three 9216-wide 923 / 914 / 912; one row 659 / 661 / 663, 696 / 721 / 716, 542 / 533 / 538, 641 / 628 / 641, 504 / 507 / 508,
        // 833 / 830 / 839: what sixteen rows gain a single one nearly loses.  Twelve 2048-wide layers 687 / 670 / 659, 585 / 594 / 610.
        const int G = p->nw[1], K = kd.H * kd.Dh;
        if (G % 2 == 0 && G / 2 <= nts[1] && (nts[1] + G / 2 - 1) / (G / 2) <= 8 && K >= 2048) p->ks[1] = 2;
        if (p->ks[1] == 2 && G % 4 == 0 && (nts[1] + G / 4 - 1) / (G / 4) <= 8 && K >= 4096) p->ks[1] = 4;
    }
    // down projection: K is long and the columns few, so every workgroup would read far more activation
    // bytes than weight bytes (one / two / four / eight slices, us: eight layers of the 7B shape 903 / 862 / 850 / 859, six of 13B
    // 935 / 876 / 859 / 881, two of 70B 678 / 648 / 642; two / four of 24 rows, two 8192-wide layers 676 / 655, eight 4096-wide 888 / 845)
    if (kd.F >= 2 * kd.d && kd.F >= 4096 && p->nw[3] % 4 == 0 && p->nw[3] / 4 <= nts[3] && (nts[3] + p->nw[3] / 4 - 1) / (p->nw[3] / 4) <= 8) p->ks[3] = 4;
    // QKV with few columns over many inputs (grouped K/V heads), one -> two slices, us, 24 / 16 rows / one row: two 8192-wide layers 678 -> 671, 557 -> 552,
    // 507 -> 509, three 9216-wide 1131 -> 1116, 933 -> 925, 836 -> 833.  Narrower layers of 24 rows would gain more (four 6144-wide 681 -> 651, six 5120-wide
    // 849 -> 819) and lose with one row (547 -> 551, 647 -> 650, eight 4096-wide 702 -> 713); with heads of their own slices lose (4096-wide 724 -> 736,
    // 663 -> 681)
    if (kd.d >= 8192 && nts[0] < 3 * fc_num_cus() && p->nw[0] % 2 == 0 && (nts[0] + p->nw[0] / 2 - 1) / (p->nw[0] / 2) <= 8) p->ks[0] = 2;
    p->co_single = 2;
    for (int i = 0; i < 5; ++i) p->co_sb[0][i] = p->co_sb[1][i] = p->co_rot[0][i] = p->co_rot[1][i] = 2;
    if (p->ks[1] == 4) p->ks_rule[1] = 4;
    // 17..32 rows (two row tiles per workgroup, up to 16 output tiles): the same grids where the partial tiles
    // fit the LDS, K slices halved until they divide the grid
    const int kin[5] = {kd.d, kd.H * kd.Dh, kd.d, kd.F, kd.d};
    const bool gained[5] = {true, false, true, false, true};
    for (int i = 0; i < 5; ++i) {
        const int most = fc_gemmco_most(32, kin[i], gained[i]);
        int G2 = p->nw[i];
        const int own = G2 > 0 ? G2 / p->ks[i] : 0;
        if (own < 1 || (nts[i] + own - 1) / own > most) G2 = fc_gemmco_grid(nts[i], most);
        int k2 = p->ks[i];
        if (i == 1 && k2 == 2) k2 = 4;       // (twice the activations: slices pay earlier; eight 2048-wide layers, 24 / 32 rows, two -> four slices 564 / 595 -> 557 / 584 us)
        while (k2 > 1 && (G2 % k2 || G2 / k2 > nts[i] || (nts[i] + G2 / k2 - 1) / (G2 / k2) > most)) k2 >>= 1;
        p->nw2[i] = G2; p->ks2[i] = k2;
    }
}

// Layout of the many-row (more than 32 rows) part of the GEMM scratch, offsets in bytes
struct ManyRowScratch { size_t af_x, af_att, af_h, ssq, part, end; };
static ManyRowScratch many_row_scratch(const KernelDims& kd) {
    auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
    ManyRowScratch m;
    const size_t MP = (size_t)((kd.M + 15) / 16) * 16;
    m.af_x = 0;
    m.af_att = m.af_x + up(fc_split_bytes(kd.M, kd.d));
    m.af_h = m.af_att + up(fc_split_bytes(kd.M, kd.H * kd.Dh));
    m.ssq = m.af_h + up(fc_split_bytes(kd.M, kd.F));
    m.part = m.ssq + up((size_t)(kd.d / 16) * MP * 4);      // at most one partial sum per column tile
    m.end = m.part + (size_t)FC_GEMM256_MAX_SK * kd.M * kd.d * 4;
    return m;
}

void fc_fast_scratch_sizes(const KernelDims& kd, size_t* gemm_part_bytes, size_t* attn_part_bytes) {
    if (!fc_fast_supported(kd, 1)) { *gemm_part_bytes = *attn_part_bytes = 4096; return; }   // the plain kernels use neither
    // column-owner kernel with K slices per owner: per workgroup up to 16 partial tiles of 1 KB and 32 partial row
    // sums; at most as many workgroups as the widest matrix has n-tiles
    int nmax = 2 * kd.F;
    if (kd.qkvN > nmax) nmax = kd.qkvN;
    if (kd.V > nmax) nmax = kd.V;
    *gemm_part_bytes = (size_t)(nmax / 16 + 1) * (16 * 1024 + 32 * 4) + 4096;
    // many-row path: activation fragments, row statistics and split-K partial tiles live in the same scratch
    const size_t big = many_row_scratch(kd).end + 4096;
    if (*gemm_part_bytes < big) *gemm_part_bytes = big;
    *attn_part_bytes = fc_attn16_part_bytes(kd.B * kd.H, FC_MAX_ATTN_SPLITS, kd.Wcap > kd.W ? kd.Wcap : kd.W) + 4096;
}

#define FLAUNCH(kind, call)                                                          \
    do {                                                                             \
        hipError_t e_;                                                               \
        if (a.prof && (e_ = a.prof_mark(a.prof, kind)) != hipSuccess) return e_;     \
        if ((e_ = (call)) != hipSuccess) return e_;                                  \
        if (a.prof && (e_ = a.prof_mark(a.prof, -1)) != hipSuccess) return e_;       \
    } while (0)

// Windows of more than 16 rows at a small batch: workgroups of one query tile each instead of two.  They read K/V twice,
// which costs nothing while the launch is latency-bound, up to so many key blocks per wave (crossing points of both forms'
// launch times over 8 to 64 heads, 1 to 8 sequences, 24 to 128 rows, 250 to 15500 positions as hi + lo pairs):
//   7 with key splits (32 heads 5.8-6.3, 40 heads 6.8), 9 with one split, which saves the merge (8.4-10.6);
//   more where the second reading comes out of the L2: 1.5 times that for 32 or more heads in groups of at least four
//   (10.5-11.2), twice for 64 or more (15.5-22);
//   1.5 times for windows above 32 rows, which the two-tile form reads more than once as well (9.2-12.6), 1.75 times where
//   half of its last unit is empty (12.2-15);
//   30 where the two-tile units need more than two workgroups per CU (24-31, 128 rows);
//   no limit where they leave half of the CUs idle (16 heads on 4, 15500 positions: 51.8 / 65.8 us).
// The choice is within 12 % of the faster form everywhere there, 0.2 % on average.  us with one / two tiles, 32 rows: 7B
// prompt 128 10.1 / 15.6, 6000 50.5 / 45.1; batch 4, 512 21.5 / 27.4, 3000 90.4 / 76.4; 64 heads on 8, 512 14.4 / 18.1, 12000
// 106.7 / 88.3.  The line is drawn at the context, not at the cache's capacity: short contexts are common in large caches.
bool fc_attn_one_tile(const KernelDims& kd, int Bact, const FastPlan& plan, int ctx_len, int* splits) {
    const int cus = fc_num_cus(), tiles = (kd.W + 15) / 16, units = Bact * kd.H * tiles, two = Bact * kd.H * ((tiles + 1) / 2) * plan.attn_splits;
    *splits = plan.attn_splits;
    if (kd.W <= 16 || units > cus) return false;
    int sp = plan.attn_splits;
    while (sp > 1 && units * sp > cus) --sp;
    float most = sp == 1 ? 9.f : 7.f;                            // key blocks per wave
    if (kd.H >= 4 * kd.Hkv && kd.H >= 32) most *= kd.H >= 64 ? 2.f : 1.5f;
    if (tiles > 2) most *= tiles % 2 ? 1.75f : 1.5f;
    if (two > 2 * cus && most < 30.f) most = 30.f;
    if ((float)((ctx_len + 31) / 32) > most * (float)(4 * sp) && 2 * two > cus) return false;
    *splits = sp;
    return true;
}

// passes with many rows per sequence (prompt chunks): one walk over the keys per 128 rows, where that still gives at least half
// of the CUs a workgroup
static bool attn_many_rows(const KernelDims& kd, int Bact, const FastPlan& plan) {
    if (kd.kvp == 3) return false;
    return plan.attn_many == 2 ? kd.W > 32 : (plan.attn_many == 1 && kd.W >= 64 && 2 * fc_attnp_workgroups(Bact, kd.H, kd.W) >= fc_num_cus());
}

int fc_attn_form(const KernelDims& kd, int Bact, const FastPlan& plan, int ctx_len) {
    if (attn_many_rows(kd, Bact, plan)) return 4;            // (one form for every length)
    int splits, rest_splits;
    const int one = fc_attn_one_tile(kd, Bact, plan, ctx_len, &splits), rows = kd.W <= 16 || one ? 16 : 32;
    return one | (fc_attn16_rest(kd.W, one ? 16 : 0, Bact * kd.H * ((kd.W + rows - 1) / rows), splits, kd.kvp, plan.attn_cut ? ctx_len : 0, &rest_splits) ? 2 : 0);
}

hipError_t fc_fast_forward(const FastArgs& a) {
    const KernelDims& kd = a.kd;
    const ModelMap& mm = *a.mm; const WorkspaceMap& wm = *a.wm;
    const int M = kd.M, d = kd.d, qd = kd.H * kd.Dh;
    char* ws = a.ws; const char* wt = a.weights;
    int32_t* stp = (int32_t*)(ws + wm.state);
    float* x = (float*)(ws + wm.x); float* q = (float*)(ws + wm.qkv); float* att = (float*)(ws + wm.att);
    float* h = (float*)(ws + wm.h);
    struct { const int32_t* n_state; const float* cosT; const float* sinT; bf16_t* kc; bf16_t* vc; float* amax_val; int layer; } g;
    g.n_state = stp + wm.st.n; g.cosT = (const float*)(ws + wm.rope_cos); g.sinT = (const float*)(ws + wm.rope_sin);
    g.kc = (bf16_t*)(ws + wm.kc); g.vc = (bf16_t*)(ws + wm.vc);
    g.amax_val = (float*)(ws + wm.amax_part); g.layer = 0;
    AttnArgs at; memset(&at, 0, sizeof(at));
    at.q = q; at.ldq = qd; at.kc = g.kc; at.vc = g.vc; at.B = kd.B; at.H = kd.H; at.Hkv = kd.Hkv; at.S = kd.S; at.W = kd.W; at.kvp = kd.kvp;
    at.rstart = a.rm.rstart;
    at.n_state = g.n_state; at.out = att; at.ldo = qd; at.part = (float*)(ws + wm.attn_part); at.cnt = (int32_t*)(ws + wm.attn_cnt); at.bpw = a.plan->attn_bpw;

    GemmCoArgs co; memset(&co, 0, sizeof(co));
    co.M = M; co.eps = kd.eps; co.n_state = g.n_state; co.cosT = g.cosT; co.sinT = g.sinT; co.kc = g.kc; co.vc = g.vc;
    co.H = kd.H; co.Hkv = kd.Hkv; co.B = kd.B; co.S = kd.S; co.Wn = kd.W; co.kvp = kd.kvp; co.kvq = kd.kvq;
    co.amax_val = g.amax_val; co.single_buffer = 2; co.rm = a.rm;
    co.stamp = (const uint64_t*)(wt + mm.stamp_off); co.record = (const uint64_t*)(ws + wm.code_record);
    Gemm256Args big; memset(&big, 0, sizeof(big));
    big.M = M; big.n_state = g.n_state; big.cosT = g.cosT; big.sinT = g.sinT; big.kc = g.kc; big.vc = g.vc;
    big.H = kd.H; big.Hkv = kd.Hkv; big.B = kd.B; big.S = kd.S; big.Wn = kd.W; big.kvp = kd.kvp; big.kvq = kd.kvq;
    big.amax_stride = (M + 15) / 16 * 16; big.rm = a.rm;
    // many-row scratch: the fragments of x, of the attention output and of the hidden activations, the partial
    // row sums of squares of x, then the split-K partial tiles
    const ManyRowScratch mrs = many_row_scratch(kd);
    bf16_t* af_x = (bf16_t*)(ws + wm.gemm_part + mrs.af_x); bf16_t* af_att = (bf16_t*)(ws + wm.gemm_part + mrs.af_att);
    bf16_t* af_h = (bf16_t*)(ws + wm.gemm_part + mrs.af_h); float* ssq = (float*)(ws + wm.gemm_part + mrs.ssq);
    big.part = (float*)(ws + wm.gemm_part + mrs.part);
    big.eps = kd.eps;
    // the fragment buffers hold what their fp32 twins would: x (with the gain of the norm that comes next, row scale
    // still to be applied by the consumer from x_nssq partial sums of squares), attention output, hidden activations
    int x_nssq = d / 256;
    const float* next_gain = nullptr;          // gain the next residual GEMM folds into the fragments of x
    // LM head: one winner per row and column block
    const int lm_ncb = fc_gemm256_plan(M, kd.V / 16, 1, 2).ncb;
    big.amax_val = g.amax_val; big.amax_idx = (int32_t*)(g.amax_val + (size_t)lm_ncb * big.amax_stride);
    int gi = 0;        // which GEMM of the plan
    auto gemm = [&](int epi, const char* base, const FusedMat& fm, const float* X, const float* gain, float* out, int ldo) {
        const char* W = base + fm.off;
        const int K = fm.K, N = fm.N, ldx = fm.K;
        // workgroups of the column-owner kernel and its K slices per owner
        const int nw = M <= 16 ? a.plan->nw[gi] : (M <= 32 ? a.plan->nw2[gi] : 0);
        const int ksl = M <= 16 ? a.plan->ks[gi] : a.plan->ks2[gi];
        if (nw > 0) {
            co.W = (const bf16_t*)W; co.K = K; co.NT = N / 16; co.X = X; co.ldx = ldx; co.gain = gain; co.out = out; co.ldo = ldo;
            co.C = a.coded && g.layer < wm.code_layers[gi] ? ws + wm.code[gi] + (size_t)g.layer * wm.code_stride[gi] : nullptr;
            co.layer = g.layer; co.ks = epi != EPI_LMHEAD ? ksl : 1; co.hi_only = (kd.actq >> gi) & 1;
            co.single_buffer = a.plan->co_single == 2 ? a.plan->co_sb[M > 16][gi] : a.plan->co_single;
            co.rotate = a.plan->co_rot[M > 16][gi];
            co.xpart = (float*)(ws + wm.gemm_part); co.xcnt = (int32_t*)(ws + wm.gemm_cnt);
            co.amax_idx = (int32_t*)(co.amax_val + (size_t)nw * (M > 16 ? 32 : 16));
            return fc_gemmco(epi, co, nw, a.st);
        }
        if (M > 32) {        // many rows: the input is fragments its producer has written
            bf16_t* af = X == x ? af_x : (X == att ? af_att : af_h);
            big.ssq = X == x ? ssq : nullptr; big.nssq = X == x ? x_nssq : 0;
            big.sk = epi == EPI_RESID ? fc_gemm256_sk(M, K, N / 16) : 1;
            big.W = (const bf16_t*)W; big.K = K; big.NT = N / 16; big.AF = af; big.out = out; big.ldo = ldo; big.layer = g.layer;
            big.hfrag = nullptr; big.rf_AF = nullptr; big.rf_gain = nullptr; big.rf_ssq = nullptr;
            if (epi == EPI_SWIGLU) {            // the hidden activations leave as fragments (fp32 copy only for debugging)
                big.hfrag = af_h;
                if (a.dbg_stop < 0) big.out = nullptr;
            }
            if (epi == EPI_RESID) {
                big.rf_AF = af_x; big.rf_gain = next_gain; big.rf_ssq = ssq;
                x_nssq = fc_gemm256_nssq(M, N / 16, big.sk);
            }
            return fc_gemm256(epi, big, a.st);
        }
        return hipErrorInvalidValue;       // every plan gives the column-owner kernel a grid
    };

    if (M > 32)
        FLAUNCH(KK_EMBED, fc_embed_split(wt + mm.emb_off, stp + wm.st.win, x, M, d, kd.V, a.rm, kd.W,
                                         (const float*)(kd.L > 0 ? wt + mm.layers_off + mm.g1_off : wt + mm.gf_off), af_x, ssq, a.st));
    else
        FLAUNCH(KK_EMBED, fc_embed(wt + mm.emb_off, FASTCOT_BF16, stp + wm.st.win, x, M, d, kd.V, a.st, a.rm, kd.W));
    int nstage = 0;
#define DBG_STOP() do { if (a.dbg_stop >= 0 && nstage++ >= a.dbg_stop) return hipSuccess; } while (0)
    for (int l = 0; l < kd.L; ++l) {
        const char* lb = wt + mm.layers_off + (size_t)l * mm.layer_stride;
        g.layer = l; at.layer = l;
        DBG_STOP();
        gi = 0;
        FLAUNCH(KK_QKV, gemm(EPI_QKV, lb, mm.qkv, x, (const float*)(lb + mm.g1_off), q, qd));
        DBG_STOP();
        if (M > 32) {                  // the many-row O projection reads fragments: attention writes them itself
            at.ofrag = af_att;
            at.out = a.dbg_stop >= 0 ? att : nullptr;
        }
        int attn_splits;
        at.subrows = fc_attn_one_tile(kd, a.Bact, *a.plan, a.ctx_len, &attn_splits) ? 16 : 0;
        at.ctx = a.plan->attn_cut ? a.ctx_len : 0;
        if (attn_many_rows(kd, a.Bact, *a.plan))
            FLAUNCH(KK_ATTN, fc_attnp(at, a.Bact, a.st));
        else
        FLAUNCH(KK_ATTN, fc_attn16(at, a.Bact, attn_splits, a.st));
        DBG_STOP();
        gi = 1;
        next_gain = (const float*)(lb + mm.g2_off);
        FLAUNCH(KK_O, gemm(EPI_RESID, lb, mm.o, att, nullptr, x, d));
        DBG_STOP();
        gi = 2;
        FLAUNCH(KK_GU, gemm(EPI_SWIGLU, lb, mm.gu, x, (const float*)(lb + mm.g2_off), h, kd.F));
        DBG_STOP();
        gi = 3;
        next_gain = l + 1 < kd.L ? (const float*)(wt + mm.layers_off + (size_t)(l + 1) * mm.layer_stride + mm.g1_off) : (const float*)(wt + mm.gf_off);
        FLAUNCH(KK_DOWN, gemm(EPI_RESID, lb, mm.down, h, nullptr, x, d));
    }
    if (a.dbg_stop >= 0 && nstage >= a.dbg_stop) return hipSuccess;
    if (a.lmhead) {
        const int stride = M > 16 ? 32 : 16;
        const int nwlm = M <= 16 ? a.plan->nw[4] : (M <= 32 ? a.plan->nw2[4] : 0);
        const int nwin = nwlm;                                // partial winners to reduce
        gi = 4; g.layer = 0;
        FLAUNCH(KK_LM, gemm(EPI_LMHEAD, wt, mm.lm, x, (const float*)(wt + mm.gf_off), a.dbg_logits, kd.V));
        if (a.accept && fc_tail_fits(a.Bact, kd.W, M, nwin, true)) {
            FLAUNCH(KK_ARGMAX, fc_tail_winners(g.amax_val, (const int32_t*)(g.amax_val + (size_t)nwin * stride), nwin, stride, M, (float*)(ws + wm.topv),
                                               a.rm, stp, wm.st, a.Bact, kd.W, kd.S, a.st));
            *a.accepted = true;
        } else if (M <= 32)
            FLAUNCH(KK_ARGMAX, fc_argmax_final(g.amax_val, (const int32_t*)(g.amax_val + (size_t)nwin * stride), nwin, stride, M, stp + wm.st.o,
                                               (float*)(ws + wm.topv), a.st, a.rm, kd.W));
        else
            FLAUNCH(KK_ARGMAX, fc_argmax_final(big.amax_val, big.amax_idx, lm_ncb, big.amax_stride, M,
                                               stp + wm.st.o, (float*)(ws + wm.topv), a.st, a.rm, kd.W));
    }
    return hipSuccess;
}

// ------------------------------------------------------------------ isolation launchers
static int iso_attn_splits(int S) {
    int nb = (S + 31) / 32, sp = (nb + 1) / 2;
    return sp < 1 ? 1 : (sp > 8 ? 8 : sp);
}
// scratch: 256 bytes unused, the arrival counters of FC_MAX_COUNTERS units, then split partials: the counters (zero
// between calls) lie where no call of another shape keeps partials, so one scratch serves calls of different shapes
#define ISO_PART_OFF (256 + (size_t)FC_MAX_COUNTERS * 4)
size_t fc_attn_iso_scratch_bytes(int W, int H, int Dh) {
    return ISO_PART_OFF + fc_attn16_part_bytes(H, FC_MAX_ATTN_SPLITS, W);
}
// The committed length travels as a kernel argument: with a launch in front that stored it for the kernel to read the
// call took 15.6 us, without 13.8 us (32 heads, 2064 keys, 16 rows).
hipError_t fc_attn_iso(const float* q, const void* kc, const void* vc, int n, int W, int H, int Hkv, int Dh, int S,
                       int dt, float* out, void* scratch, hipStream_t st) {
    char* sc = (char*)scratch;
    const int units = H * (W > 32 ? (W + 15) / 16 : 1);
    if (dt != FASTCOT_BF16 || Dh != 128 || S % 32 || units > FC_MAX_COUNTERS) {
        KernelDims kd{}; kd.L = 1; kd.H = H; kd.Hkv = Hkv; kd.Dh = Dh; kd.B = 1; kd.S = S; kd.W = W; kd.M = W; kd.kvp = 1;
        return fc_attn_plain(q, H * Dh, kc, vc, dt, kd, 0, nullptr, n, out, st);
    }
    AttnArgs at; memset(&at, 0, sizeof(at));
    at.q = q; at.ldq = H * 128; at.kc = (const bf16_t*)kc; at.vc = (const bf16_t*)vc; at.layer = 0; at.B = 1; at.H = H;
    at.Hkv = Hkv; at.S = S; at.W = W; at.kvp = 1; at.n_host = n; at.ctx = n + W; at.out = out; at.ldo = H * 128;
    at.cnt = (int32_t*)(sc + 256); at.bpw = 2;
    at.part = (float*)(sc + ISO_PART_OFF);
    int splits = iso_attn_splits(n + W);
    // More than 32 rows: units of 16 rows, queries and probabilities as three bf16 parts, because such a call has
    // always computed in fp32 (error against 64 bits 7e-7; two parts would be 3e-6, three are 3.4e-7).
    // 64 rows, 1088 keys, 40 heads: plain kernel 172 us, this 14.0 us.
    // Key splits only while every workgroup has a CU to itself (64 heads on 8, 782 keys, 5 rows: 8 splits 11.3 us, 4 splits
    // 10.4 us; 17 rows, 1024 keys: 16.6 and 13.3 us).  Units of two query tiles are built for two workgroups per CU and may
    // have them where heads share K/V and a wave would otherwise walk more than eight key blocks, of more than 96 (64 heads
    // on 8, 17 rows: 5000 keys 26.3 -> 22.5 us, 15000 keys 65.2 -> 45.2; at 2048 keys 15.5 us without and 17.8 with; 40 heads
    // with K/V of their own, 15000 keys: 58.4 without and 63.1 with).
    if (W > 32) { at.terms = 3; at.subrows = 16; }
    const int most = splits;
    while (splits > 1 && units * splits > fc_num_cus()) --splits;
    const int nb = (n + W + 31) / 32;
    if (W > 16 && W <= 32 && H > Hkv && nb > 8 * 4 * splits && nb > 96)
        for (splits = most; splits > 1 && units * splits > 2 * fc_num_cus();) --splits;
    return fc_attn16(at, 1, splits, st);
}

// scratch: winners per workgroup [workgroups][32] value + index, then room for logits (where they are not asked for),
// then, for more than 32 rows, the activations as three bf16 parts and the winners per column block
static int lm_iso_grid(int M, int d, int V) { return fc_gemmco_grid(V / 16, M > 16 ? fc_gemmco_most(32, d, false) : 8, M <= 16); }
// more than 32 rows of a width the many-row kernel takes, within its 32-bit byte offsets
static bool lm_iso_many(int M, int d, int V) {
    return M > 32 && d % 256 == 0 && (size_t)V * d * 2 < ((size_t)1 << 32) && fc_split_bytes(M, d, 3) < ((size_t)1 << 32);
}
static size_t lm_iso_logits_end(int M, int V) { return FC_ALIGN((size_t)(V / 16 + 1) * 32 * 8 + 256 + (size_t)M * V * 4); }
size_t fc_lmhead_iso_scratch_bytes(int M, int d, int V) {
    const size_t base = lm_iso_logits_end(M, V);
    if (!lm_iso_many(M, d, V)) return base;
    return base + FC_ALIGN(fc_split_bytes(M, d, 3)) + (size_t)(V / 16) * ((M + 15) / 16 * 16) * 8;
}
// largest logit of every row among the ids other than the row's winner
__global__ void k_top2(const float* logits, int V, const int32_t* ids, float* top2) {
    __shared__ float sv[4];
    const int m = blockIdx.x, win = ids[m];
    float best = -INFINITY;
    for (int n = threadIdx.x; n < V; n += blockDim.x) { const float v = logits[(size_t)m * V + n]; if (n != win && v > best) best = v; }
    for (int o = 32; o > 0; o >>= 1) best = fmaxf(best, __shfl_xor(best, o, 64));
    if ((threadIdx.x & 63) == 0) sv[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) top2[m] = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
}
hipError_t fc_lmhead_iso(const float* act, const void* packed, int M, int d, int V, int32_t* ids, float* top, float* top2,
                         float* logits, void* scratch, hipStream_t st) {
    char* sc = (char*)scratch;
    float* lg_scratch = (float*)(sc + (size_t)(V / 16 + 1) * 32 * 8 + 256);
    if (top2 && !logits) logits = lg_scratch;              // the runner-up is read off the logits
    if (lm_iso_many(M, d, V)) {
        // the many-row kernel on activations in three bf16 parts: such a call has always computed in fp32, and two
        // parts would leave the logits 2.3e-6 off.  256 rows x 5120 x 32000: the plain product of that time 3.19 ms, this 192 us.
        const size_t off = lm_iso_logits_end(M, V);
        Gemm256Args g; memset(&g, 0, sizeof(g));
        g.W = (const bf16_t*)packed; g.K = d; g.NT = V / 16; g.AF = (bf16_t*)(sc + off); g.planes = 3; g.M = M; g.out = logits; g.ldo = V;
        g.sk = 1; g.amax_stride = (M + 15) / 16 * 16;
        g.amax_val = (float*)(sc + off + FC_ALIGN(fc_split_bytes(M, d, 3)));
        const int ncb = fc_gemm256_plan(M, V / 16, 1, 3).ncb;
        g.amax_idx = (int32_t*)(g.amax_val + (size_t)ncb * g.amax_stride);
        hipError_t e = fc_split3(act, d, M, d, (bf16_t*)(sc + off), st);
        if (e == hipSuccess) e = fc_gemm256(EPI_LMHEAD, g, st);
        if (e == hipSuccess) e = fc_argmax_final(g.amax_val, g.amax_idx, ncb, g.amax_stride, M, ids, top, st);
        if (e != hipSuccess || !top2) return e;
        k_top2<<<M, 256, 0, st>>>(logits, V, ids, top2);
        return hipGetLastError();
    }
    if (M > 32 || d % 256) {
        float* lg = logits ? logits : lg_scratch;
        hipError_t e = fc_gemm_plain(packed, FASTCOT_BF16, d, V, V, act, d, lg, V, M, 0, st);
        if (e != hipSuccess) return e;
        e = fc_argmax_plain(lg, M, V, ids, top, st);
        if (e != hipSuccess || !top2) return e;
        k_top2<<<M, 256, 0, st>>>(lg, V, ids, top2);
        return hipGetLastError();
    }
    GemmCoArgs co; memset(&co, 0, sizeof(co));
    const int nwg = lm_iso_grid(M, d, V), stride = M > 16 ? 32 : 16;
    co.W = (const bf16_t*)packed; co.C = (const char*)packed + wc_off(d, V / 16); co.K = d; co.NT = V / 16; co.X = act; co.ldx = d; co.M = M; co.out = logits; co.ldo = V;
    co.stamp = co.record = (const uint64_t*)packed;        // (the copy was packed with the tiles)
    co.single_buffer = co.rotate = 2;
    co.amax_val = (float*)sc;
    co.amax_idx = (int32_t*)(co.amax_val + (size_t)nwg * stride);
    hipError_t e = fc_gemmco(EPI_LMHEAD, co, nwg, st);
    if (e != hipSuccess) return e;
    e = fc_argmax_final(co.amax_val, co.amax_idx, nwg, stride, M, ids, top, st);
    if (e != hipSuccess || !top2) return e;
    k_top2<<<M, 256, 0, st>>>(logits, V, ids, top2);
    return hipGetLastError();
}
