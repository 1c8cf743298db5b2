// Window-causal attention on matrix cores (bf16 KV cache, head_dim 128).
//
// The queries of a step are the W window rows of a sequence; the keys are the committed cache
// positions 0..n-1 plus the window positions n..n+W-1, row j seeing positions <= n+j -- the causal
// mask that lets one forward do lossless and Jacobi decoding together (Sec. 4.3, Eq. 2/4).
//
// One workgroup (4 waves) per (sequence, query head, key split); waves take 32-key blocks round
// robin.  Per block the wave computes S^T = K . Q^T with v_mfma_f32_16x16x32_bf16 (K rows as the
// A operand, straight from the cache with 16-byte loads; Q as the B operand, bf16 hi + lo), a
// running-max softmax in fp32, and O^T += V^T . P^T with V^T rows as the A operand (the V cache is
// stored transposed, [Dh][positions], so these are 16-byte loads too) and P^T, which is exactly the
// register layout the score tiles already have, as the B operand.  The two 16-key score tiles of a
// block interleave keys (tile t row r <-> key 8*(r/4) + 4*t + r%4) so that a lane ends with 8
// consecutive keys.  Waves are merged through LDS (each wave finishes a quarter of the head), key
// splits through a scratch buffer by the last workgroup to arrive, always in index order, so results
// do not depend on timing.  How many of the launched splits work on a sequence is decided at run
// time from its length.
#include "attn16.h"
#include "gemmco.h"      // fc_num_cus
#include "xwg.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4_t;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2_t;
union Frag { u32x4_t u; bf16x8_t v; };

__device__ inline void split8(const float* v, Frag& hi, Frag& lo) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) pk_bf16_hilo(v[2 * e], v[2 * e + 1], h[e], l[e]);
    hi.u = (u32x4_t){h[0], h[1], h[2], h[3]};
    lo.u = (u32x4_t){l[0], l[1], l[2], l[3]};
}

// three bf16 parts: what hi and lo leave over of a fp32 value fits a third
__device__ inline void split8(const float* v, Frag& hi, Frag& lo, Frag& lo2) {
    uint32_t h[4], l[4], m[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float a = v[2 * e], b = v[2 * e + 1];
        h[e] = pk_bf16(a, b);
        const float ra = a - __uint_as_float(h[e] << 16), rb = b - __uint_as_float(h[e] & 0xFFFF0000u);
        pk_bf16_hilo(ra, rb, l[e], m[e]);
    }
    hi.u = (u32x4_t){h[0], h[1], h[2], h[3]};
    lo.u = (u32x4_t){l[0], l[1], l[2], l[3]};
    lo2.u = (u32x4_t){m[0], m[1], m[2], m[3]};
}

#define NEG_BIG (-1.0e30f)
#define REST_BLOCKS(two) ((two) ? 56 : 16)   // key blocks times planes from which a unit of the last round is worth cutting, two / one query tiles
#define PART_FLOATS (8 * 64 * 4 + 128)   // per split of a unit and query tile: O^T tiles, then m[64], l[64] per lane.  Units lie by number with all the
                                         // launch's splits, or, where only the last units are cut, by their number among those

// the bf16 lo operand of eight cached values kept as bf16 hi (h, four words) + 8-bit residual (two words of bytes):
// value - hi = byte * 2^-15 * 2^(exponent of hi), exact in bf16
__device__ inline void expand_lo8(const u32x4_t& h, uint32_t b0, uint32_t b1, Frag& lo) {
    uint32_t o[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t w = h[p], bw = p < 2 ? b0 : b1;
        // scale of the residual's unit: sign and exponent of hi, times 2^-15 (a hi of zero or below the normal
        // range has exponent field 0: its residual is dropped, an error below 2^-126)
        const float s0 = __uint_as_float((w << 16) & 0xFF800000u) * 3.0517578125e-05f;
        const float s1 = __uint_as_float(w & 0xFF800000u) * 3.0517578125e-05f;
        const float d0 = (float)((bw >> (16 * (p & 1))) & 0xFFu) * s0;
        const float d1 = (float)((bw >> (16 * (p & 1) + 8)) & 0xFFu) * s1;
        o[p] = pk_bf16(d0, d1);
    }
    lo.u = (u32x4_t){o[0], o[1], o[2], o[3]};
}

// KVP: 1 = one bf16 plane, 2 = bf16 hi + bf16 lo planes, 3 = bf16 hi plane + a plane of 8-bit residuals
// TERMS: bf16 parts of a query or probability: 2 (17 bits, what the step's path uses) or 3 (25 bits: all of the fp32
// value, for windows of more than 32 rows of the isolated call, whose results are those of fp32 arithmetic; KVP 1 only)
template <int QT, int KVP, int TERMS = 2>
__global__ __launch_bounds__(256, QT) void k_attn16(AttnArgs a) {
    extern __shared__ float lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    // the wave index as a scalar: the block loop below is then uniform control flow
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, g = lane >> 4;
    // a window of more rows than a workgroup takes (16 per query tile) is cut into sub-windows: sub-window `sub` of a sequence is a
    // unit of its own whose rows see the committed positions plus the window rows up to their own (the
    // K/V of all window rows are already in the cache when this kernel starts)
    constexpr int SUBR = 16 * QT;                            // rows of a unit
    const int nsub = (a.W + SUBR - 1) / SUBR;
    // workgroups go to the eight XCDs (each with an L2 of its own) round robin by index, so with grouped
    // K/V heads consecutive indices take different K/V heads: the query heads that share one then follow
    // each other at a stride of Hkv, land on the same XCD when Hkv is a multiple of eight, and fetch the
    // shared planes from memory once instead of once per query head
    // (a launch whose last units are cut in key splits while the others are whole has a grid of one dimension: pieces first, see fc_attn16)
    int bh = blockIdx.x, sp = blockIdx.y, nsp_max = gridDim.y, slot = bh * nsp_max + sp;
    if (a.rest > 0) {
        const int pieces = a.rest * a.rest_splits;
        nsp_max = bh < pieces ? a.rest_splits : 1;
        sp = bh < pieces ? bh / a.rest : 0;
        slot = (bh % a.rest) * a.rest_splits + sp;
        bh = bh < pieces ? a.whole + bh % a.rest : bh - pieces;
    }
    const int hr = bh % a.H, G = a.H / a.Hkv, kvh = hr % a.Hkv, h = kvh * G + hr / a.Hkv;
    const int sub = (bh / a.H) % nsub, b = bh / (a.H * nsub);
    const int Wb = a.rstart ? a.rstart[b + 1] - a.rstart[b] : a.W, rbase = a.rstart ? a.rstart[b] : b * a.W;
    const int row0 = SUBR * sub, Wr = Wb - row0 < SUBR ? Wb - row0 : SUBR;        // rows of this unit
    if (Wr <= 0) return;                                     // a sequence with a smaller window of its own
    const int n = (a.n_state ? a.n_state[b] : a.n_host) + row0;                       // positions every row of the unit sees
    int T = n + Wr;
    if (T > a.S) T = a.S;                                    // capacity guard (the host checks first)
    const int NB = (T + 31) >> 5;
    // splits actually used: about a.bpw key blocks per workgroup (the launch provides nsp_max for the
    // longest context; every workgroup of this (sequence, head) derives the same number from n)
    int nsp = (NB + a.bpw - 1) / a.bpw;
    if (nsp > nsp_max) nsp = nsp_max;
    // a unit of the last round stays whole where its keys are read in less time than its merge costs (see fc_attn16_rest)
    if (a.rest > 0 && NB * (KVP == 1 ? 1 : 2) < REST_BLOCKS(QT == 2)) nsp = 1;
    if (sp >= nsp) return;
    const int blk0 = (int)(((unsigned)sp * (unsigned)NB) / (unsigned)nsp);
    const int blk1 = (int)(((unsigned)(sp + 1) * (unsigned)NB) / (unsigned)nsp);
    const size_t plane = (size_t)a.S * 128;
    constexpr int NPL = KVP == 1 ? 1 : 2;                   // planes of S * 128 elements a block occupies; register sets
    const bf16_t* kbase = a.kc + ((((size_t)a.layer * a.B + b) * a.Hkv + kvh) * NPL) * plane;
    const bf16_t* vbase = a.vc + ((((size_t)a.layer * a.B + b) * a.Hkv + kvh) * NPL) * plane;

    // The softmax runs in powers of two: the queries are multiplied by log2(e) / sqrt(128) before they are split, so scores,
    // maxima and partial results are in that unit.  (Multiplied into the exponent's fused multiply-add instead, the largest
    // score's own exponent was what rounding had left of the maximum: beyond 2^31 its weight was infinite or zero.)
    const float scale2 = 0.08838834764831845f * 1.4426950408889634f;
    // Q as B operand: lane (row lm, dh 32*g + 8*s + e), hi and lo.  The rows are requested here and split where they are
    // first needed, behind the requests for the first block.
    Frag qh[QT][4], ql[QT][4], qm[TERMS == 3 ? QT : 1][4];
    float4 qx[QT][4][2];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        int j = qt * 16 + lm;
        if (j >= Wr) j = Wr - 1;
        const float* qr = a.q + (size_t)(rbase + row0 + j) * a.ldq + h * 128 + 32 * g;
#pragma unroll
        for (int s = 0; s < 4; ++s) { qx[qt][s][0] = *(const float4*)(qr + 8 * s); qx[qt][s][1] = *(const float4*)(qr + 8 * s + 4); }
    }
    auto split_q = [&]() {
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const float4 x0 = qx[qt][s][0], x1 = qx[qt][s][1];
                const float v[8] = {x0.x * scale2, x0.y * scale2, x0.z * scale2, x0.w * scale2, x1.x * scale2, x1.y * scale2, x1.z * scale2, x1.w * scale2};
                if constexpr (TERMS == 3) split8(v, qh[qt][s], ql[qt][s], qm[qt][s]);
                else split8(v, qh[qt][s], ql[qt][s]);
            }
    };

    f32x4_t acc[QT][8];
    float mrun[QT], lrun[QT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        mrun[qt] = NEG_BIG; lrun[qt] = 0.f;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) acc[qt][dt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    }
    // one 32-key block: K tiles and V^T tiles of block `blk` into registers
    struct KV { Frag kf[NPL][2][4], vf[NPL][8]; };
    auto load = [&](KV& r, int blk_want) {
        const int blk = blk_want < NB ? blk_want : NB - 1;       // past the end (two query tiles): a valid block, never used
        Frag (&kf)[NPL][2][4] = r.kf; Frag (&vf)[NPL][8] = r.vf;
        // K tiles (A operand): tile t row r=lm <-> key 32*blk + 8*(lm/4) + 4*t + lm%4 ; dh 32*g + 8*s..
        // (the cache stores each block as these eight fragments, one contiguous kilobyte each; the loads are
        // non-temporal: K and V are read once per step, and letting them allocate in L2 cost 40% at batch 8)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const u32x4_t* kp = (const u32x4_t*)(kbase + (size_t)blk * 4096) + lane;
#pragma unroll
            for (int s = 0; s < 4; ++s) kf[0][t][s].u = __builtin_nontemporal_load(kp + (t * 4 + s) * 64);
            if (KVP == 2) {
                const u32x4_t* kl = (const u32x4_t*)(kbase + plane + (size_t)blk * 4096) + lane;
#pragma unroll
                for (int s = 0; s < 4; ++s) kf[NPL - 1][t][s].u = __builtin_nontemporal_load(kl + (t * 4 + s) * 64);
            } else if (KVP == 3) {      // eight residual bytes per lane and fragment; expanded in compute()
                const u32x2_t* kl = (const u32x2_t*)((const uint8_t*)(kbase + plane) + (size_t)blk * 4096) + lane;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const u32x2_t bw = __builtin_nontemporal_load(kl + (t * 4 + s) * 64);
                    kf[NPL - 1][t][s].u = (u32x4_t){bw[0], bw[1], 0u, 0u};
                }
            }
        }
        // V^T tiles (A operand): row 16*dt + lm, keys kb + 8*g .. +7
        // (stored as eight fragments per block as well)
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
            vf[0][dt].u = __builtin_nontemporal_load((const u32x4_t*)(vbase + (size_t)blk * 4096) + dt * 64 + lane);
            if (KVP == 2) vf[NPL - 1][dt].u = __builtin_nontemporal_load((const u32x4_t*)(vbase + plane + (size_t)blk * 4096) + dt * 64 + lane);
            else if (KVP == 3) {
                const u32x2_t bw = __builtin_nontemporal_load((const u32x2_t*)((const uint8_t*)(vbase + plane) + (size_t)blk * 4096) + dt * 64 + lane);
                vf[NPL - 1][dt].u = (u32x4_t){bw[0], bw[1], 0u, 0u};
            }
        }
    };
    auto compute = [&](KV& r, int blk) {
        const int kb = blk << 5;
        // every row sees all 32 keys: no test (with two query tiles the branch costs registers that are not there)
        const bool whole = QT == 1 && kb + 31 <= n && kb + 31 < T;
        if (KVP == 3) {          // the residual bytes become bf16 lo operands
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int s = 0; s < 4; ++s) { const u32x4_t bw = r.kf[NPL - 1][t][s].u; expand_lo8(r.kf[0][t][s].u, bw[0], bw[1], r.kf[NPL - 1][t][s]); }
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) { const u32x4_t bw = r.vf[NPL - 1][dt].u; expand_lo8(r.vf[0][dt].u, bw[0], bw[1], r.vf[NPL - 1][dt]); }
        }
        const Frag (&kf)[NPL][2][4] = r.kf; const Frag (&vf)[NPL][8] = r.vf;
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            f32x4_t sc[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                sc[t] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[0][t][s].v, qh[qt][s].v, sc[t], 0, 0, 0);
                    sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[0][t][s].v, ql[qt][s].v, sc[t], 0, 0, 0);
                    if constexpr (TERMS == 3) sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[0][t][s].v, qm[qt][s].v, sc[t], 0, 0, 0);
                    if (KVP >= 2)   // lo x lo is below fp32 resolution and is dropped
                        sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[NPL - 1][t][s].v, qh[qt][s].v, sc[t], 0, 0, 0);
                }
            }
            // lane: row j = qt*16 + lm, keys kb + 8*g + e  (e = 4*t + r)
            const int j = qt * 16 + lm;
            const int lastvis = n + (j < Wr ? j : Wr - 1);
            float p[8];
            float bm = NEG_BIG;
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = sc[e >> 2][e & 3];
            if (!whole) {
#pragma unroll
                for (int e = 0; e < 8; ++e) { const int key = kb + 8 * g + e; p[e] = key > lastvis || key >= T ? NEG_BIG : p[e]; }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                bm = fmaxf(bm, p[e]);
            }
            bm = fmaxf(bm, __shfl_xor(bm, 16, 64));
            bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
            // (a block in which a row sees nothing leaves bm at NEG_BIG: every weight is 0)
            const float mnew = fmaxf(mrun[qt], bm);
            const float alpha = __builtin_amdgcn_exp2f(mrun[qt] - mnew);
            float ps = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float w = __builtin_amdgcn_exp2f(p[e] - mnew);
                p[e] = !whole && p[e] == NEG_BIG ? 0.f : w;
                ps += p[e];
            }
            mrun[qt] = mnew;
            lrun[qt] = lrun[qt] * alpha + ps;
            Frag ph, pl, pm;
            if constexpr (TERMS == 3) split8(p, ph, pl, pm);
            else split8(p, ph, pl);
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) {
                acc[qt][dt] *= alpha;
                acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[0][dt].v, ph.v, acc[qt][dt], 0, 0, 0);
                acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[0][dt].v, pl.v, acc[qt][dt], 0, 0, 0);
                if constexpr (TERMS == 3) acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[0][dt].v, pm.v, acc[qt][dt], 0, 0, 0);
                if (KVP >= 2)
                    acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[NPL - 1][dt].v, ph.v, acc[qt][dt], 0, 0, 0);
            }
        }
    };
    // two register sets: the next block of this wave travels while the current one is used.
    int blk = blk0 + wv, left = blk < blk1 ? (blk1 - blk + 3) >> 2 : 0;      // this wave's blocks: blk, blk + 4, ...
    if constexpr (QT == 1) {
        // There are registers to spare: all loads of the next block stay ahead of the current block's arithmetic.  The loop
        // has one exit and the last one or two blocks follow it: with an exit after each block the paths met again at the
        // loop's head, where a register set may or may not have had loads pending, and the compiler waited there for everything
        // in flight before it requested the next block (7B heads: 1500 keys as hi + lo pairs 18.9 -> 14.0 us, 272 keys
        // 10.6 -> 8.4 us; one plane, 2064 keys 12.0 -> 10.8 us).
        if (left > 0) {
            KV ra, rb;
            load(ra, blk);
            __builtin_amdgcn_sched_barrier(0);
            split_q();
            for (; left > 2; left -= 2, blk += 8) {
                load(rb, blk + 4);
                __builtin_amdgcn_sched_barrier(0);
                compute(ra, blk);
                load(ra, blk + 8);
                __builtin_amdgcn_sched_barrier(0);
                compute(rb, blk + 4);
            }
            if (left == 2) {
                load(rb, blk + 4);
                __builtin_amdgcn_sched_barrier(0);
                compute(ra, blk);
                compute(rb, blk + 4);
            } else
                compute(ra, blk);
        }
    } else {
        // two query tiles: the compiler is left to reuse each register as soon as it is free (two workgroups share a CU
        // instead; the form above spills)
        split_q();
        KV ra, rb;
        if (left > 0) {
            load(ra, blk);
            for (;;) {
                load(rb, blk + 4);
                compute(ra, blk);
                blk += 4;
                if (blk >= blk1) break;
                load(ra, blk + 4);
                compute(rb, blk);
                blk += 4;
                if (blk >= blk1) break;
            }
        }
    }
    // row sums over the 4 lanes of a row
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        lrun[qt] += __shfl_xor(lrun[qt], 16, 64);
        lrun[qt] += __shfl_xor(lrun[qt], 32, 64);
    }

    // ---- merge the 4 waves: everyone publishes to LDS, then wave w finishes output tiles 2w and 2w+1
    // (16 head elements each) over the four partials, in wave order
    {
        float* dst = lds + (size_t)wv * QT * PART_FLOATS;
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) *(f32x4_t*)(dst + qt * PART_FLOATS + (dt * 64 + lane) * 4) = acc[qt][dt];
            dst[qt * PART_FLOATS + 2048 + lane] = mrun[qt];
            dst[qt * PART_FLOATS + 2112 + lane] = lrun[qt];
        }
    }
    __syncthreads();
    f32x4_t o2[QT][2];
    float mw[QT], lw[QT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        float mv[4], m = NEG_BIG;
#pragma unroll
        for (int v = 0; v < 4; ++v) { mv[v] = lds[(size_t)(v * QT + qt) * PART_FLOATS + 2048 + lane]; m = fmaxf(m, mv[v]); }
        float l = 0.f;
        o2[qt][0] = o2[qt][1] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float* src = lds + (size_t)(v * QT + qt) * PART_FLOATS;
            const float wgt = __builtin_amdgcn_exp2f(mv[v] - m);
            l += src[2112 + lane] * wgt;
#pragma unroll
            for (int t = 0; t < 2; ++t) o2[qt][t] += *(const f32x4_t*)(src + ((2 * wv + t) * 64 + lane) * 4) * wgt;
        }
        mw[qt] = m; lw[qt] = l;
    }

    if (nsp > 1) {
        // ---- key splits: partial tiles go to memory with agent-scope stores; the last workgroup to
        // arrive reads all of them back -- every load of the merge is in flight at once (each wave its
        // two tiles of every split), splits folded in index order
        float* mine = a.part + (size_t)slot * QT * PART_FLOATS;
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                float* dst = mine + qt * PART_FLOATS + (2 * wv + t) * 256 + lane * 2;
                st_agent_f32x2(dst, o2[qt][t][0], o2[qt][t][1]);
                st_agent_f32x2(dst + 128, o2[qt][t][2], o2[qt][t][3]);
            }
            if (wv == 0) {
                st_agent_f32(mine + qt * PART_FLOATS + 2048 + lane, mw[qt]);
                st_agent_f32(mine + qt * PART_FLOATS + 2112 + lane, lw[qt]);
            }
        }
        wait_vmem_done();
        __syncthreads();                                   // all four waves' stores have completed
        int* flag = (int*)(lds + 4 * QT * PART_FLOATS);
        if (tid == 0) *flag = arrive_agent(a.cnt + bh);
        __syncthreads();
        if (*flag != nsp - 1) return;
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            float m = NEG_BIG, l = 0.f;
            o2[qt][0] = o2[qt][1] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
            for (int s0 = 0; s0 < nsp; s0 += 8) {          // eight splits' loads in flight at a time
                float ms[8], ls[8];
                f32x4_t os[8][2];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int s2 = s0 + u < nsp ? s0 + u : nsp - 1;
                    const float* src = a.part + (size_t)(slot - sp + s2) * QT * PART_FLOATS + qt * PART_FLOATS;
                    ms[u] = ld_agent_f32(src + 2048 + lane);
                    ls[u] = ld_agent_f32(src + 2112 + lane);
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const float* p4 = src + (2 * wv + t) * 256 + lane * 2;
                        float v0, v1, v2, v3;
                        ld_agent_f32x2(p4, v0, v1);
                        ld_agent_f32x2(p4 + 128, v2, v3);
                        os[u][t] = (f32x4_t){v0, v1, v2, v3};
                    }
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const bool valid = s0 + u < nsp;
                    const float mu = valid ? ms[u] : NEG_BIG;
                    const float mnew = fmaxf(m, mu);
                    const float wa = __builtin_amdgcn_exp2f(m - mnew), wb = valid ? __builtin_amdgcn_exp2f(mu - mnew) : 0.f;
                    l = l * wa + ls[u] * wb;
                    o2[qt][0] = o2[qt][0] * wa + os[u][0] * wb;
                    o2[qt][1] = o2[qt][1] * wa + os[u][1] * wb;
                    m = mnew;
                }
            }
            lw[qt] = l;
        }
        if (tid == 0) st_agent_i32(a.cnt + bh, 0);
    }
    // out[row][h*128 + 16*dt + 4*g + r] = O / l, this wave's tiles dt = 2*wv, 2*wv + 1
    float nans[QT];                                          // 0, or NaN where something of the row is not finite
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        const int j = qt * 16 + lm;
        nans[qt] = 0.f;
        if (j < Wr) {
            const float inv = 1.0f / lw[qt];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                o2[qt][t] *= inv;
                if constexpr (KVP == 1) nans[qt] += o2[qt][t][0] * 0.f + o2[qt][t][1] * 0.f + o2[qt][t][2] * 0.f + o2[qt][t][3] * 0.f;
            }
            const int row = rbase + row0 + j;
            if (a.out) {
                float* o = a.out + (size_t)row * a.ldo + h * 128 + 4 * g;
#pragma unroll
                for (int t = 0; t < 2; ++t) *(f32x4_t*)(o + 16 * (2 * wv + t)) = o2[qt][t];
            }
            if (a.ofrag) {
                // head elements 32 * wv + 16 * t + 4 * g + r: k-tile 4 * h + wv, octet 2 * t + g / 2, elements 4 * (g % 2) + r
                const size_t KTo = (size_t)a.H * 4;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const f32x4_t v = o2[qt][t];
                    uint32_t h0, l0, h1, l1;
                    pk_bf16_hilo(v[0], v[1], h0, l0);
                    pk_bf16_hilo(v[2], v[3], h1, l1);
                    char* dst = (char*)a.ofrag + ((((size_t)(row >> 4) * KTo + 4 * h + wv) * 2) * 64 + (row & 15) + 16 * (2 * t + (g >> 1))) * 16 + 8 * (g & 1);
                    *(uint2*)dst = make_uint2(h0, h1);
                    *(uint2*)(dst + 1024) = make_uint2(l0, l1);
                }
            }
        }
    }
    if constexpr (KVP == 1) {
        // A row with a NaN in it is computed once more, key by key in fp32 and over the keys it sees only.  The matrix
        // instructions multiply what a row does not see by a weight of zero (positions past the window, which nobody has
        // to fill, and later window rows), and zero times an infinity or NaN in V is NaN; so is a query or a product of
        // its parts past the range of bf16.  A row whose own keys make it NaN (or infinite) stays so.  Each wave redoes
        // the 32 head elements it has stored; the test runs behind the stores, where it costs 0.0-0.1 us with one
        // query tile and 0.1-0.2 us with two (in front of them 0.1 and 0.4).
        uint32_t rows = 0;
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            const unsigned long long lanes = __ballot(nans[qt] != 0.f);
            rows |= ((uint32_t)(lanes | lanes >> 16 | lanes >> 32 | lanes >> 48) & 0xFFFFu) << (16 * qt);
        }
        if (__builtin_expect(rows == 0, 1)) return;
        wait_vmem_done();                                    // the stores above come first
        const int e = lane & 31;                             // lane = (parity of the key, head element)
        while (rows) {
            const int j = __builtin_ctz(rows), row = rbase + row0 + j;
            rows &= rows - 1;
            int last = n + j;
            if (last >= T) last = T - 1;
            const float* qr = a.q + (size_t)row * a.ldq + h * 128;
            auto score = [&](int t) {
#pragma clang fp contract(off)
                // (uncontracted: the caller's difference to the maximum then takes the product as it was rounded there)
                float s = 0.f;
#pragma unroll 1
                for (int i = 0; i < 128; i += 8) {
                    const u32x4_t kw = *(const u32x4_t*)(kbase + k_index(t, i, 128));
#pragma unroll
                    for (int u = 0; u < 4; ++u) { s += qr[i + 2 * u] * __uint_as_float(kw[u] << 16); s += qr[i + 2 * u + 1] * __uint_as_float(kw[u] & 0xFFFF0000u); }
                }
                return s * 0.08838834764831845f;
            };
            float mx = -3.0e38f;
            for (int t = lane; t <= last; t += 64) mx = fmaxf(mx, score(t));
            for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
            float den = 0.f, sum = 0.f;
            for (int t0 = 0; t0 <= last; t0 += 64) {
                const float p = t0 + lane <= last ? expf(score(t0 + lane) - mx) : 0.f;       // lane = key
                den += p;
#pragma unroll 1
                for (int u = lane >> 5; u < 64; u += 2) {
                    const float pu = __shfl(p, u, 64);
                    if (t0 + u <= last) sum += pu * __uint_as_float((uint32_t)vbase[v_index(32 * wv + e, t0 + u, 128)] << 16);
                }
            }
            for (int o = 32; o > 0; o >>= 1) den += __shfl_xor(den, o, 64);
            sum += __shfl_xor(sum, 32, 64);
            sum /= den;
            if (a.out && lane < 32) a.out[(size_t)row * a.ldo + h * 128 + 32 * wv + e] = sum;
            if (a.ofrag && lane < 32) {
                uint32_t hi, lo;
                pk_bf16_hilo(sum, 0.f, hi, lo);
                bf16_t* dst = a.ofrag + ((((size_t)(row >> 4) * a.H * 4 + 4 * h + wv) * 2) * 64 + (row & 15) + 16 * (e >> 3)) * 8 + (e & 7);
                dst[0] = (bf16_t)hi;
                dst[512] = (bf16_t)lo;
            }
        }
    }
}

size_t fc_attn16_part_bytes(int BH, int nsplit, int W) {      // covers both unit sizes
    const int tiles = W > 16 ? 2 * ((W + 31) / 32) : 1;
    return (size_t)BH * tiles * nsplit * PART_FLOATS * 4;
}

// More units than CUs, and one key split each: the CUs that take a unit more than the others decide when the launch ends.  The
// units past the last full round of the CUs are therefore cut into three to eight key splits, as many as still give every
// CU at most one, and start first, so that their merges are over long before the whole units.  A launch, whole -> cut, pairs of hi
// and lo planes: 13B heads, 8 sequences x 16 rows, 1024 positions 71.6 -> 63.0 us, 300 30.4 -> 28.2; 7 sequences, 2000 116.6 -> 94.9;
// 64 heads on 8, 5 x 16 rows, 2000 69.3 -> 54.2; two query tiles (8 x 32 rows), 1024 73.5 -> 70.7.  Not for two splits (12 x 32 heads 74.7
// both ways) nor for more pieces than CUs (40 heads x 10 tiles, 144 units in seven 24.9 -> 37.2), nor for short contexts (100
// positions 11.6 -> 13.5 with one tile, 300 33.3 -> 35.4 with two): by the longest one as the host knows it, and for each unit
// by its own length.  Returns the number of units cut and their *splits.
int fc_attn16_rest(int W, int subrows, int units, int nsplit, int kvp, int ctx, int* splits) {
    const int cus = fc_num_cus(), r = units % cus, two = W > 16 && subrows != 16;
    *splits = 1;
    if (nsplit != 1 || units < cus || r == 0 || cus / r < 3 || (ctx + 31) / 32 * (kvp == 1 ? 1 : 2) < REST_BLOCKS(two)) return 0;
    *splits = cus / r < 8 ? cus / r : 8;
    return r;
}

hipError_t fc_attn16(const AttnArgs& a0, int Bact, int nsplit, hipStream_t st) {
    AttnArgs a = a0;
    const int QT = a.W > 16 && a.subrows != 16 ? 2 : 1, nsub = (a.W + 16 * QT - 1) / (16 * QT);
    if (a.W < 1 || nsplit < 1 || nsplit > FC_MAX_ATTN_SPLITS || Bact * nsub * a.H > FC_MAX_COUNTERS || a.S < 32 || a.S % 32 || a.bpw < 1)
        return hipErrorInvalidValue;
    const int units = Bact * nsub * a.H;
    dim3 grid(units, nsplit);
    a.rest = fc_attn16_rest(a.W, a.subrows, units, nsplit, a.kvp, a.ctx, &a.rest_splits);
    if (a.rest) { a.whole = units - a.rest; grid = dim3(a.whole + a.rest * a.rest_splits); }
    const size_t l1 = (size_t)4 * PART_FLOATS * 4 + 16, l2 = (size_t)8 * PART_FLOATS * 4 + 16;
    static bool lds_ok = false;                          // two query tiles need more than the default 64 KB
    if (!lds_ok) {
        hipError_t e = hipFuncSetAttribute((const void*)k_attn16<2, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)l2);
        if (e == hipSuccess) e = hipFuncSetAttribute((const void*)k_attn16<2, 1>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)l2);
        if (e == hipSuccess) e = hipFuncSetAttribute((const void*)k_attn16<2, 3>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)l2);
        if (e != hipSuccess) return e;
        lds_ok = true;
    }
    if (a.kvp == 2) {
        if (QT == 2) k_attn16<2, 2><<<grid, 256, l2, st>>>(a);
        else k_attn16<1, 2><<<grid, 256, l1, st>>>(a);
    } else if (a.kvp == 1 && a.terms == 3) {
        if (QT == 2) return hipErrorInvalidValue;        // (three parts of two query tiles do not fit the registers)
        k_attn16<1, 1, 3><<<grid, 256, l1, st>>>(a);
    } else if (a.kvp == 1) {
        if (QT == 2) k_attn16<2, 1><<<grid, 256, l2, st>>>(a);
        else k_attn16<1, 1><<<grid, 256, l1, st>>>(a);
    } else if (a.kvp == 3) {
        if (QT == 2) k_attn16<2, 3><<<grid, 256, l2, st>>>(a);
        else k_attn16<1, 3><<<grid, 256, l1, st>>>(a);
    } else return hipErrorInvalidValue;
    return hipGetLastError();
}
