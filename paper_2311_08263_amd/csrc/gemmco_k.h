// Column-owner weight-streaming bf16 GEMM for up to 32 activation rows (MT = 1 or 2 row tiles of 16).
//
// A workgroup of 8 waves owns NW n-tiles (16 output columns each) over the whole of K; wave w
// takes the w-th eighth of K.  No workgroup ever needs another workgroup's result: the eight
// partial tiles meet in LDS, then waves 0..NW-1 each finish one tile and run the fused epilogue.
// For the residual GEMMs with long K and few columns (down, O) the workgroups of a launch can also be
// grouped ks to an owner, each taking 1/ks of K and so reading only 1/ks of the activations (at the 7B
// shape the down projection reads 704 KB of activations per workgroup against 352 KB of weights); the ks
// partial tiles (1 KB each) meet through memory and the last workgroup to arrive adds them in slice order.
// Compared with slicing K across workgroups everywhere this trades the global hand-off (partial tiles through
// memory, an atomic counter, a second pass by the last arriver) for more activation reads out of
// L2: every workgroup reads all 16 x K activations, straight into registers in MFMA B-fragment
// order (lane = row % 16 + 16 * k-octet: two 16-byte loads per k-tile), converts them to a bf16
// hi + lo pair and reuses each fragment for its NW weight tiles.  Weights stream HBM -> VGPR once,
// in MFMA fragment order, a pair of k-tiles x NW n-tiles at a time; from the coded copy (wcode.h) where the matrix has one: 13/16
// of the bytes for 21 vector instructions a tile, which the memory-bound loop has room for (13, without the code for zeros, leave a step
// 1-2 % shorter; leaving those 13 out as well gained 1 us of 31).
//
// What bounds a launch (7B gate/up, 16 rows, 146 MB coded, 29.1 us; from the plain tiles, 180 MB, 33.6): the bytes a CU is sent, weights
// and activations alike (six n-tiles of 64 pairs and 256 KB of activations on the fullest CUs; without activations 27.2 us), then
// 4-5 us of head, first round trip, and tail.  Activations through a ring in LDS, asked for in front of the first weights, cost what they saved:
// 256 KB a CU take 2.5 us to arrive there and 3.3 among the weights (gate/up 30.6-31.1 us against 29.1, QKV 22.4 against 21.3).
// 7B / 13B / 70B shape, 16 rows, plain tiles with a plan tuned per shape -> coded, steps of 8 / 6 / 2 layers: 871 / 912 / 704 -> 805 / 835 / 636 us
// (before the code for zeros; with it, and one round of up to 14 n-tiles a workgroup, the 70B shape's step takes 622).
#pragma once
#include "gemmco.h"
#include "wcode.h"
#include "xwg.h"
#include <type_traits>

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
union Frag { u32x4_t u; bf16x8_t v; };

__device__ inline uint32_t rne16(float f) {
    uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ inline float up16(uint32_t b) { return __uint_as_float(b << 16); }

constexpr bool co_gained(int epi) { return epi != EPI_RESID && epi != EPI_LMHEAD_BARE; }       // a norm in front
// A pair of k-tiles of a wave: its weights for the wave's n-tiles, its activation octets.
template <typename WP, int NW, int MT> struct Pair { float4 x[2][MT][2]; WP w[NW]; };

// NW * MT <= 16 output tiles per workgroup: after the K slices of the eight waves have met in LDS, wave
// w finishes tiles ti = w and w + 8, tile ti = j * MT + mt (n-tile j of the workgroup, row tile mt).
// D = pairs of k-tiles a wave has under way or in use.
template <typename WP, int EPI, int NW, int D, int MT>
__global__ __launch_bounds__(512) void k_gemmco(GemmCoArgs a) {
    extern __shared__ char lds[];
    constexpr int TW = NW * MT;                          // output tiles per workgroup
    // up to 8 output tiles: all eight waves publish at once (one barrier); more: in two rounds of four sets
    constexpr int SETS = TW <= 8 ? 8 : 4;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, g4 = lane >> 4;
    // LDS: partial tiles [SETS][TW][64 lanes], then
    float* lds_ss = (float*)(lds + SETS * TW * 1024);   // [8][MT * 16]
    float* lds_amv = lds_ss + 8 * MT * 16;              // [8][16]
    int* lds_ami = (int*)(lds_amv + 8 * 16);            // [8][16]
    float* lds_gain = (float*)(lds_ami + 8 * 16) + w * a.gain_wave;      // this wave's part of the gain [pairs][64]
    auto part_of = [&](int wave) { return (f32x4_t*)lds + (SETS == 8 ? wave : wave & 3) * (TW * 64); };
    // workgroup i owns n-tiles [i*NT/G, (i+1)*NT/G): at most NW of them
    const int ks = (EPI != EPI_LMHEAD && EPI != EPI_LMHEAD_BARE && a.ks > 1) ? a.ks : 1;
    const int G = gridDim.x / ks, owner = blockIdx.x / ks, slice = blockIdx.x % ks;
    const int nt0 = (int)(((unsigned)owner * (unsigned)a.NT) / (unsigned)G);
    const int nt1 = (int)(((unsigned)(owner + 1) * (unsigned)a.NT) / (unsigned)G);
    // this workgroup's K slice in pairs of k-tiles, cut in eight for the waves (ragged cuts allowed)
    const int PT = a.K >> 6;
    const int s_lo = (int)((unsigned)PT * (unsigned)slice / (unsigned)ks), s_len = (int)((unsigned)PT * (unsigned)(slice + 1) / (unsigned)ks) - s_lo;
    const int p_begin = s_lo + ((w * s_len) >> 3), n = ((s_lo + (((w + 1) * s_len) >> 3))) - p_begin;
    // With a.rotate every wave walks its pairs in a rotated order that differs from wave to wave and
    // workgroup to workgroup (fc_gemmco).
    const int rot = (a.rotate && n > 0) ? (int)(((unsigned)blockIdx.x * 7u + (unsigned)w * 3u) % (unsigned)n) : 0;
    auto pair_no = [&](int i) { const int r = i + rot; return p_begin + (r >= n ? r - n : r); };      // i < n
    uint32_t xoff[MT];                                  // byte offsets of this lane's rows and octet; rows past M repeat a valid row, never written
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) xoff[mt] = ((uint32_t)(mt * 16 + lm < a.M ? mt * 16 + lm : a.M - 1) * (uint32_t)a.ldx + 8 * g4) * 4;

    // A coded copy: the columns' bases, and which pairs of this wave's part of K hold weights that the copy does not; asked for
    // in front of everything else.  Pair p's bit is p - p_begin mod 64.
    constexpr bool CODED = std::is_same<WP, WCoded>::value;
    const int nt_last = nt1 > nt0 ? nt1 - 1 : (nt0 < a.NT ? nt0 : a.NT - 1);       // (tiles this workgroup does not own: its last one again)
    auto tile_no = [&](int j) { return nt0 + j < nt_last ? nt0 + j : nt_last; };
    uint32_t base4[NW], flag[NW];
    const uint8_t* flags = (const uint8_t*)a.C + wc_flag_off(a.K, a.NT);
    u32x2_t mark;                                        // lane 0: stamp, lane 1: record (a vector load, in the row of the flags: scalar ones cost 0.15 us a launch)
    if constexpr (CODED) {
        mark = *(const u32x2_t*)((lane & 1 ? a.record : a.stamp));
        const uint8_t* bases = (const uint8_t*)a.C + wc_base_off(a.K, a.NT);
        const int p = p_begin + lane < PT ? p_begin + lane : PT - 1;
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            base4[j] = bases[tile_no(j) * 16 + lm];
            flag[j] = flags[(size_t)tile_no(j) * PT + p];
        }
    }

    // All loads are unconditional (a conditionally loaded register batch would be copied, and a copy
    // waits for every load in flight): past the end of the slice, or for n-tiles this workgroup does not own, the address
    // stays at the last tile or pair of its own, which has just been requested.  (With one fixed tile of the matrix there, every
    // workgroup of fewer tiles than the widest one asked the same L2 channels for the same kilobyte.)
    // Loads return in order, so the activations of a pair are requested before its weights.
    auto load = [&](auto& b, int i) {
        const int p = n > 0 ? pair_no(i < n ? i : n - 1) : (p_begin < PT ? p_begin : PT - 1);
        const float* base = a.X + p * 64;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) b.x[u][mt][hf] = *(const float4*)((const char*)base + (xoff[mt] + u * 128 + hf * 16));
#pragma unroll
        for (int j = 0; j < NW; ++j) wc_load(b.w[j], (const char*)a.W, a.C, (size_t)tile_no(j) * PT + p, lane);
    };

    f32x4_t acc[NW][MT];
    float ss[MT];
    constexpr bool GAINED = co_gained(EPI), LMHEAD = EPI == EPI_LMHEAD || EPI == EPI_LMHEAD_BARE;       // (gain: from LDS)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        ss[mt] = 0.f;
#pragma unroll
        for (int j = 0; j < NW; ++j) acc[j][mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    }

    // one k-tile (tile t of pair p): activations -> bf16 hi + lo fragments (row statistics on the way), then NW x MT x 2 MFMAs
    auto ktile = [&](const auto& wk, int t, const float4 (&x)[MT][2], int p) {
        float4 g0, g1;
        if (GAINED) { const float* gp = lds_gain + (p - p_begin) * 64 + t * 32 + 8 * g4; g0 = *(const float4*)gp; g1 = *(const float4*)(gp + 4); }
        Frag hi[MT], lo[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            float v[8] = {x[mt][0].x, x[mt][0].y, x[mt][0].z, x[mt][0].w, x[mt][1].x, x[mt][1].y, x[mt][1].z, x[mt][1].w};
            if (GAINED) {
#pragma unroll
                for (int e = 0; e < 8; ++e) ss[mt] += v[e] * v[e];
                v[0] *= g0.x; v[1] *= g0.y; v[2] *= g0.z; v[3] *= g0.w; v[4] *= g1.x; v[5] *= g1.y; v[6] *= g1.z; v[7] *= g1.w;
            }
            uint32_t h[4], l[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) pk_bf16_hilo(v[2 * e], v[2 * e + 1], h[e], l[e]);
            hi[mt].u = (u32x4_t){h[0], h[1], h[2], h[3]};
            lo[mt].u = a.hi_only ? (u32x4_t){0u, 0u, 0u, 0u} : (u32x4_t){l[0], l[1], l[2], l[3]};
        }
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            Frag wf; wf.u = wc_tile(wk[j], t, base4[j]);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                acc[j][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf.v, hi[mt].v, acc[j][mt], 0, 0, 0);
                acc[j][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf.v, lo[mt].v, acc[j][mt], 0, 0, 0);
            }
        }
    };
    auto compute = [&](const auto& b, int p) {
        ktile(b.w, 0, b.x[0], p);
        if (NW * MT >= 12) __builtin_amdgcn_sched_barrier(0);           // (registers for one tile's fragments)
        ktile(b.w, 1, b.x[1], p);
    };
    uint64_t flagged = 0;
    // The walk over the wave's pairs with DD of them in registers; the first DD are there.  Branches are on scalar conditions alone (a matrix
    // instruction runs whatever the lane mask says); the scheduling barriers keep the loads behind the arithmetic they follow.
    auto walk = [&](auto ddc, auto& b, auto skip_flagged) {
        constexpr int DD = decltype(ddc)::value;
        auto use = [&](const auto& bd, int i) {
            const int p = pair_no(i);
            if (!(decltype(skip_flagged)::value && ((flagged >> ((p - p_begin) & 63)) & 1))) compute(bd, p);
            __builtin_amdgcn_sched_barrier(0);
        };
        int i = 0;
        for (; i + 2 * DD <= n; i += DD) {
#pragma unroll
            for (int d = 0; d < DD; ++d) {
                use(b[d], i + d);
                load(b[d], i + d + DD);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // fewer than 2 DD are left: refill what is still needed (all of the slots but the last, or none)
        const bool more = i + DD < n;
#pragma unroll
        for (int d = 0; d < DD; ++d) {
            if (i + d < n) use(b[d], i + d);
            if (d + 1 < DD && more) load(b[d], i + d + DD);
        }
#pragma unroll
        for (int d = 0; d + 1 < DD; ++d)
            if (i + DD + d < n) use(b[d], i + DD + d);
    };

    // What the epilogue will need from memory is requested now, a whole K loop ahead of its use: the rotary
    // factors of this wave's output tiles (behind a dependent load of the sequence length) and the residual
    // tile that the result is added to.
    constexpr int NF = (TW + 7) / 8;
    float rcos[NF][4], rsin[NF][4];
    f32x4_t xold[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int ti = w + 8 * f, nt = nt0 + ti / MT, m = (w % MT) * 16 + lm;
        const bool mine = ti < TW && nt < nt1 && m < a.M;
        xold[f] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) { rcos[f][e] = 1.0f; rsin[f][e] = 0.0f; }
        if (EPI == EPI_RESID) {
            if (mine) xold[f] = *(const f32x4_t*)(a.out + (size_t)m * a.ldo + nt * 16 + 4 * g4);
        } else if (EPI == EPI_QKV) {
            const int hh = nt >> 3, t = nt & 7;
            if (mine && hh < a.H + a.Hkv) {
                const int pos = a.rm.rowb ? a.n_state[a.rm.rowb[m]] + a.rm.rowj[m] : a.n_state[m / a.Wn] + m % a.Wn;
                if (pos < a.S) {
                    const f32x4_t c4 = *(const f32x4_t*)(a.cosT + (size_t)pos * 64 + 8 * t + 4 * (g4 & 1));
                    const f32x4_t s4 = *(const f32x4_t*)(a.sinT + (size_t)pos * 64 + 8 * t + 4 * (g4 & 1));
#pragma unroll
                    for (int e = 0; e < 4; ++e) { rcos[f][e] = c4[e]; rsin[f][e] = s4[e]; }
                }
            }
        }
    }

    // The gain of this wave's part of K goes through its part of LDS.  It is requested before the
    // weights: its store to LDS would otherwise wait for every weight load in front of it.
    f32x4_t gr[4];
    auto gain_at = [&](int q) { const int k = p_begin * 64 + q * 256 + lane * 4; return *(const f32x4_t*)(a.gain + (k < a.K ? k : 0)); };
    if (GAINED) {
#pragma unroll
        for (int q = 0; q < 4; ++q) gr[q] = gain_at(q);
    }
    Pair<WP, NW, MT> b[D];
#pragma unroll
    for (int d = 0; d < D; ++d) load(b[d], d);
    if (GAINED) {
        auto mine = [&](int q) { return q * 256 + lane * 4 < n * 64; };
#pragma unroll
        for (int q = 0; q < 4; ++q) if (mine(q)) *(f32x4_t*)(lds_gain + q * 256 + lane * 4) = gr[q];
        for (int q = 4; 4 * q < n; ++q) if (mine(q)) *(f32x4_t*)(lds_gain + q * 256 + lane * 4) = gain_at(q);
    }
    if constexpr (CODED) {
        uint32_t any = 0;
#pragma unroll
        for (int j = 0; j < NW; ++j) { base4[j] *= 0x01010101u; any |= lane < n ? flag[j] : 0; }
        if (n > 64)
            for (int j = 0; j < NW; ++j)
                for (int p = p_begin + 64 + lane; p < p_begin + n; p += 64) any |= flags[(size_t)tile_no(j) * PT + p];
        flagged = __ballot(any != 0);
        // Flagged pairs are left out of the walk over the copy and taken from the plain tiles behind it, one after the other;
        // where a wave has more than two of them, or the copy is not of these weights, it walks the plain tiles instead.
        const uint32_t stale = (__builtin_amdgcn_readlane(mark[0], 0) ^ __builtin_amdgcn_readlane(mark[0], 1)) | (__builtin_amdgcn_readlane(mark[1], 0) ^ __builtin_amdgcn_readlane(mark[1], 1));
        if (__builtin_expect(stale || __popcll(flagged) > 2, 0)) {
            constexpr int DP = NW * MT * D <= 12 ? D : 1;
            Pair<WPlain, NW, MT> bp[DP];
#pragma unroll
            for (int d = 0; d < DP; ++d) load(bp[d], d);
            walk(std::integral_constant<int, DP>(), bp, std::false_type());
        } else {
            walk(std::integral_constant<int, D>(), b, std::true_type());
            for (uint64_t m = flagged; m; m &= m - 1)
                for (int p = p_begin + __builtin_ctzll(m); p < p_begin + n; p += 64) {
                    Pair<WPlain, NW, MT> bp;
                    const int r = p - p_begin - rot;
                    load(bp, r < 0 ? r + n : r);
                    compute(bp, p);
                }
        }
    } else walk(std::integral_constant<int, D>(), b, std::false_type());

    // the eight K slices meet in LDS: with up to eight output tiles every wave publishes its partial tiles and one
    // barrier later each tile's finisher adds the eight in wave order; with more tiles in two rounds, so that
    // four partial sets (4 x TW KB) are enough: waves 4..7 publish, waves 0..3 add those to their own and
    // publish the sums
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        ss[mt] += __shfl_xor(ss[mt], 16, 64);
        ss[mt] += __shfl_xor(ss[mt], 32, 64);
        if (g4 == 0) lds_ss[(w * MT + mt) * 16 + lm] = ss[mt];
    }
    if constexpr (SETS == 8) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int j = 0; j < NW; ++j) part_of(w)[(j * MT + mt) * 64 + lane] = acc[j][mt];
        __syncthreads();
    } else {
    if (w >= 4) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int j = 0; j < NW; ++j) part_of(w)[(j * MT + mt) * 64 + lane] = acc[j][mt];
    }
    __syncthreads();
    if (w < 4) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int j = 0; j < NW; ++j) acc[j][mt] += part_of(w)[(j * MT + mt) * 64 + lane];
    }
    __syncthreads();
    if (w < 4) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int j = 0; j < NW; ++j) part_of(w)[(j * MT + mt) * 64 + lane] = acc[j][mt];
    }
    __syncthreads();
    }

    // wave w finishes tiles w and (with more than 8 tiles) w + 8: lane holds row tm*16 + lm, columns
    // nt*16 + 4*g4 + r.  MT divides 8, so both tiles of a wave belong to the same row tile tm.
    const int tm = w % MT;
    const int m = tm * 16 + lm;
    int ntf[NF];
    bool fin[NF];
    f32x4_t v[NF];
    float rs = 1.0f, ssrow = 0.f;
    if (GAINED) {
#pragma unroll
        for (int q = 0; q < 8; ++q) ssrow += lds_ss[(q * MT + tm) * 16 + lm];
        rs = 1.0f / sqrtf(ssrow / (float)a.K + a.eps);
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int ti = w + 8 * f;
        ntf[f] = nt0 + ti / MT;
        fin[f] = ti < TW && ntf[f] < nt1;
        v[f] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
        if (fin[f]) {
#pragma unroll
            for (int q = 0; q < SETS; ++q) v[f] += part_of(q)[ti * 64 + lane];
            if (ks == 1) v[f] *= rs;
        }
    }
    if (!LMHEAD && ks > 1) {
        // partial tiles of the ks slices (and, with a norm in front, each slice's share of the row sums of
        // squares) meet through memory; the last workgroup to arrive adds them in slice order
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            float* mine = a.xpart + ((size_t)blockIdx.x * (8 * NF) + w + 8 * f) * 256 + lane * 2;
            if (fin[f]) {
                st_agent_f32x2(mine, v[f][0], v[f][1]);
                st_agent_f32x2(mine + 128, v[f][2], v[f][3]);
            }
        }
        float* sspart = a.xpart + (size_t)gridDim.x * (8 * NF) * 256;       // [workgroup][MT * 16]
        if (GAINED && w < MT && g4 == 0) st_agent_f32(sspart + (size_t)blockIdx.x * (MT * 16) + tm * 16 + lm, ssrow);
        wait_vmem_done();
        __syncthreads();
        int* flag = (int*)lds_ss;
        if (tid == 0) *flag = arrive_agent(a.xcnt + owner);
        __syncthreads();
        if (*flag != ks - 1) return;
        if (GAINED) {
            float s = 0.f;
#pragma unroll
            for (int s2 = 0; s2 < 8; ++s2) {
                const float p = ld_agent_f32(sspart + (size_t)(owner * ks + (s2 < ks ? s2 : 0)) * (MT * 16) + tm * 16 + lm);
                if (s2 < ks) s += p;
            }
            rs = 1.0f / sqrtf(s / (float)a.K + a.eps);
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (!fin[f]) continue;
            f32x4_t part[8];
#pragma unroll
            for (int s2 = 0; s2 < 8; ++s2) {
                const float* src = a.xpart + ((size_t)(owner * ks + (s2 < ks ? s2 : 0)) * (8 * NF) + w + 8 * f) * 256 + lane * 2;
                float p0, p1, p2, p3;
                ld_agent_f32x2(src, p0, p1);
                ld_agent_f32x2(src + 128, p2, p3);
                part[s2] = (f32x4_t){p0, p1, p2, p3};
            }
            v[f] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s2 = 0; s2 < 8; ++s2) if (s2 < ks) v[f] += part[s2];
            v[f] *= rs;
        }
        if (tid == 0) st_agent_i32(a.xcnt + owner, 0);
    }
    float best = -INFINITY; int bi = 0x7fffffff;          // LM head: the wave's winner per row over its tiles
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int nt = ntf[f];
        const f32x4_t vv = v[f];
        if (!fin[f]) continue;
        if (EPI == EPI_RESID) {
            if (m < a.M) *(f32x4_t*)(a.out + (size_t)m * a.ldo + nt * 16 + 4 * g4) = xold[f] + vv;
        } else if (EPI == EPI_SWIGLU) {
            // columns 0..7 of a tile: gate of features 8*nt..; columns 8..15: their up values (lane ^ 32)
            f32x4_t h;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float other = __shfl_xor(vv[r], 32, 64);
                h[r] = vv[r] / (1.0f + expf(-vv[r])) * other;
            }
            if (g4 < 2 && m < a.M) *(f32x4_t*)(a.out + (size_t)m * a.ldo + nt * 8 + 4 * g4) = h;
        } else if (EPI == EPI_QKV) {
            // q/k heads: tile t of a head holds elements 8t..8t+7 (columns 0..7) and their rotary partners
            // 64+8t.. (columns 8..15, lane ^ 32); v heads are in natural order
            const int hh = nt >> 3, t = nt & 7;
            const int mc = m < a.M ? m : 0;
            const int b = a.rm.rowb ? a.rm.rowb[mc] : m / a.Wn, j = a.rm.rowb ? a.rm.rowj[mc] : m % a.Wn;
            const int pos = m < a.M ? a.n_state[b] + j : a.S;
            const bool ok = m < a.M && pos < a.S;               // capacity guard
            const size_t plane = (size_t)a.S * 128;
            if (hh < a.H + a.Hkv) {
                const int i0 = 8 * t + 4 * (g4 & 1);            // element index within the half
                f32x4_t r;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float other = __shfl_xor(vv[e], 32, 64);
                    const float c = rcos[f][e], s = rsin[f][e];
                    r[e] = g4 < 2 ? vv[e] * c - other * s : vv[e] * c + other * s;
                    if (hh >= a.H) r[e] = kv_round(r[e], a.kvq & 15);
                }
                const int el = (g4 < 2 ? 0 : 64) + i0;          // element index within the head
                if (ok) {
                    if (hh < a.H) *(f32x4_t*)(a.out + (size_t)m * a.ldo + hh * 128 + el) = r;
                    else {
                        bf16_t* kb = a.kc + ((((size_t)a.layer * a.B + b) * a.Hkv + (hh - a.H)) * kv_alloc_planes(a.kvp)) * plane;
                        const size_t ki = k_index(pos, el, 128);
                        bf16_t* kr = kb + ki;
                        uint32_t h[4];
                        if (a.kvp == 3) {
                            uint32_t l[4];
#pragma unroll
                            for (int e = 0; e < 4; ++e) kv24_split(r[e], h[e], l[e]);
                            *(uint2*)kr = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
                            *(uint32_t*)((uint8_t*)(kb + plane) + ki) = l[0] | (l[1] << 8) | (l[2] << 16) | (l[3] << 24);
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e) h[e] = rne16(r[e]);
                            *(uint2*)kr = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
                            if (a.kvp == 2) {
                                uint32_t l[4];
#pragma unroll
                                for (int e = 0; e < 4; ++e) l[e] = rne16(r[e] - up16(h[e]));
                                *(uint2*)(kr + plane) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
                            }
                        }
                    }
                }
            } else if (ok) {
                const int kh = hh - a.H - a.Hkv;
                bf16_t* vb = a.vc + ((((size_t)a.layer * a.B + b) * a.Hkv + kh) * kv_alloc_planes(a.kvp)) * plane;
                const size_t vi = v_index(16 * t + 4 * g4, pos, 128);
                bf16_t* vr = vb + vi;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float vq = kv_round(vv[e], a.kvq >> 4);
                    if (a.kvp == 3) {
                        uint32_t h0, l0; kv24_split(vq, h0, l0);
                        vr[e * 8] = (bf16_t)h0;
                        ((uint8_t*)(vb + plane))[vi + e * 8] = (uint8_t)l0;
                    } else {
                        const uint32_t h0 = rne16(vq);
                        vr[e * 8] = (bf16_t)h0;
                        if (a.kvp == 2) vr[e * 8 + plane] = (bf16_t)rne16(vq - up16(h0));
                    }
                }
            }
        } else if (LMHEAD) {
            const int n0 = nt * 16 + 4 * g4;
            if (a.out && m < a.M) *(f32x4_t*)(a.out + (size_t)m * a.ldo + n0) = vv;
#pragma unroll
            for (int r = 0; r < 4; ++r) if (vv[r] > best || (vv[r] == best && n0 + r < bi)) { best = vv[r]; bi = n0 + r; }
        }
    }
    if (LMHEAD) {
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
            const float ov = __shfl_xor(best, o, 64); const int oi = __shfl_xor(bi, o, 64);
            if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
        }
        if (g4 == 0) { lds_amv[w * 16 + lm] = best; lds_ami[w * 16 + lm] = bi; }
        __syncthreads();
        if (tid < 16 * MT) {                 // row tid: the waves whose tiles are row tile tid / 16
            const int rt = tid >> 4, r16 = tid & 15;
            float bv = -INFINITY; int bx = 0x7fffffff;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (q % MT != rt) continue;
                const float ov = lds_amv[q * 16 + r16]; const int oi = lds_ami[q * 16 + r16];
                if (ov > bv || (ov == bv && oi < bx)) { bv = ov; bx = oi; }
            }
            a.amax_val[(size_t)blockIdx.x * (16 * MT) + tid] = bv;
            a.amax_idx[(size_t)blockIdx.x * (16 * MT) + tid] = bx;
        }
    }
}

// LDS of a launch: the partial tiles (in two rounds of four sets where there are more than eight), row sums and winners, the waves' parts of the gain
static constexpr size_t CO_LDS_MOST = 150 * 1024;
static size_t co_lds_plan(GemmCoArgs& a, int nw, int mt, bool gain) {
    const int ks = a.ks > 1 ? a.ks : 1, PT = a.K >> 6, pairs = ((PT + ks - 1) / ks + 7) / 8;        // most pairs of a wave
    a.gain_wave = gain ? pairs * 64 : 0;
    return (size_t)(nw * mt <= 8 ? 8 : 4) * nw * mt * 1024 + (size_t)(8 * mt * 16 + 2 * 8 * 16) * 4 + (size_t)a.gain_wave * 32 + 64;
}

template <typename WP, int EPI, int NW, int D, int MT>
static hipError_t launch_k(const GemmCoArgs& a0, int G, hipStream_t st) {
    GemmCoArgs a = a0;
    const size_t lds = co_lds_plan(a, NW, MT, co_gained(EPI));
    if (lds > CO_LDS_MOST) return hipErrorInvalidValue;
    static bool raised = false;
    if (!raised) {
        hipError_t e = hipFuncSetAttribute((const void*)k_gemmco<WP, EPI, NW, D, MT>, hipFuncAttributeMaxDynamicSharedMemorySize, CO_LDS_MOST);
        if (e != hipSuccess) return e;
        raised = true;
    }
    k_gemmco<WP, EPI, NW, D, MT><<<G, 512, lds, st>>>(a);
    return hipGetLastError();
}
template <typename WP, int EPI>
static hipError_t launch_epi(const GemmCoArgs& a, int G, hipStream_t st) {
    const int owners = G / (a.ks > 1 ? a.ks : 1);
    const int nw = (a.NT + owners - 1) / owners;  // most n-tiles any workgroup owns
    // Pairs of k-tiles under way per wave: what it takes to keep the CU's loads busy (its eight waves hold at least 40 KB of requests either way)
    // and no more: with up to 16 rows one pair of up to four n-tiles, two of more (steps of eight 7B layers, one / two under way, us: QKV
    // 853 / 860, O 869 / 885, gate/up 817 / 814, LM head 883 / 881; gate/up of eight 2048-wide layers, three n-tiles, 506 / 512).
    const bool one = a.single_buffer == 1 || (a.single_buffer == 2 && a.M <= 16 && nw <= 4);
    if (a.M > 16) {
        if (one) switch (nw) {
            case 1: return launch_k<WP, EPI, 1, 2, 2>(a, G, st);
            case 2: return launch_k<WP, EPI, 2, 2, 2>(a, G, st);
            case 3: return launch_k<WP, EPI, 3, 1, 2>(a, G, st);
            case 4: return launch_k<WP, EPI, 4, 1, 2>(a, G, st);
            case 5: case 6: return launch_k<WP, EPI, 6, 1, 2>(a, G, st);
            case 7: case 8: return launch_k<WP, EPI, 8, 1, 2>(a, G, st);
        } else switch (nw) {
            case 1: return launch_k<WP, EPI, 1, 3, 2>(a, G, st);
            case 2: return launch_k<WP, EPI, 2, 3, 2>(a, G, st);
            case 3: return launch_k<WP, EPI, 3, 2, 2>(a, G, st);
            case 4: return launch_k<WP, EPI, 4, 2, 2>(a, G, st);
            case 5: case 6: return launch_k<WP, EPI, 6, 1, 2>(a, G, st);          // (registers for one)
            case 7: case 8: return launch_k<WP, EPI, 8, 1, 2>(a, G, st);
        }
        return hipErrorInvalidValue;
    }
    if (one) switch (nw) {
        case 1: return launch_k<WP, EPI, 1, 3, 1>(a, G, st);
        case 2: return launch_k<WP, EPI, 2, 2, 1>(a, G, st);
        case 3: return launch_k<WP, EPI, 3, 1, 1>(a, G, st);
        case 4: return launch_k<WP, EPI, 4, 1, 1>(a, G, st);
        case 5: case 6: return launch_k<WP, EPI, 6, 1, 1>(a, G, st);
        case 7: case 8: return launch_k<WP, EPI, 8, 1, 1>(a, G, st);
        case 9: case 10: case 11: case 12: return launch_k<WP, EPI, 12, 1, 1>(a, G, st);
        case 13: case 14: return launch_k<WP, EPI, 14, 1, 1>(a, G, st);
    } else switch (nw) {
        case 1: return launch_k<WP, EPI, 1, 4, 1>(a, G, st);
        case 2: return launch_k<WP, EPI, 2, 3, 1>(a, G, st);
        case 3: return launch_k<WP, EPI, 3, 2, 1>(a, G, st);
        case 4: return launch_k<WP, EPI, 4, 2, 1>(a, G, st);
        case 5: case 6: return launch_k<WP, EPI, 6, 2, 1>(a, G, st);
        case 7: case 8: return launch_k<WP, EPI, 8, 2, 1>(a, G, st);
        case 9: case 10: case 11: case 12: return launch_k<WP, EPI, 12, 1, 1>(a, G, st);
        case 13: case 14: return launch_k<WP, EPI, 14, 1, 1>(a, G, st);
    }
    return hipErrorInvalidValue;
}
template <typename WP>
static hipError_t launch_co(int epi, const GemmCoArgs& a, int G, hipStream_t st) {
    switch (epi) {
        case EPI_RESID: return launch_epi<WP, EPI_RESID>(a, G, st);
        case EPI_SWIGLU: return launch_epi<WP, EPI_SWIGLU>(a, G, st);
        case EPI_QKV: return launch_epi<WP, EPI_QKV>(a, G, st);
        case EPI_LMHEAD: return a.gain ? launch_epi<WP, EPI_LMHEAD>(a, G, st) : launch_epi<WP, EPI_LMHEAD_BARE>(a, G, st);
    }
    return hipErrorInvalidValue;
}
