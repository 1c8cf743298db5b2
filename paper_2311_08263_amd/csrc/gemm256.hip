// bf16 GEMM for steps with many rows (batch x window up to a few hundred): out = act . W with the
// weights in MFMA fragment order and the activations pre-split into bf16 hi + lo fragments.
//
// At 256 rows the step is no longer a pure weight stream: 2 x 256 x params x 2 (hi, lo) flops per step put it on the
// matrix-core side of the ridge.  Tiling: a workgroup of eight waves computes 64 (or 48) rows of a block of column tiles;
// every activation fragment read from LDS feeds a wave's 3 or 4 column tiles and every weight fragment (read straight
// from global memory, four k-tiles ahead) all row tiles.  Activation fragments of 4 k-tiles at a time are copied
// global -> LDS by the whole workgroup, double buffered, one barrier per stage.  The row blocks of a column block re-read
// the same weights: HBM sees them once, the repeats come from L2; workgroup ids are mapped so that they run on the same
// XCD (ids that are equal mod 8 share an XCD and its L2), back to back.
// What bounds the K loop (7B down, 1024 rows, one 64 x 256 tile per CU, 143 us = 1290 TFLOP/s issued; a library product of
// 8192^3 reaches 1135, of 16384^3 1358 on the same card): power and the bytes that move.  The same loop takes 98 us with
// matrix instructions alone, 93 us with LDS reads, 125 us with the weight loads, and on all-zero data 126 us complete and
// 84 us with matrix instructions alone.  Without effect: software-pipelined LDS reads, activations loaded straight into
// LDS, weights two stages further ahead, another order of the k-tiles per wave (the order of the matrix instructions has one:
// MFMA_TILE); slower: 128-row tiles in every form tried
// (weights through LDS, shared by two row halves, 128 accumulator registers per wave), 8 x 2 tiles per wave.
// Matrices with few columns (O and down projections) are also split along K so that the launch fills the chip; the
// slices store partial tiles and k_resid_reduce_split adds them to the residual stream in slice order.
//
// The activations arrive as bf16 hi + lo in B-fragment order [row tile][k-tile][hi|lo][lane][8], written by whoever
// computed them (embedding, residual GEMM, attention, SwiGLU); a norm's row scale is applied in the epilogue.
#include "gemm256.h"
#include "gemmco.h"      // fc_num_cus

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4_t;
union Frag { u32x4_t u; bf16x8_t v; };

__device__ inline uint32_t rne16(float f) {
    uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ inline float up16(uint32_t b) { return __uint_as_float(b << 16); }

// ------------------------------------------------------------------ activation fragments
// grid (row tiles of 16 rows, K chunks); X [M][K] fp32 -> AF [MT][KT][3][64][8] bf16: hi, lo and what the two leave
// over, all 24 bits of the value down to 2^-110 (bf16's denormals end at 2^-133: rows of 1e-34 are as exact as in fp32, of
// 1e-37 to 2.7e-4; normalised rows are of the order of one).
__global__ __launch_bounds__(512) void k_split3(const float* X, int ldx, int M, int K, bf16_t* AF) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int lm = lane & 15, g4 = lane >> 4;
    const int mt = blockIdx.x, KT = K >> 5;
    const int kt_lo = (int)((unsigned)KT * blockIdx.y / gridDim.y), kt_hi = (int)((unsigned)KT * (blockIdx.y + 1) / gridDim.y);
    const int row = mt * 16 + lm < M ? mt * 16 + lm : M - 1;
    const float* xr = X + (size_t)row * ldx + 8 * g4;
    u32x4_t* dst = (u32x4_t*)AF + (size_t)mt * KT * 3 * 64 + lane;
    for (int kt = kt_lo + w; kt < kt_hi; kt += 8) {
        const float4 a = *(const float4*)(xr + kt * 32), b = *(const float4*)(xr + kt * 32 + 4);
        const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        uint32_t h[4], l[4], l2[4], bad = 0;
        float r[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            h[e] = pk_bf16(v[2 * e], v[2 * e + 1]);
            r[2 * e] = v[2 * e] - __uint_as_float(h[e] << 16);
            r[2 * e + 1] = v[2 * e + 1] - __uint_as_float(h[e] & 0xFFFF0000u);
            bad |= (h[e] & 0x7F807F80u) + 0x00800080u;
        }
        if (__builtin_expect((bad & 0x80008000u) != 0, 0)) {
            // A hi part that is not finite.  Finite values that round up to infinity are cut off instead; infinities and NaN
            // leave nothing over (their difference would be NaN, and so every logit of a row whose logits are infinite).
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t hi = (h[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
                if ((hi & 0x7F80u) != 0x7F80u) continue;
                r[e] = 0.f;
                if ((__float_as_uint(v[e]) & 0x7F800000u) == 0x7F800000u) continue;
                h[e >> 1] -= 1u << (16 * (e & 1));                       // the largest finite bf16 of that sign
                r[e] = v[e] - __uint_as_float((hi - 1) << 16);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) pk_bf16_hilo(r[2 * e], r[2 * e + 1], l[e], l2[e]);
        dst[(size_t)kt * 192] = (u32x4_t){h[0], h[1], h[2], h[3]};
        dst[(size_t)kt * 192 + 64] = (u32x4_t){l[0], l[1], l[2], l[3]};
        dst[(size_t)kt * 192 + 128] = (u32x4_t){l2[0], l2[1], l2[2], l2[3]};
    }
}

hipError_t fc_split3(const float* X, int ldx, int M, int K, bf16_t* AF, hipStream_t st) {
    if (M < 1 || K % 256) return hipErrorInvalidValue;
    const int MT = (M + 15) / 16;
    int kc = (512 + MT - 1) / MT;                       // about 512 workgroups, at least 8 k-tiles each
    if (kc > K / 256) kc = K / 256;
    k_split3<<<dim3(MT, kc), 512, 0, st>>>(X, ldx, M, K, AF);
    return hipGetLastError();
}

// Eight residual values (lane (row lm, octet g4) of a k-tile): times g0, g1, the gain of the norm that comes next, as bf16
// hi + lo fragments, and their sum of squares.
__device__ inline float frag_out8(const f32x4_t& x0, const f32x4_t& x1, const f32x4_t& g0, const f32x4_t& g1, bf16_t* AF, size_t tile, int lane) {
    uint32_t h[4], l[4];
    pk_bf16_hilo(x0[0] * g0[0], x0[1] * g0[1], h[0], l[0]);
    pk_bf16_hilo(x0[2] * g0[2], x0[3] * g0[3], h[1], l[1]);
    pk_bf16_hilo(x1[0] * g1[0], x1[1] * g1[1], h[2], l[2]);
    pk_bf16_hilo(x1[2] * g1[2], x1[3] * g1[3], h[3], l[3]);
    u32x4_t* dst = (u32x4_t*)AF + tile * 128 + lane;
    dst[0] = (u32x4_t){h[0], h[1], h[2], h[3]};
    dst[64] = (u32x4_t){l[0], l[1], l[2], l[3]};
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) ss += x0[e] * x0[e] + x1[e] * x1[e];
    return ss;
}
// A pass over the rows of the residual stream: workgroups of eight rows x 256 columns (grid (row tiles x 2, N / 256)), a wave
// two rows, a lane eight columns: a row is read in runs of a kilobyte and the eight rows fill whole 128-byte lines of the
// fragments.  Such passes are bound by the latency of data that other XCDs have just written, so a lane requests all it reads
// at once.  (With 16 rows x 256 columns to a workgroup, lanes as in the fragments: 77 rows are 80 workgroups instead of 160, a
// row comes in runs of 128 bytes: reduction of eight K slices of 77 rows x 4096 7.5 us, now 5.3; of three of 256 rows x
// 5120 9.8, now 8.2.)
struct RowPass {
    int m, c, lane; size_t tile;         // row, first column; place in the fragments
    __device__ inline RowPass(int N) {
        const int oct = threadIdx.x & 31;
        m = blockIdx.x * 8 + (threadIdx.x >> 5); c = blockIdx.y * 256 + oct * 8;
        tile = (size_t)(m >> 4) * (N >> 5) + blockIdx.y * 8 + (oct >> 2); lane = (m & 15) + 16 * (oct & 3);
    }
    // partial row sums of squares [column block][row], from each lane's ss
    __device__ inline void ssq_out(float ss, float* ssq) const {
#pragma unroll
        for (int s = 1; s <= 16; s <<= 1) ss += __shfl_xor(ss, s, 64);
        if ((threadIdx.x & 31) == 0) ssq[(size_t)blockIdx.y * (gridDim.x * 8) + m] = ss;
    }
};

// Embedding gather of a many-row pass: the residual rows, and in the same pass the first layer's input fragments and
// row sums of squares.  (As two launches, the gather and a pass that read every row once per 512 workgroups for its norm,
// 256 rows of 13B: 28 us, now 7 us.)
__global__ __launch_bounds__(256) void k_embed_split(const bf16_t* emb, const int32_t* win, float* x, int M, int d, int V, RowMap rm, int W,
                                                     const float* gain, bf16_t* AF, float* ssq) {
    const RowPass r(d);
    float ss = 0.f;
    if (r.m < M) {
        const f32x4_t g0 = *(const f32x4_t*)(gain + r.c), g1 = *(const f32x4_t*)(gain + r.c + 4);       // (requested before the token is known)
        int t = win[rm.rowb ? rm.rowb[r.m] * W + rm.rowj[r.m] : r.m];
        if (t < 0 || t >= V) t = 0;
        const uint4 v = *(const uint4*)(emb + (size_t)t * d + r.c);
        const f32x4_t x0 = {__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xFFFF0000u)};
        const f32x4_t x1 = {__uint_as_float(v.z << 16), __uint_as_float(v.z & 0xFFFF0000u), __uint_as_float(v.w << 16), __uint_as_float(v.w & 0xFFFF0000u)};
        f32x4_t* o = (f32x4_t*)(x + (size_t)r.m * d + r.c);
        o[0] = x0; o[1] = x1;
        ss = frag_out8(x0, x1, g0, g1, AF, r.tile, r.lane);
    }
    r.ssq_out(ss, ssq);
}
hipError_t fc_embed_split(const void* emb, const int32_t* win, float* x, int M, int d, int V, RowMap rm, int W, const float* gain,
                          bf16_t* AF, float* ssq, hipStream_t st) {
    if (M < 1 || d % 256) return hipErrorInvalidValue;
    k_embed_split<<<dim3((M + 15) / 16 * 2, d / 256), 256, 0, st>>>((const bf16_t*)emb, win, x, M, d, V, rm, W, gain, AF, ssq);
    return hipGetLastError();
}

// ------------------------------------------------------------------ the GEMM
// Eight waves per workgroup, RT row tiles per row block (4, or 3 where that pads fewer rows: 65..96 rows are two blocks of
// 48 instead of two of 64), each wave RT x (up to CW) output tiles of 16 x 16.  Two forms:
//  KSPLIT: two groups of four waves take the first and the second pair of k-tiles of every stage for the same up to 4 * CW column
//    tiles and add their accumulators through LDS at the end; used where the launch has at most one workgroup per CU.
//    The weights of a wave's next four k-tiles (two stages) travel ahead.
//  else: the eight waves own neighbouring column tiles (up to 8 * CW) and share the activation stage.
// The column tiles are dealt evenly: ncb column blocks of NT / ncb tiles (one more in some), a block's tiles evenly to its
// waves, and ncb is what fills whole rounds of the chip (fc_gemm256_plan).  A wave with CW - 1 tiles skips the last
// one's matrix instructions on a scalar branch.
// NPL = bf16 parts of an activation: 2 (hi + lo), or 3 for the isolated LM head, whose logits are those of fp32
// arithmetic.
template <int EPI, int CW, bool KSPLIT, int RT, int NPL>
__global__ __launch_bounds__(512, 1) void k_gemm256(Gemm256Args a) {
    constexpr int STG = 4 * RT * NPL * 64;               // one stage: [k-tile][row tile][part][lane], 16 bytes each (32 KB: RT = 4, NPL = 2)
    constexpr int H0 = (RT + 1) / 2;                     // KSPLIT: row tiles that k-group 0 finishes
    constexpr int RED = KSPLIT ? 8 * CW * H0 * 64 : 0;   // accumulators the two k-groups exchange
    __shared__ u32x4_t lds[2 * STG > RED ? 2 * STG : RED];
    __shared__ float rowpart[8][16 * RT];
    constexpr int SL = RT * NPL / 2;                     // 16-byte stage loads per thread
    constexpr int CWV = KSPLIT ? 4 : 8;                  // waves a column block is dealt to
    const int tid = threadIdx.x, lane = tid & 63, w8 = __builtin_amdgcn_readfirstlane(tid >> 6), w = w8 & 3, kg = w8 >> 2;
    const int lm = lane & 15, g4 = lane >> 4;
    const int KT = a.K >> 5, NS = KT >> 2, MT = (a.M + 15) >> 4;
    // id -> (XCD x, sequence number q on that XCD) -> row block q % nrb of unit 8 * (q / nrb) + x
    const int nrb = (MT + RT - 1) / RT;
    const int xq = blockIdx.x >> 3, unit = (xq / nrb) * 8 + (blockIdx.x & 7), rb = xq % nrb;
    if (unit >= a.ncb * a.sk) return;                    // grid padding (whole workgroup leaves together)
    const int cb = unit / a.sk, ks = unit % a.sk;
    const int s_lo = (int)((unsigned)NS * (unsigned)ks / (unsigned)a.sk), s_hi = (int)((unsigned)NS * (unsigned)(ks + 1) / (unsigned)a.sk);
    // this workgroup's column tiles, and of those this wave's: nt0 .. ntend - 1
    const int cb0 = (int)((unsigned)a.NT * (unsigned)cb / (unsigned)a.ncb), cbn = (int)((unsigned)a.NT * (unsigned)(cb + 1) / (unsigned)a.ncb) - cb0;
    const int wc = KSPLIT ? w : w8;
    const int nt0 = cb0 + wc * cbn / CWV, ntend = cb0 + (wc + 1) * cbn / CWV;
    const bool full = __builtin_amdgcn_readfirstlane(ntend - nt0) >= CW;
    const int mt0 = rb * RT;
    // QKV: the cache positions of this wave's rows (a dependent load of the sequence length) are fetched here,
    // a whole K loop ahead of the epilogue that needs them
    int qpos[RT], qb[RT];
    if (EPI == EPI_QKV) {
#pragma unroll
        for (int m = 0; m < RT; ++m) {
            const int row = (mt0 + m) * 16 + lm;
            const bool rok = (!KSPLIT || kg == (m >= H0)) && mt0 + m < MT && row < a.M;
            qb[m] = rok ? (a.rm.rowb ? a.rm.rowb[row] : row / a.Wn) : 0;
            qpos[m] = rok ? a.n_state[qb[m]] + (a.rm.rowb ? a.rm.rowj[row] : row % a.Wn) : a.S;
        }
    }

    // stage copy: wave w8 copies fragments w8, w8 + 8, ... of the stage's 4 * RT * NPL.  Addresses are a uniform 64-bit
    // base (scalar registers, advanced per stage) plus a per-thread 32-bit byte offset fixed for the whole kernel:
    // no 64-bit vector arithmetic in the loop.
    const __amdgpu_buffer_rsrc_t Ar = __builtin_amdgcn_make_buffer_rsrc((void*)a.AF, 0, (uint32_t)MT * KT * NPL * 1024, 0x00020000);
    uint32_t aoff[SL];
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const int f = w8 + 8 * i, ktl = f / (RT * NPL), mtl = (f / NPL) % RT, part = f % NPL;
        const int mt = mt0 + mtl < MT ? mt0 + mtl : MT - 1;
        aoff[i] = ((((uint32_t)mt * KT + ktl) * NPL + part) * 64 + lane) * 16;
    }
    auto stage_load = [&](u32x4_t (&r)[SL], int s) {
#pragma unroll
        for (int i = 0; i < SL; ++i) r[i] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(Ar, aoff[i], s * (4096 * NPL), 0));   // 4 k-tiles x parts x 1 KB
    };
    auto stage_store = [&](const u32x4_t (&r)[SL], int buf) {
#pragma unroll
        for (int i = 0; i < SL; ++i) lds[buf * STG + (w8 + 8 * i) * 64 + lane] = r[i];
    };
    // Weights: a descriptor of the matrix and a scalar offset per pair of k-tiles, a 32-bit offset per lane fixed for the whole
    // kernel (as a base pointer plus offset the compiler kept 64-bit vector addresses, since the loads of a pair stand in
    // several blocks).
    const __amdgpu_buffer_rsrc_t Wr = __builtin_amdgcn_make_buffer_rsrc((void*)a.W, 0, (uint32_t)a.NT * KT * 1024, 0x00020000);
    uint32_t woff[CW];
#pragma unroll
    for (int j = 0; j < CW; ++j) {
        const uint32_t nt = nt0 + j < ntend ? nt0 + j : (ntend > nt0 ? ntend - 1 : cb0);     // no tile of its own: one that is being read anyway
        woff[j] = (nt * KT * 64 + lane) * 16;
    }
    struct Pair { Frag t[2]; };
    auto wload = [&](Pair& w, int j, int pair) {
        const int pc = pair < 2 * s_hi ? pair : 2 * s_hi - 1;     // past the end of the slice: its last pair again (never used, no new line)
#pragma unroll
        for (int t = 0; t < 2; ++t)                               // (not past the caches: the row blocks of a column block share these lines in L2)
            w.t[t].u = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(Wr, woff[j], pc * 2048 + t * 1024, 0));
    };

    f32x4_t acc[CW][RT];
#pragma unroll
    for (int j = 0; j < CW; ++j)
#pragma unroll
        for (int m = 0; m < RT; ++m) acc[j][m] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

    u32x4_t sr[SL];
    Pair P0[CW], P1[CW];                                 // the two pairs of a stage; KSPLIT: pair kg of a stage and of the next
    stage_load(sr, s_lo);
#pragma unroll
    for (int j = 0; j < CW; ++j) wload(P0[j], j, 2 * s_lo + (KSPLIT ? kg : 0));
#pragma unroll
    for (int j = 0; j < CW; ++j) wload(P1[j], j, 2 * s_lo + (KSPLIT ? 2 + kg : 1));
    stage_store(sr, 0);
    if (EPI != EPI_RESID && a.ssq) {
        // row statistics of the rows (activations that come without their norm scale): wave w adds every
        // eighth partial sum, all its loads in flight together; the epilogue adds the eight
        const int MP = MT * 16;
        const int row = mt0 * 16 + lane < MP ? mt0 * 16 + lane : MP - 1;
        float ssum = 0.f;
#pragma unroll 8
        for (int c = w8; c < a.nssq; c += 8) ssum += a.ssq[(size_t)c * MP + row];
        if (lane < 16 * RT) rowpart[w8][lane] = ssum;
    }
    __syncthreads();

// One accumulator: the NPL parts of one k-tile of row tile M.  The order of the matrix instructions is fixed (nothing of them
// passes the scheduling barrier, everything else does): power bounds this loop, and instructions in a row that add to
// the same accumulator take less of it.  16 x 16 x 32 alone on random data, TFLOP/s issued: another accumulator every
// instruction (the order the compiler takes, which puts dependent instructions apart) 1780-1850, two in a row 1890-1940, four
// 1940-1990, eight 2010-2030; 32 x 32 x 16 1650-1710 in any order.
#define MFMA_TILE(W, J, AP, M)                                                                      \
    do {                                                                                            \
        _Pragma("unroll") for (int p = 0; p < NPL; ++p) {                                           \
            acc[J][M] = __builtin_amdgcn_mfma_f32_16x16x32_bf16((W).v, AP[M][p].v, acc[J][M], 0, 0, 0); \
            __builtin_amdgcn_sched_barrier(0x3F6);                                                  \
        }                                                                                           \
    } while (0)
#define READ_AP(AP, KTL)                                                                            \
    _Pragma("unroll") for (int m = 0; m < RT; ++m)                                                  \
        _Pragma("unroll") for (int p = 0; p < NPL; ++p) AP[m][p].u = lds[buf * STG + (((KTL) * RT + m) * NPL + p) * 64 + lane]
// Pair U of the stage, from registers WSET: a column tile's two k-tiles row tile by row tile (four instructions in a row to
// an accumulator), then its next weights are requested: requests are spread over the pair and a weight has almost two pairs'
// time to arrive.  (A k-tile at a time for all columns, then all their requests, in the compiler's order: 7B prompt of
// 2048 7211 -> 6870 us, 13B step of 256 rows 1800 -> 1746, isolated LM head of 256 rows 196 -> 190, 77 rows 822 -> 814; the
// requests alone gave 1.3 % of the prompt and nothing of the 13B step.)  Three parts of an activation leave registers for one k-tile's only.
#define STEP(WSET, U, AHEAD)                                                                        \
    do {                                                                                            \
        const int next = 2 * s + (U) + (AHEAD);                                                     \
        if (NPL == 2) {                                                                             \
            Frag a0[RT][NPL], a1[RT][NPL];                                                          \
            READ_AP(a0, 2 * (U)); READ_AP(a1, 2 * (U) + 1);                                         \
            _Pragma("unroll") for (int j = 0; j < CW; ++j) {                                        \
                if (j < CW - 1 || full) {                                                           \
                    _Pragma("unroll") for (int m = 0; m < RT; ++m) { MFMA_TILE(WSET[j].t[0], j, a0, m); MFMA_TILE(WSET[j].t[1], j, a1, m); } \
                }                                                                                   \
                wload(WSET[j], j, next);                                                            \
                __builtin_amdgcn_sched_barrier(0);                                                  \
            }                                                                                       \
        } else {                                                                                    \
            _Pragma("unroll") for (int t = 0; t < 2; ++t) {                                         \
                Frag ap[RT][NPL];                                                                   \
                READ_AP(ap, 2 * (U) + t);                                                           \
                _Pragma("unroll") for (int j = 0; j < CW; ++j) {                                    \
                    if (j < CW - 1 || full) {                                                       \
                        _Pragma("unroll") for (int m = 0; m < RT; ++m) MFMA_TILE(WSET[j].t[t], j, ap, m); \
                    }                                                                               \
                    if (t == 1) wload(WSET[j], j, next);                                            \
                    __builtin_amdgcn_sched_barrier(0);                                              \
                }                                                                                   \
            }                                                                                       \
        }                                                                                           \
    } while (0)

    int buf = 0, s = s_lo;
    // the next stage's activations travel while this one is used (the scheduling barrier keeps their loads at the top:
    // left alone the scheduler sinks all loads to the end of the stage)
#define STAGE_BEGIN() do { stage_load(sr, s + 1 < s_hi ? s + 1 : s); __builtin_amdgcn_sched_barrier(0); } while (0)
#define STAGE_END() do { stage_store(sr, buf ^ 1); __syncthreads(); buf ^= 1; ++s; } while (0)
    while (s < s_hi) {
        STAGE_BEGIN();
        if (!KSPLIT) {
            STEP(P0, 0, 2);
            STEP(P1, 1, 2);
        } else {
            STEP(P0, kg, 4);
            STAGE_END();
            if (s >= s_hi) break;
            STAGE_BEGIN();
            STEP(P1, kg, 4);
        }
        STAGE_END();
    }
#undef STAGE_BEGIN
#undef STAGE_END
#undef STEP
#undef READ_AP
#undef MFMA_TILE

    if (KSPLIT) {
        // the two k-groups meet: each publishes the part of its accumulators that the other group will finish (group 0
        // keeps row tiles 0 .. H0 - 1, group 1 the others; the stage buffers are free after the loop's last barrier),
        // adds what it receives and runs the epilogue for its own part
        f32x4_t* red = (f32x4_t*)lds;
#pragma unroll
        for (int j = 0; j < CW; ++j)
#pragma unroll
            for (int mm = 0; mm < H0; ++mm) {
                if (kg == 1) red[((w8 * CW + j) * H0 + mm) * 64 + lane] = acc[j][mm];
                else if (H0 + mm < RT) red[((w8 * CW + j) * H0 + mm) * 64 + lane] = acc[j][H0 + mm < RT ? H0 + mm : 0];
            }
        __syncthreads();
        const int pw = kg == 0 ? w + 4 : w;             // the wave of the other group with the same n-tiles
#pragma unroll
        for (int j = 0; j < CW; ++j)
#pragma unroll
            for (int mm = 0; mm < H0; ++mm) {
                if (kg == 0) acc[j][mm] += red[((pw * CW + j) * H0 + mm) * 64 + lane];
                else if (H0 + mm < RT) acc[j][H0 + mm < RT ? H0 + mm : 0] += red[((pw * CW + j) * H0 + mm) * 64 + lane];
            }
        __syncthreads();
    }
    // ---- epilogue: acc[j][m]: rows (mt0 + m) * 16 + lm, columns (nt0 + j) * 16 + 4 * g4 + r
    float best[RT]; int bidx[RT];
    float rscale[RT];
#pragma unroll
    for (int m = 0; m < RT; ++m) {
        best[m] = -INFINITY; bidx[m] = 0x7fffffff;
        rscale[m] = 1.0f;
        if (EPI != EPI_RESID && a.ssq) {
            const int r = m * 16 + lm;
            float ssum = 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) ssum += rowpart[q][r];
            rscale[m] = 1.0f / sqrtf(ssum / (float)a.K + a.eps);
        }
    }
    // QKV: positions and rotary factors are requested a row tile ahead of their use, in front of the stores of
    // the tile before (a load behind a store that might alias it is not moved up by the compiler, and sixteen
    // tiles each waiting for their own factors cost sixteen round trips)
    f32x4_t qc[2][CW], qs[2][CW];
    auto qfactors = [&](int m, f32x4_t (&c)[CW], f32x4_t (&sn)[CW]) {
#pragma unroll
        for (int j = 0; j < CW; ++j) {
            const int nt = nt0 + j, hh = nt >> 3, t = nt & 7;
            c[j] = (f32x4_t){1.0f, 1.0f, 1.0f, 1.0f};
            sn[j] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
            if (qpos[m] < a.S && nt < ntend && hh < a.H + a.Hkv) {
                c[j] = *(const f32x4_t*)(a.cosT + (size_t)qpos[m] * 64 + 8 * t + 4 * (g4 & 1));
                sn[j] = *(const f32x4_t*)(a.sinT + (size_t)qpos[m] * 64 + 8 * t + 4 * (g4 & 1));
            }
        }
    };
    if (EPI == EPI_QKV) qfactors(0, qc[0], qs[0]);
    // RESID without K slices: the old residual rows, for the same reason a row tile ahead; and the next norm's gain
    f32x4_t xo[2][CW], gn[CW];
    float ss[RT];
    auto xold = [&](int m, f32x4_t (&x)[CW]) {
        const int row = (mt0 + m) * 16 + lm;
        const bool rok = (!KSPLIT || kg == (m >= H0)) && mt0 + m < MT && row < a.M;
#pragma unroll
        for (int j = 0; j < CW; ++j) x[j] = rok && nt0 + j < ntend ? *(const f32x4_t*)(a.out + (size_t)row * a.ldo + (nt0 + j) * 16 + 4 * g4) : (f32x4_t){0.f, 0.f, 0.f, 0.f};
    };
    if (EPI == EPI_RESID && a.sk == 1) {
        xold(0, xo[0]);
#pragma unroll
        for (int j = 0; j < CW; ++j) gn[j] = a.rf_AF && nt0 + j < ntend ? *(const f32x4_t*)(a.rf_gain + (nt0 + j) * 16 + 4 * g4) : (f32x4_t){0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int m = 0; m < RT; ++m) {
        const int row = (mt0 + m) * 16 + lm;
        const bool rok = (!KSPLIT || kg == (m >= H0)) && mt0 + m < MT && row < a.M;
        ss[m] = 0.f;
        if (EPI == EPI_QKV && m + 1 < RT) qfactors(m + 1, qc[(m + 1) & 1], qs[(m + 1) & 1]);
        if (EPI == EPI_RESID && a.sk == 1 && m + 1 < RT) xold(m + 1, xo[(m + 1) & 1]);
#pragma unroll
        for (int j = 0; j < CW; ++j) {
            const int nt = nt0 + j;
            const bool ok = rok && nt < ntend;
            f32x4_t v = acc[j][m];
            if (EPI != EPI_RESID && a.ssq) v *= rscale[m];
            if (EPI == EPI_RESID) {
                if (ok) {
                    if (a.sk > 1) *(f32x4_t*)(a.part + ((size_t)ks * a.M + row) * (a.NT * 16) + nt * 16 + 4 * g4) = v;
                    else {
                        v += xo[m & 1][j];
                        *(f32x4_t*)(a.out + (size_t)row * a.ldo + nt * 16 + 4 * g4) = v;
                        if (a.rf_AF) {
                            // the next GEMM's input: columns 16 * nt + 4 * g4 + r are k-tile nt / 2, octet 2 * (nt % 2) + g4 / 2,
                            // elements 4 * (g4 % 2) + r
                            uint32_t h0, l0, h1, l1;
                            pk_bf16_hilo(v[0] * gn[j][0], v[1] * gn[j][1], h0, l0);
                            pk_bf16_hilo(v[2] * gn[j][2], v[3] * gn[j][3], h1, l1);
                            char* dst = (char*)a.rf_AF + ((((size_t)(mt0 + m) * (a.NT >> 1) + (nt >> 1)) * 2) * 64 + lm + 16 * (2 * (nt & 1) + (g4 >> 1))) * 16 + 8 * (g4 & 1);
                            *(uint2*)dst = make_uint2(h0, h1);
                            *(uint2*)(dst + 1024) = make_uint2(l0, l1);
                            ss[m] += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
                        }
                    }
                }
            } else if (EPI == EPI_SWIGLU) {
                f32x4_t h;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float other = __shfl_xor(v[r], 32, 64);
                    h[r] = v[r] / (1.0f + expf(-v[r])) * other;
                }
                if (ok && g4 < 2) {
                    if (a.out) *(f32x4_t*)(a.out + (size_t)row * a.ldo + nt * 8 + 4 * g4) = h;
                    if (a.hfrag) {
                        // features 8 * nt + 4 * g4 + r of row `row`: k-tile nt / 4, octet nt % 4, elements 4 * g4 + r
                        uint32_t h0, l0, h1, l1;
                        pk_bf16_hilo(h[0], h[1], h0, l0);
                        pk_bf16_hilo(h[2], h[3], h1, l1);
                        const size_t KTh = (size_t)(a.ldo >> 5);
                        char* dst = (char*)a.hfrag + ((((size_t)(mt0 + m) * KTh + (nt >> 2)) * 2) * 64 + lm + 16 * (nt & 3)) * 16 + 8 * g4;
                        *(uint2*)dst = make_uint2(h0, h1);
                        *(uint2*)(dst + 1024) = make_uint2(l0, l1);
                    }
                }
            } else if (EPI == EPI_QKV) {
                const int hh = nt >> 3, t = nt & 7;
                const int b = qb[m], pos = qpos[m];
                const bool pk = ok && pos < a.S;                 // capacity guard
                const size_t plane = (size_t)a.S * 128;
                if (hh < a.H + a.Hkv) {
                    const int i0 = 8 * t + 4 * (g4 & 1);
                    f32x4_t rr;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float other = __shfl_xor(v[e], 32, 64);
                        const float c = qc[m & 1][j][e], s = qs[m & 1][j][e];
                        rr[e] = g4 < 2 ? v[e] * c - other * s : v[e] * c + other * s;
                        if (hh >= a.H) rr[e] = kv_round(rr[e], a.kvq & 15);
                    }
                    const int el = (g4 < 2 ? 0 : 64) + i0;
                    if (pk) {
                        if (hh < a.H) *(f32x4_t*)(a.out + (size_t)row * a.ldo + hh * 128 + el) = rr;
                        else {
                            bf16_t* kb = a.kc + ((((size_t)a.layer * a.B + b) * a.Hkv + (hh - a.H)) * kv_alloc_planes(a.kvp)) * plane;
                            const size_t ki = k_index(pos, el, 128);
                            bf16_t* kr = kb + ki;
                            uint32_t h[4];
                            if (a.kvp == 3) {
                                uint32_t l[4];
#pragma unroll
                                for (int e = 0; e < 4; ++e) kv24_split(rr[e], h[e], l[e]);
                                *(uint2*)kr = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
                                *(uint32_t*)((uint8_t*)(kb + plane) + ki) = l[0] | (l[1] << 8) | (l[2] << 16) | (l[3] << 24);
                            } else {
#pragma unroll
                                for (int e = 0; e < 4; ++e) h[e] = rne16(rr[e]);
                                *(uint2*)kr = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
                                if (a.kvp == 2) {
                                    uint32_t l[4];
#pragma unroll
                                    for (int e = 0; e < 4; ++e) l[e] = rne16(rr[e] - up16(h[e]));
                                    *(uint2*)(kr + plane) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
                                }
                            }
                        }
                    }
                } else if (pk) {
                    const int kh = hh - a.H - a.Hkv;
                    bf16_t* vb = a.vc + ((((size_t)a.layer * a.B + b) * a.Hkv + kh) * kv_alloc_planes(a.kvp)) * plane;
                    const size_t vi = v_index(16 * t + 4 * g4, pos, 128);
                    bf16_t* vr = vb + vi;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float vq = kv_round(v[e], a.kvq >> 4);
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
            } else if (EPI == EPI_LMHEAD) {
                const int n0 = nt * 16 + 4 * g4;
                if (ok && a.out) *(f32x4_t*)(a.out + (size_t)row * a.ldo + n0) = v;
                if (nt < ntend) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) if (v[r] > best[m]) { best[m] = v[r]; bidx[m] = n0 + r; }
                }
            }
        }
    }
    if (EPI == EPI_RESID && a.sk == 1 && a.rf_AF) {
        // partial row sums of squares over this workgroup's columns: [column block][row]
#pragma unroll
        for (int m = 0; m < RT; ++m) {
            ss[m] += __shfl_xor(ss[m], 16, 64);
            ss[m] += __shfl_xor(ss[m], 32, 64);
            if (g4 == 0) rowpart[w8][m * 16 + lm] = ss[m];
        }
        __syncthreads();
        if (tid < 16 * RT && mt0 * 16 + tid < MT * 16) {
            float t = 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) t += rowpart[q][tid];
            a.rf_ssq[(size_t)cb * (MT * 16) + mt0 * 16 + tid] = t;
        }
    }
    if (EPI == EPI_LMHEAD) {
        // winner per row over this workgroup's columns: lanes of a row, then the waves (the
        // stage buffers are free after the last barrier of the main loop)
        float (*amv)[16 * RT] = (float (*)[16 * RT])lds;
        int (*ami)[16 * RT] = (int (*)[16 * RT])(lds + STG);
#pragma unroll
        for (int m = 0; m < RT; ++m) {
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                const float ov = __shfl_xor(best[m], o, 64); const int oi = __shfl_xor(bidx[m], o, 64);
                if (ov > best[m] || (ov == best[m] && oi < bidx[m])) { best[m] = ov; bidx[m] = oi; }
            }
            if (g4 == 0 && (!KSPLIT || kg == (m >= H0))) { amv[wc][m * 16 + lm] = best[m]; ami[wc][m * 16 + lm] = bidx[m]; }
        }
        __syncthreads();
        if (tid < 16 * RT) {
            float bv = amv[0][tid]; int bx = ami[0][tid];
            for (int q = 1; q < CWV; ++q)
                if (amv[q][tid] > bv || (amv[q][tid] == bv && ami[q][tid] < bx)) { bv = amv[q][tid]; bx = ami[q][tid]; }
            const int row = mt0 * 16 + tid;
            if (row < a.M) {
                a.amax_val[(size_t)cb * a.amax_stride + row] = bv;
                a.amax_idx[(size_t)cb * a.amax_stride + row] = bx;
            }
        }
    }
}

// out[m][n] += part[0][m][n] + part[1][m][n] + ... (slice order: the result does not depend on timing), and in the same
// pass the input of the next GEMM: the new residual rows times the next norm's gain as bf16 hi + lo B-fragments, plus partial
// row sums of squares (the consumer applies the norm's row scale in its epilogue).  Rows past M of the last row tile are not written.
template <int SK>
__global__ __launch_bounds__(256) void k_resid_reduce_split(const float* part, int M, int N, float* out, int ldo,
                                                            const float* gain, bf16_t* AF, float* ssq) {
    const RowPass r(N);
    float ss = 0.f;
    if (r.m < M) {
        f32x4_t p0[SK], p1[SK];
#pragma unroll
        for (int k = 0; k < SK; ++k) {
            const f32x4_t* p = (const f32x4_t*)(part + ((size_t)k * M + r.m) * N + r.c);
            p0[k] = p[0]; p1[k] = p[1];
        }
        f32x4_t* o = (f32x4_t*)(out + (size_t)r.m * ldo + r.c);
        const f32x4_t o0 = o[0], o1 = o[1], g0 = *(const f32x4_t*)(gain + r.c), g1 = *(const f32x4_t*)(gain + r.c + 4);
#pragma unroll
        for (int k = 1; k < SK; ++k) { p0[0] = p0[0] + p0[k]; p1[0] = p1[0] + p1[k]; }
        const f32x4_t x0 = o0 + p0[0], x1 = o1 + p1[0];
        o[0] = x0; o[1] = x1;
        ss = frag_out8(x0, x1, g0, g1, AF, r.tile, r.lane);
    }
    r.ssq_out(ss, ssq);
}

// K slices for a matrix with few columns: as many as give every CU at most one workgroup (measured at 256 rows,
// 13B O / down: 240 workgroups 41 / 77 us, 480 workgroups 46 / 81 us, 320 workgroups 50 / 99 us; 7B prefill of
// 256 rows: 256 workgroups 9.4 ms, 384 10.0 ms, 512 9.9 ms: a second workgroup on a CU gains little and the
// partial tiles cost); where one per CU would leave a quarter of the CUs idle, about two per CU instead
int fc_gemm256_sk(int M, int K, int NT) {
    const int nwg = ((NT + 15) / 16) * (((M + 15) / 16 + 3) / 4), NS = K / 128;
    if (nwg >= 200) return 1;
    const int cus = fc_num_cus();
    int sk = cus / nwg;
    if (sk < 1 || nwg * sk < (3 * cus) / 4) sk = (2 * cus - 32 + nwg - 1) / nwg;
    if (sk > FC_GEMM256_MAX_SK) sk = FC_GEMM256_MAX_SK;
    if (sk > NS / 2) sk = NS / 2;
    return sk < 1 ? 1 : sk;
}

// Tiling of a launch.  Row blocks of 3 tiles where 4 would pad at least 15 % more rows.  Where blocks of 16 column tiles
// give at most one workgroup per CU of every XCD: KSPLIT, and (K slices aside, which fill the chip themselves and want the
// reuse of wide blocks) as many column blocks as there are CUs for: at these sizes a workgroup's time is what it loads.
// Else the eight waves side by side, in as few rounds of the XCDs as blocks of 32 column tiles allow and the columns dealt
// evenly over those rounds.  (Counting CUs and not each XCD's: 51 blocks x 5 row blocks are 255 workgroups, but 35 on
// three of the XCDs, a second round that cost 7B passes of 320 rows 22 %.)  Measured, blocks of fixed width (and four row tiles) -> dealt evenly: 7B QKV of 1024 rows 205 -> 185 us;
// of 77 rows gate/up 64 -> 54 us, QKV 42 -> 40 us, LM head 71 -> 67 us; 13B gate/up of 256 rows 122 us either way (216 busy
// CUs run at a higher clock than 256 do).
Gemm256Plan fc_gemm256_plan(int M, int NT, int sk, int planes) {
    Gemm256Plan p;
    const int MT = (M + 15) / 16, cus = fc_num_cus();
    const int b3 = (MT + 2) / 3, b4 = (MT + 3) / 4;
    p.rt = planes != 3 && 100 * 4 * b4 >= 115 * 3 * b3 ? 3 : 4;
    // the row blocks of a column block (and K slice) share an XCD: per round each of the eight takes cus / 8 / nrb such units
    const int nrb = p.rt == 3 ? b3 : b4, per = cus >= 8 ? cus / 8 : 1, once = 8 * (per / nrb);
    const int narrow = (NT + 15) / 16, wide = (NT + 31) / 32;
    p.ksplit = narrow * sk <= once || (sk > 1 && narrow * sk * nrb <= cus);
    if (p.ksplit) p.ncb = sk > 1 ? narrow : once;
    else {
        const int need = (wide * sk + 7) / 8, rounds = (int)(((long)need * nrb + per - 1) / per);    // units per XCD, rounds they take
        p.ncb = (int)(8 * ((long)rounds * per / nrb) / sk);
    }
    if (p.ncb > NT) p.ncb = NT;
    const int most = (NT + p.ncb - 1) / p.ncb, waves = p.ksplit ? 4 : 8;
    p.cw = (most + waves - 1) / waves;
    if (!p.ksplit && p.cw < 3) p.cw = 3;                           // (blocks of the side-by-side form have more than 16 tiles)
    return p;
}

template <int CW, bool KSPLIT, int RT>
static hipError_t launch256(int epi, const Gemm256Args& a, dim3 grid, hipStream_t st) {
    if constexpr (RT == 4) {
        if (a.planes == 3) {
            if (epi != EPI_LMHEAD) return hipErrorInvalidValue;
            k_gemm256<EPI_LMHEAD, CW, KSPLIT, 4, 3><<<grid, 512, 0, st>>>(a);
            return hipGetLastError();
        }
    }
    switch (epi) {
        case EPI_RESID: k_gemm256<EPI_RESID, CW, KSPLIT, RT, 2><<<grid, 512, 0, st>>>(a); break;
        case EPI_SWIGLU: k_gemm256<EPI_SWIGLU, CW, KSPLIT, RT, 2><<<grid, 512, 0, st>>>(a); break;
        case EPI_QKV: k_gemm256<EPI_QKV, CW, KSPLIT, RT, 2><<<grid, 512, 0, st>>>(a); break;
        case EPI_LMHEAD: k_gemm256<EPI_LMHEAD, CW, KSPLIT, RT, 2><<<grid, 512, 0, st>>>(a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <int RT>
static hipError_t launch256_rt(const Gemm256Plan& p, int epi, const Gemm256Args& a, dim3 grid, hipStream_t st) {
    if (p.ksplit) switch (p.cw) {
        case 1: return launch256<1, true, RT>(epi, a, grid, st);
        case 2: return launch256<2, true, RT>(epi, a, grid, st);
        case 3: return launch256<3, true, RT>(epi, a, grid, st);
        case 4: return launch256<4, true, RT>(epi, a, grid, st);
    } else switch (p.cw) {
        case 3: return launch256<3, false, RT>(epi, a, grid, st);
        case 4: return launch256<4, false, RT>(epi, a, grid, st);
    }
    return hipErrorInvalidValue;
}

hipError_t fc_gemm256(int epi, const Gemm256Args& a0, hipStream_t st) {
    Gemm256Args a = a0;
    if (a.M < 1 || a.K < 256 || a.K % 256 || a.NT < 1 || a.sk < 1 || a.sk > FC_GEMM256_MAX_SK || a.sk > a.K / 128) return hipErrorInvalidValue;
    if (a.sk > 1 && (epi != EPI_RESID || !a.part || !a.rf_AF)) return hipErrorInvalidValue;
    if (a.rf_AF && ((a.NT * 16) % 256 || !a.rf_gain || !a.rf_ssq)) return hipErrorInvalidValue;
    // the kernel addresses weights and fragments with 32-bit byte offsets from their bases
    if ((size_t)a.NT * 16 * a.K * 2 >= ((size_t)1 << 32) || (size_t)((a.M + 15) / 16) * 16 * a.K * (a.planes == 3 ? 6 : 4) >= ((size_t)1 << 32)) return hipErrorInvalidValue;
    const Gemm256Plan p = fc_gemm256_plan(a.M, a.NT, a.sk, a.planes);
    a.ncb = p.ncb;
    if ((size_t)a.NT * (a.ncb + 1) >= ((size_t)1 << 32)) return hipErrorInvalidValue;
    const size_t nrb = ((a.M + 15) / 16 + p.rt - 1) / p.rt, units = (size_t)p.ncb * a.sk;
    const dim3 grid((unsigned)((units + 7) / 8 * 8 * nrb));
    const hipError_t e = p.rt == 3 ? launch256_rt<3>(p, epi, a, grid, st) : launch256_rt<4>(p, epi, a, grid, st);
    if (e != hipSuccess || a.sk == 1) return e;
    const dim3 rgrid((a.M + 15) / 16 * 2, a.NT * 16 / 256);
#define REDUCE(SK) case SK: k_resid_reduce_split<SK><<<rgrid, 256, 0, st>>>(a.part, a.M, a.NT * 16, a.out, a.ldo, a.rf_gain, a.rf_AF, a.rf_ssq); break;
    switch (a.sk) { REDUCE(2) REDUCE(3) REDUCE(4) REDUCE(5) REDUCE(6) REDUCE(7) REDUCE(8) }
#undef REDUCE
    static_assert(FC_GEMM256_MAX_SK == 8, "a case per number of slices");
    return hipGetLastError();
}
