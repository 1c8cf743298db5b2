// Plain kernels: fp32 arithmetic.  They run fp32 models (the small parity configuration) and bf16 shapes the bf16
// matrix-core kernels do not cover, and serve as the on-device cross-check of those.  Products of fp32 weights run on the fp32
// matrix instructions (k_gemm_f32); products of bf16 weights, the cross-check, and attention stay on vector instructions.  Each
// follows the model definition the benchmark configurations fix (RMSNorm, rotary embedding pairing i with
// i + Dh/2, grouped-query attention with the causal mask of Eq. (2), SwiGLU).  Like the MFMA path a layer is five
// launches: QKV (norm, rotary embedding and cache write inside), attention, O, gate/up (norm and SwiGLU inside), down.
#include "kernels.h"
#include "wcode.h"
#include "gemmco.h"      // fc_num_cus

template <int DT> __device__ inline float wat(const void* W, size_t i) {
    if (DT == FASTCOT_F32) return ((const float*)W)[i];
    return bf16_to_f32(((const bf16_t*)W)[i]);
}
// cached value: fp32 models one fp32 plane; bf16 models a bf16 hi plane plus (kvp == 2) a bf16 lo plane or
// (kvp == 3) a plane of 8-bit residuals; i is the element index of plane 0's entry, `plane` the elements per plane
template <int DT> __device__ inline void kvstore(void* C, size_t i, size_t plane, int kvp, float v) {
    if (DT == FASTCOT_F32) { ((float*)C)[i] = v; return; }
    if (kvp == 3) {
        // (the block's base is part of i: the byte plane of a block starts one plane after its hi plane)
        uint32_t h, l; kv24_split(v, h, l);
        ((bf16_t*)C)[i] = (bf16_t)h;
        const size_t blk = i / plane * plane;
        ((uint8_t*)((bf16_t*)C + blk + plane))[i - blk] = (uint8_t)l;
        return;
    }
    bf16_t hi = f32_to_bf16(v);
    ((bf16_t*)C)[i] = hi;
    if (kvp == 2) ((bf16_t*)C)[i + plane] = f32_to_bf16(v - bf16_to_f32(hi));
}
// eight cached values that lie next to each other in plane 0 (i a multiple of 8)
template <int DT> __device__ inline void kvload8(const void* C, size_t i, size_t plane, int kvp, float (&v)[8]) {
    if (DT == FASTCOT_F32) {
        const float4 a = *(const float4*)((const float*)C + i), b = *(const float4*)((const float*)C + i + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
        return;
    }
    const uint4 h = *(const uint4*)((const bf16_t*)C + i);
    const uint32_t hw[4] = {h.x, h.y, h.z, h.w};
    if (kvp == 3) {
        const size_t blk = i / plane * plane;
        const uint2 r = *(const uint2*)((const uint8_t*)((const bf16_t*)C + blk + plane) + (i - blk));
        const uint32_t rw[2] = {r.x, r.y};
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = kv24_join((hw[e >> 1] >> (16 * (e & 1))) & 0xFFFFu, (rw[e >> 2] >> (8 * (e & 3))) & 0xFFu);
        return;
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) { v[2 * p] = __uint_as_float(hw[p] << 16); v[2 * p + 1] = __uint_as_float(hw[p] & 0xFFFF0000u); }
    if (kvp == 2) {
        const uint4 l = *(const uint4*)((const bf16_t*)C + i + plane);
        const uint32_t lw[4] = {l.x, l.y, l.z, l.w};
#pragma unroll
        for (int p = 0; p < 4; ++p) { v[2 * p] += __uint_as_float(lw[p] << 16); v[2 * p + 1] += __uint_as_float(lw[p] & 0xFFFF0000u); }
    }
}

// ------------------------------------------------------------------ embedding gather
template <int DT>
__global__ void k_embed(const void* emb, const int32_t* win, float* x, int d, int V, RowMap rm, int W) {
    int m = blockIdx.x;
    int t = win[rm.rowb ? rm.rowb[m] * W + rm.rowj[m] : m];
    if (t < 0 || t >= V) t = 0;
    if (DT == FASTCOT_BF16 && d % 8 == 0) {          // eight elements (16 bytes) per thread and pass
        const uint4* src = (const uint4*)((const bf16_t*)emb + (size_t)t * d);
        float4* dst = (float4*)(x + (size_t)m * d);
        for (int i = threadIdx.x; i < d / 8; i += blockDim.x) {
            const uint4 v = src[i];
            dst[2 * i] = make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xFFFF0000u));
            dst[2 * i + 1] = make_float4(__uint_as_float(v.z << 16), __uint_as_float(v.z & 0xFFFF0000u), __uint_as_float(v.w << 16), __uint_as_float(v.w & 0xFFFF0000u));
        }
        return;
    }
    for (int i = threadIdx.x; i < d; i += blockDim.x) x[(size_t)m * d + i] = wat<DT>(emb, (size_t)t * d + i);
}
hipError_t fc_embed(const void* emb, int dt, const int32_t* win, float* x, int M, int d, int V, hipStream_t st, RowMap rm, int W) {
    if (dt == FASTCOT_F32) k_embed<FASTCOT_F32><<<M, 256, 0, st>>>(emb, win, x, d, V, rm, W);
    else k_embed<FASTCOT_BF16><<<M, 256, 0, st>>>(emb, win, x, d, V, rm, W);
    return hipGetLastError();
}

// ------------------------------------------------------------------ GEMM  Y[m][n] (+)= sum_k norm(X)[m][k] W[k][n]
// A norm in front (gain != NULL) costs no pass of its own: the gain multiplies the inputs, the row's 1 / rms the sums.
// K is spread wide and nothing is staged.
//
// bf16 weights (k_gemm_plain): eight waves, wave w on k-tiles of 32 inputs w, w + 8, ...; lane (column lm, octet g) loads 8
// weights of its column and the 8 inputs of every row (the 16 lanes of an octet share the address), and the partial sums meet by
// two lane exchanges and one LDS round.  A workgroup computes 8 rows x 16 * NC columns: NC = 1 gives the most workgroups;
// NC = 4 reads the activations once for four tiles.
enum { PEPI_STORE = 0, PEPI_ADD = 1, PEPI_SWIGLU = 2, PEPI_QKV = 3 };
// One thread of the workgroup finishes an output: product v of row m and column n (16-column tile nt, column c of it) and the value
// eight columns away; yold, fcos, fsin and pos as plain_request fetched them.
struct PlainRest { float yold, fcos, fsin; int pos; };
template <int EPI>
__device__ inline void plain_request_first(const PlainGemm& a, int m, PlainRest& r, int& tok) {
    r.pos = 0; tok = 0;
    if (EPI == PEPI_QKV) r.pos = a.n_state[m / a.kd.W] + m % a.kd.W;
    if (EPI == PEPI_ADD && a.emb) { tok = a.tok[m]; if (tok < 0 || tok >= a.V) tok = 0; }
}
template <int EPI>
__device__ inline void plain_request(const PlainGemm& a, int m, int n, int c, int tok, PlainRest& r) {
    r.yold = 0.f; r.fcos = 1.f; r.fsin = 0.f;
    if (EPI == PEPI_ADD) r.yold = a.emb ? a.emb[(size_t)tok * a.ldy + (n < a.N ? n : 0)] : a.Y[(size_t)m * a.ldy + (n < a.N ? n : 0)];
    if (EPI == PEPI_QKV) {
        const int half = a.kd.Dh >> 1, hh = n / a.kd.Dh, i = 8 * ((n % a.kd.Dh) >> 4) + (c & 7), p = r.pos < a.kd.S ? r.pos : 0;
        if (hh < a.kd.H + a.kd.Hkv) { r.fcos = a.cosT[(size_t)p * half + i]; r.fsin = a.sinT[(size_t)p * half + i]; }
    }
}
template <int DT, int EPI>
__device__ inline void plain_finish(const PlainGemm& a, int m, int nt, int c, float v, float other, const PlainRest& rest) {
    const int n = nt * 16 + c;
    if (EPI == PEPI_STORE) { if (n < a.N) a.Y[(size_t)m * a.ldy + n] = v; }
    else if (EPI == PEPI_ADD) { if (n < a.N) a.Y[(size_t)m * a.ldy + n] = rest.yold + v; }
    else if (EPI == PEPI_SWIGLU) {                         // columns 0..7 of a tile: gate of features 8 * nt ..; 8..15: their up values
        if (c < 8) a.Y[(size_t)m * a.ldy + nt * 8 + c] = v / (1.0f + expf(-v)) * other;
    } else {
        // row m = b*W + j sits at absolute position n[b] + j; the product is in packed column order (head_col).
        // Rotated q goes to qrot in natural order, k heads are rotated and stored to the K cache, v heads stored to
        // the transposed V cache.
        const KernelDims& kd = a.kd;
        const int b = m / kd.W, pos = rest.pos, half = kd.Dh >> 1, hh = n / kd.Dh, cc = n % kd.Dh;
        a.Y[(size_t)m * a.ldy + n] = v;                    // read by fastcot_debug_read alone
        if (pos >= kd.S) return;                           // capacity guard: never write outside the cache
        const size_t plane = (size_t)kd.S * kd.Dh;
        if (hh < kd.H + kd.Hkv) {
            const int i = 8 * (cc >> 4) + (c & 7), el = c < 8 ? i : i + half;
            const float rot = c < 8 ? v * rest.fcos - other * rest.fsin : v * rest.fcos + other * rest.fsin;
            if (hh < kd.H) a.qrot[(size_t)m * kd.H * kd.Dh + (size_t)hh * kd.Dh + el] = rot;
            else kvstore<DT>(a.kc, kv_block(kd, a.layer, b, hh - kd.H) + k_index(pos, el, kd.Dh), plane, kd.kvp, rot);
        } else
            kvstore<DT>(a.vc, kv_block(kd, a.layer, b, hh - kd.H - kd.Hkv) + v_index(cc, pos, kd.Dh), plane, kd.kvp, v);
    }
}

template <int EPI, int NC>
__global__ __launch_bounds__(512) void k_gemm_plain(PlainGemm a) {
    constexpr int RB = 8;
    __shared__ float part[8][NC][RB][16];
    __shared__ float part_ss[8][RB];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lm = lane & 15, g = lane >> 4;
    const int nt0 = blockIdx.x * NC, m0 = blockIdx.y * RB, NT = a.NP >> 4, KT = a.K >> 5;
    const float* xr[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) xr[r] = a.X + (size_t)(m0 + r < a.M ? m0 + r : a.M - 1) * a.ldx;   // rows past M repeat the last one, never written
    float acc[NC][RB], ss[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        ss[r] = 0.f;
#pragma unroll
        for (int j = 0; j < NC; ++j) acc[j][r] = 0.f;
    }
    auto ktile = [&](int kt) {
        const int k0 = kt * 32 + 8 * g;
        float wv[NC][8];
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int nt = nt0 + j < NT ? nt0 + j : NT - 1;
            const uint4 h = *((const uint4*)a.W + ((size_t)nt * (a.K >> 5) + kt) * 64 + lane);
            const uint32_t hw[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
            for (int p = 0; p < 4; ++p) { wv[j][2 * p] = __uint_as_float(hw[p] << 16); wv[j][2 * p + 1] = __uint_as_float(hw[p] & 0xFFFF0000u); }
        }
        float gv[8];
        if (a.gain) {
            const float4 g0 = *(const float4*)(a.gain + k0), g1 = *(const float4*)(a.gain + k0 + 4);
            gv[0] = g0.x; gv[1] = g0.y; gv[2] = g0.z; gv[3] = g0.w; gv[4] = g1.x; gv[5] = g1.y; gv[6] = g1.z; gv[7] = g1.w;
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const float4 x0 = *(const float4*)(xr[r] + k0), x1 = *(const float4*)(xr[r] + k0 + 4);
            float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (a.gain) { ss[r] += x[e] * x[e]; x[e] *= gv[e]; }
#pragma unroll
                for (int j = 0; j < NC; ++j) acc[j][r] += x[e] * wv[j][e];
            }
        }
    };
    // (one tile per workgroup: two workgroups share a CU instead of two k-tiles of one wave, which would take 175 registers)
#pragma unroll (NC == 1 ? 1 : 2)
    for (int kt = w; kt < KT; kt += 8) ktile(kt);
    // octets: two exchanges; then each of the four octet groups publishes two rows of the wave's sums
#pragma unroll
    for (int r = 0; r < RB; ++r) {
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            acc[j][r] += __shfl_xor(acc[j][r], 16, 64);
            acc[j][r] += __shfl_xor(acc[j][r], 32, 64);
            if (g == (r >> 1)) part[w][j][r][lm] = acc[j][r];
        }
        if (a.gain) {
            ss[r] += __shfl_xor(ss[r], 16, 64);
            ss[r] += __shfl_xor(ss[r], 32, 64);
            if (lane == 0) part_ss[w][r] = ss[r];
        }
    }
    __syncthreads();
    if (tid >= NC * 128) return;
    const int j = tid >> 7, r = (tid >> 4) & 7, c = tid & 15, m = m0 + r, nt = nt0 + j;
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) v += part[q][j][r][c];
    if (a.gain) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) s += part_ss[q][r];
        v *= 1.0f / sqrtf(s / (float)a.K + a.eps);
    }
    const float other = __shfl_xor(v, 8, 64);             // the value 8 columns away: rotary partner, or gate <-> up
    if (m >= a.M || nt >= NT) return;
    PlainRest rest; int tok;
    plain_request_first<EPI>(a, m, rest, tok);
    plain_request<EPI>(a, m, nt * 16 + c, c, tok, rest);
    plain_finish<FASTCOT_BF16, EPI>(a, m, nt, c, v, other, rest);
}

// fp32 weights: the fp32 matrix instructions (16 x 16 outputs x 4 inputs, products and sums in fp32).  Bound by latency at the
// sizes it is meant for (256-wide layers: all weights in L2, a launch is a few load round trips), so the point is few
// instructions and one round trip: a workgroup computes 16 rows x 16 * NC columns; wave w of eight takes the groups of 16 inputs w,
// w + 8, ..., U of them requested together; lane (row or column lm, quarter g) holds inputs 4 g .. 4 g + 3 of the group: one
// 16-byte load of its row and four weights of its column, which are the operands of four instructions.  What the epilogue needs
// besides the product is requested up front.  (On vector instructions, a lane loading the inputs of all eight rows, a launch's X
// loads alone kept the CU's load path busy for 0.9 us.)  8 rows of the 256-wide model, traced, that
// form -> this: QKV 6.1 -> 4.6 us, O 3.8 -> 2.1, gate/up 5.5 -> 4.6, down 8.0 -> 4.7, LM head 4.9 -> 4.1; steps of fp32 models of 96 to 2048
// inputs and 1 to 128 rows 1.15 to 2.0 times as fast as a whole.
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
template <int EPI, int NC>
__global__ __launch_bounds__(512) void k_gemm_f32(PlainGemm a) {
    constexpr int U = NC == 1 ? 6 : 4;
    __shared__ float part[8][NC][16 * 17];
    __shared__ float part_ss[8][16];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), lm = lane & 15, g = lane >> 4;
    const int nt0 = blockIdx.x * NC, m0 = blockIdx.y * 16, NT = a.NP >> 4, GT = a.K >> 4;
    // the output this thread finishes (the first NC * 256 threads)
    const int fj = (tid >> 8) % NC, fr = (tid >> 4) & 15, fc = tid & 15, fm = m0 + fr < a.M ? m0 + fr : a.M - 1;
    const int fnt = nt0 + fj < NT ? nt0 + fj : NT - 1;
    PlainRest rest; int ftok;
    plain_request_first<EPI>(a, fm, rest, ftok);
    const int row = m0 + lm < a.M ? m0 + lm : a.M - 1;     // rows past M repeat the last one, never written
    const float* xr = a.X + (size_t)row * a.ldx;
    if (EPI == PEPI_QKV && a.emb) { const int t = a.tok[row]; xr = a.emb + (size_t)(t < 0 || t >= a.V ? 0 : t) * a.ldx; }
    uint32_t wo[NC];                                       // (weights: a uniform base per input, a fixed 32-bit offset per lane)
#pragma unroll
    for (int j = 0; j < NC; ++j) wo[j] = (uint32_t)(4 * g) * (uint32_t)a.NP + (nt0 + j < NT ? nt0 + j : NT - 1) * 16 + lm;
    f32x4_t acc[NC][4];                                    // (short chains: with one accumulator the sums lose a bit against 64 bits)
#pragma unroll
    for (int j = 0; j < NC; ++j) acc[j][0] = acc[j][1] = acc[j][2] = acc[j][3] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    float ss = 0.f;
    bool first = true;
    for (int g0 = w; g0 < GT || first; g0 += 8 * U) {      // (waves without a group still request what they finish)
        float wv[U][NC][4];
        float4 x[U], gn[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int gi = g0 + 8 * u;
            if (gi < GT) {
#pragma unroll
                for (int j = 0; j < NC; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) wv[u][j][i] = ((const float*)a.W + (size_t)(gi * 16 + i) * a.NP)[wo[j]];
                x[u] = *(const float4*)(xr + gi * 16 + 4 * g);
                if (a.gain) gn[u] = *(const float4*)(a.gain + gi * 16 + 4 * g);
            }
        }
        if (first) plain_request<EPI>(a, fm, fnt * 16 + fc, fc, ftok, rest);
        first = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (g0 + 8 * u < GT) {
                float xv[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
                if (a.gain) {
                    const float gv[4] = {gn[u].x, gn[u].y, gn[u].z, gn[u].w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) { ss += xv[i] * xv[i]; xv[i] *= gv[i]; }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < NC; ++j) acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[u][j][i], xv[i], acc[j][i], 0, 0, 0);
            }
        }
    }
    // lane: row lm, columns 4 g + e
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const f32x4_t s = (acc[j][0] + acc[j][1]) + (acc[j][2] + acc[j][3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) part[w][j][lm * 17 + 4 * g + e] = s[e];
    }
    if (a.gain) {
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (g == 0) part_ss[w][lm] = ss;
    }
    __syncthreads();
    if (tid >= NC * 256) return;
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) v += part[q][fj][fr * 17 + fc];
    if (a.gain) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) s += part_ss[q][fr];
        v *= 1.0f / sqrtf(s / (float)a.K + a.eps);
    }
    const float other = __shfl_xor(v, 8, 64);             // the value 8 columns away: rotary partner, or gate <-> up
    if (m0 + fr >= a.M || nt0 + fj >= NT) return;
    plain_finish<FASTCOT_F32, EPI>(a, m0 + fr, nt0 + fj, fc, v, other, rest);
}
template <int DT, int EPI> static hipError_t launch_gemm_plain(const PlainGemm& a, hipStream_t st) {
    const int NT = a.NP >> 4;
    if constexpr (DT == FASTCOT_F32) {
        const int rb = (a.M + 15) / 16;
        // two column tiles per workgroup where one would give more than eight workgroups per CU
        if ((size_t)NT * rb > 2048) k_gemm_f32<EPI, 2><<<dim3((NT + 1) / 2, rb), 512, 0, st>>>(a);
        else k_gemm_f32<EPI, 1><<<dim3(NT, rb), 512, 0, st>>>(a);
    } else {
        const int rb = (a.M + 7) / 8;
        // four tiles per workgroup only where that leaves several workgroups per CU
        if ((size_t)NT * rb >= 4096) k_gemm_plain<EPI, 4><<<dim3((NT + 3) / 4, rb), 512, 0, st>>>(a);
        else k_gemm_plain<EPI, 1><<<dim3(NT, rb), 512, 0, st>>>(a);
    }
    return hipGetLastError();
}
template <int DT> static hipError_t launch_gemm_plain_epi(int epi, const PlainGemm& a, hipStream_t st) {
    switch (epi) {
        case PEPI_STORE: return launch_gemm_plain<DT, PEPI_STORE>(a, st);
        case PEPI_ADD: return launch_gemm_plain<DT, PEPI_ADD>(a, st);
        case PEPI_SWIGLU: return launch_gemm_plain<DT, PEPI_SWIGLU>(a, st);
        case PEPI_QKV: return launch_gemm_plain<DT, PEPI_QKV>(a, st);
    }
    return hipErrorInvalidValue;
}
static hipError_t gemm_plain_any(int epi, int dt, const PlainGemm& a, hipStream_t st) {
    if (a.M < 1 || a.K < 16 || a.K % (dt == FASTCOT_F32 ? 16 : 32) || a.NP < 16 || a.NP % 16 || a.ldx % 4) return hipErrorInvalidValue;
    return dt == FASTCOT_F32 ? launch_gemm_plain_epi<FASTCOT_F32>(epi, a, st) : launch_gemm_plain_epi<FASTCOT_BF16>(epi, a, st);
}
hipError_t fc_gemm_plain(const void* W, int dt, int K, int NP, int N, const float* X, int ldx, float* Y, int ldy,
                         int M, int accumulate, hipStream_t st, const float* gain, float eps, TokenRows tr) {
    PlainGemm a{}; a.emb = tr.emb; a.tok = tr.tok; a.V = tr.V; a.W = W; a.K = K; a.NP = NP; a.N = N; a.X = X; a.ldx = ldx; a.Y = Y; a.ldy = ldy; a.M = M; a.gain = gain; a.eps = eps;
    return gemm_plain_any(accumulate ? PEPI_ADD : PEPI_STORE, dt, a, st);
}
hipError_t fc_swiglu_plain(const void* W, int dt, int K, int F, const float* X, int ldx, float* h, int M, const float* gain,
                           float eps, hipStream_t st) {
    PlainGemm a{}; a.W = W; a.K = K; a.NP = a.N = 2 * F; a.X = X; a.ldx = ldx; a.Y = h; a.ldy = F; a.M = M; a.gain = gain; a.eps = eps;
    return gemm_plain_any(PEPI_SWIGLU, dt, a, st);
}
hipError_t fc_qkv_plain(const void* W, int dt, const KernelDims& kd, int layer, const float* X, const float* gain, float* qkv, float* qrot,
                        const int32_t* n_state, const float* cosT, const float* sinT, void* kc, void* vc, hipStream_t st,
                        TokenRows tr) {
    PlainGemm a{}; a.emb = tr.emb; a.tok = tr.tok; a.V = tr.V; a.W = W; a.K = kd.d; a.NP = a.N = kd.qkvN; a.X = X; a.ldx = kd.d; a.Y = qkv; a.ldy = kd.qkvN; a.M = kd.M;
    a.gain = gain; a.eps = kd.eps; a.kd = kd; a.layer = layer; a.qrot = qrot; a.n_state = n_state; a.cosT = cosT; a.sinT = sinT; a.kc = kc; a.vc = vc;
    return gemm_plain_any(PEPI_QKV, dt, a, st);
}

// ------------------------------------------------------------------ window-causal attention
__device__ inline float block_sum(float v, float* red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    float s = 0;
    for (int i = 0; i < nw; ++i) s += red[i];
    return s;
}
// One workgroup (4 waves) per (row m, query head h): scores over cache positions 0 .. n[b]+j, softmax, weighted V.
// Both passes read the cache in its own fragment order, eight values per lane and load: a wave takes 16 keys (lane =
// key r, quarter p of the head elements; two exchanges add the quarters), then 16 head elements x 32 positions
// (lane = element, octet of positions), and the waves' sums over their blocks meet in LDS.  With a thread per key and
// a thread per head element walking all keys one by one a 64-row window over 1088 keys and 40 heads took 647 us; now 172 us.
// EARLY (heads of up to 64 elements, launches of at most two workgroups per CU, bf16 caches of at most 128 positions): each wave's first K tile and V block are
// requested before anything is known of the lengths, so that the launch is not a chain of four round trips; what lies behind the
// last position is read all the same and not used, same bits.  fp32 caches, 8 rows x 32 heads of 64, plain -> EARLY: 0 to 32 keys 6.2 -> 5.6 us,
// 200 9.9 -> 9.9, 2000 73.3 -> 72.1, 15800 525 -> 521.  bf16 caches gain while a wave has no block but its first one (128
// positions) and lose after that: 32 keys 6.9 -> 6.5 us, 127 7.6 -> 7.1, 152 10.4 -> 10.7, 700 25.0 -> 25.4; so only in caches that
// hold no more.  (Heads of 128: the unrolled copies of the long loop cost long contexts a quarter.  Four workgroups per CU: 6-8 % at 32 keys, 1 % at 2000.)
#define EARLY_BF16_KEYS 128
template <int DT, bool EARLY>
__global__ __launch_bounds__(256) void k_attn_plain(const float* q, int ldq, const void* kc, const void* vc, KernelDims kd, int layer,
                                                    const int32_t* n_state, int n_host, float* out) {
    extern __shared__ float sc[];   // [S] scores, [Dh] the query, [4][Dh] sums of the waves, [16] reduction scratch
    float* qs = sc + kd.S; float* wsum = qs + kd.Dh; float* red = wsum + 4 * kd.Dh;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 15, p = lane >> 4;
    const int m = blockIdx.x, h = blockIdx.y, b = m / kd.W, j = m % kd.W;
    int last = (n_state ? n_state[b] : n_host) + j;
    const int kh = h / (kd.H / kd.Hkv), Dh = kd.Dh, G = Dh >> 5;
    const size_t kbase = kv_block(kd, layer, b, kh), plane = (size_t)kd.S * Dh;
    constexpr int EG = EARLY ? 2 : 1;
    float kv0[EG][8], vv0[2 * EG][8];
    if (EARLY) {
        const int nblk = (kd.S + 31) >> 5, kb0 = (w >> 1) < nblk ? w >> 1 : nblk - 1, vb0 = w < nblk ? w : nblk - 1;
#pragma unroll
        for (int i = 0; i < EG; ++i)
            if (i < G) kvload8<DT>(kc, kbase + (size_t)kb0 * 32 * Dh + (size_t)(((w & 1) * 4 + p) * 16 * G + r + 16 * i) * 8, plane, kd.kvp, kv0[i]);
#pragma unroll
        for (int i = 0; i < 2 * EG; ++i)
            if (i < 2 * G) kvload8<DT>(vc, kbase + (size_t)vb0 * 32 * Dh + (size_t)(i * 64 + lane) * 8, plane, kd.kvp, vv0[i]);
    }
    for (int i = tid; i < Dh; i += 256) qs[i] = q[(size_t)m * ldq + (size_t)h * Dh + i];
    if (last >= kd.S) last = kd.S - 1;
    const int NB = (last >> 5) + 1;
    __syncthreads();
    const float scale = 1.0f / sqrtf((float)Dh);
    float mx = -3.0e38f;
    if (EARLY && w < 2 * NB) {                             // half block w, as below
        const int pos = (w >> 1) * 32 + 8 * (r >> 2) + 4 * (w & 1) + (r & 3);
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < EG; ++i)
            if (i < G)
#pragma unroll
                for (int e = 0; e < 8; ++e) s += qs[32 * i + 8 * p + e] * kv0[i][e];
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        s *= scale;
        if (pos <= last) { if (p == 0) sc[pos] = s; mx = fmaxf(mx, s); }
    }
    for (int hb = EARLY ? w + 4 : w; hb < 2 * NB; hb += 4) {   // half block: tile hb % 2 of key block hb / 2
        const int pos = (hb >> 1) * 32 + 8 * (r >> 2) + 4 * (hb & 1) + (r & 3);
        float s = 0.f;
#pragma unroll 4
        for (int i = 0; i < G; ++i) {
            float kv[8];
            kvload8<DT>(kc, kbase + (size_t)(hb >> 1) * 32 * Dh + (size_t)(((hb & 1) * 4 + p) * 16 * G + r + 16 * i) * 8, plane, kd.kvp, kv);
#pragma unroll
            for (int e = 0; e < 8; ++e) s += qs[32 * i + 8 * p + e] * kv[e];
        }
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        s *= scale;
        if (pos <= last) { if (p == 0) sc[pos] = s; mx = fmaxf(mx, s); }
    }
    for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) red[w] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    float den = 0.f;
    for (int t = tid; t <= last; t += 256) { const float e = expf(sc[t] - mx); sc[t] = e; den += e; }
    den = block_sum(den, red);                             // (its first barrier also publishes the weights)
    if constexpr (EARLY) {
#pragma unroll
        for (int dt = 0; dt < 2 * EG; ++dt) {
            if (dt >= 2 * G) break;
            float acc = 0.f;
            if (w < NB)                                    // the wave's first block, which is here already
#pragma unroll
                for (int e = 0; e < 8; ++e) acc += w * 32 + 8 * p + e <= last ? sc[w * 32 + 8 * p + e] * vv0[dt][e] : 0.f;
#pragma unroll 4
            for (int blk = w + 4; blk < NB; blk += 4) {
                float kv[8];
                kvload8<DT>(vc, kbase + (size_t)blk * 32 * Dh + (size_t)(dt * 64 + lane) * 8, plane, kd.kvp, kv);
                const int t0 = blk * 32 + 8 * p;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc += t0 + e <= last ? sc[t0 + e] * kv[e] : 0.f;
            }
            acc += __shfl_xor(acc, 16, 64);
            acc += __shfl_xor(acc, 32, 64);
            if (p == 0) wsum[w * Dh + dt * 16 + r] = acc;
        }
    } else
    for (int dt = 0; dt < Dh >> 4; ++dt) {
        float acc = 0.f;
#pragma unroll 4
        for (int blk = w; blk < NB; blk += 4) {
            float kv[8];
            kvload8<DT>(vc, kbase + (size_t)blk * 32 * Dh + (size_t)(dt * 64 + lane) * 8, plane, kd.kvp, kv);
            const int t0 = blk * 32 + 8 * p;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc += t0 + e <= last ? sc[t0 + e] * kv[e] : 0.f;
        }
        acc += __shfl_xor(acc, 16, 64);
        acc += __shfl_xor(acc, 32, 64);
        if (p == 0) wsum[w * Dh + dt * 16 + r] = acc;
    }
    __syncthreads();
    for (int i = tid; i < Dh; i += 256)
        out[(size_t)m * kd.H * Dh + (size_t)h * Dh + i] = (wsum[i] + wsum[Dh + i] + wsum[2 * Dh + i] + wsum[3 * Dh + i]) / den;
}
hipError_t fc_attn_plain(const float* q, int ldq, const void* kc, const void* vc, int dt, const KernelDims& kd,
                         int layer, const int32_t* n_state, int n_host, float* out, hipStream_t st) {
    dim3 grid(kd.M, kd.H);
    const size_t sh = ((size_t)kd.S + 5 * kd.Dh + 16) * sizeof(float);
    auto launch = [&](auto kernel) -> hipError_t {
        if (sh > 64 * 1024) {                              // the longest caches: past the default limit of a launch
            const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) return e;
        }
        kernel<<<grid, 256, sh, st>>>(q, ldq, kc, vc, kd, layer, n_state, n_host, out);
        return hipSuccess;
    };
    const bool early = kd.Dh <= 64 && kd.M * kd.H <= 2 * fc_num_cus() && (dt == FASTCOT_F32 || kd.S <= EARLY_BF16_KEYS);
    const hipError_t e = dt == FASTCOT_F32 ? (early ? launch(k_attn_plain<FASTCOT_F32, true>) : launch(k_attn_plain<FASTCOT_F32, false>))
                                           : (early ? launch(k_attn_plain<FASTCOT_BF16, true>) : launch(k_attn_plain<FASTCOT_BF16, false>));
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

// ------------------------------------------------------------------ per-row argmax, lowest index on ties
__global__ void k_argmax(const float* logits, int V, int32_t* ids, float* top) {
    __shared__ float bv[4];
    __shared__ int bi[4];
    const float* r = logits + (size_t)blockIdx.x * V;
    float best = -INFINITY; int idx = 0x7fffffff;
    for (int i = threadIdx.x; i < V; i += blockDim.x) {
        float v = r[i];
        if (v > best || (v == best && i < idx)) { best = v; idx = i; }
    }
    for (int o = 32; o > 0; o >>= 1) {
        float ov = __shfl_down(best, o, 64); int oi = __shfl_down(idx, o, 64);
        if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
    }
    if ((threadIdx.x & 63) == 0) { bv[threadIdx.x >> 6] = best; bi[threadIdx.x >> 6] = idx; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
            if (bv[w] > best || (bv[w] == best && bi[w] < idx)) { best = bv[w]; idx = bi[w]; }
        ids[blockIdx.x] = idx == 0x7fffffff ? 0 : idx; top[blockIdx.x] = best;      // nothing but NaN: an id of the vocabulary all the same
    }
}
hipError_t fc_argmax_plain(const float* logits, int M, int V, int32_t* ids, float* top, hipStream_t st) {
    k_argmax<<<M, 256, 0, st>>>(logits, V, ids, top);
    return hipGetLastError();
}

// ------------------------------------------------------------------ packing
// canonical [rows][cols] -> fused matrix columns; mode selects the column map: 0 natural at col_off,
// 1 / 2 gate / up interleave, 3 + Dh rotary-pair order inside heads of Dh columns (q and k heads).
__device__ inline int pack_col(int c, int col_off, int mode) { return mode == 0 ? col_off + c : (mode <= 2 ? gu_col(c, mode - 1) : qkv_col(col_off + c, mode - 3, 0x7fffffff)); }
__global__ void k_pack_f32(const float* src, int rows, int cols, float* dst, int NP, int col_off, int mode) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)rows * cols) return;
    const int k = (int)(i / cols), c = (int)(i % cols);
    dst[(size_t)k * NP + pack_col(c, col_off, mode)] = src[i];
}
// bf16: a thread takes eight rows of a column at a time, which are a lane's 16 bytes of the fragment: rows are read in runs of the workgroup's
// columns, sixteen neighbouring columns are written as 256 bytes.  stamp (or NULL) and stamp[tensor] take the hash of what was packed; a workgroup
// takes many rows so that few of them add to it.
__global__ void k_stamp_clear(unsigned long long* stamp, int tensor) {       // (tensors may be packed on several streams)
    atomicAdd(stamp, 0ull - stamp[tensor]);
    stamp[tensor] = 0;
}
__device__ inline unsigned long long stamp_mix(unsigned long long x) {
    x = (x ^ (x >> 31)) * 6364136223846793005ull;
    x = (x ^ (x >> 29)) * 2862933555777941757ull;
    return x ^ (x >> 32);
}
__global__ __launch_bounds__(1024) void k_pack_bf16(const bf16_t* src, int rows, int cols, bf16_t* dst, int K, int col_off, int mode, unsigned long long* stamp, int tensor) {
    __shared__ unsigned long long part[16];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63);
    unsigned long long h = 0;
    if (c < cols) {
        const int n = pack_col(c, col_off, mode);
        const unsigned long long salt = (unsigned long long)tensor << 40;
        for (int k = (blockIdx.y * 16 + (threadIdx.x >> 6)) * 8; k < rows; k += gridDim.y * 128) {
            uint32_t v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = src[(size_t)(k + e) * cols + c];
            const u32x4_t w = {v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16)};
            const size_t at = frag_index(K, k, n);
            *(u32x4_t*)(dst + at) = w;
            h += stamp_mix((w[0] | ((unsigned long long)w[1] << 32)) + stamp_mix(salt + at)) + stamp_mix((w[2] | ((unsigned long long)w[3] << 32)) + stamp_mix(salt + at + 4));
        }
    }
    if (!stamp) return;
    for (int o = 32; o > 0; o >>= 1) h += __shfl_xor(h, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = h;
    __syncthreads();
    if (threadIdx.x >= 2) return;
    h = 0;
    for (int q = 0; q < 16; ++q) h += part[q];
    atomicAdd(stamp + threadIdx.x * tensor, h);
}
// The coded copy (wcode.h) of a matrix from its plain tiles: a workgroup an n-tile, its eight waves all of K twice, for
// the columns' largest exponents and for the codes.
__global__ __launch_bounds__(512) void k_code(const char* W, char* C, int K, int NT) {
    __shared__ uint32_t top[8][16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lm = lane & 15, nt = blockIdx.x, PT = K >> 6;
    const u32x4_t* src = (const u32x4_t*)W + (size_t)nt * PT * 128 + lane;
    uint32_t hi = 0;
#pragma unroll 4
    for (int t = w; t < 2 * PT; t += 8) {
        const u32x4_t v = src[(size_t)t * 64];
#pragma unroll
        for (int i = 0; i < 4; ++i) { const uint32_t a = (v[i] >> 8) & 0x7Fu, b = (v[i] >> 24) & 0x7Fu; hi = max(hi, max(a, b)); }
    }
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, 16, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, 32, 64));
    if (lane < 16) top[w][lane] = hi;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) hi = max(hi, top[q][lm]);
    const uint32_t base = hi > 15 ? hi - 15 : 0;
    if (tid < 16) C[wc_base_off(K, NT) + (size_t)nt * 16 + tid] = (char)base;
    for (int p = w; p < PT; p += 8) {
        u32x4_t l; u32x2_t n; uint32_t s = 0, out = 0;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const u32x4_t v = src[(size_t)(2 * p + t) * 64];
            n[t] = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t lw = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t x = (v[2 * h + (j >> 1)] >> (16 * (j & 1))) & 0xFFFFu, e = (x >> 8) & 0x7Fu;
                    const bool in = e == 0 || e > base;              // (e - base <= 15: no exponent is above the largest)
                    out |= !in;
                    lw |= (x & 0xFFu) << (8 * j);
                    n[t] |= (in && e ? e - base : 0u) << (8 * j + 4 * h);
                    s |= (x >> 15) << (2 * t + h + ((j & 1) << 3) + ((j >> 1) << 2));
                }
                l[2 * t + h] = lw;
            }
        }
        char* at = C + ((size_t)nt * PT + p) * WC_PAIR;
        *(u32x4_t*)(at + lane * 16) = l;
        *(u32x2_t*)(at + 1024 + lane * 8) = n;
        *(uint16_t*)(at + 1536 + lane * 2) = (uint16_t)s;
        const bool any = __ballot(out != 0) != 0;
        if (lane == 0) C[wc_flag_off(K, NT) + (size_t)nt * PT + p] = (char)any;
    }
}
hipError_t fc_code(const void* W, void* C, int K, int NT, hipStream_t st) {
    if (K < 256 || K % 256 || NT < 1) return hipErrorInvalidValue;
    k_code<<<NT, 512, 0, st>>>((const char*)W, (char*)C, K, NT);
    return hipGetLastError();
}
hipError_t fc_pack(const void* src, int dt, int rows, int cols, void* dst_base, const FusedMat& fm, int col_off,
                   int mode, hipStream_t st, void* stamp, int tensor) {
    char* dst = (char*)dst_base + fm.off;
    if (dt == FASTCOT_F32) {
        const size_t n = (size_t)rows * cols;
        k_pack_f32<<<(unsigned)((n + 255) / 256), 256, 0, st>>>((const float*)src, rows, cols, (float*)dst, fm.NP, col_off, mode);
        return hipGetLastError();
    }
    if (rows % 32) return hipErrorInvalidValue;
    if (stamp) k_stamp_clear<<<1, 1, 0, st>>>((unsigned long long*)stamp, tensor);
    const int runs = (rows / 8 + 15) / 16, strips = (cols + 63) / 64, per = strips < 1024 ? 1024 / strips : 1;
    k_pack_bf16<<<dim3(strips, runs < per ? runs : per), 1024, 0, st>>>((const bf16_t*)src, rows, cols, (bf16_t*)dst, fm.K, col_off, mode, (unsigned long long*)stamp, tensor);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess && fm.coded ? fc_code(dst, dst + wc_off(fm.K, fm.NP / 16), fm.K, fm.NP / 16, st) : e;
}
// A packed model's stamp is the sum of hashes over all its matrices, each of every 8 bytes of it and their place (k_pack_bf16): a coded
// copy's record (the stamp of the weights it was made from, its complement while there is no copy) shows whether it is of the weights that are there.
__global__ void k_stamp_keep(const unsigned long long* stamp, unsigned long long* record, int made) { *record = made ? *stamp : ~*stamp; }
__global__ void k_stamp_look(const unsigned long long* stamp, const unsigned long long* record, int* host) { *host = *stamp != *record; }
hipError_t fc_stamp_keep(const void* stamp, void* record, int made, hipStream_t st) {
    k_stamp_keep<<<1, 1, 0, st>>>((const unsigned long long*)stamp, (unsigned long long*)record, made);
    return hipGetLastError();
}
hipError_t fc_stamp_look(const void* stamp, const void* record, int* host, hipStream_t st) {
    k_stamp_look<<<1, 1, 0, st>>>((const unsigned long long*)stamp, (const unsigned long long*)record, host);
    return hipGetLastError();
}

__global__ void k_fill_f32(float* dst, size_t n, float v) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = v;
}
hipError_t fc_fill_f32(float* dst, size_t n, float v, hipStream_t st) {
    if (n == 0) return hipSuccess;
    k_fill_f32<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(dst, n, v);
    return hipGetLastError();
}
__global__ void k_copy_u32(uint32_t* dst, const uint32_t* src, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}
hipError_t fc_copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t st) {  // bytes % 4 == 0
    size_t n = bytes / 4;
    if (n == 0) return hipSuccess;
    k_copy_u32<<<(unsigned)((n + 255) / 256), 256, 0, st>>>((uint32_t*)dst, (const uint32_t*)src, n);
    return hipGetLastError();
}

// canonical K, V [S_in][Hkv][Dh] -> cache layout of one sequence: per head [S/32 blocks][32 * Dh] in fragment order (k_index, v_index)
template <int DT>
__global__ void k_kv_scatter(const void* k, const void* v, int S_in, int Hkv, int Dh, int S, void* kc, void* vc) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)S_in * Hkv * Dh) return;
    int e = (int)(i % Dh), h = (int)((i / Dh) % Hkv), t = (int)(i / ((size_t)Dh * Hkv));
    if (DT == FASTCOT_F32) {
        ((float*)kc)[(size_t)h * S * Dh + k_index(t, e, Dh)] = ((const float*)k)[i];
        ((float*)vc)[(size_t)h * Dh * S + v_index(e, t, Dh)] = ((const float*)v)[i];
    } else {
        ((bf16_t*)kc)[(size_t)h * S * Dh + k_index(t, e, Dh)] = ((const bf16_t*)k)[i];
        ((bf16_t*)vc)[(size_t)h * Dh * S + v_index(e, t, Dh)] = ((const bf16_t*)v)[i];
    }
}
hipError_t fc_kv_scatter(const void* k, const void* v, int S_in, int Hkv, int Dh, int S, int dt, void* kc, void* vc,
                         hipStream_t st) {
    size_t n = (size_t)S_in * Hkv * Dh;
    unsigned blocks = (unsigned)((n + 255) / 256);
    if (dt == FASTCOT_F32) k_kv_scatter<FASTCOT_F32><<<blocks, 256, 0, st>>>(k, v, S_in, Hkv, Dh, S, kc, vc);
    else k_kv_scatter<FASTCOT_BF16><<<blocks, 256, 0, st>>>(k, v, S_in, Hkv, Dh, S, kc, vc);
    return hipGetLastError();
}
