// Decoding-state kernels: all per-sequence state (committed length n, generated count g, the
// Approximate Tokens Buffer, the window, done flags) lives in device memory so that a captured
// step can be replayed without host arguments.
#include "kernels.h"

// Prefill pass of R rows per sequence starting at prompt position p0: row j of sequence b carries
// prompt token p0 + j if that token is one of the first len-1 prompt tokens, else a pad (its K/V is
// never committed).
__global__ void k_prefill_window(int32_t* st, StateMap sm, int B, int R, int S, int p0) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B * R) return;
    int b = i / R, j = i % R;
    int len = st[sm.plen + b];
    int p = p0 + j;
    st[sm.win + i] = (p < len - 1) ? st[sm.prompt + (size_t)b * S + p] : 0;
}
hipError_t fc_prefill_window(int32_t* state, const StateMap& sm, int B, int R, int S, int p0, hipStream_t st) {
    k_prefill_window<<<(B * R + 255) / 256, 256, 0, st>>>(state, sm, B, R, S, p0);
    return hipGetLastError();
}

// After the forward of a prefill pass that ended at prompt position p1: commit the K/V of the real
// prompt rows.  After the last pass, set up the first Jacobi window: slot 0 = last prompt token,
// slots 1.. = buffer[0..W-2].
__global__ void k_prefill_advance(int32_t* st, StateMap sm, int B, int W, int S, int p1, int last) {
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    int len = st[sm.plen + b];
    int n = p1;
    if (n > len - 1) n = len - 1;
    st[sm.n + b] = n;
    if (last) {
        st[sm.g + b] = 0; st[sm.done + b] = 0; st[sm.steps + b] = 0; st[sm.lastK + b] = 0; st[sm.olen + b] = 0;
        int newest = st[sm.prompt + (size_t)b * S + len - 1];
        st[sm.newest + b] = newest;
        st[sm.win + b * W] = newest;
        for (int j = 1; j < W; ++j) st[sm.win + b * W + j] = st[sm.buf + (size_t)b * S + j - 1];
    }
}
hipError_t fc_prefill_advance(int32_t* state, const StateMap& sm, int B, int W, int S, int p1, int last,
                              hipStream_t st) {
    k_prefill_advance<<<(B + 63) / 64, 64, 0, st>>>(state, sm, B, W, S, p1, last);
    return hipGetLastError();
}

// Verification (Eq. 5), acceptance, cache update and window shift (Sec. 4.3), stop conditions
// (Sec. 4.4) for every sequence.  o[b][j] is the argmax of row j, i.e. the prediction for the
// token after window slot j.  Approximate slot i is verified when o[i-1] == win[i]; slots are
// checked in order and the first miss stops.  K verified slots => K+1 exact tokens o[0..K].
// Committing their K/V is the bump of n: rows 0..K of this step wrote their K/V at positions
// n..n+K already.  All W fresh outputs go back to the buffer; the window slides by K+1.
// One wave per sequence, lane j on window slot j (in rounds of 64 for wider windows): the scans of Eq. 5 and of
// the EOS rule are ballots, the copies one load and one store per lane.
// o_all [B][W]: the argmax ids of the step's rows (in memory or LDS).  Called by a whole workgroup.
__device__ inline void accept_commit(int32_t* st, const StateMap& sm, int B, int W, int S, const int32_t* o_all) {
    __shared__ int not_done;
    if (threadIdx.x == 0) not_done = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int max_new = st[sm.params + PARAM_MAX_NEW], eos = st[sm.params + PARAM_EOS];
    const int max_steps = st[sm.params + PARAM_MAX_STEPS], buf_len = st[sm.params + PARAM_BUF_LEN];
    for (int b = wave; b < B; b += nwaves) {
        if (st[sm.done + b]) { if (lane == 0) st[sm.lastK + b] = -1; continue; }
        const int32_t* w = st + sm.win + b * W;
        const int32_t* o = o_all + b * W;
        int32_t* buf = st + sm.buf + (size_t)b * S;
        int32_t* out = st + sm.out + (size_t)b * S;
        int n = st[sm.n + b], g = st[sm.g + b], steps = st[sm.steps + b];
        const int g0 = g, olen0 = st[sm.olen + b];
        // a sequence with a window of its own uses the first Wb rows of its W: the others are ignored (or not computed)
        const int ws = st[sm.wseq + b], Wb = ws > 0 && ws < W ? ws : W;
        // K = verified slots: the first i in 1..Wb-1 with o[i-1] != w[i] ends the scan (Eq. 5); E = first accepted
        // row that is an EOS (rows after it are not emitted)
        int K = Wb - 1, E = Wb;
        for (int j0 = 0; j0 < Wb - 1; j0 += 64) {
            const int j = j0 + lane;
            const bool miss = j < Wb - 1 && o[j] != w[j + 1];
            const unsigned long long mask = __ballot(miss);
            if (mask) { K = j0 + __ffsll((long long)mask) - 1; break; }
        }
        if (eos >= 0)
            for (int j0 = 0; j0 <= K; j0 += 64) {
                const int j = j0 + lane;
                const unsigned long long mask = __ballot(j <= K && o[j] == eos);
                if (mask) { E = j0 + __ffsll((long long)mask) - 1; break; }
            }
        // all Wb fresh outputs go back to the buffer ("Cache Update", Sec. 4.3); the next window is read from the
        // values themselves where they were just written (slot p of the buffer, p - g0 < Wb), else from the buffer
        const int last = E < K ? E : K;                         // last emitted row
        for (int j = lane; j < Wb; j += 64) {
            const int oj = o[j];
            if (g0 + j < buf_len) buf[g0 + j] = oj;
            if (j <= last && g0 + j < max_new && g0 + j < S) out[g0 + j] = oj;
        }
        int jmax = last;
        if (jmax > max_new - 1 - g0) jmax = max_new - 1 - g0;
        if (jmax > S - 1 - g0) jmax = S - 1 - g0;
        const int emitted = jmax >= 0 ? g0 + jmax + 1 : 0;
        int stop = E <= K;
        const int newest = o[K];
        n += K + 1; g += K + 1; ++steps;
        if (g >= max_new || (max_steps > 0 && steps >= max_steps)) stop = 1;
        bool err = false;
        if (n + W > S || g + 2 * W - 1 > buf_len) {       // no room for another window: stop, flag it
            err = !stop;
            stop = 1;
        }
        // (the window is rewritten only after every lane has read its o and w above: a wave runs in lockstep, and
        // the reads below touch o and the part of the buffer this step did not write)
        int32_t* wn = st + sm.win + b * W;
        for (int j = lane; j < W; j += 64) {
            int v;
            if (j == 0) v = newest;
            else {
                const int p = g + j - 1;
                v = p >= buf_len ? 0 : (p - g0 < Wb ? o[p - g0] : buf[p]);
            }
            wn[j] = v;
        }
        if (lane == 0) {
            if (emitted > olen0) st[sm.olen + b] = emitted;
            if (err) st[sm.flags + FLAG_ERROR] = 1;
            st[sm.n + b] = n; st[sm.g + b] = g; st[sm.steps + b] = steps; st[sm.lastK + b] = K;
            st[sm.newest + b] = newest; st[sm.done + b] = stop;
            if (!stop) atomicAdd(&not_done, 1);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) st[sm.flags + FLAG_ALL_DONE] = (not_done == 0);
}
__global__ void k_accept_commit(int32_t* st, StateMap sm, int B, int W, int S) { accept_commit(st, sm, B, W, S, st + sm.o); }

// The end of a small step in one launch: one workgroup of sixteen waves finds every row's argmax and, with the ids still in
// LDS, runs the accept step.  Two launches cost a kernel boundary more (2-4 us) than one workgroup loses against one per
// row, as long as there is little to read: see fc_tail_fits.
#define TAIL_IDS 1024                                      // one per thread
__device__ inline bool tail_better(float v, int i, float best, int bi) { return v > best || (v == best && i < bi); }
// rows of a packed step sit at entry rowb[m] * W + rowj[m] of the ids
__device__ inline int tail_dst(const RowMap& rm, int m, int W) { return rm.rowb ? rm.rowb[m] * W + rm.rowj[m] : m; }

// from the logits [M][V], a wave per row
__global__ __launch_bounds__(1024) void k_tail_logits(const float* logits, int M, int V, float* top, int32_t* st, StateMap sm, int B, int W, int S) {
    __shared__ int32_t ids[TAIL_IDS];
    const int lane = threadIdx.x & 63;
    for (int m = threadIdx.x >> 6; m < M; m += 16) {
        const float* r = logits + (size_t)m * V;
        float best = -INFINITY; int bi = 0x7fffffff;
        int i = lane;
        for (; i + 192 < V; i += 256) {                    // four loads in flight; ascending ids: a later one wins only by value
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = r[i + 64 * u];
#pragma unroll
            for (int u = 0; u < 4; ++u) if (tail_better(v[u], i + 64 * u, best, bi)) { best = v[u]; bi = i + 64 * u; }
        }
        for (; i < V; i += 64) { const float v = r[i]; if (tail_better(v, i, best, bi)) { best = v; bi = i; } }
        for (int o = 32; o > 0; o >>= 1) {
            const float ov = __shfl_xor(best, o, 64); const int oi = __shfl_xor(bi, o, 64);
            if (tail_better(ov, oi, best, bi)) { best = ov; bi = oi; }
        }
        if (lane == 0) { ids[m] = bi == 0x7fffffff ? 0 : bi; st[sm.o + m] = ids[m]; top[m] = best; }     // nothing but NaN: id 0
    }
    __syncthreads();
    accept_commit(st, sm, B, W, S, ids);
}
// from the LM head's winners per workgroup, val / idx [nparts][R], R = 16 or 32 rows: lane (row, part), so that a wave's load takes
// whole lines
template <int R>
__global__ __launch_bounds__(1024) void k_tail_winners(const float* val, const int32_t* idx, int nparts, int M, float* top, RowMap rm, int32_t* st,
                                                       StateMap sm, int B, int W, int S) {
    __shared__ int32_t ids[TAIL_IDS];
    __shared__ float bv[16][R];
    __shared__ int bi[16][R];
    const int tid = threadIdx.x, m = tid % R, wave = tid >> 6;
    float best = -INFINITY; int b = 0x7fffffff;
#pragma unroll 4
    for (int c = tid / R; c < nparts; c += 1024 / R) {
        const float v = val[(size_t)c * R + m]; const int i = idx[(size_t)c * R + m];
        if (tail_better(v, i, best, b)) { best = v; b = i; }
    }
#pragma unroll
    for (int o = R; o < 64; o <<= 1) {
        const float ov = __shfl_xor(best, o, 64); const int oi = __shfl_xor(b, o, 64);
        if (tail_better(ov, oi, best, b)) { best = ov; b = oi; }
    }
    if ((tid & 63) < R) { bv[wave][m] = best; bi[wave][m] = b; }
    for (int i = tid; i < B * W; i += 1024) ids[i] = st[sm.o + i];     // entries no row of this step fills keep what they were
    __syncthreads();
    if (tid < M) {
        for (int q = 0; q < 16; ++q) if (tail_better(bv[q][tid], bi[q][tid], best, b)) { best = bv[q][tid]; b = bi[q][tid]; }
        const int dst = tail_dst(rm, tid, W), id = b == 0x7fffffff ? 0 : b;
        ids[dst] = id; st[sm.o + dst] = id; top[dst] = best;
    }
    __syncthreads();
    accept_commit(st, sm, B, W, S, ids);
}
// What a wave walks decides: per row a fixed part and a round per 256 logits.  A step of a small one-layer model, two launches ->
// one, us: up to 16 rows (a wave each) 1 x 2048 logits 32.4 -> 31.4, 16 x 2048 33.0 -> 32.3, 1 x 4096 34.1 -> 34.2, 16 x 4096 34.6 ->
// 35.2, 1 x 8192 39.6 -> 41.2; two rows a wave 32 x 256 31.1 -> 30.6, 32 x 512 31.1 -> 31.4; 64 x 64 31.1 -> 32.1, 512 x 16 40 -> 63.
// Winners, 16 / 32 columns of them: 64 parts 56.2 -> 55.0 / 54.4 -> 53.1, 256 parts 56.4 -> 56.1 / 55.0 -> 55.4, 512 parts 61.2 ->
// 62.0 / 64.6 -> 67.1.
bool fc_tail_fits(int B, int W, int M, int V_or_parts, bool winners) {
    if (B * W > TAIL_IDS) return false;
    if (winners) return M <= 32 && V_or_parts * (M > 16 ? 32 : 16) <= 4096;
    return (M + 15) / 16 * (5 + (V_or_parts + 255) / 256) <= 13;
}
hipError_t fc_tail_logits(const float* logits, int M, int V, float* top, int32_t* state, const StateMap& sm, int B, int W, int S, hipStream_t st) {
    if (!fc_tail_fits(B, W, M, V, false) || M != B * W) return hipErrorInvalidValue;
    k_tail_logits<<<1, 1024, 0, st>>>(logits, M, V, top, state, sm, B, W, S);
    return hipGetLastError();
}
hipError_t fc_tail_winners(const float* val, const int32_t* idx, int nparts, int stride, int M, float* top, RowMap rm, int32_t* state,
                           const StateMap& sm, int B, int W, int S, hipStream_t st) {
    if (!fc_tail_fits(B, W, M, nparts, true) || (stride != 16 && stride != 32) || M > stride) return hipErrorInvalidValue;
    if (stride == 16) k_tail_winners<16><<<1, 1024, 0, st>>>(val, idx, nparts, M, top, rm, state, sm, B, W, S);
    else k_tail_winners<32><<<1, 1024, 0, st>>>(val, idx, nparts, M, top, rm, state, sm, B, W, S);
    return hipGetLastError();
}
// What fastcot_generate looks at between batches of steps, to pinned host memory: g[B], done[B], the two flags.
__global__ void k_report(const int32_t* st, StateMap sm, int B, int32_t* host) {
    for (int i = threadIdx.x; i < 2 * B + 2; i += blockDim.x)
        host[i] = i < B ? st[sm.g + i] : (i < 2 * B ? st[sm.done + i - B] : st[sm.flags + i - 2 * B]);
}
hipError_t fc_report(const int32_t* state, const StateMap& sm, int B, int32_t* host, hipStream_t st) {
    k_report<<<1, 64, 0, st>>>(state, sm, B, host);
    return hipGetLastError();
}

// A new window size between steps: the window is rebuilt from the newest exact token and the buffer
// (the buffer already holds every output of the previous steps, Sec. 4.3 "Cache Update").
__global__ void k_rewindow(int32_t* st, StateMap sm, int B, int W, int S) {
    const int buf_len = st[sm.params + PARAM_BUF_LEN];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B * W) return;
    const int b = i / W, j = i % W;
    const int p = st[sm.g + b] + j - 1;
    st[sm.win + i] = j == 0 ? st[sm.newest + b] : (p < buf_len ? st[sm.buf + (size_t)b * S + p] : 0);
}
hipError_t fc_rewindow(int32_t* state, const StateMap& sm, int B, int W, int S, hipStream_t st) {
    k_rewindow<<<(B * W + 255) / 256, 256, 0, st>>>(state, sm, B, W, S);
    return hipGetLastError();
}

hipError_t fc_accept_commit(int32_t* state, const StateMap& sm, int B, int W, int S, hipStream_t st) {
    const int waves = B < 16 ? (B < 1 ? 1 : B) : 16;
    k_accept_commit<<<1, 64 * waves, 0, st>>>(state, sm, B, W, S);
    return hipGetLastError();
}

// ------------------------------------------------------------------ sequence slots
// Two sequences trade slots: every per-sequence entry of the state block (one workgroup) ...
__global__ void k_swap_seq(int32_t* st, StateMap sm, int b1, int b2, int W, int S) {
    const int t = threadIdx.x;
    if (t < 9) {
        const int32_t offs[9] = {sm.n, sm.g, sm.done, sm.steps, sm.newest, sm.lastK, sm.plen, sm.olen, sm.wseq};
        const int32_t v1 = st[offs[t] + b1], v2 = st[offs[t] + b2];
        st[offs[t] + b1] = v2; st[offs[t] + b2] = v1;
    }
    for (int j = t; j < W; j += blockDim.x) {
        const int32_t v1 = st[sm.win + b1 * W + j], v2 = st[sm.win + b2 * W + j];
        st[sm.win + b1 * W + j] = v2; st[sm.win + b2 * W + j] = v1;
    }
    const int32_t rows[3] = {sm.buf, sm.out, sm.prompt};
    for (int r = 0; r < 3; ++r)
        for (int j = t; j < S; j += blockDim.x) {
            const int32_t v1 = st[rows[r] + b1 * S + j], v2 = st[rows[r] + b2 * S + j];
            st[rows[r] + b1 * S + j] = v2; st[rows[r] + b2 * S + j] = v1;
        }
}
// ... and their K/V cache: `count` chunks of n16 sixteen-byte words, chunk i at a + i * stride16 and b + i * stride16
__global__ void k_swap_chunks(uint4* a, uint4* b, size_t n16, size_t stride16) {
    uint4* pa = a + (size_t)blockIdx.y * stride16; uint4* pb = b + (size_t)blockIdx.y * stride16;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x) {
        const uint4 va = pa[i], vb = pb[i];
        pa[i] = vb; pb[i] = va;
    }
}
hipError_t fc_swap_sequences(int32_t* state, const StateMap& sm, int b1, int b2, int W, int S, void* kc, void* vc,
                             size_t seq_bytes, int layers, size_t layer_stride_bytes, hipStream_t st) {
    if (b1 == b2) return hipSuccess;
    if (seq_bytes % 16 || layer_stride_bytes % 16) return hipErrorInvalidValue;
    k_swap_seq<<<1, 256, 0, st>>>(state, sm, b1, b2, W, S);
    const size_t n16 = seq_bytes / 16;
    unsigned gx = (unsigned)((n16 + 255) / 256);
    if (gx > 2048) gx = 2048;
    for (int which = 0; which < 2; ++which) {
        char* base = (char*)(which ? vc : kc);
        k_swap_chunks<<<dim3(gx, (unsigned)layers), 256, 0, st>>>((uint4*)(base + (size_t)b1 * seq_bytes), (uint4*)(base + (size_t)b2 * seq_bytes),
                                                                 n16, layer_stride_bytes / 16);
    }
    return hipGetLastError();
}
