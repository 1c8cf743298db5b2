// Launches of the column-owner GEMM (gemmco_k.h): its grid, the choice between coded copy and plain tiles, and the kernels of the
// plain tiles; and the reduction behind the LM head.
#include "gemmco_k.h"

static int g_cus = 0;
static int num_cus() {
    if (!g_cus) {
        int dev = 0; hipDeviceProp_t p;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess) g_cus = p.multiProcessorCount;
        if (g_cus <= 0) g_cus = 256;
    }
    return g_cus;
}

int fc_num_cus() { return num_cus(); }

// grid: one workgroup per CU unless that would give a workgroup more than `most` n-tiles (at most 8: with two
// row tiles a workgroup then finishes 16 output tiles, whose partial sums take 64 KB of LDS).
// wide (up to 16 rows): one round also of 12 to 14 n-tiles per CU.  The second round costs a head and a tail and reads the activations
// once more; one pair of 14 tiles per wave keeps the loads as busy as two of eight.  us, two rounds / one: LM heads of 16 rows (one
// matrix, call after call), 51200 columns, 2048 / 4096 / 8192 inputs 41.7 / 37.6, 68.6 / 61.4, 122.5 / 111.7; two layers of the 70B shape (gate/up 14
// tiles per CU) 636 / 621.  Fewer tiles run as 12 and gain nothing (40000 columns, 9.8 tiles: 16 rows 56.5 / 56.7, 5 rows 51.9 / 54.8), and so do
// more rounds of wider workgroups (128256 columns: four rounds of eight 147 us, three of twelve 155).
int fc_gemmco_grid(int NT, int most, bool wide) {
    int G = num_cus();
    if (wide && NT > 11 * G && NT <= 14 * G) return G;
    if (G > NT) G = NT;
    while ((NT + G - 1) / G > most) G += num_cus();
    return G;
}

// Most n-tiles per workgroup (of 8, 6, 4, 3, 2 or 1: 5 runs as 6, 7 as 8) whose partial tiles and gain fit the LDS
int fc_gemmco_most(int M, int K, bool gain) {
    const int inst[6] = {8, 6, 4, 3, 2, 1};
    for (int i = 0; i < 6; ++i) {
        GemmCoArgs a; a.K = K; a.ks = 1;
        if (co_lds_plan(a, inst[i], M > 16 ? 2 : 1, gain) <= CO_LDS_MOST) return inst[i];
    }
    return 1;
}

bool fc_gemmco_fits(int M, int K, int NT, int G, int ks, bool gain) {
    if (M < 1 || M > 32 || K < 256 || K % 256 || NT < 1 || G < 1 || ks < 1 || ks > 8 || G % ks || G / ks > NT || K / 256 < ks) return false;
    const int inst[8] = {1, 2, 3, 4, 6, 8, 12, 14}, own = (NT + G / ks - 1) / (G / ks), most = M <= 16 ? 14 : 8;
    if (own > most || (ks > 1 && G / ks > FC_MAX_COUNTERS)) return false;
    int nw = own;
    for (int i = 7; i >= 0; --i) if (inst[i] >= own) nw = inst[i];
    GemmCoArgs a; a.K = K; a.ks = ks;
    return co_lds_plan(a, nw, M > 16 ? 2 : 1, gain) <= CO_LDS_MOST;
}

hipError_t fc_gemmco(int epi, const GemmCoArgs& a, int G, hipStream_t st) {
    const int ks = a.ks > 1 ? a.ks : 1;
    if (!fc_gemmco_fits(a.M, a.K, a.NT, G, ks, a.gain != nullptr)) return hipErrorInvalidValue;
    if (epi != EPI_LMHEAD && (a.gain != nullptr) != co_gained(epi)) return hipErrorInvalidValue;          // (no norm in front of an adding product, one in front of the others)
    if (ks > 1 && (epi == EPI_LMHEAD || !a.xpart || !a.xcnt)) return hipErrorInvalidValue;
    // Plain tiles of up to eight n-tiles per workgroup are walked in rotated order: the slices of different workgroups start at addresses that
    // differ by multiples of K * 32 bytes, in step they would all sit on the same memory channels.  us a launch in order / rotated, 16 rows:
    // down of the 7B / 13B / 70B shape 24.6 / 22.3, 30.6 / 31.0, 78.6 / 75.2 (24 rows 86.4 / 79.3), O 13.2 / 12.7, 16.4 / 16.3, 31.4 / 28.0, QKV
    // 23.2 / 23.0, 33.5 / 32.1, 37 / 35.8, gate/up 36.6 / 36.5, 54 / 50.4, LM head 49.1 / 45.1, 55.7 / 56.5, 86.8 / 83.0; with 14 n-tiles per workgroup
    // (70B gate/up) 141.3 / 143.3.  Coded pairs are 1664 bytes, so that the slices fall on different channels by themselves: as fast or faster in order.
    GemmCoArgs b = a;
    if (a.rotate == 2) b.rotate = !a.C && (a.NT + G / ks - 1) / (G / ks) <= 8;
    return b.C ? fc_gemmco_coded(epi, b, G, st) : launch_co<WPlain>(epi, b, G, st);
}

// reduction of the LM head's per-workgroup winners: lowest id on ties
__global__ void k_argmax_final(const float* val, const int32_t* idx, int nparts, int stride, int32_t* ids, float* top, RowMap rm, int W) {
    __shared__ float bv[4];
    __shared__ int bi[4];
    const int m = blockIdx.x;
    float best = -INFINITY; int b = 0x7fffffff;
    for (int c = threadIdx.x; c < nparts; c += blockDim.x) {
        float v = val[(size_t)c * stride + m]; int i = idx[(size_t)c * stride + m];
        if (v > best || (v == best && i < b)) { best = v; b = i; }
    }
    for (int o = 32; o > 0; o >>= 1) {
        float ov = __shfl_xor(best, o, 64); int oi = __shfl_xor(b, o, 64);
        if (ov > best || (ov == best && oi < b)) { best = ov; b = oi; }
    }
    if ((threadIdx.x & 63) == 0) { bv[threadIdx.x >> 6] = best; bi[threadIdx.x >> 6] = b; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < (int)(blockDim.x >> 6); ++q)
            if (bv[q] > best || (bv[q] == best && bi[q] < b)) { best = bv[q]; b = bi[q]; }
        const int dst = rm.rowb ? rm.rowb[m] * W + rm.rowj[m] : m;
        ids[dst] = b == 0x7fffffff ? 0 : b; top[dst] = best;       // nothing but NaN: an id of the vocabulary all the same
    }
}
hipError_t fc_argmax_final(const float* val, const int32_t* idx, int nparts, int stride, int M, int32_t* ids, float* top,
                           hipStream_t st, RowMap rm, int W) {
    k_argmax_final<<<M, 256, 0, st>>>(val, idx, nparts, stride, ids, top, rm, W);
    return hipGetLastError();
}
