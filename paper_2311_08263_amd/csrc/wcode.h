// Coded copy of bf16 weights: what the weight-bound kernels read is 13 bits a weight instead of 16, without loss.
//
// A weight stream is bound by its bytes, and three of a trained or scaled-random weight's eight exponent bits say nothing:
// within a column nearly all magnitudes lie within 2^-30 of the largest.  Of a weight are kept
//   its low byte (mantissa and the exponent's lowest bit), its sign, and
//   4 bits: 0 where the exponent's upper seven bits are 0 (zeros above all), else those seven bits less the column's base, which
//     is the column's largest less 15 (0 at least).
// The window reaches 2^-29 below the largest power of two of the column: of normally distributed weights a few in 10^9 lie outside.
// A pair of k-tiles that holds such a weight is flagged, and whoever walks it reads its plain tiles instead.  So any bit pattern
// comes out as it went in.  (Zeros have a code because they are not that rare: 3 in 10^8 of what torch.normal_ makes, 7 in 10^6
// of sums of eight 16-bit numbers; outside the window, the few flagged pairs of a launch cost it about 2 us each at its end.)
//
// Kernels of up to 32 rows (gemmco_k.h) read the copy.  Those of many rows, bound by the matrix cores, read the plain tiles: with
// 13 vector instructions a tile (without the code for zero) the many-row products were 8-10 % slower, and with the weights kept as two planes of bytes (4
// instructions a tile, and 21 bits a weight in memory for 29) still 3-5 %.
//
// A lane of a pair of tiles (k-tiles 2 p and 2 p + 1, column lane % 16, octet lane / 16) holds 8 weights of either tile:
//   [64 lanes][16] low bytes, [64][8] nibbles (tile t: byte j = weight j | weight 4 + j << 4), [64][2] signs
//   (weight 4 h + j of tile t: bit 2 t + h + {0, 8, 4, 12}[j]): three loads of whole 128-byte lines, 1664 bytes for 2048.
#pragma once
#include "common.h"

typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2_t;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4_t;

struct WCoded { u32x4_t l; u32x2_t n; uint32_t s; };     // a lane's part of a pair: coded
struct WPlain { u32x4_t t[2]; };                         // ... and as it is

// tile t (0 or 1) of a pair as an A operand; base4 = the column's base in every byte
__device__ inline u32x4_t wc_tile(const WPlain& p, int t, uint32_t) { return p.t[t]; }
__device__ inline u32x4_t wc_tile(const WCoded& p, int t, uint32_t base4) {
    const uint32_t sg = __builtin_amdgcn_ubfe(p.s, (threadIdx.x & 1) * 16, 16), d = sg | (sg << 12), n = p.n[t];    // (bits 0..3 of every byte: the four groups of four signs)
    const uint32_t x0 = n & 0x0F0F0F0Fu, x1 = (n >> 4) & 0x0F0F0F0Fu;
    // the base for every byte that is not zero: byte selector 8 gives the sign of a base byte, which is 0
    uint32_t u0 = x0 + __builtin_amdgcn_perm(base4, base4, (~(x0 + 0x7F7F7F7Fu) & 0x80808080u) >> 4);
    uint32_t u1 = x1 + __builtin_amdgcn_perm(base4, base4, (~(x1 + 0x7F7F7F7Fu) & 0x80808080u) >> 4);
    u0 = (u0 & 0x7F7F7F7Fu) | ((d << (7 - 2 * t)) & 0x80808080u);
    u1 = (u1 & 0x7F7F7F7Fu) | ((d << (6 - 2 * t)) & 0x80808080u);
    const uint32_t l0 = p.l[2 * t], l1 = p.l[2 * t + 1];
    return (u32x4_t){__builtin_amdgcn_perm(u0, l0, 0x05010400u), __builtin_amdgcn_perm(u0, l0, 0x07030602u),
                     __builtin_amdgcn_perm(u1, l1, 0x05010400u), __builtin_amdgcn_perm(u1, l1, 0x07030602u)};
}
// pair number `pair` of a matrix, past the caches
__device__ inline void wc_load(WPlain& p, const char* W, const char*, size_t pair, uint32_t lane) {
    const u32x4_t* t = (const u32x4_t*)(W + pair * 2048 + lane * 16);
    p.t[0] = __builtin_nontemporal_load(t); p.t[1] = __builtin_nontemporal_load(t + 64);
}
__device__ inline void wc_load(WCoded& p, const char*, const char* C, size_t pair, uint32_t lane) {
    const char* at = C + pair * WC_PAIR;
    p.l = __builtin_nontemporal_load((const u32x4_t*)(at + lane * 16));
    p.n = __builtin_nontemporal_load((const u32x2_t*)(at + (1024 + lane * 8)));
    // (two lanes' signs in a word: of 16-bit loads the compiler keeps 16-bit values through the loop, and widens them, and so waits for them,
    // in front of the next requests)
    p.s = __builtin_nontemporal_load((const uint32_t*)(at + (1536 + (lane >> 1) * 4)));
}
