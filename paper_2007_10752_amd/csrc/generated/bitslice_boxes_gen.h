// Generated by paper_2007_10752_amd/gen/emit.py from the DES tables of the
// paper's Appendix A and the verified S-box networks.  Do not edit.
#pragma once
#include <stdint.h>

#include "bitslice_gen.h"

// One S-box on 32 blocks per lane: d[q] ^= output q ^ m.o[q], x the box's six
// inputs as right-half words, m.e[i] the mask of its i-th second-use input.
template <int J>
__device__ __forceinline__ void bs_box(const uint32_t *x, uint32_t *d, const BsBoxMasks &m);

template <>
__device__ __forceinline__ void bs_box<0>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S1
    const uint32_t x0 = x[0];
    const uint32_t x1 = x[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5] ^ m.e[0];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x1, x4, x5, 0x69);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x3, x4, g6, 0xb5);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x1, g6, g7, 0x7c);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x2, g7, g8, 0x25);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x1, g7, g9, 0x4a);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x4, g9, g10, 0x2b);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x2, g7, g11, 0x39);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x0, x2, g8, 0x29);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x4, g7, g13, 0x8c);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x3, g11, g14, 0x85);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(g7, g12, g13, 0x4a);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(x3, g8, g16, 0x67);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x0, g6, g17, 0x78);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(g10, g15, g18, 0x2d);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(x0, g12, g19, 0xca);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(g8, g12, g14, 0xf6);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(x4, g19, g17, 0x99);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(x4, x5, g20, 0xe9);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(x0, x1, x3, 0xd6);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(g8, g14, g23, 0xd8);
    const uint32_t g26 = __builtin_amdgcn_bitop3_b32(g9, g17, g22, 0x8f);
    const uint32_t g27 = __builtin_amdgcn_bitop3_b32(g24, g25, g26, 0xd2);
    const uint32_t g28 = __builtin_amdgcn_bitop3_b32(g6, g23, g27, 0x96);
    const uint32_t g29 = __builtin_amdgcn_bitop3_b32(g21, g22, g28, 0x63);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g20, m.o[0], 0x96);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g29, m.o[1], 0x69);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g22, m.o[2], 0x96);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g27, m.o[3], 0x96);
}

template <>
__device__ __forceinline__ void bs_box<1>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S2
    const uint32_t x0 = x[0] ^ m.e[0];
    const uint32_t x1 = x[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x0, x1, x4, 0xd3);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x4, x5, g6, 0xd7);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x1, x5, g7, 0xf9);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x0, x5, g8, 0x96);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x2, x5, g6, 0xb4);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x2, g8, g9, 0x4d);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x3, g7, g11, 0x4b);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(g8, g10, g12, 0x93);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x4, g9, g13, 0x96);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x5, g6, g13, 0x26);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(x5, g14, g15, 0x47);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(g8, g12, g16, 0x63);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x5, g10, g12, 0xb0);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(x1, x4, g18, 0x4b);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(g7, g14, g15, 0x21);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(g17, g19, g20, 0x69);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(x0, g16, g17, 0x94);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(x5, g17, g22, 0xac);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(g17, g21, g23, 0xae);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(g7, g15, g24, 0x96);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g14, m.o[0], 0x96);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g21, m.o[1], 0x69);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g25, m.o[2], 0x96);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g17, m.o[3], 0x69);
}

template <>
__device__ __forceinline__ void bs_box<2>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S3
    const uint32_t x0 = x[0] ^ m.e[0];
    const uint32_t x1 = x[1] ^ m.e[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5] ^ m.e[2];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x1, x4, x5, 0x96);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x0, x2, g6, 0x69);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x5, g6, g7, 0xc5);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x2, x4, g8, 0x87);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x1, g7, g9, 0xc6);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x3, x4, g9, 0x5a);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x4, g7, g11, 0x39);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x5, g11, g12, 0xc6);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x1, g12, g13, 0x9c);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x0, g9, g14, 0xf6);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(x3, g10, g15, 0x39);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(g11, g14, g15, 0x6d);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x5, g8, g17, 0x1d);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(x1, g7, g17, 0xd9);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(x0, g12, g19, 0x29);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(x3, g18, g20, 0x17);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(x2, g12, g21, 0x69);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(x5, g10, g13, 0xd9);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(x0, g12, g23, 0x9c);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(x4, g16, g21, 0x96);
    const uint32_t g26 = __builtin_amdgcn_bitop3_b32(x2, g24, g25, 0x6d);
    const uint32_t g27 = __builtin_amdgcn_bitop3_b32(g9, g19, g26, 0x8d);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g16, m.o[0], 0x96);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g22, m.o[1], 0x69);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g27, m.o[2], 0x96);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g24, m.o[3], 0x69);
}

template <>
__device__ __forceinline__ void bs_box<3>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S4
    const uint32_t x0 = x[0] ^ m.e[0];
    const uint32_t x1 = x[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x0, x2, x4, 0x1c);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x1, x3, g6, 0x14);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x2, x3, x4, 0x4a);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x1, g8, g6, 0x71);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x0, g8, g9, 0x96);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x4, g7, g10, 0xe9);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x1, x3, g10, 0xb1);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x5, g11, g12, 0x65);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x3, g11, g12, 0x69);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x2, g9, g14, 0xdb);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(g9, g7, g15, 0x29);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(g13, g15, g16, 0x96);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x5, g11, g17, 0x96);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(x1, g10, g14, 0x69);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(x5, g16, g19, 0x95);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(x5, g16, g19, 0x56);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g17, m.o[0], 0x69);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g18, m.o[1], 0x96);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g20, m.o[2], 0x69);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g21, m.o[3], 0x69);
}

template <>
__device__ __forceinline__ void bs_box<4>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S5
    const uint32_t x0 = x[0] ^ m.e[0];
    const uint32_t x1 = x[1] ^ m.e[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x2, x3, x5, 0xd6);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x2, x3, x4, 0x69);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x3, x5, g7, 0x56);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x0, x3, g8, 0xd6);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x4, g6, g9, 0x4d);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x4, g6, g8, 0x59);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x2, x5, g11, 0xb5);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x0, g8, g12, 0xc5);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x0, g11, g13, 0xe7);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x3, x4, g14, 0x25);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(x1, g13, g15, 0x63);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(g6, g12, g16, 0x84);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(g7, g10, g17, 0x4b);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(g9, g10, g15, 0x91);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(x5, g17, g19, 0x65);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(g12, g14, g20, 0xf2);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(g15, g18, g21, 0xb2);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(g10, g14, g22, 0x82);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(x3, g10, g18, 0xc6);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(g9, g15, g21, 0xe1);
    const uint32_t g26 = __builtin_amdgcn_bitop3_b32(x1, g24, g25, 0x59);
    const uint32_t g27 = __builtin_amdgcn_bitop3_b32(g13, g17, g26, 0xe1);
    const uint32_t g28 = __builtin_amdgcn_bitop3_b32(x0, x3, g22, 0xed);
    const uint32_t g29 = __builtin_amdgcn_bitop3_b32(x1, g20, g28, 0x6c);
    const uint32_t g30 = __builtin_amdgcn_bitop3_b32(g23, g27, g29, 0x39);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g30, m.o[0], 0x96);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g29, m.o[1], 0x96);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g16, m.o[2], 0x96);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g26, m.o[3], 0x96);
}

template <>
__device__ __forceinline__ void bs_box<5>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S6
    const uint32_t x0 = x[0] ^ m.e[0];
    const uint32_t x1 = x[1] ^ m.e[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x1, x2, x4, 0x85);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x0, x3, x5, 0x96);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x1, x3, g7, 0xa5);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x5, g7, g8, 0x16);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x0, g7, g9, 0x51);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x2, x4, g10, 0x4b);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x0, x1, g9, 0x9b);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x2, g11, g12, 0x87);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x3, x4, g13, 0x7c);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(g6, g8, g14, 0x6c);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(x0, g8, g14, 0x6f);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(x1, x4, g16, 0xad);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x4, g15, g17, 0x47);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(g8, g10, g11, 0x76);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(g15, g18, g19, 0x74);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(x2, g12, g16, 0x1c);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(g13, g14, g21, 0x16);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(x2, x3, g19, 0x7c);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(x1, g14, g23, 0x39);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(g15, g22, g24, 0xc3);
    const uint32_t g26 = __builtin_amdgcn_bitop3_b32(g8, g11, g17, 0x87);
    const uint32_t g27 = __builtin_amdgcn_bitop3_b32(g8, g18, g23, 0x4b);
    const uint32_t g28 = __builtin_amdgcn_bitop3_b32(x0, g27, g24, 0xca);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g20, m.o[0], 0x69);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g25, m.o[1], 0x96);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g26, m.o[2], 0x96);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g28, m.o[3], 0x69);
}

template <>
__device__ __forceinline__ void bs_box<6>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S7
    const uint32_t x0 = x[0] ^ m.e[0];
    const uint32_t x1 = x[1] ^ m.e[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x1, x3, x4, 0xb4);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x0, x3, x4, 0x96);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x2, g6, g7, 0x1e);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(g6, g7, g8, 0x3a);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x0, x1, g6, 0xe4);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(g8, g9, g10, 0x4e);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x5, g9, g11, 0x5c);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x3, x5, g11, 0x1f);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x0, g12, g13, 0x91);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x0, g7, g14, 0xae);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(x0, x1, g15, 0x71);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(x0, g9, g14, 0x37);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x5, g16, g17, 0x9e);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(x1, x5, g18, 0x53);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(x0, x2, x3, 0x79);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(x5, g17, g20, 0x7a);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(x1, g15, g21, 0x93);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(x3, g7, g22, 0x16);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(g8, g14, g23, 0xc9);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(g11, g19, g24, 0x69);
    const uint32_t g26 = __builtin_amdgcn_bitop3_b32(g18, g22, g25, 0x87);
    const uint32_t g27 = __builtin_amdgcn_bitop3_b32(x3, g23, g25, 0x64);
    const uint32_t g28 = __builtin_amdgcn_bitop3_b32(g11, g26, g27, 0xa6);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g25, m.o[0], 0x96);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g22, m.o[1], 0x96);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g28, m.o[2], 0x69);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g12, m.o[3], 0x96);
}

template <>
__device__ __forceinline__ void bs_box<7>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S8
    const uint32_t x0 = x[0] ^ m.e[0];
    const uint32_t x1 = x[1] ^ m.e[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4] ^ m.e[2];
    const uint32_t x5 = x[5] ^ m.e[3];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x0, x1, x4, 0x9a);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x1, x3, g6, 0x1e);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x2, x3, x4, 0x72);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x0, g6, g8, 0x7c);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x1, g6, g8, 0x34);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x0, g6, g10, 0xca);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x2, x3, g11, 0x69);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(g7, g9, g12, 0x6a);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x5, g6, g13, 0xe9);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x0, g8, g14, 0x93);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(x1, g8, g14, 0x49);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(g12, g15, g16, 0x6d);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x5, g13, g17, 0x36);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(x2, g7, g11, 0x65);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(x0, g8, g13, 0x18);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(x1, g10, g12, 0x83);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(x5, g13, g19, 0xac);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(g20, g21, g22, 0xa3);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(x2, g15, g21, 0x76);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(g12, g23, g24, 0xe7);
    const uint32_t g26 = __builtin_amdgcn_bitop3_b32(x5, g19, g25, 0x96);
    const uint32_t g27 = __builtin_amdgcn_bitop3_b32(x3, g20, g26, 0x42);
    const uint32_t g28 = __builtin_amdgcn_bitop3_b32(x1, g15, g27, 0x63);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g18, m.o[0], 0x96);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g26, m.o[1], 0x96);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g28, m.o[2], 0x96);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g22, m.o[3], 0x96);
}
