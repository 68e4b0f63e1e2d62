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
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x0, x2, x3, 0x96);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x2, x5, g6, 0x46);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x4, g6, g7, 0x1a);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x3, g6, g8, 0xab);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x0, x3, x4, 0x43);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x5, g9, g10, 0xdc);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x2, x3, g11, 0x40);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x1, g10, g12, 0x2f);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x3, g11, g13, 0x48);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(g8, g9, g14, 0x79);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(x1, g8, g10, 0xc9);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(x4, g6, g15, 0x2c);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x2, x5, g17, 0x6a);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(g12, g16, g18, 0x3e);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(g9, g15, g19, 0x38);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(g13, g16, g17, 0x38);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(g7, g19, g21, 0x49);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(g8, g13, g18, 0xc6);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(g11, g19, g23, 0x89);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(x4, g14, g24, 0xa7);
    const uint32_t g26 = __builtin_amdgcn_bitop3_b32(g8, g14, g25, 0x8f);
    const uint32_t g27 = __builtin_amdgcn_bitop3_b32(g22, g23, g25, 0xc7);
    const uint32_t g28 = __builtin_amdgcn_bitop3_b32(x1, g26, g27, 0x69);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g20, m.o[0], 0x69);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g22, m.o[1], 0x69);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g24, m.o[2], 0x69);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g28, m.o[3], 0x96);
}

template <>
__device__ __forceinline__ void bs_box<1>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S2
    const uint32_t x0 = x[0];
    const uint32_t x1 = x[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x0, x5, m.e[0], 0x69);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x1, x4, g6, 0x7c);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x4, x5, g7, 0xd2);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x1, g6, g8, 0x76);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x2, x3, g8, 0x1b);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x5, g7, g10, 0x7b);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x2, g9, g11, 0x78);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x1, x4, g10, 0x69);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x3, g12, g13, 0x96);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x5, g6, g14, 0x8c);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(x1, g7, g15, 0x2d);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(g13, g15, g16, 0xc3);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x5, g14, g16, 0x5e);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(g10, g15, g18, 0x69);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(g17, g16, g19, 0x36);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(g6, g14, g20, 0x24);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(x5, g17, g21, 0x93);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(x5, g15, g22, 0x2f);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(g14, g20, g23, 0x69);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g14, m.o[0], 0x96);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g22, m.o[1], 0x96);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g24, m.o[2], 0x96);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g19, m.o[3], 0x69);
}

template <>
__device__ __forceinline__ void bs_box<2>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S3
    const uint32_t x0 = x[0] ^ m.e[0];
    const uint32_t x1 = x[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5] ^ m.e[2];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x3, x4, x5, 0x96);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x1, x1, m.e[1], 0xa5);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x0, x2, g7, 0x89);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x3, x4, g7, 0x95);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x2, x4, g9, 0x59);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x0, g6, g10, 0x69);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x3, x4, g11, 0x4e);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(g6, g8, g12, 0xb3);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x2, g11, g13, 0x38);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x0, x5, g14, 0xf6);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(g10, g11, g15, 0x1e);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(g13, g14, g16, 0x61);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x5, g15, g16, 0x60);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(x3, g14, g18, 0x9c);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(g6, g8, g16, 0xe2);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(x2, x3, g16, 0xd8);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(g6, g9, g21, 0x46);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(g19, g20, g22, 0x93);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(x5, g12, g23, 0x87);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(g14, g20, g24, 0x76);
    const uint32_t g26 = __builtin_amdgcn_bitop3_b32(x0, g11, g25, 0x9c);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g17, m.o[0], 0x96);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g19, m.o[1], 0x96);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g23, m.o[2], 0x69);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g26, m.o[3], 0x96);
}

template <>
__device__ __forceinline__ void bs_box<3>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S4
    const uint32_t x0 = x[0];
    const uint32_t x1 = x[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x0, x2, m.e[0], 0x69);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x4, x5, g6, 0x96);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x2, x4, x2, 0xc3);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x1, g6, g8, 0x24);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x2, x3, x4, 0x99);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x1, g8, g10, 0xd2);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(g6, g10, g11, 0xf6);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x3, g9, g12, 0x6c);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(g6, g8, g10, 0x2c);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(g11, g13, g14, 0xb4);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(g7, g13, g15, 0xc9);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(x5, g16, g15, 0x69);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(g7, g12, g14, 0x62);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(g12, g17, g18, 0x63);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(g14, g16, g18, 0x69);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g16, m.o[0], 0x96);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g17, m.o[1], 0x96);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g19, m.o[2], 0x69);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g20, m.o[3], 0x69);
}

template <>
__device__ __forceinline__ void bs_box<4>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S5
    const uint32_t x0 = x[0];
    const uint32_t x1 = x[1] ^ m.e[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x0, x0, m.e[0], 0xa5);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x2, x3, g6, 0x4b);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x3, x5, g7, 0xc2);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x2, x4, g8, 0x28);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x2, x4, g7, 0x62);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x2, x5, g6, 0x6b);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(g9, g10, g11, 0xa9);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x2, x5, g12, 0x2e);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x1, x4, g6, 0x96);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(g11, g13, g14, 0xa3);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(g15, g10, x3, 0xd8);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(x3, g11, g14, 0x4e);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(g7, g13, g14, 0xc4);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(x1, g8, g16, 0x69);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(x4, g9, g19, 0xf6);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(g17, g18, g20, 0xac);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(g13, g16, g21, 0x96);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(x3, g10, g20, 0x29);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(x1, g12, g23, 0x63);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(g14, g21, g24, 0x62);
    const uint32_t g26 = __builtin_amdgcn_bitop3_b32(g13, g14, g22, 0x0e);
    const uint32_t g27 = __builtin_amdgcn_bitop3_b32(g8, g25, g26, 0x96);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g22, m.o[0], 0x69);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g19, m.o[1], 0x69);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g27, m.o[2], 0x69);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g24, m.o[3], 0x96);
}

template <>
__device__ __forceinline__ void bs_box<5>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S6
    const uint32_t x0 = x[0];
    const uint32_t x1 = x[1] ^ m.e[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x0, x1, m.e[0], 0x96);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x5, x1, g6, 0x8d);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x4, g6, g7, 0x61);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x2, x1, g8, 0x7c);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x4, g6, g9, 0x19);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x4, g7, g9, 0x07);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x1, g10, g11, 0x97);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x3, g7, g12, 0x2d);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x5, g12, g13, 0x59);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x5, g6, g8, 0x35);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(x4, g14, g15, 0x1c);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(x2, g15, g16, 0x17);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(x2, x5, g16, 0x69);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(x1, g17, g18, 0x38);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(g8, g14, g19, 0xc9);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(x3, x5, g20, 0xd3);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(g10, g11, g21, 0xb4);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(g15, g21, g22, 0x96);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(g20, g22, g23, 0xba);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(g13, g14, g24, 0x57);
    const uint32_t g26 = __builtin_amdgcn_bitop3_b32(x1, g18, g25, 0x69);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g20, m.o[0], 0x69);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g26, m.o[1], 0x69);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g18, m.o[2], 0x69);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g23, m.o[3], 0x69);
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
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x1, x3, x5, 0x93);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x1, x5, g6, 0xa9);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x2, x3, g6, 0x68);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x1, x3, x4, 0xb4);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x2, x3, g9, 0xb7);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(g7, g8, g10, 0x78);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(g7, g8, g9, 0xe1);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x2, x5, g12, 0x3b);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(x0, g9, g13, 0xbf);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x0, x2, x5, 0x96);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(g6, g11, g15, 0xd1);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(x0, g12, g16, 0x69);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(g6, g11, g17, 0x78);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(g14, g17, g18, 0x59);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(g13, g10, g19, 0x09);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(x1, x4, g16, 0x69);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(x0, g21, g18, 0x4c);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(g11, g20, g22, 0x69);
    const uint32_t g24 = __builtin_amdgcn_bitop3_b32(g13, g19, g23, 0x9c);
    const uint32_t g25 = __builtin_amdgcn_bitop3_b32(g17, g21, g14, 0x2d);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g23, m.o[0], 0x69);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g21, m.o[1], 0x69);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g24, m.o[2], 0x96);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g25, m.o[3], 0x69);
}

template <>
__device__ __forceinline__ void bs_box<7>(const uint32_t *x, uint32_t *d,
                                           const BsBoxMasks &m) {  // S8
    const uint32_t x0 = x[0] ^ m.e[0];
    const uint32_t x1 = x[1] ^ m.e[1];
    const uint32_t x2 = x[2];
    const uint32_t x3 = x[3];
    const uint32_t x4 = x[4];
    const uint32_t x5 = x[5] ^ m.e[3];
    const uint32_t g6 = __builtin_amdgcn_bitop3_b32(x4, x1, m.e[2], 0x96);
    const uint32_t g7 = __builtin_amdgcn_bitop3_b32(x0, x1, g6, 0x9a);
    const uint32_t g8 = __builtin_amdgcn_bitop3_b32(x0, x1, x5, 0x9c);
    const uint32_t g9 = __builtin_amdgcn_bitop3_b32(x3, g7, g8, 0x19);
    const uint32_t g10 = __builtin_amdgcn_bitop3_b32(x0, x2, g9, 0xc9);
    const uint32_t g11 = __builtin_amdgcn_bitop3_b32(x3, g7, g10, 0x87);
    const uint32_t g12 = __builtin_amdgcn_bitop3_b32(x1, x5, g11, 0x69);
    const uint32_t g13 = __builtin_amdgcn_bitop3_b32(x1, g8, g9, 0xcb);
    const uint32_t g14 = __builtin_amdgcn_bitop3_b32(g6, g10, g11, 0x63);
    const uint32_t g15 = __builtin_amdgcn_bitop3_b32(x0, g12, g14, 0x7d);
    const uint32_t g16 = __builtin_amdgcn_bitop3_b32(x5, g12, g15, 0x93);
    const uint32_t g17 = __builtin_amdgcn_bitop3_b32(x1, g14, g16, 0x5c);
    const uint32_t g18 = __builtin_amdgcn_bitop3_b32(g7, g13, g17, 0x69);
    const uint32_t g19 = __builtin_amdgcn_bitop3_b32(g8, g16, g18, 0xd2);
    const uint32_t g20 = __builtin_amdgcn_bitop3_b32(x5, g14, g19, 0xc6);
    const uint32_t g21 = __builtin_amdgcn_bitop3_b32(g12, g13, g20, 0x4b);
    const uint32_t g22 = __builtin_amdgcn_bitop3_b32(g12, g13, g20, 0x2e);
    const uint32_t g23 = __builtin_amdgcn_bitop3_b32(g20, g16, g19, 0x69);
    d[0] = __builtin_amdgcn_bitop3_b32(d[0], g21, m.o[0], 0x96);
    d[1] = __builtin_amdgcn_bitop3_b32(d[1], g22, m.o[1], 0x96);
    d[2] = __builtin_amdgcn_bitop3_b32(d[2], g18, m.o[2], 0x69);
    d[3] = __builtin_amdgcn_bitop3_b32(d[3], g23, m.o[3], 0x96);
}
