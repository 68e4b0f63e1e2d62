// Generated by paper_2007_10752_amd/gen/emit.py from the DES tables of the
// paper's Appendix A and the verified S-box networks.  Do not edit.
#pragma once
#include <stdint.h>

// Initial permutation as renaming: L[i] / R[i] read plane BS_IP_L[i] / BS_IP_R[i]
static constexpr int BS_IP_L[32] = {
    62, 54, 46, 38, 30, 22, 14, 6, 60, 52, 44, 36, 28, 20, 12, 4,
    58, 50, 42, 34, 26, 18, 10, 2, 56, 48, 40, 32, 24, 16, 8, 0,
};
static constexpr int BS_IP_R[32] = {
    63, 55, 47, 39, 31, 23, 15, 7, 61, 53, 45, 37, 29, 21, 13, 5,
    59, 51, 43, 35, 27, 19, 11, 3, 57, 49, 41, 33, 25, 17, 9, 1,
};
// Final permutation as renaming: output plane q is preoutput bit BS_FP_SRC[q]
// (preoutput = R16 || L16: 0..31 from R16, 32..63 from L16)
static constexpr int BS_FP_SRC[64] = {
    31, 63, 23, 55, 15, 47, 7, 39, 30, 62, 22, 54, 14, 46, 6, 38,
    29, 61, 21, 53, 13, 45, 5, 37, 28, 60, 20, 52, 12, 44, 4, 36,
    27, 59, 19, 51, 11, 43, 3, 35, 26, 58, 18, 50, 10, 42, 2, 34,
    25, 57, 17, 49, 9, 41, 1, 33, 24, 56, 16, 48, 8, 40, 0, 32,
};

// S-box gate counts: S1=23, S2=19, S3=21, S4=15, S5=22, S6=21, S7=20, S8=18 (total 159 per round)
#define BS_SBOX_GATES_PER_ROUND 159
// XORs per round: 32 of S-box outputs into the other half, and the second
// uses whose masks are not folded into the gates (6 of 16 are)
#define BS_XORS_PER_ROUND 42


// Number of second-use inputs of each S-box (mask words e[] it reads).
static constexpr int BS_BOX_NDUP[8] = {
    1, 1, 3, 1, 2, 2, 2, 4,
};

// Key masks of one S-box in registers: o[q] is folded into the XOR of output q
// into the other half, e[i] is the mask of the box's i-th second-use input.
struct BsBoxMasks {
    uint32_t o[4], e[4];
};

// One Feistel round on 32 blocks per lane (Sec. III-B): d ^= P(S(E(r) ^ K)).
// The halves are stored XORed with key masks: each word of r already carries the
// round-key bit of its primary expansion position, so only second uses need their
// mask: XORed in, or taken as the third operand of the gates that read the input;
// the output masks re-mask the updated words of d for their next use.  Masks are
// laid out by round and S-box (8 words per box, 64 per round: o[0..3], e[0..3])
// and software-pipelined D boxes ahead: before box j
// runs, load(pm[(j + D) % 8], q, n) requests the masks of the box D places
// later, q = p + 8 * (j + D), or past the last box pn + 8 * (j + D - 8) (pn: the
// next round's masks).
// A scheduling barrier between boxes keeps each request and each box's
// arithmetic in place, so the request's latency overlaps D boxes of work.
// On entry pm[0..D-1] hold this round's first D boxes; on exit the next round's.
// n = BS_BOX_NDUP of the requested box: load fills o[0..3] and e[0..n-1] only.
// P: the pointer type of p and pn (a generic or an LDS pointer).
template <int D, class LOAD, class P>
__device__ __forceinline__ void bs_round_piped(uint32_t (&d)[32], const uint32_t (&r)[32],
                                               P p, P pn, BsBoxMasks (&pm)[8],
                                               const LOAD &load) {
    static_assert(D >= 1 && D <= 7, "pipeline depth");
    {  // S1
        __builtin_amdgcn_sched_barrier(0);
        load(pm[(0 + D) % 8],
             0 + D < 8 ? p + 8 * (0 + D) : pn + 8 * (0 + D - 8),
             BS_BOX_NDUP[(0 + D) % 8]);
        const BsBoxMasks &m = pm[0];
        const uint32_t x0 = r[31];
        const uint32_t x1 = r[0];
        const uint32_t x2 = r[1];
        const uint32_t x3 = r[2];
        const uint32_t x4 = r[3];
        const uint32_t x5 = r[4] ^ m.e[0];
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
        d[8] = __builtin_amdgcn_bitop3_b32(d[8], g20, m.o[0], 0x69);
        d[16] = __builtin_amdgcn_bitop3_b32(d[16], g22, m.o[1], 0x69);
        d[22] = __builtin_amdgcn_bitop3_b32(d[22], g24, m.o[2], 0x69);
        d[30] = __builtin_amdgcn_bitop3_b32(d[30], g28, m.o[3], 0x96);
    }
    {  // S2
        __builtin_amdgcn_sched_barrier(0);
        load(pm[(1 + D) % 8],
             1 + D < 8 ? p + 8 * (1 + D) : pn + 8 * (1 + D - 8),
             BS_BOX_NDUP[(1 + D) % 8]);
        const BsBoxMasks &m = pm[1];
        const uint32_t x0 = r[3];  // mask folded into its gates
        const uint32_t x1 = r[4];
        const uint32_t x2 = r[5];
        const uint32_t x3 = r[6];
        const uint32_t x4 = r[7];
        const uint32_t x5 = r[8];
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
        d[12] = __builtin_amdgcn_bitop3_b32(d[12], g14, m.o[0], 0x96);
        d[27] = __builtin_amdgcn_bitop3_b32(d[27], g22, m.o[1], 0x96);
        d[1] = __builtin_amdgcn_bitop3_b32(d[1], g24, m.o[2], 0x96);
        d[17] = __builtin_amdgcn_bitop3_b32(d[17], g19, m.o[3], 0x69);
    }
    {  // S3
        __builtin_amdgcn_sched_barrier(0);
        load(pm[(2 + D) % 8],
             2 + D < 8 ? p + 8 * (2 + D) : pn + 8 * (2 + D - 8),
             BS_BOX_NDUP[(2 + D) % 8]);
        const BsBoxMasks &m = pm[2];
        const uint32_t x0 = r[7] ^ m.e[0];
        const uint32_t x1 = r[8];  // mask folded into its gates
        const uint32_t x2 = r[9];
        const uint32_t x3 = r[10];
        const uint32_t x4 = r[11];
        const uint32_t x5 = r[12] ^ m.e[2];
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
        d[23] = __builtin_amdgcn_bitop3_b32(d[23], g17, m.o[0], 0x96);
        d[15] = __builtin_amdgcn_bitop3_b32(d[15], g19, m.o[1], 0x96);
        d[29] = __builtin_amdgcn_bitop3_b32(d[29], g23, m.o[2], 0x69);
        d[5] = __builtin_amdgcn_bitop3_b32(d[5], g26, m.o[3], 0x96);
    }
    {  // S4
        __builtin_amdgcn_sched_barrier(0);
        load(pm[(3 + D) % 8],
             3 + D < 8 ? p + 8 * (3 + D) : pn + 8 * (3 + D - 8),
             BS_BOX_NDUP[(3 + D) % 8]);
        const BsBoxMasks &m = pm[3];
        const uint32_t x0 = r[11];  // mask folded into its gates
        const uint32_t x1 = r[12];
        const uint32_t x2 = r[13];
        const uint32_t x3 = r[14];
        const uint32_t x4 = r[15];
        const uint32_t x5 = r[16];
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
        d[25] = __builtin_amdgcn_bitop3_b32(d[25], g16, m.o[0], 0x96);
        d[19] = __builtin_amdgcn_bitop3_b32(d[19], g17, m.o[1], 0x96);
        d[9] = __builtin_amdgcn_bitop3_b32(d[9], g19, m.o[2], 0x69);
        d[0] = __builtin_amdgcn_bitop3_b32(d[0], g20, m.o[3], 0x69);
    }
    {  // S5
        __builtin_amdgcn_sched_barrier(0);
        load(pm[(4 + D) % 8],
             4 + D < 8 ? p + 8 * (4 + D) : pn + 8 * (4 + D - 8),
             BS_BOX_NDUP[(4 + D) % 8]);
        const BsBoxMasks &m = pm[4];
        const uint32_t x0 = r[15];  // mask folded into its gates
        const uint32_t x1 = r[16] ^ m.e[1];
        const uint32_t x2 = r[17];
        const uint32_t x3 = r[18];
        const uint32_t x4 = r[19];
        const uint32_t x5 = r[20];
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
        d[7] = __builtin_amdgcn_bitop3_b32(d[7], g22, m.o[0], 0x69);
        d[13] = __builtin_amdgcn_bitop3_b32(d[13], g19, m.o[1], 0x69);
        d[24] = __builtin_amdgcn_bitop3_b32(d[24], g27, m.o[2], 0x69);
        d[2] = __builtin_amdgcn_bitop3_b32(d[2], g24, m.o[3], 0x96);
    }
    {  // S6
        __builtin_amdgcn_sched_barrier(0);
        load(pm[(5 + D) % 8],
             5 + D < 8 ? p + 8 * (5 + D) : pn + 8 * (5 + D - 8),
             BS_BOX_NDUP[(5 + D) % 8]);
        const BsBoxMasks &m = pm[5];
        const uint32_t x0 = r[19];  // mask folded into its gates
        const uint32_t x1 = r[20] ^ m.e[1];
        const uint32_t x2 = r[21];
        const uint32_t x3 = r[22];
        const uint32_t x4 = r[23];
        const uint32_t x5 = r[24];
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
        d[3] = __builtin_amdgcn_bitop3_b32(d[3], g20, m.o[0], 0x69);
        d[28] = __builtin_amdgcn_bitop3_b32(d[28], g26, m.o[1], 0x69);
        d[10] = __builtin_amdgcn_bitop3_b32(d[10], g18, m.o[2], 0x69);
        d[18] = __builtin_amdgcn_bitop3_b32(d[18], g23, m.o[3], 0x69);
    }
    {  // S7
        __builtin_amdgcn_sched_barrier(0);
        load(pm[(6 + D) % 8],
             6 + D < 8 ? p + 8 * (6 + D) : pn + 8 * (6 + D - 8),
             BS_BOX_NDUP[(6 + D) % 8]);
        const BsBoxMasks &m = pm[6];
        const uint32_t x0 = r[23] ^ m.e[0];
        const uint32_t x1 = r[24] ^ m.e[1];
        const uint32_t x2 = r[25];
        const uint32_t x3 = r[26];
        const uint32_t x4 = r[27];
        const uint32_t x5 = r[28];
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
        d[31] = __builtin_amdgcn_bitop3_b32(d[31], g23, m.o[0], 0x69);
        d[11] = __builtin_amdgcn_bitop3_b32(d[11], g21, m.o[1], 0x69);
        d[21] = __builtin_amdgcn_bitop3_b32(d[21], g24, m.o[2], 0x96);
        d[6] = __builtin_amdgcn_bitop3_b32(d[6], g25, m.o[3], 0x69);
    }
    {  // S8
        __builtin_amdgcn_sched_barrier(0);
        load(pm[(7 + D) % 8],
             7 + D < 8 ? p + 8 * (7 + D) : pn + 8 * (7 + D - 8),
             BS_BOX_NDUP[(7 + D) % 8]);
        const BsBoxMasks &m = pm[7];
        const uint32_t x0 = r[27] ^ m.e[0];
        const uint32_t x1 = r[28] ^ m.e[1];
        const uint32_t x2 = r[29];
        const uint32_t x3 = r[30];
        const uint32_t x4 = r[31];  // mask folded into its gates
        const uint32_t x5 = r[0] ^ m.e[3];
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
        d[4] = __builtin_amdgcn_bitop3_b32(d[4], g21, m.o[0], 0x96);
        d[26] = __builtin_amdgcn_bitop3_b32(d[26], g22, m.o[1], 0x96);
        d[14] = __builtin_amdgcn_bitop3_b32(d[14], g18, m.o[2], 0x69);
        d[20] = __builtin_amdgcn_bitop3_b32(d[20], g23, m.o[3], 0x96);
    }
}
