// Generated by paper_2007_10752_amd/gen/emit.py from the DES tables of the
// paper's Appendix A and the verified S-box networks.  Do not edit.
#pragma once
#include <stdint.h>

// Expansion E (Appendix A): source word of each of the 48 S-box inputs,
// the primary input of each word, and the 16 second-use inputs in order.
static constexpr int kBsESrc[48] = {
    31, 0, 1, 2, 3, 4, 3, 4, 5, 6, 7, 8, 7, 8, 9, 10,
    11, 12, 11, 12, 13, 14, 15, 16, 15, 16, 17, 18, 19, 20, 19, 20,
    21, 22, 23, 24, 23, 24, 25, 26, 27, 28, 27, 28, 29, 30, 31, 0,
};
static constexpr int kBsPrimaryE[32] = {
    1, 2, 3, 4, 7, 8, 9, 10, 11, 14, 15, 16, 19, 20, 21, 22,
    23, 26, 27, 28, 29, 32, 33, 34, 35, 38, 39, 40, 41, 44, 45, 0,
};
static constexpr int kBsDupE[16] = {
    5, 6, 12, 13, 17, 18, 24, 25, 30, 31, 36, 37, 42, 43, 46, 47,
};
// Straight permutation P: half-word receiving S-box output 4*box+q.
static constexpr int kBsOutWord[32] = {
    8, 16, 22, 30, 12, 27, 1, 17, 23, 15, 29, 5, 25, 19, 9, 0,
    7, 13, 24, 2, 3, 28, 10, 18, 31, 11, 21, 6, 4, 26, 14, 20,
};
// Second-use index k of mask slot 4 + i of S-box j: kBsBoxDup[4*j + i] (-1: unused).
static constexpr int kBsBoxDup[32] = {
    0, -1, -1, -1, 1, -1, -1, -1, 2, 3, 4, -1, 5, -1, -1, -1,
    6, 7, -1, -1, 8, 9, -1, -1, 10, 11, -1, -1, 12, 13, 14, 15,
};

// Places of the masks widened from the key words, as a table: round t, box j at
// kBsRoundMasks*t + kBsBoxMasks*j (outputs 0..3, then second uses); then the four
// 32-word extra groups.  The kernels use a box's kBsBoxMasks places (a row of the
// batched kernel's table), the CPU emulation of the tests the whole.
enum { kBsBoxMasks = 8, kBsRoundMasks = 64, kBsInitY = 3072, kBsRemask16 = 3104,
       kBsRemask32 = 3136, kBsFinalX = 3168, kBsNumMasks = 3200 };
