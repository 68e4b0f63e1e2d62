// Host check of the key expansion that the GPU runs (keysched_device.h): round keys
// from the transposed key and fields, the schedules' words lane by lane, and the
// table kernel's keys, each against the sequential schedule of keysched_core.h.
// Built and run by test_keysched_device.py.
#include <cstdint>
#include <cstdio>

#include "keysched_device.h"

using namespace tdes;

int main() {
    uint64_t state = 0x3DE5DE71ull;
    auto next_byte = [&]() {
        state = state * 6364136223846793005ull + 1442695040888963407ull;
        return (uint8_t)(state >> 56);
    };
    int bad = 0, n = 0;
    // all zeros, all ones, every single key bit, then random bundles
    for (int trial = 0; trial < 2 + 192 + 2000; trial++, n++) {
        alignas(8) uint8_t key24[24];
        for (int i = 0; i < 24; i++)
            key24[i] = trial == 1 ? 0xFF : trial < 2 ? 0 : trial < 194 ? 0 : next_byte();
        if (trial >= 2 && trial < 194) key24[(trial - 2) / 8] = (uint8_t)(1u << (trial - 2) % 8);
        uint64_t k[3][16];
        for (int b = 0; b < 3; b++) des_round_keys(key24 + 8 * b, k[b]);
        uint32_t primary[48], out[48], dup[48];
        for (int slot = 0; slot < 48; slot++) {
            const uint64_t key = load_key(key24 + 8 * (slot / 16), true);
            bad += key != load_key(key24 + 8 * (slot / 16), false);
            const RoundMasks m = round_masks(key, slot % 16);
            primary[slot] = m.primary;
            out[slot] = m.out;
            dup[slot] = m.dup;
            const SpboxRound got = table_round_keys(key, slot % 16);
            const SpboxRound want = spbox_round_keys(k[slot / 16][slot % 16]);
            for (int i = 0; i < 4; i++) bad += got.w[i] != want.w[i];
        }
        for (int dir = 0; dir < 2; dir++) {
            uint32_t want[kDirWords];
            bitslice_mask_words(k, dir, want);
            for (int t = 0; t < kDirWords / 2; t++) {
                const WordPair w = schedule_words(primary, out, dup, dir, t);
                bad += (w.x != want[2 * t]) + (w.y != want[2 * t + 1]);
            }
        }
    }
    printf("%s %d bundles\n", bad ? "FAIL" : "ok", n);
    return bad ? 1 : 0;
}
