// Host side of the key formats: round order per direction, bitsliced key
// masks (keysched_core.h) and the table kernel's key chunks.
#include <string.h>

#include "internal.h"

namespace tdes {

void round_sequence(const tdes_schedule &ks, int dir, RoundSequence *seq) {
    for (int t = 0; t < 48; t++) seq->rk[t] = round_key_at(ks.k, dir, t);
}

void bitslice_keys(const tdes_schedule &ks, int dir, BitsliceKeys *out) {
    bitslice_mask_words(ks.k, dir, out->w);
}

void device_schedule_words(const tdes_schedule &ks, uint32_t out[kDeviceScheduleWords]) {
    bitslice_mask_words(ks.k, 0, out);
    bitslice_mask_words(ks.k, 1, out + kDirWords);
}

void spbox_keys(const RoundSequence &seq, SpboxKeys *out) {
    for (int r = 0; r < 48; r++) {
        const SpboxRound k = spbox_round_keys(seq.rk[r]);
        for (int i = 0; i < 4; i++) out->w[r][i] = k.w[i];
    }
}

}  // namespace tdes
