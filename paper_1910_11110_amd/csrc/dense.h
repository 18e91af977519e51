// dense.h -- host interface of the dense check: the statuses of a whole id space in LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace vc {

// largest id space whose table (3 bits an id, 8 ids a word) a wave holds in LDS: 32 KiB
constexpr uint32_t DENSE_MAX_IDS = 1u << 16;

// Events from which on chunks over many ids are folded forwards, by a launch of their own
// that leaves those of skewed ids to the backward fold: 2^22 events x 2^16 ids 24.4 us by the
// fold alone and 26.7 + 7.6 by both (whole check 80 and 79), 2^24 67 and 48 + 6, 2^26 231 and
// 161 + 6; 2^24 of Zipf(1.1) ids 111 and 7 + 89.
constexpr uint64_t DENSE_FORWARD_FROM = 1ull << 22;

size_t dense_scratch_bytes(uint64_t n, uint32_t n_ids);

// plain check of n events over n_ids <= DENSE_MAX_IDS ids: status bytes, final table (all
// of it), violations (count into ctl->n_viol).  Resets ctl first.
void launch_dense_check(const uint32_t *events, uint64_t n, uint32_t n_ids, const uint8_t *init, uint8_t *status,
                        uint8_t *final_out, uint32_t *viol, void *scratch, Control *ctl, hipStream_t s);

// A combined stream as 32-bit words (an event's, then its induced items', op 5; probes,
// which change nothing, DENSE_OP_PROBE), by tiles of `tile` events: tile t's words start at
// tpos[t] (device, tiles + 1 entries), m words in all.  Every chunk's functions first: by
// the fold, which resets ctl and reports malformed words, or (well-formed words only) with
// the functions that the probes see (pre, m bytes, at their positions: 3 bits, as in the
// table) and the statuses from `init` entering every chunk.  Then, from an `init` again, the
// events' status bytes in their order, all final statuses and the number of flagged induced
// items (ctl->n_induced_stuck).
constexpr uint32_t DENSE_OP_PROBE = 6;
struct DenseWords {
    const uint32_t *words;
    uint64_t m;
    const uint64_t *tpos;
    uint64_t tiles;
    uint32_t n_ids;
};
size_t dense_words_scratch_bytes(uint64_t tiles, uint32_t n_ids, bool probes);
void launch_dense_words_fold(const DenseWords &W, void *scratch, Control *ctl, hipStream_t s);
struct DenseEntering { // chunk c's statuses at rows[c * row], 8 ids a word; the words of tiles [c * per, ...)
    const uint32_t *rows;
    uint32_t row;
    uint64_t per;
};
DenseEntering launch_dense_words_probe(const DenseWords &W, const uint8_t *init, uint8_t *pre, void *scratch,
                                       Control *ctl, hipStream_t s);
void launch_dense_words_apply(const DenseWords &W, bool probes, const uint8_t *init, uint64_t n, uint32_t tile,
                              uint8_t *status, uint8_t *final_out, void *scratch, Control *ctl, hipStream_t s);

// initial statuses of the check of a dynamic trace from the functions that the probes see:
// a create's probe lies after it (pos32[create] + 1 of m words)
void launch_dyn_inherit_dense(const uint32_t *mother, const uint32_t *cpos, const uint8_t *pre, const uint32_t *pos32,
                              uint64_t n, uint64_t m, const DenseEntering &E, const uint8_t *init, uint32_t n_ids,
                              uint8_t *init2, hipStream_t s);

} // namespace vc
