// dense.h -- host interface of the dense check: the statuses of a whole id space in LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace vc {

// largest id space whose table (3 bits an id, 8 ids a word) a wave holds in LDS: 32 KiB
constexpr uint32_t DENSE_MAX_IDS = 1u << 16;

size_t dense_scratch_bytes(uint64_t n, uint32_t n_ids);

// plain check of n events over n_ids <= DENSE_MAX_IDS ids: status bytes, final table (all
// of it), violations (count into ctl->n_viol).  Resets ctl first.
void launch_dense_check(const uint32_t *events, uint64_t n, uint32_t n_ids, const uint8_t *init, uint8_t *status,
                        uint8_t *final_out, uint32_t *viol, void *scratch, Control *ctl, hipStream_t s);

// A combined stream as 32-bit words (an event's, then its induced items', op 5; probes,
// which change nothing, DENSE_OP_PROBE), by tiles of `tile` events: tile t's words start at
// tpos[t] (device, tiles + 1 entries), m words in all.  The fold resets ctl and reports
// malformed words; then, with probes, the statuses the probes see from `init` (pre, m
// bytes, at their positions); then, from another `init`, the events' status bytes in
// their order, all final statuses and the number of flagged induced items
// (ctl->n_induced_stuck).
constexpr uint32_t DENSE_OP_PROBE = 6;
struct DenseWords {
    const uint32_t *words;
    uint64_t m;
    const uint64_t *tpos;
    uint64_t tiles;
    uint32_t n_ids;
};
size_t dense_words_scratch_bytes(uint64_t tiles, uint32_t n_ids, bool probes);
void launch_dense_words_fold(const DenseWords &W, bool probes, void *scratch, Control *ctl, hipStream_t s);
void launch_dense_words_probe(const DenseWords &W, const uint8_t *init, uint8_t *pre, void *scratch, hipStream_t s);
void launch_dense_words_apply(const DenseWords &W, bool probes, const uint8_t *init, uint64_t n, uint32_t tile,
                              uint8_t *status, uint8_t *final_out, void *scratch, Control *ctl, hipStream_t s);

} // namespace vc
