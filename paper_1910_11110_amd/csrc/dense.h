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

} // namespace vc
