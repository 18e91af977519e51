// wide.h -- scan of partitioned events, a bucket's ids in LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace vc {

// The events of bucket b (ids with id >> bits == b) lie at part[base[b], base[b + 1]) in
// their order; a chunk is at most `per` events of one bucket.  The bases and the chunks
// come from the buckets' counts (tot, nb <= 1024): cbase[b] is bucket b's first chunk (nb +
// 1 entries), cb[c] chunk c's bucket, marked when it is the bucket's first
// (wide_max_chunks entries).
struct WideChunks {
    const uint32_t *part;
    const uint32_t *tot;
    uint64_t *base;
    uint32_t *cbase, *cb;
    uint32_t nb, n_ids, bits;
    uint64_t n, per;
};
// events per chunk and the most chunks n events can need
uint64_t wide_chunk_events(uint64_t n, uint32_t row);
uint32_t wide_max_chunks(uint64_t n, uint32_t nb, uint64_t per);
void launch_wide_bases(const WideChunks &W, hipStream_t s);

// rows of the scans: words per chunk, and the scratch of `max_chunks` of them
uint32_t wide_row_events(uint32_t bits);
uint32_t wide_row_spaces(uint32_t bits);
size_t wide_rows_bytes(uint32_t max_chunks, uint32_t row);

// event words: the status byte of every word at its place, final statuses of the buckets
// with events
void launch_wide_scan_events(const WideChunks &W, const uint8_t *init, uint8_t *final_out, void *rows, uint8_t *res,
                             Control *ctl, hipStream_t s);
// k-space words: the uint16 status of every word at its place, final statuses of the
// buckets with events
void launch_wide_scan_spaces(const WideChunks &W, const uint8_t *init, uint8_t *final_out, void *rows, uint16_t *res,
                             Control *ctl, hipStream_t s);

} // namespace vc
