// batch.h -- descriptor of one trace inside a batched launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace vc {

struct TraceDesc {
    const uint32_t *events; // the trace's events (device)
    const uint8_t *init;    // initial statuses or null for (V,I)
    const uint64_t *off;    // overlap CSR offsets or null when the trace has no arrays
    const uint32_t *nbr;    // overlap CSR neighbours
    uint64_t n;             // events
    uint64_t ev_base;       // first global event index
    uint32_t n_ids;
    uint32_t key_base;      // first global key
    Control *ctl;           // the trace's counters (errors, violations, induced)
    uint8_t *status;        // the trace's result buffers
    uint8_t *fin;
    uint32_t *viol;
    uint64_t m;             // its combined items (events and induced items)
    uint64_t item_base;     // bucket route: first combined position (a multiple of 16)
    uint64_t first_chunk;   // index of its first chunk
    uint32_t key_local;     // bucket route: first key inside its group
    // dense route: words of its rows, where its rows and its groups' rows lie, its chunks
    uint32_t row;
    uint64_t row_base, grp_base, first_dense;
    uint32_t dense_chunks;
};

// a run of consecutive events of one trace: the unit of work of the relocation passes,
// one wave each (a chunk never straddles two traces).  At most BATCH_CHUNK events for a
// trace with arrays (its items are staged per event), BATCH_CHUNK_PLAIN otherwise.
constexpr uint32_t BATCH_CHUNK = 512;
constexpr uint32_t BATCH_CHUNK_PLAIN = 4096;
struct ChunkDesc {
    uint64_t start; // first event, trace-relative
    uint32_t trace;
    uint32_t len;
};
// per chunk: induced items its events add (chunks of traces without arrays add none)
void launch_batch_chunk_count(const TraceDesc *d, const ChunkDesc *ch, uint64_t n_chunks, uint32_t *chunk_cnt,
                              hipStream_t s);
// items of every chunk at its events' global indices shifted by the induced items of
// the chunks before it (chunk_pos) and of its own events before each one
void launch_batch_chunk_emit(const TraceDesc *d, const ChunkDesc *ch, uint64_t n_chunks, const uint64_t *chunk_pos,
                             uint64_t *items, uint64_t cap, hipStream_t s);

// bucket route: every chunk's items as 32-bit words (group-local keys, induced items op
// 5), each trace's at item_base on; an item past the trace's range is not written and
// reported, and slots of the range that no item reaches, and those after it up to the
// next multiple of 16 (below cap), get a no-op word; `plain`: the chunks of traces
// without arrays too
void launch_batch_chunk_words(const TraceDesc *d, const ChunkDesc *ch, uint64_t n_chunks, const uint64_t *chunk_pos,
                              uint32_t *words, uint64_t cap, bool plain, hipStream_t s);
// bucket route, after the bucket pass of one group (items [g_lo, g_lo + g_m), results
// res in the partitioned order through dstidx, or in combined order when dstidx is
// null), for the chunks [c_lo, c_hi) of its traces: every chunk's primaries' status
// bytes into its trace's status buffer, the number of them flagged into vcnt[chunk], and
// per trace the flagged induced items into ind
void launch_batch_chunk_status(const TraceDesc *d, const ChunkDesc *ch, uint64_t c_lo, uint64_t c_hi,
                               const uint64_t *chunk_pos, const uint8_t *res, const uint32_t *dstidx, uint64_t g_lo,
                               uint64_t g_m, uint32_t *vcnt, unsigned long long *ind, hipStream_t s);
// every chunk's flagged events into its trace's violation list (ascending, trace-relative),
// from vpos = the exclusive prefix of vcnt over the batch (dense: the dense route's chunks)
void launch_batch_chunk_viol(const TraceDesc *d, const ChunkDesc *ch, uint64_t n_chunks, const uint32_t *vcnt,
                             const uint64_t *vpos, bool dense, hipStream_t s);
// bucket route: every trace's final statuses and counts
void launch_batch_finish(const TraceDesc *d, uint32_t n_traces, uint64_t n_chunks, const uint64_t *vpos,
                         const uint8_t *fin_all, const Control *bctl, const unsigned long long *ind, hipStream_t s);

// dense route, the traces without arrays over at most small_max_ids() ids and with an event
// at least: checked by strands, a chunk (strand_chunk() events, a trace's last one the rest) a
// tile; flagged events per chunk into vcnt.  The final statuses stay in the last chunks'
// words of lbv (batch_strands_bytes(chunks)), STRAND_WORDS a chunk of STRAND_IDS ids each,
// for launch_batch_counts.
constexpr uint32_t STRAND_WORDS = 4, STRAND_IDS = 20;
uint32_t strand_chunk();
size_t batch_strands_bytes(uint64_t chunks);
void launch_batch_strands(const TraceDesc *d, const ChunkDesc *ch, uint32_t chunks, uint32_t *vcnt, uint64_t *lbv,
                          uint32_t *ticket, hipStream_t s);
// dense route, the others (every trace over at most DENSE_CLASS[last] * 8 ids): the chunks of all
// traces by classes of row sizes, a trace's consecutive; the groups of B_GROUP chunks of
// every trace, BLOCK words of their rows a job
constexpr uint32_t B_GROUP = 32;
struct PrefixJob {
    uint32_t trace, group, word;
};
constexpr int DENSE_CLASSES = 4;
constexpr uint32_t DENSE_CLASS[DENSE_CLASSES] = {1024, 2048, 4096, 8192}; // words of a row (8 ids each), at most
uint32_t dense_class_waves(int k); // waves of a class the device holds
struct DenseBatch {
    const TraceDesc *d;
    const ChunkDesc *ch;
    uint32_t class_at[DENSE_CLASSES + 1]; // first chunk of every class
    const uint32_t *words;
    const uint64_t *pos;
    const PrefixJob *jobs;
    uint32_t n_jobs;
    bool grouped; // a trace has more than one group
    uint32_t *rows, *grp, *vcnt;
};
// status bytes, final statuses, flagged induced items, flagged events per chunk (vcnt)
void launch_batch_dense(const DenseBatch &B, hipStream_t s);
// every trace's number of violations, from vpos = the exclusive prefix of vcnt, and the final
// statuses of the traces checked by strands (the batch's first `strands` chunks)
void launch_batch_counts(const TraceDesc *d, uint32_t n_traces, const uint64_t *vpos, uint32_t strands,
                         const uint64_t *lbv, const Control *bctl, hipStream_t s);

void launch_batch_reset(const TraceDesc *d, uint32_t n_traces, unsigned long long *ind, hipStream_t s);
// every trace's initial statuses into its key range of init_all and fin_all (K keys)
void launch_batch_init(const TraceDesc *d, uint32_t n_traces, uint64_t K, uint8_t *init_all, uint8_t *fin_all,
                       hipStream_t s);
// general route: every trace's status bytes, final statuses, violations and counts
void launch_batch_distribute(const TraceDesc *d, uint32_t n_traces, const uint8_t *status_all, const uint8_t *fin_all,
                             const uint32_t *viol_all, const Control *bctl, const unsigned long long *ind,
                             hipStream_t s);

} // namespace vc
