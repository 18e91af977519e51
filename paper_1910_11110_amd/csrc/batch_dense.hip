// batch_dense.hip -- batched check of traces over at most 2^16 ids each: no event is moved.
//
// Every trace is walked in its order with the statuses of all its ids in LDS (see
// dense_steps.h), all traces of the batch together: a trace without arrays straight from
// its events, one with arrays from its combined words.  The traces are cut into chunks,
// one wave each; a launch takes the chunks whose rows fit its tables (a wave of 2^16 ids
// takes 32 KB of LDS, and one over few ids shall not wait for that room).
// 1. fold: every chunk's functions, backwards, into its row.
// 2. groups, prefix: per trace and word of its rows, the statuses entering every chunk,
//    by groups of B_GROUP chunks.
// 3. apply: the status bytes, the flagged events of every chunk and the flagged induced
//    items of every trace; a trace's last chunk leaves its final statuses.
// 4. the violation lists, from a scan of the chunks' counts, and the counts.
// A trace's initial and final statuses may lie in the same place: a launch that writes final
// ones (3, and 4 of the traces checked by strands) comes after all that read initial ones (2
// and the strands).
// Bound like the dense check by the walks' LDS round trips and their instructions.  1,024
// traces of 100 to 10^6 events over 8 to 65,536 ids, a fifth of them over arrays (110 M
// events): kernels 2,133 us through the bucket engine (which relocates every event to a
// word, partitions, scans and takes the results back), 1,018 this way, 950 with the plain
// traces over few ids by strands (small.hip), 940 with the items' bounds by one load: of
// them the folds 247, the applies 357, the strands 55 and the words of the traces with
// arrays 141.
#include "batch.h"
#include "dense_steps.h"
#include "prof.h"

namespace vc {

namespace {

constexpr int B_PAIR = 2;

// the chunks [first, first + chunks) of the batch
struct BatchChunks {
    const TraceDesc *d;
    const ChunkDesc *ch;
    const uint32_t *words; // of the traces with arrays
    const uint64_t *pos;   // their chunks' induced items, as exclusive sums
    uint32_t first, chunks;

    struct Chunk {
        const uint32_t *ev;
        uint64_t begin, end, row_at;
        uint64_t start; // first event, trace-relative
        const TraceDesc *t;
        uint32_t row, bits, n_ids, len, index; // (index: of the chunk in the batch)
        bool arrays, last;
        __device__ uint32_t local(uint32_t w) const { return w & 0xFFFFu; }
        __device__ uint32_t clamped(uint32_t w) const
        {
            const uint32_t x = w & 0xFFFFFFu;
            return x < n_ids ? x : n_ids - 1;
        }
        __device__ bool bad(uint32_t w) const
        {
            return (w >> 28) != 0 || ((w >> 24) & 7u) > (arrays ? (uint32_t)OP_RWIND : (uint32_t)OP_NOOP) ||
                   (w & 0xFFFFFFu) >= n_ids;
        }
        // (the words' own pass reported theirs)
        __device__ Control *report_to(Control *) const { return arrays ? nullptr : t->ctl; }
    };
    __device__ uint32_t count() const { return chunks; }
    __device__ Chunk chunk(uint32_t c) const
    {
        Chunk C;
        C.index = first + c;
        const ChunkDesc cd = ch[C.index];
        const TraceDesc *t = C.t = d + cd.trace;
        C.start = cd.start;
        C.len = cd.len;
        C.n_ids = t->n_ids;
        C.bits = 32u - (uint32_t)__builtin_clz(C.n_ids | 1u);
        C.row = t->row;
        C.row_at = t->row_base + (C.index - t->first_dense) * (uint64_t)C.row;
        C.last = cd.start + cd.len == t->n;
        C.arrays = t->off != nullptr;
        if (C.arrays) {
            const uint64_t tile = t->first_chunk + cd.start / BATCH_CHUNK, p0 = pos[t->first_chunk];
            const uint64_t next = tile + ceil_div((uint64_t)cd.len, (uint64_t)BATCH_CHUNK);
            auto at = [&](uint64_t p) { return p < t->m ? p : t->m; }; // (events that changed since they were sized)
            C.ev = words + t->item_base;
            C.begin = at(cd.start + (pos[tile] - p0));
            C.end = at(cd.start + cd.len + (pos[next] - p0));
        } else {
            C.ev = t->events;
            C.begin = cd.start;
            C.end = cd.start + cd.len;
        }
        return C;
    }
};

// the status bytes of the events, in their order; flagged events and induced items counted
struct BatchOut {
    uint32_t *vcnt;
    const TraceDesc *t;
    uint8_t *status; // of the chunk's first event
    uint32_t len, row, n_ids, index;
    bool arrays, last;
    uint32_t next, flagged, induced;
    uint64_t from;
    __device__ void begin(const BatchChunks::Chunk &C, uint32_t)
    {
        t = C.t;
        status = C.t->status + C.start;
        len = C.len;
        row = C.row;
        n_ids = C.n_ids;
        index = C.index;
        arrays = C.arrays;
        last = C.last;
        from = C.begin;
        next = flagged = induced = 0;
    }
    __device__ void step(uint32_t lane, uint32_t, uint64_t i, uint32_t w, uint32_t byte, bool valid)
    {
        if (!arrays) {
            if (valid)
                status[i - from + lane] = (uint8_t)byte;
            flagged += (uint32_t)__builtin_popcountll(__ballot(valid && (byte & 0x80u)));
            return;
        }
        const bool event = valid && ((w >> 24) & 7u) <= OP_NOOP;
        const uint64_t m = __ballot(event), f = __ballot(valid && (byte & 0x80u));
        const uint32_t at = next + mask_rank(m);
        if (event && at < len)
            status[at] = (uint8_t)byte;
        next += (uint32_t)__builtin_popcountll(m);
        flagged += (uint32_t)__builtin_popcountll(f & m);
        induced += (uint32_t)__builtin_popcountll(f & ~m);
    }
    __device__ void round(uint32_t, uint64_t, uint32_t, bool) const {}
    __device__ void chunk(uint32_t lane, const uint32_t *s_t) const
    {
        if (lane == 0) {
            vcnt[index] = flagged;
            if (induced)
                atomicAdd(reinterpret_cast<unsigned long long *>(&t->ctl->n_induced_stuck),
                          (unsigned long long)induced);
        }
        if (last)
            for (uint32_t w = lane; w * 8 < n_ids; w += WAVE)
                Two::put_final(s_t[w], t->fin, w * 8, n_ids);
    }
};

// a group of a trace's chunks, and BLOCK words of its rows
__global__ __launch_bounds__(BLOCK) void k_batch_groups(const TraceDesc *__restrict__ d,
                                                        const PrefixJob *__restrict__ jobs,
                                                        const uint32_t *__restrict__ rows, uint32_t *__restrict__ grp)
{
    const PrefixJob J = jobs[blockIdx.x];
    const TraceDesc &t = d[J.trace];
    const uint32_t w = J.word + threadIdx.x, row = t.row, c0 = J.group * B_GROUP, c1 = c0 + B_GROUP;
    if (w >= row || c1 >= t.dense_chunks)
        return; // (nothing follows the last group)
    uint32_t f = 0;
#pragma unroll 8
    for (uint32_t c = c0; c < c1; c++)
        f = tw_compose(rows[t.row_base + (uint64_t)c * row + w], f);
    grp[t.grp_base + (uint64_t)J.group * row + w] = f;
}

__global__ __launch_bounds__(BLOCK) void k_batch_prefix(const TraceDesc *__restrict__ d,
                                                        const PrefixJob *__restrict__ jobs, uint32_t *rows,
                                                        const uint32_t *__restrict__ grp)
{
    const PrefixJob J = jobs[blockIdx.x];
    const TraceDesc &t = d[J.trace];
    const uint32_t w = J.word + threadIdx.x, row = t.row, c0 = J.group * B_GROUP;
    if (w >= row)
        return;
    const uint32_t c1 = c0 + B_GROUP < t.dense_chunks ? c0 + B_GROUP : t.dense_chunks;
    uint32_t st = Two::initial(t.init, w * 8, t.n_ids);
#pragma unroll 8
    for (uint32_t q = 0; q < J.group; q++)
        st = tw_compose(grp[t.grp_base + (uint64_t)q * row + w], st);
    uint32_t *const r = rows + t.row_base + w;
#pragma unroll 8
    for (uint32_t c = c0; c < c1; c++) {
        const uint32_t f = r[(uint64_t)c * row];
        r[(uint64_t)c * row] = st;
        st = tw_compose(f, st);
    }
}

// a wave a trace: its number of violations and, checked by strands, its final statuses, which
// its last chunk's words hold as constants
__global__ __launch_bounds__(BLOCK) void k_batch_counts(const TraceDesc *__restrict__ d, uint32_t n_traces,
                                                        const uint64_t *__restrict__ vpos, uint32_t strands,
                                                        const uint64_t *__restrict__ lbv,
                                                        const Control *__restrict__ bctl)
{
    const uint32_t t = blockIdx.x * (BLOCK / WAVE) + threadIdx.x / WAVE, lane = lane_id();
    if (t >= n_traces)
        return;
    const TraceDesc &td = d[t];
    const uint64_t end = td.first_dense + td.dense_chunks;
    if (td.first_dense < strands && lane < td.n_ids) { // (at most 64 ids)
        const Planes st = pl_unpack(lbv[(end - 1) * STRAND_WORDS + lane / STRAND_IDS]);
        const uint32_t k = lane % STRAND_IDS;
        td.fin[lane] = (uint8_t)(((st.x >> k) & 1u) | (((st.y >> k) & 1u) << 1));
    }
    if (lane)
        return;
    td.ctl->n_viol = vpos[end] - vpos[td.first_dense];
    if (bctl->err_code) // an internal error of the shared scan concerns every trace
        atomicOr(&td.ctl->err_code, bctl->err_code);
}

size_t table_lds(uint32_t table) { return ((size_t)table + 32) * 4; }

} // namespace

uint32_t dense_class_waves(int k)
{
    const uint64_t waves = 163840 / table_lds(DENSE_CLASS[k]);
    return 256 * (uint32_t)(waves > 24 ? 24 : waves);
}

// The launches of a walk: the chunks of consecutive classes together, with the tables of the
// widest, while the device holds them all at once.  A launch that leaves it idle lasts as long
// as a chunk does, 10 to 25 us (kernels of 32 traces, 3.7 M events, 7 of the traces over more
// than 8,192 ids: the folds 61 us and the applies 91 in a launch a class, 42 and 54 this way).
template <class LAUNCH> static void by_launches(const DenseBatch &B, LAUNCH launch)
{
    for (int hi = DENSE_CLASSES - 1, lo; hi >= 0; hi = lo - 1) {
        lo = hi;
        if (B.class_at[hi + 1] == B.class_at[hi])
            continue;
        while (lo > 0 && B.class_at[hi + 1] - B.class_at[lo - 1] <= dense_class_waves(hi))
            lo--;
        launch(BatchChunks{B.d, B.ch, B.words, B.pos, B.class_at[lo], B.class_at[hi + 1] - B.class_at[lo]},
               DENSE_CLASS[hi]);
    }
}

void launch_batch_dense(const DenseBatch &B, hipStream_t s)
{
    by_launches(B, [&](const BatchChunks &T, uint32_t table) {
        ProfScope p(s, "batch_fold");
        k_dense_fold<Fold<Two>, B_PAIR, BatchChunks>
            <<<T.chunks, WAVE, table_lds(table), s>>>(T, table, B.rows, nullptr, nullptr);
    });
    if (B.grouped) {
        ProfScope p(s, "batch_groups");
        k_batch_groups<<<B.n_jobs, BLOCK, 0, s>>>(B.d, B.jobs, B.rows, B.grp);
    }
    if (B.n_jobs) {
        ProfScope p(s, "batch_prefix");
        k_batch_prefix<<<B.n_jobs, BLOCK, 0, s>>>(B.d, B.jobs, B.rows, B.grp);
    }
    by_launches(B, [&](const BatchChunks &T, uint32_t table) {
        ProfScope p(s, "batch_apply");
        k_dense_apply<Apply<Two>, B_PAIR, BatchChunks, BatchOut><<<T.chunks, WAVE, table_lds(table), s>>>(
            T, table, B.rows, BatchOut{B.vcnt, nullptr, nullptr, 0, 0, 0, 0, false, false, 0, 0, 0, 0});
    });
}

void launch_batch_counts(const TraceDesc *d, uint32_t n_traces, const uint64_t *vpos, uint32_t strands,
                         const uint64_t *lbv, const Control *bctl, hipStream_t s)
{
    ProfScope p(s, "batch_counts");
    k_batch_counts<<<(unsigned)ceil_div(n_traces, BLOCK / WAVE), BLOCK, 0, s>>>(d, n_traces, vpos, strands, lbv, bctl);
}

} // namespace vc
