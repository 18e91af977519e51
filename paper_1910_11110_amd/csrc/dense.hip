// dense.hip -- check of a trace in program order, the statuses of all its ids in LDS
// (gfx950).
//
// For id spaces up to 2^16.  The trace is cut into chunks, one wave each, and no event is
// moved:
// 1. fold: a wave walks its chunk backwards, 64 events a step, and composes every id's
//    transition function over the chunk in a table in LDS (3 bits an id); the table is
//    the chunk's row in memory.  Going backwards, an id whose function has become a
//    constant (its last write) is done, so frequent ids soon cost nothing.
// 2. prefix: per word of the rows (8 ids at once by bit operations), the rows composed
//    in order from the initial statuses give the statuses entering every chunk, in
//    place, and the final ones.
// 3. apply: a wave walks its chunk forwards from its entering statuses; an event reads
//    its id's status, leaves the new one and its status byte is stored.
// A step's 64 events update the table in one go unless two of them share an id: each event
// sets its id's touch bit by the same atomic that reads the id's table word, so a lane
// that finds the bit set knows.  The lanes of a shared id (rare over many ids, the rule
// over few or over skewed ones) are put in order by composing their functions along them.
#include "dense.h"
#include "dense_steps.h"
#include "prof.h"

namespace vc {

namespace {

constexpr uint32_t OP_PROBE = DENSE_OP_PROBE;
constexpr int D_PAIR = 2;

// the chunks of one trace: `per` events each (a multiple of 64), the last one the rest
struct TraceChunks {
    const uint32_t *ev;
    uint64_t n, per;
    uint32_t n_ids, row, chunks;
    __device__ uint32_t op_mask() const { return 0x1F1Fu; }
    __device__ OneChunk<TraceChunks> chunk(uint32_t c) const { return {*this, c}; }
    __device__ Control *report_to(Control *ctl) const { return ctl; }
    __device__ uint32_t count() const { return chunks; }
    __device__ uint32_t id_bits() const { return 32u - (uint32_t)__builtin_clz(n_ids | 1u); }
    __device__ uint32_t local(uint32_t w) const { return w & 0xFFFFu; }
    __device__ uint32_t clamped(uint32_t w) const
    {
        const uint32_t x = w & 0xFFFFFFu;
        return x < n_ids ? x : n_ids - 1;
    }
    __device__ uint64_t begin_of(uint32_t c) const { return (uint64_t)c * per; }
    __device__ uint64_t end_of(uint32_t c) const
    {
        const uint64_t e = (uint64_t)(c + 1) * per;
        return e < n ? e : n;
    }
    __device__ bool bad(uint32_t w) const
    {
        return (w >> 28) != 0 || ((w >> 24) & 7u) > OP_NOOP || (w & 0xFFFFFFu) >= n_ids;
    }
};

// the chunks of a combined stream: the words of `per` tiles of events each
struct TileChunks {
    const uint32_t *ev;
    const uint64_t *tpos; // first word of every tile, their number at the end
    uint64_t n, tiles, per;
    uint32_t n_ids, row, chunks;
    __device__ uint32_t op_mask() const { return 0x7F7Fu; }
    __device__ OneChunk<TileChunks> chunk(uint32_t c) const { return {*this, c}; }
    __device__ Control *report_to(Control *ctl) const { return ctl; }
    __device__ uint32_t count() const { return chunks; }
    __device__ uint32_t id_bits() const { return 32u - (uint32_t)__builtin_clz(n_ids | 1u); }
    __device__ uint32_t local(uint32_t w) const { return w & 0xFFFFu; }
    __device__ uint32_t clamped(uint32_t w) const
    {
        const uint32_t x = w & 0xFFFFFFu;
        return x < n_ids ? x : n_ids - 1;
    }
    __device__ uint64_t at(uint64_t tile) const
    {
        const uint64_t p = tpos[tile < tiles ? tile : tiles];
        return p < n ? p : n; // (events that changed since the stream was sized)
    }
    __device__ uint64_t begin_of(uint32_t c) const { return at((uint64_t)c * per); }
    __device__ uint64_t end_of(uint32_t c) const { return at((uint64_t)(c + 1) * per); }
    __device__ bool bad(uint32_t w) const
    {
        return (w >> 28) != 0 || ((w >> 24) & 7u) > OP_PROBE || (w & 0xFFFFFFu) >= n_ids;
    }
};

// 2. prefix over the rows, by groups of D_GROUP chunks: a thread per word and group.  The
// first kernel folds every group's rows; the second walks them from the statuses entering
// the group (the initial ones and the groups before) and leaves the statuses entering
// every chunk (`entering` may be `rows`); the last group's end is the final table.
constexpr uint32_t D_GROUP = 32;

__global__ __launch_bounds__(BLOCK) void k_dense_groups(const uint32_t *__restrict__ rows, uint32_t row,
                                                        uint32_t chunks, uint32_t *__restrict__ grp)
{
    const uint32_t w = blockIdx.x * BLOCK + threadIdx.x, g = blockIdx.y;
    if (w >= row)
        return;
    const uint32_t c0 = g * D_GROUP, c1 = c0 + D_GROUP < chunks ? c0 + D_GROUP : chunks;
    uint32_t f = 0;
#pragma unroll 8
    for (uint32_t c = c0; c < c1; c++)
        f = tw_compose(rows[(uint64_t)c * row + w], f);
    grp[(uint64_t)g * row + w] = f;
}

__global__ __launch_bounds__(BLOCK) void k_dense_prefix(const uint32_t *rows, uint32_t *entering, uint32_t row,
                                                        uint32_t chunks, const uint32_t *__restrict__ grp,
                                                        uint32_t n_ids,
                                                        const uint8_t *__restrict__ init,
                                                        uint8_t *__restrict__ final_out)
{
    const uint32_t w = blockIdx.x * BLOCK + threadIdx.x, g = blockIdx.y;
    if (w >= row)
        return;
    uint32_t st = Two::initial(init, w * 8, n_ids);
#pragma unroll 8
    for (uint32_t q = 0; q < g; q++)
        st = tw_compose(grp[(uint64_t)q * row + w], st);
    const uint32_t c0 = g * D_GROUP, c1 = c0 + D_GROUP < chunks ? c0 + D_GROUP : chunks;
#pragma unroll 8
    for (uint32_t c = c0; c < c1; c++) {
        const uint32_t f = rows[(uint64_t)c * row + w];
        entering[(uint64_t)c * row + w] = st;
        st = tw_compose(f, st);
    }
    if (c1 == chunks && final_out)
        Two::put_final(st, final_out, w * 8, n_ids);
}

// 3. what becomes of the events' statuses
constexpr uint32_t D_TILE = 512;
static_assert(D_TILE % (D_UNROLL * WAVE) == 0, "whole rounds of steps a tile");

// a trace: status bytes; per step of 64 events the mask of the flagged ones, per tile of
// D_TILE events their number
struct TraceOut {
    uint8_t *status;
    uint64_t *masks;
    uint32_t *tcnt;
    uint64_t mask; // lane u: the flagged events of step u
    uint32_t flagged;
    template <class CHUNKS>
    __device__ void begin(const CHUNKS &, uint32_t)
    {
        flagged = 0;
    }
    __device__ void step(uint32_t lane, uint32_t u, uint64_t i, uint32_t, uint32_t byte, bool valid)
    {
        if (valid)
            status[i + lane] = (uint8_t)byte;
        const uint64_t m = __ballot(valid && (byte & 0x80u));
        mask = lane == u ? m : mask;
        flagged += (uint32_t)__builtin_popcountll(m);
    }
    __device__ void round(uint32_t lane, uint64_t i, uint32_t steps, bool last)
    {
        if (lane < steps)
            masks[i / WAVE + lane] = mask;
        if (last || (i / (D_UNROLL * WAVE) + 1) % (D_TILE / (D_UNROLL * WAVE)) == 0) {
            if (lane == 0)
                tcnt[i / D_TILE] = flagged;
            flagged = 0;
        }
    }
    __device__ void chunk(uint32_t, const uint32_t *) const {}
};

// a combined stream: the status bytes of the events, in their order; flagged induced
// items are counted
struct PrimaryOut {
    uint8_t *status;
    uint64_t n; // events
    uint32_t tile; // events per tile
    unsigned long long *induced;
    uint64_t next;
    uint32_t count;
    __device__ void begin(const OneChunk<TileChunks> &T, uint32_t c)
    {
        next = (uint64_t)c * T.per * tile;
        count = 0;
    }
    __device__ void step(uint32_t lane, uint32_t, uint64_t, uint32_t w, uint32_t byte, bool valid)
    {
        const uint32_t op = (w >> 24) & 7u;
        const bool event = valid && op <= OP_NOOP;
        const uint64_t m = __ballot(event);
        const uint64_t at = next + mask_rank(m);
        if (event && at < n)
            status[at] = (uint8_t)byte;
        next += (uint32_t)__builtin_popcountll(m);
        count += (uint32_t)__builtin_popcountll(__ballot(valid && op == OP_RWIND && (byte & 0x80u)));
    }
    __device__ void round(uint32_t, uint64_t, uint32_t, bool) const {}
    __device__ void chunk(uint32_t lane, const uint32_t *) const
    {
        if (lane == 0 && count)
            atomicAdd(induced, (unsigned long long)count);
    }
};

// The functions that the probes see, from their chunk's beginning, at their positions: with
// them a stream with probes is walked twice, not three times (34 M words over 2^16 ids, of
// 2^23 events with 48,000 creates: fold 146, a walk for the probes 125 and the apply 125 us
// before; composed forwards 126 and the apply 132).
struct ProbeOut {
    uint8_t *pre;
    __device__ void begin(const OneChunk<TileChunks> &, uint32_t) const {}
    __device__ void step(uint32_t lane, uint32_t, uint64_t i, uint32_t w, uint32_t byte, bool valid) const
    {
        if (valid && ((w >> 24) & 7u) == OP_PROBE)
            pre[i + lane] = (uint8_t)byte;
    }
    __device__ void round(uint32_t, uint64_t, uint32_t, bool) const {}
    __device__ void chunk(uint32_t, const uint32_t *) const {}
};

// ascending indices of the flagged events, one wave per tile (SUM: the tiles' offsets are
// the sums of their counts, worked out by every workgroup for its own)
template <bool SUM>
__global__ __launch_bounds__(BLOCK) void k_mask_scatter(const uint64_t *__restrict__ masks, uint64_t n,
                                                        const uint64_t *__restrict__ offs,
                                                        const uint32_t *__restrict__ tcnt, uint64_t ntiles,
                                                        uint32_t *__restrict__ viol, unsigned long long *n_viol)
{
    constexpr uint32_t STEPS = D_TILE / WAVE, WAVES = BLOCK / WAVE;
    const uint32_t lane = lane_id(), wave = threadIdx.x / WAVE;
    uint64_t before = 0;
    if constexpr (SUM) { // (one tile a wave)
        const uint32_t t0 = blockIdx.x * WAVES;
        before = sum_before<BLOCK>(tcnt, t0);
        for (uint32_t w = 0; w < wave; w++)
            before += t0 + w < ntiles ? tcnt[t0 + w] : 0u;
    }
    for (uint64_t t = (uint64_t)blockIdx.x * WAVES + wave; t < ntiles; t += (uint64_t)gridDim.x * WAVES) {
        uint64_t o = SUM ? before : offs[t];
        if (SUM && t + 1 == ntiles && lane == 0)
            *n_viol = o + tcnt[t];
        const uint64_t nsteps = ceil_div(n, (uint64_t)WAVE);
        const uint64_t mine = lane < STEPS && t * STEPS + lane < nsteps ? masks[t * STEPS + lane] : 0ull;
#pragma unroll
        for (uint32_t q = 0; q < STEPS; q++) {
            const uint64_t m = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), q) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, q);
            if ((m >> lane) & 1u)
                viol[o + mask_rank(m)] = (uint32_t)(t * D_TILE + q * WAVE + lane);
            o += (uint64_t)__builtin_popcountll(m);
        }
    }
}

// LDS of a wave: its table and the step table
size_t dense_lds(uint32_t row) { return ((size_t)row + 32) * 4; }

// a row's words (a multiple of 64 of them, 8 ids each)
uint32_t dense_row(uint32_t n_ids) { return ((uint32_t)ceil_div(n_ids ? n_ids : 1, 8) + 63u) & ~63u; }

// Chunks that fill the device: as many waves as have their tables in a CU's 160 KB (4 of
// 2^16 ids; 5 would leave no room for the step table), at most 24, on 256 CUs.
uint64_t dense_chunks(uint32_t n_ids)
{
    const uint64_t waves = 163840 / dense_lds(dense_row(n_ids));
    return 256 * (waves > 24 ? 24 : waves);
}

struct Rows { // chunks' rows and groups' rows
    uint32_t row, chunks, groups;
    uint32_t *rows, *entering, *grp;
    uint32_t *left; // chunks that the forward fold leaves to the backward one
};

class Carve {
public:
    explicit Carve(void *scratch) : p0(reinterpret_cast<char *>(scratch)) {}
    template <class T>
    T *take(size_t n)
    {
        T *r = p0 ? reinterpret_cast<T *>(p0 + off) : nullptr;
        off += (n * sizeof(T) + 255) & ~size_t(255);
        return r;
    }
    size_t bytes() const { return off; }

private:
    char *p0;
    size_t off = 0;
};

// (keep: the chunks' functions stay beside the entering statuses, for another prefix)
Rows take_rows(Carve &c, uint32_t n_ids, uint32_t chunks, bool keep)
{
    Rows R{};
    R.row = dense_row(n_ids);
    R.chunks = chunks;
    R.groups = (uint32_t)ceil_div(chunks, D_GROUP);
    R.rows = c.take<uint32_t>((size_t)chunks * R.row);
    R.entering = keep ? c.take<uint32_t>((size_t)chunks * R.row) : R.rows;
    R.grp = c.take<uint32_t>((size_t)R.groups * R.row);
    R.left = c.take<uint32_t>(chunks);
    return R;
}

void launch_groups(const Rows &R, hipStream_t s)
{
    if (R.groups < 2)
        return;
    ProfScope p(s, "dense_groups");
    k_dense_groups<<<dim3((unsigned)ceil_div(R.row, BLOCK), R.groups - 1), BLOCK, 0, s>>>(R.rows, R.row, R.chunks, R.grp);
}

template <class CHUNKS>
void launch_fold(const CHUNKS &T, const Rows &R, Control *ctl, hipStream_t s)
{
    if (!T.chunks)
        return;
    const unsigned lds = dense_lds(R.row);
    if (T.n_ids > FORWARD_IDS && T.n >= DENSE_FORWARD_FROM) {
        {
            ProfScope p(s, "dense_forward");
            k_dense_forward<Two, D_PAIR, CHUNKS><<<T.chunks, WAVE, lds, s>>>(T, R.row, R.rows, ctl, R.left);
        }
        ProfScope p(s, "dense_fold"); // (of the chunks of skewed ids)
        k_dense_fold<Fold<Two>, D_PAIR, CHUNKS><<<T.chunks, WAVE, lds, s>>>(T, R.row, R.rows, ctl, R.left);
    } else {
        ProfScope p(s, "dense_fold");
        k_dense_fold<Fold<Two>, D_PAIR, CHUNKS><<<T.chunks, WAVE, lds, s>>>(T, R.row, R.rows, ctl, nullptr);
    }
    launch_groups(R, s);
}

void launch_prefix(const Rows &R, uint32_t chunks, uint32_t n_ids, const uint8_t *init, uint8_t *final_out,
                   hipStream_t s)
{
    ProfScope p(s, "dense_prefix");
    k_dense_prefix<<<dim3((unsigned)ceil_div(R.row, BLOCK), R.groups), BLOCK, 0, s>>>(
        R.rows, R.entering, R.row, chunks, R.grp, n_ids, init, final_out);
}

template <class CHUNKS, class OUT>
void launch_apply(const CHUNKS &T, const Rows &R, const OUT &out, hipStream_t s)
{
    if (!T.chunks)
        return;
    ProfScope p(s, "dense_apply");
    k_dense_apply<Apply<Two>, D_PAIR, CHUNKS, OUT><<<T.chunks, WAVE, dense_lds(R.row), s>>>(T, R.row, R.entering, out);
}

// rows, masks and tile counts of a trace
struct TraceLayout {
    Rows R;
    uint64_t per, tiles;
    uint32_t *tcnt;
    uint64_t *masks, *offs;
    void *xscan;
    size_t bytes;
};

TraceLayout trace_layout(void *scratch, uint64_t n, uint32_t n_ids)
{
    TraceLayout L{};
    L.tiles = ceil_div(n ? n : 1, (uint64_t)D_TILE);
    L.per = ceil_div(L.tiles, dense_chunks(n_ids)) * D_TILE;
    Carve c(scratch);
    L.R = take_rows(c, n_ids, (uint32_t)ceil_div(n ? n : 1, L.per), false);
    L.masks = c.take<uint64_t>(L.tiles * (D_TILE / WAVE));
    L.tcnt = c.take<uint32_t>(L.tiles);
    L.offs = c.take<uint64_t>(L.tiles + 1);
    L.xscan = c.take<char>(excl_scan_scratch_bytes(L.tiles));
    L.bytes = c.bytes();
    return L;
}

// tiles of events per chunk of a combined stream
uint64_t tiles_per_chunk(uint64_t tiles, uint32_t n_ids) { return ceil_div(tiles ? tiles : 1, dense_chunks(n_ids)); }

Rows words_layout(Carve &c, uint64_t tiles, uint32_t n_ids, bool keep)
{
    return take_rows(c, n_ids, (uint32_t)ceil_div(tiles ? tiles : 1, tiles_per_chunk(tiles, n_ids)), keep);
}

TileChunks words_chunks(const DenseWords &W, const Rows &R)
{
    const uint64_t per = tiles_per_chunk(W.tiles, W.n_ids);
    return TileChunks{W.words, W.tpos, W.m, W.tiles, per, W.n_ids, R.row, W.m ? R.chunks : 0u};
}

} // namespace

size_t dense_scratch_bytes(uint64_t n, uint32_t n_ids) { return trace_layout(nullptr, n, n_ids).bytes; }

void launch_dense_check(const uint32_t *events, uint64_t n, uint32_t n_ids, const uint8_t *init, uint8_t *status,
                        uint8_t *final_out, uint32_t *viol, void *scratch, Control *ctl, hipStream_t s)
{
    const TraceLayout L = trace_layout(scratch, n, n_ids);
    const FillJob job{L.xscan, excl_scan_scratch_bytes(L.tiles), 0};
    launch_prep(ctl, nullptr, &job, 1, s);
    const TraceChunks T{events, n, L.per, n_ids, L.R.row, n ? L.R.chunks : 0u};
    launch_fold(T, L.R, ctl, s);
    launch_prefix(L.R, T.chunks, n_ids, init, final_out, s);
    if (!n)
        return;
    launch_apply(T, L.R, TraceOut{status, L.masks, L.tcnt, 0, 0}, s);
    const uint64_t blocks = ceil_div(L.tiles, BLOCK / WAVE);
    if (L.tiles <= SUM_TILES) {
        ProfScope p(s, "mask_scatter");
        k_mask_scatter<true><<<(unsigned)blocks, BLOCK, 0, s>>>(L.masks, n, nullptr, L.tcnt, L.tiles, viol, &ctl->n_viol);
        return;
    }
    launch_excl_scan(L.tcnt, L.tiles, L.offs, reinterpret_cast<uint64_t *>(&ctl->n_viol), L.xscan, ctl->tickets[10], s,
                     true);
    ProfScope p(s, "mask_scatter");
    k_mask_scatter<false><<<(unsigned)(blocks < 8192 ? blocks : 8192), BLOCK, 0, s>>>(L.masks, n, L.offs, L.tcnt, L.tiles,
                                                                                      viol, nullptr);
}

size_t dense_words_scratch_bytes(uint64_t tiles, uint32_t n_ids, bool probes)
{
    Carve c(nullptr);
    (void)words_layout(c, tiles, n_ids, probes);
    return c.bytes();
}

void launch_dense_words_fold(const DenseWords &W, void *scratch, Control *ctl, hipStream_t s)
{
    launch_reset_control(ctl, s);
    Carve c(scratch);
    const Rows R = words_layout(c, W.tiles, W.n_ids, false);
    launch_fold(words_chunks(W, R), R, ctl, s);
}

DenseEntering launch_dense_words_probe(const DenseWords &W, const uint8_t *init, uint8_t *pre, void *scratch,
                                       Control *ctl, hipStream_t s)
{
    launch_reset_control(ctl, s);
    Carve c(scratch);
    const Rows R = words_layout(c, W.tiles, W.n_ids, true);
    const TileChunks T = words_chunks(W, R);
    if (T.chunks) {
        ProfScope p(s, "dense_onto");
        k_dense_apply<Onto<Two>, D_PAIR, TileChunks, ProbeOut>
            <<<T.chunks, WAVE, dense_lds(R.row), s>>>(T, R.row, R.rows, ProbeOut{pre});
        launch_groups(R, s);
    }
    launch_prefix(R, T.chunks, W.n_ids, init, nullptr, s);
    return DenseEntering{R.entering, R.row, T.per};
}

void launch_dense_words_apply(const DenseWords &W, bool probes, const uint8_t *init, uint64_t n, uint32_t tile,
                              uint8_t *status, uint8_t *final_out, void *scratch, Control *ctl, hipStream_t s)
{
    Carve c(scratch);
    const Rows R = words_layout(c, W.tiles, W.n_ids, probes);
    const TileChunks T = words_chunks(W, R);
    launch_prefix(R, T.chunks, W.n_ids, init, final_out, s);
    launch_apply(T, R, PrimaryOut{status, n, tile, &ctl->n_induced_stuck, 0, 0}, s);
}

} // namespace vc
