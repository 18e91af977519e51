// wide.hip -- scan of partitioned events, a bucket's ids in LDS (gfx950).
//
// For id spaces whose table does not fit a wave's LDS the events are first partitioned by
// buckets of ids; a chunk is then a run of one bucket's events, and the walks are those of
// the dense check (dense_steps.h) on the bucket's table.  The prefix over the chunks'
// rows starts from the initial statuses at every bucket's first chunk.
#include "dense_steps.h"
#include "prof.h"
#include "spaces.h"
#include "wide.h"

namespace vc {

namespace {

// k memory spaces: a word per id, its function (17 bits) and the touch bit
struct Spaces {
    static constexpr uint32_t SELF = 0x8421u; // every location reaches itself
    static constexpr bool BY_MASKS = false, CLOSES = false;
    static constexpr int ALIKE = 0;
    static constexpr uint32_t MASK = 0x1FFFFu, IDENTITY = KF_ID, NOOP = 3u << 24, IDS = 1, ROW_IDENTITY = KF_ID;
    __device__ static uint32_t word(uint32_t id) { return id; }
    __device__ static uint32_t shift(uint32_t) { return 0; }
    __device__ static uint32_t touch(uint32_t) { return 1u << 31; }
    __device__ static uint32_t fold_entry(const uint32_t *, uint32_t w) { return w >> 24; }
    __device__ static bool fold_part(uint32_t ob) { return (ob & 3u) == K_OP_W || (ob & 3u) == K_OP_COPY; }
    // a write at a, then h: the constant h({a}); a copy from a to b, then h: what b reaches
    // joins a's row
    __device__ static uint32_t fold_next(uint32_t ob, uint32_t h)
    {
        const bool wr = (ob & 3u) == K_OP_W;
        const uint32_t a4 = ob & 12u, from = wr ? a4 : (ob >> 2) & 12u;
        const uint32_t reach = ((h | SELF) >> from) & 15u;
        return (h & KF_CONST) ? h : wr ? KF_CONST | reach : h | (reach << a4);
    }
    __device__ static bool fold_open(uint32_t h) { return (h & KF_CONST) == 0; }
    __device__ static uint32_t apply_entry(const uint32_t *, uint32_t w) { return w >> 24; }
    __device__ static uint32_t apply_next(uint32_t ob, uint32_t h, uint32_t &st)
    {
        const uint32_t op = ob & 3u, pre = h & 15u, at_a = (pre >> ((ob >> 2) & 3u)) & 1u;
        const uint32_t a = (SELF >> (ob & 12u)) & 15u, b = (SELF >> ((ob >> 2) & 12u)) & 15u;
        const uint32_t copied = op == K_OP_COPY ? b & (0u - at_a) : 0u; // nothing when stuck
        const uint32_t post = op == K_OP_W ? a : pre | copied;
        const uint32_t stuck = (op == K_OP_R || op == K_OP_COPY) ? at_a ^ 1u : 0u;
        st = post | (pre << 4) | (stuck << 15);
        return KF_CONST | post;
    }
    __device__ static uint32_t function(const uint32_t *, uint32_t w) { return kf_of(w >> 24); }
    __device__ static uint32_t compose(uint32_t g, uint32_t f) { return kf_compose(g, f); }
    __device__ static bool constant(uint32_t f) { return (f & KF_CONST) != 0; }
    __device__ static uint32_t pack(uint32_t f, uint32_t p) { return f | (p << 17); }
    __device__ static uint32_t packed_function(uint32_t v) { return v & MASK; }
    __device__ static uint32_t packed_lane(uint32_t v) { return v >> 17; }
    __device__ static uint32_t fold_all(uint32_t h, uint32_t f) { return kf_compose(h, f); }
    __device__ static uint32_t status_after(uint32_t f, uint32_t h) { return kf_apply(f, h & 15u); }
    // rows, as in Two
    __device__ static uint32_t compose_word(uint32_t g, uint32_t f) { return kf_compose(g, f); }
    __device__ static uint32_t initial(const uint8_t *init, uint32_t id, uint32_t n_ids)
    {
        return KF_CONST | (init && id < n_ids ? init[id] & 15u : 1u);
    }
    __device__ static void put_final(uint32_t st, uint8_t *final_out, uint32_t id, uint32_t n_ids)
    {
        if (id < n_ids)
            final_out[id] = (uint8_t)(st & 15u);
    }
};

// steps whose reads share one wait: two over the 2^14 ids of a plain bucket, where they
// seldom meet, one over a k-space bucket's 2^12
constexpr int PAIR = 2, K_PAIR = 1;

// a chunk's bucket (cb), with a mark on a bucket's first chunk
constexpr uint32_t W_FIRST = 1u << 31, W_BUCKET = W_FIRST - 1;

struct BucketChunks {
    const uint32_t *ev;
    const uint64_t *base;
    const uint32_t *cbase, *cb;
    uint32_t nb, bits;
    uint64_t per;
    uint32_t row;
    __device__ OneChunk<BucketChunks> chunk(uint32_t c) const { return {*this, c}; }
    __device__ Control *report_to(Control *) const { return nullptr; } // (the histogram did)
    __device__ uint32_t count() const { return cbase[nb]; }
    __device__ uint32_t id_bits() const { return bits; }
    __device__ uint32_t local(uint32_t w) const { return w & ((1u << bits) - 1u); }
    __device__ uint32_t clamped(uint32_t w) const { return local(w); }
    __device__ uint64_t begin_of(uint32_t c) const
    {
        const uint32_t b = cb[c] & W_BUCKET;
        return base[b] + (uint64_t)(c - cbase[b]) * per;
    }
    __device__ uint64_t end_of(uint32_t c) const
    {
        const uint64_t e = begin_of(c) + per, last = base[(cb[c] & W_BUCKET) + 1];
        return e < last ? e : last;
    }
    __device__ bool bad(uint32_t) const { return false; } // (reported; its bits stay inside the table)
};

template <class R>
struct StatusOut {
    R *res;
    template <class CHUNKS>
    __device__ void begin(const CHUNKS &, uint32_t) const {}
    __device__ void step(uint32_t lane, uint32_t, uint64_t i, uint32_t, uint32_t st, bool valid) const
    {
        if (valid)
            res[i + lane] = (R)st;
    }
    __device__ void round(uint32_t, uint64_t, uint32_t, bool) const {}
    __device__ void chunk(uint32_t, const uint32_t *) const {}
};

// bases of the buckets' events and chunks, and every chunk's bucket
__global__ __launch_bounds__(1024) void k_wide_bases(const uint32_t *__restrict__ tot, uint32_t nb, uint64_t per,
                                                     uint64_t *__restrict__ base, uint32_t *__restrict__ cbase,
                                                     uint32_t *__restrict__ cb)
{
    __shared__ uint32_t s_t[1024];
    __shared__ uint64_t s_wa[1024 / WAVE];
    __shared__ uint32_t s_wt[1024 / WAVE];
    const uint32_t i = threadIdx.x, lane = lane_id(), wave = i / WAVE;
    const uint32_t c = i < nb ? tot[i] : 0, k = (uint32_t)ceil_div((uint64_t)c, per);
    const uint64_t ainc = wave_scan_add((uint64_t)c, lane);
    const uint32_t tinc = wave_scan_add(k, lane);
    if (lane == WAVE - 1) {
        s_wa[wave] = ainc;
        s_wt[wave] = tinc;
    }
    __syncthreads();
    uint64_t a0 = ainc - c;
    uint32_t t0 = tinc - k, chunks = 0;
    for (uint32_t w2 = 0; w2 < 1024 / WAVE; w2++) {
        a0 += w2 < wave ? s_wa[w2] : 0;
        t0 += w2 < wave ? s_wt[w2] : 0;
        chunks += s_wt[w2];
    }
    s_t[i] = t0 + k;
    if (i < nb) {
        base[i] = a0;
        cbase[i] = t0;
    }
    if (i == nb - 1) {
        base[nb] = a0 + c;
        cbase[nb] = t0 + k;
    }
    __syncthreads();
    // s_t: the first chunk after bucket i's; a chunk's bucket is the first that ends past it
    for (uint32_t q = i; q < chunks; q += 1024) {
        uint32_t lo = 0, hi = nb - 1;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) / 2;
            if (s_t[mid] > q)
                hi = mid;
            else
                lo = mid + 1;
        }
        cb[q] = lo | (q == (lo ? s_t[lo - 1] : 0u) ? W_FIRST : 0u);
    }
}

// Prefix over the rows by groups of W_GROUP chunks, as in the dense check; a group's row is
// the composition since the last bucket that starts in it.
constexpr uint32_t W_GROUP = 32, W_BATCH = 8;
static_assert(W_GROUP % W_BATCH == 0, "whole batches but for the last group's");

template <class D>
__global__ __launch_bounds__(BLOCK) void k_wide_groups(const uint32_t *__restrict__ rows, uint32_t row, uint32_t nb,
                                                       const uint32_t *__restrict__ cbase,
                                                       const uint32_t *__restrict__ cb, uint32_t *__restrict__ grp)
{
    const uint32_t w = blockIdx.x * BLOCK + threadIdx.x, g = blockIdx.y, chunks = cbase[nb];
    const uint32_t c0 = g * W_GROUP, c1 = c0 + W_GROUP < chunks ? c0 + W_GROUP : chunks;
    if (w >= row || c0 >= chunks)
        return;
    uint32_t f = D::ROW_IDENTITY;
    for (uint32_t q = c0; q < c1; q += W_BATCH) {
        uint32_t v[W_BATCH], b[W_BATCH]; // a batch's loads together
#pragma unroll
        for (uint32_t k = 0; k < W_BATCH; k++) {
            const uint32_t c = q + k < c1 ? q + k : c1 - 1;
            b[k] = cb[c];
            v[k] = rows[(uint64_t)c * row + w];
        }
#pragma unroll
        for (uint32_t k = 0; k < W_BATCH; k++)
            if (q + k < c1)
                f = (b[k] & W_FIRST) ? v[k] : D::compose_word(v[k], f);
    }
    grp[(uint64_t)g * row + w] = f;
}

template <class D>
__global__ __launch_bounds__(BLOCK) void k_wide_prefix(uint32_t *__restrict__ rows, uint32_t row, uint32_t nb,
                                                       const uint32_t *__restrict__ cbase,
                                                       const uint32_t *__restrict__ cb,
                                                       const uint32_t *__restrict__ grp, uint32_t n_ids, uint32_t bits,
                                                       const uint8_t *__restrict__ init,
                                                       uint8_t *__restrict__ final_out)
{
    const uint32_t w = blockIdx.x * BLOCK + threadIdx.x, g = blockIdx.y, chunks = cbase[nb];
    const uint32_t c0 = g * W_GROUP, c1 = c0 + W_GROUP < chunks ? c0 + W_GROUP : chunks;
    if (w >= row || c0 >= chunks)
        return;
    auto first_id = [&](uint32_t b) { return (b << bits) + w * D::IDS; };
    const uint32_t b0 = cb[c0] & W_BUCKET, first = cbase[b0];
    uint32_t st = D::initial(init, first_id(b0), n_ids);
    if (first < c0)
#pragma unroll 8
        for (uint32_t q = first / W_GROUP; q < g; q++)
            st = D::compose_word(grp[(uint64_t)q * row + w], st);
    for (uint32_t q = c0; q < c1; q += W_BATCH) {
        uint32_t v[W_BATCH], b[W_BATCH + 1];
#pragma unroll
        for (uint32_t k = 0; k < W_BATCH; k++) {
            const uint32_t c = q + k < c1 ? q + k : c1 - 1;
            b[k] = cb[c];
            v[k] = rows[(uint64_t)c * row + w];
        }
        b[W_BATCH] = q + W_BATCH < chunks ? cb[q + W_BATCH] : W_FIRST;
#pragma unroll
        for (uint32_t k = 0; k < W_BATCH; k++) {
            const uint32_t c = q + k;
            if (c >= c1)
                continue;
            if ((b[k] & W_FIRST) && c > c0)
                st = D::initial(init, first_id(b[k] & W_BUCKET), n_ids);
            rows[(uint64_t)c * row + w] = st;
            st = D::compose_word(v[k], st);
            if (c + 1 == chunks || ((c + 1 < c1 || k + 1 == W_BATCH ? b[k + 1] : cb[c + 1]) & W_FIRST))
                D::put_final(st, final_out, first_id(b[k] & W_BUCKET), n_ids); // the bucket's last chunk
        }
    }
}

size_t wide_lds(uint32_t row) { return ((size_t)row + 32) * 4; }

uint32_t groups_of(uint32_t max_chunks) { return (uint32_t)ceil_div(max_chunks, W_GROUP); }

} // namespace

// Chunks that fill the device (as many waves as have their tables in a CU's 160 KB, at most
// 24, on 256 CUs), of whole rounds of steps and long enough that a chunk's walk outweighs
// its row.
uint64_t wide_chunk_events(uint64_t n, uint32_t row)
{
    const uint64_t waves = 163840 / wide_lds(row), chunks = 256 * (waves > 24 ? 24 : waves);
    const uint64_t round = WAVE * D_UNROLL, per = ceil_div(n ? n : 1, chunks);
    return ceil_div(per, round) * round;
}

uint32_t wide_max_chunks(uint64_t n, uint32_t nb, uint64_t per) { return (uint32_t)(n / per) + nb; }

void launch_wide_bases(const WideChunks &W, hipStream_t s)
{
    ProfScope p(s, "wide_bases");
    k_wide_bases<<<1, 1024, 0, s>>>(W.tot, W.nb, W.per, W.base, W.cbase, W.cb);
}

uint32_t wide_row_events(uint32_t bits) { return (1u << bits) / Two::IDS; }
uint32_t wide_row_spaces(uint32_t bits) { return (1u << bits) / Spaces::IDS; }

size_t wide_rows_bytes(uint32_t max_chunks, uint32_t row)
{
    return ((size_t)max_chunks + groups_of(max_chunks)) * row * 4;
}

template <class D, int Q, class R>
static void wide_scan(const WideChunks &W, uint32_t row, const uint8_t *init, uint8_t *final_out, void *scratch, R *res,
                      Control *ctl, hipStream_t s)
{
    const uint32_t most = wide_max_chunks(W.n, W.nb, W.per), groups = groups_of(most);
    uint32_t *rows = (uint32_t *)scratch, *grp = rows + (size_t)most * row;
    const BucketChunks T{W.part, W.base, W.cbase, W.cb, W.nb, W.bits, W.per, row};
    const dim3 pg((unsigned)ceil_div(row, BLOCK), groups);
    {
        ProfScope p(s, "wide_fold");
        k_dense_fold<Fold<D>, Q, BucketChunks><<<most, WAVE, wide_lds(row), s>>>(T, row, rows, ctl, nullptr);
    }
    if (groups > 1) {
        ProfScope p(s, "wide_groups");
        k_wide_groups<D><<<pg, BLOCK, 0, s>>>(rows, row, W.nb, W.cbase, W.cb, grp);
    }
    {
        ProfScope p(s, "wide_prefix");
        k_wide_prefix<D><<<pg, BLOCK, 0, s>>>(rows, row, W.nb, W.cbase, W.cb, grp, W.n_ids, W.bits, init, final_out);
    }
    ProfScope p(s, "wide_apply");
    k_dense_apply<Apply<D>, Q, BucketChunks, StatusOut<R>><<<most, WAVE, wide_lds(row), s>>>(T, row, rows, StatusOut<R>{res});
}

void launch_wide_scan_events(const WideChunks &W, const uint8_t *init, uint8_t *final_out, void *rows, uint8_t *res,
                             Control *ctl, hipStream_t s)
{
    wide_scan<Two, PAIR>(W, wide_row_events(W.bits), init, final_out, rows, res, ctl, s);
}

void launch_wide_scan_spaces(const WideChunks &W, const uint8_t *init, uint8_t *final_out, void *rows, uint16_t *res,
                             Control *ctl, hipStream_t s)
{
    wide_scan<Spaces, K_PAIR>(W, wide_row_spaces(W.bits), init, final_out, rows, res, ctl, s);
}

} // namespace vc
