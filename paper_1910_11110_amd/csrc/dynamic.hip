// dynamic.hip -- partial vectors created and destroyed during a trace (gfx950).
//
// The registry of a vector's live partial vectors (Section 4.3, "Towards an
// implementation in VectorPU") is not kept as a sequential structure: every array's
// lifetime is read off the trace at once (the position of its create and destroy
// events), the overlap sets of all arrays come from the interval sweep, and an array y
// belongs to the registry at position t exactly when its lifetime contains t.  So a
// write at t induces RW on the neighbours of its array whose lifetime contains t, and
// the liveness rules of every event are checked in parallel against the lifetimes.
//
// A created partial vector inherits its mother's status (appendix "Partial
// Vectors").  That status depends only on the mother's own events and on the induced
// writes it receives, never on a partial vector's status, so the check runs the
// segmented scan twice on the same sorted items: first for the statuses before
// "probe" items placed on the mother's segment at every creation (the inherited
// statuses), then, with those as the created arrays' initial statuses, for every
// status byte and the final table.  (The dense check finds the functions that the probes
// see while it composes its chunks', and needs no first scan.)
#include "dense.h"
#include "device.h"
#include "internal.h"
#include "prof.h"

namespace vc {

constexpr uint32_t OP_CREATE = 6, OP_DESTROY = 7;
constexpr uint32_t NO_POS = 0xFFFFFFFFu;
constexpr uint32_t NO_MOTHER = 0xFFFFFFFFu;

namespace {

__device__ __forceinline__ void report_bad(Control *ctl, uint64_t i)
{
    atomicMin(reinterpret_cast<unsigned long long *>(&ctl->err_index_lo), (unsigned long long)i);
}

// a well-formed word of a dynamic trace: ops 0-4, or create / destroy on side 0
__device__ __forceinline__ bool word_ok(uint32_t e, uint32_t n_ids)
{
    const uint32_t op = (e >> 24) & 7u;
    return (e >> 28) == 0 && op != OP_RWIND && (e & 0xFFFFFFu) < n_ids && (op < OP_CREATE || ((e >> 27) & 1u) == 0);
}

__global__ void k_dyn_clear(uint32_t *cpos, uint32_t *dpos, uint32_t n_ids)
{
    for (uint32_t x = blockIdx.x * blockDim.x + threadIdx.x; x < n_ids; x += gridDim.x * blockDim.x) {
        cpos[x] = NO_POS;
        dpos[x] = NO_POS;
    }
}

// first create and first destroy position of every array
__global__ void k_dyn_life(const uint32_t *__restrict__ ev, uint64_t n, uint32_t n_ids, uint32_t *cpos,
                           uint32_t *dpos)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += stride) {
        const uint32_t e = ev[t], op = (e >> 24) & 7u, x = e & 0xFFFFFFu;
        if (!word_ok(e, n_ids))
            continue;
        if (op == OP_CREATE)
            atomicMin(&cpos[x], (uint32_t)t);
        else if (op == OP_DESTROY)
            atomicMin(&dpos[x], (uint32_t)t);
    }
}

// a lifetime as it is asked: live at t when x <= t < y
__device__ __forceinline__ bool life_holds(uint2 lf, uint64_t t)
{
    return lf.x <= (uint32_t)t && (uint32_t)t < lf.y; // (t < 2^30)
}

// lifetimes of every entry of the overlap CSR, so that the neighbours of a write read
// theirs in order instead of gathering them, and then of every array
__global__ void k_dyn_nbr_life(const uint32_t *__restrict__ nbr, uint64_t n_nbr, uint32_t n_ids,
                               const uint32_t *__restrict__ cpos, const uint32_t *__restrict__ dpos,
                               uint2 *__restrict__ life)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n_nbr + n_ids; j += stride) {
        const uint32_t y = j < n_nbr ? nbr[j] : (uint32_t)(j - n_nbr);
        const uint32_t c = cpos[y];
        life[j] = make_uint2(c == NO_POS ? 0u : c + 1, dpos[y]);
    }
}

// The combined items by wave tiles of DTILE events: each event, a probe on its mother (a
// partial vector's create) and, at a write, an induced RW item on every neighbour of its
// array that is live at the write.  A count pass checks the events, finds the live
// neighbours of their writes and leaves the number of items of every event and tile and,
// where they fit, the live ones' bits; the emit pass, with the tiles' scanned positions,
// writes the items.  A write's neighbours are looked at after the tile's events: of a write
// with at most D_SMALL by one lane, 64 writes together, of one with more by the whole wave,
// 64 neighbours a step and several steps' loads issued together.
// Bound by the requests of the gathers and scattered stores and, nearly half of the time,
// by vector instructions.  2^23 events over 1,024 vectors and 64,512 partial vectors (50 M
// neighbours of writes, 25 M of them live): walking the neighbours 64 consecutive ones at a
// time in both passes, with a search for the event of each, took 200 and 266 us; both in
// one pass behind a look-back over its workgroups 310 (their polls, from 8 dies, cost more
// than the second reading); this way 118 and 147.
constexpr int D_PER = 8;                   // events per lane
constexpr uint32_t DTILE = WAVE * D_PER;   // events per wave tile
constexpr uint32_t DWAVES = BLOCK / WAVE;
constexpr uint32_t D_SMALL = 24;           // neighbours one lane looks at
constexpr int D_AHEAD = 4;                 // neighbours a lane looks at together
constexpr int D_WAHEAD = 8;                // writes the wave looks at together

struct __attribute__((packed, aligned(8))) Bounds { // two entries of the neighbours' offsets
    uint64_t begin, end;
};

// a wave tile: its events' words (D_PROBE: a probe follows), their items (later
// where these start), and its writes with neighbours (from the front of `list` those with
// few, from its back the others) with their number and the bits of the live ones
constexpr uint32_t D_PROBE = 1u << 30;
struct DynTile {
    uint32_t word[DTILE], items[DTILE];
    uint32_t deg[DTILE]; // count: of a write, its neighbours; emit: what the count pass left
    uint16_t list[DTILE];
};
static_assert(D_SMALL < 30, "a bit each beside the mark");

__device__ __forceinline__ void wave_lds_fence() { asm volatile("" ::: "memory"); } // (a wave's LDS operations are in order)
__device__ __forceinline__ uint32_t lane32(uint32_t v, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ uint64_t lane64(uint32_t lo, uint32_t hi, int l)
{
    return ((uint64_t)lane32(hi, l) << 32) | lane32(lo, l);
}

// 64 writes with more than D_SMALL neighbours, one a lane: the event, where its neighbours
// start and their number, and the bits of the first 128 live ones
struct Writes {
    uint32_t k, deg, count;
    uint32_t o_lo, o_hi, live[4];
    __device__ __forceinline__ void take(const DynTile &T, uint32_t i0, uint32_t many, const uint64_t *__restrict__ off,
                                         uint32_t lane)
    {
        k = T.list[DTILE - 1 - (i0 + lane < many ? i0 + lane : many - 1)];
        const Bounds at = *reinterpret_cast<const Bounds *>(off + (T.word[k] & 0xFFFFFFu));
        deg = (uint32_t)(at.end - at.begin);
        o_lo = (uint32_t)at.begin;
        o_hi = (uint32_t)(at.begin >> 32);
        count = 0;
    }
    __device__ __forceinline__ uint64_t first(int l) const { return lane64(o_lo, o_hi, l); }
    __device__ __forceinline__ uint64_t bits(int l, int h) const { return lane64(live[2 * h], live[2 * h + 1], l); }
    // the live neighbours of the first cnt writes: their number and bits
    __device__ __forceinline__ void look(uint32_t cnt, uint64_t t0, const uint2 *__restrict__ life, uint32_t lane)
    {
        for (uint32_t i = 0; i < cnt; i += D_WAHEAD) {
            uint32_t d[D_WAHEAD];
            uint2 v[D_WAHEAD][2];
#pragma unroll
            for (int u = 0; u < D_WAHEAD; u++) {
                const int l = (int)(i + u < cnt ? i + u : cnt - 1);
                d[u] = lane32(deg, l);
                const uint2 *p = life + first(l);
                v[u][0] = v[u][1] = make_uint2(~0u, 0);
                if (lane < d[u])
                    v[u][0] = p[lane];
                if (lane + WAVE < d[u])
                    v[u][1] = p[lane + WAVE];
            }
#pragma unroll
            for (int u = 0; u < D_WAHEAD; u++) {
                const int l = (int)(i + u < cnt ? i + u : cnt - 1);
                const uint64_t t = t0 + lane32(k, l);
                const uint64_t a = __ballot(life_holds(v[u][0], t)), b = __ballot(life_holds(v[u][1], t));
                uint32_t c = (uint32_t)__builtin_popcountll(a) + (uint32_t)__builtin_popcountll(b);
                for (uint32_t q = 2 * WAVE; q < d[u]; q += WAVE) // uniform, and rare
                    c += (uint32_t)__builtin_popcountll(__ballot(
                        q + lane < d[u] && life_holds(life[first(l) + (q + lane < d[u] ? q + lane : 0)], t)));
                const bool me = lane == (uint32_t)l;
                count = me ? c : count;
                live[0] = me ? (uint32_t)a : live[0];
                live[1] = me ? (uint32_t)(a >> 32) : live[1];
                live[2] = me ? (uint32_t)b : live[2];
                live[3] = me ? (uint32_t)(b >> 32) : live[3];
            }
        }
    }
};

// what the count pass leaves of an event: its items (E_MANY: a write with many neighbours),
// or of a write with few neighbours the live ones' bits
constexpr uint32_t E_FEW = 1u << 31, E_MANY = 1u << 30;
__device__ __forceinline__ uint32_t items_of(uint32_t e)
{
    return (e & E_FEW) ? 1u + (uint32_t)__builtin_popcount(e & ~E_FEW) : e & ~E_MANY;
}

// the items of every event (left) and tile (tcnt), and the bits of the live ones among the
// first 128 neighbours of a tile's first 64 writes with many (bits, 4 words a lane)
__global__ __launch_bounds__(BLOCK) void k_dyn_count(const uint32_t *__restrict__ ev, uint64_t n, uint32_t n_ids,
                                                     const uint32_t *__restrict__ mother,
                                                     const uint64_t *__restrict__ off,
                                                     const uint2 *__restrict__ life, const uint2 *__restrict__ own,
                                                     uint64_t ntiles, uint32_t *__restrict__ left,
                                                     uint4 *__restrict__ bits, uint32_t *__restrict__ tcnt, Control *ctl)
{
    __shared__ DynTile s_tiles[DWAVES];
    const uint32_t lane = lane_id(), wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const uint64_t tile = (uint64_t)blockIdx.x * DWAVES + wv, i0 = tile * DTILE;
    if (tile >= ntiles)
        return; // whole waves; no workgroup barriers below
    DynTile &T = s_tiles[wv];
    // ---- the events: their words, lifetimes and neighbours' bounds, each loaded together.
    // Malformed words and liveness errors are reported at their index (the smallest one
    // is the first error of a sequential reading) and have only the event itself.
    uint32_t w[D_PER], few = 0, many = 0;
#pragma unroll
    for (int j = 0; j < D_PER; j++) {
        const uint64_t t = i0 + j * WAVE + lane;
        w[j] = t < n ? ev[t] : (uint32_t)OP_NOOP << 24;
    }
    uint2 lf[D_PER];
    uint32_t bad = 0; // bit j
#pragma unroll
    for (int j = 0; j < D_PER; j++) {
        const bool ok = word_ok(w[j], n_ids);
        bad |= ok || i0 + j * WAVE + lane >= n ? 0u : 1u << j;
        w[j] = ok ? w[j] : (uint32_t)OP_NOOP << 24;
        lf[j] = own[w[j] & 0xFFFFFFu];
    }
    Bounds at[D_PER];
#pragma unroll
    for (int j = 0; j < D_PER; j++) {
        at[j] = Bounds{0, 0};
        if (((w[j] >> 24) & 7u) == OP_W)
            at[j] = *reinterpret_cast<const Bounds *>(off + (w[j] & 0xFFFFFFu));
    }
#pragma unroll
    for (int j = 0; j < D_PER; j++) {
        const uint32_t k = j * WAVE + lane, op = (w[j] >> 24) & 7u;
        const uint64_t t = i0 + k;
        const bool in = t < n;
        bool wrong, probe = false;
        if (__ballot(op >= OP_CREATE)) { // (uniform, and rare)
            wrong = !life_holds(lf[j], t);
            if (op == OP_CREATE) {
                const uint32_t m = mother[w[j] & 0xFFFFFFu];
                probe = m != NO_MOTHER;
                wrong = lf[j].x != (uint32_t)t + 1 || (probe && !life_holds(own[m], t));
            } else if (op == OP_DESTROY) {
                wrong = lf[j].y != (uint32_t)t || lf[j].x > (uint32_t)t;
            }
        } else {
            wrong = !life_holds(lf[j], t);
        }
        if (!in || ((bad >> j) & 1u)) // (a malformed word is no event on its array)
            wrong = false;
        bad |= wrong ? 1u << j : 0u;
        probe = probe && !wrong;
        const uint32_t deg = wrong ? 0u : (uint32_t)(at[j].end - at[j].begin); // (0 but for writes)
        const bool f = deg != 0 && deg <= D_SMALL, m = deg > D_SMALL;
        const uint64_t fm = __ballot(f), mm = __ballot(m);
        T.word[k] = w[j] | (probe ? D_PROBE : 0u);
        T.items[k] = in ? 1u + (probe ? 1u : 0u) : 0u;
        T.deg[k] = deg;
        if (f)
            T.list[few + mask_rank(fm)] = (uint16_t)k;
        if (m)
            T.list[DTILE - 1 - (many + mask_rank(mm))] = (uint16_t)k;
        few += (uint32_t)__builtin_popcountll(fm);
        many += (uint32_t)__builtin_popcountll(mm);
    }
    if (bad)
        report_bad(ctl, i0 + (uint32_t)__builtin_ctz(bad) * WAVE + lane);
    wave_lds_fence();
    // ---- live neighbours of the writes with few
    for (uint32_t i = lane; i < few; i += WAVE) {
        const uint32_t k = T.list[i], deg = T.deg[k];
        const uint64_t o = off[T.word[k] & 0xFFFFFFu];
        uint32_t live = 0;
        for (uint32_t q = 0; q < deg; q += D_AHEAD) {
            uint2 lf[D_AHEAD];
#pragma unroll
            for (int u = 0; u < D_AHEAD; u++)
                lf[u] = life[o + (q + u < deg ? q + u : deg - 1)];
#pragma unroll
            for (int u = 0; u < D_AHEAD; u++)
                live |= q + u < deg && life_holds(lf[u], i0 + k) ? 1u << (q + u) : 0u;
        }
        T.items[k] = E_FEW | live;
    }
    // ---- and of the others, 64 at a time
    for (uint32_t i0w = 0; i0w < many; i0w += WAVE) {
        Writes W;
        W.take(T, i0w, many, off, lane);
        W.look(many - i0w < WAVE ? many - i0w : WAVE, i0, life, lane);
        if (i0w + lane < many)
            T.items[W.k] = E_MANY | (1u + W.count);
        if (i0w == 0 && lane < many)
            bits[tile * WAVE + lane] = make_uint4(W.live[0], W.live[1], W.live[2], W.live[3]);
    }
    wave_lds_fence();
    uint32_t total = 0;
#pragma unroll
    for (int j = 0; j < D_PER; j++) {
        const uint32_t k = j * WAVE + lane, c = T.items[k];
        if (i0 + k < n)
            left[i0 + k] = c;
        total += items_of(c);
    }
    total = wave_total_u32(total);
    if (lane == 0)
        tcnt[tile] = total;
}

__device__ __forceinline__ uint32_t below(uint32_t n) { return n < 32 ? (1u << n) - 1u : ~0u; } // the lowest n bits

// MODE: D_ITEMS: 64-bit sort items from tpos[tile] on (cap at most; probes carry payload
// n + t, induced items INDUCED_BIT).  D_WORDS: words for the bucket engine (a create, a
// destroy and a probe are no-ops on their array, induced items op 5) and over left[t] event
// t's position.  D_DENSE: words for the dense check, probes of their own op, and the
// creates' positions.
enum { D_ITEMS, D_WORDS, D_DENSE };
template <int MODE>
__global__ __launch_bounds__(BLOCK) void k_dyn_emit(const uint32_t *__restrict__ ev, uint64_t n, uint32_t n_ids,
                                                    const uint32_t *__restrict__ mother,
                                                    const uint64_t *__restrict__ off,
                                                    const uint2 *__restrict__ life,
                                                    const uint32_t *__restrict__ nbr, uint64_t ntiles,
                                                    const uint64_t *__restrict__ tpos, uint32_t *left,
                                                    const uint4 *__restrict__ bits, void *__restrict__ out, uint64_t cap,
                                                    Control *ctl)
{
    __shared__ DynTile s_tiles[DWAVES];
    const uint32_t lane = lane_id(), wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const uint64_t tile = (uint64_t)blockIdx.x * DWAVES + wv, i0 = tile * DTILE;
    if (tile >= ntiles)
        return; // whole waves; no workgroup barriers below
    DynTile &T = s_tiles[wv];
    const uint64_t base = tpos[tile];
    // ---- the events' words and items, and their writes' neighbours
    uint32_t w[D_PER], c[D_PER], few = 0, many = 0, total = 0;
#pragma unroll
    for (int j = 0; j < D_PER; j++) {
        const uint64_t t = i0 + j * WAVE + lane;
        w[j] = t < n ? ev[t] : (uint32_t)OP_NOOP << 24;
        c[j] = t < n ? left[t] : 0u;
    }
#pragma unroll
    for (int j = 0; j < D_PER; j++) {
        w[j] = word_ok(w[j], n_ids) ? w[j] : (uint32_t)OP_NOOP << 24; // (a malformed one was reported)
        const uint32_t k = j * WAVE + lane, op = (w[j] >> 24) & 7u;
        const bool f = op == OP_W && c[j] > E_FEW, m = op == OP_W && !(c[j] & E_FEW) && (c[j] & E_MANY);
        const uint64_t fm = __ballot(f), mm = __ballot(m);
        const uint32_t it = items_of(c[j]), inc = wave_scan_add(it, lane);
        T.word[k] = w[j] | (op == OP_CREATE && c[j] > 1 ? D_PROBE : 0u);
        T.items[k] = total + inc - it;
        T.deg[k] = c[j];
        total += (uint32_t)__builtin_amdgcn_readlane((int)inc, WAVE - 1);
        if (f)
            T.list[few + mask_rank(fm)] = (uint16_t)k;
        if (m)
            T.list[DTILE - 1 - (many + mask_rank(mm))] = (uint16_t)k;
        few += (uint32_t)__builtin_popcountll(fm);
        many += (uint32_t)__builtin_popcountll(mm);
    }
    wave_lds_fence();
    // ---- the items (past the capacity: the events changed since they were sized)
    const uint32_t room = base < cap ? (uint32_t)(cap - base < total ? cap - base : total) : 0u;
    if (room < total)
        for (uint32_t k = lane; k < DTILE; k += WAVE)
            if (T.items[k] <= room && room < (k + 1 < DTILE ? T.items[k + 1] : total))
                report_bad(ctl, i0 + k);
    if (lane == 0 && base + total != tpos[tile + 1])
        report_bad(ctl, i0); // the events changed since the items were counted
    uint64_t *const items = reinterpret_cast<uint64_t *>(out) + base;
    uint32_t *const words = reinterpret_cast<uint32_t *>(out) + base;
    auto induced = [&](uint32_t p, uint32_t y, uint32_t head) { // (head: op and side)
        if (p >= room)
            return;
        if (MODE == D_ITEMS)
            items[p] = make_item(y, fcode(OP_RWIND, (head >> 27) & 1u), INDUCED_BIT);
        else
            words[p] = y | head;
    };
#pragma unroll
    for (int j = 0; j < D_PER; j++) {
        const uint32_t k = j * WAVE + lane;
        const uint64_t t = i0 + k;
        if (t >= n)
            continue;
        const uint32_t w = T.word[k], p = T.items[k];
        const uint32_t op = (w >> 24) & 7u, x = w & 0xFFFFFFu, side = (w >> 27) & 1u;
        if (p < room) {
            if (MODE == D_ITEMS)
                items[p] = make_item(x, op >= OP_CREATE ? fcode(OP_NOOP, 0) : fcode(op, side), (uint32_t)t);
            else
                words[p] = x | (op >= OP_CREATE ? (uint32_t)OP_NOOP << 24 : (w & (15u << 24)));
        }
        if (op == OP_CREATE || MODE == D_WORDS)
            if (MODE != D_ITEMS)
                left[t] = (uint32_t)base + p; // below 2^32 on these routes
        if ((w & D_PROBE) && p + 1 < room) {
            const uint32_t m = mother[x];
            if (MODE == D_ITEMS)
                items[p + 1] = make_item(m, fcode(OP_NOOP, 0), (uint32_t)(n + t));
            else
                words[p + 1] = m | (MODE == D_DENSE ? DENSE_OP_PROBE : (uint32_t)OP_NOOP) << 24;
        }
    }
    for (uint32_t i = lane; i < few; i += WAVE) {
        const uint32_t k = T.list[i], w = T.word[k];
        const Bounds at = *reinterpret_cast<const Bounds *>(off + (w & 0xFFFFFFu));
        const uint64_t o = at.begin;
        uint32_t p = T.items[k] + 1, live = T.deg[k] & below((uint32_t)(at.end - o) < D_SMALL ? (uint32_t)(at.end - o) : D_SMALL);
        while (live) {
            uint32_t y[D_AHEAD], c = 0;
#pragma unroll
            for (int u = 0; u < D_AHEAD; u++)
                if (live) {
                    y[u] = nbr[o + __builtin_ctz(live)];
                    live &= live - 1;
                    c++;
                }
#pragma unroll
            for (int u = 0; u < D_AHEAD; u++)
                if (u < (int)c)
                    induced(p + u, y[u], OP_RWIND << 24 | (w & (1u << 27)));
            p += c;
        }
    }
    for (uint32_t i0w = 0; i0w < many; i0w += WAVE) {
        const uint32_t cnt = many - i0w < WAVE ? many - i0w : WAVE;
        Writes W0;
        W0.take(T, i0w, many, off, lane);
        if (i0w == 0) {
            const uint4 b = bits[tile * WAVE + (lane < many ? lane : many - 1)];
            // (inside its neighbours, whatever became of the event since)
            W0.live[0] = b.x & below(W0.deg);
            W0.live[1] = b.y & below(W0.deg > 32 ? W0.deg - 32 : 0);
            W0.live[2] = b.z & below(W0.deg > 64 ? W0.deg - 64 : 0);
            W0.live[3] = b.w & below(W0.deg > 96 ? W0.deg - 96 : 0);
        } else { // (looked at again)
            W0.look(cnt, i0, life, lane);
        }
        const uint32_t start = T.items[W0.k] + 1, head = OP_RWIND << 24 | (T.word[W0.k] & (1u << 27));
        for (uint32_t i = 0; i < cnt; i += D_WAHEAD) {
            uint32_t y[D_WAHEAD][2];
#pragma unroll
            for (int u = 0; u < D_WAHEAD; u++) {
                const int l = (int)(i + u < cnt ? i + u : cnt - 1);
                const uint32_t *p = nbr + W0.first(l);
                y[u][0] = y[u][1] = 0;
                if (__builtin_amdgcn_inverse_ballot_w64(W0.bits(l, 0)))
                    y[u][0] = p[lane];
                if (__builtin_amdgcn_inverse_ballot_w64(W0.bits(l, 1)))
                    y[u][1] = p[WAVE + lane];
            }
#pragma unroll
            for (int u = 0; u < D_WAHEAD; u++) {
                if (i + u >= cnt)
                    break; // uniform
                const int l = (int)(i + u);
                const uint32_t h = lane32(head, l), deg = lane32(W0.deg, l);
                uint32_t p = lane32(start, l);
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    const uint64_t m = W0.bits(l, q);
                    if (__builtin_amdgcn_inverse_ballot_w64(m))
                        induced(p + mask_rank(m), y[u][q], h);
                    p += (uint32_t)__builtin_popcountll(m);
                }
                for (uint32_t q = 2 * WAVE; q < deg; q += WAVE) { // uniform, and rare
                    const uint64_t at = W0.first(l) + (q + lane < deg ? q + lane : 0);
                    const uint64_t m = __ballot(q + lane < deg && life_holds(life[at], i0 + lane32(W0.k, l)));
                    if (__builtin_amdgcn_inverse_ballot_w64(m))
                        induced(p + mask_rank(m), nbr[at], h);
                    p += (uint32_t)__builtin_popcountll(m);
                }
            }
        }
    }
}

// initial statuses of the second scan: a created partial vector starts at the status
// its mother had at the creation (the probe's pre-status); every other array at its
// initial status (init, or (V,I))
__global__ void k_dyn_inherit(const uint32_t *__restrict__ mother, const uint32_t *__restrict__ cpos,
                              const uint8_t *__restrict__ probe_pre, uint64_t n, const uint8_t *__restrict__ init,
                              uint32_t n_ids, uint8_t *__restrict__ init2, uint8_t *__restrict__ fin)
{
    for (uint32_t x = blockIdx.x * blockDim.x + threadIdx.x; x < n_ids; x += gridDim.x * blockDim.x) {
        const uint32_t c = cpos[x];
        uint8_t s = init ? init[x] : (uint8_t)1;
        if (c != NO_POS && c < n && mother[x] != NO_MOTHER)
            s = probe_pre[n + c];
        init2[x] = s;
        fin[x] = s;
    }
}

// the same from the words' pre-statuses (bits 0-1 of pre[i], through dstidx[i] when it
// is given): a create's probe sits right after the create, at pos32[c] + 1
__global__ void k_dyn_inherit_words(const uint32_t *__restrict__ mother, const uint32_t *__restrict__ cpos,
                                    const uint8_t *__restrict__ pre, const uint32_t *__restrict__ dstidx,
                                    const uint32_t *__restrict__ pos32, uint64_t n, uint64_t m,
                                    const uint8_t *__restrict__ init, uint32_t n_ids, uint8_t *__restrict__ init2,
                                    uint8_t *__restrict__ fin)
{
    for (uint32_t x = blockIdx.x * blockDim.x + threadIdx.x; x < n_ids; x += gridDim.x * blockDim.x) {
        const uint32_t c = cpos[x];
        uint8_t s = init ? init[x] : (uint8_t)1;
        if (c != NO_POS && c < n && mother[x] != NO_MOTHER) {
            uint64_t p = (uint64_t)pos32[c] + 1;
            p = p < m ? p : m - 1;
            if (dstidx) {
                p = dstidx[p];
                p = p < m ? p : m - 1; // (in range for consistent counts)
            }
            s = (uint8_t)(pre[p] & 3u);
        }
        init2[x] = s;
        fin[x] = s;
    }
}

// the same from the functions that the probes see (pre, at a create's position + 1) and the
// statuses entering the create's chunk
__global__ void k_dyn_inherit_dense(const uint32_t *__restrict__ mother, const uint32_t *__restrict__ cpos,
                                    const uint8_t *__restrict__ pre, const uint32_t *__restrict__ pos32, uint64_t n,
                                    uint64_t m, DenseEntering E, const uint8_t *__restrict__ init, uint32_t n_ids,
                                    uint8_t *__restrict__ init2)
{
    for (uint32_t x = blockIdx.x * blockDim.x + threadIdx.x; x < n_ids; x += gridDim.x * blockDim.x) {
        const uint32_t c = cpos[x], mo = mother[x];
        uint8_t s = init ? init[x] : (uint8_t)1;
        if (c != NO_POS && c < n && mo != NO_MOTHER) {
            const uint64_t p = (uint64_t)pos32[c] + 1;
            const uint32_t f = pre[p < m ? p : m - 1];
            const uint32_t h = (E.rows[c / DTILE / E.per * E.row + (mo >> 3)] >> (3 * (mo & 7u))) & 3u;
            // f of h: a constant, or the copies valid before and those a transfer makes valid
            s = (uint8_t)((f & 4u) ? f & 3u : h | (f & (h >> 1) & 1u) | ((f & (h << 1)) & 2u));
        }
        init2[x] = s;
    }
}

unsigned grid_of(uint64_t n, unsigned per = BLOCK * 4)
{
    uint64_t g = ceil_div(n ? n : 1, per);
    return (unsigned)(g > 8192 ? 8192 : g);
}

} // namespace

void launch_dyn_life(const uint32_t *ev, uint64_t n, uint32_t n_ids, uint32_t *cpos, uint32_t *dpos, hipStream_t s)
{
    {
        ProfScope p(s, "dyn_clear");
        k_dyn_clear<<<grid_of(n_ids), BLOCK, 0, s>>>(cpos, dpos, n_ids);
    }
    if (n) {
        ProfScope p(s, "dyn_life");
        k_dyn_life<<<grid_of(n), BLOCK, 0, s>>>(ev, n, n_ids, cpos, dpos);
    }
}

uint32_t dyn_tile_events() { return DTILE; }

uint64_t dyn_tiles(uint64_t n) { return ceil_div(n, (uint64_t)DTILE); }

void launch_dyn_near(const OverlapSets *o, uint32_t n_ids, const uint32_t *cpos, const uint32_t *dpos, uint2 *life,
                     hipStream_t s)
{
    ProfScope p(s, "dyn_nbr_life");
    k_dyn_nbr_life<<<grid_of(o->n_nbr + n_ids), BLOCK, 0, s>>>(o->nbr, o->n_nbr, n_ids, cpos, dpos, life);
}

size_t dyn_bits_bytes(uint64_t n) { return dyn_tiles(n) * WAVE * sizeof(uint4); }

void launch_dyn_count(const DynTrace &D, uint32_t *left, void *bits, uint32_t *tcnt, Control *ctl, hipStream_t s)
{
    const uint64_t ntiles = dyn_tiles(D.n);
    if (ntiles) {
        ProfScope p(s, "dyn_count");
        k_dyn_count<<<(unsigned)ceil_div(ntiles, (uint64_t)DWAVES), BLOCK, 0, s>>>(
            D.ev, D.n, D.n_ids, D.mother, D.sets->off, D.life, D.life + D.sets->n_nbr, ntiles, left, (uint4 *)bits, tcnt,
            ctl);
    }
}

namespace {

template <int MODE>
void launch_emit(const DynTrace &D, const uint64_t *tpos, uint32_t *left, const void *bits, void *out, uint64_t cap,
                 Control *ctl, hipStream_t s)
{
    const uint64_t ntiles = dyn_tiles(D.n);
    if (ntiles) {
        ProfScope p(s, "dyn_emit");
        k_dyn_emit<MODE><<<(unsigned)ceil_div(ntiles, (uint64_t)DWAVES), BLOCK, 0, s>>>(
            D.ev, D.n, D.n_ids, D.mother, D.sets->off, D.life, D.sets->nbr, ntiles, tpos, left, (const uint4 *)bits, out,
            cap, ctl);
    }
}

} // namespace

void launch_dyn_items(const DynTrace &D, const uint64_t *tpos, uint32_t *left, const void *bits, uint64_t *items,
                      uint64_t cap, Control *ctl, hipStream_t s)
{
    launch_emit<D_ITEMS>(D, tpos, left, bits, items, cap, ctl, s);
}

void launch_dyn_words(const DynTrace &D, bool dense, const uint64_t *tpos, uint32_t *left, const void *bits,
                      uint32_t *words, uint64_t cap, Control *ctl, hipStream_t s)
{
    if (dense)
        launch_emit<D_DENSE>(D, tpos, left, bits, words, cap, ctl, s);
    else
        launch_emit<D_WORDS>(D, tpos, left, bits, words, cap, ctl, s);
}

void launch_dyn_inherit_words(const uint32_t *mother, const uint32_t *cpos, const uint8_t *pre, const uint32_t *dstidx,
                              const uint32_t *pos32, uint64_t n, uint64_t m, const uint8_t *init, uint32_t n_ids,
                              uint8_t *init2, uint8_t *fin, hipStream_t s)
{
    ProfScope p(s, "dyn_inherit");
    k_dyn_inherit_words<<<grid_of(n_ids), BLOCK, 0, s>>>(mother, cpos, pre, dstidx, pos32, n, m ? m : 1, init, n_ids,
                                                         init2, fin);
}

void launch_dyn_inherit_dense(const uint32_t *mother, const uint32_t *cpos, const uint8_t *pre, const uint32_t *pos32,
                              uint64_t n, uint64_t m, const DenseEntering &E, const uint8_t *init, uint32_t n_ids,
                              uint8_t *init2, hipStream_t s)
{
    ProfScope p(s, "dyn_inherit");
    k_dyn_inherit_dense<<<grid_of(n_ids), BLOCK, 0, s>>>(mother, cpos, pre, pos32, n, m ? m : 1, E, init, n_ids, init2);
}

void launch_dyn_inherit(const uint32_t *mother, const uint32_t *cpos, const uint8_t *probe_pre, uint64_t n,
                        const uint8_t *init, uint32_t n_ids, uint8_t *init2, uint8_t *fin, hipStream_t s)
{
    ProfScope p(s, "dyn_inherit");
    k_dyn_inherit<<<grid_of(n_ids), BLOCK, 0, s>>>(mother, cpos, probe_pre, n, init, n_ids, init2, fin);
}

} // namespace vc
