// dense_steps.h -- 64 events at a time on a table of all ids' functions or statuses in LDS
// (one wave; used by the dense and the wide check).
//
// A domain says what a table word holds: Two, the two memory spaces, 8 ids a word; its
// functions are passed between lanes in 4-byte form.  Fold walks events backwards and
// composes every id's function, Apply walks them forwards on the ids' statuses.
#pragma once
#include "device.h"
#include "internal.h"

namespace vc {
namespace {

// ----------------------------------------------------------------------------------
// Table words: 8 ids of 3 bits and, in the top byte, a touch bit for each (zero between
// steps).  An id's bits are a monoid element: bit 2 a constant, whose status is bits 0
// (CPU copy valid) and 1 (GPU); else bit 0 "CPU |= GPU" and bit 1 "GPU |= CPU".
// ----------------------------------------------------------------------------------
constexpr uint32_t T_TOUCH = 1u << 24;
constexpr uint32_t MX = 011111111u, MY = MX << 1, MT = MX << 2;

// h o f (f first), 8 ids at once (counters zero)
__device__ __forceinline__ uint32_t tw_compose(uint32_t h, uint32_t f)
{
    const uint32_t ftx = (f >> 2) & MX, htx = (h >> 2) & MX;
    const uint32_t ex = f | (h & (~ftx | (f >> 1)));
    const uint32_t ey = f | (h & (~(ftx << 1) | (f << 1)));
    const uint32_t hx = htx | (htx << 1); // fields that h makes constant
    return ((h | f) & MT) | (((h & hx) | (((ex & MX) | (ey & MY)) & ~hx)));
}

// the same on one id's 3 bits
__device__ __forceinline__ uint32_t el_compose(uint32_t h, uint32_t f)
{
    const uint32_t ft = f >> 2;
    const uint32_t ex = f | (h & ((ft ^ 1u) | (f >> 1)));
    const uint32_t ey = f | (h & (((ft ^ 1u) << 1) | (f << 1)));
    const uint32_t r = ((h | f) & 4u) | (ex & 1u) | (ey & 2u);
    return (h & 4u) ? h : r;
}

// Per (op | side << 3): an effect's element; for the backward walk the element h o f for
// every h, 3 bits each; for the forward walk the status byte for every status before the
// event, 8 bits each.  In constant memory, copied to LDS by every wave.
constexpr uint32_t host_compose(uint32_t h, uint32_t f)
{
    if (h & 4u)
        return h;
    const uint32_t x = (f & 1u) | ((h & 1u) & ((f & 4u) ? (f >> 1) & 1u : 1u));
    const uint32_t y = ((f >> 1) & 1u) | (((h >> 1) & 1u) & ((f & 4u) ? f & 1u : 1u));
    return (f & 4u) | x | (y << 1);
}
struct StepTable {
    uint32_t fold[16];  // (h o f) << 3h, the element in bits 24-26
    uint32_t onto[16];  // (f o h) << 3h, the same
    uint32_t apply[16]; // status byte << 8s
};
constexpr StepTable make_step_table()
{
    StepTable t{};
    for (uint32_t i = 0; i < 16; i++) {
        const uint32_t op = i & 7u, side = i >> 3, own = side ? 2u : 1u;
        uint32_t e = 0;
        if (op == OP_W || op == OP_RWIND)
            e = 4u | own;
        else if (op == OP_PUSH)
            e = side ? 1u : 2u;
        else if (op == OP_PULL)
            e = side ? 2u : 1u;
        for (uint32_t h = 0; h < 8; h++)
            t.fold[i] |= host_compose(h, e) << (3 * h), t.onto[i] |= host_compose(e, h) << (3 * h);
        t.fold[i] |= e << 24, t.onto[i] |= e << 24;
        const Effect x = make_effect(op <= OP_RWIND ? op : (uint32_t)OP_NOOP, side);
        for (uint32_t s = 0; s < 4; s++) {
            const uint32_t post = (x.f4 >> (8 * s)) & 3u;
            t.apply[i] |= (post | (s << 2) | (((x.stuck >> s) & 1u) << 7)) << (8 * s);
        }
    }
    return t;
}
__constant__ constexpr StepTable STEPS = make_step_table();

__device__ __forceinline__ void compiler_fence() { asm volatile("" ::: "memory"); }

// (relaxed: one wave, whose LDS operations execute in order)
__device__ __forceinline__ uint32_t tab_touch(uint32_t *p, uint32_t bit)
{
    return __hip_atomic_fetch_or(p, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void tab_untouch(uint32_t *p, uint32_t bit)
{
    (void)__hip_atomic_fetch_and(p, ~bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void tab_xor(uint32_t *p, uint32_t v)
{
    (void)__hip_atomic_fetch_xor(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ uint32_t tab_load(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// ----------------------------------------------------------------------------------
// Domains: where an id lies in the table, and an event's part in each walk (`entry`, from
// its word; `next`: the id's bits after it, and its result; `open`: whether an event can
// still change the id in the fold), and how the functions of lanes that share an id are
// composed (BY_MASKS: from ballots; else they are passed along, with the lane they came
// from (64: none) in spare bits).  ALIKE: the ids of a step that are looked for before all are
// matched; CLOSES: chunks of skewed ids close constants first (k spaces, a bucket of 2^12 ids of
// which half a lane a step meets, gain by neither: uniform ids 187 and 207 us, 2^26 events).
// ----------------------------------------------------------------------------------
struct __attribute__((packed)) Bytes8 { // at any address
    uint32_t lo, hi;
};

struct Two {
    static constexpr uint32_t MASK = 7, NOOP = (uint32_t)OP_NOOP << 24;
    static constexpr bool BY_MASKS = true, CLOSES = true;
    static constexpr int ALIKE = 1;
    // The lanes of a step by what their events do, in their order from bit 0 on: constants
    // (t), of them those that leave the CPU copy (c: one event leaves one copy), and the others
    // that add the CPU copy to a status with the GPU copy valid (x) or the other way round (y).
    struct Kinds {
        uint64_t t, c, x, y;
    };
    template <bool BACK>
    __device__ static uint64_t in_order(uint64_t m)
    {
        return BACK ? __builtin_bitreverse64(m) : m; // (lower lanes are later events)
    }
    // from an element's bits (of the fold's table entries), or a status byte's (the walk's: the
    // statuses after (I,I), (V,I) and (I,V))
    template <bool BACK>
    __device__ static Kinds kinds(bool constant, bool cpu, bool gpu)
    {
        const uint64_t t = in_order<BACK>(__ballot(constant)), x = in_order<BACK>(__ballot(cpu));
        return Kinds{t, t & x, x & ~t, in_order<BACK>(__ballot(gpu)) & ~t};
    }
    template <bool BACK>
    __device__ static Kinds fold_kinds(uint32_t e)
    {
        return kinds<BACK>((e >> 26) & 1u, (e >> 24) & 1u, (e >> 25) & 1u);
    }
    __device__ static Kinds apply_kinds(uint32_t e) { return kinds<false>((e & 3u) != 0, (e >> 16) & 1u, (e >> 9) & 1u); }
    // The functions of the lanes of `set` composed (any set for each lane): a constant forgets
    // what was before it, and the others can be taken in any order.  So it is the latest
    // constant (k: there is one, left: its status) and whether any lane after it adds either
    // copy (x, y: bits 0 and 1).  Of two sets without common lanes the one with the latest lane
    // is the larger number.  (2^24 events over 2^16 ids in runs of 128 an id, the apply pass: 149
    // us by the position of the latest constant, with shifts and masks, and as functions in
    // 4-byte form, 96 this way, 88 with the rest of what steps that share ids do.)
    struct Composed {
        bool k;
        uint32_t left, x, y;
        __device__ uint32_t status(uint32_t h) const // after it, from status h
        {
            const uint32_t s = k ? left : h;
            return s | ((s >> 1) & x) | ((s << 1) & y);
        }
        __device__ uint32_t element() const { return k ? 4u | status(0) : x | y; }
    };
    __device__ static Composed compose_set(uint64_t set, const Kinds &K)
    {
        const uint64_t k = set & K.t, c = set & K.c;
        return Composed{k != 0, c > (k ^ c) ? 1u : 2u, (set & K.x) > k ? 1u : 0u, (set & K.y) > k ? 2u : 0u};
    }
    __device__ static uint32_t word(uint32_t id) { return id >> 3; }
    __device__ static uint32_t shift(uint32_t id) { return 3u * (id & 7u); }
    __device__ static uint32_t touch(uint32_t id) { return T_TOUCH << (id & 7u); }
    __device__ static uint32_t fold_entry(const uint32_t *tab, uint32_t w) { return tab[(w >> 24) & 15u]; }
    __device__ static bool fold_part(uint32_t e) { return (e >> 24) != 0; }
    __device__ static uint32_t fold_next(uint32_t e, uint32_t h) { return (e >> (3u * h)) & 7u; }
    __device__ static bool fold_open(uint32_t h) { return (h & 4u) == 0; }
    __device__ static uint32_t onto_next(uint32_t e, uint32_t h) { return (e >> (3u * h)) & 7u; }
    __device__ static uint32_t onto_all(const Composed &f, uint32_t h) { return el_compose(f.element(), h); }
    __device__ static uint32_t apply_entry(const uint32_t *tab, uint32_t w) { return tab[16 + ((w >> 24) & 15u)]; }
    __device__ static uint32_t apply_next(uint32_t e, uint32_t h, uint32_t &byte)
    {
        byte = e >> (8u * (h & 3u));
        return 4u | (byte & 3u);
    }
    __device__ static uint32_t fold_all(uint32_t h, const Composed &f) { return el_compose(h, f.element()); }
    __device__ static uint32_t status_after(const Composed &f, uint32_t h) { return f.status(h & 3u); }
    // rows: a word's composition, the initial statuses of its ids (from id on, n_ids in all)
    // as constants, and its statuses as final ones
    static constexpr uint32_t IDS = 8, ROW_IDENTITY = 0;
    __device__ static uint32_t compose_word(uint32_t g, uint32_t f) { return tw_compose(g, f); }
    __device__ static uint32_t initial(const uint8_t *init, uint32_t id, uint32_t n_ids)
    {
        if (!init)
            return MT | MX; // (V,I) eight times
        uint32_t st = MT;
        if (id + 8 <= n_ids) {
            const Bytes8 b = *reinterpret_cast<const Bytes8 *>(init + id);
#pragma unroll
            for (uint32_t k = 0; k < 8; k++)
                st |= (((k < 4 ? b.lo : b.hi) >> (8u * (k & 3u))) & 3u) << (3 * k);
        } else {
            for (uint32_t k = 0; k < 8; k++)
                st |= (id + k < n_ids ? init[id + k] & 3u : 1u) << (3 * k);
        }
        return st;
    }
    __device__ static void put_final(uint32_t st, uint8_t *final_out, uint32_t id, uint32_t n_ids)
    {
        if (id + 8 <= n_ids) {
            Bytes8 b{0, 0};
#pragma unroll
            for (uint32_t k = 0; k < 4; k++) {
                b.lo |= ((st >> (3 * k)) & 3u) << (8 * k);
                b.hi |= ((st >> (3 * k + 12)) & 3u) << (8 * k);
            }
            *reinterpret_cast<Bytes8 *>(final_out + id) = b;
        } else {
            for (uint32_t k = 0; k < 8; k++)
                if (id + k < n_ids)
                    final_out[id + k] = (uint8_t)((st >> (3 * k)) & 3u);
        }
    }
};

// The lanes of `among` with this lane's id (ids of `bits` bits, at most 16); of a lane that is
// not among them, anything.  The first FIRST ids are taken one by one (a run of events on an id
// fills steps), and if there are more all lanes are matched bit by bit.
template <int FIRST>
__device__ __forceinline__ uint64_t same_id(uint32_t id, uint64_t among, uint32_t bits)
{
    uint64_t rest = among, mine = 0;
#pragma unroll
    for (int k = 0; k < FIRST && rest; k++) {
        const bool eq = id == (uint32_t)__builtin_amdgcn_readlane((int)id, __builtin_ctzll(rest));
        const uint64_t with = among & __ballot(eq);
        mine = eq ? with : mine;
        rest &= ~with;
    }
    if (FIRST && !rest)
        return mine;
    uint32_t lo = (uint32_t)among, hi = (uint32_t)(among >> 32);
    match_bits<0, 4>(id, lo, hi);
    if (bits > 4)
        match_bits<4, 8>(id, lo, hi);
    if (bits > 8)
        match_bits<8, 12>(id, lo, hi);
    if (bits > 12)
        match_bits<12, 14>(id, lo, hi);
    if (bits > 14)
        match_bits<14, 16>(id, lo, hi);
    return ((uint64_t)hi << 32) | lo;
}

// Composition of the functions of the lanes of a lane's id up to and with it, by pointer
// jumping along them; p is the nearest lower one, 64 if none.  BACK: lower lanes are later
// events (their function comes last).  Q steps at once, independent of each other.
template <class D, bool BACK, int Q>
__device__ __forceinline__ void compose_along(uint32_t (&f)[Q], uint32_t (&p)[Q])
{
    for (;;) {
        bool more = false;
#pragma unroll
        for (int q = 0; q < Q; q++) {
            if (!BACK && D::constant(f[q])) // nothing before a constant matters
                p[q] = 64u;
            more = more || p[q] < 64u;
        }
        if (!__ballot(more))
            break;
        uint32_t v[Q];
#pragma unroll
        for (int q = 0; q < Q; q++)
            v[q] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(p[q] * 4u), (int)D::pack(f[q], p[q]));
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const uint32_t g = p[q] < 64u ? D::packed_function(v[q]) : D::IDENTITY;
            f[q] = BACK ? D::compose(g, f[q]) : D::compose(f[q], g);
            p[q] = p[q] < 64u ? D::packed_lane(v[q]) : 64u;
        }
    }
}

template <class D>
struct Fold {
    static constexpr bool BACK = true;
    using Dom = D;
    __device__ static uint32_t entry(const uint32_t *tab, uint32_t w) { return D::fold_entry(tab, w); }
    __device__ static bool takes_part(uint32_t e) { return D::fold_part(e); }
    __device__ static bool open(uint32_t h) { return D::fold_open(h); }
    __device__ static uint32_t next(uint32_t e, uint32_t h, uint32_t &) { return D::fold_next(e, h); }
    __device__ static uint32_t first_table(uint32_t i) { return STEPS.fold[i]; }
    __device__ static auto kinds(uint32_t e) { return D::template fold_kinds<true>(e); }
};
template <class D>
struct Apply {
    static constexpr bool BACK = false;
    using Dom = D;
    __device__ static uint32_t entry(const uint32_t *tab, uint32_t w) { return D::apply_entry(tab, w); }
    __device__ static bool takes_part(uint32_t) { return true; }
    __device__ static bool open(uint32_t) { return true; }
    __device__ static uint32_t next(uint32_t e, uint32_t h, uint32_t &result) { return D::apply_next(e, h, result); }
    // the status after the functions before the event
    template <class F>
    __device__ static uint32_t after(const F &f, uint32_t h)
    {
        return D::status_after(f, h);
    }
    static constexpr bool FUNCTIONS = false;
    __device__ static uint32_t first_table(uint32_t i) { return STEPS.fold[i]; }
    __device__ static auto kinds(uint32_t e) { return D::apply_kinds(e); }
};
// every id's function composed forwards; an event's result is the one before it
template <class D>
struct Onto {
    static constexpr bool BACK = false;
    using Dom = D;
    __device__ static uint32_t entry(const uint32_t *tab, uint32_t w) { return D::fold_entry(tab, w); }
    __device__ static bool takes_part(uint32_t) { return true; }
    __device__ static bool open(uint32_t) { return true; }
    __device__ static uint32_t next(uint32_t e, uint32_t h, uint32_t &result)
    {
        result = h;
        return D::onto_next(e, h);
    }
    template <class F>
    __device__ static uint32_t after(const F &f, uint32_t h)
    {
        return D::onto_all(f, h);
    }
    static constexpr bool FUNCTIONS = true;
    __device__ static uint32_t first_table(uint32_t i) { return STEPS.onto[i]; } // (in the fold's place)
    __device__ static auto kinds(uint32_t e) { return D::template fold_kinds<false>(e); }
};

template <class DIR>
struct Lane { // one lane's event in a step
    using D = typename DIR::Dom;
    uint32_t *p;
    uint32_t id, w, entry, old;
    bool part;
    __device__ uint32_t touch() const { return D::touch(id); }
    __device__ uint32_t field(uint32_t word) const { return (word >> D::shift(id)) & D::MASK; }
    __device__ uint32_t change(uint32_t h, uint32_t nh) const { return (h ^ nh) << D::shift(id); }
    __device__ bool met() const { return part && (old & touch()) != 0; }
    __device__ void enter()
    {
        old = 0;
        if (part)
            old = tab_touch(p, touch());
    }
    __device__ void leave() const
    {
        if (part)
            tab_untouch(p, touch());
    }
};

template <class DIR>
__device__ __forceinline__ Lane<DIR> make_lane(uint32_t *s_t, const uint32_t *s_tab, uint32_t w, uint32_t id, bool in)
{
    Lane<DIR> L;
    L.id = id;
    L.w = w;
    L.p = s_t + DIR::Dom::word(id);
    L.entry = DIR::entry(s_tab, w);
    L.part = in && DIR::takes_part(L.entry);
    L.old = 0;
    return L;
}

// no two lanes share an id (all have entered)
template <class DIR>
__device__ __forceinline__ uint32_t step_apart(const Lane<DIR> &L)
{
    const uint32_t h = L.field(L.old);
    uint32_t result = 0;
    const uint32_t nh = DIR::next(L.entry, h, result);
    if (L.part)
        tab_xor(L.p, L.change(h, nh) | L.touch());
    return result;
}

// few lanes share ids (`met`: all but the first of each id to enter; none is in the table
// any more): the lanes of an id take turns in their order
template <class DIR>
__device__ __forceinline__ uint32_t step_in_turn(const Lane<DIR> &L, uint64_t met)
{
    uint32_t turn = 0, turns = 0;
    while (met) {
        const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)L.id, __builtin_ctzll(met));
        const bool mine = L.part && L.id == other;
        const uint64_t same = __ballot(mine);
        if (mine)
            turn = mask_rank(same);
        const uint32_t n = (uint32_t)__builtin_popcountll(same) - 1;
        turns = turns > n ? turns : n;
        met &= ~same;
    }
    uint32_t result = 0;
    for (uint32_t k = 0; k <= turns; k++) {
        if (L.part && turn == k) {
            const uint32_t h = L.field(tab_load(L.p));
            tab_xor(L.p, L.change(h, DIR::next(L.entry, h, result)));
        }
        compiler_fence();
    }
    return result;
}

// lanes of a step that share ids with others, at most, for which taking turns is the shorter way
// (2^24 uniform events over 512 ids, all kernels: 155 us, 161 with 5, 166 with 2, 155 with 16)
constexpr int D_FEW = 10;

// Q steps whose lanes may share ids, one after the other; no lane is in the table.  What
// the lanes of an id do together does not depend on the table, so the steps work it out
// side by side.  `shared` counts the steps where any did (backwards, where the open ids go on
// getting fewer, those where more than few did, and those without an open id).
template <class DIR, int Q>
__device__ __forceinline__ void steps_together(const Lane<DIR> (&L)[Q], uint32_t (&result)[Q], const uint32_t *s_tab,
                                               uint32_t bits, uint32_t lane, uint32_t &shared)
{
    using D = typename DIR::Dom;
    bool in[Q], any = false;
    uint64_t same[Q];
    const uint64_t under = (1ull << lane) - 1;
#pragma unroll
    for (int q = 0; q < Q; q++) { // (a later step's id may close before it: it then changes nothing)
        in[q] = L[q].part && (!DIR::BACK || DIR::open(L[q].field(tab_load(L[q].p))));
        any = any || in[q];
    }
    if (DIR::BACK && !__ballot(any)) { // nothing changes (and the next steps may be as much alike)
        shared += Q;
        return;
    }
#pragma unroll
    for (int q = 0; q < Q; q++) {
        const uint64_t among = __ballot(in[q]);
        same[q] = same_id<D::ALIKE>(L[q].id, among, bits);
        same[q] = in[q] ? same[q] : 0ull;
        const uint64_t m = __ballot((same[q] & under) != 0);
        shared += (DIR::BACK ? !among || __builtin_popcountll(m) > D_FEW : m != 0) ? 1u : 0u;
    }
    // writes the table: the last lane of its id
    auto last = [&](int q) { return (same[q] & ~under) == 1ull << lane; };
    if constexpr (D::BY_MASKS) {
        typename D::Composed f[Q]; // BACK: of all lanes of the id; else of those before
#pragma unroll
        for (int q = 0; q < Q; q++) {
            f[q] = D::compose_set(DIR::BACK ? D::template in_order<true>(same[q]) : same[q] & under,
                                  DIR::kinds(L[q].entry));
        }
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const uint32_t h = L[q].field(tab_load(L[q].p));
            uint32_t nh;
            if constexpr (DIR::BACK)
                nh = D::fold_all(h, f[q]);
            else
                nh = DIR::next(L[q].entry, DIR::after(f[q], h), result[q]);
            if (last(q))
                tab_xor(L[q].p, L[q].change(h, nh));
            compiler_fence();
        }
    } else {
        uint32_t f[Q], p[Q], prev[Q], g[Q];
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const uint64_t below = same[q] & under;
            prev[q] = p[q] = below ? 63u - (uint32_t)__builtin_clzll(below) : 64u;
            f[q] = D::function(s_tab, L[q].w);
        }
        compose_along<D, DIR::BACK, Q>(f, p);
        if constexpr (!DIR::BACK)
#pragma unroll
            for (int q = 0; q < Q; q++)
                g[q] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((prev[q] & 63u) * 4u), (int)f[q]);
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const uint32_t h = L[q].field(tab_load(L[q].p));
            uint32_t nh;
            if constexpr (DIR::BACK)
                nh = D::fold_all(h, f[q]);
            else
                nh = DIR::next(L[q].entry, prev[q] < 64 ? DIR::after(g[q], h) : h, result[q]);
            if (last(q))
                tab_xor(L[q].p, L[q].change(h, nh));
            compiler_fence();
        }
    }
}

// PAIR steps at once: all enter, and when no lane met a touched id, neither of its own
// step nor of the ones before it, their reads are one wait and their changes independent.
// Otherwise all leave and the steps take their turns; lanes that share ids within a step
// take turns too when they are few, else they work their changes out together.
// CLOSE: ids that are constants already leave before the lanes enter (only backwards; a read
// more a step).
template <class DIR, int PAIR, bool CLOSE = false>
__device__ __forceinline__ void steps(Lane<DIR> (&L)[PAIR], uint32_t (&result)[PAIR], const uint32_t *s_tab,
                                      uint32_t bits, uint32_t lane, uint32_t &shared_steps)
{
    bool met = false;
    if constexpr (CLOSE)
#pragma unroll
        for (int q = 0; q < PAIR; q++)
            L[q].part = L[q].part && DIR::open(L[q].field(tab_load(L[q].p)));
#pragma unroll
    for (int q = 0; q < PAIR; q++)
        L[q].enter();
#pragma unroll
    for (int q = 0; q < PAIR; q++)
        met = met || L[q].met();
    if (!__ballot(met)) {
#pragma unroll
        for (int q = 0; q < PAIR; q++)
            result[q] = step_apart<DIR>(L[q]);
        return;
    }
    compiler_fence();
    if (PAIR > 1 || DIR::BACK) {
#pragma unroll
        for (int q = 0; q < PAIR; q++)
            L[q].leave();
        compiler_fence();
    }
#pragma unroll
    for (int q = 0; q < PAIR; q++) {
        if (DIR::BACK && L[q].part) // ids that are constants already take no part
            L[q].part = DIR::open(L[q].field(tab_load(L[q].p)));
        if (PAIR > 1 || DIR::BACK)
            L[q].enter();
        const uint64_t m = __ballot(L[q].met());
        if (!m) {
            result[q] = step_apart<DIR>(L[q]);
        } else {
            L[q].leave();
            compiler_fence();
            if (__builtin_popcountll(m) <= D_FEW) {
                result[q] = step_in_turn<DIR>(L[q], m);
            } else {
                const Lane<DIR> one[1] = {L[q]};
                uint32_t r[1] = {0};
                steps_together<DIR, 1>(one, r, s_tab, bits, lane, shared_steps);
                result[q] = r[0];
            }
        }
        compiler_fence();
    }
}

constexpr int D_UNROLL = 8; // steps whose events are loaded together
// a round whose last one worked out at least so many of its steps together does so for all
constexpr uint32_t D_TOGETHER = D_UNROLL / 2;

// a round's words turned by PAIR: a loop over the round's steps takes the first ones, so that
// its code is not there for every step, nor are the words read from memory again (2^24 events
// over 2^16 ids in runs of 128 an id: fold 130 -> 116 us)
template <int PAIR>
__device__ __forceinline__ void turn_words(uint32_t (&w)[D_UNROLL])
{
    uint32_t v[D_UNROLL];
#pragma unroll
    for (int u = 0; u < D_UNROLL; u++)
        v[u] = w[(u + PAIR) % D_UNROLL];
#pragma unroll
    for (int u = 0; u < D_UNROLL; u++)
        w[u] = v[u];
}

// The first round of a chunk goes that way when so many of its events have their neighbour's
// id: about 500 times the chance that two events share theirs, which is 14 for Zipf(1.1) ids over
// 2^16 and 4 for uniform ones over 128, where a step has about 2,000 times that of lanes that
// meet; on one address the lanes' atomics take turns (2^24 events over 2^20 ids in runs of 128
// an id: fold 70 -> 59, apply 72 -> 47 us; uniform ids over 512, of which 2 % of the chunks have
// 4, fold 47.7 with 8 and 48-57 with 4).
constexpr uint32_t D_ALIKE = 8;
__device__ __forceinline__ uint32_t first_shared(const uint32_t (&w)[D_UNROLL])
{
    uint32_t alike = 0;
#pragma unroll
    for (int u = 0; u < D_UNROLL; u++)
        alike += (uint32_t)__builtin_popcountll(
            __ballot(((dpp_move<DPP_WAVE_SHR1>(~w[u], w[u]) ^ w[u]) & 0xFFFFFFu) == 0));
    return alike >= D_ALIKE ? D_TOGETHER : 0u;
}

template <class DIR>
__device__ __forceinline__ void load_step_table(uint32_t *s_tab, uint32_t lane)
{
    if (lane < 32)
        s_tab[lane] = lane < 16 ? DIR::first_table(lane) : STEPS.apply[lane - 16];
    compiler_fence();
}

// ----------------------------------------------------------------------------------
// The walks: one wave per chunk.  CHUNKS: the number of chunks, and of a chunk its words
// (ev + [begin, end)), its row (words of it, and where it lies), the bits of its ids,
// malformed words (op_mask: bit op + 8 side of the known ones, of chunks that go forwards),
// and the table's id of a word (local: of a well-formed one; clamped: inside the table for
// any).  `table`: words of LDS for the table, a row of any chunk.
// ----------------------------------------------------------------------------------
// a chunk of a trace, or stream, whose chunks are all alike
template <class CHUNKS>
struct OneChunk : CHUNKS {
    uint64_t begin, end, row_at;
    uint32_t bits;
    __device__ OneChunk(const CHUNKS &T, uint32_t c)
        : CHUNKS(T), begin(T.begin_of(c)), end(T.end_of(c)), row_at((uint64_t)c * T.row), bits(T.id_bits())
    {
    }
};

// malformed words among a round's: the words' upper bits, their largest id and the bits of
// their ops in C.op_mask together, then (rarely) one by one
template <class C>
__device__ __forceinline__ bool any_bad(const C &c, const uint32_t (&w)[D_UNROLL])
{
    uint32_t bits = 0, top = 0, known = 1;
#pragma unroll
    for (int u = 0; u < D_UNROLL; u++) {
        const uint32_t id = w[u] & 0xFFFFFFu;
        bits |= w[u];
        top = top > id ? top : id;
        known &= c.op_mask() >> ((w[u] >> 24) & 31u);
    }
    return (bits >> 28) != 0 || top >= c.n_ids || !(known & 1u);
}

// Whole rounds forwards from round 0, whose words are in nxt, then the words past them one
// step at a time: out takes every event's result.  A malformed word only has to stay inside
// the table (what a trace with one comes to is not read); PUT sees the words.
template <class DIR, int PAIR, class C, class PUT, class OUT>
__device__ __forceinline__ void walk_forward(const C &c, uint32_t *s_t, const uint32_t *s_tab, uint32_t lane,
                                             uint32_t (&nxt)[D_UNROLL], PUT &&put, OUT &out)
{
    using D = typename DIR::Dom;
    const uint64_t i0 = c.begin;
    const uint32_t bits = c.bits, len = (uint32_t)(c.end - i0), rounds = len / (D_UNROLL * WAVE);
    uint32_t shared_steps = rounds ? first_shared(nxt) : 0u;
    for (uint32_t r = 0; r < rounds; r++) {
        uint32_t w[D_UNROLL];
#pragma unroll
        for (int u = 0; u < D_UNROLL; u++)
            w[u] = nxt[u];
        const uint64_t i = i0 + (uint64_t)r * (D_UNROLL * WAVE);
        if (r + 1 < rounds) {
            const uint32_t *e = c.ev + i + D_UNROLL * WAVE + lane;
#pragma unroll
            for (int u = 0; u < D_UNROLL; u++)
                nxt[u] = e[u * WAVE];
        }
        if (shared_steps >= D_TOGETHER) {
            shared_steps = 0;
#pragma unroll 1
            for (int u = 0; u < D_UNROLL; u += PAIR) {
                Lane<DIR> L[PAIR];
                uint32_t byte[PAIR];
#pragma unroll
                for (int q = 0; q < PAIR; q++)
                    L[q] = make_lane<DIR>(s_t, s_tab, w[q], c.clamped(w[q]), true);
                steps_together<DIR, PAIR>(L, byte, s_tab, bits, lane, shared_steps);
#pragma unroll
                for (int q = 0; q < PAIR; q++)
                    out.step(lane, u + q, i + (u + q) * WAVE, w[q], byte[q], true);
                turn_words<PAIR>(w);
            }
        } else {
            shared_steps = 0;
#pragma unroll
            for (int u = 0; u < D_UNROLL; u += PAIR) {
                Lane<DIR> L[PAIR];
                uint32_t byte[PAIR];
#pragma unroll
                for (int q = 0; q < PAIR; q++)
                    L[q] = make_lane<DIR>(s_t, s_tab, w[u + q], c.clamped(w[u + q]), true);
                steps<DIR, PAIR>(L, byte, s_tab, bits, lane, shared_steps);
#pragma unroll
                for (int q = 0; q < PAIR; q++)
                    out.step(lane, u + q, i + (u + q) * WAVE, w[u + q], byte[q], true);
            }
        }
        put.round(w, i);
        out.round(lane, i, D_UNROLL, (r + 1) * (D_UNROLL * WAVE) == len);
    }
    // the events past the whole rounds, one step at a time
    const uint32_t past = rounds * (D_UNROLL * WAVE);
    for (uint32_t k = past; k < len; k += WAVE) {
        const bool valid = k + lane < len;
        const uint32_t w = valid ? c.ev[i0 + k + lane] : D::NOOP;
        put.one(w, i0 + k + lane);
        const Lane<DIR> one[1] = {make_lane<DIR>(s_t, s_tab, w, c.clamped(w), valid)};
        uint32_t b[1];
        steps_together<DIR, 1>(one, b, s_tab, bits, lane, shared_steps);
        out.step(lane, (k - past) / WAVE, i0 + k, w, b[0], valid);
    }
    if (past < len)
        out.round(lane, i0 + past, (len - past + WAVE - 1) / WAVE, true);
}

// words that were checked before
struct Checked {
    __device__ void round(const uint32_t (&)[D_UNROLL], uint64_t) const {}
    __device__ void one(uint32_t, uint64_t) const {}
};

// words checked here, a round's after its steps (nothing waits for the round's last words
// before its first steps): malformed ones are reported
template <class C>
struct Unchecked {
    const C &c;
    Control *ctl;
    uint32_t lane;
    __device__ void one(uint32_t w, uint64_t i) const
    {
        if (c.bad(w))
            if (Control *const to = c.report_to(ctl))
                atomicMin(reinterpret_cast<unsigned long long *>(&to->err_index_lo), (unsigned long long)i);
    }
    __device__ void round(const uint32_t (&w)[D_UNROLL], uint64_t i) const
    {
        if (__ballot(any_bad(c, w)))
#pragma unroll
            for (int u = 0; u < D_UNROLL; u++)
                one(w[u], i + u * WAVE + lane);
    }
};

struct NoOut {
    __device__ void step(uint32_t, uint32_t, uint64_t, uint32_t, uint32_t, bool) const {}
    __device__ void round(uint32_t, uint64_t, uint32_t, bool) const {}
};

// Every chunk's functions into its row (left: of the chunks marked there, of skewed ids, only).
// In chunks of skewed ids, or whose first words show it, few still meet when those that are
// constants leave first (2^24 events of Zipf(1.1) ids over 2^16: 106 -> 89 us, 2^26 over 2^20
// 211 -> 140; uniform ids 231 -> 273 us at 2^26 over 2^16).
template <class F, int PAIR, class CHUNKS>
__global__ __launch_bounds__(WAVE) void k_dense_fold(CHUNKS T, uint32_t table, uint32_t *__restrict__ rows,
                                                     Control *ctl, const uint32_t *__restrict__ left)
{
    using D = typename F::Dom;
    extern __shared__ __align__(16) uint32_t s_t[];
    uint32_t *const s_tab = s_t + table;
    const uint32_t lane = threadIdx.x, chunks = T.count();
    load_step_table<F>(s_tab, lane);
    for (uint32_t c = blockIdx.x; c < chunks; c += gridDim.x) {
        if (left && !left[c])
            continue;
        const auto C = T.chunk(c);
        const uint64_t i0 = C.begin, i1 = C.end;
        const uint32_t row = C.row, bits = C.bits;
        const uint32_t len = (uint32_t)(i1 - i0), rounds = len / (D_UNROLL * WAVE);
        for (uint32_t i = lane; i < row / 4; i += WAVE)
            reinterpret_cast<uint4 *>(s_t)[i] = make_uint4(0, 0, 0, 0);
        compiler_fence();
        // (a malformed word is a Noop on id 0)
        auto clean = [&](uint32_t w, bool bad) { return bad ? D::NOOP : w; };
        auto report = [&](uint64_t i) {
            if (Control *const to = C.report_to(ctl))
                atomicMin(reinterpret_cast<unsigned long long *>(&to->err_index_lo), (unsigned long long)i);
        };
        uint32_t shared_steps = 0;
        bool close = left != nullptr;
        // the events past the whole rounds, one step at a time
        for (uint32_t left = len - rounds * (D_UNROLL * WAVE); left;) {
            const uint32_t m = left < WAVE ? left : WAVE;
            const uint64_t i = i0 + rounds * (D_UNROLL * WAVE) + left - 1 - lane;
            const bool in = lane < m;
            uint32_t w = in ? C.ev[i] : D::NOOP;
            if (C.bad(w)) {
                report(i);
                w = clean(w, true);
            }
            const Lane<F> one[1] = {make_lane<F>(s_t, s_tab, w, C.local(w), in)};
            uint32_t none[1];
            steps_together<F, 1>(one, none, s_tab, bits, lane, shared_steps);
            left -= m;
        }
        // whole rounds: lane l takes the round's last event but l, then 64 before, ...
        const uint32_t *const e0 = C.ev + i0 - 1 - lane;
        uint32_t nxt[D_UNROLL];
        auto load = [&](uint32_t r) {
            const uint32_t *e = e0 + (uint64_t)r * (D_UNROLL * WAVE);
#pragma unroll
            for (int u = 0; u < D_UNROLL; u++)
                nxt[u] = e[-(u * WAVE)];
        };
        if (rounds) {
            load(rounds);
            shared_steps = first_shared(nxt);
            close = close || shared_steps;
        }
        for (uint32_t r = rounds; r > 0; r--) {
            uint32_t w[D_UNROLL], badm = 0;
#pragma unroll
            for (int u = 0; u < D_UNROLL; u++) {
                const bool bad = C.bad(nxt[u]);
                badm |= bad ? 1u << u : 0u;
                w[u] = clean(nxt[u], bad);
            }
            if (r > 1)
                load(r - 1);
            if (__ballot(badm != 0)) {
                if (badm) // the lane's first malformed event is its last step's
                    report(i0 + (uint64_t)r * (D_UNROLL * WAVE) - 1 - lane -
                           WAVE * (31u - (uint32_t)__builtin_clz(badm)));
            }
            if (shared_steps >= D_TOGETHER) {
                shared_steps = 0;
#pragma unroll 1
                for (int u = 0; u < D_UNROLL; u += PAIR) {
                    Lane<F> L[PAIR];
                    uint32_t none[PAIR];
#pragma unroll
                    for (int q = 0; q < PAIR; q++)
                        L[q] = make_lane<F>(s_t, s_tab, w[q], C.local(w[q]), true);
                    steps_together<F, PAIR>(L, none, s_tab, bits, lane, shared_steps);
                    turn_words<PAIR>(w);
                }
                continue;
            }
            shared_steps = 0;
            if (D::CLOSES && close) { // (a loop of its own: a branch a step costs uniform ids 4 %)
#pragma unroll 1
                for (int u = 0; u < D_UNROLL; u += PAIR) {
                    Lane<F> L[PAIR];
                    uint32_t byte[PAIR];
#pragma unroll
                    for (int q = 0; q < PAIR; q++)
                        L[q] = make_lane<F>(s_t, s_tab, w[q], C.local(w[q]), true);
                    steps<F, PAIR, true>(L, byte, s_tab, bits, lane, shared_steps);
                    turn_words<PAIR>(w);
                }
                continue;
            }
#pragma unroll
            for (int u = 0; u < D_UNROLL; u += PAIR) {
                Lane<F> L[PAIR];
                uint32_t byte[PAIR];
#pragma unroll
                for (int q = 0; q < PAIR; q++)
                    L[q] = make_lane<F>(s_t, s_tab, w[u + q], C.local(w[u + q]), true);
                steps<F, PAIR>(L, byte, s_tab, bits, lane, shared_steps);
            }
        }
        compiler_fence();
        uint4 *out = reinterpret_cast<uint4 *>(rows + C.row_at);
        for (uint32_t i = lane; i < row / 4; i += WAVE)
            out[i] = reinterpret_cast<const uint4 *>(s_t)[i];
        compiler_fence();
    }
}

// The same forwards: an id whose function has become a constant still takes part, but a step
// is shorter.  A chunk of skewed ids is left to the backward walk (marked in `left`): one in
// whose first two pairs of steps so many events meet an id again as uniform ids above
// FORWARD_IDS practically never do (4 of 256 at 4,096 ids; a single chunk that is left costs
// as long as all of them).
constexpr uint32_t FORWARD_IDS = 4096, FORWARD_MET = 16;
template <class D, int PAIR, class CHUNKS>
__global__ __launch_bounds__(WAVE) void k_dense_forward(CHUNKS T, uint32_t table, uint32_t *__restrict__ rows,
                                                        Control *ctl, uint32_t *__restrict__ left)
{
    extern __shared__ __align__(16) uint32_t s_t[];
    uint32_t *const s_tab = s_t + table;
    const uint32_t lane = threadIdx.x, chunks = T.count();
    load_step_table<Onto<D>>(s_tab, lane);
    for (uint32_t c = blockIdx.x; c < chunks; c += gridDim.x) {
        const auto C = T.chunk(c);
        const uint32_t row = C.row;
        uint32_t nxt[D_UNROLL];
        const bool whole = C.end - C.begin >= D_UNROLL * WAVE;
        if (whole) {
            const uint32_t *e = C.ev + C.begin + lane;
#pragma unroll
            for (int u = 0; u < D_UNROLL; u++)
                nxt[u] = e[u * WAVE];
        }
        for (uint32_t i = lane; i < row / 4; i += WAVE)
            reinterpret_cast<uint4 *>(s_t)[i] = make_uint4(0, 0, 0, 0);
        compiler_fence();
        uint32_t again = 0; // events that meet an id again
        if (whole) {
#pragma unroll
            for (int q = 0; q < 2 * PAIR; q += PAIR) {
                uint32_t *at[PAIR], touch[PAIR];
#pragma unroll
                for (int u = 0; u < PAIR; u++) {
                    const uint32_t id = C.clamped(nxt[q + u]);
                    at[u] = s_t + D::word(id);
                    touch[u] = D::touch(id);
                    again += (uint32_t)__builtin_popcountll(__ballot((tab_touch(at[u], touch[u]) & touch[u]) != 0));
                }
                compiler_fence();
#pragma unroll
                for (int u = 0; u < PAIR; u++)
                    tab_untouch(at[u], touch[u]);
                compiler_fence();
            }
        }
        if (lane == 0)
            left[c] = again >= FORWARD_MET ? 1u : 0u;
        if (again >= FORWARD_MET)
            continue; // uniform
        const Unchecked<decltype(C)> put{C, ctl, lane};
        NoOut none;
        walk_forward<Onto<D>, PAIR>(C, s_t, s_tab, lane, nxt, put, none);
        compiler_fence();
        uint4 *out = reinterpret_cast<uint4 *>(rows + C.row_at);
        for (uint32_t i = lane; i < row / 4; i += WAVE)
            out[i] = reinterpret_cast<const uint4 *>(s_t)[i];
        compiler_fence();
    }
}

// The events' results from their chunk's entering statuses (Apply), or every chunk's
// functions into its row, the events' results the functions before them (Onto).  OUT takes
// the results: step() a step's (u: its number in its round or in the chunk's last, partial
// one), round() at the end of each, chunk() at the chunk's.
template <class DIR, int PAIR, class CHUNKS, class OUT>
__global__ __launch_bounds__(WAVE) void k_dense_apply(CHUNKS T, uint32_t table, uint32_t *__restrict__ rows, OUT out)
{
    extern __shared__ __align__(16) uint32_t s_t[];
    uint32_t *const s_tab = s_t + table;
    const uint32_t lane = threadIdx.x, chunks = T.count();
    load_step_table<DIR>(s_tab, lane);
    for (uint32_t c = blockIdx.x; c < chunks; c += gridDim.x) {
        const auto C = T.chunk(c);
        uint4 *const chunk_row = reinterpret_cast<uint4 *>(rows + C.row_at);
        const uint32_t row = C.row;
        out.begin(C, c);
        uint32_t nxt[D_UNROLL];
        if (C.end - C.begin >= D_UNROLL * WAVE) {
            const uint32_t *e = C.ev + C.begin + lane;
#pragma unroll
            for (int u = 0; u < D_UNROLL; u++)
                nxt[u] = e[u * WAVE];
        }
        for (uint32_t i = lane; i < row / 4; i += WAVE)
            reinterpret_cast<uint4 *>(s_t)[i] = DIR::FUNCTIONS ? make_uint4(0, 0, 0, 0) : chunk_row[i];
        compiler_fence();
        const Checked put;
        walk_forward<DIR, PAIR>(C, s_t, s_tab, lane, nxt, put, out);
        out.chunk(lane, s_t);
        compiler_fence();
        if (DIR::FUNCTIONS)
            for (uint32_t i = lane; i < row / 4; i += WAVE)
                chunk_row[i] = reinterpret_cast<const uint4 *>(s_t)[i];
        compiler_fence();
    }
}

} // namespace
} // namespace vc
