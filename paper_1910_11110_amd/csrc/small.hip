// small.hip -- single-pass check of a trace over at most 64 variables (gfx950).
//
// No sort.  The trace is cut into tiles of 256 strands of EP consecutive events, one per
// lane (EP 64, or 16 for short traces).  A lane walks its strand event by event with the
// 64 variables' functions, then statuses, one byte each in an LDS column of its own, so
// that neither a variable nor a lane ever waits for another.
//   1. The tile's events are read in order, packed to 16 bits and handed to their lanes
//      through LDS.
//   2. Each lane composes its strand's functions: per event one byte read, one shift of a
//      table word, one byte written.
//   3. The bytes become 64-bit planes (T, X, Y: an element of the 7-element monoid per
//      variable); a wave scan of the planes (DPP) and the wave totals give every lane the
//      composition of the tile's strands before it.
//   4. The tiles chain their statuses with a decoupled look-back on the tile's function:
//      four self-flagged 64-bit words of 20 variables each (one wave per word).  A word
//      whose variables were all written in the tile is final at once, so in an ordinary
//      trace no tile waits for more than the one before it.
//   5. Each lane applies its prefix to the statuses entering the tile and walks its strand
//      again for the status bytes, which go out in order through LDS, and the final
//      statuses come from the last tile.  The count of flagged events and, per 16 events,
//      their mask and offset inside the tile are stored; a scan of the counts and a scatter
//      pass then write the ascending violation indices (no second chain of tiles).
#include "batch.h"
#include "device.h"
#include "internal.h"
#include "prof.h"

namespace vc {

namespace {

constexpr int SK = 64;               // variables
constexpr int SB = 256;              // threads per tile
constexpr int SW = SB / WAVE;        // waves per tile
constexpr int SPW = (SK + 19) / 20;  // look-back words per tile (20 variables each)
static_assert(SPW <= SW, "one wave per look-back word");
static_assert(SPW == (int)STRAND_WORDS && PL_MASK == (1u << STRAND_IDS) - 1, "the words that a batch's last pass reads");

// Events per lane: long strands share the cost of a strand's planes and scan, short ones
// keep a short trace on more lanes and its walks short.  The line lies where the long ones
// fill the device: 2^22 events take 20.1 us with 64 a lane and 17.7 with 16, 2^23 events
// 22.8 and 30.0; 2^13 events 18.2 and 10.0.
constexpr int EP_LONG = 64, EP_SHORT = 16;
constexpr uint64_t LONG_FROM = 3ull << 21; // events
constexpr int strand_of(uint64_t n) { return n >= LONG_FROM ? EP_LONG : EP_SHORT; }

// Per effect (op | side << 3): for the composition walk the element after it for every
// element before it, a nibble each (bit 2 a constant, whose status is bits 0 CPU and 1
// GPU; else bit 0 "CPU |= GPU", bit 1 "GPU |= CPU"), with bit 3 of nibble 0 set for an op
// past Noop; for the status walk the status byte for every status before it, a byte each.
struct StrandTable {
    uint32_t fold[16], apply[16];
};
constexpr StrandTable make_strand_table()
{
    StrandTable t{};
    for (uint32_t i = 0; i < 16; i++) {
        const uint32_t op = i & 7u;
        const Effect e = make_effect(op <= OP_NOOP ? op : (uint32_t)OP_NOOP, i >> 3);
        for (uint32_t h = 0; h < 8; h++) {
            // the element as a function, followed by the effect, as an element again
            uint32_t f[4] = {};
            for (uint32_t s = 0; s < 4; s++) {
                const uint32_t x = h & 1u, y = (h >> 1) & 1u, c = s & 1u, g = s >> 1;
                const uint32_t m = (h & 4u) ? (h & 3u) : ((c | (x & g)) | ((g | (y & c)) << 1));
                f[s] = (e.f4 >> (8 * m)) & 3u;
            }
            const uint32_t r = (h & 4u) || (f[0] == f[3]) ? 4u | f[0] : (f[2] & 1u) | (f[1] & 2u);
            t.fold[i] |= r << (4 * h);
        }
        t.fold[i] |= op > OP_NOOP ? 8u : 0u;
        for (uint32_t s = 0; s < 4; s++)
            t.apply[i] |= (((e.f4 >> (8 * s)) & 3u) | (s << 2) | (((e.stuck >> s) & 1u) << 7)) << (8 * s);
    }
    return t;
}
__constant__ constexpr StrandTable STRAND = make_strand_table();

// A packed event: variable >> 2 in bits 8-11 and variable & 3 in bits 0-1, the place of its
// byte in a column of words WAVE apart; 4 * (op | side << 3) in bits 2-5, the place of its
// table word.
__device__ __forceinline__ uint32_t pack_event(uint32_t w)
{
    return ((w & 0x3Cu) << 6) | (w & 3u) | ((w >> 22) & 0x3Cu);
}
constexpr uint32_t PLACE = 0xF03u, TABLE_AT = 0x3Cu;

// bits `bit` of the four bytes of v as bits 0-3, added to acc << bit
__device__ __forceinline__ uint32_t gather4(uint32_t v, uint32_t mask, uint32_t weights, uint32_t acc)
{
    return __builtin_amdgcn_udot4(v & mask, weights, acc, false);
}
constexpr uint32_t W_LO = 0x08040201u, W_HI = 0x80402010u;

// four event words from an address that is a multiple of 4 bytes only
struct __attribute__((packed, aligned(4))) Words4 {
    uint32_t x, y, z, w;
};

__device__ __forceinline__ void lds_fence() { asm volatile("" ::: "memory"); } // a wave's LDS operations are in order

// one 32-bit half of the function planes of up to 64 variables
struct Fn32 {
    uint32_t t, x, y;
};

// h o f (f first) on one half of the planes
__device__ __forceinline__ Fn32 fn_compose(Fn32 h, Fn32 f)
{
    const uint32_t ex = f.x | (h.x & (~f.t | f.y));
    const uint32_t ey = f.y | (h.y & (~f.t | f.x));
    return Fn32{h.t | f.t, (h.t & h.x) | (~h.t & ex), (h.t & h.y) | (~h.t & ey)};
}

// statuses (c, g) after f, on one half of the planes
__device__ __forceinline__ void fn_apply(Fn32 f, uint32_t &c, uint32_t &g)
{
    const uint32_t nc = (f.t & f.x) | (~f.t & (c | (f.x & g)));
    const uint32_t ng = (f.t & f.y) | (~f.t & (g | (f.y & c)));
    c = nc;
    g = ng;
}

template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ Fn32 fn_move(Fn32 f)
{
    return Fn32{dpp_move<CTRL, ROWS>(0u, f.t), dpp_move<CTRL, ROWS>(0u, f.x), dpp_move<CTRL, ROWS>(0u, f.y)};
}

// inclusive scan of the function planes across the wave (lane 0 first); a lane
// without a source combines with the identity (all planes zero)
__device__ __forceinline__ void fn_wave_scan(Fn32 &lo, Fn32 &hi)
{
#define VC_FN_STEP(CTRL, ROWS)                                                                                         \
    {                                                                                                                  \
        const Fn32 gl = fn_move<CTRL, ROWS>(lo), gh = fn_move<CTRL, ROWS>(hi);                                         \
        lo = fn_compose(lo, gl);                                                                                       \
        hi = fn_compose(hi, gh);                                                                                       \
    }
    VC_FN_STEP(DPP_ROW_SHR + 1, 0xF)
    VC_FN_STEP(DPP_ROW_SHR + 2, 0xF)
    VC_FN_STEP(DPP_ROW_SHR + 4, 0xF)
    VC_FN_STEP(DPP_ROW_SHR + 8, 0xF)
    VC_FN_STEP(DPP_ROW_BCAST15, 0xA)
    VC_FN_STEP(DPP_ROW_BCAST31, 0xC)
#undef VC_FN_STEP
}

__device__ __forceinline__ uint32_t bits20(uint32_t lo, uint32_t hi, uint32_t k)
{
    const uint64_t v = ((uint64_t)hi << 32) | lo;
    return (uint32_t)(v >> (20 * k)) & PL_MASK;
}

// flag words per scatter tile (512 or 256)
template <int EP>
constexpr uint32_t scatter_threads()
{
    return EP == EP_LONG ? 512 : 256;
}

// Bound by the issue of about 25 VALU instructions and 7 LDS operations per event, with
// three workgroups per CU (the packed events and the columns take 53 KB).  Composing 16
// events a lane in registers, with 64-bit planes, took about 100 instructions per event:
// 2^28 events x 64 variables 877 us, 746 with words final at once, 391 this way (3.4 TB/s
// of events in and status bytes out); 2^26 events 229 and 110 us; 10^4 events 12.8 and 10.7.
//
// SRC: the traces.  OneTrace: one, whose flagged events are left as flag words and counts of
// the scatter tiles.  BatchStrands: a batch's traces over few ids, a chunk a tile (consecutive
// ones of a trace), whose flagged events are counted per tile; 200 of them of 100 to 10^6
// events (23 M) take 55 us, 120 by the walks of the dense check.
// A last tile does not wait for the first one (a constant word ends its look-back), so nothing
// here orders its final statuses after the first tile's read of the initial ones: a batch's,
// which may be the same table, stay in the last tile's look-back words for a later launch
// (OneTrace: never the same table).
struct StrandTile {
    const uint32_t *ev;
    uint64_t n; // of the trace
    uint32_t n_ids;
    const uint8_t *init;
    uint8_t *status, *final_out;
    Control *ctl;
    uint64_t first; // event
    bool starts, ends; // the trace
};
struct OneTrace {
    const uint32_t *ev;
    uint64_t n;
    uint32_t n_ids;
    const uint8_t *init;
    uint8_t *status, *final_out;
    Control *ctl;
    uint32_t *fw;
    static constexpr bool FLAGS = true;
    __device__ StrandTile tile(uint32_t t, uint64_t ntiles, uint64_t events) const
    {
        return StrandTile{ev, n, n_ids, init, status, final_out, ctl, t * events, t == 0, t + 1 == ntiles};
    }
};
struct BatchStrands {
    const TraceDesc *d;
    const ChunkDesc *ch;
    static constexpr bool FLAGS = false;
    __device__ StrandTile tile(uint32_t t, uint64_t, uint64_t) const
    {
        const ChunkDesc c = ch[t];
        const TraceDesc &T = d[c.trace];
        return StrandTile{T.events, T.n, T.n_ids, T.init, T.status, nullptr, T.ctl, c.start, c.start == 0,
                          c.start + c.len == T.n};
    }
};

template <int EP, class SRC>
__global__ __launch_bounds__(SB) void k_small_check(SRC S, uint64_t *__restrict__ lbv, uint32_t *__restrict__ tcnt,
                                                    uint32_t *__restrict__ ticket, uint64_t ntiles)
{
    constexpr int ROW = EP / 2 + 4;          // words of a lane's packed events, padded (16-byte rows on all banks)
    constexpr int WE = WAVE * EP;            // events of a wave
    constexpr int GROUPS = EP / FLAG_EVENTS; // flag words per lane
    __shared__ __align__(16) uint32_t s_ev[SW][WAVE * ROW];
    __shared__ __align__(16) uint8_t s_fn[SW * SK * WAVE];
    __shared__ uint32_t s_fold[16], s_apply[16];
    __shared__ Fn32 s_wtot[SW][2];           // per wave: composition of its threads
    __shared__ uint32_t s_in[SPW][2];        // statuses entering the tile, 20 variables a word
    __shared__ uint32_t s_wsum[SW];
    __shared__ uint32_t s_tile;

    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / WAVE;
    if (tid < 16) {
        s_fold[tid] = STRAND.fold[tid];
        s_apply[tid] = STRAND.apply[tid];
    }
    __syncthreads();
    uint32_t *const rows = s_ev[wave], *const row = rows + lane * ROW;
    const uint32_t column = wave * (SK * WAVE) + lane * 4; // this lane's bytes: s_fn[place | column]
    uint32_t *const colw = reinterpret_cast<uint32_t *>(s_fn + column);
    auto table = [](const uint32_t *t, uint32_t x) {
        return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const uint8_t *>(t) + (x & TABLE_AT));
    };

    for (;;) {
        const uint32_t tile = take_ticket(ticket, &s_tile);
        if (tile >= ntiles)
            break;
        const StrandTile X = S.tile(tile, ntiles, (uint64_t)SW * WE);
        const uint32_t *const ev = X.ev;
        uint8_t *const status = X.status, *const final_out = X.final_out;
        const uint64_t n = X.n, wb = X.first + wave * WE; // the wave's first event
        const uint32_t n_ids = X.n_ids;

        // ---- 1. the wave's events, four consecutive ones a lane, packed to their rows ----
        uint32_t badm = 0, top = 0;
        constexpr int LOADS = EP / 4, BATCH = LOADS < 8 ? LOADS : 8;
        for (int q0 = 0; q0 < LOADS; q0 += BATCH) {
            uint4 v[BATCH];
#pragma unroll
            for (int q = 0; q < BATCH; q++) {
                const uint64_t g = wb + (uint32_t)(q0 + q) * (4 * WAVE) + lane * 4;
                if (g + 4 <= n) {
                    const Words4 e4 = *reinterpret_cast<const Words4 *>(ev + g);
                    v[q] = make_uint4(e4.x, e4.y, e4.z, e4.w);
                } else {
                    constexpr uint32_t NOOP = (uint32_t)OP_NOOP << 24;
                    v[q].x = g < n ? ev[g] : NOOP;
                    v[q].y = g + 1 < n ? ev[g + 1] : NOOP;
                    v[q].z = g + 2 < n ? ev[g + 2] : NOOP;
                    v[q].w = g + 3 < n ? ev[g + 3] : NOOP;
                }
            }
#pragma unroll
            for (int q = 0; q < BATCH; q++) {
                const uint32_t e = (uint32_t)(q0 + q) * (4 * WAVE) + lane * 4;
                badm |= (v[q].x | v[q].y | v[q].z | v[q].w) & 0xF0FFFFC0u;
                if (n_ids < SK) {
                    const uint32_t a = v[q].x & 63u, b = v[q].y & 63u, c = v[q].z & 63u, d = v[q].w & 63u;
                    const uint32_t ab = a > b ? a : b, cd = c > d ? c : d, m = ab > cd ? ab : cd;
                    top = top > m ? top : m;
                }
                *reinterpret_cast<uint2 *>(rows + (e / EP) * ROW + (e % EP) / 2) =
                    make_uint2(pack_event(v[q].x) | (pack_event(v[q].y) << 16),
                               pack_event(v[q].z) | (pack_event(v[q].w) << 16));
            }
        }
#pragma unroll
        for (int k = 0; k < SK / 4; k++)
            colw[k * WAVE] = 0; // identity
        lds_fence();

        // ---- 2. this strand's functions ------------------------------------------------
        uint32_t seen = 0;
        for (int c = 0; c < EP / 8; c++) {
            const uint4 v = reinterpret_cast<const uint4 *>(row)[c];
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            uint32_t t[8];
#pragma unroll
            for (int j = 0; j < 8; j++) {
                t[j] = table(s_fold, w[j >> 1] >> (16 * (j & 1)));
                seen |= t[j];
            }
#pragma unroll
            for (int j = 0; j < 8; j++) {
                uint8_t &h = s_fn[((w[j >> 1] >> (16 * (j & 1))) & PLACE) | column];
                h = (uint8_t)(t[j] >> ((4u * h) & 31u)); // (bits above the element are left over)
            }
        }
        // malformed words: the first index is reported (the walks stay inside the columns)
        if (__ballot(badm != 0 || top >= n_ids || (seen & 8u))) {
            for (uint32_t k = 0; k < (uint32_t)EP; k++) {
                const uint64_t g = wb + (uint64_t)lane * EP + k;
                const uint32_t x = g < n ? ev[g] : (uint32_t)OP_NOOP << 24;
                if ((x >> 28) != 0 || ((x >> 24) & 7u) > OP_NOOP || (x & 0xFFFFFFu) >= n_ids) {
                    if (g < n)
                        atomicMin(reinterpret_cast<unsigned long long *>(&X.ctl->err_index_lo), (unsigned long long)g);
                    break;
                }
            }
        }

        // ---- 3. the functions as planes; the composition of the strands before this one --
        Fn32 lo{0, 0, 0}, hi{0, 0, 0};
#pragma unroll
        for (int k = 0; k < SK / 4; k += 2) {
            const uint32_t a = colw[k * WAVE], b = colw[(k + 1) * WAVE];
            // eight variables a pair of words
            const uint32_t x = gather4(b, 0x01010101u, W_HI, gather4(a, 0x01010101u, W_LO, 0));
            const uint32_t y = gather4(b, 0x02020202u, W_HI, gather4(a, 0x02020202u, W_LO, 0)) >> 1;
            const uint32_t z = gather4(b, 0x04040404u, W_HI, gather4(a, 0x04040404u, W_LO, 0)) >> 2;
            Fn32 &f = k < SK / 8 ? lo : hi;
            f.x |= x << (4 * (k % (SK / 8)));
            f.y |= y << (4 * (k % (SK / 8)));
            f.t |= z << (4 * (k % (SK / 8)));
        }
        fn_wave_scan(lo, hi);
        if (lane == WAVE - 1) {
            s_wtot[wave][0] = lo;
            s_wtot[wave][1] = hi;
        }
        // exclusive: the inclusive prefix of the lane before (lane 0: identity)
        const Fn32 xlo = fn_move<DPP_WAVE_SHR1>(lo), xhi = fn_move<DPP_WAVE_SHR1>(hi);
        __syncthreads();
        // earlier waves, then the wave's own prefix
        Fn32 plo{0, 0, 0}, phi{0, 0, 0}, alo{0, 0, 0}, ahi{0, 0, 0};
#pragma unroll
        for (uint32_t w2 = 0; w2 < SW; w2++) {
            if (w2 == wave) {
                plo = alo;
                phi = ahi;
            }
            alo = fn_compose(s_wtot[w2][0], alo);
            ahi = fn_compose(s_wtot[w2][1], ahi);
        }
        plo = fn_compose(xlo, plo);
        phi = fn_compose(xhi, phi);

        // ---- 4. statuses entering the tile: look-back, one wave per word of 20 --------
        if (wave < SPW) {
            const uint32_t k = wave;
            // (places past the ids count as constants, so that a word can be all constant)
            const uint32_t past = n_ids > k * 20 + 20 ? 0u : PL_MASK & ~((1u << (n_ids > k * 20 ? n_ids - k * 20 : 0)) - 1u);
            const Planes agg{bits20(alo.t, ahi.t, k) | past, bits20(alo.x, ahi.x, k), bits20(alo.y, ahi.y, k)};
            Planes first{PL_MASK, 0, 0};
            if (X.starts) {
                const uint32_t v = k * 20 + lane;
                const uint32_t s0 = (X.init && lane < 20 && v < n_ids) ? X.init[v] : 1u;
                first.x = (uint32_t)__ballot(s0 & 1u) & PL_MASK;
                first.y = (uint32_t)__ballot((s0 >> 1) & 1u) & PL_MASK;
            }
            const Planes st = lb_planes_exclusive(lbv, SPW, tile, X.starts, k, agg, first);
            if (lane == 0) {
                s_in[k][0] = st.x;
                s_in[k][1] = st.y;
            }
            if (X.ends && final_out && lane < 20) {
                const uint32_t v = k * 20 + lane;
                const Planes inc = pl_compose(agg, st);
                if (v < n_ids)
                    final_out[v] = (uint8_t)(((inc.x >> lane) & 1u) | (((inc.y >> lane) & 1u) << 1));
            }
        }
        __syncthreads();
        uint64_t c64 = 0, g64 = 0;
#pragma unroll
        for (int k = 0; k < SPW; k++) {
            c64 |= (uint64_t)s_in[k][0] << (20 * k);
            g64 |= (uint64_t)s_in[k][1] << (20 * k);
        }
        uint32_t clo = (uint32_t)c64, chi = (uint32_t)(c64 >> 32), glo = (uint32_t)g64, ghi = (uint32_t)(g64 >> 32);
        fn_apply(plo, clo, glo);
        fn_apply(phi, chi, ghi);

        // ---- 5. the strand's statuses --------------------------------------------------
#pragma unroll
        for (int k = 0; k < SK / 4; k++) {
            const uint32_t c = k < SK / 8 ? clo : chi, g = k < SK / 8 ? glo : ghi, at = 4 * (k % (SK / 8));
            // four variables' bits to four bytes (the partial products land on distinct bits)
            const uint32_t cb = __umul24((c >> at) & 15u, 0x204081u) & 0x01010101u;
            const uint32_t gb = __umul24((g >> at) & 15u, 0x204081u) & 0x01010101u;
            colw[k * WAVE] = cb | (gb << 1);
        }
        lds_fence();
        uint32_t flags[GROUPS];
        uint32_t cnt = 0;
#pragma unroll 1
        for (int c = 0; c < EP / 16; c++) {
            uint32_t out[4];
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const uint4 v = reinterpret_cast<const uint4 *>(row)[2 * c + h];
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
                uint32_t t[8], r[8];
#pragma unroll
                for (int j = 0; j < 8; j++)
                    t[j] = table(s_apply, w[j >> 1] >> (16 * (j & 1)));
#pragma unroll
                for (int j = 0; j < 8; j++) {
                    uint8_t &s8 = s_fn[((w[j >> 1] >> (16 * (j & 1))) & PLACE) | column];
                    r[j] = t[j] >> ((8u * s8) & 31u); // (the status is the byte's low bits)
                    s8 = (uint8_t)r[j];
                }
#pragma unroll
                for (int j = 0; j < 8; j += 4) // the low bytes of four words
                    out[2 * h + j / 4] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(r[j + 3], r[j + 2], 0x0C0C0400u),
                                                               __builtin_amdgcn_perm(r[j + 1], r[j], 0x0C0C0400u),
                                                               0x05040100u);
            }
            // the row's words up to 8c + 7 have been read: the status words take their place
            reinterpret_cast<uint4 *>(row)[c] = make_uint4(out[0], out[1], out[2], out[3]);
            const uint32_t m = (gather4(out[1], 0x80808080u, W_HI, gather4(out[0], 0x80808080u, W_LO, 0)) >> 7) |
                               (gather4(out[3], 0x80808080u, W_HI, gather4(out[2], 0x80808080u, W_LO, 0)) << 1);
#pragma unroll
            for (int q = 0; q < GROUPS; q++)
                flags[q] = q == c ? m : flags[q];
            cnt += __builtin_popcount(m);
        }
        lds_fence();
        // the wave's status bytes, 16 consecutive ones a lane
#pragma unroll
        for (int q = 0; q < EP / 16; q++) {
            const uint32_t e = (q * WAVE + lane) * 16;
            const uint4 v = *reinterpret_cast<const uint4 *>(rows + (e / EP) * ROW + (e % EP) / 4);
            const uint64_t g = wb + e;
            if (g + 16 <= n) {
                *reinterpret_cast<uint4 *>(status + g) = v;
            } else {
                const uint32_t o[4] = {v.x, v.y, v.z, v.w};
                for (int j = 0; j < 16; j++)
                    if (g + j < n)
                        status[g + j] = (uint8_t)(o[j >> 2] >> (8 * (j & 3)));
            }
        }

        // ---- flagged events: per 16 their mask and offset inside the scatter tile, per
        // scatter tile the count
        const uint32_t inc = wave_scan_add(cnt, lane);
        if (lane == WAVE - 1)
            s_wsum[wave] = inc;
        __syncthreads();
        if constexpr (!SRC::FLAGS) {
            if (tid == 0)
                tcnt[tile] = s_wsum[0] + s_wsum[1] + s_wsum[2] + s_wsum[3];
            __syncthreads(); // (the next tile's sums)
            continue;
        } else {
        constexpr uint32_t TW = scatter_threads<EP>() / (WAVE * GROUPS); // waves per scatter tile
        uint32_t woff = 0, total = 0;
#pragma unroll
        for (uint32_t w2 = 0; w2 < SW; w2++) {
            if (w2 / TW == wave / TW) {
                if (w2 < wave)
                    woff += s_wsum[w2];
                total += s_wsum[w2];
            }
        }
        uint32_t o = woff + inc - cnt;
        uint32_t *const f = S.fw + ((uint64_t)tile * SB + tid) * GROUPS;
        uint32_t words[GROUPS];
#pragma unroll
        for (int q = 0; q < GROUPS; q++) {
            words[q] = flags[q] | (o << 16);
            o += __builtin_popcount(flags[q]);
        }
        if constexpr (GROUPS == 4)
            *reinterpret_cast<uint4 *>(f) = make_uint4(words[0], words[1], words[2], words[3]);
        else
#pragma unroll
            for (int q = 0; q < GROUPS; q++)
                f[q] = words[q];
        if (lane == 0 && wave % TW == 0)
            tcnt[(uint64_t)tile * (SW / TW) + wave / TW] = total;
        }
    }
}

} // namespace

// scratch: look-back words, tile counts, their offsets, the chunk scan's scratch, the
// per-thread flag words
struct SmallLayout {
    uint64_t tiles, stiles; // tiles of the check, tiles of the scatter
    uint64_t *lbv;
    uint32_t *tcnt;
    uint64_t *offs;
    void *xscan;
    uint32_t *fw;
    size_t bytes;
};

static SmallLayout small_layout(void *scratch, uint64_t n)
{
    const int ep = strand_of(n);
    const uint64_t tiles = ceil_div(n ? n : 1, (uint64_t)SB * ep);
    const uint64_t words = tiles * SB * (ep / FLAG_EVENTS);
    const uint64_t stiles = words / (ep == EP_LONG ? scatter_threads<EP_LONG>() : scatter_threads<EP_SHORT>());
    char *p = reinterpret_cast<char *>(scratch);
    size_t off = 0;
    auto take = [&](size_t sz) {
        char *r = p ? p + off : nullptr;
        off += (sz + 255) & ~size_t(255);
        return r;
    };
    SmallLayout L;
    L.tiles = tiles;
    L.stiles = stiles;
    L.lbv = reinterpret_cast<uint64_t *>(take(tiles * SPW * sizeof(uint64_t)));
    L.tcnt = reinterpret_cast<uint32_t *>(take(stiles * 4));
    L.offs = reinterpret_cast<uint64_t *>(take((stiles + 1) * 8));
    L.xscan = take(excl_scan_scratch_bytes(stiles));
    L.fw = reinterpret_cast<uint32_t *>(take(words * 4));
    L.bytes = off;
    return L;
}

// (the most a trace of n events or fewer takes: the longest one by short strands has more
// look-back words than the first by long ones)
size_t small_scratch_bytes(uint64_t n)
{
    const size_t own = small_layout(nullptr, n).bytes;
    const size_t shorter = small_layout(nullptr, n < LONG_FROM ? n : LONG_FROM - 1).bytes;
    return own > shorter ? own : shorter;
}

uint32_t small_max_ids() { return SK; }

void excl_scan_warm_launch_shape();

// computes the persistent grids of the small check once, so that later launches make
// no host-side allocation
void small_warm_launch_shapes()
{
    (void)resident_grid((const void *)k_small_check<EP_LONG, OneTrace>, 1, 0, SB);
    (void)resident_grid((const void *)k_small_check<EP_SHORT, OneTrace>, 1, 0, SB);
    excl_scan_warm_launch_shape();
}

void launch_small_check(const uint32_t *events, uint64_t n, uint32_t n_ids, const uint8_t *init, uint8_t *status,
                        uint8_t *final_out, uint32_t *viol, void *scratch, Control *ctl, hipStream_t s,
                        unsigned grid_cap, const FillJob *fin_fill)
{
    const SmallLayout L = small_layout(scratch, n);
    // one set-up launch: the control block, both look-back arrays, the caller's fill
    FillJob jobs[3] = {FillJob{L.lbv, (size_t)L.tiles * SPW * sizeof(uint64_t), 0},
                       FillJob{L.xscan, excl_scan_scratch_bytes(L.stiles), 0}, FillJob{nullptr, 0, 0}};
    if (fin_fill)
        jobs[2] = *fin_fill;
    launch_prep(ctl, nullptr, jobs, 3, s);
    if (n == 0)
        return;
    const bool is_long = strand_of(n) == EP_LONG;
    {
        const auto kernel = is_long ? k_small_check<EP_LONG, OneTrace> : k_small_check<EP_SHORT, OneTrace>;
        const unsigned grid = resident_grid((const void *)kernel, L.tiles, grid_cap, SB);
        ProfScope prof_(s, "small_check");
        kernel<<<grid, SB, 0, s>>>(OneTrace{events, n, n_ids, init, status, final_out, ctl, L.fw}, L.lbv, L.tcnt,
                                   ctl->tickets[7], L.tiles);
    }
    launch_flag_list(FlagList{L.fw, L.tcnt, L.offs, L.xscan, L.stiles},
                     is_long ? (int)scatter_threads<EP_LONG>() : (int)scatter_threads<EP_SHORT>(), viol, ctl,
                     ctl->tickets[8], s);
}

uint32_t strand_chunk() { return SB * EP_LONG; }
size_t batch_strands_bytes(uint64_t chunks) { return chunks * SPW * sizeof(uint64_t); }

void launch_batch_strands(const TraceDesc *d, const ChunkDesc *ch, uint32_t chunks, uint32_t *vcnt, uint64_t *lbv,
                          uint32_t *ticket, hipStream_t s)
{
    if (!chunks)
        return;
    launch_clear_lookback(lbv, (size_t)chunks * SPW, ticket, s);
    ProfScope p(s, "batch_strands");
    const auto kernel = k_small_check<EP_LONG, BatchStrands>;
    kernel<<<resident_grid((const void *)kernel, chunks, 0, SB), SB, 0, s>>>(BatchStrands{d, ch}, lbv, vcnt, ticket,
                                                                            chunks);
}

} // namespace vc
