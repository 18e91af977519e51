// declared.hip -- well-declaredness of component programs with explicit bodies (gfx950).
//
// Definition "Well-declared program" (Section 3.4), its array form (Section 3.5) and
// the naive rule for overlapping arrays (Section 4.1), checked for every component at
// once.  Every body event is checked on its own against its component's declarations
// (transfers, undeclared reads and writes, and, for arrays, cells shared with an
// overlapping array that is not declared for writing); the obligation of a W
// declaration (every element written on its side) is a coverage question, answered
// with one bit per element: the body's writes set their bits, and the component's end
// finds any bit left clear.  A wave has a tile of consecutive components to itself and
// works out in LDS, once per declaration, what its body events will ask (k_wd_tiles); the
// tiles that do not fit there, malformed ones among them, are listed for k_wd_big, which
// asks per event and keeps its bits in global memory.  With the extension O(M) (Table
// "Extension of access mode annotations to deal with overlapping arrays"), whether a
// variable is declared for reading or writing in O(M) is decided from M directly:
//   W or RW y in O(M)  iff  W or RW y in M, or some W or RW x in M overlaps y;
//   R or RW y in O(M)  iff  R or RW y in M, or some RW x in M overlaps y, or some
//                           W x in M overlaps y while y is not declared W;
//   W y stays W        iff  no RW x in M overlaps y  (else it is upgraded to RW);
// all on the same side.  Errors are reported with a key that orders them as a
// sequential reading does: component, then declarations before body, then index.
#include "declared.h"
#include "device.h"
#include "internal.h"
#include "prof.h"

namespace vc {

constexpr uint32_t WD_TRANSFER = 1, WD_READ = 2, WD_WRITE = 4, WD_UNWRITTEN = 8, WD_OVERLAP = 16, WD_ILL = 128;

namespace {

// error key: component << 33 | (0 declaration, 1 body word) << 32 | index
__device__ __forceinline__ void report_key(Control *ctl, uint64_t c, uint32_t kind, uint64_t index)
{
    const unsigned long long key = ((unsigned long long)c << 33) | ((unsigned long long)kind << 32) | (index & 0xFFFFFFFFull);
    atomicMin(reinterpret_cast<unsigned long long *>(&ctl->err_index_lo), key);
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, uint32_t lane)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), (int)lane) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, (int)lane);
}

struct Decl {
    uint32_t var, mode, side;
};
__device__ __forceinline__ Decl decl_of(uint32_t w) { return Decl{w & 0xFFFFFFu, (w >> 24) & 3u, (w >> 27) & 1u}; }

// what a staged declaration says of its own variable on its own side
constexpr uint32_t P_READ = 1, P_WRITE = 2, P_OBLIGED = 4, P_FORBIDDEN = 8;

// A component's declarations with the intervals of their variables: read from global
// memory (GlobalDecls) or staged in LDS for a tile of components (StagedDecls, with the
// obligation of every declaration worked out when it is staged).
// (a malformed declaration's variable, reported by the declaration pass, has the empty
// interval [0, 0))
struct GlobalDecls {
    const uint32_t *w, *lo, *hi;
    uint32_t n_vars;
    __device__ __forceinline__ bool obliged(uint64_t a, uint64_t b, uint64_t d, bool extend) const;
    __device__ __forceinline__ uint32_t word(uint64_t d) const { return w[d]; }
    __device__ __forceinline__ uint32_t vlo(uint64_t d) const
    {
        const uint32_t x = w[d] & 0xFFFFFFu;
        return x < n_vars ? lo[x] : 0u;
    }
    __device__ __forceinline__ uint32_t vhi(uint64_t d) const
    {
        const uint32_t x = w[d] & 0xFFFFFFu;
        return x < n_vars ? hi[x] : 0u;
    }
};
struct StagedDecls {
    const uint32_t *w, *lo, *hi;
    const uint8_t *perm;
    __device__ __forceinline__ bool obliged(uint64_t, uint64_t, uint64_t d, bool) const
    {
        return (perm[d] & P_OBLIGED) != 0;
    }
    __device__ __forceinline__ uint32_t word(uint64_t d) const { return w[d]; }
    __device__ __forceinline__ uint32_t vlo(uint64_t d) const { return lo[d]; }
    __device__ __forceinline__ uint32_t vhi(uint64_t d) const { return hi[d]; }
};

// the declaration of y on side s in M (index in [a, b)), or b if none
template <class D>
__device__ __forceinline__ uint64_t find_decl(const D &M, uint64_t a, uint64_t b, uint32_t y, uint32_t s)
{
    for (uint64_t d = a; d < b; d++) {
        const Decl q = decl_of(M.word(d));
        if (q.var == y && q.side == s)
            return d;
    }
    return b;
}

// is y (interval [ylo, yhi)) declared for writing (W or RW) on side s, in M or in O(M)
template <class D>
__device__ __forceinline__ bool writable(const D &M, uint64_t a, uint64_t b, uint32_t y, uint32_t s, uint32_t ylo,
                                         uint32_t yhi, bool extend)
{
    bool ok = false;
    for (uint64_t d = a; d < b; d++) {
        const Decl q = decl_of(M.word(d));
        if (q.side != s || q.mode == 0)
            continue;
        ok |= q.var == y || (extend && M.vlo(d) < yhi && ylo < M.vhi(d));
    }
    return ok;
}

// is y (interval [ylo, yhi)) declared for reading (R or RW) on side s, in M or in O(M)
template <class D>
__device__ __forceinline__ bool readable(const D &M, uint64_t a, uint64_t b, uint32_t y, uint32_t s, uint32_t ylo,
                                         uint32_t yhi, bool extend)
{
    bool own_r = false, own_w = false, by_rw = false, by_w = false;
    for (uint64_t d = a; d < b; d++) {
        const Decl q = decl_of(M.word(d));
        if (q.side != s)
            continue;
        if (q.var == y) {
            own_r |= q.mode == 0 || q.mode == 2;
            own_w |= q.mode == 1;
        } else if (extend && M.vlo(d) < yhi && ylo < M.vhi(d)) {
            by_rw |= q.mode == 2;
            by_w |= q.mode == 1;
        }
    }
    return own_r || by_rw || (by_w && !own_w);
}

// W declaration d of component [a, b) that keeps its obligation (not upgraded)
template <class D>
__device__ __forceinline__ bool obliged_scan(const D &M, uint64_t a, uint64_t b, uint64_t d, bool extend)
{
    const Decl q = decl_of(M.word(d));
    if (q.mode != 1)
        return false;
    if (!extend)
        return true;
    const uint32_t qlo = M.vlo(d), qhi = M.vhi(d);
    for (uint64_t e = a; e < b; e++) {
        const Decl r = decl_of(M.word(e));
        if (r.side == q.side && r.mode == 2 && r.var != q.var && M.vlo(e) < qhi && qlo < M.vhi(e))
            return false;
    }
    return true;
}
__device__ __forceinline__ bool GlobalDecls::obliged(uint64_t a, uint64_t b, uint64_t d, bool extend) const
{
    return obliged_scan(*this, a, b, d, extend);
}

// what the kernels read
struct WdInputs {
    const uint64_t *comp_off, *body_off;
    const uint32_t *decls, *body, *idx, *lo, *hi;
    const uint64_t *off; // the arrays' neighbours
    const uint32_t *nbr;
    uint64_t n_comp, n_decl, n_body;
    uint32_t n_vars;
    bool ext; // the extension, with arrays
};

// The declarations of component c checked (as the translation does), and the number of
// coverage bits of every one (the length of an obliged declaration's variable); returns
// their sum.
__device__ __forceinline__ uint64_t check_decls(const GlobalDecls &M, uint64_t c, uint64_t a, uint64_t b, bool ext,
                                                uint32_t *__restrict__ wlen, Control *ctl)
{
    bool bad = false;
    for (uint64_t d = a; d < b && !bad; d++) {
        const uint32_t w = M.w[d];
        bool ok = (w >> 28) == 0 && ((w >> 26) & 1u) == 0 && ((w >> 24) & 3u) != 3 && (w & 0xFFFFFFu) < M.n_vars;
        for (uint64_t e = a; e < d && ok; e++)
            ok = ((M.w[e] ^ w) & 0xFFFFFFu) != 0;
        if (!ok) {
            report_key(ctl, c, 0, d);
            bad = true;
        }
    }
    uint64_t sum = 0;
    for (uint64_t d = a; d < b; d++) {
        uint32_t len = 0;
        if (!bad && obliged_scan(M, a, b, d, ext))
            len = M.lo ? M.vhi(d) - M.vlo(d) : 1u;
        wlen[d] = len;
        sum += len;
    }
    return sum;
}

__global__ void k_wd_decls(WdInputs I, uint32_t *__restrict__ wlen, Control *ctl)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const GlobalDecls G{I.decls, I.lo, I.hi, I.n_vars};
    for (uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; c < I.n_comp; c += stride) {
        const uint64_t a = I.comp_off[c], b = I.comp_off[c + 1];
        if (b < a || b > I.n_decl)
            report_key(ctl, c, 0, c);
        else
            (void)check_decls(G, c, a, b, I.ext, wlen, ctl);
    }
}

// The conditions that body event j (word e, element i) of component c breaks, against its
// declarations [a, b) of M.  A malformed event is reported.
template <class D>
__device__ __forceinline__ uint32_t body_event(uint64_t c, const D &M, uint64_t a, uint64_t b, uint64_t j, uint32_t e,
                                               uint32_t i, const WdInputs &I, Control *ctl)
{
    const uint32_t x = e & 0xFFFFFFu, op = (e >> 24) & 7u, s = (e >> 27) & 1u;
    const uint32_t xlo = I.lo && x < I.n_vars ? I.lo[x] : 0u, xhi = I.lo && x < I.n_vars ? I.hi[x] : 1u;
    if ((e >> 28) != 0 || op > OP_NOOP || x >= I.n_vars || (I.lo ? i >= xhi - xlo : i != 0)) {
        report_key(ctl, c, 1, j);
        return 0;
    }
    uint32_t v = 0;
    if (op == OP_PUSH || op == OP_PULL)
        v |= WD_TRANSFER;
    if (op == OP_R && !readable(M, a, b, x, s, xlo, xhi, I.ext))
        v |= WD_READ;
    if (op == OP_W) {
        if (!writable(M, a, b, x, s, xlo, xhi, I.ext))
            v |= WD_WRITE;
        if (I.lo) {
            // the naive rule: every other array holding the written cell
            const uint32_t addr = xlo + i;
            for (uint64_t q = I.off[x]; q < I.off[x + 1]; q++) {
                const uint32_t y = I.nbr[q], ylo = I.lo[y], yhi = I.hi[y];
                if (ylo <= addr && addr < yhi && !writable(M, a, b, y, s, ylo, yhi, I.ext))
                    v |= WD_OVERLAP;
            }
        }
    }
    return v;
}

// the obliged declaration (index in [a, b)) that body word e writes, or b if none
template <class D>
__device__ __forceinline__ uint64_t obliged_decl(const D &M, uint64_t a, uint64_t b, uint32_t e, bool ext)
{
    if (((e >> 24) & 7u) != OP_W)
        return b;
    const uint64_t d = find_decl(M, a, b, e & 0xFFFFFFu, (e >> 27) & 1u);
    return d < b && M.obliged(a, b, d, ext) ? d : b;
}

constexpr uint32_t WD_STAGE = 384;   // declarations of a tile
constexpr uint32_t WD_CELLS = 8192;  // elements of its W and RW declarations
constexpr int WD_BIG = 12;           // counter of the listed tiles (tickets[WD_BIG][0])

__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); } // (a wave's LDS operations are in order)

// Tiles of up to 64 consecutive components, a wave each.  The tile's declarations (at most
// WD_STAGE) are staged with their variables' intervals; a component's lane checks them and
// works out for each what it permits on its own variable and side, and where the bits of
// its elements lie (W and RW; at most WD_CELLS a tile): `cover` takes the body's writes,
// `forbid` holds the cells of an overlapping array that the component may not write.  With
// the extension there are none: an overlapping array of a writable one is writable too.
// The tile's body events are consecutive and walked 64 at a time; the lane of each finds
// its component from a ballot of the components' starts among the 64 and its declaration
// among the component's.  An event whose variable is not declared on its side asks as
// k_wd_big does.
// Bound by the chains of dependent LDS reads of a step, and of loads for the few events
// that are not declared.  2^18 components of 1-4 arrays of 1-64 elements with the extension
// (7.4 M body events): asking for every event with the bits in global memory 268 us, with
// the declarations' lengths, their scan, two clears and the end in passes of their own
// (37, 15 and 18 us); this way 63 in all.  256 components 105 and 20, 2^17 without the
// extension 196 and 45; 2^14 of 8 arrays of up to 1,024 elements, none of whose tiles fit,
// 2.9 ms and 0.8.
__global__ __launch_bounds__(WAVE) void k_wd_tiles(WdInputs I, uint32_t per, uint8_t *__restrict__ out,
                                                   uint32_t *__restrict__ big, Control *ctl)
{
    __shared__ uint32_t s_w[WD_STAGE], s_lo[WD_STAGE], s_hi[WD_STAGE];
    __shared__ uint16_t s_base[WD_STAGE];
    __shared__ uint8_t s_perm[WD_STAGE], s_comp[WD_STAGE];
    __shared__ uint32_t s_cover[WD_CELLS / 32], s_forbid[WD_CELLS / 32];
    __shared__ uint32_t s_dstart[WAVE + 1], s_start[WAVE + 1], s_lane[WAVE], s_mark[WAVE], s_verdict[WAVE];
    const uint32_t lane = threadIdx.x;
    const StagedDecls S{s_w, s_lo, s_hi, s_perm};
    const uint64_t tile = blockIdx.x, c0 = tile * per, c = c0 + lane;
    const uint32_t nc = (uint32_t)(I.n_comp - c0 < per ? I.n_comp - c0 : per);
    const bool mine = lane < nc;
    const uint64_t a = I.comp_off[mine ? c : c0 + nc], b = I.comp_off[mine ? c + 1 : c0 + nc];
    const uint64_t j0 = I.body_off[mine ? c : c0 + nc], j1 = I.body_off[mine ? c + 1 : c0 + nc];
    const uint64_t A = readlane64(a, 0), J = readlane64(j0, 0);
    const uint64_t B = readlane64(b, nc - 1), E = readlane64(j1, nc - 1);
    const bool well = a <= b && b <= I.n_decl && j0 <= j1 && j1 <= I.n_body;
    if (__ballot(!well) || B - A > WD_STAGE || E - J >= (1u << 30)) { // (uniform)
        if (lane == 0)
            big[atomicAdd(&ctl->tickets[WD_BIG][0], 1u)] = (uint32_t)tile;
        return;
    }
    const uint32_t nd = (uint32_t)(B - A), total = (uint32_t)(E - J);
    const uint32_t da = (uint32_t)(a - A), db = (uint32_t)(b - A);
    // the first events, on their way while the declarations are worked out
    constexpr uint32_t AHEAD = 4;
    uint32_t ev[AHEAD], ix[AHEAD];
    auto load = [&](uint32_t q0) {
#pragma unroll
        for (uint32_t u = 0; u < AHEAD; u++) {
            const uint32_t q = q0 + u * WAVE + lane;
            ev[u] = q < total ? I.body[J + q] : 0u;
            ix[u] = q < total && I.idx ? I.idx[J + q] : 0u;
        }
    };
    load(0);
    for (uint32_t k = lane; k < nd; k += WAVE) {
        const uint32_t w = I.decls[A + k], x = w & 0xFFFFFFu;
        const bool known = x < I.n_vars;
        s_w[k] = w;
        s_lo[k] = I.lo && known ? I.lo[x] : 0u;
        s_hi[k] = !known ? 0u : I.lo ? I.hi[x] : 1u;
    }
    s_dstart[lane] = da;
    if (lane == WAVE - 1)
        s_dstart[WAVE] = nd;
    s_verdict[lane] = 0;
    lds_order();
    // the component's declarations: well formed, each variable once; their cells
    bool bad = false;
    uint64_t cells = 0;
    for (uint32_t d = da; d < db && !bad; d++) {
        const uint32_t w = s_w[d];
        bool ok = (w >> 28) == 0 && ((w >> 26) & 1u) == 0 && ((w >> 24) & 3u) != 3 && (w & 0xFFFFFFu) < I.n_vars;
        for (uint32_t e = da; e < d && ok; e++)
            ok = ((s_w[e] ^ w) & 0xFFFFFFu) != 0;
        if (!ok) {
            report_key(ctl, c, 0, A + d);
            bad = true;
        }
        cells += ok && decl_of(w).mode ? s_hi[d] - s_lo[d] : 0u;
    }
    const uint32_t own_cells = bad ? 0u : (uint32_t)(cells < WD_CELLS + 1 ? cells : WD_CELLS + 1);
    const uint32_t upto = wave_scan_add(own_cells, lane);
    const uint32_t ncells = (uint32_t)__builtin_amdgcn_readlane((int)upto, WAVE - 1);
    if (ncells > WD_CELLS) { // (uniform)
        if (lane == 0)
            big[atomicAdd(&ctl->tickets[WD_BIG][0], 1u)] = (uint32_t)tile;
        return;
    }
    for (uint32_t k = lane; k < ceil_div(ncells, 32u); k += WAVE) {
        s_cover[k] = 0;
        s_forbid[k] = 0;
    }
    uint32_t base = upto - own_cells;
    for (uint32_t d = da; d < db; d++) {
        const Decl q = decl_of(s_w[d]);
        const uint32_t qlo = s_lo[d], qhi = s_hi[d];
        bool by_rw = false; // overlapped by one of its side declared RW
        if (I.ext)
            for (uint32_t e = da; e < db; e++) {
                const Decl r = decl_of(s_w[e]);
                by_rw |= r.mode == 2 && r.side == q.side && r.var != q.var && s_lo[e] < qhi && qlo < s_hi[e];
            }
        uint32_t p = 0;
        if (q.mode == 0 || q.mode == 2 || by_rw) // (W stays W unless it is upgraded)
            p |= P_READ;
        if (q.mode != 0)
            p |= P_WRITE;
        if (q.mode == 1 && !by_rw && !bad)
            p |= P_OBLIGED;
        s_perm[d] = (uint8_t)p;
        s_comp[d] = (uint8_t)lane;
        s_base[d] = (uint16_t)base;
        base += !bad && q.mode ? qhi - qlo : 0u;
    }
    const uint64_t bad_comps = __ballot(bad);
    lds_order();
    if (I.off && !I.ext)
        for (uint32_t k = lane; k < nd; k += WAVE) {
            const uint32_t comp = s_comp[k];
            const Decl q = decl_of(s_w[k]);
            if (q.mode == 0 || ((bad_comps >> comp) & 1u))
                continue;
            const uint32_t ca = s_dstart[comp], cb = s_dstart[comp + 1];
            const uint64_t n1 = I.off[q.var + 1];
            for (uint64_t n = I.off[q.var]; n < n1; n++) {
                const uint32_t y = I.nbr[n], ylo = I.lo[y], yhi = I.hi[y];
                if (writable(S, ca, cb, y, q.side, ylo, yhi, false))
                    continue;
                const uint32_t from = (ylo > s_lo[k] ? ylo : s_lo[k]) - s_lo[k];
                const uint32_t to = (yhi < s_hi[k] ? yhi : s_hi[k]) - s_lo[k];
                for (uint32_t p = s_base[k] + from, e = s_base[k] + to; p < e;) {
                    const uint32_t b0 = p & 31u, span = e - p < 32u - b0 ? e - p : 32u - b0;
                    atomicOr(&s_forbid[p >> 5], (span == 32u ? ~0u : ((1u << span) - 1u)) << b0);
                    p += span;
                }
                s_perm[k] = (uint8_t)(s_perm[k] | P_FORBIDDEN);
            }
        }
    // the components' starts among the tile's events
    const uint32_t len = (uint32_t)(j1 - j0);
    const uint64_t nonempty = __ballot(len > 0);
    const uint32_t nne = (uint32_t)__builtin_popcountll(nonempty);
    if (len > 0) {
        const uint32_t r = mask_rank(nonempty);
        s_start[r] = (uint32_t)(j0 - J);
        s_lane[r] = lane;
    }
    lds_order();
    uint32_t ec = 0; // the component (by rank) covering slot q0 - 1
    for (uint32_t q0 = 0; q0 < total; q0 += AHEAD * WAVE) {
        uint32_t now[AHEAD], nix[AHEAD];
#pragma unroll
        for (uint32_t u = 0; u < AHEAD; u++) {
            now[u] = ev[u];
            nix[u] = ix[u];
        }
        load(q0 + AHEAD * WAVE);
#pragma unroll
        for (uint32_t u = 0; u < AHEAD; u++) {
            const uint32_t qc = q0 + u * WAVE, q = qc + lane;
            if (qc >= total)
                break; // (uniform)
            const uint32_t r = ec + 1 + lane;
            const uint32_t st = r < nne ? s_start[r] : total;
            s_mark[lane] = 0;
            lds_order();
            if (st < total && st < qc + WAVE)
                s_mark[st - qc] = 1;
            lds_order();
            const uint64_t heads = __ballot(s_mark[lane] != 0);
            const uint32_t own = ec + mask_rank(heads) + (uint32_t)((heads >> lane) & 1u);
            ec += (uint32_t)__builtin_popcountll(heads);
            if (q >= total)
                continue;
            const uint32_t e = now[u], op = (e >> 24) & 7u, i = nix[u];
            const uint32_t ol = s_lane[own], ca = s_dstart[ol], cb = s_dstart[ol + 1];
            uint32_t d = cb; // the event's variable's declaration (four read together)
            for (uint32_t k = ca; k < cb && d == cb; k += 4) {
#pragma unroll
                for (uint32_t t = 4; t-- > 0;) {
                    const uint32_t at = k + t < cb ? k + t : cb - 1;
                    d = ((s_w[at] ^ e) & 0xFFFFFFu) ? d : at;
                }
            }
            uint32_t v = 0;
            const uint32_t p = d < cb ? s_perm[d] : 0u;
            if (d < cb && ((s_w[d] ^ e) & (1u << 27)) == 0 && (op != OP_W || (p & P_WRITE)) &&
                (e >> 28) == 0 && op <= OP_NOOP && i < s_hi[d] - s_lo[d] && !((bad_comps >> ol) & 1u)) {
                if (op == OP_PUSH || op == OP_PULL)
                    v = WD_TRANSFER;
                if (op == OP_R && !(p & P_READ))
                    v = WD_READ;
                if (op == OP_W) {
                    const uint32_t cell = s_base[d] + i, bit = 1u << (cell & 31u);
                    if (p & P_OBLIGED)
                        atomicOr(&s_cover[cell >> 5], bit);
                    if ((p & P_FORBIDDEN) && (s_forbid[cell >> 5] & bit))
                        v = WD_OVERLAP;
                }
            } else {
                v = body_event(c0 + ol, S, ca, cb, J + q, e, i, I, ctl);
            }
            if (v)
                atomicOr(&s_verdict[ol], v);
        }
    }
    lds_order();
    if (mine) {
        uint32_t v = s_verdict[lane];
        for (uint32_t d = da; d < db && !(v & WD_UNWRITTEN); d++)
            if (s_perm[d] & P_OBLIGED) {
                const uint32_t p0 = s_base[d], e = p0 + (s_hi[d] - s_lo[d]);
                for (uint32_t p = p0; p < e;) {
                    const uint32_t b0 = p & 31u, span = e - p < 32u - b0 ? e - p : 32u - b0;
                    const uint32_t mask = (span == 32u ? ~0u : ((1u << span) - 1u)) << b0;
                    if ((s_cover[p >> 5] & mask) != mask) {
                        v |= WD_UNWRITTEN;
                        break;
                    }
                    p += span;
                }
            }
        out[c] = (uint8_t)(v | (v ? WD_ILL : 0u));
    }
}

// The listed tiles, a wave each, 64 body events at a time of the tile's components (those
// with an empty or malformed body range take no slot; a malformed one is reported).  Every
// event is checked against its component's declarations, which are staged when they are at
// most WD_STAGE.  The coverage bits of the tile's obliged declarations are a piece of
// `bits` (at most nbits in all), taken and cleared by the wave.
__global__ __launch_bounds__(WAVE) void k_wd_big(WdInputs I, uint32_t per, const uint32_t *__restrict__ big,
                                                 uint32_t *__restrict__ wlen, uint64_t *__restrict__ boff,
                                                 uint32_t *__restrict__ bits, uint64_t nbits,
                                                 uint32_t *__restrict__ verdict, uint8_t *__restrict__ out, Control *ctl)
{
    __shared__ uint32_t s_start[WAVE + 1], s_lane[WAVE], s_mark[WAVE];
    __shared__ uint64_t s_bo[WAVE];
    __shared__ uint32_t s_w[WD_STAGE], s_lo[WD_STAGE], s_hi[WD_STAGE];
    __shared__ uint8_t s_obl[WD_STAGE];
    const uint32_t lane = threadIdx.x, tiles = ctl->tickets[WD_BIG][0];
    const GlobalDecls G{I.decls, I.lo, I.hi, I.n_vars};
    const StagedDecls S{s_w, s_lo, s_hi, s_obl};
    for (uint32_t k = blockIdx.x; k < tiles; k += gridDim.x) {
        const uint64_t c0 = (uint64_t)big[k] * per, c = c0 + lane;
        const uint32_t nc = (uint32_t)(I.n_comp - c0 < per ? I.n_comp - c0 : per);
        uint64_t a = 0, b = 0, j0 = 0, cells = 0;
        uint32_t len = 0;
        bool ok = true;
        if (lane < nc) {
            a = I.comp_off[c];
            b = I.comp_off[c + 1];
            ok = a <= b && b <= I.n_decl;
            if (!ok)
                report_key(ctl, c, 0, c);
            j0 = I.body_off[c];
            const uint64_t j1 = I.body_off[c + 1];
            if (j1 < j0 || j1 > I.n_body)
                report_key(ctl, c, 1, j0);
            else
                len = (uint32_t)(j1 - j0); // below 2^32 (n_body < 2^32)
            if (ok)
                cells = check_decls(G, c, a, b, I.ext, wlen, ctl);
            verdict[c] = 0;
        }
        // where the coverage bits lie
        uint64_t upto = cells;
        for (uint32_t d = 1; d < WAVE; d <<= 1) {
            const uint64_t t = __shfl_up(upto, d);
            upto += lane >= d ? t : 0;
        }
        const uint64_t all = readlane64(upto, WAVE - 1), room = (all + 31) & ~(uint64_t)31;
        uint64_t base = 0;
        if (lane == 0 && room)
            base = atomicAdd(&ctl->n_out, (unsigned long long)room); // (the bits handed out)
        base = readlane64(base, 0);
        if (lane < nc && ok) {
            uint64_t p = base + upto - cells;
            for (uint64_t d = a; d < b; d++) {
                boff[d] = p;
                p += wlen[d];
            }
        }
        for (uint64_t p = base + 32u * lane; p < base + room && p < nbits; p += 32u * WAVE)
            bits[p >> 5] = 0;
        // stage the tile's declarations when the offsets are well formed
        const uint64_t A = readlane64(a, 0), B = readlane64(b, nc - 1);
        const bool staged = __ballot(!ok) == 0 && B - A <= (uint64_t)WD_STAGE;
        if (staged) {
            const uint32_t nd = (uint32_t)(B - A);
            for (uint32_t d = lane; d < nd; d += WAVE) {
                s_w[d] = I.decls[A + d];
                s_lo[d] = G.lo ? G.vlo(A + d) : 0u;
                s_hi[d] = G.lo ? G.vhi(A + d) : 0u;
                s_obl[d] = 0;
            }
            lds_order();
            if (lane < nc)
                for (uint64_t d = a - A; d < b - A; d++)
                    s_obl[d] = obliged_scan(S, a - A, b - A, d, I.ext) ? P_OBLIGED : 0u;
        }
        const uint64_t ne = __ballot(len > 0);
        const uint32_t r = mask_rank(ne);
        const uint32_t inc = wave_scan_add(len, lane);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, WAVE - 1);
        const uint32_t nne = (uint32_t)__builtin_popcountll(ne);
        if (len > 0) {
            s_start[r] = inc - len;
            s_lane[r] = lane;
            s_bo[r] = j0;
        }
        if (lane == 0)
            s_start[nne] = total;
        __threadfence(); // (the cleared bits and the offsets, before other lanes use them)
        uint32_t ec = 0; // the component (by rank) covering slot qc - 1
        for (uint32_t qc = 0; qc < total; qc += WAVE) {
            // ranks ec + 1 .. ec + 64 hold every start inside [qc, qc + 64)
            const uint32_t e = ec + 1 + lane;
            const uint32_t st = e <= nne ? s_start[e] : total;
            s_mark[lane] = 0;
            lds_order();
            if (st < total && st < qc + WAVE)
                s_mark[st - qc] = 1;
            lds_order();
            const uint64_t heads = __ballot(s_mark[lane] != 0);
            const uint32_t own = ec + mask_rank(heads) + (uint32_t)((heads >> lane) & 1u);
            const uint32_t q = qc + lane;
            // the owner's declaration range, from its lane
            const uint32_t ol = q < total ? s_lane[own] : 0u;
            const uint64_t oa = __shfl(a, (int)ol), ob = __shfl(b, (int)ol);
            const bool ook = __shfl(ok ? 1 : 0, (int)ol) != 0;
            if (q < total) {
                const uint64_t j = s_bo[own] + (q - s_start[own]);
                const uint32_t w = I.body[j], i = I.idx ? I.idx[j] : 0u;
                uint32_t v;
                uint64_t d = 0, last = 0;
                if (staged) {
                    v = body_event(c0 + ol, S, oa - A, ob - A, j, w, i, I, ctl);
                    d = A + obliged_decl(S, oa - A, ob - A, w, I.ext);
                    last = ob;
                } else {
                    // (a malformed declaration range was reported)
                    v = body_event(c0 + ol, G, ook ? oa : 0, ook ? ob : 0, j, w, i, I, ctl);
                    d = ook ? obliged_decl(G, oa, ob, w, I.ext) : 0;
                    last = ook ? ob : 0;
                }
                if (d < last && i < wlen[d]) {
                    const uint64_t bit = boff[d] + i;
                    if (bit < nbits)
                        atomicOr(&bits[bit >> 5], 1u << (bit & 31u));
                }
                if (v && ook)
                    atomicOr(&verdict[c0 + ol], v);
            }
            ec += (uint32_t)__builtin_popcountll(heads);
            lds_order();
        }
        __threadfence();
        if (lane < nc) {
            uint32_t v = __hip_atomic_load(&verdict[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (ok)
                for (uint64_t d = a; d < b && !(v & WD_UNWRITTEN); d++) {
                    // the declaration's obligation bits [p0, p1), a 32-bit word at a time
                    const uint64_t p0 = boff[d], e = p0 + wlen[d], p1 = e < nbits ? e : nbits;
                    for (uint64_t p = p0; p < p1;) {
                        const uint32_t b0 = (uint32_t)(p & 31u);
                        const uint64_t span = p1 - p < 32u - b0 ? p1 - p : 32u - b0;
                        const uint32_t mask = (span == 32 ? ~0u : ((1u << span) - 1u)) << b0;
                        if ((__hip_atomic_load(&bits[p >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & mask) !=
                            mask) {
                            v |= WD_UNWRITTEN;
                            break;
                        }
                        p += span;
                    }
                }
            out[c] = (uint8_t)(v | (v ? WD_ILL : 0u));
        }
        lds_order();
    }
}

unsigned grid_w(uint64_t n)
{
    uint64_t g = ceil_div(n ? n : 1, (uint64_t)BLOCK * 4);
    return (unsigned)(g > 16384 ? 16384 : g);
}

} // namespace

static WdInputs wd_inputs(const WdProgram &P)
{
    const OverlapSets *o = P.sets;
    return WdInputs{P.comp_off, P.body_off, P.decls, P.body, P.idx, P.lo, P.hi, o ? o->off : nullptr,
                    o ? o->nbr : nullptr, P.n_comp, P.n_decl, P.n_body, P.n_vars, P.extend && P.lo};
}

// Components a tile: 64, fewer (but 8) while the tiles are too few for 16 waves a CU (2^18
// components: 63 us by 64, 69 by 32, 78 by 16).
static uint32_t wd_per(uint64_t n_comp)
{
    uint32_t per = WAVE;
    while (per > 8 && n_comp < (uint64_t)per * 4096)
        per /= 2;
    return per;
}

uint64_t wd_tiles(uint64_t n_comp) { return ceil_div(n_comp, (uint64_t)wd_per(n_comp)); }

void launch_wd_decls(const WdProgram &P, uint32_t *wlen, Control *ctl, hipStream_t s)
{
    if (P.n_comp) {
        ProfScope p(s, "wd_decls");
        k_wd_decls<<<grid_w(P.n_comp), BLOCK, 0, s>>>(wd_inputs(P), wlen, ctl);
    }
}

void launch_wd_check(const WdProgram &P, uint32_t *big, uint32_t *wlen, uint64_t *boff, uint32_t *bits,
                     uint64_t nbits, uint32_t *verdict, uint8_t *out, Control *ctl, hipStream_t s)
{
    if (!P.n_comp)
        return;
    const WdInputs I = wd_inputs(P);
    const uint32_t per = wd_per(P.n_comp);
    const uint64_t tiles = wd_tiles(P.n_comp);
    {
        ProfScope p(s, "wd_tiles");
        k_wd_tiles<<<(unsigned)tiles, WAVE, 0, s>>>(I, per, out, big, ctl);
    }
    // (the waves that the device holds when most tiles may be listed, judged by what the
    // program had when it was loaded; a few, which mostly find no tile, otherwise)
    const bool most = P.n_decl / tiles > WD_STAGE / 2 || nbits / tiles > WD_CELLS / 2;
    const uint64_t grid = most ? 256 * 20 : 512;
    ProfScope p(s, "wd_big");
    k_wd_big<<<(unsigned)(tiles < grid ? tiles : grid), WAVE, 0, s>>>(I, per, big, wlen, boff, bits, nbits, verdict, out,
                                                                      ctl);
}

} // namespace vc
