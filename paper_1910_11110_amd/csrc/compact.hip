// compact.hip -- coalesced compaction of violation flags (gfx950).
//
// Reads the per-event status bytes in program order (16 bytes per thread and load), counts
// flagged events per tile, obtains the tile's output offset by decoupled look-back, stages
// ascending indices in LDS, 4096 events at a time, and writes each as one contiguous run.
#include "device.h"
#include "internal.h"
#include "prof.h"

namespace vc {

namespace {

constexpr int CITEMS = 16;
constexpr int CPART = BLOCK * CITEMS; // events staged together

// Parts a tile: the look-back, whose cost grows with the number of tiles that poll, bounds
// long traces; short ones want the workgroups.  2^24 events: 34.5 us by 4,096 and 21.5 by
// 16,384; 2^22 16.2 and 12.6; 2^21 12.7 and no better.
constexpr int C_LONG = 4;
constexpr uint64_t C_LONG_FROM = 1ull << 22;
int parts_of(uint64_t n) { return n >= C_LONG_FROM ? C_LONG : 1; }

template <int PARTS>
__global__ __launch_bounds__(BLOCK) void k_compact(const uint8_t *__restrict__ status, uint64_t n,
                                                   uint32_t *__restrict__ viol, uint64_t *__restrict__ lb,
                                                   uint32_t *__restrict__ ticket, uint64_t ntiles, Control *ctl,
                                                   const unsigned long long *__restrict__ flagged,
                                                   const unsigned long long *__restrict__ n_dev)
{
    constexpr uint64_t CTILE = (uint64_t)PARTS * CPART;
    __shared__ uint32_t s_idx[CPART];
    __shared__ uint32_t s_wsum[PARTS][BLOCK / WAVE];
    __shared__ uint32_t s_tile;
    __shared__ unsigned long long s_excl;

    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / WAVE;
    if (flagged && *flagged == 0)
        return; // nothing flagged: the list is empty (n_viol stays 0)
    if (n_dev && *n_dev < n) {
        n = *n_dev;
        ntiles = ceil_div(n, CTILE);
    }
    for (;;) {
        const uint32_t tile = take_ticket(ticket, &s_tile);
        if (tile >= ntiles)
            break;
        const uint64_t base = (uint64_t)tile * CTILE;
        uint4 v[PARTS];
#pragma unroll
        for (int p = 0; p < PARTS; p++) {
            const uint64_t my0 = base + (uint64_t)p * CPART + (uint64_t)tid * CITEMS;
            v[p] = make_uint4(0, 0, 0, 0);
            if (my0 + CITEMS <= n) {
                v[p] = *reinterpret_cast<const uint4 *>(status + my0);
            } else if (my0 < n) {
                uint32_t w[4] = {0, 0, 0, 0};
                for (int k = 0; k < CITEMS; k++)
                    if (my0 + k < n)
                        w[k >> 2] |= (uint32_t)status[my0 + k] << (8 * (k & 3));
                v[p] = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
        uint32_t bits[PARTS], off[PARTS]; // off: of the thread's flagged events in their part
#pragma unroll
        for (int p = 0; p < PARTS; p++) {
            const uint32_t w[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
            bits[p] = 0;
#pragma unroll
            for (int q = 0; q < 4; q++) // bits 7, 15, 23, 31 to four neighbouring ones
                bits[p] |= (((w[q] & 0x80808080u) * 0x00204081u) >> 28) << (4 * q);
            const uint32_t cnt = __builtin_popcount(bits[p]);
            const uint32_t inc = wave_scan_add(cnt, lane);
            off[p] = inc - cnt;
            if (lane == WAVE - 1)
                s_wsum[p][wave] = inc;
        }
        __syncthreads();
        uint32_t total = 0, part[PARTS];
#pragma unroll
        for (int p = 0; p < PARTS; p++) {
            part[p] = 0;
            for (uint32_t w = 0; w < BLOCK / WAVE; w++) {
                if (w < wave)
                    off[p] += s_wsum[p][w];
                part[p] += s_wsum[p][w];
            }
            total += part[p];
        }
        if (wave == 0) {
            const uint64_t excl = lb_count_exclusive(lb, tile, total);
            if (lane == 0) {
                s_excl = excl;
                if (base + CTILE >= n)
                    ctl->n_viol = excl + total;
            }
        }
        uint64_t to = 0;
#pragma unroll
        for (int p = 0; p < PARTS; p++) {
            const uint32_t my0 = (uint32_t)(base + (uint64_t)p * CPART + (uint64_t)tid * CITEMS);
            uint32_t k = off[p], m = bits[p];
            while (m) {
                s_idx[k++] = my0 + __builtin_ctz(m);
                m &= m - 1;
            }
            __syncthreads();
            if (p == 0)
                to = s_excl;
            for (uint32_t i = tid; i < part[p]; i += BLOCK)
                viol[to + i] = s_idx[i];
            to += part[p];
            __syncthreads();
        }
    }
}

// Violation indices from per-thread flag words of 16 consecutive events (flag mask |
// the thread's offset among its tile's flagged events << 16) and the tiles' offsets
// among all flagged events: offs (ntiles + 1 entries), or, without it, the sums of the
// tiles' counts tcnt, which every workgroup works out (one workgroup a tile), the last one
// the whole number.  Each thread lists its flagged indices in LDS at its offset, then the
// tile's run is written out contiguously.
template <int TB, bool SUM>
__global__ __launch_bounds__(TB) void k_flag_scatter(const uint32_t *__restrict__ fw, const uint64_t *__restrict__ offs,
                                                     const uint32_t *__restrict__ tcnt, uint64_t ntiles,
                                                     uint32_t *__restrict__ viol, unsigned long long *n_viol)
{
    constexpr uint32_t TE = TB * FLAG_EVENTS; // events per tile
    __shared__ uint32_t s_idx[TE];
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        uint64_t o0, total;
        if constexpr (SUM) {
            o0 = sum_before<TB>(tcnt, (uint32_t)tile);
            total = tcnt[tile];
            if (tile + 1 == ntiles && threadIdx.x == 0)
                *n_viol = o0 + total;
        } else {
            o0 = offs[tile];
            total = offs[tile + 1] - o0;
        }
        if (total == 0)
            continue; // uniform: no flagged event in the tile
        const uint32_t word = fw[tile * TB + threadIdx.x];
        uint32_t flags = word & 0xFFFFu, o = word >> 16;
        const uint32_t my0 = (uint32_t)(tile * TE) + threadIdx.x * FLAG_EVENTS;
        while (flags) {
            const uint32_t b = __builtin_ctz(flags);
            flags &= flags - 1;
            if (o < TE)
                s_idx[o] = my0 + b;
            o++;
        }
        __syncthreads();
        const uint32_t cnt = total < (uint64_t)TE ? (uint32_t)total : TE;
        for (uint32_t i = threadIdx.x; i < cnt; i += TB)
            viol[o0 + i] = s_idx[i];
        __syncthreads();
    }
}

template <int TB>
void flag_list(const FlagList &F, uint32_t *viol, Control *ctl, uint32_t *ticket, hipStream_t s)
{
    auto *const n_viol = &ctl->n_viol;
    if (F.tiles <= SUM_TILES) {
        ProfScope prof_(s, "flag_scatter");
        k_flag_scatter<TB, true><<<(unsigned)F.tiles, TB, 0, s>>>(F.fw, nullptr, F.tcnt, F.tiles, viol, n_viol);
        return;
    }
    launch_excl_scan(F.tcnt, F.tiles, F.offs, reinterpret_cast<uint64_t *>(n_viol), F.xscan, ticket, s, true);
    ProfScope prof_(s, "flag_scatter");
    const unsigned grid = (unsigned)(F.tiles < 8192 ? F.tiles : 8192);
    k_flag_scatter<TB, false><<<grid, TB, 0, s>>>(F.fw, F.offs, F.tcnt, F.tiles, viol, nullptr);
}

} // namespace

void launch_flag_list(const FlagList &F, int tb, uint32_t *viol, Control *ctl, uint32_t *ticket, hipStream_t s)
{
    if (!F.tiles)
        return;
    if (tb == 512)
        flag_list<512>(F, viol, ctl, ticket, s);
    else
        flag_list<256>(F, viol, ctl, ticket, s);
}

// (the most a trace of n events or fewer takes: a shorter one by single parts)
size_t compact_scratch_bytes(uint64_t n)
{
    const uint64_t part = n < C_LONG_FROM ? n : C_LONG_FROM;
    const uint64_t a = ceil_div(n ? n : 1, (uint64_t)parts_of(n) * CPART), b = ceil_div(part ? part : 1, (uint64_t)CPART);
    return (a > b ? a : b) * sizeof(uint64_t);
}

void launch_compact(const uint8_t *status, uint64_t n, uint32_t *viol, void *scratch, Control *ctl, hipStream_t s,
                    const unsigned long long *flagged, const unsigned long long *n_dev, bool lookback_cleared)
{
    if (n == 0)
        return;
    const bool is_long = parts_of(n) == C_LONG;
    const uint64_t tiles = ceil_div(n, (uint64_t)parts_of(n) * CPART);
    uint64_t *lb = reinterpret_cast<uint64_t *>(scratch);
    if (!lookback_cleared)
        launch_clear_lookback(lb, tiles, ctl->tickets[2], s);
    const auto kernel = is_long ? k_compact<C_LONG> : k_compact<1>;
    ProfScope prof_(s, "compact");
    kernel<<<resident_grid((const void *)kernel, tiles), BLOCK, 0, s>>>(status, n, viol, lb, ctl->tickets[2], tiles, ctl,
                                                                       flagged, n_dev);
}

} // namespace vc
