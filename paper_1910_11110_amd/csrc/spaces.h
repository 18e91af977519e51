// spaces.h -- functions on the statuses of k memory spaces (sets of valid locations), shared
// by the sorted and the wide check.
#pragma once
#include "device.h"

namespace vc {
namespace {

constexpr uint32_t KF_CONST = 1u << 16;
constexpr uint32_t KF_ID = 0u;
constexpr uint32_t K_OP_R = 0, K_OP_W = 1, K_OP_COPY = 2;

// function of an event (op byte: op | a << 2 | b << 4)
__device__ __forceinline__ uint32_t kf_of(uint32_t ob)
{
    const uint32_t op = ob & 3u, a = (ob >> 2) & 3u, b = (ob >> 4) & 3u;
    if (op == K_OP_W)
        return KF_CONST | (1u << a);
    if (op == K_OP_COPY)
        return (1u << b) << (4u * a);
    return KF_ID;
}

// the locations a set reaches through a relation (the rows the set selects): each bit a
// of the set is spread to a mask of row a (bit a to bit 4a, times 15), and the selected
// rows are folded together
__device__ __forceinline__ uint32_t kf_reach(uint32_t rel, uint32_t s)
{
    const uint32_t t = (s | (s << 3) | (s << 6) | (s << 9)) & 0x1111u;
    uint32_t r = rel & (t * 15u);
    r |= r >> 8;
    r |= r >> 4;
    return r & 15u;
}

__device__ __forceinline__ uint32_t kf_apply(uint32_t f, uint32_t s)
{
    return (f & KF_CONST) ? (f & 15u) : (s | kf_reach(f & 0xFFFFu, s));
}

// g o f (f first).  For two relations, row a of the product is the union of the rows b
// of g that row a of f selects: column b of f (bits 4a + b, shifted to 4a) times row b
// of g places row b of g in every row a that selects it, without carries.
__device__ __forceinline__ uint32_t kf_compose(uint32_t g, uint32_t f)
{
    if (g & KF_CONST)
        return g;
    if (f & KF_CONST)
        return KF_CONST | kf_apply(g, f & 15u);
    uint32_t p = 0;
#pragma unroll
    for (uint32_t b = 0; b < 4; b++)
        p |= ((f >> b) & 0x1111u) * ((g >> (4u * b)) & 15u);
    return f | g | p;
}

// a malformed k-space word (what vc_trace_load_spaces refuses)
__device__ __forceinline__ bool k_malformed(uint32_t e, uint32_t n_ids, uint32_t k)
{
    const uint32_t op = (e >> 24) & 3u, a = (e >> 26) & 3u, b = (e >> 28) & 3u;
    return (e >> 30) != 0 || (e & 0xFFFFFFu) >= n_ids || a >= k || b >= k || (op != K_OP_COPY && b != 0) ||
           (op == 3 && a != 0);
}

// stuck: a read at a, or a copy from a, with location a invalid
__device__ __forceinline__ uint32_t k_stuck(uint32_t ob, uint32_t pre)
{
    const uint32_t op = ob & 3u, a = (ob >> 2) & 3u;
    return (op == K_OP_R || op == K_OP_COPY) ? (((pre >> a) & 1u) ^ 1u) : 0u;
}

} // namespace
} // namespace vc
