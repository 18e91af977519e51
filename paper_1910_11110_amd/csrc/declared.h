// declared.h -- host interface of the well-declaredness check's kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace vc {

// a program of components: declarations [comp_off[c], comp_off[c + 1]), body events
// [body_off[c], ...) with their element indices (idx, or none), the variables' intervals
// and overlap sets (or none)
struct WdProgram {
    const uint64_t *comp_off, *body_off;
    const uint32_t *decls, *body, *idx, *lo, *hi;
    const OverlapSets *sets;
    uint64_t n_comp, n_decl, n_body;
    uint32_t n_vars;
    bool extend;
};

// the number of coverage bits of every declaration (n_decl words); checks the declarations
void launch_wd_decls(const WdProgram &P, uint32_t *wlen, Control *ctl, hipStream_t s);

// tiles of consecutive components that are checked together
uint64_t wd_tiles(uint64_t n_comp);

// every component's verdict byte (out).  For the tiles that do not fit in LDS: their list
// (big, a word a tile), lengths and places of their declarations' bits (wlen, boff, one a
// declaration), the bits (nbits of them, in words; a tile's are rounded up to a word), and
// a verdict word a component.  ctl reset before.
void launch_wd_check(const WdProgram &P, uint32_t *big, uint32_t *wlen, uint64_t *boff, uint32_t *bits,
                     uint64_t nbits, uint32_t *verdict, uint8_t *out, Control *ctl, hipStream_t s);

} // namespace vc
