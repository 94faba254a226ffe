// The streaming pass's segment arithmetic (csrc/segment.h) for a host test.
#include "../../paper_2312_08053_amd/csrc/segment.h"

using namespace kimad;

extern "C" {

// out: [0] the new limit, [1] whether the stretch goes on
void limit_after(uint32_t seg_end, uint32_t allowed, uint32_t taken, uint32_t most, uint32_t open, uint32_t* out) {
    const StretchLimit l = stretch_limit_after(seg_end, allowed, taken, most, open);
    out[0] = l.end; out[1] = l.on;
}

}  // extern "C"
