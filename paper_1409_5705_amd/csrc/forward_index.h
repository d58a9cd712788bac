// Index arithmetic of the streaming bf16 forward (forward_bf16.hip).  Plain C++: the kernel and host programs use the
// same functions.
#pragma once
#include <stdint.h>

namespace sfb {

// First of the four fp32 columns of W that a lane loads for column group `part` (0 .. 15) of the k-slice that starts at
// column k0, in a row of D columns (D % 4 == 0, D >= 4).  Groups past the row load its last one (they count as zero): the
// load is unconditional, and behind the last row there may be no memory.
constexpr int64_t fwd_w_column(int64_t k0, int part, int64_t D)
{
    return k0 + 4 * part < D ? k0 + 4 * part : D - 4;
}

}  // namespace sfb
