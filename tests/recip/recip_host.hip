// Host build of the division by a host-made reciprocal that the kernels take an item's
// chain with. Only the host pass is built (no device code runs).
#include <stdint.h>

#include "launch.h"

extern "C" uint32_t recip_div(uint32_t n, uint32_t d)
{
    return fastrack::div_recip(n, d, fastrack::div_recip_of(d));
}
