// The packed linear at 2- and 3-bit codes.
#include "packed_linear.h"

namespace oq {
template hipError_t linear_bits<2>(const LinArgs&, int64_t, const uint16_t*, int64_t, void*);
template hipError_t linear_bits<3>(const LinArgs&, int64_t, const uint16_t*, int64_t, void*);
}  // namespace oq
