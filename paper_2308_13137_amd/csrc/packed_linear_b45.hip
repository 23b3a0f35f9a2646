// The packed linear at 4- and 5-bit codes.
#include "packed_linear.h"

namespace oq {
template hipError_t linear_bits<4>(const LinArgs&, int64_t, const uint16_t*, int64_t, void*);
template hipError_t linear_bits<5>(const LinArgs&, int64_t, const uint16_t*, int64_t, void*);
}  // namespace oq
