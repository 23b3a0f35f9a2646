// The packed linear at 6- and 7-bit codes.
#include "packed_linear.h"

namespace oq {
template hipError_t linear_bits<6>(const LinArgs&, int64_t, const uint16_t*, int64_t, void*);
template hipError_t linear_bits<7>(const LinArgs&, int64_t, const uint16_t*, int64_t, void*);
}  // namespace oq
