// Deployment of the calibrated weights (Sec. 4.5, Table "tab:speed"): the
// integer codes W_q of Eq.2 stored as low-bit strings, and the weight-only
// quantised linear Y = X W^T + B that reads them, with W = (W_q - z) * h per
// group (Eq.2's dequantisation) and 16-bit activations.
//
// Storage: each output row's codes form one little-endian bit string (code j
// at bits j*bits .. j*bits + bits - 1), rows back to back.  Because c_in is a
// multiple of 32, every run of 32 codes is exactly `bits` whole dwords: the
// unit a lane loads.
//
// The linear's kernels are in packed_linear.h, one code width per instantiation.
#include <algorithm>

#include "common.h"
#include "packed.h"

namespace oq {
namespace {

constexpr int PACK_THREADS = 256;

// ------------------------------------------------------------------ packing
// One thread per run of 32 codes: 32 input bytes -> BITS output dwords.  Only
// the low BITS bits of each code are stored.
template <int BITS>
__global__ __launch_bounds__(PACK_THREADS) void pack_codes_kernel(const uint8_t* __restrict__ codes,
                                                                  int64_t n_runs,
                                                                  uint32_t* __restrict__ out) {
  const int64_t stride = int64_t(gridDim.x) * PACK_THREADS;
  for (int64_t i = int64_t(blockIdx.x) * PACK_THREADS + threadIdx.x; i < n_runs; i += stride) {
    const uint4* src = reinterpret_cast<const uint4*>(codes + 32 * i);
    const uint4 a = src[0], b = src[1];
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t o[BITS];
#pragma unroll
    for (int k = 0; k < BITS; ++k) o[k] = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
      const uint32_t c = (w[j >> 2] >> (8 * (j & 3))) & ((1u << BITS) - 1);
      const int pos = j * BITS;
      o[pos >> 5] |= c << (pos & 31);
      if ((pos & 31) + BITS > 32) o[(pos >> 5) + 1] |= c >> (32 - (pos & 31));
    }
    uint32_t* dst = out + i * BITS;
#pragma unroll
    for (int k = 0; k < BITS; ++k) dst[k] = o[k];
  }
}

}  // namespace

hipError_t pack_codes(const uint8_t* codes, int64_t c_out, int64_t c_in, int bits, uint8_t* packed,
                      hipStream_t stream) {
  const int64_t n_runs = c_out * (c_in / 32);
  if (n_runs == 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n_runs + PACK_THREADS - 1) / PACK_THREADS, 4096);
  uint32_t* out = reinterpret_cast<uint32_t*>(packed);
  const dim3 g{unsigned(blocks)}, b{unsigned(PACK_THREADS)};
  switch (bits) {
    case 2: hipLaunchKernelGGL(pack_codes_kernel<2>, g, b, 0, stream, codes, n_runs, out); break;
    case 3: hipLaunchKernelGGL(pack_codes_kernel<3>, g, b, 0, stream, codes, n_runs, out); break;
    case 4: hipLaunchKernelGGL(pack_codes_kernel<4>, g, b, 0, stream, codes, n_runs, out); break;
    case 5: hipLaunchKernelGGL(pack_codes_kernel<5>, g, b, 0, stream, codes, n_runs, out); break;
    case 6: hipLaunchKernelGGL(pack_codes_kernel<6>, g, b, 0, stream, codes, n_runs, out); break;
    case 7: hipLaunchKernelGGL(pack_codes_kernel<7>, g, b, 0, stream, codes, n_runs, out); break;
    case 8: hipLaunchKernelGGL(pack_codes_kernel<8>, g, b, 0, stream, codes, n_runs, out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t packed_linear(const uint16_t* X, int64_t n_tok, int64_t c_in, const uint8_t* packed,
                         int bits, int64_t group, const float* h, const float* z,
                         const float* bias, int64_t c_out, void* Y, bool y_bf16,
                         hipStream_t stream) {
  if (n_tok == 0 || c_out == 0) return hipSuccess;
  const LinArgs a{c_in, reinterpret_cast<const uint32_t*>(packed), int(c_in / group),
                  uint32_t(((uint64_t(1) << 31) + uint64_t(group / 32) - 1) / uint64_t(group / 32)), h, z, bias, c_out,
                  y_bf16, stream};
  switch (bits) {
    case 2: return linear_bits<2>(a, group, X, n_tok, Y);
    case 3: return linear_bits<3>(a, group, X, n_tok, Y);
    case 4: return linear_bits<4>(a, group, X, n_tok, Y);
    case 5: return linear_bits<5>(a, group, X, n_tok, Y);
    case 6: return linear_bits<6>(a, group, X, n_tok, Y);
    case 7: return linear_bits<7>(a, group, X, n_tok, Y);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace oq
