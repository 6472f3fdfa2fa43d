// The fused encoder for at most 96 positions: blocks of 32, 64 or 96 tokens instead of
// 128, in a translation unit of its own (the 128-token kernel's code is generated as
// if it were the only instantiation).
//
// A block's time is its products' and, the fewer tokens share a weight fragment, the
// stream of the packed weights from L2 (3.4 MB a candidate at 2 layers and 1024
// hidden units).  us, 2 layers, 1024 hidden units, 4 heads, before (128-token block)
// and after:
//   24 candidates   T 20: 106 -> 62    60: 107 -> 76    90: 107 -> 93
//   500 candidates  T 20: 241 -> 140   40: 242 -> 174   70: 243 -> 214
// A deeper look-ahead (24 or 32 fragments in place of 16) gains nothing: T 20 64, 66.
#include "encoder_fused_device.h"

namespace tav2 {

hipError_t launch_encoder_fused_short(const fz::Args& a, int T, unsigned grid, hipStream_t st) {
  if (T <= 32)
    fz::encoder_fused_kernel<false, 1><<<grid, fz::NT, 0, st>>>(a);
  else if (T <= 64)
    fz::encoder_fused_kernel<false, 2><<<grid, fz::NT, 0, st>>>(a);
  else
    fz::encoder_fused_kernel<false, 3><<<grid, fz::NT, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace tav2
