// Row-strip kernels for tiles of 256 and 128 (stored frames, 2 to 5 levels):
// the 16-row chain schedule, in grid form.  Each lane owns 4 (2) columns of a
// luma row instead of 8, so units are half (a quarter) as large and need fewer
// registers and less LDS.
// What bounds them: latency, the dependent levels of a strip (a frame of 30
// tiles of 256: 10.4 us for 5.9 MB; the 64 x 64 block kernel took 38).
#pragma once
#include "wv_strip.h"

namespace wv {
namespace strip {

template <class LF, int FMT, int P, int L>
static hipError_t launch_small_one(const WorkArgs& a, hipStream_t s) {
  // waves per SIMD to leave register room for
  constexpr int WPE = std::is_same<LF, Inv53>::value ? (P == 256 ? 6 : 8) : (P == 256 ? 4 : 5);
  if (a.total <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_strip<LF, FMT, P, L, 16, 4, false, WPE, 1, false>), dim3(a.total), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <class LF, int FMT, int P>
static hipError_t launch_small_levels(int L, const WorkArgs& a, hipStream_t s) {
  switch (L) {
    case 2: return launch_small_one<LF, FMT, P, 2>(a, s);
    case 3: return launch_small_one<LF, FMT, P, 3>(a, s);
    case 4: return launch_small_one<LF, FMT, P, 4>(a, s);
    case 5: return launch_small_one<LF, FMT, P, 5>(a, s);
  }
  return hipErrorInvalidValue;
}

template <class LF>
static hipError_t launch_small(int format, int tile, int L, const WorkArgs& a, hipStream_t s) {
  if (tile == 256)
    return format == WV_YUV420 ? launch_small_levels<LF, WV_YUV420, 256>(L, a, s)
                               : launch_small_levels<LF, WV_GRAY8, 256>(L, a, s);
  return format == WV_YUV420 ? launch_small_levels<LF, WV_YUV420, 128>(L, a, s)
                             : launch_small_levels<LF, WV_GRAY8, 128>(L, a, s);
}

}  // namespace strip
}  // namespace wv
