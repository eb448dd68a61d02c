// Row-strip fused decode kernels for the 5/3 wavelet, tiles of 256 and 128.
#include "wv_strip_small.h"

namespace wv {

hipError_t launch_strip53_small(int format, int tile, int L, const WorkArgs& a, hipStream_t s) {
  return strip::launch_small<Inv53>(format, tile, L, a, s);
}

}  // namespace wv
