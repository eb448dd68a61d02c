// Device helpers shared by the fused, plain and encoder kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wv_internal.h"
#include "wv_lift.h"

namespace wv {

// ----------------------------------------------------------------- helpers
constexpr int kMaxTile = 512;
__device__ __forceinline__ int floor_even(int x) { return x & ~1; }
__device__ __forceinline__ int ceil_even(int x) { return (x + 1) & ~1; }

template <class LF>
struct CoefT;
template <>
struct CoefT<Inv53> { using T = int16_t; using R = uint8_t; };
template <>
struct CoefT<Inv97> { using T = float; using R = float; };

// q is an int16 index and step <= 65535: both fit the 24-bit multiplier.
__device__ __forceinline__ int deq(int16_t q, int step) { return __mul24((int)q, step); }
__device__ __forceinline__ float deq(float q, int) { return q; }

__device__ __forceinline__ int clip255(int v) { return min(max(v, 0), 255); }
__device__ __forceinline__ float clip255(float v) { return fminf(fmaxf(v, 0.0f), 255.0f); }

// YUV -> RGB, JFIF full range.  Integer: Q16 constants round(65536 k).
__device__ __forceinline__ void to_rgb(int y, int cb, int cr, int& r, int& g, int& b) {
  cb -= 128;
  cr -= 128;
  r = clip255(((y << 16) + 91881 * cr + 32768) >> 16);
  g = clip255(((y << 16) - 22554 * cb - 46802 * cr + 32768) >> 16);
  b = clip255(((y << 16) + 116130 * cb + 32768) >> 16);
}
__device__ __forceinline__ void to_rgb(float y, float cb, float cr, float& r, float& g,
                                       float& b) {
  cb -= 128.0f;
  cr -= 128.0f;
  r = clip255(y + 1.402f * cr);
  g = clip255(y - 0.344136f * cb - 0.714136f * cr);
  b = clip255(y + 1.772f * cb);
}

// Byte permutation (V_PERM_B32): byte i of the result is byte sel_i of the
// eight bytes {lo (0..3), hi (4..7)}; selector 0x0c gives 0x00, 0x0d 0xff.
__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_amdgcn_perm(hi, lo, sel);
}
// Byte packing of values already clipped to 0..255, as byte permutations.
// Packing with shifts and ORs let instruction selection fold a preceding
// shift and clamp of two values into V_ASHR_PK_U8_I32, which writes only the
// low half of its destination, while the code this toolchain generated after
// it ORed further bytes into the upper half as if it were zero: the
// register's stale bytes reached the output (clipped odd rows of the 5/3
// inverse, (a + b) >> 1 with no residual).  A permutation of whole registers
// offers no such pattern.
__device__ __forceinline__ uint32_t pack4(int a, int b, int c, int d) {
  const uint32_t ab = perm((uint32_t)b, (uint32_t)a, 0x0c0c0400u);   // a0 b0 0 0
  const uint32_t cd = perm((uint32_t)d, (uint32_t)c, 0x0c0c0400u);   // c0 d0 0 0
  return perm(cd, ab, 0x05040100u);                                   // a0 b0 c0 d0
}

// Level windows of a block, one dimension.  Level 1's computed window C_1
// is the block itself.  Level k needs the low-band samples
// [C_k.a/2 - S_LO, C_k.b/2 + S_HI) of level k+1's output; that range rounded
// out to even bounds is the layout window W_{k+1} (kept in LDS), and the part
// of it inside the level k+1 region [0, P >> k) is what level k+1 computes,
// C_{k+1}.  The rest of W_{k+1} lies outside the region and is filled by
// mirroring: the low band of a whole-sample-symmetric signal is itself
// symmetric about its first sample on the left and about the point between
// its last two samples on the right, which differs from the extension a
// coarser level's output would get on its own -- so those samples are
// copied, never computed.  The approximation band (level L+1) is stored:
// its whole window W_{L+1} is loaded with that mirroring.
template <class LF>
__device__ __forceinline__ void level_window(int k, int P, int L, int a1, int n1, int& ca, int& cb,
                                             int& wa, int& wb) {
  ca = a1;
  cb = a1 + n1;
  wa = ca;
  wb = cb;
  for (int j = 1; j < k; ++j) {
    wa = floor_even((ca >> 1) - LF::S_LO);
    wb = ceil_even((cb >> 1) + LF::S_HI);
    if (j + 1 <= L) {
      ca = max(wa, 0);
      cb = min(wb, P >> j);
    } else {
      ca = wa;
      cb = wb;
    }
  }
}

// Compile-time bound of every level's window length for a level-1 block of B.
template <class LF>
constexpr int win_max(int B) {
  int len = B, mx = B;
  for (int k = 0; k < 14; ++k) {
    int nxt = len / 2 + LF::S_LO + LF::S_HI + 2;
    nxt += nxt & 1;
    if (nxt > mx) mx = nxt;
    len = nxt;
  }
  return mx;
}

__device__ __forceinline__ int xcd_remap(int b, int g) {
  // Work groups are dealt to the XCDs round-robin; give each XCD a
  // contiguous range of work units so neighbouring blocks of one tile (which
  // share coefficient halos) meet in the same L2.
  return xcd_first(b % kXcds, g) + b / kXcds;
}

// Ordering of one wave's LDS writes before its own later reads (DS
// instructions of a wave execute in order; this only keeps the compiler from
// moving them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

}  // namespace wv
