// wv_encode_intra's host side against the counting runtime: what a call leaves
// behind when a launch fails.
#include "hip_stub.h"

#include "wv_api.cpp"

#include <cstdio>

namespace {

wv::Variant block{"block", 64, 64, 256, false, 0, true, 0, -1, 0, -1, -1};
std::atomic<int> queued{0};      // kernels enqueued and not yet waited for
bool fail_second = false;        // the launcher's second kernel cannot be launched

hipError_t drain(hipStream_t) {
  queued = 0;
  return hipSuccess;
}

int check(bool ok, const char* what) {
  if (!ok) std::printf("FAILED: %s\n", what);
  return ok ? 0 : 1;
}

}  // namespace

namespace wv {
int fused_variant_count(int, int) { return 1; }
const Variant* fused_variant(int, int, int v) { return v == 0 ? &block : nullptr; }
int default_variant(const wv_desc&) { return 0; }
int few_tiles_variant(const wv_desc&) { return -1; }
hipError_t launch_fused(int, int, int, const WorkArgs&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_plain(int, int, const PlainArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_strip53_set(int, int, int, const WorkArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_strip97_set(int, int, int, const WorkArgs&, hipStream_t) { return hipSuccess; }
size_t encode_workspace_bytes(int, int, int, int, int) { return 64; }
hipError_t launch_encode(int, int, int, int, int, int, const void* const*, void* const*, void*, int*, hipStream_t) {
  ++queued;
  if (fail_second) return hipErrorLaunchFailure;
  ++queued;
  return hipSuccess;
}
}  // namespace wv

int main() {
  int bad = 0;
  stub::stream_sync = drain;
  wv_desc d = {};
  d.width = d.height = d.tile = 256;
  d.levels = 3;
  d.wavelet = WV_W53;
  d.format = WV_GRAY8;
  wv_ctx* c = nullptr;
  bad += check(wv_create(&c, &d) == WV_OK, "wv_create");
  unsigned char src[16];
  short coef[16];
  const void* s[1] = {src};
  void* k[1] = {coef};
  bad += check(wv_encode_intra(c, s, k, 1, nullptr) == WV_OK && queued == 0, "a call waits for its kernels");
  // the kernels write the caller's planes and a workspace that the next call uses
  fail_second = true;
  bad += check(wv_encode_intra(c, s, k, 1, nullptr) == WV_EDEVICE, "a launch error is reported");
  bad += check(queued == 0, "a call whose second launch failed waits for its first kernel");
  wv_destroy(c);
  bad += check(stub::live_device == 0 && stub::live_host == 0, "everything is given back");
  if (!bad) std::printf("ok\n");
  return bad;
}
