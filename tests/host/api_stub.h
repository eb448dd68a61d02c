// wv_api.cpp with launchers that do nothing, for the host tests; a test may put
// its own launch_encode (STUB_ENCODE) or variants and decode launchers
// (STUB_DECODE) in place.
#pragma once

#include "hip_stub.h"

#include "wv_api.cpp"

#include <cstdio>

inline wv::Variant stub_block{"block", 64, 64, 256, false, 0, true, 0, -1, 0, -1, -1};

inline int check(bool ok, const char* what) {
  if (!ok) std::printf("FAILED: %s\n", what);
  return ok ? 0 : 1;
}

namespace wv {
#ifndef STUB_DECODE
int fused_variant_count(int, int) { return 1; }
const Variant* fused_variant(int, int, int v) { return v == 0 ? &stub_block : nullptr; }
int default_variant(const wv_desc&) { return 0; }
int alternative_variant(const wv_desc&) { return -1; }
hipError_t launch_fused(int, int, int, const WorkArgs&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_strip53_set(int, int, int, const WorkArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_strip97_set(int, int, int, const WorkArgs&, hipStream_t) { return hipSuccess; }
#endif
hipError_t launch_plain(int, int, const PlainArgs&, hipStream_t) { return hipSuccess; }
size_t encode_workspace_bytes(int, int, int, int, int) { return 64; }
#ifndef STUB_ENCODE
hipError_t launch_encode(int, int, int, int, int, int, const void* const*, void* const*, void*, int*, hipStream_t) {
  return hipSuccess;
}
#endif
}  // namespace wv
