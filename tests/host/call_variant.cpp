// Which variant a call runs in: until the caller chooses one, 5/3 calls on tiles of
// 512 take the 16-row or the 32-row strips by their number of tiles; a choice
// holds for every call.
#define STUB_DECODE
#include "api_stub.h"

namespace {

// 0: 32-row strips, 1: 16-row chain strips
wv::Variant strips[2] = {{"r32", 512, 32, 256, false, 0, false, 3, 0, 2, -1, -1},
                         {"r16", 512, 16, 256, false, 0, false, 3, 4, 2, -1, -1}};
int ran = -1;   // the variant of the last launch

hipError_t set_launch(int shape) {
  ran = shape == 4;
  return hipSuccess;
}

}  // namespace

namespace wv {
int fused_variant_count(int, int) { return 2; }
const Variant* fused_variant(int, int, int v) { return v >= 0 && v < 2 ? &strips[v] : nullptr; }
int default_variant(const wv_desc& d) { return d.format == WV_YUV420; }
int alternative_variant(const wv_desc& d) { return d.wavelet == WV_W53 ? d.format != WV_YUV420 : -1; }
hipError_t launch_fused(int, int, int v, const WorkArgs&, int, hipStream_t) {
  ran = v;
  return hipSuccess;
}
hipError_t launch_strip53_set(int, int shape, int, const WorkArgs&, hipStream_t) { return set_launch(shape); }
hipError_t launch_strip97_set(int, int shape, int, const WorkArgs&, hipStream_t) { return set_launch(shape); }
}  // namespace wv

namespace {

alignas(16) unsigned char buf[64];

struct Calls {
  wv_ctx* c = nullptr;
  std::vector<uint8_t> mask;
  std::vector<int32_t> stamp;
  explicit Calls(int wavelet, int format) {
    wv_desc d = {};
    d.width = 512 * 256;
    d.height = d.tile = 512;
    d.levels = 3;
    d.wavelet = wavelet;
    d.format = format;
    if (wv_create(&c, &d) != WV_OK) std::printf("FAILED: wv_create\n");
    mask.assign(256, 0);
    stamp.assign(256, -1);
  }
  ~Calls() { wv_destroy(c); }
  void visible(int n) {
    for (int i = 0; i < 256; ++i) mask[i] = i < n;
    ran = -1;
  }
  int gop(int n, int frames) {
    visible(n);
    std::vector<wv_frame> f(frames);
    for (int i = 0; i < frames; ++i) f[i] = wv_frame{{buf, buf, buf}, i, i == 0, 1, 0};
    wv_ref ref{{buf, buf, buf}, stamp.data()};
    if (wv_decode_gop(c, frames, f.data(), nullptr, mask.data(), &ref, nullptr, nullptr) != WV_OK)
      std::printf("FAILED: wv_decode_gop: %s\n", wv_last_error());
    return ran;
  }
  int frame(int n) {
    visible(n);
    wv_frame f{{buf, buf, buf}, 0, 1, 1, 0};
    wv_ref ref{{buf, buf, buf}, stamp.data()};
    if (wv_decode_viewport(c, &f, nullptr, mask.data(), &ref, nullptr, nullptr) != WV_OK)
      std::printf("FAILED: wv_decode_viewport: %s\n", wv_last_error());
    return ran;
  }
  int set(int n, int frames) {
    visible(n);
    wv_set st = {};
    st.planes[0] = st.planes[1] = st.planes[2] = buf;
    st.n = 4;
    for (int b = 0; b < 4; ++b) st.qstep[b] = 1;
    void* outs[4] = {buf, buf, buf, buf};
    if (wv_decode_set(c, &st, 0, frames, nullptr, mask.data(), outs, nullptr) != WV_OK)
      std::printf("FAILED: wv_decode_set: %s\n", wv_last_error());
    return ran;
  }
};

int expect(int got, int want, const char* call, int n) {
  if (got == want) return 0;
  std::printf("FAILED: %s of %d tiles ran in variant %d\n", call, n, got);
  return 1;
}

}  // namespace

int main() {
  int bad = 0;
  for (int n : {1, 24, 25, 32, 33, 40, 41, 48, 49, 80, 81, 96, 97, 128, 129, 144, 145, 256}) {
    const bool r32_gop = n > 40 && n <= 48, r32_set = (n - 1) % 48 >= 32;
    Calls y(WV_W53, WV_YUV420), g(WV_W53, WV_GRAY8), f(WV_W97, WV_YUV420);
    bad += expect(y.frame(n), 1, "a 5/3 YUV420 frame", n);
    bad += expect(y.gop(n, 8), !r32_gop, "a 5/3 YUV420 GOP", n);
    bad += expect(y.gop(n, 1), 1, "a 5/3 YUV420 GOP of one frame", n);
    for (int k : {1, 2, 4}) bad += expect(y.set(n, k), !r32_set, "a 5/3 YUV420 set", n);
    bad += expect(g.frame(n), n <= 24, "a 5/3 grey frame", n);
    bad += expect(g.gop(n, 8), n <= 24, "a 5/3 grey GOP", n);
    bad += expect(g.set(n, 4), 0, "a 5/3 grey set", n);
    bad += expect(f.gop(n, 8), 1, "a 9/7 GOP", n);
    bad += expect(f.set(n, 4), 1, "a 9/7 set", n);
    for (int v = 0; v < 2; ++v) {   // a chosen variant
      wv_set_variant(y.c, v);
      wv_set_variant(g.c, v);
      bad += expect(y.gop(n, 8), v, "a GOP in a chosen variant", n);
      bad += expect(y.set(n, 4), v, "a set in a chosen variant", n);
      bad += expect(g.frame(n), v, "a grey frame in a chosen variant", n);
    }
  }
  if (!bad) std::printf("ok\n");
  return bad;
}
