// wv_encode_intra's host side against the counting runtime: what a call leaves
// behind when a launch fails, and calls of several threads on one context.
#define STUB_ENCODE
#include "api_stub.h"

#include <chrono>
#include <condition_variable>
#include <set>
#include <thread>

namespace {

std::atomic<int> queued{0};      // kernels enqueued and not yet waited for
bool fail_second = false;        // the launcher's second kernel cannot be launched

// Calls of several threads: every call waits in its stream synchronisation until
// `meet` of them are there.
std::mutex mu;
std::condition_variable cv;
int meet = 0, there = 0, overflow_stream = 0;
bool alone = false;              // somebody waited in vain
std::multiset<void*> workspaces; // of the calls between launch and synchronisation
bool shared_ws = false;

hipError_t meet_all(hipStream_t) {
  std::unique_lock<std::mutex> lock(mu);
  ++there;
  cv.notify_all();
  if (!cv.wait_for(lock, std::chrono::seconds(5), [] { return there >= meet; })) alone = true;
  return hipSuccess;
}

hipError_t drain(hipStream_t) {
  queued = 0;
  return hipSuccess;
}

}  // namespace

namespace wv {
hipError_t launch_encode(int, int, int, int, int, int, const void* const*, void* const*, void* ws,
                         int* flag, hipStream_t st) {
  if (meet) {
    std::lock_guard<std::mutex> lock(mu);
    shared_ws |= workspaces.count(ws) != 0;
    workspaces.insert(ws);
    if ((size_t)st == (size_t)overflow_stream) *flag = 1;
    return hipSuccess;
  }
  ++queued;
  if (fail_second) return hipErrorLaunchFailure;
  ++queued;
  return hipSuccess;
}
}  // namespace wv

int errors(wv_ctx* c) {
  int bad = 0;
  stub::stream_sync = drain;
  unsigned char src[16];
  short coef[16];
  const void* s[1] = {src};
  void* k[1] = {coef};
  bad += check(wv_encode_intra(c, s, k, 1, nullptr) == WV_OK && queued == 0, "a call waits for its kernels");
  // the kernels write the caller's planes and a workspace that the next call uses
  fail_second = true;
  bad += check(wv_encode_intra(c, s, k, 1, nullptr) == WV_EDEVICE, "a launch error is reported");
  bad += check(queued == 0, "a call whose second launch failed waits for its first kernel");
  return bad;
}

int threads(wv_ctx* c, int n) {
  int bad = 0;
  const int before = stub::live_device, before_host = stub::live_host;
  stub::stream_sync = meet_all;
  for (int round = 0; round < 2; ++round) {
    meet = n;
    there = 0;
    workspaces.clear();
    overflow_stream = 1 + round;
    std::vector<wv_status> st(n);
    std::vector<std::thread> t;
    for (int i = 0; i < n; ++i)
      t.emplace_back([&, i] {
        unsigned char src[16];
        short coef[16];
        const void* s[1] = {src};
        void* k[1] = {coef};
        st[i] = wv_encode_intra(c, s, k, 1, (hipStream_t)(size_t)(i + 1));
      });
    for (auto& x : t) x.join();
    for (int i = 0; i < n; ++i)
      bad += check(st[i] == (i == round ? WV_EINVAL : WV_OK), "the overflow belongs to the call that made it");
    const int kept = stub::live_device - before;
    bad += check(kept <= n && kept <= 4, "at most four workspaces are kept");
  }
  bad += check(stub::live_host == before_host, "no flag is left over");
  bad += check(!alone, "calls of several threads do not wait for each other");
  bad += check(!shared_ws, "every call has a workspace of its own");
  return bad;
}

int main(int argc, char** argv) {
  int bad = 0;
  wv_desc d = {};
  d.width = d.height = d.tile = 256;
  d.levels = 3;
  d.wavelet = WV_W53;
  d.format = WV_GRAY8;
  wv_ctx* c = nullptr;
  bad += check(wv_create(&c, &d) == WV_OK, "wv_create");
  bad += argc > 1 ? threads(c, std::atoi(argv[1])) : errors(c);
  wv_destroy(c);
  bad += check(stub::live_device == 0 && stub::live_host == 0, "everything is given back");
  if (!bad) std::printf("ok\n");
  return bad;
}
