// The storage order of a tile's blocks as the rebuild kernel gets it (made by
// counting) against the encoder's (a stable sort by level).
#include "api_stub.h"

#include "wv_format.cpp"

namespace wv {
hipError_t launch_rebuild(int, const RebuildArgs&, hipStream_t) { return hipSuccess; }
}  // namespace wv

int main() {
  int bad = 0;
  for (int p = 8; p <= 512; p *= 2)
    for (int levels = 1; (p >> levels) >= 1; ++levels) {
      const auto want = storage_order(p, levels);
      uint16_t got[wv::kRebuildMaxBlocks];
      bad += check((int)want.size() <= wv::kRebuildMaxBlocks, "blocks per tile");
      storage_order_packed(p, levels, got);
      for (size_t j = 0; j < want.size(); ++j)
        if (got[j] != ((want[j].first << 8) | want[j].second)) {
          std::printf("FAILED: edge %d, %d levels, block %zu\n", p, levels, j);
          ++bad;
          break;
        }
    }
  // a frame's table: luma, then the order that both chroma planes share
  for (int tile = 16; tile <= 512; tile *= 2) {
    wv_ctx c = {};
    c.d.tile = tile;
    c.d.levels = 3;
    c.d.format = WV_YUV420;
    c.nplanes = 3;
    wv::RebuildArgs a;
    rebuild_geometry(&c, a);
    const auto chroma = storage_order(tile / 2, 3);
    bad += check(a.plane[1].order0 == a.plane[0].nb && a.plane[2].order0 == a.plane[0].nb &&
                     a.per_item == a.plane[0].nb + 2 * a.plane[1].nb && a.plane[1].nb == (int)chroma.size(),
                 "the parts of the table");
    for (size_t j = 0; j < chroma.size(); ++j)
      bad += check(a.order[a.plane[1].order0 + j] == ((chroma[j].first << 8) | chroma[j].second), "the chroma order");
  }
  if (!bad) std::printf("ok\n");
  return bad;
}
