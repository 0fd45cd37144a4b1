// Workspace of one lagkv_compress call that needs any: [scores][kept], as include/lagkv.h states it for callers that
// size it by hand.  Host code only: for the library and for the binding.
#pragma once
#include <cstddef>
#include <cstdint>

namespace lagkv {

constexpr size_t kWsAlign = 256;
inline size_t ws_align_up(size_t x) { return (x + kWsAlign - 1) / kWsAlign * kWsAlign; }

struct CompressWs {
  size_t off_scores, off_kept, total;
};
// need_scores: the caller gives no array for them
inline CompressWs compress_ws(int64_t streams, int64_t n_s, int64_t L, int64_t k, bool need_scores) {
  CompressWs w;
  w.off_scores = 0;
  w.off_kept = need_scores ? ws_align_up((size_t)streams * n_s * L * 4) : 0;
  w.total = w.off_kept + ws_align_up((size_t)streams * n_s * k * 4);
  return w;
}

}  // namespace lagkv
