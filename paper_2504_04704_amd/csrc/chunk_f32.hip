// The chunk-at-a-time kernel for fp32 (an element type a file, so that they compile side by side), and
// what its callers ask about it.
#include "chunk_pass.hpp"

namespace lagkv {

bool chunk_supported(int D, int esize, int L, int64_t st) {
  const int64_t rowbytes = (int64_t)D * esize;
  if (rowbytes < 16 || rowbytes > 512 || rowbytes % 4 != 0 || L > 512) return false;
  if (chunk_slices(D, esize, L) > 32) return false;
  return st * (int64_t)L < (1LL << 31);  // lane offsets inside a chunk are 32 bit
}

int chunk_slices(int D, int esize, int L) {
  const int R = chunk_step(chunk_lpr(D * esize));
  return (L + R - 1) / R;
}

int chunk_places(int D, int esize, int L) { return chunk_slices(D, esize, L) <= 8 ? 2 : 1; }

hipError_t launch_chunk_pass(const PassArgs& args, hipStream_t s) {
  PassArgs a = args;
  if (!chunk_supported(a.D, a.esize, a.L, a.st) || a.nseg < 1 || a.nseg > a.n_s) return hipErrorInvalidValue;
  a.edge = edge_parts(a, 4 * kChunkWaves * (kWave / chunk_lpr(a.D * a.esize)));
  if (a.esize == 4) return launch_chunk_f32(a, s);
  return a.f16 ? launch_chunk_f16(a, s) : launch_chunk_bf16(a, s);
}

hipError_t launch_chunk_f32(const PassArgs& a, hipStream_t s) { return launch_chunk_t<F32>(a, s); }

}  // namespace lagkv
