// The single-round append kernel for fp32 (an element type a file, so that they compile side by side), the
// plain append, and what their callers ask about them.
#include "round_pass.hpp"

namespace lagkv {

// The call that completes no chunk: new rows behind the tail, one 16-byte slice per thread, K and V in
// grid.y.  At one row per stream a workgroup per stream had 32 of its 256 threads at work (3.0 us a call at
// 512 streams, 2.8 us this way; rows of partial slices took three launches).
template <bool A4>
__global__ void __launch_bounds__(256) append_rows_kernel(const AppendArgs a, uint32_t units, uint32_t total) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= total) return;
  const int rowbytes = a.D * a.esize;
  const uint32_t row = i / units, n_new = (uint32_t)a.n_new;  // over streams and new rows
  const int u = (int)(i - row * units);
  const uint32_t st = row / n_new, bb = st / (uint32_t)a.H;
  const int64_t stream = st, r = row - st * n_new, b = bb, h = st - bb * (uint32_t)a.H;
  const int coff = u * 16 < rowbytes - 16 ? u * 16 : rowbytes - 16;
  const char* src = (blockIdx.y ? a.V_new : a.K_new) + b * a.nsb + h * a.nsh + r * a.nst + coff;
  const int64_t to = stream * a.capacity + a.n_static + a.n_tail + r;
  char* dst = (blockIdx.y ? a.V : a.K) + to * rowbytes + coff;
  if constexpr (A4) st16_a4(dst, ld16_a4(src));
  else st16(dst, ld16(src));
  if (a.pos && blockIdx.y == 0 && u == 0) a.pos[to] = (int32_t)(a.n_seen + r);
}

static int64_t append_slices(const AppendArgs& a) {
  return (int64_t)a.B * a.H * a.n_new * (((int64_t)a.D * a.esize + 15) / 16);
}

bool append_rows_supported(const AppendArgs& a) {
  const int64_t rowbytes = (int64_t)a.D * a.esize;
  return a.rounds == 0 && rowbytes >= 16 && rowbytes % 4 == 0 && rowbytes <= 512 &&
         append_slices(a) < (1LL << 31);  // slice numbers are 32 bit
}

hipError_t launch_append_rows(const AppendArgs& a, hipStream_t s) {
  if (!append_rows_supported(a)) return hipErrorInvalidValue;
  const int rowbytes = a.D * a.esize, units = (rowbytes + 15) / 16;
  const int64_t total = append_slices(a), nb = (total + 255) / 256;
  if (total <= 0) return hipSuccess;
  const bool a4 = ((rowbytes | a.nsb | a.nsh | a.nst | (int64_t)(uintptr_t)a.K | (int64_t)(uintptr_t)a.V |
                    (int64_t)(uintptr_t)a.K_new | (int64_t)(uintptr_t)a.V_new) & 15) != 0;
  const dim3 grid((unsigned)nb, 2), block(256);
  if (a4) append_rows_kernel<true><<<grid, block, 0, s>>>(a, (uint32_t)units, (uint32_t)total);
  else append_rows_kernel<false><<<grid, block, 0, s>>>(a, (uint32_t)units, (uint32_t)total);
  return hipGetLastError();
}

bool append_round_supported(const AppendArgs& a) {
  if (a.rounds != 1 || !chunk_supported(a.D, a.esize, a.L, (int64_t)a.D * a.esize)) return false;
  // a sink that is still filling has no tail behind it
  if (a.n_seen < a.S && (a.n_tail != 0 || a.n_static != a.n_seen)) return false;
  return round_lds_bytes(a.D, a.L) <= kMaxLdsBytes && grid_fits((int64_t)a.B * a.H, kChunkThreads);
}

hipError_t launch_append_round(const AppendArgs& args, hipStream_t s) {
  AppendArgs a = args;
  if (!append_round_supported(a)) return hipErrorInvalidValue;
  a.n_sink = 0;
  if (a.n_seen < a.S) {  // (a round happens only behind a full sink)
    a.n_sink = (int32_t)(a.S - a.n_seen);
    a.n_static = a.S;
  }
  const int64_t tail = a.n_tail + a.n_new - a.n_sink;
  if (tail < 2 * (int64_t)a.L || tail >= 3 * (int64_t)a.L) return hipErrorInvalidValue;
  if (a.esize == 4) return launch_round_f32(a, s);
  return a.f16 ? launch_round_f16(a, s) : launch_round_bf16(a, s);
}

hipError_t launch_round_f32(const AppendArgs& a, hipStream_t s) { return launch_round_t<F32>(a, s); }

}  // namespace lagkv
