// The ring kernel for fp32 (an element type a file, so that they compile side by side), and what its callers ask
// about it.
#include "ring_pass.hpp"

namespace lagkv {

bool ring_supported(int D, int esize, int L, int64_t st) {
  if (row_units(D, esize) == 0 || ring_shape(D, esize, L).gw == 0) return false;
  return st * ((int64_t)L + 128) < (1LL << 32);  // lane offsets of whole pairs of steps are 32 bit
}

bool ring_pays(int D, int esize, int L) {
  const RingShape f = ring_shape(D, esize, L);
  return f.nsl == 0 ? ring_stream_pays(D, esize, L) : ring_hold_pays(f, D, esize, L);
}

bool ring_holds(int D, int esize, int L) { return ring_shape(D, esize, L).nsl != 0; }

int ring_threads(int D, int esize, int L) { return ring_shape(D, esize, L).gw * 2 * kWave; }

int ring_steps(int D, int esize, int L, int waves) {
  const int rows = waves * (kWave / chunk_lpr(D * esize));
  return (L + rows - 1) / rows;
}

int ring_places(int D, int esize, int L) {
  const RingShape f = ring_shape(D, esize, L);
  const int lds = kRingMaxLds / ring_lds(D, esize, L, f.nsl, f.gw).total, regs = (f.nsl == 32 ? 8 : 16) / (2 * f.gw);
  return 256 * (lds < regs ? lds : regs);
}

hipError_t launch_ring_pass(const PassArgs& args, hipStream_t s) {
  PassArgs a = args;
  const int64_t chunks = (int64_t)a.B * a.H * a.n_s;
  if (!ring_supported(a.D, a.esize, a.L, a.st) || a.variant == 2) return hipErrorInvalidValue;
  if (a.walks < 1 || a.walks > chunks || chunks >= (1LL << 31)) return hipErrorInvalidValue;
  a.edge = edge_parts(a, 4 * 2 * ring_shape(a.D, a.esize, a.L).gw * (kWave / chunk_lpr(a.D * a.esize)));
  if (a.esize == 4) return launch_ring_f32(a, s);
  return a.f16 ? launch_ring_f16(a, s) : launch_ring_bf16(a, s);
}

bool direct_supported(int D, int esize, int L, int64_t st) {
  if (!chunk_supported(D, esize, L, st) || st * ((int64_t)L + 128) >= (1LL << 32)) return false;
  const int gw = direct_waves(D, esize, L);
  return gw != 0 && direct_lds(D, esize, L, gw) <= kRingMaxLds;
}

int direct_threads(int D, int esize, int L) { return direct_waves(D, esize, L) * 2 * kWave; }

int direct_places(int D, int esize, int L) {
  const int gw = direct_waves(D, esize, L), lds = kRingMaxLds / direct_lds(D, esize, L, gw), regs = 16 / (2 * gw);
  return 256 * (lds < regs ? lds : regs);
}

hipError_t launch_direct_pass(const PassArgs& args, hipStream_t s) {
  PassArgs a = args;
  const int64_t chunks = (int64_t)a.B * a.H * a.n_s;
  if (!direct_supported(a.D, a.esize, a.L, a.st) || a.variant == 2) return hipErrorInvalidValue;
  if (a.walks < 1 || a.walks > chunks || chunks >= (1LL << 31)) return hipErrorInvalidValue;
  a.edge = edge_parts(a, 4 * 2 * direct_waves(a.D, a.esize, a.L) * (kWave / chunk_lpr(a.D * a.esize)));
  if (a.esize == 4) return launch_direct_f32(a, s);
  return a.f16 ? launch_direct_f16(a, s) : launch_direct_bf16(a, s);
}

hipError_t launch_ring_f32(const PassArgs& a, hipStream_t s) { return launch_ring_t<F32>(a, s); }
hipError_t launch_direct_f32(const PassArgs& a, hipStream_t s) { return launch_direct_t<F32>(a, s); }

}  // namespace lagkv
