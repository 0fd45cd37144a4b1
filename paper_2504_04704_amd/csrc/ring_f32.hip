// The ring kernel for fp32 (an element type a file, so that they compile side by side), and what its callers ask
// about it.
#include "ring_pass.hpp"

namespace lagkv {

bool ring_supported(int D, int esize, int L, int64_t st) {
  if (row_units(D, esize) == 0 || ring_shape(D, esize, L).gw == 0) return false;
  return st * ((int64_t)L + 128) < (1LL << 32);  // lane offsets of whole pairs of steps are 32 bit
}

// Where the workgroup has a compute unit to itself, nothing runs beside its selection, and lanes without rows of
// their own - rows of fewer slices than lanes, steps past the end of the chunk - count.  Its gain over the streaming
// kernel there (60 to 700 MB, both variants) by the share of the lanes' slices that hold rows:
//   16 wavefronts, 2-byte elements   0.52 0.83, 0.62 0.87 to 1.00, 0.75 0.95 to 1.10, 0.76 0.79, 0.79 0.93,
//                                    0.85 1.07 to 1.36, 0.9 and more 1.04 to 1.35; fp32 1.12 to 1.46 from 0.62 on
//   32 slices, 2-byte elements       0.57 0.93, 0.62 1.01 to 1.20, 0.75 and more 1.02 to 1.36
//   32 slices, fp32                  0.62 0.94, 0.70 1.00, 0.95 and more 1.06 to 1.22
bool ring_pays(int D, int esize, int L) {
  const RingShape f = ring_shape(D, esize, L);
  if (f.gw < 8 && f.nsl == 8) return true;
  const int lpr = chunk_lpr(D * esize), R = f.gw * (kWave / lpr), steps = ((L + R - 1) / R + 1) & ~1;
  const int64_t filled = (int64_t)L * row_units(D, esize) * 100 / ((int64_t)steps * R * lpr);
  if (f.nsl == 8) return esize == 4 || filled >= 80;
  return filled >= (esize == 4 ? 70 : 62);
}

int ring_threads(int D, int esize, int L) { return ring_shape(D, esize, L).gw * 2 * kWave; }

int ring_places(int D, int esize, int L) {
  const RingShape f = ring_shape(D, esize, L);
  const int lds = kRingMaxLds / ring_lds(D, esize, L, f.nsl, f.gw).total, regs = (f.nsl == 8 ? 16 : 8) / (2 * f.gw);
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

hipError_t launch_ring_f32(const PassArgs& a, hipStream_t s) { return launch_ring_t<F32>(a, s); }

}  // namespace lagkv
