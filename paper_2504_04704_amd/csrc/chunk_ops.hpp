// What the kernels that take one chunk per workgroup share (chunk_pass.hpp, round_pass.hpp): rows as
// 16-byte slices on 4-byte addresses, statistics, variances and the selection.
//
// Rows: `D` channels of 4 or 2 bytes, 16 to 512 bytes in all and a multiple of 4, on 4-byte aligned
// addresses.  LPR lanes hold a row, 16 bytes each; a lane whose 16 bytes would reach past the end of the
// row takes the row's LAST 16 bytes instead.  The channels it shares with the lane before it (`dead`
// leading ones, all of them in a lane beyond the row) change no minimum or maximum, are stored twice with
// the same bytes, and are left out of the sums.
#pragma once
#include "lagkv_internal.hpp"
#include "lds_dma.hpp"
#include "row_ops.hpp"
#include "wave_ops.hpp"
#include "wg_select.hpp"

namespace lagkv {

constexpr int kChunkWaves = 8;
static_assert(kChunkWaves * kWave == kChunkThreads, "");

struct ChunkLds {
  int off_vK, off_vV, off_slot, off_rank, off_sel, off_stat, off_ref, total;  // bytes
};
// room for the rows of a whole pair of steps (at most 128)
__host__ __device__ inline int chunk_pad(int L) { return (L + 127) & ~127; }
__host__ __device__ inline ChunkLds chunk_lds(int D, int L) {
  ChunkLds l;
  const int lp = chunk_pad(L);
  l.off_vK = 0;
  l.off_vV = lp * 4;
  l.off_slot = 2 * lp * 4;                                    // int32 [L]: output slot within the chunk, or -1
  l.off_rank = 3 * lp * 4;                                    // uint32 [L]
  l.off_sel = 4 * lp * 4;
  l.off_stat = l.off_sel + ((group_sel_bytes() + 15) & ~15);  // float [wave][mn|mx][D]
  l.off_ref = l.off_stat + kChunkWaves * 2 * D * 4;           // float [K|V][mn|iv][D]
  l.total = l.off_ref + 4 * D * 4;
  return l;
}

// min(a, b) where lanes [0,32) receive the minimum of `a` over both halves of the wavefront and lanes
// [32,64) that of `b`; the same over the even and odd rows of 16 lanes.
__device__ __forceinline__ float fold_min32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float fold_min16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Folds the running statistics over the row groups of a wavefront and leaves them in w[0 .. D) (minima)
// and w[D .. 2D) (maxima); ch0 is the lane's first channel.  Scattered: after the exchange across 32
// lanes one half holds minima and the other negated maxima, after the exchange across 16 lanes each row
// holds half of the lane's channels.
template <int LPR, int VEC>
__device__ __forceinline__ void park_stats(const TStats<VEC>& acc, float* w, int D, int ch0, int lane) {
  const bool hi32 = (lane & 32) != 0, hi16 = (lane & 16) != 0;
  float v[VEC];
#pragma unroll
  for (int j = 0; j < VEC; ++j) v[j] = fold_min32(acc.mn[j], -acc.mx[j]);
  constexpr int N = LPR <= 16 ? VEC / 2 : VEC;
  float* dst = w + (hi32 ? D : 0) + ch0;
  if constexpr (LPR <= 16) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      v[j] = fold_min16(v[j], v[N + j]);
      if constexpr (LPR <= 8) v[j] = fminf(v[j], dpp_mov<0x128>(v[j]));   // row_ror:8
      if constexpr (LPR <= 4) v[j] = fminf(v[j], dpp_mov<0x124>(v[j]));   // row_ror:4
    }
    dst += hi16 ? N : 0;
  }
#pragma unroll
  for (int j = 0; j < N; ++j) dst[j] = hi32 ? -v[j] : v[j];
}

// Sum of squares of the lane's own channels (Eq. 16).
template <bool PART, int VEC>
__device__ __forceinline__ float sum_squares(const float (&x)[VEC], int dead) {
  if constexpr (PART) {
    float s[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      const float y = i < dead ? 0.f : x[i];
      s[i & 1] = fmaf(y, y, s[i & 1]);
    }
    return s[0] + s[1];
  } else {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < VEC; ++i) s = fmaf(x[i], x[i], s);
    return s;
  }
}

// What a lane of the chunk kernels holds and does: `NSL` slices of a chunk's rows, four wavefronts per
// tensor, R rows of a tensor per step.
template <typename ET, int LPR, int NSL, bool PART>
struct ChunkLane {
  static constexpr int VEC = ET::VEC, RPW = kWave / LPR, G = kChunkWaves / 2, R = G * RPW, ESIZE = 16 / VEC;
  int tid, lane, wave;
  int tensor;          // 0: this wavefront handles K rows, 1: V rows
  int row0, cl;        // the lane's row of a step, its slice of the row
  int rowbytes, coff;  // bytes of a dense row, byte its slice starts at
  int dead, ch0;       // leading channels that belong to the lane before it, first channel
  int D, L;
  float inv_D, inv_dof;
  TStats<VEC> acc;
  float mn[VEC], iv[VEC];

  __device__ __forceinline__ void init(int D_, int L_, int ddof) {
    tid = threadIdx.x;
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    tensor = wave >= G ? 1 : 0;
    cl = lane % LPR;
    row0 = (wave - tensor * G) * RPW + lane / LPR;
    D = D_;
    L = L_;
    rowbytes = PART ? D * ESIZE : LPR * 16;
    coff = PART && cl * 16 > rowbytes - 16 ? rowbytes - 16 : cl * 16;
    dead = PART ? ((cl * 16 - coff) / ESIZE < VEC ? (cl * 16 - coff) / ESIZE : VEC) : 0;
    ch0 = coff / ESIZE;
    inv_D = 1.0f / (float)D;
    inv_dof = 1.0f / (float)(D - ddof);
  }
  // steps of R rows, in pairs (a step past the end repeats the chunk's last row), at most NSL
  __device__ __forceinline__ int steps() const { return ((L + R - 1) / R + 1) & ~1; }
  // (whole rows may lie on 4-byte addresses too, by their stride or base: one instruction either way)
  static __device__ __forceinline__ uint4 ld(const char* p) { return ld16_a4(p); }

  __device__ __forceinline__ void fold_pair(const uint4& q0, const uint4& q1) {
    float x0[VEC], x1[VEC];
    unpack<ET>(q0, x0);
    unpack<ET>(q1, x1);
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      acc.mn[i] = fminf(fminf(acc.mn[i], x0[i]), x1[i]);
      acc.mx[i] = fmaxf(fmaxf(acc.mx[i], x0[i]), x1[i]);
    }
    pin(acc);
  }
  __device__ __forceinline__ void park(float* statbuf) { park_stats<LPR, VEC>(acc, statbuf + wave * 2 * D, D, ch0, lane); }
  // combine what the wavefronts parked: one thread per channel (2 * D <= 512), behind a barrier
  __device__ __forceinline__ void publish(const float* statbuf, float* refbuf) {
    if (tid < 2 * D) {
      const int tn = tid >= D ? 1 : 0, ch = tid - tn * D;
      float lo = INFINITY, hi = -INFINITY;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float* rd = statbuf + (tn * G + g) * 2 * D + ch;
        lo = fminf(lo, rd[0]);
        hi = fmaxf(hi, rd[D]);
      }
      refbuf[tn * 2 * D + ch] = lo;
      refbuf[(tn * 2 + 1) * D + ch] = inv_range(lo, hi);
    }
  }
  // the published statistics of the lane's channels, behind another barrier
  __device__ __forceinline__ void take_ref(const float* refbuf) {
    const float* rd = refbuf + tensor * 2 * D + ch0;
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      mn[i] = rd[i];
      iv[i] = PART && i < dead ? 0.f : rd[D + i];
    }
  }
  // out[r] (LDS, chunk_pad(L) floats): channel variance of the lane's rows (Eq. 9-10), or minus the key
  // norm (Eq. 16); with `stats` also the running min/max.  Rows past the end go into the padding.
  __device__ __forceinline__ void variances(const uint4 (&hold)[NSL], int n, float* out, bool l2, bool stats) {
#pragma unroll
    for (int j = 0; j < NSL; j += 2) {
      if (j < n) {
        float x0[VEC], x1[VEC];
        // (opaque copies: unpacked here and not kept alive across the loops)
        uint4 t0 = hold[j], t1 = hold[j + 1];
        asm volatile("" : "+v"(t0.x), "+v"(t0.y), "+v"(t0.z), "+v"(t0.w));
        asm volatile("" : "+v"(t1.x), "+v"(t1.y), "+v"(t1.z), "+v"(t1.w));
        unpack<ET>(t0, x0);
        unpack<ET>(t1, x1);
        float v0, v1;
        if (l2) {
          v0 = -sqrtf(group_sum<LPR>(sum_squares<PART>(x0, dead)));
          v1 = -sqrtf(group_sum<LPR>(sum_squares<PART>(x1, dead)));
        } else {
          v0 = token_var_sub<LPR, VEC, PART>(x0, mn, iv, inv_D, inv_dof, dead);
          v1 = token_var_sub<LPR, VEC, PART>(x1, mn, iv, inv_D, inv_dof, dead);
        }
        if (cl == 0) {
          out[j * R] = v0;
          out[(j + 1) * R] = v1;
        }
        if (stats) {
#pragma unroll
          for (int i = 0; i < VEC; ++i) {
            acc.mn[i] = fminf(fminf(acc.mn[i], x0[i]), x1[i]);
            acc.mx[i] = fmaxf(fmaxf(acc.mx[i], x0[i]), x1[i]);
          }
          pin(acc);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
};

// Opaque copies for one pass over the slices: what is worked out from them (row offsets, step counts)
// is not moved out of a loop over chunks, where it would hold registers across everything.
__device__ __forceinline__ int here_v(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ int here_s(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

// Chunk softmax, K+V sum and top-k (Eq. 10-11; Eq. 16 with `l2`) from the variances in vK / vV; the slot
// map is complete behind the caller's next barrier.  `rank` is zero for tokens < L and `selbuf` (when
// L > kRankSelMax) cleared, both visible.
__device__ __forceinline__ void chunk_select(float* vK, float* vV, bool l2, int L, int k, bool do_select,
                                             float* gs, uint32_t* rank, uint32_t* selbuf, int32_t* slotmap,
                                             int tid, int32_t* gp, uint32_t pos0) {
  const int tn = here_v(tid), ln = tn & 63, wv = __builtin_amdgcn_readfirstlane(tn >> 6);
  const int Ls = here_s(L), ks = here_s(k);
  if (Ls <= 64) group_rank_select<1>(vK, vV, l2, Ls, ks, do_select, gs, rank, slotmap, ln, wv, gp, pos0);
  else if (Ls <= 128) group_rank_select<2>(vK, vV, l2, Ls, ks, do_select, gs, rank, slotmap, ln, wv, gp, pos0);
  else if (Ls <= kRankSelMax) group_rank_select<4>(vK, vV, l2, Ls, ks, do_select, gs, rank, slotmap, ln, wv, gp, pos0);
  else if (l2) {
    if (gs && tn < Ls) st4_out_at(gs, (uint32_t)tn * 4u, __float_as_uint(vK[tn]));
    if (do_select)
      group_topk(tn < Ls ? ordered_key(vK[tn]) : 0u, Ls, ks, selbuf, nullptr, slotmap, tn, kChunkWaves, gp, pos0);
  } else {
    group_score_select<false, true>(vK, vV, Ls, ks, do_select, gs, selbuf, nullptr, slotmap, tn, kChunkWaves * kWave,
                                    gp, pos0);
  }
}

// ------------------------------------------------------------------------ host side
inline int chunk_lpr(int rowbytes) {
  const int units = (rowbytes + 15) / 16;
  return units <= 4 ? 4 : units <= 8 ? 8 : units <= 16 ? 16 : 32;
}
// rows a workgroup takes per step
inline int chunk_step(int lpr) { return (kChunkWaves / 2) * (kWave / lpr); }

}  // namespace lagkv
