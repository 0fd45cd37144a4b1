// Chunk-at-a-time LagKV kernel for gfx950: the one-shot pass for calls that do not fill the chip with
// long walks (few or short streams), and for rows that are not whole 16-byte slices.
//
// What bounds such a call is latency: one launch, a chain of dependent memory reads, the selection.  So a
// workgroup of eight wavefronts (four on K rows, four on V rows) takes ONE chunk, or a short run of them
// when there are more chunks than places, and asks for everything it will need at once: the rows of the
// reference chunk (Eq. 7-8) and the rows of its own chunk are in flight together, the chunk stays in
// registers until the selection is known, and the kept rows are stored from there.  A neighbour reads
// the reference rows as its own chunk at about the same time, so their second read is served by a cache.
// The walking kernels, which read every row once and keep a stream of loads in flight, take over where
// memory bandwidth is the limit (the rule and the figures stand at the choice, in lagkv_api.hip).
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

// Workgroup barrier for LDS traffic only (see hold_pass.hip): rows still in flight are not waited for.
__device__ __forceinline__ void lds_only_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

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

// NSL: 16-byte row slices a lane holds: chunks of up to NSL * R rows, R = 4 * 64 / LPR per step.
// PART: rows shorter than LPR slices.
template <typename ET, int LPR, int NSL, bool PART>
__global__ void __launch_bounds__(512, NSL <= 8 ? 4 : 2) chunk_pass_kernel(const PassArgs a) {
  constexpr int VEC = ET::VEC, RPW = kWave / LPR, G = kChunkWaves / 2, R = G * RPW;
  constexpr int ESIZE = 16 / VEC;
  constexpr int UR = NSL < 8 ? NSL : 8;  // reference rows in flight per lane beside the chunk's
  extern __shared__ float4 lds_raw[];
  char* lds = reinterpret_cast<char*>(lds_raw);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D, L = a.L, k = a.k, S = a.S;
  const ChunkLds lay = chunk_lds(D, L);
  float* vK = reinterpret_cast<float*>(lds + lay.off_vK);
  float* vV = reinterpret_cast<float*>(lds + lay.off_vV);
  int32_t* slotmap = reinterpret_cast<int32_t*>(lds + lay.off_slot);
  uint32_t* rank = reinterpret_cast<uint32_t*>(lds + lay.off_rank);
  uint32_t* selbuf = reinterpret_cast<uint32_t*>(lds + lay.off_sel);
  float* statbuf = reinterpret_cast<float*>(lds + lay.off_stat);
  float* refbuf = reinterpret_cast<float*>(lds + lay.off_ref);

  const int tensor = wave >= G ? 1 : 0;  // 0: this wavefront handles K rows, 1: V rows
  const int rl = lane / LPR, cl = lane % LPR;
  const int row0 = (wave - tensor * G) * RPW + rl;
  const int rowbytes = PART ? D * ESIZE : LPR * 16;
  const int coff = PART && cl * 16 > rowbytes - 16 ? rowbytes - 16 : cl * 16;
  const int dead = PART ? ((cl * 16 - coff) / ESIZE < VEC ? (cl * 16 - coff) / ESIZE : VEC) : 0;
  const int ch0 = coff / ESIZE;
  // steps of R rows, in pairs (a step past the end repeats the chunk's last row), at most NSL
  const int n_iter = ((L + R - 1) / R + 1) & ~1;

  const int64_t streams = (int64_t)a.B * a.H, n_score = streams * a.nseg;
  const bool edge = blockIdx.x >= n_score;
  const int64_t stream = edge ? (blockIdx.x - n_score) / a.edge : blockIdx.x / a.nseg;
  const int seg = blockIdx.x % a.nseg;
  const int64_t b = stream / a.H, h = stream % a.H;
  const char* kin = a.K + b * a.sb + h * a.sh;
  const char* vin = a.V + b * a.sb + h * a.sh;
  // (Eq. 16 scores read no values: there need not be any)
  const char* tin = tensor && (a.variant != 2 || a.K_out) ? vin : kin;
  const bool gather = a.K_out != nullptr;
  char* kout = gather ? a.K_out + stream * a.T_out * rowbytes : nullptr;
  char* vout = gather ? a.V_out + stream * a.T_out * rowbytes : nullptr;
  char* tout = tensor ? vout : kout;
  int32_t* iout = (gather && a.idx_out) ? a.idx_out + stream * a.T_out : nullptr;
  float* sout = a.scores ? a.scores + stream * a.n_s * L : nullptr;
  float* myvar = tensor ? vV : vK;
  const float inv_D = 1.0f / (float)D;
  const float inv_dof = 1.0f / (float)(D - a.ddof);
  const bool l2 = a.variant == 2, local = a.variant == 1;

  if (edge) {
    copy_edge_rows<LPR, PART>(kin, vin, a.st, kout, vout, iout, rowbytes, S, S + a.n_s * L, S + a.n_s * k,
                              a.T - (S + a.n_s * L), (int)((blockIdx.x - n_score) % a.edge), a.edge, coff, tid,
                              kChunkWaves * kWave);
    return;
  }

  const int64_t p0 = (int64_t)seg * a.n_s / a.nseg;
  const int64_t p1 = (int64_t)(seg + 1) * a.n_s / a.nseg;
  const uint32_t st = (uint32_t)a.st;
  // Opaque copies for one pass over the slices: what is worked out from them (row offsets, step counts)
  // is not moved out of the loop over the chunks, where it would hold registers across everything.
  auto here_v = [](int v) __attribute__((always_inline)) {
    asm volatile("" : "+v"(v));
    return v;
  };
  auto here_s = [](int v) __attribute__((always_inline)) {
    asm volatile("" : "+s"(v));
    return v;
  };
  // 16 bytes of row `r` of the chunk at `base`; rows past the end repeat its last row
  auto load = [&](const char* base, int r) __attribute__((always_inline)) {
    const uint32_t off = (uint32_t)(r < L ? r : L - 1) * st + (uint32_t)coff;
    return PART ? ld16_a4(base + off) : ld16(base + off);
  };

  uint4 hold[NSL];
  TStats<VEC> acc;
  float mn[VEC], iv[VEC], bias = 0.f;
  auto fold_pair = [&](const uint4& q0, const uint4& q1) __attribute__((always_inline)) {
    float x0[VEC], x1[VEC];
    unpack<ET>(q0, x0);
    unpack<ET>(q1, x1);
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      acc.mn[i] = fminf(fminf(acc.mn[i], x0[i]), x1[i]);
      acc.mx[i] = fmaxf(fmaxf(acc.mx[i], x0[i]), x1[i]);
    }
    pin(acc);
  };
  auto park = [&]() __attribute__((always_inline)) {
    park_stats<LPR, VEC>(acc, statbuf + wave * 2 * D, D, ch0, lane);
  };
  // combine what the wavefronts parked: one thread per channel (2 * D <= 512), behind a barrier
  auto publish = [&]() __attribute__((always_inline)) {
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
  };
  // the published statistics of the lane's channels, behind another barrier
  auto take_ref = [&]() __attribute__((always_inline)) {
    const float* rd = refbuf + tensor * 2 * D + ch0;
    bias = 0.f;
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      mn[i] = rd[i];
      iv[i] = PART && i < dead ? 0.f : rd[D + i];
      bias -= mn[i] * iv[i];
    }
  };

  const char* cb = tin + (S + (p1 - 1) * L) * a.st;  // first row of the chunk
  // 0. everything the first chunk needs is asked for at once
  if (tid >= L && tid < chunk_pad(L)) slotmap[tid] = -1;  // rows past the end are never stored
  {
    const int row = here_v(row0), n = here_s(n_iter);
    if (!l2 && !local) {
      const char* rb = cb + (int64_t)L * a.st;
      acc.reset();
#pragma unroll
      for (int j0 = 0; j0 < NSL; j0 += UR) {
        uint4 q[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u)
          if (j0 + u < n) q[u] = load(rb, row + (j0 + u) * R);
#pragma unroll
        for (int u = 0; u < UR; ++u)
          if (j0 + u < n) hold[j0 + u] = load(cb, row + (j0 + u) * R);
#pragma unroll
        for (int u = 0; u < UR; u += 2)
          if (j0 + u < n) fold_pair(q[u], q[u + 1]);
      }
      park();
      lds_only_barrier();
      publish();
      lds_only_barrier();
      take_ref();
    } else {
#pragma unroll
      for (int j = 0; j < NSL; ++j)
        if (j < n) hold[j] = load(cb, row + j * R);
    }
  }

  for (int64_t p = p1 - 1; p >= p0; --p) {
    const bool more = p > p0;
    if (tid < L) rank[tid] = 0;
    if (local) {
      acc.reset();
      const int n = here_s(n_iter);
#pragma unroll
      for (int j = 0; j < NSL; j += 2)
        if (j < n) {
          fold_pair(hold[j], hold[j + 1]);
          __builtin_amdgcn_sched_barrier(0);
        }
      park();
      lds_only_barrier();
      publish();
      lds_only_barrier();
      take_ref();
    }
    // 1. channel variance of every row (Eq. 9-10), or minus the key norm (Eq. 16); the running
    // min/max of the chunk when it is the next one's reference
    const bool stats = !l2 && !local && more;
    if (stats) acc.reset();
    {
      const int n = here_s(n_iter);
      float* out = myvar + here_v(row0);
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
          } else if constexpr (PART) {
            v0 = token_var_part<LPR, VEC>(x0, mn, iv, bias, inv_D, inv_dof, dead);
            v1 = token_var_part<LPR, VEC>(x1, mn, iv, bias, inv_D, inv_dof, dead);
          } else {
            v0 = token_var<LPR, VEC>(x0, mn, iv, bias, inv_D, inv_dof);
            v1 = token_var<LPR, VEC>(x1, mn, iv, bias, inv_D, inv_dof);
          }
          if (cl == 0) {  // (rows past the end: into the padding)
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
    if (stats) park();
    if (L > kRankSelMax) group_sel_clear(selbuf, tid, kChunkWaves * kWave);
    lds_only_barrier();
    if (stats) publish();
    // 2. chunk softmax, K+V sum and top-k (Eq. 10-11)
    float* gs = sout ? sout + p * L : nullptr;
    int32_t* gp = iout ? iout + S + p * k : nullptr;
    const uint32_t pos0 = (uint32_t)(S + p * L);
    {
      const int ln = here_v(lane), tn = here_v(tid), wv = here_s(wave), Ls = here_s(L), ks = here_s(k);
      if (Ls <= 64) group_rank_select<1>(vK, vV, l2, Ls, ks, gather, gs, rank, slotmap, ln, wv, gp, pos0);
      else if (Ls <= 128) group_rank_select<2>(vK, vV, l2, Ls, ks, gather, gs, rank, slotmap, ln, wv, gp, pos0);
      else if (Ls <= kRankSelMax) group_rank_select<4>(vK, vV, l2, Ls, ks, gather, gs, rank, slotmap, ln, wv, gp, pos0);
      else if (l2) {
        if (gs && tn < Ls) st4_out_at(gs, (uint32_t)tn * 4u, __float_as_uint(vK[tn]));
        if (gather)
          group_topk(tn < Ls ? ordered_key(vK[tn]) : 0u, Ls, ks, selbuf, nullptr, slotmap, tn, kChunkWaves, gp, pos0);
      } else {
        group_score_select<false, true>(vK, vV, Ls, ks, gather, gs, selbuf, nullptr, slotmap, tn, kChunkWaves * kWave, gp, pos0);
      }
    }
    lds_only_barrier();
    // 3. kept rows out of the registers, the next chunk's rows in
    const char* nb = cb - (int64_t)L * a.st;
    {
      char* dst = tout + (S + p * k) * rowbytes;
      const int row = here_v(row0), n = here_s(n_iter);
#pragma unroll
      for (int j = 0; j < NSL; ++j) {
        if (j < n) {
          if (gather) {
            const int sl = slotmap[row + j * R];
            if (sl >= 0) st16_out_at(dst, (uint32_t)sl * (uint32_t)rowbytes + (uint32_t)coff, hold[j]);
          }
          if (more) hold[j] = load(nb, row + j * R);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (stats) take_ref();
    cb = nb;
  }
}

// ------------------------------------------------------------------------ host side
inline int chunk_lpr(int rowbytes) {
  const int units = (rowbytes + 15) / 16;
  return units <= 4 ? 4 : units <= 8 ? 8 : units <= 16 ? 16 : 32;
}
// rows a workgroup takes per step
inline int chunk_step(int lpr) { return (kChunkWaves / 2) * (kWave / lpr); }

template <typename ET>
hipError_t launch_chunk_t(const PassArgs& a, hipStream_t s) {
  constexpr int ESIZE = 16 / ET::VEC;
  const int rowbytes = a.D * ESIZE, lpr = chunk_lpr(rowbytes);
  const bool part = rowbytes != lpr * 16;
  const int R = chunk_step(lpr), steps = (a.L + R - 1) / R;
  const int nsl = steps <= 8 ? 8 : steps <= 16 ? 16 : 32;
  const int64_t nblocks = (int64_t)a.B * a.H * (a.nseg + a.edge);
  if (steps > 32 || nblocks <= 0 || nblocks > 0x7fffffffLL) return hipErrorInvalidValue;
  const size_t lds = (size_t)chunk_lds(a.D, a.L).total;
  const dim3 grid((unsigned)nblocks), block(kChunkWaves * kWave);
#define LAGKV_CHUNK_CASE(LPR, NSL)                                                          \
  case LPR * 64 + NSL:                                                                      \
    if (part) chunk_pass_kernel<ET, LPR, NSL, true><<<grid, block, lds, s>>>(a);            \
    else chunk_pass_kernel<ET, LPR, NSL, false><<<grid, block, lds, s>>>(a);                \
    break;
  switch (lpr * 64 + nsl) {
    LAGKV_CHUNK_CASE(4, 8)
    LAGKV_CHUNK_CASE(8, 8)
    LAGKV_CHUNK_CASE(8, 16)
    LAGKV_CHUNK_CASE(16, 8)
    LAGKV_CHUNK_CASE(16, 16)
    LAGKV_CHUNK_CASE(16, 32)
    LAGKV_CHUNK_CASE(32, 8)
    LAGKV_CHUNK_CASE(32, 16)
    LAGKV_CHUNK_CASE(32, 32)
    default: return hipErrorInvalidValue;
  }
#undef LAGKV_CHUNK_CASE
  return hipGetLastError();
}

}  // namespace lagkv
