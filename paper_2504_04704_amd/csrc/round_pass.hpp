// One compression round of a decode cache (gfx950), in place, one workgroup per stream: the call in which
// the appended rows complete exactly one more chunk, for up to one stream per CU at any shape that the chunk
// kernels take, for rows that are not whole 16-byte slices at any stream count, and above that for chunks of
// up to 8 row slices a lane and some of up to 16 (the rule and the figures stand at round_is_faster, lagkv_api.hip).
//
// Such calls come a lag at a time while a prompt is prefilled, on few streams: a stream's chain of
// dependent steps is what bounds them, not bandwidth.  As in chunk_pass.hpp everything is asked for at
// once - the chunk's rows and the reference's - and stays in registers until it is stored at its final
// place, so that the chain is one memory latency, the scoring, the selection and the stores.  Measured on
// 32 streams, lag 256, rows of 256 bytes: 17.4 us a call against 31.8 us with the general kernel, which appends
// first and then scans, gathers and slides through memory.
//
// The tail is addressed virtually, as in decode_step_kernel: row v is in the cache when v < n_tail, else it
// is a new row.  Rows [0, L) are scored and the kept ones go to [0, k); the reference rows [L, 2L) go to
// [k, k + L) and what lies behind them to [k + L, ..).  Every store's place is among or below rows that
// every wavefront has loaded before the barrier in front of it.  (Storing the reference rows before the
// selection, which their places do not depend on, is 10 % slower at 512 to 2048 streams.)
#pragma once
#include "chunk_ops.hpp"

namespace lagkv {

// chunk_lds and the positions of the (fewer than 3L) tail rows
__host__ __device__ inline int round_lds_bytes(int D, int L) { return chunk_lds(D, L).total + 3 * L * 4; }

template <typename ET, int LPR, int NSL, bool PART>
__global__ void __launch_bounds__(512, 2) append_round_kernel(const AppendArgs a) {
  using Lane = ChunkLane<ET, LPR, NSL, PART>;
  constexpr int R = Lane::R;
  constexpr bool KEEP = NSL <= 16;       // the reference rows stay in registers too; else they are read again
  constexpr int UR = 8;
  extern __shared__ float4 lds_raw[];
  char* lds = reinterpret_cast<char*>(lds_raw);
  Lane g;
  g.init(a.D, a.L, a.ddof);
  const int tid = g.tid, row0 = g.row0, rowbytes = g.rowbytes, coff = g.coff;
  const int L = a.L, k = a.k, nthreads = kChunkWaves * kWave;
  const ChunkLds lay = chunk_lds(a.D, L);
  float* vK = reinterpret_cast<float*>(lds + lay.off_vK);
  float* vV = reinterpret_cast<float*>(lds + lay.off_vV);
  int32_t* slotmap = reinterpret_cast<int32_t*>(lds + lay.off_slot);
  uint32_t* rank = reinterpret_cast<uint32_t*>(lds + lay.off_rank);
  uint32_t* selbuf = reinterpret_cast<uint32_t*>(lds + lay.off_sel);
  float* statbuf = reinterpret_cast<float*>(lds + lay.off_stat);
  float* refbuf = reinterpret_cast<float*>(lds + lay.off_ref);
  int32_t* ptail = reinterpret_cast<int32_t*>(lds + lay.total);
  const bool l2 = a.variant == 2, local = a.variant == 1;
  const int n_iter = g.steps();

  const int64_t stream = blockIdx.x;
  const int64_t b = stream / a.H, h = stream % a.H;
  const int n_sink = a.n_sink, n_tail = (int)a.n_tail, n_all = (int)(a.n_tail + a.n_new) - n_sink;
  // tail row 0 of this wavefront's tensor, and the new rows behind the ones that complete the sink
  char* ct = (g.tensor ? a.V : a.K) + (stream * a.capacity + a.n_static) * rowbytes;
  const char* fresh = a.n_new > 0 ? (g.tensor ? a.V_new : a.K_new) + b * a.nsb + h * a.nsh + n_sink * a.nst : ct;
  auto src = [&](int v) __attribute__((always_inline)) {
    return (v < n_tail ? ct + (int64_t)v * rowbytes : fresh + (int64_t)(v - n_tail) * a.nst) + coff;
  };
  // row `r` of the `n` tail rows from `v0` on; rows past the end repeat the last one
  auto load = [&](int v0, int r, int n) __attribute__((always_inline)) {
    return Lane::ld(src(v0 + (r < n ? r : n - 1)));
  };
  auto store = [&](int to, const uint4& q) __attribute__((always_inline)) {
    st16_out_at(ct, (uint32_t)to * (uint32_t)rowbytes + (uint32_t)coff, q);
  };
  int32_t* pc = a.pos ? a.pos + stream * a.capacity + a.n_static : nullptr;

  // 0. everything is asked for at once; where the reference rows are kept, they come first
  uint4 hold[NSL], rq[KEEP ? NSL : 1];
  {
    const int row = here_v(row0), n = here_s(n_iter);
    if constexpr (KEEP) {
#pragma unroll
      for (int j = 0; j < NSL; ++j)
        if (j < n) {
          rq[j] = load(L, row + j * R, L);
          __builtin_amdgcn_sched_barrier(0);  // (one address at a time)
        }
    }
#pragma unroll
    for (int j = 0; j < NSL; ++j)
      if (j < n) {
        hold[j] = load(0, row + j * R, L);
        __builtin_amdgcn_sched_barrier(0);
      }
    if (tid < L) rank[tid] = 0;
    if (L > kRankSelMax) group_sel_clear(selbuf, tid, nthreads);
    if (tid >= L && tid < chunk_pad(L)) slotmap[tid] = -1;  // rows past the end are never stored
    if (pc)
      for (int v = tid; v < n_all; v += nthreads)
        ptail[v] = v < n_tail ? pc[v] : (int32_t)(a.n_seen + n_sink + (v - n_tail));
    // 1. statistics of the reference (Eq. 7-8), or of the chunk itself (Eq. 14-15)
    g.acc.reset();
    if (!l2 && !local) {
      if constexpr (KEEP) {
#pragma unroll
        for (int j = 0; j < NSL; j += 2)
          if (j < n) g.fold_pair(rq[j], rq[j + 1]);
      } else {
#pragma unroll
        for (int j0 = 0; j0 < NSL; j0 += UR) {
          uint4 q[UR];
#pragma unroll
          for (int u = 0; u < UR; ++u)
            if (j0 + u < n) {
              q[u] = load(L, row + (j0 + u) * R, L);
              __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
          for (int u = 0; u < UR; u += 2)
            if (j0 + u < n) g.fold_pair(q[u], q[u + 1]);
        }
      }
    } else if (local) {
#pragma unroll
      for (int j = 0; j < NSL; j += 2)
        if (j < n) g.fold_pair(hold[j], hold[j + 1]);
    }
  }
  if (!l2) {
    g.park(statbuf);
    lds_barrier();
    g.publish(statbuf, refbuf);
    lds_barrier();
    g.take_ref(refbuf);
  }
  // 2. variances, scores, selection (Eq. 9-11, Eq. 16)
  g.variances(hold, here_s(n_iter), (g.tensor ? vV : vK) + here_v(row0), l2, false);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // whatever was asked for above has been read
  lds_barrier();
  chunk_select(vK, vV, l2, L, k, true, nullptr, rank, selbuf, slotmap, tid, nullptr, 0);
  lds_barrier();
  // 3. kept rows -> [0, k)
  {
    const int row = here_v(row0), n = here_s(n_iter);
#pragma unroll
    for (int j = 0; j < NSL; ++j)
      if (j < n) {
        const int sl = slotmap[row + j * R];
        if (sl >= 0) store(sl, hold[j]);
      }
  }
  // 4. reference rows -> [k, k + L), over dead rows of the chunk and their own old places, and the rest of
  // the tail -> [k + L, ..); what was not kept is loaded by every wavefront before any of it is stored
  const int nrem = n_all - 2 * L;
  auto ask = [&](int from, int rows) __attribute__((always_inline)) {
    const int row = here_v(row0), n = here_s(n_iter);
#pragma unroll
    for (int j = 0; j < NSL; ++j)
      if (j < n) {
        hold[j] = load(from, row + j * R, rows);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  auto put = [&](int to, int rows) __attribute__((always_inline)) {
    const int row = here_v(row0), n = here_s(n_iter);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
#pragma unroll
    for (int j = 0; j < NSL; ++j)
      if (j < n && row + j * R < rows) store(to + row + j * R, hold[j]);
  };
  if constexpr (KEEP) {
    if (nrem > 0) ask(2 * L, nrem);  // (in flight while the reference rows leave)
    const int row = here_v(row0), n = here_s(n_iter);
#pragma unroll
    for (int j = 0; j < NSL; ++j)
      if (j < n && row + j * R < L) store(k + row + j * R, rq[j]);
  } else {
    ask(L, L);
    put(k, L);
    if (nrem > 0) ask(2 * L, nrem);
  }
  if (nrem > 0) put(k + L, nrem);
  if (pc) {
    for (int t = tid; t < L; t += nthreads) {
      const int sl = slotmap[t];
      if (sl >= 0) pc[sl] = ptail[t];
    }
    for (int i = tid; i < n_all - L; i += nthreads) pc[k + i] = ptail[L + i];
  }
  // the new rows that complete the sink: into places no tail row is in
  for (int r = row0; r < n_sink; r += R) {
    const uint4 q = Lane::ld(fresh + (int64_t)(r - n_sink) * a.nst + coff);
    st16_out(ct + (int64_t)(r - n_sink) * rowbytes + coff, q);
  }
  if (pc)
    for (int r = tid; r < n_sink; r += nthreads) pc[r - n_sink] = (int32_t)(a.n_seen + r);
}

template <typename ET>
hipError_t launch_round_t(const AppendArgs& a, hipStream_t s) {
  constexpr int ESIZE = 16 / ET::VEC;
  const int rowbytes = a.D * ESIZE, lpr = chunk_lpr(rowbytes);
  const bool part = rowbytes != lpr * 16;
  const int R = chunk_step(lpr), steps = (a.L + R - 1) / R;
  const int nsl = steps <= 8 ? 8 : steps <= 16 ? 16 : 32;
  const int64_t streams = (int64_t)a.B * a.H;
  if (steps > 32 || streams <= 0 || streams > 0x7fffffffLL) return hipErrorInvalidValue;
  const size_t lds = (size_t)round_lds_bytes(a.D, a.L);
  if (lds > (size_t)kMaxLdsBytes) return hipErrorInvalidValue;
  const dim3 grid((unsigned)streams), block(kChunkWaves * kWave);
#define LAGKV_ROUND_CASE(LPR, NSL)                                                            \
  case LPR * 64 + NSL:                                                                        \
    if (part) append_round_kernel<ET, LPR, NSL, true><<<grid, block, lds, s>>>(a);            \
    else append_round_kernel<ET, LPR, NSL, false><<<grid, block, lds, s>>>(a);                \
    break;
  switch (lpr * 64 + nsl) {
    LAGKV_ROUND_CASE(4, 8)
    LAGKV_ROUND_CASE(8, 8)
    LAGKV_ROUND_CASE(8, 16)
    LAGKV_ROUND_CASE(16, 8)
    LAGKV_ROUND_CASE(16, 16)
    LAGKV_ROUND_CASE(16, 32)
    LAGKV_ROUND_CASE(32, 8)
    LAGKV_ROUND_CASE(32, 16)
    LAGKV_ROUND_CASE(32, 32)
    default: return hipErrorInvalidValue;
  }
#undef LAGKV_ROUND_CASE
  return hipGetLastError();
}

}  // namespace lagkv
