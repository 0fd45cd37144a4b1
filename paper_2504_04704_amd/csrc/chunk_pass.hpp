// Chunk-at-a-time LagKV kernel for gfx950: the one-shot pass for calls that do not fill the chip with
// long walks (few or short streams), and for rows that are not whole 16-byte slices.  The ring kernel (ring_pass.hpp) has
// taken most of these; left are Eq. 16, rows of partial slices of which a lane holds 9 to 32, and short calls by Eq. 14-15 of
// chunks that it would go over twice.
//
// What bounds such a call is latency: one launch, a chain of dependent memory reads, the selection.  So a
// workgroup of eight wavefronts (four on K rows, four on V rows) takes ONE chunk, or a short run of them
// when there are more chunks than places, and asks for everything it will need at once: the rows of the
// reference chunk (Eq. 7-8) and the rows of its own chunk are in flight together, the chunk stays in
// registers until the selection is known, and the kept rows are stored from there.  A neighbour reads
// the reference rows as its own chunk at about the same time, so their second read is served by a cache.
// The walking kernels, which read every row once and keep a stream of loads in flight, take over where
// memory bandwidth is the limit (the rule and the figures stand at the choice, in lagkv_api.hip).
#pragma once
#include "chunk_ops.hpp"

namespace lagkv {

// NSL: 16-byte row slices a lane holds: chunks of up to NSL * R rows, R = 4 * 64 / LPR per step.  All NSL are asked for
// in one go (behind a branch of its own every load would wait for the one before it), those past the chunk's end of one
// row.  So chunks of one or two steps have a kernel of their own: with the six or seven loads too many of the next larger one,
// 216 streams of 52 chunks of 64 rows of 36 bytes, scores by Eq. 16, took 53.9 us and not 45.9, calls of up to 1024
// such chunks 3 % longer.
// PART: rows shorter than LPR slices.
template <typename ET, int LPR, int NSL, bool PART>
__global__ void __launch_bounds__(512, NSL <= 8 ? 4 : 2) chunk_pass_kernel(const PassArgs a) {
  using Lane = ChunkLane<ET, LPR, NSL, PART>;
  constexpr int R = Lane::R;
  constexpr int UR = NSL < 8 ? NSL : 8;  // reference rows in flight per lane beside the chunk's
  extern __shared__ float4 lds_raw[];
  char* lds = reinterpret_cast<char*>(lds_raw);
  Lane g;
  g.init(a.D, a.L, a.ddof);
  const int tid = g.tid, row0 = g.row0, rowbytes = g.rowbytes, coff = g.coff, tensor = g.tensor;
  const int D = a.D, L = a.L, k = a.k, S = a.S;
  const ChunkLds lay = chunk_lds(D, L);
  float* vK = reinterpret_cast<float*>(lds + lay.off_vK);
  float* vV = reinterpret_cast<float*>(lds + lay.off_vV);
  int32_t* slotmap = reinterpret_cast<int32_t*>(lds + lay.off_slot);
  uint32_t* rank = reinterpret_cast<uint32_t*>(lds + lay.off_rank);
  uint32_t* selbuf = reinterpret_cast<uint32_t*>(lds + lay.off_sel);
  float* statbuf = reinterpret_cast<float*>(lds + lay.off_stat);
  float* refbuf = reinterpret_cast<float*>(lds + lay.off_ref);

  const int n_iter = g.steps();

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
  const bool l2 = a.variant == 2, local = a.variant == 1;

  if (edge) {
    copy_edge_rows<LPR, true>(kin, vin, a.st, kout, vout, iout, rowbytes, S, S + a.n_s * L, S + a.n_s * k,
                              a.T - (S + a.n_s * L), (int)((blockIdx.x - n_score) % a.edge), a.edge, coff, tid,
                              kChunkWaves * kWave);
    return;
  }

  const int64_t p0 = (int64_t)seg * a.n_s / a.nseg;
  const int64_t p1 = (int64_t)(seg + 1) * a.n_s / a.nseg;
  const uint32_t st = (uint32_t)a.st;
  // 16 bytes of row `r` of the chunk at `base`; rows past the end repeat its last row
  auto load = [&](const char* base, int r) __attribute__((always_inline)) {
    const uint32_t off = (uint32_t)(r < L ? r : L - 1) * st + (uint32_t)coff;
    return Lane::ld(base + off);
  };

  uint4 hold[NSL];
  const char* cb = tin + (S + (p1 - 1) * L) * a.st;  // first row of the chunk
  // 0. everything the first chunk needs is asked for at once
  if (tid >= L && tid < chunk_pad(L)) slotmap[tid] = -1;  // rows past the end are never stored
  {
    const int row = here_v(row0), n = here_s(n_iter);
    if (!l2 && !local) {
      const char* rb = cb + (int64_t)L * a.st;
      g.acc.reset();
#pragma unroll
      for (int j0 = 0; j0 < NSL; j0 += UR) {
        if (j0 < n) {  // (a batch in one go: behind a branch of its own every load would wait for the one before it)
          uint4 q[UR];
#pragma unroll
          for (int u = 0; u < UR; ++u) q[u] = load(rb, row + (j0 + u) * R);
#pragma unroll
          for (int u = 0; u < UR; ++u) hold[j0 + u] = load(cb, row + (j0 + u) * R);
#pragma unroll
          for (int u = 0; u < UR; u += 2)
            if (j0 + u < n) g.fold_pair(q[u], q[u + 1]);
        }
      }
      g.park(statbuf);
      lds_barrier();
      g.publish(statbuf, refbuf);
      lds_barrier();
      g.take_ref(refbuf);
    } else {
#pragma unroll
      for (int j = 0; j < NSL; ++j) hold[j] = load(cb, row + j * R);
    }
  }

  for (int64_t p = p1 - 1; p >= p0; --p) {
    const bool more = p > p0;
    if (tid < L) rank[tid] = 0;
    if (local) {
      g.acc.reset();
      const int n = here_s(n_iter);
#pragma unroll
      for (int j = 0; j < NSL; j += 2)
        if (j < n) {
          g.fold_pair(hold[j], hold[j + 1]);
          __builtin_amdgcn_sched_barrier(0);
        }
      g.park(statbuf);
      lds_barrier();
      g.publish(statbuf, refbuf);
      lds_barrier();
      g.take_ref(refbuf);
    }
    // 1. channel variance of every row (Eq. 9-10), or minus the key norm (Eq. 16); the running
    // min/max of the chunk when it is the next one's reference
    const bool stats = !l2 && !local && more;
    if (stats) g.acc.reset();
    g.variances(hold, here_s(n_iter), myvar + here_v(row0), l2, stats);
    if (stats) g.park(statbuf);
    if (L > kRankSelMax) group_sel_clear(selbuf, tid, kChunkWaves * kWave);
    lds_barrier();
    if (stats) g.publish(statbuf, refbuf);
    // 2. chunk softmax, K+V sum and top-k (Eq. 10-11)
    float* gs = sout ? sout + p * L : nullptr;
    int32_t* gp = iout ? iout + S + p * k : nullptr;
    chunk_select(vK, vV, l2, L, k, gather, gs, rank, selbuf, slotmap, tid, gp, (uint32_t)(S + p * L));
    lds_barrier();
    // 3. kept rows out of the registers, the next chunk's rows in
    const char* nb = cb - (int64_t)L * a.st;
    {
      char* dst = tout + (S + p * k) * rowbytes;
      const int row = here_v(row0), n = here_s(n_iter);
#pragma unroll
      for (int j = 0; j < NSL; ++j) {
        if (gather && j < n) {
          const int sl = slotmap[row + j * R];
          if (sl >= 0) st16_out_at(dst, (uint32_t)sl * (uint32_t)rowbytes + (uint32_t)coff, hold[j]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (more) {
#pragma unroll
        for (int j = 0; j < NSL; ++j) hold[j] = load(nb, row + j * R);
      }
    }
    if (stats) g.take_ref(refbuf);
    cb = nb;
  }
}

// ------------------------------------------------------------------------ host side
template <typename ET>
hipError_t launch_chunk_t(const PassArgs& a, hipStream_t s) {
  constexpr int ESIZE = 16 / ET::VEC;
  const int rowbytes = a.D * ESIZE, lpr = chunk_lpr(rowbytes);
  const bool part = rowbytes != lpr * 16;
  const int R = chunk_step(lpr), steps = (a.L + R - 1) / R;
  const int nsl = steps <= 2 ? 2 : steps <= 8 ? 8 : steps <= 16 ? 16 : 32;
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
    LAGKV_CHUNK_CASE(4, 2)
    LAGKV_CHUNK_CASE(4, 8)
    LAGKV_CHUNK_CASE(8, 2)
    LAGKV_CHUNK_CASE(8, 8)
    LAGKV_CHUNK_CASE(8, 16)
    LAGKV_CHUNK_CASE(16, 2)
    LAGKV_CHUNK_CASE(16, 8)
    LAGKV_CHUNK_CASE(16, 16)
    LAGKV_CHUNK_CASE(16, 32)
    LAGKV_CHUNK_CASE(32, 2)
    LAGKV_CHUNK_CASE(32, 8)
    LAGKV_CHUNK_CASE(32, 16)
    LAGKV_CHUNK_CASE(32, 32)
    default: return hipErrorInvalidValue;
  }
#undef LAGKV_CHUNK_CASE
  return hipGetLastError();
}

}  // namespace lagkv
