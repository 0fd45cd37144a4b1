// The one-shot pass with one chunk at a time in registers and the rows behind it on their way, for gfx950: rows of
// whole 16-byte slices, any lag whose chunk fits (ring_shape), Eq. 7-11 and Eq. 14-15.
//
// What bounds the pass is memory, as long as the loads never stop.  So every wavefront asks for rows through an LDS
// ring of its own (asynchronous global->LDS loads), always one chunk ahead: the slots that a pair of steps leaves are
// filled with the rows of the next chunk at once, across selections, stores and the borders between streams.  A chunk
// stays in registers until its selection is known and the kept rows are stored from there, so no row is read
// twice (the streaming kernel in split_pass.hip reads kept rows again, and so does this one where a chunk does not
// fit: its rows then pass through the ring only).  A compute unit holds 16 wavefronts of up to 128 registers each, as
// one workgroup or as many as eight: the smallest workgroup whose lanes hold a chunk in eight slices is taken, because
// the others then have the unit to themselves while one of them selects.  Longer chunks take eight wavefronts of 256
// registers, alone on their unit.
//
// The scored chunks of a call are cut into equal shares, one per place that the chip has, without regard to where a
// stream ends: with whole segments of streams 112 streams of 31 chunks left the longest workgroup 9 chunks to read
// where 6.8 was the mean.  What a share costs beyond its chunks is its first reference (Eq. 7-8), read once more than
// needed, and another wherever it goes over into the next stream.
//
// Issue slots come second (half of them are taken with 2-byte elements): the variance of a pair of rows shares its
// reductions, one wavefront selects while the others wait - all of them counting ranks took ten times the
// instructions - and the statistics are parked in the element type of the rows, which holds them exactly.
//
// Against the streaming kernel, 600 MB of K and V on 96 streams (lag | own chunk as reference, Eq. 14-15), us:
//   rows of 128 bytes (bf16), lag  64   277 -> 178 | 284 -> 176        lag 256   209 -> 176 | 230 -> 186
//   rows of 160 bytes (f16),  lag 100   254 -> 228 | 289 -> 260        rows of 192, lag 128   207 -> 178 | 233 -> 193
//   rows of 256 bytes (bf16), lag  64   199 -> 179 | 221 -> 174        lag 300   235 -> 190 | 250 -> 224
//   rows of 512 bytes (bf16), lag 128   208 -> 177 | 232 -> 207        lag 256   212 -> 189 | 233 -> 218
//   rows of 512 bytes (fp32), lag 128   217 -> 170 | 244 -> 174        lag 256   210 -> 178 | 232 -> 195
//   lag 1024, rows of 128 bytes (bf16)  223 -> 195 | 253 -> 228        of 512 bytes (bf16)  311 -> 248 | 309 -> 256
#pragma once
#include "chunk_ops.hpp"

namespace lagkv {

// Ring slots (1 KiB steps) per wavefront: a whole chunk, or half of one where a lane holds 32 slices; six or
// eight where it holds none (nsl = 0: chunks that do not fit).
__host__ __device__ constexpr int ring_slots(int nsl, int gw) { return nsl == 32 ? 16 : nsl == 0 && gw == 4 ? 6 : 8; }

struct RingLds {
  int off_vK, off_vV, off_slot, off_ref, off_stat, off_ring, total;  // bytes
};
// nsl: slices a lane holds; gw: wavefronts per tensor
__host__ __device__ inline RingLds ring_lds(int D, int esize, int L, int nsl, int gw) {
  RingLds l;
  const int lp = chunk_pad(L);
  l.off_vK = 0;
  l.off_vV = lp * 4;
  // int32 [L]: where the row goes, in bytes from the first kept row of its chunk, or -1; nsl = 0: [k]: the kept rows
  l.off_slot = 2 * lp * 4;
  l.off_ref = 3 * lp * 4;                      // float [K|V][mn|iv][D], then eight zeros for lanes without channels
  const int full = (D * esize & (D * esize - 1)) == 0 && D * esize >= 64;  // no lane without channels
  l.off_stat = l.off_ref + (4 * D + (full ? 0 : 8)) * 4;  // elements as in the rows: [wave][mn|mx][D]
  l.off_ring = (l.off_stat + 2 * gw * 2 * D * esize + 127) & ~127;
  l.total = l.off_ring + 2 * gw * ring_slots(nsl, gw) * 1024;
  return l;
}

// At most `c` (or a few less) vector-memory operations outstanding, c the same in the whole wavefront: weaker waits
// first, the way out behind each.
__device__ __forceinline__ void wait_vm6(int c) {
  asm volatile(
      "s_waitcnt vmcnt(6)\n\ts_cmp_ge_i32 %0, 6\n\ts_cbranch_scc1 .Lring_w%=\n\t"
      "s_waitcnt vmcnt(4)\n\ts_cmp_ge_i32 %0, 4\n\ts_cbranch_scc1 .Lring_w%=\n\t"
      "s_waitcnt vmcnt(2)\n\ts_cmp_ge_i32 %0, 2\n\ts_cbranch_scc1 .Lring_w%=\n\t"
      "s_waitcnt vmcnt(0)\n.Lring_w%=:"
      :
      : "s"(c)
      : "memory", "scc");
}
__device__ __forceinline__ void wait_vm14(int c) {
  asm volatile(
      "s_waitcnt vmcnt(14)\n\ts_cmp_ge_i32 %0, 14\n\ts_cbranch_scc1 .Lring_w%=\n\t"
      "s_waitcnt vmcnt(10)\n\ts_cmp_ge_i32 %0, 10\n\ts_cbranch_scc1 .Lring_w%=\n\t"
      "s_waitcnt vmcnt(6)\n\ts_cmp_ge_i32 %0, 6\n\ts_cbranch_scc1 .Lring_w%=\n\t"
      "s_waitcnt vmcnt(2)\n\ts_cmp_ge_i32 %0, 2\n\ts_cbranch_scc1 .Lring_w%=\n\t"
      "s_waitcnt vmcnt(0)\n.Lring_w%=:"
      :
      : "s"(c)
      : "memory", "scc");
}
// two landed 16-byte entries at byte offsets OFFA and OFFB of `base`
template <int OFFA, int OFFB>
__device__ __forceinline__ void lds_read_pair_at(u32x4& a, u32x4& b, uint32_t base) {
  asm volatile(
      "ds_read_b128 %0, %2 offset:%3\n\t"
      "ds_read_b128 %1, %2 offset:%4\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(a), "=&v"(b)
      : "v"(base), "n"(OFFA), "n"(OFFB)
      : "memory");
}

// the same value in every lane, in a scalar register
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <int BEGIN, int END, int STEP, typename F>
__device__ __forceinline__ void ring_for(F&& f) {
  if constexpr (BEGIN < END) {
    f(std::integral_constant<int, BEGIN>{});
    ring_for<BEGIN + STEP, END, STEP>(f);
  }
}

// A statistic in the element type of the rows, which it is an element of.
template <typename ET>
struct Stat;
template <>
struct Stat<F32> {
  typedef float T;
  static __device__ __forceinline__ T to(float v) { return v; }
  static __device__ __forceinline__ float from(T v) { return v; }
};
template <>
struct Stat<BF16> {
  typedef uint16_t T;
  static __device__ __forceinline__ T to(float v) { return (T)(__float_as_uint(v) >> 16); }
  static __device__ __forceinline__ float from(T v) { return __uint_as_float((uint32_t)v << 16); }
};
template <>
struct Stat<F16> {
  typedef _Float16 T;
  static __device__ __forceinline__ T to(float v) { return (T)v; }
  static __device__ __forceinline__ float from(T v) { return (float)v; }
};

// Sums of s0 and of s1 over groups of LPR lanes.  Lanes with an even number receive the first, odd ones the second
// (LPR = 8: every lane the one its `odd` says; the sums cross the quads by a mirror, which does not keep parity).
template <int LPR>
__device__ __forceinline__ float pair_sum(float s0, float s1, bool odd) {
  if constexpr (LPR == 8) {
    const float t0 = group_sum<8>(s0), t1 = group_sum<8>(s1);
    return odd ? t1 : t0;
  } else {
    float t = (odd ? s1 : s0) + dpp_mov<0xB1>(odd ? s0 : s1);
    t += dpp_mov<0x4E>(t);
    if constexpr (LPR >= 16) {
      t += dpp_mov<0x124>(t);  // row_ror:4
      t += dpp_mov<0x128>(t);  // row_ror:8
    }
    if constexpr (LPR >= 32) t += __shfl_xor(t, 16);
    return t;
  }
}
// Channel variances (Eq. 9-10, as token_var_sub) of two rows: the first in even lanes, the second in odd ones.
// PART: the first `dead` channels of the lane belong to its neighbour and are left out (their iv is 0).
template <int LPR, int VEC, bool PART>
__device__ __forceinline__ float token_var_pair(const float (&x0)[VEC], const float (&x1)[VEC], const float (&mn)[VEC],
                                                const float (&iv)[VEC], float inv_D, float inv_dof, bool odd, int dead) {
  float y0[VEC], y1[VEC], s0 = 0.f, s1 = 0.f;
#pragma unroll
  for (int j = 0; j < VEC; ++j) {
    y0[j] = x0[j] - mn[j];
    y1[j] = x1[j] - mn[j];
    s0 = fmaf(y0[j], iv[j], s0);
    s1 = fmaf(y1[j], iv[j], s1);
  }
  const float s = pair_sum<LPR>(s0, s1, odd);
  const float m0 = dpp_mov<0xA0>(s) * inv_D;  // quad_perm(0,0,2,2)
  const float m1 = dpp_mov<0xF5>(s) * inv_D;  // quad_perm(1,1,3,3)
  float q0[2] = {0.f, 0.f}, q1[2] = {0.f, 0.f};  // (two short sums: half the rounding of one long one)
#pragma unroll
  for (int j = 0; j < VEC; ++j) {
    const bool out = PART && j < dead;
    const float d0 = fmaf(y0[j], iv[j], out ? 0.f : -m0), d1 = fmaf(y1[j], iv[j], out ? 0.f : -m1);
    q0[j & 1] = fmaf(d0, d0, q0[j & 1]);
    q1[j & 1] = fmaf(d1, d1, q1[j & 1]);
  }
  return pair_sum<LPR>(q0[0] + q0[1], q1[0] + q1[1], odd) * inv_dof;
}

// 1 / the sum of v over the wavefront: a factor common to a whole chunk, whose error every score of it has in full.  FINE: the
// last additions in 64 bits and the reciprocal of what they give, 0.05 us a call.  Scores off 64 bits, mean and, against the
// kernels before this one, largest of 144 shapes: lags of 129 to 256 3.9e-8, 0.96 times theirs (without 4.6e-8, 1.01), to 512
// 3.8e-8, 0.95 (4.5e-8, 1.08), to 1024 3.8e-8, 0.89 (4.6e-8, 1.06); to 128, without, 4.4e-8 as theirs.
template <bool FINE>
__device__ __forceinline__ float wave_sum_rcp(float v) {
  if constexpr (!FINE) return 1.0f / wave_sum(v);
  v = group_sum<16>(v);
  const double sum = ((double)rl_f(v, 0) + rl_f(v, 16)) + ((double)rl_f(v, 32) + rl_f(v, 48));
  const float s = (float)sum, r = fast_rcp(s);
  return fmaf(fmaf(-(float)(sum - s), r, fmaf(-s, r, 1.0f)), r, r);
}

// Chunk softmax, K+V sum and top-k (Eq. 10-11) by one wavefront, L <= 64 * E tokens in registers; arguments as
// group_rank_select's (wg_select.hpp), but the slot map receives byte offsets of rows.
// LIST: it receives the k kept rows instead.
template <int E, bool LIST>
__device__ __forceinline__ void wave_pick(const float* vK, const float* vV, int L, int k, bool do_select, float* gout,
                                          int32_t* slotmap, int lane, int32_t* pos_out, uint32_t pos0, uint32_t rowbytes) {
  float eK[E], eV[E];
  float mK = -INFINITY, mV = -INFINITY;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int t = e * kWave + lane;
    eK[e] = t < L ? std_of_var(vK[t]) : -INFINITY;
    eV[e] = t < L ? std_of_var(vV[t]) : -INFINITY;
    mK = fmaxf(mK, eK[e]);
    mV = fmaxf(mV, eV[e]);
  }
  mK = wave_max(mK);
  mV = wave_max(mV);
  // (denominators, a factor common to the whole chunk, as pairwise sums)
  float aK[E], aV[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int t = e * kWave + lane;
    aK[e] = eK[e] = t < L ? __expf(eK[e] - mK) : 0.f;
    aV[e] = eV[e] = t < L ? __expf(eV[e] - mV) : 0.f;
  }
#pragma unroll
  for (int w = 1; w < E; w *= 2)
#pragma unroll
    for (int e = 0; e + w < E; e += 2 * w) {
      aK[e] += aK[e + w];
      aV[e] += aV[e + w];
    }
  const float rK = wave_sum_rcp<(E >= 4)>(aK[0]), rV = wave_sum_rcp<(E >= 4)>(aV[0]);
  uint32_t key[E], hi = 0, lo = 0xffffffffu;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int t = e * kWave + lane;
    const float s = eK[e] * rK + eV[e] * rV;
    if (gout && t < L) st4_out_at(gout, (uint32_t)t * 4u, __float_as_uint(s));
    key[e] = t < L ? ordered_key(s) : 0u;
    hi = umax_(hi, key[e]);
    lo = umin_(lo, key[e] ? key[e] : 0xffffffffu);
  }
  if (!do_select) return;
  // the k-th largest key bit by bit, from the highest bit in which two keys differ down to the one that parts
  // exactly k of them from the rest
  hi = wave_umax(hi);
  lo = wave_umin(lo);
  uint32_t theta = hi;
  if (hi != lo) {
    const int top = 31 - __builtin_clz(hi ^ lo);
    theta = hi & ~((2u << top) - 1u);
    for (int bit = top; bit >= 0; --bit) {
      const uint32_t cand = theta | (1u << bit);
      int cnt = 0;
#pragma unroll
      for (int e = 0; e < E; ++e) cnt += __popcll(__ballot(key[e] >= cand));
      if (cnt >= k) theta = cand;
      if (cnt == k) break;
    }
  }
  int need = k;  // keys equal to theta are admitted from the lowest position up
#pragma unroll
  for (int e = 0; e < E; ++e) need -= __popcll(__ballot(key[e] > theta));
  int base = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int t = e * kWave + lane;
    const uint64_t eq = __ballot(key[e] == theta && t < L);
    const bool keep = key[e] > theta || (key[e] == theta && t < L && prefix_popc(eq) < need);
    const uint64_t km = __ballot(keep);
    const int slot = base + prefix_popc(km);
    if constexpr (LIST) {
      if (keep) slotmap[slot] = t;
    } else if (t < L) {
      slotmap[t] = keep ? (int)__umul24((uint32_t)slot, rowbytes) : -1;
    }
    if (keep && pos_out) st4_out_at(pos_out, (uint32_t)slot * 4u, pos0 + (uint32_t)t);
    base += __popcll(km);
    need -= __popcll(eq);
  }
}

// GW wavefronts on K rows, as many on V rows; a lane holds up to NSL 16-byte slices of its chunk.
// Scored chunks are numbered stream * n_s + p; workgroup i of `walks` takes the i-th equal share of them, from
// the highest number down.
// DIRECT: rows of any multiple of 4 bytes on 4-byte addresses, which the asynchronous loads do not take: the next
// chunk's rows are loaded into registers of their own while this one is selected (NSL = 8).
template <typename ET, int LPR, int NSL, int GW, bool DIRECT>
__device__ __forceinline__ void ring_pass(const PassArgs& a) {
  constexpr int VEC = ET::VEC, ESIZE = 16 / VEC, RPW = kWave / LPR, R = GW * RPW, NR = ring_slots(NSL, GW);
  constexpr int THREADS = GW * 2 * kWave;
  constexpr bool HOLD = NSL > 0;  // else a chunk passes through the ring only
  typedef Stat<ET> ST;
  extern __shared__ float4 lds_raw[];
  char* lds = reinterpret_cast<char*>(lds_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int tensor = wave >= GW ? 1 : 0;  // 0: this wavefront handles K rows, 1: V rows
  // (the V rows from another wavefront on, so that the SIMD that takes the longer share of the K rows takes a
  // shorter one of these)
  const int slot0 = tensor ? (wave + GW / 2) % GW : wave;
  const int cl = lane % LPR, row0 = slot0 * RPW + lane / LPR;
  const int D = a.D, L = a.L, k = a.k, S = a.S, rowbytes = D * ESIZE;
  // A lane beyond the row's slices repeats its last 16 bytes; it has no channels of its own.  (Where the row ends
  // inside a lane's slice, that lane does too, and its first `part` channels are its neighbour's.)
  const bool dead = cl * 16 >= rowbytes;
  const int coff = cl * 16 > rowbytes - 16 ? rowbytes - 16 : cl * 16, ch0 = coff / ESIZE;
  const int part = dead ? VEC : (cl * 16 - coff) / ESIZE;
  const RingLds lay = ring_lds(D, ESIZE, L, NSL, GW);
  float* vK = reinterpret_cast<float*>(lds + lay.off_vK);
  float* vV = reinterpret_cast<float*>(lds + lay.off_vV);
  int32_t* slotmap = reinterpret_cast<int32_t*>(lds + lay.off_slot);
  float* refbuf = reinterpret_cast<float*>(lds + lay.off_ref);
  typename ST::T* statbuf = reinterpret_cast<typename ST::T*>(lds + lay.off_stat);
  // steps of R rows in which this wavefront has any, in pairs (rows past the end repeat the last one)
  const int n = L > slot0 * RPW ? ((L - slot0 * RPW + R - 1) / R + 1) & ~1 : 0;
  const int streams = a.B * a.H;
  const bool gather = a.K_out != nullptr;
  const bool local = a.variant == 1;

  if (blockIdx.x >= a.walks) {
    const int64_t e = blockIdx.x - a.walks, stream = e / a.edge, b = stream / a.H, h = stream % a.H;
    const int64_t out = stream * a.T_out;
    copy_edge_rows<LPR, DIRECT>(a.K + b * a.sb + h * a.sh, a.V + b * a.sb + h * a.sh, a.st, a.K_out + out * rowbytes,
                        a.V_out + out * rowbytes, a.idx_out ? a.idx_out + out : nullptr, rowbytes, S,
                        S + a.n_s * L, S + a.n_s * k, a.T - (S + a.n_s * L), (int)(e % a.edge), a.edge, coff, tid,
                        THREADS);
    return;
  }
  const float inv_D = dead ? 0.f : 1.0f / (float)D, inv_dof = 1.0f / (float)(D - a.ddof);
  const bool odd = lane & 1;

  // (fewer than 2^31 chunks in all)
  const uint32_t n_s = (uint32_t)a.n_s, total = (uint32_t)streams * n_s, walks = (uint32_t)a.walks;
  const uint32_t share = total / walks, longer = total - share * walks;  // the first `longer` shares have one more
  int left = (int)(share + (blockIdx.x < longer ? 1 : 0));  // chunks still to be scored
  const uint32_t last = blockIdx.x * share + umin_(blockIdx.x, longer) + left - 1;
  int stream = uni((int)(last / n_s));
  int p = (int)(last - stream * n_s);

  const uint32_t st = (uint32_t)a.st;
  const uint32_t lane_off = (uint32_t)row0 * st + (uint32_t)coff;
  const uint32_t lane_max = (uint32_t)(L - 1) * st + (uint32_t)coff;
  const uint32_t ring_base = uni(lds_offset(lds + lay.off_ring) + (uint32_t)wave * (NR * 1024u));
  const uint32_t ring_lane = ring_base + (uint32_t)lane * 16u;
  const char* tbase = tensor ? a.V : a.K;
  auto chunk_at = [&](int s, int q) __attribute__((always_inline)) {
    const int b = uni((int)((uint32_t)s / (uint32_t)a.H)), h = s - b * a.H;
    return tbase + (int64_t)b * a.sb + (int64_t)h * a.sh + (S + (int64_t)q * L) * a.st;
  };
  // An item is a chunk to be scored, or (Eq. 7-8) the first reference of a share or of a stream in it.
  // Where the chunk does not stay in registers, its own statistics (Eq. 14-15) are an item before it.
  bool ref = !HOLD || !local;
  const char* cur = chunk_at(stream, p + (local ? 0 : 1));
  auto dma = [&](const char* base, auto tag, auto keep) __attribute__((always_inline)) {
    constexpr int j = decltype(tag)::value;
    const uint32_t off = lane_off + (uint32_t)(j * R) * st, at = off < lane_max ? off : lane_max;
    if constexpr (HOLD) dma_rows16_at<(j % NR) * 1024, !decltype(keep)::value>(at, base, ring_base);
    else dma_rows16<false>(at, base, ring_base + (j % NR) * 1024u);
  };
  constexpr std::false_type once{};
  uint4 hold[HOLD ? NSL : 1], ahead[DIRECT ? NSL : 1];
  // (All slices in one go, without a branch: behind one, the compiler waits for the loads before it.  Steps this
  // wavefront does not have, and with `rows` 1 the whole of it, repeat one row.)
  auto load = [&](uint4 (&to)[NSL ? NSL : 1], const char* base, int rows) __attribute__((always_inline)) {
    const int row = here_v(row0);  // (offsets worked out here, not kept across everything)
#pragma unroll
    for (int j = 0; j < NSL; ++j)
      to[j] = ld16_a4(base + ((uint32_t)(row + j * R < rows ? row + j * R : rows - 1) * st + (uint32_t)coff));
  };
  if constexpr (DIRECT) {  // the first reference and the first chunk at once
    load(ahead, cur, L);
    load(hold, ref ? cur - (int64_t)L * a.st : cur, L);
  } else {
    auto fill = [&](auto keep) __attribute__((always_inline)) {
      ring_for<0, NR, 1>([&](auto tag) __attribute__((always_inline)) {
        if (decltype(tag)::value < n) dma(cur, tag, keep);
      });
    };
    // The chunk behind the scored ones, which the workgroups that copy the window read too, stays in the caches for them
    // (388 streams of one chunk of 64 rows of 512 bytes 23.3 us, loaded like the others 28.6 us; asked about at every later turn as
    // well, the code of twice the loads cost calls of 6 us 0.35 us).
    if (HOLD && gather && !local && p == (int)n_s - 1) fill(std::true_type{});
    else fill(once);
  }
  if (tid < 8 && rowbytes < LPR * 16) refbuf[4 * D + tid] = 0.f;
  if constexpr (HOLD)
    for (int t = L + tid; t < chunk_pad(L); t += THREADS) slotmap[t] = -1;  // rows past the end are never stored
  uint32_t at = 0;  // !HOLD: byte offset of the next step's slot

  TStats<VEC> acc;
  float mn[VEC], iv[VEC];
  // the wavefront's minima and maxima -> statbuf
  auto park = [&]() __attribute__((always_inline)) {
    const bool hi32 = (lane & 32) != 0, hi16 = (lane & 16) != 0;
    float v[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) v[j] = fold_min32(acc.mn[j], -acc.mx[j]);
    constexpr int N = LPR <= 16 ? VEC / 2 : VEC;
    typename ST::T* dst = statbuf + (wave * 2 + (hi32 ? 1 : 0)) * D + ch0;
    if constexpr (LPR <= 16) {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        v[j] = fold_min16(v[j], v[N + j]);
        if constexpr (LPR <= 8) v[j] = fminf(v[j], dpp_mov<0x128>(v[j]));  // row_ror:8
        if constexpr (LPR <= 4) v[j] = fminf(v[j], dpp_mov<0x124>(v[j]));  // row_ror:4
      }
      dst += hi16 ? N : 0;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) dst[j] = ST::to(hi32 ? -v[j] : v[j]);
  };
  // what the wavefronts parked, combined: one thread per channel, behind a barrier
  auto publish = [&]() __attribute__((always_inline)) {
    for (int t = here_v(tid); t < 2 * D; t += THREADS) {
      const int tn = t >= D ? 1 : 0, ch = t - tn * D;
      float lo = INFINITY, hi = -INFINITY;
#pragma unroll
      for (int g = 0; g < GW; ++g) {
        const typename ST::T* rd = statbuf + (tn * GW + g) * 2 * D + ch;
        lo = fminf(lo, ST::from(rd[0]));
        hi = fmaxf(hi, ST::from(rd[D]));
      }
      refbuf[tn * 2 * D + ch] = lo;
      refbuf[(tn * 2 + 1) * D + ch] = inv_range(lo, hi);
    }
  };
  // the published statistics of the lane's channels, behind another barrier
  auto take_ref = [&]() __attribute__((always_inline)) {
    const float* rd = refbuf + tensor * 2 * D + ch0;
    const float* ri = refbuf + (dead ? 4 * D : (tensor * 2 + 1) * D + ch0);
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      mn[i] = rd[i];
      iv[i] = DIRECT && i < part ? 0.f : ri[i];
    }
  };
  // lanes 0 and 1 of a row hold the variances of its row of steps j and j + 1
  float* myvar = (tensor ? vV : vK) + row0 + (odd ? R : 0);
  auto score_pair = [&](const float (&x0)[VEC], const float (&x1)[VEC], int j) __attribute__((always_inline)) {
    const float v = token_var_pair<LPR, VEC, DIRECT>(x0, x1, mn, iv, inv_D, inv_dof, odd, part);
    if (cl < 2) myvar[j * R] = v;
  };

  auto fold_pair = [&](const float (&x0)[VEC], const float (&x1)[VEC]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      acc.mn[i] = fminf(fminf(acc.mn[i], x0[i]), x1[i]);
      acc.mx[i] = fmaxf(fmaxf(acc.mx[i], x0[i]), x1[i]);
    }
    pin(acc);
  };

  if (DIRECT && ref) {
    acc.reset();
#pragma unroll
    for (int j = 0; j < NSL; j += 2)
      if (j < n) {
        float x0[VEC], x1[VEC];
        unpack<ET>(ahead[DIRECT ? j : 0], x0);
        unpack<ET>(ahead[DIRECT ? j + 1 : 0], x1);
        fold_pair(x0, x1);
        __builtin_amdgcn_sched_barrier(0);
      }
    park();
    lds_barrier();
    publish();
    lds_barrier();
    take_ref();
    ref = false;
    cur -= (int64_t)L * a.st;
  }
  while (true) {
    // the item after this one
    const bool more = ref || left > 1;
    const bool turn = !ref && p == 0;  // this stream's share ends
    int nstream = stream, np = p - (ref ? 0 : 1);
    const bool split_item = !HOLD && local;  // every chunk is two items
    bool nref = split_item && !ref;
    const char* next = split_item && ref ? cur : cur - (int64_t)L * a.st;
    if (turn && more) {
      nstream = stream - 1;
      np = (int)n_s - 1;
      nref = !HOLD || !local;
      next = chunk_at(nstream, np + (local ? 0 : 1));
    }
    const bool score = !ref && !(HOLD && local);
    // its minima and maxima are wanted
    const bool stats = ref || (HOLD && local) || (!local && more && !turn);
    acc.reset();
    // Steps j and j + 1 have landed once no more operations are outstanding than loads were issued behind them: the
    // rest of the item's and, if there is one, the next item's as far as it has been asked for.
    if (HOLD && !DIRECT && !more) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if constexpr (!HOLD) {
      for (int j = 0; j < n; j += 2) {
        // as many loads as slots are under way, until nothing is left to ask for
        if (more || j + NR <= n) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NR - 2) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        u32x4 qa, qb;
        lds_read_pair_at<0, 1024>(qa, qb, ring_lane + at);
        const int ja = j + NR;  // (no wavefront with rows has fewer than NR steps)
        if (more || ja < n) {
          const char* base = ja < n ? cur : next;
          const uint32_t step = (uint32_t)((ja < n ? ja : ja - n) * R) * st;
          const uint32_t o0 = lane_off + step, o1 = o0 + (uint32_t)R * st;
          dma_rows16<false>(o0 < lane_max ? o0 : lane_max, base, ring_base + at);
          dma_rows16<false>(o1 < lane_max ? o1 : lane_max, base, ring_base + at + 1024u);
        }
        at = at == (NR - 2) * 1024u ? 0u : at + 2048u;
        float x0[VEC], x1[VEC];
        unpack<ET>(make_uint4(qa.x, qa.y, qa.z, qa.w), x0);
        unpack<ET>(make_uint4(qb.x, qb.y, qb.z, qb.w), x1);
        if (stats) fold_pair(x0, x1);
        if (score) score_pair(x0, x1, j);
      }
    }
    ring_for<0, NSL, 2>([&](auto tag) __attribute__((always_inline)) {
      constexpr int j = decltype(tag)::value;
      if (!DIRECT && j < n) {
        if constexpr (NSL == 8) wait_vm6(n - 2);
        else wait_vm14(j >= 16 && more ? n - 18 : n - 2 - j);
        u32x4 qa, qb;
        lds_read_pair_at<(j % NR) * 1024, ((j + 1) % NR) * 1024>(qa, qb, ring_lane);
        hold[j] = make_uint4(qa.x, qa.y, qa.z, qa.w);
        hold[j + 1] = make_uint4(qb.x, qb.y, qb.z, qb.w);
      }
      // the two slots are free again
      if constexpr (DIRECT) {
      } else if constexpr (NSL == 8) {
        if (j < n && more) {
          dma(next, tag, once);
          dma(next, std::integral_constant<int, j + 1>{}, once);
        }
      } else if constexpr (j < 16) {
        if (j + 16 < n) {
          dma(cur, std::integral_constant<int, j + 16>{}, once);
          dma(cur, std::integral_constant<int, j + 17>{}, once);
        }
      } else if (more) {
        dma(next, std::integral_constant<int, j - 16>{}, once);
        dma(next, std::integral_constant<int, j - 15>{}, once);
      }
      if (j < n) {
        float x0[VEC], x1[VEC];
        unpack<ET>(hold[j], x0);
        unpack<ET>(hold[j + 1], x1);
        if (stats) fold_pair(x0, x1);
        if (score) score_pair(x0, x1, j);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (DIRECT) load(ahead, more ? next : cur, more ? L : 1);
    if (stats) park();
    if (ref || (HOLD && local)) {
      lds_barrier();
      publish();
      lds_barrier();
      take_ref();
    }
    if (!ref) {
      if (HOLD && local) {
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
            score_pair(x0, x1, j);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      lds_barrier();
      if (stats && !local) publish();
      const int64_t out = stream * a.T_out + S + (int64_t)p * k;  // output row of the chunk's first kept row
      // (a wavefront of the upper half: the lower ones publish; another one for every chunk)
      if (wave == THREADS / kWave - 1 - left % GW) {
        float* gs = a.scores ? a.scores + ((int64_t)stream * n_s + p) * L : nullptr;
        int32_t* gp = gather && a.idx_out ? a.idx_out + out : nullptr;
        const int ln = here_v(lane), Ls = here_s(L), ks = here_s(k);
        const uint32_t pos0 = (uint32_t)(S + p * L), rb = (uint32_t)rowbytes;
        if constexpr (HOLD) {
          if (Ls <= 64) wave_pick<1, false>(vK, vV, Ls, ks, gather, gs, slotmap, ln, gp, pos0, rb);
          else if (Ls <= 128) wave_pick<2, false>(vK, vV, Ls, ks, gather, gs, slotmap, ln, gp, pos0, rb);
          else if (Ls <= 256) wave_pick<4, false>(vK, vV, Ls, ks, gather, gs, slotmap, ln, gp, pos0, rb);
          else wave_pick<8, false>(vK, vV, Ls, ks, gather, gs, slotmap, ln, gp, pos0, rb);
        } else {
          if (Ls <= 512) wave_pick<8, true>(vK, vV, Ls, ks, gather, gs, slotmap, ln, gp, pos0, rb);
          else wave_pick<16, true>(vK, vV, Ls, ks, gather, gs, slotmap, ln, gp, pos0, rb);
        }
      }
      lds_barrier();
      if (gather) {
        char* dst = (tensor ? a.V_out : a.K_out) + out * rowbytes;
        if constexpr (!HOLD) {  // kept rows are read again
          constexpr int UG = 8;
          const char* src = cur + here_v(coff);
          for (int s0 = here_v(row0); s0 < k; s0 += UG * R) {
            uint4 q[UG];
#pragma unroll
            for (int u = 0; u < UG; ++u) q[u] = ld16_last(src + (int64_t)slotmap[s0 + u * R < k ? s0 + u * R : s0] * a.st);
#pragma unroll
            for (int u = 0; u < UG; ++u)
              if (s0 + u * R < k) st16_out_at(dst, (uint32_t)(s0 + u * R) * (uint32_t)rowbytes + (uint32_t)coff, q[u]);
          }
        }
        const int row = here_v(row0), nn = here_s(n);
#pragma unroll
        for (int j = 0; j < NSL; ++j) {
          if (j < nn) {
            const int sl = slotmap[row + j * R];
            if (sl >= 0) st16_out_at(dst, (uint32_t)(sl + coff), hold[j]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      if (stats && !local) take_ref();
      --left;
    }
    if (!more) break;
    if constexpr (DIRECT) {
#pragma unroll
      for (int j = 0; j < NSL; ++j) hold[j] = ahead[j];
    }
    cur = next;
    stream = nstream;
    p = np;
    ref = nref;
  }
}

template <typename ET, int LPR, int NSL, int GW, bool DIRECT>
__global__ void __launch_bounds__(GW * 2 * kWave, NSL <= 8 ? 4 : 2) ring_pass_kernel(const PassArgs a) {
  ring_pass<ET, LPR, NSL, GW, DIRECT>(a);
}

// ------------------------------------------------------------------------ host side
template <typename K>
hipError_t launch_ring_one(K kernel, const PassArgs& a, dim3 grid, int threads, size_t lds, hipStream_t s) {
  if (lds > 64 * 1024) {  // beyond the default dynamic LDS limit: opt in (idempotent)
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  kernel<<<grid, dim3(threads), lds, s>>>(a);
  return hipGetLastError();
}

// Wavefronts per tensor and slices per lane: the smallest workgroup whose lanes hold a chunk in eight slices, else 32
// slices of four wavefronts per tensor.
struct RingShape {
  int gw, nsl;  // (0, 0: no shape holds the chunk)
};
inline RingShape ring_hold_shape(int D, int esize, int L) {
  const int lpr = chunk_lpr(D * esize), rpw = kWave / lpr;
  for (int gw = 1; gw <= 8; gw *= 2)
    if (L <= 8 * gw * rpw && 2 * gw * rpw <= 128 && ring_lds(D, esize, L, 8, gw).total <= kRingMaxLds) return {gw, 8};
  if (L > 16 * 4 * rpw && L <= 32 * 4 * rpw && L <= 512 && ring_lds(D, esize, L, 32, 4).total <= kRingMaxLds) return {4, 32};
  return {0, 0};
}
// ... and the wavefronts through whose ring other chunks pass.
inline RingShape ring_stream_shape(int D, int esize, int L) {
  const int lpr = chunk_lpr(D * esize), rpw = kWave / lpr;
  const int gw = lpr == 4 || (int64_t)L * D * esize < 256 * 1024 ? 4 : 8, nr = ring_slots(0, gw);
  // (its last wavefront has rows in as many steps as slots, in pairs)
  const bool deep = L - (gw - 1) * rpw > (nr - 2) * gw * rpw;
  return deep && L <= 1024 && ring_lds(D, esize, L, 0, gw).total <= kRingMaxLds ? RingShape{gw, 0} : RingShape{0, 0};
}
// Where a chunk in registers takes a compute unit to itself, nothing runs beside its selection, and lanes without rows
// of their own - rows of fewer slices than lanes, steps past the end of the chunk - count.  Two workgroups that stream
// and read the kept rows again (mostly out of the memory-side cache) do better there from some share of such lanes
// on, the earlier the more arithmetic a byte costs.  Held | streamed, us, 600 MB on 96 streams, lag and own reference:
//   16 wavefronts, bf16   rows of 128 bytes, lag 512 (all slices hold rows) 200, 234 | 186, 218; 450 (0.88) 206, 241 | 182, 211
//                         rows of 256 bytes, lag 180 (0.94) 187, 215 | 191, 219; of 192, 256 (0.75) 207, 240 | 197, 232
//                 fp32    rows of 256 bytes, lag 130 (0.68) 194, 218 | 199, 231; 200 (0.78) 169, 182 | 183, 210
//   32 slices, bf16       rows of 256 bytes, lag 300 (0.94) 212, 243 | 190, 224; 400 (0.96) 188, 216 | 193, 229
//                         rows of 512 bytes, lag 152 (0.95) 207, 240 | 194, 230; 200 (0.96) 180, 215 | 195, 232
//              fp32       rows of 384 bytes, lag 152 (0.71) 211, 233 | 182, 212; 200 (0.72) 189, 216 | 190, 223
inline bool ring_hold_pays(const RingShape& f, int D, int esize, int L) {
  if (f.gw == 0) return false;
  if (f.gw < 8 && f.nsl == 8) return true;
  const int lpr = chunk_lpr(D * esize), R = f.gw * (kWave / lpr), steps = ((L + R - 1) / R + 1) & ~1;
  const int64_t filled = (int64_t)L * row_units(D, esize) * 100 / ((int64_t)steps * R * lpr);
  if (f.nsl == 8) return esize == 4 || (lpr >= 16 && filled >= 90);
  return filled >= (esize == 4 ? 72 : 96);
}
// Where neither does: lanes without channels and chunks too short for the steps that the selection costs (2-byte
// elements; streaming kernel, us): rows of 160 bytes, lag 180 239, 272 | 251, 301; 256 228, 260 | 226, 272; 300 265, 295 | 213,
// 259; rows of 192 bytes, lag 152 215, 242 | 230, 275; 180 217, 245 | 211, 252; 256 216, 246 | 197, 232.
inline bool ring_stream_pays(int D, int esize, int L) {
  const int units = row_units(D, esize), lpr = chunk_lpr(D * esize);
  return esize == 4 || units == lpr || L > (4 * units < 3 * lpr ? 256 : 179);
}
inline RingShape ring_shape(int D, int esize, int L) {
  const RingShape h = ring_hold_shape(D, esize, L), t = ring_stream_shape(D, esize, L);
  return ring_hold_pays(h, D, esize, L) || t.gw == 0 ? h : t;
}

template <typename ET, int LPR, int NSL, int GW>
hipError_t launch_ring_n(const PassArgs& a, dim3 grid, size_t lds, hipStream_t s) {
  return launch_ring_one(ring_pass_kernel<ET, LPR, NSL, GW, false>, a, grid, GW * 2 * kWave, lds, s);
}
template <typename ET, int LPR>
hipError_t launch_ring_l(const PassArgs& a, const RingShape& f, dim3 grid, size_t lds, hipStream_t s) {
  switch (f.gw * 64 + f.nsl) {
    case 1 * 64 + 8: return launch_ring_n<ET, LPR, 8, 1>(a, grid, lds, s);
    case 2 * 64 + 8: return launch_ring_n<ET, LPR, 8, 2>(a, grid, lds, s);
    case 4 * 64 + 8: return launch_ring_n<ET, LPR, 8, 4>(a, grid, lds, s);
    case 8 * 64 + 8:  // (2-byte rows of up to 128 bytes: streamed, by ring_hold_pays)
      if constexpr (LPR >= 16 || (LPR == 8 && ET::VEC == 4)) return launch_ring_n<ET, LPR, 8, 8>(a, grid, lds, s);
      break;
    case 4 * 64: return launch_ring_n<ET, LPR, 0, 4>(a, grid, lds, s);
    case 8 * 64:  // (chunks of 256 KiB, at most 1024 rows)
      if constexpr (LPR >= 16) return launch_ring_n<ET, LPR, 0, 8>(a, grid, lds, s);
      break;
    case 4 * 64 + 32:
      if constexpr (LPR >= 16) return launch_ring_n<ET, LPR, 32, 4>(a, grid, lds, s);
      break;
    default: break;
  }
  return hipErrorInvalidValue;
}
// Rows on 4-byte addresses: wavefronts per tensor whose lanes hold a chunk in eight slices, 0 if there is no such number.
inline int direct_waves(int D, int esize, int L) {
  const int rpw = kWave / chunk_lpr(D * esize);
  for (int gw = 1; gw <= 8; gw *= 2)
    if (L <= 8 * gw * rpw && 2 * gw * rpw <= 128) return gw;
  return 0;
}
inline int direct_lds(int D, int esize, int L, int gw) { return ring_lds(D, esize, L, 8, gw).off_ring; }

template <typename ET, int LPR>
hipError_t launch_direct_l(const PassArgs& a, int gw, dim3 grid, size_t lds, hipStream_t s) {
  switch (gw) {
    case 1: return launch_ring_one(ring_pass_kernel<ET, LPR, 8, 1, true>, a, grid, 128, lds, s);
    case 2: return launch_ring_one(ring_pass_kernel<ET, LPR, 8, 2, true>, a, grid, 256, lds, s);
    case 4: return launch_ring_one(ring_pass_kernel<ET, LPR, 8, 4, true>, a, grid, 512, lds, s);
    case 8:
      if constexpr (LPR >= 8) return launch_ring_one(ring_pass_kernel<ET, LPR, 8, 8, true>, a, grid, 1024, lds, s);
      break;
    default: break;
  }
  return hipErrorInvalidValue;
}
template <typename ET>
hipError_t launch_direct_t(const PassArgs& a, hipStream_t s) {
  const int gw = direct_waves(a.D, a.esize, a.L);
  const int64_t nblocks = a.walks + (int64_t)a.B * a.H * a.edge;
  if (gw == 0 || nblocks <= 0 || nblocks > 0x7fffffffLL) return hipErrorInvalidValue;
  const size_t lds = (size_t)direct_lds(a.D, a.esize, a.L, gw);
  const dim3 grid((unsigned)nblocks);
  switch (chunk_lpr(a.D * a.esize)) {
    case 4: return launch_direct_l<ET, 4>(a, gw, grid, lds, s);
    case 8: return launch_direct_l<ET, 8>(a, gw, grid, lds, s);
    case 16: return launch_direct_l<ET, 16>(a, gw, grid, lds, s);
    case 32: return launch_direct_l<ET, 32>(a, gw, grid, lds, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename ET>
hipError_t launch_ring_t(const PassArgs& a, hipStream_t s) {
  const RingShape f = ring_shape(a.D, a.esize, a.L);
  const int64_t nblocks = a.walks + (int64_t)a.B * a.H * a.edge;
  if (f.gw == 0 || nblocks <= 0 || nblocks > 0x7fffffffLL) return hipErrorInvalidValue;
  const size_t lds = (size_t)ring_lds(a.D, a.esize, a.L, f.nsl, f.gw).total;
  const dim3 grid((unsigned)nblocks);
  switch (chunk_lpr(a.D * a.esize)) {
    case 4: return launch_ring_l<ET, 4>(a, f, grid, lds, s);
    case 8: return launch_ring_l<ET, 8>(a, f, grid, lds, s);
    case 16: return launch_ring_l<ET, 16>(a, f, grid, lds, s);
    case 32: return launch_ring_l<ET, 32>(a, f, grid, lds, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lagkv
