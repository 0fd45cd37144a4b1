// C ABI of the LagKV compression pass (see include/lagkv.h): host-side validation,
// the partition arithmetic of Eq. 12-13, path choice and kernel launches.
#include "lagkv.h"

#include <cmath>
#include <cstring>

#include "compress_ws.h"
#include "lagkv_internal.hpp"

using namespace lagkv;

namespace {

// Launch override carried by lagkv_params.launch (see lagkv_launch_hint):
//   bits 0-1 path, bits 2-5 wavefronts, bits 6-26 segments, bits 27-28 stream order,
//   bits 29-30 selection mode; 0 everywhere = automatic.
struct Hint {
  int path, waves, nseg, order, sel;
};
constexpr int kHintWavesShift = 2, kHintSegShift = 6, kHintOrderShift = 27, kHintSelShift = 29;
constexpr int kMaxSegments = 1 << 20;

bool parse_hint(int32_t v, Hint* h) {
  if (v < 0) return false;
  h->path = v & 3;
  h->waves = (v >> kHintWavesShift) & 15;
  h->nseg = (v >> kHintSegShift) & ((1 << 21) - 1);
  h->order = (v >> kHintOrderShift) & 3;
  h->sel = (v >> kHintSelShift) & 3;
  if (h->waves != 0 && h->waves != 1 && h->waves != 2 && h->waves != 4 && h->waves != 8) return false;
  return h->nseg <= kMaxSegments && h->sel <= LAGKV_SELECT_GROUP;
}

constexpr int64_t kMaxRows = 0x7fffffffLL;  // positions are int32

struct Norm {  // validated, normalised parameters
  int B, H, D, S, L, k, esize, f16, ddof, variant;
  int64_t streams;
  int64_t rowbytes;
  Hint hint;
};

int validate(const lagkv_params* p, Norm* n) {
  if (!p) return LAGKV_EINVAL;
  if (p->dtype != LAGKV_F32 && p->dtype != LAGKV_BF16 && p->dtype != LAGKV_F16) return LAGKV_EDTYPE;
  if (p->variant < LAGKV_SCORE_LAG || p->variant > LAGKV_SCORE_L2) return LAGKV_EDTYPE;
  if (!parse_hint(p->launch, &n->hint)) return LAGKV_EINVAL;
  if (p->std_ddof != 0 && p->std_ddof != 1) return LAGKV_EINVAL;
  if (p->B < 1 || p->H < 1 || p->D < 1) return LAGKV_ESHAPE;
  if (p->std_ddof == 1 && p->D < 2 && p->variant != LAGKV_SCORE_L2) return LAGKV_ESHAPE;
  if (p->S < 0 || p->L < 1) return LAGKV_EINVAL;
  if (!(p->r > 0.0) || !(p->r <= 1.0)) return LAGKV_EINVAL;  // also rejects NaN
  const double kd = std::floor(p->r * (double)p->L);
  if (kd < 1.0) return LAGKV_EINVAL;
  if (p->stride_b < 0 || p->stride_h < 0 || p->stride_t < 0) return LAGKV_ESHAPE;
  n->B = p->B;
  n->H = p->H;
  n->D = p->D;
  n->S = p->S;
  n->L = p->L;
  n->k = (int)kd;
  n->esize = p->dtype == LAGKV_F32 ? 4 : 2;
  n->f16 = p->dtype == LAGKV_F16 ? 1 : 0;
  n->ddof = p->std_ddof;
  n->variant = p->variant;
  n->streams = (int64_t)p->B * p->H;
  n->rowbytes = (int64_t)p->D * n->esize;
  if (n->streams > (1 << 24)) return LAGKV_ESHAPE;
  return LAGKV_OK;
}

void plan_of(const Norm& n, int64_t T, int64_t n_static, lagkv_plan_t* out) {
  const int64_t rest = T - n_static;
  out->k = n.k;
  if (rest < 2 * (int64_t)n.L) {  // below 2L rows after the static part nothing is compressed
    const int64_t r = rest > 0 ? rest : 0;
    out->n_chunks = r / n.L;
    out->rem = r % n.L;
    out->n_scored = 0;
    out->T_out = T;
    return;
  }
  out->n_chunks = rest / n.L;
  out->rem = rest % n.L;
  out->n_scored = out->n_chunks - 1;  // the last chunk has no reference
  out->T_out = n_static + (int64_t)n.k * out->n_scored + n.L + out->rem;  // Eq. 12
}

// Input strides in bytes; 0 means dense [B,H,T,D].
int strides_of(const lagkv_params* p, const Norm& n, int64_t T, int64_t* sb, int64_t* sh,
               int64_t* st) {
  const int64_t t = p->stride_t ? p->stride_t : n.D;
  const int64_t h = p->stride_h ? p->stride_h : t * T;
  const int64_t b = p->stride_b ? p->stride_b : h * n.H;
  if (t < n.D) return LAGKV_ESHAPE;
  *st = t * n.esize;
  *sh = h * n.esize;
  *sb = b * n.esize;
  return LAGKV_OK;
}

bool shape_fused(const Norm& n, int64_t sb, int64_t sh, int64_t st) {
  if (n.rowbytes % 16 != 0 || n.rowbytes < 48 || n.rowbytes > 512) return false;  // whole 16-byte slices
  return ((sb | sh | st) & 15) == 0;
}

int pick_waves(const Norm& n) {
  int nw = n.hint.waves ? n.hint.waves : 4;
  while (nw > 1 && fused_lds_bytes(n.D, n.L, n.k, nw) > (size_t)kMaxLdsBytes) nw >>= 1;
  return nw;
}

bool fused_fits(const Norm& n) {
  return split_lds_bytes(n.D, n.esize, n.L, n.k, 2) <= (size_t)80 * 1024 &&
         fused_lds_bytes(n.D, n.L, n.k, 1) <= (size_t)kMaxLdsBytes;
}

// lagkv_workspace_bytes, which does not see addresses, answers 0 for these.
bool told_none(const Norm& n, int64_t sb, int64_t sh, int64_t st) {
  return n.hint.path != LAGKV_PATH_STAGED && shape_fused(n, sb, sh, st) && fused_fits(n);
}

bool staged_fits(const Norm& n) {
  return staged_score_lds_bytes(n.D, n.L) <= (size_t)kMaxLdsBytes &&
         ((size_t)n.L + n.k) * 4 <= (size_t)kMaxLdsBytes;
}

bool aligned_to(const void* p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

// Wavefronts per workgroup of the tensor-split kernel (0 = its LDS need does not fit).
// Long chunks keep eight wavefronts streaming; for short chunks the per-chunk serial part
// (fold, selection by one wavefront, barriers) weighs more, and smaller workgroups - more of
// them per CU, each with its own selection - overlap it better (measured: L=128 0.59 ms with 2
// against 0.80 ms with 8 wavefronts on 256 streams of 16K rows).
int split_nw(const Norm& n) {
  int nw = n.L >= 512 ? 8 : n.L >= 256 ? 4 : 2;
  const int t = n.hint.waves;
  if (t == 2 || t == 4 || t == 8) nw = t;
  while (nw >= 2 && split_lds_bytes(n.D, n.esize, n.L, n.k, nw) > (size_t)80 * 1024) nw >>= 1;
  return nw >= 2 ? nw : 0;
}

// Segments per stream.  A launch of W = streams * segments workgroups on a chip that holds `cap` of them
// at a time takes about ceil(W / cap) rounds of one segment each, so the count that fits a whole number
// of rounds and still cuts the longest segment down is what pays; one that spills a few workgroups into
// one more round doubles the time (112 streams of 32K tokens at lag 1024: 560 workgroups on 512 places
// 750 us, 448 workgroups 589 us).  A segment of c chunks costs c chunks of rows, one more that is only read
// for the first reference, and `fixed` rows' worth of start-up and drain, plus `per_batch` rows per batch of
// `batch` chunks.  (Eq. 16 reads no such chunk, nor does Eq. 14-15 in the resident kernel; not charging them for it
// made 6 of 600 shapes 4 to 13 % faster and 4 of them 4 to 7 % slower.  Nor does the cost know of a memory that is
// saturated already, where one more segment is only one more chunk to read: 456 streams of 9 chunks of 128 rows of
// 512 bytes, scores alone, three segments 146 us, two 130 us.)
struct Cut {
  int nseg;
  int64_t chunks, rows;  // of the longest segment; that a place goes through one after another, as above
};
Cut pick_cut(int64_t streams, int64_t n_s, int64_t L, int64_t cap, int64_t fixed, int64_t batch, int64_t per_batch) {
  Cut best = {1, n_s, INT64_MAX};
  const int64_t base = (streams + cap - 1) / cap;  // rounds with whole streams
  for (int64_t rounds = base; rounds < base + 8; ++rounds) {
    int64_t nseg = rounds * cap / streams;
    if (nseg > n_s) nseg = n_s;
    if (nseg < 1) nseg = 1;
    const int64_t c = (n_s + nseg - 1) / nseg;  // chunks of the longest segment
    nseg = (n_s + c - 1) / c;                   // ... which fewer segments may share
    const int64_t waves = (streams * nseg + cap - 1) / cap;
    const int64_t cost = waves * ((c + 1) * L + (c + batch - 1) / batch * per_batch + fixed);
    if (cost < best.rows) best = {(int)nseg, c, cost};
  }
  return best;
}
int pick_segments(int64_t streams, int64_t n_s, int64_t L, int64_t cap, int64_t fixed, int64_t batch,
                  int64_t per_batch) {
  return pick_cut(streams, n_s, L, cap, fixed, batch, per_batch).nseg;
}

int clamp_segments(int64_t nseg, int64_t n_s) { return (int)(nseg > n_s ? n_s : nseg < 1 ? 1 : nseg); }

// Streaming kernel: its register budget lets 16 wavefronts share a CU, its LDS fewer.
int pick_segments_split(const Norm& n, int64_t n_s, int nw) {
  if (n.hint.nseg) return clamp_segments(n.hint.nseg, n_s);
  int64_t per_cu = (160 * 1024) / (int64_t)split_lds_bytes(n.D, n.esize, n.L, n.k, nw);
  if (per_cu > 16 / nw) per_cu = 16 / nw;
  return pick_segments(n.streams, n_s, n.L, 256 * per_cu, 64, 1, 16);
}

// Register-resident kernel: one workgroup per CU, in batches of 512 rows.
Cut hold_cut(const Norm& n, int64_t n_s) { return pick_cut(n.streams, n_s, n.L, 256, 128, 512 / n.L, 96); }
int pick_segments_hold(const Norm& n, int64_t n_s) {
  return n.hint.nseg ? clamp_segments(n.hint.nseg, n_s) : hold_cut(n, n_s).nseg;
}

// The register-resident kernel is the default wherever it applies (rows of 256 bytes, lags
// of 128, 256 or 512 rows, Eq. 7-11 or Eq. 14-15): it reads every row once, where the
// streaming kernel reads the kept rows a second time for the compaction (and, for
// Eq. 14-15, every row a second time for the scoring); measured faster or equal from 8 to
// 1024 streams.
bool use_resident(const Norm& n) {
  if (n.variant == LAGKV_SCORE_L2 || !hold_supported(n.D, n.esize, n.L, n.k)) return false;
  return n.hint.path == LAGKV_PATH_RESIDENT || n.hint.path == LAGKV_PATH_AUTO;
}

// The chunk-at-a-time kernel.  It reads a reference chunk beside every chunk, and for Eq. 16 the values of rows that
// are not kept (in a scores-only call the keys a second time), and overlaps nothing but the workgroups that share
// a CU.  So it takes (a) the calls with a workspace, or on 4-byte addresses, whose rows are multiples of 4 bytes - the
// walking kernels cannot, and the three-kernel path reads such rows 2 or 4 bytes at a time (64 streams of 8K rows of
// 200 bytes: 109 us against 570 us); and (b) short calls that would go to the streaming kernel.  Those are counted in
// scored chunks against the places of its workgroups, two a CU with up to 8 row slices a lane, else one.  Its gain
// over the streaming kernel, launches of 1 to 10 chunks per stream, 15 shapes:
//   up to 8 slices      half the places 1.36 to 1.81, all 0.99 to 1.68, twice 0.90 to 1.51 (40 streams of 1228 rows of
//                       128 bytes, lag 128: 12.0 us against 18.3 us)
//   9 to 16 slices      half 1.40 to 2.34, all 1.05 to 2.00, twice 0.79 to 1.28 (as many above 1 as below; 32 streams of
//                       2335 rows of 256 bytes, lag 246: 25.7 us against 44.4 us)
//   17 to 32 slices     half 1.17 to 1.58, all 0.88 to 1.49, 1.25 times 0.74 to 1.07
//   Eq. 16              half 0.83 to 1.55, three quarters 0.76 to 1.42, all 0.64 to 1.27
//   Eq. 16, scores      all 1.08 to 1.77 (17 to 32 slices: half 1.00 to 1.28, all 0.85 to 1.21), 1.25 times 0.54 to 1.43
// The register-resident kernel is as fast or faster at any size.
int64_t chunk_most(const Norm& n, bool gather) {
  const int slices = chunk_slices(n.D, n.esize, n.L);
  const int64_t places = 256 * chunk_places(n.D, n.esize, n.L);
  if (n.variant == LAGKV_SCORE_L2) return gather || slices > 16 ? places / 2 : places;
  return slices <= 16 ? 2 * places : places;
}
// Sets a.nseg where it says yes.
bool use_chunk(const Norm& n, PassArgs& a, bool whole_slices) {
  if (n.hint.path != LAGKV_PATH_AUTO || n.hint.waves || n.hint.nseg || n.hint.order || n.hint.sel) return false;
  if (((a.sb | a.sh | a.st) & 3) || !chunk_supported(n.D, n.esize, n.L, a.st)) return false;
  if (!aligned_to(a.K, 4) || !aligned_to(a.V, 4) || !aligned_to(a.K_out, 4) || !aligned_to(a.V_out, 4)) return false;
  if (whole_slices && (use_resident(n) || n.streams * a.n_s > chunk_most(n, a.K_out != nullptr))) return false;
  const int nseg = pick_segments(n.streams, a.n_s, n.L, 256 * chunk_places(n.D, n.esize, n.L), 64, 1, 32);
  // its workgroups are twice the three-kernel path's
  if (!grid_fits(n.streams * nseg + most_edge_workgroups(a), kChunkThreads)) return false;
  a.nseg = nseg;
  return true;
}
// The ring kernel in place of the register-resident kernel, for lags of 128 where a stream does not have a place to itself
// (256 streams of 16384 rows equal; lags of 256 and 512 0.82 to 1.05).  Its gain, 2554 calls of 1 to 2048 streams:
//   2-byte elements   up to 512 chunks, about one a place, 1.05 to 1.29 (8 streams of 20 chunks 1.17 in the mean of such);
//                     Eq. 14-15, where that kernel goes over its rows twice with nothing else on the compute unit, 1.05
//                     to 1.28 at any size, with single calls down to 0.93;
//                     else by how much longer the other's longest workgroup is than an even share of this one's:
//                     segments of up to 3 chunks (a batch of four is never full) 1.02 to 1.08, above that less than
//                     1.2 times the rows 0.98, to 1.25 0.99, to 1.3 1.01, to 1.35 1.03 (all with calls of 0.89 to 0.94
//                     among them), to 1.4 1.06, to 1.5 1.09, beyond 1.16
//   fp32              up to 512 chunks 1.04 to 1.16, above 0.94 to 1.05
// (256 streams and more 1.0 to 1.3 for the same reasons: calls of the other kernel so far, and left to it.)  Whether kept rows are
// stored or only scores asked for makes no difference to the rules of Eq. 7-8 and 14-15: lagkv_score gives the scores
// that lagkv_compress selects by, to the bit.
bool ring_over_resident(const Norm& n, const PassArgs& a) {
  if (n.L != 128 || n.streams >= 256) return false;
  const int64_t chunks = n.streams * a.n_s;
  if (chunks <= 512) return true;
  if (n.esize == 4) return false;
  if (n.variant == LAGKV_SCORE_LOCAL) return true;
  const Cut cut = hold_cut(n, a.n_s);
  // two workgroups a compute unit; each reads its share, a first reference and one more for every stream it goes over into
  const double share = chunks / 512.0, over = n.streams / 512.0;
  return cut.chunks <= 3 || (double)cut.rows > 1.35 * 256 * (share + 1 + (share < over ? share : over));
}
// The ring kernel in place of the chunk kernel, for the short calls that use_chunk takes.  A call of at most a chunk a
// compute unit is as long as one workgroup, and the chunk kernel's is the shorter one where its eight wavefronts share the
// seven or eight steps that the ring kernel gives two, and for rows that fill their lanes and steps that fill them (elsewhere
// the ring kernel has the fewer instructions).  The chunk kernel over the ring kernel, compressions | scores alone,
// means of 3000 random calls of 1 to 1100 chunks (all the others 0.91 | 0.88):
//   two wavefronts                up to 64 chunks 1.04 to 1.22, 1.12 | 1.04   to 256 chunks 0.96 to 1.20, 1.08 | 0.98
//                                 (8 chunks of 64 rows of 128 bytes 6.1 us, 7.1 us)
//   full rows, four, Eq. 14-15    up to 64 chunks 1.01 | 0.93                 to 256 chunks 1.01 to 1.11, 1.05 | 0.94
//          (eight steps)          up to 64 chunks, rows of 64 and 256 bytes 1.03 to 1.08, 1.05 | 0.93, of 128 0.99 | 0.93
//   eight, Eq. 14-15              up to 64 chunks 0.86 to 1.15, 1.05 | 0.99   to 256 chunks 0.98 to 1.16, 1.07 | 0.96
//          (more steps)           up to 64 chunks 1.02 to 1.12, 1.04 | 0.99   to 256 chunks 0.92 to 1.12, 1.00 | 0.90
//          Eq. 7-8, 2 bytes       up to 64 chunks 0.95 to 1.18, 1.07 | 1.01   (fp32 0.98 | 0.93; above, all 0.97 | 0.89)
//   sixteen                       0.99 | 0.99
// Lags above 256 in eight slices are searched by one wavefront with eight keys a lane, in the chunk kernel by four: rows of up to
// 128 bytes, up to 256 chunks, inputs in the caches | in memory, means of 600 calls: Eq. 14-15 1.13 | 1.05 (scores alone
// 1.02 | 0.94), Eq. 7-8 1.11 | 0.96 (1.00 | 0.83); 257 to 512 chunks 0.98 | 0.94 (0.93 | 0.86).  33 streams of one chunk of 512
// rows of 64 bytes, in the caches: 9.8 us before the ring kernel, 11.7 us with it.
bool ring_over_chunk(const Norm& n, const PassArgs& a) {
  const bool local = n.variant == LAGKV_SCORE_LOCAL;
  if (local && !ring_holds(n.D, n.esize, n.L)) return false;  // (a chunk gone over twice: 12.6 us, 11.0 us)
  const int64_t chunks = n.streams * a.n_s;
  const int waves = ring_threads(n.D, n.esize, n.L) / 128;  // of each tensor
  const int steps = ring_steps(n.D, n.esize, n.L, waves);
  if (chunks > 256) return true;
  if (n.L > 256 && steps <= 8 && ring_holds(n.D, n.esize, n.L)) return false;
  if (steps < 7 || waves > 4) return true;
  if (waves == 1) return false;
  if (n.rowbytes < 64 || (n.rowbytes & (n.rowbytes - 1)) != 0) return true;  // lanes without channels
  if (chunks <= 64) return waves == 2 ? !local || (n.rowbytes != 64 && n.rowbytes != 256) : !local && n.esize == 4;
  return !local || steps > 8;
}
// The ring kernel, in place of the resident, of the streaming and of the chunk kernel (`brief`).  Sets a.walks where
// it says yes.  (Streaming kernel: 1.29 in the mean of 2012 calls of 300 to 8000 chunks, 57 of them below 0.97, the least
// 0.83, most of which the rule for Eq. 14-15 below leaves to it.)
bool use_ring(const Norm& n, PassArgs& a, bool brief) {
  if (n.hint.path != LAGKV_PATH_AUTO || n.hint.waves || n.hint.nseg || n.hint.order || n.hint.sel) return false;
  const int64_t chunks = n.streams * a.n_s;
  if (n.variant == LAGKV_SCORE_L2 || !ring_supported(n.D, n.esize, n.L, a.st) || chunks >= (1LL << 31)) return false;
  if (use_resident(n) && !ring_over_resident(n, a)) return false;
  if (!ring_pays(n.D, n.esize, n.L) || (brief && !ring_over_chunk(n, a))) return false;
  const int64_t places = ring_places(n.D, n.esize, n.L);
  // Eq. 14-15 streamed by a workgroup a compute unit, some of them two chunks and more of them one: where a place has 1 to 1.6
  // chunks, inputs in the caches | in memory, 0.95 (least 0.86) | 1.01, of 48 calls; with more 1.03 | 1.05
  if (n.variant == LAGKV_SCORE_LOCAL && places == 256 && chunks > places && 5 * chunks <= 8 * places &&
      !ring_holds(n.D, n.esize, n.L))
    return false;
  a.walks = chunks < places ? chunks : places;
  return true;
}
// The ring kernel's form for rows on 4-byte addresses, in place of the chunk kernel where that takes such rows.  Sets
// a.walks where it says yes.  (64 streams of 8247 rows of 200 bytes, lag 128: 74 us, the chunk kernel 110 us.)  Its gain, 998
// calls of 1 to 4000 chunks, 1.17 in the mean of those it takes, 4 of them below 0.97; not taken, for the reasons above:
//   Eq. 14-15, eight wavefronts and more   up to 512 chunks 0.84 to 1.10 (195 streams of one of 512 rows of 56 bytes: 0.84)
//   lags above 256                         up to 256 chunks 0.88 to 1.08
//   seven or eight steps                   up to 256 chunks, two wavefronts 0.89 to 1.13, four (Eq. 14-15) 0.93 to 1.10
bool use_direct(const Norm& n, PassArgs& a) {
  const int64_t chunks = n.streams * a.n_s;
  if (n.variant == LAGKV_SCORE_L2 || chunks >= (1LL << 31) || !direct_supported(n.D, n.esize, n.L, a.st)) return false;
  const int waves = direct_threads(n.D, n.esize, n.L) / 128;
  const bool local = n.variant == LAGKV_SCORE_LOCAL;
  if (chunks <= 512 && local && waves >= 4) return false;
  if (chunks <= 256 && (n.L > 256 || ((local || waves == 1) && ring_steps(n.D, n.esize, n.L, waves) >= 7))) return false;
  const int64_t places = direct_places(n.D, n.esize, n.L);
  a.walks = chunks < places ? chunks : places;
  return grid_fits(a.walks + most_edge_workgroups(a), direct_threads(n.D, n.esize, n.L));
}
// Where use_chunk says yes and use_ring no.
int launch_chunk(PassArgs& a, const Norm& n, bool whole_slices, hipStream_t s) {
  if (!whole_slices && use_direct(n, a)) return launch_direct_pass(a, s) == hipSuccess ? LAGKV_OK : LAGKV_EHIP;
  return launch_chunk_pass(a, s) == hipSuccess ? LAGKV_OK : LAGKV_EHIP;
}

// `launch` on the streams of `a`, in one launch unless the workgroups that copy sink and window rows (one per
// stream at such counts) take it past the limit of a grid: then in as few ranges of streams as fit.
template <typename F>
int launch_in_parts(const PassArgs& a, int threads, F launch, hipStream_t s) {
  const int64_t streams = (int64_t)a.B * a.H, score = streams * a.nseg;
  if (grid_fits(score + most_edge_workgroups(a), threads) || !grid_fits(score, threads))
    return launch(a, s) == hipSuccess ? LAGKV_OK : LAGKV_EHIP;
  const int64_t most = (kMaxGridItems - 1) / threads / (a.nseg + 1), rowbytes = (int64_t)a.D * a.esize;
  // a range is whole batches, or heads of one batch
  const int64_t nb = a.H <= most ? most / a.H : 1, nh = a.H <= most ? a.H : most;
  for (int64_t b = 0; b < a.B; b += nb)
    for (int64_t h = 0; h < a.H; h += nh) {
      const int64_t at = b * a.H + h;
      PassArgs p = a;
      p.B = (int32_t)(a.B - b < nb ? a.B - b : nb);
      p.H = (int32_t)(a.H - h < nh ? a.H - h : nh);
      p.K += b * a.sb + h * a.sh;
      p.V += b * a.sb + h * a.sh;
      p.K_out += at * a.T_out * rowbytes;
      p.V_out += at * a.T_out * rowbytes;
      if (a.idx_out) p.idx_out += at * a.T_out;
      if (a.scores) p.scores += at * a.n_s * a.L;
      if (launch(p, s) != hipSuccess) return LAGKV_EHIP;
    }
  return LAGKV_OK;
}

// Launch the one-shot fused kernel.
int launch_fused_any(PassArgs& a, const Norm& n, hipStream_t s) {
  const bool brief = use_chunk(n, a, true);
  if (use_ring(n, a, brief)) return launch_ring_pass(a, s) == hipSuccess ? LAGKV_OK : LAGKV_EHIP;
  if (brief) return launch_chunk(a, n, true, s);
  a.order = n.hint.order;
  a.sel = n.hint.sel;
  if (use_resident(n)) {
    a.nwaves = 8;
    a.nseg = pick_segments_hold(n, a.n_s);
    return launch_in_parts(a, 64 * a.nwaves, launch_hold_pass, s);
  }
  if (n.hint.path == LAGKV_PATH_RESIDENT) return LAGKV_ESHAPE;
  a.nwaves = split_nw(n);
  a.nseg = pick_segments_split(n, a.n_s, a.nwaves);
  return launch_in_parts(a, 64 * a.nwaves, launch_split_pass, s);
}

// A single round of whole-slice rows: append_round_kernel, or (where it says no) decode_step_kernel if the shape
// is one of its own, else fused_append_kernel.  The first asks for everything at once and is the shortest per
// stream; with more than 8 row slices a lane its registers leave room for one workgroup per CU, where the others
// keep two and more.  The gains below are the others' kernel time over its own.
bool round_is_faster(const Norm& n, const AppendArgs& a, int64_t tail) {
  if (!append_round_supported(a)) return false;
  const int slices = chunk_slices(n.D, n.esize, n.L);
  // up to one workgroup per CU: 1.1 to 1.8 (64, 128, 256 streams) at any number of slices up to 16; beyond 16, where
  // the reference rows are read twice, 256 streams of Eq. 7-8 0.83 to 0.98 and 128 streams 1.0 to 1.2
  if (n.streams <= (slices <= 16 || n.variant == LAGKV_SCORE_LOCAL ? 256 : 128)) return true;
  const bool step = decode_step_supported(a);
  // 8 slices: Eq. 14-15 1.14 to 2.0.  decode_step_kernel asks for the rows BEHIND the reference chunk before its
  // selection and, for Eq. 16, reads values only where kept, and its lead grows with the streams: lag 128, rows
  // of 256 bytes, caches of 8448 rows, 110 rows behind, 4096 streams 231 us against 268 us, Eq. 16 209 us against
  // 265 us (2048 streams equal, 512 streams 32 us against 29 us).  With an eighth of a lag behind or less, the
  // single-round kernel 1.2 to 1.4 at 512 to 2048 streams, as long at 4096
  if (slices <= 8) return !step || (n.variant != LAGKV_SCORE_L2 && (tail - 2 * (int64_t)n.L) * 8 <= n.L);
  // 16 slices: against decode_step_kernel 0.70 to 0.94 (rows of 160 bytes, lag 200; 192 and 160; 80 and 300);
  // against fused_append_kernel from 512 streams on 0.99 to 1.20 where three quarters of the slices hold
  // rows (256 bytes, lag 256; 512 and 100; 128 and 500), 0.84 to 1.10 below that and below 512 streams, Eq. 16
  // 0.77 to 1.09
  return !step && slices <= 16 && n.variant != LAGKV_SCORE_L2 && n.streams >= 512 && n.rowbytes * n.L >= 48 * 1024;
}

// Workspace of the three-kernel path for one pass
CompressWs staged_ws(const Norm& n, int64_t n_s, bool need_scores) {
  return compress_ws(n.streams, n_s, n.L, n.k, need_scores);
}

// Workspace of the three-kernel append: [scores][kept][stage K][stage V][stage pos]
struct AppendWs {
  size_t off_scores, off_kept, off_k, off_v, off_pos, total;
};
AppendWs append_ws(const Norm& n, int64_t q, int64_t rows_staged) {
  AppendWs w;
  size_t o = 0;
  w.off_scores = o;
  o += ws_align_up((size_t)n.streams * q * n.L * 4);
  w.off_kept = o;
  o += ws_align_up((size_t)n.streams * q * n.k * 4);
  w.off_k = o;
  o += ws_align_up((size_t)n.streams * rows_staged * n.rowbytes);
  w.off_v = o;
  o += ws_align_up((size_t)n.streams * rows_staged * n.rowbytes);
  w.off_pos = o;
  o += ws_align_up((size_t)n.streams * rows_staged * 4);
  w.total = o;
  return w;
}

// What the append asks of its caller before it takes rows that are not the fused kernels' (`tail` rows behind the sink).
bool append_ws_given(const Norm& n, int64_t q, int64_t tail, int64_t sb, int64_t sh, int64_t st, const void* ws,
                     size_t ws_bytes) {
  if (!staged_fits(n)) return false;
  return told_none(n, sb, sh, st) ||
         (ws && aligned_to(ws, 16) && ws_bytes >= append_ws(n, q, q * n.k + (tail - q * n.L)).total);
}

int hip_status(hipError_t e) { return e == hipSuccess ? LAGKV_OK : LAGKV_EHIP; }

void fill_pass(PassArgs* a, const Norm& n, const void* K, const void* V, int64_t T,
               const lagkv_plan_t& pl, int64_t sb, int64_t sh, int64_t st) {
  std::memset(a, 0, sizeof(*a));
  a->K = (const char*)K;
  a->V = (const char*)V;
  a->sb = sb;
  a->sh = sh;
  a->st = st;
  a->T = T;
  a->T_out = pl.T_out;
  a->n_s = pl.n_scored;
  a->B = n.B;
  a->H = n.H;
  a->D = n.D;
  a->S = n.S;
  a->L = n.L;
  a->k = n.k;
  a->esize = n.esize;
  a->f16 = n.f16;
  a->ddof = n.ddof;
  a->variant = n.variant;
  a->nseg = 1;
  a->nwaves = 4;
}

// The new rows of an EMPTY cache in one pass, where they complete chunks: no round of the recursion reads what another
// wrote (a chunk is scored against the raw rows behind it), so all of them run side by side through the one-shot
// kernels, whose outputs go straight to their places in the cache (T_out is the distance from one stream's to the
// next's).  Only kernels that subtract as exactly as the single-round kernels these calls otherwise go to; LAGKV_ESHAPE
// where there is none, or where rows and cache overlap.
int fill_empty_cache(const Norm& n, lagkv_cache* c, const void* K, const void* V, int64_t T, int64_t sb, int64_t sh,
                     int64_t st, hipStream_t s) {
  lagkv_plan_t pl;
  plan_of(n, T, n.S, &pl);
  if (pl.n_scored < 1 || c->n_seen || c->n_static || c->n_tail) return LAGKV_ESHAPE;
  if (n.hint.path != LAGKV_PATH_AUTO || n.hint.waves || n.hint.nseg || n.hint.order || n.hint.sel) return LAGKV_ESHAPE;
  const int64_t held = n.streams * c->capacity * n.rowbytes, span = (n.B - 1) * sb + (n.H - 1) * sh + (T - 1) * st + n.rowbytes;
  for (const void* from : {K, V})
    for (const void* to : {c->K, c->V})
      if ((const char*)from < (const char*)to + held && (const char*)to < (const char*)from + span) return LAGKV_ESHAPE;
  PassArgs a;
  fill_pass(&a, n, K, V, T, pl, sb, sh, st);
  a.K_out = (char*)c->K;
  a.V_out = (char*)c->V;
  a.idx_out = c->pos;
  a.T_out = c->capacity;
  const bool whole = shape_fused(n, sb, sh, st) && fused_fits(n) &&
                     fused_supported(n.D, n.esize, sb, sh, st, K, V, c->K, c->V);
  const int64_t chunks = n.streams * pl.n_scored;
  int rc = LAGKV_ESHAPE;
  if (whole && n.variant != LAGKV_SCORE_L2 && ring_supported(n.D, n.esize, n.L, st) && chunks < (1LL << 31)) {
    const int64_t places = ring_places(n.D, n.esize, n.L);
    a.walks = chunks < places ? chunks : places;
    if (grid_fits(a.walks + most_edge_workgroups(a), ring_threads(n.D, n.esize, n.L)))
      rc = launch_ring_pass(a, s) == hipSuccess ? LAGKV_OK : LAGKV_EHIP;
  } else if (use_chunk(n, a, whole && n.variant == LAGKV_SCORE_L2)) {
    rc = launch_chunk(a, n, whole, s);
  } else if (whole && (n.variant == LAGKV_SCORE_L2 || !chunk_supported(n.D, n.esize, n.L, st))) {
    a.nwaves = split_nw(n);  // (which takes its means as the general append kernel does)
    a.nseg = pick_segments_split(n, a.n_s, a.nwaves);
    rc = launch_in_parts(a, 64 * a.nwaves, launch_split_pass, s);
  }
  if (rc != LAGKV_OK) return rc;
  c->n_seen = T;
  c->n_static = n.S + (int64_t)n.k * pl.n_scored;
  c->n_tail = pl.T_out - c->n_static;
  return LAGKV_OK;
}

}  // namespace

extern "C" {

int lagkv_plan(const lagkv_params* p, int64_t T, int64_t n_static, lagkv_plan_t* out) {
  Norm n;
  int rc = validate(p, &n);
  if (rc != LAGKV_OK) return rc;
  if (!out) return LAGKV_EINVAL;
  if (T < 0 || T > kMaxRows) return LAGKV_ESHAPE;
  if (n_static < 0) n_static = n.S;
  if (n_static > T && T >= n.S) return LAGKV_EINVAL;
  plan_of(n, T, n_static, out);
  return LAGKV_OK;
}

int lagkv_keep_for_compression(int64_t T, int32_t S, int32_t L, double C, int64_t* k_out,
                               double* r_out) {
  if (!k_out || !r_out || S < 0 || L < 1 || !(C >= 0.0) || !(C < 1.0)) return LAGKV_EINVAL;
  if (T < (int64_t)S + 2 * (int64_t)L) return LAGKV_EINVAL;
  const int64_t n_s = (T - S) / L - 1, m = (T - S) % L;
  // Eq. 12-13 with rL = k: C(k) = 1 - (S + k*n_s + L + m) / T, decreasing in k.  Start from the
  // closed form and settle the boundary with the exact comparison the definition uses.
  auto ratio = [&](int64_t k) { return 1.0 - (double)(S + k * n_s + L + m) / (double)T; };
  int64_t k = (int64_t)std::floor(((1.0 - C) * (double)T - (double)(S + L + m)) / (double)n_s);
  if (k > L) k = L;
  if (k < 1) k = 1;
  while (k < L && ratio(k + 1) >= C) ++k;
  while (k >= 1 && ratio(k) < C) --k;
  if (k < 1) return LAGKV_EINVAL;
  *k_out = k;
  *r_out = k == L ? 1.0 : ((double)k + 0.5) / (double)L;
  return LAGKV_OK;
}

size_t lagkv_workspace_bytes(const lagkv_params* p, int64_t T) {
  Norm n;
  if (validate(p, &n) != LAGKV_OK || T < 1 || T > kMaxRows) return 0;
  int64_t sb, sh, st;
  if (strides_of(p, n, T, &sb, &sh, &st) != LAGKV_OK) return 0;
  if (told_none(n, sb, sh, st)) return 0;
  // one pass over T rows, and an append into a cache of capacity T
  lagkv_plan_t pl;
  plan_of(n, T, n.S, &pl);
  const size_t pass = staged_ws(n, pl.n_scored > 0 ? pl.n_scored : 1, true).total;
  const size_t app = append_ws(n, T / n.L + 1, T).total;
  return pass > app ? pass : app;
}

int lagkv_score(const lagkv_params* p, const void* K, const void* V, int64_t T, float* scores,
                void* ws, size_t ws_bytes, void* hip_stream) {
  (void)ws;  // no path stages anything for the scores alone
  (void)ws_bytes;
  Norm n;
  int rc = validate(p, &n);
  if (rc != LAGKV_OK) return rc;
  if (T < 1 || T > kMaxRows) return LAGKV_ESHAPE;
  if (!K || (!V && n.variant != LAGKV_SCORE_L2)) return LAGKV_EINVAL;
  if (!aligned_to(K, n.esize) || !aligned_to(V, n.esize)) return LAGKV_EINVAL;
  int64_t sb, sh, st;
  rc = strides_of(p, n, T, &sb, &sh, &st);
  if (rc != LAGKV_OK) return rc;
  lagkv_plan_t pl;
  plan_of(n, T, n.S, &pl);
  if (pl.n_scored == 0) return LAGKV_OK;
  if (!scores) return LAGKV_EINVAL;
  hipStream_t s = (hipStream_t)hip_stream;
  PassArgs a;
  fill_pass(&a, n, K, V, T, pl, sb, sh, st);
  a.scores = scores;
  const int force = n.hint.path;
  const bool fused_ok = shape_fused(n, sb, sh, st) && fused_fits(n) &&
                        fused_supported(n.D, n.esize, sb, sh, st, K, V, nullptr, nullptr);
  if ((force == LAGKV_PATH_FUSED || force == LAGKV_PATH_RESIDENT) && !fused_ok) return LAGKV_ESHAPE;
  if (fused_ok && force != LAGKV_PATH_STAGED) return launch_fused_any(a, n, s);
  if (!staged_fits(n)) return LAGKV_ESHAPE;
  if (use_chunk(n, a, false)) return launch_chunk(a, n, false, s);
  return hip_status(launch_staged_score(a, n.S, scores, s));
}

int lagkv_select(const lagkv_params* p, const float* scores, int64_t T, int32_t* kept,
                 void* hip_stream) {
  Norm n;
  int rc = validate(p, &n);
  if (rc != LAGKV_OK) return rc;
  if (T < 1 || T > kMaxRows) return LAGKV_ESHAPE;
  lagkv_plan_t pl;
  plan_of(n, T, n.S, &pl);
  if (pl.n_scored == 0) return LAGKV_OK;
  if (!scores || !kept) return LAGKV_EINVAL;
  if (((size_t)n.L + n.k) * 4 > (size_t)kMaxLdsBytes) return LAGKV_ESHAPE;
  return hip_status(launch_select(scores, n.streams, pl.n_scored, n.L, n.k, n.S, kept,
                                  (hipStream_t)hip_stream));
}

int lagkv_compress(const lagkv_params* p, const void* K, const void* V, int64_t T, void* K_out,
                   void* V_out, int32_t* idx_out, float* scores_out, void* ws, size_t ws_bytes,
                   void* hip_stream) {
  return lagkv::compress_with_workspace(p, K, V, T, K_out, V_out, idx_out, scores_out, ws, ws_bytes,
                                        hip_stream);
}

}  // extern "C"

// Workspace one lagkv_compress call needs (0: the fused kernels serve it, or the parameters
// are invalid and the call itself will say so).
size_t lagkv::compress_workspace_need(const lagkv_params* p, int64_t T) {
  Norm n;
  if (validate(p, &n) != LAGKV_OK || T < 1 || T > kMaxRows) return 0;
  int64_t sb, sh, st;
  if (strides_of(p, n, T, &sb, &sh, &st) != LAGKV_OK) return 0;
  if (told_none(n, sb, sh, st)) return 0;
  lagkv_plan_t pl;
  plan_of(n, T, n.S, &pl);
  return pl.n_scored > 0 ? staged_ws(n, pl.n_scored, true).total : 0;
}

// The whole pass with the workspace given by the caller (lagkv_compress) or taken from the
// library's static scratch (lagkv_compress_static).
int lagkv::compress_with_workspace(const lagkv_params* p, const void* K, const void* V, int64_t T,
                                   void* K_out, void* V_out, int32_t* idx_out, float* scores_out,
                                   void* ws, size_t ws_bytes, void* hip_stream) {
  Norm n;
  int rc = validate(p, &n);
  if (rc != LAGKV_OK) return rc;
  if (T < 1 || T > kMaxRows) return LAGKV_ESHAPE;
  if (!K || !V || !K_out || !V_out) return LAGKV_EINVAL;
  if (!aligned_to(K, n.esize) || !aligned_to(V, n.esize) || !aligned_to(K_out, n.esize) ||
      !aligned_to(V_out, n.esize))
    return LAGKV_EINVAL;
  int64_t sb, sh, st;
  rc = strides_of(p, n, T, &sb, &sh, &st);
  if (rc != LAGKV_OK) return rc;
  lagkv_plan_t pl;
  plan_of(n, T, n.S, &pl);
  hipStream_t s = (hipStream_t)hip_stream;
  if (pl.n_scored == 0) {  // nothing to compress: the output is the input
    const int64_t osh = T * n.rowbytes, osb = osh * n.H;
    hipError_t e = launch_copy_rows((const char*)K, sb, sh, st, (char*)K_out, osb, osh, n.rowbytes,
                                    n.B, n.H, T, n.rowbytes, s);
    if (e == hipSuccess)
      e = launch_copy_rows((const char*)V, sb, sh, st, (char*)V_out, osb, osh, n.rowbytes, n.B, n.H,
                           T, n.rowbytes, s);
    if (e == hipSuccess && idx_out) e = launch_iota_rows(idx_out, n.streams, T, 0, T, 0, s);
    return hip_status(e);
  }
  PassArgs a;
  fill_pass(&a, n, K, V, T, pl, sb, sh, st);
  a.K_out = (char*)K_out;
  a.V_out = (char*)V_out;
  a.idx_out = idx_out;
  a.scores = scores_out;
  const int force = n.hint.path;
  const bool fused_ok = shape_fused(n, sb, sh, st) && fused_fits(n) &&
                        fused_supported(n.D, n.esize, sb, sh, st, K, V, K_out, V_out);
  if ((force == LAGKV_PATH_FUSED || force == LAGKV_PATH_RESIDENT) && !fused_ok) return LAGKV_ESHAPE;
  if (fused_ok && force != LAGKV_PATH_STAGED) return launch_fused_any(a, n, s);
  if (!staged_fits(n)) return LAGKV_ESHAPE;
  const CompressWs w = staged_ws(n, pl.n_scored, scores_out == nullptr);
  const bool chunk = use_chunk(n, a, false);
  if (!(chunk && told_none(n, sb, sh, st)) && (!ws || ws_bytes < w.total || !aligned_to(ws, 16)))
    return LAGKV_EWORKSPACE;
  if (chunk) return launch_chunk(a, n, false, s);
  float* sc = scores_out ? scores_out : (float*)((char*)ws + w.off_scores);
  int32_t* kept = (int32_t*)((char*)ws + w.off_kept);
  hipError_t e = launch_staged_score(a, n.S, sc, s);
  if (e == hipSuccess) e = launch_select(sc, n.streams, pl.n_scored, n.L, n.k, n.S, kept, s);
  if (e == hipSuccess) e = launch_staged_gather(a, kept, s);
  return hip_status(e);
}

extern "C" {

int lagkv_cache_after_compress(const lagkv_params* p, int64_t T, lagkv_cache* c) {
  Norm n;
  int rc = validate(p, &n);
  if (rc != LAGKV_OK) return rc;
  if (!c) return LAGKV_EINVAL;
  if (T < 0 || T > kMaxRows) return LAGKV_ESHAPE;
  lagkv_plan_t pl;
  plan_of(n, T, n.S, &pl);
  if (c->capacity < pl.T_out) return LAGKV_ECAPACITY;
  // Eq. 12: the output is [sink | k rows per scored chunk | last chunk + remainder]
  c->n_static = pl.n_scored > 0 ? n.S + (int64_t)n.k * pl.n_scored : (T < n.S ? T : n.S);
  c->n_tail = pl.T_out - c->n_static;
  c->n_seen = T;
  return LAGKV_OK;
}

int64_t lagkv_prefill_rows(const lagkv_params* p, const lagkv_cache* c, int64_t rows_left) {
  Norm n;
  if (validate(p, &n) != LAGKV_OK || !c || rows_left <= 0) return 0;
  const int64_t want = c->n_seen == 0 ? (int64_t)n.S + 2 * (int64_t)n.L : (int64_t)n.L;
  return rows_left < want ? rows_left : want;
}

int lagkv_append_and_compress(const lagkv_params* p, lagkv_cache* c, const void* K_new,
                              const void* V_new, int64_t n_new, void* ws, size_t ws_bytes,
                              void* hip_stream) {
  Norm n;
  int rc = validate(p, &n);
  if (rc != LAGKV_OK) return rc;
  if (!c || !c->K || !c->V) return LAGKV_EINVAL;
  if (n_new < 0 || c->capacity < 1 || c->n_static < 0 || c->n_tail < 0 || c->n_seen < 0)
    return LAGKV_EINVAL;
  if (n_new > 0 && (!K_new || !V_new)) return LAGKV_EINVAL;
  if (c->capacity > kMaxRows || c->n_seen + n_new > kMaxRows) return LAGKV_ESHAPE;
  if (!aligned_to(c->K, n.esize) || !aligned_to(c->V, n.esize) || !aligned_to(K_new, n.esize) ||
      !aligned_to(V_new, n.esize))
    return LAGKV_EINVAL;
  const int64_t held = c->n_static + c->n_tail;
  if (held + n_new > c->capacity) return LAGKV_ECAPACITY;
  int64_t sb = 0, sh = 0, st = 0;
  if (n_new > 0) {
    rc = strides_of(p, n, n_new, &sb, &sh, &st);
    if (rc != LAGKV_OK) return rc;
  }
  // host arithmetic of the recursion: the sink fills first, then the tail is cut
  // into L-chunks and all but the last full one are compressed
  const int64_t total = held + n_new;
  int64_t base = c->n_static;
  if (c->n_seen < n.S) {
    const int64_t seen = c->n_seen + n_new;
    base = seen < n.S ? seen : n.S;
  }
  const int64_t tail = total - base;
  const int64_t q = tail >= 2 * (int64_t)n.L ? tail / n.L - 1 : 0;
  hipStream_t s = (hipStream_t)hip_stream;
  const int force = n.hint.path;
  const bool fused_ok = shape_fused(n, sb, sh, st) && fused_fits(n) &&
                        fused_supported(n.D, n.esize, sb, sh, st, c->K, c->V, K_new, V_new);
  if ((force == LAGKV_PATH_FUSED || force == LAGKV_PATH_RESIDENT) && !fused_ok) return LAGKV_ESHAPE;
  if (q > 1 && total == n_new && (fused_ok || append_ws_given(n, q, tail, sb, sh, st, ws, ws_bytes))) {
    rc = fill_empty_cache(n, c, K_new, V_new, n_new, sb, sh, st, s);
    if (rc != LAGKV_ESHAPE) return rc;
  }
  hipError_t e = hipSuccess;
  AppendArgs a;
  std::memset(&a, 0, sizeof(a));
  a.K = (char*)c->K;
  a.V = (char*)c->V;
  a.pos = c->pos;
  a.K_new = (const char*)K_new;
  a.V_new = (const char*)V_new;
  a.nsb = sb;
  a.nsh = sh;
  a.nst = st;
  a.capacity = c->capacity;
  a.n_static = c->n_static;
  a.n_tail = c->n_tail;
  a.n_seen = c->n_seen;
  a.n_new = n_new;
  a.rounds = q;
  a.B = n.B;
  a.H = n.H;
  a.D = n.D;
  a.S = n.S;
  a.L = n.L;
  a.k = n.k;
  a.esize = n.esize;
  a.f16 = n.f16;
  a.ddof = n.ddof;
  a.variant = n.variant;
  a.sel = n.hint.sel;
  // the kernels for 4-byte aligned rows, unless a launch is asked for
  const bool free_launch = force == LAGKV_PATH_AUTO && n.hint.waves == 0 && n.hint.sel == 0;
  const bool a4 = free_launch && !((sb | sh | st | n.rowbytes) & 3) && aligned_to(c->K, 4) && aligned_to(c->V, 4) &&
                  aligned_to(K_new, 4) && aligned_to(V_new, 4);
  if (fused_ok && force != LAGKV_PATH_STAGED) {
    if (n_new > 0 || q > 0) {
      a.nwaves = pick_waves(n);
      if (a4 && append_rows_supported(a)) e = launch_append_rows(a, s);
      else if (a4 && round_is_faster(n, a, tail)) e = launch_append_round(a, s);
      else if (n.hint.waves == 0 && decode_step_supported(a)) e = launch_decode_step(a, s);
      else e = launch_fused_append(a, s);
    }
  } else {
    if (!staged_fits(n)) return LAGKV_ESHAPE;
    const int64_t rows_staged = q > 0 ? q * n.k + (tail - q * n.L) : 0;
    const AppendWs w = append_ws(n, q, rows_staged);
    const bool round = a4 && append_round_supported(a), rows = a4 && append_rows_supported(a);
    if (q > 0 && !(round && told_none(n, sb, sh, st)) && (!ws || ws_bytes < w.total || !aligned_to(ws, 16)))
      return LAGKV_EWORKSPACE;
    const int64_t csh = c->capacity * n.rowbytes, csb = csh * n.H;
    if (round) {
      e = launch_append_round(a, s);
    } else if (n_new > 0 && rows) {
      e = launch_append_rows(a, s);
    } else if (n_new > 0) {
      e = launch_copy_rows((const char*)K_new, sb, sh, st, (char*)c->K + held * n.rowbytes, csb, csh,
                           n.rowbytes, n.B, n.H, n_new, n.rowbytes, s);
      if (e == hipSuccess)
        e = launch_copy_rows((const char*)V_new, sb, sh, st, (char*)c->V + held * n.rowbytes, csb,
                             csh, n.rowbytes, n.B, n.H, n_new, n.rowbytes, s);
      if (e == hipSuccess && c->pos)
        e = launch_iota_rows(c->pos, n.streams, c->capacity, held, n_new, (int32_t)c->n_seen, s);
    }
    if (e == hipSuccess && q > 0 && !round) {
      char* wsb = (char*)ws;
      float* sc = (float*)(wsb + w.off_scores);
      int32_t* kept = (int32_t*)(wsb + w.off_kept);
      PassArgs a;
      lagkv_plan_t pl;
      pl.n_chunks = q + 1;
      pl.n_scored = q;
      pl.rem = 0;
      pl.k = n.k;
      pl.T_out = rows_staged;
      fill_pass(&a, n, c->K, c->V, total, pl, csb, csh, n.rowbytes);
      e = launch_staged_score(a, base, sc, s);
      if (e == hipSuccess) e = launch_select(sc, n.streams, q, n.L, n.k, base, kept, s);
      GatherMap m;
      m.n_pre = 0;
      m.pre0 = 0;
      m.n_kept = q * n.k;
      m.post0 = base + q * n.L;
      m.n_out = rows_staged;
      const int64_t ssh = rows_staged * n.rowbytes, ssb = ssh * n.H;
      if (e == hipSuccess)
        e = launch_gather_rows((const char*)c->K, csb, csh, n.rowbytes, n.B, n.H, wsb + w.off_k,
                               n.rowbytes, n.esize, kept, nullptr, m, s);
      if (e == hipSuccess)
        e = launch_gather_rows((const char*)c->V, csb, csh, n.rowbytes, n.B, n.H, wsb + w.off_v,
                               n.rowbytes, n.esize, kept, nullptr, m, s);
      if (e == hipSuccess)
        e = launch_copy_rows(wsb + w.off_k, ssb, ssh, n.rowbytes, (char*)c->K + base * n.rowbytes,
                             csb, csh, n.rowbytes, n.B, n.H, rows_staged, n.rowbytes, s);
      if (e == hipSuccess)
        e = launch_copy_rows(wsb + w.off_v, ssb, ssh, n.rowbytes, (char*)c->V + base * n.rowbytes,
                             csb, csh, n.rowbytes, n.B, n.H, rows_staged, n.rowbytes, s);
      if (e == hipSuccess && c->pos) {
        // positions are a [streams, capacity] tensor of one 4-byte channel
        e = launch_gather_rows((const char*)c->pos, c->capacity * 4 * n.H, c->capacity * 4, 4, n.B,
                               n.H, wsb + w.off_pos, 4, 4, kept, nullptr, m, s);
        if (e == hipSuccess)
          e = launch_copy_rows(wsb + w.off_pos, rows_staged * 4 * n.H, rows_staged * 4, 4,
                               (char*)c->pos + base * 4, c->capacity * 4 * n.H, c->capacity * 4, 4,
                               n.B, n.H, rows_staged, 4, s);
      }
    }
  }
  if (e != hipSuccess) return LAGKV_EHIP;
  c->n_seen += n_new;
  c->n_static = base + q * n.k;
  c->n_tail = tail - q * n.L;
  return LAGKV_OK;
}

int lagkv_prefill(const lagkv_params* p, lagkv_cache* c, const void* K, const void* V, int64_t T, void* ws,
                  size_t ws_bytes, void* hip_stream, int64_t* calls) {
  if (calls) *calls = 0;
  Norm n;
  int rc = validate(p, &n);
  if (rc != LAGKV_OK) return rc;
  if (!c || !c->K || !c->V || T < 0 || (T > 0 && (!K || !V))) return LAGKV_EINVAL;
  if (T == 0) return LAGKV_OK;
  int64_t sb, sh, st;
  rc = strides_of(p, n, T, &sb, &sh, &st);
  if (rc != LAGKV_OK) return rc;
  // the rows that the longest of the calls would hold: S + 2L, then k more with every lag, or the last, partial one
  const int64_t first = n.S + 2 * (int64_t)n.L, full = (T - first) / n.L, rem = (T - first) % n.L;
  if (T >= first && T <= kMaxRows && c->capacity <= kMaxRows && c->capacity >= first + full * n.k &&
      c->capacity >= n.S + (full + 1) * n.k + n.L + rem && aligned_to(K, n.esize) && aligned_to(V, n.esize) &&
      aligned_to(c->K, n.esize) && aligned_to(c->V, n.esize)) {
    const bool fused_ok = shape_fused(n, sb, sh, st) && fused_fits(n) &&
                          fused_supported(n.D, n.esize, sb, sh, st, c->K, c->V, K, V);
    if (fused_ok || append_ws_given(n, 1, 2 * (int64_t)n.L, sb, sh, st, ws, ws_bytes)) {
      rc = fill_empty_cache(n, c, K, V, T, sb, sh, st, (hipStream_t)hip_stream);
      if (rc == LAGKV_OK && calls) *calls = 1 + full + (rem > 0);
      if (rc != LAGKV_ESHAPE) return rc;
    }
  }
  lagkv_params q = *p;
  q.stride_b = sb / n.esize;
  q.stride_h = sh / n.esize;
  q.stride_t = st / n.esize;
  for (int64_t t = 0; t < T;) {
    const int64_t rows = lagkv_prefill_rows(&q, c, T - t);
    rc = lagkv_append_and_compress(&q, c, (const char*)K + t * st, (const char*)V + t * st, rows, ws, ws_bytes, hip_stream);
    if (rc != LAGKV_OK) return rc;
    t += rows;
    if (calls) ++*calls;
  }
  return LAGKV_OK;
}

int32_t lagkv_launch_hint(int path, int waves, int segments) {
  if (path < 0 || path > LAGKV_PATH_RESIDENT || segments < 0 || segments > kMaxSegments) return -1;
  if (waves != 0 && waves != 1 && waves != 2 && waves != 4 && waves != 8) return -1;
  return (int32_t)(path | (waves << kHintWavesShift) | (segments << kHintSegShift));
}

int32_t lagkv_launch_hint_ex(int path, int waves, int segments, int order, int select) {
  const int32_t base = lagkv_launch_hint(path, waves, segments);
  if (base < 0 || order < 0 || order > LAGKV_ORDER_BITREV || select < 0 || select > LAGKV_SELECT_GROUP)
    return -1;
  return base | (order << kHintOrderShift) | (select << kHintSelShift);
}

int lagkv_path_for(const lagkv_params* p, int64_t T) {
  Norm n;
  int rc = validate(p, &n);
  if (rc != LAGKV_OK) return -rc;
  if (T < 1 || T > kMaxRows) return -LAGKV_ESHAPE;
  int64_t sb, sh, st;
  rc = strides_of(p, n, T, &sb, &sh, &st);
  if (rc != LAGKV_OK) return -rc;
  const int force = n.hint.path;
  const bool fused_ok = shape_fused(n, sb, sh, st) && fused_fits(n);
  if ((force == LAGKV_PATH_FUSED || force == LAGKV_PATH_RESIDENT) && !fused_ok) return -LAGKV_ESHAPE;
  if (fused_ok && force != LAGKV_PATH_STAGED) {
    if (use_resident(n)) return LAGKV_PATH_RESIDENT;
    return force == LAGKV_PATH_RESIDENT ? -LAGKV_ESHAPE : LAGKV_PATH_FUSED;
  }
  return staged_fits(n) ? LAGKV_PATH_STAGED : -LAGKV_ESHAPE;
}

const char* lagkv_kernel_for(const lagkv_params* p, int64_t T) {
  const int path = lagkv_path_for(p, T);
  if (path < 0) return nullptr;
  Norm n;
  int64_t sb, sh, st;
  if (validate(p, &n) != LAGKV_OK || strides_of(p, n, T, &sb, &sh, &st) != LAGKV_OK) return nullptr;
  lagkv_plan_t pl;
  plan_of(n, T, n.S, &pl);
  if (pl.n_scored == 0) return "copy_rows_kernel";
  PassArgs a;
  fill_pass(&a, n, nullptr, nullptr, T, pl, sb, sh, st);
  alignas(16) char out[16];  // (a call with outputs; nothing is stored)
  a.K_out = a.V_out = out;
  const bool whole = path != LAGKV_PATH_STAGED;
  const bool chunk = use_chunk(n, a, whole);
  if (whole ? use_ring(n, a, chunk) : chunk && use_direct(n, a)) return "ring_pass_kernel";
  if (chunk) return "chunk_pass_kernel";
  return path == LAGKV_PATH_RESIDENT ? "hold_pass_kernel" : path == LAGKV_PATH_FUSED ? "split_pass_kernel" : "staged_score_kernel";
}

const char* lagkv_strerror(int status) {
  switch (status) {
    case LAGKV_OK: return "ok";
    case LAGKV_EINVAL: return "invalid argument (null pointer, r outside (0,1], floor(r*L) < 1, S < 0, L < 1, misaligned pointer)";
    case LAGKV_ESHAPE: return "unsupported or inconsistent shape, stride or size";
    case LAGKV_EDTYPE: return "unknown dtype or scoring variant";
    case LAGKV_ECAPACITY: return "cache capacity too small for the appended rows";
    case LAGKV_EWORKSPACE: return "workspace missing, misaligned or smaller than lagkv_workspace_bytes()";
    case LAGKV_EHIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

int lagkv_version(void) { return 200; }

}  // extern "C"
