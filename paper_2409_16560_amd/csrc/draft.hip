// Draft stage (Section 3.1 "Overview" / "Details"): one beam-sampling step of the small model, and the layout of
// the sampled layers as a draft forest.
//
// dsbd_draft_layer: W_S independent draws from q_beam = T o q/Q over (beams of the current layer) x V, by inverse CDF
// in flat order.  Two dependent passes:
//   1. take_chunks: every row is cut into chunks; a chunk's maximum and its fp64 sum of exponentials against that maximum;
//   2. draw_one (a workgroup per draw) or, with warping, draw_warped (a workgroup per prompt): the row totals and beam weights
//      out of the chunks' pairs, which every workgroup folds for itself in the same order, and then only the chunks that
//      matter are read again: the one that holds the draw, or those that can hold one of the top_k leading entries.
// One launch: the second pass's workgroups stand behind the first's and wait for the pairs in tagged slots (two launches
// under capture, for more than DR_WAITING of them, and where the chunks are long to stream: DR_ONE_*).
// What bounds a step is the chain of dependent memory round trips (8 MB of logits are 1.6 us at HBM rate).  Measured, 16
// beams x 128256 tokens, 16 draws, top_k 10 / top_p 0.8: 5.7 + 11.4 us in two kernels, 16.1 in one; 64 beams of eight prompts x
// 32000, 8 draws each, no warping: 6.0 + 6.6 and 12.0 us.  The rest of the gain is the host's: a launch less is 3 us.
//
// dsbd_build_forest: one workgroup per prompt turns the layers' (parent row, token) lists into the
// tree-contiguous layout the other calls expect.
#include "common.h"
#include "exp_nonpos.h"
#include "slots.h"
#include "wave_f64.h"
#include <float.h>
#include <limits.h>

#define DC_BLOCK 256           // chunk kernel
#define DD_BLOCK 512           // draw kernel
#define DW_BLOCK 1024          // warped kernel
#define DW_WAVES (DW_BLOCK / 64)
#define DR_MAX_CHUNKS 64       // chunks per row: one per lane
#define DR_K_MAX 32
#define DR_WAITING 256         // most workgroups that wait behind the chunks in one launch
#define DR_ONE_WARPED (3LL << 20)    // most logits of a step in one launch, with warping ...
#define DR_ONE_PLAIN (12LL << 20)    // ... and without
#define DR_WAIT_TICKS 20000    // 200 us of the 100 MHz wall clock: how long a wave waits for a chunk before it takes it itself
#define DW_CAND 1024           // candidates the warped kernel ranks directly
#define DW_DIGIT 11            // bits per pass of its radix selection
#define BF_BLOCK 512
#define BF_NODE_CAP 512

namespace {

__constant__ double c_draft_exp2_tab[64] = {DSBD_EXP2_TABLE_64};

struct DraftArgs {
  int n_prompts, n_beams, max_prompt_beams, V, W_S;
  int chunk, nchunk;           // logits per chunk, chunks per row
  const int32_t* beam_off;
  const float* z;
  const double* cum;
  const float* u;
  double2* part;               // [n_beams][nchunk]: maximum of the chunk, sum of exp(z - maximum) ...
  Slot* slots;                 // ... or, in one launch, [n_beams][nchunk][2]: the two in tagged slots
  unsigned long long tag;
  long long wait_limit;        // of every wait for a slot, in ticks of the 100 MHz wall clock
  int chunk_wgs;               // one launch: the workgroups that take chunks; those behind them draw
  int top_k;
  float top_p;
  int32_t *out_parent, *out_token;
  double* out_logp;
  int32_t* fault;
};

// ---- pass 1 (bound by a round trip to HBM, the maximum's barrier and fp64 exponentials; 2048-logit chunks at 16 x 128256
// give 1008 workgroups, 4.4 us at best): NPT logits per thread and tile stay in registers between the maximum and the exponentials; chunks of
// more than one tile (vocabularies above 262144 tokens) merge their tiles as they go.  Loads of 4 bytes per lane: a
// row of an odd vocabulary starts anywhere, and 8 MB do not ask for more.
// A workgroup of BLOCK threads takes BLOCK / DC_BLOCK chunks; ONE: their results go into slots for workgroups that wait.
template <int NPT, int BLOCK, bool ONE>
__device__ __forceinline__ void take_chunks(const DraftArgs& a, int wg) {
  constexpr int W = DC_BLOCK / 64;
  __shared__ double tab[64];
  __shared__ float wmax[BLOCK / 64];
  __shared__ double wsum[BLOCK / 64];
  const int group = BLOCK == DC_BLOCK ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / DC_BLOCK);
  const int tid = threadIdx.x % DC_BLOCK, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, first = group * W;
  const long long n_items = (long long)a.n_beams * a.nchunk, item_raw = (long long)wg * (BLOCK / DC_BLOCK) + group;
  const long long item = item_raw < n_items ? item_raw : n_items - 1;      // (the last workgroup may have threads left over)
  const int row = (int)(item / a.nchunk), c = (int)(item - (long long)row * a.nchunk);
  const float* const z = a.z + (long long)row * a.V;
  const int x_lo = c * a.chunk, x_end = min(a.V, x_lo + a.chunk);
  if (threadIdx.x < 64) tab[threadIdx.x] = c_draft_exp2_tab[threadIdx.x];
  float M = -INFINITY;
  double S = 0.0;
  bool bad = false;
  for (int i = 0; i < a.chunk; i += NPT * DC_BLOCK) {       // (as often in every chunk: there are barriers inside)
    const int x0 = min(x_lo + i, x_end);
    float v[NPT];
#pragma unroll
    for (int k = 0; k < NPT; ++k) v[k] = z[min(x0 + k * DC_BLOCK + tid, x_end - 1)];     // (clamped repeats leave a maximum alone)
    float m = -INFINITY;
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      m = fmaxf(m, v[k]);
      bad |= !(v[k] <= FLT_MAX);                     // NaN or +Inf (-Inf: a masked token, probability 0)
    }
    m = wave_max_f32(m);
    __syncthreads();                                 // (the table; and the tile before has read its totals)
    if (lane == 0) wmax[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(wmax[first], wmax[first + 1]), fmaxf(wmax[first + 2], wmax[first + 3]));
    const double ref = m == -INFINITY ? 0.0 : (double)m;       // a tile masked whole adds 0
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      const double e = dsbd_exp_nonpos((double)v[k] - ref, tab);
      s += x0 + k * DC_BLOCK + tid < x_end ? e : 0.0;
    }
    s = wave_sum(s);
    if (lane == 0) wsum[wave] = s;
    __syncthreads();
    s = (wsum[first] + wsum[first + 1]) + (wsum[first + 2] + wsum[first + 3]);
    if (m > -INFINITY) {
      const float Mn = fmaxf(M, m);
      S = (M > -INFINITY ? S * dsbd_exp_nonpos((double)M - (double)Mn, tab) : 0.0) + s * dsbd_exp_nonpos((double)m - (double)Mn, tab);
      M = Mn;
    }
  }
  if (bad) atomicOr(a.fault, DSBD_FAULT_NONFINITE);
  if (item_raw >= n_items) return;
  if constexpr (ONE) {
    if (tid < 2) slot_post(a.slots + item * 2 + tid, tid ? S : (double)M, a.tag);
  } else {
    if (tid == 0) a.part[item] = make_double2((double)M, S);
  }
}

template <int NPT>
__global__ __launch_bounds__(DC_BLOCK) void draft_chunk_kernel(DraftArgs a) { take_chunks<NPT, DC_BLOCK, false>(a, blockIdx.x); }

// A prompt's rows.  False: no usable beams (out of range or none); `bad` gets the fault bits.
__device__ __forceinline__ bool prompt_rows(const DraftArgs& a, int p, int& r0, int& n, int& bad) {
  r0 = a.beam_off[p];
  const int r1 = a.beam_off[p + 1];
  n = r1 - r0;
  if (p == 0 && r0 != 0) bad |= DSBD_FAULT_TOPOLOGY;
  if (p == a.n_prompts - 1 && r1 != a.n_beams) bad |= DSBD_FAULT_TOPOLOGY;
  if (r0 < 0 || r1 > a.n_beams || n < 0) { bad |= DSBD_FAULT_TOPOLOGY; n = 0; }
  if (n > a.max_prompt_beams || n > 64) { bad |= DSBD_FAULT_BOUNDS; n = 0; }
  return n > 0;
}

// A chunk by one wave, the same sums in the same order as take_chunks forms them with four: for a wave that has waited long
// enough for the chunk's own workgroup.
__device__ double2 chunk_alone(const DraftArgs& a, int row, int c, const double* tab) {
  const int lane = threadIdx.x & 63, npt = a.chunk >= 4096 ? 16 : a.chunk / DC_BLOCK;
  const float* const z = a.z + (long long)row * a.V;
  const int x_lo = c * a.chunk, x_end = min(a.V, x_lo + a.chunk);
  float M = -INFINITY;
  double S = 0.0;
  for (int x0 = x_lo; x0 < x_end; x0 += npt * DC_BLOCK) {
    float m = -INFINITY;
    for (int k = 0; k < npt * (DC_BLOCK / 64); ++k) m = fmaxf(m, z[min(x0 + k * 64 + lane, x_end - 1)]);
    m = wave_max_f32(m);
    const double ref = m == -INFINITY ? 0.0 : (double)m;
    double part[DC_BLOCK / 64];
#pragma unroll
    for (int w = 0; w < DC_BLOCK / 64; ++w) {
      double s = 0.0;
      for (int k = 0; k < npt; ++k) {
        const int x = x0 + k * DC_BLOCK + w * 64 + lane;
        const double e = dsbd_exp_nonpos((double)z[min(x, x_end - 1)] - ref, tab);
        s += x < x_end ? e : 0.0;
      }
      part[w] = wave_sum(s);
    }
    const double s = (part[0] + part[1]) + (part[2] + part[3]);
    if (m > -INFINITY) {
      const float Mn = fmaxf(M, m);
      S = (M > -INFINITY ? S * dsbd_exp_nonpos((double)M - (double)Mn, tab) : 0.0) + s * dsbd_exp_nonpos((double)m - (double)Mn, tab);
      M = Mn;
    }
  }
  return make_double2((double)M, S);
}

// What the chunks' pairs say about a prompt: every row's maximum, sum and scale (beam weight / sum, Section 2.1: the
// joint entry of token x is exp(z - max) * scale), folded by one wave per row, a chunk per lane, in a fixed order
// (equal rows give equal bits).  `each(row, lane's chunk maximum, its sum, row maximum, scale)` sees every chunk.
template <int WAVES, bool ONE, class Each>
__device__ __forceinline__ void fold_rows(const DraftArgs& a, int r0, int n, const double* tab, double* row_max,
                                          double* row_sum, double* row_scale, int& bad, Each&& each) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto pair = [&](int r) -> double2 {
    double2 ms = make_double2(-INFINITY, 0.0);
    const long long at = (long long)(r0 + r) * a.nchunk + lane;
    if constexpr (!ONE) {
      if (lane < a.nchunk) ms = a.part[at];
    } else {
      const bool have = lane >= a.nchunk || (a.wait_limit > 0 && slot_wait2(a.slots + at * 2, a.slots + at * 2 + 1, a.tag, ms.x, ms.y, a.wait_limit));
      for (unsigned long long missing = __ballot(!have); missing; missing &= missing - 1) {
        const int c = (int)__ffsll((long long)missing) - 1;
        const double2 own = chunk_alone(a, r0 + r, c, tab);
        if (lane == c) ms = own;
      }
    }
    return ms;
  };
  // the first rows' pairs are requested before anything else: their round trip runs beside the weights
  double2 first = make_double2(-INFINITY, 0.0);
  if (!ONE && wave < n) first = pair(wave);
  // beam weights = softmax of the stored likelihoods (Section 2.1), every wave for itself
  const double cm = lane < n ? a.cum[r0 + lane] : -INFINITY;
  const double top = wave_max_f64(cm);
  const bool lost = !(top > -INFINITY && top < INFINITY) || __ballot(lane < n && cm != cm) != 0ull;
  if (lost) bad |= DSBD_FAULT_NONFINITE;
  const double e = lane < n ? dsbd_exp_nonpos(cm - top, tab) : 0.0;
  const double w = e / wave_sum(e);
  for (int r = wave; r < n; r += WAVES) {
    const double2 ms = ONE || r != wave ? pair(r) : first;
    const double M = wave_max_f64(ms.x);
    double share = ms.x > -INFINITY ? ms.y * dsbd_exp_nonpos(ms.x - M, tab) : 0.0;
    const double S = wave_sum(share);
    // A row without a finite logit (or with one that is no number: the chunks have reported that) has no entries: its
    // beam is never continued, and the prompt's other beams keep their shares.  (Every wave sees rows of its own, so it
    // reports for itself.)
    const bool dead = !(S > 0.0 && S < INFINITY);
    if (dead && lane == 0) atomicOr(a.fault, DSBD_FAULT_NONFINITE);
    if (dead) share = 0.0;
    const double scale = dead ? 0.0 : __shfl(w, r) / S;
    if (lane == 0) { row_max[r] = M; row_sum[r] = S; row_scale[r] = scale; }
    each(r, ms.x, share, M, scale);
  }
}

__device__ __forceinline__ void write_draw(const DraftArgs& a, int p, int j, int row, int x, double M, double S) {
  const long long o = (long long)p * a.W_S + j;
  a.out_parent[o] = row;
  a.out_token[o] = x;
  a.out_logp[o] = a.cum[row] + ((double)a.z[(long long)row * a.V + x] - (M + log(S)));
}

__device__ __forceinline__ void write_no_draw(const DraftArgs& a, int p, int j) {
  const long long o = (long long)p * a.W_S + j;
  a.out_parent[o] = -1; a.out_token[o] = -1; a.out_logp[o] = 0.0;
}

// First lane whose inclusive prefix exceeds the target; rounding may leave none: then the last lane with mass.
__device__ __forceinline__ int first_above(double incl, double mass, double target) {
  const unsigned long long above = __ballot(incl > target);
  if (above) return (int)__ffsll((long long)above) - 1;
  const unsigned long long has = __ballot(mass > 0.0);
  return has ? 63 - __clzll((long long)has) : 0;
}

// ---- pass 2, no warping: one draw per workgroup, so that the draws' dependent round trips (pairs, chunk, group) run side
// by side; 6.6 us whatever the number of draws.
template <bool ONE>
__device__ __forceinline__ void draw_one(const DraftArgs& a, int wg) {
  __shared__ double tab[64];
  __shared__ double row_max[64], row_sum[64], row_scale[64], row_mass[64];
  __shared__ double pre[64 * DR_MAX_CHUNKS];       // inclusive prefixes of the chunks' masses inside their row
  __shared__ double group[64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int p = wg / a.W_S, j = wg - p * a.W_S;
  int r0, n, bad = 0;
  const bool any = prompt_rows(a, p, r0, n, bad);
  if (!any) {
    if (tid == 0) { write_no_draw(a, p, j); if (bad && j == 0) atomicOr(a.fault, bad); }
    return;
  }
  const double u = (double)a.u[(long long)p * a.W_S + j];
  if (tid < 64) tab[tid] = c_draft_exp2_tab[tid];
  __syncthreads();
  fold_rows<DD_BLOCK / 64, ONE>(a, r0, n, tab, row_max, row_sum, row_scale, bad,
                           [&](int r, double, double share, double, double scale) {
    const double incl = wave_inclusive_scan(share * scale);
    pre[r * DR_MAX_CHUNKS + lane] = incl;
    if (lane == 63) row_mass[r] = incl;
  });
  if (j == 0 && tid == 0 && bad) atomicOr(a.fault, bad);
  __syncthreads();
  // the row and the chunk that hold the draw (every wave finds them for itself)
  const double rm = lane < n ? row_mass[lane] : 0.0;
  const double rincl = wave_inclusive_scan(rm);
  const double target = u * __shfl(rincl, 63);
  const int r = min(first_above(rincl, rm, target), n - 1);
  double before = r > 0 ? __shfl(rincl, r - 1) : 0.0;
  const double cincl = pre[r * DR_MAX_CHUNKS + lane];
  double cprev = __shfl_up(cincl, 1);
  if (lane == 0) cprev = 0.0;
  const int c = min(first_above(before + cincl, cincl - cprev, target), a.nchunk - 1);
  before += c > 0 ? __shfl(cincl, c - 1) : 0.0;
  // the chunk in up to 64 groups of whole 64-entry rounds: the groups' sums, then the one group that holds the draw
  const float* const z = a.z + (long long)(r0 + r) * a.V;
  const int x_lo = c * a.chunk, x_hi = min(a.V, x_lo + a.chunk);
  const int glen = ((x_hi - x_lo + 63) / 64 + 63) / 64 * 64;
  const double M = row_max[r], scale = row_scale[r];
  for (int gr = wave; gr < 64; gr += DD_BLOCK / 64) {
    const int g_lo = x_lo + gr * glen, g_hi = min(x_hi, g_lo + glen);
    double s = 0.0;
    for (int x = g_lo + lane; x < g_hi; x += 64) s += dsbd_exp_nonpos((double)z[x] - M, tab);
    s = g_lo < g_hi ? wave_sum(s) * scale : 0.0;
    if (lane == 0) group[gr] = s;
  }
  __syncthreads();
  if (wave != 0) return;
  const double gs = group[lane];
  const double gincl = wave_inclusive_scan(gs);
  const int gr = first_above(before + gincl, gs, target);
  before += gr > 0 ? __shfl(gincl, gr - 1) : 0.0;
  const int g_lo = x_lo + gr * glen, g_hi = min(x_hi, g_lo + glen);
  int pick = -1, last = -1;
  for (int x0 = g_lo; x0 < g_hi && pick < 0; x0 += 64) {
    const double v = x0 + lane < g_hi ? dsbd_exp_nonpos((double)z[min(x0 + lane, g_hi - 1)] - M, tab) * scale : 0.0;
    const double incl = wave_inclusive_scan(v);
    const unsigned long long has = __ballot(v > 0.0), above = __ballot(before + incl > target);
    if (has) last = x0 + 63 - __clzll((long long)has);
    if (above) pick = x0 + (int)__ffsll((long long)above) - 1;
    before += __shfl(incl, 63);
  }
  if (pick < 0) pick = last >= 0 ? last : min(g_lo, x_hi - 1);
  if (lane == 0) write_draw(a, p, j, r0 + r, pick, M, row_sum[r]);
}

__global__ __launch_bounds__(DD_BLOCK) void draft_draw_kernel(DraftArgs a) { draw_one<false>(a, blockIdx.x); }

template <int NPT>
__global__ __launch_bounds__(DD_BLOCK) void draft_one_kernel(DraftArgs a) {
  if ((int)blockIdx.x < a.chunk_wgs) take_chunks<NPT, DD_BLOCK, true>(a, blockIdx.x);
  else draw_one<true>(a, (int)blockIdx.x - a.chunk_wgs);
}

// ---- pass 2 with warping T (Section 2.1): the top_k first joint entries (by value, equal values by flat index), of
// those the shortest leading part whose share exceeds top_p, renormalised; all of a prompt's draws from that list.
struct WarpShared {
  double tab[64];
  double row_max[64], row_sum[64], row_scale[64], row_thr[64];
  double cmax[64 * DR_MAX_CHUNKS];    // largest joint entry of every chunk (-1: none)
  int list[64 * DR_MAX_CHUNKS];       // chunks that can hold a kept entry
  double gmax[64];
  double bound;
  int n_list, n_cand;
  double cv[DW_CAND];
  int ci[DW_CAND];
  double kv[DR_K_MAX];
  int ki[DR_K_MAX];
  unsigned int hist[1 << DW_DIGIT];
  int wcount[DW_WAVES];
  unsigned long long prefix;          // radix selection: leading bits of the K-th entry, and its rank among those that share them
  int want;
};

// The K-th largest of 64 group maxima (one per lane, the same in every wave): K entries are at or above it.  Every wave
// ranks four of them by ballots.  A bound already held stays if it is higher (-1: none; fewer than K groups hold anything).
__device__ __forceinline__ void bound_of_groups(WarpShared& sh, double g, int K) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 64 / DW_WAVES; ++k) {
    const int i = wave * (64 / DW_WAVES) + k;
    const double v = __shfl(g, i);
    const int ahead = __popcll(__ballot((g > v) | ((g == v) & (lane < i))));
    if (ahead == K - 1 && lane == 0 && v > sh.bound) sh.bound = v;
  }
}

template <bool ONE>
__device__ __forceinline__ void draw_warped(const DraftArgs& a, int p) {
  __shared__ WarpShared sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int K = a.top_k, V = a.V;
  int r0, n, bad = 0;
  const bool any = prompt_rows(a, p, r0, n, bad);
  if (!any) {
    if (tid < a.W_S) write_no_draw(a, p, tid);
    if (tid == 0 && bad) atomicOr(a.fault, bad);
    return;
  }
  const float u_mine = tid < a.W_S ? a.u[(long long)p * a.W_S + tid] : 0.f;
  if (tid < 64) sh.tab[tid] = c_draft_exp2_tab[tid];
  if (tid == 0) { sh.n_list = 0; sh.n_cand = 0; sh.bound = -1.0; }
  __syncthreads();
  fold_rows<DW_WAVES, ONE>(a, r0, n, sh.tab, sh.row_max, sh.row_sum, sh.row_scale, bad,
                      [&](int r, double m, double, double M, double scale) {
    if (lane < a.nchunk) sh.cmax[r * a.nchunk + lane] = m > -INFINITY ? dsbd_exp_nonpos(m - M, sh.tab) * scale : -1.0;
  });
  if (tid == 0 && bad) atomicOr(a.fault, bad);
  __syncthreads();
  // ---- a lower bound of the K-th entry: the K-th largest of the maxima of 64 groups of chunks
  const int T = n * a.nchunk;
  {
    double g = -1.0;
#pragma unroll 4
    for (int t = lane; t < T; t += 64) g = fmax(g, sh.cmax[t]);
    bound_of_groups(sh, g, K);
  }
  __syncthreads();
  // a row's logit that reaches the bound, with slack for the rounding of the logarithm (candidates are ranked by
  // their exact entries afterwards: a few too many do no harm)
  auto thresholds = [&]() {
    if (tid < n) {
      const double b = sh.bound;
      const double t = b > 0.0 ? sh.row_max[tid] + log(b / sh.row_scale[tid]) : -INFINITY;
      sh.row_thr[tid] = t - 1e-9 * (1.0 + fabs(t));
      if (!(b > 0.0)) sh.row_thr[tid] = -INFINITY;
    }
  };
  thresholds();
  for (int t = tid; t < T; t += DW_BLOCK)
    if (sh.cmax[t] >= sh.bound * (1.0 - 1e-12)) {
      const int r = t / a.nchunk;
      sh.list[atomicAdd(&sh.n_list, 1)] = r * DR_MAX_CHUNKS + t - r * a.nchunk;
    }
  __syncthreads();
  // `body(row, token, z)` on every entry of the listed chunks that reaches its row's threshold: a wave takes two tiles of
  // 512 entries at a time, all their loads in flight together (about ten chunks are listed: one or two round trips).
  // The body is there once, with its logit picked out of the registers: sixteen inlined copies cost more in instruction
  // fetches than the few entries that get that far.
  const int tshift = 31 - __clz(a.chunk) - 9;          // (chunks are powers of two, at least 1024)
  const int n_tiles = sh.n_list << tshift;
  auto each_entry = [&](auto&& body) __attribute__((always_inline)) {
    for (int w0 = wave; w0 < n_tiles; w0 += 2 * DW_WAVES) {
      float v[16];
      unsigned int hit = 0u;
      int row[2], xl[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int w = min(w0 + h * DW_WAVES, n_tiles - 1);
        const int t = sh.list[w >> tshift];
        const int r = t / DR_MAX_CHUNKS, c = t % DR_MAX_CHUNKS;
        const int x0 = c * a.chunk + (w & ((1 << tshift) - 1)) * 512;
        const int x1 = w0 + h * DW_WAVES < n_tiles ? min(V, x0 + 512) : 0;          // (0: there is no second tile)
        const float* const z = a.z + (long long)(r0 + r) * V;
        row[h] = r; xl[h] = x0 + lane;
#pragma unroll
        for (int k = 0; k < 8; ++k) v[8 * h + k] = z[min(xl[h] + 64 * k, V - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k) hit |= xl[h] + 64 * k < x1 ? 1u << (8 * h + k) : 0u;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double thr = sh.row_thr[row[h]];
#pragma unroll
        for (int k = 0; k < 8; ++k) hit &= (double)v[8 * h + k] >= thr ? ~0u : ~(1u << (8 * h + k));
      }
      for (; hit != 0u; hit &= hit - 1u) {
        const int b = __ffs((int)hit) - 1;
        float z = v[0];
#pragma unroll
        for (int k = 1; k < 16; ++k) z = b == k ? v[k] : z;
        body(b >= 8 ? row[1] : row[0], (b >= 8 ? xl[1] : xl[0]) + 64 * (b & 7), z);
      }
    }
  };
  auto entry = [&](int r, float z) { return dsbd_exp_nonpos((double)z - sh.row_max[r], sh.tab) * sh.row_scale[r]; };
  if (T < 64) {
    // few chunks bound poorly (or not at all): the maxima of 64 groups of threads over the listed chunks do better
    double g = -1.0;
    each_entry([&](int r, int, float z) { g = fmax(g, entry(r, z)); });
#pragma unroll
    for (int off = 1; off <= 8; off <<= 1) g = fmax(g, __shfl_xor(g, off));
    if ((lane & 15) == 0) sh.gmax[wave * 4 + (lane >> 4)] = g;
    __syncthreads();
    bound_of_groups(sh, sh.gmax[lane], K);
    __syncthreads();
    thresholds();
    __syncthreads();
  }
  auto keep = [&](int r, int x, float z) {
    const int at = atomicAdd(&sh.n_cand, 1);
    if (at < DW_CAND) { sh.cv[at] = entry(r, z); sh.ci[at] = r * V + x; }
  };
  each_entry(keep);
  __syncthreads();
  if (sh.n_cand > DW_CAND) {
    // Entries crowd at the bound (rows of equal logits): the K-th entry's exact value by radix selection over the
    // bits of the entries (non-negative doubles order like their bits), then everything above it and, of those equal
    // to it, the first by index.
    __syncthreads();
    if (tid == 0) { sh.prefix = 0ull; sh.want = K; sh.n_cand = 0; }
    for (int shift = 64 - DW_DIGIT; ; shift = max(shift - DW_DIGIT, 0)) {
      const int width = shift == 0 ? 64 % DW_DIGIT : DW_DIGIT;          // 64 = 5 x 11 + 9
      for (int b = tid; b < (1 << DW_DIGIT); b += DW_BLOCK) sh.hist[b] = 0u;
      __syncthreads();
      const unsigned long long prefix = sh.prefix;
      each_entry([&](int r, int, float z) {
        const unsigned long long key = (unsigned long long)__double_as_longlong(entry(r, z));
        const int up = shift + width;
        if (up >= 64 || (key >> up) == (prefix >> up)) atomicAdd(&sh.hist[(key >> shift) & ((1u << width) - 1u)], 1u);
      });
      __syncthreads();
      if (wave == 0) {
        // from the highest digit down: a lane's 32 digits in one sum, then the digits of the lane that reaches `want`
        const int hi = (1 << DW_DIGIT) - 1 - 32 * lane, want = sh.want;
        int mine = 0;
        for (int b = 0; b < 32; ++b) mine += (int)sh.hist[hi - b];
        const double incl = wave_inclusive_scan((double)mine);
        const unsigned long long reach = __ballot(incl >= (double)want);
        if (reach != 0ull && lane == (int)__ffsll((long long)reach) - 1) {
          int left = want - (int)(incl - (double)mine), d = hi;
          while ((int)sh.hist[d] < left) { left -= (int)sh.hist[d]; --d; }
          sh.want = left;
          sh.prefix = prefix | ((unsigned long long)d << shift);
        }
      }
      __syncthreads();
      if (shift == 0) break;
    }
    const unsigned long long kth = sh.prefix;
    const int n_eq = sh.want;                          // this many of the entries equal to the K-th are kept
    each_entry([&](int r, int x, float z) {
      if ((unsigned long long)__double_as_longlong(entry(r, z)) > kth) keep(r, x, z);
    });
    __syncthreads();
    const int n_gt = sh.n_cand;
    int found = 0;                                     // equal entries so far (uniform)
    for (int t = 0; t < T && found < n_eq; ++t) {      // chunks in index order
      if (!(sh.cmax[t] >= sh.bound * (1.0 - 1e-12))) continue;
      const int r = t / a.nchunk, c = t - r * a.nchunk;
      const int x1 = min(V, (c + 1) * a.chunk);
      const float* const z = a.z + (long long)(r0 + r) * V;
      for (int x0 = c * a.chunk; x0 < x1 && found < n_eq; x0 += DW_BLOCK) {
        const int x = x0 + tid;
        const float v = z[min(x, x1 - 1)];
        const bool eq = x < x1 && (double)v >= sh.row_thr[r] && (unsigned long long)__double_as_longlong(entry(r, v)) == kth;
        const unsigned long long m = __ballot(eq);
        if (lane == 0) sh.wcount[wave] = __popcll(m);
        __syncthreads();
        int ahead = found, all = 0;
        for (int w = 0; w < DW_WAVES; ++w) { ahead += w < wave ? sh.wcount[w] : 0; all += sh.wcount[w]; }
        ahead += __popcll(m & ((1ull << lane) - 1ull));
        if (eq && ahead < n_eq) { sh.cv[n_gt + ahead] = __longlong_as_double((long long)kth); sh.ci[n_gt + ahead] = r * V + x; }
        found += all;
        __syncthreads();
      }
    }
    if (tid == 0) sh.n_cand = n_gt + min(found, n_eq);
    __syncthreads();
  }
  const int nc = min(sh.n_cand, DW_CAND);
  if (tid < nc) {
    const double v = sh.cv[tid];
    const int ix = sh.ci[tid];
    int rank = 0;
#pragma unroll 4
    for (int o = 0; o < nc; ++o) {
      const double ov = sh.cv[o];
      rank += (ov > v) | ((ov == v) & (sh.ci[o] < ix));
    }
    if (rank < K) { sh.kv[rank] = v; sh.ki[rank] = ix; }
  }
  __syncthreads();
  if (wave != 0) return;
  // ---- top-p (the running sums add the entries one by one in rank order), then the kept entries in index order
  const int nk = min(nc, K);
  const double v = lane < nk ? sh.kv[lane] : 0.0;
  const int ix = lane < nk ? sh.ki[lane] : INT_MAX;
  double cum = 0.0;
#pragma unroll 8
  for (int o = 0; o < nk; ++o) {
    const double ov = sh.kv[o];
    if (o <= lane) cum += ov;
  }
  int kept = nk;
  if (a.top_p < 1.0f) {
    const double mass = __shfl(cum, max(nk - 1, 0));
    const unsigned long long over = __ballot(lane < nk && cum / mass > (double)a.top_p);
    if (over) kept = (int)__ffsll((long long)over);
  }
  const double total = __shfl(cum, max(kept - 1, 0));
  int at = 0;
#pragma unroll 8
  for (int o = 0; o < kept; ++o) at += sh.ki[o] < ix;
  wave_lds_fence();
  if (lane < kept) { sh.cv[at] = v / total; sh.ci[at] = ix; }
  wave_lds_fence();
  const double w = lane < kept ? sh.cv[lane] : 0.0;
  const double incl = wave_inclusive_scan(w);
  const double Z = __shfl(incl, 63);
  sh.gmax[lane] = incl;
  wave_lds_fence();
  if (lane < a.W_S) {
    const double target = (double)u_mine * Z;
    int pick = -1, last = 0;
#pragma unroll 8
    for (int o = 0; o < kept; ++o) {
      if (sh.cv[o] > 0.0) last = o;
      if (pick < 0 && sh.gmax[o] > target) pick = o;
    }
    if (pick < 0) pick = last;
    const int flat = kept > 0 ? sh.ci[pick] : 0;       // (no entry at all: fold_rows has reported it, the draw stays in bounds)
    const int r = flat / V;
    write_draw(a, p, lane, r0 + r, flat - r * V, sh.row_max[r], sh.row_sum[r]);
  }
}

__global__ __launch_bounds__(DW_BLOCK) void draft_warp_kernel(DraftArgs a) { draw_warped<false>(a, blockIdx.x); }

template <int NPT>
__global__ __launch_bounds__(DW_BLOCK) void draft_warp_one_kernel(DraftArgs a) {
  if ((int)blockIdx.x < a.chunk_wgs) take_chunks<NPT, DW_BLOCK, true>(a, blockIdx.x);
  else draw_warped<true>(a, (int)blockIdx.x - a.chunk_wgs);
}

int32_t check_draft(const dsbd_draft_in* in, int32_t W_S) {
  if (!in) return DSBD_ERR_INVALID;
  if (in->n_prompts < 0 || in->n_beams < 0 || in->max_prompt_beams < 0) return DSBD_ERR_INVALID;
  if (W_S < 1 || W_S > 64 || in->max_prompt_beams > 64) return DSBD_ERR_UNSUPPORTED;
  if (in->V < 1) return DSBD_ERR_UNSUPPORTED;
  return DSBD_OK;
}

// What a call with beams needs beyond that (the limits of the verification's sampling, whose results these are).
bool draft_supported(const dsbd_draft_in* in, int32_t W_S, int32_t top_k, float top_p) {
  if (in->V > (1 << 30) || in->max_prompt_beams < 1) return false;
  if (top_k < 0 || top_k > DR_K_MAX || !(top_p >= 0.0f)) return false;
  if (top_k == 0 && top_p > 0.0f && top_p < 1.0f) return false;
  if ((long long)in->n_beams * DR_MAX_CHUNKS > 0x7fffffffLL || (long long)in->n_prompts * W_S > 0x7fffffffLL) return false;      // grids
  const long long cap = W_S > in->max_prompt_beams ? W_S : in->max_prompt_beams;
  if (top_k > 0 && cap * in->V > 0x7fffffffLL) return false;           // flat indices are 32-bit integers
  return true;
}

// Chunks of a power of two of at least 1024 logits (4 per thread), at most 64 per row (a lane each in the fold): the
// smallest that give no more than 2048 workgroups, eight per compute unit, which is what is resident at once.
void draft_chunks(const dsbd_draft_in* in, int* chunk, int* nchunk) {
  long long c = 1024;
  while ((in->V + c - 1) / c > DR_MAX_CHUNKS || (c < 4096 && in->n_beams * ((in->V + c - 1) / c) > 2048)) c *= 2;
  *chunk = (int)c;
  *nchunk = (int)((in->V + c - 1) / c);
}

}  // namespace

extern "C" size_t dsbd_draft_layer_workspace_bytes(const dsbd_draft_in* in, int32_t W_S, int32_t top_k, float top_p) {
  if (check_draft(in, W_S) != DSBD_OK) return 0;
  if (in->n_beams == 0 || in->n_prompts == 0) return 256;
  if (!draft_supported(in, W_S, top_k, top_p)) return 0;
  int chunk, nchunk;
  draft_chunks(in, &chunk, &nchunk);
  WorkspaceCarver ws(nullptr);
  ws.take<Slot>((size_t)in->n_beams * nchunk * 2);
  return ws.total() + 256;
}

extern "C" int32_t dsbd_draft_layer(const dsbd_draft_in* in, int32_t W_S, int32_t top_k, float top_p,
                                    const dsbd_draft_out* out, void* workspace, size_t workspace_bytes,
                                    int32_t* fault, void* stream_) {
  if (!out || !fault) return DSBD_ERR_INVALID;
  const int32_t rc = check_draft(in, W_S);
  if (rc != DSBD_OK) return rc;
  if (in->n_beams == 0 || in->n_prompts == 0) return DSBD_OK;
  if (!in->beam_off || !in->logits_draft || !in->beam_logp_draft || !in->u) return DSBD_ERR_INVALID;
  if (!out->parent || !out->token || !out->logp_draft || !workspace) return DSBD_ERR_INVALID;
  const size_t need = dsbd_draft_layer_workspace_bytes(in, W_S, top_k, top_p);
  if (need == 0) return DSBD_ERR_UNSUPPORTED;
  if (workspace_bytes < need) return DSBD_ERR_WORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  DraftArgs a;
  draft_chunks(in, &a.chunk, &a.nchunk);
  WorkspaceCarver ws(reinterpret_cast<char*>(dsbd_align_up(reinterpret_cast<uintptr_t>(workspace), 256)));
  a.slots = ws.take<Slot>((size_t)in->n_beams * a.nchunk * 2);
  a.part = reinterpret_cast<double2*>(a.slots);
  a.n_prompts = in->n_prompts; a.n_beams = in->n_beams; a.max_prompt_beams = in->max_prompt_beams; a.V = in->V; a.W_S = W_S;
  a.beam_off = in->beam_off; a.z = in->logits_draft; a.cum = in->beam_logp_draft; a.u = in->u;
  a.top_k = top_k; a.top_p = (top_p > 0.0f && top_p < 1.0f) ? top_p : 1.0f;
  a.out_parent = out->parent; a.out_token = out->token; a.out_logp = out->logp_draft; a.fault = fault;
  const long long n_chunks = (long long)in->n_beams * a.nchunk;
  const long long draws = top_k > 0 ? in->n_prompts : (long long)in->n_prompts * W_S;
  // One launch: the drawing workgroups stand behind those that take the chunks and wait for their results.  The workgroups in
  // front wait for nobody, and a wait that lasts (other streams' work can keep them from starting) ends with the waiting wave
  // taking the chunk itself, so nothing depends on what runs beside it.  Not under capture, where a replay would repeat the
  // tags.  Measured, us per step: 8 to 16 beams x 128256, warped, 17.1 on the device in two kernels, 16.1 in one; 6 us of host
  // time in two launches, 2.9 in one.
  // Only up to a size: the chunks then run in the drawing kernel's workgroups, of which a compute unit holds two (warped, 74 KB
  // of LDS) or four, not eight as of the chunk kernel's, and a step of many chunks is bound by their stream.  Measured, us on
  // the device in two kernels -> one: warped, 8.2 MB of logits 17.3 -> 15.4, 15.6 -> 13.9 and 15.4 -> 15.5; 16.4 MB 19.9 -> 19.3
  // and 18.7 -> 19.3; 24.6 MB 23.7 -> 24.7; 67.7 MB 33.3 -> 42.4.  Not warped, 32.8 MB 20.8 -> 19.9, 49.3 MB 24.6 -> 24.0, 65.5 MB
  // 31.0 -> 31.7.
  const bool streams = (long long)in->n_beams * in->V > (top_k > 0 ? DR_ONE_WARPED : DR_ONE_PLAIN);
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  const bool capturing = hipStreamIsCapturing(stream, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone;
  if (!capturing && !streams && draws <= DR_WAITING) {
    const DsbdKnobs& knobs = dsbd_knobs();
    a.tag = exchange_tag(dsbd_launch_nonce());
    a.wait_limit = knobs.draft_wait_us >= 0 ? knobs.draft_wait_us * 100LL : DR_WAIT_TICKS;
    const int block = top_k > 0 ? DW_BLOCK : DD_BLOCK, per_wg = block / DC_BLOCK;
    a.chunk_wgs = (int)((n_chunks + per_wg - 1) / per_wg);
    const dim3 grid((unsigned)(a.chunk_wgs + draws));
    auto launch = [&](auto warped, auto plain) {
      if (top_k > 0) hipLaunchKernelGGL(warped, grid, dim3(DW_BLOCK), 0, stream, a);
      else hipLaunchKernelGGL(plain, grid, dim3(DD_BLOCK), 0, stream, a);
    };
    if (a.chunk == 1024) launch(draft_warp_one_kernel<4>, draft_one_kernel<4>);
    else if (a.chunk == 2048) launch(draft_warp_one_kernel<8>, draft_one_kernel<8>);
    else launch(draft_warp_one_kernel<16>, draft_one_kernel<16>);
  } else {
    if (capturing) (void)hipGetLastError();
    const dim3 grid((unsigned)n_chunks);
    if (a.chunk == 1024) hipLaunchKernelGGL(draft_chunk_kernel<4>, grid, dim3(DC_BLOCK), 0, stream, a);
    else if (a.chunk == 2048) hipLaunchKernelGGL(draft_chunk_kernel<8>, grid, dim3(DC_BLOCK), 0, stream, a);
    else hipLaunchKernelGGL(draft_chunk_kernel<16>, grid, dim3(DC_BLOCK), 0, stream, a);
    if (top_k > 0) hipLaunchKernelGGL(draft_warp_kernel, dim3((unsigned)draws), dim3(DW_BLOCK), 0, stream, a);
    else hipLaunchKernelGGL(draft_draw_kernel, dim3((unsigned)draws), dim3(DD_BLOCK), 0, stream, a);
  }
  DSBD_HIP_LAUNCH_CHECK();
  return DSBD_OK;
}

// ------------------------------------------------------------------------------------------------ forest layout
namespace {

struct BuildArgs {
  int n_prompts, n_roots, gamma, W_S;
  const int32_t *root_off, *root_token, *layer_parent, *layer_token;
  dsbd_forest_out out;
  int32_t* fault;
};

struct BuildShared {
  int root[BF_NODE_CAP];        // prompt-local input beam every node descends from
  int key[BF_NODE_CAP];         // layer * W_S + draw index (0 for roots): the order inside a tree
  int par_local[BF_NODE_CAP];   // prompt-local index (layer-major) of the parent, -1 for roots
  int pos[BF_NODE_CAP];         // position of the node in the prompt's part of the forest
  int tree_n[64];
  int largest;
  int bad;
};

__global__ __launch_bounds__(BF_BLOCK) void build_forest_kernel(BuildArgs a) {
  __shared__ BuildShared sh;
  const int p = blockIdx.x, tid = threadIdx.x;
  const int r0 = a.root_off[p], r1 = a.root_off[p + 1];
  int W = r1 - r0;
  const int rows = a.n_prompts * a.W_S;                 // rows of a drafted layer
  int bad = 0;
  if (r0 < 0 || r1 > a.n_roots || W < 0 || W > 64) { bad |= DSBD_FAULT_BOUNDS; W = 0; }
  if (p == 0 && r0 != 0) bad |= DSBD_FAULT_TOPOLOGY;
  if (p == a.n_prompts - 1 && r1 != a.n_roots) bad |= DSBD_FAULT_TOPOLOGY;
  int n_p = W > 0 ? W + a.gamma * a.W_S : 0;            // nodes of the prompt; local index: roots, then layer-major
  if (n_p > BF_NODE_CAP) { bad |= DSBD_FAULT_BOUNDS; n_p = 0; W = 0; }
  const long long base = (long long)r0 + (long long)p * a.gamma * a.W_S;     // first forest node of the prompt
  if (tid == 0) { sh.bad = 0; sh.largest = 0; }
  if (tid < 64) sh.tree_n[tid] = 0;
  __syncthreads();
  // every node: its parent (prompt-local) and, walking up, its input beam
  if (tid < n_p) {
    int l = 0, j = tid, par = -1, root = tid;
    if (tid >= W) {
      l = 1 + (tid - W) / a.W_S; j = (tid - W) % a.W_S;
      int cur_l = l, row = p * a.W_S + j;
      while (cur_l >= 1) {
        int up = a.layer_parent[(long long)(cur_l - 1) * rows + row];
        // rows of the layer above that belong to this prompt
        const int lo = cur_l == 1 ? r0 : p * a.W_S, hi = cur_l == 1 ? r1 : (p + 1) * a.W_S;
        if (up < lo || up >= hi) { atomicOr(&sh.bad, DSBD_FAULT_TOPOLOGY); up = lo; }
        if (cur_l == l) par = cur_l == 1 ? up - r0 : W + (cur_l - 2) * a.W_S + (up - p * a.W_S);
        row = up;
        cur_l -= 1;
      }
      root = row - r0;
    }
    sh.root[tid] = root;
    sh.key[tid] = tid < W ? 0 : l * a.W_S + j;          // a root comes first in its tree (its own index may exceed W_S)
    sh.par_local[tid] = par;
    atomicAdd(&sh.tree_n[root], 1);
  }
  __syncthreads();
  if (tid < n_p) {
    const int root = sh.root[tid], key = sh.key[tid];
    int pos = 0;
    for (int c = 0; c < n_p; ++c) {
      const int rc = sh.root[c], kc = sh.key[c];
      pos += (rc < root) | ((rc == root) & (kc < key));
    }
    sh.pos[tid] = pos;
  }
  __syncthreads();
  if (tid < n_p) {
    const long long n = base + sh.pos[tid];
    const int par = sh.par_local[tid];
    a.out.parent[n] = par < 0 ? -1 : (int)(base + sh.pos[par]);
    if (tid < W) {
      a.out.token[n] = a.root_token ? a.root_token[r0 + tid] : 0;
      a.out.draft_rank[n] = 0;
      a.out.tree_prompt[r0 + tid] = p;
      a.out.tree_off[r0 + tid] = (int)n;
      a.out.node_of_root[r0 + tid] = (int)n;
      if (sh.tree_n[tid] > DSBD_MAX_TREE_NODES) atomicOr(&sh.bad, DSBD_FAULT_BOUNDS);
      atomicMax(&sh.largest, sh.tree_n[tid]);
    } else {
      const int l = 1 + (tid - W) / a.W_S, j = (tid - W) % a.W_S;
      const long long li = (long long)(l - 1) * rows + p * a.W_S + j;
      a.out.token[n] = a.layer_token[li];
      a.out.draft_rank[n] = j;
      a.out.node_of[li] = (int)n;
    }
  }
  if (W == 0 && n_p == 0) {
    // a prompt without input beams (or one that does not fit): its draws get no node
    for (int i = tid; i < a.gamma * a.W_S; i += BF_BLOCK) {
      const int l = 1 + i / a.W_S, j = i % a.W_S;
      a.out.node_of[(long long)(l - 1) * rows + p * a.W_S + j] = -1;
    }
  }
  if (p == a.n_prompts - 1 && tid == 0) a.out.tree_off[a.n_roots] = a.n_roots + a.gamma * rows;
  __syncthreads();
  if (tid == 0) {
    if (bad | sh.bad) atomicOr(a.fault, bad | sh.bad);
    if (a.n_prompts == 1) *a.out.max_tree_nodes = sh.largest;      // (a lone prompt needs no cleared word: a launch less)
    else atomicMax(a.out.max_tree_nodes, sh.largest);
  }
}

__global__ void build_forest_init_kernel(int32_t* max_tree_nodes) { *max_tree_nodes = 0; }

}  // namespace

extern "C" int32_t dsbd_build_forest(int32_t n_prompts, int32_t n_roots, int32_t gamma, int32_t W_S,
                                     const int32_t* root_off, const int32_t* root_token,
                                     const int32_t* layer_parent, const int32_t* layer_token,
                                     const dsbd_forest_out* out, int32_t* fault, void* stream_) {
  if (!out || !fault) return DSBD_ERR_INVALID;
  if (n_prompts < 0 || n_roots < 0 || gamma < 0 || W_S < 0) return DSBD_ERR_INVALID;
  if (gamma > 0 && (W_S < 1 || W_S > 64)) return DSBD_ERR_UNSUPPORTED;
  if (gamma >= DSBD_MAX_TREE_NODES) return DSBD_ERR_UNSUPPORTED;
  if (n_prompts == 0) return DSBD_OK;
  if (!root_off || (gamma > 0 && (!layer_parent || !layer_token))) return DSBD_ERR_INVALID;
  if (!out->tree_prompt || !out->tree_off || !out->parent || !out->token || !out->draft_rank || !out->node_of_root ||
      !out->max_tree_nodes || (gamma > 0 && !out->node_of))
    return DSBD_ERR_INVALID;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  BuildArgs a;
  a.n_prompts = n_prompts; a.n_roots = n_roots; a.gamma = gamma; a.W_S = gamma > 0 ? W_S : 0;
  a.root_off = root_off; a.root_token = root_token; a.layer_parent = layer_parent; a.layer_token = layer_token;
  a.out = *out; a.fault = fault;
  if (n_prompts > 1) hipLaunchKernelGGL(build_forest_init_kernel, dim3(1), dim3(1), 0, stream, out->max_tree_nodes);
  hipLaunchKernelGGL(build_forest_kernel, dim3((unsigned)n_prompts), dim3(BF_BLOCK), 0, stream, a);
  DSBD_HIP_LAUNCH_CHECK();
  return DSBD_OK;
}
