// Row work of a warped verification (paper Section 2.1: T cuts the joints to their top_k first entries, then by top-p):
// for every row of both models its maximum, its fp64 sum of exponentials and its top_k first entries, plus the per-node
// fp32 outputs (log-sum-exp of a node's row, log-probability of a node's token under its parent's row).
//
// A joint's top_k first entries are among the top_k first entries of its rows, so the layer walk gets by with these records
// and never touches the logits again: it needs no slices of the joint and no partner workgroups (verify.hip).  All rows
// are taken at once, whether the walk reaches them or not: their sums are outputs anyway.  (Before, every layer formed its
// joint over I x V on up to 256 workgroups and selected from it by exchanges: 15 us of a layer's 22; now 4 of 11.)
//
// Two kernels:
//  1. verify_chunk_kernel: a wave per chunk of a row, no barrier: maximum, sum, and the maxima of the chunk's parts.
//     Bound by fp64 exponentials as soon as there are many: both models' rows of 53 nodes x 128256 (54 MB) take 15 us, of 248
//     nodes (254 MB) 60; without the exponentials 13 and 36 (7.1 TB/s).  Fewer instructions per exponential (rounding by an
//     addition, the power of two put into the table entry's exponent) changed nothing, a table of 256 entries with a
//     polynomial of degree 4 took 5 us off 248 nodes and nothing off 53.
//  2. verify_row_kernel: a workgroup per row folds the chunks, bounds the row's K-th entry by the K-th largest of the
//     maxima of groups of parts (K entries reach it) and reads again only the parts that reach the bound.  A chain of round
//     trips: 6 us for 106 rows, 9 for 496 (with 256 threads per row, which take the parts three after the other: 14).
#include "verify_rows.h"
#include "exp_nonpos.h"
#include "wave_f64.h"
#include <float.h>
#include <limits.h>
#include <algorithm>

#define VR_BLOCK 256           // chunk kernel
#define VR_ROW_BLOCK 1024      // row kernel, few rows: short chains of round trips ...
#define VR_ROW_BLOCK_MANY 256  // ... and many: workgroups side by side
#define VR_ROWS_MANY 512       // rows up to which the large ones are all resident at once, two on every compute unit (verification, us
                               // at 1024 / 256 threads per row: 106 rows x 128256 47.3 / 49.3, 240 x 32000 top_k 32 65.5 / 73.3, 496 x
                               // 32000 73.5 / 74.3, 1154 x 32000 105 / 98, 5642 x 1000 119 / 86, 72000 x 300 788 / 367)
#define VR_PARTS 256            // most parts of a row
#define VR_LAUNCH_CHUNKS (1 << 23)     // most chunks, and so rows, of a launch (2^32 threads are the limit)
#define VR_CAND 1024           // candidates that are ranked directly

namespace {

__constant__ double c_rows_exp2_tab[64] = {DSBD_EXP2_TABLE_64};

// (rows of an odd vocabulary start anywhere; the loads are as wide all the same)
typedef float vr_f32x4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ const float* row_logits(const RowsArgs& a, int row) {
  return a.alias ? a.zp + (long long)row * a.V : ((row & 1) ? a.zq : a.zp) + (long long)(row >> 1) * a.V;
}

#define VR_TILE 1024           // logits a wave takes at a time: four 16-byte loads per lane
struct Tile { vr_f32x4 v[4]; };

__device__ __forceinline__ Tile load_tile(const float* __restrict__ z, int x0, int x_end) {
  const int lane = threadIdx.x & 63;
  Tile t;
  if (x0 + VR_TILE <= x_end) {
#pragma unroll
    for (int k = 0; k < 4; ++k) t.v[k] = __builtin_nontemporal_load(reinterpret_cast<const vr_f32x4*>(z + x0 + k * 256 + lane * 4));
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int x = x0 + k * 256 + lane * 4 + e;
        const float w = z[min(x, x_end - 1)];
        t.v[k][e] = x < x_end ? w : -INFINITY;             // (places beyond the row's end: masked tokens)
      }
  }
  return t;
}

// The maxima of a tile's parts (PARTS 2 or 4: in every lane; 16: of four lanes' rows and four loads, lane l's row's in
// part[k]), its maximum and its sum of exponentials against that.
template <int PARTS>
__device__ __forceinline__ void take_tile(const Tile& t, const double* tab, bool& bad, float (&part)[4], float& m, double& s) {
  float q[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    q[k] = fmaxf(fmaxf(t.v[k][0], t.v[k][1]), fmaxf(t.v[k][2], t.v[k][3]));
#pragma unroll
    for (int e = 0; e < 4; ++e) bad |= !(t.v[k][e] <= FLT_MAX);      // NaN or +Inf
  }
  if constexpr (PARTS == 2 || PARTS == 0) {
    part[0] = wave_max_f32(fmaxf(q[0], q[1]));
    part[1] = wave_max_f32(fmaxf(q[2], q[3]));
    m = fmaxf(part[0], part[1]);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) part[k] = PARTS == 4 ? wave_max_f32(q[k]) : row16_max_f32(q[k]);
    m = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    if constexpr (PARTS == 16) m = wave_max_f32(m);
  }
  const double ref = m == -INFINITY ? 0.0 : (double)m;     // (a tile masked whole adds 0)
  double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] += dsbd_exp_nonpos((double)t.v[k][e] - ref, tab);
  s = wave_sum((sum[0] + sum[1]) + (sum[2] + sum[3]));
}

// SINGLE: a chunk is one tile (rows of up to 131072 logits); else several, merged as they go.  A chunk per wave and as many
// waves as there are chunks: those that wait for their logits and those that work on theirs mix by themselves (four resident
// waves per SIMD that take chunk after chunk, the next two on their way: 2 us slower on 54 MB).
template <bool SINGLE, int PARTS>
__global__ __launch_bounds__(VR_BLOCK) void verify_chunk_kernel(RowsArgs a, int row0, int rows) {
  __shared__ double tab[64];
  const int lane = threadIdx.x & 63;
  const unsigned int mine = blockIdx.x * (VR_BLOCK / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool live = mine < (unsigned int)rows * (unsigned int)a.nchunk;      // (below VR_LAUNCH_CHUNKS)
  const unsigned int at = live ? mine : 0u;
  const int row = row0 + (int)(at / (unsigned int)a.nchunk), c = (int)(at % (unsigned int)a.nchunk);
  const long long item = (long long)row * a.nchunk + c;
  const float* const z = row_logits(a, row);
  const int x_lo = c * a.chunk, x_hi = min(a.V, x_lo + a.chunk);
  const Tile first = load_tile(z, x_lo, x_hi);
  if (threadIdx.x < 64) tab[threadIdx.x] = c_rows_exp2_tab[threadIdx.x];
  __syncthreads();
  if (!live) return;
  bool bad = false;
  float sub[4], M;
  double S;
  take_tile<PARTS>(first, tab, bad, sub, M, S);
  if constexpr (!SINGLE) {
    float part[2] = {M, -INFINITY};                        // (a part is half of the chunk: whole tiles)
    for (int x0 = x_lo + VR_TILE; x0 < x_hi; x0 += VR_TILE) {
      float m;
      double s;
      take_tile<2>(load_tile(z, x0, x_hi), tab, bad, sub, m, s);
      if (x0 - x_lo < a.chunk / 2) part[0] = fmaxf(part[0], m); else part[1] = fmaxf(part[1], m);
      if (m > -INFINITY) {
        const float Mn = fmaxf(M, m);
        S = (M > -INFINITY ? S * dsbd_exp_nonpos((double)M - (double)Mn, tab) : 0.0) + s * dsbd_exp_nonpos((double)m - (double)Mn, tab);
        M = Mn;
      }
    }
    sub[0] = part[0]; sub[1] = part[1];
  }
  bad = __ballot(bad) != 0ull;
  if (bad) S = -S;                                         // (sums are never negative)
  if (lane == 0) {
    if (a.part) a.part[item] = make_double2((double)M, S);
    else if (a.compact < 0) *reinterpret_cast<double*>(a.rec + item * a.rec_stride) = S;
    else { RowHead h; h.sum = S; h.max = M; h.n = 0; *reinterpret_cast<RowHead*>(a.rec + item * a.rec_stride) = h; }
  }
  if constexpr (PARTS == 16) {
    if ((lane & 15) == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) a.sub[item * 16 + 4 * k + (lane >> 4)] = sub[k];
    }
  } else if constexpr (PARTS > 0) {
    if (lane < PARTS) a.sub[item * PARTS + lane] = lane == 0 ? sub[0] : lane == 1 ? sub[1] : lane == 2 ? sub[2] : sub[3];
  }
  if (bad && a.report && lane == 0) atomicOr(a.fault, DSBD_FAULT_NONFINITE);
}

// The entry of value v and token x comes before the one of value v2 and token x2 of the same row.
template <class T>
__device__ __forceinline__ bool entry_before(T v, int x, T v2, int x2) { return (v > v2) | ((v == v2) & (x < x2)); }

template <int RB>
__global__ __launch_bounds__(RB) void verify_row_kernel(RowsArgs a, int row0) {
  constexpr int WAVES = RB / 64, PT = VR_WHOLE / RB;      // logits per thread of a row read whole
  __shared__ double tab[64];
  __shared__ __attribute__((aligned(16))) float part_max[VR_PARTS];
  __shared__ int list[VR_PARTS];
  __shared__ float cz[VR_CAND];
  __shared__ int cx[VR_CAND];
  __shared__ float bound_s;
  __shared__ int n_list, n_cand, close;
  __shared__ double best_v[WAVES];
  __shared__ int best_x[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = row0 + blockIdx.x, K = a.K, V = a.V;
  const bool second = !a.alias && (row & 1);
  const int node = a.alias ? row : row >> 1;
  const float* const z = row_logits(a, row);
  const int nsub = a.nchunk * a.parts, sub_len = a.parts > 0 ? a.chunk / a.parts : 0;
  const bool whole = a.parts == 0;            // a short row: its logits are in the threads' registers
  // everything that is read from memory first is requested together
  double2 ms[VR_MAX_CHUNKS / 64];
#pragma unroll
  for (int k = 0; k < VR_MAX_CHUNKS / 64; ++k) {
    ms[k] = make_double2(-INFINITY, 0.0);
    if (lane + 64 * k < a.nchunk) {
      if (a.part) ms[k] = a.part[(long long)row * a.nchunk + lane + 64 * k];
      else if (a.compact < 0) ms[k].y = *reinterpret_cast<const double*>(a.rec + (long long)row * a.rec_stride);
      else { const RowHead h = *reinterpret_cast<const RowHead*>(a.rec + (long long)row * a.rec_stride); ms[k] = make_double2((double)h.max, h.sum); }
    }
  }
  float mine[PT];
  if (whole) {
#pragma unroll
    for (int k = 0; k < PT; ++k) {
      const float v = z[min(tid + k * RB, V - 1)];
      mine[k] = tid + k * RB < V ? v : -INFINITY;
    }
  } else if (tid < VR_PARTS) {
    part_max[tid] = tid < nsub ? a.sub[(long long)row * nsub + tid] : -INFINITY;
  }
  // children: nodes of the same tree, behind this one, no further than a tree is long
  const int child_n = min(node + tid, a.n_nodes - 1);
  int child_par = -1, ct = -1, par = -1, tok = -1;
  if (tid < DSBD_MAX_TREE_NODES) {
    child_par = a.parent[child_n]; ct = a.token[child_n];
    par = a.parent[node]; tok = a.token[node];
  }
  if (whole) {                                // 64 groups of threads, in place of four parts each
    float gm = mine[0];
#pragma unroll
    for (int k = 1; k < PT; ++k) gm = fmaxf(gm, mine[k]);
    gm = RB == 1024 ? row16_max_f32(gm) : quad_max_f32(gm);
    if (tid % (RB / 64) == 0) part_max[tid / (RB / 64)] = gm;
  }
  if (tid < 64) tab[tid] = c_rows_exp2_tab[tid];
  if (tid == 0) { bound_s = -INFINITY; n_list = 0; n_cand = 0; close = 0; }
  __syncthreads();
  const bool child = tid >= 1 && tid < DSBD_MAX_TREE_NODES && node + tid < a.n_nodes && child_par == node && ct >= 0 && ct < V;
  const float zt = child ? z[ct] : 0.f;
  // the row's maximum and sum, every wave for itself, in a fixed order
  static_assert(VR_MAX_CHUNKS == 128, "two chunks per lane");
  if (a.compact < 0) ms[0].x = lane == 0 ? (double)wave_max_f32(part_max[lane]) : -INFINITY;      // (one chunk, read whole)
  const bool bad = __ballot((__double2hiint(ms[0].y) | __double2hiint(ms[1].y)) < 0) != 0ull;
  ms[0].y = fabs(ms[0].y); ms[1].y = fabs(ms[1].y);
  const double M = wave_max_f64(fmax(ms[0].x, ms[1].x));
  const double S = wave_sum((ms[0].x > -INFINITY ? ms[0].y * dsbd_exp_nonpos(ms[0].x - M, tab) : 0.0) +
                            (ms[1].x > -INFINITY ? ms[1].y * dsbd_exp_nonpos(ms[1].x - M, tab) : 0.0));
  float top;                                  // the row's maximum
  // the bound: the K-th largest of the maxima of 64 groups of parts (K entries reach it; fewer groups: none), one group per
  // lane, the same in every wave, each of which ranks four of them
  {
    static_assert(VR_PARTS == 4 * 64, "four parts per lane");
    static_assert(RB == 64 * 16 || RB == 64 * 4, "groups of 16 or four threads");
    float gm = part_max[lane];
    if (!whole) gm = fmaxf(fmaxf(gm, part_max[lane + 64]), fmaxf(part_max[lane + 128], part_max[lane + 192]));
#pragma unroll
    for (int k = 0; k < 64 / WAVES; ++k) {
      const int i = 64 / WAVES * wave + k;
      const float v = __shfl(gm, i);
      const int ahead = __popcll(__ballot((gm > v) | ((gm == v) & (lane < i))));
      if (ahead == K - 1 && lane == 0) bound_s = v;
    }
    top = wave_max_f32(gm);
  }
  __syncthreads();
  // (lowered by the distance that logits of equal entries can have, eight times over: the roundings of z - max and of exp)
  const float bound = bound_s - 1e-15f * (4.f + (top - bound_s));
  // Different logits can have equal entries only where they differ by no more than the bound was lowered by: both around zero
  // (neighbours are |z| 2^-24 apart).
  const float near = 4e-8f * (4.f + fabsf(top));
  auto offer = [&](float v, int x) {                         // an entry at or above the bound is a candidate
    if (v >= bound && v > -INFINITY) {
      const int at = atomicAdd(&n_cand, 1);
      if (at < VR_CAND) { cz[at] = v; cx[at] = x; }
      if (fabsf(v) <= near) close = 1;
    }
  };
  if (whole) {
#pragma unroll
    for (int k = 0; k < PT; ++k) offer(mine[k], tid + k * RB);
  } else if (tid < nsub && part_max[tid] >= bound && part_max[tid] > -INFINITY) {
    list[atomicAdd(&n_list, 1)] = tid;
  }
  __syncthreads();
  const int nl = n_list;
  for (int i = wave; i < nl; i += WAVES) {
    const int x_lo = list[i] * sub_len, x_hi = min(V, x_lo + sub_len);
    for (int x0 = x_lo; x0 < x_hi; x0 += 512) {
      float v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = z[min(x0 + k * 64 + lane, x_hi - 1)];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (x0 + k * 64 + lane < x_hi) offer(v[k], x0 + k * 64 + lane);
    }
  }
  __syncthreads();
  char* const rec = a.rec + (long long)row * a.rec_stride;
  auto put = [&](int r, float v, int x) {
    if (a.compact < 0) return;
    if (a.compact == 1) { reinterpret_cast<uint8_t*>(rec + sizeof(RowHead))[r] = (uint8_t)x; return; }
    if (a.compact == 2) { reinterpret_cast<uint16_t*>(rec + sizeof(RowHead))[r] = (uint16_t)x; return; }
    RowEntry e;
    e.z = v; e.x = x;
    reinterpret_cast<RowEntry*>(rec + sizeof(RowHead))[r] = e;
  };
  const int nc = n_cand;
  if (nc <= min(a.direct, VR_CAND) && close == 0) {
    for (int t = tid; t < nc; t += RB) {                     // (the entries' order is that of their logits)
      const float v = cz[t];
      const int x = cx[t];
      int rank = 0;
#pragma unroll 4
      for (int o = 0; o < nc; ++o) rank += entry_before(cz[o], cx[o], v, x) ? 1 : 0;
      if (rank < K) put(rank, v, x);
    }
  } else {
    // Entries crowd at the bound (equal logits), or some may be equal though their logits are not: rank after rank, every thread offers its first entry behind the last one
    // taken, and only the thread whose offer was taken looks for its next.
    double bv = -1.0, pv = INFINITY;                             // the thread's offer; the last entry taken
    float bz = 0.f;
    int bx = -1, px = -1;
    for (int r = 0; r < K; ++r) {
      if (bx == px) {
        bv = -1.0; bx = INT_MAX;
        float same = NAN;                                        // (crowds: an exponential for each change of the logit)
        double v = 0.0;
        for (int i = 0; i < (whole ? 1 : nl); ++i) {
          const int x_lo = whole ? 0 : list[i] * sub_len, x_hi = whole ? V : min(V, x_lo + sub_len);
          for (int x = x_lo + tid; x < x_hi; x += RB) {
            const float w = z[x];
            if (!(w >= bound && w > -INFINITY)) continue;
            if (w != same) { same = w; v = dsbd_exp_nonpos((double)w - M, tab); }
            if (entry_before(pv, px, v, x) && entry_before(v, x, bv, bx)) { bv = v; bz = w; bx = x; }
          }
        }
      }
      double wv = bv;
      int wx = bx;
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) {
        const double ov = __shfl_xor(wv, off);
        const int ox = __shfl_xor(wx, off);
        if (entry_before(ov, ox, wv, wx)) { wv = ov; wx = ox; }
      }
      __syncthreads();
      if (lane == 0) { best_v[wave] = wv; best_x[wave] = wx; }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < WAVES; ++w)
        if (entry_before(best_v[w], best_x[w], wv, wx)) { wv = best_v[w]; wx = best_x[w]; }
      if (wx == INT_MAX) break;                                  // (no more entries; uniform)
      if (bx == wx) put(r, bz, wx);
      pv = wv; px = wx;
    }
  }
  // ---- head and per-node outputs
  const double lse64 = M + log(S);
  const float lse = (float)lse64;
  float* const o_lse = second ? a.lse_q : a.lse_p;
  float* const o_logp = second ? a.logp_q : a.logp_p;
  int fault = 0;
  if (tid == 0) {
    RowHead h;
    h.sum = S; h.max = (float)M; h.n = min(nc, K) + (bad ? VR_ROW_BAD : 0);
    if (a.compact >= 0) *reinterpret_cast<RowHead*>(rec) = h;
    if (o_lse) o_lse[node] = lse;
    if (a.alias && a.lse_q) a.lse_q[node] = lse;
    if (!(S > 0.0)) fault = DSBD_FAULT_NONFINITE;              // a row without a finite logit (NaN and +Inf: the chunks report them)
    if (!(par >= 0 && par < node && node - par < DSBD_MAX_TREE_NODES && tok >= 0 && tok < V)) {      // a root (or a node reported elsewhere)
      if (o_logp) o_logp[node] = 0.f;
      if (a.alias && a.logp_q) a.logp_q[node] = 0.f;
    }
  }
  if (child) {
    if (zt == -INFINITY) fault = DSBD_FAULT_NONFINITE;         // a drafted token masked in its parent's row
    const float lp = (float)((double)zt - lse64);
    if (o_logp) o_logp[child_n] = lp;
    if (a.alias && a.logp_q) a.logp_q[child_n] = lp;
  }
  if (fault && a.report) atomicOr(a.fault, fault);
}

}  // namespace

hipError_t launch_verify_rows(const RowsArgs& a, hipStream_t stream) {
  const int rows = a.n_nodes * (a.alias ? 1 : 2);
  for (int row0 = 0, most = std::max(1, VR_LAUNCH_CHUNKS / a.nchunk); row0 < rows; row0 += std::min(most, rows - row0)) {
    const int n = std::min(most, rows - row0);
    const dim3 grid(((unsigned)n * (unsigned)a.nchunk + VR_BLOCK / 64 - 1) / (VR_BLOCK / 64));
    if (a.chunk > VR_TILE) hipLaunchKernelGGL((verify_chunk_kernel<false, 2>), grid, dim3(VR_BLOCK), 0, stream, a, row0, n);
    else if (a.parts == 0) hipLaunchKernelGGL((verify_chunk_kernel<true, 0>), grid, dim3(VR_BLOCK), 0, stream, a, row0, n);
    else if (a.parts == 16) hipLaunchKernelGGL((verify_chunk_kernel<true, 16>), grid, dim3(VR_BLOCK), 0, stream, a, row0, n);
    else if (a.parts == 4) hipLaunchKernelGGL((verify_chunk_kernel<true, 4>), grid, dim3(VR_BLOCK), 0, stream, a, row0, n);
    else hipLaunchKernelGGL((verify_chunk_kernel<true, 2>), grid, dim3(VR_BLOCK), 0, stream, a, row0, n);
    if (rows <= VR_ROWS_MANY) hipLaunchKernelGGL(verify_row_kernel<VR_ROW_BLOCK>, dim3((unsigned)n), dim3(VR_ROW_BLOCK), 0, stream, a, row0);
    else hipLaunchKernelGGL(verify_row_kernel<VR_ROW_BLOCK_MANY>, dim3((unsigned)n), dim3(VR_ROW_BLOCK_MANY), 0, stream, a, row0);
  }
  return hipGetLastError();
}
