// Layer-wise verification of a draft forest on gfx950 (paper Section 3.1 "Details", Algorithm 1,
// and the dynamic layer width of Section 3.2, Eq. 1-6).
//
// One launch, two kinds of workgroups that do not depend on each other:
//
// 1. The first ones walk the layers (latency-bound, persistent; all of them must be resident at once, which their place
//    at the front of the grid gives them): G workgroups per prompt.  Every decision is taken in fp64.  They derive
//    everything from the call's inputs (tree and node range of their prompt, node depths, the maxima and sums of the
//    rows they use).  For the layer's input beams I the workgroups materialise p_beam and q_beam over I x V (their
//    slice each), and every dependent reduction over I x V is one pass over the slices plus one exchange among the G
//    workgroups.
// 2. Those behind take the fp32 statistics of the rows of both models (bandwidth-bound, all nodes: the
//    per-node outputs, the O(W |V|) softmax work of Section 2.1 done once for every forest node).  They run on the
//    compute units that the layers leave free, and on all of them once the layers are done.
//
// The running residual p' is never stored.  After k consecutive rejections since the last reset
//     p'_k = max(p_beam - c_k q_beam, 0) / F(c_k),   F(c) = sum max(p_beam - c q_beam, 0),
//     c_1 = 0, F(c_1) := 1, c_{k+1} = c_k + F(c_k)
// (induction on p'_{k+1} = norm(max(0, p'_k - q_beam))), so a rejection costs one evaluation of F, the
// chain {c_k, F(c_k)} depends only on (p_beam, q_beam) and is reused after every acceptance resets p'
// to p_beam, and the conditional acceptance probabilities of Eq. 3 are alpha_k = 1 - F(c_{k+1})/F(c_k).
//
// All G workgroups of a prompt run the same sequential program on the same reduced values (summed in
// the same order), so their control flow stays identical without any broadcast.
//
// Warped joints (top-k / top-p) have at most 64 entries, which come out of the rows' records (verify_rows.hip, launched in
// front): one workgroup walks a prompt's layers and exchanges nothing (verify_layers_kernel<true>).  Measured, verification
// in us, against layers formed and selected from on up to 256 workgroups: 53 nodes x 128256 58 -> 47, 103 nodes of 3 prompts
// x 50273 88 -> 45, 577 nodes of 16 prompts x 32000 160 -> 104, 28 nodes x 32000 89 -> 46, 248 nodes x 128256 142 -> 126.
#include "common.h"
#include "topology_device.h"
#include "exp_nonpos.h"
#include "slots.h"
#include "verify_rows.h"
#include "wave_f64.h"
#include <type_traits>
#include <float.h>
#include <limits.h>
#include <math.h>
#include <stdlib.h>
#include <algorithm>
#include <atomic>
#include <mutex>

#define VL_BLOCK 512
#define NODE_CAP 512           // nodes of one prompt (all its trees)
#define NEAR_TIE 1.0e-6
#define SYNC_LIMIT_TICKS 300000000LL   // default bound of every wait: 3 s of the 100 MHz wall clock
#define DSBD_STATIC_SCRATCH_BYTES (32u << 20)   // the device array behind dsbd_verify_forest_static
#define CU_LDS_BYTES (160 * 1024)  // LDS of a compute unit (gfx950)
#define XU 4                   // logits per thread and model in flight in the exponential pass (eight, a 4008-entry piece of the
                               // benchmark's joint in one round, cost 256 vector registers)
#define VL_DYN_LDS_BYTES (84 * 1024)   // dynamic LDS of the layer kernel (its static LDS takes most of the rest) ...
#define VL_DYN_LDS_BYTES_SMALL (112 * 1024)   // ... and of its variant for prompts of at most NODE_CAP_SMALL nodes
#define NODE_CAP_SMALL 128
#define VL_LAUNCH_PROMPTS (1 << 22)    // most prompts of a launch with a workgroup each (2^32 threads are the limit)

// ------------------------------------------------------------------------------------------------ row statistics, fp32
// 2^x by the hardware instruction alone: results below 2^-126 come out as zero instead of denormal, which a sum
// of terms relative to the running maximum does not notice (the library routine spends four more instructions
// per logit on that range).
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ void online_add16(float& m, float& s, bool& bad, float4 a, float4 b, float4 c, float4 d) {
  const float L2E = 1.4426950408889634f;
  const float v[16] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w, d.x, d.y, d.z, d.w};
  float bm = v[0];
#pragma unroll
  for (int e = 1; e < 16; ++e) bm = fmaxf(bm, v[e]);
  bool nan = false;
#pragma unroll
  for (int e = 0; e < 16; ++e) nan |= (v[e] != v[e]);
  bad |= nan | !(bm <= FLT_MAX);                     // NaN or +Inf (-Inf: a masked token, probability 0)
  if (bm > m) {
    s *= fast_exp2((m - bm) * L2E);
    m = bm;
  }
  const float ref = m == -INFINITY ? 0.f : m;       // (nothing but masked tokens so far: they add 0, not exp(-Inf + Inf))
  float t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
#pragma unroll
  for (int e = 0; e < 16; e += 4) {
    t0 += fast_exp2((v[e] - ref) * L2E); t1 += fast_exp2((v[e + 1] - ref) * L2E);
    t2 += fast_exp2((v[e + 2] - ref) * L2E); t3 += fast_exp2((v[e + 3] - ref) * L2E);
  }
  s += (t0 + t1) + (t2 + t3);
}

__device__ __forceinline__ void online_add1(float& m, float& s, bool& bad, float x) {
  const float L2E = 1.4426950408889634f;
  bad |= !(x <= FLT_MAX);                            // NaN or +Inf
  if (x > m) {
    s *= fast_exp2((m - x) * L2E);
    m = x;
  }
  s += fast_exp2((x - (m == -INFINITY ? 0.f : m)) * L2E);
}

__device__ __forceinline__ void online_merge(float& m, float& s, float m2, float s2) {
  const float L2E = 1.4426950408889634f;
  const float mn = fmaxf(m, m2);
  if (mn == -INFINITY) { s = 0.f; return; }
  s = s * exp2f((m - mn) * L2E) + s2 * exp2f((m2 - mn) * L2E);
  m = mn;
}

// ------------------------------------------------------------------------------------------------ the kernel
// Where the exchanges of one prompt keep their 16-byte slots (offsets in slots from the prompt's first one).
struct SlotLayout {
  int x[2];              // the two alternating banks of the post-then-collect-from-all exchanges: G lines
  int r, r_w, r_stride;  // row sums of layer l: r + (l - 1) * r_stride, r_w slots per workgroup
  int acc;               // accumulator words of the one-hop sums: 2 banks x NACC lines
  int acc0;              // their values at launch, posted by the prompt's first workgroup: 2 x NACC slots
  int prompt_stride;
};

struct LayersArgs {
  int n_prompts, n_trees, n_nodes;
  const int32_t *tree_prompt, *tree_off, *parent, *token, *rank;
  int max_depth, max_prompt_trees;
  int V;
  const float *zp, *zq;
  const double *blp, *blq;
  const float *u_acc, *u_res, *u_fill;
  int W_L, W_min, W_cap;
  float t;
  int top_k;             // warping T (Section 2.1): keep the top_k largest entries of each joint (0: T is the identity) ...
  float top_p;           // ... then the smallest leading part of those whose share of the kept mass exceeds top_p
  dsbd_verify_out out;
  int prompt0;           // first prompt of this launch (forests of more prompts than fit the device run in groups)
  int max_tree_nodes;
  double* pb;            // [n_prompts][G][slice_cap]  p_beam slice storage, a private region per workgroup
  double* qb;            // the same for q_beam
  long long slice_cap;   // elements of a workgroup's region
  double* red;           // exchange slots of 16 bytes each, n_prompts regions laid out as in `sl`
  SlotLayout sl;
  int G, I_cap;
  long long* trace;      // optional timeline of workgroup trace_wg: pairs (label, 100 MHz wall clock)
  int trace_wg;
  int lds_elems;         // capacity (elements) of each of the two dynamic-LDS slice arrays; 0 = none
  int lds_slice;         // slices of up to this many elements are kept in the LDS (<= lds_elems)
  int alias;             // one model in both roles (same logits, same beam likelihoods): q_beam IS p_beam, kept once
  long long sync_limit;  // bound of every wait, in ticks of the 100 MHz wall clock
  unsigned long long nonce;   // base of this launch's exchange tags: no tag of an earlier launch on the same workspace can match
  const unsigned long long* replay;   // launches recorded into a graph: a word of the workspace that a small kernel in front of
                              // this one counts up at every replay (the arguments, nonce included, repeat); else null
  int mute_wg;           // test hook: this workgroup withholds its first post (-1: none), so that its partners'
                         // bounded waits give up and the error path can be exercised without a hang
  int32_t* fault;
  const char* rec;       // warping: the records of all rows (verify_rows.h), `rec_stride` bytes apart
  long long rec_stride;
  int rec_compact;
  dsbd_next_beams nx;    // next-beam plan written along with the output beams (fused selection) ...
  int nx_on;             // ... when this is set
  int layer_wgs;         // workgroups of this launch that walk layers; those behind them take the statistics of the rows ...
  int stats_threads;     // ... with so many threads per row
  float *lse_p, *lse_q, *logp_p, *logp_q;   // per-node outputs of the statistics (any may be null)
};

#define VL_WAVES (VL_BLOCK / 64)
#define NODE_DEPTH_MASK 0xff   // LayerShared::n_depth: depth of the node (below 64) ...
#define NODE_TREE_SHIFT 8      // ... and, above it, the index of its tree among the prompt's trees (below 64)
#define NACC 8                 // accumulator words of a one-hop sum (see wave_sum_accumulators)
#define ACC_FIELD_BITS 54
static_assert(NODE_CAP <= VL_BLOCK, "one thread per node of a prompt");
static_assert(VL_WAVES == 8, "the fixed reduction trees below are written for eight waves");

// NC: the most nodes a prompt may have (all its trees).  Two sizes are built: what the arrays below do not take of a
// compute unit's LDS is room for the joint slices.
template <int NC>
struct LayerShared {
  // input beams of the layer
  int I_node[64];
  double cum_p[64], cum_q[64];       // cumulative log-likelihoods of the input beams
  double lse_p[64], lse_q[64];       // fp64 log-sum-exp of their logit rows
  double max_p[64], max_q[64];       // exact row maxima
  double lm_p[64], lm_q[64];         // maxima of this workgroup's pieces of its rows (row i_lo first)
  float wmax[2][2 * VL_WAVES];       // per-wave maxima of a piece, two rows in flight
  double sp[64], sq[64];             // beam weight / row sum: p_beam(i,x) = exp(z - max) * sp[i]
  double bw_p[64], bw_q[64];         // beam weights
  // accepted beams of the layer (next layer's inputs): node and its position among the candidates
  int A_node[64], A_idx[64];
  double A_cum_p[64], A_cum_q[64];
  // the prompt's nodes (loaded once: the sequential parts must not wait for global memory)
  int n_parent[NC], n_token[NC], n_rank[NC];
  short n_depth[NC];
  float n_u[NC];               // accept uniform of each node
  // candidates
  short slot_of[NC];           // slot in I of a prompt node, -1 if not an input beam
  int S_node[NC], S_tmp[NC];
  float S_zp[NC], S_zq[NC];   // logits at the candidates' (parent, token)
  double S_pb[NC], S_qb[NC];
  float S_u[NC];               // accept uniform of each candidate
  unsigned char S_flag[NC];    // test against p_beam itself: bit 0 = accepted, bit 1 = near tie
  // residual chain and accept-count table
  double cc[NC + 2], FF[NC + 2];
  union {
    struct { double alpha[NC + 2], first[NC + 2]; } w;   // dynamic width only
    double wpart[64 * VL_WAVES * 2];                                   // per-wave row sums of the exponential pass
  } u;
  double Pa[NC + 2], Pb[NC + 2];
  double wsum[2][VL_WAVES];
  unsigned long long acc_prev[2][NACC];   // the accumulator words' values before their next exchange
  int x_have;                        // the exchange under way is collected (chain entry kx + 1 is in cc / FF)
  int stop;                          // accept loop: the chain entry on its way is not needed, its collection may be left
  unsigned int handed;               // accept loop: wave totals handed to the collecting wave so far
  double scan_w[VL_WAVES], scan_w2[VL_WAVES];
  double tsum[VL_BLOCK];
  double gpart[256];                 // one partial per workgroup of the prompt (G <= 256)
  double ptot[256];                  // p_beam total of every workgroup's slice, worked out from the layer's row sums
  int ptot_ok;                       // ... when every gathering thread saw a single piece (else 0: totals are exchanged)
  double exp_tab[64];                // 2^(j/64)
  double d_target[64];               // sampling: u * total of each draw
  // warped joints (top-k / top-p): union of the two supports, ascending flat index over I x V
  int U_idx[64];
  double U_p[64], U_q[64];
  int nU;
  unsigned long long warp_bound[2];  // bits of a lower bound of the K-th entry of either joint ...
  int warp_kept[2];                  // ... and the entries that reach it
  int last_mass[2];                  // draws: the last workgroup that holds any mass, of either kind of weights
  int state[2];                      // outcome of the decision rounds, alternating entries
  int kmax, counter, abort, found, sbad, sgamma;
  int acc_n, pos, kidx;        // accept loop: accepted so far, next candidate, chain index of p'
  int pick_th;                 // sampling from workspace slices: the thread whose chunk holds the draw
};


static_assert(sizeof(LayerShared<NODE_CAP>) + VL_DYN_LDS_BYTES + 2048 <= CU_LDS_BYTES, "the layer kernel's LDS must fit a compute unit");
static_assert(sizeof(LayerShared<NODE_CAP_SMALL>) + VL_DYN_LDS_BYTES_SMALL + 2048 <= CU_LDS_BYTES, "the layer kernel's LDS must fit a compute unit");

// 2^(j/64), j = 0..63 (exp_nonpos.h)
__constant__ double c_exp2_tab[64] = {DSBD_EXP2_TABLE_64};

__device__ __forceinline__ double exp_nonpos(double x, const double* tab) { return dsbd_exp_nonpos(x, tab); }

// floor(a / b) for 0 <= a, 0 < b, both below 2^52, without the 64-bit integer division sequence
__device__ __forceinline__ long long div_floor(long long a, long long b) {
  long long q = (long long)((double)a / (double)b);
  if (q * b > a) --q;
  else if ((q + 1) * b <= a) ++q;
  return q;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() carries a workgroup-scope fence, for which the
// compiler also drains the wave's outstanding global loads and stores: where the waves exchange nothing but LDS
// values, this form lets the first wave's status stores and slot posts stay in flight across the barrier.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---- exchange among the G workgroups of one prompt
//
// No grid-wide barrier and no cache-wide fence: a workgroup publishes each partial value in its own
// 16-byte slot as two agent-scope atomic words (value bits, value bits XOR tag) and every other
// workgroup polls exactly the slots it needs.  The tag changes with every exchange, so a slot is valid
// only once both words of the current exchange have landed.  A bank of slots is never overwritten while
// somebody may still read it:
//  * the row-sum exchange is collected only from the workgroups that share a row, so each layer has a bank of its own
//    for it, written once per launch;
//  * the accumulator words' values at launch have a bank, written once per launch;
//  * the two sampling prefixes (banks 0 and 1) are the prompt's last exchanges, written once per launch.
// Chain entries travel in the accumulator words below.  Warped layers are walked by one workgroup per prompt and
// exchange nothing.
// Single-value exchanges: workgroup w owns the slot at the start of its own 128-byte line of the bank (slot index
// w * LINE_SLOTS), so that no two workgroups ever write the same cache line.  Measured with a microbenchmark
// on this chip, all-to-all among 256 workgroups: 2.3 us with a line per workgroup, 3.1 us with the words packed
// densely (sixteen writers per line), although the packed layout needs sixteen times fewer lines per poll.
#define LINE_SLOTS 8
__device__ __forceinline__ void dense_post(Slot* bank, int G, int g, double v, unsigned long long tag) {
  (void)G;
  slot_post(bank + (long long)g * LINE_SLOTS, v, tag);
}

// One wave collects the values of all G workgroups (G <= 256): lane i gets those of workgroups i, i + 64, i + 128,
// i + 192 in v[0..3] (0 beyond G), with the loads of a polling round in flight together; `own` is the value this
// workgroup posted.  False if the wait gave up.
__device__ __forceinline__ bool wave_collect4(Slot* bank, int G, int g, double own, unsigned long long tag,
                                              double (&v)[4], long long limit) {
  const int lane = threadIdx.x & 63;
  bool have[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    have[k] = (lane + 64 * k >= G); v[k] = 0.0;
    if (lane + 64 * k == g) { have[k] = true; v[k] = own; }   // the workgroup's own value needs no round trip
  }
  long long t0 = 0;
  for (int spin = 0;; ++spin) {
    unsigned long long w0[4], w1[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      w0[k] = 0; w1[k] = 0;
      if (!have[k]) {
        Slot* s = bank + (long long)(lane + 64 * k) * LINE_SLOTS;
        w0[k] = __hip_atomic_load(&s->w0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        w1[k] = __hip_atomic_load(&s->w1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (!have[k] && (w0[k] ^ w1[k]) == tag) { v[k] = __longlong_as_double((long long)w0[k]); have[k] = true; }
    if (have[0] && have[1] && have[2] && have[3]) return true;
    if (spin == 0) t0 = wall_clock64();
    else if ((spin & 15) == 0 && wall_clock64() - t0 > limit) return false;
    __builtin_amdgcn_s_sleep(1);
  }
}

// Sum over the prompt's G workgroups of one value in [0, 4) each, in one hop: every workgroup adds its value, as a
// 2^-52 fixed-point number with a 1 in the count field above it, to one of NACC accumulator words (an agent-scope
// integer atomic: the order of the additions does not matter, so the sum is the same in every run), and one wave
// polls the NACC words until each has counted all its members.  The accumulators are never cleared: a word only ever
// grows (modulo 2^64), and what an exchange added to it is the difference to the value it had before the exchange,
// which every workgroup knows (the value it read at the end of the word's previous exchange; the values at launch are
// read by the prompt's first workgroup before anybody adds and handed round with the first layer's row sums).  The
// difference decodes as (members << 54) + sum as long as the sum stays below 2^54 units and there are fewer than 1024
// members per word.  Two banks alternate: whoever posts exchange
// n + 2 has collected n + 1, so everybody had posted n + 1 and was therefore done collecting n.  Measured among 256 workgroups: 1.8 us against
// 2.45 us for a two-hop slot exchange (a microbenchmark of both on the same box).
// Posting and collecting are separate, so that an exchange can travel beside other work; every workgroup collects what it
// posted before it posts again (only then has nobody left the bank before the last to be collected).
__device__ __forceinline__ void accumulators_post(unsigned long long* accs, int G, int g, double own) {
  if (G == 1 || (threadIdx.x & 63) != 0) return;
  const unsigned long long q = (unsigned long long)__double2ull_rn(fmin(fmax(own, 0.0), 3.999) * 4503599627370496.0);
  __hip_atomic_fetch_add(&accs[(g % NACC) * 16], (1ull << ACC_FIELD_BITS) + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
enum { ACC_DONE = 0, ACC_TIMEOUT = 1, ACC_STOPPED = 2 };
// One wave.  `stop`: a word of the LDS by which another wave of the workgroup calls the wait off (ACC_STOPPED: the exchange
// is still to be collected); null: none.
__device__ __forceinline__ int accumulators_collect(unsigned long long* accs, unsigned long long* prev, int G, double own,
                                                    long long limit, const int* stop, double& total) {
  const int lane = threadIdx.x & 63;
  if (G == 1) { total = own; return ACC_DONE; }
  unsigned long long field = 0, w = 0;
  bool have = true;
  unsigned long long members = 0, before = 0;
  if (lane < NACC) {
    members = lane < G ? (unsigned long long)((G - lane + NACC - 1) / NACC) : 0ull;
    before = prev[lane];
    have = members == 0;
  }
  long long t0 = 0;
  for (int spin = 0;; ++spin) {
    if (!have) {
      w = __hip_atomic_load(&accs[lane * 16], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const unsigned long long diff = w - before;
      if ((diff >> ACC_FIELD_BITS) == members) { field = diff & ((1ull << ACC_FIELD_BITS) - 1); have = true; }
    }
    if (__builtin_amdgcn_ballot_w64(!have) == 0ull) break;
    if (stop && __hip_atomic_load(stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0) return ACC_STOPPED;
    if (spin == 0) t0 = wall_clock64();
    else if ((spin & 15) == 0 && wall_clock64() - t0 > limit) return ACC_TIMEOUT;
    __builtin_amdgcn_s_sleep(1);
  }
  if (lane < NACC && members) prev[lane] = w;
  // the eight words' fields added up by lane moves inside the SIMD (quads, then the other quad of the eight) and the
  // first lane's total read back as a uniform value: no LDS round trips on the chain's critical path
  static_assert(NACC == 8, "the reduction below is written for eight words");
  field += dpp_move_u64<0xB1>(field);       // quad_perm [1,0,3,2]
  field += dpp_move_u64<0x4E>(field);       // quad_perm [2,3,0,1]
  field += dpp_move_u64<0x141>(field);      // row_half_mirror
  {
    const unsigned int lo = (unsigned int)__builtin_amdgcn_readfirstlane((int)(unsigned int)field);
    const unsigned int hi = (unsigned int)__builtin_amdgcn_readfirstlane((int)(unsigned int)(field >> 32));
    field = ((unsigned long long)hi << 32) | lo;
  }
  total = (double)field * (1.0 / 4503599627370496.0);
  return ACC_DONE;
}

__device__ __forceinline__ Slot* prompt_slots(const LayersArgs& a, int prompt) {
  return reinterpret_cast<Slot*>(a.red) + (long long)prompt * a.sl.prompt_stride;
}

#define WARP_K_MAX VR_K_MAX
__device__ __forceinline__ double readlane_f64(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l), hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}
// The value of the lane below (lane 0: 0.0).
__device__ __forceinline__ double lane_from_below(double v) { return dpp_move_f64<0x138, 0xf>(v); }      // wave_shr:1

// How a layer's joint over nI rows of V entries is cut among G workgroups (host and device use the same rule).
struct SliceCut {
  int rows_per_wg;       // > 0: every workgroup takes this many whole rows (nI >= G)
  int wg_per_row;        // else: every row is cut into this many pieces of `len` entries (the last ones may be empty)
  long long len;         // entries of the longest slice
};
__host__ __device__ inline SliceCut slice_cut(int nI, int V, int G) {
  SliceCut c;
  if (nI >= G) {
    c.rows_per_wg = (nI + G - 1) / G; c.wg_per_row = 0; c.len = (long long)c.rows_per_wg * V;
  } else {
    c.rows_per_wg = 0; c.wg_per_row = G / nI;
    c.len = (long long)((((unsigned int)V + c.wg_per_row - 1) / c.wg_per_row + 1) & ~1u);      // (V is at most 2^30)
  }
  return c;
}

// ---- per-node outputs (step A3 of the path: fp32 log-sum-exp of a node's row, log-probability of a node's token under its
// parent's row): the workgroups behind the layers' take the rows of both models.  A row's sum is complete inside its
// workgroup, so the log-probabilities of the row's children are its to write, and nothing has to be merged afterwards.
// (Before, a kernel per chunk of a row and a merging kernel ran on a second stream, forked from and joined to the
// caller's by events: 12 us of a call, 33 us of host time in four event calls and two launches, and exchanges that slowed
// down on every compute unit the two shared.  Measured, verification call: 28 nodes x 32000 tokens 50 -> 38 us, 120 nodes
// 75 -> 64 us, 248 nodes x 128256 123 -> 96 us, 16 prompts with 747 nodes x 32000 208 -> 188 us.)
// TR threads take a row, so a workgroup has VL_BLOCK / TR rows side by side.
#define SU 8                   // 16-byte loads in flight per thread, twice (the next round travels during this one's exponentials)
template <int TR, class Shared>
__device__ __forceinline__ void row_statistics(const LayersArgs& a, Shared& sh) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x % TR;
  const int V = a.V;
  const int rows = a.n_nodes * (a.alias ? 1 : 2);
  int item = ((int)blockIdx.x - a.layer_wgs) * (VL_BLOCK / TR) + (int)threadIdx.x / TR;
  const bool live = item < rows;           // (the last workgroup may have threads left over: they repeat the last row)
  item = min(item, rows - 1);
  const bool second = !a.alias && (item & 1);
  const int n = a.alias ? item : item >> 1;
  const float* const row = (second ? a.zq : a.zp) + (long long)n * V;
  float m = -INFINITY, s = 0.f;
  bool bad = false;
  const int head = min((int)(((16 - (reinterpret_cast<uintptr_t>(row) & 15)) & 15) >> 2), V);
  const int body4 = (V - head) >> 2, tail0 = head + 4 * body4;
  const f32x4* const r4 = reinterpret_cast<const f32x4*>(row + head);
  f32x4 nx[SU];
  auto request = [&](int i) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < SU; ++k) nx[k] = __builtin_nontemporal_load(&r4[min(i + k * TR, body4 - 1)]);
  };
  if (tid < body4) request(tid);
  // children: nodes of the same tree, behind this one, no further than a tree is long
  const int c = n + tid;
  const bool child = tid >= 1 && tid < DSBD_MAX_TREE_NODES && c < a.n_nodes && a.parent[c] == n;
  const int par = a.parent[n], tok = a.token[n];
  if (tid < head) online_add1(m, s, bad, row[tid]);
  if (tail0 + tid < V) online_add1(m, s, bad, row[tail0 + tid]);
  for (int i = tid; i < body4; i += SU * TR) {
    f32x4 y[SU];
#pragma unroll
    for (int k = 0; k < SU; ++k) y[k] = nx[k];
    if (i + SU * TR < body4) request(i + SU * TR);
#pragma unroll
    for (int k = 0; k < SU; k += 4) {
      float4 x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {     // (places beyond the end are masked tokens: they change neither maximum nor sum, and a
                                        // row of nothing else keeps its maximum of -Inf, by which it is found below)
        const bool in = i + (k + e) * TR < body4;
        x[e] = in ? make_float4(y[k + e].x, y[k + e].y, y[k + e].z, y[k + e].w) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      }
      online_add16(m, s, bad, x[0], x[1], x[2], x[3]);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const float m2 = __shfl_xor(m, off), s2 = __shfl_xor(s, off);
    online_merge(m, s, m2, s2);
  }
  bad = __ballot(bad) != 0ull;
  if constexpr (TR > 64) {
    float2* const part = reinterpret_cast<float2*>(sh.tsum);
    const int wave = threadIdx.x >> 6, first = (int)threadIdx.x / TR * (TR / 64);
    if ((threadIdx.x & 63) == 0) { part[2 * wave] = make_float2(m, s); part[2 * wave + 1].x = bad ? 1.f : 0.f; }
    __syncthreads();
    m = part[2 * first].x; s = part[2 * first].y; bad = part[2 * first + 1].x != 0.f;
#pragma unroll
    for (int w = 1; w < TR / 64; ++w) {
      online_merge(m, s, part[2 * (first + w)].x, part[2 * (first + w)].y);
      bad |= part[2 * (first + w) + 1].x != 0.f;
    }
  }
  if (!live) return;
  const float lse = m + logf(s);
  float* const o_lse = second ? a.lse_q : a.lse_p;
  float* const o_logp = second ? a.logp_q : a.logp_p;
  int fault = 0;
  if (tid == 0) {
    if (o_lse) o_lse[n] = lse;
    if (a.alias && a.lse_q) a.lse_q[n] = lse;
    if (bad || lse == -INFINITY) fault = DSBD_FAULT_NONFINITE;         // NaN or +Inf; a row without a finite logit
    if (!(par >= 0 && par < n && n - par < DSBD_MAX_TREE_NODES && tok >= 0 && tok < V)) {      // a root (or a node reported elsewhere)
      if (o_logp) o_logp[n] = 0.f;
      if (a.alias && a.logp_q) a.logp_q[n] = 0.f;
    }
  }
  if (child) {
    const int ct = a.token[c];
    if (ct >= 0 && ct < V) {
      const float zt = row[ct];
      if (zt == -INFINITY) fault = DSBD_FAULT_NONFINITE;               // a drafted token masked in its parent's row
      if (o_logp) o_logp[c] = zt - lse;
      if (a.alias && a.logp_q) a.logp_q[c] = zt - lse;
    }
  }
  if (fault) atomicOr(a.fault, fault);
}

// At most VL_MAX_VGPRS vector registers.  (The attribute counts in halves of the unified register file of this target:
// the compiler doubles the number it is given.  Without it the allocator takes whatever two waves per SIMD leave it, up
// to 256, whether it needs them or not.)
#define VL_MAX_VGPRS 240
// BARE: the rows' records hold no entries (RowsPlan::compact < 0); a build of its own, whose registers the other's place for two
// workgroups on a compute unit would not survive.
template <bool WARP, int NC, bool BARE = false>
__global__ __launch_bounds__(VL_BLOCK) __attribute__((amdgpu_num_vgpr(VL_MAX_VGPRS / 2)))
void verify_layers_kernel(LayersArgs a) {
  __shared__ LayerShared<NC> sh;
  extern __shared__ __attribute__((aligned(16))) double dyn_lds[];
  if (!WARP && (int)blockIdx.x >= a.layer_wgs) {
    if (a.stats_threads == 64) row_statistics<64>(a, sh);
    else if (a.stats_threads == 128) row_statistics<128>(a, sh);
    else if (a.stats_threads == 256) row_statistics<256>(a, sh);
    else row_statistics<VL_BLOCK>(a, sh);
    return;
  }
  const int prompt = a.prompt0 + blockIdx.x / a.G;
  const int g = blockIdx.x % a.G;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int V = a.V;
  unsigned int epoch = 0;      // exchanges so far (sets the tag); identical in every workgroup of the prompt
  Slot* const slots = WARP ? nullptr : prompt_slots(a, prompt);      // (one workgroup walks a prompt's warped layers: no exchanges)
  // (a replayed launch: the replay count, which the kernel in front of this one has just raised, sets the tags apart
  // from those of the graph's earlier replays)
  const unsigned long long nonce =
      a.nonce + (a.replay ? (__hip_atomic_load(a.replay, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) << 40) : 0ull);
  // (selected, not indexed: a run-time index into the kernel's argument block would move the whole block into scratch memory)
  const int slx0 = a.sl.x[0], slx1 = a.sl.x[1];
  unsigned int wsum_round = 0; // alternates the two wsum buffers
  unsigned int decide_round = 0;
  int trace_n = 0;
  auto stamp = [&](int label) {
    if (a.trace && (int)blockIdx.x == a.trace_wg && tid == 0 && trace_n < 255) {
      a.trace[2 * trace_n + 2] = label; a.trace[2 * trace_n + 3] = wall_clock64(); ++trace_n; a.trace[0] = trace_n;
    }
  };
  stamp(0);

  // the accumulator words of the one-hop sums as the launch finds them: read by the prompt's first workgroup before
  // anybody adds to them (nobody does before the first layer's row sums, which wait for this workgroup's), and handed
  // to the others in tagged slots, collected during the first layer
  unsigned long long* const accs = reinterpret_cast<unsigned long long*>(slots + a.sl.acc);
  const unsigned long long acc0_tag = exchange_tag(nonce + 0xFFFFFFull);
  unsigned int achg = 0;       // accumulator exchanges posted so far (alternates their two banks)
  bool x_open = false;         // the last of them is not known to be collected by every workgroup
  double x_own = 0.0;          // what this workgroup posted in it
  unsigned int handovers = 0;  // rounds of the accept loop's handing over of wave totals
  // (requested here, used at the end of the prologue: the round trip through the memory system runs beside it)
  unsigned long long acc0_w = 0;
  if (!WARP && g == 0 && tid < 2 * NACC)
    acc0_w = __hip_atomic_load(&accs[tid * 16], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  if (tid == 0) { sh.abort = 0; sh.sbad = 0; sh.sgamma = 0; sh.counter = 0; sh.found = 0; sh.handed = 0u; }
  double exp_tab_mine = 0.0;     // (the table entry travels while the prompt's trees are looked up; stored below)
  if (tid < 64) exp_tab_mine = c_exp2_tab[tid];

  // ---- trees and nodes of this prompt.  tree_prompt is non-decreasing: the prompt's trees are those behind the
  // trees of earlier prompts.  (Everything the kernel needs it derives from the call's inputs: it does not wait for
  // the statistics, which run beside it.)
  int t_first = 0, t_end = a.n_trees;
  if (a.n_prompts > 1) {
    __syncthreads();
    int lt = 0, le = 0;
    for (int t = tid; t < a.n_trees; t += VL_BLOCK) {
      const int tp = a.tree_prompt[t];
      lt += tp < prompt; le += tp <= prompt;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) { lt += __shfl_xor(lt, off); le += __shfl_xor(le, off); }
    if (lane == 0) { atomicAdd(&sh.counter, lt); atomicAdd(&sh.found, le); }
    __syncthreads();
    t_first = sh.counter; t_end = sh.found;
  }
  stamp(2);
  int n_roots = t_end - t_first;
  int bad = 0;
  if (n_roots < 0) { bad |= DSBD_FAULT_TOPOLOGY; n_roots = 0; }
  if (n_roots > a.max_prompt_trees || n_roots > a.I_cap || n_roots > 64) { bad |= DSBD_FAULT_BOUNDS; n_roots = 0; }
  int n_begin = 0, n_end = 0;
  if (n_roots > 0) { n_begin = a.tree_off[t_first]; n_end = a.tree_off[t_end]; }
  if (n_begin < 0 || n_end > a.n_nodes || n_end < n_begin) { bad |= DSBD_FAULT_TOPOLOGY; n_roots = 0; }
  if (n_end - n_begin > NC) { bad |= DSBD_FAULT_BOUNDS; n_roots = 0; }
  int n_pn = n_roots > 0 ? n_end - n_begin : 0;          // nodes of the prompt
  const int Lw = a.max_depth + 2;                        // row length of the per-layer arrays
  stamp(3);
  __syncthreads();
  if (tid < n_roots) {                                   // every tree inside the prompt's node range
    const int b = t_first + tid;
    const int r0 = a.tree_off[b], r1 = a.tree_off[b + 1];
    if (r0 < n_begin || r1 > n_end || r1 <= r0) atomicOr(&sh.sbad, DSBD_FAULT_TOPOLOGY);
    sh.I_node[tid] = r0;
    sh.cum_p[tid] = a.blp[b];
    sh.cum_q[tid] = a.blq[b];
  }
  if (tid < n_pn) {
    const int n = n_begin + tid;
    int tok = a.token[n];
    if (tok < 0 || tok >= V) { atomicOr(&sh.sbad, DSBD_FAULT_TOKEN); tok = 0; }
    sh.n_parent[tid] = a.parent[n];
    sh.n_token[tid] = tok;
    sh.n_rank[tid] = a.rank ? a.rank[n] : 0;
    sh.n_u[tid] = a.u_acc[n];
    sh.slot_of[tid] = -1;
    sh.S_tmp[tid] = 0;
  }
  if (tid < 64) sh.exp_tab[tid] = exp_tab_mine;
  __syncthreads();
  stamp(4);
  if (sh.sbad & DSBD_FAULT_TOPOLOGY) { n_roots = 0; n_pn = 0; }
  // this workgroup's share of I x V, as a function of the number of rows (worked out when that changes; 32-bit
  // divisions only: as five 64-bit ones it took 1.3 us)
  int geo_nI = -1, geo_ilo = 0, geo_ihi = -1, geo_pieces = 1;
  SliceCut geo_cut = {0, 1, 0};
  long long geo_lo = 0, geo_hi = 0;
  auto set_geometry = [&](int rows_) {
    const int rows = __builtin_amdgcn_readfirstlane(rows_);
    if (rows == geo_nI) return;
    geo_nI = rows;
    geo_cut = slice_cut(rows, V, a.G);
    int lo = 0, hi = 0;                                  // this workgroup's entries of row geo_ilo (pieces)
    if (geo_cut.rows_per_wg > 0) {
      const int first = min(rows, g * geo_cut.rows_per_wg), last = min(rows, first + geo_cut.rows_per_wg);
      geo_ilo = first; geo_ihi = last - 1; geo_pieces = 1;
      geo_lo = (long long)first * V; geo_hi = (long long)last * V;
      return;
    }
    geo_pieces = (int)(((unsigned int)V + (unsigned int)geo_cut.len - 1u) / (unsigned int)geo_cut.len);
    geo_ilo = min(rows, (int)((unsigned int)g / (unsigned int)geo_cut.wg_per_row));
    if (geo_ilo < rows) {
      const int k = g - geo_ilo * geo_cut.wg_per_row;
      lo = (int)min((long long)V, k * geo_cut.len);
      hi = (int)min((long long)V, (k + 1) * geo_cut.len);
    }
    geo_ihi = hi > lo ? geo_ilo : geo_ilo - 1;
    geo_lo = (long long)geo_ilo * V + lo;
    geo_hi = (long long)geo_ilo * V + hi;
  };
  // The first two rounds of logits of this workgroup's first row of a layer, requested as soon as the layer's rows are
  // known; the book-keeping that needs no logits runs while they travel (its barriers order the LDS only).
  float eA_p[XU], eA_q[XU], eB_p[XU], eB_q[XU];
  bool early = false;
#pragma unroll
  for (int k = 0; k < XU; ++k) { eA_p[k] = 0.f; eA_q[k] = 0.f; eB_p[k] = 0.f; eB_q[k] = 0.f; }
  auto request_first = [&](const int* row_nodes) __attribute__((always_inline)) {
    if constexpr (WARP) return;
    early = geo_ihi >= geo_ilo;
    if (!early) return;
    const int i = geo_ilo;
    const int node = row_nodes[i];
    const int x_lo = (int)(max(geo_lo, (long long)i * V) - (long long)i * V);
    const int x_hi = (int)(min(geo_hi, (long long)(i + 1) * V) - (long long)i * V);
    const float* zp = a.zp + (long long)node * V;
    const float* zq = a.zq + (long long)node * V;
    const int xA = x_lo + tid, xB = xA + XU * VL_BLOCK;
#pragma unroll
    for (int k = 0; k < XU; ++k) {
      const int xx = min(xA + k * VL_BLOCK, x_hi - 1);
      eA_p[k] = zp[xx]; eA_q[k] = zq[xx];
    }
#pragma unroll
    for (int k = 0; k < XU; ++k) {
      const int xx = min(xB + k * VL_BLOCK, x_hi - 1);
      eB_p[k] = zp[xx]; eB_q[k] = zq[xx];
    }
  };
  if (n_roots > 0) {
    set_geometry(n_roots);
    request_first(sh.I_node);
  }
  // node depths (and the validation of the parent pointers): one wave per tree walks the parent chains with lane
  // shuffles over the entries already in the LDS; depths land in S_tmp (prompt-local index)
  for (int b = wave; b < n_roots; b += VL_WAVES) {
    dsbd_tree_range t;
    t.base = sh.I_node[b];
    t.n_all = (b + 1 < n_roots ? sh.I_node[b + 1] : n_end) - t.base;
    t.n = min(t.n_all, min(a.max_tree_nodes, DSBD_MAX_TREE_NODES));
    t.bad = t.n_all > t.n ? DSBD_FAULT_BOUNDS : 0;
    t.valid = true;
    const int p_mine = lane < t.n ? sh.n_parent[t.base - n_begin + lane] : -1;
    const int fb = dsbd_tree_walk(t, lane, p_mine, a.max_depth, reinterpret_cast<int32_t*>(sh.S_tmp) - n_begin, nullptr, nullptr);
    if (fb) atomicOr(&sh.sbad, fb);
    // the tree's deepest node: the wave's maximum by lane exchanges, one LDS atomic per tree (an atomic per node, all
    // on one word, took 2 us on a prompt of 248 nodes)
    wave_lds_fence();
    const int d_mine = lane < t.n ? sh.S_tmp[t.base - n_begin + lane] : 0;
    int d = d_mine;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) d = max(d, __shfl_xor(d, off));
    if (lane == 0 && d > 0) atomicMax(&sh.sgamma, d);
    // (the node's tree within the prompt rides in the bits above its depth: the next-beam plan names it)
    if (lane < t.n) sh.S_tmp[t.base - n_begin + lane] = (d_mine & NODE_DEPTH_MASK) | (b << NODE_TREE_SHIFT);
  }
  lds_barrier();
  if (tid < n_pn) sh.n_depth[tid] = (short)sh.S_tmp[tid];      // (read after later barriers only)
  stamp(5);
  bad |= sh.sbad;
  const int gamma = min(sh.sgamma, a.max_depth);
  if (bad && g == 0 && tid == 0) atomicOr(a.fault, bad);

  // ---- initial statuses (first workgroup of the prompt)
  if (g == 0) {
    if (tid < n_pn) a.out.node_status[n_begin + tid] = (sh.n_depth[tid] & NODE_DEPTH_MASK) == 0 ? DSBD_ROOT : DSBD_NOT_REACHED;
    for (int i = tid; i < Lw; i += VL_BLOCK) a.out.layer_width[(long long)prompt * Lw + i] = i == 0 ? n_roots : 0;
  }
  // Output words are written by exactly one workgroup each (sampled beams by the workgroup that owns the
  // sample, per-node log-probabilities by the node's workgroup, everything else by the prompt's first
  // workgroup): the XCDs' L2 caches are not coherent with each other, so two workgroups must never write
  // the same word.
  const int plan_len = a.max_depth + 1;                   // row length of the plan's paths
  auto clear_out_slots = [&](int from) {
    for (int i = from + tid; i < a.W_cap; i += VL_BLOCK) {
      const long long o = (long long)prompt * a.W_cap + i;
      a.out.out_parent[o] = -1; a.out.out_token[o] = -1; a.out.out_node[o] = -1;
      a.out.out_logp_target[o] = 0.0; a.out.out_logp_draft[o] = 0.0;
      if (a.nx_on) {
        a.nx.src_tree[o] = -1; a.nx.src_out[o] = -1; a.nx.path_len[o] = 0; a.nx.token[o] = -1;
        a.nx.logp_target[o] = 0.0; a.nx.logp_draft[o] = 0.0;
        for (int k = 0; k < plan_len; ++k) a.nx.path[o * plan_len + k] = -1;
      }
    }
  };
  // Fused selection (Algorithm 1's return; Section 3.3, last paragraph): whoever writes output beam j of the prompt
  // also writes its entry of the next-beam plan: the tree whose cache it continues and the nodes root .. `node`
  // (the beam's last forest node), root first, read off the parent entries in the LDS.  One thread per beam.
  auto emit_next = [&](int j, int node, int x, double lp, double lq) {
    if (!a.nx_on) return;
    const long long o = (long long)prompt * a.W_cap + j;
    const int dt = sh.n_depth[node - n_begin];
    const int d = min(dt & NODE_DEPTH_MASK, a.max_depth);
    int32_t* const path = a.nx.path + o * plan_len;
    int cur = node;
    for (int k = d; k >= 0; --k) {
      path[k] = cur;
      cur = k > 0 ? sh.n_parent[cur - n_begin] : cur;
    }
    for (int k = d + 1; k < plan_len; ++k) path[k] = -1;
    a.nx.src_tree[o] = t_first + (dt >> NODE_TREE_SHIFT);
    a.nx.src_out[o] = j;
    a.nx.path_len[o] = d + 1;
    a.nx.token[o] = x;
    a.nx.logp_target[o] = lp;
    a.nx.logp_draft[o] = lq;
  };
  if (n_roots == 0) {
    if (g == 0) clear_out_slots(0);
    if (g == 0 && tid == 0) {
      a.out.l_last[prompt] = 0; a.out.n_out[prompt] = 0; a.out.near_tie_count[prompt] = 0;
      if (a.nx_on) a.nx.n_next[prompt] = 0;
    }
    return;   // uniform over the prompt's workgroups: nobody waits for a missing partner
  }

  const int W_in = a.W_L > 0 ? a.W_L : n_roots;
  const bool dynamic = a.t >= 0.f;
  const double thr = (double)a.t;
  // Slices that do not fit the LDS live in the workspace, each workgroup's in a region of its own: the layers
  // cut I x V differently, and an address written by workgroups of two XCDs in turn (whose L2 caches write back
  // in no particular order) could later be read back stale.
  double* pb = a.pb + (long long)blockIdx.x * a.slice_cap;
  double* qb = a.qb + (long long)blockIdx.x * a.slice_cap;
  const float* u_res = a.u_res + (long long)prompt * Lw;
  const float* u_fill = a.u_fill + (long long)prompt * Lw * a.W_cap;

  // ---- layer 1 inputs: the roots
  if (tid < n_roots) sh.slot_of[sh.I_node[tid] - n_begin] = (short)tid;
  int nI = n_roots;
  int near_tie = 0;          // meaningful in thread 0
  int l_last = gamma + 1;
  int n_out = 0;
  if (!WARP && g == 0 && tid < 2 * NACC) {
    (&sh.acc_prev[0][0])[tid] = acc0_w;
    slot_post(slots + a.sl.acc0 + tid, __longlong_as_double((long long)acc0_w), acc0_tag);
  }
  lds_barrier();
  stamp(6);

  // total over the workgroup of one value per thread: valid in every thread after the barrier inside
  auto wg_total = [&](double s, bool lds_only = false) -> double {
    s = wave_sum(s);
    double* ws = sh.wsum[wsum_round & 1];
    wsum_round += 1;
    if (lane == 0) ws[wave] = s;
    if (lds_only) lds_barrier(); else __syncthreads();
    return ((ws[0] + ws[1]) + (ws[2] + ws[3])) + ((ws[4] + ws[5]) + (ws[6] + ws[7]));
  };
  auto give_up = [&]() { sh.abort = 1; atomicOr(a.fault, DSBD_FAULT_SYNC_TIMEOUT); };

  int passed_nacc = -1;      // >= 0: the layer before passed with this many accepted beams, not yet handed over

  stamp(1);
  for (int l = 1; l <= gamma + 1; ++l) {
    stamp(10 + l);
    // The layer before passed: its accepted beams are this layer's inputs.
    if (passed_nacc >= 0) {
      const int nacc = passed_nacc;
      passed_nacc = -1;
      set_geometry(nacc);
      request_first(sh.A_node);
      // cumulative likelihoods of the accepted beams (fp64)
      if (tid < nacc) {
        const int n = sh.A_node[tid];
        const int ci = sh.A_idx[tid];
        const int slot = sh.slot_of[sh.n_parent[n - n_begin] - n_begin];
        sh.A_cum_p[tid] = sh.cum_p[slot] + ((double)sh.S_zp[ci] - sh.lse_p[slot]);
        sh.A_cum_q[tid] = sh.cum_q[slot] + ((double)sh.S_zq[ci] - sh.lse_q[slot]);
      }
      lds_barrier();
      // (no barrier between the next two steps: the old inputs and the new ones are nodes of different depths, so
      // their slot_of entries are different words, and thread t reads I_node[t] before it alone overwrites it)
      if (tid < nI) sh.slot_of[sh.I_node[tid] - n_begin] = -1;
      if (tid < nacc) {
        const int i = sh.A_node[tid] - n_begin;
        sh.I_node[tid] = sh.A_node[tid];
        sh.cum_p[tid] = sh.A_cum_p[tid];
        sh.cum_q[tid] = sh.A_cum_q[tid];
        sh.slot_of[i] = (short)tid;
      }
      nI = nacc;
      lds_barrier();
    }
    const bool bonus = (l == gamma + 1);
    const long long total = (long long)nI * V;           // elements of I x V
    // I x V is cut along the rows: with fewer rows than workgroups every row is cut into the same pieces (the
    // workgroups left over idle for the layer), otherwise every workgroup takes whole rows.  Either way a row's
    // sum is formed in an order that depends on the row's length only, so beams with equal logits and equal
    // likelihoods (duplicates are common in beam sampling) get bitwise equal joint entries, and the order of
    // equal entries (by index) is the same as in a plain row-by-row evaluation.
    set_geometry(nI);
    const SliceCut cut = geo_cut;
    const long long ch = cut.len;            // the longest slice of the layer
    const long long e_lo = geo_lo, e_hi = geo_hi;
    const long long len = e_hi - e_lo;
    const int i_lo = geo_ilo, i_hi = geo_ihi;
    // slice storage: the leading n_lds entries of the slice in the LDS (no memory latency in the dependent passes, and
    // no traffic: a batch of prompts whose slices all lived in the workspace re-read them through the memory system
    // a dozen times per layer), what does not fit behind them in the workspace
    const long long n_lds = min(len, (long long)a.lds_slice);
    const bool in_lds = n_lds == len;
    // Accessors with explicit address spaces (LDS or global): through generic pointers the compiler merges the two
    // cases into one FLAT access with a selected address, which is slower than either.
    typedef __attribute__((address_space(3))) double lds_f64;
    typedef __attribute__((address_space(1))) double glb_f64;
    lds_f64* const pl = (lds_f64*)dyn_lds;
    lds_f64* const ql = a.alias ? pl : pl + a.lds_elems;
    glb_f64* const pbg = (glb_f64*)pb;
    glb_f64* const qbg = a.alias ? pbg : (glb_f64*)qb;
    auto ldp = [&](long long j) -> double { double v; if (j < n_lds) v = pl[(int)j]; else v = pbg[j]; return v; };
    auto ldq = [&](long long j) -> double { double v; if (j < n_lds) v = ql[(int)j]; else v = qbg[j]; return v; };
    // The hot loops are written once, over a range [r0, r1) of the slice, and instantiated for both homes, with the
    // choice taken outside the loop (left per access, it becomes a pair of branches around every load and store).
    auto with_slices = [&](auto&& body) __attribute__((always_inline)) {
      if (in_lds) { body(pl, ql, 0LL, len); return; }
      if (n_lds > 0) body(pl, ql, 0LL, n_lds);
      body(pbg, qbg, n_lds, len);
    };

    // warping: entry r of row i's record of model m, for the thread's first place among 2 x nI x K
    RowHead rec_head = {1.0, 0.f, 0};
    RowEntry rec_entry = {0.f, 0};
    auto row_record = [&](int node, int m, int r, RowHead& h, RowEntry& e) {
      const char* const at = a.rec + (a.alias ? (long long)node : 2LL * node + m) * a.rec_stride;
      h = *reinterpret_cast<const RowHead*>(at);
      if (a.rec_compact) {
        if (r >= h.n % VR_ROW_BAD) e.x = 0;
        else if (a.rec_compact == 1) e.x = reinterpret_cast<const uint8_t*>(at + sizeof(RowHead))[r];
        else e.x = reinterpret_cast<const uint16_t*>(at + sizeof(RowHead))[r];
        e.z = (m ? a.zq : a.zp)[(long long)node * V + e.x];
      } else {
        e = reinterpret_cast<const RowEntry*>(at + sizeof(RowHead))[min(r, V - 1)];     // (a record has room for min(K, V); places behind its n entries are not used)
      }
    };
    if constexpr (WARP) {
      const int n_cand = nI * a.top_k;
      if (!BARE && tid < 2 * n_cand) {
        const int m = tid >= n_cand ? 1 : 0, e = tid - m * n_cand;
        row_record(sh.I_node[e / a.top_k], m, e % a.top_k, rec_head, rec_entry);
      }
    }
    // a chain entry of the layer before that nobody needed: collected now (by the wave that does nothing else here), so
    // that the words' values are known when the next exchange is posted
    if (x_open) {
      if (wave == 1 && sh.x_have == 0) {
        double unused;
        const unsigned int at = achg - 1;
        if (accumulators_collect(accs + (size_t)(at & 1) * NACC * 16, sh.acc_prev[at & 1], a.G, x_own, a.sync_limit, nullptr, unused) != ACC_DONE)
          give_up();
      }
      x_open = false;
    }
    // ===== while the first logits travel: candidates = depth-l nodes whose parent is an input beam, in (rank, node) order
    // (this and the beam weights stood behind the exponential pass, beside the wait for the row sums, and were longer
    // than that wait)
    int M = 0;
    float czp = 0.f, czq = 0.f;
    if (!bonus) {
      if (tid == 0) sh.counter = 0;
      lds_barrier();
      if (tid < n_pn && (sh.n_depth[tid] & NODE_DEPTH_MASK) == l) {
        const int n = n_begin + tid;
        const int par = sh.n_parent[tid];
        const bool cand = par >= n_begin && par < n && sh.slot_of[par - n_begin] >= 0;
        if (cand) {
          const int at = atomicAdd(&sh.counter, 1);
          sh.S_tmp[at] = n;
          sh.S_zp[at] = __int_as_float(sh.n_rank[tid]);        // (its logits are stored there later)
        } else if (g == 0) {
          a.out.node_status[n] = DSBD_PRUNED;
        }
      }
      lds_barrier();
      M = __builtin_amdgcn_readfirstlane(sh.counter);
      if (tid < M) {
        const int n = sh.S_tmp[tid], rk = __float_as_int(sh.S_zp[tid]);
        int pos = 0;
#pragma unroll 8
        for (int j = 0; j < M; ++j) {
          const int n2 = sh.S_tmp[j], rk2 = __float_as_int(sh.S_zp[j]);
          pos += (int)(rk2 < rk) | ((int)(rk2 == rk) & (int)(n2 < n));
        }
        sh.S_node[pos] = n;
      }
    }
    // ===== beside them the beam weights = softmax of the cumulative likelihoods over I (Section 2.1), by one wave
    if (wave == VL_WAVES - 1) {
      const bool valid = lane < nI;
      const double cp = sh.cum_p[min(lane, nI - 1)], cq = sh.cum_q[min(lane, nI - 1)];
      const double mp = wave_max_f64(cp), mq = wave_max_f64(cq);
      const double ep = valid ? exp_nonpos(cp - mp, sh.exp_tab) : 0.0;
      const double eq = valid ? exp_nonpos(cq - mq, sh.exp_tab) : 0.0;
      const double zp = wave_sum(ep), zq = wave_sum(eq);
      if (valid) { sh.bw_p[lane] = ep / zp; sh.bw_q[lane] = eq / zq; }
      // no beam of the layer with a likelihood above 0 under one of the models (stored likelihoods of -Inf), or a
      // likelihood that is no number: the joint is 0/0
      const bool lost = !(mp > -INFINITY && mp < INFINITY && mq > -INFINITY && mq < INFINITY) || __ballot(cp != cp || cq != cq) != 0ull;
      if (lost && g == 0 && lane == 0) atomicOr(a.fault, DSBD_FAULT_NONFINITE);
    }
    if (!bonus) {
      lds_barrier();
      if (tid < M) {      // logits at the candidate's (parent beam, token): in flight until the candidates are tested
        const int n = sh.S_node[tid];
        const int par = sh.n_parent[n - n_begin];
        const int tok = sh.n_token[n - n_begin];
        czp = a.zp[(long long)par * V + tok];
        czq = a.zq[(long long)par * V + tok];
      }
    }

    double f1 = 0.0;                         // this thread's part of F(1) = sum max(p_beam - q_beam, 0) (second entry of the chain)
    if constexpr (!WARP) {
    // ===== p_beam / q_beam over I x V: exponentials and this workgroup's share of the row sums.  The exponentials
    // are taken against the maximum of the workgroup's own piece of the row (found here, in the same pass over the
    // logits); the pieces' maxima travel with their sums and are folded into the row's maximum and total below.
    for (int i = i_lo; i <= i_hi; ++i) {
      const int node = sh.I_node[i];
      const int x_lo = (int)(max(e_lo, (long long)i * V) - (long long)i * V);      // positions in the row: below V < 2^30
      const int x_hi = (int)(min(e_hi, (long long)(i + 1) * V) - (long long)i * V);
      const float* zp = a.zp + (long long)node * V;
      const float* zq = a.zq + (long long)node * V;
      double s_p = 0.0, s_q = 0.0;
      const long long joff = (long long)i * V - e_lo;
      auto exp_pass = [&](auto store) __attribute__((always_inline)) {
      // the first two rounds of XU logits per model stay in registers (a 4008-entry piece of the benchmark's joint is
      // two rounds); longer pieces are read a second time (from the caches)
      float fpA[XU], fqA[XU], fpB[XU], fqB[XU];
      float lmp = -INFINITY, lmq = -INFINITY;
      const int xA = x_lo + tid, xB = xA + XU * VL_BLOCK;
      const bool haveB = x_lo + XU * VL_BLOCK < x_hi;                      // uniform over the workgroup
      if (early && i == i_lo) {            // requested at the top of the layer
#pragma unroll
        for (int k = 0; k < XU; ++k) { fpA[k] = eA_p[k]; fqA[k] = eA_q[k]; fpB[k] = eB_p[k]; fqB[k] = eB_q[k]; }
      } else {
#pragma unroll
        for (int k = 0; k < XU; ++k) {
          const int xx = min(xA + k * VL_BLOCK, x_hi - 1);              // clamped repeats do not change a maximum
          fpA[k] = zp[xx]; fqA[k] = zq[xx];
        }
#pragma unroll
        for (int k = 0; k < XU; ++k) {
          const int xx = min(xB + k * VL_BLOCK, x_hi - 1);
          fpB[k] = zp[xx]; fqB[k] = zq[xx];
        }
      }
      bool nonfinite = false;        // (the row statistics report these for every row; the layers for the rows they use)
#pragma unroll
      for (int k = 0; k < XU; ++k) {
        lmp = fmaxf(fmaxf(lmp, fpA[k]), fpB[k]); lmq = fmaxf(fmaxf(lmq, fqA[k]), fqB[k]);
        nonfinite |= !(fpA[k] <= FLT_MAX) | !(fqA[k] <= FLT_MAX) | !(fpB[k] <= FLT_MAX) | !(fqB[k] <= FLT_MAX);     // NaN or +Inf (-Inf: a masked token)
      }
      // (the rest of a long piece: maxima only, so four times as many logits in flight as in the rounds above)
      for (int x = xB + XU * VL_BLOCK; x < x_hi; x += 4 * XU * VL_BLOCK) {
        float fp[4 * XU], fq[4 * XU];
#pragma unroll
        for (int k = 0; k < 4 * XU; ++k) {
          const int xx = min(x + k * VL_BLOCK, x_hi - 1);
          fp[k] = zp[xx]; fq[k] = zq[xx];
        }
#pragma unroll
        for (int k = 0; k < 4 * XU; ++k) {
          lmp = fmaxf(lmp, fp[k]); lmq = fmaxf(lmq, fq[k]);
          nonfinite |= !(fp[k] <= FLT_MAX) | !(fq[k] <= FLT_MAX);
        }
      }
      if (nonfinite) atomicOr(a.fault, DSBD_FAULT_NONFINITE);
      stamp(73);
      lmp = wave_max_f32(lmp); lmq = wave_max_f32(lmq);
      float* const wm = sh.wmax[(i - i_lo) & 1];       // two buffers: a wave is at most one row ahead of the slowest
      if (lane == 0) { wm[2 * wave] = lmp; wm[2 * wave + 1] = lmq; }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < VL_WAVES; ++w) { lmp = fmaxf(lmp, wm[2 * w]); lmq = fmaxf(lmq, wm[2 * w + 1]); }
      const double mp = (double)lmp, mq = (double)lmq;
      if (tid == 0) { sh.lm_p[i - i_lo] = mp; sh.lm_q[i - i_lo] = mq; }
      // XU exponentials per model at a time (all of a round's at once would cost more registers than there are to spare)
#pragma unroll
      for (int k = 0; k < XU; ++k) {
        const int x = xA + k * VL_BLOCK;
        if (x < x_hi) {
          const double ep = exp_nonpos((double)fpA[k] - mp, sh.exp_tab);
          double eq = ep;
          if (!a.alias) eq = exp_nonpos((double)fqA[k] - mq, sh.exp_tab);
          store(joff + x, ep, eq);
          s_p += ep; s_q += eq;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (haveB) {
#pragma unroll
        for (int k = 0; k < XU; ++k) {
          const int x = xB + k * VL_BLOCK;
          if (x < x_hi) {
            const double ep = exp_nonpos((double)fpB[k] - mp, sh.exp_tab);
            double eq = ep;
            if (!a.alias) eq = exp_nonpos((double)fqB[k] - mq, sh.exp_tab);
            store(joff + x, ep, eq);
            s_p += ep; s_q += eq;
          }
        }
      }
      // the rest of a long piece, read a second time (from the caches): XU logits of each model at a time, the next
      // round's requested before this round's exponentials are taken; ragged end predicated
      {
        int x = xB + XU * VL_BLOCK;
        float np[XU], nq[XU];
        if (x < x_hi) {
#pragma unroll
          for (int k = 0; k < XU; ++k) {
            const int xx = min(x + k * VL_BLOCK, x_hi - 1);
            np[k] = zp[xx]; nq[k] = zq[xx];
          }
        }
        while (x < x_hi) {
          float fp[XU], fq[XU];
#pragma unroll
          for (int k = 0; k < XU; ++k) { fp[k] = np[k]; fq[k] = nq[k]; }
          const int xn = x + XU * VL_BLOCK;
          if (xn < x_hi) {
#pragma unroll
            for (int k = 0; k < XU; ++k) {
              const int xx = min(xn + k * VL_BLOCK, x_hi - 1);
              np[k] = zp[xx]; nq[k] = zq[xx];
            }
          }
#pragma unroll
          for (int k = 0; k < XU; ++k) {
            if (x + k * VL_BLOCK < x_hi) {
              const double ep = exp_nonpos((double)fp[k] - mp, sh.exp_tab);
              double eq = ep;
              if (!a.alias) eq = exp_nonpos((double)fq[k] - mq, sh.exp_tab);
              store(joff + x + k * VL_BLOCK, ep, eq);
              s_p += ep; s_q += eq;
            }
          }
          x = xn;
        }
      }
      };
      // (an aliased q_beam is p_beam: both stores then go to one place)
      if (in_lds) exp_pass([&](long long jj, double ep, double eq) { pl[(int)jj] = ep; ql[(int)jj] = eq; });
      else if (n_lds == 0) exp_pass([&](long long jj, double ep, double eq) { pbg[jj] = ep; qbg[jj] = eq; });
      else exp_pass([&](long long jj, double ep, double eq) {
        if (jj < n_lds) { pl[(int)jj] = ep; ql[(int)jj] = eq; } else { pbg[jj] = ep; qbg[jj] = eq; }
      });
      s_p = wave_sum(s_p);
      s_q = wave_sum(s_q);
      if (lane == 0) {
        sh.u.wpart[((i - i_lo) * VL_WAVES + wave) * 2] = s_p;
        sh.u.wpart[((i - i_lo) * VL_WAVES + wave) * 2 + 1] = s_q;
      }
    }
    early = false;
#pragma unroll
    for (int k = 0; k < XU; ++k) { eA_p[k] = 0.f; eA_q[k] = 0.f; eB_p[k] = 0.f; eB_q[k] = 0.f; }     // (not carried through the layer)
    stamp(100);
    __syncthreads();
    // ===== all-reduce of the rows' maxima and sums.  Only the workgroups that hold a piece of row i post its four
    // values (sum and maximum of the piece, both models) and only those are polled.
    epoch += 1;
    const unsigned long long rs_tag = exchange_tag(nonce + epoch);
    Slot* const rs_bank = slots + a.sl.r + (long long)(l - 1) * a.sl.r_stride;
    if (tid < 4 * (i_hi - i_lo + 1) && !(l == 1 && (int)blockIdx.x == a.mute_wg)) {
      const int r = tid >> 2, which = tid & 3;
      double v;
      if (which < 2) {
        const double* wp = &sh.u.wpart[r * VL_WAVES * 2 + which];
        v = ((wp[0] + wp[2]) + (wp[4] + wp[6])) + ((wp[8] + wp[10]) + (wp[12] + wp[14]));
      } else {
        v = which == 2 ? sh.lm_p[r] : sh.lm_q[r];
      }
      slot_post(rs_bank + (long long)g * a.sl.r_w + 4 * i_lo + tid, v, rs_tag);
    }
    stamp(102);

    if (l == 1 && g != 0 && wave == 2 && lane < 2 * NACC) {      // the accumulator words' values at launch
      double v = 0.0;
      if (!slot_wait(slots + a.sl.acc0 + lane, acc0_tag, v, a.sync_limit)) give_up();
      (&sh.acc_prev[0][0])[lane] = (unsigned long long)__double_as_longlong(v);
    }
    // ===== rows' maxima and totals: thread (r, c) gathers column c = (row, model) from every R-th workgroup that holds
    // part of it and folds the pieces (sum relative to the piece's maximum) as it goes; the R partial results of a
    // column sit in R neighbouring lanes of one wave and are put on the column's maximum and added up by lane
    // exchanges that pair the lanes symmetrically (no table in the LDS, no barrier in between): every lane of a
    // column, in every workgroup of the prompt, gets the same bits.
    {
      const int ncols = 2 * nI;
      int cshift = 0;
      while ((1 << cshift) < ncols) ++cshift;
      const int cpow = 1 << cshift;
      const int R = min(32, VL_BLOCK / cpow);                        // a power of two, 4 .. 32
      int rshift = 2;
      while ((1 << rshift) < R) ++rshift;
      const int r = tid & (R - 1), c = tid >> rshift;                // c < VL_BLOCK / R, which is at least cpow
      double accM = -INFINITY, accS = 0.0;
      bool mine = true;
      if (c < ncols) {
        const int i = c >> 1;
        const int w_lo = cut.rows_per_wg > 0 ? i / cut.rows_per_wg : i * cut.wg_per_row;
        const int w_hi = cut.rows_per_wg > 0 ? w_lo : w_lo + geo_pieces - 1;
        for (int w = w_lo + r; w <= w_hi; w += R) {
          double vs = 0.0, vm = 0.0;
          Slot* const sl0 = rs_bank + (long long)w * a.sl.r_w + 4 * i + (c & 1);
          mine = mine && slot_wait2(sl0, sl0 + 2, rs_tag, vs, vm, a.sync_limit);
          const double Mn = fmax(accM, vm);
          accS = accS * exp_nonpos(accM - Mn, sh.exp_tab) + vs * exp_nonpos(vm - Mn, sh.exp_tab);
          accM = Mn;
        }
      }
      stamp(20);
      if (!mine) give_up();
      // over aligned groups of R lanes: quads, the other quad of an eight, the other half of a sixteen (lane moves
      // inside the SIMD), then the other sixteen (one LDS exchange)
      double cm = accM;
      cm = fmax(cm, dpp_move_f64<0xB1, 0xf>(cm));                    // quad_perm [1,0,3,2]
      cm = fmax(cm, dpp_move_f64<0x4E, 0xf>(cm));                    // quad_perm [2,3,0,1]
      if (R >= 8) cm = fmax(cm, dpp_move_f64<0x141, 0xf>(cm));       // row_half_mirror
      if (R >= 16) cm = fmax(cm, dpp_move_f64<0x140, 0xf>(cm));      // row_mirror
      if (R >= 32) cm = fmax(cm, __shfl_xor(cm, 16));
      double tot = accS * exp_nonpos(accM - cm, sh.exp_tab);         // partial results without a piece: 0 x exp(-inf) = 0
      tot += dpp_move_f64<0xB1, 0xf>(tot);
      tot += dpp_move_f64<0x4E, 0xf>(tot);
      if (R >= 8) tot += dpp_move_f64<0x141, 0xf>(tot);
      if (R >= 16) tot += dpp_move_f64<0x140, 0xf>(tot);
      if (R >= 32) tot += __shfl_xor(tot, 16);
      __syncthreads();                       // the beam weights (another wave's) are there; so is a give-up
      if (sh.abort) return;
      stamp(21);
      // column totals; the scale factors of the rows, and what the fp64 log-sum-exp needs (taken later)
      if (c < ncols && r == 0) {
        const int i = c >> 1;
        if (c & 1) { sh.max_q[i] = cm; sh.sq[i] = sh.bw_q[i] / tot; sh.lse_q[i] = tot; }
        else { sh.max_p[i] = cm; sh.sp[i] = sh.bw_p[i] / tot; sh.lse_p[i] = tot; }
      }
      // every workgroup's share of p_beam follows from its piece's sum: sampling from p_beam (the additional layer,
      // the draws that fill a layer up) then needs no exchange of the workgroups' totals.  Only where a gathering
      // thread holds exactly one piece (its sum and maximum are still in its registers).
      // (entries of workgroups without a piece are never written: the reader knows which those are)
      const bool single_piece = cut.rows_per_wg == 0 && geo_pieces <= R;
      if (tid == 0) sh.ptot_ok = single_piece ? 1 : 0;
      if (single_piece && c < ncols && (c & 1) == 0 && r < geo_pieces) {
        const int i = c >> 1;
        sh.ptot[i * cut.wg_per_row + r] = (sh.bw_p[i] / tot) * (accS * exp_nonpos(accM - cm, sh.exp_tab));
      }
      __syncthreads();
    }
    stamp(24);
    // scaling, fused with this thread's part of F(1)
    for (int i = i_lo; i <= i_hi; ++i) {
      const long long j_lo = max(e_lo, (long long)i * V) - e_lo;
      const long long j_hi = min(e_hi, (long long)(i + 1) * V) - e_lo;
      // (the slice holds exponentials against the piece's own maximum: put them on the row's)
      const double fp = sh.sp[i] * exp_nonpos(sh.lm_p[i - i_lo] - sh.max_p[i], sh.exp_tab);
      const double fq = sh.sq[i] * exp_nonpos(sh.lm_q[i - i_lo] - sh.max_q[i], sh.exp_tab);
      with_slices([&](auto P, auto Q, long long r0, long long r1) {
        const long long j_end = min(j_hi, r1);
        long long j = max(j_lo, r0) + tid;
        for (; j + 3 * VL_BLOCK < j_end; j += 4 * VL_BLOCK) {      // four elements of each array in flight
          double pv[4], qv[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) { pv[k] = P[j + k * VL_BLOCK]; qv[k] = Q[j + k * VL_BLOCK]; }
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            pv[k] *= fp; qv[k] *= fq;
            P[j + k * VL_BLOCK] = pv[k]; Q[j + k * VL_BLOCK] = qv[k];
            f1 += fmax(pv[k] - qv[k], 0.0);
          }
        }
        for (; j < j_end; j += VL_BLOCK) {
          const double pv = P[j] * fp, qv = Q[j] * fq;
          P[j] = pv; Q[j] = qv;
          f1 += fmax(pv - qv, 0.0);
        }
      });
    }
    }
    if constexpr (WARP) {
      // ===== warping T: top-k / top-p on the two joints (Section 2.1; Section 3.1 "Details": p_beam = T o p/P).  A joint's
      // K first entries (by value, equal values by flat index) are among the K first of its rows, which the rows' records
      // hold: every entry's value from its logit in one form that depends on the row only (equal logits of a row give
      // equal values), then their ranks by counting.
      const int K = a.top_k, n_cand = nI * K;            // at most 64 x 32 per model
      typedef __attribute__((address_space(3))) int lds_i32;
      const int stride = n_cand;
      lds_f64* const cv = (lds_f64*)dyn_lds;             // [2][stride] values of p_beam's and q_beam's entries, row by row, then
      lds_i32* const ci = (lds_i32*)(dyn_lds + 2 * stride);      // their flat indices, and
      lds_i32* const kept = ci + 2 * stride;                     // the numbers of those that can be among the K first
      lds_f64* const lv = (lds_f64*)sh.Pa; lds_i32* const li = (lds_i32*)sh.Pb;      // the K first of either, in rank order
      if constexpr (BARE) {
        // a wave per row takes its K first entries one after the other out of its registers
        for (int t = wave; t < 2 * nI; t += VL_WAVES) {
          const int m = t >= nI ? 1 : 0, i = t - m * nI, node = sh.I_node[i];
          const float* const mine = (m ? a.zq : a.zp) + (long long)node * V + lane;
          float z[VR_BARE / 64];
#pragma unroll
          for (int k = 0; k < VR_BARE / 64; ++k) {
            z[k] = -INFINITY;
            if (64 * k + lane < V) z[k] = mine[64 * k];
            if (!(z[k] > -INFINITY)) z[k] = -INFINITY;                      // (NaN is no entry)
          }
          float top = z[0];
#pragma unroll
          for (int k = 1; k < VR_BARE / 64; ++k) top = fmaxf(top, z[k]);
          const double M = (double)wave_max_f32(top);
          if (lane == 0) (m ? sh.max_q : sh.max_p)[i] = M;
          double v[VR_BARE / 64];
#pragma unroll
          for (int k = 0; k < VR_BARE / 64; ++k) {
            v[k] = -1.0;
            if (64 * k < V && z[k] > -INFINITY) v[k] = exp_nonpos((double)z[k] - M, sh.exp_tab);
          }
          for (int r = 0; r < K; ++r) {
            double wv = -1.0;
            int wx = INT_MAX;
#pragma unroll
            for (int k = 0; k < VR_BARE / 64; ++k)
              if (v[k] > wv) { wv = v[k]; wx = lane + 64 * k; }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
              const double ov = __shfl_xor(wv, off);
              const int ox = __shfl_xor(wx, off);
              if ((ov > wv) | ((ov == wv) & (ox < wx))) { wv = ov; wx = ox; }
            }
#pragma unroll
            for (int k = 0; k < VR_BARE / 64; ++k)
              if (lane + 64 * k == wx) { v[k] = -1.0; kept[m * stride + i * K + r] = __float_as_int(z[k]); }
            if (lane == 0) ci[m * stride + i * K + r] = wx;
          }
        }
      }
      lds_barrier();                                     // the beam weights are there
      for (int t = tid; t < 2 * n_cand; t += VL_BLOCK) {
        const int m = t >= n_cand ? 1 : 0, e = t - m * n_cand, i = e / K, r = e - i * K;
        RowHead h = rec_head;
        RowEntry x = rec_entry;
        if constexpr (BARE) {
          const double s = *reinterpret_cast<const double*>(a.rec + (a.alias ? (long long)sh.I_node[i] : 2LL * sh.I_node[i] + m) * a.rec_stride);
          x.z = __int_as_float(kept[m * stride + e]); x.x = ci[m * stride + e];
          h.sum = fabs(s); h.max = (float)(m ? sh.max_q : sh.max_p)[i];
          h.n = (x.x != INT_MAX ? r + 1 : 0) + (__double2hiint(s) < 0 ? VR_ROW_BAD : 0);
        } else {
          if (t != tid) row_record(sh.I_node[i], m, r, h, x);
        }
        const double scale = (m ? sh.bw_q[i] : sh.bw_p[i]) / h.sum, top = (double)h.max;
        if (r == 0) {
          (m ? sh.max_q : sh.max_p)[i] = top; (m ? sh.sq : sh.sp)[i] = scale; (m ? sh.lse_q : sh.lse_p)[i] = h.sum;
          if (h.n >= VR_ROW_BAD) atomicOr(a.fault, DSBD_FAULT_NONFINITE);
        }
        const bool real = r < h.n % VR_ROW_BAD;
        cv[m * stride + e] = real ? exp_nonpos((double)x.z - top, sh.exp_tab) * scale : -1.0;
        ci[m * stride + e] = real ? i * V + x.x : INT_MAX;
      }
      if (tid < 2 * K) { lv[tid] = -1.0; li[tid] = INT_MAX; }      // ("none", which sorts last)
      if (tid < 2) { sh.warp_bound[tid] = 0ull; sh.warp_kept[tid] = 0; }
      __syncthreads();
      stamp(60);
      // Ranks by counting the entries ahead (of equal values the one in front has the lower index: rows are in index order, and
      // so are equal logits of a row).  A single row's list has the ranks already.
      if (nI == 1) {
        for (int t = tid; t < 2 * K; t += VL_BLOCK) {
          const int m = t >= K ? 1 : 0, r = t - m * K;
          if (cv[m * stride + r] >= 0.0) { lv[t] = cv[m * stride + r]; li[t] = ci[m * stride + r]; }
        }
      } else {
        // First a lower bound of the K-th entry: in column c of the rows' lists, the ceil(K / (c + 1))-th largest entry has
        // c + 1 entries of each of so many rows at or above it.  The best of these bounds leaves little more than K entries.
        // (Counting among all, 8 rows: K = 10 2.2 us, K = 20 7.1, K = 32 12.7.)
        for (int t = tid; t < 2 * n_cand; t += VL_BLOCK) {
          const int m = t >= n_cand ? 1 : 0, e = t - m * n_cand, i = e / K, c = e - i * K;
          const lds_f64* const all = cv + m * stride;
          const double v = all[e];
          int ahead = 0;
#pragma unroll 4
          for (int o = 0; o < nI; ++o) { const double w = all[o * K + c]; ahead += (w > v) | ((w == v) & (o < i)); }
          if (v >= 0.0 && ahead == (K + c) / (c + 1) - 1) atomicMax(&sh.warp_bound[m], (unsigned long long)__double_as_longlong(v));
        }
        __syncthreads();
        for (int t = tid; t < 2 * n_cand; t += VL_BLOCK) {
          const int m = t >= n_cand ? 1 : 0, e = t - m * n_cand;
          const double v = cv[m * stride + e];
          if (v >= 0.0 && v >= __longlong_as_double((long long)sh.warp_bound[m])) kept[m * stride + atomicAdd(&sh.warp_kept[m], 1)] = e;
        }
        __syncthreads();
        const int n_p = sh.warp_kept[0], n_all = n_p + sh.warp_kept[1];
        for (int t0 = 0; t0 < n_all; t0 += VL_BLOCK / 8) {      // eight threads an entry
          const int t = t0 + (tid >> 3);
          const bool has = t < n_all;
          const int m = has && t >= n_p ? 1 : 0;
          const lds_i32* const mine = kept + m * stride;
          const int e = has ? mine[t - m * n_p] : 0, n_m = has ? (m ? n_all - n_p : n_p) : 0;
          const double v = cv[m * stride + e];
          int rank = 0;
#pragma unroll 4
          for (int c = tid & 7; c < n_m; c += 8) {
            const int oe = mine[c];
            const double o = cv[m * stride + oe];
            rank += (o > v) | ((o == v) & (oe < e));
          }
          rank += __shfl_xor(rank, 1);
          rank += __shfl_xor(rank, 2);
          rank += __shfl_xor(rank, 4);
          if (has && (tid & 7) == 0 && rank < K) { lv[m * K + rank] = v; li[m * K + rank] = ci[m * stride + e]; }
        }
      }
      __syncthreads();
      stamp(61);
      if (wave == 0) {
        // top-p on the kept entries (rank order: the shortest leading part whose share exceeds top_p) and
        // renormalisation; lanes 0..31 carry p_beam's list, lanes 32..63 q_beam's, one rank each.  The running
        // sums add the entries one by one in rank order.
        const int r = lane & 31, half = lane & 32;
        const bool is_q = half != 0;
        const int ix = r < K ? li[(is_q ? K : 0) + r] : INT_MAX;
        const bool real = ix != INT_MAX;
        const double v = real ? lv[(is_q ? K : 0) + r] : 0.0;
        double cum = 0.0;
        int partner = -1;                  // lane of the other list's entry with the same index
        {
          // (the lists are read from the LDS, every lane of a half the same word: one read serves 32 lanes; lane
          // reads of the other lanes' registers cost a scalar round trip each)
          const int own = is_q ? K : 0, oth = is_q ? 0 : K;
#pragma unroll 8
          for (int c = 0; c < K; ++c) {
            const int i_own = li[own + c], i_oth = li[oth + c];
            const double v_own = i_own != INT_MAX ? lv[own + c] : 0.0;
            if (c <= r) cum += v_own;
            if (i_oth == ix) partner = (is_q ? 0 : 32) + c;
          }
        }
        const unsigned long long real_m = __ballot(real);
        const int n = __popcll(is_q ? (real_m >> 32) : (real_m & 0xffffffffull));     // real entries lead the list
        int keep = n;
        if (a.top_p < 1.0f) {
          const double mass = __shfl(cum, half + max(n - 1, 0));
          const unsigned long long over_m = __ballot(real && cum / mass > (double)a.top_p);
          const unsigned int mine = (unsigned int)(is_q ? (over_m >> 32) : (over_m & 0xffffffffull));
          if (mine) keep = __ffs((int)mine);
        }
        const double z = __shfl(cum, half + max(keep - 1, 0));
        const bool kept = r < keep;
        const double w = kept ? v / z : 0.0;
        // union of the two supports, ascending flat index: a q entry whose index p_beam also keeps is
        // carried by the p entry
        const double w_partner = __shfl(w, max(partner, 0));       // 0 when the partner was cut
        const int kept_partner = __shfl((int)kept, max(partner, 0));
        const bool both = real && partner >= 0 && kept_partner;
        const double other = (both && !is_q) ? w_partner : 0.0;
        const bool valid = kept && !(is_q && both);
        int rank = 0;
        {
          // the valid entries' indices side by side in the LDS (lane c: p_beam's list, 32 + c: q_beam's)
          lds_i32* const vx = (lds_i32*)sh.A_idx;
          vx[lane] = valid ? ix : INT_MAX;
          wave_lds_fence();
#pragma unroll 8
          for (int c = 0; c < K; ++c) rank += (vx[c] < ix ? 1 : 0) + (vx[32 + c] < ix ? 1 : 0);
        }
        if (valid) { sh.U_idx[rank] = ix; sh.U_p[rank] = is_q ? 0.0 : w; sh.U_q[rank] = is_q ? w : other; }
        const unsigned long long vm = __ballot(valid);
        if (lane == 0) sh.nU = __popcll(vm);
        }
      __syncthreads();
    }
    stamp(25);
    // p_beam and q_beam at every candidate's (parent beam, token)
    if (tid < M) {
      const int n = sh.S_node[tid];
      const int slot = sh.slot_of[sh.n_parent[n - n_begin] - n_begin];
      sh.S_zp[tid] = czp; sh.S_zq[tid] = czq;
      double pbx, qbx;
      if constexpr (WARP) {       // warped joints: the surviving entries, zero elsewhere
        const int flat = slot * V + sh.n_token[n - n_begin];
        int at = 0;                                  // entries with a smaller index (the list is in index order)
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1) {
          const int probe = at + step - 1;
          at += (probe < sh.nU && sh.U_idx[min(probe, 63)] < flat) ? step : 0;
        }
        const bool hit = at < sh.nU && sh.U_idx[min(at, 63)] == flat;
        pbx = hit ? sh.U_p[min(at, 63)] : 0.0;
        qbx = hit ? sh.U_q[min(at, 63)] : 0.0;
      } else {
        pbx = exp_nonpos((double)czp - sh.max_p[slot], sh.exp_tab) * sh.sp[slot];
        qbx = exp_nonpos((double)czq - sh.max_q[slot], sh.exp_tab) * sh.sq[slot];
      }
      const float uf = sh.n_u[n - n_begin];
      // the test with p' = p_beam (first candidate, and every candidate right after an acceptance) needs no chain
      const double ratio = (qbx == 0.0) ? INFINITY : pbx / qbx;
      sh.S_pb[tid] = pbx; sh.S_qb[tid] = qbx; sh.S_u[tid] = uf;
      sh.S_flag[tid] = (unsigned char)(((double)uf <= ratio ? 1 : 0) | (fabs(ratio - (double)uf) <= NEAR_TIE ? 2 : 0));
    }
    if (tid == 0) { sh.cc[1] = 0.0; sh.FF[1] = 1.0; sh.kmax = 1; sh.acc_n = 0; sh.pos = 0; sh.kidx = 1; sh.x_have = 0; sh.stop = 0; }
    // Entry 2 of the residual chain (c = 1) is needed by the first rejection of nearly every layer: its partial
    // sums are posted ahead of time.
    stamp(26);
    if (!WARP && M > 0) {
      x_own = wg_total(f1);                 // barrier inside: also publishes the scaled slices
      stamp(27);
      if (wave == 0) accumulators_post(accs + (size_t)(achg & 1) * NACC * 16, a.G, g, x_own);
      achg += 1;
      x_open = true;
    } else {
      __syncthreads();
    }

    // fp64 log-sum-exp of the input beams' rows: needed at the end of the layer only, so one wave takes the
    // logarithms while the first wave is busy with the decisions (or the others with the sampling prefix sums)
    if (wave == 2 && lane < nI) {
      sh.lse_p[lane] = sh.max_p[lane] + log(sh.lse_p[lane]);
      sh.lse_q[lane] = sh.max_q[lane] + log(sh.lse_q[lane]);
    }
    stamp(22);
    // sum over the slice of max(p_beam - c q_beam, 0); four loads in flight per thread
    // (the threads t0 .. t0+nt-1 share the work; the others return 0)
    auto slice_sum = [&](double c, int t0, int nt) -> double {
      double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
      if (tid < t0) return 0.0;
      if constexpr (WARP) {       // the whole (warped) joint is the prompt's workgroup's short list
        const int c2 = tid - t0;
        return c2 < sh.nU ? fmax(sh.U_p[c2] - c * sh.U_q[c2], 0.0) : 0.0;
      }
      with_slices([&](auto P, auto Q, long long r0, long long r1) {
        // four elements of each array in flight per thread, the ragged end predicated (one element after the other,
        // the tail of a 4008-entry slice cost four dependent LDS round trips per chain entry; eight in flight cost
        // 50 more registers)
        const int n = (int)r1;             // a slice has fewer than 2^31 entries
        const int j_first = (int)r0 + tid - t0;
        if constexpr (std::is_same<decltype(P), glb_f64*>::value) {
          // the part in the workspace (read through the caches): eight of each array in flight
          for (int j = j_first; j < n; j += 8 * nt) {
            double pv[8], qv[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) { const int jk = min(j + k * nt, n - 1); pv[k] = P[jk]; qv[k] = Q[jk]; }
#pragma unroll
            for (int k = 0; k < 8; k += 4) {
              s0 += (j + k * nt < n) ? fmax(pv[k] - c * qv[k], 0.0) : 0.0;
              s1 += (j + (k + 1) * nt < n) ? fmax(pv[k + 1] - c * qv[k + 1], 0.0) : 0.0;
              s2 += (j + (k + 2) * nt < n) ? fmax(pv[k + 2] - c * qv[k + 2], 0.0) : 0.0;
              s3 += (j + (k + 3) * nt < n) ? fmax(pv[k + 3] - c * qv[k + 3], 0.0) : 0.0;
            }
          }
        } else {
          for (int j = j_first; j < n; j += 4 * nt) {
            const int j1 = min(j + nt, n - 1), j2 = min(j + 2 * nt, n - 1), j3 = min(j + 3 * nt, n - 1);
            const double p0 = P[j], p1 = P[j1], p2 = P[j2], p3 = P[j3];
            const double q0 = Q[j], q1 = Q[j1], q2 = Q[j2], q3 = Q[j3];
            s0 += fmax(p0 - c * q0, 0.0);
            s1 += (j + nt < n) ? fmax(p1 - c * q1, 0.0) : 0.0;
            s2 += (j + 2 * nt < n) ? fmax(p2 - c * q2, 0.0) : 0.0;
            s3 += (j + 3 * nt < n) ? fmax(p3 - c * q3, 0.0) : 0.0;
          }
        }
      });
      return (s0 + s1) + (s2 + s3);
    };

    stamp(23);
    // What the last layer draws: `d_cnt` beams into the output slots from d_base on, the first of them from the residual
    // max(p_beam - d_c q_beam, 0) (d_resid), the others from p_beam.
    int d_cnt, d_base = 0;
    bool d_resid = false;
    double d_c = 0.0;
    if (bonus) {
      // ===== every draft layer passed: W_L beams from p_beam^(gamma+1)
      d_cnt = n_out = min(W_in, a.W_cap);
      if (g == 0 && tid == 0) a.out.layer_width[(long long)prompt * Lw + l] = W_in;
    } else {
    int WL = W_in;             // width of the layer, known before the first decision

    // The accept / reject decisions of Algorithm 1 in candidate order, as far as the chain allows.
    // Outcome in sh.state[round & 1]: 0 = finished, 1 = the next chain entry is needed.
    // Plain sequential form (one thread): only used when a residual without mass turns up.
    auto decide_serial = [&](unsigned int round) {
      int pos = sh.pos, nacc = sh.acc_n, k = sh.kidx;
      const int kmax = sh.kmax;
      int state = 0;
      while (true) {
        if (pos >= M || nacc >= WL) { state = 0; break; }
        if (k > kmax) { state = 1; break; }
        if (k > 1 && !(sh.FF[k] > 0.0)) {
          // a residual without mass (impossible in exact arithmetic): fall back to p_beam
          atomicOr(a.fault, DSBD_FAULT_ZERO_RESIDUAL);
          k = 1;
        }
        const int n = sh.S_node[pos];
        const double pbx = sh.S_pb[pos], qbx = sh.S_qb[pos];
        const double num = (k == 1) ? pbx : fmax(pbx - sh.cc[k] * qbx, 0.0) / sh.FF[k];
        const double ratio = (qbx == 0.0) ? INFINITY : num / qbx;
        const double u = (double)sh.S_u[pos];
        if (fabs(ratio - u) <= NEAR_TIE) near_tie++;
        if (u <= ratio) {
          sh.A_node[nacc] = n;
          sh.A_idx[nacc] = pos;
          nacc++;
          k = 1;
          if (g == 0) a.out.node_status[n] = DSBD_ACCEPTED;
        } else {
          k++;
          if (g == 0) a.out.node_status[n] = DSBD_REJECTED;
        }
        pos++;
      }
      sh.pos = pos; sh.acc_n = nacc; sh.kidx = k; sh.state[round & 1] = state;
    };
    // The same decisions taken by the first wave, a run at a time.  With p' = p_beam (chain index 1) consecutive
    // candidates are independent tests (precomputed flags): all acceptances up to the first rejection are taken
    // at once.  After a rejection candidate pos + j meets chain entry k + j for as long as the rejections last:
    // those tests run side by side and the first acceptance ends the streak.
    auto decide = [&](unsigned int round, int kmax) {    // kmax: entries of the chain that exist (uniform)
      wave_lds_fence();                                    // the newest entry was written by lane 0 a moment ago
      int pos = sh.pos, nacc = sh.acc_n, k = sh.kidx;      // uniform over the wave
      int state = 0, near_add = 0;
      while (true) {
        if (pos >= M || nacc >= WL) { state = 0; break; }
        const int cand = pos + lane;
        if (k == 1) {
          const int nv = min(64, M - pos);
          const int fl = lane < nv ? sh.S_flag[cand] : 0;
          const unsigned long long rej = __ballot(lane < nv && !(fl & 1));
          const int run = rej ? min(nv, (int)__ffsll((long long)rej) - 1) : nv;   // acceptances in a row from pos
          const int take = min(run, WL - nacc);
          if (lane < take) {
            const int n = sh.S_node[cand];
            sh.A_node[nacc + lane] = n;
            sh.A_idx[nacc + lane] = cand;
            if (g == 0) a.out.node_status[n] = DSBD_ACCEPTED;
          }
          const bool fails = take == run && run < nv && nacc + take < WL;   // candidate pos + run is tested and rejected
          near_add += __popcll(__ballot((lane < take || (fails && lane == run)) && (fl & 2)));
          nacc += take; pos += take;
          if (fails) {
            if (lane == run && g == 0) a.out.node_status[sh.S_node[cand]] = DSBD_REJECTED;
            pos += 1; k = 2;
          }
          continue;
        }
        const int navail = kmax - k + 1;                   // chain entries k .. kmax exist
        if (navail <= 0) { state = 1; break; }
        const int nv = min(min(64, navail), M - pos);
        bool acc = false, nr = false, dead = false;
        if (lane < nv) {
          const int kk = k + lane;
          const double F = sh.FF[kk];
          dead = !(F > 0.0);
          const double pbx = sh.S_pb[cand], qbx = sh.S_qb[cand];
          const double num = fmax(pbx - sh.cc[kk] * qbx, 0.0) / F;
          const double ratio = (qbx == 0.0) ? INFINITY : num / qbx;
          const double u = (double)sh.S_u[cand];
          acc = u <= ratio;
          nr = fabs(ratio - u) <= NEAR_TIE;
        }
        const unsigned long long accm = __ballot(lane < nv && acc);
        const int last = accm ? (int)__ffsll((long long)accm) - 1 : nv - 1;     // last candidate tested in this step
        if (__ballot(lane <= last && dead)) {
          // a residual without mass: hand the rest to the sequential form, which knows what to do about it
          if (lane == 0) { near_tie += near_add; sh.pos = pos; sh.acc_n = nacc; sh.kidx = k; decide_serial(round); }
          wave_lds_fence();
          return;
        }
        near_add += __popcll(__ballot(lane <= last && nr));
        if (lane <= last) {
          const int n = sh.S_node[cand];
          const bool a_here = accm && lane == last;
          if (a_here) { sh.A_node[nacc] = n; sh.A_idx[nacc] = cand; }
          if (g == 0) a.out.node_status[n] = a_here ? DSBD_ACCEPTED : DSBD_REJECTED;
        }
        pos += last + 1;
        if (accm) { nacc += 1; k = 1; } else { k += nv; }
      }
      if (lane == 0) {
        near_tie += near_add; sh.pos = pos; sh.acc_n = nacc; sh.kidx = k; sh.state[round & 1] = state;
        // (finished without the entry that is on its way)
        if (state == 0 && (nacc >= WL || k <= kmax)) __hip_atomic_store(&sh.stop, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    };

    // The open exchange's value, entry k + 1 of the chain, by the wave that calls (all its lanes).
    auto collect_entry = [&](int k, const int* stop) __attribute__((always_inline)) {
      const unsigned int at = achg - 1;
      double F;
      const int r = accumulators_collect(accs + (size_t)(at & 1) * NACC * 16, sh.acc_prev[at & 1], a.G, x_own, a.sync_limit, stop, F);
      if (r == ACC_TIMEOUT) give_up();
      if (r == ACC_DONE && lane == 0) { sh.cc[k + 1] = sh.cc[k] + sh.FF[k]; sh.FF[k + 1] = F; sh.x_have = 1; }
    };
    // Appends entry kmax+1 to the residual chain: every workgroup sums its slice (unless the entry is under way), the
    // second wave exchanges the partial sums.  All threads leave through one barrier; false = a wait gave up.
    auto extend_chain = [&]() -> bool {
      const int k = sh.kmax;
      if constexpr (WARP) {          // the workgroup holds the whole warped joint: the total is F itself
        const double c = sh.cc[k] + sh.FF[k];
        const double tot = wg_total(slice_sum(c, 0, VL_BLOCK));
        if (tid == 0) { sh.cc[k + 1] = c; sh.FF[k + 1] = tot; sh.kmax = k + 1; }
        __syncthreads();
        return true;
      }
      if (!x_open) {
        const double c = sh.cc[k] + sh.FF[k];
        stamp(46);
        const double sl = slice_sum(c, 0, VL_BLOCK);
        stamp(43);
        x_own = wg_total(sl, true);
        stamp(44);
        if (wave == 1) accumulators_post(accs + (size_t)(achg & 1) * NACC * 16, a.G, g, x_own);
        achg += 1;
      }
      if (wave == 1) {
        collect_entry(k, nullptr);
        if (lane == 0) sh.kmax = k + 1;
      }
      x_open = false;
      stamp(45);
      __syncthreads();
      return sh.abort == 0;
    };

    stamp(30);
    // ===== width of the layer
    if (dynamic) {
      // alpha_j for j = 1..M (Eq. 3) from the chain; stop early if the residual mass vanishes
      if constexpr (WARP) {
        // The warped joints are the workgroup's short list, an entry per lane: the first wave runs the
        // whole chain by itself (c_{k+1} = c_k + F(c_k), F a sum over its lanes), no barrier per entry.  The same
        // sums as extend_chain forms (there the other waves add zeros).
        if (wave == 0) {
          const bool in = lane < sh.nU;
          const double up = in ? sh.U_p[lane] : 0.0, uq = in ? sh.U_q[lane] : 0.0;
          int k = sh.kmax;               // 1: nothing is posted ahead of time for warped joints
          double c = sh.cc[k], F = sh.FF[k];
          for (int j = 1; j <= M; ++j) {
            c += F;
            F = wave_sum(fmax(up - c * uq, 0.0));
            k += 1;
            if (lane == 0) { sh.cc[k] = c; sh.FF[k] = F; }
            if (!(F > 0.0)) break;
          }
          if (lane == 0) sh.kmax = k;
        }
        __syncthreads();
      } else {
        bool dead = false;
        for (int j = 1; j <= M && !dead; ++j) {
          if (!extend_chain()) return;
          dead = !(sh.FF[j + 1] > 0.0);
        }
      }
      const int kdone = sh.kmax;     // entries 1..kdone valid
      __syncthreads();
      int Wt = 0;
      if (M < 64) {
        // up to 63 drafts (every forest of the paper's shapes): the table fits one wave, lane m = row m, and everything is
        // in its registers: the other rows' values come by lane reads and by moving a column a lane at a time.  Same sums
        // in the same order as the general form below.  (With the values in the LDS, every term a dependent read: 5.4 us
        // for 12 drafts and a few columns, now 2.)
        if (wave == 0) {
          const int m = lane;
          const bool row = m >= 1 && m <= M;
          double alpha = 1.0;              // no residual mass left: accepted with certainty
          if (row && m + 1 <= kdone && sh.FF[m] > 0.0) alpha = 1.0 - sh.FF[m + 1] / sh.FF[m];
          // first[m] = alpha_m prod_{j<m} (1 - alpha_j); Pa = P(m,0) = prod_{j<=m} (1 - alpha_j)
          double first = alpha, Pa = 1.0;
          const double rest = 1.0 - alpha;
          for (int j = 1; j <= M; ++j) {
            const double rj = readlane_f64(rest, j);
            if (j < m) first *= rj;
            if (j <= m) Pa *= rj;
          }
          double below = 0.0;              // sum_{k<K} P(M,k)
          const int Kmax = min(M, a.W_cap);
          for (int K = 1; K <= Kmax; ++K) {
            below += readlane_f64(Pa, M);  // Pa holds column K-1
            if (!(1.0 - below >= thr)) break;
            Wt = K;
            if (K == Kmax) break;
            // column K from column K-1: P(m,K) = sum_{i=1..m} first[i] P(m-i,K-1), zero for m < K (and P(m,K-1) for m < K-1)
            double tot = 0.0, moved = m >= K - 1 ? Pa : 0.0;
            for (int i = 1; i <= M; ++i) {
              moved = lane_from_below(moved);              // P(m-i,K-1); 0 from beyond row 0
              tot += readlane_f64(first, i) * moved;
            }
            Pa = m >= K && m <= M ? tot : 0.0;
          }
          if (lane == 0) sh.found = Wt;
        }
        __syncthreads();
        Wt = sh.found;
        __syncthreads();
      } else {
        // alpha_i (Eq. 3), first[i] = alpha_i prod_{j<i} (1 - alpha_j) (Eq. 2), Pa[m] = P(m,0)
        for (int i = 1 + tid; i <= M; i += VL_BLOCK) {
          double alpha = 1.0;            // no residual mass left: accepted with certainty
          if (i + 1 <= kdone && sh.FF[i] > 0.0) alpha = 1.0 - sh.FF[i + 1] / sh.FF[i];
          sh.u.w.alpha[i] = alpha;
        }
        __syncthreads();
        for (int i = 1 + tid; i <= M; i += VL_BLOCK) {
          double f = sh.u.w.alpha[i];
          for (int j = 1; j < i; ++j) f *= (1.0 - sh.u.w.alpha[j]);
          sh.u.w.first[i] = f;
        }
        if (tid == 0) {
          double none = 1.0;
          sh.Pa[0] = 1.0;
          for (int m = 1; m <= M; ++m) { none *= (1.0 - sh.u.w.alpha[m]); sh.Pa[m] = none; }
        }
        __syncthreads();
        // W~ = max{K : 1 - sum_{k<K} P(M,k) >= t}; K = 0 always qualifies
        double below = 0.0;              // sum_{k<K} P(M,k)
        const int Kmax = min(M, a.W_cap);
        for (int K = 1; K <= Kmax; ++K) {
          below += sh.Pa[M];             // column K-1 is in Pa
          if (!(1.0 - below >= thr)) break;
          Wt = K;
          if (K == Kmax) break;
          // column K from column K-1:  P(m,K) = sum_{i=1..m} first[i] P(m-i,K-1), zero for m < K
          for (int m = tid; m <= M; m += VL_BLOCK) {
            double tot = 0.0;
            if (m >= K)
              for (int i = 1; i <= m; ++i) tot += sh.u.w.first[i] * ((m - i >= K - 1) ? sh.Pa[m - i] : 0.0);
            sh.Pb[m] = tot;
          }
          __syncthreads();
          for (int m = tid; m <= M; m += VL_BLOCK) sh.Pa[m] = sh.Pb[m];
          __syncthreads();
        }
        __syncthreads();
      }
      WL = min(a.W_cap, max(a.W_min, Wt));
    }
    WL = min(WL, a.W_cap);
    if (g == 0 && tid == 0) a.out.layer_width[(long long)prompt * Lw + l] = WL;

    stamp(40);
    // ===== sequential accept / reject.  The first wave takes the decisions as far as the chain reaches.  Meanwhile the
    // other seven sum their slices for the chain entry that would come next, and the second hands the totals to the other
    // workgroups and collects theirs: entries do not depend on decisions, so an entry takes as long as the longer of
    // the two (a rejection took 2.45 us with the exchange behind the decision: 1.05 to 1.3 us and 1.2).
    if constexpr (WARP) {
      while (true) {
        const int k = sh.kmax;         // entries 1..k exist (read after a barrier: uniform)
        const double c_next = sh.cc[k] + sh.FF[k];
        stamp(41);
        if (wave == 0) decide(decide_round, k);
        const double tot = wg_total(slice_sum(c_next, 64, VL_BLOCK - 64), true);   // barrier inside
        const int st = sh.state[decide_round & 1];
        decide_round += 1;             // the next outcome goes to the other entry: nobody still reads it
        stamp(42);
        if (st != 1) break;
        if (tid == 0) { sh.cc[k + 1] = c_next; sh.FF[k + 1] = tot; sh.kmax = k + 1; }
        __syncthreads();
      }
    } else {
      int kx = sh.kmax;                // entries 1..kx exist (the same in every thread)
      while (true) {
        stamp(41);
        // (the barriers of this loop order LDS values only: chain entries, decisions, wave totals; slices are
        // read-only here and the outputs written meanwhile are read by nobody in this kernel)
        const bool produce = !x_open && kx <= M;         // (M rejections reach entry M + 1)
        if (wave == 0) {
          if (lane == 0) sh.kmax = kx;
          decide(decide_round, kx);
        } else if (produce) {
          const double c_next = sh.cc[kx] + sh.FF[kx];
          const double ts = wave_sum(slice_sum(c_next, 64, VL_BLOCK - 64));
          double* const ws = sh.wsum[wsum_round & 1];
          if (wave >= 2) {
            if (lane == 0) {
              ws[wave] = ts;
              asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
              __hip_atomic_fetch_add(&sh.handed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
          } else {
            const unsigned int want = (handovers + 1) * (VL_WAVES - 2);
            while (__hip_atomic_load(&sh.handed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != want) {}
            asm volatile("" ::: "memory");
            x_own = (ts + (ws[2] + ws[3])) + ((ws[4] + ws[5]) + (ws[6] + ws[7]));
            if (lane == 0) sh.x_have = 0;
            accumulators_post(accs + (size_t)(achg & 1) * NACC * 16, a.G, g, x_own);
          }
        }
        if (produce) { wsum_round += 1; handovers += 1; achg += 1; x_open = true; }
        if (wave == 1 && x_open) collect_entry(kx, &sh.stop);
        stamp(42);
        lds_barrier();
        const int st = sh.state[decide_round & 1];
        decide_round += 1;             // the next outcome goes to the other entry: nobody still reads it
        if (sh.abort) return;
        if (st != 1) break;
        x_open = false;                // the decisions go on with the new entry
        kx += 1;
        stamp(45);
      }
    }
    const int nacc = sh.acc_n, pos_end = sh.pos, kcur = sh.kidx, kmax_end = sh.kmax;
    if (g == 0)
      for (int i = pos_end + tid; i < M; i += VL_BLOCK) a.out.node_status[sh.S_node[i]] = DSBD_REJECTED;

    stamp(50);
    if (nacc >= WL) {          // the layer passed: handed over at the top of the next layer
      passed_nacc = nacc;
      continue;
    }
    {
      // cumulative likelihoods of the accepted beams (fp64)
      if (tid < nacc) {
        const int n = sh.A_node[tid];
        const int ci = sh.A_idx[tid];
        const int slot = sh.slot_of[sh.n_parent[n - n_begin] - n_begin];
        sh.A_cum_p[tid] = sh.cum_p[slot] + ((double)sh.S_zp[ci] - sh.lse_p[slot]);
        sh.A_cum_q[tid] = sh.cum_q[slot] + ((double)sh.S_zq[ci] - sh.lse_q[slot]);
      }
      __syncthreads();
      // ===== the layer falls short: accepted beams, one residual sample, then p_beam samples
      if (g == 0 && tid < nacc) {
        const int n = sh.A_node[tid];
        const long long o = (long long)prompt * a.W_cap + tid;
        a.out.out_parent[o] = sh.n_parent[n - n_begin];
        a.out.out_token[o] = sh.n_token[n - n_begin];
        a.out.out_node[o] = n;
        a.out.out_logp_target[o] = sh.A_cum_p[tid];
        a.out.out_logp_draft[o] = sh.A_cum_q[tid];
        emit_next(tid, sh.n_parent[n - n_begin], sh.n_token[n - n_begin], sh.A_cum_p[tid], sh.A_cum_q[tid]);
      }
      // p' = p'_kcur; its chain entry may still be missing if the last candidate was rejected
      int k = kcur;
      if (k > kmax_end) {
        if (WARP || !x_open || sh.x_have == 0) { if (!extend_chain()) return; }
      }
      if (k > 1 && !(sh.FF[k] > 0.0)) {
        if (g == 0 && tid == 0) atomicOr(a.fault, DSBD_FAULT_ZERO_RESIDUAL);
        k = 1;
      }
      d_resid = k > 1;
      d_c = sh.cc[k];
      d_base = nacc;
      d_cnt = WL - nacc;
      l_last = l;
      n_out = WL;
    }
    }

    // ===== the draws, by inverse CDF over I x V in flat order; the workgroup that owns a draw writes its output slot.
    // (One copy of this code for all draws of a prompt, and one pass for the residual's draw and the others: instructions
    // that run once come from memory.)
    const float d_u = tid >= d_cnt ? 0.f : bonus ? u_fill[(long long)l * a.W_cap + tid]
                                          : tid == 0 ? u_res[l] : u_fill[(long long)l * a.W_cap + tid - 1];
    auto emit = [&](long long pick, int j) {           // (flat index over I x V)
      const int i = (int)div_floor(pick, V);
      const int x = (int)(pick - (long long)i * V);
      const int node = sh.I_node[i];
      const long long o = (long long)prompt * a.W_cap + d_base + j;
      a.out.out_parent[o] = node;
      a.out.out_token[o] = x;
      a.out.out_node[o] = -1;
      const double lp_o = sh.cum_p[i] + ((double)a.zp[(long long)node * V + x] - sh.lse_p[i]);
      const double lq_o = sh.cum_q[i] + ((double)a.zq[(long long)node * V + x] - sh.lse_q[i]);
      a.out.out_logp_target[o] = lp_o;
      a.out.out_logp_draft[o] = lq_o;
      emit_next(d_base + j, node, x, lp_o, lq_o);
    };
    if constexpr (WARP) {
      // the weights live on the short list (ascending flat index): one wave scans it and writes the samples
      __syncthreads();           // the rows' log-sum-exps (another wave's work since the fold) are in place
      if (wave == 0 && g == 0) {
        const int nU = sh.nU;
        const double wp = lane < nU ? sh.U_p[lane] : 0.0, wr = lane < nU ? fmax(wp - d_c * sh.U_q[lane], 0.0) : 0.0;
        lds_f64* const pre = (lds_f64*)sh.tsum;          // inclusive prefixes: p_beam's, then the residual's
        pre[lane] = wave_inclusive_scan(wp);
        pre[64 + lane] = wave_inclusive_scan(wr);
        const unsigned long long mass_p = __ballot(wp > 0.0), mass_r = __ballot(wr > 0.0);
        wave_lds_fence();
        if (lane < d_cnt) {                              // a draw per lane: the first entry whose prefix exceeds the target
          const bool resid = d_resid && lane == 0;
          lds_f64* const tab = pre + (resid ? 64 : 0);
          const unsigned long long mass = resid ? mass_r : mass_p;
          const double target = (double)d_u * tab[63];
          int at = 0;
#pragma unroll
          for (int step = 32; step >= 1; step >>= 1) at += tab[at + step - 1] > target ? 0 : step;
          if (!(tab[at] > target)) at = mass ? 63 - __clzll((long long)mass) : 0;      // (rounding: the last one with mass)
          emit(nU > 0 ? sh.U_idx[at] : 0, lane);         // (no entry at all, reported as a fault: stay in bounds)
        }
      }
      break;
    } else {
    const bool d_plain = d_cnt > (d_resid ? 1 : 0);    // draws from p_beam
    lds_f64* const ts_r = (lds_f64*)sh.tsum;           // inclusive prefixes over the workgroup's threads: the residual's weights ...
    lds_f64* const ts_p = (lds_f64*)&sh.u;             // ... and p_beam's
    static_assert(sizeof(sh.u) >= sizeof(sh.tsum), "a prefix per thread");
    // every thread's total over its chunk of the slice
    long long per = (len + VL_BLOCK - 1) / VL_BLOCK;
    if (!in_lds) {                      // slices in the workspace: chunks of a power of two (at least one) entries
      long long p2 = 1;
      while (p2 < per) p2 <<= 1;
      per = p2;
    }
    const long long t_lo = min(len, per * tid), t_hi = min(len, t_lo + per);   // slice-local
    double tot_r = 0.0, tot_p = 0.0;
    if (in_lds) {
      for (int j = (int)t_lo; j < (int)t_hi; ++j) {
        const double pv = pl[j];
        if (d_resid) tot_r += fmax(pv - d_c * (double)ql[j], 0.0);
        tot_p += pv;
      }
    } else {
      for (int kind = d_resid ? 0 : 1; kind < (d_plain ? 2 : 1); ++kind) {
        const bool use_q = kind == 0;
        const double c = d_c;
        double ts = 0.0;
        // A thread walking its own chunk would make every load of a wave touch 64 cache lines (measured: 14 us for a
        // 16000-entry slice).  Instead a wave reads the 64 chunks of its threads 64 consecutive entries at a time and
        // adds them up across the lanes: `per` rounds, each holding 64 / per whole chunks or a 64th of one.
        const long long w_lo = per * 64 * wave;
        auto weight = [&](long long jj) -> double {
          if (jj >= len) return 0.0;
          if (jj < n_lds) return use_q ? fmax((double)pl[(int)jj] - c * (double)ql[(int)jj], 0.0) : (double)pl[(int)jj];
          return use_q ? fmax((double)pbg[jj] - c * (double)qbg[jj], 0.0) : (double)pbg[jj];
        };
        // eight rounds from r0 on (rounds beyond `lim` count nothing): one home for all eight in all but one group of
        // a wave, and then loads without branches between them, which the compiler keeps in flight together
        auto weights8 = [&](long long r0, long long lim, double (&w)[8]) {
          const long long b0 = w_lo + r0 * 64, b1 = w_lo + min(r0 + 8, lim) * 64;     // the group's range (uniform)
          if (b0 >= n_lds && b0 < len) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const long long jj = b0 + k * 64 + lane, jc = min(jj, len - 1);
              const double pv = pbg[jc], qv = use_q ? (double)qbg[jc] : 0.0;
              const double v = use_q ? fmax(pv - c * qv, 0.0) : pv;
              w[k] = (r0 + k < lim && jj < len) ? v : 0.0;
            }
          } else if (b1 <= n_lds) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const int jc = (int)min(b0 + k * 64 + lane, n_lds - 1);
              const double pv = pl[jc], qv = use_q ? (double)ql[jc] : 0.0;
              const double v = use_q ? fmax(pv - c * qv, 0.0) : pv;
              w[k] = (r0 + k < lim) ? v : 0.0;
            }
          } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = r0 + k < lim ? weight(b0 + k * 64 + lane) : 0.0;
          }
        };
        if (per < 64) {
          // sums over aligned groups of `per` lanes by lane moves inside the SIMD (one LDS exchange for groups of 32);
          // a group's first lane leaves the chunk's total in the table, where its thread picks it up
          const int S = 64 / (int)per;                  // chunks per round
          for (long long r0 = 0; r0 < per; r0 += 8) {
            double w[8];
            weights8(r0, per, w);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              double v = w[k];
              if (per >= 2) v += dpp_move_f64<0xB1, 0xf>(v);      // quad_perm [1,0,3,2]
              if (per >= 4) v += dpp_move_f64<0x4E, 0xf>(v);      // quad_perm [2,3,0,1]
              if (per >= 8) v += dpp_move_f64<0x141, 0xf>(v);     // row_half_mirror: the other quad of the eight
              if (per >= 16) v += dpp_move_f64<0x140, 0xf>(v);    // row_mirror: the other half of the sixteen
              if (per >= 32) v += __shfl_xor(v, 16);
              if (r0 + k < per && (lane & ((int)per - 1)) == 0)
                sh.tsum[wave * 64 + (int)(r0 + k) * S + lane / (int)per] = v;
            }
          }
          wave_lds_fence();
          ts = sh.tsum[tid];
        } else {
          const long long rpc = per / 64;                // rounds per chunk (a power of two); chunk after chunk
          double acc = 0.0;
          for (long long r0 = 0; r0 < per; r0 += 8) {
            double w[8];
            weights8(r0, per, w);                                                       // per >= 64 is a multiple of 8
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              acc += w[k];
              if (((r0 + k + 1) & (rpc - 1)) == 0) {
                const double tot = wave_sum(acc);
                if (lane == (int)((r0 + k) / rpc)) ts = tot;
                acc = 0.0;
              }
            }
          }
        }
        if (use_q) tot_r = ts; else tot_p = ts;
        wave_lds_fence();
      }
    }
    stamp(70);
    const double incl_r = wave_inclusive_scan(tot_r), incl_p = wave_inclusive_scan(tot_p);
    __syncthreads();
    if (lane == 63) { sh.scan_w[wave] = incl_r; sh.scan_w2[wave] = incl_p; }
    if (tid == 0) sh.counter = 0;
    __syncthreads();
    double before_r = 0.0, before_p = 0.0;
    for (int w = 0; w < wave; ++w) { before_r += sh.scan_w[w]; before_p += sh.scan_w2[w]; }
    ts_r[tid] = before_r + incl_r;
    ts_p[tid] = before_p + incl_p;
    // ... and over the workgroups (same order everywhere), gathered and scanned by one wave for either kind: the first for
    // the residual, whose totals have to be exchanged, the second for p_beam, whose totals are known from the row sums
    // (see above; the same in every workgroup of the prompt) unless a gathering thread saw several pieces.
    // (These are the prompt's last exchanges: nobody waits for their banks to be free again.)
    lds_f64* const pre_r = (lds_f64*)sh.gpart;
    lds_f64* const pre_p = (lds_f64*)sh.ptot;
    if ((wave == 0 && d_resid) || (wave == 1 && d_plain)) {
      const bool known_totals = wave == 1 && sh.ptot_ok != 0;
      lds_f64* const tab = wave == 0 ? pre_r : pre_p;
      double v[4];
      if (!known_totals) {
        const unsigned long long tag = exchange_tag(nonce + epoch + 1 + wave);
        Slot* const bank = slots + (wave == 0 ? slx0 : slx1);
        double mine = 0.0;
        for (int w = 0; w < VL_WAVES; ++w) mine += wave == 0 ? sh.scan_w[w] : sh.scan_w2[w];
        if (lane == 0) dense_post(bank, a.G, g, mine, tag);
        if (!wave_collect4(bank, a.G, g, mine, tag, v, a.sync_limit)) give_up();
#pragma unroll
        for (int k = 0; k < 4; ++k) if (lane + 64 * k < a.G) tab[lane + 64 * k] = v[k];
        wave_lds_fence();          // now four consecutive workgroups per lane
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int w = 4 * lane + k;
        bool holds = w < a.G;
        if (known_totals) holds = holds && w / cut.wg_per_row < nI && w % cut.wg_per_row < geo_pieces;
        v[k] = holds ? (double)tab[w] : 0.0;
      }
      int nz = -1;                 // the last workgroup that holds any mass (uniform: from ballots)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const unsigned long long has = __ballot(v[k] > 0.0);
        if (has) nz = max(nz, 4 * (63 - __clzll((long long)has)) + k);
      }
      v[1] += v[0]; v[2] += v[1]; v[3] += v[2];
      double incl = v[3];
      incl = wave_inclusive_scan(incl);
      double excl = __shfl_up(incl, 1);
      if (lane == 0) excl = 0.0;
#pragma unroll
      for (int k = 0; k < 4; ++k) if (4 * lane + k < a.G) tab[4 * lane + k] = excl + v[k];
      if (lane == 0) sh.last_mass[wave] = nz;
    }
    __syncthreads();
    stamp(71);
    if (sh.abort) return;
    if (tid < d_cnt) {
      const bool resid = d_resid && tid == 0;
      lds_f64* const tab = resid ? pre_r : pre_p;
      const double target = (double)d_u * tab[a.G - 1];
      sh.d_target[tid] = target;
      // owner: the first workgroup whose inclusive prefix exceeds the target (rounding: the last one with mass)
      int lo = 0, hi = a.G;
      while (lo < hi) { const int mid = (lo + hi) >> 1; if (tab[mid] > target) hi = mid; else lo = mid + 1; }
      const int owner = lo < a.G ? lo : max(sh.last_mass[resid ? 0 : 1], 0);
      if (owner == g) sh.S_tmp[atomicAdd(&sh.counter, 1)] = tid;
    }
    __syncthreads();
    stamp(72);
    const int n_mine = sh.counter;
    for (int k = 0; k < n_mine; ++k) {
      const int j = sh.S_tmp[k];
      const bool resid = d_resid && j == 0;
      lds_f64* const ts = resid ? ts_r : ts_p;
      const double before = g > 0 ? (double)(resid ? pre_r : pre_p)[g - 1] : 0.0;
      const double target = sh.d_target[j];
      // the thread whose inclusive prefix is the first to exceed the target (rounding: the last one with mass,
      // found by the last thread)
      const bool above = before + ts[tid] > target;
      const bool prev_above = tid > 0 && (before + ts[tid - 1] > target);
      const bool holder = (above && !prev_above) || (tid == VL_BLOCK - 1 && !above);
      if (in_lds) {
        if (holder) {
          int th = tid;
          if (!above)
            while (th > 0 && !(ts[th] > ts[th - 1])) --th;
          const long long c_lo = min(len, per * th), c_hi = min(len, c_lo + per);
          double accl = before + (th > 0 ? (double)ts[th - 1] : 0.0);
          long long pick = -1, last = -1;
          for (long long jj = c_lo; jj < c_hi; ++jj) {
            const double v = resid ? fmax((double)pl[(int)jj] - d_c * (double)ql[(int)jj], 0.0) : (double)pl[(int)jj];
            if (v > 0.0) last = jj;
            accl += v;
            if (accl > target) { pick = jj; break; }
          }
          if (pick < 0) pick = last >= 0 ? last : c_lo;
          emit(min(pick + e_lo, total - 1), j);
        }
      } else {
        // slices in the workspace: one thread walking its chunk would wait for a load per element, so the first wave
        // takes the chunk 64 entries at a time (coalesced loads, a scan across the lanes)
        if (holder) {
          int th = tid;
          if (!above)
            while (th > 0 && !(ts[th] > ts[th - 1])) --th;
          sh.pick_th = th;
        }
        __syncthreads();
        if (wave == 0) {
          const int th = sh.pick_th;
          const long long c_lo = min(len, per * th), c_hi = min(len, c_lo + per);
          double start = before + (th > 0 ? (double)ts[th - 1] : 0.0);
          long long pick = -1, last = -1;
          for (long long b0 = c_lo; b0 < c_hi && pick < 0; b0 += 64) {
            const long long jj = b0 + lane;
            double v = 0.0;
            if (jj < c_hi) v = resid ? fmax(ldp(jj) - d_c * ldq(jj), 0.0) : ldp(jj);
            double incl = v;
            incl = wave_inclusive_scan(incl);
            const unsigned long long mass = __ballot(v > 0.0);
            if (mass) last = b0 + 63 - __clzll((long long)mass);
            const unsigned long long over = __ballot(start + incl > target);
            if (over) pick = b0 + __ffsll((long long)over) - 1;
            start += __shfl(incl, 63);
          }
          if (pick < 0) pick = last >= 0 ? last : c_lo;
          if (lane == 0) emit(min(pick + e_lo, total - 1), j);
        }
        __syncthreads();                   // sh.pick_th is free again
      }
    }
    break;
    }
  }

  stamp(99);
  if (g == 0) clear_out_slots(n_out);
  if (g == 0 && tid == 0) {
    a.out.l_last[prompt] = l_last;
    a.out.n_out[prompt] = n_out;
    a.out.near_tie_count[prompt] = near_tie;
    if (a.nx_on) a.nx.n_next[prompt] = n_out;
  }
}

// ------------------------------------------------------------------------------------------------ host side
namespace {

struct VerifyPlan {
  int I_cap, G, lds_elems;
  bool small_nodes;        // the layer kernel built for prompts of at most NODE_CAP_SMALL nodes serves (more LDS for slices)
  int group;               // prompts per launch of the layer kernel (all of them, unless they do not fit the device at once)
  size_t lds_bytes;        // dynamic LDS of the layer kernel
  SlotLayout sl;
  long long slice_cap;     // elements of the largest slice of I x V a workgroup can get
};

int32_t check_verify(const dsbd_forest* f, int V, const dsbd_params* p) {
  if (!f || !p) return DSBD_ERR_INVALID;
  if (f->n_prompts < 0 || f->n_trees < 0 || f->n_nodes < 0) return DSBD_ERR_INVALID;
  if (V < 1 || V > (1 << 30)) return DSBD_ERR_UNSUPPORTED;     // positions in a row are 32-bit integers with room to step past the end
  if (p->W_cap < 1 || p->W_cap > 64) return DSBD_ERR_UNSUPPORTED;
  if (p->W_min < 1 || p->W_min > p->W_cap || p->W_L > p->W_cap) return DSBD_ERR_INVALID;
  if (!(p->t <= 1.0f)) return DSBD_ERR_INVALID;      // also rejects NaN (which would otherwise read as dynamic width 0)
  if (f->max_tree_nodes < 1 || f->max_tree_nodes > DSBD_MAX_TREE_NODES) return DSBD_ERR_UNSUPPORTED;
  if (f->max_prompt_trees < 1 || f->max_prompt_trees > 64) return DSBD_ERR_UNSUPPORTED;
  if (p->W_L <= 0 && f->max_prompt_trees > p->W_cap) return DSBD_ERR_INVALID;
  if ((long long)f->max_prompt_trees * f->max_tree_nodes > NODE_CAP) return DSBD_ERR_UNSUPPORTED;
  if (f->max_depth < 0 || f->max_depth >= DSBD_MAX_TREE_NODES) return DSBD_ERR_INVALID;
  // warping T: top_k = 0 and top_p >= 1 is the identity; otherwise the joint is cut to its top_k <= WARP_K_MAX
  // entries first (top-p alone would need an unbounded candidate list)
  if (p->top_k < 0 || !(p->top_p >= 0.0f)) return DSBD_ERR_INVALID;
  if (p->top_k > WARP_K_MAX || (p->top_k == 0 && p->top_p > 0.0f && p->top_p < 1.0f)) return DSBD_ERR_UNSUPPORTED;
  if (p->top_k > 0) {
    const long long cap = p->W_cap > f->max_prompt_trees ? p->W_cap : f->max_prompt_trees;
    if (cap * V > 0x7fffffffLL) return DSBD_ERR_UNSUPPORTED;     // flat indices travel as 32-bit integers
  }
  return DSBD_OK;
}

// What the layer kernel may occupy: all its workgroups must be resident at once.
struct DeviceLimits { int cus, blocks_per_cu; };
const DeviceLimits& device_limits() {
  static DeviceLimits lim = {0, 0};
  static std::once_flag once;
  std::call_once(once, [] {
    int dev = 0, v = 0;
    lim.cus = 256;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      lim.cus = v;
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(verify_layers_kernel<false, NODE_CAP>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, VL_DYN_LDS_BYTES);
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(verify_layers_kernel<true, NODE_CAP>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, VL_DYN_LDS_BYTES);
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(verify_layers_kernel<true, NODE_CAP, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, VL_DYN_LDS_BYTES);
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(verify_layers_kernel<false, NODE_CAP_SMALL>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, VL_DYN_LDS_BYTES_SMALL);
    int nb = 0, nb3 = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, verify_layers_kernel<false, NODE_CAP>, VL_BLOCK, VL_DYN_LDS_BYTES) != hipSuccess || nb < 1)
      nb = 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb3, verify_layers_kernel<false, NODE_CAP_SMALL>, VL_BLOCK, VL_DYN_LDS_BYTES_SMALL) != hipSuccess || nb3 < 1)
      nb3 = 1;
    lim.blocks_per_cu = nb < nb3 ? nb : nb3;
    (void)hipGetLastError();
  });
  return lim;
}

// Prompts of few nodes and no warping (whose scratch lists use the per-node arrays at full size) take the kernel variant
// with the short per-node arrays, which leaves more of the LDS to the slices.
bool small_prompts(const dsbd_forest* f, const dsbd_params* p) {
  return p->top_k == 0 && (long long)f->max_prompt_trees * f->max_tree_nodes <= NODE_CAP_SMALL;
}

// Joint entries of a slice that the LDS holds (both arrays).
long long lds_slice_entries(const dsbd_forest* f, const dsbd_params* p) {
  return (small_prompts(f, p) ? VL_DYN_LDS_BYTES_SMALL : VL_DYN_LDS_BYTES) / 16;
}

// Workgroups per prompt of the layer kernel.  `sparing`: 4000 joint entries each, whatever the problem (make_verify_plan).
int layer_workgroups(const dsbd_forest* f, int V, const dsbd_params* p, bool sparing) {
  // one workgroup per compute unit in total, shared evenly by the prompts, at least 4096 joint elements per
  // workgroup.  More prompts than workgroups fit the device at once: groups of prompts, one launch after the other
  // (Algorithm 1 runs per prompt), one workgroup per prompt.
  const DeviceLimits& lim = device_limits();
  const long long joint = (long long)f->max_prompt_trees * V;
  int G = f->n_prompts > 0 ? lim.cus / f->n_prompts : 1;
  if (sparing) {
    const long long by_work = (joint + 3999) / 4000;
    if (G > by_work) G = (int)by_work;
    return G < 1 ? 1 : G;
  }
  // ... minus compute units for the workgroups that take the rows' statistics meanwhile: one per MB of logits (30 GB/s for
  // a unit on its own, over the 35 us that the shortest walks take), at most a quarter of the device, as long as the
  // coarser slices fit the LDS.  A lone prompt loses next to nothing by it (its exchanges get shorter as its passes get
  // longer).  With several prompts it takes 90 MB of logits that would otherwise stand behind the layers (13 us), and
  // 300 MB where the slices outgrow the LDS, up to twice its size.  The dynamic width on unwarped joints passes over the slices for every entry of its chains: there a row is
  // never cut into less than 85 % of the pieces.  Measured, verification in us with 0 / a quarter of the units kept:
  // 8 beams, 248 nodes x 128256 137 / 109 (t = 0.7 310 / 286), 64 nodes 73 / 62; 2 prompts of 8
  // beams, 496 nodes x 32000 94 / 85, x 128256 199 / 181; 4 prompts, 992 nodes x 32000 120 / 111 (t = 0.7 304 / 341, an eighth
  // 316), 256 nodes 78 / 79; 16 prompts of 4 beams, 1984 nodes x 16000 105 / 97 (t = 0.7 248 /
  // 308), 341 nodes x 32000 88 / 112; 3 prompts, 103 nodes x 50273, t = 0.7: 84 / 78 / 72 / 66 workgroups each 104 / 104 / 98 / 99.
  {
    const long long bytes = 2LL * f->n_nodes * V * 4;
    long long keep = (bytes + (1 << 20) - 1) / (1 << 20);
    if (keep > lim.cus / 4) keep = lim.cus / 4;
    const int W = f->max_prompt_trees, P = f->n_prompts;
    const bool chains = p->t >= 0.0f;
    int Gk = P > 0 ? (int)((lim.cus - keep) / P) : 0;
    if (P > 1 && chains) Gk = std::max(Gk, (G / W * 85 + 99) / 100 * W);
    if (Gk >= W && Gk < G) {
      const long long slice = slice_cut(W, V, Gk).len, room = lds_slice_entries(f, p);
      if (P == 1 ? slice <= room : chains || bytes >= 300000000LL ? slice <= 2 * room : bytes >= 90000000LL && slice <= room) G = Gk;
    }
  }
  // (sized by the joint of the input beams, which is what a fixed width keeps every layer at: shorter slices make shorter
  // passes and more partners longer exchanges.  Measured, call in us at 16 / 32 / 48 / 64 / 96 / 128 / 160 / 192 workgroups
  // of a prompt: 4 x 32000 joint entries 49.4 / 38.1 / 36.1 / 36.0 / 36.6 / 36.3 / 37.6 / 37.8; 8 x 32000: 99.8 / 65.8 / 50.1 /
  // 48.2 / 48.0 / 48.1 / 48.3 / 48.4; 8 x 128256:
  // 516 / 303 / 238 / 181 / 154 / 121 / 116 / 108.  5 x 128256 plain: 324 / 201 / 140 /
  // 121 / 81 / 77 / 73 / 75.  So 2000 entries per workgroup up to 128 of them, 4000 beyond.)
  long long by_work = (joint + 1999) / 2000;
  if (by_work > 128) by_work = std::max(128LL, (joint + 3999) / 4000);
  if (G > by_work) G = (int)by_work;
  // (workgroups beyond a multiple of the rows hold no piece but take part in every exchange)
  if (f->max_prompt_trees > 0 && G > f->max_prompt_trees) G -= G % f->max_prompt_trees;
  if (G < 1) G = 1;
  return G > 256 ? 256 : G;
}

VerifyPlan plan_with_workgroups(const dsbd_forest* f, int V, const dsbd_params* p, bool alias, int G) {
  VerifyPlan pl;
  const DeviceLimits& lim = device_limits();
  const int resident = lim.cus * lim.blocks_per_cu;
  pl.I_cap = p->W_cap > f->max_prompt_trees ? p->W_cap : f->max_prompt_trees;
  pl.G = G;
  pl.group = f->n_prompts;
  if ((long long)pl.group * G > resident) pl.group = resident / G;     // G is 1 here
  if (pl.group < 1) pl.group = 1;
  pl.small_nodes = small_prompts(f, p);
  const long long cap = lds_slice_entries(f, p) * (alias ? 2 : 1);   // one array instead of two when q_beam is p_beam
  // exchange slots: every workgroup's slots of an exchange start a 128-byte line (no two writers per line)
  {
    auto up8 = [](int v) { return (v + LINE_SLOTS - 1) / LINE_SLOTS * LINE_SLOTS; };
    const int layers = f->max_depth + 1;
    SlotLayout& sl = pl.sl;
    int off = 0;
    sl.x[0] = off; off += G * LINE_SLOTS;
    sl.x[1] = off; off += G * LINE_SLOTS;
    sl.r_w = up8(4 * pl.I_cap);
    sl.r = off; sl.r_stride = G * sl.r_w; off += layers * sl.r_stride;
    sl.acc = off; off += 2 * NACC * LINE_SLOTS;
    sl.acc0 = off; off += up8(2 * NACC);
    sl.prompt_stride = off;
  }
  // dynamic LDS for the p_beam / q_beam slices: what one slice needs, at most VL_DYN_LDS_BYTES for the two arrays
  long long need = 2;                        // the longest slice any number of input rows can give
  for (int nI = 1; nI <= pl.I_cap; ++nI) {
    const long long len = slice_cut(nI, V, G).len;
    if (len > need) need = len;
  }
  need = (need + 1) & ~1LL;
  pl.slice_cap = need;
  pl.lds_elems = (int)(need < cap ? need : cap);
  pl.lds_bytes = ((size_t)pl.lds_elems * (alias ? 8 : 16) + 15) & ~(size_t)15;
  return pl;
}

size_t carve_verify(WorkspaceCarver& ws, const dsbd_forest* f, const VerifyPlan& pl, double** pb, double** qb, double** red) {
  const size_t P = (size_t)f->n_prompts;
  ws.take<long long>(512);                 // timeline of the layer kernel (diagnostics), first in the workspace
  ws.take<unsigned long long>(32);         // replay count of launches recorded into a graph (one word, a line of its own)
  // slices that do not fit the LDS: a region per workgroup of a launch (the launches of a forest that runs in groups
  // of prompts follow each other and share the regions); exchange slots: a region per prompt
  *pb = ws.take<double>((size_t)pl.group * pl.G * (size_t)pl.slice_cap);
  *qb = ws.take<double>((size_t)pl.group * pl.G * (size_t)pl.slice_cap);
  *red = ws.take<double>(P * (size_t)pl.sl.prompt_stride * 2);
  return ws.total();
}

// Warped joints: one workgroup walks a prompt's layers from the rows' records.
VerifyPlan warped_plan(const dsbd_forest* f, const dsbd_params* p) {
  (void)device_limits();                   // (the kernel's dynamic LDS is set up there)
  VerifyPlan pl = {};
  pl.I_cap = p->W_cap > f->max_prompt_trees ? p->W_cap : f->max_prompt_trees;
  pl.G = 1;
  pl.group = f->n_prompts;
  pl.lds_bytes = dsbd_align_up((size_t)2 * pl.I_cap * p->top_k * (sizeof(double) + 2 * sizeof(int)), 16);     // a layer's candidates
  return pl;
}

size_t carve_warped(WorkspaceCarver& ws, const dsbd_forest* f, const RowsPlan& rp, RowsArgs* ra) {
  const size_t rows = (size_t)f->n_nodes * 2;
  ws.take<long long>(512);                 // timeline of the layer kernel
  const bool in_records = rp.compact && rp.nchunk == 1;
  ra->part = ws.take<double2>(in_records ? 0 : rows * rp.nchunk);
  if (in_records) ra->part = nullptr;
  ra->sub = ws.take<float>(rows * rp.nchunk * rp.parts);
  ra->rec = ws.take<char>(rows * (size_t)rp.rec_stride);
  return ws.total();
}

// Records with logits, unless smaller ones bring the workspace down to the 32 MiB of dsbd_verify_forest_static where those do
// not (large batches over vocabularies of a few hundred tokens): tokens of 8 or 16 bits, a dependent load per layer more, or no
// entries at all.  `bytes`: what the call asks for.  A call with smaller records asks for the whole 32 MiB, so that the sizes
// rise with the batch: a buffer for the largest call serves the others, records with logits or not.
RowsPlan warped_rows(const dsbd_forest* f, int V, int K, size_t* bytes = nullptr) {
  auto size = [&](const RowsPlan& rp) { WorkspaceCarver ws(nullptr); RowsArgs ra; return carve_warped(ws, f, rp, &ra) + 256; };
  const size_t most = DSBD_STATIC_SCRATCH_BYTES;
  const RowsPlan plain = rows_plan(V, K, 0);
  const size_t n = size(plain);
  RowsPlan rp = plain;
  if (n > most && V <= 65536) {
    rp = rows_plan(V, K, V <= 256 ? 1 : 2);
    if (size(rp) > most && V <= VR_BARE) rp = rows_plan(V, K, -1);
    if (size(rp) > most) rp = plain;
  }
  if (bytes) *bytes = rp.compact ? most : n;
  return rp;
}

size_t verify_workspace(const dsbd_forest* f, const VerifyPlan& pl) {
  WorkspaceCarver ws(nullptr);
  double *pb, *qb, *red;
  return carve_verify(ws, f, pl, &pb, &qb, &red) + 256;
}

// More workgroups per prompt bring more exchange slots (every layer has its own) and, where rows and workgroups do not
// divide, longer slices in all.  The array behind dsbd_verify_forest_static is 32 MiB: a problem that fits it with 4000
// joint entries per workgroup keeps to those if it would outgrow it otherwise.  (Both entry points take the same plan.)
VerifyPlan make_verify_plan(const dsbd_forest* f, int V, const dsbd_params* p, bool alias = false) {
  const DsbdKnobs& knobs = dsbd_knobs();
  const DeviceLimits& lim = device_limits();
  if (knobs.verify_g >= 1 && knobs.verify_g <= 256 && (long long)knobs.verify_g * f->n_prompts <= lim.cus * lim.blocks_per_cu)   // tuning knob
    return plan_with_workgroups(f, V, p, alias, knobs.verify_g);
  const VerifyPlan pl = plan_with_workgroups(f, V, p, alias, layer_workgroups(f, V, p, false));
  if (verify_workspace(f, pl) <= (size_t)DSBD_STATIC_SCRATCH_BYTES) return pl;
  const VerifyPlan small = plan_with_workgroups(f, V, p, alias, layer_workgroups(f, V, p, true));
  return verify_workspace(f, small) <= (size_t)DSBD_STATIC_SCRATCH_BYTES ? small : pl;
}

// Two layer kernels on different streams must not share the compute units: each waits for workgroups of its own that
// the other one's keep out.  The library therefore orders its layer launches itself once it has seen calls on more
// than one stream: the first change of stream waits for the device to drain, and from then on layers_done is recorded
// behind every layer launch and a launch on another stream than the last one waits for it.  (Recording from the start
// would cost every single-stream caller 6 us per call, measured.)  Warped calls wait for nobody and take part only where
// their workspace is the static array, which they share with every other static call.  One per device; the event is
// created on first use and kept until the process ends.  enqueue makes one call's launches, records and waits a unit among
// host threads, with or without the event: the kernels of a warped call follow each other on one workspace.
struct LaunchOrder {
  bool tried = false;
  std::atomic<bool> ok{false};       // the event exists
  hipEvent_t layers_done = nullptr;
  hipStream_t last_stream = nullptr;
  bool have_last = false, several_streams = false;
  std::mutex enqueue;
};
LaunchOrder* launch_order_of_current_device(bool may_create) {
  static LaunchOrder table[64];
  static std::mutex mutex;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lock(mutex);
  LaunchOrder& s = table[dev];
  if (!s.tried && may_create) {
    s.tried = true;
    const unsigned ev = hipEventDisableTiming | (dsbd_knobs().event_fence ? 0u : (unsigned)hipEventDisableSystemFence);
    s.ok = hipEventCreateWithFlags(&s.layers_done, ev) == hipSuccess;
    if (!s.ok) (void)hipGetLastError();
  }
  return &s;
}

// Threads per row of the row statistics.  A wave with a row of its own streams without a break between its loads and waits
// for nobody; a workgroup on one row waits at its end for the slowest wave, for the row's few words and for the next
// workgroup, on a compute unit that the layers' LDS leaves to one workgroup at a time: 1, 1.06, 1.15 and 1.35 of the time
// per row for 64 to 512 threads.  Against that stand the rounds that the workgroups make on the compute units that the layers
// leave free (or on all of them, when they leave none: then the rows run behind the layers).  Measured, verification in us with 512 / 256 / 128 / 64 threads per row: 200 prompts, 8400
// rows x 1000 172 / 120 / 87 / 80, x 8000 324 / 249 / 235 / 234; 8 prompts, 3968 rows x 32000 218 / 193 / 191 / 192; 1024 rows 110 /
// 104 / 103 / 102; one prompt, 496 rows x 128256 109 / 98 / 97 / 96, 256 rows 78 / 78 / 78 / 81, 64 rows 52 / 52 / 52 / 76.
int statistics_threads(const dsbd_forest* f, const VerifyPlan& pl, unsigned rows) {
  const int cus = device_limits().cus;
  const int left = cus - pl.group * pl.G, units = left > 0 ? left : cus;
  int threads = 64;
  double best = 0.0;
  for (int t = 64; t <= VL_BLOCK; t *= 2) {
    const int rows_per_wg = VL_BLOCK / t;
    double rounds = ceil((double)rows / rows_per_wg) / units;
    rounds = rounds <= 3.0 ? ceil(rounds) : rounds + 0.5;
    const double cost = rounds * rows_per_wg * (t == 64 ? 1.0 : t == 128 ? 1.06 : t == 256 ? 1.15 : 1.35);
    if (t == 64 || cost < best) { best = cost; threads = t; }
  }
  return threads;
}

// In front of a layer kernel that is recorded into a graph: every replay repeats the launch's arguments, so what tells
// its exchange slots from those of the replay before is this count (whatever the word held to begin with).
__global__ void bump_replay_count_kernel(unsigned long long* count) { *count += 1; }

}  // namespace

extern "C" size_t dsbd_verify_forest_workspace_bytes(const dsbd_forest* f, int32_t V, const dsbd_params* p) {
  if (check_verify(f, V, p) != DSBD_OK) return 0;
  if (p->top_k > 0) {
    size_t bytes;
    (void)warped_rows(f, V, p->top_k, &bytes);
    return bytes;
  }
  return verify_workspace(f, make_verify_plan(f, V, p));
}

namespace {
// static_scratch: the workspace is the device array that all such calls share, and the call must not allocate: it takes
// part in the ordering across streams only if an earlier ordinary call or dsbd_init() has made the event.
// next: the next-beam plan to be written along with the output beams (nullptr: none).  With keep_one == 0 the layer
// kernel writes it itself; the single surviving beam of keep_one != 0 needs all of a prompt's output beams side by
// side, which sit in several workgroups' hands: there the selection kernel is launched behind the verification.
int32_t verify_impl(const dsbd_forest* f, const dsbd_verify_in* in, const dsbd_params* p, const dsbd_verify_out* out,
                    void* workspace, size_t workspace_bytes, int32_t* fault, void* stream_, bool static_scratch,
                    const dsbd_next_beams* next = nullptr, int keep_one = 0) {
  if (!in || !out || !fault) return DSBD_ERR_INVALID;
  int32_t rc = check_verify(f, in->V, p);
  if (rc != DSBD_OK) return rc;
  if (next && (!next->n_next || !next->src_tree || !next->src_out || !next->path_len || !next->path || !next->token ||
               !next->logp_target || !next->logp_draft))
    return DSBD_ERR_INVALID;
  if (f->n_nodes == 0 || f->n_trees == 0 || f->n_prompts == 0) return DSBD_OK;
  if (!f->tree_prompt || !f->tree_off || !f->parent || !f->token) return DSBD_ERR_INVALID;
  if (!in->logits_target || !in->logits_draft || !in->beam_logp_target || !in->beam_logp_draft || !in->u_accept ||
      !in->u_resid || !in->u_fill)
    return DSBD_ERR_INVALID;
  if (!out->node_status || !out->l_last || !out->layer_width || !out->n_out || !out->out_parent || !out->out_token ||
      !out->out_node || !out->out_logp_target || !out->out_logp_draft || !out->near_tie_count)
    return DSBD_ERR_INVALID;
  if (!workspace) return DSBD_ERR_INVALID;
  const DsbdKnobs& knobs = dsbd_knobs();
  // the same arrays given for both models: q_beam is p_beam and is kept, and computed, once (in the same workspace)
  const bool alias = in->logits_target == in->logits_draft && in->beam_logp_target == in->beam_logp_draft;
  const bool warped = p->top_k > 0;
  const VerifyPlan pl = warped ? warped_plan(f, p) : make_verify_plan(f, in->V, p, alias);
  if (workspace_bytes < (warped ? dsbd_verify_forest_workspace_bytes(f, in->V, p) : verify_workspace(f, pl))) return DSBD_ERR_WORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(stream_);

  char* wbase = reinterpret_cast<char*>(dsbd_align_up(reinterpret_cast<uintptr_t>(workspace), 256));
  WorkspaceCarver ws(wbase);
  double *pb = nullptr, *qb = nullptr, *red = nullptr;
  RowsArgs ra;
  const RowsPlan rp = warped_rows(f, in->V, p->top_k);
  if (warped) carve_warped(ws, f, rp, &ra); else carve_verify(ws, f, pl, &pb, &qb, &red);

  const bool want_stats = out->lse_target || out->lse_draft || out->node_logp_target || out->node_logp_draft;
  LaunchOrder* state = launch_order_of_current_device(!static_scratch);
  std::unique_lock<std::mutex> enqueue_lock;
  if (state) enqueue_lock = std::unique_lock<std::mutex>(state->enqueue);
  if (state && (!state->ok || (warped && !static_scratch))) state = nullptr;      // (no part in the order)
  // a stream under capture takes no part in the ordering of layer launches (an event recorded into a capture cannot
  // be waited for from outside it): replays of such a graph are the caller's to keep apart from other verifications
  bool capturing = false;
  {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cs) == hipSuccess) capturing = cs != hipStreamCaptureStatusNone;
    else { (void)hipGetLastError(); capturing = true; }
  }
  LayersArgs la;
  la.n_prompts = f->n_prompts; la.n_trees = f->n_trees; la.n_nodes = f->n_nodes;
  la.tree_prompt = f->tree_prompt; la.tree_off = f->tree_off; la.parent = f->parent; la.token = f->token;
  la.rank = f->draft_rank; la.max_depth = f->max_depth; la.max_prompt_trees = f->max_prompt_trees;
  la.max_tree_nodes = f->max_tree_nodes;
  la.V = in->V; la.zp = in->logits_target; la.zq = in->logits_draft;
  la.blp = in->beam_logp_target; la.blq = in->beam_logp_draft;
  la.u_acc = in->u_accept; la.u_res = in->u_resid; la.u_fill = in->u_fill;
  la.W_L = p->W_L; la.W_min = p->W_min; la.W_cap = p->W_cap; la.t = p->t;
  la.out = *out;
  la.pb = pb; la.qb = qb; la.red = red; la.slice_cap = pl.slice_cap;
  la.trace = knobs.verify_trace ? reinterpret_cast<long long*>(wbase) : nullptr;
  la.trace_wg = knobs.verify_trace_wg;
  la.sync_limit = SYNC_LIMIT_TICKS;
  if (knobs.verify_sync_limit_us >= 1 && knobs.verify_sync_limit_us <= 10000000LL)   // bound of the kernel's waits (default 3 s)
    la.sync_limit = knobs.verify_sync_limit_us * 100;
  la.mute_wg = knobs.verify_mute_wg;   // error-path test hook
  // Exchange slots carry a tag made of this number and the exchange's index: nothing an earlier launch left in the
  // workspace can pass for a value of this one, so the slots need no clearing.
  la.nonce = dsbd_launch_nonce();
  la.replay = nullptr;
  la.rec = nullptr; la.rec_stride = 0; la.rec_compact = 0;
  if (capturing && !warped) {
    unsigned long long* const count = reinterpret_cast<unsigned long long*>(wbase + 512 * sizeof(long long));
    hipLaunchKernelGGL(bump_replay_count_kernel, dim3(1), dim3(1), 0, stream, count);
    la.replay = count;
  }
  la.G = pl.G; la.I_cap = pl.I_cap; la.sl = pl.sl; la.lds_elems = pl.lds_elems; la.fault = fault;
  la.lds_slice = pl.lds_elems;
  la.alias = alias ? 1 : 0;
  la.nx_on = (next && !keep_one) ? 1 : 0;
  la.lse_p = out->lse_target; la.lse_q = out->lse_draft; la.logp_p = out->node_logp_target; la.logp_q = out->node_logp_draft;
  if (la.nx_on) la.nx = *next; else la.nx = dsbd_next_beams{};
  if (knobs.verify_lds_slice >= 0 && knobs.verify_lds_slice < la.lds_slice) la.lds_slice = knobs.verify_lds_slice;   // tuning / test knob
  la.top_k = p->top_k; la.top_p = (p->top_p > 0.0f && p->top_p < 1.0f) ? p->top_p : 1.0f;
  // Ordinary launches: a launch was sized to fit the device at once, and every wait inside the kernel is bounded.
  // (A cooperative launch would also guarantee co-residency against work on other streams, but it made rocprofv3
  // crash at process exit on ROCm 7.2 and costs extra launch latency.)
  if (state && !capturing && state->have_last && state->last_stream != stream) {
    if (!state->several_streams) {
      if (hipDeviceSynchronize() != hipSuccess) return DSBD_ERR_HIP;
      state->several_streams = true;
    } else if (hipStreamWaitEvent(stream, state->layers_done, 0) != hipSuccess) {
      return DSBD_ERR_HIP;
    }
  }
  hipError_t le;
  if (warped) {
    ra.n_nodes = f->n_nodes; ra.V = in->V; ra.K = p->top_k; ra.chunk = rp.chunk; ra.nchunk = rp.nchunk; ra.parts = rp.parts;
    ra.alias = la.alias; ra.zp = in->logits_target; ra.zq = in->logits_draft;
    ra.parent = f->parent; ra.token = f->token; ra.rec_stride = rp.rec_stride; ra.compact = rp.compact;
    ra.lse_p = out->lse_target; ra.lse_q = out->lse_draft; ra.logp_p = out->node_logp_target; ra.logp_q = out->node_logp_draft;
    ra.fault = fault; ra.report = want_stats ? 1 : 0;
    ra.direct = knobs.warp_fast ? INT_MAX : 0;
    le = launch_verify_rows(ra, stream);
    la.rec = ra.rec; la.rec_stride = rp.rec_stride; la.rec_compact = rp.compact;
    for (la.prompt0 = 0; le == hipSuccess && la.prompt0 < f->n_prompts; la.prompt0 += la.layer_wgs) {
      la.layer_wgs = std::min(f->n_prompts - la.prompt0, VL_LAUNCH_PROMPTS);
      const dim3 grid((unsigned)la.layer_wgs), block(VL_BLOCK);
      if (rp.compact < 0) dsbd_launch(DSBD_KERNEL_VERIFY_LAYERS, verify_layers_kernel<true, NODE_CAP, true>, grid, block, (unsigned int)pl.lds_bytes, stream, la);
      else dsbd_launch(DSBD_KERNEL_VERIFY_LAYERS, verify_layers_kernel<true, NODE_CAP>, grid, block, (unsigned int)pl.lds_bytes, stream, la);
      le = hipGetLastError();
    }
  } else {
    const unsigned rows = (unsigned)f->n_nodes * (alias ? 1u : 2u);
    la.stats_threads = statistics_threads(f, pl, rows);
    const unsigned rows_per_wg = VL_BLOCK / la.stats_threads;
    for (int p0 = 0; p0 < f->n_prompts; p0 += pl.group) {
      la.prompt0 = p0;
      const int np = f->n_prompts - p0 < pl.group ? f->n_prompts - p0 : pl.group;
      unsigned grid3 = (unsigned)np * (unsigned)pl.G;
      la.layer_wgs = (int)grid3;
      if (want_stats && p0 + np == f->n_prompts) grid3 += (rows + rows_per_wg - 1) / rows_per_wg;     // behind the (last) layers
      if (pl.small_nodes)
        dsbd_launch(DSBD_KERNEL_VERIFY_LAYERS, verify_layers_kernel<false, NODE_CAP_SMALL>, dim3(grid3), dim3(VL_BLOCK),
                    (unsigned int)pl.lds_bytes, stream, la);
      else
        dsbd_launch(DSBD_KERNEL_VERIFY_LAYERS, verify_layers_kernel<false, NODE_CAP>, dim3(grid3), dim3(VL_BLOCK),
                    (unsigned int)pl.lds_bytes, stream, la);
    }
    le = hipGetLastError();
  }
  if (state && !capturing) {
    if (state->several_streams && hipEventRecord(state->layers_done, stream) != hipSuccess) le = hipErrorUnknown;
    state->last_stream = stream;
    state->have_last = true;
  }
  if (le != hipSuccess) return DSBD_ERR_HIP;
  if (next && keep_one) return dsbd_select_beams(f, out, p->W_cap, keep_one, next, fault, stream_);
  return DSBD_OK;
}
}  // namespace

extern "C" int32_t dsbd_verify_forest(const dsbd_forest* f, const dsbd_verify_in* in, const dsbd_params* p,
                                      const dsbd_verify_out* out, void* workspace, size_t workspace_bytes,
                                      int32_t* fault, void* stream_) {
  return verify_impl(f, in, p, out, workspace, workspace_bytes, fault, stream_, false);
}

extern "C" int32_t dsbd_verify_forest_select(const dsbd_forest* f, const dsbd_verify_in* in, const dsbd_params* p,
                                             const dsbd_verify_out* out, int32_t keep_one, const dsbd_next_beams* next,
                                             void* workspace, size_t workspace_bytes, int32_t* fault, void* stream_) {
  if (!next) return DSBD_ERR_INVALID;
  return verify_impl(f, in, p, out, workspace, workspace_bytes, fault, stream_, false, next, keep_one != 0);
}

// ---- the same call for callers that cannot allocate device memory (code under HIP graph capture, serving loops,
// harnesses that forbid hipMalloc): the workspace is a device array that is part of the library's image.
static __device__ __align__(256) unsigned char scratch[DSBD_STATIC_SCRATCH_BYTES];

namespace {
// Address of `scratch` on the current device (every GPU holds its own copy of the array at its own address; the
// array's name is only a host-side stand-in and must never reach a kernel or a memory call).
void* static_scratch_of_current_device() {
  static void* table[64] = {nullptr};
  static std::mutex mutex;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lock(mutex);
  if (!table[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    table[dev] = ptr;
  }
  return table[dev];
}
}  // namespace

extern "C" int32_t dsbd_init(void) {
  if (!static_scratch_of_current_device()) return DSBD_ERR_HIP;
  (void)device_limits();
  (void)dsbd_knobs();
  const LaunchOrder* const order = launch_order_of_current_device(true);
  return order && order->ok ? DSBD_OK : DSBD_ERR_HIP;
}

extern "C" size_t dsbd_verify_forest_static_capacity(void) { return DSBD_STATIC_SCRATCH_BYTES; }

extern "C" int32_t dsbd_verify_forest_static(const dsbd_forest* f, const dsbd_verify_in* in, const dsbd_params* p,
                                             const dsbd_verify_out* out, int32_t* fault, void* stream_) {
  if (!in) return DSBD_ERR_INVALID;
  const int32_t rc = check_verify(f, in->V, p);
  if (rc != DSBD_OK) return rc;
  // the same plan as the ordinary call; a problem whose workspace exceeds the array is turned away, nothing is enqueued
  if (dsbd_verify_forest_workspace_bytes(f, in->V, p) > (size_t)DSBD_STATIC_SCRATCH_BYTES) return DSBD_ERR_WORKSPACE;
  void* ptr = static_scratch_of_current_device();
  if (!ptr) return DSBD_ERR_HIP;
  return verify_impl(f, in, p, out, ptr, DSBD_STATIC_SCRATCH_BYTES, fault, stream_, true);
}
