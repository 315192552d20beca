// Forest attention for gfx950 (paper Section 3.3, "Forest-based Parallel Decoding").
//
// Every node of tree b attends to beam b's prefix cache plus the tree rows of its ancestors and
// itself.  All nodes of a tree (times the query heads of one KV group) share one pass over the
// beam's K/V stream, which is what makes the step bandwidth-bound instead of re-reading the cache
// once per node.
//
// Work decomposition (split-KV): one workgroup per (tree, KV head, row block, KV split).  Inside a
// workgroup the 4 waves form RW row groups x TW token groups.  Every wave streams its own 32-token
// steps of K and V from HBM through registers into tiles of its own in the LDS (no block-level barrier in the main
// loop) and keeps 16*NRT query rows resident:
//   S^T = K Q^T   MFMA 16x16x32 bf16, A = K (tokens x d) from the tile, B = Q^T held in registers for the whole kernel;
//   online softmax per query row, entirely lane-local: in the transposed product every lane owns
//                 one query row (column l%16), its scores and its slice of the output accumulators;
//   O^T += V^T P^T  MFMA 16x16x32, B = P^T built in registers from the S^T tile, A = V^T through the transposing LDS read.
// Bound by HBM: 16 prompts, 77 beams x 32 heads, 2.9 GB: 486 us = 6.05 TB/s (530 us while K came straight from memory in
// operand layout, which takes a cache line in two instructions and so cannot be streamed past the caches); 8 beams x 32
// heads x 2048 tokens, half of them shared: 36 us (40).
// The ancestor mask never exists in memory: every wave derives the tree's topology itself (the parent array of
// a tree is one load per lane, the parent chains are walked with lane shuffles), each lane keeps the 64-bit
// ancestor bitmap of its row's node and tests bits while handling the (at most two) steps that cover the
// tree's own rows.  The first workgroup of a tree also reports what the walk found wrong with the parent array.
// Partial (m, l, O) of the KV splits go to the workspace; a second kernel merges them.
#include "common.h"
#include "topology_device.h"
#include "wave_f64.h"
#include <stdlib.h>
#include <type_traits>

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

#define NEG_BIG (-1.0e30f)
#define REF_SLACK 40.0f          // log2 headroom of the softmax reference before it is raised
#define STEP 32                 // tokens per wave step (two 16-token MFMA tiles)
#define AT_BLOCK 256            // threads of every kernel here
#define AT_MAX_SPLIT 64

struct AttnArgs {
  const int32_t* tree_off;
  const int32_t* parent;
  int max_tree_nodes, max_depth;
  uint64_t* anc_out;            // [n_nodes] ancestor-or-self bitmaps, written once per tree if not null
  const void* const* k_ptr;
  const void* const* v_ptr;
  const int32_t* len;
  const void* const* k_shared_ptr;
  const void* const* v_shared_ptr;
  const int32_t* shared_len;
  long long token_stride, head_stride;
  const __bf16* q;
  const __bf16* k_tree;
  const __bf16* v_tree;
  int n_trees, n_nodes, Hq, Hkv, group;
  float scale_log2;             // scale * log2(e): scores are kept in the log2 domain
  int max_len;
  int by_tree;                  // splits chosen tree by tree on the device (else `nsplit` for every unit)
  int nsplit, n_rowblocks;      // row blocks: of the largest tree the caller announces
  int rows_block;               // query rows per workgroup
  int wg_slots;                 // by_tree: workgroups to spread the work over
  int waves;                    // waves per workgroup of the wave-private kernel
  // Partial results, one of two layouts (the plan takes the smaller): by split, the row of split s behind those of all
  // rows of the splits before it; or a slot of part_pitch rows per workgroup, a unit's splits in consecutive slots.
  int by_split;
  int part_pitch;
  long long part_stride;        // rows between a row's partial results of consecutive splits
  long long part_rows;          // rows there is room for
  float* part_o;                // [part_rows][D]
  float* part_ml;               // [part_rows][2]
  int2* row_parts;              // [n_nodes*Hq] a row's first partial result (slots), and how many there are (null: no splits)
  __bf16* out;                  // written by the main kernel where a unit is not split, else by the merge kernel
  float* lse;
  int32_t* fault;
};

// 16-byte load through the GLOBAL address space.  The cache pointers come out of a pointer table in
// memory, so the compiler only knows them as generic pointers and would emit FLAT loads, which count on
// the LDS counter as well: every wait for an LDS read would then also wait for all K/V loads in flight.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_global_16(const void* p) {
  const u32x4 v = *(const __attribute__((address_space(1))) u32x4*)(p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
// The same with the non-temporal hint, for streams whose cache lines are consumed whole by one load instruction of a
// wave (where several instructions share a line the hint costs 20 % instead of gaining 9 to 14 %).
__device__ __forceinline__ uint4 load_global_16_nt(const void* p) {
  const u32x4 v = __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4*)(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ bf16x8 load_global_bf16x8(const void* p) {
  union { uint4 u; bf16x8 v; } c;
  c.u = load_global_16(p);
  return c.v;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() carries a workgroup-scope fence, for
// which the compiler waits for ALL outstanding memory operations (vmcnt(0)) - including the K/V loads of
// the next tile that were issued on purpose before the barrier, which would then never overlap with the
// arithmetic.  Here only the LDS counter is drained; global loads stay in flight across the barrier.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---- which part of the work a workgroup has
//
// A unit is (tree, KV head, row block); a tree of more steps than an even share of the whole work has its units split
// along the keys.  Lengths and node counts sit in device memory, so every workgroup works its place out for itself: a
// lane (up to 64 trees) or a thread (up to 256) per tree, its steps, its share of the total, the splits of its units; the
// trees' workgroups are handed out in order of falling length, so that what runs last is short.  With a lane per tree
// everything the workgroup needs to know of its tree arrives with the same round trip to memory, and no barrier is
// needed (the sums go by lane moves: twelve shuffles through the LDS cost 0.4 us in front of the first loads).  With more trees than threads, or a pinned number of splits, every unit gets `nsplit` splits and the place is
// plain arithmetic.
// (One number of splits for all units, from the bounds the host knows, gave a sampled forest - one tree of 48 nodes, four
// of one or two - a single split per unit: 92 us where 26 are enough; 24 trees of 700 to 3000 tokens: 35 us, now 25.)
struct WorkShare {
  int steps[AT_BLOCK], count[AT_BLOCK];
  float wsum[4], usum[4];
  int b, rel, nsplit, nrb;
};
struct Place {
  int b, g, rb, split, nsplit;
  int base, end;                            // the tree's nodes (unchecked)
  int Ls, Lo;                               // tokens of the shared and the own segment (unchecked)
  const __bf16 *k0, *v0, *k1, *v1;          // shared and own segment (null where not given)
};

__device__ __forceinline__ const __bf16* lane_pointer(const void* p, int l) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned int lo = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)v, l);
  const unsigned int hi = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)(v >> 32), l);
  return reinterpret_cast<const __bf16*>(((unsigned long long)hi << 32) | lo);
}

// Most splits worth their partial results for a unit of so many steps.  Wave-private kernel (32-token steps, a wave each): four
// steps per split (whole call, us at 1 / 2 / 3 / 4 / 6 / 8 splits: 8 units of 17 steps 17.4 / 15.2 / 15.5 / 13.7 / 13.2 / 13.3; 32
// units of 23 steps 15.3 / 14.3 / 13.2 / 13.1 / 11.7 / 11.7).  Tile kernel: four 64-token tiles, and as little as two tiles for
// up to four splits (at 2 / 4 / 6 / 8 / 16 splits: 32 units of 33 tiles 30.4 / 22.2 / 20.9 / 21.1 / 26.3; of 9 tiles 17.4 / 15.5 /
// 16.8 / 16.5).
__host__ __device__ __forceinline__ int split_limit(int steps, bool tiles, int waves) {
  const int four = steps / 4, two = steps / 2;
  const int most = !tiles ? (waves == 8 ? (steps + 7) / 8 : four) : (four >= 4 ? four : (two < 4 ? two : 4));
  return most < 1 ? 1 : (most > AT_MAX_SPLIT ? AT_MAX_SPLIT : most);
}

// Splits of a tree's units: one, and its share of the workgroups that are left when every unit has one.  The shares are
// rounded down, so that all workgroups together are no more than the slots (or the units, if those are more), which is
// the grid (slots and units side by side before: a ninth more workgroups and workspace, equal times).
// (What is whole in exact arithmetic must not fall below: the slack adds less than half a workgroup over all units.)
__device__ __forceinline__ int splits_of(const AttnArgs& a, int steps, float total, float units, bool tiles) {
  const float left = fmaxf((float)a.wg_slots - units, 0.f);
  const int ns = 1 + (int)((float)steps * left / total + 1e-3f);
  return max(1, min(min(ns, split_limit(steps, tiles, a.waves)), a.nsplit));
}

// False: nothing to do for this workgroup.
template <int UNIT>
__device__ __forceinline__ bool work_place(const AttnArgs& a, WorkShare& w, Place& pl) {
  const int bid = blockIdx.x, tid = threadIdx.x;
  // a tree's steps and row blocks (0 if its offsets are unusable: then no workgroup gets it)
  auto measure = [&](int base, int end, int Ls, int Lo, int& steps, int& nrb) {
    steps = 0; nrb = 0;
    if (base >= 0 && end <= a.n_nodes && end > base) {
      Lo = max(Lo, 0); Ls = max(Ls, 0);
      Ls = min(Ls, a.max_len); Lo = min(Lo, a.max_len - Ls);
      const int n = min(end - base, DSBD_MAX_TREE_NODES);
      steps = (Ls + UNIT - 1) / UNIT + (Lo + UNIT - 1) / UNIT + (n + UNIT - 1) / UNIT;
      nrb = min((n * a.group + a.rows_block - 1) / a.rows_block, a.n_rowblocks);
    }
  };
  const bool shares = a.shared_len != nullptr && a.k_shared_ptr != nullptr;
  int rel, nrb_b;
  if (a.by_tree && a.n_trees <= 64) {
    const int lane = tid & 63, t = min(lane, a.n_trees - 1);
    const int base = a.tree_off[t], end = a.tree_off[t + 1], Lo = a.len[t], Ls = shares ? a.shared_len[t] : 0;
    const void *k1 = a.k_ptr[t], *v1 = a.v_ptr[t];
    const void *k0 = shares ? a.k_shared_ptr[t] : nullptr, *v0 = shares ? a.v_shared_ptr[t] : nullptr;
    int steps, nrb;
    measure(base, end, Ls, Lo, steps, nrb);
    if (lane >= a.n_trees) { steps = 0; nrb = 0; }
    else if (bid == 0 && tid < 64 && nrb == 0) atomicOr(a.fault, DSBD_FAULT_TOPOLOGY);
    float units = (float)(nrb * a.Hkv), total = units * (float)steps;
    total = wave_sum_f32(total); units = wave_sum_f32(units);
    const int ns = splits_of(a, steps, total, units, UNIT == 64), count = a.Hkv * nrb * ns;
    int first = 0;
    for (int o = 0; o < a.n_trees; ++o) {
      const int so = __builtin_amdgcn_readlane(steps, o), co = __builtin_amdgcn_readlane(count, o);
      first += (so > steps || (so == steps && o < lane)) ? co : 0;
    }
    const unsigned long long m = __ballot(bid >= first && bid < first + count);
    if (m == 0ull) return false;
    const int l = (int)__ffsll((long long)m) - 1;
    pl.b = l;
    rel = bid - __builtin_amdgcn_readlane(first, l);
    pl.nsplit = __builtin_amdgcn_readlane(ns, l);
    nrb_b = __builtin_amdgcn_readlane(nrb, l);
    pl.base = __builtin_amdgcn_readlane(base, l); pl.end = __builtin_amdgcn_readlane(end, l);
    pl.Ls = __builtin_amdgcn_readlane(Ls, l); pl.Lo = __builtin_amdgcn_readlane(Lo, l);
    pl.k0 = lane_pointer(k0, l); pl.v0 = lane_pointer(v0, l);
    pl.k1 = lane_pointer(k1, l); pl.v1 = lane_pointer(v1, l);
  } else {
    if (a.by_tree) {
      int steps = 0, nrb = 0;
      if (tid < a.n_trees) {
        measure(a.tree_off[tid], a.tree_off[tid + 1], shares ? a.shared_len[tid] : 0, a.len[tid], steps, nrb);
        if (bid == 0 && nrb == 0) atomicOr(a.fault, DSBD_FAULT_TOPOLOGY);
      }
      float units = (float)(nrb * a.Hkv), total = units * (float)steps;
      total = wave_sum_f32(total); units = wave_sum_f32(units);
      if ((tid & 63) == 0) { w.wsum[tid >> 6] = total; w.usum[tid >> 6] = units; }
      if (tid == 0) w.b = -1;
      __syncthreads();
      const int ns = splits_of(a, steps, (w.wsum[0] + w.wsum[1]) + (w.wsum[2] + w.wsum[3]),
                               (w.usum[0] + w.usum[1]) + (w.usum[2] + w.usum[3]), UNIT == 64), count = a.Hkv * nrb * ns;
      w.steps[tid] = steps;
      w.count[tid] = count;
      __syncthreads();
      int first = 0;
#pragma unroll 4
      for (int o = 0; o < a.n_trees; ++o) {
        const int so = w.steps[o], co = w.count[o];
        first += (so > steps || (so == steps && o < tid)) ? co : 0;
      }
      if (bid >= first && bid < first + count) { w.b = tid; w.rel = bid - first; w.nsplit = ns; w.nrb = nrb; }
      __syncthreads();
      pl.b = __builtin_amdgcn_readfirstlane(w.b); rel = __builtin_amdgcn_readfirstlane(w.rel);
      pl.nsplit = __builtin_amdgcn_readfirstlane(w.nsplit); nrb_b = __builtin_amdgcn_readfirstlane(w.nrb);
      if (pl.b < 0) return false;
    } else {
      const int per = a.Hkv * a.n_rowblocks * a.nsplit;
      pl.b = bid / per; rel = bid % per; pl.nsplit = a.nsplit; nrb_b = a.n_rowblocks;
      if (pl.b >= a.n_trees) return false;
    }
    const int b = pl.b;
    pl.base = a.tree_off[b]; pl.end = a.tree_off[b + 1];
    pl.Lo = a.len[b]; pl.Ls = shares ? a.shared_len[b] : 0;
    pl.k1 = (const __bf16*)a.k_ptr[b]; pl.v1 = (const __bf16*)a.v_ptr[b];
    pl.k0 = shares ? (const __bf16*)a.k_shared_ptr[b] : nullptr;
    pl.v0 = shares ? (const __bf16*)a.v_shared_ptr[b] : nullptr;
  }
  pl.split = rel % pl.nsplit;
  pl.rb = (rel / pl.nsplit) % nrb_b;
  pl.g = rel / (pl.nsplit * nrb_b);
  return true;
}

// Where this workgroup's rows leave their results: `rows` of them (all, but for trees with more nodes than announced or that
// share nodes with others: slots hold no more), row rl at `at` + rl (slots) or + its number among all rows (by split).
struct PartPlace { long long at; int rows; };
__device__ __forceinline__ PartPlace part_place(const AttnArgs& a, int split, int nsplit, int rows) {
  PartPlace p = {split * a.part_stride, rows};
  if (!a.by_split) {
    p.at = (long long)blockIdx.x * a.part_pitch;
    if (nsplit > 1) p.rows = p.at + a.part_pitch <= a.part_rows ? min(rows, a.part_pitch) : 0;
  }
  return p;
}

// Four channels of a finished row: out = acc / L, and once per row the log-sum-exp.
template <int D>
__device__ __forceinline__ void write_row_part(const AttnArgs& a, long long row, int part, float M, float L, floatx4 acc) {
  const float inv = L > 0.f ? 1.f / L : 0.f;
  union { __bf16 h[4]; uint2 u; } pk;
#pragma unroll
  for (int i = 0; i < 4; ++i) pk.h[i] = (__bf16)(acc[i] * inv);
  *reinterpret_cast<uint2*>(&a.out[row * D + 4 * part]) = pk.u;
  if (a.lse && part == 0) a.lse[row] = (M + log2f(L)) * 0.6931471805599453f;
}

// TW: waves, each with steps of its own.
template <int D, int NRT, int TW>
__global__ __launch_bounds__(64 * TW) void forest_attention_kernel(AttnArgs a) {
  constexpr int DS = D / 32;        // MFMA k-steps over the head dimension for S^T
  constexpr int DT = D / 16;        // 16-row output tiles over the head dimension for O^T
  constexpr int ROWS_B = 16 * NRT;  // query rows
  constexpr int LPR = D / 8;        // lanes covering one K or V row with 16-byte loads
  constexpr int TG = 64 / LPR;      // rows per load instruction of a wave
  constexpr int ROUNDS = STEP / TG;

  constexpr int KP = D + 8;         // pitch of a tile row in elements (16 bytes of padding)
  constexpr int OP = D + 4;         // pitch of an output row in the merge of the waves (floats)
  static_assert(ROWS_B * OP * 4 <= 2 * STEP * KP * 2, "a wave's partial output takes the place of its tiles");
  __shared__ __attribute__((aligned(16))) __bf16 tiles[TW][2 * STEP * KP];     // every wave's K and V tile
  __shared__ float wave_ml[TW][ROWS_B][2];
  __shared__ WorkShare share;

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int col = lane & 15;        // query row within a 16-row tile / token within a 16-token tile
  const int qd = lane >> 4;         // lane group 0..3

  Place pl;
  if (!work_place<STEP>(a, share, pl)) return;
  const int nsplit = pl.nsplit, split = pl.split, rb = pl.rb, g = pl.g;

  const dsbd_tree_range tr = dsbd_tree_range_between(pl.base, pl.end, a.n_nodes, a.max_tree_nodes);
  const bool reporter = split == 0 && rb == 0 && g == 0 && wave == 0;   // one wave per tree speaks for it
  if (!tr.valid) {
    if (reporter && lane == 0) atomicOr(a.fault, tr.bad);
    return;
  }
  const int base = tr.base;
  const int n_b = min(tr.n_all, DSBD_MAX_TREE_NODES);
  const int p_mine = dsbd_tree_parent_of(tr, lane, a.parent);   // used once the first loads are on their way
  const int R = n_b * a.group;       // query rows of this (tree, KV head)
  const int row0 = rb * ROWS_B;
  if (row0 >= R) return;             // a row block beyond the tree's rows (uniform over the workgroup)

  // ---- segments of the key sequence: shared prefix, own prefix, the tree's own rows
  int Ls = max(pl.Ls, 0), Lo = max(pl.Lo, 0);
  int bad = 0;
  if ((long long)Ls + Lo > a.max_len) { bad |= DSBD_FAULT_BOUNDS; Ls = min(Ls, a.max_len); Lo = min(Lo, a.max_len - Ls); }
  const long long hoff = (long long)g * a.head_stride;
  const __bf16 *k0 = pl.k0, *v0 = pl.v0, *k1 = pl.k1, *v1 = pl.v1;
  if (Ls && (!k0 || !v0 || (((uintptr_t)k0 | (uintptr_t)v0) & 15))) { bad |= DSBD_FAULT_BOUNDS; Ls = 0; }
  if (Lo && (!k1 || !v1 || (((uintptr_t)k1 | (uintptr_t)v1) & 15))) { bad |= DSBD_FAULT_BOUNDS; Lo = 0; }
  if (bad && threadIdx.x == 0) atomicOr(a.fault, bad);   // missing or misaligned cache pointer: segment skipped
  k0 += hoff; v0 += hoff; k1 += hoff; v1 += hoff;
  const __bf16* k2 = a.k_tree + ((long long)base * a.Hkv + g) * D;
  const __bf16* v2 = a.v_tree + ((long long)base * a.Hkv + g) * D;
  const long long stride2 = (long long)a.Hkv * D;
  const int n0 = (Ls + STEP - 1) / STEP;
  const int n1 = (Lo + STEP - 1) / STEP;
  const int n2 = (n_b + STEP - 1) / STEP;
  const int total_steps = n0 + n1 + n2;
  // balanced partition: the first (total % nsplit) splits take one step more than the others
  const int st_begin = split * (total_steps / nsplit) + min(split, total_steps % nsplit);
  const int st_end = st_begin + total_steps / nsplit + (split < total_steps % nsplit ? 1 : 0);

  // ---- resident query fragments (B operand: lane holds row `col`, 8 channels 32j + 8qd ..)
  bf16x8 qf[NRT][DS];
  uint64_t anc[NRT];
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    const int r = row0 + rt * 16 + col;
    const bool live = r < R;
    const int node = live ? r / a.group : 0;
    const int head = g * a.group + (live ? r % a.group : 0);
    anc[rt] = 0ull;
    const __bf16* qp = a.q + ((long long)(base + node) * a.Hq + head) * D + 8 * qd;
#pragma unroll
    for (int j = 0; j < DS; ++j) {
      if (live) {
        qf[rt][j] = load_global_bf16x8(qp + 32 * j);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[rt][j][e] = (__bf16)0.0f;
      }
    }
  }

  floatx4 o[NRT][DT];
  float m_run[NRT], l_run[NRT];
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    m_run[rt] = NEG_BIG;
    l_run[rt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[rt][dt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  __bf16* const kt = tiles[wave];
  __bf16* const vt = kt + STEP * KP;
  const int ld_piece = lane % LPR;   // 16-byte piece of the row this lane loads
  const int ld_tok = lane / LPR;     // row among those of a load instruction

  uint4 kr[ROUNDS], vr[ROUNDS];     // the next step's rows on their way from HBM to the tiles

  // step -> (segment, first token, tokens in the segment)
  auto locate = [&](int st, const __bf16*& kp, const __bf16*& vp, long long& stride, int& tok0, int& len, bool& tree) {
    if (st < n0) { kp = k0; vp = v0; stride = a.token_stride; tok0 = st * STEP; len = Ls; tree = false; }
    else if (st < n0 + n1) { kp = k1; vp = v1; stride = a.token_stride; tok0 = (st - n0) * STEP; len = Lo; tree = false; }
    else { kp = k2; vp = v2; stride = stride2; tok0 = (st - n0 - n1) * STEP; len = n_b; tree = true; }
  };
  // Whole rows per instruction, streamed past the caches: a line consumed by one instruction may carry the non-temporal
  // hint, which the stream needs (a pure-load replay of the 16-prompt batch: 6.8 TB/s with it, 5.95 without; K loaded
  // straight in operand layout takes a line in two instructions and was 20 % slower with the hint).
  auto load_step = [&](int st) {
    const __bf16 *kp, *vp; long long stride; int tok0, len; bool tree;
    locate(st, kp, vp, stride, tok0, len, tree);
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
      const long long off = (long long)min(tok0 + TG * k + ld_tok, len - 1) * stride + 8 * ld_piece;
      kr[k] = load_global_16_nt(kp + off);
      vr[k] = load_global_16_nt(vp + off);
    }
  };

  int st = st_begin + wave;
  const bool active = st < st_end;
  if (active) load_step(st);
  // ---- topology of the tree (every wave for itself, while the first K/V loads travel): lane j = node j
  {
    uint64_t my_anc = 0;
    const int tb = dsbd_tree_walk(tr, lane, p_mine, a.max_depth, nullptr, reporter ? a.anc_out : nullptr, &my_anc);
    if (reporter && tb) atomicOr(a.fault, tb);
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) {
      const int r = row0 + rt * 16 + col;
      const int node = r < R ? r / a.group : 0;
      const unsigned lo = __shfl((unsigned)my_anc, node), hi = __shfl((unsigned)(my_anc >> 32), node);
      anc[rt] = r < R ? ((uint64_t)hi << 32) | lo : 0ull;
    }
  }

  // One step = 32 tokens of this wave: its rows move from the registers to the wave's tiles, the next step's are
  // requested, S^T = K Q^T.
  int tok0 = 0, nvalid = 0, st_next = 0;
  bool is_tree = false;
  floatx4 s[NRT][2];
  auto step_front = [&]() {
    const __bf16 *kp_, *vp_; long long stride_; int seglen;
    locate(st, kp_, vp_, stride_, tok0, seglen, is_tree);
    nvalid = min(STEP, seglen - tok0);
    st_next = st + TW;
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
      *reinterpret_cast<uint4*>(&kt[(TG * k + ld_tok) * KP + 8 * ld_piece]) = kr[k];
      *reinterpret_cast<uint4*>(&vt[(TG * k + ld_tok) * KP + 8 * ld_piece]) = vr[k];
    }
    wave_lds_fence();
    if (st_next < st_end) load_step(st_next);
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      bf16x8 kf[DS];
#pragma unroll
      for (int j = 0; j < DS; ++j) kf[j] = *reinterpret_cast<const bf16x8*>(&kt[(16 * tt + col) * KP + 32 * j + 8 * qd]);
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < DS; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[j], qf[rt][j], acc, 0, 0, 0);
        s[rt][tt] = acc;
      }
    }
  };
  // O^T += V^T P^T (V^T through the transposing LDS read, see the shared-tile kernel)
  auto step_pv = [&](const bf16x8 (&pf)[NRT]) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      union { v4i16 h[2]; bf16x8 v; } vf;
      const __bf16* rowp = &vt[(4 * qd + (col >> 2)) * KP + 16 * dt + 4 * (col & 3)];
      vf.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(rowp));
      vf.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(rowp + 16 * KP));
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) o[rt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf.v, pf[rt], o[rt][dt], 0, 0, 0);
    }
  };

  // Softmax numerators are taken against a per-row reference m_run that is NOT the exact running
  // maximum: it is set by the first step with a valid score for the row and raised only when a score
  // exceeds it by more than 2^REF_SLACK.  fp32 (and bf16, for P) have the exponent range for numerators
  // up to 2^REF_SLACK, and the final division by the row sum removes the reference.  So the hot loop
  // below is "exp2(s - m_run), accumulate": no rescaling of the output accumulators (which live in
  // accumulation registers that vector ALU instructions cannot touch), no cross-lane traffic.  Steps
  // that need a mask (tree rows, ragged tail) or a higher reference leave the hot loop and take the
  // general path once.
  while (active && st < st_end) {
    bool general = false;
    while (st < st_end) {                      // ---- hot loop
      step_front();
      if (is_tree || nvalid < STEP) { general = true; break; }
      bool raise = false;
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        float mx = fmaxf(fmaxf(s[rt][0][0], s[rt][0][1]), fmaxf(s[rt][0][2], s[rt][0][3]));
        mx = fmaxf(mx, fmaxf(fmaxf(s[rt][1][0], s[rt][1][1]), fmaxf(s[rt][1][2], s[rt][1][3])));
        raise = raise || (mx * a.scale_log2 > m_run[rt] + REF_SLACK);
      }
      if (__builtin_amdgcn_ballot_w64(raise) != 0ull) { general = true; break; }
      bf16x8 pf[NRT];
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        const float nm = -m_run[rt];
        float psum = 0.f;
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float p = __builtin_amdgcn_exp2f(fmaf(s[rt][tt][i], a.scale_log2, nm));
            psum += p;
            pf[rt][4 * tt + i] = (__bf16)p;
          }
        l_run[rt] += psum;
      }
      step_pv(pf);
      st = st_next;
    }
    if (!general) break;

    // ---- general step: masks, reference raise with rescaling
    const bool need_mask = is_tree || nvalid < STEP;
    bf16x8 pf[NRT];
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) {
      float sv[8];
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) sv[4 * tt + i] = s[rt][tt][i] * a.scale_log2;
      unsigned okbits = 0xffu;
      if (need_mask) {
        okbits = 0;
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int t = 16 * tt + 4 * qd + i;          // token within the step
            bool valid = t < nvalid;
            if (is_tree) valid = valid && ((anc[rt] >> (tok0 + t)) & 1ull);
            if (valid) okbits |= 1u << (4 * tt + i); else sv[4 * tt + i] = NEG_BIG;
          }
      }
      float mx = fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])), fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));                  // same value in the 4 lane groups of a row
      const float m_new = (mx > m_run[rt] + REF_SLACK) ? mx : m_run[rt];
      const float alpha = __builtin_amdgcn_exp2f(m_run[rt] - m_new);
      l_run[rt] *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[rt][dt] *= alpha;
      m_run[rt] = m_new;
      float psum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float p = ((okbits >> e) & 1u) ? __builtin_amdgcn_exp2f(sv[e] - m_new) : 0.f;
        psum += p;
        pf[rt][e] = (__bf16)p;
      }
      l_run[rt] += psum;
    }
    step_pv(pf);
    st = st_next;
  }

  // ---- finish the row sums (each lane group summed its own tokens)
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    l_run[rt] += __shfl_xor(l_run[rt], 16);
    l_run[rt] += __shfl_xor(l_run[rt], 32);
  }

  // ---- the waves' partial results merged through the LDS (each wave's in the place of its own tiles), a thread per
  // (row, four channels), rows written whole
  wave_lds_fence();
  float* const mine = reinterpret_cast<float*>(tiles[wave]);
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    const int rl = rt * 16 + col;
    if (qd == 0) { wave_ml[wave][rl][0] = m_run[rt]; wave_ml[wave][rl][1] = l_run[rt]; }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<floatx4*>(&mine[rl * OP + 16 * dt + 4 * qd]) = o[rt][dt];
  }
  __syncthreads();
  constexpr int QPR = D / 4;
  const PartPlace place = part_place(a, split, nsplit, min(R - row0, ROWS_B));
#pragma unroll
  for (int c = threadIdx.x; c < ROWS_B * QPR; c += 64 * TW) {
    const int rl = c / QPR, part = c % QPR, r = row0 + rl;
    if (rl >= place.rows) break;       // (rows rise with c)
    float m[TW], M = NEG_BIG, L = 0.f;
#pragma unroll
    for (int w = 0; w < TW; ++w) { m[w] = wave_ml[w][rl][0]; M = fmaxf(M, m[w]); }
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < TW; ++w) {
      const float e = __builtin_amdgcn_exp2f(m[w] - M);
      L += e * wave_ml[w][rl][1];
      acc += e * *reinterpret_cast<const floatx4*>(&reinterpret_cast<const float*>(tiles[w])[rl * OP + 4 * part]);
    }
    const int row = (base + r / a.group) * a.Hq + g * a.group + r % a.group;
    const long long prow = place.at + (a.by_split ? row : rl);
    if (part == 0 && split == 0 && a.row_parts) a.row_parts[row] = make_int2((int)prow, nsplit);
    if (nsplit == 1) {
      write_row_part<D>(a, row, part, M, L, acc);
    } else {
      if (part == 0) *reinterpret_cast<float2*>(&a.part_ml[prow * 2]) = make_float2(M, L);
      *reinterpret_cast<floatx4*>(&a.part_o[prow * D + 4 * part]) = acc;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Many query rows per K/V stream (large trees and/or grouped-query attention): the waves of a workgroup keep 32 query
// rows each (two 16-row tiles) and share a 64-token K/V tile that goes straight from memory into the LDS
// (global_load_lds_dwordx4: a wave's 64 lanes fill 1 KiB of consecutive LDS, no staging registers, no LDS stores).  K is
// read back as MFMA A operand with 16-byte reads, V through the transposing LDS read of gfx950 (ds_read_b64_tr_b16),
// which hands a lane four tokens of one channel.  Rows cannot be padded in LDS-bound loads, so bank conflicts are avoided
// by a swizzle: the 16-byte piece p of token t sits at position p ^ f(t) of the token's row, f(t) = 2 (t & 3) + ((t >> 2)
// & 1), which spreads both the K operand reads (16 consecutive tokens, one piece) and the transposing V reads (4
// consecutive tokens, two pieces) over all banks.  The two tile buffers are four separate LDS arrays and the loop is
// written out for both, so that the compiler can tell a read of one buffer from the load in flight into the other (it
// waits for every outstanding LDS-bound load before an LDS read that may alias it).
//
// A block has up to 128 rows, a wave for each 32 of them.  Blocks of at most 64 rows (small trees, the last block of a
// large one) would leave two or three waves without a row: there the waves take the two 32-token halves of a tile, two
// waves per half, and the halves are merged at the end.
#ifndef DSBD_DMA_AUX
#define DSBD_DMA_AUX 2        // cache policy of the tile loads: non-temporal
#endif
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void glb_cvoid_t;
template <int D, int WPE>
__global__ __launch_bounds__(AT_BLOCK) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
void forest_attention_dma_kernel(AttnArgs a) {
  constexpr int TILE = 64, NRT = 2;
  constexpr int DS = D / 32, DT = D / 16;
  constexpr int PPR = D / 8;                // 16-byte pieces of a row
  constexpr int ROWB = D * 2;               // bytes of a row
  constexpr int SLOTS = TILE * PPR;         // 16-byte slots of a K or V tile
  constexpr int TPI = 64 / PPR;             // tokens per load instruction of a wave
  constexpr int ROUNDS = TILE / (4 * TPI);
  constexpr int ROWS_W = 16 * NRT, ROWS_B = ROWS_W * 4;
  __shared__ __attribute__((aligned(16))) uint4 kA[SLOTS];
  __shared__ __attribute__((aligned(16))) uint4 kB[SLOTS];
  __shared__ __attribute__((aligned(16))) uint4 vA[SLOTS];
  __shared__ __attribute__((aligned(16))) uint4 vB[SLOTS];
  __shared__ float half_ml[2 * ROWS_W][2];
  __shared__ float row_ml[ROWS_B][2];
  __shared__ int row_id[ROWS_B];            // node * Hq + head
  __shared__ WorkShare share;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, qd = lane >> 4;

  Place pl;
  if (!work_place<TILE>(a, share, pl)) return;
  const int nsplit = pl.nsplit, split = pl.split, rb = pl.rb, g = pl.g;

  const dsbd_tree_range tr = dsbd_tree_range_between(pl.base, pl.end, a.n_nodes, a.max_tree_nodes);
  const bool reporter = split == 0 && rb == 0 && g == 0 && wave == 0;   // one wave per tree speaks for it
  if (!tr.valid) {
    if (reporter && lane == 0) atomicOr(a.fault, tr.bad);
    return;
  }
  const int base = tr.base;
  const int n_b = min(tr.n_all, DSBD_MAX_TREE_NODES);
  const int p_mine = dsbd_tree_parent_of(tr, lane, a.parent);   // used once the first loads are on their way
  const int R = n_b * a.group;
  if (rb * ROWS_B >= R) return;             // uniform over the workgroup
  // the waves: row groups of 32 rows, and token halves where there are at most two row groups
  const int rows_here = min(R - rb * ROWS_B, ROWS_B);
  const bool halves = rows_here <= 2 * ROWS_W;
  const int rgrp = halves ? wave & 1 : wave, half = halves ? wave >> 1 : 0;
  const bool computes = rgrp * ROWS_W < rows_here;              // (uniform over the wave)
  const int row0 = rb * ROWS_B + rgrp * ROWS_W;

  int Ls = max(pl.Ls, 0), Lo = max(pl.Lo, 0);
  int bad = 0;
  if ((long long)Ls + Lo > a.max_len) { bad |= DSBD_FAULT_BOUNDS; Ls = min(Ls, a.max_len); Lo = min(Lo, a.max_len - Ls); }
  const long long hoff = (long long)g * a.head_stride;
  const __bf16 *k0 = pl.k0, *v0 = pl.v0, *k1 = pl.k1, *v1 = pl.v1;
  if (Ls && (!k0 || !v0 || (((uintptr_t)k0 | (uintptr_t)v0) & 15))) { bad |= DSBD_FAULT_BOUNDS; Ls = 0; }
  if (Lo && (!k1 || !v1 || (((uintptr_t)k1 | (uintptr_t)v1) & 15))) { bad |= DSBD_FAULT_BOUNDS; Lo = 0; }
  if (bad && tid == 0) atomicOr(a.fault, bad);
  k0 += hoff; v0 += hoff; k1 += hoff; v1 += hoff;
  const __bf16* k2 = a.k_tree + ((long long)base * a.Hkv + g) * D;
  const __bf16* v2 = a.v_tree + ((long long)base * a.Hkv + g) * D;
  const long long stride2 = (long long)a.Hkv * D;
  const int n0 = (Ls + TILE - 1) / TILE, n1 = (Lo + TILE - 1) / TILE, n2 = (n_b + TILE - 1) / TILE;
  const int total_tiles = n0 + n1 + n2;
  // balanced partition: the first (total % nsplit) splits take one tile more than the others
  const int t_begin = split * (total_tiles / nsplit) + min(split, total_tiles % nsplit);
  const int t_end = t_begin + total_tiles / nsplit + (split < total_tiles % nsplit ? 1 : 0);

  bf16x8 qf[NRT][DS];
  uint64_t anc[NRT];
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    const int r = row0 + rt * 16 + col;
    const bool live = r < R;
    const int node = live ? r / a.group : 0;
    const int head = g * a.group + (live ? r % a.group : 0);
    anc[rt] = 0ull;
    const __bf16* qp = a.q + ((long long)(base + node) * a.Hq + head) * D + 8 * qd;
#pragma unroll
    for (int j = 0; j < DS; ++j) {
      if (live) {
        qf[rt][j] = load_global_bf16x8(qp + 32 * j);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[rt][j][e] = (__bf16)0.0f;
      }
    }
  }
  floatx4 o[NRT][DT];
  float m_run[NRT], l_run[NRT];
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    m_run[rt] = NEG_BIG; l_run[rt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[rt][dt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  auto locate = [&](int ti, const __bf16*& kp, const __bf16*& vp, long long& stride, int& tok0, int& len, bool& tree) {
    if (ti < n0) { kp = k0; vp = v0; stride = a.token_stride; tok0 = ti * TILE; len = Ls; tree = false; }
    else if (ti < n0 + n1) { kp = k1; vp = v1; stride = a.token_stride; tok0 = (ti - n0) * TILE; len = Lo; tree = false; }
    else { kp = k2; vp = v2; stride = stride2; tok0 = (ti - n0 - n1) * TILE; len = n_b; tree = true; }
  };
  auto swz = [](int t) { return ((t & 3) << 1) | ((t >> 2) & 1); };
  // tile ti -> the LDS arrays Kb / Vb: instruction r of wave w fills slots (4r + w) * 64 .. + 63, i.e. lane L fills
  // position L % PPR of token TPI (4r + w) + L / PPR and therefore fetches piece (L % PPR) ^ f(token)
  const int ld_tok = TPI * wave + lane / PPR;            // (the token of round 0; a round is 4 TPI tokens, a multiple of 8)
  const int ld_piece = (lane % PPR) ^ swz(ld_tok);
  // A whole tile (no ragged end) needs no per-lane arithmetic at all: the lane's byte offset inside the tile's
  // first round of tokens is a constant of the segment, the tile and the round are uniform.
  // (That offset is a 32-bit number: caches with 64 million elements or more from token to token take the general form.)
  const bool near = a.token_stride >= 0 && a.token_stride < (1LL << 26);
  auto issue = [&](int ti, auto& Kb, auto& Vb) {
    const __bf16 *kp, *vp; long long stride; int tok0, len; bool tree;
    locate(ti, kp, vp, stride, tok0, len, tree);
    if (near && tok0 + TILE <= len) {
      const char* const kb = reinterpret_cast<const char*>(kp + (long long)tok0 * stride);
      const char* const vb = reinterpret_cast<const char*>(vp + (long long)tok0 * stride);
      const unsigned int lo = (unsigned int)ld_tok * (unsigned int)(stride * 2) + (unsigned int)(ld_piece * 16);
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        const long long step = (long long)r * (4 * TPI) * stride * 2;
        __builtin_amdgcn_global_load_lds((glb_cvoid_t*)(kb + step + lo), (lds_void_t*)&Kb[(4 * r + wave) * 64], 16, 0, DSBD_DMA_AUX);
        __builtin_amdgcn_global_load_lds((glb_cvoid_t*)(vb + step + lo), (lds_void_t*)&Vb[(4 * r + wave) * 64], 16, 0, DSBD_DMA_AUX);
      }
      return;
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int tok = min(tok0 + 4 * TPI * r + ld_tok, len - 1);
      const long long off = (long long)tok * stride + ld_piece * 8;
      __builtin_amdgcn_global_load_lds((glb_cvoid_t*)(kp + off), (lds_void_t*)&Kb[(4 * r + wave) * 64], 16, 0, DSBD_DMA_AUX);
      __builtin_amdgcn_global_load_lds((glb_cvoid_t*)(vp + off), (lds_void_t*)&Vb[(4 * r + wave) * 64], 16, 0, DSBD_DMA_AUX);
    }
  };
  // byte offsets of this lane's operand reads inside a tile, without the token-block part
  int k_off[DS];                             // K: token col, piece (4 j + qd) ^ f(col)
#pragma unroll
  for (int j = 0; j < DS; ++j) k_off[j] = col * ROWB + (((4 * j + qd) ^ swz(col)) << 4);
  int v_off[DT];                             // V: token 4 qd + col / 4, piece (2 dt + (col & 3) / 2) ^ f, half col & 1
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    const int t = 4 * qd + (col >> 2);
    v_off[dt] = t * ROWB + (((2 * dt + ((col & 3) >> 1)) ^ swz(t)) << 4) + ((col & 1) << 3);
  }

  auto compute = [&](auto half_only, int ti, auto& Kb, auto& Vb) __attribute__((always_inline)) {
    constexpr bool HALF = decltype(half_only)::value;
    const __bf16 *kp_, *vp_; long long stride_; int tok0, seglen; bool is_tree;
    locate(ti, kp_, vp_, stride_, tok0, seglen, is_tree);
    const int nvalid = min(TILE, seglen - tok0);
    const char* const kl = reinterpret_cast<const char*>(&Kb[0]);
    const char* const vl = reinterpret_cast<const char*>(&Vb[0]);
    const bool need_mask = is_tree || nvalid < TILE;
#pragma unroll
    for (int step = 0; step < (HALF ? 1 : TILE / 32); ++step) {
      const int ks = HALF ? half : step;
      floatx4 s[NRT][2];
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) {
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) s[rt][t2] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < DS; ++j) {
          const bf16x8 kfrag = *reinterpret_cast<const bf16x8*>(kl + (32 * ks + 16 * t2) * ROWB + k_off[j]);
#pragma unroll
          for (int rt = 0; rt < NRT; ++rt)
            s[rt][t2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kfrag, qf[rt][j], s[rt][t2], 0, 0, 0);
        }
      }
      bf16x8 pf[NRT];
      bool raise = false;
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        float mx = fmaxf(fmaxf(s[rt][0][0], s[rt][0][1]), fmaxf(s[rt][0][2], s[rt][0][3]));
        mx = fmaxf(mx, fmaxf(fmaxf(s[rt][1][0], s[rt][1][1]), fmaxf(s[rt][1][2], s[rt][1][3])));
        raise = raise || (mx * a.scale_log2 > m_run[rt] + REF_SLACK);
      }
      if (!need_mask && __builtin_amdgcn_ballot_w64(raise) == 0ull) {
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) {
          const float nm = -m_run[rt];
          float psum = 0.f;
#pragma unroll
          for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float p = __builtin_amdgcn_exp2f(fmaf(s[rt][t2][i], a.scale_log2, nm));
              psum += p;
              pf[rt][4 * t2 + i] = (__bf16)p;
            }
          l_run[rt] += psum;
        }
      } else {
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) {
          float sv[8];
          unsigned okbits = 0;
#pragma unroll
          for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int t = 32 * ks + 16 * t2 + 4 * qd + i;
              bool valid = t < nvalid;
              if (is_tree) valid = valid && ((anc[rt] >> (tok0 + t)) & 1ull);
              if (valid) okbits |= 1u << (4 * t2 + i);
              sv[4 * t2 + i] = valid ? s[rt][t2][i] * a.scale_log2 : NEG_BIG;
            }
          float mx = sv[0];
#pragma unroll
          for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sv[e]);
          mx = fmaxf(mx, __shfl_xor(mx, 16));
          mx = fmaxf(mx, __shfl_xor(mx, 32));
          const float m_new = (mx > m_run[rt] + REF_SLACK) ? mx : m_run[rt];
          const float alpha = __builtin_amdgcn_exp2f(m_run[rt] - m_new);
          l_run[rt] *= alpha;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) o[rt][dt] *= alpha;
          m_run[rt] = m_new;
          float psum = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float p = ((okbits >> e) & 1u) ? __builtin_amdgcn_exp2f(sv[e] - m_new) : 0.f;
            psum += p;
            pf[rt][e] = (__bf16)p;
          }
          l_run[rt] += psum;
        }
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        // A operand = V^T: lane (channel 16dt + col, qd) needs tokens 4qd .. 4qd+3 of both 16-token blocks of the
        // half, the order the numerators have in pf.  A transposing read returns, to lane i of a group of 16, the
        // element i % 4 of the four lanes i / 4, 4 + i / 4, ...: so lane i points at token 4qd + i / 4, channels
        // 16dt + 4 (i % 4) .. + 3, and receives channel 16dt + i of tokens 4qd .. 4qd+3.
        union { v4i16 h[2]; bf16x8 v; } vf;
        const char* rowp = vl + 32 * ks * ROWB + v_off[dt];
        vf.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(rowp));
        vf.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(rowp + 16 * ROWB));
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt)
          o[rt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf.v, pf[rt], o[rt][dt], 0, 0, 0);
      }
    }
  };

  int ti = t_begin;
  if (ti < t_end) issue(ti, kA, vA);
  {
    uint64_t my_anc = 0;
    const int tb = dsbd_tree_walk(tr, lane, p_mine, a.max_depth, nullptr, reporter ? a.anc_out : nullptr, &my_anc);
    if (reporter && tb) atomicOr(a.fault, tb);
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) {
      const int r = row0 + rt * 16 + col;
      const int node = r < R ? r / a.group : 0;
      const unsigned lo = __shfl((unsigned)my_anc, node), hi = __shfl((unsigned)(my_anc >> 32), node);
      anc[rt] = r < R ? ((uint64_t)hi << 32) | lo : 0ull;
    }
  }
  // One barrier per tile: it says that every wave's part of tile ti has landed (each wave waits for its own loads
  // first) and that everybody is done reading the other buffer, into which the next tile is then requested.
  // (The loop is there twice, for waves on whole tiles and on halves: with the choice inside, the second half's LDS reads
  // could not start under the first half's arithmetic.  8 beams of 31 nodes, 32/8 heads, 4500 tokens: 49.2 -> 47.9 us, 8192
  // tokens 67.2 -> 65.0.)
  auto tiles = [&](auto half_only) __attribute__((always_inline)) {
    while (ti < t_end) {
      __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
      lds_barrier();
      if (ti + 1 < t_end) issue(ti + 1, kB, vB);
      if (computes) compute(half_only, ti, kA, vA);
      if (++ti >= t_end) break;
      __builtin_amdgcn_s_waitcnt(0x0F70);
      lds_barrier();
      if (ti + 1 < t_end) issue(ti + 1, kA, vA);
      if (computes) compute(half_only, ti, kB, vB);
      ++ti;
    }
  };
  if (halves) tiles(std::true_type{}); else tiles(std::false_type{});
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();                           // nobody reads a tile any more: the buffers become the output staging

#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    l_run[rt] += __shfl_xor(l_run[rt], 16);
    l_run[rt] += __shfl_xor(l_run[rt], 32);
  }
  // ---- rows go through the LDS so that each leaves as one contiguous write: a wave's 32 rows in "its" array, the
  // 16-byte pieces of a row swizzled by the row number
  constexpr int QPR = D / 4;
  auto array_of = [&](int w) { return w == 0 ? kA : (w == 1 ? kB : (w == 2 ? vA : vB)); };
  auto stage = [&](uint4* st) {
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        union { floatx4 f; uint4 u; } cv;
        cv.f = o[rt][dt];
        st[(rt * 16 + col) * QPR + ((4 * dt + qd) ^ (col & 7))] = cv.u;
      }
  };
  if (halves) {
    // the second half's results join the first half's (wave 2 -> wave 0, wave 3 -> wave 1)
    if (half == 1) {
      stage(array_of(wave));
      if (qd == 0)
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) { half_ml[rgrp * ROWS_W + rt * 16 + col][0] = m_run[rt]; half_ml[rgrp * ROWS_W + rt * 16 + col][1] = l_run[rt]; }
    }
    __syncthreads();
    if (half == 0) {
      const uint4* const sr = array_of(wave + 2);
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        const float m2 = half_ml[rgrp * ROWS_W + rt * 16 + col][0], l2 = half_ml[rgrp * ROWS_W + rt * 16 + col][1];
        const float m_new = fmaxf(m_run[rt], m2);
        const float a1 = __builtin_amdgcn_exp2f(m_run[rt] - m_new), a2 = __builtin_amdgcn_exp2f(m2 - m_new);
        l_run[rt] = l_run[rt] * a1 + l2 * a2;
        m_run[rt] = m_new;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          union { floatx4 f; uint4 u; } cv;
          cv.u = sr[(rt * 16 + col) * QPR + ((4 * dt + qd) ^ (col & 7))];
          o[rt][dt] = o[rt][dt] * a1 + cv.f * a2;
        }
      }
    }
  }
  if (half == 0) {
    stage(array_of(rgrp));
    if (qd == 0)
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        const int rl = rgrp * ROWS_W + rt * 16 + col, r = rb * ROWS_B + rl;
        row_ml[rl][0] = m_run[rt]; row_ml[rl][1] = l_run[rt];
        row_id[rl] = (base + r / a.group) * a.Hq + g * a.group + r % a.group;
      }
  }
  __syncthreads();
  // (a short loop on purpose: every workgroup runs this once, and instructions that are not in the cache yet cost more
  // than the LDS reads' round trips: written out over the rows 1.3 us more)
  const PartPlace place = part_place(a, split, nsplit, rows_here);
  for (int c = tid; c < place.rows * QPR; c += AT_BLOCK) {
    const int rl = c / QPR, part = c % QPR, lr = rl % ROWS_W;
    union { floatx4 f; uint4 u; } cv;
    cv.u = array_of(rl / ROWS_W)[lr * QPR + (part ^ (lr & 7))];
    const float M = row_ml[rl][0], L = row_ml[rl][1];
    const int row = row_id[rl];
    const long long prow = place.at + (a.by_split ? row : rl);
    if (part == 0 && split == 0 && a.row_parts) a.row_parts[row] = make_int2((int)prow, nsplit);
    if (nsplit == 1) {
      write_row_part<D>(a, row, part, M, L, cv.f);
    } else {
      if (part == 0) *reinterpret_cast<float2*>(&a.part_ml[prow * 2]) = make_float2(M, L);
      *reinterpret_cast<uint4*>(&a.part_o[prow * D + 4 * part]) = cv.u;
    }
  }
}

// Merge the KV splits of the rows that have several: out = sum_s 2^(m_s-M) O_s / sum_s 2^(m_s-M) l_s.  The workgroups of
// the rows' first splits have left where a row's partial results are.  SG threads share four channels of a row: each takes
// every SG-th split, eight at a time with all their loads in flight, then they meet in the LDS.  Many rows are bound by
// the partial results' bytes and take SG = 1 (8 beams x 31 nodes x 32 heads, 8 splits: 7.5 us, SG = 4: 11.1); few rows of
// many splits by a thread's round trips, SG = 4 (2 x 23 nodes x 32 heads, 32 splits: 6.8 us against 8.0).
template <int D, int SG>
__global__ __launch_bounds__(AT_BLOCK) void forest_attention_combine_kernel(AttnArgs a) {
  constexpr int QPR = D / 4;                 // float4 quads per row
  constexpr int RPB = AT_BLOCK / (QPR * SG); // rows per workgroup
  __shared__ floatx4 s_acc[SG][SG > 1 ? RPB * QPR : 1];
  __shared__ float2 s_ml[SG][RPB];
  const int lr = threadIdx.x % (RPB * QPR), sg = SG > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / (RPB * QPR)) : 0;      // (waves)
  const long long row = (long long)blockIdx.x * RPB + lr / QPR;
  const int quad = lr % QPR;
  const bool in = row < (long long)a.n_nodes * a.Hq;
  // By split, the places of a row's results are known without its entry in row_parts: the first two that a thread may need
  // travel beside it (what is read of a split that the row does not have is not used).
  const float* po = a.part_o + row * D + 4 * quad;
  const float* pml = a.part_ml + row * 2;
  auto fetch = [&](int s, float2& ml, floatx4& v) __attribute__((always_inline)) {
    const long long off = s * a.part_stride;            // (uniform)
    ml = *reinterpret_cast<const float2*>(pml + off * 2);
    v = *reinterpret_cast<const floatx4*>(po + off * D);
  };
  float2 ml[8];
  floatx4 v[8];
  if (a.by_split && in) {
#pragma unroll
    for (int j = 0; j < 2; ++j) fetch(min(sg + j * SG, a.nsplit - 1), ml[j], v[j]);
  }
  const int2 parts = in ? a.row_parts[row] : make_int2(0, 0);
  const int nsplit = parts.y;
  const long long first = a.by_split ? row : parts.x;
  // (one part: already written by the main kernel; the rows of a tree with unusable offsets hold nothing to go by)
  const bool live = nsplit >= 2 && nsplit <= a.nsplit && first >= 0 && first + (nsplit - 1) * a.part_stride < a.part_rows;
  float M = NEG_BIG, L = 0.f;
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  if (live && sg < nsplit) {
    int s0 = sg;
    if (!a.by_split) {
      po = a.part_o + first * D + 4 * quad;
      pml = a.part_ml + first * 2;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        if (s0 + j * SG < nsplit) fetch(s0 + j * SG, ml[j], v[j]);
    }
    while (true) {
#pragma unroll
      for (int j = 2; j < 8; ++j)
        if (s0 + j * SG < nsplit) fetch(s0 + j * SG, ml[j], v[j]);
      float Mb = M;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (s0 + j * SG < nsplit) Mb = fmaxf(Mb, ml[j].x);
      const float keep = exp2f(M - Mb);                   // 1 when the reference stays
      L *= keep; acc *= keep; M = Mb;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (s0 + j * SG < nsplit) {
          const float w = exp2f(ml[j].x - M);
          L += w * ml[j].y;
          acc += w * v[j];
        }
      s0 += 8 * SG;
      if (s0 >= nsplit) break;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        if (s0 + j * SG < nsplit) fetch(s0 + j * SG, ml[j], v[j]);
    }
  }
  if constexpr (SG > 1) {
    if (sg > 0) {
      s_acc[sg][lr] = acc;
      if (quad == 0) s_ml[sg][lr / QPR] = make_float2(M, L);
    }
    __syncthreads();
  }
  if (sg > 0 || !live) return;
#pragma unroll
  for (int g = 1; g < SG; ++g) {
    const float2 o = s_ml[g][lr / QPR];
    const float Mn = fmaxf(M, o.x), e1 = exp2f(M - Mn), e2 = exp2f(o.x - Mn);
    L = L * e1 + o.y * e2;
    acc = acc * e1 + s_acc[g][lr] * e2;
    M = Mn;
  }
  write_row_part<D>(a, row, quad, M, L, acc);
}

// ------------------------------------------------------------------------------------------------ host side
namespace {

struct AttnPlan {
  int nrt;                    // 16-row tiles per wave
  int waves;                  // waves per workgroup of the wave-private kernel
  bool shared;                // tiles shared by the waves (many rows per stream) instead of wave-private streams
  int rows_block, n_rowblocks;
  bool by_tree;
  int nsplit;                 // by_tree: the most splits any tree may get; else every unit's
  int slots;
  long long grid;             // workgroups of the main kernel
  bool merge;                 // some unit may be split
  bool by_split;              // layout of the partial results, see AttnArgs
  int part_pitch;
  long long part_stride, part_rows;
  long long part_room;        // rows of partial results that the workspace holds: part_rows, or more (see make_plan)
};

AttnPlan make_plan(const dsbd_forest* f, const dsbd_kv* kv, int Hq, int Hkv, int D) {
  AttnPlan p;
  const int group = Hq / Hkv;
  const int rmax = f->max_tree_nodes * group;
  p.shared = rmax > 32;
  p.nrt = rmax <= 16 ? 1 : 2;
  p.rows_block = p.shared ? 128 : 16 * p.nrt;
  p.n_rowblocks = (rmax + p.rows_block - 1) / p.rows_block;
  const int unit = p.shared ? 64 : STEP;
  // units there can be: a row block per (tree, KV head), and one more for every rows_block rows
  long long units = (long long)Hkv * (f->n_trees + (long long)f->n_nodes * group / p.rows_block);
  const long long most = (long long)f->n_trees * Hkv * p.n_rowblocks;
  if (units > most) units = most;
  const int most_steps = (kv->max_len + unit - 1) / unit + 2;
  p.by_tree = f->n_trees <= AT_BLOCK && dsbd_knobs().attn_nsplit <= 0;
  // Workgroups to spread the work over: as many as are resident at once, two per compute unit (one for 32 rows of 128
  // channels in the wave-private kernel, which take a SIMD's registers).  Wave-private work of less than four steps per
  // wave that way is quicker on one workgroup per unit: some units would have two to run and the others wait for them (us
  // at 256 / 512 workgroups or the next fewer that come out even: 64 units of 36 steps 16.1 / 16.5, 80 units of 36 steps, 24
  // rows, 20.6 / 32.7, 128 units of 65 steps 29.8 / 28.7).
  p.slots = 512;
  p.waves = 4;
  // Workgroups of eight waves, one per compute unit, where all units fit the device at once: the same waves as two workgroups
  // of four, but no or half the splits, and twice the loads in flight where a unit is not worth splitting.  Not for few
  // units of middling length, which more workgroups serve better, nor for long ones that leave units idle.  Measured, call in
  // us with four / eight waves: 128 units of 18 steps 15.7 / 13.4, 256 units of 36 steps 32.3 / 27.5, 160 units of 36 steps 26.0
  // / 21.8, 32 units of 130 steps 20.0 / 18.4, of 9 steps 11.3 / 10.0; 32 units of 36 steps (64 channels) 11.4 / 12.3, 12 units of
  // 49 steps 12.3 / 13.2, 8 units of 64 steps 12.0 / 12.8, 128 units of 130 steps (64 channels) 31.4 / 33.8.
  // The bounds where a unit is worth splitting: more than 64 units, 8448 = 128 units x 66 steps, just above the 65 at which eight
  // waves still won (the next point, 128 x 130 = 16640, lost; nothing was measured between); up to 32 units, 4096, just below the
  // 32 x 130 that won (32 x 36 lost); 33 to 64 units have no point of their own, 2048 lies between these two.
  const long long work = units * most_steps;
  const bool unsplit = most_steps < (units <= 16 ? 12 : 24);
  if (!p.shared && f->n_trees <= 64 && units <= 256 && (p.nrt == 1 || D == 64) &&
      (units > 192 || unsplit || (units > 64 ? work <= 8448 : work >= (units > 32 ? 2048 : 4096)))) { p.waves = 8; p.slots = 256; }
  else if (!p.shared && ((D == 128 && p.nrt == 2) || units * most_steps < 16LL * 512)) p.slots = 256;
  // Short units stay whole: what splitting takes off them is less than the merge's launch, the less so the more units there
  // are (us unsplit / in two / three / four: 8 units of 8 steps 12.7 / 13.0 / 12.9 / 12.9, of 11 steps 14.3 / 15.1 / 13.0 / 12.8;
  // 64 units of 11 steps 11.5 / 12.7 / 11.2 / 11.2; 96 units of 15 steps 13.0 / 13.6, of 17 steps 14.3 / 14.0; 128 units of 17
  // steps 14.5 / 15.1, of 23 steps 16.5 / 16.4; 32 units of 5 tiles 15.1 / 15.5 / - / 14.7, of 3 tiles 12.9 / 14.3 / - / 14.1).  And
  // with two rounds of workgroups none is split (a tree much longer than the others could still gain by it; not measured).
  const int worth = p.shared ? 7 : p.waves == 8 ? 24 : (units <= 64 ? 12 : (units < 128 ? 18 : 24));
  int most_split = split_limit(most_steps, p.shared, p.waves);
  if (most_steps < worth || (long long)f->n_trees * Hkv >= 2 * 512) most_split = 1;
  if (p.by_tree) {
    // (a tree's units are at least its KV heads, so its share of what the units leave is at most this; with no split there
    // is nothing to merge: 256 units of 36 steps 29.3 -> 27.4 us)
    const long long spare = p.slots - (long long)f->n_trees * Hkv;
    if (const long long share = 1 + (spare > 0 ? spare / Hkv : 0); most_split > share) most_split = (int)share;
    p.nsplit = most_split;
    p.grid = p.nsplit > 1 && units < p.slots ? p.slots : units;
  } else {
    // (more trees than threads fill the device by themselves, unless they have a single KV head)
    p.nsplit = most > 0 ? (int)((p.slots + most - 1) / most) : 1;
    if (p.nsplit > most_split) p.nsplit = most_split;
    if (const int v = dsbd_knobs().attn_nsplit; v >= 1 && v <= AT_MAX_SPLIT) p.nsplit = v;   // tuning knob: KV splits of every unit
    p.grid = most * p.nsplit;
  }
  p.merge = p.nsplit > 1;
  const long long rows = (long long)f->n_nodes * Hq;
  p.part_pitch = p.rows_block < rmax ? p.rows_block : rmax;
  // (trees are split only where all workgroups together are no more than the slots)
  const long long slot_rows = (p.by_tree && p.grid > p.slots ? p.slots : p.grid) * p.part_pitch, split_rows = rows * p.nsplit;
  p.by_split = split_rows < slot_rows;
  p.part_stride = p.by_split ? rows : p.part_pitch;
  p.part_rows = !p.merge ? 0 : (p.by_split ? split_rows : slot_rows);
  // The workspace asked for covers what any forest within these bounds (fewer trees, nodes, tokens) can need, split or
  // not, so that a buffer for a caller's largest call serves the others too.
  auto room = [&](bool tiles) -> long long {       // (smaller trees may take the other kernel)
    const int steps = (kv->max_len + (tiles ? 64 : STEP) - 1) / (tiles ? 64 : STEP) + 2;
    const int splits = steps < (tiles ? 7 : 12) ? 1 : split_limit(steps, tiles, 4), pitch = tiles ? p.part_pitch : (p.part_pitch < 32 ? p.part_pitch : 32);
    const long long by_slot = (f->n_trees > AT_BLOCK ? 1024LL : 512LL) * pitch;
    return splits < 2 ? 0 : (rows * splits < by_slot ? rows * splits : by_slot);
  };
  p.part_room = room(false);
  if (p.shared && p.part_room < room(true)) p.part_room = room(true);
  if (p.part_room < p.part_rows) p.part_room = p.part_rows;
  return p;
}

// The workspace: partial results and the rows' entries.
size_t carve_attention(WorkspaceCarver& ws, const AttnPlan& p, const dsbd_forest* f, int Hq, int D, AttnArgs* a) {
  float* const o = ws.take<float>((size_t)p.part_room * D);
  float* const ml = ws.take<float>((size_t)p.part_room * 2);
  int2* const parts = ws.take<int2>(p.part_room > 0 ? (size_t)f->n_nodes * Hq : 0);
  if (a) { a->part_o = o; a->part_ml = ml; a->row_parts = p.merge ? parts : nullptr; }
  return ws.total() + 256;
}

int32_t check_args(const dsbd_forest* f, const dsbd_kv* kv, int Hq, int Hkv, int D) {
  if (!f || !kv) return DSBD_ERR_INVALID;
  if (f->n_trees < 0 || f->n_nodes < 0 || f->n_prompts < 0) return DSBD_ERR_INVALID;
  if (Hq <= 0 || Hkv <= 0 || Hq % Hkv != 0) return DSBD_ERR_INVALID;
  if (D != 128 && D != 64) return DSBD_ERR_UNSUPPORTED;
  if (f->max_tree_nodes < 1 || f->max_tree_nodes > DSBD_MAX_TREE_NODES) return DSBD_ERR_UNSUPPORTED;
  if (kv->max_len < 0) return DSBD_ERR_INVALID;
  if (kv->token_stride % 8 != 0 || kv->head_stride % 8 != 0) return DSBD_ERR_UNSUPPORTED;
  return DSBD_OK;
}

int32_t check_pointers(const dsbd_forest* f, const dsbd_kv* kv) {
  if (f->n_trees > 0 && (!f->tree_off || !f->parent || !kv->k_ptr || !kv->v_ptr || !kv->len)) return DSBD_ERR_INVALID;
  if ((kv->shared_len != nullptr) != (kv->k_shared_ptr != nullptr) ||
      (kv->shared_len != nullptr) != (kv->v_shared_ptr != nullptr)) return DSBD_ERR_INVALID;
  return DSBD_OK;
}

template <int D>
void launch_attention(const AttnPlan& p, const AttnArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)p.grid), block(AT_BLOCK);
  if (p.shared) dsbd_launch(DSBD_KERNEL_ATTENTION, forest_attention_dma_kernel<D, D == 128 ? 2 : 3>, grid, block, 0, stream, a);
  else if (p.waves == 8) {
    const dim3 wide(512);
    if (p.nrt == 1) dsbd_launch(DSBD_KERNEL_ATTENTION, forest_attention_kernel<D, 1, 8>, grid, wide, 0, stream, a);
    else if constexpr (D == 64) dsbd_launch(DSBD_KERNEL_ATTENTION, forest_attention_kernel<D, 2, 8>, grid, wide, 0, stream, a);
  }
  else if (p.nrt == 1) dsbd_launch(DSBD_KERNEL_ATTENTION, forest_attention_kernel<D, 1, 4>, grid, block, 0, stream, a);
  else dsbd_launch(DSBD_KERNEL_ATTENTION, forest_attention_kernel<D, 2, 4>, grid, block, 0, stream, a);
  if (p.merge) {
    const long long rows = (long long)a.n_nodes * a.Hq, wgs = (rows * (D / 4) + AT_BLOCK - 1) / AT_BLOCK;
    if (wgs < 256 && p.nsplit >= 8) {         // fewer workgroups than compute units
      hipLaunchKernelGGL((forest_attention_combine_kernel<D, 4>), dim3((unsigned)((rows * D + AT_BLOCK - 1) / AT_BLOCK)), block, 0, stream, a);
    } else {
      hipLaunchKernelGGL((forest_attention_combine_kernel<D, 1>), dim3((unsigned)wgs), block, 0, stream, a);
    }
  }
}

}  // namespace

extern "C" size_t dsbd_forest_attention_workspace_bytes(const dsbd_forest* f, const dsbd_kv* kv, int32_t Hq,
                                                        int32_t Hkv, int32_t D) {
  if (check_args(f, kv, Hq, Hkv, D) != DSBD_OK) return 0;
  const AttnPlan p = make_plan(f, kv, Hq, Hkv, D);
  WorkspaceCarver ws(nullptr);
  return carve_attention(ws, p, f, Hq, D, nullptr);
}

extern "C" int32_t dsbd_forest_attention(const dsbd_forest* f, const dsbd_kv* kv, const void* q, const void* k_tree,
                                         const void* v_tree, int32_t Hq, int32_t Hkv, int32_t D, float scale,
                                         void* out, float* lse, uint64_t* anc_mask_out, void* workspace,
                                         size_t workspace_bytes, int32_t* fault, void* stream_) {
  int32_t rc = check_args(f, kv, Hq, Hkv, D);
  if (rc != DSBD_OK) return rc;
  if (!fault) return DSBD_ERR_INVALID;
  if (f->n_nodes == 0 || f->n_trees == 0) return DSBD_OK;
  rc = check_pointers(f, kv);
  if (rc != DSBD_OK) return rc;
  if (!q || !k_tree || !v_tree || !out || !workspace) return DSBD_ERR_INVALID;
  if ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k_tree) | reinterpret_cast<uintptr_t>(v_tree) |
       reinterpret_cast<uintptr_t>(out)) & 15)
    return DSBD_ERR_INVALID;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  const AttnPlan p = make_plan(f, kv, Hq, Hkv, D);
  {
    WorkspaceCarver none(nullptr);
    if (workspace_bytes < carve_attention(none, p, f, Hq, D, nullptr)) return DSBD_ERR_WORKSPACE;
  }
  // (a slot's rows are counted in 32-bit integers)
  if (p.grid > 0x7fffffffLL || (!p.by_split && p.part_rows > 0x7fffffffLL)) return DSBD_ERR_UNSUPPORTED;

  WorkspaceCarver ws(reinterpret_cast<char*>(dsbd_align_up(reinterpret_cast<uintptr_t>(workspace), 256)));
  AttnArgs a;
  carve_attention(ws, p, f, Hq, D, &a);
  a.tree_off = f->tree_off; a.parent = f->parent;
  a.max_tree_nodes = f->max_tree_nodes; a.max_depth = f->max_depth; a.anc_out = anc_mask_out;
  a.k_ptr = kv->k_ptr; a.v_ptr = kv->v_ptr; a.len = kv->len;
  a.k_shared_ptr = kv->k_shared_ptr; a.v_shared_ptr = kv->v_shared_ptr; a.shared_len = kv->shared_len;
  a.token_stride = kv->token_stride; a.head_stride = kv->head_stride;
  a.q = static_cast<const __bf16*>(q); a.k_tree = static_cast<const __bf16*>(k_tree);
  a.v_tree = static_cast<const __bf16*>(v_tree);
  a.n_trees = f->n_trees; a.n_nodes = f->n_nodes; a.Hq = Hq; a.Hkv = Hkv; a.group = Hq / Hkv;
  const float sc = scale > 0.f ? scale : 1.0f / sqrtf((float)D);
  a.scale_log2 = sc * 1.4426950408889634f;
  a.max_len = kv->max_len;
  a.by_tree = p.by_tree ? 1 : 0; a.nsplit = p.nsplit; a.n_rowblocks = p.n_rowblocks; a.rows_block = p.rows_block;
  a.wg_slots = p.slots; a.waves = p.waves;
  a.by_split = p.by_split ? 1 : 0; a.part_pitch = p.part_pitch; a.part_stride = p.part_stride; a.part_rows = p.part_rows;
  a.out = static_cast<__bf16*>(out); a.lse = lse; a.fault = fault;
  if (D == 128) launch_attention<128>(p, a, stream);
  else launch_attention<64>(p, a, stream);
  DSBD_HIP_LAUNCH_CHECK();
  return DSBD_OK;
}
