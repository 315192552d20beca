// Physical key/value cache update after an iteration (paper Section 3.3, last paragraph: the caches are
// updated to follow the output beams; Section 3.4: a single cache in the memory-reduced variant).
//
// The cache of a next-iteration beam = the own cache segment of the input beam it descends from, followed by the
// key/value rows of the forest nodes on the path root .. the node the output beam hangs from (the plan written by
// dsbd_select_beams).  A pure copy, bound by HBM bandwidth.  A destination that IS its source buffer (the beam continues
// in place) only gets the tree rows appended.
//
// A workgroup takes up to 16 tokens of K or of V of one prompt and works through the prompt's sources: 16-byte pieces, eight
// loads in flight per thread, and every piece goes to all the destinations that continue this source, so a source is read
// once however many next beams share it.  The path rows are handed out over the prompt's workgroups in units of four tokens,
// to those first that are left over by the sources.
//
// Measured, a call in us: 8 beams of 8192 tokens x 8 heads x 128, their caches copied along a plan (33.7 MB read, 235 MB
// written) 42.0; 7 prompts of 8 beams, 40 heads, prefixes of 40 tokens 12.2 (27.7 with 16 tokens per workgroup whatever their
// length: too few workgroups); eight chains of 64 nodes x 40 heads behind prefixes of 32 tokens 9.7 (57.6 with all of a
// destination's path rows in one workgroup).
#include "common.h"
#include <algorithm>

#define CM_BLOCK 256
#define CM_TOKENS 16           // most tokens per workgroup (8: 43.7 us, 24: 45.7, 32: 49.1 on the first plan above, at 43.0 for 16); fewer
                               // where a round of loads takes fewer (more than 8 heads of 128)
#define CM_CHUNKS (1LL << 20)  // most chunks of a launch: beyond, a workgroup takes several (a far bound on the lengths costs little)
#define CM_PATH_TOKENS 4       // path rows per unit (8 with eight loads in flight: 13.6 us on the last plan above)
#define CM_LOADS 8             // 16-byte loads in flight per thread (4: 46.8 us; 512 threads with 4: 45.3, at 43.0 for 8)
#define CM_GRID 2048           // workgroups that the device holds at once (grids of twice that: 47.4 us, at 43.0)

struct CommitArgs {
  int n_prompts, n_trees, n_nodes, W_cap, plen, Hkv, D, shares;
  int tokens;                  // per chunk
  const void* const* src_k; const void* const* src_v; const int32_t* src_len;
  long long token_stride, head_stride;      // elements; the same layout for sources and destinations
  const __bf16 *k_tree, *v_tree;            // [n_nodes, Hkv, D]
  const int32_t *n_next, *src_tree, *path_len, *path;
  void* const* dst_k; void* const* dst_v; int32_t* dst_len;
  int capacity, max_len;
  int32_t* fault;
};

typedef unsigned int cm_u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) cm_u32x4 cm_gvec;

__device__ __forceinline__ unsigned long long cm_lane(unsigned long long v, int l) {
  const unsigned int lo = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)v, l);
  const unsigned int hi = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)(v >> 32), l);
  return ((unsigned long long)hi << 32) | lo;
}

// Workgroup (chunk x {K, V}, share, prompt): the sources number share, share + shares, .. of the prompt.
__global__ __launch_bounds__(CM_BLOCK) void commit_kv_kernel(CommitArgs a) {
  const int chunk = blockIdx.x >> 1, share = blockIdx.y, p = blockIdx.z, is_v = blockIdx.x & 1;
  const int tid = threadIdx.x, lane = tid & 63;
  // the prompt's destinations, one per lane
  const bool slot = lane < a.W_cap;
  const int j0 = p * a.W_cap, j = j0 + min(lane, a.W_cap - 1);
  const int nn = max(0, min(a.n_next[p], a.W_cap));
  const int b = a.src_tree[j];
  const char* const dk = static_cast<const char*>(a.dst_k[j]);
  const char* const dv = static_cast<const char*>(a.dst_v[j]);
  const int pl = max(0, min(a.path_len[j], a.plen));
  const bool known = b >= 0 && b < a.n_trees;
  const int bc = known ? b : 0;
  int L_raw = 0;
  const char *sk = nullptr, *sv = nullptr;
  if (a.n_trees > 0) {
    L_raw = a.src_len[bc];
    sk = static_cast<const char*>(a.src_k[bc]); sv = static_cast<const char*>(a.src_v[bc]);
  }
  // the source length is the caller's: the grid covers max_len tokens, so a longer source cannot be copied
  const int L = max(0, min(L_raw, a.max_len));
  // Both planes are checked by every workgroup (the K and the V workgroups of a destination must take the same
  // decision: a destination with a usable K buffer and a null or misaligned V buffer is left untouched as a whole).
  const bool bad = L_raw < 0 || L_raw > a.max_len || L + pl > a.capacity || !dk || !dv || (L > 0 && (!sk || !sv)) ||
                   ((reinterpret_cast<uintptr_t>(dk) | reinterpret_cast<uintptr_t>(sk) |
                     reinterpret_cast<uintptr_t>(dv) | reinterpret_cast<uintptr_t>(sv)) & 15);
  const bool on = lane < nn, good = on && known && !bad;
  if (chunk == 0 && share == 0 && !is_v && tid == lane && slot) {      // one thread per destination reports and writes the length
    a.dst_len[j] = good ? L + pl : 0;
    if (on && !good) atomicOr(a.fault, known ? DSBD_FAULT_BOUNDS : DSBD_FAULT_TOPOLOGY);
  }
  const unsigned long long src = reinterpret_cast<unsigned long long>(is_v ? sv : sk);
  const unsigned long long dst = reinterpret_cast<unsigned long long>(is_v ? dv : dk);
  const int CG = a.D / 8;                    // 16-byte pieces per (token, head)
  const int per_tok = a.Hkv * CG;
  auto place = [&](int t, int r) -> long long {      // byte offset of piece r of token t in a cache
    return ((long long)t * a.token_stride + (long long)(r / CG) * a.head_stride + r % CG * 8) * 2;
  };

  // ---- the destinations' path rows, CM_PATH_TOKENS at a time, over the workgroups of the prompt: the last shares first, which
  // have no source where there are fewer sources than shares
  const __bf16* const rows = is_v ? a.v_tree : a.k_tree;
  const unsigned long long with_path = __builtin_amdgcn_ballot_w64(good && pl > 0);
  const int parts = (a.plen + CM_PATH_TOKENS - 1) / CM_PATH_TOKENS, n_unit = nn * parts;
  for (long long at = (long long)(a.shares - 1 - share) * (gridDim.x >> 1) + chunk; at < n_unit; at += (long long)(gridDim.x >> 1) * a.shares) {
    const int unit = (int)at;
    const int q = unit / parts, k0 = (unit - q * parts) * CM_PATH_TOKENS;
    if (!((with_path >> q) & 1)) continue;
    const int qL = __builtin_amdgcn_readlane(L, q), n_piece = (min(__builtin_amdgcn_readlane(pl, q), k0 + CM_PATH_TOKENS) - k0) * per_tok;
    char* const to = reinterpret_cast<char*>(cm_lane(dst, q));
    const int32_t* const path = a.path + (long long)(j0 + q) * a.plen + k0;
    for (int i0 = tid; i0 < n_piece; i0 += 2 * CM_BLOCK) {
      cm_u32x4 v[2];
      long long off[2];
      bool have[2];
#pragma unroll
      for (int l = 0; l < 2; ++l) {
        const int i = i0 + l * CM_BLOCK, k = i / per_tok, r = i % per_tok;
        have[l] = false;
        if (i >= n_piece) continue;
        const int node = path[k];
        if (node < 0 || node >= a.n_nodes) { atomicOr(a.fault, DSBD_FAULT_TOPOLOGY); continue; }
        v[l] = *(const cm_gvec*)(rows + ((long long)node * per_tok + r) * 8);
        off[l] = place(qL + k0 + k, r);
        have[l] = true;
      }
#pragma unroll
      for (int l = 0; l < 2; ++l)
        if (have[l]) __builtin_nontemporal_store(v[l], (cm_gvec*)(to + off[l]));
    }
  }
  // ---- the sources' tokens
  for (long long at = (long long)chunk * a.tokens; at < a.max_len; at += (long long)(gridDim.x >> 1) * a.tokens) {
    const int t0 = (int)at;
    unsigned long long left = __builtin_amdgcn_ballot_w64(good && t0 < L && dst != src);
    if (!left) break;
    for (int n = 0; left; ++n) {
      const int q0 = (int)__ffsll((long long)left) - 1;
      const unsigned long long takers = left & __builtin_amdgcn_ballot_w64(b == __builtin_amdgcn_readlane(b, q0));
      left &= ~takers;
      if (n % a.shares != share) continue;
      const char* const from = reinterpret_cast<const char*>(cm_lane(src, q0));
      const int n_piece = (min(__builtin_amdgcn_readlane(L, q0), t0 + a.tokens) - t0) * per_tok;
      for (int i0 = tid; i0 < n_piece; i0 += CM_LOADS * CM_BLOCK) {
        cm_u32x4 v[CM_LOADS];
        long long off[CM_LOADS];
#pragma unroll
        for (int k = 0; k < CM_LOADS; ++k) {
          const int i = min(i0 + k * CM_BLOCK, n_piece - 1);
          off[k] = place(t0 + i / per_tok, i % per_tok);
          v[k] = __builtin_nontemporal_load((const cm_gvec*)(from + off[k]));
        }
        for (unsigned long long m = takers; m; m &= m - 1) {
          char* const to = reinterpret_cast<char*>(cm_lane(dst, (int)__ffsll((long long)m) - 1));
#pragma unroll
          for (int k = 0; k < CM_LOADS; ++k)
            if (i0 + k * CM_BLOCK < n_piece) __builtin_nontemporal_store(v[k], (cm_gvec*)(to + off[k]));
        }
      }
    }
  }

}

extern "C" int32_t dsbd_commit_kv(const dsbd_forest* f, const dsbd_kv* src, const void* k_tree, const void* v_tree,
                                  int32_t Hkv, int32_t D, const dsbd_next_beams* next, int32_t W_cap,
                                  const dsbd_kv_dst* dst, int32_t* fault, void* stream_) {
  if (!f || !src || !next || !dst || !fault) return DSBD_ERR_INVALID;
  if (W_cap < 1 || W_cap > 64) return DSBD_ERR_UNSUPPORTED;
  if (Hkv <= 0 || D <= 0 || D % 8 != 0) return DSBD_ERR_UNSUPPORTED;
  if (f->max_depth < 0 || f->max_depth >= DSBD_MAX_TREE_NODES) return DSBD_ERR_INVALID;
  if (f->n_prompts < 0 || f->n_trees < 0 || f->n_nodes < 0 || src->max_len < 0 || dst->capacity < 0) return DSBD_ERR_INVALID;
  if (src->token_stride % 8 != 0 || src->head_stride % 8 != 0) return DSBD_ERR_UNSUPPORTED;
  if (f->n_prompts == 0) return DSBD_OK;
  if (!src->k_ptr || !src->v_ptr || !src->len || !k_tree || !v_tree) return DSBD_ERR_INVALID;
  if (!next->n_next || !next->src_tree || !next->path_len || !next->path) return DSBD_ERR_INVALID;
  if (!dst->k_ptr || !dst->v_ptr || !dst->len) return DSBD_ERR_INVALID;
  if ((reinterpret_cast<uintptr_t>(k_tree) | reinterpret_cast<uintptr_t>(v_tree)) & 15) return DSBD_ERR_INVALID;
  CommitArgs a;
  a.n_prompts = f->n_prompts; a.n_trees = f->n_trees; a.n_nodes = f->n_nodes; a.W_cap = W_cap;
  a.plen = f->max_depth + 1; a.Hkv = Hkv; a.D = D;
  a.src_k = src->k_ptr; a.src_v = src->v_ptr; a.src_len = src->len;
  a.token_stride = src->token_stride; a.head_stride = src->head_stride;
  a.k_tree = static_cast<const __bf16*>(k_tree); a.v_tree = static_cast<const __bf16*>(v_tree);
  a.n_next = next->n_next; a.src_tree = next->src_tree; a.path_len = next->path_len; a.path = next->path;
  a.dst_k = dst->k_ptr; a.dst_v = dst->v_ptr; a.dst_len = dst->len; a.capacity = dst->capacity; a.max_len = src->max_len;
  a.fault = fault;
  const long long slots = (long long)f->n_prompts * W_cap;
  if (slots > 65535) return DSBD_ERR_UNSUPPORTED;
  a.tokens = (int)std::max(1LL, std::min((long long)CM_TOKENS, CM_LOADS * CM_BLOCK / ((long long)Hkv * (D / 8))));
  const long long chunks = std::min(std::max(1LL, ((long long)src->max_len + a.tokens - 1) / a.tokens), CM_CHUNKS);
  // a prompt's sources, and the units of its path rows, side by side where its chunks leave compute units idle
  const long long units = (long long)W_cap * ((a.plen + CM_PATH_TOKENS - 1) / CM_PATH_TOKENS);
  a.shares = (int)std::max(1LL, std::min(std::max((long long)W_cap, (units + chunks - 1) / chunks), CM_GRID / (chunks * 2 * f->n_prompts)));
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  dsbd_launch(DSBD_KERNEL_KV_COMMIT, commit_kv_kernel, dim3(2 * (unsigned)chunks, (unsigned)a.shares, (unsigned)f->n_prompts), dim3(CM_BLOCK), 0, stream, a);
  DSBD_HIP_LAUNCH_CHECK();
  return DSBD_OK;
}
