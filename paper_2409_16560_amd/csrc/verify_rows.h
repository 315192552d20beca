// What the layer walk needs of the logit rows when the joints are warped (top-k / top-p, paper Section 2.1): per row its
// maximum, the fp64 sum of its exponentials and its top_k first entries, all rows of a call side by side (verify_rows.hip).
#pragma once
#include "common.h"

#define VR_MAX_CHUNKS 128      // chunks per row: two per lane where they are folded
#define VR_WHOLE 4096          // rows of up to so many logits are read whole where their entries are selected
#define VR_K_MAX 32
#define VR_BARE 1024           // rows of up to so many logits can do with records of a sum alone

// A row's record: `sum` (of exp(z - max)), `max`, the number of entries (VR_ROW_BAD added where the row holds NaN or +Inf),
// then the entries (logit, token) by descending exp(logit - max) in fp64, equal ones by ascending token (logits around zero
// differ by less than that resolves); masked tokens (-Inf) are no entries.
#define VR_ROW_BAD 256
struct RowHead { double sum; float max; int n; };
struct RowEntry { float z; int x; };

struct RowsPlan {
  int chunk, nchunk;           // logits per chunk (a power of two), chunks per row
  int parts;                   // parts of a chunk whose maxima are kept (0: none; rows of up to VR_WHOLE logits)
  int compact;                 // > 0: the entries are tokens of so many bytes (1 or 2), whose logits are looked up again; < 0: a
                               // record is the row's sum alone (sign set: the row is bad), the layers select from the logits
  long long rec_stride;        // bytes from record to record
};
// Chunks depend on the row's length alone, so that equal rows are summed in the same order and get the same bits.
inline RowsPlan rows_plan(int V, int K, int compact) {
  RowsPlan r;
  long long c = 1024;
  while ((V + c - 1) / c > VR_MAX_CHUNKS) c *= 2;
  r.chunk = (int)c;
  r.nchunk = (int)((V + c - 1) / c);
  // parts so short that a row has more of them than entries are ever asked for, and no more than 256
  r.parts = V <= VR_WHOLE ? 0 : V <= 16384 ? 16 : V <= 65536 ? 4 : 2;
  r.compact = compact;
  const size_t entries = (size_t)(K < V ? K : V);
  r.rec_stride = compact < 0 ? (long long)sizeof(double) : compact ? (long long)dsbd_align_up(sizeof(RowHead) + entries * compact, 8)
                         : (long long)dsbd_align_up(sizeof(RowHead) + entries * sizeof(RowEntry), 16);
  return r;
}

struct RowsArgs {
  int n_nodes, V, K, chunk, nchunk, parts;
  int alias;                   // one model in both roles: one row per node, whose outputs serve both
  const float *zp, *zq;
  const int32_t *parent, *token;
  double2* part;               // [rows][nchunk]: maximum of the chunk, sum of exp(z - maximum), its sign set where the chunk holds NaN or
                               // +Inf; null (rows of one chunk): in the records (without the maximum where they hold a sum alone)
  float* sub;                  // [rows][nchunk * parts]: maxima of the chunk's parts
  char* rec;                   // [rows] records, `rec_stride` bytes apart
  int compact;
  long long rec_stride;
  float *lse_p, *lse_q, *logp_p, *logp_q;     // per-node outputs (any may be null)
  int report;                  // faults of all rows are reported here (some output is wanted); else the layers report the rows they use
  int32_t* fault;
  int direct;                  // candidates that are ranked directly (fewer: a test hook for the other form)
};
// Row 2 n + m of the records: model m's logits of node n (row n where one model has both roles).
hipError_t launch_verify_rows(const RowsArgs& a, hipStream_t stream);
