// Work items as the device code uses them: validated, with the place of their keys in the pool (the scheduler, and attention kernels that find their
// units themselves).
#pragma once
#include "fcp_internal.h"

namespace fcp {

__device__ inline int32_t ceil_div(int32_t a, int32_t b) { return (a + b - 1) / b; }

// A work item as the scheduler uses it: validated, with the place of its keys in the pool.  Items are fetched once per block and kept in LDS: a list
// is built of many short dependent steps, and trips to global memory for descriptor, cu_seqlens and mask in each of them
// were most of its time.  (No arrays: indexed by a run-time segment number they would live in scratch memory.)
struct Item {
  int32_t seq;                      // -1: rejected
  int32_t q_off, q_len, q_pos;      // query rows: first local row, count, position of the first
  int32_t k0, n0, k1, n1;           // key segments: position of the first key, keys (n1 = 0: one segment)
  int32_t base;                     // pool row of the sequence's first key
  int32_t vis0, vis1;               // keys of the segment that the last row sees
  int32_t step;
  __device__ int32_t k(int s) const { return s ? k1 : k0; }
  __device__ int32_t n(int s) const { return s ? n1 : n0; }
  __device__ int32_t vis(int s) const { return s ? vis1 : vis0; }
};

// The mask in the form every kernel uses: row i sees the keys at positions 0 .. limit(i), a key is seen by the
// rows from position from(key) on; both grow with the position.  Causal: limit = the row's own position,
// from = the key's own position; with full-attention spans the tables the caller passed.
struct MaskTables {
  const int32_t* q_limit;   // [tq] by local query row, or NULL
  const int32_t* k_from;    // [tkv] by pool row, or NULL
  __device__ int64_t limit(const Item& it, int32_t row) const {
    return q_limit ? (int64_t)q_limit[it.q_off + row] : (int64_t)it.q_pos + row;
  }
  __device__ int64_t from(const Item& it, int64_t k_pos) const { return k_from ? (int64_t)k_from[it.base + k_pos] : k_pos; }
};

// keys of segment s that a row with that limit sees
__device__ inline int32_t seen_keys(const Item& it, int s, int64_t limit) {
  return (int32_t)max((int64_t)0, min((int64_t)it.n(s), limit - it.k(s) + 1));
}

struct ListArgs {                   // what a list is built from
  const fcp_work_desc* work;
  const int32_t* cu;
  int32_t n_work, n_seqs, tq, tkv, n_parts, max_seg_keys;
  bool check_step;
};
__device__ inline Item load_item(const ListArgs& a, const MaskTables& m, int32_t i) {
  const fcp_work_desc w = a.work[i];
  Item it{-1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  if (w.seq < 0 || w.seq >= a.n_seqs) return it;
  if (a.check_step && (w.step < 0 || w.step >= a.n_parts)) return it;
  if (w.q_len < 1 || w.q_local_off < 0 || w.q_seq_start < 0) return it;
  if ((int64_t)w.q_local_off + w.q_len > (int64_t)a.tq) return it;
  if ((int64_t)w.q_seq_start + w.q_len > (int64_t)(1 << 30)) return it;
  if (w.n_seg < 1 || w.n_seg > 2) return it;
  const int64_t s0 = a.cu[w.seq], s1 = a.cu[w.seq + 1];
  if (s0 < 0 || s1 < s0 || s1 > (int64_t)a.tkv) return it;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    if (s >= w.n_seg) continue;
    if (w.k_seq_start[s] < 0 || w.k_len[s] < 1 || w.k_len[s] > a.max_seg_keys) return it;
    if (s0 + (int64_t)w.k_seq_start[s] + w.k_len[s] > s1) return it;
  }
  const bool two = w.n_seg > 1;
  it = {w.seq, w.q_local_off, w.q_len, w.q_seq_start, w.k_seq_start[0], w.k_len[0], two ? w.k_seq_start[1] : 0, two ? w.k_len[1] : 0,
        (int32_t)s0, 0, 0, w.step};
  const int64_t limit = m.limit(it, it.q_len - 1);
  it.vis0 = seen_keys(it, 0, limit);
  it.vis1 = two ? seen_keys(it, 1, limit) : 0;
  return it;
}

}  // namespace fcp
