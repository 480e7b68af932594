// Declarations shared by the backward kernels' translation units (not installed).
#pragma once
#include "fcp_device.h"

namespace fcp {

struct BwdParams {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const uint16_t* d_o;
  const float* lse;
  const float* delta;
  const int32_t* q_limit;    // [tq] last key position each local query row sees, NULL = its own position (causal)
  const int32_t* k_from;     // [tkv] first query position that sees each pool key, NULL = its own position
  const float* stats;        // two planes [hq][tq]: -LSE * log2 e (-inf for a row without keys), then -delta
  SchedHeader* hdr;          // schedule region of the kernel being launched
  const Tile* tiles;
  float* dq;
  float* dk;
  float* dv;
  // Direct mode (all three set, or all NULL): a unit that owns its rows / keys in this launch (the scheduler's
  // exclusivity flags) writes its final bf16 result here; dq also carries the one-pass kernel's running sums.
  uint16_t* dq_out;
  uint16_t* dk_out;
  uint16_t* dv_out;
  // One-pass kernel: the chain record of every tile (kChainWords words: rank, first block of the next tile, flag base,
  // first block) and the flag words.
  const int32_t* chain;
  int32_t* flags;
  // Split tiles: turn words of the kernel's tiles (see wait_turn), and the word that counts waits which ran out.
  int32_t* turns;
  int32_t* n_stalled;
  // The query-tile list.
  SchedHeader* hdr_q;
  const Tile* tiles_q;
  int32_t* turns_q;
  int32_t tq, hq, hkv;
  int32_t either;            // the list decided which kernels work it (path word): the others of the launches have nothing to do
  float scale, scale_log2;
};

// The pieces of a split tile add to its rows one after the other, so that the sums do not depend on the run: each adding wave of a unit has a
// word per (tile, head) that counts the pieces whose same wave, with the same part of the rows, has added; that of piece n begins once the word stands at n.  The adds
// are atomics, performed when the memory has acknowledged them.  A piece only waits for pieces ahead of it in the list, which blocks take
// units from in order: the earliest unfinished unit never waits.  (One word for all waves, each turn as long as the slowest of
// them: 315 -> 400 us on one sequence of 4096 tokens, 8 query heads on one KV head.)
constexpr int kTurnPolls = 1 << 18;      // about half a second: a wait that does not end is given up (fcp_scratch_status reports it)
__device__ inline bool wait_turn(const int32_t* word, int piece) {
  for (int left = kTurnPolls; left > 0; --left) {
    const int32_t v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(v) >= piece) return true;
    __builtin_amdgcn_s_sleep(1);
  }
  return false;
}
__device__ inline void pass_turn(int32_t* word) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// dK / dV over key tiles and dQ over query tiles (csrc/fcp_attn_bwd_lists.hip).  `units` = upper bound of the units of both lists.
constexpr int lists_blocks_per_cu(int head_dim) { return head_dim == 64 ? 3 : 2; }
int launch_bwd_lists(const BwdParams& p, int head_dim, int head_pair, int64_t units, int n_cu, hipStream_t stream);

// dQ, dK and dV in one pass over key tiles, 128 channels per head: one block of twelve waves per CU (csrc/fcp_attn_bwd_fused.hip), or two of four
// for many short sequences (csrc/fcp_attn_bwd_short.hip).
int launch_bwd_fused(const BwdParams& p, int64_t units, int n_cu, hipStream_t stream);
int launch_bwd_short(const BwdParams& p, int64_t units, int n_cu, hipStream_t stream);

}  // namespace fcp
