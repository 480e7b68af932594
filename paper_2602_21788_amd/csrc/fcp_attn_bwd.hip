// fcp_attn_bwd_step: gradient contributions of one CP rank for its ring steps.
//
// Backward of O = softmax(scale Q K^T) V (paper Eq. 1, Sec. 3.1; causal mask, Sec. 4.3) for
// the key sets the ring steps bring (ring-style CP, Sec. 3.2).  With the merged LSE the
// probabilities of a step are recomputed exactly, P = exp(scale s - LSE), so each step adds
// its own share:  dV += P^T dO,  dS = P o (dO V^T - delta),  dQ += scale dS K,  dK += scale dS^T Q.
//
// Entry points, checks and the launches of the way that bwd_way (csrc/fcp_sizes.h) chooses: key tiles and query tiles in one launch (csrc/fcp_attn_bwd_lists.hip),
// or one pass over key tiles for lists of short whole sequences (csrc/fcp_attn_bwd_fused.hip; many of them: csrc/fcp_attn_bwd_short.hip).
#include "fcp_bwd.h"

#include <algorithm>

using fcp::fail;

// Both entry points; q_limit == k_from == NULL is the causal mask.
static int bwd_step(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                    const float* delta, const int32_t* cu_seqlens_kv, int32_t n_seqs,
                    const fcp_work_desc* work, int64_t n_work, int32_t tq, int32_t tkv, int32_t hq,
                    int32_t hkv, int32_t head_dim, float softmax_scale, const int32_t* q_limit, const int32_t* k_from,
                    float* dq_acc, float* dk_acc, float* dv_acc, void* scratch, size_t scratch_bytes, void* stream,
                    void* dq_out = nullptr, void* dk_out = nullptr, void* dv_out = nullptr) {
  fcp::clear_error();
  if (!q || !k || !v || !d_o || !lse || !delta || !cu_seqlens_kv || !dq_acc || !dk_acc || !dv_acc || !scratch)
    return fail(FCP_ERR_INVALID_ARG, "fcp_attn_bwd_step: null pointer");
  const bool direct = dq_out != nullptr;
  if (n_work > 0 && !work) return fail(FCP_ERR_INVALID_ARG, "fcp_attn_bwd_step: work is NULL");
  if (tq < 0 || tkv < 1 || n_seqs < 1 || n_work < 0 || hq < 1 || hkv < 1)
    return fail(FCP_ERR_INVALID_ARG, "fcp_attn_bwd_step: bad sizes");
  if (n_work > (1 << 24)) return fail(FCP_ERR_UNSUPPORTED, "fcp_attn_bwd_step: more than 2^24 work items");
  if (hq % hkv != 0) return fail(FCP_ERR_UNSUPPORTED, "fcp_attn_bwd_step: hq %d not a multiple of hkv %d", hq, hkv);
  if (head_dim != 64 && head_dim != 128) return fail(FCP_ERR_UNSUPPORTED, "fcp_attn_bwd_step: head_dim %d not 64/128", head_dim);
  if (!(softmax_scale > 0.f) || !(softmax_scale < 1e30f)) return fail(FCP_ERR_INVALID_ARG, "fcp_attn_bwd_step: softmax_scale must be positive and finite");
  const uintptr_t align_mask = reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k) |
                               reinterpret_cast<uintptr_t>(v) | reinterpret_cast<uintptr_t>(d_o) |
                               reinterpret_cast<uintptr_t>(dq_acc) | reinterpret_cast<uintptr_t>(dk_acc) |
                               reinterpret_cast<uintptr_t>(dv_acc);
  if (align_mask & 15u) return fail(FCP_ERR_INVALID_ARG, "fcp_attn_bwd_step: tensors must be 16-byte aligned");
  if (reinterpret_cast<uintptr_t>(scratch) & 255u) return fail(FCP_ERR_INVALID_ARG, "fcp_attn_bwd_step: scratch must be 256-byte aligned");
  const size_t need = fcp_scratch_bytes(FCP_SCRATCH_BWD, tq, tkv, hq, hkv, head_dim, n_work, 1);
  if (scratch_bytes < need) return fail(FCP_ERR_CAPACITY, "fcp_attn_bwd_step: scratch %zu < %zu bytes", scratch_bytes, need);

  // The Q / dO rows of a work item are reached through one buffer resource with 32-bit byte offsets, which the fills
  // advance a few blocks past the item's end; an item has at most tq rows.  (The accumulators and outputs are reached
  // tile by tile, the pool segment by segment: the scheduler bounds a segment.)
  if ((int64_t)tq * hq * head_dim * 2 + ((int64_t)1 << 22) >= ((int64_t)1 << 31))
    return fail(FCP_ERR_UNSUPPORTED, "fcp_attn_bwd_step: tq * hq * head_dim must stay below 2^30 - 2^21 elements");
  hipStream_t st = (hipStream_t)stream;
  const int64_t cap_kv = fcp::bwd_kv_cap(tkv, n_work);
  const int64_t cap_q = fcp::bwd_q_cap(tq, tkv, n_work);
  if (cap_kv > INT32_MAX / 64 || cap_q > INT32_MAX / 64) return fail(FCP_ERR_UNSUPPORTED, "fcp_attn_bwd_step: too many tiles");
  void* region_kv = scratch;
  void* region_q = static_cast<char*>(scratch) + fcp::sched_region_bytes(n_work, cap_kv);
  float* stats = reinterpret_cast<float*>(static_cast<char*>(region_q) + fcp::sched_region_bytes(n_work, cap_q));
  if (direct) { const int rcs = fcp::check_row_states(n_work); if (rcs != FCP_OK) return rcs; }
  int dev = 0, n_cu = 0;                            // (arguments are refused without a device)
  FCP_HIP_CHECK(hipGetDevice(&dev));
  FCP_HIP_CHECK(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
  const int group = hq / hkv;
  const int64_t key_units = (int64_t)tkv * hkv / fcp::kBwdBN;
  const auto [fused, many_short, either] = fcp::bwd_way(hq, hkv, head_dim, tq, tkv, n_work, n_cu);
  // direct mode: where every row's result comes from (and the accumulator rows that are accumulated into cleared),
  // on extra blocks of the scheduling launch
  fcp::RowStates rs{};
  if (direct) {
    rs.q_state = fcp::bwd_q_state(scratch, n_work, tq, tkv, hq);
    rs.kv_state = fcp::bwd_kv_state(scratch, n_work, tq, tkv, hq);
    rs.dq_acc = dq_acc; rs.dk_acc = dk_acc; rs.dv_acc = dv_acc;
    rs.q_row_elems = hq * head_dim; rs.kv_row_elems = hkv * head_dim;
    rs.n_parts = 1; rs.check_step = false;
  }
  if (tq == 0 || n_work == 0) {     // nothing to add; the lists are still built so that the status call works
    if (direct) {
      const int rcs = fcp::launch_row_states((int64_t)hkv * head_dim * 2, rs, q_limit, k_from, work, n_work, cu_seqlens_kv,
                                             n_seqs, tq, tkv, st);
      if (rcs != FCP_OK) return rcs;
    }
    int rc0 = fcp::launch_schedule(true, fcp::kBwdBN, fcp::kBwdBM, (int64_t)hkv * head_dim * 2, q_limit, k_from, work, n_work, cu_seqlens_kv, n_seqs, tq, tkv, 1, cap_kv, region_kv, nullptr, 0, st);
    if (rc0 != FCP_OK) return rc0;
    return fcp::launch_schedule(false, fcp::kDqBM, fcp::kDqBN, (int64_t)hkv * head_dim * 2, q_limit, k_from, work, n_work, cu_seqlens_kv, n_seqs, tq, tkv, 1, cap_q, region_q, nullptr, 0, st);
  }
  // dQ units: 128 query rows for two heads of one KV head when the heads pair up, else 256 rows for one head
  const int head_pair = ((hq / hkv) % 2 == 0) ? 1 : 0;
  const int dq_rows = 2 * fcp::kDqBM >> head_pair;
  // Split tiles (see csrc/fcp_sched.hip): worth the scheduler's time where there are a few tiles per CU at most and a serial loop can be
  // long, in 32-row blocks of all heads of a KV head or in 32-key blocks.  In sharded lists a tile's loop is the shorter for
  // the sharding, and its accumulators are mostly shared already.  Measured, scheduling and attention launches, whole and split (with one kernel per list;
  // split_sizes in csrc/fcp_sched.hip has the estimate as fitted to one kernel for both): one sequence of 4096 tokens, 8 query
  // heads on one KV head, 128 channels 952 -> 296 us; 6 on 2, 64 channels 445 -> 175 us; 30 sequences of 20011 tokens in all, 6 on 2, 489 -> 357 us
  // whole and 316 -> 245 us with the longest one over 3 ranks; 4096 tokens over 3 ranks, 4 on 4, 106 -> 86 us; 4096 tokens, 32 on 8, 609 -> 575 us.
  // (At the edge the estimate can miss: 9000 tokens over 4 ranks, 12 on 4, 128 channels 367 -> 375 us.)
  const int64_t longest = std::max((int64_t)tq * group / fcp::kBwdBM, (int64_t)tkv / fcp::kDqBN);
  const bool split = (!fused || either) && key_units <= 1024 && n_work <= 1024 && longest >= (tq == tkv ? 24 : 64);
  const fcp::SplitTiles sp{group, hkv, hq / (head_pair ? 2 : 1), n_cu, 12,         // (12 steps at least)
                           (int32_t)fcp::key_turns(tkv, n_work), (int32_t)fcp::row_turns(tq, n_work), fcp::lists_blocks_per_cu(head_dim), split, many_short};
  int32_t* const turns = fcp::bwd_turns(scratch, n_work, tq, tkv, hq);
  int32_t* const flags = fcp::bwd_chain_flags(scratch, n_work, tq, tkv, hq, hkv);
  const int64_t n_flags = fused ? fcp::chain_flag_words(tq, hq, n_work) : 0;
  int32_t* const clear = split ? turns : flags;
  const int64_t n_clear = !split ? n_flags : !fused ? fcp::turn_words(tq, tkv, hq, hkv, n_work) : flags - turns + n_flags;
  int rc = fcp::launch_schedule_bwd((int64_t)hkv * head_dim * 2, q_limit, k_from, work, n_work, cu_seqlens_kv, n_seqs, tq, tkv,
                                    cap_kv, region_kv, dq_rows, cap_q, region_q, lse, delta, (int64_t)hq * tq, stats, st,
                                    direct ? &rs : nullptr, fused ? fcp::bwd_chain(scratch, n_work, tq, tkv, hq, hkv) : nullptr, clear, n_clear, &sp, either);
  if (rc != FCP_OK) return rc;

  fcp::BwdParams p{};
  p.q = (const uint16_t*)q; p.k = (const uint16_t*)k; p.v = (const uint16_t*)v; p.d_o = (const uint16_t*)d_o;
  p.lse = lse; p.delta = delta; p.stats = stats;
  p.q_limit = q_limit; p.k_from = k_from;
  p.dq = dq_acc; p.dk = dk_acc; p.dv = dv_acc;
  p.dq_out = (uint16_t*)dq_out; p.dk_out = (uint16_t*)dk_out; p.dv_out = (uint16_t*)dv_out;
  p.tq = tq; p.hq = hq; p.hkv = hkv;
  p.scale = softmax_scale; p.scale_log2 = softmax_scale * fcp::kLog2e;

  p.either = either;
  if (fused) {
    p.chain = fcp::bwd_chain(scratch, n_work, tq, tkv, hq, hkv);
    p.flags = flags;
    p.hdr = (fcp::SchedHeader*)region_kv;
    p.tiles = fcp::sched_tiles(region_kv, n_work);
    const int64_t units = fcp::kv_tile_cap(tkv, n_work) * hkv;      // (more units, of keys shared by many items: the blocks take them in turn)
    rc = many_short ? fcp::launch_bwd_short(p, units, n_cu, st) : fcp::launch_bwd_fused(p, units, n_cu, st);
    if (rc != FCP_OK || !either) return rc;
  }
  // both lists
  p.turns = turns;
  p.turns_q = turns + fcp::key_turns(tkv, n_work) * hkv * fcp::kTurnWaves;
  p.n_stalled = &((fcp::SchedHeader*)region_kv)->n_stalled;
  p.hdr = (fcp::SchedHeader*)region_kv;
  p.tiles = fcp::sched_tiles(region_kv, n_work);
  p.hdr_q = (fcp::SchedHeader*)region_q;
  p.tiles_q = fcp::sched_tiles(region_q, n_work);
  const double pieces = split ? (double)tq * tkv * hq / sp.min_steps : 0.;      // bounds of the units that splitting adds, times a step's pairs
  const int64_t units = fcp::kv_tile_cap(tkv, n_work) * hkv + (int64_t)(pieces / (fcp::kBwdBM * fcp::kBwdBN)) +
                        2 * (fcp::q_tile_cap(tq, tkv, n_work, 1 << 20, dq_rows) * (hq / (head_pair ? 2 : 1)) + (int64_t)(pieces / (2 * fcp::kDqBM * fcp::kDqBN)));
  return fcp::launch_bwd_lists(p, head_dim, head_pair, units, n_cu, st);
}

extern "C" int fcp_attn_bwd_step(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                                 const float* delta, const int32_t* cu_seqlens_kv, int32_t n_seqs,
                                 const fcp_work_desc* work, int64_t n_work, int32_t tq, int32_t tkv, int32_t hq,
                                 int32_t hkv, int32_t head_dim, float softmax_scale, float* dq_acc, float* dk_acc,
                                 float* dv_acc, void* scratch, size_t scratch_bytes, void* stream) {
  return bwd_step(q, k, v, d_o, lse, delta, cu_seqlens_kv, n_seqs, work, n_work, tq, tkv, hq, hkv, head_dim,
                  softmax_scale, nullptr, nullptr, dq_acc, dk_acc, dv_acc, scratch, scratch_bytes, stream);
}

extern "C" int fcp_attn_bwd_step_mixed(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                                       const float* delta, const int32_t* cu_seqlens_kv, int32_t n_seqs,
                                       const fcp_work_desc* work, int64_t n_work, int32_t tq, int32_t tkv, int32_t hq,
                                       int32_t hkv, int32_t head_dim, float softmax_scale, const int32_t* q_limit,
                                       const int32_t* k_from, float* dq_acc, float* dk_acc, float* dv_acc,
                                       void* scratch, size_t scratch_bytes, void* stream) {
  if (!q_limit || !k_from) {
    fcp::clear_error();
    return fail(FCP_ERR_INVALID_ARG, "fcp_attn_bwd_step_mixed: q_limit or k_from is NULL");
  }
  return bwd_step(q, k, v, d_o, lse, delta, cu_seqlens_kv, n_seqs, work, n_work, tq, tkv, hq, hkv, head_dim,
                  softmax_scale, q_limit, k_from, dq_acc, dk_acc, dv_acc, scratch, scratch_bytes, stream);
}

extern "C" int fcp_attn_bwd_step_direct(const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                                        const float* delta, const int32_t* cu_seqlens_kv, int32_t n_seqs,
                                        const fcp_work_desc* work, int64_t n_work, int32_t tq, int32_t tkv, int32_t hq,
                                        int32_t hkv, int32_t head_dim, float softmax_scale, const int32_t* q_limit,
                                        const int32_t* k_from, float* dq_acc, float* dk_acc, float* dv_acc, void* dq_out,
                                        void* dk_out, void* dv_out, void* scratch, size_t scratch_bytes, void* stream) {
  fcp::clear_error();
  if (!dq_out || !dk_out || !dv_out) return fail(FCP_ERR_INVALID_ARG, "fcp_attn_bwd_step_direct: output pointer is NULL");
  if ((q_limit == nullptr) != (k_from == nullptr))
    return fail(FCP_ERR_INVALID_ARG, "fcp_attn_bwd_step_direct: q_limit and k_from go together");
  if ((reinterpret_cast<uintptr_t>(dq_out) | reinterpret_cast<uintptr_t>(dk_out) | reinterpret_cast<uintptr_t>(dv_out)) & 15u)
    return fail(FCP_ERR_INVALID_ARG, "fcp_attn_bwd_step_direct: outputs must be 16-byte aligned");
  return bwd_step(q, k, v, d_o, lse, delta, cu_seqlens_kv, n_seqs, work, n_work, tq, tkv, hq, hkv, head_dim,
                  softmax_scale, q_limit, k_from, dq_acc, dk_acc, dv_acc, scratch, scratch_bytes, stream, dq_out, dk_out,
                  dv_out);
}
