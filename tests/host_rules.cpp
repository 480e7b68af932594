// What csrc/fcp_sizes.h computes, for tests/host_rules.py.
#include "fcp_sizes.h"

extern "C" {
// out: tile rows, paired heads, list capacity, bytes of the list's region
void forward_plan(int head_dim, int hq, int hkv, int32_t tq, int32_t tkv, int64_t n_work, int32_t n_parts, int n_cu, int64_t area, int64_t* out) {
  const fcp::FwdPlan p = fcp::fwd_plan(head_dim, hq, hkv, tq, tkv, n_work, n_parts, n_cu, (size_t)area);
  out[0] = p.tile;
  out[1] = p.head_pair;
  out[2] = p.cap;
  out[3] = (int64_t)fcp::sched_region_bytes(n_work, p.cap);
}
int64_t static_bytes(int32_t tq, int32_t tkv, int64_t n_work, int32_t n_parts) { return (int64_t)fcp::fwd_static_bytes(tq, tkv, n_work, n_parts); }
int64_t scratch_area_bytes(int32_t tq, int32_t tkv, int64_t n_work, int32_t n_parts) { return (int64_t)fcp::fwd_area_bytes(tq, tkv, n_work, n_parts); }
int64_t bwd_kv_cap(int32_t tkv, int64_t n_work) { return fcp::bwd_kv_cap(tkv, n_work); }
int64_t bwd_q_cap(int32_t tq, int32_t tkv, int64_t n_work) { return fcp::bwd_q_cap(tq, tkv, n_work); }
int64_t persistent_blocks(int64_t resident, int64_t units) { return fcp::persistent_blocks(resident, units); }
void first_unit(int place, int places, int key_units, int n_long, int64_t* out) {
  const fcp::FirstUnit f = fcp::first_unit(place, places, key_units, n_long);
  out[0] = f.key_dealt;
  out[1] = f.key;
  out[2] = f.row;
}
int head_queues(int per_tile, int in_turn) { return fcp::head_queues(per_tile, in_turn != 0); }
void unit_numbers(int block, int queues, int in_turn, int64_t* out) {
  const fcp::UnitNumbers n = fcp::unit_numbers(block, queues, in_turn != 0);
  out[0] = n.counter;
  out[1] = n.mul;
  out[2] = n.add;
}
int deals_first(int units, int blocks, int per_block, int longest) { return fcp::deals_first(units, blocks, per_block, longest); }
int keeps_reserve(int dealt, int longest) { return fcp::keeps_reserve(dealt != 0, longest); }
int backward_way(int32_t hq, int32_t hkv, int32_t head_dim, int32_t tq, int32_t tkv, int64_t n_work, int n_cu) {
  const fcp::BwdWay w = fcp::bwd_way(hq, hkv, head_dim, tq, tkv, n_work, n_cu);
  return (w.one_pass ? 1 : 0) | (w.many_short ? 2 : 0) | (w.either ? 4 : 0);
}
int delta_streams_do(int32_t tq, int32_t hq, int32_t head_dim) { return fcp::delta_streams_do(tq, hq, head_dim); }
int alone_order(int form, int64_t n_work, int64_t units, int n_cu) { return fcp::alone_order((fcp::FwdForm)form, n_work, units, n_cu); }
int forward_alone(int form, int head_dim, int64_t n_work, int32_t n_parts, int64_t units, int n_cu) {
  return fcp::fwd_alone((fcp::FwdForm)form, head_dim, n_work, n_parts, units, n_cu);
}
}
