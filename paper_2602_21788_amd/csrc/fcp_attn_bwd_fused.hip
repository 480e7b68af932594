// dQ, dK and dV in one pass over key tiles: the backward kernel of lists of whole, mostly short sequences with 128 channels per head.
//
// Same function as the kernel that works two lists (csrc/fcp_attn_bwd_lists.hip), which forms S and dP twice: seven contractions
// where the mathematics has five, two sets of units that each begin by waiting for their first rows, and Q, dO, K and V read
// twice.  On sequences of one or two key tiles those beginnings are most of the time.  One pass needs the dQ contributions of the key
// tiles added up cheaply.  fp32 atomics cannot do that (about one element per L2 channel and clock); plain loads
// and stores through the L2 of ONE XCD can:
//   * all units (key tile, KV head) of a KV head are taken by blocks of the same XCD (the queue is chosen by the block's
//     own XCC_ID), so dQ rows travel between them through that XCD's L2 and nothing has to be written back or
//     invalidated; loads bypass the CU's vector cache (sc1);
//   * the tiles of an item add to a 32-row block of dQ in a fixed order, their `rank` in the item.  A flag word per (block, head, half
//     of the rows, 32-channel slice) counts the contributions made; a unit waits until it equals its rank, loads, adds,
//     stores, waits for the stores to arrive and sets it to rank + 1.  The order is that of the tile list, from which the blocks take
//     units in order, so a unit only ever waits for units that were taken earlier: the earliest unfinished unit
//     never waits, hence no deadlock, and the sum does not depend on the run;
//   * the first contribution loads nothing, and in direct mode the last one (no later tile reaches the block) writes the
//     final bf16 rows: the dQ of a short sequence needs neither clearing nor a second pass through memory.
// Items that share query rows with others have no chain (rank -1), their tiles add with atomics.
//
// A block is 768 threads = 12 waves, three per SIMD, 168 registers each.  A step is one 32-row query block of one head
// against the unit's 128 keys.  Per SIMD:
//   score wave   for its 32 keys S = Q K^T, P = exp2(..), dP - delta = dO V^T, dS = P o (dP - delta), P and dS left in LDS as bf16.  K and V
//                fragments in registers; S is formed a step ahead, so that the exponentials need nothing but registers when a
//                step begins and dS is formed in the shadow of the next S.  Also fills the Q / dO stages;
//   dV wave      dV += P^T dO two steps behind, 64 keys x 64 channels, operands requested from LDS an iteration ahead so that its matrix
//                instructions start right after the barrier;   dK wave: dK += dS^T Q likewise;
//                both also dQ of the step before, for 16 of its rows and a slice of 32 channels: K^T fragments in registers, dS read back
//                transposed (the query on the lane), and the way of these rows through L2.
// One barrier per step.  A step takes about 2800 clocks with the matrix units busy for 46 % of them: what bounds it is the
// longest program of the three waves (a wave issues one instruction in about five clocks, an LDS read under this load answers after 500).
// Other splits of the work were slower: dQ by one of two kinds of waves in turn (every other step too long for the barrier that
// ends it), 8 waves of 256 registers (370 instructions each), dQ on 32 x 32 x 16 instructions with dQ in flight in registers.
//
// Measured against the two lists, scheduling and attention launches: 32 query heads on 8 KV heads, 200 sequences of 60 tokens on average 169 -> 159 us;
// 8 heads on 8, 30 of 100 43 -> 41 us, 200 of 60 89 -> 83; on one sequence of 4096 tokens 167 -> 211 us (units wait for each other at the shared rows
// and the stores of dQ compete for the L2): the rule of dispatch is bwd_way in csrc/fcp_sizes.h.
#include "fcp_bwd.h"

namespace fcp {
namespace {

template <int D>
struct FusedCfg {
  static constexpr int BM = kBwdBM;                // 32 query rows per step
  static constexpr int BN = kBwdBN;                // 128 keys per unit
  using DT = DualTile<D>;
  static constexpr int TILE = DT::bytes(BM);       // one Q or dO block
  static constexpr int SLOT = 256;                 // one statistics plane of a step: 64 floats (32 used)
  static constexpr int STAGE = 2 * TILE + 2 * SLOT;
  static constexpr int FILL_AHEAD = 3;
  static constexpr int NSTAGE = 2 + FILL_AHEAD;    // one step behind, the step itself, FILL_AHEAD ahead
  static constexpr int PB = 32 * 32 * 2;           // P or dS of one key group, bf16
  static constexpr int XGROUP = 4 * PB;            // P and dS, double-buffered by step parity
  static constexpr int XOFF = NSTAGE * STAGE;      // hand-over buffers; the K tile at the start of a unit
  static constexpr int OOFF = XOFF + 4 * XGROUP;   // what a part of a dQ block holds so far: per accumulating wave 2 KB by step parity
  static constexpr int LDS_BYTES = OOFF + 8 * 4096;
  static constexpr int NS = D / 16;                // matrix instructions of one 32 x 32 block of S or dP
  static constexpr int NVA = D / 64;               // 32-channel blocks per accumulating wave (half of the channels)
  static constexpr int kAhead = 4;                 // LDS fragments requested this many matrix instructions ahead
  static constexpr int DRAIN = 2;                  // iterations after the last step's contraction
  static_assert(D == 128, "four 32-channel slices of dQ, one per SIMD");
  static_assert(4 * XGROUP >= DT::bytes(BN) && 2 * STAGE >= DT::bytes(BN), "the K and V tiles pass through these areas at the start of a unit");
  static_assert(STAGE % 256 == 0 && TILE % 256 == 0 && XOFF % 256 == 0, "the address permutations stay below bit 8");
  static_assert(LDS_BYTES <= 160 * 1024 - 512, "LDS");
};

__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N>
__device__ inline void wait_vmem() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

constexpr int kCacheBypass = 16;   // sc1: the load goes past the CU's vector cache, which may hold what the line was when this CU last read it
// Two wave-wide LDS-direct loads of 16 bytes per lane (see lds_fill_b128), 1 KB apart in LDS and `step` bytes apart in memory; v0, v1 = lane offsets.
template <bool Bypass>
__device__ inline void lds_fill_x2(i32x4 r, uint32_t lds, int v0, int v1, int soff, int step) {
  int so;
  if constexpr (Bypass)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 3\n\tbuffer_load_dwordx4 %2, %4, %5 offen sc1 lds\n\t"
                 "s_add_u32 m0, m0, 0x400\n\ts_add_u32 %0, %5, %6\n\ts_nop 0\n\tbuffer_load_dwordx4 %3, %4, %0 offen sc1 lds"
                 : "=&s"(so) : "s"(lds), "v"(v0), "v"(v1), "s"(r), "s"(soff), "s"(step) : "memory", "scc");
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 3\n\tbuffer_load_dwordx4 %2, %4, %5 offen lds\n\t"
                 "s_add_u32 m0, m0, 0x400\n\ts_add_u32 %0, %5, %6\n\ts_nop 0\n\tbuffer_load_dwordx4 %3, %4, %0 offen lds"
                 : "=&s"(so) : "s"(lds), "v"(v0), "v"(v1), "s"(r), "s"(soff), "s"(step) : "memory", "scc");
}
// The kernel's arguments, read again: a role's unit loop holds those that it needs in a unit, not all of them across everything.
__device__ inline BwdParams args_again() {
  struct Words { uint64_t w[sizeof(BwdParams) / 8]; } r;
  auto a = (const __attribute__((address_space(4))) uint64_t*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  for (int i = 0; i < (int)(sizeof(BwdParams) / 8); ++i) r.w[i] = a[i];
  return __builtin_bit_cast(BwdParams, r);
}
constexpr int kClaimed = 1 << 30;      // counter of a claimed queue: past every unit; the claiming XCD from bit kClaimShift on (home blocks count below it)
constexpr int kClaimShift = 24;
constexpr int kClaimPolls = 16;
constexpr int kSpinLimit = 1 << 18;    // polls of a wave per unit, about half a second: a chain that cannot go on ends, its rows become NaN and the
                                       // header says so

// A unit as every role sees it.
struct FusedUnit {
  KTile t;
  int rank, qb_next, flag_base;   // place in the chain (-1: atomics), first block that a later tile reaches, first flag block
  int qb0, nqb, n_iter;           // first query block, blocks per head, steps
  int kvh;
  bool exclusive;
  __device__ int pick(const int32_t (&a)[4], int grp) const { return grp == 0 ? a[0] : grp == 1 ? a[1] : grp == 2 ? a[2] : a[3]; }
  // a key group takes part in the blocks from first_active on and needs no mask from first_unmasked on (blocks from qb0)
  __device__ int first_active(int grp) const {
    const int thr = pick(t.from_first, grp) - t.q_seq_start;
    if (32 * grp >= t.n_keys || thr > t.q_len - 1) return nqb;
    return max(0, (max(thr, 0) >> 5) - qb0);
  }
  __device__ int first_unmasked(int grp) const {
    if (32 * grp + 32 > t.n_keys) return nqb;
    const int thr = pick(t.from_last, grp) - t.q_seq_start;
    return max(0, ((max(thr, 0) + 31) >> 5) - qb0);
  }
};

template <int D>
__global__ __launch_bounds__(768, 1) void bwd_fused_kernel(const BwdParams p0) {
  using C = FusedCfg<D>;
  using DT = typename C::DT;
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  __shared__ int32_t s_next_unit;
  __shared__ int32_t s_queue[2];                   // queue that units are taken from; this block's XCD
  __shared__ int32_t s_rec[20];                    // tile record, then chain record

  const BwdParams& p = p0;
  if (p.either && !(p.hdr->path & kPathOnePass)) return;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int role = wave >> 2;                      // 0: score wave, 1: dV, 2: dK
  const int pw = wave & 3;                         // SIMD: key group of a score wave; (key half, channel half) and dQ slice of an accumulating one
  const int G = p.hq / p.hkv;
  const uint32_t lds0 = lds_offset(smem);
  // the queue of the XCD this block really runs on: see the head of the file
  if (tid == 0) s_queue[0] = s_queue[1] = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & (kNumXcd - 1);   // HW_REG_XCC_ID, bits 3:0
  const int kvh_here = p.hkv / kNumXcd;
  const int n_units = p.hdr->n_tiles * kvh_here;

  // Units are taken one at a time, when the block is about to need one: a unit that a block holds in reserve would
  // hold up the units after it in its chains.
  auto publish = [&](int unit) {
    const int lane = lane_id();
    if (unit < n_units) {
      const int64_t tile = unit / kvh_here;
      if (lane < 16) s_rec[lane] = reinterpret_cast<const int32_t*>(p.tiles)[tile * 16 + lane];
      else if (lane < 20) s_rec[lane] = p.chain[tile * kChainWords + lane - 16];
    }
    if (lane == 0) s_next_unit = unit;
  };
  auto take_unit = [&]() {
    const int home = __builtin_amdgcn_readfirstlane(s_queue[1]), q = __builtin_amdgcn_readfirstlane(s_queue[0]);
    int32_t v0 = 0;
    if (lane_id() == 0) v0 = atomicAdd(q == home ? &p.hdr->counter[q] : &p.hdr->claimed[q], 1);
    publish(__builtin_amdgcn_readfirstlane(v0));
  };
  // Blocks are dealt to the XCDs in turn, so every queue has its blocks.  An XCD that has begun nothing while a block of another one
  // has run out of units is late (its CUs are held by something else) or got no block: after a few polls (about 30 us) its
  // queue is claimed as a whole for the XCD of that block, and all blocks of that XCD which run out work it off together.  None of them
  // leaves before the last claim: a block leaves when every queue is begun.
  auto take_elsewhere = [&]() {
    const int home = __builtin_amdgcn_readfirstlane(s_queue[1]);
    int unit = __builtin_amdgcn_readfirstlane(s_next_unit);
    if (unit < n_units || n_units == 0) return;
    const int lane = lane_id();
    for (int polls = 0;; ++polls) {
      int32_t c = 1;
      if (lane < kNumXcd) c = __hip_atomic_load(&p.hdr->counter[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      uint64_t ours = __builtin_amdgcn_ballot_w64(c >= kClaimed && (c - kClaimed) >> kClaimShift == home);
      const uint64_t idle = __builtin_amdgcn_ballot_w64(c == 0);
      if (idle && polls >= kClaimPolls) {
        const int q = __builtin_ctzll(idle);
        int32_t old = 0;
        if (lane == 0) old = atomicCAS(&p.hdr->counter[q], 0, kClaimed + (home << kClaimShift));
        if (__builtin_amdgcn_readfirstlane(old) == 0) ours |= (uint64_t)1 << q;
      }
      for (; ours && unit >= n_units; ours &= ours - 1) {
        const int q = __builtin_ctzll(ours);
        int32_t v = 0;
        if (lane == 0) v = atomicAdd(&p.hdr->claimed[q], 1);
        unit = __builtin_amdgcn_readfirstlane(v);
        if (lane == 0) s_queue[0] = q;
      }
      if (unit < n_units || !idle) break;
      __builtin_amdgcn_s_sleep(32);
    }
    publish(unit);
  };
  if (wave == 0) { take_unit(); take_elsewhere(); }
  __syncthreads();
  auto next_unit = [&](FusedUnit& u) {
    const int unit = __builtin_amdgcn_readfirstlane(s_next_unit);
    if (unit >= n_units) return false;
    u.t = read_record<KTile, 15>(s_rec);
    u.rank = __builtin_amdgcn_readfirstlane(s_rec[16]);
    u.qb_next = __builtin_amdgcn_readfirstlane(s_rec[17]);
    u.flag_base = __builtin_amdgcn_readfirstlane(s_rec[18]);
    u.qb0 = __builtin_amdgcn_readfirstlane(s_rec[19]);
    u.nqb = (u.t.q_len + C::BM - 1) / C::BM - u.qb0;
    u.n_iter = u.nqb * G;
    u.kvh = __builtin_amdgcn_readfirstlane(s_queue[0]) * kvh_here + unit % kvh_here;
    u.exclusive = (u.t.flags & kFlagSeg0Exclusive) != 0;
    return true;
  };
  const int q_row_bytes = p.hq * D * 2;
  const int kv_row_bytes = p.hkv * D * 2;

  // The roles run the unit loop each for itself, so that none holds registers for another's values; they meet at the same
  // barriers: one when the K tile has landed, one per iteration (n_iter + DRAIN of them), one at the end of a unit.  Step s = (query
  // head s / nqb of the KV head, query block nqb - 1 - s % nqb from qb0 on).  In iteration `it`
  //   a score wave forms P(it), dP(it), dS(it), S(it + 1) and fills step it + FILL_AHEAD,
  //   an accumulating wave adds step it - 2 to dV or dK (operands requested in the iteration before) and step it - 1 to dQ.
  FusedUnit u;
  if (role == 0) {
    __builtin_amdgcn_s_setprio(2);
    const bool fill_is_do = pw >= 2;                // fill duty: sixteen rows of Q or dO, four instructions; waves 0 and 1 a statistics plane each
    const int fill_row0 = 16 * (pw & 1);
    while (next_unit(u)) {
      const BwdParams p = args_again();
      const int lane = lane_id();                   // per-lane values are formed here, not ahead of the unit loop (registers)
      const int l32 = lane & 31, g2 = lane >> 5;
      const int n_keys = u.t.n_keys, n_iter = u.n_iter;
      // ---- fills: instruction i covers rows fill_row0 + 4 i + lane / 16 (its chunk permutation differs by i)
      const int tfill = (fill_row0 + lane / DT::CPR) * q_row_bytes + (((lane % DT::CPR) ^ DT::key(lane / DT::CPR)) << 4);
      int f_head = u.kvh * G, f_left = u.nqb, f_heads_left = G;
      const int f_row0 = (u.qb0 + u.nqb - 1) * C::BM;
      int f_soff = f_row0 * q_row_bytes, f_ssoff = f_row0 * 4;
      const uint32_t f_dst0 = lds0 + (fill_is_do ? C::TILE : 0) + DT::row_base(fill_row0);
      uint32_t f_dst = f_dst0;
      i32x4 f_r, f_rs;
      auto f_resources = [&](bool live) {
        f_r = buffer_rsrc((fill_is_do ? p.d_o : p.q) + ((int64_t)u.t.q_local_off * p.hq + f_head) * D,
                          live ? (u.t.q_len - 1) * q_row_bytes + D * 2 : 0);
        f_rs = buffer_rsrc(p.stats + ((int64_t)(pw & 1) * p.hq + f_head) * p.tq + u.t.q_local_off, live ? u.t.q_len * 4 : 0);
      };
      f_resources(true);
      auto fill_next = [&]() {
        if (f_left == 0) {
          --f_heads_left;
          ++f_head;
          f_left = u.nqb;
          f_soff = f_row0 * q_row_bytes;
          f_ssoff = f_row0 * 4;
          f_resources(f_heads_left > 0);
        }
        const int tf = fresh(tfill);
        lds_fill_x2<false>(f_r, f_dst, tf, tf ^ 16, f_soff, 4 * q_row_bytes);
        lds_fill_x2<false>(f_r, f_dst + 2048, tf ^ 32, tf ^ 48, f_soff + 8 * q_row_bytes, 4 * q_row_bytes);
        if (fresh_uniform(pw) < 2) lds_fill_b32(f_rs, f_dst + (2 * C::TILE - DT::row_base(fill_row0)) + pw * C::SLOT, 4 * lane, f_ssoff);
        --f_left;
        f_soff -= C::BM * q_row_bytes;
        f_ssoff -= C::BM * 4;
        f_dst += C::STAGE;
        if (f_dst == f_dst0 + C::NSTAGE * C::STAGE) f_dst = f_dst0;
      };
#pragma unroll
      for (int a = 0; a < C::FILL_AHEAD; ++a) fill_next();
      const int my_key = 32 * pw + l32;
      int my_key_from = u.t.k_pos0 + my_key;        // position of the first query that sees the lane's key
      if (p.k_from) my_key_from = p.k_from[(int64_t)u.t.kv_row0 + min(my_key, n_keys - 1)];
      asm volatile("s_waitcnt vmcnt(0)" : "+v"(my_key_from) :: "memory");
      my_key_from = (my_key < n_keys ? my_key_from : INT32_MAX) - 4 * g2;
      lds_barrier();                                // the K and V tiles (loaded by the accumulating waves) and the first steps have landed

      const int row0 = tile_off<DT>(l32, g2);       // row fragment ks (A or B operand: row l32, channels 16 ks + 8 g2 ..) at row0 ^ (ks << 5)
      auto rows = [&](int at, int ks) { return *reinterpret_cast<const bf16x8*>(smem + (at ^ (ks << 5))); };
      bf16x8 kf[C::NS], vf[C::NS];
#pragma unroll
      for (int ks = 0; ks < C::NS; ++ks) {
        kf[ks] = rows(C::XOFF + 32 * pw * 2 * D + row0, ks);
        vf[ks] = rows(3 * C::STAGE + 32 * pw * 2 * D + row0, ks);
      }
      // Where the wave leaves P and dS of a step: 16 bytes per lane = key l32, rows 16 t + 4 g2 + [0,4) and 16 t + 8 + 4 g2 + [0,4) (t = 0, 1).
      // In dS the key is permuted so that the transposed reads of four keys x sixteen rows (dQ) fall into different banks.
      const int x_p = C::XOFF + pw * C::XGROUP;     // + 16 lane
      const int j_act = u.first_active(pw), j_unmasked = u.first_unmasked(pw);

      f32x16 sacc = {};                             // S of step `it` at the top of iteration `it`
      int j = 0, st = (C::NSTAGE - 1) * C::STAGE;   // block and stage of step `it`
      for (int it = -1; it < n_iter + C::DRAIN; ++it) {
        // iteration -1 only forms S(0); its barrier is the one above
        if (it >= 0) {
          wait_vmem<4>();                           // all fills but the newest step's
          lds_barrier();
        }
        int st1 = st + C::STAGE;                    // stage and block of step it + 1
        if (st1 == C::NSTAGE * C::STAGE) st1 = 0;
        const int j1 = j == 0 ? u.nqb - 1 : j - 1;
        const bool act = it >= 0 && it < n_iter && j >= j_act;
        const bool act1 = it + 1 < n_iter && j1 >= j_act;
        constexpr int A = C::kAhead;
        bf16x8 fr[C::NS];
        const int at = st + C::TILE + row0;
        f32x16 pr = {}, dp = {};
        f32x4 nl[4];                                // register i of S is block row 8 (i/4) + 4 g2 + i%4
        bf16x8 pb[2], dsb[2];
        const float* const stat = reinterpret_cast<const float*>(smem + st + 2 * C::TILE) + 4 * g2;
        if (act) {
#pragma unroll
          for (int q = 0; q < 4; ++q) nl[q] = *reinterpret_cast<const f32x4*>(stat + 8 * q);
        }
        // The masked variants: the causal edge and the keys past the tile's last (always masked).  Rows past the item's last need no mask:
        // their dO and statistics arrive as zeros, so P = 1 meets zeros in dV and dS.  A masked pair is selected away, not multiplied by zero:
        // a row must not see what a key after it holds, an infinity or a NaN included.
        const bool masked = act && j < j_unmasked;
        auto clear_masked = [&](f32x16& x) {
          const int q_pos0 = u.t.q_seq_start + (u.qb0 + j) * C::BM;
          int lo = my_key_from - q_pos0;            // register i is masked below it
          asm volatile("; masked variant" : "+v"(lo));
#pragma unroll
          for (int i = 0; i < 16; ++i) x[i] = 8 * (i / 4) + (i % 4) < lo ? 0.f : x[i];
        };
        auto ds_pair = [&](int x) {
#pragma unroll
          for (int i = 2 * x; i < 2 * x + 2; ++i) dsb[i / 8][i % 8] = (__bf16)(pr[i] * dp[i]);
        };
        // ---- P(it), dP(it)
        if (act) {
#pragma unroll
          for (int x = 0; x < A; ++x) fr[x] = rows(at, x);
#pragma unroll
          for (int i = 0; i < 16; ++i) pr[i] = __builtin_amdgcn_exp2f(fmaf(sacc[i], p.scale_log2, nl[i / 4][i % 4]));
          if (masked) clear_masked(pr);
#pragma unroll
          for (int i = 0; i < 16; ++i) pb[i / 8][i % 8] = (__bf16)pr[i];
#pragma unroll
          for (int q = 0; q < 2; ++q) *reinterpret_cast<bf16x8*>(smem + fresh(lane) * 16 + (x_p + (it & 1) * C::PB) + q * 1024) = pb[q];
#pragma unroll
          for (int q = 0; q < 4; ++q) {             // the accumulator starts at -delta of its rows
            const f32x4 nd = *reinterpret_cast<const f32x4*>(stat + C::SLOT / 4 + 8 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) dp[4 * q + e] = nd[e];
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int x = 0; x < C::NS; ++x) {
            dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[x], vf[x], dp, 0, 0, 0);
            if (x + A < C::NS) fr[x + A] = rows(at, x + A);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (it >= 0) fill_next();
        // ---- S(it + 1) with dS(it)
        if (act1) {
          const int at1 = st1 + row0;
#pragma unroll
          for (int x = 0; x < A; ++x) fr[x] = rows(at1, x);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int x = 0; x < C::NS; ++x) {
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[x], kf[x], x == 0 ? zero16() : sacc, 0, 0, 0);
            if (x + A < C::NS) fr[x + A] = rows(at1, x + A);
            // (dP has arrived by now; right after its own instructions the selection costs 3 % on 1000 sequences of 128 tokens)
            if (x == 1 && masked) clear_masked(dp);
            if (x == 2) ds_pair(0);
            if (x >= 2) ds_pair(x - 1);
            if (x == 7) ds_pair(7);
            __builtin_amdgcn_sched_barrier(0);
          }
        } else if (act) {
          if (masked) clear_masked(dp);
#pragma unroll
          for (int x = 0; x < C::NS; ++x) ds_pair(x);
        }
        if (act) {
          const int l = fresh(lane), dl = (l * 16) ^ ((l & 32) << 2);   // chunk t at (dl ^ (t << 6)) + t * 1024
#pragma unroll
          for (int q = 0; q < 2; ++q) *reinterpret_cast<bf16x8*>(smem + (dl ^ (q << 6)) + (x_p + 2 * C::PB + (it & 1) * C::PB) + q * 1024) = dsb[q];
        }
        if (wave == 0 && it == n_iter) take_unit(); // the next unit, while the accumulating waves finish this one
        st = st1;
        j = j1;
      }
      if (wave == 0) take_elsewhere();              // (rare; here, where the unit's registers are free)
      wait_vmem<0>();                               // the fills past the last step (zeros) have landed: the next unit's V tile passes through their stages
      lds_barrier();                                // the LDS is free for the next unit
    }
  } else {
    // Accumulating waves: 64 keys (key groups 2 kp, 2 kp + 1) x 64 channels (half ch) of dV (m = 0) or dK (m = 1), and dQ of the rows 16 m .. 16 m + 15
    // of every block, channels 32 pw .. 32 pw + 31.
    const int kp = pw >> 1, ch = pw & 1, m = role - 1;
    const int dq_row_bytes = p.hq * D * 4;
    while (next_unit(u)) {
      const BwdParams p = args_again();
      const int lane = lane_id();
      const int l32 = lane & 31, g2 = lane >> 5;
      const int n_keys = u.t.n_keys, n_iter = u.n_iter;
      const int64_t kv_row0 = u.t.kv_row0;
      // The unit's K (dK waves) and V (dV waves) rows come in whole, 32 rows per wave: K into the hand-over buffers, V into stages 3 and 4, both free
      // until the first step's barrier.  Keys past the tile's last arrive as zeros.
      {
        const i32x4 r = buffer_rsrc((m ? p.k : p.v) + (kv_row0 * p.hkv + u.kvh) * D, (n_keys - 1) * kv_row_bytes + D * 2);
#pragma unroll
        for (int i = 0; i < 8; ++i)
          lds_fill_b128(r, lds0 + (m ? C::XOFF : 3 * C::STAGE) + DT::row_base(32 * pw + 4 * i), fill_voff<DT>(32, pw, i, lane, kv_row_bytes), 0);
      }
      // ---- dV or dK [32-channel block][key group of the pair] as [key x channel], see key_units
      f32x16 acc[C::NVA][2];
      const float mul = m ? p.scale : 1.f;
      const int n_pair_keys = n_keys - 64 * kp;
      const bool direct = u.exclusive && p.dk_out != nullptr;
      const int64_t out0 = ((kv_row0 + 64 * kp) * p.hkv + u.kvh) * D + 32 * C::NVA * ch;   // first element of the wave's part
      auto acc_rsrc = [&](void* base, int row_bytes, int bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, n_pair_keys > 0 ? (n_pair_keys - 1) * row_bytes + 32 * C::NVA * bytes : 0, 0x00020000);
      };
      auto each = [&](auto&& f) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int db = 0; db < C::NVA; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[db][kb][i] = f(acc[db][kb][i], 32 * kb + 8 * (i / 4) + (i % 4), db);
      };
      each([](float, int, int) { return 0.f; });
      if (u.exclusive && !direct) {                 // start from the caller's values
        int row_bytes = p.hkv * D * 4;
        asm volatile("" : "+s"(row_bytes));         // (the row offsets are formed here, not ahead of the unit loop)
        const __amdgpu_buffer_rsrc_t r = acc_rsrc((m ? p.dk : p.dv) + out0, row_bytes, 4);
        each([&](float, int row, int db) {
          return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, 4 * g2 * row_bytes + 4 * l32, row * row_bytes + 128 * db, 0));
        });
        const float inv = 1.f / mul;
        each([&](float a, int, int) { return a * inv; });
      }
      wait_vmem<0>();
      lds_barrier();                                // the K and V tiles and the first steps have landed

      // Transposed reads (one channel per lane): inside a 16-lane block lane i supplies the address of row i / 4, channels 4 (i % 4) + [0,4), and gets
      // channel i of the four rows.  dO^T, Q^T: k-slots = rows 16 x + {4 g2 + [0,4), 8 + 4 g2 + [0,4)}; rows eight further lie at (address ^ 32) + 8 rows.
      const int b4 = lane >> 4, i16 = lane & 15;
      const int traddr = tile_off<DT>(4 * g2 + (i16 >> 2), 4 * C::NVA * ch + 2 * (b4 & 1) + ((lane & 3) >> 1)) + 8 * (lane & 1) +
                         (m ? 0 : C::TILE);         // 32-channel block db at ^ (db << 6)
      // dQ^T[channel x query] by 16 x 16 x 32 matrix instructions: k-slots of a key group = keys 4 b + [0,4) and 16 + 4 b + [0,4), b = lane / 16; the query
      // (16 m + lane % 16) and the channel (16 c + lane % 16) on the lane.  kt[x][c]: K^T of key group x.
      bf16x8 kt[4][2];
      {
        const int at = C::XOFF + tile_off<DT>(4 * b4 + (i16 >> 2), 4 * pw + ((lane & 3) >> 1)) + 8 * (lane & 1);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int c = 0; c < 2; ++c) kt[x][c] = tr_read_8(smem + (at ^ (c << 5)) + 32 * x * DT::row_base(1), 16 * DT::row_base(1));
      }
      const int dsaddr = C::XOFF + 2 * C::PB + m * 1024 + (lane & 1) * 512 + (((4 * b4 + (i16 >> 2)) ^ (4 * (2 * (lane & 1) + m))) << 4) + ((lane & 3) >> 1) * 8;
      // P or dS of key group 2 kp as the score waves left it: chunk t at (xaddr ^ xflip t) + t * 1024
      const int xaddr = C::XOFF + 2 * kp * C::XGROUP + (m ? 2 * C::PB + (g2 * 32 + (l32 ^ (8 * g2))) * 16 : lane * 16);
      const int xflip = m ? 64 : 0;
      int j_actg[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) j_actg[g] = u.first_active(g);
      const int j_act0 = kp ? j_actg[2] : j_actg[0], j_act1 = kp ? j_actg[3] : j_actg[1];
      const int j_all = max(max(j_actg[0], j_actg[1]), max(j_actg[2], j_actg[3]));

      // ---- dQ through L2: register i of dq[c] is channel 16 c + 4 b + i of the lane's query
      const bool chained = u.rank >= 0, dq_direct = chained && p.dq_out != nullptr;
      // What the part holds so far comes in by LDS-direct loads of eight rows x 128 bytes, an iteration ahead, and leaves the same way; the 16-byte chunks
      // of a row are permuted by its number / 2 (no bank conflicts in either form of access).
      const int old_buf = C::OOFF + (4 * m + pw) * 4096;
      auto line_chunk = [](int l) { return 16 * ((l & 7) ^ (l >> 4)); };                        // in row l / 8 (^ 64 for the second eight rows)
      // One resource per unit, ending with the item's last row (rows past it read as zero and are not written); a step's place in it is a scalar offset.
      const int64_t dq0 = ((int64_t)u.t.q_local_off * p.hq + u.kvh * G) * D + 32 * pw;
      const int dq_bytes = (int)((uint32_t)(u.t.q_len - 1) * (uint32_t)dq_row_bytes) + (G - 1) * D * 4 + 128;
      const i32x4 rl = buffer_rsrc(p.dq + dq0, dq_bytes);
      const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void*)(p.dq + dq0), (short)0, dq_bytes, 0x00020000);
      const __amdgpu_buffer_rsrc_t rf = __builtin_amdgcn_make_buffer_rsrc((void*)(p.flags + ((int64_t)u.flag_base * p.hq + u.kvh * G) * kChainSlices + 4 * m + pw),
                                                                         (short)0, 1 << 30, 0x00020000);
      const int blk = C::BM * dq_row_bytes, fblk = p.hq * kChainSlices * 4;   // a block further, in dQ and in the flags
      int so0 = (u.qb0 + u.nqb - 1) * blk + 16 * m * dq_row_bytes, so1 = so0;   // steps it and it - 1
      int fo0 = (u.qb0 + u.nqb - 1) * fblk, fo1 = fo0, fo2 = fo0;              // steps it, it - 1, it - 2
      auto is_last = [&](int jj) { return dq_direct && u.qb0 + jj < u.qb_next; };
      const bool loads = chained && (u.rank > 0 || !dq_direct);
      int spin_left = kSpinLimit;

      bf16x8 bop[2][2] = {}, fr[2 * C::NVA] = {};   // operands of step it - 1 at the end of iteration `it`
      bool have = false, act0 = false, act1 = false;
      int j0 = u.nqb - 1, j1 = 0, j2 = 0;           // blocks of steps it, it - 1, it - 2
      int st1 = (C::NSTAGE - 1) * C::STAGE;         // stage of step it - 1
      for (int it = 0; it < n_iter + C::DRAIN; ++it) {
        lds_barrier();
        const bool live1 = it >= 1 && it - 1 < n_iter;
        const bool loads0 = loads && it < n_iter;
        int seen = u.rank;
        if (u.rank > 0 && loads0) seen = __builtin_amdgcn_raw_buffer_load_b32(rf, 0, fo0, kCacheBypass);
        // dS of step it - 1, the query on the lane
        bf16x8 ds[4];
        {
          const int at = fresh(dsaddr) + ((it - 1) & 1) * C::PB;
#pragma unroll
          for (int x = 0; x < 4; ++x) ds[x] = tr_read_8(smem + at + x * C::XGROUP, 256);
        }
        if (have) {                                 // dV += P^T dO or dK += dS^T Q of step it - 2
          if (!(act0 && act1)) {                    // rare (causal edge, tails): a group that left nothing counts as zero
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              if (!act0) bop[0][t] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
              if (!act1) bop[1][t] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
            }
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int x = 0; x < 2 * C::NVA; ++x)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
              acc[x % C::NVA][kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bop[kb][x / C::NVA], fr[x], acc[x % C::NVA][kb], 0, 0, 0);
              __builtin_amdgcn_sched_barrier(0);
            }
        }
        // ---- dQ of step it - 1
        f32x4 dq[2];
        if (live1) {
          if (j1 < j_all) {                         // rare: a group that the block does not see is left out (its keys may hold anything)
            dq[0] = dq[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int x = 0; x < 4; ++x)
              if (j1 >= j_actg[x]) {
#pragma unroll
                for (int c = 0; c < 2; ++c) dq[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kt[x][c], ds[x], dq[c], 0, 0, 0);
              }
          } else {
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
              for (int c = 0; c < 2; ++c)
                dq[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kt[x][c], ds[x], x == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : dq[c], 0, 0, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        // operands of step it - 1: its P and dS are visible since this iteration's barrier
        {
          act0 = live1 && j1 >= j_act0;
          act1 = live1 && j1 >= j_act1;
          have = act0 || act1;
          const int xa = fresh(xaddr) + ((it - 1) & 1) * C::PB, ta = st1 + fresh(traddr);
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int t = 0; t < 2; ++t) bop[kb][t] = *reinterpret_cast<const bf16x8*>(smem + (t ? xa ^ xflip : xa) + kb * C::XGROUP + t * 1024);
#pragma unroll
          for (int x = 0; x < 2 * C::NVA; ++x) {
            const int a = ta ^ ((x % C::NVA) << 6);
            fr[x] = tr_read_8(smem + a + (x / C::NVA) * 16 * DT::row_base(1), smem + (a ^ 32) + ((x / C::NVA) * 16 + 8) * DT::row_base(1));
          }
        }
        // what the part of step it - 1 holds so far is in LDS, the stores of step it - 2 have arrived (pass that block on), and the flag of step `it`
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(seen) :: "memory");
        if (it >= 2 && chained && !is_last(j2)) __builtin_amdgcn_raw_buffer_store_b32((unsigned)(u.rank + 1), rf, fresh(lane) == 0 ? 0 : 1 << 30, fo2, 0);
        if (loads0) {
          while (__builtin_amdgcn_readfirstlane(seen) != u.rank && spin_left > 0) {
            __builtin_amdgcn_s_sleep(1);
            seen = __builtin_amdgcn_raw_buffer_load_b32(rf, 0, fo0, kCacheBypass);
            --spin_left;
          }
          const int l = fresh(lane), lv = (l >> 3) * dq_row_bytes, lc = line_chunk(l);
          lds_fill_x2<true>(rl, lds0 + old_buf + (it & 1) * 2048, lv + lc, lv + (lc ^ 64), so0, 8 * dq_row_bytes);
        }
        if (live1) {
          const int l = fresh(lane);
          const int at = old_buf + ((it - 1) & 1) * 2048 + (l & 15) * 128 + (((l >> 4) ^ ((l >> 1) & 7)) << 4);   // chunk 4 c + b at ^ (c << 6)
          const int dq_voff = (l & 15) * dq_row_bytes + 16 * (l >> 4);
          const float dq_mul = spin_left > 0 ? p.scale : NAN;          // (see kSpinLimit)
          if (loads) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              const f32x4 v = *reinterpret_cast<const f32x4*>(smem + (at ^ (c << 6)));
#pragma unroll
              for (int e = 0; e < 4; ++e) dq[c][e] = fmaf(dq[c][e], dq_mul, v[e]);
            }
          } else {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
              for (int e = 0; e < 4; ++e) dq[c][e] *= dq_mul;
          }
          if (is_last(j1)) {
            const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)(p.dq_out + dq0), (short)0, (uint32_t)dq_bytes / 2, 0x00020000);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              const bf16x4 b = {(__bf16)dq[c][0], (__bf16)dq[c][1], (__bf16)dq[c][2], (__bf16)dq[c][3]};
              __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, b), rb, dq_voff / 2 + 32 * c, (uint32_t)so1 / 2, 0);
            }
          } else if (chained) {
#pragma unroll
            for (int c = 0; c < 2; ++c) *reinterpret_cast<f32x4*>(smem + (at ^ (c << 6))) = dq[c];
            const int lc = line_chunk(l), from = old_buf + ((it - 1) & 1) * 2048 + (l >> 3) * 128;
            f32x4 v[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) v[q] = *reinterpret_cast<const f32x4*>(smem + from + q * 1024 + (lc ^ (q << 6)));
#pragma unroll
            for (int q = 0; q < 2; ++q) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[q]), rq, (l >> 3) * dq_row_bytes + 16 * (l & 7) + so1 + q * 8 * dq_row_bytes, 0, 0);
          } else {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
              for (int e = 0; e < 4; ++e) __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(dq[c][e], rq, dq_voff + 64 * c + 4 * e, so1, 0);
          }
        }
        st1 += C::STAGE;
        if (st1 == C::NSTAGE * C::STAGE) st1 = 0;
        j2 = j1; j1 = j0;
        so1 = so0; fo2 = fo1; fo1 = fo0;
        if (--j0 < 0) {                             // the next head's last block
          j0 = u.nqb - 1;
          so0 += (u.nqb - 1) * blk + D * 4;
          fo0 += (u.nqb - 1) * fblk + kChainSlices * 4;
        } else {
          so0 -= blk;
          fo0 -= fblk;
        }
      }
      if (spin_left <= 0 && lane == 0) atomicAdd(&p.hdr->n_stalled, 1);
      // ---- epilogue
      int row_bytes = p.hkv * D * (direct ? 2 : 4);
      asm volatile("" : "+s"(row_bytes));
      const __amdgpu_buffer_rsrc_t ro = acc_rsrc(direct ? (void*)((m ? p.dk_out : p.dv_out) + out0) : (void*)((m ? p.dk : p.dv) + out0), row_bytes, direct ? 2 : 4);
      if (direct)
        each([&](float a, int row, int db) {
          __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, (__bf16)(a * mul)), ro, 4 * g2 * row_bytes + 2 * l32, row * row_bytes + 64 * db, 0);
          return a;
        });
      else if (u.exclusive)
        each([&](float a, int row, int db) {
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, a * mul), ro, 4 * g2 * row_bytes + 4 * l32, row * row_bytes + 128 * db, 0);
          return a;
        });
      else
        each([&](float a, int row, int db) {
          __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(a * mul, ro, 4 * g2 * row_bytes + 4 * l32, row * row_bytes + 128 * db, 0);
          return a;
        });
      lds_barrier();                                // the LDS is free for the next unit; these stores stay in flight
    }
  }
}

}  // namespace

int launch_bwd_fused(const BwdParams& p, int64_t units, int n_cu, hipStream_t stream) {
  const int64_t blocks = persistent_blocks(n_cu, units);               // one 768-thread block per CU
  static std::atomic<uint64_t> lds_done;
  const int rc = raise_lds_limit((const void*)bwd_fused_kernel<128>, FusedCfg<128>::LDS_BYTES, lds_done);
  if (rc != FCP_OK) return rc;
  hipLaunchKernelGGL(bwd_fused_kernel<128>, dim3((unsigned)blocks), dim3(768), FusedCfg<128>::LDS_BYTES, stream, p);
  FCP_HIP_CHECK(hipGetLastError());
  return FCP_OK;
}

}  // namespace fcp
