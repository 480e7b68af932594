// dK, dV and dQ of fcp_attn_bwd_step: the key tiles and the query tiles of a call in one launch.
//
// Backward of O = softmax(scale Q K^T) V (paper Eq. 1, Sec. 3.1; causal mask, Sec. 4.3) for the key sets the ring steps bring (ring-style CP,
// Sec. 3.2).  With the merged LSE the probabilities of a step are recomputed exactly, P = exp(scale s - LSE), so each step adds its own share:
//   dV += P^T dO,   dP = dO V^T,   dS = P o (dP - delta),   dK += scale dS^T Q,   dQ += scale dS K.
// fp32 atomics retire at about one element per L2 channel per clock on this chip (about 270 G/s), far too few to add dQ up per key tile, so S and
// dP are formed twice: over key tiles for dK and dV, over query tiles for dQ.
//
// gfx950 design
//   * blocks of four waves, one per SIMD, two blocks per CU (64 channels: three).  The waves are INDEPENDENT, each owns 32 keys (or 32 query rows) and
//     does everything for them; what they share is the tile stream, which comes in through two LDS stages (LDS-direct fills a stage
//     ahead, one barrier per stage).  The blocks of a CU run in no lock step, one's beginning, end, exponentials and LDS latency meet the others' matrix
//     work.  (Before: a kernel of 16 waves in four roles that handed P and dS over through LDS, then a kernel of eight waves in two phases
//     for dQ, one block per CU each.);
//   * key unit = 128 keys of one segment of a work item for one KV head, looping over the query heads of the KV head and over the 32-row query
//     blocks that see the tile.  K fragments in registers, V rows in LDS.  S and dP come out as [query x key] with the key on the lane, which is the A-operand layout
//     of P^T and dS^T in the accumulating contractions: P and dS never leave the wave's registers, and dS is formed from P in fp32;
//   * row unit = 64 query rows of one work item for two query heads of one KV head (128 rows of one head where they do not pair up), looping
//     over the 64-key stages of the two key segments that the rows see.  Q and dO fragments in registers; S^T and dP^T as [key x query], one query per lane;
//   * a step's matrix instructions are one stream, in which every LDS fragment is requested AHEAD instructions before its use across the borders
//     of the contractions; the exponentials stand between the instructions of dP, dS between those of dV.  AHEAD = 3 with 128 channels and 2 with
//     64 is what 256 and 168 registers hold without spills inside the loops;
//   * ONE launch for both lists.  Neither fills the chip on small problems, and each has an end in which CUs run dry.  A block takes units of
//     one list, then of the other; the first blocks begin with the key units that are longer than any row unit (a step of a key unit has 32
//     matrix instructions per wave, one of a row unit 24), of the others half begin with key units and half with row units;
//   * the last row units of the list, one per block, are worked in halves (two waves share 32 rows and divide the keys, 32 each, dQ added up in
//     LDS): the end of the launch is as long as a unit.  On small problems these are all of them.
// Backward step with its scheduling launch, two kernels one after the other / this one, us: 4096 tokens over 3 ranks, 8 heads 138 / 83; 8192 tokens,
// 32 heads on 8 1900 / 1650; 24 sequences of 32768 tokens, 32 on 8 4170 / 3950, 8 heads 1115 / 1020; 131072 tokens over 8 ranks, 32 on 8 51200 /
// 50100; 64 channels: 4096 tokens, 4 heads 133 / 85, 16 sequences of 60000 tokens, 40 on 8 15900 / 12100.
// Tried: the key tiles first and then the query tiles in every block (24 sequences of 32768 tokens, 8 heads 1230: the longest query tile begins
// last); every row unit in halves (its stages then serve half of the matrix instructions: 32768 tokens, 32 on 8 +5 %); priorities for the
// matrix stream: 0 to 1 % faster with 128 channels, 1 % slower with 64.
//   * the caller's fp32 accumulators: when the scheduler found that no other item of the launch touches the tile's rows the accumulators START from
//     the caller's values and the epilogue only stores; otherwise the epilogue adds with fp32 atomics; the pieces of a split tile in turn (see
//     wait_turn).  Direct mode: a unit that owns its rows writes the final bf16 values.
#include "fcp_bwd.h"

namespace fcp {
namespace {

template <int D>
struct KeyCfg {
  static constexpr int NWAVE = 4;
  static constexpr int BN = kBwdBN;                // 128 keys per unit, 32 per wave
  static constexpr int BM = kBwdBM;                // 32 query rows per step
  using DT = DualTile<D>;
  using VT = RowTile<D>;                           // (read as rows only)
  static constexpr int TILE = DT::bytes(BM);       // one Q or dO block
  static constexpr int SLOT = 256;                 // one statistics plane of a step: 64 floats (32 used)
  static constexpr int STAGE = 2 * TILE + 2 * SLOT;
  static constexpr int VOFF = 2 * STAGE;           // the unit's V rows
  static constexpr int max_of(int a, int b) { return a > b ? a : b; }
  static constexpr int LDS_BYTES = max_of(VOFF + VT::bytes(BN), max_of(NWAVE * RowStage<D>::BYTES, DT::bytes(BN)));
  static constexpr int NS = D / 16;                // MFMAs of one 32 x 32 block of S or dP
  static constexpr int NVA = D / 32;               // 32-channel blocks of dK, dV
  static constexpr int IPT = BM / DT::RPI / 2;     // fill instructions per wave and step: waves 0, 1 fill Q, waves 2, 3 dO
};

// what eight rows further change in a chunk's place, besides the row itself
template <int D> constexpr int kTr8 = (DualTile<D>::key(0) ^ DualTile<D>::key(8)) << 4;

template <int D, int AHEAD>
__device__ inline void key_units(const BwdParams& p, const int queues, PartQueue& uq, unsigned char* const smem, int32_t* const s_next_unit, int32_t* const s_rec) {
  using C = KeyCfg<D>;
  using DT = typename C::DT;
  using VT = typename C::VT;
  const int tid = threadIdx.x;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g2 = lane >> 5;
  const int G = p.hq / p.hkv;
  const uint32_t lds0 = lds_offset(smem);
  const int kvh_here = p.hkv / queues, kvh0 = (int)(blockIdx.x % queues) * kvh_here;    // the queue's heads

  const int q_row_bytes = p.hq * D * 2;
  const int kv_row_bytes = p.hkv * D * 2;
  const bool fill_is_do = wave >= 2;
  const int fill_row0 = 16 * (wave & 1);
  // fill instruction i covers rows fill_row0 + RPI i + lane / CPR: its chunk permutation is that of i = 0 with key(RPI i) on top
  const int tfill = (fill_row0 + lane / DT::CPR) * q_row_bytes + (((lane % DT::CPR) ^ DT::key(lane / DT::CPR)) << 4);
  const int row0 = tile_off<DT>(l32, g2);          // row fragment ks (row l32, channels 16 ks + 8 g2 ..) at row0 ^ (ks << 5)
  constexpr int NVR = D == 128 ? 2 : 4;            // V row fragments: distinct addresses, see fwd_kernel
  int vrow[NVR];
#pragma unroll
  for (int j = 0; j < NVR; ++j) vrow[j] = C::VOFF + C::VT::row_base(32) * wave + tile_off<typename C::VT>(l32, 2 * j + g2);
  // Transposed fragments (one channel per lane; k-slots = query rows 16 t + {4 g2 + [0,4), 8 + 4 g2 + [0,4)}): channel block db of the first four rows
  // at tr0 ^ (db << 6), of the four rows eight further at that ^ kTr8, eight rows on
  const int tr0 = tile_off<DT>(4 * g2 + ((lane & 15) >> 2), 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) + 8 * (lane & 1);

  for (;;) {
    const int unit = uq.current(s_next_unit);
    if (unit >= uq.n_all) break;
    const KTile t = read_record<KTile, 16>(s_rec);
    const int kvh = kvh0 + unit % kvh_here;

    const bool exclusive = (t.flags & kFlagSeg0Exclusive) != 0;
    const bool direct = exclusive && p.dk_out != nullptr;
    const int n_keys = t.n_keys;
    const int my_key = 32 * wave + l32;
    const int64_t kv_row0 = t.kv_row0;
    const int first_row = max(0, t.from_first[0] - t.q_seq_start);
    const int qb0 = first_row / C::BM;
    const int nqb = (t.q_len + C::BM - 1) / C::BM - qb0;
    const int n_iter = nqb * G;

    // ---- fills: step s = (query head s / nqb of the KV head, query block qb0 + s % nqb), strictly in order.  Rows past the item's last row lie outside the
    // resources' range and arrive as zeros.
    const int q_bytes = (t.q_len - 1) * q_row_bytes + D * 2;
    const int64_t plane = (int64_t)p.hq * p.tq;
    int f_head = kvh * G, f_left = nqb;
    int f_soff = qb0 * C::BM * q_row_bytes, f_ssoff = qb0 * C::BM * 4;
    i32x4 f_rt, f_rst;
    auto f_resources = [&]() {
      f_rt = buffer_rsrc((fill_is_do ? p.d_o : p.q) + ((int64_t)t.q_local_off * p.hq + f_head) * D, q_bytes);
      f_rst = buffer_rsrc(p.stats + (wave & 1) * plane + (int64_t)f_head * p.tq + t.q_local_off, t.q_len * 4);
    };
    f_resources();
    uint32_t f_dst = 0;
    auto fill_next = [&]() {
      if (f_left == 0) {
        ++f_head;
        f_left = nqb;
        f_soff = qb0 * C::BM * q_row_bytes;
        f_ssoff = qb0 * C::BM * 4;
        f_resources();
      }
      const int tf = fresh(tfill);
#pragma unroll
      for (int i = 0; i < C::IPT; ++i)
        lds_fill_b128(f_rt, lds0 + f_dst + (fill_is_do ? C::TILE : 0) + DT::row_base(fill_row0 + DT::RPI * i), tf ^ (DT::key(DT::RPI * i) << 4),
                      f_soff + i * DT::RPI * q_row_bytes);
      if (wave < 2) lds_fill_b32(f_rst, lds0 + f_dst + 2 * C::TILE + wave * C::SLOT, lane * 4, f_ssoff);
      --f_left;
      f_soff += C::BM * q_row_bytes;
      f_ssoff += C::BM * 4;
      f_dst = C::STAGE - f_dst;
    };

    // ---- the wave's own K (and V) rows: whole rows through LDS, K through the stages
    int my_key_from = t.k_pos0 + my_key;
    if (p.k_from) my_key_from = p.k_from[kv_row0 + min(my_key, n_keys - 1)];
    bf16x8 kf[C::NS];
    {
      int lane_p = lane;
      asm volatile("" : "+v"(lane_p));
      const int bytes = (n_keys - 1) * kv_row_bytes + D * 2;
      const int64_t base = (kv_row0 * p.hkv + kvh) * D;
      auto fill_rows = [&](auto tile, const uint16_t* src, int area) {
        using T = decltype(tile);
        const i32x4 r = buffer_rsrc(src + base, bytes);
#pragma unroll
        for (int i = 0; i < 32 / T::RPI; ++i)
          lds_fill_b128(r, lds0 + area + T::row_base(32 * wave + T::RPI * i), fill_voff<T>(32, wave, i, lane_p, kv_row_bytes), 0);
      };
      fill_rows(DT(), p.k, 0);
      fill_rows(VT(), p.v, C::VOFF);
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      const int r32 = DT::row_base(32) * wave + tile_off<DT>(lane_p & 31, lane_p >> 5);
#pragma unroll
      for (int ks = 0; ks < C::NS; ++ks) kf[ks] = *reinterpret_cast<const bf16x8*>(smem + (r32 ^ (ks << 5)));
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __syncthreads();                              // the stages are free
    }
    my_key_from = (my_key < n_keys ? my_key_from : 1 << 29) - 4 * g2;   // masked: rows (minus 4 g2) below it
    fill_next();

    auto pick = [](const int32_t (&a)[4], int grp) { return grp == 0 ? a[0] : grp == 1 ? a[1] : grp == 2 ? a[2] : a[3]; };
    int j_act, j_unmasked;
    {
      const int ta = pick(t.from_first, wave) - t.q_seq_start;
      j_act = (32 * wave >= n_keys || ta > t.q_len - 1) ? nqb : max(0, (max(ta, 0) >> 5) - qb0);
      const int tu = pick(t.from_last, wave) - t.q_seq_start;
      j_unmasked = 32 * wave + 32 > n_keys ? nqb : max(0, ((max(tu, 0) + 31) >> 5) - qb0);
    }
    // dV, dK [32-channel block] as [key x channel]: the channel is on the lane, register i is key 8 (i/4) + 4 g2 + i%4 of the wave's 32.  The keys are reached
    // through a buffer resource that ends with the tile's last key (reads past it give zero, writes are dropped).
    f32x16 dv[C::NVA], dk[C::NVA];
    const int n_wave_keys = n_keys - 32 * wave;
    const int64_t out0 = ((kv_row0 + 32 * wave) * p.hkv + kvh) * D;
    auto rsrc = [&](void* base, int row_bytes, int bytes) {
      return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, n_wave_keys > 0 ? (min(n_wave_keys, 32) - 1) * row_bytes + D * bytes : 0, 0x00020000);
    };
#pragma unroll
    for (int db = 0; db < C::NVA; ++db) dv[db] = dk[db] = zero16();
    if (exclusive && !direct) {
      const int row_bytes = fresh_uniform(p.hkv * D * 4);
      const __amdgpu_buffer_rsrc_t rv = rsrc(p.dv + out0, row_bytes, 4), rk = rsrc(p.dk + out0, row_bytes, 4);
      const float inv = 1.f / p.scale;
#pragma unroll
      for (int db = 0; db < C::NVA; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int so = (8 * (i / 4) + (i % 4)) * row_bytes + 128 * db;
          dv[db][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rv, 4 * g2 * row_bytes + 4 * l32, so, 0));
          dk[db][i] = inv * __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rk, 4 * g2 * row_bytes + 4 * l32, so, 0));
        }
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
    }

    int j = 0, st = 0;
    for (int it = 0; it < n_iter; ++it) {
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      __syncthreads();
      if (__builtin_expect(it + 1 < n_iter, 1)) fill_next(); else uq.take(wave);
      const int jb = j, at0 = st;
      if (++j == nqb) j = 0;
      st = C::STAGE - st;
      if (jb < j_act) continue;
      const float* const stat = reinterpret_cast<const float*>(smem + at0 + 2 * C::TILE) + 4 * g2;
      f32x16 s, dp;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 nd = *reinterpret_cast<const f32x4*>(stat + C::SLOT / 4 + 8 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) dp[4 * q + e] = nd[e];
      }
      // The step's 4 NS matrix instructions are one stream: the fragments of instruction k are requested A instructions ahead, across the borders
      // of S, dP, dV and dK.
      constexpr int NS = C::NS, A = AHEAD;
      static_assert(2 * C::NVA == NS, "as many instructions in each of the four parts");
      int xr[NS], ta[C::NVA];
      {
        const int r = fresh(row0);
#pragma unroll
        for (int ks = 0; ks < NS; ++ks) xr[ks] = (r ^ (ks << 5)) + at0;
      }
      bf16x8 fa[4 * NS], fb[NS];
      auto tr = [&](int tile, int x) {
        const unsigned char* b0 = smem + tile + (x / C::NVA) * (16 * DT::row_base(1));
        return tr_read_8(b0 + ta[x % C::NVA], b0 + 8 * DT::row_base(1) + (ta[x % C::NVA] ^ kTr8<D>));
      };
      auto request = [&](int k) {
        if (k < NS) fa[k] = *reinterpret_cast<const bf16x8*>(smem + xr[k]);
        else if (k < 2 * NS) {
          fa[k] = *reinterpret_cast<const bf16x8*>(smem + xr[k - NS] + C::TILE);
          fb[k - NS] = *reinterpret_cast<const bf16x8*>(smem + vrow[(k - NS) % NVR] + ((k - NS) / NVR) * (NVR * 32));
        }
        else if (k < 3 * NS) fa[k] = tr(C::TILE, k - 2 * NS);
        else if (k < 4 * NS) fa[k] = tr(0, k - 3 * NS);
      };
#pragma unroll
      for (int k = 0; k < A; ++k) request(k);
      if constexpr (D == 128) __builtin_amdgcn_s_setprio(1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int x = 0; x < NS; ++x) {                // S
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[x], kf[x], x == 0 ? zero16() : s, 0, 0, 0);
        request(x + A);
        __builtin_amdgcn_sched_barrier(0);
      }
      {
        const int r = fresh(tr0);
#pragma unroll
        for (int db = 0; db < C::NVA; ++db) ta[db] = (r ^ (db << 6)) + at0;
      }
      bf16x8 pb[2], dsb[2];
      f32x4 nl[4];
      // element i of a 16-element part belongs to instruction x of a part's NS, from the second on
      auto first_of = [](int x) { return x < 1 ? 0 : 16 * (x - 1) / (C::NS - 1); };
#pragma unroll
      for (int x = 0; x < NS; ++x) {                // dP with P in its shadow
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[NS + x], fb[x], dp, 0, 0, 0);
        request(NS + x + A);
        if (x == 0) nl[0] = *reinterpret_cast<const f32x4*>(stat);
#pragma unroll
        for (int i = first_of(x); i < first_of(x + 1); ++i) {
          if (i % 4 == 0 && i < 12) nl[i / 4 + 1] = *reinterpret_cast<const f32x4*>(stat + 2 * i + 8);
          s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], p.scale_log2, nl[i / 4][i % 4]));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (jb < j_unmasked) {
        int lo = my_key_from - (t.q_seq_start + (qb0 + jb) * C::BM);
        asm volatile("; masked variant" : "+v"(lo));
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 8 * (i / 4) + (i % 4) < lo ? 0.f : s[i];
#pragma unroll
        for (int i = 0; i < 16; ++i) dp[i] = 8 * (i / 4) + (i % 4) < lo ? 0.f : dp[i];
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) pb[i / 8][i % 8] = (__bf16)s[i];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int x = 0; x < NS; ++x) {                // dV with dS in its shadow
        dv[x % C::NVA] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pb[x / C::NVA], fa[2 * NS + x], dv[x % C::NVA], 0, 0, 0);
        request(2 * NS + x + A);
#pragma unroll
        for (int i = first_of(x); i < first_of(x + 1); ++i) dsb[i / 8][i % 8] = (__bf16)(s[i] * dp[i]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int x = 0; x < NS; ++x) {                // dK
        dk[x % C::NVA] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dsb[x / C::NVA], fa[3 * NS + x], dk[x % C::NVA], 0, 0, 0);
        request(3 * NS + x + A);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (D == 128) __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();                                // the stages are free
    if (n_iter == 0) uq.take(wave);
    uq.prefetch();
    // ---- epilogue
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    const int l32e = lane_e & 31, g2e = lane_e >> 5;
    using OUT = RowStage<D>;
    unsigned char* const obuf = smem + wave * OUT::BYTES;
    if (direct) {
      const int row_bytes = fresh_uniform(p.hkv * D * 2);
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const __amdgpu_buffer_rsrc_t r = rsrc((m ? p.dk_out : p.dv_out) + out0, row_bytes, 2);
        const float mul = m ? p.scale : 1.f;
#pragma unroll
        for (int db = 0; db < C::NVA; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) OUT::put_bf16(obuf, OUT::reg_row(i, g2e), 32 * db + l32e, (m ? dk : dv)[db][i] * mul);
        OUT::template flush<true>(obuf, lane_e, r, row_bytes, 0);
      }
    } else {
      const bool in_turn = (t.flags & kFlagInTurn) != 0;
      int32_t* const turn = p.turns + ((int64_t)t.turn * p.hkv + kvh) * kTurnWaves + wave;
      float mul = 1.f;
      if (in_turn && !wait_turn(turn, t.flags >> kPieceShift)) {
        mul = NAN;
        if (lane_e == 0) atomicAdd(p.n_stalled, 1);
      }
      const int row_bytes = fresh_uniform(p.hkv * D * 4);
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const __amdgpu_buffer_rsrc_t r = rsrc((m ? p.dk : p.dv) + out0, row_bytes, 4);
        const float mul_m = m ? p.scale * mul : mul;
#pragma unroll
        for (int db = 0; db < C::NVA; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const float val = (m ? dk : dv)[db][i] * mul_m;
            const int so = (8 * (i / 4) + (i % 4)) * row_bytes + 128 * db;
            if (exclusive) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, val), r, 4 * g2e * row_bytes + 4 * l32e, so, 0);
            else __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(val, r, 4 * g2e * row_bytes + 4 * l32e, so, 0);
          }
      }
      if (in_turn) pass_turn(turn);
    }
    uq.advance(s_next_unit, s_rec);
  }
}

template <int D, int SPLIT, int SKEYS>
struct RowCfg {
  static constexpr int NWAVE = 4;
  static constexpr int RG = NWAVE / SPLIT;         // groups of 32 rows (of one or two heads)
  static constexpr int SK = SKEYS;                 // keys per stage
  static constexpr int NB = SK / 32 / SPLIT;       // 32-key blocks of a stage per wave
  using DT = DualTile<D>;
  static constexpr int TILE = DT::bytes(SK);       // K or V of a stage
  static constexpr int STAGE = 2 * TILE;
  static constexpr int AREA = NWAVE * DT::bytes(32);   // the waves' Q, then dO rows, on their way in: the second stage
  static constexpr int max_of(int a, int b) { return a > b ? a : b; }
  static constexpr int LDS_BYTES = max_of(max_of(2 * STAGE, STAGE + AREA), SPLIT > 1 ? NWAVE * 32 * D * 4 : 0);
  static constexpr int NS = D / 16;                // k-steps of one 32 x 32 block of S^T or dP^T
  static constexpr int NCB = D / 32;               // 32-channel blocks of dQ
  static constexpr int RPW = SK / 2;               // rows each wave fills: waves 0, 1 K, waves 2, 3 V
  static constexpr int IPT = RPW / DT::RPI;
};

template <int D, int SPLIT, int SKEYS, int AHEAD>
__device__ inline void row_units(const BwdParams& p, const int head_pair, const int queues, PartQueue& uq, unsigned char* const smem, int32_t* const s_next_unit, int32_t* const s_rec) {
  using C = RowCfg<D, SPLIT, SKEYS>;
  using DT = typename C::DT;
  const int tid = threadIdx.x;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int share = wave % SPLIT, group = wave / SPLIT;
  const int l32 = lane & 31, g2 = lane >> 5;
  const int G = p.hq / p.hkv;
  const uint32_t lds0 = lds_offset(smem);
  const int hpu = head_pair ? 2 : 1;
  const int heads_here = p.hq / queues, head0 = (int)(blockIdx.x % queues) * heads_here;
  const int units_per_tile = heads_here / hpu;

  const int kv_row_bytes = p.hkv * D * 2;
  const bool fill_is_v = wave >= 2;
  // rows RPI i + lane / CPR of the wave's half: the chunk permutation has a period of 16 rows
  constexpr int NKF = 16 / DT::RPI < C::IPT ? 16 / DT::RPI : C::IPT;
  int tfill[NKF];
#pragma unroll
  for (int i = 0; i < NKF; ++i) {
    const int row = C::RPW * (wave & 1) + DT::RPI * i + lane / DT::CPR;
    tfill[i] = (row - DT::RPI * i) * kv_row_bytes + (((lane % DT::CPR) ^ DT::key(row)) << 4);
  }
  const int row0 = tile_off<DT>(l32, g2);          // row fragment ks (row l32, channels 16 ks + 8 g2 ..) at row0 ^ (ks << 5)
  auto rows = [&](int at, int ks) { return *reinterpret_cast<const bf16x8*>(smem + (at ^ (ks << 5))); };
  const int tr0 = tile_off<DT>(4 * g2 + ((lane & 15) >> 2), 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) + 8 * (lane & 1);   // see key_units

  for (;;) {
    const int unit = uq.current(s_next_unit);
    if (unit >= (SPLIT == 1 ? uq.n_full : uq.n_all)) break;
    QTile t = read_record<QTile, 12>(s_rec);
    constexpr int RGP = C::RG > 1 ? C::RG / 2 : 1;
    int whole = unit;
    if constexpr (SPLIT > 1) {                      // half of the tile's rows
      const int half = (unit - uq.n_full) & 1, first = half ? 32 * C::RG / hpu : 0;
      whole = uq.n_full + ((unit - uq.n_full) >> 1);
      t.q_row0 += first;
      t.q_pos0 += first;
      t.rows = min(t.rows - first, 32 * C::RG / hpu);
      if (t.rows <= 0) {
        uq.take(wave);
        uq.prefetch();
        __syncthreads();                            // (everybody has read the record)
        uq.advance(s_next_unit, s_rec);
        continue;
      }
    }
    const int head = head0 + (whole % units_per_tile) * hpu + (head_pair ? group / RGP : 0);
    const int kvh = head / G;

    const bool exclusive = (t.flags & kFlagQExclusive) != 0;
    const bool direct = exclusive && p.dq_out != nullptr;
    const int rows_here = t.rows;
    const int vis0 = t.vis[0], vis1 = t.vis[1], kpos0 = t.k_pos0[0], kpos1 = t.k_pos0[1];
    const int64_t kvrow0 = t.kv_row0[0], kvrow1 = t.kv_row0[1];
    const int nt0 = (vis0 + C::SK - 1) / C::SK, nt1 = (vis1 + C::SK - 1) / C::SK;
    const int n_iter = nt0 + nt1;

    const int wave_r0 = 32 * (head_pair ? group % RGP : group);
    const int my_row = wave_r0 + l32;
    const int row_ld = min(my_row, rows_here - 1);
    const bool wave_active = wave_r0 < rows_here;
    int q_lim = t.q_pos0 + my_row, first_lim = t.q_pos0 + wave_r0, last_lim = t.q_pos0 + min(wave_r0 + 31, rows_here - 1);
    if (p.q_limit) {
      const int32_t* ql = p.q_limit + t.q_row0;
      q_lim = ql[row_ld];
      first_lim = __builtin_amdgcn_readfirstlane(ql[min(wave_r0, rows_here - 1)]);
      last_lim = __builtin_amdgcn_readfirstlane(ql[min(wave_r0 + 31, rows_here - 1)]);
    }
    const float stat_p = p.stats[(int64_t)head * p.tq + t.q_row0 + row_ld];
    const float stat_d = p.stats[(int64_t)p.hq * p.tq + (int64_t)head * p.tq + t.q_row0 + row_ld];
    __builtin_amdgcn_s_waitcnt(kWaitVm0);          // before any fill is in flight: later waits count the fills only

    // ---- fills
    i32x4 f_r;
    auto f_resource = [&](int64_t row, int vis) {
      f_r = buffer_rsrc((fill_is_v ? p.v : p.k) + (row * p.hkv + kvh) * D, vis > 0 ? (vis - 1) * kv_row_bytes + D * 2 : 0);
    };
    f_resource(kvrow0, vis0);
    int f_left = nt0, f_soff = 0;
    bool f_seg0 = true;
    uint32_t f_dst = lds0 + (fill_is_v ? C::TILE : 0) + DT::row_base(C::RPW) * (wave & 1);
    const uint32_t f_sum = 2 * f_dst + C::STAGE;
    auto fill_next = [&]() {
      if (f_seg0 && f_left == 0) { f_resource(kvrow1, vis1); f_seg0 = false; f_soff = 0; }
#pragma unroll
      for (int i = 0; i < C::IPT; ++i)
        lds_fill_b128(f_r, f_dst + DT::row_base(DT::RPI * i), tfill[i % NKF], f_soff + i * DT::RPI * kv_row_bytes);
      --f_left;
      f_soff += C::SK * kv_row_bytes;
      f_dst = f_sum - f_dst;
    };
    if (n_iter > 0) fill_next();
    const int n_wave_rows = rows_here - wave_r0;
    bf16x8 qf[C::NS], dof[C::NS];
    {
      int lane_p = lane;
      asm volatile("" : "+v"(lane_p));
      const int q_row_bytes = p.hq * D * 2;
      const int64_t base = ((int64_t)(t.q_row0 + wave_r0) * p.hq + head) * D;
      const int nbytes = n_wave_rows > 0 ? (min(n_wave_rows, 32) - 1) * q_row_bytes + D * 2 : 0;
      const int area = C::STAGE + wave * DT::bytes(32);
      const int at = area + tile_off<DT>(lane_p & 31, lane_p >> 5);
      auto load_tile = [&](const uint16_t* src, bf16x8 (&f)[C::NS]) {
        const i32x4 r = buffer_rsrc(src + base, nbytes);
#pragma unroll
        for (int i = 0; i < 32 / DT::RPI; ++i)
          lds_fill_b128(r, lds0 + area + DT::row_base(DT::RPI * i), fill_voff<DT>(32, 0, i, lane_p, q_row_bytes), 0);
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
#pragma unroll
        for (int ks = 0; ks < C::NS; ++ks) f[ks] = rows(at, ks);
        __builtin_amdgcn_s_waitcnt(0xC07F);
      };
      load_tile(p.q, qf);
      load_tile(p.d_o, dof);
    }
    f32x16 acc[C::NCB];
    auto rsrc = [&](void* base, int row_bytes, int bytes) {
      return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, n_wave_rows > 0 ? (min(n_wave_rows, 32) - 1) * row_bytes + D * bytes : 0, 0x00020000);
    };
    const int64_t out0 = ((int64_t)(t.q_row0 + wave_r0) * p.hq + head) * D;
#pragma unroll
    for (int db = 0; db < C::NCB; ++db) acc[db] = zero16();
    if (exclusive && !direct && share == 0) {
      const int row_bytes = fresh_uniform(p.hq * D * 4);
      const __amdgpu_buffer_rsrc_t r = rsrc(p.dq + out0, row_bytes, 4);
      const float inv = 1.f / p.scale;
#pragma unroll
      for (int db = 0; db < C::NCB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          acc[db][i] = inv * __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, 4 * g2 * row_bytes + 4 * l32, (8 * (i / 4) + (i % 4)) * row_bytes + 128 * db, 0));
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
    }

    for (int it = 0; it < n_iter; ++it) {
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      __syncthreads();
      if (__builtin_expect(it + 1 < n_iter, 1)) fill_next(); else uq.take(wave);
      const bool seg1 = it >= nt0;
      const int base = (it - (seg1 ? nt0 : 0)) * C::SK + 32 * C::NB * share;
      for (int b = 0; b < C::NB; ++b) {
        const int k0 = base + 32 * b;
        const int k_pos = (seg1 ? kpos1 : kpos0) + k0;
        const int n_valid = (seg1 ? vis1 : vis0) - k0;
        if (!wave_active || n_valid <= 0 || k_pos > last_lim) break;
        const int so = (it & 1) * C::STAGE + (C::NB * share + b) * DT::row_base(32);
        constexpr int NS = C::NS, A = AHEAD;        // one stream of 3 NS matrix instructions, see key_units
        static_assert(2 * C::NCB == NS, "as many instructions in each of the three parts");
        bf16x8 fa[3 * NS], ds[2];
        f32x16 s, dp;
        int xr[NS], ta[2][C::NCB];
        {
          const int r = fresh(row0);
#pragma unroll
          for (int ks = 0; ks < NS; ++ks) xr[ks] = (r ^ (ks << 5)) + so;
        }
        auto request = [&](int k) {
          if (k < NS) fa[k] = *reinterpret_cast<const bf16x8*>(smem + xr[k]);
          else if (k < 2 * NS) fa[k] = *reinterpret_cast<const bf16x8*>(smem + xr[k - NS] + C::TILE);
          else if (k < 3 * NS) {
            const unsigned char* b0 = smem + ((k - 2 * NS) / C::NCB) * (16 * DT::row_base(1));
            fa[k] = tr_read_8(b0 + ta[0][k % C::NCB], b0 + ta[1][k % C::NCB] + 8 * DT::row_base(1));
          }
        };
#pragma unroll
        for (int k = 0; k < A; ++k) request(k);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < NS; ++x) {              // S^T
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[x], qf[x], x == 0 ? zero16() : s, 0, 0, 0);
          request(x + A);
          __builtin_amdgcn_sched_barrier(0);
        }
        {
          const int r = fresh(tr0);
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int db = 0; db < C::NCB; ++db) ta[h][db] = (r ^ (db << 6) ^ (h ? kTr8<D> : 0)) + so;
        }
        auto first_of = [](int x) { return x < 1 ? 0 : 16 * (x - 1) / (C::NS - 1); };
#pragma unroll
        for (int x = 0; x < NS; ++x) {              // dP^T with P^T in its shadow
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[NS + x], dof[x], x == 0 ? zero16() : dp, 0, 0, 0);
          request(NS + x + A);
#pragma unroll
          for (int i = first_of(x); i < first_of(x + 1); ++i) s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], p.scale_log2, stat_p));
          __builtin_amdgcn_sched_barrier(0);
        }
        if (k_pos + 31 > first_lim || n_valid < 32) {
          int hi = min(n_valid, q_lim - k_pos + 1) - 4 * g2;
          asm volatile("; masked variant" : "+v"(hi));
#pragma unroll
          for (int i = 0; i < 16; ++i) ds[i / 8][i % 8] = (__bf16)((8 * (i / 4) + (i % 4) < hi) ? s[i] * (dp[i] + stat_d) : 0.f);
        } else {
#pragma unroll
          for (int i = 0; i < 16; ++i) ds[i / 8][i % 8] = (__bf16)(s[i] * (dp[i] + stat_d));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < NS; ++x) {
          acc[x % C::NCB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ds[x / C::NCB], fa[2 * NS + x], acc[x % C::NCB], 0, 0, 0);
          request(2 * NS + x + A);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    __syncthreads();
    if (n_iter == 0) uq.take(wave);
    uq.prefetch();
    // ---- epilogue
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    const int l32e = lane_e & 31, g2e = lane_e >> 5;
    int n_db = C::NCB, db0 = 0;
    if constexpr (SPLIT > 1) {                      // the group's waves add up in LDS, each its channel blocks
      unsigned char* const mine = smem + wave * (32 * D * 4);
#pragma unroll
      for (int db = 0; db < C::NCB; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4 v = {acc[db][4 * j], acc[db][4 * j + 1], acc[db][4 * j + 2], acc[db][4 * j + 3]};
          *reinterpret_cast<f32x4*>(mine + (db * 4 + j) * 1024 + lane * 16) = v;
        }
      __syncthreads();
      constexpr int PARTS = SPLIT < C::NCB ? SPLIT : C::NCB;
      constexpr int NO = C::NCB / PARTS;
      n_db = share < PARTS ? NO : 0;
      db0 = (share < PARTS ? share : 0) * NO;
#pragma unroll
      for (int o = 0; o < NO; ++o)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int w = 0; w < SPLIT; ++w) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(smem + (group * SPLIT + w) * (32 * D * 4) + ((db0 + o) * 4 + j) * 1024 + lane * 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += v[e];
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[o][4 * j + e] = sum[e];
        }
    }
    if (direct) {
      const int row_bytes = fresh_uniform(p.hq * D * 2);
      const __amdgpu_buffer_rsrc_t r = rsrc(p.dq_out + out0 + 32 * db0, row_bytes, 2);
#pragma unroll
      for (int db = 0; db < C::NCB; ++db)
        if (SPLIT == 1 || db < n_db) {
#pragma unroll
          for (int i = 0; i < 16; ++i)
            __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, (__bf16)(acc[db][i] * p.scale)), r, 4 * g2e * row_bytes + 2 * l32e,
                                                  (8 * (i / 4) + (i % 4)) * row_bytes + 64 * db, 0);
        }
    } else {
      const bool in_turn = (t.flags & kFlagInTurn) != 0;
      int32_t* const turn = p.turns_q + ((int64_t)t.turn * (p.hq / hpu) + head / hpu) * kTurnWaves + wave;
      float mul = p.scale;
      if (in_turn && !wait_turn(turn, t.flags >> kPieceShift)) {
        mul = NAN;
        if (lane_e == 0) atomicAdd(p.n_stalled, 1);
      }
      const int row_bytes = fresh_uniform(p.hq * D * 4);
      const __amdgpu_buffer_rsrc_t r = rsrc(p.dq + out0 + 32 * db0, row_bytes, 4);
#pragma unroll
      for (int db = 0; db < C::NCB; ++db)
        if (SPLIT == 1 || db < n_db) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const float val = acc[db][i] * mul;
            const int so = (8 * (i / 4) + (i % 4)) * row_bytes + 128 * db;
            if (exclusive) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, val), r, 4 * g2e * row_bytes + 4 * l32e, so, 0);
            else __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(val, r, 4 * g2e * row_bytes + 4 * l32e, so, 0);
          }
        }
      if (in_turn) pass_turn(turn);
    }
    uq.advance(s_next_unit, s_rec);
  }
}

template <int D>
struct ListsCfg {
  static constexpr int max_of(int a, int b) { return a > b ? a : b; }
  static constexpr int LDS_BYTES = max_of(KeyCfg<D>::LDS_BYTES, max_of(RowCfg<D, 1, 64>::LDS_BYTES, RowCfg<D, 2, 64>::LDS_BYTES));
};

// Row units whose loop is shorter than this are not worked in halves: it is mostly their beginnings and ends that would be doubled.
constexpr int kHalfKeys = 512;

template <int D, int AHEAD>
__global__ __launch_bounds__(256, lists_blocks_per_cu(D)) void bwd_lists_kernel(const BwdParams p, const int head_pair) {
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  __shared__ int32_t s_next_unit;
  __shared__ int32_t s_rec[16];
  const int path = p.hdr->path;
  if (p.either && (path & kPathOnePass)) return;
  const bool kv_turns = (path & kPathSplitKeys) != 0, q_turns = (path & kPathSplitRows) != 0;   // units wait for earlier ones of their list
  const bool turns = kv_turns || q_turns;
  const int place = PartQueue::place(), places = PartQueue::places();
  const bool kv_xcd = (p.hkv % kNumXcd) == 0;
  const int kv_per_tile = kv_xcd ? p.hkv / kNumXcd : p.hkv;
  const int kv_tiles = p.hdr->n_tiles, q_tiles = p.hdr_q->n_tiles;      // (read here once: the counters beside them are busy later)
  const int kv_units = kv_tiles * kv_per_tile;
  const int kv_mine = PartQueue::mine(kv_units, kv_xcd);
  const int hpu = head_pair ? 2 : 1;
  const bool q_xcd = (p.hq % (kNumXcd * hpu)) == 0;
  const int q_per_tile = (q_xcd ? p.hq / kNumXcd : p.hq) / hpu;
  const int q_units = q_tiles * q_per_tile;

  // How many of the key tiles that could come first take longer than the longest query tile (lists are sorted).
  const QTile* const q_list = reinterpret_cast<const QTile*>(p.tiles_q);
  const int lane = threadIdx.x & 63;
  int q_half = 0, n_long = kv_mine;
  if (q_units > 0) {
    if (!q_turns) {
      q_half = min(q_units, q_xcd ? places : (int)gridDim.x);
      const QTile& t = q_list[(q_units - q_half) / q_per_tile];
      if (t.vis[0] + t.vis[1] < kHalfKeys) q_half = 0;
    }
    const int longest = (q_list->vis[0] + q_list->vis[1]) * 24;
    n_long = 0;
    for (int l0 = 0; l0 < places; l0 += 64) {
      const int l = l0 + lane, u = kv_xcd ? l : l * kNumXcd + (int)(blockIdx.x % kNumXcd);
      bool longer = false;
      if (l < kv_mine) {
        const KTile& t = reinterpret_cast<const KTile*>(p.tiles)[u / kv_per_tile];
        longer = (t.q_len - max(0, t.from_first[0] - t.q_seq_start)) * (p.hq / p.hkv) * 32 > longest;
      }
      n_long += __builtin_popcountll(__builtin_amdgcn_ballot_w64(longer));
    }
  }
  n_long = min(n_long, min(kv_mine, places));
  const auto [kv_dealt, kv_first, q_first] = first_unit(place, places, kv_mine, n_long);
  const int q_mine = PartQueue::mine(q_units + q_half, q_xcd);
  if (kv_first < 0 && q_first >= q_mine && kv_dealt == kv_mine) return;   // the others are enough
  const int longest_row = q_units > 0 ? q_list->vis[0] + q_list->vis[1] : 0;
  const bool deal = !turns && deals_first(kv_mine + q_mine, places, kDealLists, longest_row), reserve = keeps_reserve(deal, longest_row);
  bool keys = kv_first >= 0;
#pragma unroll 1
  for (int turn = 0; turn < 2; ++turn, keys = !keys) {
    PartQueue uq;
    if (turn) __syncthreads();                     // (everybody has seen the end of the other list)
    const bool dealt = deal && turn == 0;
    if (keys) {
      const int queues = head_queues(p.hkv, kv_turns);
      const int per_tile = p.hkv / queues;
      uq.open(p.hdr, p.tiles, kv_tiles * per_tile, 0, per_tile, unit_numbers(blockIdx.x, queues, kv_turns), turns, reserve, dealt ? kv_first : -1,
              deal ? kv_dealt : 0, &s_next_unit, s_rec);
      key_units<D, AHEAD>(p, queues, uq, smem, &s_next_unit, s_rec);
    } else {
      const int queues = head_queues(p.hq / hpu, q_turns);
      const int per_tile = p.hq / hpu / queues;
      uq.open(p.hdr_q, p.tiles_q, q_tiles * per_tile, q_half, per_tile, unit_numbers(blockIdx.x, queues, q_turns), turns, reserve, dealt ? q_first : -1,
              deal ? places - kv_dealt : 0, &s_next_unit, s_rec);
      row_units<D, 1, 64, 4>(p, head_pair, queues, uq, smem, &s_next_unit, s_rec);
      row_units<D, 2, 64, 4>(p, head_pair, queues, uq, smem, &s_next_unit, s_rec);
    }
  }
}

template <int D, int AHEAD>
int launch_one(const BwdParams& p, int head_pair, int64_t units, int n_cu, hipStream_t stream) {
  using C = ListsCfg<D>;
  static std::atomic<uint64_t> lds_done;
  const auto kernel = bwd_lists_kernel<D, AHEAD>;
  const int rc = raise_lds_limit((const void*)kernel, C::LDS_BYTES, lds_done);
  if (rc != FCP_OK) return rc;
  const int64_t blocks = persistent_blocks((int64_t)n_cu * lists_blocks_per_cu(D), units);
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), C::LDS_BYTES, stream, p, head_pair);
  FCP_HIP_CHECK(hipGetLastError());
  return FCP_OK;
}

}  // namespace

int launch_bwd_lists(const BwdParams& p, int head_dim, int head_pair, int64_t units, int n_cu, hipStream_t stream) {
  if (head_dim == 128) return launch_one<128, 3>(p, head_pair, units, n_cu, stream);
  return launch_one<64, 2>(p, head_pair, units, n_cu, stream);
}

}  // namespace fcp
