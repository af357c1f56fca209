// Fused attention forward for gfx950: S = scale*Q K^T, online row softmax, O = P V, LSE saved.
//
// Structure (paper Sec. 3.2): one workgroup owns one tile of 128 query rows of one (batch,
// head) and loops over tiles of 64 keys; per iteration it computes the score tile on the
// matrix cores, updates the running row max / row sum (Sec. 3.2.1, Eq. 3), rescales the O
// accumulator by exp(m_pre - m_cur), and accumulates P V on the matrix cores.  O is written
// once at the end, so HBM sees three reads and one write.
//
// What is specific to CDNA4 here:
//   * Each of the 4 waves owns 32 query rows.  The score tile is computed TRANSPOSED,
//     S^T = K Q^T (keys on the MFMA M axis, queries on the N axis), so a lane owns ONE query
//     column and its 32 accumulator registers are 32 of the tile's 64 keys.  Row max and row
//     sum are then in-lane reductions plus one exchange with the lane 32 positions away
//     (the counterpart of the paper's shuffle step for fp32 accumulators).
//   * O is accumulated transposed as well, O^T = V^T P^T.  The packed accumulator registers
//     of S^T are directly the B operand of that MFMA (see mma_gfx950.hpp), and the V^T
//     operand comes from the row-major V tile in LDS through transposing LDS reads.  P never
//     touches LDS or HBM (the paper's Sec. 3.2.2 layout transform becomes register renaming).
//   * K/V tiles are double-buffered in LDS and arrive there by direct global->LDS loads (no
//     staging registers, no LDS store instructions), requested at the top of the round before the one
//     that reads them and awaited before the one barrier that ends a round.
//   * The tiles are unpadded and XOR-swizzled (tiles_gfx950.hpp) so that the 16-byte row reads
//     of K and the 4-row transposing reads of V both spread over all banks.
//   * Each 64-key tile runs as two 32-key online-softmax steps.  V runs one tile behind K, so that the VALU work of
//     every step is interleaved, in program order (a wave issues in order), with the score MFMAs of
//     the step after it and the PV MFMAs of the step before it; LDS operand reads are issued
//     several MFMAs ahead and pinned there with scheduler fences.  (Within one tile the first scores and the last
//     products had no VALU work beside them.  Forward, us, that -> this: bf16, d = 128, 64 heads x 1024 over
//     4096 keys 133.8 -> 128.1, causal 64 x 4096 256.6 -> 251.2; fp16, causal 16 x 16384 1006 -> 984, d = 64 32 x
//     8192 597 -> 590.  The loop takes 26.5 ns per MFMA and SIMD at d = 128 in bf16 (64 heads x 1024, 2048
//     keys against 4096) and 36.5 at d = 64 in fp16; its instructions in a straight line take 24 and 32
//     (mix_floor_bench), the MFMAs alone 18 and 20.)
//   * Workgroups of 4 waves (128 queries, two per CU) or of 8 waves (256 queries, one per CU):
//     with 8 waves each K/V tile that is brought into LDS serves twice as many MFMAs (measured
//     -4 % at d = 128 on long sequences, +2 % at d = 64); the host picks per problem.  The 8-wave
//     form has the CU's LDS to itself: it holds two stages of two tiles each, requests tiles two
//     at a time and meets at a barrier every second round only (PAIR; at d = 64 that is equal to 4 % slower).
//   * Causal: the loop ends at the diagonal, only diagonal tiles are masked, waves skip tiles
//     wholly above their rows, and a workgroup takes the complementary pair of query tiles
//     (nqt-1-p, p) so every workgroup carries the same amount of work.
#pragma once
#include "dropout_gfx950.hpp"
#include "mma_gfx950.hpp"
#include "tiles_gfx950.hpp"

namespace spark {

// PAIR: the K/V buffers hold two stages of TWO 64-key tiles each instead of two single tiles: tiles
// are requested two at a time and the workgroup meets at a barrier every second round only.
template <int D, int NW = 4, bool PAIR = false> struct FwdCfg {
  static constexpr int BM = 32 * NW;  // query rows per workgroup (32 per wave)
  static constexpr int BN = 64;   // keys per iteration
  static constexpr int ROWB = lds_row<D> * 2;  // bytes per (swizzled, unpadded) row
  static constexpr int TILE = BN * ROWB;  // one of K, V
  static constexpr int STAGE = 2 * TILE;  // power of two: the buffer is switched by one XOR
  static constexpr int OSTR = lds_row<D> * 2 + 16;  // epilogue staging row stride
  static constexpr int SLOTS = PAIR ? 4 : 2;  // tiles resident or in flight
  static constexpr int SMEM = SLOTS * STAGE > NW * 32 * OSTR ? SLOTS * STAGE : NW * 32 * OSTR;  // tiles / epilogue
  static_assert((STAGE & (STAGE - 1)) == 0, "XOR buffer switch");
};

// Workgroups per CU: at D = 64 three of four waves, which costs the causal kernel with dropout 8 of its 176 registers
// (us, 256 heads x 2048 256 -> 236); at D = 128 the registers allow two.
template <typename T, int D, bool CAUSAL, bool DROP, int NW = 4, bool PAIR = false>
__global__ __launch_bounds__(64 * NW, NW == 4 ? (D == 64 ? 3 : 2) : 1) void mha_fwd_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    T* __restrict__ O, float* __restrict__ LSE, TensorMap mq, TensorMap mk, TensorMap mv,
    TensorMap mo, int H, int Nq, int Nk, int dh, int nqt, int paired, float scale_log2, Dropout dr) {
  using F = Frag<T>;
  using v8 = typename F::v8;
  using v4 = typename F::v4;
  using C = FwdCfg<D, NW, PAIR>;
  constexpr int KS = D / 16;   // k-steps of the score contraction
  constexpr int DT = D / 32;   // 32-row tiles of O^T
  constexpr int CPR = lds_row<D> / 8;  // 16-byte chunks per row of a tile
  static_assert(2 * DT == KS, "as many products of S as of O per half");

  // Causal kernels hold their read offsets in few registers: with dropout they otherwise spill (fp16, d = 128, 512
  // heads x 512 72.3 -> 77.0 us; without dropout equal).  A spilled value that is reloaded in front of the loop
  // makes the compiler wait, inside it, for every outstanding vector memory operation, that is for the tile the
  // round has just requested.
  using LaneOffsets = std::conditional_t<CAUSAL, SwzLaneLean<D>, SwzLane<D>>;
  SPARK_LDS char* const smem = lds_origin();

  // uniform: the rows of the wave, its loop limits and its share of the loads then take scalar registers.  (With that and
  // the lane index read anew in the epilogue, 17 ... 25 vector registers less and no spills: causal d = 64 128 x 1024
  // 31.8 -> 29.3 us, d = 80 36 x 1333 29.4 -> 27.1, d = 64 96 x 512 14.4 -> 13.2.)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr Lanes LANES = DROP && (D == 64 || NW == 8) ? FAR : IN_ORDER;
  const int g = lane >> 5, c32 = column_row<LANES>(lane);
  const uint32_t k_row_bytes = (uint32_t)mk.row * 2, v_row_bytes = (uint32_t)mv.row * 2;
  const uint32_t k_lane_src = dma_lane_src<D>(wave & 3, lane, k_row_bytes, dh);
  const uint32_t v_lane_src = dma_lane_src<D>(wave & 3, lane, v_row_bytes, dh);

  // Work items.  Non-causal, or a causal grid too small for pairs: one query tile per workgroup.
  // Otherwise a causal workgroup takes the pair of tiles (nqt-1-p, p), whose loop lengths add up to
  // the same total for every p, so that all workgroups carry equal work and the launch has no
  // tail of long tiles.
  const int items = paired ? causal_items<CAUSAL>(nqt) : nqt;
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int head = logical / items;
  const int item = logical - head * items;

  // Nq query rows and Nk key rows per head (equal for self-attention; causal needs them equal)
  const T* Qh = Q + head_base(mq, head, H);
  const T* Kh = K + head_base(mk, head, H);
  const T* Vh = V + head_base(mv, head, H);

  for (int rep = 0; rep < (CAUSAL && paired ? 2 : 1); ++rep) {
    const int qt = CAUSAL && rep == 0 ? nqt - 1 - item : item;
    if (CAUSAL && rep == 1) {
      if (qt == nqt - 1 - item) break;  // odd tile count: the middle tile has no partner
      __syncthreads();                  // the first tile's epilogue is done with the LDS
    }

    const int q0 = qt * C::BM + wave * 32;  // first query row of this wave
    const int qrow = q0 + c32;              // this lane's query row
    const int qrow_c = qrow < Nq ? qrow : Nq - 1;

    v8 qf[KS];
    load_row_frags(qf, Qh + (size_t)qrow_c * (size_t)mq.row, g, dh);

    int kv_end = Nk;
    if (CAUSAL) {
      const int lim = (qt + 1) * C::BM;
      kv_end = lim < Nk ? lim : Nk;
    }
    const int nt = (kv_end + C::BN - 1) / C::BN;

    // K / V tiles: global -> LDS directly; rows past the end of the sequence arrive as zeros.  Tile t lives in slot
    // t mod SLOTS.
    const BufView kview(Kh, head_span_bytes(mk, Nk, dh)), vview(Vh, head_span_bytes(mv, Nk, dh));
    auto fetch_k = [&](int t) {  // four waves move a tile
      if (t >= nt || (NW > 4 && wave >= 4)) return;
      tile_dma<D, C::BN>(kview, t * C::BN, smem + (t & (C::SLOTS - 1)) * C::STAGE, wave, k_lane_src, k_row_bytes);
    };
    auto fetch_v = [&](int t) {
      if (t >= nt || (NW > 4 && wave >= 4)) return;
      tile_dma<D, C::BN>(vview, t * C::BN, smem + (t & (C::SLOTS - 1)) * C::STAGE + C::TILE, wave, v_lane_src,
                         v_row_bytes);
    };
    LaneOffsets off(lane);  // read offsets: rows of K tile i, columns of V tile i - 1
    off.flip_tr((C::SLOTS - 1) * C::STAGE);

    f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    // reference of the row's exponentials (log2 domain).  Finite, so that a masked score (-inf)
    // minus the reference is -inf and not NaN before the first valid key has set it.
    float m_run = -1e30f;
    float l_run = 0.f;        // running row sum over this lane's keys only (halves merged at the end)

    fetch_k(0);
    if (PAIR) {
      fetch_k(1);
      fetch_v(0);
    }
    // The Q fragments must have arrived before the loop: otherwise the waits for them would sit
    // inside the loop body.
    wait_vmem_all();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]));
    __syncthreads();

    // last key this lane's query attends to, less the 4 g that every register's key contains: the mask is one
    // compare with a constant per score (with both limits compared, four instructions; us, causal, d = 64, 256
    // heads x 512 22.8 -> 21.6, d = 80, 36 x 1333 35.9 -> 31.9)
    const int last_key = (CAUSAL && qrow < Nk ? qrow : Nk - 1) - 4 * g;

    // Carried from round to round: raw scores of the second half of tile i - 1, P of its first half and their sum.
    f32x16 s0, s1;
    v8 pf0[2];
    float rs0 = 0.f;

    // Round i of the loop:
    //   S_0(i), O += P_0(i-1) V_0(i-1)   ||  exponentials of half 1 of tile i-1
    //   S_1(i), O += P_1(i-1) V_1(i-1)   ||  exponentials of half 0 of tile i
    // The fences keep the scheduler from regrouping the instructions.
    // FIRST: there is no tile i-1; LAST: no tile i.  MASKED for tiles that the diagonal or the end of the keys
    // crosses: compiled apart, since the compiler evaluates a run-time mask for every score of every tile.
    auto round = [&](const int i, auto first_tag, auto last_tag, auto masked_tag) {
      constexpr bool FIRST = decltype(first_tag)::value, LAST = decltype(last_tag)::value;
      constexpr bool MASKED = decltype(masked_tag)::value;
      SPARK_LDS const char* kb = smem;  // + off.* (which carry the slot)
      SPARK_LDS const char* vb = smem + C::TILE;

      // Step u (0 .. 2 KS - 1) has one MFMA of S (half u / KS, k-step u % KS) and one of O (16 keys u / DT, d-tile
      // u % DT); operands are read PF steps ahead (with four, kernels spill; causal, two and three are equal).
      constexpr int PF = CAUSAL ? 2 : 3;
      v8 kf[PF], vf[PF];
      auto load_step = [&](int u) {
        if (!LAST) kf[u % PF] = lds_read16<v8>(kb, off.row_at(u % KS) + (u / KS) * 32 * C::ROWB);
        if (!FIRST) {
          const int ro = (u / DT) * 16 * C::ROWB;
          vf[u % PF] = read_tr_pair<T>(vb, off.tr_at(0, u % DT) + ro, off.tr_at(1, u % DT) + ro);
        }
      };

      float t[16];
      // Online softmax (Eq. 3) with a lazy reference point.  P is formed against the current
      // reference m_run straight away, WITHOUT computing the row maximum first; the row sum of the
      // result (needed anyway) tells whether the reference was too low: if no lane's partial sum
      // exceeds 2^8, no P exceeds 2^8 either, which fp32 sums and the 16-bit MFMA operand hold
      // without loss, and the reference stays (the final O = acc / l and LSE = m + log l do not
      // depend on it).  Otherwise (the first tile, and afterwards only when a row's maximum grows
      // by more than ~2^8) the maximum is computed after all, the reference moved there, the
      // accumulators rescaled by exp(m_pre - m_cur) as in Eq. 3, and the half's P formed again.
      // key0: first key of the half.
      auto score = [&](const f32x16& s, int r, int key0) {
        return MASKED && 8 * (r / 4) + (r % 4) > last_key - key0 ? -INFINITY : s[r];
      };
      auto exp_elem = [&](const f32x16& s, int r, int key0, float& rs) {
        t[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(score(s, r, key0), scale_log2, -m_run));
        rs += t[r];
        // materialise here, between the MFMAs around this call: nothing uses the values before the
        // end of the half, and the compiler otherwise moves the arithmetic there
        asm volatile("" : "+v"(t[r]), "+v"(rs));
      };
      // Returns the rescale factor.
      auto renorm = [&](const f32x16& s, int key0, float& rs) {
        float mx = score(s, 0, key0);
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, score(s, r, key0));
        mx = half_pair_max(mx) * scale_log2;  // scale > 0 commutes with the maximum
        const float m_new = fmaxf(m_run, mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
        rs = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) exp_elem(s, r, key0, rs);
        return alpha;
      };
      // The generator's rounds sit between the MFMAs, too, but in the causal kernel at d = 64, which has no registers for
      // their state there (us, 256 heads x 512 30.6 -> 28.6, 256 x 2048 244.8 -> 238.7, 128 x 1024 44.2 -> 41.1).
      constexpr bool SPREAD = DROP && !(D == 64 && CAUSAL);
      // Dropout acts on P after the row sums are taken: dropped entries become zero in the
      // operand of O += P V; the survivors' factor 1/(1-p) is applied once, to O, at the end.
      auto finish_half = [&](v8 (&pf)[2], Philox& rng) {
        if (DROP) {
          uint32_t kb4[4];
          if (!SPREAD) {
#pragma unroll
            for (int q = 0; q < 10; ++q) philox_round<true>(rng, dr.key0, dr.key1, q);
          }
          keep_query_lane_finish<LANES>(rng, lane, kb4);
          // converted first, then dropped in pairs: six instructions for four entries, where a compare and a
          // select of each fp32 value are eight
          uint32_t pk[2][4];
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            uint32_t mask[2];
            keep_pairs(keep_flags(kb4[a], dr), mask);
#pragma unroll
            for (int x = 0; x < 2; ++x)
              pk[a / 2][2 * (a % 2) + x] = pack2<T>(t[4 * a + 2 * x], t[4 * a + 2 * x + 1]) & mask[x];
          }
          pf[0] = join_pairs<T>(pk[0]);
          pf[1] = join_pairs<T>(pk[1]);
        } else {
          pf[0] = pack8<T>(&t[0]);
          pf[1] = pack8<T>(&t[8]);
        }
      };
      // One half of the round: steps KS h .. KS h + KS - 1, between them the exponentials of `s` and the rounds of the
      // dropout generator for them (EXP).
      auto half = [&](auto h_tag, f32x16& s_new, const f32x16& s, int key0, float& rs, const v8 (&pf)[2], Philox& rng) {
        constexpr int h = decltype(h_tag)::value;
        constexpr bool EXP = h == 0 ? !FIRST : !LAST;
        if (DROP && EXP) {
          rng = keep_query_lane_begin<LANES>(dr, head, qrow, key0, lane);
          // Opaque there: otherwise products of the first rounds are held across the loop, spilled, and their reload
          // awaited inside it together with the tile just requested (us, 256 heads x 512 25.2 -> 24.7, 512 x 300
          // 27.9 -> 27.0, equal at 256 x 2048).
          if (!SPREAD) asm volatile("" : "+v"(rng.c0), "+v"(rng.c1));
        }
        if (!LAST) {
#pragma unroll
          for (int r = 0; r < 16; ++r) s_new[r] = 0.f;
        }
#pragma unroll
        for (int e = 0; e < KS; ++e) {
          const int u = KS * h + e;
          const int x0 = e * 16 / KS, x2 = (e + 1) * 16 / KS, x1 = (x0 + x2) / 2;
          if (!LAST) s_new = F::mfma(kf[u % PF], qf[e], s_new);
          if (EXP) {
#pragma unroll
            for (int x = x0; x < x1; ++x) exp_elem(s, x, key0, rs);
          }
          if (SPREAD && EXP) {
#pragma unroll
            for (int q = e * 10 / KS; q < (e + 1) * 10 / KS; ++q) philox_round<true>(rng, dr.key0, dr.key1, q);
          }
          sched_fence();
          if (!FIRST) o[u % DT] = F::mfma(vf[u % PF], pf[(u / DT) & 1], o[u % DT]);
          if (EXP) {
#pragma unroll
            for (int x = x1; x < x2; ++x) exp_elem(s, x, key0, rs);
          }
          if (u + PF < 2 * KS) load_step(u + PF);
          sched_fence();
        }
      };
      Philox rng{0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < PF; ++u) load_step(u);
      sched_fence();
      v8 pf1[2];
      float rs1 = 0.f;
      const int kp = (i - 1) * C::BN + 32, kc = i * C::BN;
      half(std::integral_constant<int, 0>{}, s0, s1, kp, rs1, pf0, rng);
      if (!FIRST) {
        if (__any(!(rs1 <= 256.0f))) rs0 *= renorm(s1, kp, rs1);  // also true for inf / NaN
        l_run += rs0 + rs1;
        finish_half(pf1, rng);
        sched_fence();
      }
      rs0 = 0.f;
      half(std::integral_constant<int, 1>{}, s1, s0, kc, rs0, pf1, rng);
      if (!LAST) {
        if (__any(!(rs0 <= 256.0f))) renorm(s0, kc, rs0);
        finish_half(pf0, rng);
        sched_fence();
      }
    };
    // Requests of round i, into slots everybody left before the last barrier: the next round's tiles, or with PAIR, in
    // even rounds, those of the next two.
    auto request = [&](int i) {
      if (PAIR) {
        if ((i & 1) == 0) {
          fetch_k(i + 2);
          fetch_k(i + 3);
          fetch_v(i + 1);
          fetch_v(i + 2);
        }
      } else {
        fetch_k(i + 1);
        fetch_v(i);
      }
    };
    auto end_round = [&](int i) {
      // next slot: 0 -> 1 -> 2 -> 3 -> 0 with PAIR (XOR with STAGE, then with 3 STAGE), else 0 <-> 1
      off.flip_rows(PAIR && (i & 1) ? 3 * C::STAGE : C::STAGE);
      off.flip_tr(PAIR && !(i & 1) ? 3 * C::STAGE : C::STAGE);
      if (!PAIR || (i & 1) || i >= nt) {
        wait_vmem_all();  // requested at the top of this round (pair of rounds)
        __syncthreads();
      }
    };
    // Tiles [0, n_plain) end within the keys and, if causal, at or below the diagonal for every
    // row of this wave, and tiles from n_wave on are wholly above it.  Both differ between the waves of a workgroup; the
    // number of rounds, and with it the number of barriers, does not.
    int n_plain = Nk / C::BN, n_wave = nt;
    if (CAUSAL) {
      if ((q0 + 1) / C::BN < n_plain) n_plain = (q0 + 1) / C::BN;
      if ((q0 + 31) / C::BN + 1 < n_wave) n_wave = (q0 + 31) / C::BN + 1;
    }
    if (n_plain > nt) n_plain = nt;
    using no = std::false_type;
    using yes = std::true_type;
    request(0);
    if (n_plain > 0)
      round(0, yes{}, no{}, no{});
    else
      round(0, yes{}, no{}, yes{});
    end_round(0);
    int i = 1;
    for (; i < n_plain; ++i) {
      request(i);
      round(i, no{}, no{}, no{});
      end_round(i);
    }
    for (; i < n_wave; ++i) {
      request(i);
      round(i, no{}, no{}, yes{});
      end_round(i);
    }
    request(i);
    if (n_plain == n_wave)
      round(i, no{}, yes{}, no{});
    else
      round(i, no{}, yes{}, yes{});
    end_round(i);
    for (++i; i <= nt; ++i) {
      request(i);
      end_round(i);
    }

    // Epilogue: normalise, round once, transpose through this wave's LDS slice, store rows.
    // The lane index is read anew: addresses formed from it would otherwise be held in registers across the loop.
    int elane = lane;
    asm volatile("" : "+v"(elane));
    const int eg = elane >> 5, ec32 = column_row<LANES>(elane);
    l_run = half_pair_sum(l_run);
    const float inv = (DROP ? dr.rescale : 1.0f) / l_run;
    SPARK_LDS char* ob = smem + wave * 32 * C::OSTR;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        v4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[e] = (T)(o[dt][r4 * 4 + e] * inv);
        lds_write(ob, ec32 * C::OSTR + (dt * 32 + 8 * r4 + 4 * eg) * 2, pk);
      }
    T* Oh = O + head_base(mo, head, H);
    constexpr int RPP = 64 / CPR;  // rows per pass of the wave
#pragma unroll
    for (int p = 0; p < 32 / RPP; ++p) {
      const int row = p * RPP + elane / CPR, cc = elane % CPR;
      const u32x4 v = lds_read16<u32x4>(ob, row * C::OSTR + cc * 16);
      if (q0 + row < Nq && cc * 8 < dh)
        *reinterpret_cast<u32x4*>(Oh + (size_t)(q0 + row) * (size_t)mo.row + cc * 8) = v;
    }
    if (eg == 0 && q0 + ec32 < Nq)
      LSE[(size_t)head * Nq + q0 + ec32] = (m_run + __builtin_amdgcn_logf(l_run)) * 0.6931471805599453f;
  }  // rep
}

}  // namespace spark
