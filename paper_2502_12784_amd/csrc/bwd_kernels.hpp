// Attention backward for gfx950 (paper Sec. 3.3, Eq. 4), two kernels on one stream, in this order:
//
//   mha_bwd_dq_kernel        : one workgroup per tile of 128 queries; first forms
//                              D_i = sum_k dO_ik O_ik (the paper's "dPsum") for its rows from the
//                              fragments it loads anyway and writes D and LSE*log2(e) to the
//                              workspace, then loops over key tiles, recomputes P and dS and
//                              accumulates dQ = scale * dS K.
//   mha_bwd_dkdv_pipe_kernel : one workgroup per tile of 128 keys, loops over query tiles,
//                              recomputes P = exp(S - LSE), accumulates dV = P^T dO and
//                              dK = scale * dS^T Q in registers, writes them once (as in
//                              Sec. 3.3, where each thread block owns a slice of dK and dV).
//                              Software-pipelined inside the wave.  Reads D and LSE*log2(e) from
//                              the workspace.
//
// The paper adds every block's dQ contribution into HBM with atomic adds.  Here dQ has its
// own pass with the forward's loop structure instead: it costs two recomputed contractions
// (7 executed for 5 counted) but needs no fp32 dQ buffer to zero and convert, no atomics, and
// gives bitwise reproducible gradients.  Both variants exist and were timed on the same inputs
// (the atomic one is in bwd_atomic_kernels.hpp): with 128 keys per workgroup it adds N/128 fp32
// values per dQ element, 2.2 GB for N = 4096, d = 128, 64 heads, causal; MI355X performs
// device-scope atomics at the memory side, at 1.3 TB/s, so that variant takes 1.75 ms where these
// two kernels take 0.91 ms.
//
// Register layouts follow mma_gfx950.hpp.  In the dK/dV kernels the score tile is computed as
// S = Q K^T (lane = key column, registers = query rows) so that P and dS, packed to 16 bits,
// are directly the B operands of dV^T = dO^T P and dK^T = Q^T dS; the dO^T / Q^T operands
// come from the row-major LDS tiles through transposing reads.  In the dQ kernel everything
// is transposed as in the forward (lane = query column), so LSE_i and D_i are per-lane
// scalars and dS^T is directly the B operand of dQ^T = K^T dS^T.
#pragma once
#include "dropout_gfx950.hpp"
#include "mma_gfx950.hpp"
#include "tiles_gfx950.hpp"

namespace spark {

// ---------------------------------------------------------------------------------------
// dK, dV: software-pipelined.
//
// At d = 128 the accumulators (dK^T, dV^T: 128 registers) and the resident K / V fragments
// (64) leave room for one wave per SIMD only, so nothing but the wave itself can hide its
// softmax arithmetic and LDS latency.  (At d = 64 two workgroups share a CU and the same
// schedule still pays: measured 9 % faster on causal N = 8192 than an unpipelined loop.)  A wave issues in order, and an MFMA occupies the matrix
// core for ~34 cycles while the wave can issue about half a dozen other instructions; so the
// loop is skewed by one 32-query step and written as units of {one MFMA, a few VALU / LDS
// instructions}:
//   region 1:  scores of step i+1 (MFMA)   ||  second half of P, dS of step i      (VALU)
//   region 2:  dV, dK of step i   (MFMA)   ||  first half of P, dS of step i+1     (VALU)
// Because step i+1 may lie in the next 64-query stage, stages live in a ring of three LDS
// slots: stage m+1 is resident while stage m is processed, and stage m+2 is being written by
// direct global->LDS loads (no staging registers, no LDS store instructions).  No step is
// skipped: blocks above the causal diagonal are masked to zero (first two stages of a workgroup
// only); rows past the end of the sequence read as zeros (Q = dO = 0), so they add nothing.
// ---------------------------------------------------------------------------------------
template <int D> struct BwdKvPipeCfg {
  static constexpr int BN = 128, BM = 64, SLOTS = 3;
  static constexpr int ROWB = lds_row<D> * 2;
  static constexpr int TILE = BM * ROWB;
  static constexpr int STAGE = 2 * TILE;
  static constexpr int STAT = 2 * BM * 4;  // LSE*log2(e) and D of the stage's rows
  static constexpr int OSTR = lds_row<D> * 2 + 16;
  static constexpr int STAT0 = SLOTS * STAGE;  // LDS = [slot 0..2 | stat 0..2]
  static constexpr int SMEM = SLOTS * STAGE + SLOTS * STAT;
  static_assert(4 * 32 * OSTR <= SLOTS * STAGE, "epilogue staging must fit");
};

// dS of one entry under dropout in the dK/dV kernels, P o (M o dP + d): pe = P, pm = M o P, d = -D (1-p).  With
// the mask already in pm one instruction is saved, but only where dP cannot overflow: 0 * inf would turn a dropped
// entry whose dP is past fp32's range into NaN.  (bf16 without that saving, a select then: dK/dV 639 -> 648 us at 64
// heads x 4096 causal, d = 128.)  keep: ones or zeros.
template <typename T>
static __device__ __forceinline__ float dropout_ds(uint32_t keep, float pe, float pm, float dp, float d) {
  if (Frag<T>::FINITE_DOT) return __builtin_fmaf(pm, dp, pe * d);
  return pe * (keep_float(keep, dp) + d);
}

// The workgroup's part: key tile `item` of `head`, and its partner if the causal tiles are paired.
template <typename T, int D, bool CAUSAL, bool DROP, Lanes M, bool COMPARE = false>
static __device__ __forceinline__ void bwd_dkdv_pipe(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const T* __restrict__ dO, const float* __restrict__ LSE2, const float* __restrict__ Dws,
    T* __restrict__ dK, T* __restrict__ dV, const TensorMap& mq, const TensorMap& mk, const TensorMap& mv,
    const TensorMap& mdo, const TensorMap& mdk, const TensorMap& mdv, int H, int Nq, int Nk, int dh, int nkt,
    int paired, float scale, const Dropout& dr, int head, int item) {
  using F = Frag<T>;
  using v8 = typename F::v8;
  using C = BwdKvPipeCfg<D>;
  constexpr int KS = D / 16, DT = D / 32;

  // D = 64: few offset registers; with dropout the kernel needs 247 to 254 of its 256 and spilled with all of them
  // (dK/dV, us, 256 causal heads x 512 44.1 -> 41.4; without dropout 0 ... 1 % less)
  using LaneOffsets = std::conditional_t<D == 64, SwzLaneLean<D>, SwzLane<D>>;
  SPARK_LDS char* const smem = lds_origin();

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, c32 = column_row<M>(lane);

  const T* Kh = K + head_base(mk, head, H);
  const T* Vh = V + head_base(mv, head, H);
  const BufView qview(Q + head_base(mq, head, H), head_span_bytes(mq, Nq, dh));
  const BufView doview(dO + head_base(mdo, head, H), head_span_bytes(mdo, Nq, dh));
  const uint32_t q_row_bytes = (uint32_t)mq.row * 2, do_row_bytes = (uint32_t)mdo.row * 2;
  const BufView lview(LSE2 + (size_t)head * Nq, (uint32_t)Nq * 4), dview(Dws + (size_t)head * Nq, (uint32_t)Nq * 4);
  const uint32_t q_lane_src = dma_lane_src<D>(wave, lane, q_row_bytes, dh);
  const uint32_t do_lane_src = dma_lane_src<D>(wave, lane, do_row_bytes, dh);
  const float scale_log2 = scale * 1.4426950408889634f;

  for (int rep = 0; rep < (CAUSAL && paired ? 2 : 1); ++rep) {
    const int kt = rep == 0 ? item : nkt - 1 - item;  // the long tile first
    if (CAUSAL && rep == 1) {
      if (kt == item) break;  // odd tile count: the middle tile has no partner
      __syncthreads();        // the first tile's epilogue is done with the LDS
    }
    const int k0w = kt * C::BN + wave * 32;
    const int krow = k0w + c32;
    const int krow_c = krow < Nk ? krow : Nk - 1;

    v8 kf[KS], vf[KS];
    const T* const kp = Kh + (size_t)krow_c * (size_t)mk.row;
    const T* const vp = Vh + (size_t)krow_c * (size_t)mv.row;
    if constexpr (!CAUSAL && D < 128) {  // us, 150 heads x 300, d = 56 16.7 -> 16.3, d = 64 96 x 512 equal
      load_row_chunks(kf, kp, g, dh);
      load_row_chunks(vf, vp, g, dh);
    } else {
      load_row_frags(kf, kp, g, dh);
      load_row_frags(vf, vp, g, dh);
    }

    f32x16 dk[DT], dv[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) { dk[dt][r] = 0.f; dv[dt][r] = 0.f; }

    const int ns = (Nq + C::BM - 1) / C::BM;
    const int s_begin = CAUSAL ? (kt * C::BN) / C::BM : 0;

    const LaneOffsets lane_off(lane);  // offsets inside slot 0
    const int lane_stat = C::STAT0 + 16 * g;

    // global -> LDS slot, asynchronously (completion is awaited with wait_vmem_all + barrier)
    auto fetch_stage = [&](int m, int slot) {
      SPARK_LDS char* sb = smem + slot * C::STAGE;
      tile_dma<D, C::BM>(qview, m * C::BM, sb, wave, q_lane_src, q_row_bytes);
      tile_dma<D, C::BM>(doview, m * C::BM, sb + C::TILE, wave, do_lane_src, do_row_bytes);
      // 64 floats of LSE*log2(e) (wave 0) and of D (wave 1): 4 bytes per lane
      SPARK_LDS char* st = smem + C::STAT0 + slot * C::STAT;
      if (wave == 0) lview.load4_to_lds(st, lane * 4, (uint32_t)m * C::BM * 4);
      if (wave == 1) dview.load4_to_lds(st + C::BM * 4, lane * 4, (uint32_t)m * C::BM * 4);
    };

    // LDS read offsets of the step whose scores are being formed (row reads, statistics) ...
    LaneOffsets offA(lane_off);
    int statA;
    // ... and of the step whose dV / dK are being accumulated (transposing reads)
    LaneOffsets offC(lane_off);
    auto point_A = [&](int slot) {
      offA.point_rows(lane_off, slot * C::STAGE);
      statA = lane_stat + slot * C::STAT;
    };
    auto point_C = [&](int slot) { offC.point_tr(lane_off, slot * C::STAGE); };

    v8 fa[2][4];
    auto load_agroup = [&](int gi, int sub) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        fa[gi & 1][2 * e] = lds_read16<v8>(smem, offA.row_at(2 * gi + e) + sub * 32 * C::ROWB);
        fa[gi & 1][2 * e + 1] = lds_read16<v8>(smem + C::TILE, offA.row_at(2 * gi + e) + sub * 32 * C::ROWB);
      }
    };
    // statistics of 8 of the 16 query rows a lane holds (half = 0: registers 0..7, 1: 8..15) of the
    // step offA / statA point at
    auto load_stats = [&](f32x4 (&l)[2], f32x4 (&d)[2], int sub, int half) {
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const int o = statA + (sub * 32 + 8 * (2 * half + x)) * 4;
        l[x] = lds_read16<f32x4>(smem, o);
        if (DROP) d[x] = lds_read16<f32x4>(smem, o + C::BM * 4);
      }
    };
    // RING (dropout at D = 64): the statistics go through two slots of four query rows each, refilled as soon as their
    // four elements are done, instead of being held for a half step (8 rows) and the next one.  With that the kernel
    // fits 256 registers and two workgroups share a CU (us, 256 heads x 2048 852 -> 660, causal 509 -> 386).
    constexpr bool RING = DROP && D == 64;
    auto load_quad = [&](f32x4 (&l)[2], f32x4 (&d)[2], int stat, int sub, int x) {
      const int o = stat + (sub * 32 + 8 * x) * 4;
      l[x & 1] = lds_read16<f32x4>(smem, o);
      d[x & 1] = lds_read16<f32x4>(smem, o + C::BM * 4);
    };
    // The workspace holds -D.  Without dropout dS = P o (dP - D) needs no subtraction: the dP
    // accumulator of a step starts from -D of its 16 query rows instead of from zero (the four
    // 16-byte reads below deliver them in exactly the accumulator's row order), so the MFMAs
    // themselves leave dP - D there.  (Under dropout the mask must act on dP alone, so the
    // accumulator starts from zero and -D is added afterwards.)
    auto dp_start = [&](int sub) {
      f32x16 c;
      if (DROP) {
#pragma unroll
        for (int r = 0; r < 16; ++r) c[r] = 0.f;
      } else {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const f32x4 v = lds_read16<f32x4>(smem, statA + (sub * 32 + 8 * x) * 4 + C::BM * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) c[4 * x + e] = v[e];
        }
      }
      return c;
    };
    constexpr int NG = KS / 2;
    constexpr int NTG = DT;  // the 2 DT pairs of operands (one dO^T, one Q^T) of dV and dK, two to a group
    v8 ft[2][4];
    // half e of transposed-fragment group tg (one pair of operands: four reads); issued in halves so that no
    // MFMA slot carries more than a few LDS reads
    auto load_thalf = [&](int tg, int sub, int e) {
      const int kk = (2 * tg + e) / DT, dt = (2 * tg + e) % DT;
      const int o = sub * 32 * C::ROWB + kk * 16 * C::ROWB;
      ft[tg & 1][2 * e] = read_tr_pair<T>(smem + C::TILE, offC.tr_at(0, dt) + o, offC.tr_at(1, dt) + o);
      ft[tg & 1][2 * e + 1] = read_tr_pair<T>(smem, offC.tr_at(0, dt) + o, offC.tr_at(1, dt) + o);
    };

    uint32_t strip = 0;
    // One element of P and dS from finished scores: the unit of VALU work that is placed between
    // MFMAs.  r8 = register index within the half (0..7).  ahead: how far the lane's key lies behind the
    // step's first query of this lane, so that the causal mask is one compare with a constant per element.
    // Under dropout (kb: the step's decision bytes) the dV operand is the dropped P, and
    // dS = r P o (M o dPraw - D (1-p)): the workspace holds D (1-p), r goes into the final scales.
    auto softmax_elem = [&](const f32x16& s, const f32x16& dp, int half, int r8, const f32x4 (&l)[2],
                            const f32x4 (&d)[2], int ahead, bool mask, const uint32_t (&kb)[4], float* p,
                            float* ds, uint32_t (&pk_p)[4], uint32_t (&pk_ds)[4]) {
      const int r = 8 * half + r8;
      float pe = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], scale_log2, -l[r8 >> 2][r8 & 3]));
      if (mask) pe = ahead > 8 * (r / 4) + (r % 4) ? 0.f : pe;
      if (DROP) {
        uint32_t keep;
        if (COMPARE) {
          keep = keep_reg(kb, r, dr.thr) ? 0xFFFFFFFFu : 0u;
        } else {
          if ((r & 3) == 0) strip = keep_strip(kb[r >> 2], dr);  // in the slot of the first of four entries
          keep = keep_mask(strip, r & 3);
        }
        p[r8] = keep_float(keep, pe);
        asm volatile("" : "+v"(p[r8]));  // keeps the mask in front of the packed conversion
        ds[r8] = dropout_ds<T>(keep, pe, p[r8], dp[r], d[r8 >> 2][r8 & 3]);
      } else {
        p[r8] = pe;
        ds[r8] = pe * dp[r];  // the accumulator started from -D
      }
      // materialise dS here, between the MFMAs around this call: it is not used before the packing
      // at the end of the region, and the compiler would otherwise move its arithmetic there,
      // where no MFMA hides it
      asm volatile("" : "+v"(ds[r8]));
      if (r8 & 1) {  // a pair is complete: convert it now
        pk_p[r8 >> 1] = pack2<T>(p[r8 - 1], p[r8]);
        pk_ds[r8 >> 1] = pack2<T>(ds[r8 - 1], ds[r8]);
      }
    };
    // In fp16 with dropout at D = 64, rows far apart, there is one register too few for krow - 4 g across the loop: formed anew
    // where a mask needs it.  Spilled, it is awaited inside the loop, together with the stage just requested (us, backward,
    // 512 heads x 192 44.5 -> 42.3, 256 x 512 70.2 -> 68.4).  The other kernels hold it and are slower without it (bf16
    // 64 x 2048 162.4 -> 164.4, 140 x 512 60.1 -> 60.5; fp16, rows in order, d = 48 140 x 512 55.0 -> 55.4).
    constexpr bool ANEW = DROP && D == 64 && F::FINITE_DOT && M == FAR;
    auto ahead_of = [&](int q0s) {
      int l = lane;
      if (ANEW) asm volatile("" : "+v"(l));
      return ANEW ? k0w - q0s + column_row<M>(l) - 4 * (l >> 5) : krow - q0s - 4 * g;
    };
    uint32_t kbCur[4] = {0, 0, 0, 0}, kbNew[4] = {0, 0, 0, 0};  // decision bytes of the current / next step

    // ---- prologue: stages s_begin and s_begin+1 resident, scores of the first step formed ----
    fetch_stage(s_begin, 0);
    if (s_begin + 1 < ns) fetch_stage(s_begin + 1, 1);
    wait_vmem_all();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(kf[ks]), "+v"(vf[ks]));
    __syncthreads();

    point_A(0);
    point_C(0);
    f32x16 sX, dpX, sY, dpY;
    f32x4 lL[2], dL[2], lH[2], dH[2];  // statistics: first half of the next step / second half of the current
#pragma unroll
    for (int r = 0; r < 16; ++r) sX[r] = 0.f;
    dpX = dp_start(0);
    load_agroup(0, 0);
    load_agroup(1, 0);
    load_stats(lL, dL, 0, 0);
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        sX = F::mfma(fa[gi & 1][2 * e], kf[2 * gi + e], sX);
        dpX = F::mfma(fa[gi & 1][2 * e + 1], vf[2 * gi + e], dpX);
      }
      if (gi + 2 < NG) load_agroup(gi + 2, 0);
      sched_fence();
    }
    // Every step requests the first two fragment groups of its successor half-way through its own dV / dK region, so
    // that no step starts by waiting for LDS (D = 128, causal 64 heads x 4096: backward -3 %; D = 64, us, 32 x 8192
    // 1776 -> 1748, causal 128 x 1024 85.0 -> 83.9, both sides in one grid 24 x 1024 36.0 -> 34.6); here those
    // of step (s_begin, 1).
    load_agroup(0, 1);
    load_agroup(1, 1);
    // With more than 256 registers per lane the MFMAs deliver the scores in accumulation registers,
    // which the VALU reaches through one v_accvgpr_read per element.  Such a read co-issues with
    // executing MFMAs as long as none of them writes the register read (measured), so each element
    // is read where its softmax arithmetic sits, between the MFMAs of the following regions; the
    // two score buffers X / Y alternate so that the one being read is never the one being formed.
    // P / dS operands of the current step: registers 0..7 (pfL, dsfL) are formed one region
    // early, registers 8..15 (pfH, dsfH) while the next step's scores are on the matrix cores.
    v8 pfL, dsfL;
    {
      float p[8], ds[8];
      uint32_t pk_p[4], pk_ds[4];
      const int ahead_first = CAUSAL ? ahead_of(s_begin * C::BM) : 0;
      if (DROP) keep_bytes_key_lane<M>(dr, head, krow, s_begin * C::BM, lane, kbCur);
#pragma unroll
      for (int r = 0; r < 8; ++r)
        softmax_elem(sX, dpX, 0, r, lL, dL, ahead_first, CAUSAL, kbCur, p, ds, pk_p, pk_ds);
      pfL = join_pairs<T>(pk_p);
      dsfL = join_pairs<T>(pk_ds);
    }
    if (RING) {
      load_quad(lL, dL, statA, 0, 2);
      load_quad(lL, dL, statA, 0, 3);
    } else {
      load_stats(lH, dH, 0, 1);
    }

    // One stage: steps (m, 0) and (m, 1).  On entry sX / dpX hold the scores of (m, 0), pfL / dsfL
    // their first half and lH / dH (RING: lL / dL, quads 2 and 3) the statistics of their second half;
    // offA, statA and offC point at stage m.  On exit the same holds for (m+1, 0).
    auto stage = [&](int m, int slot, bool mask) {
      const int slot1 = slot == 2 ? 0 : slot + 1;
      const int slot2 = slot1 == 2 ? 0 : slot1 + 1;
      // stage m+2 goes into the slot that stage m-1 used; everybody left it before the last barrier
      if (m + 2 < ns) fetch_stage(m + 2, slot2);

      // One step.  cur: scores complete, first half of P / dS packed.  new: the step after it
      // (sub_new inside the stage offA / statA point at).
      auto step = [&](f32x16& s_new, f32x16& dp_new, int sub_new, int q0_new, const f32x16& s_cur,
                      const f32x16& dp_cur, int sub_cur, int q0_cur, auto&& request_next) {
        const int ahead_cur = mask ? ahead_of(q0_cur) : 0, ahead_new = mask ? ahead_of(q0_new) : 0;
        const int stat_new = statA;  // request_next may move statA on before the last of its quads is read
        // ---- region 1: scores of the next step  ||  second half of P, dS of the current step ----
        float p[8], ds[8];
        uint32_t pk_p[4], pk_ds[4];
        // dropout decisions of the next step: the ten generator rounds ride in the MFMA slots below
        Philox rng;
        if (DROP) rng = keep_key_lane_begin<M>(dr, head, krow, q0_new, lane);
        if (!RING) load_stats(lL, dL, sub_new, 0);
        load_thalf(0, sub_cur, 0);
#pragma unroll
        for (int i = 0; i < 4 * NG; ++i) {
          const int gi = i / 4, e = (i / 2) & 1;
          if ((i & 1) == 0)
            s_new = F::mfma(fa[gi & 1][2 * e], kf[2 * gi + e], s_new);
          else
            dp_new = F::mfma(fa[gi & 1][2 * e + 1], vf[2 * gi + e], dp_new);
          if ((i & 3) == 3 && gi + 2 < NG) load_agroup(gi + 2, sub_new);
          if (i == 1) load_thalf(0, sub_cur, 1);
          if (i == 2 * NG) load_thalf(1, sub_cur, 0);
          if (i == 2 * NG + 1) load_thalf(1, sub_cur, 1);
          if (i & 1) {
#pragma unroll
            for (int x = (i / 2) * 4 / NG; x < (i / 2 + 1) * 4 / NG; ++x)  // 8 elements in 2 NG slots
              softmax_elem(s_cur, dp_cur, 1, x, RING ? lL : lH, RING ? dL : dH, ahead_cur, mask, kbCur, p, ds,
                           pk_p, pk_ds);
            if (RING && (i & 3) == 3) load_quad(lL, dL, stat_new, sub_new, i / 4);  // first half of the next step
          }
          if (DROP) {
#pragma unroll
            for (int round = i * 10 / (4 * NG); round < (i + 1) * 10 / (4 * NG); ++round)
              philox_round<true>(rng, dr.key0, dr.key1, round);
          }
          sched_fence();
        }
        if (DROP) keep_key_lane_finish<M>(rng, lane, kbNew);
        const v8 pfH = join_pairs<T>(pk_p), dsfH = join_pairs<T>(pk_ds);
        if (!RING) load_stats(lH, dH, sub_new, 1);
        sched_fence();
        // ---- region 2: dV, dK of the current step  ||  first half of P, dS of the next step ----
#pragma unroll
        for (int tg = 0; tg < NTG; ++tg) {
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int slot = 2 * tg + e, kk = slot / DT, dt = slot % DT;
            dv[dt] = F::mfma(ft[tg & 1][2 * e], kk ? pfH : pfL, dv[dt]);
            dk[dt] = F::mfma(ft[tg & 1][2 * e + 1], kk ? dsfH : dsfL, dk[dt]);
            if (NTG == 2) {  // two elements a slot, of different pairs
              softmax_elem(s_new, dp_new, 0, 4 * tg + e, lL, dL, ahead_new, mask, kbNew, p, ds, pk_p, pk_ds);
              softmax_elem(s_new, dp_new, 0, 4 * tg + 2 + e, lL, dL, ahead_new, mask, kbNew, p, ds, pk_p, pk_ds);
            } else {
#pragma unroll
              for (int x = slot * 4 / NTG; x < (slot + 1) * 4 / NTG; ++x)
                softmax_elem(s_new, dp_new, 0, x, lL, dL, ahead_new, mask, kbNew, p, ds, pk_p, pk_ds);
            }
            if (tg + 2 < NTG) load_thalf(tg + 2, sub_cur, e);  // into the operands just used
            sched_fence();
          }
          if (RING) load_quad(lL, dL, stat_new, sub_new, 2 + tg);  // second half of the next step
          // the fragment buffers are free since region 1 ended; one group per slot keeps the number
          // of LDS reads in flight under the 15 the wave's counter can track
          if (tg == (NTG - 1) / 2) request_next(0);
          if (tg == (NTG + 1) / 2) request_next(1);
          sched_fence();
        }
        pfL = join_pairs<T>(pk_p);
        dsfL = join_pairs<T>(pk_ds);
        // materialise here: otherwise this arithmetic sinks to its use in the next step and
        // runs there with no MFMA to hide it
        asm volatile("" : "+v"(pfL), "+v"(dsfL));
        if (DROP) {
#pragma unroll
          for (int a = 0; a < 4; ++a) kbCur[a] = kbNew[a];
        }
      };

      // (m, 1) scores  ||  (m, 0) softmax; then (m, 0) dV / dK
#pragma unroll
      for (int r = 0; r < 16; ++r) sY[r] = 0.f;
      dpY = dp_start(1);  // statA points at stage m here
      auto request_B = [&](int part) {
        if (part == 0) point_A(slot1);  // stage m+1 has been resident since the end of stage m-1
        load_agroup(part, 0);
      };
      auto request_A = [&](int part) { load_agroup(part, 1); };
      sched_fence();
      step(sY, dpY, 1, m * C::BM + 32, sX, dpX, 0, m * C::BM, request_B);
      // (m+1, 0) scores  ||  (m, 1) softmax; then (m, 1) dV / dK
#pragma unroll
      for (int r = 0; r < 16; ++r) sX[r] = 0.f;
      dpX = dp_start(0);  // statA points at stage m + 1 by now (request_B moved it)
      sched_fence();
      step(sX, dpX, 0, (m + 1) * C::BM, sY, dpY, 1, m * C::BM + 32, request_A);

      point_C(slot1);
      wait_vmem_all();  // stage m+2 has landed (it was requested a whole stage ago)
      __syncthreads();
    };

    int m = s_begin, slot = 0;
    if (CAUSAL) {  // the diagonal crosses the first two stages only
      const int m_end = s_begin + 2 < ns ? s_begin + 2 : ns;
      for (; m < m_end; ++m) {
        stage(m, slot, true);
        slot = slot == 2 ? 0 : slot + 1;
      }
    }
    for (; m < ns; ++m) {
      stage(m, slot, false);
      slot = slot == 2 ? 0 : slot + 1;
    }

    SPARK_LDS char* ob = smem + wave * 32 * C::OSTR;
    store_transposed<T, D, C::OSTR, M>(dk, DROP ? scale * dr.rescale : scale, ob, dK + head_base(mdk, head, H), k0w,
                                    Nk, lane, (size_t)mdk.row, dh);
    store_transposed<T, D, C::OSTR, M>(dv, DROP ? dr.rescale : 1.0f, ob, dV + head_base(mdv, head, H), k0w, Nk,
                                    lane, (size_t)mdv.row, dh);
  }  // rep
}

template <typename T, int D, bool CAUSAL, bool DROP>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void mha_bwd_dkdv_pipe_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const T* __restrict__ dO, const float* __restrict__ LSE2, const float* __restrict__ Dws,
    T* __restrict__ dK, T* __restrict__ dV, TensorMap mq, TensorMap mk, TensorMap mv, TensorMap mdo,
    TensorMap mdk, TensorMap mdv, int H, int Nq, int Nk, int dh, int nkt, int paired, float scale,
    Dropout dr) {
  const int items = paired ? causal_items<CAUSAL>(nkt) : nkt;  // causal: key tiles (p, nkt-1-p)
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int head = logical / items;
  // decisions of dropout by a compare and a select each in fp16 at 128 columns, causal (backward, us, masks -> so: 140 x 512,
  // d = 112 101.3 -> 100.5, d = 128 140 x 700 135.7 -> 134.8; without the causal mask, d = 112 115.7 -> 116.5)
  constexpr bool COMPARE = D == 128 && CAUSAL && Frag<T>::FINITE_DOT;
  bwd_dkdv_pipe<T, D, CAUSAL, DROP, IN_ORDER, COMPARE>(Q, K, V, dO, LSE2, Dws, dK, dV, mq, mk, mv, mdo, mdk, mdv, H, Nq,
                                                       Nk, dh, nkt, paired, scale, dr, head, logical - head * items);
}

// With dropout, the rows far apart in the lanes (column_row); the rule is far_rows.
template <typename T, int D, bool CAUSAL>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void mha_bwd_dkdv_pipe_far_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const T* __restrict__ dO, const float* __restrict__ LSE2, const float* __restrict__ Dws,
    T* __restrict__ dK, T* __restrict__ dV, TensorMap mq, TensorMap mk, TensorMap mv, TensorMap mdo,
    TensorMap mdk, TensorMap mdv, int H, int Nq, int Nk, int dh, int nkt, int paired, float scale,
    Dropout dr) {
  const int items = paired ? causal_items<CAUSAL>(nkt) : nkt;  // causal: key tiles (p, nkt-1-p)
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int head = logical / items;
  bwd_dkdv_pipe<T, D, CAUSAL, true, FAR>(Q, K, V, dO, LSE2, Dws, dK, dV, mq, mk, mv, mdo, mdk, mdv, H, Nq, Nk, dh,
                                         nkt, paired, scale, dr, head, logical - head * items);
}

// ---------------------------------------------------------------------------------------
// dQ
// ---------------------------------------------------------------------------------------
template <int D, bool CAUSAL, bool DROP> struct BwdQCfg {
  static constexpr int BM = 128;  // query rows per workgroup (32 per wave)
  // keys per iteration: 32 at D = 128 keeps the kernel within 256 registers, so that two
  // workgroups share a CU and one hides the other's softmax arithmetic and LDS latency.  At D = 96 (dQ, us, 32 -> 64
  // keys, causal 36 heads x 1333 40.9 -> 36.8, 64 x 4096 309 -> 297) only the causal kernel with dropout spills.
  static constexpr int BN = D == 128 || (D == 96 && CAUSAL && DROP) ? 32 : 64;
  static constexpr int ROWB = lds_row<D> * 2;
  static constexpr int TILE = BN * ROWB;  // one of K, V (swizzled, unpadded)
  static constexpr int STAGE = 2 * TILE;  // power of two: the buffer is switched by one XOR
  static constexpr int OSTR = lds_row<D> * 2 + 16;
  static constexpr int SMEM = 2 * STAGE > 4 * 32 * OSTR ? 2 * STAGE : 4 * 32 * OSTR;  // tiles / epilogue
  static_assert((STAGE & (STAGE - 1)) == 0, "XOR buffer switch");
};

// The workgroup's part: query tile `item` of `head`, and its partner if the causal tiles are paired.
// STATS: the workspace holds -D and LSE * log2(e) already (mha_bwd_stats_kernel); otherwise they are
// formed here and left there for the dK/dV kernel.
template <typename T, int D, bool CAUSAL, bool DROP, bool STATS, Lanes M>
static __device__ __forceinline__ void bwd_dq(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const T* __restrict__ O, const T* __restrict__ dO, const float* __restrict__ LSE,
    float* __restrict__ Dws, float* __restrict__ LSE2ws, T* __restrict__ dQ, const TensorMap& mq,
    const TensorMap& mk, const TensorMap& mv, const TensorMap& mo, const TensorMap& mdo, const TensorMap& mdq, int H,
    int Nq, int Nk, int dh, int nqt, int paired, float scale, float scale_log2, const Dropout& dr, int head,
    int item) {
  using F = Frag<T>;
  using v8 = typename F::v8;
  using C = BwdQCfg<D, CAUSAL, DROP>;
  // The exchange of the generator's words behind one score product or two: far apart in one slot causal kernels at D > 64 lost 1 %, in
  // order in two slots all of them 1 to 5 % (us, fp16, both sides, 4 heads x 4096, d = 112 146.5 -> 139.8 in one).
  constexpr bool TWO_SLOTS = D == 64 || M == FAR;
  constexpr int KS = D / 16, DT = D / 32;

  // few offset registers in the causal kernels: with dropout at D = 128 all of them spill (dQ, us, 512 heads x 512 115.7 ->
  // 108.4, bf16 64 x 2048 122.3 -> 118.3; the others are equal)
  using LaneOffsets = std::conditional_t<CAUSAL, SwzLaneLean<D>, SwzLane<D>>;
  SPARK_LDS char* const smem = lds_origin();

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, c32 = column_row<M>(lane);

  const T* Qh = Q + head_base(mq, head, H);
  const T* dOh = dO + head_base(mdo, head, H);
  const T* Oh = STATS ? nullptr : O + head_base(mo, head, H);
  const BufView kview(K + head_base(mk, head, H), head_span_bytes(mk, Nk, dh));
  const BufView vview(V + head_base(mv, head, H), head_span_bytes(mv, Nk, dh));
  const uint32_t k_row_bytes = (uint32_t)mk.row * 2, v_row_bytes = (uint32_t)mv.row * 2;
  const uint32_t k_lane_src = dma_lane_src<D>(wave, lane, k_row_bytes, dh);
  const uint32_t v_lane_src = dma_lane_src<D>(wave, lane, v_row_bytes, dh);
  // K / V tiles go global -> LDS directly (no staging registers, no LDS store instructions);
  // completion is awaited with wait_vmem_all + barrier at the end of the iteration before use.
  auto fetch_tile = [&](int j, int buf) {
    tile_dma<D, C::BN>(kview, j * C::BN, smem + buf * C::STAGE, wave, k_lane_src, k_row_bytes);
    tile_dma<D, C::BN>(vview, j * C::BN, smem + buf * C::STAGE + C::TILE, wave, v_lane_src, v_row_bytes);
  };

  for (int rep = 0; rep < (CAUSAL && paired ? 2 : 1); ++rep) {
    const int qt = CAUSAL && rep == 0 ? nqt - 1 - item : item;  // the long tile first
    if (CAUSAL && rep == 1) {
      if (qt == nqt - 1 - item) break;  // odd tile count: the middle tile has no partner
      __syncthreads();                  // the first tile's epilogue is done with the LDS
    }
    const int q0 = qt * C::BM + wave * 32;
    const int qrow = q0 + c32;
    const int qrow_c = qrow < Nq ? qrow : Nq - 1;

    v8 qf[KS], dof[KS], of[KS];  // of: the row of O, needed for D only
    if constexpr (CAUSAL) {
      load_row_frags(qf, Qh + (size_t)qrow_c * (size_t)mq.row, g, dh);
      load_row_frags(dof, dOh + (size_t)qrow_c * (size_t)mdo.row, g, dh);
      if constexpr (!STATS) load_row_frags(of, Oh + (size_t)qrow_c * (size_t)mo.row, g, dh);
    } else {
      load_row_frags(qf, BufView(Qh, head_span_bytes(mq, Nq, dh)), (uint32_t)qrow_c * ((uint32_t)mq.row * 2), g, dh);
      load_row_frags(dof, BufView(dOh, head_span_bytes(mdo, Nq, dh)), (uint32_t)qrow_c * ((uint32_t)mdo.row * 2), g, dh);
      if constexpr (!STATS)
        load_row_frags(of, BufView(Oh, head_span_bytes(mo, Nq, dh)), (uint32_t)qrow_c * ((uint32_t)mo.row * 2), g, dh);
    }
    float lse2 = STATS ? LSE2ws[(size_t)head * Nq + qrow_c] : LSE[(size_t)head * Nq + qrow_c];
    float Dq = STATS ? -Dws[(size_t)head * Nq + qrow_c] : 0.f;

    int kv_end = Nk;
    if (CAUSAL) {
      const int lim = (qt + 1) * C::BM;
      kv_end = lim < Nk ? lim : Nk;
    }
    const int nt = (kv_end + C::BN - 1) / C::BN;

    LaneOffsets off(lane);  // read offsets of the current buffer

    f32x16 dq[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) dq[dt][r] = 0.f;

    fetch_tile(0, 0);
    // the tile is requested before the wait for O and dO that forming D takes, not behind it (the scheduler's
    // choice; us, causal 256 heads x 512, d = 128 54.5 -> 48.8, d = 64 31.4 -> 27.9)
    sched_fence();
    wait_vmem_all();  // Q / dO / O fragments and LSE are in registers before the loop
    // D_i = sum_k dO_ik O_ik (the paper's "dPsum"): a lane holds half of its query's row, the lane
    // 32 further on the other half.  Under dropout dS = r P o (M o dPraw - D (1-p)), so D is kept
    // multiplied by the keep probability.  The dK/dV kernel runs after this one and reads D and
    // LSE * log2(e) from the workspace.
    if (!STATS) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int i = 0; i < 8; ++i) Dq = __builtin_fmaf((float)of[ks][i], (float)dof[ks][i], Dq);
      Dq = half_pair_sum(Dq) * (DROP ? dr.keep_prob : 1.0f);
      lse2 *= 1.4426950408889634f;
      if (g == 0 && qrow < Nq) {
        Dws[(size_t)head * Nq + qrow] = -Dq;  // negated: the dK/dV kernel starts its dP accumulators from it
        LSE2ws[(size_t)head * Nq + qrow] = lse2;
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]), "+v"(dof[ks]));
    asm volatile("" : "+v"(lse2), "+v"(Dq));
    // dS = P o (dP - D) needs no subtraction: every dP accumulator starts from -D
    // (one value per lane here: lane = query), handed to the first MFMA as its addend.  That costs 16
    // registers for the whole loop (dQ kernel at D = 64 -2 ... -3 %; backward, us, D = 128, causal 64 x 4096 923.7 ->
    // 913.3, 16 x 16384 3536 -> 3513, D = 96 90 x 1500 344 -> 340, with dropout equal).
    f32x16 dneg;
#pragma unroll
    for (int r = 0; r < 16; ++r) dneg[r] = -Dq;
    asm volatile("" : "+v"(dneg));
    __syncthreads();

    // last key this lane's query attends to, less the 4 g that every register's key contains: the mask is one
    // compare with a constant per element
    const int last_key = (CAUSAL && qrow < Nk ? qrow : Nk - 1) - 4 * g;
    // One iteration, compiled twice: MASKED for tiles that the diagonal or the end of the keys
    // crosses, and without any mask arithmetic for all the others.
    auto iteration = [&](const int j, auto masked_tag) {
      constexpr bool MASKED = decltype(masked_tag)::value;
      const int buf = j & 1;
      if (j + 1 < nt) fetch_tile(j + 1, buf ^ 1);  // everybody left that buffer before the last barrier
      const int k0 = j * C::BN;
      // wave-uniform: skip tiles entirely above the diagonal (they are among the masked ones)
      if (!MASKED || !CAUSAL || k0 <= q0 + 31) {
        SPARK_LDS const char* kb = smem;  // + off.* (which carry the buffer bit)
        SPARK_LDS const char* vb = smem + C::TILE;

        // S^T = K Q^T first, then dP^T = V dO^T (lane = query column, registers = keys), so that
        // P = exp2(S c - LSE) can be formed under the MFMAs of dP, and the second half of dS under
        // the first MFMAs of dQ.  A wave issues in order: what overlaps is decided by program
        // order, so the arithmetic is placed between the MFMAs by hand, pinned by empty asm
        // statements (the compiler would move it to its first use) and scheduling fences.
        // Row fragments (step i < KS: K at k-step i; step i >= KS: V at k-step i - KS) are read
        // four steps ahead of their MFMAs.
        constexpr int MT = C::BN / 32;  // 32-key blocks per tile
        f32x16 s[MT], dp[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
          for (int r = 0; r < 16; ++r) s[mt][r] = 0.f;
          dp[mt] = dneg;
        }
        constexpr int AHEAD = 4;
        v8 fa[AHEAD][MT];
        auto load_step = [&](int i) {
          const int ks = i < KS ? i : i - KS;
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            fa[i % AHEAD][mt] = lds_read16<v8>(i < KS ? kb : vb, off.row_at(ks) + mt * 32 * C::ROWB);
        };
        // Dropout: dS = r P o (M o dPraw - D (1-p)); the workspace holds D (1-p) and the factor r
        // goes into the final scale of dQ.  The generator's rounds ride between the MFMAs of S, its exchange between
        // the first ones of dP (backward, us, causal fp16 d = 64 256 heads x 2048 685 -> 662, 512 x 512 170.8 -> 169.4;
        // bf16 d = 128 64 x 4096 1067 -> 1039; d = 80 36 x 1333 95.7 -> 92.2).
        uint32_t keep[MT][4];
        Philox rng[MT];
        if (DROP) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) rng[mt] = keep_query_lane_begin<M>(dr, head, qrow, k0 + 32 * mt, lane);
        }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) load_step(i);
        sched_fence();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            s[mt] = F::mfma(fa[ks % AHEAD][mt], qf[ks], s[mt]);
            if (DROP) {
#pragma unroll
              for (int round = ks * 10 / KS; round < (ks + 1) * 10 / KS; ++round)
                philox_round<true>(rng[mt], dr.key0, dr.key1, round);
              sched_fence();
            }
          }
          load_step(ks + AHEAD);  // KS >= AHEAD: always a valid step
          sched_fence();
        }

        float pe[16 * MT];
        auto p_elem = [&](int e) {  // e = mt * 16 + r
          const int mt = e / 16, r = e % 16;
          float x = __builtin_amdgcn_exp2f(__builtin_fmaf(s[mt][r], scale_log2, -lse2));
          if (MASKED) x = mt * 32 + 8 * (r / 4) + (r % 4) > last_key - k0 ? 0.f : x;
          pe[e] = x;
          asm volatile("" : "+v"(pe[e]));
        };
        // K^T fragments, one group per 16-key step of dQ; the first two groups are requested in
        // the second half of the dP phase, when the row fragments have all been requested (one
        // burst of all of them would exceed the 15 LDS reads a wave can have in flight)
        constexpr int NKK = C::BN / 16;
        v8 ft[2][DT];
        auto load_tgroup = [&](int kk) {
          const int o = kk * 16 * C::ROWB;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt)
            ft[kk & 1][dt] = read_tr_pair<T>(kb, off.tr_at(0, dt) + o, off.tr_at(1, dt) + o);
        };
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            dp[mt] = F::mfma(fa[(KS + ks) % AHEAD][mt], dof[ks], dp[mt]);
            if (DROP && ks == 0) {
              keep[mt][0] = rng[mt].c0; keep[mt][1] = rng[mt].c1; keep[mt][2] = rng[mt].c2; keep[mt][3] = rng[mt].c3;
              exchange_bit0<M>(keep[mt], lane);
              if (TWO_SLOTS) asm volatile("" : "+v"(keep[mt][0]), "+v"(keep[mt][1]), "+v"(keep[mt][2]), "+v"(keep[mt][3]));
            }
            if (DROP && ks == (TWO_SLOTS ? 2 : 0)) {
              exchange_bit1<M>(keep[mt], lane);
              asm volatile("" : "+v"(keep[mt][0]), "+v"(keep[mt][1]), "+v"(keep[mt][2]), "+v"(keep[mt][3]));
            }
#pragma unroll
            for (int x = ks * 16 / KS; x < (ks + 1) * 16 / KS; ++x) p_elem(mt * 16 + x);  // 16 in KS MFMAs
            sched_fence();
          }
          if (KS + ks + AHEAD < 2 * KS) load_step(KS + ks + AHEAD);
          if (ks == KS - AHEAD) load_tgroup(0);
          if (ks == KS - AHEAD / 2) load_tgroup(1);
          sched_fence();
        }

        float ds[16 * MT];
        auto ds_elem = [&](int e) {
          const int mt = e / 16, r = e % 16;
          // the accumulator started from -D, which is also what a dropped entry has instead of M o dP - D
          ds[e] = pe[e] * (DROP && !keep_reg(keep[mt], r, dr.thr) ? -Dq : dp[mt][r]);
          asm volatile("" : "+v"(ds[e]));
        };
        // dQ^T += K^T dS^T, 16 keys per step; step kk uses elements 8 kk .. 8 kk + 7.  Those of
        // step 0 are formed up front, those of step kk + 1 under the MFMAs of step kk.
        v8 dsf[NKK];
#pragma unroll
        for (int x = 0; x < 8; ++x) ds_elem(x);
        dsf[0] = pack8<T>(&ds[0]);
        sched_fence();
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            dq[dt] = F::mfma(ft[kk & 1][dt], dsf[kk], dq[dt]);
            if (kk + 1 < NKK) {
#pragma unroll
              for (int x = dt * 8 / DT; x < (dt + 1) * 8 / DT; ++x) ds_elem(8 * (kk + 1) + x);
            }
            sched_fence();
          }
          if (kk + 1 < NKK) {
            dsf[kk + 1] = pack8<T>(&ds[8 * (kk + 1)]);
            asm volatile("" : "+v"(dsf[kk + 1]));
          }
          if (kk + 2 < NKK) load_tgroup(kk + 2);
          sched_fence();
        }
      }
      off.flip(C::STAGE);
      wait_vmem_all();  // the next tile has landed (requested at the top of the iteration)
      __syncthreads();
    };
    // Tiles [0, n_plain) end within the keys and, if causal, at or below the diagonal for every
    // row of this wave.  The split differs between the waves of a workgroup; the number of
    // iterations, and with it the number of barriers, does not.
    int n_plain = Nk / C::BN;
    if (CAUSAL && (q0 + 1) / C::BN < n_plain) n_plain = (q0 + 1) / C::BN;
    if (n_plain > nt) n_plain = nt;
    int j = 0;
    for (; j < n_plain; ++j) iteration(j, std::false_type{});
    for (; j < nt; ++j) iteration(j, std::true_type{});

    SPARK_LDS char* ob = smem + wave * 32 * C::OSTR;
    store_transposed<T, D, C::OSTR, M>(dq, DROP ? scale * dr.rescale : scale, ob, dQ + head_base(mdq, head, H), q0,
                                    Nq, lane, (size_t)mdq.row, dh);
  }  // rep
}

template <typename T, int D, bool CAUSAL, bool DROP>
__global__ __launch_bounds__(256, 2) void mha_bwd_dq_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const T* __restrict__ O, const T* __restrict__ dO, const float* __restrict__ LSE,
    float* __restrict__ Dws, float* __restrict__ LSE2ws, T* __restrict__ dQ, TensorMap mq, TensorMap mk,
    TensorMap mv, TensorMap mo, TensorMap mdo, TensorMap mdq, int H, int Nq, int Nk, int dh, int nqt, int paired,
    float scale, float scale_log2, Dropout dr) {
  const int items = paired ? causal_items<CAUSAL>(nqt) : nqt;  // causal: query tiles (nqt-1-p, p)
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int head = logical / items;
  bwd_dq<T, D, CAUSAL, DROP, false, IN_ORDER>(Q, K, V, O, dO, LSE, Dws, LSE2ws, dQ, mq, mk, mv, mo, mdo, mdq, H, Nq,
                                              Nk, dh, nqt, paired, scale, scale_log2, dr, head, logical - head * items);
}

// With dropout, the rows far apart in the lanes (column_row); the rule is far_rows.
template <typename T, int D, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void mha_bwd_dq_far_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const T* __restrict__ O, const T* __restrict__ dO, const float* __restrict__ LSE,
    float* __restrict__ Dws, float* __restrict__ LSE2ws, T* __restrict__ dQ, TensorMap mq, TensorMap mk,
    TensorMap mv, TensorMap mo, TensorMap mdo, TensorMap mdq, int H, int Nq, int Nk, int dh, int nqt, int paired,
    float scale, float scale_log2, Dropout dr) {
  const int items = paired ? causal_items<CAUSAL>(nqt) : nqt;  // causal: query tiles (nqt-1-p, p)
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int head = logical / items;
  bwd_dq<T, D, CAUSAL, true, false, FAR>(Q, K, V, O, dO, LSE, Dws, LSE2ws, dQ, mq, mk, mv, mo, mdo, mdq, H, Nq,
                                         Nk, dh, nqt, paired, scale, scale_log2, dr, head, logical - head * items);
}

// ---------------------------------------------------------------------------------------
// Both in one grid, for problems of which neither kernel fills the chip by itself.  The dK/dV side
// needs D and LSE * log2(e) of all queries, so these are formed by a pass of their own first (2 us).
// Measured at 16 heads x 1024, d = 64 (128 workgroups per side on 256 CUs): 36.9 -> 26.5 us.
// ---------------------------------------------------------------------------------------

// -D (times the keep probability under dropout) and LSE * log2(e): D / 8 lanes per query row.
template <typename T, int D>
__global__ __launch_bounds__(256) void mha_bwd_stats_kernel(const T* __restrict__ O, const T* __restrict__ dO,
                                                            const float* __restrict__ LSE, float* __restrict__ Dws,
                                                            float* __restrict__ LSE2ws, TensorMap mo, TensorMap mdo,
                                                            int H, int Nq, int dh, int rows, float keep_prob) {
  using v8 = typename Frag<T>::v8;
  constexpr int LPR = lds_row<D> / 8;
  const int row = blockIdx.x * (256 / LPR) + threadIdx.x / LPR;  // flat (head, query) index
  const int col = (threadIdx.x % LPR) * 8;
  const bool live = row < rows;
  const int r = live ? row : rows - 1;
  const int head = r / Nq, q = r - head * Nq;
  const v8 o = load_row_chunk<v8>(O + head_base(mo, head, H) + (size_t)q * (size_t)mo.row, col, dh);
  const v8 g = load_row_chunk<v8>(dO + head_base(mdo, head, H) + (size_t)q * (size_t)mdo.row, col, dh);
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) acc = __builtin_fmaf((float)o[i], (float)g[i], acc);
#pragma unroll
  for (int m = LPR / 2; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, LPR);
  if (live && col == 0) {
    Dws[r] = -acc * keep_prob;
    LSE2ws[r] = LSE[r] * 1.4426950408889634f;
  }
}

template <int D> struct BwdMergedCfg {
  static constexpr int SMEM = BwdKvPipeCfg<D>::SMEM;
  static_assert(SMEM >= BwdQCfg<D, false, false>::SMEM, "the dK/dV side needs more, whatever the other's tile");
};

// dK/dV's decisions of dropout by a compare and a select each in the causal merged kernels that gain by it (backward, us, masks ->
// so): 96 columns, 6 heads x 4000, d = 80 fp16 147.5 -> 146.2, bf16 152.4 -> 150.7, 24 x 1024 47.5 -> 47.0, 49.9 -> 49.4; fp16 at
// d = 64, 64 x 384 21.3 -> 21.2, 24 x 1024 36.7 -> 36.6 (bf16 36.8 -> 38.2); bf16 at d = 128, rows far apart, 7 x 2240 87.7 -> 86.0
// (fp16 85.3 -> 86.3; in order, 60 x 400, 37.5 -> 38.0 in both types).  With one grid per side masks are as fast or faster
// at those (bf16, 140 x 512, d = 96 89.6 -> 90.5, d = 64 61.2 -> 62.9; 64 x 2048, d = 128 291 -> 295).
template <typename T, int D, bool CAUSAL, Lanes M>
constexpr bool merged_compares = CAUSAL && (D == 96 || (D == 64 ? Frag<T>::FINITE_DOT : !Frag<T>::FINITE_DOT && M == FAR));

template <typename T, int D, bool CAUSAL, bool DROP>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void mha_bwd_merged_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ dO,
    float* __restrict__ Dws, float* __restrict__ LSE2ws, T* __restrict__ dQ, T* __restrict__ dK, T* __restrict__ dV,
    TensorMap mq, TensorMap mk, TensorMap mv, TensorMap mdo, TensorMap mdq, TensorMap mdk, TensorMap mdv, int H,
    int Nq, int Nk, int dh, int nqt, int nkt, int paired, float scale, Dropout dr) {
  const int qitems = paired ? causal_items<CAUSAL>(nqt) : nqt, kitems = paired ? causal_items<CAUSAL>(nkt) : nkt;
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int head = logical / (qitems + kitems);
  const int item = logical - head * (qitems + kitems);
  constexpr bool COMPARE = merged_compares<T, D, CAUSAL, IN_ORDER>;
  if (item < kitems)  // the longer ones first
    bwd_dkdv_pipe<T, D, CAUSAL, DROP, IN_ORDER, COMPARE>(Q, K, V, dO, LSE2ws, Dws, dK, dV, mq, mk, mv, mdo, mdk, mdv, H, Nq,
                                                         Nk, dh, nkt, paired, scale, dr, head, item);
  else
    bwd_dq<T, D, CAUSAL, DROP, true, IN_ORDER>(Q, K, V, nullptr, dO, nullptr, Dws, LSE2ws, dQ, mq, mk, mv, mdo, mdo, mdq, H,
                                               Nq, Nk, dh, nqt, paired, scale, scale * 1.4426950408889634f, dr, head,
                                               item - kitems);
}

// With dropout, the rows far apart in the lanes (column_row); the rule is far_rows.
template <typename T, int D, bool CAUSAL>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void mha_bwd_merged_far_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ dO,
    float* __restrict__ Dws, float* __restrict__ LSE2ws, T* __restrict__ dQ, T* __restrict__ dK, T* __restrict__ dV,
    TensorMap mq, TensorMap mk, TensorMap mv, TensorMap mdo, TensorMap mdq, TensorMap mdk, TensorMap mdv, int H,
    int Nq, int Nk, int dh, int nqt, int nkt, int paired, float scale, Dropout dr) {
  const int qitems = paired ? causal_items<CAUSAL>(nqt) : nqt, kitems = paired ? causal_items<CAUSAL>(nkt) : nkt;
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int head = logical / (qitems + kitems);
  const int item = logical - head * (qitems + kitems);
  if (item < kitems)  // the longer ones first
    bwd_dkdv_pipe<T, D, CAUSAL, true, FAR, merged_compares<T, D, CAUSAL, FAR>>(
        Q, K, V, dO, LSE2ws, Dws, dK, dV, mq, mk, mv, mdo, mdk, mdv, H, Nq, Nk, dh, nkt, paired, scale, dr, head, item);
  else
    bwd_dq<T, D, CAUSAL, true, true, FAR>(Q, K, V, nullptr, dO, nullptr, Dws, LSE2ws, dQ, mq, mk, mv, mdo, mdo, mdq, H,
                                          Nq, Nk, dh, nqt, paired, scale, scale * 1.4426950408889634f, dr, head,
                                          item - kitems);
}

}  // namespace spark
