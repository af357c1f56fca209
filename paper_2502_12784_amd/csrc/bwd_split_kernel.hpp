// Attention backward for grids that leave most of the chip idle, in one launch: small batches, few heads,
// short sequences.
//
// The two kernels of bwd_kernels.hpp give a workgroup 128 rows and walk the other sequence in one serial
// chain, one kernel after the other; with 32 such workgroups seven eighths of the CUs idle through both.
// Here a workgroup owns 32 rows and its waves split the OTHER dimension: wave w of NW takes the 32-row tiles
// w, w + NW, ..., and the partial gradients are added once at the end through LDS, in a fixed order (the
// result is reproducible).  Workgroups of both kinds, dQ for 32 queries and dK, dV for 32 keys, share one
// grid and run side by side; what lets them is that the dK/dV side forms D = rowsum(dO o O) of its query
// tiles itself instead of reading it from the workspace (KS 16-byte loads and 8 KS multiply-adds a lane
// and tile, which only an otherwise idle chip has to spare).
//
// Every wave fills its own double-buffered LDS tiles by direct global->LDS loads, so the loops have no
// barrier.  Eight waves (two per SIMD) at D = 64; at D = 128 the accumulators of dK and dV, the K and V
// fragments and the row of O take about 300 registers, so four waves run, one per SIMD, and the 128 KB of
// tiles are the same.  Bound: the chain of one tile (load, two score contractions, softmax, two accumulations),
// 1.7 us per round of eight tiles at D = 64 and of four at D = 128.  Measured against the two kernels, fp16:
// 2 heads x 128, d = 64: 11.6 -> 6.4 us; 4 heads x 1024: 35.3 -> 13.2 us, d = 128 58.4 -> 23.5 us.
#pragma once
#include "bwd_kernels.hpp"
#include "dropout_gfx950.hpp"
#include "mma_gfx950.hpp"
#include "tiles_gfx950.hpp"

namespace spark {

template <int D> struct BwdSplitCfg {
  static constexpr int NW = D == 64 ? 8 : 4;  // waves of a workgroup = streams over the other dimension
  static constexpr int BM = 32;   // rows a workgroup owns, and rows per tile of the other dimension
  static constexpr int ROWB = D * 2;
  static constexpr int TILE = BM * ROWB;
  static constexpr int NLOAD = TILE / 1024;    // direct loads per tile
  static constexpr int STAGE = 2 * TILE;       // one tile of each operand; every wave has two stages
  static constexpr int GROUPS = D / 8;         // accumulator quads (4 registers) per lane
  static constexpr int GPW = GROUPS / NW;      // ... that each wave sums in the merge
  static constexpr int OSTR = D * 2 + 16;
  static constexpr int STG0 = NW * 2 * STAGE;  // 16-bit rows on their way out
  static constexpr int STAT0 = STG0 + BM * OSTR;  // [wave][-D, LSE*log2(e)][row]
  static constexpr int SMEM = STAT0 + NW * 2 * BM * 4;
  static_assert(NW * GROUPS * 1024 <= STG0, "partial results of all waves");
};

// Sum of the accumulators (D x 32, lane = column) of waves 0 .. used-1, times `mul`, stored as 32 rows of D
// 16-bit values: rows < N, columns < dh.  All waves call it; the LDS tiles are overwritten.
template <typename T, int D>
static __device__ __forceinline__ void merge_store(const f32x16 (&acc)[D / 32], float mul, int used,
                                                   SPARK_LDS char* smem, int tid, T* __restrict__ out, int row0, int N,
                                                   size_t row_stride, int dh) {
  using C = BwdSplitCfg<D>;
  using v4 = typename Frag<T>::v4;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, c32 = lane & 31;
  __syncthreads();  // every wave has left its tiles, and an earlier merge its staging rows
  if (wave < used) {
#pragma unroll
    for (int q = 0; q < C::GROUPS; ++q) {
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = acc[q / 4][(q % 4) * 4 + e];
      lds_write(smem, (wave * C::GROUPS + q) * 1024 + lane * 16, x);
    }
  }
  __syncthreads();
#pragma unroll
  for (int gi = 0; gi < C::GPW; ++gi) {
    const int q = wave * C::GPW + gi;
    f32x4 sum = lds_read16<f32x4>(smem, q * 1024 + lane * 16);
    for (int w = 1; w < used; ++w) sum += lds_read16<f32x4>(smem, (w * C::GROUPS + q) * 1024 + lane * 16);
    v4 pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = (T)(sum[e] * mul);
    lds_write(smem + C::STG0, c32 * C::OSTR + (8 * q + 4 * g) * 2, pk);
  }
  __syncthreads();
  constexpr int CPR = D / 8, RPP = 64 * C::NW / CPR;  // chunks per row, rows per pass of the workgroup
  const int cc = tid % CPR;
  for (int row = tid / CPR; row < C::BM; row += RPP)
    if (row0 + row < N && cc * 8 < dh)
      *reinterpret_cast<u32x4*>(out + (size_t)(row0 + row) * row_stride + cc * 8) =
          lds_read16<u32x4>(smem + C::STG0, row * C::OSTR + cc * 16);
}

template <typename T, int D, bool CAUSAL, bool DROP>
__global__ __launch_bounds__(64 * BwdSplitCfg<D>::NW, 1) void mha_bwd_split_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ O,
    const T* __restrict__ dO, const float* __restrict__ LSE, T* __restrict__ dQ, T* __restrict__ dK,
    T* __restrict__ dV, TensorMap mq, TensorMap mk, TensorMap mv, TensorMap mo, TensorMap mdo, TensorMap mdq,
    TensorMap mdk, TensorMap mdv, int H, int Nq, int Nk, int dh, int nqt, int nkt, float scale, DropoutLean drop) {
  using F = Frag<T>;
  using v8 = typename F::v8;
  using C = BwdSplitCfg<D>;
  constexpr int KS = D / 16, DT = D / 32;

  SPARK_LDS char* const smem = lds_origin();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, c32 = lane & 31;
  SPARK_LDS char* const wbuf = smem + wave * 2 * C::STAGE;
  const float scale_log2 = scale * 1.4426950408889634f;
  // With the word more of `Dropout` the causal kernels at 128 columns loaded an argument inside the loop and awaited it
  // there (us, fp16, causal 2 x 128, d = 128 10.6 -> 10.4, bf16 10.8 -> 10.6; bf16 4 x 1024 25.6 -> 25.5).
  const Dropout dr{drop.key0, drop.key1, drop.offset, drop.thr, (256u - drop.thr) * 0x01010101u, drop.keep_prob,
                   drop.rescale};

  // per head first the key tiles, then the query tiles (the former have twice the accumulation work);
  // causal: the longest of each kind first
  const int logical = xcd_contiguous(blockIdx.x, gridDim.x);
  const int head = logical / (nqt + nkt);
  const int item = logical - head * (nqt + nkt);

  const T* Qh = Q + head_base(mq, head, H);
  const T* Kh = K + head_base(mk, head, H);
  const T* Vh = V + head_base(mv, head, H);
  const T* Oh = O + head_base(mo, head, H);
  const T* dOh = dO + head_base(mdo, head, H);
  const SwzLane<D> off(lane);

  if (item >= nkt) {
    // ------------------------------------------------------------------ dQ of 32 queries
    // As in mha_bwd_dq_kernel: S^T = K Q^T, dP^T = V dO^T (lane = query), dQ^T += K^T dS^T.
    const int qt = CAUSAL ? nqt - 1 - (item - nkt) : item - nkt;
    const int q0 = qt * C::BM, qrow = q0 + c32;
    const int qrow_c = qrow < Nq ? qrow : Nq - 1;
    const int kv_end = CAUSAL && q0 + C::BM < Nk ? q0 + C::BM : Nk;
    const int nt = (kv_end + C::BM - 1) / C::BM;
    int n_plain = Nk / C::BM;  // tiles [0, n_plain) need no mask
    if (CAUSAL && qt < n_plain) n_plain = qt;

    const BufView kview(Kh, head_span_bytes(mk, Nk, dh)), vview(Vh, head_span_bytes(mv, Nk, dh));
    const uint32_t k_row_bytes = (uint32_t)mk.row * 2, v_row_bytes = (uint32_t)mv.row * 2;
    const WaveDma<D> kdma(lane, k_row_bytes, dh), vdma(lane, v_row_bytes, dh);
    auto fetch = [&](int j, int b) {  // stage b: K, V
      kdma.template tile<C::BM>(kview, j * C::BM, wbuf + b * C::STAGE, k_row_bytes);
      vdma.template tile<C::BM>(vview, j * C::BM, wbuf + b * C::STAGE + C::TILE, v_row_bytes);
    };

    v8 qf[KS], dof[KS], of[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qf[ks] = load_row_chunk<v8>(Qh + (size_t)qrow_c * (size_t)mq.row, ks * 16 + g * 8, dh);
      dof[ks] = load_row_chunk<v8>(dOh + (size_t)qrow_c * (size_t)mdo.row, ks * 16 + g * 8, dh);
      of[ks] = load_row_chunk<v8>(Oh + (size_t)qrow_c * (size_t)mo.row, ks * 16 + g * 8, dh);
    }
    float lse2 = LSE[(size_t)head * Nq + qrow_c];
    if (wave < nt) fetch(wave, 0);
    float Dq = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int i = 0; i < 8; ++i) Dq = __builtin_fmaf((float)of[ks][i], (float)dof[ks][i], Dq);
    Dq = half_pair_sum(Dq) * (DROP ? dr.keep_prob : 1.0f);
    lse2 *= 1.4426950408889634f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]), "+v"(dof[ks]));

    f32x16 dq[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) dq[dt][r] = 0.f;

    const int last_key = (CAUSAL && qrow < Nk ? qrow : Nk - 1) - 4 * g;  // the mask: one compare with a constant
    auto tile = [&](const int j, const int b, auto masked_tag, const bool next) {
      constexpr bool MASKED = decltype(masked_tag)::value;
      SPARK_LDS char* const kb = wbuf + b * C::STAGE;
      SPARK_LDS char* const vb = kb + C::TILE;
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = DROP ? 0.f : -Dq; }
      if (next) {
        wait_lds_all();  // every read of that stage has returned
        fetch(j + C::NW, b ^ 1);
        wait_vmem<2 * C::NLOAD>();  // this tile is here, the next one on its way
      } else {
        wait_vmem<0>();
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) dp = F::mfma(lds_read16<v8>(vb, off.row[ks]), dof[ks], dp);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s = F::mfma(lds_read16<v8>(kb, off.row[ks]), qf[ks], s);
      uint32_t keep[4];
      if (DROP) keep_bytes_query_lane<IN_ORDER>(dr, head, qrow, j * C::BM, lane, keep);
      float ds[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], scale_log2, -lse2));
        if (MASKED && 8 * (r / 4) + (r % 4) > last_key - j * C::BM) p = 0.f;
        ds[r] = DROP ? p * ((keep_reg(keep, r, dr.thr) ? dp[r] : 0.f) - Dq) : p * dp[r];
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const v8 dsf = pack8<T>(&ds[8 * kk]);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const int ro = kk * 16 * C::ROWB;
          dq[dt] = F::mfma(read_tr_pair<T>(kb, off.tr[0][dt] + ro, off.tr[1][dt] + ro), dsf, dq[dt]);
        }
      }
    };
    int b = 0;
    for (int j = wave; j < nt; j += C::NW) {
      if (j < n_plain)
        tile(j, b, std::false_type{}, j + C::NW < nt);
      else
        tile(j, b, std::true_type{}, j + C::NW < nt);
      b ^= 1;
    }
    merge_store<T, D>(dq, DROP ? scale * dr.rescale : scale, nt < C::NW ? nt : C::NW, smem, tid,
                      dQ + head_base(mdq, head, H), q0, Nq, (size_t)mdq.row, dh);
  } else {
    // ------------------------------------------------------------------ dK, dV of 32 keys
    // As in mha_bwd_dkdv_pipe_kernel: S = Q K^T, dP = dO V^T (lane = key), dV^T += dO^T P, dK^T += Q^T dS.
    const int kt = item;
    const int k0 = kt * C::BM, krow = k0 + c32;
    const int t0 = CAUSAL ? kt : 0;  // first query tile
    const BufView qview(Qh, head_span_bytes(mq, Nq, dh)), doview(dOh, head_span_bytes(mdo, Nq, dh));
    const uint32_t q_row_bytes = (uint32_t)mq.row * 2, do_row_bytes = (uint32_t)mdo.row * 2;
    const WaveDma<D> qdma(lane, q_row_bytes, dh), dodma(lane, do_row_bytes, dh);
    auto fetch = [&](int t, int b) {  // stage b: Q, dO
      qdma.template tile<C::BM>(qview, t * C::BM, wbuf + b * C::STAGE, q_row_bytes);
      dodma.template tile<C::BM>(doview, t * C::BM, wbuf + b * C::STAGE + C::TILE, do_row_bytes);
    };
    const BufView oview(Oh, head_span_bytes(mo, Nq, dh));
    // row of O and LSE of this lane's query in tile t; zeros past the end (there dO reads as zeros, too)
    v8 of[KS];
    float lse = 0.f;
    auto load_o = [&](int t) {
      const int row = t * C::BM + c32;
      const bool valid = row < Nq;
      load_row_frags(of, oview, (uint32_t)row * ((uint32_t)mo.row * 2), g, dh, valid);
      lse = valid ? LSE[(size_t)head * Nq + row] : 0.f;
    };

    v8 kf[KS], vf[KS];
    const int krow_c = krow < Nk ? krow : Nk - 1;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      kf[ks] = load_row_chunk<v8>(Kh + (size_t)krow_c * (size_t)mk.row, ks * 16 + g * 8, dh);
      vf[ks] = load_row_chunk<v8>(Vh + (size_t)krow_c * (size_t)mv.row, ks * 16 + g * 8, dh);
    }
    if (t0 + wave < nqt) {
      fetch(t0 + wave, 0);
      load_o(t0 + wave);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(kf[ks]), "+v"(vf[ks]));

    f32x16 dk[DT], dv[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) { dk[dt][r] = 0.f; dv[dt][r] = 0.f; }
    SPARK_LDS char* const stat = smem + C::STAT0 + wave * 2 * C::BM * 4;

    auto tile = [&](const int t, const int b, const bool next) {
      SPARK_LDS char* const qb = wbuf + b * C::STAGE;
      SPARK_LDS char* const dob = qb + C::TILE;
      wait_vmem<0>();  // Q, dO, O and LSE of this tile
      // D of the tile's rows: a lane holds half of row c32
      v8 dof[KS];
      float Dq = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        dof[ks] = lds_read16<v8>(dob, off.row[ks]);
#pragma unroll
        for (int i = 0; i < 8; ++i) Dq = __builtin_fmaf((float)of[ks][i], (float)dof[ks][i], Dq);
      }
      Dq = half_pair_sum(Dq) * (DROP ? dr.keep_prob : 1.0f);
      if (g == 0) {
        lds_write(stat, c32 * 4, -Dq);
        lds_write(stat, (C::BM + c32) * 4, lse * 1.4426950408889634f);
      }
      if (next) {
        wait_lds_all();  // every read of that stage has returned
        fetch(t + C::NW, b ^ 1);
        load_o(t + C::NW);
      }
      f32x16 s, dp;
      f32x4 l[4], d[4];  // statistics of the 16 query rows a lane holds in its accumulator registers
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        d[x] = lds_read16<f32x4>(stat, (8 * x + 4 * g) * 4);
        l[x] = lds_read16<f32x4>(stat, (C::BM + 8 * x + 4 * g) * 4);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = DROP ? 0.f : d[r >> 2][r & 3]; }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) dp = F::mfma(dof[ks], vf[ks], dp);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s = F::mfma(lds_read16<v8>(qb, off.row[ks]), kf[ks], s);
      uint32_t keep[4];
      if (DROP) keep_bytes_key_lane<IN_ORDER>(dr, head, krow, t * C::BM, lane, keep);
      const bool diag = CAUSAL && t == kt;
      float p[16], ds[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float pe = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], scale_log2, -l[r >> 2][r & 3]));
        if (diag) pe = c32 - 4 * g > 8 * (r / 4) + (r % 4) ? 0.f : pe;  // krow - t * BM = c32
        if (DROP) {
          // fp16: a compare and a select, behind which dS and its conversion are one v_fma_mix (us, masks -> so: causal
          // 2 x 128, d = 128 10.5 -> 10.4; 4 x 1024 equal).  bf16: masks (compare and select: 4 x 1024, d = 64 14.5
          // against 13.7, causal d = 128 26.4 against 25.5), but not at more than 64 columns without the causal mask (masks -> so: 2 x
          // 1000, d = 128 24.5 -> 24.0, d = 96 23.4 -> 22.9; 4 x 200, d = 128 12.3 -> 12.1).
          constexpr bool COMPARE = F::FINITE_DOT || (D > 64 && !CAUSAL);
          uint32_t kept;
          if (COMPARE) {
            kept = keep_reg(keep, r, dr.thr) ? 0xFFFFFFFFu : 0u;
          } else {
            if ((r & 3) == 0) keep[r >> 2] = keep_strip(keep[r >> 2], dr);
            kept = keep_mask(keep[r >> 2], r & 3);
          }
          p[r] = keep_float(kept, pe);
          ds[r] = dropout_ds<T>(kept, pe, p[r], dp[r], d[r >> 2][r & 3]);
        } else {
          p[r] = pe;
          ds[r] = pe * dp[r];
        }
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const v8 pf = pack8<T>(&p[8 * kk]), dsf = pack8<T>(&ds[8 * kk]);
        const int ro = kk * 16 * C::ROWB;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          dv[dt] = F::mfma(read_tr_pair<T>(dob, off.tr[0][dt] + ro, off.tr[1][dt] + ro), pf, dv[dt]);
          dk[dt] = F::mfma(read_tr_pair<T>(qb, off.tr[0][dt] + ro, off.tr[1][dt] + ro), dsf, dk[dt]);
        }
      }
    };
    int b = 0;
    for (int t = t0 + wave; t < nqt; t += C::NW) {
      tile(t, b, t + C::NW < nqt);
      b ^= 1;
    }
    const int used = nqt - t0 < C::NW ? nqt - t0 : C::NW;
    merge_store<T, D>(dk, DROP ? scale * dr.rescale : scale, used, smem, tid, dK + head_base(mdk, head, H), k0, Nk,
                      (size_t)mdk.row, dh);
    merge_store<T, D>(dv, DROP ? dr.rescale : 1.0f, used, smem, tid, dV + head_base(mdv, head, H), k0, Nk,
                      (size_t)mdv.row, dh);
  }
}

}  // namespace spark
