// Attention forward for grids that leave most of the chip idle: few queries (down to one row per
// head), few heads, short sequences.
//
// mha_fwd_kernel gives a workgroup 128 query rows and walks the keys in one serial chain; with 64
// such workgroups three quarters of the CUs have nothing to do and the others run one wave per
// SIMD, so the time is the chain of N_k / 64 iterations (0.7 us each at d = 64, 1.0 us at d = 128).
// Here a workgroup owns 32 query rows and its 8 waves split the KEYS: wave w takes key tiles w,
// w + 8, ..., keeps its own (m, l, O) and the eight partial results are merged once at the end
// through LDS with Eq. 3 of Sec. 3.2.1.  That gives four times as many workgroups, two waves per
// SIMD, and chains an eighth as long.
//
// Every wave has its own K and V buffer in LDS (8 KB each) and fills it itself by direct
// global->LDS loads, so the loop has no barrier at all: the next K tile is requested as soon as
// the scores have consumed the present one, the next V tile as soon as P V has, and each wait is a
// vmcnt that leaves the other request in flight.  128 KB per CU are then in flight or in use, which
// is what a single query row, a pure read of K and V, needs to approach the memory rate.
// The price is operand traffic: K and V are read from L2 once per 32 query rows instead of once per
// 128 (8 waves on 8 KB + 8 KB of their own per 32 x 32 ... 64 block, against 64 B per clock from L2:
// about the rate of one wave per SIMD of the other kernel), hence only for grids that fit the chip in
// one go, or in two where the chains are long (the rule and its times: split_forward).  With a few rows against a long memory even these are few (8 heads: 8 workgroups on 256 CUs); then
// several workgroups share the keys of a query tile and a small kernel merges them (2 queries, 8 heads, 8318
// keys, d = 128: 64.0 -> 19.3 us).  Measured: 1 head, N = 8192: d = 64 fp16 91 -> 29 us, d = 128 134 -> 51 us; one query row
// against 2048 keys, 128 heads, d = 128: 40.7 -> 29.3 us (4.6 TB/s, the rate of a large copy).
#pragma once
#include "dropout_gfx950.hpp"
#include "mma_gfx950.hpp"
#include "tiles_gfx950.hpp"

namespace spark {

template <int D> struct FwdSplitCfg {
  static constexpr int NW = 8;                   // waves = key streams of a workgroup
  static constexpr int BM = 32;                  // query rows per workgroup
  static constexpr int BN = D == 64 ? 64 : 32;   // keys per tile: 8 KB of K, 8 KB of V
  static constexpr int ROWB = D * 2;
  static constexpr int TILE = BN * ROWB;
  static constexpr int NLOAD = TILE / 1024;      // direct loads per tile of K or V
  static constexpr int GROUPS = D / 8;           // accumulator quads (4 registers) per lane
  static constexpr int GPW = GROUPS / NW;        // ... that each wave sums in the merge
  static constexpr int XCH = NW * NW * GPW * 1024;  // partial O: [source wave][summing wave][quad][lane]
  static constexpr int BUF = NW * 2 * TILE > XCH ? NW * 2 * TILE : XCH;
  static constexpr int STAT0 = BUF;              // m and l: [wave][row]
  static constexpr int OSTR = D * 2 + 16;
  static constexpr int STG0 = STAT0 + 2 * NW * BM * 4;  // 16-bit rows on their way out
  static constexpr int SMEM = STG0 + BM * OSTR;
};

// PART (not causal): `parts` workgroups share the keys of a query tile; each leaves its m, l and unnormalised
// O of the rows below Nq in fp32, and mha_fwd_combine_kernel merges them.
template <typename T, int D, bool CAUSAL, bool DROP, bool PART = false>
__global__ __launch_bounds__(512, 1) void mha_fwd_split_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ LSE, TensorMap mq, TensorMap mk, TensorMap mv, TensorMap mo, int H, int Nq, int Nk,
    int dh, int nqt, int paired, float scale_log2, Dropout dr, int parts, float* __restrict__ partial) {
  using F = Frag<T>;
  using v8 = typename F::v8;
  using v4 = typename F::v4;
  using C = FwdSplitCfg<D>;
  constexpr int KS = D / 16, DT = D / 32, HALVES = C::BN / 32;

  SPARK_LDS char* const smem = lds_origin();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr Lanes LANES = DROP && !(CAUSAL && D == 128) ? NEAR : IN_ORDER;
  const int g = lane >> 5, c32 = column_row<LANES>(lane);
  SPARK_LDS char* const kb = smem + wave * 2 * C::TILE;
  SPARK_LDS char* const vb = kb + C::TILE;

  // causal: query tiles (nqt-1-p, p) are paired for equal work, unless there are so few tiles that
  // each gets a CU of its own
  const int items = paired ? causal_items<CAUSAL>(nqt) : nqt;
  const int flat = xcd_contiguous(blockIdx.x, gridDim.x);
  const int logical = PART ? flat / parts : flat, part = PART ? flat - logical * parts : 0;
  const int head = logical / items;
  const int item = logical - head * items;

  const BufView kview(K + head_base(mk, head, H), head_span_bytes(mk, Nk, dh));
  const BufView vview(V + head_base(mv, head, H), head_span_bytes(mv, Nk, dh));
  const uint32_t k_row_bytes = (uint32_t)mk.row * 2, v_row_bytes = (uint32_t)mv.row * 2;
  const WaveDma<D> kdma(lane, k_row_bytes, dh), vdma(lane, v_row_bytes, dh);
  const SwzLane<D> off(lane);

  for (int rep = 0; rep < (CAUSAL && paired ? 2 : 1); ++rep) {
    const int qt = CAUSAL && rep == 0 ? nqt - 1 - item : item;
    if (CAUSAL && rep == 1) {
      if (qt == nqt - 1 - item) break;  // odd tile count: the middle tile has no partner
      __syncthreads();                  // the first tile's output has left the LDS
    }
    const int q0 = qt * C::BM, qrow = q0 + c32;
    const T* qp = Q + head_base(mq, head, H) + (size_t)(qrow < Nq ? qrow : Nq - 1) * (size_t)mq.row;

    int kv_end = Nk;
    if (CAUSAL && q0 + C::BM < Nk) kv_end = q0 + C::BM;
    int nt = (kv_end + C::BN - 1) / C::BN;
    int j0 = 0;  // this workgroup's tiles are [j0, nt)
    if (PART) {
      const int per = (nt + parts - 1) / parts;
      j0 = part * per;
      nt = j0 + per < nt ? j0 + per : nt;  // the host leaves no part without a tile
    }
    // tiles [0, n_plain) need no mask: they end within the keys and, if causal, at or below row q0
    int n_plain = Nk / C::BN;
    if (CAUSAL && (q0 + 1) / C::BN < n_plain) n_plain = (q0 + 1) / C::BN;

    v8 qf[KS];
    load_row_frags(qf, qp, g, dh);

    f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    float m_run = -1e30f;  // finite, so that a masked score (-inf) minus the reference is not NaN
    float l_run = 0.f;

    auto fetch_k = [&](int j) { kdma.template tile<C::BN>(kview, j * C::BN, kb, k_row_bytes); };
    auto fetch_v = [&](int j) { vdma.template tile<C::BN>(vview, j * C::BN, vb, v_row_bytes); };
    if (j0 + wave < nt) {
      fetch_k(j0 + wave);
      fetch_v(j0 + wave);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]));  // Q is awaited here, not in the loop

    const int last_key = (CAUSAL && qrow < Nk ? qrow : Nk - 1) - 4 * g;  // as in mha_fwd_kernel
    // One tile; next: this wave has another one.  On entry at most NLOAD loads of K and, behind them,
    // NLOAD of V are outstanding.
    auto tile = [&](const int j, auto masked_tag, const bool next) {
      constexpr bool MASKED = decltype(masked_tag)::value;
      const int k0 = j * C::BN;
      f32x16 s[HALVES];
#pragma unroll
      for (int h = 0; h < HALVES; ++h)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[h][r] = 0.f;
      wait_vmem<C::NLOAD>();  // K is here; V may still be on its way
      v8 kf[HALVES][KS];
#pragma unroll
      for (int h = 0; h < HALVES; ++h)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[h][ks] = lds_read16<v8>(kb, off.row[ks] + h * 32 * C::ROWB);
#pragma unroll
      for (int h = 0; h < HALVES; ++h)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s[h] = F::mfma(kf[h][ks], qf[ks], s[h]);
      if (next) {
        wait_lds_all();  // every read of this K tile has returned
        fetch_k(j + C::NW);
      }

      float t[HALVES * 16];
      auto load_scores = [&](int h) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          t[h * 16 + r] = s[h][r];
          if (MASKED) {
            if (h * 32 + 8 * (r / 4) + (r % 4) > last_key - k0) t[h * 16 + r] = -INFINITY;
          }
        }
      };
      auto exp_all = [&]() {
        float rs = 0.f;
#pragma unroll
        for (int i = 0; i < HALVES * 16; ++i) {
          t[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(t[i], scale_log2, -m_run));
          rs += t[i];
        }
        return rs;
      };
#pragma unroll
      for (int h = 0; h < HALVES; ++h) load_scores(h);
      // lazy reference as in mha_fwd_kernel: exponentials against the present one first; only if
      // the row sum shows that it was too low, the maximum, the rescale of Eq. 3 and P once more
      float rs = exp_all();
      if (__any(!(rs <= 256.0f))) {
#pragma unroll
        for (int h = 0; h < HALVES; ++h) load_scores(h);
        float mx = t[0];
#pragma unroll
        for (int i = 1; i < HALVES * 16; ++i) mx = fmaxf(mx, t[i]);
        const float m_new = fmaxf(m_run, half_pair_max(mx) * scale_log2);
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
        rs = exp_all();
      }
      l_run += rs;
      if (DROP) {
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
          uint32_t keep[4];
          keep_bytes_query_lane<LANES>(dr, head, qrow, k0 + 32 * h, lane, keep);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            if (!keep_reg(keep, r, dr.thr)) t[h * 16 + r] = 0.f;
            asm volatile("" : "+v"(t[h * 16 + r]));  // the select stays in front of the packed conversion
          }
        }
      }
      if (next)
        wait_vmem<C::NLOAD>();  // V is here; the next K may still be on its way
      else
        wait_vmem<0>();
#pragma unroll
      for (int kk = 0; kk < 2 * HALVES; ++kk) {
        const v8 pf = pack8<T>(&t[8 * kk]);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const int ro = kk * 16 * C::ROWB;
          o[dt] = F::mfma(read_tr_pair<T>(vb, off.tr[0][dt] + ro, off.tr[1][dt] + ro), pf, o[dt]);
        }
      }
      if (next) {
        wait_lds_all();
        fetch_v(j + C::NW);
      }
    };
    int j = j0 + wave;
    if (n_plain > nt) n_plain = nt;
    for (; j < n_plain; j += C::NW) tile(j, std::false_type{}, j + C::NW < nt);
    for (; j < nt; j += C::NW) tile(j, std::true_type{}, j + C::NW < nt);

    // ---- merge of the partial results (Eq. 3) ----
    l_run = half_pair_sum(l_run);
    SPARK_LDS float* const stat = reinterpret_cast<SPARK_LDS float*>(smem + C::STAT0);
    if (g == 0) {
      stat[wave * C::BM + c32] = m_run;
      stat[(C::NW + wave) * C::BM + c32] = l_run;
    }
    __syncthreads();  // also: every wave has left its tiles
    const int used = nt - j0 < C::NW ? nt - j0 : C::NW;  // the waves behind that had no tile
    float m_all = stat[c32];
    for (int w = 1; w < used; ++w) m_all = fmaxf(m_all, stat[w * C::BM + c32]);
    float l_all = 0.f;
    for (int w = 0; w < used; ++w)
      l_all += stat[(C::NW + w) * C::BM + c32] * __builtin_amdgcn_exp2f(stat[w * C::BM + c32] - m_all);
    const float mul = __builtin_amdgcn_exp2f(m_run - m_all) * (PART ? 1.0f : (DROP ? dr.rescale : 1.0f) / l_all);
    const size_t prow = ((size_t)head * Nq + qrow) * (size_t)(PART ? parts : 1) + part;  // row of the partial result
    if (wave < used) {
#pragma unroll
      for (int q = 0; q < C::GROUPS; ++q) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = o[q / 4][(q % 4) * 4 + e] * mul;
        // quad q goes to wave q / GPW, in the lane order of the accumulators (no bank conflicts)
        lds_write(smem, (wave * C::GROUPS + q) * 1024 + lane * 16, x);
      }
    }
    __syncthreads();
#pragma unroll
    for (int gi = 0; gi < C::GPW; ++gi) {
      const int q = wave * C::GPW + gi;
      f32x4 sum = lds_read16<f32x4>(smem, q * 1024 + lane * 16);
      for (int w = 1; w < used; ++w) sum += lds_read16<f32x4>(smem, (w * C::GROUPS + q) * 1024 + lane * 16);
      if (PART) {
        if (qrow < Nq) *reinterpret_cast<f32x4*>(partial + prow * (D + 4) + 8 * q + 4 * g) = sum;
        continue;
      }
      v4 pk;
#pragma unroll
      for (int e = 0; e < 4; ++e) pk[e] = (T)sum[e];
      lds_write(smem + C::STG0, c32 * C::OSTR + (8 * q + 4 * g) * 2, pk);
    }
    if (PART) {
      if (wave == 0 && g == 0 && qrow < Nq) {
        *reinterpret_cast<f32x4*>(partial + prow * (D + 4) + D) = f32x4{m_all, l_all, 0.f, 0.f};
      }
      return;
    }
    __syncthreads();
    constexpr int CPR = D / 8;
    const int row = tid / CPR, cc = tid % CPR;
    if (row < C::BM && q0 + row < Nq && cc * 8 < dh)
      *reinterpret_cast<u32x4*>(O + head_base(mo, head, H) + (size_t)(q0 + row) * (size_t)mo.row + cc * 8) =
          lds_read16<u32x4>(smem + C::STG0, row * C::OSTR + cc * 16);
    if (wave == 0 && g == 0 && qrow < Nq)
      LSE[(size_t)head * Nq + qrow] = (m_all + __builtin_amdgcn_logf(l_all)) * 0.6931471805599453f;
  }  // rep
}

// Merge of the partial results of a row (Eq. 3): D / 4 lanes per row.  A partial result is D + 4 floats: O, m,
// l, two unused (16-byte alignment).
template <typename T, int D, bool DROP>
__global__ __launch_bounds__(256) void mha_fwd_combine_kernel(const float* __restrict__ partial, T* __restrict__ O,
                                                              float* __restrict__ LSE, TensorMap mo, int H, int Nq,
                                                              int dh, int rows, int parts, float rescale) {
  using v4 = typename Frag<T>::v4;
  constexpr int LPR = D / 4;
  const int row = blockIdx.x * (256 / LPR) + threadIdx.x / LPR;  // flat (head, query) index
  const int col = (threadIdx.x % LPR) * 4;
  if (row >= rows) return;
  const float* p = partial + (size_t)row * (size_t)parts * (D + 4);
  // four parts at a time, so that their loads are in flight together; behind the last part its weight is 0
  float m = p[D];
  for (int s = 1; s < parts; s += 4) {
    float x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = p[(size_t)(s + u < parts ? s + u : 0) * (D + 4) + D];
#pragma unroll
    for (int u = 0; u < 4; ++u) m = fmaxf(m, x[u]);
  }
  float l = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < parts; s += 4) {
    f32x4 x[4], st[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float* ps = p + (size_t)(s + u < parts ? s + u : 0) * (D + 4);
      st[u] = *reinterpret_cast<const f32x4*>(ps + D);
      x[u] = *reinterpret_cast<const f32x4*>(ps + col);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (s + u >= parts) break;
      const float w = __builtin_amdgcn_exp2f(st[u][0] - m);
      l += st[u][1] * w;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = __builtin_fmaf(x[u][e], w, o[e]);
    }
  }
  const int head = row / Nq, q = row - head * Nq;
  const float inv = (DROP ? rescale : 1.0f) / l;
  if (col < dh) {
    v4 pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = (T)(o[e] * inv);
    *reinterpret_cast<v4*>(O + head_base(mo, head, H) + (size_t)q * (size_t)mo.row + col) = pk;
  }
  if (col == 0) LSE[row] = (m + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
}

}  // namespace spark
