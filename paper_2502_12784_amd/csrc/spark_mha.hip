// C ABI of the fused MHA library: argument validation and kernel dispatch (host side).
// The operations are defined in include/spark_mha.h.
#include "../../include/spark_mha.h"

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <atomic>

#include "bwd_atomic_kernels.hpp"
#include "bwd_kernels.hpp"
#include "bwd_split_kernel.hpp"
#include "fwd_kernel.hpp"
#include "fwd_split_kernel.hpp"
#include "layout_probe.hpp"

// Scratch memory of spark_mha_bwd_static: the backward's workspace (D and LSE * log2(e)) for callers
// that cannot allocate.  One copy per GPU, at its own address on each, held until the process ends.
// In host code this name is only a handle for hipGetSymbolAddress, never a device address.
#define SPARK_STATIC_SCRATCH_BYTES (8u << 20)
static __device__ __align__(256) unsigned char scratch[SPARK_STATIC_SCRATCH_BYTES];

namespace {

using namespace spark;

// Device address of `scratch` on the current device, looked up once per device with that device
// current and kept; nullptr if the runtime cannot resolve it.
void* static_scratch_ptr() {
  static std::atomic<void*> ptrs[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  void* p = ptrs[dev].load(std::memory_order_acquire);
  if (p) return p;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
  ptrs[dev].store(p, std::memory_order_release);  // every thread resolves the same address
  return p;
}

// hipGetLastError() == hipSuccess, and with SPARK_MHA_DEBUG set in the environment the runtime's own
// description of a failure on stderr (the C ABI itself only returns SPARK_ERR_LAUNCH).
bool launch_ok(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return true;
  static const bool verbose = getenv("SPARK_MHA_DEBUG") != nullptr;
  if (verbose) fprintf(stderr, "spark_mha: %s: %s\n", what, hipGetErrorString(e));
  return false;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Everything one problem is made of; the entry points fill it and hand it to the launchers.
struct Problem {
  int B, H, Nq, Nk, d;
  float scale;
  int causal;
  int dtype;
  int thr;  // dropout threshold, 0 = no dropout
  unsigned long long seed;
  unsigned offset;
  // element strides of the [B,H,N,d] tensors
  TensorMap mq, mk, mv, mo, mdo, mdq, mdk, mdv;
  hipStream_t st;
  void* fwd_ws;  // the forward's optional workspace, large enough, or nullptr
};

TensorMap contiguous(int H, int N, int d) {
  return TensorMap{(long long)H * N * d, (long long)N * d, (long long)d};
}

// Nq queries attend to Nk keys; self-attention passes the same N twice.
int check_common(int B, int H, int Nq, int Nk, int d, float scale, int causal, int dtype) {
  if (dtype != SPARK_F16 && dtype != SPARK_BF16) return SPARK_ERR_DTYPE;
  if (B < 1 || H < 1 || Nq < 1 || Nk < 1) return SPARK_ERR_SHAPE;
  if (causal && Nq != Nk) return SPARK_ERR_SHAPE;  // the mask is defined for a square S only
  if (d < 8 || d > 128 || (d & 7)) return SPARK_ERR_SHAPE;  // rows of 16-byte chunks, tiles up to 128 wide
  if (!isfinite(scale) || !(scale > 0.f)) return SPARK_ERR_SHAPE;
  const int64_t bh = (int64_t)B * H;
  const int64_t nmax = Nq > Nk ? Nq : Nk;
  const int64_t tiles64 = (nmax + 63) / 64;
  if (bh * tiles64 >= (int64_t)1 << 31) return SPARK_ERR_SHAPE;
  // 31-bit byte offsets inside one head, including the rows a ragged last tile reaches past N
  if ((nmax + 256) * d * 2 >= (int64_t)1 << 31) return SPARK_ERR_SHAPE;
  return SPARK_OK;
}

// A strided tensor is usable if rows hold d contiguous elements, every stride keeps 16-byte
// alignment, and one head's rows span less than 4 GiB (the kernels address a head through a
// 32-bit buffer descriptor).
// An output tensor must in addition give every (batch, head) its own rows: a zero batch or head stride
// (a broadcast, fine for an input) would make all those workgroups store to the same memory.
int check_strides(const spark_strides_t* s, int N, int d, TensorMap* out, bool is_output = false, int B = 1,
                  int H = 1) {
  if (!s) return SPARK_ERR_NULL;
  if (s->batch < 0 || s->head < 0 || s->row < d) return SPARK_ERR_SHAPE;
  if (is_output && ((B > 1 && s->batch == 0) || (H > 1 && s->head == 0))) return SPARK_ERR_SHAPE;
  if ((s->batch | s->head | s->row) & 7) return SPARK_ERR_ALIGN;
  // 31-bit byte offsets inside one head, including the rows a ragged last tile reaches past N
  // (offsets from 2^31 on are how the kernels mark chunks that must read as zeros)
  if ((int64_t)(N + 256) * s->row * 2 >= (int64_t)1 << 31) return SPARK_ERR_SHAPE;
  *out = TensorMap{s->batch, s->head, s->row};
  return SPARK_OK;
}

// Dropout rate -> 8-bit threshold: an entry is dropped iff its random byte < thr, i.e. with
// probability thr / 256.  -1 if the rate is not a number in [0, 255.5/256).
int drop_threshold(float p_drop) {
  if (!(p_drop >= 0.f) || !(p_drop < 1.f)) return -1;
  const int thr = (int)floorf(p_drop * 256.0f + 0.5f);
  return thr <= 255 ? thr : -1;
}

Dropout make_dropout(int thr, unsigned long long seed, unsigned offset) {
  Dropout dr;
  dr.key0 = (uint32_t)seed;
  dr.key1 = (uint32_t)(seed >> 32);
  dr.offset = offset;
  dr.thr = (uint32_t)thr;
  dr.keep_add = thr ? (uint32_t)(256 - thr) * 0x01010101u : 0;  // of use to kernels with dropout only
  dr.keep_prob = (float)(256 - thr) / 256.0f;
  dr.rescale = 256.0f / (float)(256 - thr);
  return dr;
}

template <typename KernelT>
int set_smem(KernelT kernel, int bytes) {
  // The kernels address LDS from 0 (lds_origin): that holds only without static LDS in front.
  hipFuncAttributes fa;
  if (hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(kernel)) != hipSuccess || fa.sharedSizeBytes != 0) {
    if (getenv("SPARK_MHA_DEBUG")) fprintf(stderr, "spark_mha: kernel attributes unavailable or static LDS present\n");
    return SPARK_ERR_LAUNCH;
  }
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess && getenv("SPARK_MHA_DEBUG"))
    fprintf(stderr, "spark_mha: hipFuncSetAttribute(%d bytes of LDS): %s\n", bytes, hipGetErrorString(e));
  return e == hipSuccess ? SPARK_OK : SPARK_ERR_LAUNCH;
}

// set_smem once per kernel and device: the attribute belongs to the function on the current
// device, so a process that drives several GPUs needs it on each of them.  `done` holds one bit
// per device ordinal; a failure is not remembered, the next call tries again.
template <typename KernelT>
int ensure_smem(KernelT kernel, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return SPARK_ERR_LAUNCH;
  if (dev < 64 && ((done.load(std::memory_order_acquire) >> dev) & 1u)) return SPARK_OK;
  const int rc = set_smem(kernel, bytes);
  if (rc == SPARK_OK && dev < 64) done.fetch_or(uint64_t(1) << dev, std::memory_order_release);
  return rc;
}

// Workgroups of 8 waves (256 query rows, one per CU) instead of 4 (128 rows, two per CU): each
// K/V tile brought into LDS then serves twice as many MFMAs.  Pays at d = 128 when the loop over the keys is
// long enough to outweigh running one workgroup per CU with nothing to overlap its prologue and epilogue
// (measured on the grid of Sec. 4.1, hidden size 2048: -5 ... -7 % from 2048 keys on, +7 ... +10 %
// at 512, equal at 1024; at d = 64 it costs 2 %) and the last round of one per CU is not nearly empty:
// two rounds or more, almost two, or one round where the narrow grid puts two workgroups on some CU (the time is
// that CU's).  Forward, bf16, us, narrow -> wide (n wide workgroups):
//   16 heads x 4096 (256) 125.6 -> 117.0   24 x 2048 (192) 59.1 -> 52.8   40 x 1024 over 4096 keys (160) 105.8 -> 93.8
//   causal 8 x 16384 (256) 503.7 -> 456.9   24 x 4096 (192) 122.3 -> 111.7   64 x 2048 (256) 80.6 -> 81.4 (one run each; below)
//   not taken: 40 x 2048 (320) 95.1 -> 107.5   12 x 8192 (384) 369 -> 394   causal 40 x 4096 (320) 211.7 -> 225.4
//   almost two: 56 x 2048 (448) 121.2 -> 113.7   causal 112 x 2048 (448) 145.8 -> 140.0
// Checked over 68 problems around these two classes (medians in alternating order; with dropout and d = 72 ... 104 among them):
// 0.85 ... 0.99 of the narrow kernel's time at all that are taken, among them causal 64 x 2048 83.9 -> 78.5 and with dropout
// 101.7 -> 98.5, 43 x 700 over 2048 (129 against 258, the fewest) 56.1 -> 52.4, 450 x 250 over 2100 152.9 -> 150.9; not
// taken 1.08 ... 1.76, except 20 x 5000 (400, d = 96) 273.6 -> 247.3.  The kernels of 96 columns, over 19 problems on both
// sides: taken 0.91 ... 0.98 (43 x 700 over 2048 42.6 -> 39.2, causal 24 x 4096 93.4 -> 84.8, 128 x 2048 118.5 -> 115.9), not
// taken 1.07 ... 1.14, except 20 x 5000 232.0 -> 210.3 and, with fewer keys, 64 x 1024 30.9 -> 29.2.
template <bool CAUSAL>
bool wide_workgroups(const Problem& p) {
  const int64_t bh = (int64_t)p.B * p.H;
  const int64_t wide = bh * causal_items<CAUSAL>((p.Nq + 255) / 256);
  const int64_t narrow = bh * causal_items<CAUSAL>((p.Nq + 127) / 128);
  return p.d > 64 && p.Nk >= 2048 && (wide >= 512 || narrow >= 896 || (wide <= 256 && narrow > 256));
}

// Whether a causal grid runs as complementary pairs of tiles, (n-1-p, p) in one workgroup: equal work for
// every workgroup, at the price of half as many of them, each with two prologues and epilogues in
// series.  `n` tiles per head, `bh` heads, `per_cu` workgroups of the kernel on a CU.  Not paired:
//  * up to one tile per CU: the longest tile alone is shorter than a pair (forward / dQ / dK/dV, paired ->
//    unpaired us, 256 tiles: N = 256 d = 64 11.9/16.9/17.1 -> 8.0/12.1/12.4; N = 1024 d = 128
//    30.3/42.0/44.2 -> 24.8/33.6/37.1; N = 4096 d = 64 53.6/61.9/75.8 -> 49.3/55.6/70.4; from 320 tiles on
//    the pairs win: N = 4096 53.5/61.5/75.9 against 67.8/81.3/100.8);
//  * two tiles per head while all are resident: lengths differ by a factor of two at most (512 tiles, d = 64
//    12.2/19.5/18.6 -> 10.5/17.0/17.8; dK/dV with dropout 130 x 256 19.5 -> 18.4, 256 x 256 21.4 -> 20.5, 256 x 192
//    equal; both sides in one grid 66 x 256 19.5 -> 18.2, 128 x 200 19.9 -> 19.4);
//  * three tiles per head: the middle one stays alone in a workgroup with half the others' work (2049 tiles,
//    d = 128: 79/135/175 -> 65/108/139), unless a kernel with one workgroup per CU fits its pairs in one round and
//    its tiles not (dK/dV, d = 128, paired / unpaired: 92 heads 28.4 / 30.8, 118 heads 24.8 / 30.0, 127 heads
//    30.1 / 34.0; both sides in one grid, 47 heads 25.3 / 27.2, 59 heads 26.8 / 32.4; but 86 heads, two tiles
//    too many, 24.2 / 19.2, and 132 heads, pairs in two rounds, unpaired is 0.7 of it; d = 64, two per CU, with dropout
//    100 x 384 22.5 / 21.5, both sides 64 x 384 22.8 / 20.2, 45 x 300 18.7 / 17.7; 96 columns as 128: 92 heads x 384
//    23.8 / 25.3, 127 24.8 / 28.6, but 86 23.7 / 19.6, 129 42.6 / 28.7; two tiles 140 x 256 21.2 / 25.6, 250 25.3 / 29.8).
int pair_tiles(bool causal, int64_t bh, int n, int per_cu) {
  if (!causal || bh * n <= 256) return 0;
  if (n == 3) return per_cu == 1 && bh > 88 && bh <= 128;
  return !(n == 2 && bh * n <= 256 * per_cu);
}

template <typename T, int D, bool CAUSAL, bool DROP, int NW, bool PAIR = false>
int launch_fwd_nw(const Problem& p, const void* Q, const void* K, const void* V, void* O, float* LSE) {
  using C = FwdCfg<D, NW, PAIR>;
  auto kernel = mha_fwd_kernel<T, D, CAUSAL, DROP, NW, PAIR>;
  static std::atomic<uint64_t> ready{0};
  const int attr = ensure_smem(kernel, C::SMEM, ready);
  if (attr != SPARK_OK) return attr;
  const int BH = p.B * p.H;
  const int nqt = (p.Nq + C::BM - 1) / C::BM;
  const float scale_log2 = p.scale * 1.4426950408889634f;
  // Three tiles per head at two workgroups per CU: paired only where the pairs fit one round and the tiles are well
  // past it, and only here (d = 128, paired / unpaired us: 188 x 384 27.1 / 25.6, 200 x 300 23.6 / 24.4, 233 x 270
  // 24.1 / 26.0, 257 x 306 34.6 / 25.7; with dropout 228 x 384 35.3 / 34.8; at d = 64 three workgroups fit, and dQ
  // gains unpaired: 244 heads 0.9 of it; at 96 columns 200 x 300 16.4 / 16.2, 233 x 270 16.6 / 17.0, 256 x 384 20.2 / 19.6).
  const bool one_round = D > 64 && !DROP && nqt == 3 && BH > 192 && BH <= 256;
  const int paired = CAUSAL && one_round ? 1 : pair_tiles(CAUSAL, BH, nqt, NW == 4 ? 2 : 1);
  hipLaunchKernelGGL(kernel, dim3((unsigned)(BH * (paired ? causal_items<true>(nqt) : nqt))), dim3(64 * NW), C::SMEM,
                     p.st, static_cast<const T*>(Q), static_cast<const T*>(K), static_cast<const T*>(V),
                     static_cast<T*>(O), LSE, p.mq, p.mk, p.mv, p.mo, p.H, p.Nq, p.Nk, p.d, nqt, paired, scale_log2,
                     make_dropout(p.thr, p.seed, p.offset));
  return launch_ok("forward kernel") ? SPARK_OK : SPARK_ERR_LAUNCH;
}

// Grid of mha_fwd_split_kernel (32 query rows per workgroup, one workgroup per CU).  Causal tiles are
// paired for equal work only when they would not each get a CU of their own.
template <bool CAUSAL>
int64_t fwd_split_workgroups(const Problem& p, int* paired) {
  const int nqt = (p.Nq + 31) / 32;
  const int64_t bh = (int64_t)p.B * p.H;
  *paired = CAUSAL && bh * nqt > 256;
  return bh * (*paired ? causal_items<true>(nqt) : nqt);
}

// The split forward needs keys to split (up to 256 of them the merge costs what the shorter chain
// gains: 5.1 -> 5.2 us at N = 192, d = 64) and every workgroup resident at once, or long chains in two rounds
// (an eighth of the chain, twice): measured, fp16
// d = 64 / bf16 d = 128, us, mha_fwd_kernel -> split:
//   1 head, N = 8192 (256 workgroups)       91 -> 29  / 134 -> 51
//   8 heads, N = 1024 (256)                14.6 -> 8.0 / 20.6 -> 11.7
//   1 query, 128 heads, 2048 keys (128)          -    / 40.7 -> 29.3
//   1 query, 256 heads, 2048 keys (256)    30.8 -> 26.0 / 50.3 -> 50.5
//   16 heads, N = 1024 (512)               14.7 -> 14.9 / 21.1 -> 23.6 (not taken)
//   8 heads, N = 2048 (512)                26.4 -> 20.1 / 37.6 -> 31.9   1 head, N = 16384  184 -> 103 / 266 -> 190
//   causal, 6 heads, N = 4096 (384)        48.9 -> 39.5 / 85.0 -> 61.4   12 heads, N = 2048 (384) 27.1 -> 29.6 (not)
//   12 heads, N = 2048 (768)               26.6 -> 29.0 / 37.9 -> 46.6 (not)
// Not beyond one round where a few rows per head of nearly 128 columns make the time a read of K and V: a second,
// mostly empty round then costs more than the split saves (mha_fwd_kernel's heads of one tile fit at once).  So for up to 32
// rows below 320 workgroups, up to 64 rows, and up to 128 rows from 400 MB of K and V on, which no cache holds (d = 128,
// rows x heads over keys: 15 x 257 over 3840 101 -> 118, 32 x 288 over 6541 186 -> 207, 40 x 150 over 5000 101 -> 106,
// 85 x 150 over 11264 216 -> 230; equal at 1 x 350 over 3071 and 96 x 100 over 8191).  With 512 heads and more the other kernel would be
// the 8-wave one (2 x 512 over 2048 146 -> 104).  Nor, in a nearly full round, up to 704 keys for heads of one tile: two or
// three key tiles per wave (32 x 256, d = 128, over 384 12.0 -> 13.2, over 512 14.3 -> 15.3).  With dropout the split wins
// at all of these.
template <bool CAUSAL>
bool split_forward(const Problem& p) {
  int paired;
  const int64_t bh = (int64_t)p.B * p.H, n = fwd_split_workgroups<CAUSAL>(p, &paired);
  if (p.Nk <= 256 || n > (p.Nk >= (CAUSAL ? 4096 : 2048) ? 512 : 256)) return false;
  if (CAUSAL || p.thr || p.d <= 96) return true;
  if (n <= 256) return !(p.d > 112 && n > 224 && p.Nq <= 32 && p.Nk <= 704);
  if (bh >= 512 || p.Nq > 128) return true;
  if (p.Nq > 64) return bh * p.Nk * p.d * 4 < (int64_t)400 << 20;
  return p.d <= 112 || (p.Nq <= 32 && (p.d <= 120 || n >= 320));
}

// Workgroups that share the keys of one query tile, 1 = no sharing.  For grids of at most half the CUs: as
// many as give every CU a workgroup, with two rounds of tiles left to each of its 8 waves (one round left
// costs more in the merge than it saves), at most 16 (the merge walks them).  Worth the merge kernel, 3 us,
// from four rounds saved on; near 128 workgroups the memory rate is reached without sharing, and only long
// memories gain.  Forward, fp16, us, one workgroup -> shared, queries x heads over keys:
//   d = 64:   1 x 2 over 4096 15.2 -> 10.1    2 x 8 over 8318 25.7 -> 13.3    40 x 48 over 12096 58.3 -> 38.9
//             1 x 100 over 8192 50.0 -> 42.5  1 x 128 over 4096 29.3 -> 29.7 (not taken)
//   d = 128:  1 x 2 over 2048 15.6 -> 11.0    2 x 8 over 8318 64.0 -> 19.3    16 x 24 over 4067 42.9 -> 19.3
//             1 x 128 over 16384 204 -> 181   1 x 128 over 2048 29.9 -> 30.9 (not taken)
int fwd_parts(const Problem& p) {
  if (p.causal) return 1;
  const int64_t w = (int64_t)p.B * p.H * ((p.Nq + 31) / 32);
  if (w > 128) return 1;
  const int nt = p.d <= 64 ? (p.Nk + 63) / 64 : (p.Nk + 31) / 32;
  const int rounds = (nt + 7) / 8;
  int parts = (int)(256 / w);
  if (parts > rounds / 2) parts = rounds / 2;
  if (parts > 16) parts = 16;
  if (parts < 2 || rounds - rounds / parts < (w > 96 ? 8 : 4)) return 1;
  const int per = (nt + parts - 1) / parts;
  return (nt + per - 1) / per;  // no part without a tile
}

size_t fwd_workspace_bytes(const Problem& p) {
  const int parts = fwd_parts(p);
  return parts == 1 ? 0 : (size_t)p.B * p.H * p.Nq * parts * ((p.d <= 64 ? 64 : 128) + 4) * sizeof(float);
}

template <typename T, int D, bool DROP>
int launch_fwd_parts(const Problem& p, const void* Q, const void* K, const void* V, void* O, float* LSE, int parts) {
  using C = FwdSplitCfg<D>;
  auto kernel = mha_fwd_split_kernel<T, D, false, DROP, true>;
  static std::atomic<uint64_t> ready{0};
  const int attr = ensure_smem(kernel, C::SMEM, ready);
  if (attr != SPARK_OK) return attr;
  const int nqt = (p.Nq + C::BM - 1) / C::BM, rows = p.B * p.H * p.Nq;
  const Dropout dr = make_dropout(p.thr, p.seed, p.offset);
  float* partial = static_cast<float*>(p.fwd_ws);
  hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H * nqt * parts)), dim3(64 * C::NW), C::SMEM, p.st,
                     static_cast<const T*>(Q), static_cast<const T*>(K), static_cast<const T*>(V),
                     static_cast<T*>(O), LSE, p.mq, p.mk, p.mv, p.mo, p.H, p.Nq, p.Nk, p.d, nqt, 0,
                     p.scale * 1.4426950408889634f, dr, parts, partial);
  if (!launch_ok("forward kernel (shared keys)")) return SPARK_ERR_LAUNCH;
  constexpr int RPB = 256 * 4 / D;
  hipLaunchKernelGGL((mha_fwd_combine_kernel<T, D, DROP>), dim3((unsigned)((rows + RPB - 1) / RPB)), dim3(256), 0,
                     p.st, partial, static_cast<T*>(O), LSE, p.mo, p.H, p.Nq, p.d, rows, parts, dr.rescale);
  return launch_ok("forward merge kernel") ? SPARK_OK : SPARK_ERR_LAUNCH;
}

template <typename T, int D, bool CAUSAL, bool DROP>
int launch_fwd_split(const Problem& p, const void* Q, const void* K, const void* V, void* O, float* LSE) {
  using C = FwdSplitCfg<D>;
  auto kernel = mha_fwd_split_kernel<T, D, CAUSAL, DROP>;
  static std::atomic<uint64_t> ready{0};
  const int attr = ensure_smem(kernel, C::SMEM, ready);
  if (attr != SPARK_OK) return attr;
  const int nqt = (p.Nq + C::BM - 1) / C::BM;
  int paired;
  const int64_t grid = fwd_split_workgroups<CAUSAL>(p, &paired);
  hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * C::NW), C::SMEM, p.st,
                     static_cast<const T*>(Q), static_cast<const T*>(K), static_cast<const T*>(V),
                     static_cast<T*>(O), LSE, p.mq, p.mk, p.mv, p.mo, p.H, p.Nq, p.Nk, p.d, nqt, paired,
                     p.scale * 1.4426950408889634f, make_dropout(p.thr, p.seed, p.offset), 1, nullptr);
  return launch_ok("forward kernel (split keys)") ? SPARK_OK : SPARK_ERR_LAUNCH;
}

template <typename T, int D, bool CAUSAL, bool DROP>
int launch_fwd(const Problem& p, const void* Q, const void* K, const void* V, void* O, float* LSE) {
  if constexpr (!CAUSAL) {
    const int parts = p.fwd_ws ? fwd_parts(p) : 1;
    if (parts > 1) return launch_fwd_parts<T, lds_row<D>, DROP>(p, Q, K, V, O, LSE, parts);
  }
  if (split_forward<CAUSAL>(p)) return launch_fwd_split<T, lds_row<D>, CAUSAL, DROP>(p, Q, K, V, O, LSE);
  if constexpr (D > 64) {
    // ... with the K/V tiles requested two at a time and one barrier every second iteration (the
    // workgroup has the CU's LDS to itself): another -1 ... -3 % on the forward.
    if (wide_workgroups<CAUSAL>(p)) return launch_fwd_nw<T, D, CAUSAL, DROP, 8, true>(p, Q, K, V, O, LSE);
  }
  return launch_fwd_nw<T, D, CAUSAL, DROP, 4>(p, Q, K, V, O, LSE);
}

// Grid of mha_bwd_split_kernel: 32 queries or 32 keys per workgroup, one workgroup per CU.
int64_t bwd_split_workgroups(const Problem& p) {
  return (int64_t)p.B * p.H * ((p.Nq + 31) / 32 + (p.Nk + 31) / 32);
}
// It is taken while every CU has one workgroup, and up to two where the chains are long enough for their
// split to outweigh the second round (at d = 128 four waves split them instead of eight: only if causal, where
// the two rounds differ in length).  Measured against mha_bwd_merged_kernel, which is next, fp16, us,
// merged -> split (n workgroups), square problems of BH heads:
//   d = 64:   16 x 256 (256) 10.7 -> 8.4    4 x 1024 (256) 22.2 -> 13.2    32 x 256 (512) 11.0 -> 15.1
//             16 x 512 (512) 15.4 -> 18.3   8 x 1024 (512) 23.2 -> 22.5    2 x 4096 (512) 69.7 -> 57.8
//             16 x 1024 (1024) 24.9 -> 43.0     causal 8 x 1024 23.7 -> 18.6, 2 x 4096 71.3 -> 47.5
//   d = 128:  4 x 1024 (256) 35.6 -> 23.1   2 x 4096 (512) 122 -> 129      causal 2 x 4096 128 -> 102
bool split_backward(const Problem& p) {
  const int64_t n = bwd_split_workgroups(p);
  return n <= 256 || (n <= 512 && p.Nq >= 1024 && p.Nk >= 1024 && (p.d <= 64 || p.causal));
}

template <typename T, int D, bool CAUSAL, bool DROP>
int launch_bwd_split(const Problem& p, const void* Q, const void* K, const void* V, const void* O, const float* LSE,
                     const void* dO, void* dQ, void* dK, void* dV) {
  using C = BwdSplitCfg<D>;
  auto kernel = mha_bwd_split_kernel<T, D, CAUSAL, DROP>;
  static std::atomic<uint64_t> ready{0};
  const int attr = ensure_smem(kernel, C::SMEM, ready);
  if (attr != SPARK_OK) return attr;
  const Dropout dr = make_dropout(p.thr, p.seed, p.offset);
  hipLaunchKernelGGL(kernel, dim3((unsigned)bwd_split_workgroups(p)), dim3(64 * C::NW), C::SMEM, p.st,
                     static_cast<const T*>(Q), static_cast<const T*>(K), static_cast<const T*>(V),
                     static_cast<const T*>(O), static_cast<const T*>(dO), LSE, static_cast<T*>(dQ),
                     static_cast<T*>(dK), static_cast<T*>(dV), p.mq, p.mk, p.mv, p.mo, p.mdo, p.mdq, p.mdk, p.mdv,
                     p.H, p.Nq, p.Nk, p.d, (p.Nq + C::BM - 1) / C::BM, (p.Nk + C::BM - 1) / C::BM, p.scale,
                     DropoutLean{dr.key0, dr.key1, dr.offset, dr.thr, dr.keep_prob, dr.rescale});
  return launch_ok("backward kernel (split)") ? SPARK_OK : SPARK_ERR_LAUNCH;
}

// Both sides of the backward in one grid of 128-row tiles (mha_bwd_merged_kernel): where a kernel per side
// leaves CUs idle one after the other, at the price of a small kernel that forms D first.  Two workgroups of the
// grid fit a CU at d = 64, one at d = 128.  Backward, fp16, us, one kernel per side -> merged (n tiles of
// both sides), square problems of BH heads:
//   up to one tile per CU:  d = 64 128 x 128 (256) 12.3 -> 9.6, 16 x 1024 (256) 36.9 -> 26.5;
//                           d = 128 32 x 512 (256) 36.9 -> 25.7, 4 x 4096 (256) 198 -> 130
//   two per CU, d = 64:     8 x 4096 (512) 129 -> 118, 24 x 1024 (384) 36.9 -> 35.6, but 48 x 512 (384) equal and
//                           128 x 256 (512) 17.0 -> 17.7: only from 1024 rows on, and not beyond one round
//                           (36 x 1333 (792) 76.7 -> 81.1, 96 x 512 (768) 37.1 -> 37.9)
//   d = 128 beyond one:     the dQ side, two workgroups per CU in its own kernel, is held to one here:
//                           24 x 1024 (384) 62.7 -> 71.6
//   causal, paired, while the pairs of both sides are resident together: d = 64 32 x 1024 (512) 39.1 -> 30.2,
//                           3 x 8192 (384) 229 -> 140, 36 x 1333 (792) 58.2 -> 51.1, but 128 x 1024 (2048) 90.2 -> 91.1;
//                           d = 128 32 x 1024 (512) 65.3 -> 50.1, 8 x 4096 (512) 203 -> 142, but 96 x 512 (768)
//                           59.7 -> 64.2
//   causal, one tile per head (nothing to pair): while all are resident, three per CU at d = 64 without dropout;
//                           64 rows 114 heads (228) 10.4 -> 7.7, 359 (718) 14.3 -> 13.2, but 399 (798) 14.7 -> 15.0;
//                           d = 128 109 (218) 14.9 -> 10.7, but 213 (426) 16.2 -> 18.4; dropout, d = 64 114 x 128 (228)
//                           16.5 -> 11.6, but 133 x 128 (266) 21.9 -> 23.1, 256 x 128 (512) 22.9 -> 24.1
//   dropout, d = 64, causal: two and three tiles per head keep the line of one workgroup per CU (150 x 300 (900) 37.6 ->
//                           39.7), longer ones that of two (96 x 512 (768) 54.4 -> 50.0, 36 x 1333 (792) 85.4 -> 74.5,
//                           16 x 4096 (1024) 202 -> 182); not causal as without it (24 x 1024 (384) 53.9 -> 52.0, but
//                           128 x 256 (512) 25.6 -> 27.6)
//   d = 128 with few queries over many keys: the time is the dQ side's chain over the keys, whose iterations are
//                           slower here (more than 256 registers, so matrix results come through accumulation registers:
//                           1.3 of them without dropout, 1.15 with), against a launch and the other side's chain: 6 x 323 over 1457 50.5 -> 47.6,
//                           9 x 669 over 2235 73.9 -> 69.8, but 1 x 2 over 10565 227 -> 294, 4 x 32 over 4379 105 -> 127,
//                           6 x 254 over 1858 58.6 -> 59.8, 2 x 992 over 5424 146 -> 155; dropout 6 x 450 over 2837
//                           106 -> 102, but 2 x 592 over 4902 169 -> 172 (the line is where both are equal within 2 %; at 96 columns
//                           one grid wins up to 5 % further: 8 x 256 over 1536 37.3 -> 35.2, 1900 43.2 -> 42.3, 2400 50.4 -> 51.5,
//                           4 x 512 over 2400 55.6 -> 51.3, 3000 63.9 -> 61.8, 3500 equal; dropout 6 x 450 over 2837 79.1 -> 74.6,
//                           4500 111.4 -> 113.4)
bool merged_backward(const Problem& p) {
  const int per_cu = p.d <= 64 && !(p.thr && p.causal && p.Nq <= 384) ? 2 : 1;  // which line, as measured above
  if (p.d > 64 && !p.causal && p.Nk > (p.thr ? 7 * (int64_t)p.Nq + 640 : 4 * (int64_t)p.Nq + 512)) return false;
  const int64_t n = (int64_t)p.B * p.H * ((p.Nq + 127) / 128 + (p.Nk + 127) / 128);
  if (p.causal && p.Nq <= 128) return n <= 256 * (per_cu == 2 ? 3 : 1);
  if (p.causal) return n <= 512 * per_cu;
  return n <= 256 || (per_cu == 2 && n <= 512 && p.Nq >= 1024 && p.Nk >= 1024);
}

template <int D> constexpr int dkdv_per_cu = D == 64 ? 2 : 1;  // workgroups of the dK/dV and of the merged kernel on a CU

// How the kernels of 128-row tiles spread their rows over the lanes under dropout (column_row): far apart the exchange of the
// generator's words is cheaper, which is kept where no operand's rows load faster in order.  Neighbouring lanes' addresses agree
// in bit 6, in order if rows are a multiple of 128 bytes apart, far apart already at a multiple of 32.  Backward, us, fp16 / bf16,
// in order -> far:
//   d = 64:   64 heads x 2048 299 / 291 -> 292 / 283      512 x 192 48.0 / 47.5 -> 48.4 / 47.7
//             both sides in one grid: 8 x 2048 49.0 / 49.9 -> 48.3 / 48.9, causal 6 x 4000 96.0 / 99.1 -> 94.5 / 96.1
//   d = 128:  64 x 2048 524 / 505 -> 513 / 493, causal 301 / 291 -> 297 / 287      140 x 512 120.2 / 117.9 -> 119.8 / 117.6
//             but 512 x 192 94.1 / 93.0 -> 95.1 / 94.5, causal 140 x 512 109.1 / 107.9 -> 110.2 / 109.0: from 512 rows of the loop on
//   rows of 96 and 224 bytes, causal 140 x 512: d = 48 55.0 / 56.3 -> 57.2 / 58.4, d = 112 100.0 / 100.5 -> 106.2 / 106.4
//   odd multiples of 16 bytes, which agree less often: d = 56 causal 140 x 512 56.1 / 57.4 -> 57.2 / 57.8, 64 x 2048 290 / 282 -> 284 / 277: from
//             1024 rows on
// Not at 96 columns (d = 80, 64 x 2048 equal; causal 140 x 512 85.7 / 86.7 -> 90.3 / 91.5).
bool far_rows(const Problem& p) {
  const int loop = p.Nq < p.Nk ? p.Nq : p.Nk;
  if (p.d > 64 && loop < (p.causal ? 1024 : 512)) return false;
  for (const TensorMap* m : {&p.mq, &p.mk, &p.mv, &p.mo, &p.mdo}) {
    const long long bytes = m->row * 2;
    if (bytes % 128 != 0 && (bytes % 32 == 0 || loop < 1024)) return false;
  }
  return true;
}

template <typename T, int D, bool CAUSAL, bool DROP>
int launch_bwd_merged(const Problem& p, const void* Q, const void* K, const void* V, const void* O, const float* LSE,
                      const void* dO, void* dQ, void* dK, void* dV, float* Dws) {
  auto kernel = mha_bwd_merged_kernel<T, D, CAUSAL, DROP>;
  static std::atomic<uint64_t> ready[2] = {};
  bool far = false;
  if constexpr (DROP && D != 96) {
    far = far_rows(p);
    if (far) kernel = mha_bwd_merged_far_kernel<T, D, CAUSAL>;
  }
  constexpr int SMEM = BwdMergedCfg<D>::SMEM;
  const int attr = ensure_smem(kernel, SMEM, ready[far]);
  if (attr != SPARK_OK) return attr;
  const int BH = p.B * p.H, rows = BH * p.Nq;
  const Dropout dr = make_dropout(p.thr, p.seed, p.offset);
  float* LSE2ws = Dws + (size_t)rows;
  constexpr int RPB = 256 * 8 / lds_row<D>;  // rows per workgroup of the statistics kernel
  hipLaunchKernelGGL((mha_bwd_stats_kernel<T, D>), dim3((unsigned)((rows + RPB - 1) / RPB)), dim3(256), 0, p.st,
                     static_cast<const T*>(O), static_cast<const T*>(dO), LSE, Dws, LSE2ws, p.mo, p.mdo, p.H, p.Nq,
                     p.d, rows, DROP ? dr.keep_prob : 1.0f);
  if (!launch_ok("backward statistics kernel")) return SPARK_ERR_LAUNCH;
  const int nqt = (p.Nq + 127) / 128, nkt = (p.Nk + 127) / 128;
  const int paired = pair_tiles(CAUSAL, 2 * (int64_t)BH, nqt, dkdv_per_cu<D>);
  const int items = paired ? 2 * causal_items<true>(nqt) : nqt + nkt;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(BH * items)), dim3(256), SMEM, p.st, static_cast<const T*>(Q),
                     static_cast<const T*>(K), static_cast<const T*>(V), static_cast<const T*>(dO), Dws, LSE2ws,
                     static_cast<T*>(dQ), static_cast<T*>(dK), static_cast<T*>(dV), p.mq, p.mk, p.mv, p.mdo, p.mdq,
                     p.mdk, p.mdv, p.H, p.Nq, p.Nk, p.d, nqt, nkt, paired, p.scale, dr);
  return launch_ok("backward kernel (both sides)") ? SPARK_OK : SPARK_ERR_LAUNCH;
}

// Optional profiling marks between the kernels of a backward (spark_mha_bwd_marked).
bool mark(const Problem& p, void* const* ev, int i) {
  return !ev || hipEventRecord(static_cast<hipEvent_t>(ev[i]), p.st) == hipSuccess;
}

// One kernel per side.
template <typename T, int D, bool CAUSAL, bool DROP, bool FAR_ROWS>
int launch_bwd_sides(const Problem& p, const T* q, const T* k, const T* v, const T* o, const float* LSE, const T* dout,
                     T* dq, T* dk, T* dv, float* Dws, void* const* ev) {
  const int BH = p.B * p.H;
  const Dropout dr = make_dropout(p.thr, p.seed, p.offset);
  float* LSE2ws = Dws + (size_t)BH * p.Nq;  // second half of the workspace: LSE * log2(e)
  {  // dQ: one workgroup per tile of 128 queries (8-wave workgroups measured 3 % slower here).
     // Also writes D = rowsum(dO o O) and LSE * log2(e) for the dK/dV kernel.
    using C = BwdQCfg<D, CAUSAL, DROP>;
    auto kernel = mha_bwd_dq_kernel<T, D, CAUSAL, DROP>;
    if constexpr (FAR_ROWS) kernel = mha_bwd_dq_far_kernel<T, D, CAUSAL>;
    static std::atomic<uint64_t> ready{0};
    const int attr = ensure_smem(kernel, C::SMEM, ready);
    if (attr != SPARK_OK) return attr;
    const int nqt = (p.Nq + C::BM - 1) / C::BM;
    const int paired = pair_tiles(CAUSAL, BH, nqt, 2);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(BH * (paired ? causal_items<true>(nqt) : nqt))), dim3(256), C::SMEM, p.st,
                       q, k, v, o, dout, LSE, Dws, LSE2ws, dq, p.mq, p.mk, p.mv, p.mo,
                       p.mdo, p.mdq, p.H, p.Nq, p.Nk, p.d, nqt, paired, p.scale, p.scale * 1.4426950408889634f, dr);
    if (!launch_ok("dQ kernel") || !mark(p, ev, 1)) return SPARK_ERR_LAUNCH;
  }
  {  // dK, dV: one workgroup per tile of 128 keys, software-pipelined
    using C = BwdKvPipeCfg<D>;
    auto kernel = mha_bwd_dkdv_pipe_kernel<T, D, CAUSAL, DROP>;
    if constexpr (FAR_ROWS) kernel = mha_bwd_dkdv_pipe_far_kernel<T, D, CAUSAL>;
    static std::atomic<uint64_t> ready{0};
    const int attr = ensure_smem(kernel, C::SMEM, ready);
    if (attr != SPARK_OK) return attr;
    const int nkt = (p.Nk + C::BN - 1) / C::BN;
    const int paired = pair_tiles(CAUSAL, BH, nkt, dkdv_per_cu<D>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(BH * (paired ? causal_items<true>(nkt) : nkt))), dim3(256), C::SMEM, p.st,
                       q, k, v, dout, LSE2ws, Dws, dk, dv, p.mq, p.mk,
                       p.mv, p.mdo, p.mdk, p.mdv, p.H, p.Nq, p.Nk, p.d, nkt, paired, p.scale, dr);
    if (!launch_ok("dK/dV kernel") || !mark(p, ev, 2)) return SPARK_ERR_LAUNCH;
  }
  return SPARK_OK;
}

template <typename T, int D, bool CAUSAL, bool DROP>
int launch_bwd(const Problem& p, const void* Q, const void* K, const void* V, const void* O,
               const float* LSE, const void* dO, void* dQ, void* dK, void* dV, float* Dws,
               void* const* ev) {
  if (!mark(p, ev, 0)) return SPARK_ERR_LAUNCH;
  if (split_backward(p)) {  // one kernel: both later marks follow it
    const int rc = launch_bwd_split<T, lds_row<D>, CAUSAL, DROP>(p, Q, K, V, O, LSE, dO, dQ, dK, dV);
    if (rc != SPARK_OK) return rc;
    return mark(p, ev, 1) && mark(p, ev, 2) ? SPARK_OK : SPARK_ERR_LAUNCH;
  }
  if (merged_backward(p)) {
    const int rc = launch_bwd_merged<T, D, CAUSAL, DROP>(p, Q, K, V, O, LSE, dO, dQ, dK, dV, Dws);
    if (rc != SPARK_OK) return rc;
    return mark(p, ev, 1) && mark(p, ev, 2) ? SPARK_OK : SPARK_ERR_LAUNCH;
  }
  auto sides = launch_bwd_sides<T, D, CAUSAL, DROP, false>;
  if constexpr (DROP && D != 96) {
    if (far_rows(p)) sides = launch_bwd_sides<T, D, CAUSAL, DROP, true>;
  }
  return sides(p, static_cast<const T*>(Q), static_cast<const T*>(K), static_cast<const T*>(V), static_cast<const T*>(O),
               LSE, static_cast<const T*>(dO), static_cast<T*>(dQ), static_cast<T*>(dK), static_cast<T*>(dV), Dws, ev);
}

size_t workspace_bytes(int B, int H, int Nq) { return 2 * (size_t)B * H * Nq * sizeof(float); }
size_t workspace_bytes_stats(int B, int H, int Nq) { return workspace_bytes(B, H, Nq); }

// The paper's own backward (Sec. 3.3): prepare (D, LSE * log2(e), cleared fp32 dQ accumulator), one
// fused kernel that adds dQ contributions with atomics, conversion of the accumulator to dQ.
size_t atomic_dq_offset(int B, int H, int Nq) { return (workspace_bytes_stats(B, H, Nq) + 255) & ~(size_t)255; }

template <typename T, int D, bool CAUSAL>
int launch_bwd_atomic(const Problem& p, const void* Q, const void* K, const void* V, const void* O,
                      const float* LSE, const void* dO, void* dQ, void* dK, void* dV, void* workspace) {
  const int BH = p.B * p.H;
  const long long rows = (long long)BH * p.Nq;
  float* Dws = static_cast<float*>(workspace);
  float* LSE2ws = Dws + rows;
  float* dQacc = reinterpret_cast<float*>(static_cast<char*>(workspace) + atomic_dq_offset(p.B, p.H, p.Nq));
  hipLaunchKernelGGL(mha_bwd_prep_kernel<T>, dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, p.st,
                     static_cast<const T*>(O), static_cast<const T*>(dO), LSE, Dws, LSE2ws, dQacc, p.mo, p.mdo,
                     p.H, p.Nq, p.d, rows);
  if (hipGetLastError() != hipSuccess) return SPARK_ERR_LAUNCH;
  {
    using C = BwdAtomicCfg<D>;
    auto kernel = mha_bwd_fused_atomic_kernel<T, D, CAUSAL>;
    static std::atomic<uint64_t> ready{0};
    const int attr = ensure_smem(kernel, C::SMEM, ready);
    if (attr != SPARK_OK) return attr;
    const int nkt = (p.Nk + C::BN - 1) / C::BN;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(BH * causal_items<CAUSAL>(nkt))), dim3(256), C::SMEM, p.st,
                       static_cast<const T*>(Q), static_cast<const T*>(K), static_cast<const T*>(V),
                       static_cast<const T*>(dO), LSE2ws, Dws, dQacc, static_cast<T*>(dK), static_cast<T*>(dV),
                       p.mq, p.mk, p.mv, p.mdo, p.mdk, p.mdv, p.H, p.Nq, p.Nk, p.d, nkt, p.scale);
    if (hipGetLastError() != hipSuccess) return SPARK_ERR_LAUNCH;
  }
  const long long chunks = rows * (p.d >> 3);
  hipLaunchKernelGGL(mha_bwd_dq_convert_kernel<T>, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, p.st,
                     dQacc, static_cast<T*>(dQ), p.mdq, p.H, p.Nq, p.d, p.scale, chunks);
  return hipGetLastError() == hipSuccess ? SPARK_OK : SPARK_ERR_LAUNCH;
}

// Expand the (dtype, d, causal, dropout) runtime tuple into a template instantiation.  A threshold of 0 must not reach the
// kernels with dropout: what they add to a byte to decide it has no byte for it.
#define SPARK_DISPATCH_CD(FN, T, D, ...)                                                    \
  do {                                                                                      \
    if (p.causal) return p.thr ? FN<T, D, true, true>(__VA_ARGS__)                          \
                               : FN<T, D, true, false>(__VA_ARGS__);                        \
    return p.thr ? FN<T, D, false, true>(__VA_ARGS__) : FN<T, D, false, false>(__VA_ARGS__); \
  } while (0)
// The row width a kernel is built for: 64, 96 or 128.  From d = 72 to 96 the kernels of 96 columns leave out a quarter of
// the products and of the accumulators of the 128-column ones; rows in LDS keep 256 bytes in both, a power of two for the
// swizzle, and the kernels for small grids exist for 64 and 128 only.  Forward / dQ / dK/dV, us, 128 -> 96 columns:
//   d = 96 causal 64 x 4096 238/352/514 -> 209/296/454      88, 64 x 1024 over 4096 keys 113/167/258 -> 98/145/229
//   d = 80, 36 x 1333 32.5/44.9/48.2 -> 29.3/36.8/43.3      72, causal with dropout, 256 x 512 32.4/43.2/67.7 -> 30.3/40.4/62.6
#define SPARK_DISPATCH(FN, ...)                                              \
  do {                                                                       \
    if (p.dtype == SPARK_F16) {                                              \
      if (p.d <= 64) SPARK_DISPATCH_CD(FN, _Float16, 64, __VA_ARGS__);       \
      if (p.d <= 96) SPARK_DISPATCH_CD(FN, _Float16, 96, __VA_ARGS__);       \
      SPARK_DISPATCH_CD(FN, _Float16, 128, __VA_ARGS__);                     \
    }                                                                        \
    if (p.d <= 64) SPARK_DISPATCH_CD(FN, __bf16, 64, __VA_ARGS__);           \
    if (p.d <= 96) SPARK_DISPATCH_CD(FN, __bf16, 96, __VA_ARGS__);           \
    SPARK_DISPATCH_CD(FN, __bf16, 128, __VA_ARGS__);                         \
  } while (0)

// Shape, scale, dtype and dropout checks common to forward and backward; fills `p` with
// contiguous strides (the strided entry points overwrite them afterwards).
int make_problem(Problem* p, int B, int H, int Nq, int Nk, int d, float scale, int causal, int thr,
                 unsigned long long seed, unsigned offset, spark_dtype_t dtype, void* stream) {
  const int rc = check_common(B, H, Nq, Nk, d, scale, causal, (int)dtype);
  if (rc != SPARK_OK) return rc;
  if (thr < 0) return SPARK_ERR_SHAPE;
  p->B = B; p->H = H; p->Nq = Nq; p->Nk = Nk; p->d = d;
  p->scale = scale;
  p->causal = causal != 0;
  p->dtype = (int)dtype;
  p->thr = thr;
  p->seed = seed;
  p->offset = offset;
  p->mq = p->mo = p->mdo = p->mdq = contiguous(H, Nq, d);
  p->mk = p->mv = p->mdk = p->mdv = contiguous(H, Nk, d);
  p->st = static_cast<hipStream_t>(stream);
  p->fwd_ws = nullptr;
  return SPARK_OK;
}

int run_fwd(const Problem& p, const void* Q, const void* K, const void* V, void* O, float* LSE) {
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O) || !aligned16(LSE))
    return SPARK_ERR_ALIGN;
  SPARK_DISPATCH(launch_fwd, p, Q, K, V, O, LSE);
}

int run_bwd(const Problem& p, const void* Q, const void* K, const void* V, const void* O,
            const float* LSE, const void* dO, void* dQ, void* dK, void* dV, void* workspace,
            size_t ws_bytes, void* const* ev) {
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O) || !aligned16(LSE) ||
      !aligned16(dO) || !aligned16(dQ) || !aligned16(dK) || !aligned16(dV) || !aligned16(workspace))
    return SPARK_ERR_ALIGN;
  if (ws_bytes < workspace_bytes(p.B, p.H, p.Nq)) return SPARK_ERR_WORKSPACE;
  float* Dws = static_cast<float*>(workspace);
  SPARK_DISPATCH(launch_bwd, p, Q, K, V, O, LSE, dO, dQ, dK, dV, Dws, ev);
}

}  // namespace

extern "C" {

int spark_mha_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int H,
                  int N, int d, float scale, int causal, spark_dtype_t dtype, void* stream) {
  return spark_mha_cross_fwd(Q, K, V, O, LSE, B, H, N, N, d, scale, causal, dtype, stream);
}

int spark_mha_cross_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int B,
                        int H, int Nq, int Nk, int d, float scale, int causal,
                        spark_dtype_t dtype, void* stream) {
  return spark_mha_dropout_fwd(Q, K, V, O, LSE, B, H, Nq, Nk, d, scale, causal, 0.0f, 0, 0, dtype,
                               stream);
}

int spark_mha_dropout_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int B,
                          int H, int Nq, int Nk, int d, float scale, int causal, float p_drop,
                          unsigned long long seed, unsigned offset, spark_dtype_t dtype,
                          void* stream) {
  if (!Q || !K || !V || !O || !LSE) return SPARK_ERR_NULL;
  Problem p;
  const int rc = make_problem(&p, B, H, Nq, Nk, d, scale, causal, drop_threshold(p_drop), seed,
                              offset, dtype, stream);
  if (rc != SPARK_OK) return rc;
  return run_fwd(p, Q, K, V, O, LSE);
}

int spark_mha_strided_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE,
                          const spark_strides_t* sQ, const spark_strides_t* sK,
                          const spark_strides_t* sV, const spark_strides_t* sO, int B, int H, int Nq,
                          int Nk, int d, float scale, int causal, float p_drop,
                          unsigned long long seed, unsigned offset, spark_dtype_t dtype,
                          void* stream) {
  return spark_mha_workspace_fwd(Q, K, V, O, LSE, sQ, sK, sV, sO, nullptr, 0, B, H, Nq, Nk, d, scale, causal, p_drop,
                                 seed, offset, dtype, stream);
}

size_t spark_mha_fwd_workspace_bytes(int B, int H, int Nq, int Nk, int d, int causal, spark_dtype_t dtype) {
  Problem p;
  if (make_problem(&p, B, H, Nq, Nk, d, 1.0f, causal, 0, 0, 0, dtype, nullptr) != SPARK_OK) return 0;
  return fwd_workspace_bytes(p);
}

int spark_mha_workspace_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE,
                            const spark_strides_t* sQ, const spark_strides_t* sK,
                            const spark_strides_t* sV, const spark_strides_t* sO, void* workspace,
                            size_t workspace_bytes, int B, int H, int Nq, int Nk, int d, float scale,
                            int causal, float p_drop, unsigned long long seed, unsigned offset,
                            spark_dtype_t dtype, void* stream) {
  if (!Q || !K || !V || !O || !LSE) return SPARK_ERR_NULL;
  Problem p;
  int rc = make_problem(&p, B, H, Nq, Nk, d, scale, causal, drop_threshold(p_drop), seed, offset,
                        dtype, stream);
  if (rc != SPARK_OK) return rc;
  if ((rc = check_strides(sQ, Nq, d, &p.mq)) != SPARK_OK) return rc;
  if ((rc = check_strides(sK, Nk, d, &p.mk)) != SPARK_OK) return rc;
  if ((rc = check_strides(sV, Nk, d, &p.mv)) != SPARK_OK) return rc;
  if ((rc = check_strides(sO, Nq, d, &p.mo, true, B, H)) != SPARK_OK) return rc;
  if (workspace) {
    if (!aligned16(workspace)) return SPARK_ERR_ALIGN;
    const size_t need = fwd_workspace_bytes(p);
    if (workspace_bytes < need) return SPARK_ERR_WORKSPACE;
    if (need) p.fwd_ws = workspace;
  }
  return run_fwd(p, Q, K, V, O, LSE);
}

size_t spark_mha_cross_bwd_workspace_bytes(int B, int H, int Nq, int Nk, int d,
                                           spark_dtype_t dtype) {
  if (check_common(B, H, Nq, Nk, d, 1.0f, 0, (int)dtype) != SPARK_OK) return 0;
  return workspace_bytes(B, H, Nq);  // D and LSE*log2(e), fp32 [B,H,Nq] each
}

int spark_mha_bwd_grids(int B, int H, int Nq, int Nk, int d, int causal, float p_drop, spark_dtype_t dtype) {
  Problem p;
  const int rc = make_problem(&p, B, H, Nq, Nk, d, 1.0f, causal, drop_threshold(p_drop), 0, 0, dtype, nullptr);
  if (rc != SPARK_OK) return rc;
  return split_backward(p) || merged_backward(p) ? 1 : 2;
}

size_t spark_mha_bwd_workspace_bytes(int B, int H, int N, int d, spark_dtype_t dtype) {
  return spark_mha_cross_bwd_workspace_bytes(B, H, N, N, d, dtype);
}

int spark_mha_bwd(const void* Q, const void* K, const void* V, const void* O, const float* LSE,
                  const void* dO, void* dQ, void* dK, void* dV, void* workspace,
                  size_t workspace_bytes, int B, int H, int N, int d, float scale, int causal,
                  spark_dtype_t dtype, void* stream) {
  return spark_mha_cross_bwd(Q, K, V, O, LSE, dO, dQ, dK, dV, workspace, workspace_bytes, B, H, N, N,
                             d, scale, causal, dtype, stream);
}

int spark_mha_cross_bwd(const void* Q, const void* K, const void* V, const void* O,
                        const float* LSE, const void* dO, void* dQ, void* dK, void* dV,
                        void* workspace, size_t workspace_bytes, int B, int H, int Nq, int Nk,
                        int d, float scale, int causal, spark_dtype_t dtype, void* stream) {
  return spark_mha_dropout_bwd(Q, K, V, O, LSE, dO, dQ, dK, dV, workspace, workspace_bytes, B, H, Nq,
                               Nk, d, scale, causal, 0.0f, 0, 0, dtype, stream);
}

int spark_mha_dropout_bwd(const void* Q, const void* K, const void* V, const void* O,
                          const float* LSE, const void* dO, void* dQ, void* dK, void* dV,
                          void* workspace, size_t workspace_bytes, int B, int H, int Nq, int Nk,
                          int d, float scale, int causal, float p_drop, unsigned long long seed,
                          unsigned offset, spark_dtype_t dtype, void* stream) {
  if (!Q || !K || !V || !O || !LSE || !dO || !dQ || !dK || !dV || !workspace) return SPARK_ERR_NULL;
  Problem p;
  const int rc = make_problem(&p, B, H, Nq, Nk, d, scale, causal, drop_threshold(p_drop), seed,
                              offset, dtype, stream);
  if (rc != SPARK_OK) return rc;
  return run_bwd(p, Q, K, V, O, LSE, dO, dQ, dK, dV, workspace, workspace_bytes, nullptr);
}

int spark_mha_strided_bwd(const void* Q, const void* K, const void* V, const void* O,
                          const float* LSE, const void* dO, void* dQ, void* dK, void* dV,
                          const spark_strides_t* sQ, const spark_strides_t* sK,
                          const spark_strides_t* sV, const spark_strides_t* sO,
                          const spark_strides_t* sdO, const spark_strides_t* sdQ,
                          const spark_strides_t* sdK, const spark_strides_t* sdV, void* workspace,
                          size_t workspace_bytes, int B, int H, int Nq, int Nk, int d, float scale,
                          int causal, float p_drop, unsigned long long seed, unsigned offset,
                          spark_dtype_t dtype, void* stream) {
  if (!Q || !K || !V || !O || !LSE || !dO || !dQ || !dK || !dV || !workspace) return SPARK_ERR_NULL;
  Problem p;
  int rc = make_problem(&p, B, H, Nq, Nk, d, scale, causal, drop_threshold(p_drop), seed, offset,
                        dtype, stream);
  if (rc != SPARK_OK) return rc;
  if ((rc = check_strides(sQ, Nq, d, &p.mq)) != SPARK_OK) return rc;
  if ((rc = check_strides(sK, Nk, d, &p.mk)) != SPARK_OK) return rc;
  if ((rc = check_strides(sV, Nk, d, &p.mv)) != SPARK_OK) return rc;
  if ((rc = check_strides(sO, Nq, d, &p.mo)) != SPARK_OK) return rc;
  if ((rc = check_strides(sdO, Nq, d, &p.mdo)) != SPARK_OK) return rc;
  if ((rc = check_strides(sdQ, Nq, d, &p.mdq, true, B, H)) != SPARK_OK) return rc;
  if ((rc = check_strides(sdK, Nk, d, &p.mdk, true, B, H)) != SPARK_OK) return rc;
  if ((rc = check_strides(sdV, Nk, d, &p.mdv, true, B, H)) != SPARK_OK) return rc;
  return run_bwd(p, Q, K, V, O, LSE, dO, dQ, dK, dV, workspace, workspace_bytes, nullptr);
}

int spark_mha_bwd_marked(const void* Q, const void* K, const void* V, const void* O,
                         const float* LSE, const void* dO, void* dQ, void* dK, void* dV,
                         void* workspace, size_t workspace_bytes, int B, int H, int N, int d,
                         float scale, int causal, spark_dtype_t dtype, void* stream,
                         void* const events[3]) {
  if (!Q || !K || !V || !O || !LSE || !dO || !dQ || !dK || !dV || !workspace) return SPARK_ERR_NULL;
  if (!events || !events[0] || !events[1] || !events[2]) return SPARK_ERR_NULL;
  Problem p;
  const int rc = make_problem(&p, B, H, N, N, d, scale, causal, 0, 0, 0, dtype, stream);
  if (rc != SPARK_OK) return rc;
  return run_bwd(p, Q, K, V, O, LSE, dO, dQ, dK, dV, workspace, workspace_bytes, events);
}

size_t spark_mha_bwd_static_max_rows(void) { return SPARK_STATIC_SCRATCH_BYTES / (2 * sizeof(float)); }

int spark_mha_bwd_static(const void* Q, const void* K, const void* V, const void* O, const float* LSE,
                         const void* dO, void* dQ, void* dK, void* dV, int B, int H, int N, int d,
                         float scale, int causal, spark_dtype_t dtype, void* stream) {
  if (!Q || !K || !V || !O || !LSE || !dO || !dQ || !dK || !dV) return SPARK_ERR_NULL;
  Problem p;
  const int rc = make_problem(&p, B, H, N, N, d, scale, causal, 0, 0, 0, dtype, stream);
  if (rc != SPARK_OK) return rc;
  if (workspace_bytes(B, H, N) > SPARK_STATIC_SCRATCH_BYTES) return SPARK_ERR_WORKSPACE;
  void* ws = static_scratch_ptr();
  if (!ws) return SPARK_ERR_LAUNCH;
  return run_bwd(p, Q, K, V, O, LSE, dO, dQ, dK, dV, ws, SPARK_STATIC_SCRATCH_BYTES, nullptr);
}

size_t spark_mha_bwd_atomic_workspace_bytes(int B, int H, int Nq, int Nk, int d, spark_dtype_t dtype) {
  if (check_common(B, H, Nq, Nk, d, 1.0f, 0, (int)dtype) != SPARK_OK) return 0;
  return atomic_dq_offset(B, H, Nq) + (size_t)B * H * Nq * d * sizeof(float);
}

int spark_mha_bwd_atomic(const void* Q, const void* K, const void* V, const void* O, const float* LSE,
                         const void* dO, void* dQ, void* dK, void* dV, void* workspace,
                         size_t workspace_bytes, int B, int H, int Nq, int Nk, int d, float scale,
                         int causal, spark_dtype_t dtype, void* stream) {
  if (!Q || !K || !V || !O || !LSE || !dO || !dQ || !dK || !dV || !workspace) return SPARK_ERR_NULL;
  Problem p;
  const int rc = make_problem(&p, B, H, Nq, Nk, d, scale, causal, 0, 0, 0, dtype, stream);
  if (rc != SPARK_OK) return rc;
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O) || !aligned16(LSE) ||
      !aligned16(dO) || !aligned16(dQ) || !aligned16(dK) || !aligned16(dV) || !aligned16(workspace))
    return SPARK_ERR_ALIGN;
  // the two elementwise kernels are gridded over rows / 16 and over 8-element chunks / 256
  if (((int64_t)B * H * Nq + 15) / 16 >= (int64_t)1 << 31 ||
      ((int64_t)B * H * Nq * (d >> 3) + 255) / 256 >= (int64_t)1 << 31)
    return SPARK_ERR_SHAPE;
  if (workspace_bytes < spark_mha_bwd_atomic_workspace_bytes(B, H, Nq, Nk, d, dtype)) return SPARK_ERR_WORKSPACE;
#define SPARK_ATOMIC_CD(T, D)                                                                          \
  return p.causal ? launch_bwd_atomic<T, D, true>(p, Q, K, V, O, LSE, dO, dQ, dK, dV, workspace)       \
                  : launch_bwd_atomic<T, D, false>(p, Q, K, V, O, LSE, dO, dQ, dK, dV, workspace)
  if (p.dtype == SPARK_F16) {
    if (p.d <= 64) SPARK_ATOMIC_CD(_Float16, 64);
    SPARK_ATOMIC_CD(_Float16, 128);
  }
  if (p.d <= 64) SPARK_ATOMIC_CD(__bf16, 64);
  SPARK_ATOMIC_CD(__bf16, 128);
#undef SPARK_ATOMIC_CD
}

int spark_mha_dropout_bwd_marked(const void* Q, const void* K, const void* V, const void* O,
                                 const float* LSE, const void* dO, void* dQ, void* dK, void* dV,
                                 void* workspace, size_t workspace_bytes, int B, int H, int Nq, int Nk,
                                 int d, float scale, int causal, float p_drop, unsigned long long seed,
                                 unsigned offset, spark_dtype_t dtype, void* stream,
                                 void* const events[3]) {
  if (!Q || !K || !V || !O || !LSE || !dO || !dQ || !dK || !dV || !workspace) return SPARK_ERR_NULL;
  if (!events || !events[0] || !events[1] || !events[2]) return SPARK_ERR_NULL;
  Problem p;
  const int rc = make_problem(&p, B, H, Nq, Nk, d, scale, causal, drop_threshold(p_drop), seed,
                              offset, dtype, stream);
  if (rc != SPARK_OK) return rc;
  return run_bwd(p, Q, K, V, O, LSE, dO, dQ, dK, dV, workspace, workspace_bytes, events);
}

int spark_dropout_threshold(float p_drop) { return drop_threshold(p_drop); }

int spark_dropout_mask(unsigned char* M, int B, int H, int Nq, int Nk, float p_drop,
                       unsigned long long seed, unsigned offset, void* stream) {
  if (!M) return SPARK_ERR_NULL;
  if (B < 1 || H < 1 || Nq < 1 || Nk < 1) return SPARK_ERR_SHAPE;
  const int thr = drop_threshold(p_drop);
  if (thr < 0) return SPARK_ERR_SHAPE;
  const int qblocks = (Nq + 3) / 4, kblocks = (Nk + 3) / 4;
  const long long total = (long long)B * H * qblocks * kblocks;
  if (total >= ((long long)1 << 31) * 256) return SPARK_ERR_SHAPE;
  const unsigned grid = (unsigned)((total + 255) / 256);
  hipLaunchKernelGGL(dropout_mask_kernel, dim3(grid), dim3(256), 0, static_cast<hipStream_t>(stream),
                     M, Nq, Nk, qblocks, kblocks, total, make_dropout(thr, seed, offset));
  return hipGetLastError() == hipSuccess ? SPARK_OK : SPARK_ERR_LAUNCH;
}

int spark_layout_probe(float* out, spark_dtype_t dtype, void* stream) {
  if (!out) return SPARK_ERR_NULL;
  if (dtype != SPARK_F16 && dtype != SPARK_BF16) return SPARK_ERR_DTYPE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (dtype == SPARK_F16)
    hipLaunchKernelGGL(layout_probe_kernel<_Float16>, dim3(1), dim3(64), 16 * 64 * 2, st, out);
  else
    hipLaunchKernelGGL(layout_probe_kernel<__bf16>, dim3(1), dim3(64), 16 * 64 * 2, st, out);
  return hipGetLastError() == hipSuccess ? SPARK_OK : SPARK_ERR_LAUNCH;
}

const char* spark_status_str(int status) {
  switch (status) {
    case SPARK_OK: return "ok";
    case SPARK_ERR_NULL: return "a required pointer is NULL";
    case SPARK_ERR_SHAPE:
      return "unsupported shape, scale, dropout rate or stride (need B,H,N >= 1, d a multiple of 8 with "
             "8 <= d <= 128, finite scale > 0, Nq == Nk if causal, 0 <= p_drop < 0.998, row stride >= d, "
             "nonzero batch/head strides for outputs, sizes within the documented limits)";
    case SPARK_ERR_DTYPE: return "unsupported dtype (need SPARK_F16 or SPARK_BF16)";
    case SPARK_ERR_ALIGN: return "a pointer or stride is not 16-byte aligned";
    case SPARK_ERR_WORKSPACE:
      return "workspace smaller than spark_mha_bwd_workspace_bytes() or spark_mha_fwd_workspace_bytes(), or "
             "B*H*N above spark_mha_bwd_static_max_rows() for spark_mha_bwd_static";
    case SPARK_ERR_LAUNCH: return "the HIP runtime refused a kernel launch";
    default: return "unknown status";
  }
}

}  // extern "C"
