// Attention dropout for the fused kernels on gfx950: the keep/drop decisions are regenerated
// inside every kernel from a counter-based generator, so the forward and the two backward
// kernels see the same mask without storing it (paper Sec. 4.2: the backward repeats the
// forward's dropout; Sec. 4.1: rate 0.1 in every measurement).
//
// Definition of the mask (the library's own; the paper does not give one).  The decision for
// entry (head h, query i, key j) is one byte of the output of Philox4x32 with 10 rounds
// (Salmon, Moraes, Dror, Shaw, SC'11):
//   x = Philox(counter = (j / 4, i / 4, h, offset), key = (seed low word, seed high word))
//   u = byte (j mod 4) of x[i mod 4];   keep iff u >= thr;   survivors scaled by 256 / (256 - thr)
// One call therefore covers a block of 4 queries x 4 keys.  In the MFMA accumulator layout a
// lane holds, per 32 x 32 block, four strips of four consecutive rows of one column: four 1 x 4
// (or 4 x 1) pieces of four different calls.  Four lanes hold the complementary pieces of the same
// four calls, so each of them evaluates one call and they exchange the words (a 4 x 4
// transpose): one generator call per 16 entries, none wasted.
#pragma once
#include <stdint.h>

namespace spark {

struct Dropout {
  uint32_t key0, key1;  // seed, low and high word
  uint32_t offset;      // counter word 3: distinguishes calls that share a seed
  uint32_t thr;         // drop iff byte < thr (1..255 in the kernels below; a rate of 0 runs the kernels without dropout)
  uint32_t keep_add;    // 256 - thr in every byte, which holds none for 0: byte + (256 - thr) carries iff byte >= thr
  float keep_prob;      // (256 - thr) / 256
  float rescale;        // 256 / (256 - thr)
};
// The same without what a kernel can form from `thr`: an argument fewer to hold.
struct DropoutLean {
  uint32_t key0, key1, offset, thr;
  float keep_prob, rescale;
};

// Philox4x32-10, one round at a time so that a kernel can place the rounds between its MFMAs.
// The key schedule (key + round * Weyl constant) is uniform across the wave: scalar registers.
struct Philox {
  uint32_t c0, c1, c2, c3;
};
// The two exclusive ors of three words are one v_bitop3_b32 each (truth table 0x96): 4 vector
// instructions a round instead of 6.
static __device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0x96);
}
template <bool SPREAD = false>
static __device__ __forceinline__ void philox_round(Philox& s, uint32_t key0, uint32_t key1, int round) {
  const uint32_t k0 = key0 + (uint32_t)round * 0x9E3779B9u, k1 = key1 + (uint32_t)round * 0xBB67AE85u;
  uint64_t p0 = (uint64_t)0xD2511F53u * s.c0;
  uint64_t p1 = (uint64_t)0xCD9E8D57u * s.c2;
  // SPREAD (rounds spread over MFMA slots): kept whole, so that each product is one v_mad_u64_u32; the compiler
  // otherwise splits every second one into v_mul_lo_u32 and v_mul_hi_u32, quarter-rate instructions like it (48
  // per stage of the dK/dV loop instead of 32).  The first products are loop-invariant or uniform.
  if (SPREAD && round >= 1) asm("" : "+v"(p0));
  if (SPREAD && round >= 2) asm("" : "+v"(p1));
  // Head, offset and keys are uniform: in rounds 0 and 1 most of these words are scalar and the scalar unit joins
  // them.  v_bitop3_b32 takes one scalar operand only; the others would sit in vector registers for the
  // whole loop, and the causal wide forward at D = 128 spilled inside its masked loop (scratch 140 -> 108 bytes).
  const uint32_t h1 = (uint32_t)(p1 >> 32), h0 = (uint32_t)(p0 >> 32);
  const uint32_t n0 = round < 2 ? h1 ^ s.c1 ^ k0 : xor3(h1, s.c1, k0);
  const uint32_t n2 = round < 2 ? h0 ^ s.c3 ^ k1 : xor3(h0, s.c3, k1);
  s.c1 = (uint32_t)p1;
  s.c3 = (uint32_t)p0;
  s.c0 = n0;
  s.c2 = n2;
}
static __device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                     uint32_t k0, uint32_t k1, uint32_t (&out)[4]) {
  Philox s{c0, c1, c2, c3};
#pragma unroll
  for (int round = 0; round < 10; ++round) philox_round(s, k0, k1, round);
  out[0] = s.c0; out[1] = s.c1; out[2] = s.c2; out[3] = s.c3;
}

// How the 32 rows of a block, the products' columns, are spread over the lanes.  With dropout the four rows of a call swap words
// (exchange_words), which is cheap across lane bits 3 and 4 and dear inside a quad; but a kernel also loads its rows by 16 bytes
// a lane, and such a load takes up to three times as long where neighbouring lanes' addresses agree in bit 6 (ns for a load by
// a wave, eight waves on a CU, rows of 64 / 96 / 128 / 160 / 192 / 224 / 256 bytes in L2):
//             bits 0, 1 of a row are lane bits   exchange, instructions   row load
//   IN_ORDER  0, 1                               16                       15.4 /  9.2 / 27 / 13.0 / 14.1 / 14.0 / 27
//   NEAR      0, 4                               10                       15.5 / 14.5 / 27 / 14.3 / 14.1 / 15.1 / 27
//   FAR       3, 4                                8                       28.8 / 27.9 / 27 / 27.5 / 27.3 / 27.2 / 27
// FAR in the forward at 64 columns and in its workgroups of eight waves, which load one operand's rows for a long loop, and in the
// backward's 128-row tiles as far_rows decides; NEAR in mha_fwd_split_kernel, whose eight waves load the same rows (IN_ORDER where its
// causal form has 128 columns: 4 heads x 512 10.8 -> 10.6 us); IN_ORDER elsewhere.  (FAR in all of them, us, fp16: forward 4 x 512,
// d = 96 9.0 -> 9.6, now 8.8; 100 x 384, d = 112 17.9 -> 18.2, now 17.2; backward causal 140 x 512, d = 48 55.0 -> 57.2, d = 96
// 87.9 -> 92.3; 4 x 512, d = 48 8.2 -> 8.9.  IN_ORDER with eight waves: causal 10 x 7168, d = 128 207.3 -> 210.9.)
enum Lanes { IN_ORDER, NEAR, FAR };
template <Lanes M> static __device__ __forceinline__ int column_row(int lane) {
  return M == NEAR  ? (lane & 14) << 1 | ((lane >> 3) & 2) | (lane & 1)
         : M == FAR ? (lane & 7) << 2 | ((lane >> 3) & 3)
                    : lane & 31;
}
template <Lanes M> static __device__ __forceinline__ int call_strip(int lane) { return column_row<M>(lane) & 3; }

// 4 x 4 transpose over the four lanes of a call: on return x[a] holds what the lane of strip a had in x[w], w = this lane's
// strip.  Two butterfly steps, each exchanging the two words that differ in that bit of w: across lane bit 3 a DPP move
// into half of the lanes for each word (row_ror:8, banks of four lanes), across bit 4 one swap for two words; inside a quad,
// where a move cannot be held to some of the lanes, a move and three selects for two words.
template <Lanes M, int B> static __device__ __forceinline__ void exchange_pair(uint32_t& lo, uint32_t& hi, int lane) {
  const uint32_t a = lo, b = hi;
  if (M == IN_ORDER || (M == NEAR && B == 0)) {
    const bool upper = lane & (B == 0 ? 1 : 2);
    const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)(upper ? a : b), B == 0 ? 0xB1 : 0x4E, 0xF, 0xF, true);
    lo = upper ? got : a;
    hi = upper ? b : got;
  } else if (B == 0) {
    lo = (uint32_t)__builtin_amdgcn_update_dpp((int)a, (int)b, 0x128, 0xF, 0xC, false);
    hi = (uint32_t)__builtin_amdgcn_update_dpp((int)b, (int)a, 0x128, 0xF, 0x3, false);
  } else {
    const auto s = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    lo = s[0];
    hi = s[1];
  }
}
template <Lanes M> static __device__ __forceinline__ void exchange_bit0(uint32_t (&x)[4], int lane) {
  exchange_pair<M, 0>(x[0], x[1], lane);
  exchange_pair<M, 0>(x[2], x[3], lane);
}
template <Lanes M> static __device__ __forceinline__ void exchange_bit1(uint32_t (&x)[4], int lane) {
  exchange_pair<M, 1>(x[0], x[2], lane);
  exchange_pair<M, 1>(x[1], x[3], lane);
}
template <Lanes M> static __device__ __forceinline__ void exchange_words(uint32_t (&x)[4], int lane) {
  exchange_bit0<M>(x, lane);
  exchange_bit1<M>(x, lane);
}

// Decisions of four entries at once: v_lerp_u8 halves the nine-bit sums byte + (256 - thr), so bit 7 of byte b is the
// carry, set iff entry b is kept.  v_perm_b32 copies bits 15 and 31 of its sources into whole bytes; the word shifted up by one
// byte brings the others there.  A compare and a select for each entry are eight instructions for four; in pairs it is six, by
// strips seven, whose last four (v_and_b32 of a sign-extended byte) sit where the entries are used (us, forward, d = 64 256
// heads x 2048 403 -> 386, causal d = 128 64 x 4096 352 -> 339; dK/dV, d = 64, the same 640 -> 629).  In the dQ kernel, whose
// entries choose between two values, a compare and a select stay the shorter form.  mha_fwd_split_kernel, too, compares and selects
// each entry (masks have not been measured there), and so do the dK/dV kernels that were faster so (COMPARE in each).
static __device__ __forceinline__ uint32_t keep_flags(uint32_t bytes, const Dropout& dr) {
  return __builtin_amdgcn_lerp(bytes, dr.keep_add, 0);
}
// ones or zeros for 16-bit values in pairs: entries 0, 1 of the strip, and 2, 3
static __device__ __forceinline__ void keep_pairs(uint32_t flags, uint32_t (&mask)[2]) {
  mask[0] = __builtin_amdgcn_perm(flags, flags << 8, 0x0A0A0808u);
  mask[1] = __builtin_amdgcn_perm(flags, flags << 8, 0x0B0B0909u);
}
// ones or zeros in byte b for entry b of the strip; entry b's extended to 32 bits (in the instruction that uses it)
static __device__ __forceinline__ uint32_t keep_strip(uint32_t bytes, const Dropout& dr) {
  const uint32_t flags = keep_flags(bytes, dr);
  return __builtin_amdgcn_perm(flags, flags << 8, 0x0B090A08u);
}
static __device__ __forceinline__ uint32_t keep_mask(uint32_t strip, int b) {
  return (uint32_t)(int32_t)(int8_t)(strip >> (8 * b));
}
static __device__ __forceinline__ float keep_float(uint32_t mask, float x) {
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) & mask);
}

// Lane = query column (S^T layouts of the forward and dQ kernels).  The lane's query is
// `qrow` (row column_row<M>(lane) of its block) and it holds keys kblk + 8a + 4g + b of the 32-key block
// starting at kblk (a multiple of 32), g = lane / 32.  kb[a] receives the four decision bytes of
// strip a: byte b belongs to accumulator register 4a + b.
// In three parts (counter, ten rounds of philox_round, exchange), see keep_key_lane_begin.
template <Lanes M>
static __device__ __forceinline__ Philox keep_query_lane_begin(const Dropout& dr, int head, int qrow, int kblk,
                                                               int lane) {
  const int w = call_strip<M>(lane), g = lane >> 5;  // this lane evaluates the call of strip a = w
  return Philox{(uint32_t)((kblk >> 2) + 2 * w + g), (uint32_t)(qrow >> 2), (uint32_t)head, dr.offset};
}
template <Lanes M>
static __device__ __forceinline__ void keep_query_lane_finish(const Philox& s, int lane, uint32_t (&kb)[4]) {
  // strip a needs word (query mod 4) = w of the call that the lane of strip a evaluated
  kb[0] = s.c0; kb[1] = s.c1; kb[2] = s.c2; kb[3] = s.c3;
  exchange_words<M>(kb, lane);
}
template <Lanes M>
static __device__ __forceinline__ void keep_bytes_query_lane(const Dropout& dr, int head, int qrow,
                                                             int kblk, int lane, uint32_t (&kb)[4]) {
  Philox s = keep_query_lane_begin<M>(dr, head, qrow, kblk, lane);
#pragma unroll
  for (int round = 0; round < 10; ++round) philox_round(s, dr.key0, dr.key1, round);
  keep_query_lane_finish<M>(s, lane, kb);
}

// Lane = key column (S layouts of the dK/dV kernel).  The lane's key is `krow`
// (row column_row<M>(lane) of its block) and it holds queries qblk + 8a + 4g + b of the 32-query block
// starting at qblk (a multiple of 32).  kb[a] as above: byte b belongs to register 4a + b.
// In three parts (counter, ten rounds of philox_round, exchange) so that the kernel can spread
// the rounds over its MFMA slots; keep_bytes_key_lane runs them back to back.
template <Lanes M>
static __device__ __forceinline__ Philox keep_key_lane_begin(const Dropout& dr, int head, int krow, int qblk,
                                                             int lane) {
  const int w = call_strip<M>(lane), g = lane >> 5;  // this lane evaluates the call of strip a = w
  return Philox{(uint32_t)(krow >> 2), (uint32_t)((qblk >> 2) + 2 * w + g), (uint32_t)head, dr.offset};
}
template <Lanes M>
static __device__ __forceinline__ void keep_key_lane_finish(const Philox& s, int lane, uint32_t (&kb)[4]);
template <Lanes M>
static __device__ __forceinline__ void keep_bytes_key_lane(const Dropout& dr, int head, int krow,
                                                           int qblk, int lane, uint32_t (&kb)[4]) {
  Philox s = keep_key_lane_begin<M>(dr, head, krow, qblk, lane);
#pragma unroll
  for (int round = 0; round < 10; ++round) philox_round(s, dr.key0, dr.key1, round);
  keep_key_lane_finish<M>(s, lane, kb);
}
template <Lanes M>
static __device__ __forceinline__ void keep_key_lane_finish(const Philox& s, int lane, uint32_t (&kb)[4]) {
  // byte k of the call's four words (queries) belongs to the lane with key mod 4 = k: 4 x 4 byte transpose
  // inside the lane (8 byte permutes), then word k of strip a's call to lane k
  const uint32_t a01 = __builtin_amdgcn_perm(s.c1, s.c0, 0x05010400u);  // c0[0] c1[0] c0[1] c1[1]
  const uint32_t b01 = __builtin_amdgcn_perm(s.c1, s.c0, 0x07030602u);  // c0[2] c1[2] c0[3] c1[3]
  const uint32_t a23 = __builtin_amdgcn_perm(s.c3, s.c2, 0x05010400u);
  const uint32_t b23 = __builtin_amdgcn_perm(s.c3, s.c2, 0x07030602u);
  kb[0] = __builtin_amdgcn_perm(a23, a01, 0x05040100u);
  kb[1] = __builtin_amdgcn_perm(a23, a01, 0x07060302u);
  kb[2] = __builtin_amdgcn_perm(b23, b01, 0x05040100u);
  kb[3] = __builtin_amdgcn_perm(b23, b01, 0x07060302u);
  exchange_words<M>(kb, lane);
}

// decision for accumulator register r (0..15) from the bytes of its strip
static __device__ __forceinline__ bool keep_reg(const uint32_t (&kb)[4], int r, uint32_t thr) {
  return ((kb[r >> 2] >> (8 * (r & 3))) & 0xFFu) >= thr;
}

// The keep mask itself, one byte per entry (1 = keep), [B*H][Nq][Nk]: one thread per 4 x 4 block.
__global__ void dropout_mask_kernel(unsigned char* __restrict__ M, int Nq, int Nk, int qblocks,
                                    int kblocks, long long total_blocks, Dropout dr) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total_blocks) return;
  const int jb = (int)(t % kblocks);
  const long long rest = t / kblocks;
  const int ib = (int)(rest % qblocks);
  const int h = (int)(rest / qblocks);
  uint32_t x[4];
  philox4x32_10((uint32_t)jb, (uint32_t)ib, (uint32_t)h, dr.offset, dr.key0, dr.key1, x);
  for (int r = 0; r < 4; ++r) {
    const int i = 4 * ib + r;
    if (i >= Nq) break;
    for (int c = 0; c < 4; ++c) {
      const int j = 4 * jb + c;
      if (j >= Nk) break;
      M[((size_t)h * Nq + i) * Nk + j] = ((x[r] >> (8 * c)) & 0xFFu) >= dr.thr ? 1 : 0;
    }
  }
}

}  // namespace spark
