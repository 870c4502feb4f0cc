// rlx_mfma.hpp -- the generator step X <- A X mod m on the int8 matrix cores
// of gfx950 (v_mfma_i32_32x32x32_i8), for a multiplier A that is the same for
// the whole launch.
//
// The product by a constant is a dense contraction (paper, section 2.1: the
// 576 x 576-bit multiply is the larger part of the generator's time).  With
// X = sum_i x_i 256^i (72 bytes x_i) and C_i = A 256^i mod m,
//
//   A X = sum_i x_i C_i  (mod m),
//
// a [72 x 72] matrix of byte digits of the C_i applied to the byte vector of
// X.  The matrix cores multiply signed bytes exactly into 32-bit sums, so:
//
//  * each byte of X enters as the signed digit d_i = x_i - 128 (the byte with
//    its top bit flipped);
//  * each C_i enters as its balanced base-256 digits (in [-128, 127], up to
//    76 of them), and the constant K = 128 sum_i C_i (the exact integer, not
//    reduced) as one more column multiplied by a constant input byte 1, so
//    that sum_i d_i C_i + K = sum_i x_i C_i exactly: a non-negative integer
//    below 72 * 255 * 2^576 < 2^591;
//  * output row r of the product is the digit sum S_r of weight 256^r; every
//    |S_r| < 2^21, so the 32-bit sums are exact, and four rows make the
//    signed 64-bit sum W_w of 32-bit word w (w < 19);
//  * a signed carry chain over W_0..W_18 gives the 19 words of
//    sum_i x_i C_i: 18 words of X' and the word h above 2^576 (h < 2^15),
//    which is folded back with 2^576 = 2^240 - 1 (mod m) as in step()
//    (section 2.2), ending in the canonical residue.
//
// One wave holds 64 independent states (one per lane).  The contraction runs
// as 18 MFMAs of 32 x 32 x 32: three tiles of 32 output rows (73 used) by
// three steps of 32 input bytes (72 used plus the constant) by two tiles of
// 32 states.  The matrix core pairs byte j of lane l's A operand with byte j
// of lane l's B operand for every (l div 32, j), and returns in lane l, value
// 4q + u of a tile, output row 8q + 4 (l div 32) + u of state column l mod 32.
// Each lane's state is split in halves: E = words 0..8 and F = words 9..17.
// In every lane the halves of the inputs are exchanged with the lane 32 away
// (v_permlane32_swap), so that one register file holds, in lanes 0..31, the
// E half of states 0..31 and, in lanes 32..63, their F half (the B operand of
// state tile 0), and the other one the same for states 32..63 (tile 1); the
// A operand's byte (l div 32, j) of each K step is the column of the input
// byte that sits there.  On the output side the halves are exchanged back:
// lanes 0..31 of tile 0 hold the even words of states 0..31, lanes 32..63
// their odd words, and the same for tile 1, so one exchange per word pair
// gives every lane all 19 words of its own state.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rlx_arith.hpp"

namespace rlx {

typedef int mf_v4i __attribute__((ext_vector_type(4)));
typedef int mf_v16i __attribute__((ext_vector_type(16)));

constexpr int MF_FRAGS = 9;         // A operands: 3 output-row tiles x 3 input steps
constexpr int MF_BYTES = 72;        // input bytes of X
constexpr int MF_ROWS = 96;         // output rows (balanced digits) kept per column
constexpr int MF_COLS = MF_BYTES + 1;  // the 72 C_i and K
// words of one luxury level's table: for each g < RLX_FOLD_G (multiplier
// A^(2^g)), MF_FRAGS fragments of 64 lanes x 4 words
constexpr size_t MF_FRAG_WORDS = (size_t)64 * 4;
constexpr size_t MF_LEVEL_WORDS = (size_t)MF_FRAGS * MF_FRAG_WORDS;

// Input column of A-operand byte j of lane half h in input step ks: the byte
// of X that the B operand holds there (0..71), MF_BYTES for K (the constant
// input byte 1), or -1 for a zero column.  Half h = 0 holds E = words 0..8,
// h = 1 holds F = words 9..17, four words per step: word e = 4 ks + j / 4 of
// the half; e = 9 is the register holding the constant 1 (in both halves;
// only h = 0 carries K), e = 10, 11 pad.
RLX_HD constexpr int mf_input_column(int h, int ks, int j) {
  return (4 * ks + j / 4) < 9 ? 4 * (4 * ks + j / 4 + 9 * h) + j % 4
         : ((4 * ks + j / 4) == 9 && j % 4 == 0 && h == 0) ? MF_BYTES
                                                           : -1;
}

// Balanced base-256 digits of the non-negative number in words w[0..n): the
// digits b_r in [-128, 127] with sum_r b_r 256^r equal to it; writes MF_ROWS
// digits (the number must be below 128 * 256^(MF_ROWS - 1)).
template <int N>
RLX_HD void balanced_digits(const uint32_t (&w)[N], int8_t (&d)[MF_ROWS]) {
  int carry = 0;
  for (int r = 0; r < MF_ROWS; ++r) {
    const int byte = (r / 4 < N) ? (int)((w[r / 4] >> (8 * (r % 4))) & 0xFFu) : 0;
    const int v = byte + carry;
    carry = v >= 128;
    d[r] = (int8_t)(v - 256 * carry);
  }
}

// Opaque 32-bit constant: keeps the compiler from turning multiply-adds by
// it into shifts and sign extensions (a multiply-add is one instruction).
__device__ __forceinline__ uint32_t mf_opaque(uint32_t v) {
  asm volatile("" : "+s"(v));
  return v;
}

// Exchange register a of lanes 32..63 with register b of lanes 0..31.
__device__ __forceinline__ void mf_swap(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

// LDS writes of a wave become visible to the whole wave.
__device__ __forceinline__ void mf_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef unsigned mf_v2u __attribute__((ext_vector_type(2)));

// The 64-bit value with low word lo and high word hi (a register pair).
__device__ __forceinline__ int64_t mf_pair(uint32_t lo, uint32_t hi) {
  return __builtin_bit_cast(int64_t, mf_v2u{lo, hi});
}

// Signed 64-bit sum of output rows 4q .. 4q + 3 of a tile (weights 2^0,
// 2^8, 2^16, 2^24), as four multiply-adds (k1 = 1, the first one sign-
// extends).
__device__ __forceinline__ int64_t mf_word(const mf_v16i& s, int q, int32_t k1, int32_t k8, int32_t k16,
                                           int32_t k24) {
  int64_t w = (int64_t)s[4 * q] * k1;
  w = (int64_t)s[4 * q + 1] * k8 + w;
  w = (int64_t)s[4 * q + 2] * k16 + w;
  w = (int64_t)s[4 * q + 3] * k24 + w;
  return w;
}

// Copy a step's A operands (MF_FRAGS x 64 lanes x 16 bytes) from global
// memory into the block's LDS array `dst`; all `nthreads` threads of the
// block call it, then synchronise before the first step.
__device__ __forceinline__ void mf_stage_operands(mf_v4i* __restrict__ dst, const uint32_t* __restrict__ src,
                                                  uint32_t tid, uint32_t nthreads) {
  const mf_v4i* s = reinterpret_cast<const mf_v4i*>(src);
  for (uint32_t k = tid; k < (uint32_t)MF_FRAGS * 64; k += nthreads) dst[k] = s[k];
}

// Operand fetch from an array af[64 f + lane] (LDS, or any memory).
struct MfFromArray {
  const mf_v4i* __restrict__ af;
  uint32_t lane;
  __device__ __forceinline__ mf_v4i operator()(int f) const { return af[64 * f + lane]; }
};

// Operand fetch from global memory through a buffer resource: the
// wave-uniform table address lives in scalar registers and each fetch is one
// buffer load at this lane's 32-bit offset (no 64-bit address per lane).
// dword 3 of the resource is the raw-buffer format word of gfx9 parts.
struct MfFromBuffer {
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t off;  // 16 * lane
  __device__ __forceinline__ MfFromBuffer(const uint32_t* table, uint32_t lane)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(table), (short)0,
                                               (int)(MF_LEVEL_WORDS * sizeof(uint32_t)), 0x00020000)),
        off(16u * lane) {}
  __device__ __forceinline__ mf_v4i operator()(int f) const {
    return __builtin_bit_cast(mf_v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 1024 * f, 0));
  }
};

// X <- A X mod m with the A operands of the wave's multiplier delivered by
// `fetch(3 mt + ks)` (output-row tile mt, input step ks: this lane's 16
// bytes; read just before its two MFMAs, from LDS or global memory).  Must
// run with all 64 lanes of the wave active.  Returns the canonical residue;
// `force_general` sends the fold through its general branch.
template <class Fetch>
__device__ __forceinline__ void mfma_step(uint32_t (&x)[NW], const Fetch& fetch, bool force_general) {
  // signed input digits, halves exchanged across the two lane halves
  uint32_t a[9], b[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    a[k] = x[k] ^ 0x80808080u;
    b[k] = x[9 + k] ^ 0x80808080u;
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) mf_swap(a[k], b[k]);
  const mf_v4i b0[3] = {mf_v4i{(int)a[0], (int)a[1], (int)a[2], (int)a[3]},
                        mf_v4i{(int)a[4], (int)a[5], (int)a[6], (int)a[7]}, mf_v4i{(int)a[8], 1, 0, 0}};
  const mf_v4i b1[3] = {mf_v4i{(int)b[0], (int)b[1], (int)b[2], (int)b[3]},
                        mf_v4i{(int)b[4], (int)b[5], (int)b[6], (int)b[7]}, mf_v4i{(int)b[8], 1, 0, 0}};
  const int32_t k1 = (int32_t)mf_opaque(1u), k8 = (int32_t)mf_opaque(256u);
  const int32_t k16 = (int32_t)mf_opaque(65536u), k24 = (int32_t)mf_opaque(1u << 24);
  const mf_v16i zero = {};
  int32_t c = 0;      // signed carry of the chain
  uint32_t h = 0;     // word 18
#pragma unroll
  for (int mt = 0; mt < 3; ++mt) {
    const mf_v4i f0 = fetch(3 * mt), f1 = fetch(3 * mt + 1), f2 = fetch(3 * mt + 2);
    mf_v16i s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f0, b0[0], zero, 0, 0, 0);
    mf_v16i s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f0, b1[0], zero, 0, 0, 0);
    s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f1, b0[1], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f1, b1[1], s1, 0, 0, 0);
    s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f2, b0[2], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f2, b1[2], s1, 0, 0, 0);
    // rows 64 + 8q + ... of the last tile are zero from q = 2 on (the
    // digits end at row 75)
    const int nq = mt < 2 ? 4 : 2;
#pragma unroll
    for (int q = 0; q < nq; ++q) {
      const int64_t w0 = mf_word(s0, q, k1, k8, k16, k24);
      const int64_t w1 = mf_word(s1, q, k1, k8, k16, k24);
      uint32_t lo0 = (uint32_t)w0, hi0 = (uint32_t)((uint64_t)w0 >> 32);
      uint32_t lo1 = (uint32_t)w1, hi1 = (uint32_t)((uint64_t)w1 >> 32);
      mf_swap(lo0, lo1);
      mf_swap(hi0, hi1);
      // this lane's state: word 8 mt + 2 q in (lo0, hi0), the next in (lo1, hi1)
      const int e = 8 * mt + 2 * q;
      const int64_t we = mf_pair(lo0, hi0);
      const int64_t te = (int64_t)c * k1 + we;
      c = (int32_t)((uint64_t)te >> 32);
      if (e < NW) {
        x[e] = (uint32_t)te;
      } else {
        h = (uint32_t)te;
      }
      if (e + 1 < NW) {
        const int64_t wo = mf_pair(lo1, hi1);
        const int64_t to = (int64_t)c * k1 + wo;
        c = (int32_t)((uint64_t)to >> 32);
        x[e + 1] = (uint32_t)to;
      }
    }
  }
  // fold h (< 2^15) with 2^576 = 2^240 - 1: x - h at words 0-1, + (h << 16)
  // at words 7-9 (as in step())
  const uint32_t w0 = x[0], w1 = x[1], w7 = x[7], w8 = x[8], w9 = x[9];
  uint32_t br = 0;
  x[0] = subb(w0, h, br);
  x[1] = subb(w1, 0u, br);
  uint32_t cy = 0;
  x[7] = addc(w7, h << 16, cy);
  x[8] = addc(w8, h >> 16, cy);
  x[9] = addc(w9, 0u, cy);
  const bool rare = (br | cy) != 0 || x[17] == 0xFFFFFFFFu || force_general;
  if (rare) {
    x[0] = w0; x[1] = w1; x[7] = w7; x[8] = w8; x[9] = w9;
    fold_word_general(x, h);
  }
}

// ---------------------------------------------------------------------------
// the step with contiguous output halves
//
// The same product with the output digits placed differently: A row
// 32 mt + 8 q + 4 h + u is digit u of word 4 mt + q of the low half for h = 0
// (words 0..8) and of the high half for h = 1 (words 9..18), so lanes 0..31
// of a tile receive the low words of its states and lanes 32..63 the high
// ones.  Each lane then carries through nine words of two states on its own,
// and one exchange per word pair gives every lane its state: 10 exchanges and
// 20 short chain links against 20 and 19 (v_permlane32_swap takes 8 cycles,
// a link 16 with one multiply-add, 20 with five).  The carry into word 9 and
// word 18 are joined after the exchange.  About 560 vector cycles per wave
// against 720.
constexpr int MF_SPLIT_STEPS = 17;  // step sizes 2^g with operands of this form: up to 65 536 lanes per record

// Digit row of row `row` of output tile mt in this placement, or -1.
RLX_HD constexpr int mf_split_row(int mt, int row) {
  return ((row >> 2) & 1) == 0 ? (4 * mt + (row >> 3) < 9 ? 4 * (4 * mt + (row >> 3)) + (row & 3) : -1)
                               : (4 * mt + (row >> 3) < 10 ? 4 * (9 + 4 * mt + (row >> 3)) + (row & 3) : -1);
}

// Next word of a signed carry chain over output rows: rows 4q .. 4q + 3 of a
// tile (weights 2^0, 2^8, 2^16, 2^24) plus the carry c so far; returns the low
// 32 bits and leaves the carry in c.  With |S| < 2^21, lo = S_0 + S_1 2^8 + c
// and hi = S_2 + S_3 2^8 are below 2^30 in magnitude: two 32-bit shift-adds,
// an add, and one multiply-add by an opaque 2^16.
__device__ __forceinline__ uint32_t mf_chain(const mf_v16i& s, int q, int32_t k16, int32_t& c) {
  const int32_t lo = (int32_t)((uint32_t)s[4 * q] + ((uint32_t)s[4 * q + 1] << 8)) + c;
  const int32_t hi = (int32_t)((uint32_t)s[4 * q + 2] + ((uint32_t)s[4 * q + 3] << 8));
  const int64_t w = (int64_t)hi * k16 + (int64_t)lo;
  c = (int32_t)((uint64_t)w >> 32);
  return (uint32_t)w;
}

// x + the pending carries of mfma_step_split, exact and canonical: p2, p9 and
// p11 (-1, 0 or 1) at words 2, 9 and 11, and h2 (0 or -1, the upper half of a
// negative word 18) with the weight of word 19's share of the fold.
__device__ __forceinline__ void mf_settle(uint32_t (&x)[NW], int32_t p2, int32_t p9, int32_t p11, int32_t h2) {
  int64_t acc = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    int64_t add = 0;
    if (k == 1) add = -(int64_t)h2;
    if (k == 2) add = p2;
    if (k == 8) add = (int64_t)h2 * 65536;
    if (k == 9) add = p9;
    if (k == 11) add = p11;
    acc += (int64_t)x[k] + add;
    x[k] = (uint32_t)acc;
    acc >>= 32;
  }
  // x + top 2^576 = x + top (2^240 - 1), top in {-1, 0, 1}; x is then so far
  // from the other end that nothing passes 2^576 or 0 again
  const int64_t top = acc;
  acc = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    const int64_t add = k == 0 ? -top : k == 7 ? top * 65536 : 0;
    acc += (int64_t)x[k] + add;
    x[k] = (uint32_t)acc;
    acc >>= 32;
  }
  canonicalize(x);
}

// X <- A X mod m with operands in the split placement: fetch0 for the states
// of lanes 0..31, fetch1 for lanes 32..63 (ONE: fetch0 for both).  Must run
// with all 64 lanes of the wave active; returns the canonical residue;
// `force_general` sends the end of it through its general branch.  With two
// multipliers a tile's MFMAs of the one are issued before the other's operands
// are read: 12 operand registers at a time, so that the levels kernels fit 128
// VGPRs (both at once: 142, or 64 bytes of spills).
template <bool ONE, int CROSS, class Fetch0, class Fetch1>
__device__ __forceinline__ void mfma_step_split(uint32_t (&x)[NW], const Fetch0& fetch0, const Fetch1& fetch1,
                                                bool force_general) {
  uint32_t a[9], b[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    a[k] = x[k] ^ 0x80808080u;
    b[k] = x[9 + k] ^ 0x80808080u;
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) mf_swap(a[k], b[k]);
  const mf_v4i b0[3] = {mf_v4i{(int)a[0], (int)a[1], (int)a[2], (int)a[3]},
                        mf_v4i{(int)a[4], (int)a[5], (int)a[6], (int)a[7]}, mf_v4i{(int)a[8], 1, 0, 0}};
  const mf_v4i b1[3] = {mf_v4i{(int)b[0], (int)b[1], (int)b[2], (int)b[3]},
                        mf_v4i{(int)b[4], (int)b[5], (int)b[6], (int)b[7]}, mf_v4i{(int)b[8], 1, 0, 0}};
  const int32_t k16 = (int32_t)mf_opaque(65536u);
  const mf_v16i zero = {};
  int32_t c0 = 0, c1 = 0;  // carries of the two states' chains
  uint32_t t0 = 0, t1 = 0;
#pragma unroll
  for (int mt = 0; mt < 3; ++mt) {
    mf_v16i s0, s1;
    if constexpr (ONE) {
      const mf_v4i f0 = fetch0(3 * mt), f1 = fetch0(3 * mt + 1), f2 = fetch0(3 * mt + 2);
      s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f0, b0[0], zero, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f0, b1[0], zero, 0, 0, 0);
      s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f1, b0[1], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f1, b1[1], s1, 0, 0, 0);
      s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f2, b0[2], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f2, b1[2], s1, 0, 0, 0);
    } else {
      __builtin_amdgcn_sched_barrier(0);
      const mf_v4i f0 = fetch0(3 * mt), f1 = fetch0(3 * mt + 1), f2 = fetch0(3 * mt + 2);
      s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f0, b0[0], zero, 0, 0, 0);
      s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f1, b0[1], s0, 0, 0, 0);
      s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f2, b0[2], s0, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      const mf_v4i g0 = fetch1(3 * mt), g1 = fetch1(3 * mt + 1), g2 = fetch1(3 * mt + 2);
      s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(g0, b1[0], zero, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(g1, b1[1], s1, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(g2, b1[2], s1, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < (mt < 2 ? 4 : 2); ++q) {
      const int j = 4 * mt + q;
      uint32_t w0 = mf_chain(s0, q, k16, c0), w1 = mf_chain(s1, q, k16, c1);
      mf_swap(w0, w1);
      if (j < 9) {
        x[j] = w0;
        x[9 + j] = w1;
      } else {
        t0 = w0;  // the carry out of the low half
        t1 = w1;  // word 18
      }
    }
    if (mt == 0) __builtin_amdgcn_sched_barrier(ONE ? CROSS : 0);
  }
  // t0 (signed) enters at word 9, t1 = h (< 2^15) is folded with 2^576 =
  // 2^240 - 1: - h at word 0, + (h << 16) at word 7.  Each sum is carried two
  // words; what runs further (p2, p9, p11), or a top word that allows a
  // result >= m, is settled in the rare branch.
  uint32_t br = 0, cy = 0, cf = 0;
  const uint32_t sgn = (uint32_t)((int32_t)t0 >> 31);
  x[0] = subb(x[0], t1, br);
  x[1] = subb(x[1], 0u, br);
  x[7] = addc(x[7], t1 << 16, cy);
  x[8] = addc(x[8], t1 >> 16, cy);
  x[9] = addc(x[9], t0, cf);
  x[10] = addc(x[10], sgn, cf);
  const uint32_t p11 = cf + sgn;
  if ((br | cy | p11) != 0 || x[17] == 0xFFFFFFFFu || force_general)
    mf_settle(x, -(int32_t)br, (int32_t)cy, (int32_t)p11, (int32_t)t1 >> 31);
}

// What may be moved across the end of the first tile: MFMAs and LDS reads of the
// next tiles, or LDS reads only, where 128 VGPRs hold no more (normals, levels,
// batches).  With
// nothing moved a step of a lone wave takes 5% longer: 64 streams x 10 000 at 8
// lanes 130 us against 124 (normals 248, 245 with LDS reads, 250 and spills with
// MFMAs); 65 536 x 4096 is even.
// Operands through the L1 wait longer: 20 streams x 60 000 normals of several
// levels at 64 lanes 220 us with LDS reads only, 180 with MFMAs and such reads.
constexpr int MF_CROSS_ALL = 0x108, MF_CROSS_LDS = 0x100, MF_CROSS_BUFFER = 0x28;

template <int CROSS = MF_CROSS_ALL, class Fetch>
__device__ __forceinline__ void mfma_step_split(uint32_t (&x)[NW], const Fetch& fetch, bool force_general) {
  mfma_step_split<true, CROSS>(x, fetch, fetch, force_general);
}

// ---------------------------------------------------------------------------
// product by a factor that 32 lanes share
//
// Y <- X Y mod m with one X per half-wave and a Y of each lane's own: the
// lanes of a record start this way (X the record's state, Y = A^l).  The
// digits of the product are a contraction too, with the Toeplitz matrix of
// X's digits, P_r = sum_i x_{r-i} y_i, as the A operand:
//
//  * X and Y enter as balanced base-256 digits, 72 and a last one in {0, 1}:
//    the bytes of X + 0x8080...80 with their top bits flipped, and the carry
//    out of that sum;
//  * Y's digits are placed as the step places them (halves exchanged across
//    the lane halves), and the output rows as mfma_step_split places them:
//    lanes 0..31 receive words 0..17 of the product, lanes 32..63 words
//    18..35.  Lane (rr, h) = (l mod 32, l div 32) of the A operand for output
//    tile mt and input step ks then holds x_{r - 16 ks - 36 h - j}, j < 16,
//    for the row r = 16 mt + 4 (rr div 8) + rr mod 4 + 72 (rr div 4 mod 2):
//    seven windows d = mt - ks = -2..4 of X's digits in reversed order, bytes
//    151 - r + 16 mt - 16 d + 36 h and up of an array Z that holds digit q at
//    151 - q between zeros (the digit y_72 falls on byte 4 of step 2 of the
//    upper half by itself);
//  * the windows start at any byte, and LDS reads that are not word-aligned
//    run at a fraction of the rate (start-up 20% slower than mulmod_generic
//    with them, 20% faster without), so Z is kept four times, copy c shifted
//    down by 3 - c bytes, and lane rr reads whole words of copy rr mod 4;
//  * |P_r| <= 73 128 128 < 2^21, and the 36 words of the product follow by
//    the step's chain and are reduced by mod_m.
constexpr int MF_SHARED_COPY = 320;                  // bytes between copies (bank offset 16)
constexpr int MF_SHARED_BYTES = 4 * MF_SHARED_COPY;  // per half-wave
// The B operands of one tile of 32 lanes in memory: 3 steps x 64 lanes x 16
// bytes; a level's table holds the two tiles of Y = A^l, l < 64.
constexpr size_t MF_START_WORDS = (size_t)2 * 3 * 64 * 4;

// Bytes of x + 0x8080...80 with the top bits flipped: digits 0..71; returns
// digit 72.
__device__ __forceinline__ uint32_t mf_balance(const uint32_t (&x)[NW], uint32_t (&d)[NW]) {
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) d[k] = addc(x[k], 0x80808080u, c) ^ 0x80808080u;
  return c;
}

// The shared factor's digits to LDS, each half-wave its own X at lds + h
// MF_SHARED_BYTES: lane rr < 18 of a half holds word rr of X, the others 0.
// The carries of X + 0x8080...80 come from one add of the wave's generate and
// propagate masks, so no lane runs an 18-word chain.  Words 0..57 of each
// copy are written: all that the windows cover.
__device__ __forceinline__ void mf_shared_digits(uint32_t w, uint8_t* __restrict__ lds, uint32_t lane) {
  const uint32_t rr = lane & 31u, h = lane >> 5;
  const uint64_t gen = __ballot(w > 0x7F7F7F7Fu), prop = __ballot(w == 0x7F7F7F7Fu);
  const uint64_t carry = ((gen | prop) + gen) ^ prop;
  // word 37 - rr of Z; lane 18 holds digit 72, lanes above it zero digits
  const uint32_t z =
      __builtin_bswap32((w + 0x80808080u + ((uint32_t)(carry >> lane) & 1u)) ^ 0x80808080u);
  const uint32_t up = __builtin_amdgcn_update_dpp(0, z, 0x138, 0xF, 0xF, true);  // wave_shr:1: word 38 - rr
  uint32_t* const base = reinterpret_cast<uint32_t*>(lds + h * MF_SHARED_BYTES);
#pragma unroll
  for (uint32_t c = 0; c < 4; ++c) {
    uint32_t* const copy = base + c * (MF_SHARED_COPY / 4);
    copy[37u - rr] = __builtin_amdgcn_alignbyte(up, z, 3u - c);
    if (rr < 26) copy[rr < 6 ? rr : 32u + rr] = 0u;
  }
  mf_wave_sync();
}

// B operands of the lanes' own factors y: b[0..2] of state tile 0 (lanes
// 0..31), b[3..5] of tile 1.
__device__ __forceinline__ void mf_shared_operands(const uint32_t (&y)[NW], mf_v4i (&b)[6]) {
  uint32_t lo[9], hi[9], d[NW];
  uint32_t l9 = 0, h9 = mf_balance(y, d);
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    lo[k] = d[k];
    hi[k] = d[9 + k];
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) mf_swap(lo[k], hi[k]);
  mf_swap(l9, h9);
  b[0] = mf_v4i{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3]};
  b[1] = mf_v4i{(int)lo[4], (int)lo[5], (int)lo[6], (int)lo[7]};
  b[2] = mf_v4i{(int)lo[8], (int)l9, 0, 0};
  b[3] = mf_v4i{(int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
  b[4] = mf_v4i{(int)hi[4], (int)hi[5], (int)hi[6], (int)hi[7]};
  b[5] = mf_v4i{(int)hi[8], (int)h9, 0, 0};
}

// r = X Y mod m from the digits that mf_shared_digits wrote and the operands
// of mf_shared_operands (ONE: both halves have the same X).  Must run with
// all 64 lanes of the wave active.
template <bool ONE>
__device__ __forceinline__ void mf_shared_product(const uint8_t* __restrict__ lds, const mf_v4i (&b)[6],
                                                  uint32_t (&r)[NW], uint32_t lane) {
  const uint32_t rr = lane & 31u, h = lane >> 5;
  // lane (rr, h)'s window d in its copy: bytes 0..231 for d = -2..4
  const uint8_t* f0 = lds + ((rr & 3u) * MF_SHARED_COPY + 148u - 4u * (rr >> 3) - 72u * ((rr >> 2) & 1u) + 36u * h - 64u);
  typedef uint32_t words4 __attribute__((ext_vector_type(4), aligned(4)));
  auto window = [&](int half, int d) {
    return __builtin_bit_cast(mf_v4i, *reinterpret_cast<const words4*>(f0 + half * MF_SHARED_BYTES + 16 * (4 - d)));
  };
  const int32_t k16 = (int32_t)mf_opaque(65536u);
  // the first fold of mod_m word by word as the two halves L and H arrive:
  // T1 = L + H 2^240 - H
  uint32_t t[26], hw[NW];
  uint32_t cy = 0, br = 0;
  int32_t c0 = 0, c1 = 0;
  uint32_t e0 = 0, e1 = 0;
#pragma unroll
  for (int mt = 0; mt < 5; ++mt) {
    mf_v16i s0 = {}, s1 = {};
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) {
      const mf_v4i f = window(0, mt - ks);
      s0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(f, b[ks], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(ONE ? f : window(1, mt - ks), b[3 + ks], s1, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < (mt < 4 ? 4 : 2); ++q) {
      const int j = 4 * mt + q;
      uint32_t w0 = mf_chain(s0, q, k16, c0), w1 = mf_chain(s1, q, k16, c1);
      mf_swap(w0, w1);
      hw[j] = w1;
      if (j >= 7) w0 = addc(w0, j == 7 ? hw[0] << 16 : __builtin_amdgcn_alignbit(hw[j - 7], hw[j - 8], 16), cy);
      t[j] = subb(w0, w1, br);
    }
    if (mt == 4) {
      // with row 144 (x_72 y_72) a high half carries nothing past word 35
      e0 = (uint32_t)(c0 + s0[8]);
      e1 = (uint32_t)(c1 + s1[8]);
    }
    // one tile's words before the next tile's MFMAs: fits the generate
    // kernels' 128 VGPRs
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int k = NW; k < 26; ++k) {
    const uint32_t w = addc(k < 25 ? __builtin_amdgcn_alignbit(hw[k - 7], hw[k - 8], 16) : hw[17] >> 16, 0u, cy);
    t[k] = subb(w, 0u, br);
  }
  // H lacks the carry `low` out of L, and has one of its own, `high`, only
  // when that addition would wrap: T1 += (low + high 2^576) (2^240 - 1)
  uint32_t low = (uint32_t)c0, other = (uint32_t)c1, b2 = 0, c9 = 0;
  mf_swap(low, other);
  mf_swap(e0, e1);
  const uint32_t high = e1;
  const uint32_t sgn = (uint32_t)((int32_t)low >> 31);
  t[0] = subb(t[0], low, b2);
  t[1] = subb(t[1], sgn, b2);
  t[7] = addc(t[7], low << 16, c9);
  t[8] = addc(t[8], (uint32_t)((int32_t)low >> 16), c9);
  const int32_t p2 = -(int32_t)(b2 + sgn), p9 = (int32_t)(c9 + sgn);
  if ((p2 | p9 | (int32_t)high) != 0) {
    int64_t acc = 0;
#pragma unroll
    for (int k = 0; k < 26; ++k) {
      int64_t add = 0;
      if (k == 2) add = p2;
      if (k == 9) add = p9;
      if (k == 18) add = -(int64_t)(int32_t)high;
      if (k == 25) add = (int64_t)(int32_t)high * 65536;
      acc += (int64_t)t[k] + add;
      t[k] = (uint32_t)acc;
      acc >>= 32;
    }
  }
  mod_m_folded(t, r);
}

}  // namespace rlx
