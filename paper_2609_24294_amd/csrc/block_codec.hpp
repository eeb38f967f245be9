// block_codec.hpp -- per-block ZFP fixed-rate coding, one block per lane.
//
// Everything here works on one 4x4x4 block held in registers of a single
// lane: block exponent, block-floating-point cast, separable integer lifting,
// sequency reordering, negabinary conversion, a 64x32 bit-matrix transpose
// into bit planes, and the embedded bit-plane coder/decoder cut at the fixed
// budget of 64*rate bits (the paper's Section II-C: independent 4^3 blocks,
// lifting transform, precision reduction, exactly r bits per value; the
// in-block steps as in ZFP's published algorithm description).
//
// Stream layout of one block (64*rate bits, least significant bit first in
// little-endian 64-bit words):
//   bit 0        1 if the block has a nonzero value, else 0 and the rest is 0
//   bits 1..8    emax + 127, emax = largest exponent e with |v| = f 2^e,
//                f in [1/2,1) (values below 2^-126 count as e = -126)
//   then, planes 31..0 of the negabinary coefficients in sequency order:
//   the first n bits verbatim, then group tests and unary scans that make
//   further coefficients significant; the last position is implied when a
//   scan reaches it; when the budget runs out the rest is zero.
//
// Variable-size modes (fixed precision, fixed accuracy) run the same coder
// but stop after the bit planes 31 .. 32 - p, p = min(maxprec, max(0,
// emax - minexp + 2 (d + 1))) with d = 3 (ZFP's rule for its precision and
// accuracy modes, which the paper names as the variable-size alternative);
// p = 0 makes the block the single bit 0.  The defaults of maxprec and minexp
// give p = 32 for every float block, which is fixed rate.
//
// The functions are __host__ __device__ so that the same logic can be built
// for the CPU when debugging; the library itself only runs them on the GPU.
#pragma once

#include <stdint.h>

#if defined(__HIP_DEVICE_COMPILE__)
#define ZFPX_HD __host__ __device__ __attribute__((always_inline)) inline
#elif defined(__HIPCC__)
#define ZFPX_HD __host__ __device__ inline
#else
#define ZFPX_HD inline
#endif

namespace zfpx {

constexpr uint32_t kNegabinaryMask = 0xaaaaaaaau;
constexpr int kMinExpNone = -1074;  // no exponent floor: every block keeps maxprec planes

// Bit planes coded for a block with exponent emax.
ZFPX_HD int block_precision(int emax, int maxprec, int minexp) {
  const int p = emax - minexp + 8;
  return p < 0 ? 0 : (p > maxprec ? maxprec : p);
}

// ---------------------------------------------------------------------------
// Sequency order, computed at compile time by sorting the 64 block-local
// indices i = 16 z + 4 y + x on the key (x+y+z, x^2+y^2+z^2, i).
// ---------------------------------------------------------------------------
struct SeqOrder {
  int8_t idx[64];  // idx[s] = block-local index at sequency position s
};

constexpr int seq_key(int i) {
  int x = i & 3, y = (i >> 2) & 3, z = i >> 4;
  return ((x + y + z) * 64 + (x * x + y * y + z * z)) * 64 + i;
}

constexpr SeqOrder make_seq_order() {
  SeqOrder o{};
  int a[64] = {};
  for (int i = 0; i < 64; i++) a[i] = i;
  for (int i = 1; i < 64; i++) {  // insertion sort
    int v = a[i], j = i - 1;
    while (j >= 0 && seq_key(a[j]) > seq_key(v)) {
      a[j + 1] = a[j];
      j--;
    }
    a[j + 1] = v;
  }
  for (int i = 0; i < 64; i++) o.idx[i] = (int8_t)a[i];
  return o;
}

constexpr SeqOrder kSeq = make_seq_order();

// ---------------------------------------------------------------------------
// Scalar helpers
// ---------------------------------------------------------------------------
ZFPX_HD uint32_t f32_bits(float f) { return __builtin_bit_cast(uint32_t, f); }

ZFPX_HD float scale_pow2(float f, int e) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_ldexpf(f, e);
#else
  return __builtin_ldexpf(f, e);
#endif
}

ZFPX_HD int ctz64(uint64_t x) {  // x != 0
  return __builtin_ctzll(x);
}

// ---------------------------------------------------------------------------
// Lifting (wrapping int32 arithmetic, arithmetic shifts)
// ---------------------------------------------------------------------------
ZFPX_HD void lift_fwd(int32_t& x0, int32_t& x1, int32_t& x2, int32_t& x3) {
  // done in uint32 so that wrap-around is defined; >> on int32 is arithmetic
  auto add = [](int32_t a, int32_t b) { return (int32_t)((uint32_t)a + (uint32_t)b); };
  auto sub = [](int32_t a, int32_t b) { return (int32_t)((uint32_t)a - (uint32_t)b); };
  x0 = add(x0, x3) >> 1; x3 = sub(x3, x0);
  x2 = add(x2, x1) >> 1; x1 = sub(x1, x2);
  x0 = add(x0, x2) >> 1; x2 = sub(x2, x0);
  x3 = add(x3, x1) >> 1; x1 = sub(x1, x3);
  x3 = add(x3, x1 >> 1); x1 = sub(x1, x3 >> 1);
}

ZFPX_HD void lift_inv(int32_t& x0, int32_t& x1, int32_t& x2, int32_t& x3) {
  auto add = [](int32_t a, int32_t b) { return (int32_t)((uint32_t)a + (uint32_t)b); };
  auto sub = [](int32_t a, int32_t b) { return (int32_t)((uint32_t)a - (uint32_t)b); };
  // The steps "a += b; b = 2b - a" leave b = 2b - (a + b) = b - a (mod 2^32):
  // two operations instead of three.
  auto step = [&](int32_t& a, int32_t& b) {
    const int32_t a0 = a;
    a = add(a0, b);
    b = sub(b, a0);
  };
  x1 = add(x1, x3 >> 1); x3 = sub(x3, x1 >> 1);
  step(x1, x3);
  step(x2, x0);
  step(x1, x2);
  step(x3, x0);
}

// Forward 3-D transform of q[16 z + 4 y + x]: x-lines, y-lines, z-lines.
ZFPX_HD void xform_fwd(int32_t* q) {
#pragma unroll
  for (int zy = 0; zy < 16; zy++) lift_fwd(q[4 * zy], q[4 * zy + 1], q[4 * zy + 2], q[4 * zy + 3]);
#pragma unroll
  for (int z = 0; z < 4; z++)
#pragma unroll
    for (int x = 0; x < 4; x++)
      lift_fwd(q[16 * z + x], q[16 * z + 4 + x], q[16 * z + 8 + x], q[16 * z + 12 + x]);
#pragma unroll
  for (int yx = 0; yx < 16; yx++) lift_fwd(q[yx], q[16 + yx], q[32 + yx], q[48 + yx]);
}

// Inverse: z-lines, y-lines, x-lines.
ZFPX_HD void xform_inv(int32_t* q) {
#pragma unroll
  for (int yx = 0; yx < 16; yx++) lift_inv(q[yx], q[16 + yx], q[32 + yx], q[48 + yx]);
#pragma unroll
  for (int z = 0; z < 4; z++)
#pragma unroll
    for (int x = 0; x < 4; x++)
      lift_inv(q[16 * z + x], q[16 * z + 4 + x], q[16 * z + 8 + x], q[16 * z + 12 + x]);
#pragma unroll
  for (int zy = 0; zy < 16; zy++) lift_inv(q[4 * zy], q[4 * zy + 1], q[4 * zy + 2], q[4 * zy + 3]);
}

// ---------------------------------------------------------------------------
// Bit transpose
// ---------------------------------------------------------------------------

// Two independent 32x32 transposes at once on 64-bit words: a[r] holds row r
// of the first matrix in its low half and of the second in its high half;
// afterwards a[r] low/high bit c = old a[c] low/high bit r.  The classic
// five-stage block-swap transpose: stage J swaps, between rows r and r+J
// (r & J == 0), the bits whose column has bit J set in row r with the bits
// whose column has it clear in row r+J.  Stages 16 and 8 move whole bytes
// (one byte permute per output half); stages 4, 2, 1 are a shift and a
// bit-field select per output half.

// Byte permute: result byte i = byte sel_i of (hi:lo), bytes 0-3 from lo.
ZFPX_HD uint32_t byte_perm(uint32_t hi, uint32_t lo, uint32_t sel) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_perm(hi, lo, sel);
#else
  uint64_t x = ((uint64_t)hi << 32) | lo;
  uint32_t r = 0;
  for (int i = 0; i < 4; i++) r |= (uint32_t)((x >> (8 * ((sel >> (8 * i)) & 7))) & 0xff) << (8 * i);
  return r;
#endif
}

template <int J>
ZFPX_HD void transpose_bytes64(uint64_t* a) {
  // J = 16: new a = [a.b0 a.b1 b.b0 b.b1], new b = [a.b2 a.b3 b.b2 b.b3]
  // J = 8 : new a = [a.b0 b.b0 a.b2 b.b2], new b = [a.b1 b.b1 a.b3 b.b3]
  constexpr uint32_t sa = J == 16 ? 0x05040100u : 0x06020400u;
  constexpr uint32_t sb = J == 16 ? 0x07060302u : 0x07030501u;
#pragma unroll
  for (int r = 0; r < 32; r++) {
    if ((r & J) == 0) {
      uint32_t alo = (uint32_t)a[r], ahi = (uint32_t)(a[r] >> 32);
      uint32_t blo = (uint32_t)a[r + J], bhi = (uint32_t)(a[r + J] >> 32);
      a[r] = byte_perm(blo, alo, sa) | ((uint64_t)byte_perm(bhi, ahi, sa) << 32);
      a[r + J] = byte_perm(blo, alo, sb) | ((uint64_t)byte_perm(bhi, ahi, sb) << 32);
    }
  }
}

// Bit select: (a & m) | (b & ~m), one three-input logic instruction; INV
// returns its complement, still one instruction.
template <bool INV = false>
ZFPX_HD uint32_t bit_select(uint32_t m, uint32_t a, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_bitop3_b32(m, a, b, INV ? 0x35 : 0xCA);
#else
  return INV ? ~((a & m) | (b & ~m)) : (a & m) | (b & ~m);
#endif
}

// Any three-input bitwise function in one instruction: bit i of TT is the
// result for the inputs (s0, s1, s2) = (bit 2, bit 1, bit 0 of i).
template <uint32_t TT>
ZFPX_HD uint32_t bitop3(uint32_t s0, uint32_t s1, uint32_t s2) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_bitop3_b32(s0, s1, s2, TT);
#else
  uint32_t r = 0;
  for (int i = 0; i < 8; i++)
    if ((TT >> i) & 1) r |= ((i & 4) ? s0 : ~s0) & ((i & 2) ? s1 : ~s1) & ((i & 1) ? s2 : ~s2);
  return r;
#endif
}

// The bit stages 4, 2 and 1 stay inside groups of eight rows: a points to the
// first row of one group.  INV_HI complements the rows r + J written by the
// stage (the odd rows when J = 1), at no cost.
template <int J, uint32_t MASK, bool INV_HI = false>
ZFPX_HD void transpose_bits64(uint64_t* a) {
  // Each half is shifted on its own: the bits a 64-bit shift would carry
  // across the halves land where the select mask discards them.
  constexpr uint32_t HM = MASK << J;
#pragma unroll
  for (int r = 0; r < 8; r++) {
    if ((r & J) == 0) {
      uint32_t xl = (uint32_t)a[r], xh = (uint32_t)(a[r] >> 32);
      uint32_t yl = (uint32_t)a[r + J], yh = (uint32_t)(a[r + J] >> 32);
      a[r + J] = (uint64_t)bit_select<INV_HI>(MASK, xl >> J, yl) |
                 ((uint64_t)bit_select<INV_HI>(MASK, xh >> J, yh) << 32);
      a[r] = (uint64_t)bit_select(HM, yl << J, xl) | ((uint64_t)bit_select(HM, yh << J, xh) << 32);
    }
  }
}

// The J = 1 stage reading the odd rows complemented (the input rows r + 1),
// at no cost: each output is one three-input function of the two rows.
ZFPX_HD void transpose_bits64_odd_in_inverted(uint64_t* a) {
  constexpr uint32_t M = 0x55555555u, HM = M << 1;
#pragma unroll
  for (int r = 0; r < 8; r += 2) {
    uint32_t xl = (uint32_t)a[r], xh = (uint32_t)(a[r] >> 32);
    uint32_t yl = (uint32_t)a[r + 1], yh = (uint32_t)(a[r + 1] >> 32);
    // odd row: (M & x >> 1) | (~M & ~y); even row: (HM & ~(y << 1)) | (~HM & x)
    a[r + 1] = (uint64_t)bitop3<0xC5>(M, xl >> 1, yl) | ((uint64_t)bitop3<0xC5>(M, xh >> 1, yh) << 32);
    a[r] = (uint64_t)bitop3<0x3A>(HM, yl << 1, xl) | ((uint64_t)bitop3<0x3A>(HM, yh << 1, xh) << 32);
  }
}

// Make N values available at this point (an empty asm that reads and writes
// each).  Without it the compiler moves each output of a transpose stage to
// its use behind the next branch: both inputs then stay live beside the
// outputs already made, twice the registers.
template <int N>
ZFPX_HD void pin_values(uint64_t* a) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int i = 0; i < N; i++) asm volatile("" : "+v"(a[i]));
#else
  (void)a;
#endif
}
template <int N>
ZFPX_HD void pin_values(int32_t* a) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int i = 0; i < N; i++) asm volatile("" : "+v"(a[i]));
#else
  (void)a;
#endif
}

// Each stage swaps one bit of the row index with the same bit of the column
// index; the stages commute, so any order gives the transpose.  It is done in
// two parts: the byte stages over all rows, and the bit stages for each group
// of eight rows (bit planes 8 g .. 8 g + 7), which the coder runs as it
// reaches the group (and not at all for planes past the last one coded).
ZFPX_HD void transpose_bytes(uint64_t* a) {
  transpose_bytes64<16>(a);
  transpose_bytes64<8>(a);
}

// Bit stages of a group, encoder.  INVERT_ODD: afterwards rows 1, 3, 5, 7 are
// complemented.  XOR with a constant commutes with the transpose, so the
// encoder's negabinary XOR with 0xaaaaaaaa (the odd bits of every coefficient)
// becomes exactly this.
template <bool INVERT_ODD = false>
ZFPX_HD void transpose_group(uint64_t* a) {
  transpose_bits64<4, 0x0f0f0f0fu>(a);
  transpose_bits64<2, 0x33333333u>(a);
  transpose_bits64<1, 0x55555555u, INVERT_ODD>(a);
}

// The whole transpose at once: the same stages, for the mapping probe.  The
// library runs the two parts apart (the decoder in the other order).
template <bool INVERT_ODD = false>
ZFPX_HD void transpose32x2(uint64_t* a) {
  transpose_bytes(a);
#pragma unroll
  for (int g = 0; g < 4; g++) transpose_group<INVERT_ODD>(a + 8 * g);
}

// Bit stages of a group, decoder: of rows 1, 3, 5, 7 complemented (the J = 1
// stage first, reading them inverted).  Eight zero rows become kZeroGroup.
constexpr uint64_t kZeroGroup = 0xaaaaaaaaaaaaaaaaull;
ZFPX_HD void transpose_group_odd_in_inverted(uint64_t* a) {
  transpose_bits64_odd_in_inverted(a);
  transpose_bits64<2, 0x33333333u>(a);
  transpose_bits64<4, 0x0f0f0f0fu>(a);
}

// ---------------------------------------------------------------------------
// Coded-stream access in LDS
// ---------------------------------------------------------------------------
// Each lane owns a slice of LDS words for its block: `rate` words of stream
// followed by slack words that are always zero, so that windows and writes
// that run past the budget stay inside the slice.

constexpr int kSlackWords = 2;

// OR the (up to 64-bit) value `code` into the slice at bit position `pos`.
// The word index of bit position pos, kept opaque so that the address
// becomes one shift-add of it (not a shift, a mask and an add).
ZFPX_HD uint32_t word_of(uint32_t pos) {
  uint32_t w = pos >> 6;
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(w));
#endif
  return w;
}

ZFPX_HD void or_bits(uint64_t* s, uint32_t pos, uint64_t code) {
  uint32_t w = word_of(pos), b = pos & 63;
  uint64_t lo = code << b;
  uint64_t hi = (code >> 1) >> (63 - b);
#if defined(__HIP_DEVICE_COMPILE__)
  __hip_atomic_fetch_or(s + w, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  __hip_atomic_fetch_or(s + w + 1, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
#else
  s[w] |= lo;
  s[w + 1] |= hi;
#endif
}

// The 64 stream bits starting at bit position `pos`.
// Read as 32-bit words (the low word of each 64-bit word first): three words
// from word pos / 32 hold the window, and two funnel shifts by pos % 32 (which
// the instruction takes from the low 5 bits of its count) assemble it.
typedef uint32_t __attribute__((may_alias)) u32_alias;
ZFPX_HD uint32_t funnel32(uint32_t hi, uint32_t lo, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_alignbit(hi, lo, b);
#else
  return (uint32_t)((((uint64_t)hi << 32) | lo) >> (b & 31));
#endif
}
// The 32-bit word index of bit position pos, opaque as word_of.
ZFPX_HD uint32_t word32_of(uint32_t pos) {
  uint32_t w = pos >> 5;
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(w));
#endif
  return w;
}
ZFPX_HD uint64_t window64(const uint64_t* s, uint32_t pos) {
  const u32_alias* d = reinterpret_cast<const u32_alias*>(s) + word32_of(pos);
  const uint32_t d0 = d[0], d1 = d[1], d2 = d[2];
  return (uint64_t)funnel32(d1, d0, pos) | ((uint64_t)funnel32(d2, d1, pos) << 32);
}

// The three 32-bit words that hold the window at pos, and the window itself.
struct Words3 {
  uint32_t w0, w1, w2;
};
ZFPX_HD Words3 window_words(const uint64_t* s, uint32_t pos) {
  const u32_alias* d = reinterpret_cast<const u32_alias*>(s) + word32_of(pos);
  return Words3{d[0], d[1], d[2]};
}
ZFPX_HD uint64_t window_of(const Words3& w, uint32_t pos) {
  return (uint64_t)funnel32(w.w1, w.w0, pos) | ((uint64_t)funnel32(w.w2, w.w1, pos) << 32);
}

// Make the words of a window available at this point (an empty asm that reads
// and writes all three): the reads are issued first and waited for together.
ZFPX_HD void pin_words(Words3& a) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(a.w0), "+v"(a.w1), "+v"(a.w2));
#else
  (void)a;
#endif
}

// x as 64 bits, x not known to the compiler (which would keep a constant upper
// half in a register of its own throughout a loop around the coder).
ZFPX_HD uint64_t sign_extended(int32_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(x));
#endif
  return (uint64_t)(int64_t)x;
}

// A value that is the same in every active lane, in a scalar register.
ZFPX_HD int uniform_int(int x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_readfirstlane(x);
#else
  return x;
#endif
}

// Any three-input bitwise function of 64-bit words (bitop3 on both halves).
template <uint32_t TT>
ZFPX_HD uint64_t bitop3_64(uint64_t s0, uint64_t s1, uint64_t s2) {
  return (uint64_t)bitop3<TT>((uint32_t)s0, (uint32_t)s1, (uint32_t)s2) |
         ((uint64_t)bitop3<TT>((uint32_t)(s0 >> 32), (uint32_t)(s1 >> 32), (uint32_t)(s2 >> 32))
          << 32);
}

// (a << S) + b, one instruction for S <= 4 (opaque: the compiler would make
// a multiply of two of them).
template <int S>
ZFPX_HD uint64_t shift_add64(uint64_t a, uint64_t b) {
  uint64_t r = (a << S) + b;
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(r));
#endif
  return r;
}

// Population count of a 64-bit word.
ZFPX_HD int popc64(uint64_t x) { return __builtin_popcountll(x); }

// Whether any active lane of the wavefront holds a nonzero value (a scalar
// branch: loops on it keep every lane, so their body must do nothing where
// x = 0).
ZFPX_HD bool any_lane(uint64_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_ballot_w64(x != 0) != 0;
#else
  return x != 0;
#endif
}

// e without its lowest one.
ZFPX_HD uint64_t drop_lowest(uint64_t e) { return e & (e - 1); }

// Each one of y moved up by the number of ones below it (mod 2^64): y, plus
// for t = 0, 1, ... y without its lowest t + 1 ones shifted up by t.  Steps
// come in pairs (a step past a lane's last one adds nothing), the first with
// constant shifts, which one shift-add instruction takes.
ZFPX_HD uint64_t spread_ranks(uint64_t y) {
  uint64_t sp = y, e = drop_lowest(y);
  if (any_lane(e)) {
    sp = shift_add64<0>(e, sp);
    e = drop_lowest(e);
    sp = shift_add64<1>(e, sp);
    e = drop_lowest(e);
    if (any_lane(e)) {
      sp = shift_add64<2>(e, sp);
      e = drop_lowest(e);
      sp = shift_add64<3>(e, sp);
      e = drop_lowest(e);
      for (int t = 4; any_lane(e); t += 2) {
        const int st = uniform_int(t);
        sp += e << st;
        e = drop_lowest(e);
        sp += e << (st + 1);
        e = drop_lowest(e);
      }
    }
  }
  return sp;
}

// Each one of y moved down by the number of ones below it: y, minus for
// t = 1, 2, ... y without its lowest t ones shifted down by t.
ZFPX_HD uint64_t gather_ranks(uint64_t y) {
  uint64_t down = 0, e = drop_lowest(y);
  if (any_lane(e)) {
    down = e >> 1;
    e = drop_lowest(e);
    down += e >> 2;
    e = drop_lowest(e);
    if (any_lane(e)) {
      down += e >> 3;
      e = drop_lowest(e);
      down += e >> 4;
      e = drop_lowest(e);
      for (int t = 5; any_lane(e); t += 2) {
        const int st = uniform_int(t);
        down += e >> st;
        e = drop_lowest(e);
        down += e >> (st + 1);
        e = drop_lowest(e);
      }
    }
  }
  return y - down;
}

// ---------------------------------------------------------------------------
// Encoder
// ---------------------------------------------------------------------------

// Encode one block of 64 floats (v[16 z + 4 y + x]) into the slice `out`,
// which must hold rate + kSlackWords zero words.  Bits are ORed in place;
// the slack words may receive bits past the budget and are not part of the
// stream.  v is clobbered.  Returns the block's length in bits (at most
// 64 * rate; 1 for a block coded as the single bit 0).
//
// The coder is the larger half of the work and runs at the vector unit's issue
// rate, so it is written for few instructions per bit plane:
//  - a plane without newly significant coefficients in any lane is one mask,
//    one OR into the slice and one compare: positions advance by `adv`, kept
//    across planes and updated only when n changes;
//  - bits may run past the budget into the slack words (a plane starts below
//    the budget, so its verbatim bits end before bit maxbits + 63 and a code
//    word of at most 64 bits stays in the two slack words): no test of the
//    budget inside a plane;
//  - the groups of a plane are one code word, also when they reach coefficient
//    63; only a word of more than 64 bits takes the loop over groups.
// VAR = false is fixed rate (every plane may be coded).
template <int RATE, bool VAR = false>
ZFPX_HD uint32_t encode_block(float* v, uint64_t* out, int rate_rt, int maxprec = 32,
                              int minexp = kMinExpNone) {
  const int rate = RATE > 0 ? RATE : rate_rt;
  const uint32_t maxbits = 64u * (uint32_t)rate;
  // block exponent from the largest magnitude (its biased exponent field)
  float amax = 0.0f;
#pragma unroll
  for (int i = 0; i < 64; i++) amax = __builtin_fmaxf(amax, __builtin_fabsf(v[i]));
  uint32_t mx = f32_bits(amax);
  if (mx == 0) return 1;  // empty block: the single bit 0, all zero
  int emax = (int)(mx >> 23) - 126;  // subnormal maximum (field 0) gives -126
  const int kmin = VAR ? 32 - block_precision(emax, maxprec, minexp) : 0;
  if (VAR && kmin == 32) return 1;  // no plane to code: the single bit 0
  or_bits(out, 0, 1u | ((uint64_t)((emax + 127) & 0xff) << 1));
  // X[s] = coefficients s and 32+s (negabinary); after the transpose X[k] is
  // bit plane k: bit s of X[k] = bit k of coefficient s
  uint64_t X[32];
  {
    int32_t q[64];
    // 2^(30 - emax) is a normal float for emax >= -97: one multiply per value
    // is the exact scaling (a product below 1 in magnitude truncates to 0
    // whatever its rounding).  Smaller blocks are first scaled by 2^64,
    // exactly: a step of its own, so that one cast and transform follows.
    int sh = 30 - emax;
    if (emax < -97) {
#pragma unroll
      for (int i = 0; i < 64; i++) v[i] *= 0x1p64f;
      sh -= 64;
    }
    const float sc = scale_pow2(1.0f, sh);
#pragma unroll
    for (int i = 0; i < 64; i++) q[i] = (int32_t)(v[i] * sc);
    xform_fwd(q);
    // negabinary (q + mask) ^ mask: the add here, the XOR in the transpose
#pragma unroll
    for (int s = 0; s < 32; s++) {
      uint32_t lo = (uint32_t)q[kSeq.idx[s]] + kNegabinaryMask;
      uint32_t hi = (uint32_t)q[kSeq.idx[32 + s]] + kNegabinaryMask;
      X[s] = (uint64_t)lo | ((uint64_t)hi << 32);
    }
  }
  static_assert(kNegabinaryMask == 0xaaaaaaaau, "the transpose complements the odd planes");
  transpose_bytes(X);
  pin_values<32>(X);
  uint32_t pos = 9;
  uint32_t n = 0;    // coefficients significant so far
  uint32_t adv = 1;  // verbatim bits and a group test of 0: n + (n < 64)
  uint64_t vm = 0;   // mask of the low n bits
#pragma unroll
  for (int g = 3; g >= 0; g--) {
    if (!any_lane(pos < maxbits && (!VAR || 8 * g + 7 >= kmin))) break;
    transpose_group<true>(X + 8 * g);
    pin_values<8>(X + 8 * g);
#pragma unroll
    for (int k = 8 * g + 7; k >= 8 * g; k--) {
      if (pos < maxbits && (!VAR || k >= kmin)) {
        const uint64_t x = X[k];
        or_bits(out, pos, x & vm);  // the first n bits verbatim
        uint32_t gpos = pos + n;    // the group test
        pos += adv;
        if (x > vm) {  // a bit at or above n (so n < 64)
          // Each newly significant coefficient costs a group test 1, the zeros
          // up to it and its own 1 (that one is implied, and not written, for
          // coefficient 63).  With the newly significant coefficients at
          // positions q_0 < ... < q_(m-1) of y, the code word has a group test
          // 1 at bit 0 and, for each i, the coefficient's one at bit
          // q_i + i + 1, followed (unless i is the last) by the next group test
          // 1 at bit q_i + i + 2.  With sp = sum_i 2^(q_i + i), whose top bit is
          // hs, the word is 1 + 2 sp + 4 (sp - 2^hs): parts that share no bit.
          uint64_t y = x >> n;
          const uint32_t hx = 63u - (uint32_t)__builtin_clzll(x);  // coefficient of the last one
          const uint32_t last = hx == 63 ? 1u : 0u;  // its one is implied
          const uint32_t hs = hx - n + (uint32_t)popc64(y) - 1;
          if (hs <= 62) {
            // -2^(hs+2) for the group test that does not follow the last one,
            // and -2^(hs+1) for its own one if implied
            const uint64_t cut = sign_extended(last ? -3 : -2) << (hs + 1);
            const uint64_t sp = spread_ranks(y);
            or_bits(out, gpos, shift_add64<2>(sp, shift_add64<1>(sp, cut + 1)));
            pos = gpos + hs + 3 - 2 * last;  // and the closing group test 0
          } else {
            // group by group, within the budget
            uint32_t c = n;
            pos = gpos;
            while (y != 0 && pos < maxbits) {
              const uint32_t p = (uint32_t)ctz64(y);
              const uint32_t end = c + p == 63 ? 1u : 0u;
              or_bits(out, pos, end ? uint64_t(1) : (uint64_t(1) | (uint64_t(2) << p)));
              pos += p + 2 - end;
              c += p + 1;
              y = (y >> p) >> 1;
            }
            pos += 1 - last;
          }
          n = hx + 1;
          adv = hx < 62 ? hx + 2 : 64;
          vm = ((uint64_t)2 << hx) - 1;
        }
      }
    }
  }
  return pos < maxbits ? pos : maxbits;
}

// ---------------------------------------------------------------------------
// Decoder
// ---------------------------------------------------------------------------

// The group tests and scans that follow a group test of 1, parsed from the
// 64 stream bits v after it (bit 0 first), without a loop over the groups.
// Each group is zeros up to a one (the newly significant coefficient), and
// the group test after it is 1 if another group follows: so inside every
// maximal run of ones that starts right after a zero (or at bit 0) the bits
// alternate coefficient-one, group-test, coefficient-one, ...; a run that
// ends on a coefficient-one is followed by the closing group test 0.
// Returns the coefficient-ones up to the first that a closing group test
// follows, and through upto the mask of the bits up to it (all ones if the
// window has none; bit 63 counts as followed by a 0).
ZFPX_HD uint64_t parse_groups(uint64_t v, uint64_t& upto) {
  constexpr uint64_t kEven = 0x5555555555555555ull;
  // runs that start at an even position turn to zeros when their start bit
  // is added (the carry runs through them); the others are unchanged
  const uint64_t t = v + bitop3_64<0x40>(kEven, v, v << 1);  // v & ~(v << 1) & kEven
  // coefficient-ones: even positions of even-started runs, odd positions of
  // odd-started runs
  const uint64_t e = bitop3_64<0x48>(kEven, v, t);  // v & (t ^ kEven)
  const uint64_t ends = e & ~(v >> 1);
  upto = ends ^ (ends - 1);
  return e & upto;
}

// Decode the slice `in` (rate words followed by kSlackWords zero words) into
// 64 floats (block-local order).
//
// Per bit plane the verbatim bits and the group test are the low n + 1 bits of
// the window at pos: as a number they pass 2^n - 1 exactly when the group
// test is 1.  A plane whose group test is 0 (most of them) is done with that;
// positions advance by `adv`, kept across planes and updated when n changes.
// Reads past the budget return the zero slack, which is what a budget that
// has run out yields for verbatim bits and group tests.
// After a group test of 1 the groups are parsed from the window behind it
// (parse_groups).  The run of groups ends, whichever comes first,
//  - at a closing group test 0;
//  - at coefficient 63, whose one is implied, not coded, with no test after;
//  - at the end of the budget, where the coefficient that the scan has
//    reached becomes significant.
// A run that the window does not hold whole takes the loop over groups.
// VAR = false is fixed rate (every plane may be coded).
template <int RATE, bool VAR = false>
ZFPX_HD void decode_block(const uint64_t* in, float* vout, int rate_rt, int maxprec = 32,
                          int minexp = kMinExpNone) {
  const int rate = RATE > 0 ? RATE : rate_rt;
  const uint32_t maxbits = 64u * (uint32_t)rate;
  // the header (bits 0..8) and the first plane's window (from bit 9) are in
  // the first three words: one round trip
  Words3 wfirst = window_words(in, 0);
  pin_words(wfirst);
  const uint32_t head = wfirst.w0;
  uint32_t pos = maxbits;  // an empty block decodes to zeros
  int emax = 0, kmin = 0;
  if (head & 1) {
    emax = (int)((head >> 1) & 0xff) - 127;
    pos = 9;
    if (VAR) kmin = 32 - block_precision(emax, maxprec, minexp);
  }
  uint64_t X[32];  // bit planes, then (after the transpose) coefficients s, 32+s
  uint32_t n = 0;     // coefficients significant so far
  uint32_t adv = 1;   // verbatim bits and a group test of 0: n + (n < 64)
  uint64_t vm = 0;    // mask of the low n bits
  uint64_t vm1 = 1;   // mask of the low min(n + 1, 64) bits
#pragma unroll
  for (int g = 3; g >= 0; g--) {
    if (!any_lane(pos < maxbits && (!VAR || 8 * g + 7 >= kmin))) {
#pragma unroll
      for (int k = 8 * g; k < 8 * g + 8; k++) X[k] = kZeroGroup;
      continue;
    }
#pragma unroll
    for (int k = 8 * g + 7; k >= 8 * g; k--) {
      uint64_t x = 0;
      if (pos < maxbits && (!VAR || k >= kmin)) {
        const uint64_t w = k == 31 ? window_of(wfirst, pos) : window64(in, pos);
        x = w & vm1;
        pos += adv;
        if (x > vm) {  // group test 1 (so n < 64); pos is the bit after it
          x &= vm;
          uint64_t upto;
          const uint64_t ev = parse_groups(window64(in, pos), upto);
          const uint32_t len = (uint32_t)popc64(upto);  // through the last one
          uint64_t y = gather_ranks(ev);  // bit i: coefficient n + i
          uint32_t hx = n + len - (uint32_t)popc64(ev);  // coefficient of the last one
          uint32_t used = len + 1;                       // with the closing group test
          uint32_t slow = 0;
          if (len == 64 || hx > 62) {
            // no closing group test before coefficient 63 or the window's end
            const uint32_t left = maxbits - pos;  // budget behind the first test
            const uint32_t d = 63 - n;
            const uint64_t low = ((uint64_t)1 << d) - 1;
            used = d + (uint32_t)popc64(y & low);  // bits that reach coefficient 63
            if (used <= 64 && used <= left) {
              y = (y & low) | (low + 1);
              hx = 63;
            } else if (left < 64) {
              // all ones found lie within the budget
              hx = n + left - (uint32_t)popc64(ev);
              y |= (uint64_t)1 << (hx - n);
              used = left;
            } else {
              slow = 1;
              y = 0;
              hx = n - 1;
              used = 0;
            }
          }
          x |= y << n;
          pos += used;
          n = hx + 1;
          // group by group: zeros up to the next one, at most up to
          // coefficient 63 (implied) or the end of the budget (a second stage
          // that runs no step when the first applied, not an alternative to it:
          // the compiler would carry this block's planes through a loop around
          // the decoder in extra registers)
          while (slow) {
            uint32_t lim = 63 - n;
            if (maxbits - pos < lim) lim = maxbits - pos;
            const uint64_t s = window64(in, pos);
            const uint32_t z = s ? (uint32_t)ctz64(s) : 64;
            const uint32_t t = z < lim ? z : lim;
            const uint32_t found = z < lim ? 1u : 0u;
            x |= uint64_t(1) << (n + t);
            n += t + 1;
            pos += t + found;
            slow = 0;
            if (n < 64 && pos < maxbits) {
              slow = (uint32_t)((s >> (t + found)) & 1);  // t + found <= 63
              pos += 1;
            }
          }
          vm = ((uint64_t)2 << (n - 1)) - 1;  // n >= 1 after a group test of 1
          vm1 = shift_add64<1>(vm, 1);
          adv = n < 63 ? n + 1 : 64;
        }
      }
      X[k] = x;
    }
    // odd planes complemented as the transpose reads them: every coefficient
    // comes out XORed with the negabinary mask 0xaaaaaaaa (bits 1, 3, ..., 31)
    transpose_group_odd_in_inverted(X + 8 * g);
    pin_values<8>(X + 8 * g);
  }
  transpose_bytes(X);
  int32_t q[64];
#pragma unroll
  for (int s = 0; s < 32; s++) {
    // negabinary to two's complement: (u ^ mask) - mask, the XOR done above
    q[kSeq.idx[s]] = (int32_t)((uint32_t)X[s] - kNegabinaryMask);
    q[kSeq.idx[32 + s]] = (int32_t)((uint32_t)(X[s] >> 32) - kNegabinaryMask);
  }
  xform_inv(q);
  pin_values<64>(q);
  // Reconstruction is one rounding of q 2^(emax - 30): float(q), then a
  // power-of-two scale that is exact.  It is exact also where the result is
  // subnormal, as long as float32's smallest step 2^-149 is no more than one
  // unit of q (emax >= -119): |q| < 2^23 there.  For smaller exponents the step
  // is 2^k units, k = 1 .. 8, and q is first replaced, in place, by the result
  // in units of 2^-149: a normal one (|q| >= 2^(23 + k)) is float(q) / 2^k, an
  // integer; a subnormal one is q / 2^k rounded to the nearest integer (ties
  // to even), and one that rounds to zero keeps q's sign.  Branches of the
  // whole wavefront, on values replaced in place: with two alternative
  // reconstructions the values of both would be live at once.
  uint64_t minus_zero = 0;
  if (any_lane(emax < -119)) {
    const int k = emax < -119 ? -119 - emax : 0;
    const uint32_t below = k > 0 ? 1u << (23 + k) : 0;
    const uint32_t half = k > 0 ? 1u << (k - 1) : 1;
    const float down = scale_pow2(1.0f, -k);
#pragma unroll
    for (int i = 0; i < 64; i++) {
      const int32_t qi = q[i];
      const uint32_t mag = qi < 0 ? 0u - (uint32_t)qi : (uint32_t)qi;
      const uint32_t rem = (uint32_t)qi & (2 * half - 1);  // |q| may reach 2^31 - 1: no carry past it
      const int32_t sub = k > 0 ? (qi >> k) + (int32_t)((rem + half - 1 + ((qi >> k) & 1)) >> k) : 0;
      const int32_t nor = k > 0 ? (int32_t)((float)qi * down) : qi;
      q[i] = mag < below ? sub : nor;
      minus_zero |= (uint64_t)(qi < 0 && q[i] == 0) << i;
      pin_values<1>(q + i);
    }
  }
  const float sc = scale_pow2(1.0f, emax < -119 ? -149 : emax - 30);
#pragma unroll
  for (int i = 0; i < 64; i++) vout[i] = (float)q[i] * sc;
  if (any_lane(minus_zero)) {
#pragma unroll
    for (int i = 0; i < 64; i++) vout[i] = (minus_zero >> i) & 1 ? -0.0f : vout[i];
  }
}

}  // namespace zfpx
