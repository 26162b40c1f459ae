// Bit layouts of the packed int4 / int2 codes as matrix-instruction operands (gfx950), shared by
// the decode kernels.
#pragma once

#include "bd_common.h"
#include "bd_device.h"

namespace bd {
namespace {

// A mask in a scalar register: an instruction with a literal is twice as long, and a wave alone on its SIMD issues one of
// those every 5.1 cycles, the short form every 4.
__device__ __forceinline__ uint32_t scalar_mask(uint32_t m) {
  asm("" : "+s"(m));
  return m;
}

// ---- format traits ---------------------------------------------------------------------
// One lane loads WORDS 32-bit words (32 codes) per 16-row tile.  k-step j (of 4) of the tile
// consumes 8 codes as 4 VGPRs; VGPR v holds two codes that arrive multiplied by 1/un(v).
// The B operand must present the other factor in the same order: "slot group" sg = 4*g + j
// (g = lane/16) holds 8 entries, entry e = 2*i + run for the i-th channel of one of two runs
// of 4 consecutive channels.
template <int BITS>
struct Fmt;

template <>
struct Fmt<4> {
  static constexpr int WORDS = 4;
  static constexpr float kQmax = 15.0f;
  // first channel of run `run` (0/1) of slot group sg: word sg, nibbles 0..3 / 4..7
  __device__ static int run_base(int sg, int run) { return 8 * sg + 4 * run; }
  __device__ static constexpr float un(int v) { return (v & 1) ? (1.0f / 16.0f) : 1.0f; }
  __device__ static constexpr float inv_un(int v) { return (v & 1) ? 16.0f : 1.0f; }
  // k-step j = 2*half + jj of the second product contracts the tokens of two S^T tiles of that
  // half: tile_lo(jj) fills the low fp16 half of the P' registers, tile_hi(jj) the high one
  __device__ static constexpr int tile_lo(int jj) { return 2 * jj; }
  __device__ static constexpr int tile_hi(int jj) { return 2 * jj + 1; }
  // position of block token t in the k-ordered P' / V operand: lane group t/32, then k-step j,
  // register r, half -- tile T = (t%32)/4 feeds k-step T/2, half T%2
  __device__ static int p_slot(int t) {
    const int T = (t & 31) >> 2, r = t & 3;
    return (t & ~31) + 8 * (T >> 1) + 2 * r + (T & 1);
  }
  // position (8 * slot group + entry) of channel / block token t in that operand order
  __device__ static int operand_pos(int t) { return (t & ~7) + 2 * (t & 3) + ((t >> 2) & 1); }
  __device__ static h8_t dequant(const uint32_t* w, int j) {
    const uint32_t x = w[j], y = x >> 8;
    u4_t r;
    r[0] = x & scalar_mask(0x000F000Fu);   // nibbles 0, 4
    r[1] = x & scalar_mask(0x00F000F0u);   // nibbles 1, 5 (x16)
    r[2] = y & scalar_mask(0x000F000Fu);   // nibbles 2, 6
    r[3] = y & scalar_mask(0x00F000F0u);   // nibbles 3, 7 (x16)
    return __builtin_bit_cast(h8_t, r);
  }
};

template <>
struct Fmt<2> {
  static constexpr int WORDS = 2;
  static constexpr float kQmax = 3.0f;
  // slot group sg = 2*W + jj: word W, crumbs 4*jj + 0..3 (run 0) and 8 + 4*jj + 0..3 (run 1)
  __device__ static int run_base(int sg, int run) { return 16 * (sg >> 1) + 4 * (sg & 1) + 8 * run; }
  __device__ static constexpr float un(int v) { return 1.0f / (float)(1 << (2 * v)); }
  __device__ static constexpr float inv_un(int v) { return (float)(1 << (2 * v)); }
  __device__ static constexpr int tile_lo(int jj) { return jj; }
  __device__ static constexpr int tile_hi(int jj) { return jj + 2; }
  // tile T = (t%32)/4 feeds k-step 2*(T/4) + T%2, half (T%4)/2
  __device__ static int p_slot(int t) {
    const int T = (t & 31) >> 2, r = t & 3;
    return (t & ~31) + 8 * (2 * (T >> 2) + (T & 1)) + 2 * r + ((T & 3) >> 1);
  }
  __device__ static int operand_pos(int t) {
    return 8 * (2 * (t >> 4) + ((t >> 2) & 1)) + 2 * (t & 3) + ((t >> 3) & 1);
  }
  __device__ static h8_t dequant(const uint32_t* w, int j) {
    const uint32_t x = (j & 1) ? (w[j >> 1] >> 8) : w[j >> 1];
    u4_t r;
    r[0] = x & scalar_mask(0x00030003u);   // crumbs 0, 8      (of the selected byte pair)
    r[1] = x & scalar_mask(0x000C000Cu);   // crumbs 1, 9  (x4)
    r[2] = x & scalar_mask(0x00300030u);   // crumbs 2, 10 (x16)
    r[3] = x & scalar_mask(0x00C000C0u);   // crumbs 3, 11 (x64)
    return __builtin_bit_cast(h8_t, r);
  }
};

template <int WORDS>
struct RawTile {
  uint32_t w[WORDS];
};

template <int WORDS>
__device__ __forceinline__ RawTile<WORDS> load_raw(const uint32_t* p) {
  RawTile<WORDS> t;
  if constexpr (WORDS == 4) {
    u4_t v = __builtin_nontemporal_load(reinterpret_cast<const u4_t*>(p));
    t.w[0] = v[0]; t.w[1] = v[1]; t.w[2] = v[2]; t.w[3] = v[3];
  } else {
    u2_t v = __builtin_nontemporal_load(reinterpret_cast<const u2_t*>(p));
    t.w[0] = v[0]; t.w[1] = v[1];
  }
  return t;
}

// ---- the same codes as operands of v_mfma_scale_f32_16x16x128_f8f6f4 --------------------
// One instruction contracts all 128 channels (tokens) of a 16-row tile: lane group g supplies the 32 codes it loads.
// An int4 code in the low nibble of a byte is the e4m3 number code * 2^-9 (the first 16 e4m3 bit patterns are
// linear), a 2-bit code in the low half of a nibble the e2m1 number code / 2, so the A operand is again word & mask,
// 3 instructions per word (8 int4 or 16 int2 codes), and the instruction's block scale undoes the power of two.
// The B operand is e4m3: eight registers of four bytes per lane, (half h, register j of the half, byte b).
// Measured operand order: an 8-bit operand's lane group g holds contraction indices 16g + .. in half 0 and
// 64 + 16g + .. in half 1; a 4-bit operand's holds 32g + ...
// Measured accumulation: the products of one instruction are aligned to the largest and cut at 2^-15 or so of it
// (values over the whole e4m3 range: 6e-5 of the sum of magnitudes, towards zero); with B values of at most 2^kTop
// every product is a multiple of the smallest e4m3 number within that window and the sums are exact.  (An operand's
// subnormals are aligned as if they were its smallest normal number: centre codes enter as normal numbers.)
template <int BITS>
struct FmtF8;

// e4m3 pieces of the weights P' <= 1, 2^-5 apart: 19 bits of every weight, down to a last step of 2^-25 (4 bits) or
// 2^-27 (2 bits) of the largest, so that no weight is held to less than in fp16 (11 bits, last step 2^-24).  Three end
// at 2^-22 with 2-bit codes, which loses a tail of 6144 tokens at 2^-23.5 of one dominating weight, 1.7e-4 of the result
// (with four 1e-6), and is 1.3e-5 off for 4096 ordinary tokens (5e-7); the fourth costs 0.5 us of 32.8 a step at 8 x 32K.
constexpr int kWeightPieces = 4;

template <>
struct FmtF8<4> {   // both operands 8 bits wide: byte by byte the same order on both sides
  static constexpr int kFormatA = 0, kScaleA = 127 + 9;
  static constexpr int kTop = 1;
  __device__ static i8_t a_operand(const uint32_t* w) {
    i8_t r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      r[2 * i] = (int)(w[i] & scalar_mask(0x0F0F0F0Fu));              // codes 0, 2, 4, 6
      r[2 * i + 1] = (int)((w[i] >> 4) & scalar_mask(0x0F0F0F0Fu));   // codes 1, 3, 5, 7
    }
    return r;
  }
  // block token of row 4 * gamma + r (r = 0) of S^T tile T: a lane group's 32 tokens are consecutive
  __device__ static int token(int gamma, int T) { return 32 * gamma + 4 * T; }
  __device__ static int par_slot(int t) { return t + (t >> 5); }   // LDS slot of a token's parameters: spreads the lane groups over the banks
  // where the channel (token) x of the 128 sits in the B operand: lane group, half, register, byte
  __device__ static int b_group(int x) { return x >> 5; }
  __device__ static int b_half(int x) { return (x >> 4) & 1; }
  __device__ static constexpr int b_reg(int x) { return 2 * ((x >> 3) & 1) + (x & 1); }
  __device__ static constexpr int b_byte(int x) { return (x & 7) >> 1; }
};

template <>
struct FmtF8<2> {
  static constexpr int kFormatA = 4, kScaleA = 127 + 1;
  static constexpr int kTop = 3;
  __device__ static i8_t a_operand(const uint32_t* w) {
    i8_t r = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      r[2 * i] = (int)(w[i] & scalar_mask(0x33333333u));              // codes 0, 2, .. 14
      r[2 * i + 1] = (int)((w[i] >> 2) & scalar_mask(0x33333333u));   // codes 1, 3, .. 15
    }
    return r;
  }
  __device__ static int token(int gamma, int T) { return 64 * (T >> 2) + 16 * gamma + 4 * (T & 3); }
  __device__ static int par_slot(int t) { return t + (t >> 4); }
  __device__ static int b_group(int x) { return (x >> 4) & 3; }
  __device__ static int b_half(int x) { return x >> 6; }
  __device__ static constexpr int b_reg(int x) { return ((x >> 3) & 1) + 2 * (x & 1); }
  __device__ static constexpr int b_byte(int x) { return (x & 7) >> 1; }
};

// A register that is about to be written in two halves.  (A zero, or an undefined value, costs a move each time.)
__device__ __forceinline__ uint32_t any_bits() {
  uint32_t x;
  asm volatile("" : "=v"(x));
  return x;
}
// Two values as e4m3 pieces in units of `unit` (a power of two), rounded to nearest, into half `hi` of a register;
// the values are left with what the piece does not hold: at most 2^-5 of the largest, so that pieces in units 2^-5
// apart stay below the same bound and take five more bits each.
template <bool HI>
__device__ __forceinline__ uint32_t e4m3_piece(uint32_t reg, float& x, float& y, float unit) {
  typedef short s2_t __attribute__((ext_vector_type(2)));
  typedef float f2v_t __attribute__((ext_vector_type(2)));
  const s2_t r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(__builtin_bit_cast(s2_t, reg), x, y, unit, HI);
  const uint32_t u = __builtin_bit_cast(uint32_t, r);
  const f2v_t f = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(u, unit, HI);
  x -= f[0];
  y -= f[1];
  return u;
}
// (the last piece: nothing is left to be computed)
template <bool HI>
__device__ __forceinline__ uint32_t e4m3_last(uint32_t reg, float x, float y, float unit) {
  typedef short s2_t __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(__builtin_bit_cast(s2_t, reg), x, y, unit, HI));
}

// ---- K codes and Q' as operands of v_mfma_i32_16x16x64_i8 --------------------------------
// Two instructions contract the 128 channels of a 16-token tile, 64 each, 16 of every lane group.  A lane group's 32 codes of a
// token are bytes after masks as above: 4-bit ones in the order of the words, words 0 and 1 first; 2-bit ones a word each, the
// odd crumbs of a nibble where they are, that is times 4, and Q' there a quarter.  Q' is an integer x below 2^30; x + 0x808080
// has the bytes of its four signed digits, the lower three plus 128.
//
// What rounding to x takes may show, and the block's scores take it as well (in units of 2^-30), where K is by channel and one
// of a head's products q * scale counts kFineScore and more in the scores (log2 units, per code step) while the channel's zero
// is below kFineZero scales.  Below that score, T, the roundings of 128 channels add 4e-8 T (2 bits: 2.5e-8 T) to a score, less
// than the 4e-7 .. 8e-7 that an output is off anyway (T = 2.6 .. 8, and 13 with 2 bits: no difference).  And with a larger
// zero the fp32 sums lose as much: either other tokens have codes there, whose scores are that much larger, or the zero
// term is (a channel of 200 among others of 1, one key of 1200, a query of -30: 3e-5 with or without).  So a channel that is an
// outlier as a whole, its zero at half its range, takes nothing extra.  Per-token K, whose Q' is Q: where anything was lost.
// (Issued one by one, no block / every block with them: 32K tokens 10.8 / 11.4 us, 1K 6.5 / 7.6; 2 bits, 4 x 32K 17.5 / 20.5.)
template <int BITS>
struct FmtI8;
template <>
struct FmtI8<4> {
  __device__ static i8_t a_operand(const uint32_t* w) { return FmtF8<4>::a_operand(w); }
  __device__ static constexpr float position(int) { return 1.0f; }   // what channel n of a lane's eight is to be multiplied by
  static constexpr float kFineZero = 5.0f, kFineScore = 8.0f;
};
template <>
struct FmtI8<2> {
  __device__ static i8_t a_operand(const uint32_t* w) {
    i8_t r;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t x = w[i], y = x >> 4;
      r[4 * i] = (int)(x & scalar_mask(0x03030303u));       // codes 0, 4, 8, 12
      r[4 * i + 1] = (int)(x & scalar_mask(0x0C0C0C0Cu));   // codes 1, 5, 9, 13
      r[4 * i + 2] = (int)(y & scalar_mask(0x03030303u));
      r[4 * i + 3] = (int)(y & scalar_mask(0x0C0C0C0Cu));
    }
    return r;
  }
  __device__ static constexpr float position(int n) { return n & 1 ? 0.25f : 1.0f; }
  static constexpr float kFineZero = 1.25f, kFineScore = 16.0f;
};
constexpr float kFineUnits = 1073741824.0f;   // 2^30
// Bytes of a, b, c, d: out[k] has byte k of each.
__device__ __forceinline__ void transpose_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&out)[4]) {
  const uint32_t t0 = __builtin_amdgcn_perm(b, a, 0x05010400u), t1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
  const uint32_t t2 = __builtin_amdgcn_perm(d, c, 0x05010400u), t3 = __builtin_amdgcn_perm(d, c, 0x07030602u);
  out[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
  out[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
  out[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
  out[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}
// An accumulator starts at the bits of 1.5 * 2^23: as a float it is then 1.5 * 2^23 + sum, for sums below 2^22 (at most 128 *
// 15 * 128).
constexpr int kSumBits = 0x4B400000;
constexpr float kSumBase = 12582912.0f;

// DPP move into the column groups (4 lanes of each 16) named by BANKS; the others keep `old`
template <int CTRL, int BANKS>
__device__ __forceinline__ uint32_t dpp_banks(uint32_t old, uint32_t src) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)src, CTRL, 0xF, BANKS, false);
}
// Column group k gets u[k] of all four column groups c, as g[c].
__device__ __forceinline__ void exchange_pieces(const uint32_t (&u)[4], uint32_t (&g)[4]) {
  const uint32_t x0 = dpp_banks<kRowRor8, 0xC>(u[0], u[2]), x1 = dpp_banks<kRowRor8, 0xC>(u[1], u[3]);
  const uint32_t y0 = dpp_banks<kRowRor8, 0x3>(u[2], u[0]), y1 = dpp_banks<kRowRor8, 0x3>(u[3], u[1]);
  g[0] = dpp_banks<kRowShr4, 0xA>(x0, x1);
  g[1] = dpp_banks<kRowShl4, 0x5>(x1, x0);
  g[2] = dpp_banks<kRowShr4, 0xA>(y0, y1);
  g[3] = dpp_banks<kRowShl4, 0x5>(y1, y0);
}
// Sum over the four column groups, shared out: column group c gets the totals of v[c][0 .. 3].  Groups 2 and 3 (the upper banks
// of a row) keep v[2] and v[3] in the first step, the odd ones the second of the two in the next: bank masks write just those,
// where the compiler's own would take 12 selects.  (No DPP move reads a register that one of the two instructions before it has
// written; the first wait covers the operands.)
__device__ __forceinline__ void reduce_scatter(const f4_t (&v)[4], float (&out)[4]) {
  float y0, y1, y2, y3;
#define BD_ADD(d, s, how, banks) "v_add_f32_dpp " d ", " s ", " s " " how " row_mask:0xf bank_mask:" banks "\n\t"
  asm("s_nop 1\n\t"
      BD_ADD("%0", "%8", "row_ror:8", "0xf") BD_ADD("%1", "%9", "row_ror:8", "0xf") BD_ADD("%2", "%10", "row_ror:8", "0xf")
      BD_ADD("%3", "%11", "row_ror:8", "0xf") BD_ADD("%4", "%12", "row_ror:8", "0xf") BD_ADD("%5", "%13", "row_ror:8", "0xf")
      BD_ADD("%6", "%14", "row_ror:8", "0xf") BD_ADD("%7", "%15", "row_ror:8", "0xf")
      BD_ADD("%0", "%16", "row_ror:8", "0xc") BD_ADD("%1", "%17", "row_ror:8", "0xc") BD_ADD("%2", "%18", "row_ror:8", "0xc")
      BD_ADD("%3", "%19", "row_ror:8", "0xc") BD_ADD("%4", "%20", "row_ror:8", "0xc") BD_ADD("%5", "%21", "row_ror:8", "0xc")
      BD_ADD("%6", "%22", "row_ror:8", "0xc") BD_ADD("%7", "%23", "row_ror:8", "0xc")
      BD_ADD("%0", "%0", "row_shl:4", "0x5") BD_ADD("%1", "%1", "row_shl:4", "0x5") BD_ADD("%2", "%2", "row_shl:4", "0x5")
      BD_ADD("%3", "%3", "row_shl:4", "0x5") BD_ADD("%0", "%4", "row_shr:4", "0xa") BD_ADD("%1", "%5", "row_shr:4", "0xa")
      BD_ADD("%2", "%6", "row_shr:4", "0xa") BD_ADD("%3", "%7", "row_shr:4", "0xa")
      : "=&v"(out[0]), "=&v"(out[1]), "=&v"(out[2]), "=&v"(out[3]), "=&v"(y0), "=&v"(y1), "=&v"(y2), "=&v"(y3)
      : "v"(v[0][0]), "v"(v[0][1]), "v"(v[0][2]), "v"(v[0][3]), "v"(v[1][0]), "v"(v[1][1]), "v"(v[1][2]), "v"(v[1][3]),
        "v"(v[2][0]), "v"(v[2][1]), "v"(v[2][2]), "v"(v[2][3]), "v"(v[3][0]), "v"(v[3][1]), "v"(v[3][2]), "v"(v[3][3]));
#undef BD_ADD
}
// Nearest integer (halves up).
__device__ __forceinline__ int nearest(float x) {
  int n;
  asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(n) : "v"(x));
  return n;
}

}  // namespace
}  // namespace bd
