// Decode attention over the MXFP4 cache (Sec. IV-D(2): native low-precision matrix
// instructions on packed 4-bit data with block scales, no dequantization for QK^T), gfx950.
//
//   S^T[token, head] = sum_c K[token, c] * Q[head, c]  on v_mfma_scale_f32_16x16x128_f8f6f4:
//     A = the token's 128 e2m1 codes exactly as stored (each lane: one MX block of 32 codes,
//     16 bytes, with its e8m0 scale applied by the instruction); B = Q.  Q stays bf16 in the
//     interface; a bf16 (8 significant bits) is the exact sum of two e4m3 numbers (4 + 4 bits),
//     so B is fed as a high and a low fp8 piece with their own block scales: two MFMAs per
//     16-token tile give the exact products, accumulated in fp32.  (The paper quantizes Q to
//     fp4, Sec. II Challenge 2; keeping it exact costs one more MFMA and no ALU work.)
//   O^T[c, head] = sum_t V[t, c] * P'[t, head]  on v_mfma_f32_16x16x32_f16:
//     V's MX blocks run along channels, i.e. across the M dimension of this product, where the
//     hardware cannot apply them (it scales along the contraction).  So V codes are expanded
//     e2m1 -> fp16 with v_cvt_scalef32_pk_f16_fp4 (scale 1) and the block scale 2^e(t, c/32) is
//     folded into the probabilities instead: four variants of P', one per 32-channel block,
//     each an exact exponent shift of p.  This is the re-quantization of P that the paper
//     names as the new bottleneck of the native path (Sec. II Challenge 2); here it is 8 values
//     per lane and block thanks to the same column-group trick as the integer kernel.
//   V codes are stored channel-major inside each 128-token block (two tokens per byte), so the
//   A operand of the second product is contraction-contiguous: 16-byte loads, no transposition.
#include "bd_common.h"
#include "bd_device.h"
#include "bd_mx_token.h"

namespace bd {
namespace {

constexpr int kWaves = 4;
constexpr float kLog2e = 1.4426950408889634f;

struct MxArgs {
  const uint8_t* k_codes;
  const uint8_t* v_codes;
  const uint8_t* k_scales;
  const uint8_t* v_scales;
  const uint16_t* q;
  float* part_o;
  float* part_ml;
  void* out;   // one split only: the output [B][Hq][128], written instead of the partials; else nullptr
  int out_kind;     // element type of `out` (kOutF16 / kOutBf16 / kOutF32)
  int n_q_heads, n_kv_heads, gq;
  int length;      // tokens in the cache
  int capacity;
  int num_splits;
  float scale_log2;
  // paged cache only: block n of sequence b is page block_table[b * max_pages + n]
  const int32_t* block_table;
  const int32_t* seq_lens;
  int32_t* status;
  int max_pages, num_pages;
  int step;   // paged: 1 when this launch is the attention of a fused step
  // fused step without an append launch: the step's token ([B][Hkv][128] bf16), which the workgroup that
  // reads its block quantizes into the cache first (contiguous: at index `length`, and the kernel attends
  // length + 1 tokens; paged: at seq_lens[b], with `step`); nullptr otherwise
  const uint16_t* k_new;
  const uint16_t* v_new;
  RaiseArgs raise;   // paged
};

// Fused step: the workgroup that reads block `blk` (the one the step's token falls into; one workgroup per
// split and KV head) quantizes the token into position i of that block (array index bi) before it
// requests anything of the block.
__device__ __forceinline__ void mx_append_here(const MxArgs& a, size_t unit, size_t bi, int i) {
  if (threadIdx.x < 128)
    mx_quantize_token(a.k_new + unit * kD, a.v_new + unit * kD, const_cast<uint8_t*>(a.k_codes),
                      const_cast<uint8_t*>(a.k_scales), const_cast<uint8_t*>(a.v_codes),
                      const_cast<uint8_t*>(a.v_scales), (long)bi, i);
  workgroup_global_sync();   // read back below by other threads of this workgroup
}

struct MergeLdsMx {
  float o[kWaves][4][kD];
  float m[kWaves][4], l[kWaves][4];
};

__device__ __forceinline__ float bf2f(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// The query as the B operand of the scaled MFMA: exact split of each bf16 into two e4m3 pieces.
// P' = p * 2^(e - e_run + kPTop) goes to the second product as fp16, with e the e8m0 exponent of the token's
// channel block and e_run the largest exponent the wave has met so far (a running value, carried like the
// running maximum: the accumulators are rescaled when it grows).  So P' < 2^(kPTop + 1) whatever the
// magnitude of V is, the largest terms sit at the top of the fp16 range, and only blocks far below the
// largest one sink into the subnormals.
constexpr int kPTop = 13;
// largest byte of a u4_t, over all lanes of the wave.  Bytes are compared as the high bytes of 16-bit halves
// (packed 16-bit maxima: the odd bytes of a word as it is, the even ones after a shift by 8; whatever sits in
// the low byte of a half cannot change which high byte wins).
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
  uint32_t d;
  asm("v_pk_max_u16 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
template <int N>
__device__ __forceinline__ int wave_max_byte(const u4_t (&x)[N]) {
  uint32_t mo = 0, me = 0;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      mo = pk_max_u16(mo, x[i][d]);
      me = pk_max_u16(me, x[i][d] << 8);
    }
  uint32_t m = max(max(mo >> 24, (mo >> 8) & 0xFFu), max(me >> 24, (me >> 8) & 0xFFu));
  m = max(m, dpp_u<kQuadSwap1>(m));
  m = max(m, dpp_u<kQuadSwap2>(m));
  m = max(m, dpp_u<kRowHalfMirror>(m));
  m = max(m, dpp_u<kRowMirror>(m));
  return (int)max(max(__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 16)),
                  max(__builtin_amdgcn_readlane(m, 32), __builtin_amdgcn_readlane(m, 48)));
}
// 2^e as a float, e clamped to the normal range
__device__ __forceinline__ float pow2_clamped(int e) { return __uint_as_float((uint32_t)(min(max(e, -126), 127) + 127) << 23); }

// Operand layout of the 8-bit side (measured): lane (column, g) holds contraction indices
// 16g .. 16g+15 in bytes 0..15 and 64+16g .. 64+16g+15 in bytes 16..31, while the 4-bit
// side holds 32g .. 32g+31 per lane.  One block scale per head (all 128 channels) is used
// for B, so its value does not depend on which lane the instruction reads it from.
// qp: the head's query row + 16 * (lane / 16), or nullptr for a padding column (all zero).
// Every lane of the wave must call this (it exchanges the head's maximum across lane groups).
__device__ __forceinline__ void mx_query_operand(const uint16_t* qp, i8_t& bhi, i8_t& blo, int& sb_hi, int& sb_lo) {
  float x[32];
  u4_t raw[4] = {};
  if (qp) {
    raw[0] = *reinterpret_cast<const u4_t*>(qp);
    raw[1] = *reinterpret_cast<const u4_t*>(qp + 8);
    raw[2] = *reinterpret_cast<const u4_t*>(qp + 64);
    raw[3] = *reinterpret_cast<const u4_t*>(qp + 72);
  }
  float amax = 0.0f;
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    x[i] = bf2f((raw[i >> 3][(i >> 1) & 3] >> (16 * (i & 1))) & 0xFFFFu);
    amax = fmaxf(amax, fabsf(x[i]));
  }
  amax = fmaxf(amax, __shfl_xor(amax, 16));
  amax = fmaxf(amax, __shfl_xor(amax, 32));
  int eb = 0;
  if (amax > 0.0f) eb = (int)((__float_as_uint(amax) >> 23) & 0xFFu) - 127 - 7;   // amax * 2^-eb in [128, 256)
  eb = min(max(eb, -123), 127);
  sb_hi = eb + 127;
  sb_lo = eb - 4 + 127;
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    int hi = 0, lo = 0;
    float rem[4];
#pragma unroll
    for (int hw = 0; hw < 2; ++hw) {
      const float x0 = ldexpf(x[4 * v + 2 * hw], -eb), x1 = ldexpf(x[4 * v + 2 * hw + 1], -eb);
      hi = hw ? __builtin_amdgcn_cvt_pk_fp8_f32(x0, x1, hi, true) : __builtin_amdgcn_cvt_pk_fp8_f32(x0, x1, hi, false);
      rem[2 * hw] = x0;
      rem[2 * hw + 1] = x1;
    }
    rem[0] = (rem[0] - __builtin_amdgcn_cvt_f32_fp8(hi, 0)) * 16.0f;
    rem[1] = (rem[1] - __builtin_amdgcn_cvt_f32_fp8(hi, 1)) * 16.0f;
    rem[2] = (rem[2] - __builtin_amdgcn_cvt_f32_fp8(hi, 2)) * 16.0f;
    rem[3] = (rem[3] - __builtin_amdgcn_cvt_f32_fp8(hi, 3)) * 16.0f;
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(rem[0], rem[1], lo, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(rem[2], rem[3], lo, true);
    bhi[v] = hi;
    blo[v] = lo;
  }
}

template <int GQP>
struct MergeLdsMxG {
  float o[kWaves][GQP][kD];
  float m[kWaves][GQP], l[kWaves][GQP];
};

#define BD_RAISE false
#define BD_KERNEL(name) decode_##name##_kernel
#include "bd_mx_kernels.h"
#undef BD_RAISE
#undef BD_KERNEL
#define BD_RAISE true
#define BD_KERNEL(name) step_##name##_kernel
#include "bd_mx_kernels.h"
#undef BD_RAISE
#undef BD_KERNEL

}  // namespace

template <bool PAGED>
static hipError_t launch_mx(const MxArgs& a, int batch, hipStream_t st) {
  const dim3 block(256), grid(a.num_splits, a.n_kv_heads * ((a.gq + 15) / 16), batch);
  auto launch = [&](auto kernel, int gqp) {
    if (PAGED) kernel<<<grid, block, 0, st>>>(BD_HOT_PAGED(a, paged_grid(grid.x, grid.y, batch, false, 512, mx_waves_per_simd(gqp, PAGED), a.max_pages), batch), a);
    else   // (tokens and capacity in tokens in the places of the block counts)
      kernel<<<grid, block, 0, st>>>(a.q, a.k_codes, a.k_scales, nullptr, a.gq, a.n_kv_heads, a.num_splits, a.length, a.capacity,
                                 hot_word(0, 0, a.k_new != nullptr), a);
  };
  if (a.gq <= 4) launch(PAGED && a.raise.words ? step_mx_kernel<true> : decode_mx_kernel<PAGED>, 4);
  else if (a.gq <= 8) launch(PAGED && a.raise.words ? step_mxg_kernel<8, true> : decode_mxg_kernel<8, PAGED>, 8);
  else launch(PAGED && a.raise.words ? step_mxg_kernel<16, true> : decode_mxg_kernel<16, PAGED>, 16);
  return hipGetLastError();
}

hipError_t launch_decode_mx(const bd_cache* c, const void* q, int length, float softmax_scale, int num_splits,
                            float* part_o, float* part_ml, const void* k_new, const void* v_new, void* out,
                            hipStream_t st) {
  MxArgs a{};
  a.k_new = (const uint16_t*)k_new;
  a.v_new = (const uint16_t*)v_new;
  a.out = num_splits == 1 ? out : nullptr;
  a.out_kind = out_kind(c->format, c->out_type);
  a.k_codes = (const uint8_t*)c->k_codes;
  a.v_codes = (const uint8_t*)c->v_codes;
  a.k_scales = (const uint8_t*)c->k_params;
  a.v_scales = (const uint8_t*)c->v_params;
  a.q = (const uint16_t*)q;
  a.part_o = part_o;
  a.part_ml = part_ml;
  a.n_q_heads = c->n_q_heads;
  a.n_kv_heads = c->n_kv_heads;
  a.gq = c->n_q_heads / c->n_kv_heads;
  a.length = length;
  a.capacity = c->capacity;
  a.num_splits = num_splits;
  a.scale_log2 = softmax_scale * kLog2e;
  return launch_mx<false>(a, c->batch, st);
}

hipError_t launch_decode_mx_paged(const bd_paged_cache* c, const void* q, float softmax_scale, int num_splits,
                                  float* part_o, float* part_ml, bool step, const void* k_new, const void* v_new,
                                  void* out, hipStream_t st, void* counters) {
  MxArgs a{};
  a.k_new = (const uint16_t*)k_new;
  a.v_new = (const uint16_t*)v_new;
  a.out = num_splits == 1 ? out : nullptr;
  a.out_kind = out_kind(c->format, c->out_type);
  a.step = step ? 1 : 0;
  a.k_codes = (const uint8_t*)c->k_codes;
  a.v_codes = (const uint8_t*)c->v_codes;
  a.k_scales = (const uint8_t*)c->k_params;
  a.v_scales = (const uint8_t*)c->v_params;
  a.q = (const uint16_t*)q;
  a.part_o = part_o;
  a.part_ml = part_ml;
  a.n_q_heads = c->n_q_heads;
  a.n_kv_heads = c->n_kv_heads;
  a.gq = c->n_q_heads / c->n_kv_heads;
  a.capacity = kBlock;
  a.num_splits = num_splits;
  a.scale_log2 = softmax_scale * kLog2e;
  a.block_table = c->block_table;
  a.seq_lens = c->seq_lens;
  a.status = c->status;
  a.max_pages = c->max_pages_per_seq;
  a.num_pages = c->num_pages;
  a.raise = raise_args(c, step && a.out, (long)a.n_kv_heads * ((a.gq + 15) / 16), counters);
  const hipError_t e = launch_mx<true>(a, c->batch, st);
  return e == hipSuccess && step && a.out && !a.raise.words ? launch_paged_bump(c, st) : e;
}

}  // namespace bd
