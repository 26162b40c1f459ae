// Decode-step attention over the packed int4 / int2 cache: the paper's Packing Kernel
// (Sec. IV-C: fused dequantize + QK^T + softmax + PV) and the attention half of its
// Residual Kernel (Sec. IV-B), split over the context, for gfx950.
//
// How the contraction is mapped onto v_mfma_f32_16x16x32_f16 (wave64; A and B operands hold,
// per lane, 8 contraction-contiguous fp16 for row/column lane%16; the fp32 result holds rows
// 4*(lane/16)+r, r = 0..3, of column lane%16):
//
//   S^T[token, head] = sum_c K[token, c] * Q'[head, c]      A = K codes (M = 16 tokens),
//                                                           B = Q'^T (N = query group, padded to 16)
//   O^T[c, head]     = sum_t V[t, c] * P'[t, head]          A = V codes^T (M = 16 channels),
//                                                           B = P' (contraction over tokens)
//
// The query group of one KV head forms the N dimension (query transformation, Sec. IV-A).
// Because S^T comes out with 4 consecutive rows (tokens) per lane for one head, it is already
// in the B-operand layout of the second product: probabilities go exp -> fp16 -> MFMA without
// an LDS round trip.  The row -> token assignment of each S^T tile and the order of codes
// inside a word are chosen so that this holds (the analogue, for MFMA, of inducing the packed
// layout from the consumer instruction, Sec. III-A(1)).
//
// Query groups of up to 4 heads have the 16 columns for four parts of each number, part k of head h in column 4 k + h:
// * Q' in fixed point, 30 bits from the head's largest of the block down, as four signed bytes, on v_mfma_i32_16x16x64_i8 with
//   the codes as bytes (masking again, bd_fmt.h): two instructions of 16 cycles contract the 128 channels of a 16-token tile in
//   exact integers.
// * P' as a sum of e4m3 pieces, 2^-5 apart, on v_mfma_scale_f32_16x16x128_f8f6f4: one instruction of 32 cycles for the 128
//   tokens of a 16-channel tile.  Every product of codes and pieces is exact, and the instruction adds to its accumulator as
//   fp32 does (measured: 1e-7 of the larger of the two).
// The parts' partial scores are added over the column groups with DPP moves, column group c keeping tiles c and 4 + c (8
// values per lane per block, every lane doing useful work); the pieces of the weights are exchanged between the column
// groups likewise, and the column groups' partial O^T are added once, after the loop.
//
// The bytes hold the 22-bit product q * scale whole down to 2^-8 of the head's largest in the block (2-bit codes: odd channels
// 2^-6); smaller ones are rounded at 2^-30 (2^-28) of that largest.  Where that may show in the scores, a second four bytes hold
// what the rounding took, down to 2^-60, and the block's keys are multiplied by those as well (FmtI8, kFineScore, has the rule:
// one key of 10^4 among others of 1 makes its channel's products the largest of the block while the other tokens' codes
// there are 0).  Relative L2 error of fp32 outputs, against 64 bits, seven e4m3 pieces (two
// f8f6f4 instructions of 32 cycles a tile; the pieces' conversions take 8 cycles each, 52 a block) / bytes: 2048 tokens of
// normal keys 8.7e-7 / 8.6e-7, 2 bits 7.9e-7 / 4.4e-7; one key a block of 10^3 .. 6 * 10^4 with a query of -30 there 8.2e-7 /
// 7.7e-7, 2 bits 7.5e-7 / 6.0e-7 (without the second four 3e-6 .. 2e-4, 2 bits 2e-5 .. 1e-3); an outlier channel in q that is
// not K's, x 30 .. x 1000, 9e-7 .. 2e-6 either way.  A step, seven pieces / bytes (the eight waves of wide_int_kernel and the
// present merge included): 4 bits, 1K tokens 7.9 / 7.2 us, 32K 11.65 / 11.3, 128K 27.8 / 27.0; 2 bits, 8 x 32K 31.1 / 29.2.
// fp32 outputs are 4e-7 .. 5e-7 off at 4096 tokens, with fp16 weights 1.8e-4 .. 2.2e-4.
// Groups of 5 .. 16 heads have no columns to spare for the pieces and stay on fp16.
//
// Groups of 5 .. 16 heads carry the heads twice or once over the 16 columns (column c holds head c % GQP).
//
// Dequantization is reduced to masking (Sec. III-A(3) uses lop3 to the same end):
//   * a masked code sitting in the low bits of an fp16 lane IS the fp16 subnormal code * 2^-24
//     (times a power of two when it sits at bit 4..7); gfx950's MFMA takes subnormal inputs
//     exactly, so the MFMAs consume  word & mask  directly: 5 ALU ops per 8 int4 codes,
//     9 per 16 int2 codes; the power-of-two factors are folded into Q' / P'.
//   * K is quantized per channel, so  S = sum_c (Q_c s_c) code_c + sum_c Q_c z_c : the query is
//     rescaled once per 128-token block and the zero term is one scalar per head and block.
//     Q' = Q*s, 22 bits, is carried whole, as an fp16 high + low pair (two MFMAs on the same A
//     operand) or in bytes: a single fp16 Q' is not enough when a channel holds outliers.
//   * V is quantized per token, so  O = sum_t (P_t s_t) code_t + sum_t P_t z_t.
//   * Raw codes are offset by the token's zero-point, so sum_t P'_t code_t and sum_t P_t z_t are
//     two large numbers that nearly cancel; the fp16 rounding of P' and the last bits of two
//     separately accumulated fp32 sums would then show in the result.  Both are avoided by
//     writing  x_hat = s_t (code - c_t) + (z_t + s_t c_t)  with the integer c_t = rint(-z_t/s_t)
//     (the code of the value 0): a ninth A tile holds c_t for every token, so the same MFMA
//     chain also yields sum_t P'_t c_t, which is subtracted from every channel at the end; what
//     is left outside the MFMAs is sum_t P_t (z_t + s_t c_t), at most half a quantization step
//     per token.
//
// Range.  The fp16 operands are kept clear of overflow and of the subnormals whatever the magnitudes
// of Q, K and V are: every head's queries are scaled by a power of two to below 2^7 before they meet the
// K scales (a column of the B operand may carry any factor; it comes out of that column's scores), so
// |Q'| < 2^15 with the block's K scales normalised likewise; and the per-token V scale is folded into the exponent of the softmax,
// P'_t = 2^(S_t + log2 scale_t - m) with m the running maximum of S + log2 scale, so P' <= 1 with the
// largest term at 1, while the weights proper are P'_t / scale_t in fp32.
//
// The fp16 residual tail (Sec. IV-B) is shared out evenly over the workgroups of a
// (sequence, KV head): each takes a slice of the <= 128 residual tokens (bd_residual.h) and joins
// it to its partial in the final merge, so no workgroup does the tail alone.
#include "bd_common.h"
#include "bd_device.h"
#include "bd_fmt.h"
#include "bd_quant_block.h"
#include "bd_residual.h"

namespace bd {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kTwo24 = 16777216.0f;          // codes enter the MFMAs as code * 2^-24
constexpr float kTwoM24 = 1.0f / 16777216.0f;

struct DecodeArgs {
  const uint32_t* k_codes;
  const uint32_t* v_codes;
  const uint32_t* k_params;
  const uint32_t* v_params;
  const uint16_t* k_res;
  const uint16_t* v_res;
  const uint16_t* q;
  const uint16_t* k_new;   // fused step: the newest token, [B][Hkv][128], not yet in the residual buffers
  const uint16_t* v_new;
  int new_slot;            // its residual slot (res_len - 1), or -1 when the residual buffers are complete
  float* part_o;    // [nparts][B][Hq][128]
  float* part_ml;   // [nparts][B][Hq][2]   (running max in log2 units, running sum)
  void* out;    // one split only: the output [B][Hq][128], written instead of the partials; else nullptr
  int out_kind;     // element type of `out` (kOutF16 / kOutBf16 / kOutF32)
  int n_q_heads, n_kv_heads, gq;
  int nb;           // packed 128-token blocks
  int nbcap;
  int res_len;
  int num_splits;
  float scale_log2; // softmax_scale * log2(e)
  uint32_t res_scale;   // residual_scale(num_splits)
  // paged cache: block n of sequence b is page block_table[b][n], pool index page * Hkv + head;
  // nb and res_len then come from seq_lens[b]
  const int32_t* block_table;
  const int32_t* seq_lens;
  int32_t* status;
  int max_pages, num_pages;
  int step;            // paged: 1 when this launch is the attention of a fused step (see the kernel)
  // Contiguous cache, fused step whose token fills the residual block (Sec. IV-B(1)): the 127 rows of the
  // residual buffers plus k_new / v_new become packed block flush_blk inside this launch.
  //   kFlushFirst: block flush_blk counts as packed (nb includes it); the one workgroup that reads it
  //                quantizes it before it attends (the step is append, flush, then attention).
  //   kFlushAfter: the step attends the 128 fp16 rows (the paper's Residual Kernel: attention on the
  //                half-precision block, quantization of it in the same launch); one extra workgroup per
  //                (sequence, KV head), blockIdx.x == 0, does nothing but quantize.
  // (kFlushLast, paged: the same with the extra workgroups last, paged_grid)
  int flush_mode, flush_blk;
  int batch;
  RaiseArgs raise;   // paged
};

// Per-wave LDS scratch.  GQP = query heads per KV head, padded to 4, 8 or 16.
template <int GQP>
struct WaveLds {
  // (rows padded by 16 bytes: lanes of different heads read the same offset of their rows, and rows a
  // multiple of 256 bytes apart would all fall on the same LDS banks)
  uint16_t qhi[GQP][kD + 8];   // Q' per head, high fp16 piece, in B-operand slot order
  uint16_t qlo[GQP][kD + 8];   // low piece
  float4 vpar[kParSlots];  // per V token of the block: (log2 scale, 1 / scale, value of the centre code / scale, -)
  float2 kpar[kParSlots];  // per-token K only: (scale * 2^24, zero) of the block's tokens
  uint16_t c16[kBlock];    // per V token: centre code * position factor, in the A-operand order of P'
  float zq[GQP];           // per head: sum_c Q_c z_c * 2^-24 (Q as normalised below)
};
// Groups of up to 4 heads: Q' as signed bytes, the B operands of two i8 instructions per tile as their lanes read them:
// [..][instruction][lane group][column = 4 * byte + head][register].  (Four columns of padding spread the lanes that prepare eight
// consecutive channels of a head over the banks.)
template <>
struct WaveLds<4> {
  uint32_t qd[2][2][4][20][4];   // [0]: of Q'; [1]: of what their rounding took
  float4 vpar[kParSlots];
  float2 kpar[kParSlots];  // per-token K only: (scale, zero)
  uint32_t c8[4][8];       // per V token: centre code as e4m3, in B-operand order ([lane group][register])
  float2 zq[4];            // per head: (sum_c Q_c z_c, what a unit of the bytes' integer is of Q')
};
// (every column's partial result, the copies of a head included; rows padded by 16 bytes: the 16 columns write the same
// offset of their rows)
template <int GQP, int WAVES>
struct MergeLds {
  float o[WAVES][16][kD + 4];
  float m[WAVES][GQP], l[WAVES][GQP], z[WAVES][GQP];
};

constexpr size_t cmax(size_t x, size_t y) { return x > y ? x : y; }

#define BD_WAVES 4
#define BD_RAISE false
#define BD_KERNEL(name) decode_##name##_kernel
#include "bd_int_kernel.h"
#undef BD_RAISE
#undef BD_KERNEL
#define BD_RAISE true
#define BD_KERNEL(name) step_##name##_kernel
#include "bd_int_kernel.h"
#undef BD_RAISE
#undef BD_KERNEL
#undef BD_WAVES
#define BD_WAVES 8
#define BD_RAISE false
#define BD_KERNEL(name) wide_##name##_kernel
#include "bd_int_kernel.h"
#undef BD_WAVES
#undef BD_RAISE
#undef BD_KERNEL

// Log-sum-exp merge of the split partials into the final output rows (fp16 or bf16).
// One workgroup per output row: 128 channels x kGroups interleaved groups of partials.  The
// kernel is pure latency (a few hundred KB in total), so every thread issues all its loads at
// once -- up to kBatch partials per round, one round for up to kGroups * kBatch partials -- and
// merges them with a running maximum; the groups meet in LDS.
constexpr int kCombineGroups = 8, kCombineBatch = 8;
// Fused step of a paged cache: the merge is the last kernel of the step, so it also raises the
// length of every sequence whose token was appended (same test as the append kernel).
struct StepBump {
  int32_t* seq_lens;            // nullptr: nothing to raise
  const int32_t* block_table;
  int n_q_heads, max_pages, num_pages;
  int every_token;              // a page is needed by every token (MXFP4), not only by the 128th
};

template <int G>
__global__ __launch_bounds__(128 * G) void combine_kernel(const float* __restrict__ part_o,
                                                           const float* __restrict__ part_ml,
                                                           int nparts, int nrows,
                                                           void* __restrict__ out, int kind, StepBump bump) {
  constexpr int kBatch = kCombineBatch;
  __shared__ float sm[G][128], sl[G][128], so[G][128];
  const int row = blockIdx.x, tid = threadIdx.x, c = tid & 127, grp = tid >> 7;
  float M = -INFINITY, L = 0.f, o = 0.f;
  float2 ml[kBatch];
  float ov[kBatch];
  auto request = [&](int p0) {
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int p = p0 + G * i;
      const size_t r = (size_t)(p < nparts ? p : 0) * nrows + row;
      ml[i] = *reinterpret_cast<const float2*>(part_ml + r * 2);
      ov[i] = part_o[r * kD + c];
    }
  };
  request(grp);
  // one thread per sequence (here, with the partials on their way: its arguments are not among the preloaded ones)
  if (bump.seq_lens && tid == 128 * G - 1 && row % bump.n_q_heads == 0) {
    const int b = row / bump.n_q_heads;
    raise_length(bump.seq_lens, bump.block_table, b, bump.max_pages, bump.num_pages, bump.every_token != 0);
  }
  for (int p0 = grp; p0 < nparts; p0 += G * kBatch) {
    if (p0 != grp) request(p0);
#pragma unroll
    for (int i = 0; i < kBatch; ++i)
      if (p0 + G * i >= nparts) ml[i].x = -INFINITY;
    // (all weights relative to the round's maximum: a chain of running maxima and rescalings is 8 times as long and has twice
    // the exponentials: a step of 4 x 4000 tokens 8.74 -> 8.63 us, 32K 11.19 -> 11.12, one head of 64K 10.12 -> 9.95)
    float Mn = M;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) Mn = fmaxf(Mn, ml[i].x);
    const float base = Mn > -INFINITY ? Mn : 0.0f;   // (nothing so far: all weights 0)
    const float fo = __builtin_amdgcn_exp2f(M - base);
    L *= fo;
    o *= fo;
    M = Mn;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const float fn = __builtin_amdgcn_exp2f(ml[i].x - base);
      L = __builtin_fmaf(fn, ml[i].y, L);
      o = __builtin_fmaf(fn, ov[i], o);
    }
  }
  sm[grp][c] = M;
  sl[grp][c] = L;
  so[grp][c] = o;
  __syncthreads();
  if (tid < 128) {
    float Mt = sm[0][c];
#pragma unroll
    for (int g = 1; g < G; ++g) Mt = fmaxf(Mt, sm[g][c]);
    float res = 0.f;
    if (Mt > -INFINITY) {
      float Lt = 0.f, ot = 0.f;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float Mg = sm[g][c];
        const float f = Mg > -INFINITY ? __builtin_amdgcn_exp2f(Mg - Mt) : 0.f;
        Lt += f * sl[g][c];
        ot += f * so[g][c];
      }
      res = Lt > 0.f ? ot / Lt : 0.f;
    }
    const size_t idx = (size_t)row * kD + c;
    if (kind == kOutF32) reinterpret_cast<float*>(out)[idx] = res;
    else reinterpret_cast<uint16_t*>(out)[idx] = kind == kOutBf16 ? f2bf(res) : f2h(res);
  }
}

}  // namespace

namespace {

template <int BITS, int GQP, bool KT>
void launch_mode(int blocks, bool paged, const DecodeArgs& a, dim3 grid, dim3 block, hipStream_t st) {
  if (paged) {
    const PagedGrid g = paged_grid(grid.x, grid.y, grid.z, a.flush_mode != kFlushNone, INT32_MAX, 2, a.max_pages);
    if (a.raise.words) step_int_kernel<BITS, GQP, kManyBlocks, true, KT><<<dim3(g.x, g.y, g.z), block, 0, st>>>(BD_HOT_PAGED(a, g, (int)grid.z), a);
    else decode_int_kernel<BITS, GQP, kManyBlocks, true, KT><<<dim3(g.x, g.y, g.z), block, 0, st>>>(BD_HOT_PAGED(a, g, (int)grid.z), a);
  } else if (blocks == kOneBlockWide) {
    if constexpr (GQP == 4 && !KT) wide_int_kernel<BITS, GQP, kOneBlockWide, false, KT><<<grid, dim3(512), 0, st>>>(BD_HOT_CONTIGUOUS(a), a);
  } else if (blocks == kOneBlock) {
    decode_int_kernel<BITS, GQP, kOneBlock, false, KT><<<grid, block, 0, st>>>(BD_HOT_CONTIGUOUS(a), a);
  } else if (blocks == kOneBlockSlice) {
    decode_int_kernel<BITS, GQP, kOneBlockSlice, false, KT><<<grid, block, 0, st>>>(BD_HOT_CONTIGUOUS(a), a);
  } else {
    decode_int_kernel<BITS, GQP, kManyBlocks, false, KT><<<grid, block, 0, st>>>(BD_HOT_CONTIGUOUS(a), a);
  }
}

template <int BITS, bool KT>
void launch_group(int gq, int blocks, bool paged, const DecodeArgs& a, dim3 grid, dim3 block, hipStream_t st) {
  if (gq <= 4) launch_mode<BITS, 4, KT>(blocks, paged, a, grid, block, st);
  else if (gq <= 8) launch_mode<BITS, 8, KT>(blocks, paged, a, grid, block, st);
  else launch_mode<BITS, 16, KT>(blocks, paged, a, grid, block, st);
}

// picks the kernel instance: format, query group padded to 4 / 8 / 16 heads, loop structure
void launch_instance(int format, int gq, int blocks, bool paged, const DecodeArgs& a, dim3 grid, dim3 block,
                     hipStream_t st) {
  switch (format) {
    case BD_FMT_INT4: launch_group<4, false>(gq, blocks, paged, a, grid, block, st); break;
    case BD_FMT_INT2: launch_group<2, false>(gq, blocks, paged, a, grid, block, st); break;
    case BD_FMT_INT4_KT: launch_group<4, true>(gq, blocks, paged, a, grid, block, st); break;
    default: launch_group<2, true>(gq, blocks, paged, a, grid, block, st); break;
  }
}

}  // namespace

hipError_t launch_decode_int(const bd_cache* c, const void* q, int packed_len, int res_len, float softmax_scale,
                             int num_splits, float* part_o, float* part_ml, const void* k_new, const void* v_new,
                             void* out, hipStream_t st, int flush) {
  DecodeArgs a;
  a.out = num_splits == 1 ? out : nullptr;
  a.out_kind = out_kind(c->format, c->out_type);
  a.k_codes = (const uint32_t*)c->k_codes;
  a.v_codes = (const uint32_t*)c->v_codes;
  a.k_params = (const uint32_t*)c->k_params;
  a.v_params = (const uint32_t*)c->v_params;
  a.k_res = (const uint16_t*)c->k_res;
  a.v_res = (const uint16_t*)c->v_res;
  a.q = (const uint16_t*)q;
  a.k_new = (const uint16_t*)k_new;
  a.v_new = (const uint16_t*)v_new;
  // flush 1: the step's token fills the residual block, which this launch packs first (packed_len counts it,
  // res_len is 0); flush 2: ... which this launch attends in fp16 (res_len is 128) and packs as well
  a.flush_mode = flush == 1 ? kFlushFirst : flush == 2 ? kFlushAfter : kFlushNone;
  a.flush_blk = flush == 1 ? packed_len / kBlock - 1 : packed_len / kBlock;
  a.new_slot = k_new && flush != 1 ? res_len - 1 : -1;
  a.part_o = part_o;
  a.part_ml = part_ml;
  a.batch = c->batch;
  a.raise = {nullptr, 0};
  a.n_q_heads = c->n_q_heads;
  a.n_kv_heads = c->n_kv_heads;
  a.gq = c->n_q_heads / c->n_kv_heads;
  a.nb = packed_len / kBlock;
  a.nbcap = c->capacity / kBlock;
  a.res_len = res_len;
  a.num_splits = num_splits;
  a.scale_log2 = softmax_scale * kLog2e;
  a.res_scale = residual_scale(num_splits);
  a.block_table = nullptr;
  a.seq_lens = nullptr;
  a.status = nullptr;
  a.max_pages = a.num_pages = 0;
  a.step = 0;
  dim3 grid(num_splits + (flush == 2 ? 1 : 0), c->n_kv_heads * ((a.gq + 15) / 16), c->batch), block(256);
  const int blocks = contiguous_form(a.nb, num_splits, res_len, fmt_bits(c->format), a.gq, fmt_kt(c->format), (long)grid.y * grid.z, flush == 2);
  launch_instance(c->format, a.gq, blocks, false, a, grid, block, st);
  return hipGetLastError();
}

hipError_t launch_decode_paged(const bd_paged_cache* c, const void* q, float softmax_scale, int num_splits,
                               float* part_o, float* part_ml, bool step, const void* k_new, const void* v_new,
                               void* out, hipStream_t st, bool lazy, void* counters) {
  DecodeArgs a;
  a.step = step ? 1 : 0;
  a.out = num_splits == 1 ? out : nullptr;
  a.out_kind = out_kind(c->format, c->out_type);
  a.k_codes = (const uint32_t*)c->k_codes;
  a.v_codes = (const uint32_t*)c->v_codes;
  a.k_params = (const uint32_t*)c->k_params;
  a.v_params = (const uint32_t*)c->v_params;
  a.k_res = (const uint16_t*)c->k_res;
  a.v_res = (const uint16_t*)c->v_res;
  a.q = (const uint16_t*)q;
  a.k_new = (const uint16_t*)k_new;   // non-null: the step's token, which this launch appends itself
  a.v_new = (const uint16_t*)v_new;
  a.new_slot = -1;
  // lazy: a sequence whose residual this step's token fills is attended with its 128 fp16 rows, and one extra
  // workgroup per (sequence, KV head) packs them into the sequence's next page
  a.flush_mode = lazy ? kFlushAfter : kFlushNone;
  a.flush_blk = 0;
  a.part_o = part_o;
  a.part_ml = part_ml;
  a.batch = c->batch;
  a.n_q_heads = c->n_q_heads;
  a.n_kv_heads = c->n_kv_heads;
  a.gq = c->n_q_heads / c->n_kv_heads;
  a.nb = a.nbcap = a.res_len = 0;   // per sequence, from seq_lens
  a.num_splits = num_splits;
  a.scale_log2 = softmax_scale * kLog2e;
  a.res_scale = residual_scale(num_splits);
  a.block_table = c->block_table;
  a.seq_lens = c->seq_lens;
  a.status = c->status;
  a.max_pages = c->max_pages_per_seq;
  a.num_pages = c->num_pages;
  dim3 grid(num_splits, c->n_kv_heads * ((a.gq + 15) / 16), c->batch), block(256);   // (paged_grid)
  a.raise = raise_args(c, step && a.out, (long)grid.y * (lazy ? 2 : 1), counters);
  launch_instance(c->format, a.gq, kManyBlocks, true, a, grid, block, st);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess && step && a.out && !a.raise.words ? launch_paged_bump(c, st) : e;
}

hipError_t launch_combine(const bd_cache* c, const float* part_o, const float* part_ml, int nparts, void* out,
                          hipStream_t st, const bd_paged_cache* step_of) {
  const int nrows = c->batch * c->n_q_heads;
  StepBump bump{};
  if (step_of) {
    bump.seq_lens = step_of->seq_lens;
    bump.block_table = step_of->block_table;
    bump.n_q_heads = step_of->n_q_heads;
    bump.max_pages = step_of->max_pages_per_seq;
    bump.num_pages = step_of->num_pages;
    bump.every_token = step_of->format == BD_FMT_MXFP4;
  }
  // thread groups per row: enough to request every partial in one round (8 per group), no more -- a launch of
  // 1024-thread workgroups costs about a microsecond more than one of 128-thread workgroups
  const int kind = out_kind(c->format, c->out_type);
#define BD_COMBINE(G) combine_kernel<G><<<dim3(nrows), dim3(128 * G), 0, st>>>(part_o, part_ml, nparts, nrows, out, kind, bump)
  if (nparts <= kCombineBatch) BD_COMBINE(1);
  else if (nparts <= 2 * kCombineBatch) BD_COMBINE(2);
  else if (nparts <= 4 * kCombineBatch) BD_COMBINE(4);
  else BD_COMBINE(kCombineGroups);
#undef BD_COMBINE
  return hipGetLastError();
}

}  // namespace bd
