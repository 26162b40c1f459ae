// Decode attention over int4 / int2 caches whose quantization group is smaller than the
// 128-token block (Sec. IV-C(1): K_p of shape (T_n/group, d), V_p of shape (T_n, d/group)),
// gfx950.  Same contract as the group-128 kernel (split partials (m, l, O) per query head); a
// plainer schedule, because the parameters now change inside a block:
//
//   S^T[token, head] = sum_c code[token, c] * Q'[c, head] + zq[head],  Q' = Q * s_c * log2(e) / sqrt(d).
//     s_c and z_c belong to (channel, token group), so every 16-token tile lies inside one
//     32-token chunk of the block and the B operand (Q', an fp16 high + low pair: the high piece in
//     the even copies of a head's MFMA column, the low piece in the odd ones, their partial
//     products added with one DPP move) is another one in every token group.
//   O^T[c, head] = sum_t code[t, c] * P'_g[t, head],  P'_g = p * s_(t, g) for the channel group g of
//     c: one variant of P' per channel group, each feeding the M tiles of its channels.  The
//     variants pass through LDS, which also carries them from the lanes that hold a token's
//     score (its row of S^T) to the lanes that need it as contraction index.
//   The centre of each token's codes is taken out of the second product and added back in fp32
//   with the zero terms, as in the group-128 kernel, so that fp16 rounding of P' acts on
//   centred codes.
//   Both fp16 operands are range-normalised by powers of two, so accuracy does not depend on the
//   magnitude of K, V or Q: each head's query is brought below 2^7 and a token group's K scales
//   below 2^8 before Q' is formed (undone when the first product becomes a score), and channel
//   group v's P' carries s * 2^(15 - e_run[v]) with e_run[v] the largest exponent field of the
//   group's V scales so far (accumulators rescaled when it grows, undone before the waves merge).
#include "bd_common.h"
#include "bd_device.h"
#include "bd_fmt.h"
#include "bd_quant_block.h"
#include "bd_residual.h"

namespace bd {
namespace {

constexpr int kWaves = 4;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kTwo24 = 16777216.0f;   // codes enter the MFMAs as code * 2^-24
constexpr int kGrpHeads = 8;            // query heads per workgroup, at most

struct GrpArgs {
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
  float* part_ml;   // [nparts][B][Hq][2]
  void* out;    // one split only: the output [B][Hq][128], written instead of the partials; else nullptr
  int out_kind;     // element type of `out` (kOutF16 / kOutBf16 / kOutF32)
  int n_q_heads, n_kv_heads, gq;
  int nb, nbcap, res_len, num_splits;
  float scale_log2; // softmax_scale * log2(e)
  uint32_t res_scale;   // residual_scale(num_splits)
  // paged cache: block n of sequence b is page block_table[b][n], pool index page * Hkv + head;
  // nb and res_len then come from seq_lens[b]
  const int32_t* block_table;
  const int32_t* seq_lens;
  int32_t* status;
  int max_pages, num_pages;
  int step;   // paged: 1 when this launch is the attention of a fused step
  // Contiguous cache, fused step whose token fills the residual block: as in the group-128 kernel
  // (kFlushFirst: the workgroup that reads block flush_blk packs it first; kFlushAfter: the step attends the
  // 128 fp16 rows and one extra workgroup per KV head, blockIdx.x == 0, packs them)
  int flush_mode, flush_blk;
  int batch;
  RaiseArgs raise;   // paged
};

// Q' of K by channel: QB token groups at a time, per head the high fp16 pieces and the low ones, in B-operand slot order
// (rows here and of P' padded by 16 bytes: lanes of different heads read the same offset of their
// rows, and rows a multiple of 256 bytes apart would all fall on the same LDS banks)
template <int GQP, int QB>
struct GrpQueries {
  uint16_t q[QB][2][GQP][kD + 8];
  float zq[QB][GQP];           // sum_c Q_c z_c of the token group
  float ksb[QB][GQP];          // what turns the first product into scores (undoes the range normalisation of Q')
};
template <int GQP, int NV, int QB, bool KT>
struct GrpWaveLds {
  float2 vpar[NV][kParSlots];  // per (channel group, token): (scale * position factor, zero + scale * centre code)
  uint16_t c16[NV][kBlock];    // centre code * position factor, in A-operand slot order
  union {                      // Q' is used up before P' is made
    GrpQueries<GQP, QB> qs;
    uint16_t pbuf[GQP][kBlock + 8];   // P' of the channel group in work, in B-operand slot order
  };
};
template <int GQP, int NV, int QB>
struct GrpWaveLds<GQP, NV, QB, true> {
  __attribute__((aligned(16))) uint16_t zeros[8];   // what a lane outside a chain's channel group feeds the matrix unit
  uint16_t qhi[GQP][kD + 8];   // Q' per head, high fp16 piece, in B-operand slot order
  uint16_t qlo[GQP][kD + 8];   // low piece
  float2 vpar[NV][kParSlots];
  uint16_t c16[NV][kBlock];
  uint16_t pbuf[GQP][kBlock + 8];
  // K parameters (scale * 2^24, zero) per (channel group, token) of the block, and per head the sums of the
  // (normalised, scaled) query over each channel group
  float2 ktpar[NV][kParSlots];
  float qsum[GQP][NV];
};
template <int GQP, int NV>
struct GrpMergeLds {
  float o[kWaves][GQP][kD];
  float m[kWaves][GQP], l[kWaves][GQP], z[kWaves][GQP][NV];
};

constexpr size_t gmax(size_t x, size_t y) { return x > y ? x : y; }

#define BD_RAISE false
#define BD_KERNEL(name) decode_##name##_kernel
#include "bd_grp_kernel.h"
#undef BD_RAISE
#undef BD_KERNEL
#define BD_RAISE true
#define BD_KERNEL(name) step_##name##_kernel
#include "bd_grp_kernel.h"
#undef BD_RAISE
#undef BD_KERNEL

template <int BITS, int G, int GQP, bool KT>
void launch_mode(const GrpArgs& a, bool paged, dim3 grid, hipStream_t st) {
  if (paged) {
    const PagedGrid g = paged_grid(grid.x, grid.y, grid.z, a.flush_mode != kFlushNone, INT32_MAX, grp_waves_per_simd(BITS, G, GQP, KT), a.max_pages);
    if (a.raise.words) step_grp_kernel<BITS, G, GQP, true, KT><<<dim3(g.x, g.y, g.z), dim3(256), 0, st>>>(BD_HOT_PAGED(a, g, (int)grid.z), a);
    else decode_grp_kernel<BITS, G, GQP, true, KT><<<dim3(g.x, g.y, g.z), dim3(256), 0, st>>>(BD_HOT_PAGED(a, g, (int)grid.z), a);
  } else {
    decode_grp_kernel<BITS, G, GQP, false, KT><<<grid, dim3(256), 0, st>>>(BD_HOT_CONTIGUOUS(a), a);
  }
}

template <int BITS, int G, bool KT = false>
void launch_heads(const GrpArgs& a, bool paged, dim3 grid, hipStream_t st) {
  if (a.gq <= 4) launch_mode<BITS, G, 4, KT>(a, paged, grid, st);
  else launch_mode<BITS, G, 8, KT>(a, paged, grid, st);
}

hipError_t launch_format(int format, const GrpArgs& a, bool paged, int batch, hipStream_t st) {
  dim3 grid(a.num_splits + (!paged && a.flush_mode == kFlushAfter ? 1 : 0), a.n_kv_heads * ((a.gq + kGrpHeads - 1) / kGrpHeads), batch);
  switch (format) {
    case BD_FMT_INT4_G64: launch_heads<4, 64>(a, paged, grid, st); break;
    case BD_FMT_INT4_G32: launch_heads<4, 32>(a, paged, grid, st); break;
    case BD_FMT_INT2_G64: launch_heads<2, 64>(a, paged, grid, st); break;
    case BD_FMT_INT2_G32: launch_heads<2, 32>(a, paged, grid, st); break;
    case BD_FMT_INT4_KT_G64: launch_heads<4, 64, true>(a, paged, grid, st); break;
    case BD_FMT_INT4_KT_G32: launch_heads<4, 32, true>(a, paged, grid, st); break;
    case BD_FMT_INT2_KT_G64: launch_heads<2, 64, true>(a, paged, grid, st); break;
    case BD_FMT_INT2_KT_G32: launch_heads<2, 32, true>(a, paged, grid, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_grp(const bd_cache* c, const void* q, int packed_len, int res_len, float softmax_scale,
                             int num_splits, float* part_o, float* part_ml, const void* k_new, const void* v_new,
                             void* out, hipStream_t st, int flush) {
  GrpArgs a;
  a.k_new = (const uint16_t*)k_new;
  a.v_new = (const uint16_t*)v_new;
  // flush 1: the step's token fills the residual block, which this launch packs first (packed_len counts it,
  // res_len is 0); flush 2: ... which this launch attends in fp16 (res_len is 128) and packs as well
  a.flush_mode = flush == 1 ? kFlushFirst : flush == 2 ? kFlushAfter : kFlushNone;
  a.flush_blk = flush == 1 ? packed_len / kBlock - 1 : packed_len / kBlock;
  a.new_slot = k_new && flush != 1 ? res_len - 1 : -1;
  a.out = num_splits == 1 ? out : nullptr;
  a.out_kind = out_kind(c->format, c->out_type);
  a.k_codes = (const uint32_t*)c->k_codes;
  a.v_codes = (const uint32_t*)c->v_codes;
  a.k_params = (const uint32_t*)c->k_params;
  a.v_params = (const uint32_t*)c->v_params;
  a.k_res = (const uint16_t*)c->k_res;
  a.v_res = (const uint16_t*)c->v_res;
  a.q = (const uint16_t*)q;
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
  a.max_pages = a.num_pages = a.step = 0;
  return launch_format(c->format, a, false, c->batch, st);
}

hipError_t launch_decode_grp_paged(const bd_paged_cache* c, const void* q, float softmax_scale, int num_splits,
                                   float* part_o, float* part_ml, bool step, const void* k_new, const void* v_new,
                                   void* out, hipStream_t st, bool lazy, void* counters) {
  GrpArgs a;
  a.k_new = (const uint16_t*)k_new;   // non-null: the step's token, which this launch appends itself
  a.v_new = (const uint16_t*)v_new;
  a.new_slot = -1;
  a.out = num_splits == 1 ? out : nullptr;
  a.out_kind = out_kind(c->format, c->out_type);
  a.k_codes = (const uint32_t*)c->k_codes;
  a.v_codes = (const uint32_t*)c->v_codes;
  a.k_params = (const uint32_t*)c->k_params;
  a.v_params = (const uint32_t*)c->v_params;
  a.k_res = (const uint16_t*)c->k_res;
  a.v_res = (const uint16_t*)c->v_res;
  a.q = (const uint16_t*)q;
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
  a.step = step ? 1 : 0;
  a.flush_mode = lazy ? kFlushAfter : kFlushNone;   // (as in launch_decode_paged)
  a.flush_blk = 0;
  a.raise = raise_args(c, step && a.out, (long)a.n_kv_heads * ((a.gq + kGrpHeads - 1) / kGrpHeads) * (lazy ? 2 : 1), counters);
  const hipError_t e = launch_format(c->format, a, true, c->batch, st);
  return e == hipSuccess && step && a.out && !a.raise.words ? launch_paged_bump(c, st) : e;
}

}  // namespace bd
