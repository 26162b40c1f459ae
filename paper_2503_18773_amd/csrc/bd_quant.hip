// Online quantize-and-pack kernels: the quantize half of the paper's Residual Kernel
// (Sec. IV-B) and the prefill quantization (Sec. IV-B(1)).
//
// Bit-exactness contract: every stored scale, zero and code is the result of IEEE fp32
// subtract / divide / round-half-even in a fixed order, so contraction into FMAs is switched
// off for this file and no fast-math substitution is allowed.
#include "bd_common.h"
#include "bd_device.h"
#include "bd_quant_block.h"
#include "bd_mx_token.h"

#pragma clang fp contract(off)

namespace bd {
namespace {

// Copies `ntok` token rows (0 <= ntok < 128) of K and of V (PART: or of one of them), the end of a prompt, to the residual
// buffers (whole workgroup); a thread has four pieces of each tensor on the way at a time.
template <int PART>
__device__ __forceinline__ void copy_tail(const uint16_t* __restrict__ ksrc, const uint16_t* __restrict__ vsrc,
                                          uint16_t* __restrict__ kdst, uint16_t* __restrict__ vdst, int ntok) {
  const int n = ntok * (kD / 8);   // 16-byte pieces of a tensor
#pragma unroll 1
  for (int at0 = threadIdx.x; at0 < n; at0 += 4 * 256) {
    u4_t k[4], v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int at = min(at0 + 256 * i, n - 1);
      if (PART & kPartK) k[i] = reinterpret_cast<const u4_t*>(ksrc)[at];
      if (PART & kPartV) v[i] = reinterpret_cast<const u4_t*>(vsrc)[at];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (at0 + 256 * i >= n) break;
      if (PART & kPartK) reinterpret_cast<u4_t*>(kdst)[at0 + 256 * i] = k[i];
      if (PART & kPartV) reinterpret_cast<u4_t*>(vdst)[at0 + 256 * i] = v[i];
    }
  }
}

// K and V of a block go to workgroups of their own (blockIdx.z): a block's chain of loads, statistics and codes is half as
// long.  A launch in a graph, both in one workgroup / each in its own: 4 bits, 8 heads of 128 tokens 6.4 / 4.4 us, 1333 6.7 / 4.7,
// 4000 7.2 / 6.35, 6000 9.4 / 7.9, 64 of 4096 30.6 / 29.5; 2 bits 64K 55.3 / 54.1; MXFP4 128 6.1 / 4.2, 32 of 3000 12.2 / 10.9, 64 of
// 4096 29.1 / 28.8.
// With 80 registers six share a unit, with the 84 that K by channel takes unasked five.  Six while that is one round (32 of
// 3000 tokens 12.2 us, five 13.3), five past it, where six have more streams under way than the memory serves well (128K, issued
// one by one, 113.0 us, five 108.3); per-token K six always (64K 57.3, five 58.6), but five where the 80 registers do not hold it: in groups
// of 64 and 32 and in pages (in scratch, six: groups of 32, 4 of 32K 115.5 us, 2 bits 111.0, 16 of 3000 46.3; five 113.7, 108.1, 45.2,
// and scratch costs a process's first launch some 100 us).
static inline bool six_on_a_unit(bool kt, long blocks) { return kt || 2 * blocks <= 6 * 256; }
template <class Run>
__device__ __forceinline__ void run_part(Run run) {
  if (blockIdx.z == 0) run(std::integral_constant<int, kPartK>{});
  else run(std::integral_constant<int, kPartV>{});
}

// Contiguous cache: block blockIdx.x of unit blockIdx.y; the workgroups past the last whole block (tail > 0) take
// the rest of a prompt, `tail` token rows that go to the residual buffers as they are.  (A launch of its own for
// those rows cost a short prompt 3 us: 8 paged prompts of up to 1333 tokens 11.3 us each with it, 8.3 without.)
template <int BITS, bool KT, int G, int WAVES>
__global__ __launch_bounds__(256, WAVES) void quant_block_kernel(const uint16_t* __restrict__ ksrc,
                                                           const uint16_t* __restrict__ vsrc,
                                                           long src_unit_stride, int src_tok0,
                                                           uint32_t* __restrict__ k_codes,
                                                           uint32_t* __restrict__ v_codes,
                                                           uint32_t* __restrict__ k_params,
                                                           uint32_t* __restrict__ v_params, int nbcap,
                                                           int dst_blk0, uint16_t* __restrict__ k_res,
                                                           uint16_t* __restrict__ v_res, int tail) {
  const int unit = blockIdx.y, blk = blockIdx.x;
  const size_t dblk = (size_t)unit * nbcap + dst_blk0 + blk;
  const size_t src_off = (size_t)unit * src_unit_stride + ((size_t)src_tok0 + (size_t)blk * kBlock) * kD;
  if (tail > 0 && blk == (int)gridDim.x - 1) {
    const size_t res = (size_t)unit * kBlock * kD;
    run_part([&](auto part) { copy_tail<part>(ksrc + src_off, vsrc + src_off, k_res + res, v_res + res, tail); });
    return;
  }
  run_part([&](auto part) {
    quant_block_at<BITS, KT, G, part>(ksrc + src_off, vsrc + src_off, k_codes, v_codes, k_params, v_params, [&] { return (long)dblk; });
  });
}

// ---- paged cache (page = one 128-token block; pool index of (page, head) = page * H + head) ---

struct PagedArgs {
  uint32_t *k_codes, *v_codes, *k_params, *v_params;
  uint16_t *k_res, *v_res;
  const int32_t* block_table;
  int32_t* seq_lens;
  int32_t* status;
  int n_kv_heads, num_pages, max_pages;
};

// Page of block n of sequence b, or -1 (and bit `flag` of *status set) if the table has no
// valid entry for it.
__device__ __forceinline__ int page_of(const PagedArgs& a, int b, int n, int flag) {
  int page = -1;
  if (n < a.max_pages) page = a.block_table[(size_t)b * a.max_pages + n];
  if (page < 0 || page >= a.num_pages) {
    if (a.status && threadIdx.x == 0) atomicOr(a.status, flag);
    return -1;
  }
  return page;
}

// Prefill of one sequence: block blockIdx.x of KV head blockIdx.y, source [H][L][128]; the last workgroup of a head
// copies the L mod 128 newest tokens to the sequence's residual, and that of head 0 records the length.
template <int BITS, bool KT, int G, int WAVES>
__global__ __launch_bounds__(256, WAVES) void paged_quant_kernel(PagedArgs a, const uint16_t* __restrict__ ksrc,
                                                           const uint16_t* __restrict__ vsrc, int seq, int L) {
  const int blk = blockIdx.x, h = blockIdx.y;
  const size_t src_off = ((size_t)h * L + (size_t)blk * kBlock) * kD;
  if (blk == (int)gridDim.x - 1) {
    const size_t res = ((size_t)seq * a.n_kv_heads + h) * kBlock * kD;
    run_part([&](auto part) { copy_tail<part>(ksrc + src_off, vsrc + src_off, a.k_res + res, a.v_res + res, L % kBlock); });
    if (h == 0 && threadIdx.x == 0 && blockIdx.z == 0) a.seq_lens[seq] = L;
    return;
  }
  // (the page's number comes while the rows do)
  const int entry = blk < a.max_pages ? scalar_load(a.block_table + (size_t)seq * a.max_pages + blk) : -1;
  run_part([&](auto part) {
    quant_block_at<BITS, KT, G, part>(ksrc + src_off, vsrc + src_off, a.k_codes, a.v_codes, a.k_params, a.v_params, [&]() -> long {
      if (entry >= 0 && entry < a.num_pages) return (long)entry * a.n_kv_heads + h;
      if (a.status && threadIdx.x == 0) atomicOr(a.status, 2);
      return -1;
    });
  });
}

// One decode step of sequence blockIdx.y, KV head blockIdx.x: the new token row goes to residual
// slot len mod 128; if that fills the residual it is quantized into the sequence's next page
// (Sec. IV-B(1)).  Lengths are bumped by paged_bump_kernel afterwards, so every workgroup of
// the sequence sees the same length here.
template <int BITS, bool KT, int G>
__global__ __launch_bounds__(256) void paged_append_kernel(PagedArgs a, const uint16_t* __restrict__ k_new,
                                                            const uint16_t* __restrict__ v_new) {
  const int h = blockIdx.x, b = blockIdx.y;
  const int len = a.seq_lens[b];
  if (len < 0) return;
  const int nb = len / kBlock, r = len % kBlock;
  const size_t unit = (size_t)b * a.n_kv_heads + h;
  int page = 0;
  if (r == kBlock - 1) {
    page = page_of(a, b, nb, 2);
    if (page < 0) return;   // the token is dropped; the length stays
  }
  uint16_t* kr = a.k_res + unit * kBlock * kD;
  uint16_t* vr = a.v_res + unit * kBlock * kD;
  if (threadIdx.x < 32) {
    const bool is_v = threadIdx.x >= 16;
    const int c8 = 8 * (threadIdx.x & 15);
    const u4_t val = *reinterpret_cast<const u4_t*>((is_v ? v_new : k_new) + unit * kD + c8);
    *reinterpret_cast<u4_t*>((is_v ? vr : kr) + (size_t)r * kD + c8) = val;
  }
  if (r != kBlock - 1) return;
  // the row just written is read back below by other threads of this workgroup
  __threadfence();
  __syncthreads();
  quant_block<BITS, KT, G>(kr, vr, a.k_codes, a.v_codes, a.k_params, a.v_params, (size_t)page * a.n_kv_heads + h);
}

// seq_lens[b] += 1 for every sequence whose step went through (same test as the append kernel).
__global__ void paged_bump_kernel(PagedArgs a, int batch, bool every_token) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= batch) return;
  raise_length(a.seq_lens, a.block_table, b, a.max_pages, a.num_pages, every_token);
}

// Copies `ntok` token rows of K and of V between [unit][token][128] arrays of 16-bit values (an append: one row).
__global__ __launch_bounds__(256) void copy_rows_kernel(const u4_t* __restrict__ ksrc,
                                                         const u4_t* __restrict__ vsrc, long src_unit_stride,
                                                         int src_tok0, u4_t* __restrict__ kdst,
                                                         u4_t* __restrict__ vdst, long dst_unit_stride,
                                                         int dst_tok0, int ntok) {
  const int unit = blockIdx.x;
  const size_t so = ((size_t)unit * src_unit_stride + (size_t)src_tok0 * kD) / 8;
  const size_t dn = ((size_t)unit * dst_unit_stride + (size_t)dst_tok0 * kD) / 8;
  const int n = ntok * (kD / 8);
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    kdst[dn + i] = ksrc[so + i];
    vdst[dn + i] = vsrc[so + i];
  }
}

// ---- MXFP4 -------------------------------------------------------------------------------

// Where the 128-token blocks of an MXFP4 launch go: block `blk` of unit `u` is block
// u * nbcap + blk of the arrays (contiguous cache), or, for one sequence of a paged cache, block
// page * H + u with page = table_row[blk] (u = KV head).  -1 (and bit 1 of *status) if the table has
// no valid page for it.  Inside a block: K codes [128][64], scales [128][4], V codes [128 ch][64].
struct MxDst {
  uint8_t *k_codes, *k_scales, *v_codes, *v_scales;
  int nbcap;
  const int32_t* table_row;
  int32_t* status;
  int n_kv_heads, num_pages, max_pages;
};
// (entry: the table's for that block, -1 past its end)
__device__ __forceinline__ int mx_table_entry(const MxDst& d, int blk) {
  return d.table_row && blk < d.max_pages ? scalar_load(d.table_row + blk) : -1;
}
__device__ __forceinline__ long mx_block_index(const MxDst& d, int u, int blk, int entry) {
  if (!d.table_row) return (long)u * d.nbcap + blk;
  if (entry < 0 || entry >= d.num_pages) {
    if (d.status && threadIdx.x == 0) atomicOr(d.status, 2);
    return -1;
  }
  return (long)entry * d.n_kv_heads + u;
}

// Prefill of an MXFP4 cache, two workgroups per 128-token block (K and V), in the tiling of the integer block
// quantizer: 256 threads, a thread holds 8 token rows x 8 consecutive channels of each tensor (one 16-byte
// load per row; 16 lanes per token row, so every load of a wave covers 1 KB of contiguous source and the
// four lanes of a DPP quad hold one MX group).  K rows are four apart inside the wave's 32 tokens, so that
// one store of the wave covers four consecutive token rows of codes; V rows are consecutive: a channel's
// 8 tokens are one 32-bit word of the channel-major block layout, which is the 4-bit integer layout
// (transposed in registers, put in address order through an LDS tile, stored 16 bytes at a time).
// The group maximum is taken on the bf16 magnitudes as loaded (packed 16-bit maxima, then the quad);
// codes come from v_cvt_scalef32_pk_fp4_f32 (nearest e2m1, ties to the even code, saturating: measured
// identical to the definition) except that it keeps the sign of values that round to zero, which is
// cleared afterwards; groups with a very small maximum (shared exponent below -120, where elements can be
// fp32 subnormals) take the explicit path.  Source rows and codes are streaming (non-temporal) accesses.
// TAIL: the block holds only `ntok` < 128 tokens (the end of a prompt).  Rows past them are neither read nor
// written, and V's bytes past them stay as they are (an odd last token's byte gets a zero high nibble).  (A
// kernel of its own with a thread per token -- 128 values in turn, 47 us for 31 tokens -- served this block
// before, whatever the prompt's length: 57.5 us for 4 prompts of 2079 tokens.)
// place(): the block's index in the arrays, asked for when the rows are on their way; negative: nowhere.
template <bool TAIL, int PART, class Place>
__device__ __forceinline__ void mx_quant_block(const uint16_t* __restrict__ ksrc, const uint16_t* __restrict__ vsrc,
                                               size_t src_blk, const MxDst& d, Place place, int ntok,
                                               uint32_t (*vw)[kBlock / 8 + 1]) {
  constexpr int C = 8, T = 8, NCG = kD / C, WPC = kBlock / 8;   // 16 lanes per row; 16 words per channel
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cg = tid % NCG, tg = tid / NCG;
  auto krow = [&](int t) { return 32 * wave + (lane >> 4) + 4 * t; };
  auto vrow = [&](int t) { return T * tg + t; };
  auto live = [&](int row) { return !TAIL || row < ntok; };
  const uint16_t* src = PART == kPartK ? ksrc : vsrc;
  u4_t raw[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int row = PART == kPartK ? krow(t) : vrow(t);
    raw[t] = (u4_t){0u, 0u, 0u, 0u};
    if (live(row)) raw[t] = __builtin_nontemporal_load(reinterpret_cast<const u4_t*>(src + src_blk + (size_t)row * kD + C * cg));
  }
  const long bi = place();
  if (bi < 0) return;

  // the 8 codes of one row of this lane (channel C*cg + n at nibble n) and the group's scale byte
  auto row_codes = [&](const u4_t& raw, uint32_t& word, uint32_t& ebyte) {
    typedef unsigned short us2_t __attribute__((ext_vector_type(2)));
    us2_t m2 = {0, 0};
#pragma unroll
    for (int w = 0; w < 4; ++w) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(us2_t, raw[w] & 0x7FFF7FFFu));
    uint32_t mag = m2[0] > m2[1] ? m2[0] : m2[1];   // bf16 bits of the largest magnitude of this lane's 8 values
    mag = max(mag, dpp_u<kQuadSwap1>(mag));
    mag = max(mag, dpp_u<kQuadSwap2>(mag));        // ... of the MX group (the quad)
    int e = 0;
    if (mag != 0) {
      e = (int)(mag >> 7) - 127 - 2;   // floor(log2 amax) - 2 from the exponent field
      e = e < -127 ? -127 : e;
    }
    uint32_t c = 0;
    if (mag != 0) {
      if (e >= -120) {
        const float scale = __uint_as_float((uint32_t)(e + 127) << 23);
#define BD_CVT_PAIR(b)                                                                                          \
  c = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c, __uint_as_float(raw[b] << 16), __uint_as_float(raw[b] & 0xFFFF0000u), \
                                               scale, b)
        BD_CVT_PAIR(0);
        BD_CVT_PAIR(1);
        BD_CVT_PAIR(2);
        BD_CVT_PAIR(3);
#undef BD_CVT_PAIR
        // a value that rounds to zero is stored as +0: drop the sign of nibbles with no magnitude
        const uint32_t m = c & 0x77777777u;
        c = (((m + 0x77777777u) & c) & 0x88888888u) | m;
      } else {
#pragma unroll
        for (int n = 0; n < 8; ++n) {
          const uint32_t r = raw[n >> 1];
          const float x = __uint_as_float((n & 1) ? (r & 0xFFFF0000u) : (r << 16));
          c |= e2m1_code(x, e) << (4 * n);
        }
      }
    }
    word = c;
    ebyte = (uint32_t)(e + 127);
  };
  // the four scale bytes of a token row, gathered in the row's first lane
  auto row_scales = [&](uint32_t ebyte) {
    return ebyte | (dpp_u<kRowShl4>(ebyte) << 8) | (dpp_u<kRowShl8>(ebyte) << 16) | (dpp_u<kRowShl12>(ebyte) << 24);
  };

  // ---- K: token-major codes, one word per lane and row
  if constexpr (PART == kPartK) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
      uint32_t word, ebyte;
      row_codes(raw[t], word, ebyte);
      const size_t tok = (size_t)bi * kBlock + krow(t);
      const uint32_t sc4 = row_scales(ebyte);
      if (live(krow(t))) {
        __builtin_nontemporal_store(word, reinterpret_cast<uint32_t*>(d.k_codes + tok * (kD / 2)) + cg);
        if (cg == 0) *reinterpret_cast<uint32_t*>(d.k_scales + tok * 4) = sc4;
      }
    }
    return;
  }
  // ---- V: channel-major codes
  uint32_t lo[T], hi[T];   // per token: the codes of channels 0..3 / 4..7 of this lane, one per byte
#pragma unroll
  for (int t = 0; t < T; ++t) {
    uint32_t word, ebyte;
    row_codes(raw[t], word, ebyte);
    const size_t tok = (size_t)bi * kBlock + vrow(t);
    const uint32_t sc4 = row_scales(ebyte);
    if (cg == 0 && live(vrow(t))) *reinterpret_cast<uint32_t*>(d.v_scales + tok * 4) = sc4;
    const uint32_t x = word & 0x0F0F0F0Fu, y = (word >> 4) & 0x0F0F0F0Fu;   // even / odd channels, one per byte
    lo[t] = __builtin_amdgcn_perm(y, x, 0x05010400u);   // x.b0 y.b0 x.b1 y.b1
    hi[t] = __builtin_amdgcn_perm(y, x, 0x07030602u);   // x.b2 y.b2 x.b3 y.b3
  }
  uint32_t words[C];   // channel c: its 8 tokens' codes, token t at nibble t
  transpose_code_bytes<4>(lo, words);
  transpose_code_bytes<4>(hi, words + 4);
#pragma unroll
  for (int c = 0; c < C; ++c) vw[C * cg + c][tg] = words[c];
  __syncthreads();
  uint32_t* vdst = reinterpret_cast<uint32_t*>(d.v_codes) + (size_t)bi * (kD * WPC);
#pragma unroll
  for (int k = 0; k < kD * WPC / 1024; ++k) {
    const int idx = 4 * (tid + 256 * k);
    const uint32_t* row = &vw[idx / WPC][idx % WPC];
    const u4_t w4 = {row[0], row[1], row[2], row[3]};
    const int t0 = 8 * (idx % WPC);   // the 32 tokens t0 .. of channel idx / WPC
    if (live(t0 + 31)) {
      __builtin_nontemporal_store(w4, reinterpret_cast<u4_t*>(vdst + idx));
    } else {
      uint8_t* bytes = reinterpret_cast<uint8_t*>(vdst + idx);
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (t0 + 2 * j < ntok) bytes[j] = (uint8_t)(w4[j / 4] >> (8 * (j % 4)));
    }
  }
}

// Tokens [0, L) of every unit; with `seq_len` (one sequence of a paged cache) the length is recorded too.
__global__ __launch_bounds__(256, 4) void mx_quant_block_kernel(const uint16_t* __restrict__ ksrc,
                                                                 const uint16_t* __restrict__ vsrc,
                                                                 long src_unit_stride, MxDst d, int L, int32_t* seq_len) {
  const int unit = blockIdx.y, blk = blockIdx.x;
  if (seq_len && unit == 0 && blk == 0 && blockIdx.z == 0 && threadIdx.x == 0) *seq_len = L;
  const size_t src_blk = (size_t)unit * src_unit_stride + (size_t)blk * kBlock * kD;
  const int ntok = L - blk * kBlock;
  const int entry = mx_table_entry(d, blk);   // (comes while the rows do)
  auto place = [&] { return mx_block_index(d, unit, blk, entry); };
  __shared__ uint32_t vw[kD][kBlock / 8 + 1];
  run_part([&](auto part) {
    if (ntok >= kBlock) mx_quant_block<false, part>(ksrc, vsrc, src_blk, d, place, kBlock, vw);
    else mx_quant_block<true, part>(ksrc, vsrc, src_blk, d, place, ntok, vw);
  });
}

// Decode-step append for MXFP4: one token of one (sequence, KV head) goes to position i of block bi
// (mx_quantize_token, 128 threads).
__device__ __forceinline__ void mx_append_token(const uint16_t* __restrict__ k_row, const uint16_t* __restrict__ v_row,
                                                const MxDst& d, long bi, int i) {
  mx_quantize_token(k_row, v_row, d.k_codes, d.k_scales, d.v_codes, d.v_scales, bi, i);
}

// Contiguous cache: token t of every unit.
__global__ __launch_bounds__(128) void mx_append_kernel(const uint16_t* __restrict__ k_new,
                                                         const uint16_t* __restrict__ v_new, MxDst d, int t) {
  const int unit = blockIdx.x;
  mx_append_token(k_new + (size_t)unit * kD, v_new + (size_t)unit * kD, d, (long)unit * d.nbcap + t / kBlock,
                  t % kBlock);
}

// Paged cache, one decode step: the token of sequence blockIdx.y, KV head blockIdx.x goes to
// position len mod 128 of the page of block len / 128.  Without a valid page the token is dropped
// (bit 1 of *status) and paged_bump_kernel leaves the length as it is.
__global__ __launch_bounds__(128) void mx_paged_append_kernel(MxDst d, const int32_t* __restrict__ block_table,
                                                               const int32_t* __restrict__ seq_lens,
                                                               const uint16_t* __restrict__ k_new,
                                                               const uint16_t* __restrict__ v_new) {
  const int h = blockIdx.x, b = blockIdx.y;
  const int len = seq_lens[b];
  if (len < 0) return;
  d.table_row = block_table + (size_t)b * d.max_pages;
  const long bi = mx_block_index(d, h, len / kBlock, mx_table_entry(d, len / kBlock));
  if (bi < 0) return;
  const size_t unit = (size_t)b * d.n_kv_heads + h;
  mx_append_token(k_new + unit * kD, v_new + unit * kD, d, bi, len % kBlock);
}

__global__ void set_len_kernel(int32_t* seq_lens, int seq, int L) {
  if (threadIdx.x == 0 && blockIdx.x == 0) seq_lens[seq] = L;
}

}  // namespace

// Tokens [0, L) of every unit, L > 0.
static hipError_t launch_mx_prefill(const void* k, const void* v, int L, int units, const MxDst& d, int32_t* seq_len,
                                    hipStream_t st) {
  mx_quant_block_kernel<<<dim3((L + kBlock - 1) / kBlock, units, 2), dim3(256), 0, st>>>(
      (const uint16_t*)k, (const uint16_t*)v, (long)L * kD, d, L, seq_len);
  return hipGetLastError();
}

hipError_t launch_quant_blocks(const void* k, const void* v, long src_unit_stride, int src_tok0, int nblocks,
                               int units, const bd_cache* c, int dst_blk0, int tail, hipStream_t st) {
  if (nblocks <= 0 && tail <= 0) return hipSuccess;
  dim3 grid(nblocks + (tail > 0 ? 1 : 0), units, 2), block(256);
  const int nbcap = c->capacity / kBlock;
  const uint16_t *kk = (const uint16_t*)k, *vv = (const uint16_t*)v;
  uint32_t *kc = (uint32_t*)c->k_codes, *vc = (uint32_t*)c->v_codes, *kp = (uint32_t*)c->k_params,
           *vp = (uint32_t*)c->v_params;
  uint16_t *kr = (uint16_t*)c->k_res, *vr = (uint16_t*)c->v_res;
  const bool six = six_on_a_unit(fmt_kt(c->format), (long)grid.x * units);
#define BD_QUANT_CASE(FMT, BITS, KT, G)                                                                                         \
  case FMT: {                                                                                                                   \
    constexpr int kSix = KT && G < 128 ? 5 : 6, kFive = KT && G == 128 ? 6 : 5;                                                 \
    const auto kernel = six ? quant_block_kernel<BITS, KT, G, kSix> : quant_block_kernel<BITS, KT, G, kFive>;                   \
    kernel<<<grid, block, 0, st>>>(kk, vv, src_unit_stride, src_tok0, kc, vc, kp, vp, nbcap, dst_blk0, kr, vr, tail);           \
  } break;
  switch (c->format) {
    BD_QUANT_CASE(BD_FMT_INT4, 4, false, 128)
    BD_QUANT_CASE(BD_FMT_INT2, 2, false, 128)
    BD_QUANT_CASE(BD_FMT_INT4_KT, 4, true, 128)
    BD_QUANT_CASE(BD_FMT_INT2_KT, 2, true, 128)
    BD_QUANT_CASE(BD_FMT_INT4_G64, 4, false, 64)
    BD_QUANT_CASE(BD_FMT_INT4_G32, 4, false, 32)
    BD_QUANT_CASE(BD_FMT_INT2_G64, 2, false, 64)
    BD_QUANT_CASE(BD_FMT_INT2_G32, 2, false, 32)
    BD_QUANT_CASE(BD_FMT_INT4_KT_G64, 4, true, 64)
    BD_QUANT_CASE(BD_FMT_INT4_KT_G32, 4, true, 32)
    BD_QUANT_CASE(BD_FMT_INT2_KT_G64, 2, true, 64)
    BD_QUANT_CASE(BD_FMT_INT2_KT_G32, 2, true, 32)
    default: return hipErrorInvalidValue;
  }
#undef BD_QUANT_CASE
  return hipGetLastError();
}

static PagedArgs paged_args(const bd_paged_cache* c) {
  PagedArgs a;
  a.k_codes = (uint32_t*)c->k_codes;
  a.v_codes = (uint32_t*)c->v_codes;
  a.k_params = (uint32_t*)c->k_params;
  a.v_params = (uint32_t*)c->v_params;
  a.k_res = (uint16_t*)c->k_res;
  a.v_res = (uint16_t*)c->v_res;
  a.block_table = c->block_table;
  a.seq_lens = c->seq_lens;
  a.status = c->status;
  a.n_kv_heads = c->n_kv_heads;
  a.num_pages = c->num_pages;
  a.max_pages = c->max_pages_per_seq;
  return a;
}

static MxDst paged_mx_dst(const bd_paged_cache* c) {
  MxDst d{};
  d.k_codes = (uint8_t*)c->k_codes;
  d.k_scales = (uint8_t*)c->k_params;
  d.v_codes = (uint8_t*)c->v_codes;
  d.v_scales = (uint8_t*)c->v_params;
  d.nbcap = 1;
  d.status = c->status;
  d.n_kv_heads = c->n_kv_heads;
  d.num_pages = c->num_pages;
  d.max_pages = c->max_pages_per_seq;
  return d;
}

hipError_t launch_paged_prefill(const bd_paged_cache* c, int seq, const void* k, const void* v, int L,
                                hipStream_t st) {
  if (c->format == BD_FMT_MXFP4) {
    // every token is quantized on arrival: the last, partly filled block lives in a page as well
    MxDst d = paged_mx_dst(c);
    d.table_row = c->block_table + (size_t)seq * c->max_pages_per_seq;
    if (L > 0) return launch_mx_prefill(k, v, L, c->n_kv_heads, d, c->seq_lens + seq, st);
    set_len_kernel<<<dim3(1), dim3(64), 0, st>>>(c->seq_lens, seq, L);
    return hipGetLastError();
  }
  const PagedArgs a = paged_args(c);
  dim3 grid(L / kBlock + 1, c->n_kv_heads, 2), block(256);
  const uint16_t *kk = (const uint16_t*)k, *vv = (const uint16_t*)v;
  const bool six = six_on_a_unit(fmt_kt(c->format), (long)grid.x * grid.y);
#define BD_PAGED_QUANT_CASE(FMT, BITS, KT, G)                                                                   \
  case FMT: {                                                                                                   \
    const auto kernel = six ? paged_quant_kernel<BITS, KT, G, KT ? 5 : 6> : paged_quant_kernel<BITS, KT, G, 5>; \
    kernel<<<grid, block, 0, st>>>(a, kk, vv, seq, L);                                                          \
  } break;
  switch (c->format) {
    BD_PAGED_QUANT_CASE(BD_FMT_INT4, 4, false, 128)
    BD_PAGED_QUANT_CASE(BD_FMT_INT2, 2, false, 128)
    BD_PAGED_QUANT_CASE(BD_FMT_INT4_KT, 4, true, 128)
    BD_PAGED_QUANT_CASE(BD_FMT_INT2_KT, 2, true, 128)
    BD_PAGED_QUANT_CASE(BD_FMT_INT4_G64, 4, false, 64)
    BD_PAGED_QUANT_CASE(BD_FMT_INT4_G32, 4, false, 32)
    BD_PAGED_QUANT_CASE(BD_FMT_INT2_G64, 2, false, 64)
    BD_PAGED_QUANT_CASE(BD_FMT_INT2_G32, 2, false, 32)
    BD_PAGED_QUANT_CASE(BD_FMT_INT4_KT_G64, 4, true, 64)
    BD_PAGED_QUANT_CASE(BD_FMT_INT4_KT_G32, 4, true, 32)
    BD_PAGED_QUANT_CASE(BD_FMT_INT2_KT_G64, 2, true, 64)
    BD_PAGED_QUANT_CASE(BD_FMT_INT2_KT_G32, 2, true, 32)
    default: return hipErrorInvalidValue;
  }
#undef BD_PAGED_QUANT_CASE
  return hipGetLastError();
}

hipError_t launch_paged_append(const bd_paged_cache* c, const void* k_new, const void* v_new, bool bump,
                               hipStream_t st) {
  const PagedArgs a = paged_args(c);
  dim3 grid(c->n_kv_heads, c->batch), block(256);
  const uint16_t *kk = (const uint16_t*)k_new, *vv = (const uint16_t*)v_new;
  if (c->format == BD_FMT_MXFP4) {
    mx_paged_append_kernel<<<grid, dim3(128), 0, st>>>(paged_mx_dst(c), c->block_table, c->seq_lens, kk, vv);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !bump) return e;
    paged_bump_kernel<<<dim3((c->batch + 63) / 64), dim3(64), 0, st>>>(a, c->batch, true);
    return hipGetLastError();
  }
  switch (c->format) {
    case BD_FMT_INT4: paged_append_kernel<4, false, 128><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT2: paged_append_kernel<2, false, 128><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT4_KT: paged_append_kernel<4, true, 128><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT2_KT: paged_append_kernel<2, true, 128><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT4_G64: paged_append_kernel<4, false, 64><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT4_G32: paged_append_kernel<4, false, 32><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT2_G64: paged_append_kernel<2, false, 64><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT2_G32: paged_append_kernel<2, false, 32><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT4_KT_G64: paged_append_kernel<4, true, 64><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT4_KT_G32: paged_append_kernel<4, true, 32><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT2_KT_G64: paged_append_kernel<2, true, 64><<<grid, block, 0, st>>>(a, kk, vv); break;
    case BD_FMT_INT2_KT_G32: paged_append_kernel<2, true, 32><<<grid, block, 0, st>>>(a, kk, vv); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !bump) return e;
  paged_bump_kernel<<<dim3((c->batch + 63) / 64), dim3(64), 0, st>>>(a, c->batch, false);
  return hipGetLastError();
}

hipError_t launch_paged_bump(const bd_paged_cache* c, hipStream_t st) {
  paged_bump_kernel<<<dim3((c->batch + 63) / 64), dim3(64), 0, st>>>(paged_args(c), c->batch, c->format == BD_FMT_MXFP4);
  return hipGetLastError();
}

// Measurement aid: reads the packed codes of the first `packed_len` tokens of every (sequence, KV head)
// unit with the decode kernel's loads (16 bytes per lane, non-temporal) and does nothing else: the time
// of this launch is the floor that the memory system sets for a decode launch over the same cache.
__global__ __launch_bounds__(256) void stream_probe_kernel(const u4_t* __restrict__ kc, const u4_t* __restrict__ vc,
                                                             size_t unit_stride_u4, size_t unit_u4, uint32_t* sink) {
  // blockIdx.y = 2 * unit + tensor.  Workgroup x: the 1 KB pieces x * 4 + wave, + 4 * gridDim.x, ... of that
  // unit's K (or V) codes, eight in flight per wave.
  const size_t pieces = unit_u4 / 64;   // whole 1 KB pieces (unit_u4 is a multiple of 64: blocks are 8 KB or 4 KB)
  const u4_t* base = (blockIdx.y & 1 ? vc : kc) + (blockIdx.y >> 1) * unit_stride_u4;
  const int lane = threadIdx.x & 63;
  const size_t first = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6), step = (size_t)gridDim.x * 4;
  u4_t acc = {0u, 0u, 0u, 0u};
  for (size_t p0 = first; p0 < pieces; p0 += 8 * step) {
    u4_t x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const size_t p = p0 + u * step < pieces ? p0 + u * step : p0;   // (past the end: the piece at p0 again)
      x[u] = __builtin_nontemporal_load(base + p * 64 + lane);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= x[u];
  }
  if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x9E3779B9u && sink) sink[0] = 1u;   // keeps the loads alive
}

hipError_t launch_stream_probe(const bd_cache* c, int packed_len, void* sink, hipStream_t st) {
  const int units = c->batch * c->n_kv_heads;
  const size_t block_bytes = (size_t)kBlock * kD * fmt_bits(c->format) / 8;   // K codes (and V codes) of one block
  const size_t unit_u4 = (size_t)(packed_len / kBlock) * block_bytes / 16;
  const size_t stride_u4 = (size_t)(c->capacity / kBlock) * block_bytes / 16;
  if (unit_u4 == 0) return hipSuccess;
  int wgs = (1024 + 2 * units - 1) / (2 * units);   // about 1024 workgroups in all: four resident per compute unit
  stream_probe_kernel<<<dim3(wgs, 2 * units), dim3(256), 0, st>>>((const u4_t*)c->k_codes, (const u4_t*)c->v_codes, stride_u4,
                                                                  unit_u4, (uint32_t*)sink);
  return hipGetLastError();
}

hipError_t launch_copy_rows(const void* ksrc, const void* vsrc, long src_unit_stride, int src_tok0, void* kdst,
                            void* vdst, long dst_unit_stride, int dst_tok0, int ntok, int units,
                            hipStream_t st) {
  if (ntok <= 0) return hipSuccess;
  const int threads = ntok * (kD / 8) >= 256 ? 256 : 64;
  copy_rows_kernel<<<dim3(units), dim3(threads), 0, st>>>((const u4_t*)ksrc, (const u4_t*)vsrc,
                                                          src_unit_stride, src_tok0, (u4_t*)kdst, (u4_t*)vdst,
                                                          dst_unit_stride, dst_tok0, ntok);
  return hipGetLastError();
}

static MxDst mx_dst(const bd_cache* c) {
  MxDst d{};
  d.k_codes = (uint8_t*)c->k_codes;
  d.k_scales = (uint8_t*)c->k_params;
  d.v_codes = (uint8_t*)c->v_codes;
  d.v_scales = (uint8_t*)c->v_params;
  d.nbcap = c->capacity / kBlock;
  return d;
}

hipError_t launch_mx_quant(const void* k, const void* v, int L, int units, const bd_cache* c, hipStream_t st) {
  return L > 0 ? launch_mx_prefill(k, v, L, units, mx_dst(c), nullptr, st) : hipSuccess;
}

hipError_t launch_mx_append(const void* k_new, const void* v_new, int units, const bd_cache* c, int t, hipStream_t st) {
  mx_append_kernel<<<dim3(units), dim3(128), 0, st>>>((const uint16_t*)k_new, (const uint16_t*)v_new, mx_dst(c), t);
  return hipGetLastError();
}

}  // namespace bd
