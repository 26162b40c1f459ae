// Device-side helpers shared by the decode kernels (gfx950, wave64).
#pragma once

#include "bd_common.h"
#include "bd_rules.h"

namespace bd {
namespace {

__device__ __forceinline__ float h2f(uint16_t b) {
  _Float16 h;
  __builtin_memcpy(&h, &b, 2);
  return (float)h;
}
__device__ __forceinline__ uint16_t f2h(float f) {
  _Float16 h = (_Float16)f;
  uint16_t b;
  __builtin_memcpy(&b, &h, 2);
  return b;
}

// DPP lane movement inside rows of 16 lanes.
constexpr int kRowShl4 = 0x104, kRowShl8 = 0x108, kRowShl12 = 0x10C, kRowShr4 = 0x114, kRowShr8 = 0x118, kRowRor4 = 0x124, kRowRor8 = 0x128;
constexpr int kQuadSwap1 = 0xB1 /* [1,0,3,2] */, kQuadSwap2 = 0x4E /* [2,3,0,1] */;
constexpr int kRowHalfMirror = 0x141, kRowMirror = 0x140;

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
// The value of the lane 16 (32) away joined to this lane's: v_permlane16_swap / 32_swap of two copies leave the pair's
// values in the two results, in the same order in both lanes.  (8 cycles and no wait; a shuffle through LDS takes 56.)
template <class Op>
__device__ __forceinline__ float join_xor16(float x, Op op) {
  const u2_t r = __builtin_bit_cast(u2_t, __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false));
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <class Op>
__device__ __forceinline__ float join_xor32(float x, Op op) {
  const u2_t r = __builtin_bit_cast(u2_t, __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false));
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
struct Add {
  __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct Max {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
// over the four lane groups (lanes col, col + 16, col + 32, col + 48)
template <class Op>
__device__ __forceinline__ float join_groups(float x, Op op) { return join_xor32(join_xor16(x, op), op); }

// sum over the 16 lanes of a row, result in every lane
__device__ __forceinline__ float row_sum16(float x) {
  x += dpp_f<kQuadSwap1>(x);
  x += dpp_f<kQuadSwap2>(x);
  x += dpp_f<kRowHalfMirror>(x);
  x += dpp_f<kRowMirror>(x);
  return x;
}
// 2^e for e in [-126, 127]
__device__ __forceinline__ float pow2i(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }
// the power of two that brings fp16 magnitudes up to `bits` (the largest one's bit pattern) below 2^top
__device__ __forceinline__ int norm_exponent(uint32_t bits, int top) { return top + 14 - (int)(bits >> 10); }
// Q' = q * scale * position factor goes to the matrix unit as an fp16 high + low pair: queries are brought
// below 2^7 and a block's K scales below 2^8, so |Q'| < 2^15 (finite) and the low pieces of all but
// negligible entries stay above the subnormals.
constexpr int kQTop = 7, kSTop = 8;
__device__ __forceinline__ uint32_t row_max16_u(uint32_t m) {
  m = max(m, dpp_u<kQuadSwap1>(m));
  m = max(m, dpp_u<kQuadSwap2>(m));
  m = max(m, dpp_u<kRowHalfMirror>(m));
  m = max(m, dpp_u<kRowMirror>(m));
  return m;
}
// largest of a non-negative value over the wave, as a wave-uniform result
__device__ __forceinline__ uint32_t wave_max_u(uint32_t m) {
  m = row_max16_u(m);
  return max(max(__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 16)),
             max(__builtin_amdgcn_readlane(m, 32), __builtin_amdgcn_readlane(m, 48)));
}
// reductions over the lanes that carry the same head (column % (16 / COPIES)): COPIES column
// groups x 4 lane groups
template <int COPIES>
__device__ __forceinline__ float head_sum(float x) {
  if (COPIES == 4) x += dpp_f<kRowRor4>(x);
  if (COPIES >= 2) x += dpp_f<kRowRor8>(x);
  return join_groups(x, Add());
}
template <int COPIES>
__device__ __forceinline__ float head_max(float x) {
  if (COPIES == 4) x = fmaxf(x, dpp_f<kRowRor4>(x));
  if (COPIES >= 2) x = fmaxf(x, dpp_f<kRowRor8>(x));
  return join_groups(x, Max());
}

// Element type of the output rows: the format's own half type (fp16; bf16 for MXFP4) or fp32
// (bd_cache.out_type).
constexpr int kOutF16 = 0, kOutBf16 = 1, kOutF32 = 2;
__host__ __device__ __forceinline__ int out_kind(int format, int out_type) {
  return out_type == BD_OUT_F32 ? kOutF32 : format == BD_FMT_MXFP4 ? kOutBf16 : kOutF16;
}
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// A launch with one split needs no merge: the workgroup's (L, o) is the result, stored as two
// adjacent outputs o / L at elements idx, idx + 1 of `out`, exactly as the merge kernel would
// compute them (a head that attended nothing, L == 0, gives zeros).
__device__ __forceinline__ void store_final_pair(void* out, size_t idx, int kind, float o0, float o1, float L) {
  const float r0 = L > 0.f ? o0 / L : 0.f, r1 = L > 0.f ? o1 / L : 0.f;
  if (kind == kOutF32) {
    *reinterpret_cast<float2*>(reinterpret_cast<float*>(out) + idx) = make_float2(r0, r1);
    return;
  }
  const uint32_t lo = kind == kOutBf16 ? f2bf(r0) : f2h(r0), hi = kind == kOutBf16 ? f2bf(r1) : f2h(r1);
  *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(out) + idx) = lo | (hi << 16);
}

__device__ __forceinline__ void wave_sync() {
  // LDS operations of one wave execute in order; this only stops the compiler from moving
  // accesses across the exchange point.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Makes global stores of this workgroup visible to its own later loads, for data that the workgroup
// writes and then reads back inside one launch: wait until the stores have been written through to
// L2, then meet.  The waves of a workgroup share their compute unit's vector cache, which its own
// stores keep current, so workgroup scope is all this needs -- and all it can afford: measured at one
// such workgroup per (sequence, KV head) and decode step, a device-scope release (__threadfence(),
// which also writes back the XCD's L2) cost 45 us per launch and a device-scope acquire (which
// invalidates the vector cache) 7 us.
__device__ __forceinline__ void workgroup_global_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Index of per-token float2 parameters staged in LDS: lanes that work on different 32-token chunks read
// the same offset of their chunks at once, and entries 32 apart (256 bytes) share their banks, so every
// chunk is shifted by two entries (arrays hold kParSlots entries).
constexpr int kParSlots = 128 + 8;
__device__ __forceinline__ int par_slot(int t) { return t + 2 * (t >> 5); }

// The arguments that a wave's first loads wait for come as scalars ahead of an attention kernel's struct: those are in
// registers when it starts (build.py; there is room for 14 words), the struct has to be fetched first, 0.3 us.  With the
// merge's arguments likewise: 6K tokens, 8 units 9.15 -> 8.9 us a step, 4 x 8K in groups of 32 16.7 -> 16.1.
#define BD_HOT_PARAMS const uint16_t *hq, const void *hk, const void *hx, const void *hy, int hgq, int hkvh, int hns, int hi, int hj, int hm
#define BD_HOT_NAMES hq, hk, hx, hy, hgq, hkvh, hns, hi, hj, hm
#define BD_HOT_CONTIGUOUS(a) \
  a.q, a.k_codes, a.k_params, a.k_res, a.gq, a.n_kv_heads, a.num_splits, a.nb, a.nbcap, hot_word(a.res_len, a.flush_mode, a.new_slot + 1)
#define BD_HOT_PAGED(a, grid, batch) \
  a.q, a.k_codes, a.seq_lens, a.block_table, a.gq, a.n_kv_heads, a.num_splits, a.max_pages, a.num_pages, \
      hot_word((grid).order, (grid).flush_mode, a.step + 2 * (a.k_new != nullptr) + 4 * ((grid).flush_mode == kFlushLast ? batch : 0))
static inline int hot_word(int low, int flush_mode, int high) { return (int)((uint32_t)low | (uint32_t)flush_mode << 8 | (uint32_t)high << 16); }
template <bool PAGED, class Codes = uint32_t>
struct HotArgs {
  const uint16_t *q, *k_res;
  const Codes *k_codes, *k_params;
  const int32_t *seq_lens, *block_table;
  int gq, n_kv_heads, num_splits, flush_mode;
  int nb, nbcap, res_len, new_slot;    // contiguous
  int max_pages, num_pages;            // paged
  int sorted, second;                  // ... sequences to be sorted, those of the second layer (paged_sequence)
  int batch;                           // ... kFlushLast: sequences
  bool step;                           // ... the launch is the attention of a fused step
  bool append;                         // the launch appends the step's token itself
  // k_params_, k_res_: the struct's, for the paged form
  __device__ __forceinline__ HotArgs(BD_HOT_PARAMS, const Codes* k_params_, const uint16_t* k_res_)
      : q(hq), k_res(PAGED ? k_res_ : (const uint16_t*)hy), k_codes((const Codes*)hk),
        k_params(PAGED ? k_params_ : (const Codes*)hx), seq_lens(PAGED ? (const int32_t*)hx : nullptr),
        block_table(PAGED ? (const int32_t*)hy : nullptr), gq(hgq), n_kv_heads(hkvh), num_splits(hns),
        flush_mode((hm >> 8) & 3), nb(PAGED ? 0 : hi), nbcap(PAGED ? 0 : hj), res_len(PAGED ? 0 : hm & 255),
        new_slot(PAGED ? -1 : (hm >> 16) - 1), max_pages(PAGED ? hi : 0), num_pages(PAGED ? hj : 0),
        sorted(PAGED ? hm & 255 : 0), second(PAGED ? (hm >> 10) & 63 : 0), batch(PAGED ? (int)((uint32_t)hm >> 18) : 0), step(PAGED && (hm >> 16 & 1)), append(PAGED ? (hm >> 16 & 2) != 0 : hm >> 16 > 0) {}
};

// Waits until at most N vector loads are outstanding.  Where the loads before them are known to have been used, this costs
// nothing and tells the compiler so: after a load and its use behind one and the same condition it takes the load for
// possibly outstanding, and waits for everything where its register is written next, be it in the loop that follows.
template <int N>
__device__ __forceinline__ void loads_left() {
  static_assert(N >= 0 && N < 16, "vmcnt, low bits");
  __builtin_amdgcn_s_waitcnt(0xF70 | N);
}

// A word that this launch does not write, at an address that is the same for the whole wave, through the scalar cache:
// it comes past the wave's queue of vector loads, and what is computed from it stays scalar (page numbers: 8 sequences of
// up to 3K tokens, one split 20.2 -> 18.7 us, 40 in groups of 64 32.4 -> 30.4).
__device__ __forceinline__ int32_t scalar_load(const int32_t* p) {
  typedef const __attribute__((address_space(4))) int32_t* Const;
  return *(Const)p;
}

// A length.  RAISE: not to be loaded again later, when LengthRaise may have changed it.
template <bool RAISE>
__device__ __forceinline__ int32_t length_of(const int32_t* p) {
  int32_t x = scalar_load(p);
  if constexpr (RAISE) asm volatile("" : "+s"(x));
  return x;
}

// Raises the length of sequence b if its step went through: a page is needed when the step fills the residual, or, if
// `every_token`, by every token.
__device__ __forceinline__ void raise_length(int32_t* seq_lens, const int32_t* block_table, int b, int max_pages, int num_pages,
                                             bool every_token) {
  const int len = seq_lens[b];
  if (len < 0) return;
  if (every_token || len % kBlock == kBlock - 1) {
    const int n = len / kBlock;
    const int page = n < max_pages ? block_table[(size_t)b * max_pages + n] : -1;
    if (page < 0 || page >= num_pages) return;
  }
  seq_lens[b] = len + 1;
}

// Paged cache: the sequence of grid row z and its length.  A ragged batch of 257 workgroups and more (one per compute unit
// is 256) is dealt by length (to 1/16, then by index):
// - Up to 384 workgroups, 512 where the table has eight blocks a split and more.  An instance of which two share a compute
//   unit runs them all from the start, and workgroup 256 + j goes to j's unit (as the times show).  The shortest sequences
//   form the second layer, shortest first, on top of the next shortest in order; the longest have a unit to themselves.  40
//   sequences of 1K to 3.1K tokens, one split, 2 bits, 8 heads per KV head 23.4 -> 21.3 us a call against longest first;
//   against the order as given 56 of 0.3K to 3.1K 26.7 -> 21.1, 4 bits 64 of 0.4K to 4K 33.4 -> 29.7, 20 of 2K to 6K in three
//   splits 24.6 -> 23.6, MXFP4 60 of 0.3K to 3K 25.4 -> 23.0.
// - An instance that fills a unit alone (MXFP4 with 9 and more heads per KV head, groups of 32 with more than 4) runs the
//   rest as units come free: longest first.  MXFP4, 16 heads, 48 sequences of 1K to 3K tokens 48.3 us a step (two layers
//   51.6, as given 59 for 56 of them, where this takes 51.7); groups of 32, 8 heads, 56 of 1K to 3K 74.5 as given, 62.7.
// - Past that, rounds follow as units come free: where the last would fill at most half of them, longest first, so that they
//   get short ones.  24 of up to 5K, three splits, groups of 32 42.4 -> 39.3; not MXFP4 (29.4 / 30.1).
// The lengths' load then stands before everything else of the workgroup, which costs up to 0.6 us where the lengths are
// equal after all (64 of 2000, 4 bits 27.9 -> 28.2 us, groups of 32 with 8 heads 62.3 -> 62.9; MXFP4 64 of 3000 46.5 -> 46.7)
// and more than it gives where all are short (64 of 100 to 300 10.3 -> 10.7): hence the table's width, which is what the host
// knows of the lengths.  Every wave selects its sequence itself, a bit of the key at a time; batches of more than 64
// sequences stay as they are.
// A sequence whose residual this step's token fills is packed before it is attended: 5 us, the time of kFillWork tokens,
// which count as length (steps of 40 / 56 sequences, one of which fills, 2 bits, 8 heads 26.7 -> 24.1 / 30.9 -> 27.5 us).
// One number for all formats, though their time a token differs: it only has to keep such a sequence from a shared unit, and
// 450 and 1800 give what 900 does within 2 % from 2 bits with 4 heads to groups of 32 with 8.
constexpr int kFillWork = 900;
template <bool RAISE>
__device__ __forceinline__ int paged_sequence(const int32_t* __restrict__ seq_lens, int lane, int& seq_len, int n, int second,
                                              int fill_work) {
  if (n == 0) {
    seq_len = length_of<RAISE>(seq_lens + blockIdx.z);
    return blockIdx.z;
  }
  const int len = seq_lens[min(lane, n - 1)];
  // exponent and four bits of the length: 0 .. 30 * 16 + 15
  const float work = (float)len + ((len & 127) == 127 ? (float)fill_work : 0.0f);
  const uint32_t key = len > 0 ? (__float_as_uint(work) >> 19) - (127u << 4) : 0u;
  uint64_t cand = __ballot(lane < n);   // those that share the key's leading bits
  if (__all(key == (uint32_t)__builtin_amdgcn_readfirstlane(key))) {
    seq_len = __builtin_amdgcn_readlane(len, blockIdx.z);
    return blockIdx.z;
  }
  int z = place_by_length(blockIdx.z, n, second);   // the wanted one's place among them
#pragma unroll
  for (int bit = 8; bit >= 0; --bit) {
    const uint64_t ones = __ballot(((key >> bit) & 1u) != 0) & cand;
    const int c = __builtin_popcountll(ones);
    if (z < c) {
      cand = ones;
    } else {
      z -= c;
      cand &= ~ones;
    }
  }
  const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(cand >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)cand, 0u));
  const int b = __builtin_ctzll(__ballot((cand >> lane & 1u) != 0 && before == z));
  seq_len = __builtin_amdgcn_readlane(len, b);
  return b;
}

// Raises the lengths of a paged step in its only launch.  Every workgroup reads its sequence's length, where
// sequences are sorted everybody's, so no length may change before all workgroups have read.  Each counts itself once its waves have,
// at the counter of its sequence's shard; the one that completes a shard's count counts the shard, and the one that completes
// those raises.  The atomics are relaxed and at device scope (no cache to write back: the counters are all that is exchanged).
// A step against a launch of its own for the lengths, one by one: 40 sequences of 1K to 3.1K tokens, 2 bits, 8 heads per KV
// head 23.4 -> 22.0 us; 58 of 0.5K to 1.5K, 2 bits, 5 heads 21.1 -> 19.5; 9 of up to 26 tokens, 4 bits 9.3 -> 6.5; MXFP4 9 of up
// to 242 9.2 -> 6.9.  In a graph: groups of 32, 32 of up to 1000 17.7 -> 16.7; groups of 64, 2 bits, 8 heads, 33 of up to 3000
// 30.6 -> 29.3.
// The counters are zero between launches: the last to count leaves each so.
struct LengthRaise {
  uint32_t seen;   // the shard's counter as it was

  __device__ __forceinline__ static uint32_t* word(const RaiseArgs& r, int i) { return r.words + kRaiseStride * i; }
  __device__ __forceinline__ static uint32_t add(uint32_t* w) {
    return __hip_atomic_fetch_add(w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ static void clear(uint32_t* w) {
    __hip_atomic_store(w, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // The whole workgroup, which has read all lengths that it needs; `b` its sequence.
  __device__ __forceinline__ void arrive(const RaiseArgs& r, int b, int batch) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (not __syncthreads: vector loads stay on their way)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    seen = 0;
    if (threadIdx.x == blockDim.x - 64) seen = add(word(r, 1 + b % raise_shards(batch)));   // (the last wave has the fewest blocks)
  }
  // Behind the workgroup's first loads and what else it can do meanwhile.
  template <class Hot>
  __device__ __forceinline__ void finish(const RaiseArgs& r, int b, int batch, const Hot& hot, bool every_token) const {
    if (threadIdx.x < blockDim.x - 64) return;
    const int shards = raise_shards(batch), s = b % shards;
    bool last = false;
    if (threadIdx.x == blockDim.x - 64 && seen + 1 == (uint32_t)raise_arrivals(s, r.per_seq, batch)) {
      clear(word(r, 1 + s));
      if (add(word(r, 0)) + 1 == (uint32_t)shards) {
        clear(word(r, 0));
        last = true;
      }
    }
    if (!__any(last)) return;
    for (int i = threadIdx.x & 63; i < batch; i += 64)
      raise_length(const_cast<int32_t*>(hot.seq_lens), hot.block_table, i, hot.max_pages, hot.num_pages, every_token);
  }
};

// For the attention launch of a step in one split: `per_seq` workgroups of a sequence.
static inline RaiseArgs raise_args(const bd_paged_cache* c, bool wanted, long per_seq, void* counters) {
  if (!wanted || !counters || !raises_in_launch(per_seq, c->batch, BD_STEP_COUNTER_BYTES)) return {nullptr, 0};
  return {reinterpret_cast<uint32_t*>(counters), (int)per_seq};
}

// Of an integer format's workgroup: its sequence, the sequence's length, and whether it only packs (split -1).  False: it has
// nothing to do.
template <bool RAISE, class Hot>
__device__ __forceinline__ bool paged_workgroup(const Hot& hot, int lane, int& split, int& b, int& seq_len) {
  if (hot.flush_mode == kFlushLast && (int)blockIdx.z >= hot.batch) {
    split = -1;
    b = packed_sequence(blockIdx.x, blockIdx.z, hot.num_splits, hot.batch);
    if (b >= hot.batch) return false;
    seq_len = length_of<RAISE>(hot.seq_lens + b);
    return true;
  }
  b = paged_sequence<RAISE>(hot.seq_lens, lane, seq_len, hot.sorted, hot.second, hot.append && hot.flush_mode == kFlushNone ? kFillWork : 0);
  return true;
}

}  // namespace
}  // namespace bd
