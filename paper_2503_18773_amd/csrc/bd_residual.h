// The fp16 residual tokens (Sec. IV-B) in the decode kernels of the integer formats, gfx950.
//
// A workgroup attends a slice of at most 128 residual tokens on the matrix unit: S^T[token, head], key rows as A and
// queries as B, 16 tokens a tile, then O^T[c, head] = sum_t V[t, c] p[t, head].  The accumulator layout of the scores
// (tokens 4g .. 4g + 3 of a tile in lane group g) is the B-operand layout of the second product, so that no weight
// passes between lanes; the lane groups are joined for the maximum and the sum alone.  Of a slice of up to 32 tokens
// every wave scores all and multiplies its own 32 channels of the value rows, and nothing passes between waves: a lane
// of wave w loads the channel pair 32w + 2 (lane % 16) of a token, and the halves of the loaded words are two A tiles
// (row i of tile u: channel 32w + 2i + u).  Weights are fp32 up to the product, which takes all 24 bits of p * 2^14 as three fp16 pieces: the last
// is clear of the subnormals' step for every weight above 2^-15, and what a smaller one loses is below 2^-39.
//
// The rows are requested when the kernel starts, ahead of the first packed block, and attended while that block is
// on its way (where their registers allow it; else before it is requested): an idle wave's time.  What bounds a slice is latency: folding its tokens in one by one at the end of
// the kernel, each behind a load of its own, took 50 us of a launch with up to 127 tokens in a slice (40 ragged
// sequences of up to 3.1K tokens, 2-bit codes, 8 heads per KV head, one split: 77 us a step, now 35; 24 of up to
// 5K, 4-bit codes, three splits: 38.2, now 29.0).  The same products at the end of the kernel cost a slice of one
// token 0.9 us (32K tokens, 64 splits: 14.2 against 13.3 us a step).
//
// A slice of more than 32 tokens would take a second round of loads and another 1.3 us for each 32.  It is shared out over
// the waves instead, 32 tokens of all channels each, and their maxima and sums meet in LDS, behind three barriers: 40 ragged sequences of up to 3.1K
// tokens, one split, 2 bits and 8 heads per KV head 29.5 -> 26.6 us a step, 4 bits 31.0 -> 27.2; 750 tokens, 8 units
// 11.6 -> 10.2.  (A short slice that way, a few tokens a wave, would cost two barriers and more matrix instructions.)
#pragma once

#include "bd_common.h"
#include "bd_device.h"

namespace bd {
namespace {

constexpr float kResTop = 16384.0f;
// Tokens [first, last) of the residual's `res_len` are split `split`'s slice (scale: ceil(2^32 / number of splits), so that
// no workgroup starts with a division).
__device__ __forceinline__ int residual_bound(int res_len, int split, int num_splits, uint32_t scale) {
  return split >= num_splits ? res_len : min((int)__umulhi((uint32_t)(res_len * split), scale), res_len);
}
static inline uint32_t residual_scale(int num_splits) {
  return num_splits <= 1 ? 0xFFFFFFFFu : (uint32_t)(((1ull << 32) + num_splits - 1) / num_splits);
}

// The rows of a slice: the residual buffers' from its first token on, and the newest token of a fused step, which is
// still where the caller left it (token new_at of the slice; kn, vn: its rows less new_at rows).
struct ResidualRows {
  const uint16_t *k, *v, *kn, *vn;
  int new_at;
};

// LDS alone is exchanged: loads on their way stay there (__syncthreads would wait for them)
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// p * kResTop of 8 weights, as three fp16 pieces
struct ResidualWeights {
  h8_t high = {}, mid = {}, low = {};
  __device__ __forceinline__ void put(int i, float p) {
    high[i] = (_Float16)(p * kResTop);
    const float rest = __builtin_fmaf(p, kResTop, -(float)high[i]);
    mid[i] = (_Float16)rest;
    low[i] = (_Float16)(rest - (float)mid[i]);
  }
  // o0 += v0 p, o1 += v1 p, the smallest piece first
  __device__ __forceinline__ void multiply(h8_t v0, h8_t v1, f4_t& o0, f4_t& o1) const {
#pragma unroll
    for (const h8_t& piece : {low, mid, high}) {
      o0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(v0, piece, o0, 0, 0, 0);
      o1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(v1, piece, o1, 0, 0, 0);
    }
  }
};

struct ResidualSlice {
  // 16-token tiles in flight.  (Four would hide more of a long slice's latency, but the 80 registers they hold
  // are more than the single-block instances have: three of their workgroups share a compute unit.)
  static constexpr int kTiles = 2;
  h8_t q[4];                 // queries (B operand), column = head
  h8_t k[kTiles][4];         // key rows of tile i (A operand)
  uint32_t v[kTiles][4];     // short slices, value words: token 4g + r of tile i
  u4_t vl[kTiles][4];        // long slices: 8 channels of the token

  // The queries and the slice's n > 0 tokens, of a long one the wave's 32: qbase the group's first query row, gq its heads.
  // (SHORT, LONG: the lengths that the caller has.  MORE: the workgroup has more than the four waves that share a slice.)
  template <bool SHORT = true, bool LONG = true, bool MORE = false>
  __device__ __forceinline__ void start(const uint16_t* qbase, int gq, int n, const ResidualRows& rows, int wave, int lane) {
    const int col = lane & 15, g = lane >> 4;
    const bool is_short = !LONG || (SHORT && n <= kResShort);
    if (MORE && wave >= 4) return;
    const int t0 = is_short ? 0 : 32 * wave;
    // (rows past the slice repeat its last token)
    const uint16_t *kl = rows.k + 8 * g, *knl = rows.kn + 8 * g;
    auto request_keys = [&](int i) {
      const int t = min(t0 + 16 * i + col, n - 1);
      const uint16_t* kr = (t == rows.new_at ? knl : kl) + (uint32_t)(t * kD);
#pragma unroll
      for (int j = 0; j < 4; ++j) k[i][j] = *reinterpret_cast<const h8_t*>(kr + 32 * j);
    };
    const int c0 = is_short ? 32 * wave + 2 * col : 8 * col;
    const uint16_t *vl0 = rows.v + c0, *vnl = rows.vn + c0;
    auto value = [&](int i, int r) {
      const int t = min(t0 + 16 * i + 4 * g + r, n - 1);
      return (t == rows.new_at ? vnl : vl0) + (uint32_t)(t * kD);
    };
    const uint16_t* qp = qbase + (uint32_t)(min(col, gq - 1) * kD + 8 * g);   // (columns past the group repeat its last head)
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = *reinterpret_cast<const h8_t*>(qp + 32 * j);
    if (is_short) {
#pragma unroll
      for (int i = 0; i < kTiles; ++i) {
        if (i && 16 * i >= n) break;
        request_keys(i);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[i][r] = *reinterpret_cast<const uint32_t*>(value(i, r));
      }
    } else if (t0 < n) {
#pragma unroll
      for (int i = 0; i < kTiles; ++i) {
        request_keys(i);
#pragma unroll
        for (int r = 0; r < 4; ++r) vl[i][r] = *reinterpret_cast<const u4_t*>(value(i, r));
      }
    }
  }

  // Scores (log2 units) of the 32 tokens, of which `live` count; the largest.
  __device__ __forceinline__ float score(int live, float scale_log2, int g, float (&s)[2][4]) const {
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (u && live <= 16) break;   // (the same for the whole wave)
      f4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(k[u][j], q[j], acc, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[u][r] = 16 * u + 4 * g + r < live ? acc[r] * scale_log2 : -INFINITY;
        m = fmaxf(m, s[u][r]);
      }
    }
    return join_groups(m, Max());
  }
  // Weights relative to 2^m; their sum.
  __device__ __forceinline__ static float weigh(int live, const float (&s)[2][4], float m, ResidualWeights& p) {
    float l = 0.0f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (u && live <= 16) break;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float e = __builtin_amdgcn_exp2f(s[u][r] - m);
        l += e;
        p.put(4 * u + r, e);
      }
    }
    return join_groups(l, Add());
  }

  // Leaves the slice's partial result in LDS for the merge: out_o[head][128], relative to 2^out_m[head], and the
  // sum of weights out_l[head].  The caller synchronises before it reads them.  ml: LDS of the final merge (MergeLds),
  // free until then; every wave of the workgroup calls this.
  template <int GQP, bool SHORT = true, bool LONG = true, bool MORE = false, class ML>
  __device__ __forceinline__ void attend(int n, float scale_log2, ML& ml, float (*out_o)[kD], float* out_m, float* out_l,
                                         int wave, int lane) {
    const int col = lane & 15, g = lane >> 4;
    ResidualWeights p;
    float s[2][4];
    if (!LONG || (SHORT && n <= kResShort)) {
      if (MORE && wave >= 4) return;
      const float m = score(n, scale_log2, g, s), l = weigh(n, s, m, p);
      u4_t a0 = {0u, 0u, 0u, 0u}, a1 = a0;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (u && n <= 16) break;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          a0[2 * u + h] = __builtin_amdgcn_perm(v[u][2 * h + 1], v[u][2 * h], 0x05040100u);   // even channel
          a1[2 * u + h] = __builtin_amdgcn_perm(v[u][2 * h + 1], v[u][2 * h], 0x07060302u);   // odd channel
        }
      }
      f4_t o0 = {0.f, 0.f, 0.f, 0.f}, o1 = o0;
      p.multiply(__builtin_bit_cast(h8_t, a0), __builtin_bit_cast(h8_t, a1), o0, o1);
      if (col >= GQP) return;
#pragma unroll
      for (int r = 0; r < 4; ++r)   // row 4g + r of the two tiles
        *reinterpret_cast<float2*>(&out_o[col][32 * wave + 2 * (4 * g + r)]) =
            make_float2(o0[r] * (1.0f / kResTop), o1[r] * (1.0f / kResTop));
      if (wave == 0 && g == 0) {
        out_m[col] = m;
        out_l[col] = l;
      }
      return;
    }
    if constexpr (!LONG) return;
    // A long slice: the wave's 32 tokens of all channels; row i of M tile e is channel 8i + e.  The weights of all are
    // relative to the same maximum, so that they are added as they are.
    const int live = min(n - 32 * wave, 32);
    float m = -INFINITY, l = 0.0f;
    if (live > 0) m = score(live, scale_log2, g, s);
    if (lane < GQP) ml.m[wave][col] = m;
    lds_barrier();
    const int waves = (n + 31) / 32;
    m = ml.m[0][col % GQP];
    for (int w = 1; w < waves; ++w) m = fmaxf(m, ml.m[w][col % GQP]);
    f4_t o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (f4_t){0.f, 0.f, 0.f, 0.f};
    if (live > 0) {
      l = weigh(live, s, m, p);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        u4_t a0, a1;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            a0[2 * u + h] = __builtin_amdgcn_perm(vl[u][2 * h + 1][i], vl[u][2 * h][i], 0x05040100u);
            a1[2 * u + h] = __builtin_amdgcn_perm(vl[u][2 * h + 1][i], vl[u][2 * h][i], 0x07060302u);
          }
        p.multiply(__builtin_bit_cast(h8_t, a0), __builtin_bit_cast(h8_t, a1), o[2 * i], o[2 * i + 1]);
      }
    }
    if (col < GQP) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          f4_t x;
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = o[4 * half + e][r];
          *reinterpret_cast<f4_t*>(&ml.o[wave][col][8 * (4 * g + r) + 4 * half]) = x;
        }
      if (g == 0) ml.l[wave][col] = l;
    }
    lds_barrier();
#pragma unroll
    for (int h0 = 0; h0 < GQP; h0 += 4) {
      if (MORE && wave >= 4) break;
      const int h = h0 + wave, c0 = 2 * lane;
      float L = 0.f, x = 0.f, y = 0.f;
      for (int w = 0; w < waves; ++w) {
        L += ml.l[w][h];
        x += ml.o[w][h][c0];
        y += ml.o[w][h][c0 + 1];
      }
      *reinterpret_cast<float2*>(&out_o[h][c0]) = make_float2(x * (1.0f / kResTop), y * (1.0f / kResTop));
      if (lane == 0) out_l[h] = L;
    }
    if (wave == 0 && lane < GQP) out_m[col] = m;
    lds_barrier();   // the space is the waves' scratch from here on
  }
};

}  // namespace
}  // namespace bd
