// The fp16 residual tokens (Sec. IV-B) in the decode kernels of the integer formats, gfx950.
//
// A workgroup attends a slice of at most 128 residual tokens, on the matrix unit and in registers only.  Every
// wave scores the whole slice (S^T[token, head], key rows as A and queries as B, 16 tokens a tile) and multiplies
// its own 32 channels of the value rows, O^T[c, head] = sum_t V[t, c] p[t, head]: the accumulator layout of the
// scores (tokens 4g .. 4g + 3 of a tile in lane group g) is the B-operand layout of the second product, so nothing
// passes between lanes or waves.  Wave w takes channels 32w .. 32w + 31; a lane loads the channel pair
// 32w + 2 (lane % 16) of a token, and the halves of the loaded words are two A tiles (row i of tile u: channel
// 32w + 2i + u).  Weights are fp32 up to the product, which takes all 24 bits of p * 2^14 as three fp16 pieces: the last
// is clear of the subnormals' step for every weight above 2^-15, and what a smaller one loses is below 2^-39.
//
// The rows are requested when the kernel starts, ahead of the first packed block, and attended while that block is
// on its way: an idle wave's time.  What bounds a slice is latency: folding its tokens in one by one at the end of
// the kernel, each behind a load of its own, took 50 us of a launch with up to 127 tokens in a slice (40 ragged
// sequences of up to 3.1K tokens, 2-bit codes, 8 heads per KV head, one split: 77 us a step, now 35; 24 of up to
// 5K, 4-bit codes, three splits: 38.2, now 29.0).  The same products at the end of the kernel cost a slice of one
// token 0.9 us (32K tokens, 64 splits: 14.2 against 13.3 us a step).
#pragma once

#include "bd_common.h"
#include "bd_device.h"

namespace bd {
namespace {

constexpr float kResTop = 16384.0f;

struct ResidualSlice {
  // 16-token tiles in flight.  (Four would hide more of a long slice's latency, but the 80 registers they hold
  // are more than the single-block instances have: three of their workgroups share a compute unit.)
  static constexpr int kTiles = 2;
  h8_t q[4];                 // queries (B operand), column = head, zero past the group
  h8_t k[kTiles][4];         // key rows of tile i (A operand)
  uint32_t v[kTiles][4];     // value words: token 4g + r of tile i

  // krow(t), vrow(t): rows of slice token t (0 <= t < n).  Requests tokens t0 .. t0 + 31.
  template <class KRow, class VRow>
  __device__ __forceinline__ void request(int t0, int n, KRow krow, VRow vrow, int wave, int lane) {
    const int col = lane & 15, g = lane >> 4;
#pragma unroll
    for (int i = 0; i < kTiles; ++i) {
      if (i && t0 + 16 * i >= n) break;
      const uint16_t* kr = krow(min(t0 + 16 * i + col, n - 1)) + 8 * g;   // rows past the slice repeat its last token
#pragma unroll
      for (int j = 0; j < 4; ++j) k[i][j] = *reinterpret_cast<const h8_t*>(kr + 32 * j);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        v[i][r] = *reinterpret_cast<const uint32_t*>(vrow(min(t0 + 16 * i + 4 * g + r, n - 1)) + 32 * wave + 2 * col);
    }
  }

  // The queries and the first tokens: qbase the group's first query row, gq its heads; n > 0.
  template <class KRow, class VRow>
  __device__ __forceinline__ void start(const uint16_t* qbase, int gq, int n, KRow krow, VRow vrow, int wave, int lane) {
    const int col = lane & 15, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const h8_t zero = {0, 0, 0, 0, 0, 0, 0, 0};
      q[j] = col < gq ? *reinterpret_cast<const h8_t*>(qbase + col * kD + 32 * j + 8 * g) : zero;
    }
    request(0, n, krow, vrow, wave, lane);
  }

  // Leaves the slice's partial result in LDS for the merge: out_o[head][128], relative to 2^out_m[head], and the
  // sum of weights out_l[head].  The caller synchronises before it reads them.
  template <int GQP, class KRow, class VRow>
  __device__ __forceinline__ void attend(int n, float scale_log2, KRow krow, VRow vrow, float (*out_o)[kD], float* out_m,
                                         float* out_l, int wave, int lane) {
    const int col = lane & 15, g = lane >> 4;
    float m = -INFINITY, l = 0.0f;   // running maximum (log2 units), this lane's share of the running sum
    f4_t o[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    for (int t0 = 0; t0 < n; t0 += 32) {   // one k-step of the second product
      if (t0) request(t0, n, krow, vrow, wave, lane);
      const bool two = t0 + 16 < n;   // (the same for the whole workgroup)
      float s[2][4];
      float mx = -INFINITY;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (u && !two) break;
        f4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(k[u][j], q[j], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          s[u][r] = t0 + 16 * u + 4 * g + r < n ? acc[r] * scale_log2 : -INFINITY;
          mx = fmaxf(mx, s[u][r]);
        }
      }
      mx = join_groups(mx, Max());
      if (t0) {
        mx = fmaxf(m, mx);
        const float alpha = __builtin_amdgcn_exp2f(m - mx);
        l *= alpha;
        o[0] *= alpha;
        o[1] *= alpha;
      }
      m = mx;
      h8_t ph = {}, pm = {}, pl = {};
      u4_t a0 = {0u, 0u, 0u, 0u}, a1 = a0;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (u && !two) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = __builtin_amdgcn_exp2f(s[u][r] - m);
          l += p;
          ph[4 * u + r] = (_Float16)(p * kResTop);
          const float rest = __builtin_fmaf(p, kResTop, -(float)ph[4 * u + r]);
          pm[4 * u + r] = (_Float16)rest;
          pl[4 * u + r] = (_Float16)(rest - (float)pm[4 * u + r]);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          a0[2 * u + h] = __builtin_amdgcn_perm(v[u][2 * h + 1], v[u][2 * h], 0x05040100u);   // even channel
          a1[2 * u + h] = __builtin_amdgcn_perm(v[u][2 * h + 1], v[u][2 * h], 0x07060302u);   // odd channel
        }
      }
      const h8_t v0 = __builtin_bit_cast(h8_t, a0), v1 = __builtin_bit_cast(h8_t, a1);
#pragma unroll
      for (const h8_t& piece : {pl, pm, ph}) {
        o[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v0, piece, o[0], 0, 0, 0);
        o[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v1, piece, o[1], 0, 0, 0);
      }
    }
    l = join_groups(l, Add());
    if (col >= GQP) return;
#pragma unroll
    for (int r = 0; r < 4; ++r)   // row 4g + r of the two tiles
      *reinterpret_cast<float2*>(&out_o[col][32 * wave + 2 * (4 * g + r)]) =
          make_float2(o[0][r] * (1.0f / kResTop), o[1][r] * (1.0f / kResTop));
    if (wave == 0 && g == 0) {
      out_m[col] = m;
      out_l[col] = l;
    }
  }
};

}  // namespace
}  // namespace bd
