// The kernels of bd_decode_mx.hip, included twice there: as decode_*_kernel, and, with BD_RAISE, as step_*_kernel, the instances in pages
// that are a step's only launch and raise the lengths as well (LengthRaise).  (Two sets: the instances that do not raise are up
// to 5 % slower where they carry the code along, and another wrapping of the same code moves their registers.)
// Query groups of up to 4 heads: the 16 MFMA columns carry the heads four times, and the softmax work
// of a block is shared out over the copies (larger groups: decode_mxg_kernel).
// PAGED: blocks are found through the block table and every sequence has its own length.
template <bool PAGED>
__global__ __launch_bounds__(256, mx_waves_per_simd(4, PAGED)) void BD_KERNEL(mx)(BD_HOT_PARAMS, MxArgs a) {
  constexpr bool RAISE = BD_RAISE;
  const HotArgs<PAGED, uint8_t> hot(BD_HOT_NAMES, a.k_scales, nullptr);
  __shared__ MergeLdsMx ml;
  const int split = blockIdx.x, hkv = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int seq_len = 0;
  // (the first page's number for the order as given, beside the lengths' load, for batches whose lengths are equal after all:
  // 64 sequences of 3000 tokens 46.9 -> 46.7 us a step, 56 of them 43.0 -> 42.75, where an order as given takes 46.5 and 42.7)
  const int first_entry = PAGED ? scalar_load(hot.block_table + (size_t)blockIdx.z * hot.max_pages + min(split * kWaves + wave, hot.max_pages - 1)) : 0;
  const int b = PAGED ? paged_sequence<RAISE>(hot.seq_lens, lane, seq_len, hot.sorted, hot.second, 0) : blockIdx.z;
  const int col = lane & 15, g = lane >> 4;
  const int head = col & 3, cg = col >> 2;
  const int head0 = hkv * hot.gq;                  // first query head of this workgroup
  const int nheads = min(4, hot.gq);
  const size_t unit = (size_t)b * hot.n_kv_heads + hkv;
  int length = hot.nb;
  long app_bi = -1;   // fused step without an append launch: array index of the block the token goes to
  int app_pos = 0;
  if (PAGED) {
    length = seq_len;
    if (hot.step && length >= 0) {
      // fused step: this step's token counts if the table names a page for it (a preceding kernel
      // has appended it, or, with a.k_new, this launch does); the length is raised only after this kernel
      const int n = length / kBlock;
      const int e = n < hot.max_pages ? scalar_load(hot.block_table + (size_t)b * hot.max_pages + n) : -1;
      const bool ok = e >= 0 && e < hot.num_pages;
      if (hot.append) {
        if (ok) {
          app_bi = (long)e * hot.n_kv_heads + hkv;
          app_pos = length % kBlock;
        } else if (a.status && tid == 0 && split == 0) {
          atomicOr(a.status, 2);   // the token is dropped
        }
      }
      length += ok ? 1 : 0;
    }
    length = max(0, length);
  } else if (hot.append) {
    app_bi = (long)(unit * (hot.nbcap / kBlock) + length / kBlock);
    app_pos = length % kBlock;
    length += 1;
  }
  const int nb = (length + kBlock - 1) / kBlock;
  if (app_bi >= 0 && split == ((nb - 1) / kWaves) % hot.num_splits) mx_append_here(a, unit, (size_t)app_bi, app_pos);
  // blocks are dealt to the splits four at a time (one per wave), round robin: the workgroups of a
  // unit read one contiguous window of the cache at any moment
  const int blk0 = split * kWaves, blk1 = nb, bstep = kWaves * hot.num_splits;
  const int nbcap = hot.nbcap / kBlock;
  const int tok_base = 32 * (col >> 2) + (col & 3);   // row `col` of tile T holds token tok_base + 4T

  i8_t bhi, blo;      // Q[head][32g .. 32g+31] as two fp8 (e4m3) pieces
  int sb_hi, sb_lo;   // their e8m0 block scales
  u4_t kraw[8], vraw[8];
  uint32_t ksc[8];
  u4_t vsc[2];
  // A wave keeps 8 KB in flight, not a whole block: keys (and their scales) of the next block
  // are requested when the current block is done, the values of a block when its keys are about
  // to be consumed.  The waves of a compute unit share one in-order memory pipeline; a shorter
  // queue serves everybody sooner and shortens the ramp at both ends of the kernel.
  // bi = index of a 128-token block in the arrays: unit * nbcap + block, or page * H + KV head
  auto issue_k = [&](size_t bi) {
    const size_t tok0 = bi * kBlock;
#pragma unroll
    for (int T = 0; T < 8; ++T) {
      const size_t t = tok0 + tok_base + 4 * T;
      ksc[T] = *reinterpret_cast<const uint32_t*>(hot.k_params + t * 4);
      kraw[T] = __builtin_nontemporal_load(reinterpret_cast<const u4_t*>(hot.k_codes + t * 64 + 16 * g));
    }
  };
  auto issue_v = [&](size_t bi) {
    const size_t tok0 = bi * kBlock;
#pragma unroll
    for (int half = 0; half < 2; ++half)
      vsc[half] = *reinterpret_cast<const u4_t*>(a.v_scales + (tok0 + 32 * g + 16 * half + 4 * cg) * 4);
    const uint8_t* vp = a.v_codes + bi * (size_t)(kD * 64) + 16 * g;
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
      vraw[mt] = __builtin_nontemporal_load(reinterpret_cast<const u4_t*>(vp + (size_t)(16 * mt + col) * 64));
  };
  // Paged: table entry of block n (-1 past the end of the row), and the first block at or after
  // n, in this wave's stride, whose entry names a page of the pool; entries that do not are
  // skipped and reported in *status.
  auto table_entry = [&](int n) { return n < hot.max_pages ? scalar_load(hot.block_table + (size_t)b * hot.max_pages + n) : -1; };
  auto first_valid = [&](int n, int entry, size_t& bi) {
    while (n < blk1) {
      if (entry >= 0 && entry < hot.num_pages) {
        bi = (size_t)entry * hot.n_kv_heads + hkv;
        break;
      }
      if (a.status && lane == 0) atomicOr(a.status, 1);
      n += bstep;
      entry = n < blk1 ? table_entry(n) : -1;
    }
    return n;
  };
  int blk = blk0 + wave;
  size_t bi = unit * nbcap + blk;
  if (PAGED) blk = first_valid(blk, blk < blk1 ? (b == (int)blockIdx.z && blk < hot.max_pages ? first_entry : table_entry(blk)) : -1, bi);
  if (blk < blk1) issue_k(bi);

  mx_query_operand(head < nheads ? hot.q + ((size_t)b * (hot.gq * hot.n_kv_heads) + head0 + head) * kD + 16 * g : nullptr, bhi, blo,
                   sb_hi, sb_lo);
  LengthRaise raise;
  if (RAISE) raise.arrive(a.raise, b, (int)gridDim.z);

  float m_run = -INFINITY, l_run = 0.0f;
  int e_run = 0;   // largest V exponent byte so far (biased by 127)
  f4_t oacc[8];
#pragma unroll
  for (int mt = 0; mt < 8; ++mt) oacc[mt] = (f4_t){0.f, 0.f, 0.f, 0.f};
  if (RAISE) raise.finish(a.raise, b, (int)gridDim.z, hot, true);

  while (blk < blk1) {
    int nblk = blk + bstep;
    size_t nbi = bi + bstep;
    int next_entry = -1;   // requested a block ahead
    if (PAGED && nblk < blk1) next_entry = table_entry(nblk);
    issue_v(bi);
    // ---- S^T tiles straight from the packed codes; column group cg keeps tiles cg and 4+cg
    float s[2][4];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      f4_t st[4];
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        const int T = 4 * half + tt;
        const i8_t ak = {(int)kraw[T][0], (int)kraw[T][1], (int)kraw[T][2], (int)kraw[T][3], 0, 0, 0, 0};
        const int sa = (int)((ksc[T] >> (8 * g)) & 0xFFu);
        f4_t acc = {0.f, 0.f, 0.f, 0.f};
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(ak, bhi, acc, 4, 0, 0, sa, 0, sb_hi);
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(ak, blo, acc, 4, 0, 0, sa, 0, sb_lo);
        st[tt] = acc;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float lo = cg & 1 ? st[1][r] : st[0][r], hi = cg & 1 ? st[3][r] : st[2][r];
        const int t = blk * kBlock + 32 * g + 16 * half + 4 * cg + r;
        s[half][r] = t < length ? (cg & 2 ? hi : lo) * a.scale_log2 : -INFINITY;   // tokens past the end
      }
    }
    // ---- online softmax (Alg. 1): this lane owns head `head`, tokens 32g + 16*half + 4cg + r
    float bmax = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                       fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
    bmax = head_max<4>(bmax);
    const float m_new = fmaxf(m_run, bmax);
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    m_run = m_new;
    l_run *= alpha;
    const int e_new = max(e_run, wave_max_byte(vsc));
    const float alpha_o = alpha * pow2_clamped(e_run - e_new);
    e_run = e_new;
    if (__any(alpha_o != 1.0f)) {
#pragma unroll
      for (int mt = 0; mt < 8; ++mt) oacc[mt] *= alpha_o;
    }
    float p[2][4];
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[half][r] = __builtin_amdgcn_exp2f(s[half][r] - m_new);
        l_run += p[half][r];
      }
    // ---- O^T += V^T P'_cb for the four 32-channel blocks cb (M tiles 2cb, 2cb+1)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      uint32_t pk[2][2];   // [half][rows 0,1 | rows 2,3] as packed fp16
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        float pe[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int e = (int)((vsc[half][r] >> (8 * cb)) & 0xFFu) - e_run + kPTop;   // <= kPTop
          pe[r] = ldexpf(p[half][r], e);
        }
        pk[half][0] = (uint32_t)f2h(pe[0]) | ((uint32_t)f2h(pe[1]) << 16);
        pk[half][1] = (uint32_t)f2h(pe[2]) | ((uint32_t)f2h(pe[3]) << 16);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int half = j >> 1;
        u4_t pb;
        if ((j & 1) == 0) {
          pb[0] = pk[half][0];
          pb[1] = pk[half][1];
          pb[2] = dpp_u<kRowShl4>(pk[half][0]);
          pb[3] = dpp_u<kRowShl4>(pk[half][1]);
        } else {
          pb[0] = dpp_u<kRowShl8>(pk[half][0]);
          pb[1] = dpp_u<kRowShl8>(pk[half][1]);
          pb[2] = dpp_u<kRowShl12>(pk[half][0]);
          pb[3] = dpp_u<kRowShl12>(pk[half][1]);
        }
        const h8_t bp = __builtin_bit_cast(h8_t, pb);
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) {
          const int mt = 2 * cb + mm;
          const uint32_t w = vraw[mt][j];
          h2_t c0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 0);
          h2_t c1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 1);
          h2_t c2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 2);
          h2_t c3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 3);
          const h8_t av = {c0[0], c0[1], c1[0], c1[1], c2[0], c2[1], c3[0], c3[1]};
          oacc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bp, oacc[mt], 0, 0, 0);
        }
      }
    }
    if (PAGED) nblk = first_valid(nblk, next_entry, nbi);
    if (nblk < blk1) issue_k(nbi);
    blk = nblk;
    bi = nbi;
  }

  // ---- merge the waves of the workgroup (the accumulators go back to the true scale first)
  const float back = pow2_clamped(e_run - 127 - kPTop);
  l_run = head_sum<4>(l_run);
  if (col < 4) {
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) ml.o[wave][col][16 * mt + 4 * g + r] = oacc[mt][r] * back;
    if (g == 0) {
      ml.m[wave][col] = m_run;
      ml.l[wave][col] = l_run;
    }
  }
  __syncthreads();
  {
    const int h = tid >> 6, c0 = 2 * (tid & 63);
    if (h < nheads) {
      float M = ml.m[0][h];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) M = fmaxf(M, ml.m[w][h]);
      float L = 0.f, o0 = 0.f, o1 = 0.f;
      if (M > -INFINITY) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
          const float f = __builtin_amdgcn_exp2f(ml.m[w][h] - M);
          L += f * ml.l[w][h];
          o0 += f * ml.o[w][h][c0];
          o1 += f * ml.o[w][h][c0 + 1];
        }
      }
      const size_t row = ((size_t)split * gridDim.z + b) * a.n_q_heads + head0 + h;
      if (a.out) {   // one split: row == the output row
        store_final_pair(a.out, row * kD + c0, a.out_kind, o0, o1, L);
      } else {
        float2 o = {o0, o1};
        *reinterpret_cast<float2*>(a.part_o + row * kD + c0) = o;
        if ((tid & 63) == 0) {
          a.part_ml[row * 2] = M;
          a.part_ml[row * 2 + 1] = L;
        }
      }
    }
  }
}


// ---- groups of 5..16 heads per workgroup: GQP = 8 (the 16 MFMA columns carry 8 heads twice) or 16
//
// Every copy of a head's column receives the same S^T.  Copy cg keeps the tiles of its share of
// the block (GQP = 8: the four tiles of half cg, tokens 32g + 16cg .. + 15 of every lane group g;
// GQP = 16: all eight), runs their softmax, and presents their P' as its part of the B operand of
// the second product: the k-steps that contract those tokens, zero in the others.  Nothing moves
// between lanes; the copies' partial O^T are added once, after the loop.  The keys, the values
// and every matrix instruction are shared by all heads, so a group of 8 or 16 costs what a
// group of 4 costs, except for 2x / 4x the softmax work per lane.
template <int GQP, bool PAGED>
__global__ __launch_bounds__(256, mx_waves_per_simd(GQP, PAGED)) void BD_KERNEL(mxg)(BD_HOT_PARAMS, MxArgs a) {
  constexpr bool RAISE = BD_RAISE;
  const HotArgs<PAGED, uint8_t> hot(BD_HOT_NAMES, a.k_scales, nullptr);
  constexpr int COPIES = 16 / GQP;     // 2 or 1
  constexpr int NT = 8 / COPIES;       // S^T tiles a lane keeps
  __shared__ MergeLdsMxG<GQP> ml;
  const int nwg = (hot.gq + GQP - 1) / GQP;        // workgroups per (split, KV head)
  const int split = blockIdx.x, hkv = blockIdx.y / nwg, sub0 = GQP * (blockIdx.y % nwg);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int seq_len = 0;
  const int first_entry = PAGED ? scalar_load(hot.block_table + (size_t)blockIdx.z * hot.max_pages + min(split * kWaves + wave, hot.max_pages - 1)) : 0;
  const int b = PAGED ? paged_sequence<RAISE>(hot.seq_lens, lane, seq_len, hot.sorted, hot.second, 0) : blockIdx.z;
  const int col = lane & 15, g = lane >> 4;
  const int head = col % GQP, cg = col / GQP;
  const int head0 = hkv * hot.gq + sub0;           // first query head of this workgroup
  const int nheads = min(GQP, hot.gq - sub0);
  const size_t unit = (size_t)b * hot.n_kv_heads + hkv;
  int length = hot.nb;
  long app_bi = -1;   // fused step without an append launch (see decode_mx_kernel)
  int app_pos = 0;
  if (PAGED) {
    length = seq_len;
    if (hot.step && length >= 0) {
      const int n = length / kBlock;
      const int e = n < hot.max_pages ? scalar_load(hot.block_table + (size_t)b * hot.max_pages + n) : -1;
      const bool ok = e >= 0 && e < hot.num_pages;
      if (hot.append) {
        if (ok) {
          app_bi = (long)e * hot.n_kv_heads + hkv;
          app_pos = length % kBlock;
        } else if (a.status && tid == 0 && split == 0) {
          atomicOr(a.status, 2);   // the token is dropped
        }
      }
      length += ok ? 1 : 0;
    }
    length = max(0, length);
  } else if (hot.append) {
    app_bi = (long)(unit * (hot.nbcap / kBlock) + length / kBlock);
    app_pos = length % kBlock;
    length += 1;
  }
  const int nb = (length + kBlock - 1) / kBlock;
  if (app_bi >= 0 && split == ((nb - 1) / kWaves) % hot.num_splits) mx_append_here(a, unit, (size_t)app_bi, app_pos);
  // blocks are dealt to the splits four at a time (one per wave), round robin: the workgroups of a
  // unit read one contiguous window of the cache at any moment
  const int blk0 = split * kWaves, blk1 = nb, bstep = kWaves * hot.num_splits;
  const int nbcap = hot.nbcap / kBlock;
  const int tok_base = 32 * (col >> 2) + (col & 3);   // row `col` of tile T holds token tok_base + 4T

  i8_t bhi, blo;
  int sb_hi, sb_lo;
  u4_t kraw[8], vraw[8];
  uint32_t ksc[8];
  u4_t vsc[NT];   // e8m0 scales (4 channel blocks) of this lane's 4 * NT tokens, 4 tokens per register
  auto issue_k = [&](size_t bi) {
    const size_t tok0 = bi * kBlock;
#pragma unroll
    for (int T = 0; T < 8; ++T) {
      const size_t t = tok0 + tok_base + 4 * T;
      ksc[T] = *reinterpret_cast<const uint32_t*>(hot.k_params + t * 4);
      kraw[T] = __builtin_nontemporal_load(reinterpret_cast<const u4_t*>(hot.k_codes + t * 64 + 16 * g));
    }
  };
  auto issue_v = [&](size_t bi) {
    const size_t tok0 = bi * kBlock;
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
      vsc[tt] = *reinterpret_cast<const u4_t*>(a.v_scales + (tok0 + 32 * g + 4 * NT * cg + 4 * tt) * 4);
    const uint8_t* vp = a.v_codes + bi * (size_t)(kD * 64) + 16 * g;
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
      vraw[mt] = __builtin_nontemporal_load(reinterpret_cast<const u4_t*>(vp + (size_t)(16 * mt + col) * 64));
  };
  auto table_entry = [&](int n) { return n < hot.max_pages ? scalar_load(hot.block_table + (size_t)b * hot.max_pages + n) : -1; };
  auto first_valid = [&](int n, int entry, size_t& bi) {
    while (n < blk1) {
      if (entry >= 0 && entry < hot.num_pages) {
        bi = (size_t)entry * hot.n_kv_heads + hkv;
        break;
      }
      if (a.status && lane == 0) atomicOr(a.status, 1);
      n += bstep;
      entry = n < blk1 ? table_entry(n) : -1;
    }
    return n;
  };
  int blk = blk0 + wave;
  size_t bi = unit * nbcap + blk;
  if (PAGED) blk = first_valid(blk, blk < blk1 ? (b == (int)blockIdx.z && blk < hot.max_pages ? first_entry : table_entry(blk)) : -1, bi);
  if (blk < blk1) issue_k(bi);

  mx_query_operand(head < nheads ? hot.q + ((size_t)b * (hot.gq * hot.n_kv_heads) + head0 + head) * kD + 16 * g : nullptr, bhi, blo,
                   sb_hi, sb_lo);
  LengthRaise raise;
  if (RAISE) raise.arrive(a.raise, b, (int)gridDim.z);

  float m_run = -INFINITY, l_run = 0.0f;
  int e_run = 0;   // largest V exponent byte so far (biased by 127)
  f4_t oacc[8];
#pragma unroll
  for (int mt = 0; mt < 8; ++mt) oacc[mt] = (f4_t){0.f, 0.f, 0.f, 0.f};
  if (RAISE) raise.finish(a.raise, b, (int)gridDim.z, hot, true);

  while (blk < blk1) {
    int nblk = blk + bstep;
    size_t nbi = bi + bstep;
    int next_entry = -1;
    if (PAGED && nblk < blk1) next_entry = table_entry(nblk);
    issue_v(bi);
    // ---- S^T tiles straight from the packed codes; copy cg keeps tiles NT*cg .. NT*cg + NT-1
    float s[NT][4];
#pragma unroll
    for (int T = 0; T < 8; ++T) {
      const i8_t ak = {(int)kraw[T][0], (int)kraw[T][1], (int)kraw[T][2], (int)kraw[T][3], 0, 0, 0, 0};
      const int sa = (int)((ksc[T] >> (8 * g)) & 0xFFu);
      f4_t acc = {0.f, 0.f, 0.f, 0.f};
      acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(ak, bhi, acc, 4, 0, 0, sa, 0, sb_hi);
      acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(ak, blo, acc, 4, 0, 0, sa, 0, sb_lo);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int t = blk * kBlock + 32 * g + 4 * T + r;
        const float v = t < length ? acc[r] * a.scale_log2 : -INFINITY;   // tokens past the end
        if (T < NT) s[T][r] = v;                      // (first half: kept where cg == 0)
        else s[T - NT][r] = cg ? v : s[T - NT][r];    // the second half replaces it in the other copy
      }
    }
    // ---- online softmax (Alg. 1): this lane owns head `head`, tokens 32g + 4*NT*cg + 4tt + r
    float bmax = s[0][0];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
      for (int r = 0; r < 4; ++r) bmax = fmaxf(bmax, s[tt][r]);
    bmax = head_max<COPIES>(bmax);
    const float m_new = fmaxf(m_run, bmax);
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    m_run = m_new;
    l_run *= alpha;
    const int e_new = max(e_run, wave_max_byte(vsc));
    const float alpha_o = alpha * pow2_clamped(e_run - e_new);
    e_run = e_new;
    if (__any(alpha_o != 1.0f)) {
#pragma unroll
      for (int mt = 0; mt < 8; ++mt) oacc[mt] *= alpha_o;
    }
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[tt][r] = __builtin_amdgcn_exp2f(s[tt][r] - m_new);
        l_run += s[tt][r];
      }
    // ---- O^T += V^T P'_cb for the four 32-channel blocks cb (M tiles 2cb, 2cb+1)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      uint32_t pk[NT][2];   // [tile][rows 0,1 | rows 2,3] as packed fp16
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        float pe[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int e = (int)((vsc[tt][r] >> (8 * cb)) & 0xFFu) - e_run + kPTop;   // <= kPTop
          pe[r] = ldexpf(s[tt][r], e);
        }
        pk[tt][0] = (uint32_t)f2h(pe[0]) | ((uint32_t)f2h(pe[1]) << 16);
        pk[tt][1] = (uint32_t)f2h(pe[2]) | ((uint32_t)f2h(pe[3]) << 16);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        // k-step j contracts tokens 32g + 8j .. + 7: tiles 2j and 2j+1, owned by copy 2j / NT
        const int jo = j % (NT / 2);
        u4_t pb = {pk[2 * jo][0], pk[2 * jo][1], pk[2 * jo + 1][0], pk[2 * jo + 1][1]};
        if (COPIES > 1 && (2 * j) / NT != cg) pb = (u4_t){0u, 0u, 0u, 0u};
        const h8_t bp = __builtin_bit_cast(h8_t, pb);
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) {
          const int mt = 2 * cb + mm;
          const uint32_t w = vraw[mt][j];
          h2_t c0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 0);
          h2_t c1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 1);
          h2_t c2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 2);
          h2_t c3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, 3);
          const h8_t av = {c0[0], c0[1], c1[0], c1[1], c2[0], c2[1], c3[0], c3[1]};
          oacc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bp, oacc[mt], 0, 0, 0);
        }
      }
    }
    if (PAGED) nblk = first_valid(nblk, next_entry, nbi);
    if (nblk < blk1) issue_k(nbi);
    blk = nblk;
    bi = nbi;
  }

  // ---- the copies' partial O^T, then the waves of the workgroup
  const float back = pow2_clamped(e_run - 127 - kPTop);   // the accumulators go back to the true scale
  l_run = head_sum<COPIES>(l_run);
  if (COPIES == 2) {
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) oacc[mt][r] += dpp_f<kRowShl8>(oacc[mt][r]);
  }
  if (col < GQP) {
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) ml.o[wave][col][16 * mt + 4 * g + r] = oacc[mt][r] * back;
    if (g == 0) {
      ml.m[wave][col] = m_run;
      ml.l[wave][col] = l_run;
    }
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < GQP / 4; ++p) {
    const int h = 4 * p + wave, c0 = 2 * (tid & 63);
    if (h < nheads) {
      float M = ml.m[0][h];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) M = fmaxf(M, ml.m[w][h]);
      float L = 0.f, o0 = 0.f, o1 = 0.f;
      if (M > -INFINITY) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
          const float f = __builtin_amdgcn_exp2f(ml.m[w][h] - M);
          L += f * ml.l[w][h];
          o0 += f * ml.o[w][h][c0];
          o1 += f * ml.o[w][h][c0 + 1];
        }
      }
      const size_t row = ((size_t)split * gridDim.z + b) * a.n_q_heads + head0 + h;
      if (a.out) {   // one split: row == the output row
        store_final_pair(a.out, row * kD + c0, a.out_kind, o0, o1, L);
      } else {
        float2 o = {o0, o1};
        *reinterpret_cast<float2*>(a.part_o + row * kD + c0) = o;
        if ((tid & 63) == 0) {
          a.part_ml[row * 2] = M;
          a.part_ml[row * 2 + 1] = L;
        }
      }
    }
  }
}
