// The kernel of bd_decode_grp.hip, included twice there: as decode_*_kernel, and, with BD_RAISE, as step_*_kernel, the instances in pages
// that are a step's only launch and raise the lengths as well (LengthRaise).  (Two sets: the instances that do not raise are up
// to 5 % slower where they carry the code along, and another wrapping of the same code moves their registers.)
// G: quantization group (64 or 32).  GQP: heads per workgroup, padded to 4 or 8 (larger query groups
// take ceil(g_q / 8) workgroups per split and KV head; 16 heads' LDS scratch would not fit); MFMA
// column c carries head c % GQP (the copies compute the same numbers).
// PAGED: blocks are found through the block table and every sequence has its own length.
// KT: K is quantized per token and channel group like V (parameters [token][D/G]):
//   S[t, h] = sum_g s_(t,g) * (sum_{c in g} code_tc Q_c) + sum_g z_(t,g) * (sum_{c in g} Q_c).
//   A lane group holds 32 consecutive channels of a token and the matrix instruction sums over the lane
//   groups, so the channel groups are kept apart in the COLUMNS instead: Q' = Q (normalised, fp16 high + low
//   pair, prepared once per kernel) enters 2 * NG "virtual columns" per head -- (piece, channel group), zero
//   in the lane groups outside that channel group -- which the COPIES copies of the head's column carry in
//   2 * NG / COPIES chains of MFMAs; each partial product is scaled with the (token, channel group)
//   parameters in fp32 and the copies are added with DPP row rotations, after which every copy holds S^T as
//   in the channel-wise case.
template <int BITS, int G, int GQP, bool PAGED, bool KT>
__global__ __launch_bounds__(256, grp_waves_per_simd(BITS, G, GQP, KT)) void BD_KERNEL(grp)(BD_HOT_PARAMS, GrpArgs a) {
  constexpr bool RAISE = BD_RAISE;
  const HotArgs<PAGED> hot(BD_HOT_NAMES, a.k_params, a.k_res);
  // With one wave per SIMD nothing but the wave's own arithmetic hides its memory latency, so it
  // requests a block's values before its keys are consumed and the next block's keys right after
  // ("deep").  With two waves the other one covers and the short queue of the group-128 kernel is
  // better (measured, groups of 64: 13.2 against 13.7 us at 32K, 30.9 against 33.2 us at 128K),
  // except for 2-bit codes, whose blocks are half the bytes (42.9 against 45.3 us at 8 x 32K) -- but not for
  // per-token K in groups of 32 at 2 bits, where the deep queue's registers would spill.
  constexpr bool kDeep = (BITS == 2 && !(KT && G == 32)) || grp_waves_per_simd(BITS, G, GQP, KT) == 1;
  using F = Fmt<BITS>;
  constexpr int WORDS = F::WORDS;
  constexpr int KROW = kD * BITS / 32;       // K words per token
  constexpr int VROW = kBlock * BITS / 32;   // V words per channel per block
  constexpr int NG = kBlock / G;             // token groups per block == channel groups per token
  constexpr int NV = NG;
  constexpr int HP = GQP / 4;
  constexpr int COPIES = 16 / GQP;           // MFMA columns per head
  static_assert(COPIES >= 2 && COPIES % 2 == 0, "the high / low pieces of Q' need an even number of copies");
  constexpr int OWN = 4 / COPIES;            // 32-token chunks whose softmax a lane runs
  // token groups whose Q' is made at a time: all four of 8 heads would leave no LDS for a second workgroup
  constexpr int QB = GQP * NG > 16 && grp_waves_per_simd(BITS, G, GQP, KT) > 1 ? 2 : NG;
  using WL = GrpWaveLds<GQP, NV, QB, KT>;
  constexpr int CH = KT ? 2 * NG / COPIES : 0;   // per-token K: MFMA chains per S^T tile
  static_assert(!KT || (2 * NG) % COPIES == 0, "virtual columns per head must fill the copies");
  using ML = GrpMergeLds<GQP, NV>;

  __shared__ __attribute__((aligned(16))) unsigned char smem_raw[gmax(sizeof(ML), kWaves * sizeof(WL))];
  __shared__ float res_o[GQP][kD], res_m[GQP], res_l[GQP];   // result of the residual slice
  // queries * softmax_scale * log2(e), each head brought below 2^kQTop by a power of two whose inverse is
  // qinv_s[head]; padding heads zero
  __shared__ __attribute__((aligned(16))) float q_s[GQP][kD];
  __shared__ float qinv_s[GQP];

  const bool flush_after = hot.flush_mode == kFlushAfter || (PAGED && hot.flush_mode == kFlushLast);
  int split = (int)blockIdx.x - (hot.flush_mode == kFlushAfter ? 1 : 0);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int seq_len = 0;
  int b = blockIdx.z;
  if (PAGED && !paged_workgroup<RAISE>(hot, lane, split, b, seq_len)) return;
  const int col = lane & 15, g = lane >> 4;
  // Every copy of a head's column receives the same S^T; copy cp keeps the chunks c with
  // c % COPIES == cp, runs their softmax and writes their P', so that work is shared out.
  const int head = col % GQP, cp = col / GQP;
  int hkv = blockIdx.y, head0 = 0;
  if (hot.gq > kGrpHeads) {
    const int nchunk = (hot.gq + kGrpHeads - 1) / kGrpHeads;
    hkv = blockIdx.y / nchunk;
    head0 = kGrpHeads * (blockIdx.y % nchunk);
  }
  const int gq = min(hot.gq - head0, kGrpHeads);
  WL& wl = reinterpret_cast<WL*>(smem_raw)[wave];

  const size_t unit = (size_t)b * hot.n_kv_heads + hkv;
  int nb = hot.nb, res_len = hot.res_len;
  int new_slot = hot.new_slot;   // fused step: residual slot of the token that is still in the caller's buffer, or -1
  int flush_page = -1;         // paged fused step that fills the residual: the page the block goes to
  if (PAGED) {
    int len = seq_len;
    new_slot = -1;
    if (hot.step && len >= 0) {
      // fused step: this step's token counts (unless it needs a page the table does not name) and
      // the length is raised only after this kernel.  With a.k_new no kernel has appended the token:
      // it is read from the caller's buffer and filed by this launch, and if it fills the residual,
      // the workgroup that reads the new block quantizes it first (as in the main kernel).
      bool ok = true;
      int e = -1;
      if (len % kBlock == kBlock - 1) {
        const int n = len / kBlock;
        e = n < hot.max_pages ? scalar_load(hot.block_table + (size_t)b * hot.max_pages + n) : -1;
        ok = e >= 0 && e < hot.num_pages;
      }
      if (hot.append) {
        if (!ok) {
          if (a.status && tid == 0 && split == 0) atomicOr(a.status, 2);   // the token is dropped
        } else if (len % kBlock < kBlock - 1) {
          new_slot = len % kBlock;
        } else {
          flush_page = e;
        }
      }
      len += ok ? 1 : 0;
    }
    len = len < 0 ? 0 : len;
    nb = len / kBlock;
    res_len = len % kBlock;
    if (flush_after && flush_page >= 0) {   // lazy flush: this step attends the 128 residual rows in fp16
      nb -= 1;
      res_len = kBlock;
      new_slot = kBlock - 1;
    }
  }
  // blocks are dealt to the splits four at a time (one per wave), round robin: the workgroups of a
  // unit read one contiguous window of the cache at any moment
  const int blk0 = split * kWaves, blk1 = nb, bstep = kWaves * hot.num_splits;
  LengthRaise raise;
  if (RAISE && split < 0) {   // a packing workgroup: it has read what it needs
    raise.arrive(a.raise, b, a.batch);
    raise.finish(a.raise, b, a.batch, hot, false);
  }
  if (flush_after && split < 0 && head0 != 0) return;   // (one quantizing workgroup per KV head is enough)
  if (!PAGED && hot.flush_mode != kFlushNone && head0 == 0 &&
      (flush_after ? split < 0 : split == (a.flush_blk / kWaves) % hot.num_splits)) {
    // the step's token completes the residual block: file it, then pack the 128 rows as block flush_blk
    // (kFlushFirst: this workgroup is the block's only reader in this launch -- up to 8 heads per KV head)
    uint16_t* kr = const_cast<uint16_t*>(hot.k_res) + unit * kBlock * kD;
    uint16_t* vr = const_cast<uint16_t*>(a.v_res) + unit * kBlock * kD;
    if (tid < 32) {
      const bool is_v = tid >= 16;
      const uint16_t* src = (is_v ? a.v_new : a.k_new) + unit * kD + 8 * (tid & 15);
      *reinterpret_cast<u4_t*>((is_v ? vr : kr) + (kBlock - 1) * kD + 8 * (tid & 15)) = *reinterpret_cast<const u4_t*>(src);
    }
    workgroup_global_sync();
    quant_block<BITS, KT, G>(kr, vr, const_cast<uint32_t*>(hot.k_codes), const_cast<uint32_t*>(a.v_codes),
                             const_cast<uint32_t*>(hot.k_params), const_cast<uint32_t*>(a.v_params),
                             unit * hot.nbcap + a.flush_blk);
    if (flush_after) return;   // (the whole workgroup: split < 0 is uniform)
    workgroup_global_sync();
  }
  if (PAGED && flush_after && split < 0) {
    // lazy flush: the extra workgroup of a (sequence, KV head) packs the 128 rows into the page if this
    // step's token completes them, and does nothing else
    if (flush_page >= 0 && head0 == 0) {
      uint16_t* kr = const_cast<uint16_t*>(hot.k_res) + unit * kBlock * kD;
      uint16_t* vr = const_cast<uint16_t*>(a.v_res) + unit * kBlock * kD;
      if (tid < 32) {
        const bool is_v = tid >= 16;
        const uint16_t* src = (is_v ? a.v_new : a.k_new) + unit * kD + 8 * (tid & 15);
        *reinterpret_cast<u4_t*>((is_v ? vr : kr) + (kBlock - 1) * kD + 8 * (tid & 15)) = *reinterpret_cast<const u4_t*>(src);
      }
      workgroup_global_sync();
      quant_block<BITS, KT, G>(kr, vr, const_cast<uint32_t*>(hot.k_codes), const_cast<uint32_t*>(a.v_codes),
                               const_cast<uint32_t*>(hot.k_params), const_cast<uint32_t*>(a.v_params),
                               (size_t)flush_page * hot.n_kv_heads + hkv);
    }
    return;
  }
  if (PAGED && !flush_after && flush_page >= 0 && split == ((nb - 1) / kWaves) % hot.num_splits) {
    // the 128 residual rows become block nb - 1, which this workgroup alone reads in this launch (one
    // workgroup per split and KV head: the host takes this path for up to 8 heads per KV head)
    uint16_t* kr = const_cast<uint16_t*>(hot.k_res) + unit * kBlock * kD;
    uint16_t* vr = const_cast<uint16_t*>(a.v_res) + unit * kBlock * kD;
    if (tid < 32) {
      const bool is_v = tid >= 16;
      const uint16_t* src = (is_v ? a.v_new : a.k_new) + unit * kD + 8 * (tid & 15);
      *reinterpret_cast<u4_t*>((is_v ? vr : kr) + (kBlock - 1) * kD + 8 * (tid & 15)) = *reinterpret_cast<const u4_t*>(src);
    }
    workgroup_global_sync();
    quant_block<BITS, KT, G>(kr, vr, const_cast<uint32_t*>(hot.k_codes), const_cast<uint32_t*>(a.v_codes),
                                const_cast<uint32_t*>(hot.k_params), const_cast<uint32_t*>(a.v_params),
                                (size_t)flush_page * hot.n_kv_heads + hkv);
    workgroup_global_sync();
  }
  const int rt0 = residual_bound(res_len, split, hot.num_splits, a.res_scale), rt1 = residual_bound(res_len, split + 1, hot.num_splits, a.res_scale);
  const uint16_t* qbase = hot.q + ((size_t)b * (hot.gq * hot.n_kv_heads) + hkv * hot.gq + head0) * kD;

  // rows of the residual slice: the newest token of a fused step is read from where the caller left it
  const int nres = rt1 - rt0;
  const uint16_t *kres = hot.k_res + unit * kBlock * kD, *vres = a.v_res + unit * kBlock * kD;
  ResidualRows rows;
  rows.new_at = new_slot >= 0 ? new_slot - rt0 : -1;
  rows.k = kres + (size_t)rt0 * kD;
  rows.v = vres + (size_t)rt0 * kD;
  rows.kn = a.k_new + ((long)unit - rows.new_at) * kD;
  rows.vn = a.v_new + ((long)unit - rows.new_at) * kD;
  constexpr bool kResidualFirst = grp_waves_per_simd(BITS, G, GQP, KT) > 1 && (PAGED || !KT);   // (see below)
  ResidualSlice res;
  if (!kResidualFirst && nres > 0) res.start(qbase, gq, nres, rows, wave, lane);

  // ---- queries, scaled, for everybody in the workgroup
#pragma unroll
  for (int p = 0; p < HP; ++p) {
    const int h = 4 * p + wave;
    const uint32_t raw = h < gq ? *reinterpret_cast<const uint32_t*>(qbase + h * kD + 2 * lane) : 0u;
    float2 qq = {h2f((uint16_t)(raw & 0xFFFFu)) * a.scale_log2, h2f((uint16_t)(raw >> 16)) * a.scale_log2};
    const uint32_t mb = wave_max_u(max(__float_as_uint(fabsf(qq.x)), __float_as_uint(fabsf(qq.y))));
    const int kq = mb ? min(max(kQTop - 1 - ((int)(mb >> 23) - 127), -60), 60) : 0;   // max |q| * 2^kq < 2^kQTop
    const float up = pow2i(kq);
    qq.x *= up;
    qq.y *= up;
    *reinterpret_cast<float2*>(&q_s[h][2 * lane]) = qq;
    if (lane == 0) qinv_s[h] = pow2i(-kq);
  }
  if (RAISE) raise.arrive(a.raise, b, a.batch);

  if (new_slot >= 0 && split == 0 && head0 == 0 && tid < 32 && res_len < kBlock && (PAGED || hot.flush_mode == kFlushNone)) {   // fused step: file the new token for later steps
    const bool is_v = tid >= 16;
    const uint16_t* src = (is_v ? a.v_new : a.k_new) + unit * kD + 8 * (tid & 15);
    uint16_t* dst = const_cast<uint16_t*>(is_v ? a.v_res : hot.k_res) + (unit * kBlock + new_slot) * kD + 8 * (tid & 15);
    *reinterpret_cast<u4_t*>(dst) = *reinterpret_cast<const u4_t*>(src);
  }
  __syncthreads();   // q_s is complete

  float m_run = -INFINITY, l_run = 0.0f;
  float z_run[NV];
  // Channel group v's products accumulate in units of 2^(e_run[v] - 15): e_run is the largest exponent field
  // seen so far among the group's (fp16) V scales, so that scale * 2^(15 - e_run) < 2 whatever the magnitude
  // of V, and the accumulators are rescaled when it grows, together with the softmax's own rescaling.
  int e_run[NV];
  f4_t xacc[NV], oacc[8];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    z_run[v] = 0.0f;
    e_run[v] = 0;
    xacc[v] = (f4_t){0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int mt = 0; mt < 8; ++mt) oacc[mt] = (f4_t){0.f, 0.f, 0.f, 0.f};

  // Row rho = 4*gamma + r of S^T tile T = 2*chunk + run holds block token run_base(4*chunk + gamma, run) + r:
  // the tile lies inside one 32-token chunk, and lane group g ends up with exactly the 8 tokens
  // (slot group 4*chunk + g) that one 16-byte piece of the second product's B operand holds.
  const int row_gamma = col >> 2, row_r = col & 3;
  const int prep_sg = lane & 15;
  const int run0 = F::run_base(prep_sg, 0), run1 = F::run_base(prep_sg, 1);
  RawTile<WORDS> kraw[8], vraw[8];
  u4_t kp0, kp1;              // K parameters (half2) of this lane's two channel runs, token group g % NG
  uint32_t vp[2 * NV];        // V parameters (half2) of tokens 2*lane, 2*lane+1, per channel group

  uint32_t ktp[KT ? 2 * NV : 1];   // per-token K: K parameters (half2) of tokens 2*lane, 2*lane+1, per channel group
  auto issue_params = [&](size_t bi) {
    if constexpr (KT) {
      const uint32_t* kpp = hot.k_params + (bi * kBlock + 2 * lane) * NV;
      if constexpr (NV == 4) {
        const u4_t x = *reinterpret_cast<const u4_t*>(kpp), y = *reinterpret_cast<const u4_t*>(kpp + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          ktp[i] = x[i];
          ktp[4 + i] = y[i];
        }
      } else {
        const u4_t x = *reinterpret_cast<const u4_t*>(kpp);
#pragma unroll
        for (int i = 0; i < 4; ++i) ktp[i] = x[i];
      }
    } else {
      // lane group g fetches token group g % NG, whose Q' it makes (its 16 lanes cover the 128 channels)
      const uint32_t* pp = hot.k_params + (bi * NG + (g % NG)) * kD;
      kp0 = *reinterpret_cast<const u4_t*>(pp + run0);
      kp1 = *reinterpret_cast<const u4_t*>(pp + run1);
    }
    const uint32_t* vpp = a.v_params + (bi * kBlock + 2 * lane) * NV;
    if constexpr (NV == 4) {
      const u4_t x = *reinterpret_cast<const u4_t*>(vpp), y = *reinterpret_cast<const u4_t*>(vpp + 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        vp[i] = x[i];
        vp[4 + i] = y[i];
      }
    } else {
      const u4_t x = *reinterpret_cast<const u4_t*>(vpp);
#pragma unroll
      for (int i = 0; i < 4; ++i) vp[i] = x[i];
    }
  };
  auto issue_keys = [&](size_t bi) {
    const uint32_t* kp = hot.k_codes + bi * (size_t)(kBlock * KROW) + WORDS * g;
#pragma unroll
    for (int T = 0; T < 8; ++T) {
      const int tok = F::run_base(4 * (T >> 1) + row_gamma, T & 1) + row_r;
      kraw[T] = load_raw<WORDS>(kp + (size_t)tok * KROW);
    }
  };
  auto issue_values = [&](size_t bi, int mt0, int mt1) {
    const uint32_t* vpp = a.v_codes + bi * (size_t)(kD * VROW) + WORDS * g;
#pragma unroll
    for (int mt = mt0; mt < mt1; ++mt) vraw[mt] = load_raw<WORDS>(vpp + (size_t)(16 * mt + col) * VROW);
  };

  // Q' = Q * s_c as an fp16 high + low pair in B-operand order and the zero term sum_c Q_c z_c for the token groups
  // tg0 .. tg0 + QB - 1.  A lane has its channels' parameters of one token group in registers and makes Q' for that
  // group and every head (two token groups at a time: every other head, since two lane groups share a token group),
  // so scales are converted and normalised once, the token groups are worked on at the same time and their parameters
  // do not pass through LDS.  Before, the wave made one token group's Q' for all heads when a chunk opened it, from
  // parameters in LDS: 4 sequences of 8K tokens in 4 splits, 4 bits, groups of 32 25.6 -> 24.4 us a step, 2 bits, 8 heads
  // per KV head 31.2 -> 29.1; 4 of 4000 tokens, 4 bits, 8 heads 19.7 -> 18.5; one of 32K in 4 splits 76.5 -> 70.9.
  auto prep_queries = [&](int tg0) {
    if constexpr (!KT) {
      const int tg = g % QB;
      u4_t k0 = kp0, k1 = kp1;
      if constexpr (QB < NG) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          k0[i] = __shfl(kp0[i], 16 * (tg0 + tg) + prep_sg);
          k1[i] = __shfl(kp1[i], 16 * (tg0 + tg) + prep_sg);
        }
      }
      // the token group's K scales are brought below 2^kSTop (queries are below 2^kQTop): |Q'| < 2^15
      uint32_t sb = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) sb = max(sb, max(k0[i] & 0xFFFFu, k1[i] & 0xFFFFu));
      const int ek = -norm_exponent(row_max16_u(sb), kSTop);
      const float dn = pow2i(-ek), ksb = pow2i(24 + ek);   // codes enter as code * 2^-24
      float s[8], z[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t pr = i & 1 ? k1[i >> 1] : k0[i >> 1];
        s[i] = h2f((uint16_t)(pr & 0xFFFFu)) * dn * F::un(i >> 1);
        z[i] = h2f((uint16_t)(pr >> 16));
      }
#pragma unroll
      for (int i0 = 0; i0 < GQP * QB / 4; ++i0) {
        const int ph = i0 * (4 / QB) + g / QB;
        const f4_t qa = *reinterpret_cast<const f4_t*>(&q_s[ph][run0]);
        const f4_t qb = *reinterpret_cast<const f4_t*>(&q_s[ph][run1]);
        const float qinv = qinv_s[ph];
        float zsum = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) zsum = __builtin_fmaf(qa[i], z[2 * i], zsum);
#pragma unroll
        for (int i = 0; i < 4; ++i) zsum = __builtin_fmaf(qb[i], z[2 * i + 1], zsum);
        u4_t phi, plo;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float t0 = qa[v] * s[2 * v], t1 = qb[v] * s[2 * v + 1];
          const uint16_t h0 = f2h(t0), h1 = f2h(t1);
          phi[v] = (uint32_t)h0 | ((uint32_t)h1 << 16);
          plo[v] = (uint32_t)f2h(t0 - h2f(h0)) | ((uint32_t)f2h(t1 - h2f(h1)) << 16);
        }
        zsum = row_sum16(zsum) * qinv;
        *reinterpret_cast<u4_t*>(&wl.qs.q[tg][0][ph][8 * prep_sg]) = phi;
        *reinterpret_cast<u4_t*>(&wl.qs.q[tg][1][ph][8 * prep_sg]) = plo;
        if (prep_sg == 0) {
          wl.qs.zq[tg][ph] = zsum;
          wl.qs.ksb[tg][ph] = ksb * qinv;
        }
      }
    }
  };

  // Per-token K: Q' = Q * position factor (no K scale in it), once per kernel, and the sums of Q over each
  // channel group for the zero terms.
  float zq_k[KT ? CH : 1];      // chain k of this lane's copy: sum of Q over its channel group if it carries the high piece, else 0
  float qinv = 1.0f;            // undoes the query's normalisation
  constexpr bool kKeepB = CH == 1;     // the chains' B operands stay in registers when there is one chain, else they are read per chunk
  h8_t bqk[1][4];
  auto chain_operand = [&](int k, int j) -> h8_t {
    if constexpr (KT) {
      const int v = k * COPIES + cp;                       // virtual column: piece v & 1, channel group v >> 1
      const bool live = (g >> (G == 64 ? 1 : 0)) == (v >> 1);
      const uint16_t* row = (v & 1) ? &wl.qlo[head][8 * (4 * g + j)] : &wl.qhi[head][8 * (4 * g + j)];
      return *reinterpret_cast<const h8_t*>(live ? row : wl.zeros);
    }
    return h8_t{};
  };
  // Paged: table entry of block n (-1 past the end of the row), and the first block at or after
  // n, in this wave's stride, whose entry names a page of the pool; entries that do not are
  // skipped and reported in *status.
  auto table_entry = [&](int n) { return n < hot.max_pages ? scalar_load(hot.block_table + (size_t)b * hot.max_pages + n) : -1; };
  auto first_valid = [&](int n, int entry, size_t& idx) {
    while (n < blk1) {
      if (entry >= 0 && entry < hot.num_pages) {
        idx = (size_t)entry * hot.n_kv_heads + hkv;
        break;
      }
      if (a.status && lane == 0) atomicOr(a.status, 1);
      n += bstep;
      entry = n < blk1 ? table_entry(n) : -1;
    }
    return n;
  };
  int blk = blk0 + wave;
  size_t bi = unit * hot.nbcap + blk;
  if (PAGED) blk = first_valid(blk, blk < blk1 ? table_entry(blk) : -1, bi);
  // The residual slice is attended as in the group-128 kernel, its rows requested ahead and the first block on its way
  // meanwhile -- but with two workgroups per compute unit, where the registers of both (and the page's, or the parameters of
  // K by channel) are more than the 256 there are (up to 11 spilled in the loop; now at most 4), it comes first: in pages, 8
  // sequences of up to 8.2K tokens, per-token K, 4 bits, 4 heads, groups of 64 / 32 22.7 -> 22.3 / 26.9 -> 25.4 us, 2 bits,
  // groups of 32 25.5 -> 24.7, groups of 64 with 8 heads 25.3 -> 24.4; contiguous, 16 of 2K tokens, 2 bits, groups of 32
  // 18.1 -> 17.2, of 64 15.1 -> 14.8.  (Per-token K, contiguous, has the registers and is as fast either way; one workgroup
  // per compute unit would lose by it: groups of 32, 8 heads, contiguous 36.6 -> 38.7, in pages 36.6 -> 37.0.)
  if constexpr (kResidualFirst) {
    if (nres > 0) {
      res.start(qbase, gq, nres, rows, wave, lane);
      res.template attend<GQP>(nres, a.scale_log2, *reinterpret_cast<ML*>(smem_raw), res_o, res_m, res_l, wave, lane);
    }
    if (blk < blk1) {
      issue_params(bi);
      issue_keys(bi);
    }
  } else if (blk < blk1) {
    issue_params(bi);
    issue_keys(bi);
    if (nres > 0) res.template attend<GQP>(nres, a.scale_log2, *reinterpret_cast<ML*>(smem_raw), res_o, res_m, res_l, wave, lane);
  } else if (nres > 0) {
    res.template attend<GQP>(nres, a.scale_log2, *reinterpret_cast<ML*>(smem_raw), res_o, res_m, res_l, wave, lane);
  }
  if constexpr (KT) {
    if (lane < 8) wl.zeros[lane] = 0;
#pragma unroll
    for (int p = 0; p < HP; ++p) {
      const int ph = 4 * p + (lane >> 4);
      const f4_t qa = *reinterpret_cast<const f4_t*>(&q_s[ph][run0]);
      const f4_t qb = *reinterpret_cast<const f4_t*>(&q_s[ph][run1]);
      uint16_t qh[8], ql[8];
      float part[2] = {0.0f, 0.0f};
#pragma unroll
      for (int run = 0; run < 2; ++run)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float qc = run ? qb[i] : qa[i];
          const float t = qc * F::un(i);
          const uint16_t hi = f2h(t);
          qh[2 * i + run] = hi;
          ql[2 * i + run] = f2h(t - h2f(hi));
          part[run] += qc;
        }
      u4_t phi, plo;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        phi[v] = (uint32_t)qh[2 * v] | ((uint32_t)qh[2 * v + 1] << 16);
        plo[v] = (uint32_t)ql[2 * v] | ((uint32_t)ql[2 * v + 1] << 16);
      }
      *reinterpret_cast<u4_t*>(&wl.qhi[ph][8 * prep_sg]) = phi;
      *reinterpret_cast<u4_t*>(&wl.qlo[ph][8 * prep_sg]) = plo;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const float x = row_sum16((run0 / G == v ? part[0] : 0.0f) + (run1 / G == v ? part[1] : 0.0f));
        if (prep_sg == 0) wl.qsum[ph][v] = x;
      }
    }
    wave_sync();
    qinv = qinv_s[head];
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      const int v = k * COPIES + cp;
      zq_k[k] = (v & 1) ? 0.0f : wl.qsum[head][v >> 1];
    }
    if constexpr (kKeepB) {
#pragma unroll
      for (int j = 0; j < 4; ++j) bqk[0][j] = chain_operand(0, j);
    }
  }
  if (RAISE) raise.finish(a.raise, b, a.batch, hot, false);
  // this lane's 8 tokens of chunk c are block tokens tok0 + 32*c + {run_base offsets}: slot group 4*c + g
  while (blk < blk1) {
    int nblk = blk + bstep;
    size_t nbi = bi + bstep;
    if (PAGED) nblk = first_valid(nblk, nblk < blk1 ? table_entry(nblk) : -1, nbi);
    const bool has_next = nblk < blk1;
    if constexpr (kDeep) issue_values(bi, 0, 8);
    if constexpr (KT) {   // K parameters of the block's tokens, per channel group
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const uint32_t pr = ktp[u * NV + v];
          wl.ktpar[v][par_slot(2 * lane + u)] = make_float2(h2f((uint16_t)(pr & 0xFFFFu)) * kTwo24, h2f((uint16_t)(pr >> 16)));
        }
    }
    // ---- V parameters of the block's tokens, per channel group
    int e_new[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v)
      e_new[v] = max(e_run[v], (int)(wave_max_u(max(vp[v] & 0x7FFFu, vp[NV + v] & 0x7FFFu)) >> 10));
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const uint32_t pr = vp[u * NV + v];
        const float sv = h2f((uint16_t)(pr & 0xFFFFu)), zv = h2f((uint16_t)(pr >> 16));
        const int t = 2 * lane + u;
        const int r = t & 3;
        const float ct = sv > 0.0f ? rintf(fminf(fmaxf(-zv * __builtin_amdgcn_rcpf(sv), 0.0f), F::kQmax)) : 0.0f;
        wl.vpar[v][par_slot(t)] = make_float2(sv * pow2i(15 - e_new[v]) * F::un(r), __builtin_fmaf(ct, sv, zv));
        wl.c16[v][F::operand_pos(t)] = (uint16_t)(ct * F::inv_un(r));   // an integer: the fp16 subnormal code * 2^-24
      }
    // ---- S^T, chunk by chunk
    float sc[OWN][2][4];   // [owned chunk][run][row]
    h8_t bq[4];   // the high piece of Q' in the even copies of a head's column, the low piece in the odd ones
    float zq = 0.0f, ksb = 0.0f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      __builtin_amdgcn_sched_barrier(0);
      // the short queue: values into the registers that the chunk before has left (all of them behind the last chunk: one of
      // 32K tokens, 4 bits, groups of 32, 4 splits 70.9 -> 69.7 us, 4 of 8K, groups of 64, 4 splits 20.4 -> 19.6)
      if (!kDeep && c > 0) issue_values(bi, 2 * c - 2, 2 * c);
      if constexpr (KT) {
        if (c == 0) wave_sync();   // the block's K parameters are staged
        h8_t bload[kKeepB ? 1 : CH][4];
        if constexpr (!kKeepB) {
#pragma unroll
          for (int k = 0; k < CH; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) bload[k][j] = chain_operand(k, j);
        }
        auto bop = [&](int k, int j) -> h8_t {
          if constexpr (!kKeepB) return bload[k][j];
          else return bqk[k][j];
        };
        const bool mine = c % COPIES == cp;
#pragma unroll
        for (int run = 0; run < 2; ++run) {
          const int T = 2 * c + run;
          h8_t ak[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) ak[j] = F::dequant(kraw[T].w, j);
          float val[4] = {0.f, 0.f, 0.f, 0.f};
          const int slot = par_slot(F::run_base(4 * c + g, run));
#pragma unroll
          for (int k = 0; k < CH; ++k) {
            f4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < 4; ++j)
              acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(ak[j], bop(k, j), acc, 0, 0, 0);
            const float2* par = &wl.ktpar[(k * COPIES + cp) >> 1][slot];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float2 sz = par[r];
              val[r] = __builtin_fmaf(sz.x, acc[r], __builtin_fmaf(sz.y, zq_k[k], val[r]));
            }
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float x = val[r];
            if (COPIES == 4) x += dpp_f<kRowRor4>(x);
            if (COPIES >= 2) x += dpp_f<kRowRor8>(x);
            x *= qinv;
            sc[c / COPIES][run][r] = mine ? x : sc[c / COPIES][run][r];
          }
        }
      } else {
        if ((32 * c) % (G * QB) == 0) {
          if (c > 0) wave_sync();   // the previous Q' has been read by every lane
          prep_queries((32 * c) / G);
          wave_sync();
        }
        if ((32 * c) % G == 0) {   // the chunk opens a token group
          const int tg = (32 * c) / G % QB;
#pragma unroll
          for (int j = 0; j < 4; ++j) bq[j] = *reinterpret_cast<const h8_t*>(&wl.qs.q[tg][cp & 1][head][8 * (4 * g + j)]);
          zq = wl.qs.zq[tg][head];
          ksb = wl.qs.ksb[tg][head];
        }
#pragma unroll
        for (int run = 0; run < 2; ++run) {
          const int T = 2 * c + run;
          f4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const h8_t ak = F::dequant(kraw[T].w, j);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(ak, bq[j], acc, 0, 0, 0);
          }
          // the chunk's owner (copy c % COPIES) adds the other piece's partial product, which the
          // neighbouring copy computed: GQP lanes up for an even owner, GQP lanes down for an odd one
          const bool mine = c % COPIES == cp;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float x = acc[r];
            if (c & 1) x += dpp_f<GQP == 4 ? kRowShr4 : kRowShr8>(x);
            else x += dpp_f<GQP == 4 ? kRowShl4 : kRowShl8>(x);
            const float val = __builtin_fmaf(x, ksb, zq);
            sc[c / COPIES][run][r] = mine ? val : sc[c / COPIES][run][r];
          }
        }
      }
    }
    if constexpr (!kDeep) issue_values(bi, 6, 8);
    if (kDeep && has_next) {   // parameters first: they are the next block's first consumers
      issue_params(nbi);
      issue_keys(nbi);
    }
    // ---- online softmax (Alg. 1) over this lane's 8 * OWN tokens of head `head`
    float bmax = sc[0][0][0];
#pragma unroll
    for (int o = 0; o < OWN; ++o)
#pragma unroll
      for (int run = 0; run < 2; ++run)
#pragma unroll
        for (int r = 0; r < 4; ++r) bmax = fmaxf(bmax, sc[o][run][r]);
    bmax = head_max<COPIES>(bmax);
    const float m_new = fmaxf(m_run, bmax);
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on the first block (m_run = -inf)
    m_run = m_new;
    l_run *= alpha;
    bool grew = false;
#pragma unroll
    for (int v = 0; v < NV; ++v) grew |= e_new[v] != e_run[v];
    if (grew || __any(alpha != 1.0f)) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const float av = alpha * pow2i(e_run[v] - e_new[v]);
#pragma unroll
        for (int mm = 0; mm < 8 / NV; ++mm) oacc[v * (8 / NV) + mm] *= av;
        xacc[v] *= av;
        z_run[v] *= alpha;
        e_run[v] = e_new[v];
      }
    }
#pragma unroll
    for (int o = 0; o < OWN; ++o)
#pragma unroll
      for (int run = 0; run < 2; ++run)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          sc[o][run][r] = __builtin_amdgcn_exp2f(sc[o][run][r] - m_new);
          l_run += sc[o][run][r];
        }
    // ---- O^T += V^T P'_v, one channel group after the other
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      __builtin_amdgcn_sched_barrier(0);   // one variant at a time: interleaving them costs a wave per SIMD in registers
      wave_sync();   // the previous variant (or Q') has been read by every lane
#pragma unroll
      for (int o = 0; o < OWN; ++o) {
        const int sg = 4 * (o * COPIES + cp) + g;   // slot group of this lane's 8 tokens of its o-th chunk
        u4_t w;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          uint32_t hv[2];
#pragma unroll
          for (int run = 0; run < 2; ++run) {
            const float p = sc[o][run][r];
            const float2 par = wl.vpar[v][par_slot(F::run_base(sg, run)) + r];
            z_run[v] = __builtin_fmaf(p, par.y, z_run[v]);
            hv[run] = (uint32_t)f2h(p * par.x);
          }
          w[r] = hv[0] | (hv[1] << 16);   // entries 2r, 2r + 1 of the slot group
        }
        *reinterpret_cast<u4_t*>(&wl.pbuf[head][8 * sg]) = w;   // every (head, slot group) has one owner
      }
      wave_sync();
      h8_t bp[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) bp[j] = *reinterpret_cast<const h8_t*>(&wl.pbuf[head][8 * (4 * g + j)]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const h8_t ac = *reinterpret_cast<const h8_t*>(&wl.c16[v][8 * (4 * g + j)]);
        xacc[v] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ac, bp[j], xacc[v], 0, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int mm = 0; mm < 8 / NV; ++mm) {
          const int mt = v * (8 / NV) + mm;
          oacc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(F::dequant(vraw[mt].w, j), bp[j], oacc[mt], 0, 0, 0);
        }
    }
    if (!kDeep && has_next) {
      issue_params(nbi);
      issue_keys(nbi);
    }
    wave_sync();   // the next block's parameters overwrite this wave's LDS scratch
    blk = nblk;
    bi = nbi;
  }

  // ---- merge the waves of the workgroup (cross-wave step of the cooperative softmax)
  l_run = head_sum<COPIES>(l_run);
#pragma unroll
  for (int v = 0; v < NV; ++v) z_run[v] = head_sum<COPIES>(z_run[v]);
  __syncthreads();   // every wave is done with its per-wave LDS before the space is reused
  ML& ml = *reinterpret_cast<ML*>(smem_raw);
  if (col < GQP) {
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        ml.o[wave][col][16 * mt + 4 * g + r] =
            (oacc[mt][r] - xacc[mt / (8 / NV)][0]) * (kTwo24 * pow2i(e_run[mt / (8 / NV)] - 15));
    if (g == 0) {
      ml.m[wave][col] = m_run;
      ml.l[wave][col] = l_run;
#pragma unroll
      for (int v = 0; v < NV; ++v) ml.z[wave][col][v] = z_run[v];
    }
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < HP; ++p) {
    const int h = 4 * p + wave, c0 = 2 * lane;
    if (h < gq) {
      const int v = c0 / G;   // channel group of channels c0, c0 + 1
      float M = ml.m[0][h];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) M = fmaxf(M, ml.m[w][h]);
      if (nres > 0) M = fmaxf(M, res_m[h]);
      float L = 0.f, Z = 0.f, o0 = 0.f, o1 = 0.f;
      if (M > -INFINITY) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
          const float f = __builtin_amdgcn_exp2f(ml.m[w][h] - M);
          L += f * ml.l[w][h];
          Z += f * ml.z[w][h][v];
          o0 += f * ml.o[w][h][c0];
          o1 += f * ml.o[w][h][c0 + 1];
        }
        if (nres > 0) {
          const float f = __builtin_amdgcn_exp2f(res_m[h] - M);
          L += f * res_l[h];
          o0 += f * res_o[h][c0];
          o1 += f * res_o[h][c0 + 1];
        }
      }
      const size_t row = ((size_t)split * (PAGED ? (uint32_t)a.batch : gridDim.z) + b) * a.n_q_heads + hkv * hot.gq + head0 + h;
      float2 o = {o0 + Z, o1 + Z};
      if (a.out) {   // one split: row == the output row
        store_final_pair(a.out, row * kD + c0, a.out_kind, o.x, o.y, L);
      } else {
        *reinterpret_cast<float2*>(a.part_o + row * kD + c0) = o;
        if (lane == 0) {
          a.part_ml[row * 2] = M;
          a.part_ml[row * 2 + 1] = L;
        }
      }
    }
  }
}
