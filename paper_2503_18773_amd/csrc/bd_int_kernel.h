// The kernel of bd_decode.hip, included three times there: as decode_*_kernel; with BD_RAISE, as step_*_kernel, the instances in
// pages that are a step's only launch and raise the lengths as well (LengthRaise); and in BD_WAVES eight waves, as
// wide_*_kernel (kOneBlockWide).  (Sets of their own: the instances that do not raise are up
// to 5 % slower where they carry the code along, and another wrapping of the same code moves their registers.)
// GQP: the query group padded to 4, 8 or 16 heads; the 16 MFMA columns carry it 16/GQP times
//      (column c holds head c % GQP, "column group" c / GQP) and the softmax work of a block
//      is shared out over the column groups.
//      GQP = 4: see the top of the file; column group cg keeps S^T tiles cg and 4 + cg.
//      GQP = 8, 16: each column group owns 4 / COPIES of the block's four 32-token k-steps of
//      the second product: it keeps the S^T tiles of those tokens, runs their softmax, and
//      presents their P' as its part of the B operand (zero in the k-steps it does not own);
//      no probability moves between lanes, and the column groups' partial O^T are added
//      once, after the loop.
// BLOCKS: kManyBlocks, or no wave has more than one (short contexts): kOneBlock, and no residual slice more than kResShort
//      tokens; kOneBlockSlice, and residual slices of any length (one_block_instance picks).  kOneBlockWide: the same in eight
//      waves, the slice beside the block (wide_instance).
// PAGED: blocks are found through the block table and every sequence has its own length.
// KT: K is quantized per token (Sec. IV-C(1)):  S[t] = s_t * sum_c Q_c code_tc + z_t * sum_c Q_c,
//     so Q' = Q is prepared once per kernel instead of once per block and the per-token scale
//     and zero are applied to the kept S^T values.
template <int BITS, int GQP, int BLOCKS, bool PAGED, bool KT>
__global__ __launch_bounds__(64 * BD_WAVES, 2) void BD_KERNEL(int)(BD_HOT_PARAMS, DecodeArgs a) {
  constexpr bool RAISE = BD_RAISE;
  constexpr int kWaves = BD_WAVES;   // all spread along the token axis (W_m = 1)
  static_assert(kWaves == 4 || (GQP == 4 && BLOCKS == kOneBlockWide && !PAGED && !RAISE), "heads and slices are shared out over four waves");
  const HotArgs<PAGED> hot(BD_HOT_NAMES, a.k_params, a.k_res);
  constexpr bool kSingle = BLOCKS != kManyBlocks, kShortSlices = BLOCKS != kOneBlockSlice, kLongSlices = BLOCKS != kOneBlock;
  using F = Fmt<BITS>;
  using WL = WaveLds<GQP>;
  using ML = MergeLds<GQP, kWaves>;
  constexpr int WORDS = F::WORDS;            // words per lane per tile
  constexpr int KROW = kD * BITS / 32;       // K words per token
  constexpr int VROW = kBlock * BITS / 32;   // V words per channel per block
  constexpr int COPIES = 16 / GQP;           // column groups
  constexpr int OWN = 4 / COPIES;            // k-steps owned by a column group
  constexpr int HP = GQP / 4;                // passes over the heads where 16 lanes work on one head
  constexpr bool kF8 = GQP == 4;             // QK on i8 instructions, PV on f8f6f4 (see the top of bd_decode.hip)
  using E = FmtF8<BITS>;
  using I = FmtI8<BITS>;
  // The next block's keys are requested as soon as this block's are consumed, not at the block's end, where the
  // arithmetic is short or the blocks are (8 x 32K tokens, 2 bits: 32.5 -> 29.3 us, with 8 heads 39.0 -> 37.7; 128K
  // tokens, 4 bits: 26.3 -> 25.8, but with 8 heads 26.8 -> 28.2; up to 4 heads measured with QK on f8f6f4 instructions, Q' in four e4m3
  // pieces).
  constexpr bool kEarly = kF8 || (BITS == 2 && GQP == 8);

  __shared__ __attribute__((aligned(16))) unsigned char smem_raw[cmax(sizeof(ML), kWaves * sizeof(WL))];
  __shared__ float res_o[GQP][kD], res_m[GQP], res_l[GQP];   // result of the residual slice
  __shared__ __attribute__((aligned(16))) float q_s[HP > 1 ? GQP : 1][kD];   // larger groups: queries, normalised; padding heads zero
  __shared__ int kq_s[HP > 1 ? GQP : 1];                                     // larger groups: each head's normalising exponent

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool flush_after = hot.flush_mode == kFlushAfter || (PAGED && hot.flush_mode == kFlushLast);
  int split = (int)blockIdx.x - (hot.flush_mode == kFlushAfter ? 1 : 0);
  int seq_len = 0;
  int b = blockIdx.z;
  if (PAGED && !paged_workgroup<RAISE>(hot, lane, split, b, seq_len)) return;
  const int col = lane & 15, g = lane >> 4;            // MFMA column and contraction group
  const int head = col % GQP, cg = col / GQP;          // head carried by the column; column group
  // Query groups of more than 16 heads are taken 16 at a time by ceil(g_q / 16) workgroups per
  // (split, KV head), each of which reads the cache once.
  int hkv = blockIdx.y, head0 = 0;
  if (GQP == 16 && hot.gq > 16) {
    const int nchunk = (hot.gq + 15) >> 4;
    hkv = blockIdx.y / nchunk;
    head0 = 16 * (blockIdx.y % nchunk);
  }
  const int gq = min(hot.gq - head0, 16);                // heads of this workgroup
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
      // the length is raised only after this kernel.  With a.k_new the token has not been appended
      // by a kernel of its own: it is read from the caller's buffer and filed by this launch, and
      // if it fills the residual, the workgroup that reads the new block quantizes it first.
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
  // Blocks are dealt to the splits four at a time (one per wave), round robin: at any moment the
  // workgroups of a (sequence, KV head) unit read one contiguous window of the cache.  (Contiguous
  // ranges per split put the workgroups' streams a power of two apart for the usual split counts,
  // and then all of them march over the same memory channels.)
  const int blk0 = split * kWaves, blk1 = nb, bstep = kWaves * hot.num_splits;
  LengthRaise raise;
  if (RAISE && split < 0) {   // a packing workgroup: it has read what it needs
    raise.arrive(a.raise, b, a.batch);
    raise.finish(a.raise, b, a.batch, hot, false);
  }
  if (flush_after && split < 0 && head0 != 0) return;   // (one quantizing workgroup per KV head is enough)
  if (!PAGED && hot.flush_mode != kFlushNone && head0 == 0 &&
      (flush_after ? split < 0 : split == (a.flush_blk / kWaves) % hot.num_splits)) {
    // The step's token completes the residual block: file it, then quantize the 128 rows as block
    // flush_blk.  kFlushFirst: this workgroup is the block's only reader in this launch (one workgroup per
    // split and KV head: query groups of up to 16 heads).  kFlushAfter: nobody reads the block here, and
    // the others read the residual rows, which only gain the row they take from k_new / v_new anyway.
    uint16_t* kr = const_cast<uint16_t*>(hot.k_res) + unit * kBlock * kD;
    uint16_t* vr = const_cast<uint16_t*>(a.v_res) + unit * kBlock * kD;
    if (tid < 32) {
      const bool is_v = tid >= 16;
      const uint16_t* src = (is_v ? a.v_new : a.k_new) + unit * kD + 8 * (tid & 15);
      *reinterpret_cast<u4_t*>((is_v ? vr : kr) + (kBlock - 1) * kD + 8 * (tid & 15)) = *reinterpret_cast<const u4_t*>(src);
    }
    workgroup_global_sync();
    if (kWaves == 4 || wave < 4) {
      quant_block<BITS, KT, kBlock>(kr, vr, const_cast<uint32_t*>(hot.k_codes), const_cast<uint32_t*>(a.v_codes),
                                    const_cast<uint32_t*>(hot.k_params), const_cast<uint32_t*>(a.v_params),
                                    unit * hot.nbcap + a.flush_blk);
    } else {
      for (int i = 0; i < quant_block_barriers(KT); ++i) __syncthreads();
    }
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
      quant_block<BITS, KT, kBlock>(kr, vr, const_cast<uint32_t*>(hot.k_codes), const_cast<uint32_t*>(a.v_codes),
                                    const_cast<uint32_t*>(hot.k_params), const_cast<uint32_t*>(a.v_params),
                                    (size_t)flush_page * hot.n_kv_heads + hkv);
    }
    return;
  }
  if (PAGED && !flush_after && flush_page >= 0 && split == ((nb - 1) / kWaves) % hot.num_splits) {
    // This step's token completes the residual (Sec. IV-B(1)): the 128 rows become block nb - 1, which
    // this workgroup alone reads in this launch.  (One workgroup per split and KV head: the host takes
    // this path only for query groups of up to 16 heads.)
    uint16_t* kr = const_cast<uint16_t*>(hot.k_res) + unit * kBlock * kD;
    uint16_t* vr = const_cast<uint16_t*>(a.v_res) + unit * kBlock * kD;
    if (tid < 32) {
      const bool is_v = tid >= 16;
      const uint16_t* src = (is_v ? a.v_new : a.k_new) + unit * kD + 8 * (tid & 15);
      *reinterpret_cast<u4_t*>((is_v ? vr : kr) + (kBlock - 1) * kD + 8 * (tid & 15)) = *reinterpret_cast<const u4_t*>(src);
    }
    workgroup_global_sync();   // the row is read back below, and the block further down, by other threads of this workgroup
    quant_block<BITS, KT, kBlock>(kr, vr, const_cast<uint32_t*>(hot.k_codes), const_cast<uint32_t*>(a.v_codes),
                                  const_cast<uint32_t*>(hot.k_params), const_cast<uint32_t*>(a.v_params),
                                  (size_t)flush_page * hot.n_kv_heads + hkv);
    workgroup_global_sync();
  }
  // this workgroup's slice of the fp16 residual tokens
  const int rt0 = residual_bound(res_len, split, hot.num_splits, a.res_scale), rt1 = residual_bound(res_len, split + 1, hot.num_splits, a.res_scale);
  const uint16_t* qbase = hot.q + ((size_t)b * (hot.gq * hot.n_kv_heads) + hkv * hot.gq + head0) * kD;

  float m_run = -INFINITY;   // running max of this lane's head (log2 units), equal in all lanes of the head
  float l_run = 0.0f;        // running sum of p over this lane's own tokens
  float z_run = 0.0f;        // running sum of p * zero_t over this lane's own tokens
  f4_t xacc = {0.f, 0.f, 0.f, 0.f};   // sum_t P'_t * centre code of token t (every row the same)
  f4_t oacc[8];
#pragma unroll
  for (int mt = 0; mt < 8; ++mt) oacc[mt] = (f4_t){0.f, 0.f, 0.f, 0.f};

  // A wave keeps little in flight: the keys of its next block are requested when the current
  // block is done (kEarly: when its keys are consumed), the values of a block when its keys are about to be consumed.  The eight
  // waves of a compute unit share one in-order memory pipeline, so whatever one wave requests
  // early only delays what the others are waiting for: 8 KB per wave (16 MB over the chip) keeps
  // HBM busy, and a shorter queue shortens the ramp at both ends of the kernel.
  const int prep_sg = lane & 15;
  const int run0 = kF8 ? 8 * prep_sg : F::run_base(prep_sg, 0), run1 = kF8 ? run0 + 4 : F::run_base(prep_sg, 1);
  // block token in row `col` of tile T
  auto row_token = [&](int T) { return (kF8 ? E::token(col >> 2, T) : 32 * (col >> 2) + 4 * T) + (col & 3); };
  auto slot = [&](int t) { return kF8 ? E::par_slot(t) : par_slot(t); };
  RawTile<WORDS> kraw[8], vraw[8];
  u4_t kp0, kp1;   // K parameters (half2) of this lane's two channel runs
  u2_t kp2;        // per-token K: parameters of tokens 2*lane, 2*lane+1
  u2_t vp2;        // V parameters (half2) of tokens 2*lane, 2*lane+1
  // All four take the index `bi` of the block in the packed arrays: unit * nbcap + block for the
  // contiguous cache, page * Hkv + head for the paged one.
  auto issue_kpar = [&](size_t bi) {
    if constexpr (KT) {
      kp2 = *reinterpret_cast<const u2_t*>(hot.k_params + bi * kBlock + 2 * lane);
    } else {
      const uint32_t* pp = hot.k_params + bi * kD;
      kp0 = *reinterpret_cast<const u4_t*>(pp + run0);
      kp1 = *reinterpret_cast<const u4_t*>(pp + run1);
    }
  };
  auto issue_vpar = [&](size_t bi) {
    vp2 = *reinterpret_cast<const u2_t*>(a.v_params + bi * kBlock + 2 * lane);
  };
  auto issue_ktile = [&](size_t bi, int T) {
    const uint32_t* kp = hot.k_codes + bi * (size_t)(kBlock * KROW) + WORDS * g;
    kraw[T] = load_raw<WORDS>(kp + (size_t)row_token(T) * KROW);
  };
  auto issue_vtile = [&](size_t bi, int mt) {
    const uint32_t* vp = a.v_codes + bi * (size_t)(kD * VROW) + WORDS * g;
    vraw[mt] = load_raw<WORDS>(vp + (size_t)(16 * mt + col) * VROW);
  };
  // Loads return in order, so what is needed first is requested first: the queries and this
  // wave's first residual key rows, then the first block.
  // A group of up to 4 heads: every lane keeps the query slice it rescales per block (head
  // lane / 16, two runs of 4 channels) in registers.  Larger groups go through LDS (q_s).
  uint32_t qld[HP];
  u2_t qraw0 = {0u, 0u}, qraw1 = {0u, 0u};
  if constexpr (HP == 1) {
    if ((lane >> 4) < gq) {
      qraw0 = *reinterpret_cast<const u2_t*>(qbase + (lane >> 4) * kD + run0);
      qraw1 = *reinterpret_cast<const u2_t*>(qbase + (lane >> 4) * kD + run1);
    }
  } else {
#pragma unroll
    for (int p = 0; p < HP; ++p) {
      const int h = 4 * p + wave;   // thread tid: head h, channels 2*(tid%64), +1
      qld[p] = h < gq ? *reinterpret_cast<const uint32_t*>(qbase + h * kD + 2 * lane) : 0u;
    }
  }
  // fused step: the new token, which goes to the residual buffers for later steps, at the end of the kernel (a store here
  // would wait for all that is requested above and below)
  const bool files = new_slot >= 0 && split == 0 && head0 == 0 && tid < 32 && res_len < kBlock && (PAGED || hot.flush_mode == kFlushNone);
  const u4_t filed = *reinterpret_cast<const u4_t*>((files ? (tid >= 16 ? a.v_new : a.k_new) + unit * kD : qbase) + 8 * (tid & 15));
  const uint16_t *kres = hot.k_res + unit * kBlock * kD, *vres = a.v_res + unit * kBlock * kD;
  // rows of the residual slice: the newest token of a fused step is read from where the caller left it
  const int nres = rt1 - rt0;
  ResidualRows rows;
  rows.new_at = new_slot >= 0 ? new_slot - rt0 : -1;
  rows.k = kres + (size_t)rt0 * kD;
  rows.v = vres + (size_t)rt0 * kD;
  rows.kn = a.k_new + ((long)unit - rows.new_at) * kD;
  rows.vn = a.v_new + ((long)unit - rows.new_at) * kD;
  ResidualSlice res;
  auto start_slice = [&]() {
    if (nres > 0) res.template start<kShortSlices, kLongSlices, (kWaves > 4)>(qbase, gq, nres, rows, wave, lane);
  };
  auto attend_slice = [&]() {
    if (nres > 0) res.template attend<GQP, kShortSlices, kLongSlices, (kWaves > 4)>(nres, a.scale_log2, *reinterpret_cast<ML*>(smem_raw), res_o, res_m, res_l, wave, lane);
  };
  // (Where exactly the values are requested is fixed at compile time, so that the compiler knows
  // how many loads are in flight behind the one it waits for: half way through QK^T.)
  const int my_blocks = blk1 > blk0 + wave ? (blk1 - blk0 - wave + bstep - 1) / bstep : 0;
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
  size_t bi = unit * hot.nbcap + blk;
  if (PAGED) blk = first_valid(blk, blk < blk1 ? table_entry(blk) : -1, bi);
  constexpr int kBlockLoads = (KT ? 1 : 2) + 1 + 8;   // parameters and key tiles
  auto issue_first = [&]() {   // parameters first: they are the block's first consumers
    issue_kpar(bi);
    issue_vpar(bi);
#pragma unroll
    for (int T = 0; T < 8; ++T) issue_ktile(bi, T);
  };
  // Every head's queries times the power of two that brings the largest below 1 (kq); the factor comes
  // back out of the scores, together with softmax_scale * log2(e) and the 2^24 of the subnormal codes (kS).
  float qv[2][4];
  float fine_from = 0.0f;   // up to 4 heads: kFineScore as a product of head lane / 16
  int kq_head = 0;   // of the head this lane's column carries
  auto scale_queries = [&]() {
    if constexpr (HP > 1) {   // larger groups: for everybody in the workgroup
#pragma unroll
      for (int p = 0; p < HP; ++p) {
        const int h = 4 * p + wave;   // this wave holds all 128 channels of head h
        uint32_t qb = row_max16_u(max(qld[p] & 0x7FFFu, (qld[p] >> 16) & 0x7FFFu));
        qb = max(max(__builtin_amdgcn_readlane(qb, 0), __builtin_amdgcn_readlane(qb, 16)),
                 max(__builtin_amdgcn_readlane(qb, 32), __builtin_amdgcn_readlane(qb, 48)));
        const int kqh = norm_exponent(qb, kQTop);
        const float f = pow2i(kqh);
        float2 qq = {h2f((uint16_t)(qld[p] & 0xFFFFu)) * f, h2f((uint16_t)(qld[p] >> 16)) * f};
        *reinterpret_cast<float2*>(&q_s[h][2 * lane]) = qq;
        if (lane == 0) kq_s[h] = kqh;
      }
      lds_barrier();
      kq_head = kq_s[head];
    } else {
      uint32_t qb = 0;
#pragma unroll
      for (int i = 0; i < 2; ++i)
        qb = max(max(qb, max(qraw0[i] & 0x7FFFu, (qraw0[i] >> 16) & 0x7FFFu)), max(qraw1[i] & 0x7FFFu, (qraw1[i] >> 16) & 0x7FFFu));
      qb = row_max16_u(qb);   // largest |q| of head lane / 16
      const float f = pow2i(norm_exponent(qb, 0));
      fine_from = f * (I::kFineScore / fabsf(a.scale_log2));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        qv[0][i] = h2f((uint16_t)((qraw0[i >> 1] >> (16 * (i & 1))) & 0xFFFFu)) * f;
        qv[1][i] = h2f((uint16_t)((qraw1[i >> 1] >> (16 * (i & 1))) & 0xFFFFu)) * f;
      }
      kq_head = norm_exponent((uint32_t)__shfl((int)qb, 16 * head), 0);   // (head h's queries sit in lanes 16h ..)
    }
  };
  auto count_in = [&]() {
    if (RAISE) raise.arrive(a.raise, b, a.batch);
  };
  auto raise_if_last = [&]() {   // (at the workgroup's end the launch would wait for the second atomic: 22.45 us a step for 22.0)
    if (RAISE) raise.finish(a.raise, b, a.batch, hot, false);
  };
  float kS = 0.0f;   // what the kept scores still have to be multiplied by
  float kZ = 0.0f;   // ... and the zero term sum_c Q_c z_c
  // tokens whose softmax this lane runs: for its o-th owned k-step j = cg * OWN + o, the low
  // (lh = 0) and high (lh = 1) fp16 halves of the P' registers come from tiles tile_lo / tile_hi
  // of half j / 2; token = 32 g + 4 tile + row
  int tb[OWN][2];
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    const int j = cg * OWN + o;
    tb[o][0] = 32 * g + 4 * (4 * (j >> 1) + ((j & 1) ? F::tile_lo(1) : F::tile_lo(0)));
    tb[o][1] = 32 * g + 4 * (4 * (j >> 1) + ((j & 1) ? F::tile_hi(1) : F::tile_hi(0)));
  }
  if constexpr (kF8) {   // tiles cg and 4 + cg
    tb[0][0] = E::token(g, cg);
    tb[0][1] = E::token(g, 4 + cg);
  }

  // Q' = Q * s_c in B-operand order, as an fp16 high + low pair or in bytes, and the zero term sum_c Q_c z_c, per
  // head: once per block for channel-wise K (with the block's parameters), once per kernel for
  // per-token K.  16 lanes per head (slot group lane % 16: two runs of 4 consecutive channels).
  // The pair, channel-wise K: the block's scales are first brought below 1 by a power of two (2^-ek, from the largest
  // of the block), so that with |q| < 1 the products neither overflow nor sink into the fp16 subnormals;
  // the factor comes back out of the scores with kS.  Returns ek.
  // Bytes: `fine` says whether the block (per-token K: every block) takes the second four as well.
  bool fine = false;
  auto prep_queries = [&]() -> int {
    int ek = 0;
    float nrm[4];   // 2^-ek times the position factor of register i
#pragma unroll
    for (int i = 0; i < 4; ++i) nrm[i] = F::un(i);
    if constexpr (kF8) {
      float t[8], zsum = 0.0f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float qc = qv[i >> 2][i & 3];
        if constexpr (KT) {
          t[i] = qc;
          zsum += qc;
        } else {
          const h2_t pr = __builtin_bit_cast(h2_t, i < 4 ? kp0[i] : kp1[i - 4]);   // (scale, zero)
          t[i] = qc * (float)pr[0];   // exact: 11 bits times 11 bits
          zsum = __builtin_fmaf(qc, (float)pr[1], zsum);
        }
      }
      zsum = row_sum16(zsum);
      // the power of two that brings the head's largest into [2^29, 2^30), and back (all zero: any; an integer holds no NaN
      // and no infinity, which the way back hands to all of the head's scores)
      float top = fabsf(t[0]);
#pragma unroll
      for (int i = 1; i < 8; ++i) top = __builtin_elementwise_maximum(top, fabsf(t[i]));   // (NaN if one is)
      const uint32_t most = row_max16_u(__float_as_uint(top)), e = max(most & 0x7F800000u, 30u << 23);
      const float up = __uint_as_float((283u << 23) - e), down = __builtin_fmaf(__uint_as_float(most), 0.0f, __uint_as_float(e - (29u << 23)));
      const int h = lane >> 4;
      auto put_bytes = [&](const int (&n)[8], int level) {
        uint32_t x[8], d0[4], d1[4];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = (uint32_t)n[i] + 0x00808080u;
        if constexpr (BITS == 4) {
          transpose_bytes(x[0], x[2], x[4], x[6], d0);
          transpose_bytes(x[1], x[3], x[5], x[7], d1);
        } else {
          transpose_bytes(x[0], x[4], x[1], x[5], d0);
          transpose_bytes(x[2], x[6], x[3], x[7], d1);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t sign = k < 3 ? 0x80808080u : 0u;
          d0[k] ^= sign;
          d1[k] ^= sign;
          uint32_t* const reg = wl.qd[level][(prep_sg >> 1) & 1][prep_sg >> 2][4 * k + h];
          if constexpr (BITS == 4) {   // word prep_sg % 4 of the lane group's four: even channels, odd channels
            *reinterpret_cast<u2_t*>(reg + 2 * (prep_sg & 1)) = (u2_t){d0[k], d1[k]};
          } else {                     // half of a word of its two: two bytes of each register
            uint16_t* dst = reinterpret_cast<uint16_t*>(reg) + (prep_sg & 1);
            dst[0] = (uint16_t)d0[k];
            dst[2] = (uint16_t)(d0[k] >> 16);
            dst[4] = (uint16_t)d1[k];
            dst[6] = (uint16_t)(d1[k] >> 16);
          }
        }
      };
      int n[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) n[i] = nearest(t[i] * (up * I::position(i)));
      put_bytes(n, 0);
      float rest[8];   // what the rounding took (exact)
      auto rests = [&]() {
#pragma unroll
        for (int i = 0; i < 8; ++i) rest[i] = __builtin_fmaf(t[i], up * I::position(i), -(float)n[i]);
      };
      if constexpr (KT) {
        rests();
        bool some = false;
#pragma unroll
        for (int i = 0; i < 8; ++i) some |= rest[i] != 0.0f;
        fine = __any(some);
      } else {
        fine = __any(top > fine_from);
        if (fine) {
          bool some = false;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const h2_t pr = __builtin_bit_cast(h2_t, i < 4 ? kp0[i] : kp1[i - 4]);
            some |= fabsf(t[i]) > fine_from && fabsf((float)pr[1]) < I::kFineZero * (float)pr[0];
          }
          fine = __any(some);
        }
      }
      if (fine) {
        if constexpr (!KT) rests();
#pragma unroll
        for (int i = 0; i < 8; ++i) n[i] = nearest(rest[i] * kFineUnits);
        put_bytes(n, 1);
      }
      if (prep_sg == 0) wl.zq[h] = make_float2(KT ? zsum * up : zsum, down);   // (per-token K adds it to the sums)
      return 0;
    }
    if constexpr (!KT) {
      uint32_t sb = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) sb = max(sb, max(kp0[i] & 0xFFFFu, kp1[i] & 0xFFFFu));
      ek = -norm_exponent(row_max16_u(sb), kSTop);   // scale * 2^-ek < 2^kSTop for every channel of the block
      const float f = pow2i(-ek);
#pragma unroll
      for (int i = 0; i < 4; ++i) nrm[i] = f * F::un(i);
    }
    if constexpr (!kF8) {
#pragma unroll
      for (int p = 0; p < HP; ++p) {
        const int ph = 4 * p + (lane >> 4);
        const f4_t qa = *reinterpret_cast<const f4_t*>(&q_s[ph][run0]), qb = *reinterpret_cast<const f4_t*>(&q_s[ph][run1]);
        float zsum = 0.0f;
        h2_t qh[4], ql[4];   // register i: entries 2i (run 0) and 2i + 1 (run 1)
#pragma unroll
        for (int run = 0; run < 2; ++run)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float qc = run ? qb[i] : qa[i];
            float t = qc;   // per-token K: Q' = Q, and the "zero term" is sum_c Q_c
            float z = 1.0f;
            if constexpr (!KT) {
              const h2_t pr = __builtin_bit_cast(h2_t, run ? kp1[i] : kp0[i]);   // (scale, zero)
              t = qc * (float)pr[0];   // exact: 11 bits times 11 bits
              z = (float)pr[1];
            }
            // high piece, and the rest in one rounding: fma(t, nrm, -high)
            const _Float16 hi = (_Float16)(t * nrm[i]);
            qh[i][run] = hi;
            ql[i][run] = (_Float16)__builtin_fmaf(t, nrm[i], -(float)hi);
            zsum = __builtin_fmaf(qc, z, zsum);
          }
        zsum = row_sum16(zsum);
        u4_t phi, plo;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          phi[v] = __builtin_bit_cast(uint32_t, qh[v]);
          plo[v] = __builtin_bit_cast(uint32_t, ql[v]);
        }
        *reinterpret_cast<u4_t*>(&wl.qhi[ph][8 * prep_sg]) = phi;
        *reinterpret_cast<u4_t*>(&wl.qlo[ph][8 * prep_sg]) = plo;
        if (prep_sg == 0) wl.zq[ph] = zsum;
      }
    }
    return ek;
  };
  // Groups of 5 .. 8 heads: the high piece of Q' goes to the even column groups and the low piece to
  // the odd ones, so one MFMA per k-step produces both partial products (added across the column
  // groups afterwards); groups of 9..16 have no columns to spare and run two MFMAs per k-step.
  constexpr bool kSplitCols = COPIES == 2;
  h8_t bqh[4], bql[4];
  i4_t bq8[2];   // groups of up to 4 heads: byte cg of Q', the two halves of the contraction
  const float w_q = pow2i(8 * cg);            // what the byte counts
  const int sb_p = 127 - E::kTop - 5 * cg;    // that of piece cg of P'
  auto load_bq = [&](int j) {
    if constexpr (kF8) {
      if (j < 2) bq8[j] = __builtin_bit_cast(i4_t, *reinterpret_cast<const u4_t*>(wl.qd[0][j][g][col]));
    } else if constexpr (kSplitCols) {
      bqh[j] = *reinterpret_cast<const h8_t*>(cg & 1 ? &wl.qlo[head][8 * (4 * g + j)] : &wl.qhi[head][8 * (4 * g + j)]);
    } else {
      bqh[j] = *reinterpret_cast<const h8_t*>(&wl.qhi[head][8 * (4 * g + j)]);
      bql[j] = *reinterpret_cast<const h8_t*>(&wl.qlo[head][8 * (4 * g + j)]);
    }
  };
  // per-token K: the operand stays in registers; 9 .. 16 heads have not enough of them (25 spilled: 32K tokens, 16 heads,
  // 19.9 us a step) and read it for every block
  constexpr bool kKeepQ = KT && GQP < 16;
  float zq = 0.0f, qsum = 0.0f;
  auto set_scales = [&]() {
    kS = a.scale_log2 * pow2i((KT || kF8 ? 0 : 24) - kq_head);
    kZ = a.scale_log2 * pow2i(-kq_head);
    if constexpr (KT) {
      (void)prep_queries();
      wave_sync();
      if constexpr (kKeepQ) {
#pragma unroll
        for (int j = 0; j < 4; ++j) load_bq(j);
      }
      if constexpr (kF8) {
        qsum = wl.zq[head].x;
        kS *= wl.zq[head].y;
      } else {
        qsum = wl.zq[head];
      }
    }
  };

  // Two waves of different workgroups share each SIMD and the issue arbiter favours the older
  // one, which then runs a block ahead, finishes early and leaves the other to drain alone with
  // half the loads in flight.  Priority by remaining work keeps the pair in step.
  int done = 0;
  bool first = true;
  float sc[OWN][2][4];   // scores of the block's tokens that this lane keeps
  float kSb = 0.0f;      // kS for the block's K exponent
  int nblk = blk1, next_entry = -1;
  size_t nbi = 0;
  bool has_next = false;
  // the keys' registers are free: request the next block's
  auto request_next = [&]() {
    if (PAGED || kEarly) {   // parameters first: the next block's first consumers
      issue_kpar(nbi);
      issue_vpar(nbi);
    }
#pragma unroll
    for (int T = 0; T < 8; ++T) issue_ktile(nbi, T);
  };
  auto attend_block = [&]() {
  if constexpr (KT) {   // per-token scale and zero of K
#pragma unroll
    for (int o = 0; o < OWN; ++o)
#pragma unroll
      for (int lh = 0; lh < 2; ++lh)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float2 kq = wl.kpar[slot(tb[o][lh]) + r];
          sc[o][lh][r] = __builtin_fmaf(sc[o][lh][r], kq.x, kq.y * qsum);
        }
  }
  // ---- online softmax (Alg. 1) over this lane's 8 * OWN tokens of head `head`, on S + log2 of the
  //      token's V scale (see "Range" at the top): av = score in log2 units, but for the block's zero term
#pragma unroll
  for (int o = 0; o < OWN; ++o)
#pragma unroll
    for (int lh = 0; lh < 2; ++lh)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        sc[o][lh][r] = __builtin_fmaf(sc[o][lh][r], kSb, wl.vpar[slot(tb[o][lh]) + r].x);
  float bmax = sc[0][0][0];
#pragma unroll
  for (int o = 0; o < OWN; ++o)
#pragma unroll
    for (int lh = 0; lh < 2; ++lh)
#pragma unroll
      for (int r = 0; r < 4; ++r) bmax = fmaxf(bmax, sc[o][lh][r]);
  bmax = head_max<COPIES>(bmax);
  // channel-wise K: every score of the head still lacks the block's zero term
  const float zqs = zq * kZ;
  const float m_new = fmaxf(m_run, bmax + zqs);
  const float zoff = zqs - m_new;
  const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on the first block (m_run = -inf)
  m_run = m_new;
  l_run *= alpha;
  z_run *= alpha;
  if (!kSingle && !first && __any(alpha != 1.0f)) {   // nothing to rescale on the first block
#pragma unroll
    for (int mt = 0; mt < 8; ++mt) oacc[mt] *= alpha;
    xacc *= alpha;
  }
  u4_t pb[4];   // P' as the B operand of the 4 k-steps of O^T += V^T P'
  i8_t pb8;     // groups of up to 4 heads: piece cg of P'
  if constexpr (kF8) {   // the e4m3 pieces of this lane's 8 weights, to the column groups that take them
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      float e[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        e[r] = __builtin_amdgcn_exp2f(sc[0][half][r] + zoff);   // P' = weight * V scale, <= 1
        const float4& par = wl.vpar[slot(tb[0][half]) + r];
        l_run = __builtin_fmaf(e[r], par.y, l_run);
        z_run = __builtin_fmaf(e[r], par.z, z_run);
      }
      uint32_t u[4] = {any_bits(), any_bits(), any_bits(), any_bits()}, from[4];
      float unit = 1.0f / (1 << E::kTop);
#pragma unroll
      for (int k = 0; k < kWeightPieces; ++k) {
        if (k < kWeightPieces - 1)
          u[k] = e4m3_piece<true>(e4m3_piece<false>(u[k], e[0], e[2], unit), e[1], e[3], unit);
        else
          u[k] = e4m3_last<true>(e4m3_last<false>(u[k], e[0], e[2], unit), e[1], e[3], unit);
        unit *= 1.0f / 32;
      }
      exchange_pieces(u, from);
      // rows 0, 2 (low halves) and 1, 3 (high halves) of two neighbouring tiles make a register each
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        pb8[4 * half + E::b_reg(8 * w)] = (int)__builtin_amdgcn_perm(from[2 * w + 1], from[2 * w], 0x05040100u);
        pb8[4 * half + E::b_reg(8 * w + 1)] = (int)__builtin_amdgcn_perm(from[2 * w + 1], from[2 * w], 0x07060302u);
      }
    }
  } else {                       // zero where another column group owns the k-step
    u4_t pair[OWN];
#pragma unroll
    for (int o = 0; o < OWN; ++o)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        uint32_t hv[2];
#pragma unroll
        for (int lh = 0; lh < 2; ++lh) {
          const float e = __builtin_amdgcn_exp2f(sc[o][lh][r] + zoff);
          const float4& par = wl.vpar[slot(tb[o][lh]) + r];
          l_run = __builtin_fmaf(e, par.y, l_run);
          z_run = __builtin_fmaf(e, par.z, z_run);
          hv[lh] = (uint32_t)f2h(e * F::un(r));
        }
        pair[o][r] = hv[0] | (hv[1] << 16);
      }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (COPIES == 1) pb[j][r] = pair[j][r];
        else pb[j][r] = cg == (j >> 1) ? pair[j & 1][r] : 0u;
      }
  }
  // ---- O^T += V^T P'
  if constexpr (kF8) {
    const u4_t c0 = *reinterpret_cast<const u4_t*>(&wl.c8[g][0]), c1 = *reinterpret_cast<const u4_t*>(&wl.c8[g][4]);
    const i8_t ac = {(int)c0[0], (int)c0[1], (int)c0[2], (int)c0[3], (int)c1[0], (int)c1[1], (int)c1[2], (int)c1[3]};
    xacc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(ac, pb8, xacc, 0, 0, 0, 127, 0, sb_p);
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
      oacc[mt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(E::a_operand(vraw[mt].w), pb8, oacc[mt], E::kFormatA, 0,
                                                                  0, E::kScaleA, 0, sb_p);
  } else {   // k-step j contracts 32 tokens (8 per lane group)
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const h8_t ac = *reinterpret_cast<const h8_t*>(&wl.c16[8 * (4 * g + j)]);
    xacc = __builtin_amdgcn_mfma_f32_16x16x32_f16(ac, __builtin_bit_cast(h8_t, pb[j]), xacc, 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {   // k-step outermost: consecutive MFMAs go to different accumulators
    const h8_t bp = __builtin_bit_cast(h8_t, pb[j]);
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
      oacc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(F::dequant(vraw[mt].w, j), bp, oacc[mt], 0, 0, 0);
  }
  }
  };
  auto next_page = [&]() {
    if (PAGED && has_next) {
      nblk = first_valid(nblk, next_entry, nbi);
      has_next = nblk < blk1;
    }
  };
  // Prepares and scores block `blk`, up to the request of its values.
  auto score_block = [&]() {
    nblk = kSingle ? blk1 : blk + bstep;
    nbi = bi + bstep;
    next_entry = -1;   // requested a block ahead, like the parameters
    if (PAGED && nblk < blk1) next_entry = table_entry(nblk);
    if (!kSingle) {
      // (quarter of the work done)
      if (4 * done < my_blocks) __builtin_amdgcn_s_setprio(3);
      else if (4 * done < 2 * my_blocks) __builtin_amdgcn_s_setprio(2);
      else if (4 * done < 3 * my_blocks) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(0);
      ++done;
    }
    kSb = kS;
    if constexpr (!KT) {
      const int ek = prep_queries();
      if constexpr (!kF8) kSb *= pow2i(ek);
    }
    if constexpr (KT) {   // K parameters of the block's 128 tokens
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const float sk = h2f((uint16_t)(kp2[u] & 0xFFFFu)), zk = h2f((uint16_t)(kp2[u] >> 16));
        wl.kpar[slot(2 * lane + u)] = make_float2(kF8 ? sk : sk * kTwo24, zk);
      }
    }
    // V parameters of the block's 128 tokens
    float centre[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float sv = h2f((uint16_t)(vp2[u] & 0xFFFFu)), zv = h2f((uint16_t)(vp2[u] >> 16));
      const int t = 2 * lane + u;
      const int r = t & 3;                // row of the token inside its S^T tile
      // (a token whose values are all equal has scale 0 and all-zero codes: any scale does, take 1)
      const float se = sv > 0.0f ? sv : 1.0f, rs = __builtin_amdgcn_rcpf(se);
      const float ct = sv > 0.0f ? rintf(fminf(fmaxf(-zv * rs, 0.0f), F::kQmax)) : 0.0f;
      wl.vpar[slot(t)] = make_float4(__builtin_amdgcn_logf(se), rs, __builtin_fmaf(ct, sv, zv) * rs, 0.0f);
      centre[u] = ct;
      if constexpr (!kF8) wl.c16[F::p_slot(t)] = (uint16_t)(ct * F::inv_un(r));
    }
    if constexpr (kF8) {
      const uint32_t c2 = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(centre[0], centre[1], 0, false);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int t = 2 * lane + u;
        reinterpret_cast<uint8_t*>(&wl.c8[E::b_group(t)][4 * E::b_half(t) + E::b_reg(t)])[E::b_byte(t)] = (uint8_t)(c2 >> (8 * u));
      }
    }
    wave_sync();
    if constexpr (!kKeepQ) {
#pragma unroll
      for (int j = 0; j < 4; ++j) load_bq(j);
    }
    if constexpr (!KT && kF8) {
      const float2 z = wl.zq[head];
      zq = z.x;
      kSb = kS * z.y;
    } else if constexpr (!KT) {
      zq = wl.zq[head];
    }
    has_next = !kSingle && nblk < blk1;
    if (!PAGED && !kEarly && has_next) {   // small, and the next block's first consumers: requested a block ahead
      issue_kpar(nbi);
      issue_vpar(nbi);
    }
    // groups of 9..16 heads: only once the keys' registers are free, which lets two waves fit a SIMD
    constexpr bool kValuesAfterQK = GQP == 16;

    // bytes: the partial scores of a tile, `weight` what the byte counts
    auto tile_scores = [&](const uint32_t* codes, const i4_t (&bytes)[2], float weight) {
      const i8_t ak = I::a_operand(codes);
      i4_t n = {kSumBits, kSumBits, kSumBits, kSumBits};
      n = __builtin_amdgcn_mfma_i32_16x16x64_i8((i4_t){ak[0], ak[1], ak[2], ak[3]}, bytes[0], n, 0, 0, 0);
      n = __builtin_amdgcn_mfma_i32_16x16x64_i8((i4_t){ak[4], ak[5], ak[6], ak[7]}, bytes[1], n, 0, 0, 0);
      f4_t acc;
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = __builtin_fmaf(__int_as_float(n[r]), weight, -kSumBase * weight);   // exact
      return acc;
    };
    // ---- S^T tiles (rows = tokens 32*(row/4) + 4T + row%4, all 16 columns valid); each lane
    //      keeps the tiles of the k-steps its column group owns: sc[o][low/high half][row]
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      f4_t s[4];
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        f4_t acc = {0.f, 0.f, 0.f, 0.f};   // (the zero term, one number per head, joins in the softmax)
        if constexpr (kF8) {
          acc = tile_scores(kraw[4 * half + tt].w, bq8, w_q);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const h8_t ak = F::dequant(kraw[4 * half + tt].w, j);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(ak, bqh[j], acc, 0, 0, 0);
            if constexpr (!kSplitCols) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(ak, bql[j], acc, 0, 0, 0);
          }
        }
        s[tt] = acc;
      }
      if (half == 0 && !kValuesAfterQK) {
#pragma unroll
        for (int mt = 0; mt < 8; ++mt) issue_vtile(bi, mt);
      }
      // k-steps 2*half and 2*half+1 draw on this half's four tiles
      if constexpr (COPIES == 1) {
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            sc[2 * half + jj][0][r] = s[F::tile_lo(jj)][r];
            sc[2 * half + jj][1][r] = s[F::tile_hi(jj)][r];
          }
      } else if constexpr (COPIES == 2) {   // column group cg owns k-steps 2cg, 2cg+1: half cg
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            // own partial product plus the other column group's (half 0 is kept by group 0, half 1 by group 1)
            float lo = s[F::tile_lo(jj)][r], hi = s[F::tile_hi(jj)][r];
            lo += half == 0 ? dpp_f<kRowShl8>(lo) : dpp_f<kRowShr8>(lo);
            hi += half == 0 ? dpp_f<kRowShl8>(hi) : dpp_f<kRowShr8>(hi);
            sc[jj][0][r] = (half == 0 || cg == 1) ? lo : sc[jj][0][r];
            sc[jj][1][r] = (half == 0 || cg == 1) ? hi : sc[jj][1][r];
          }
      } else {                              // column group cg keeps tile cg of each half: the sum of the four bytes' products
        reduce_scatter(s, sc[0][half]);
      }
    }
    if constexpr (kF8) {
      if (fine) {
        const float w_f = w_q * (1.0f / kFineUnits);
        i4_t f8[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) f8[j] = __builtin_bit_cast(i4_t, *reinterpret_cast<const u4_t*>(wl.qd[1][j][g][col]));
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          f4_t s[4];
          float rest[4];
#pragma unroll
          for (int tt = 0; tt < 4; ++tt) {
            RawTile<WORDS> again = kraw[4 * half + tt];   // (hidden: the masked codes would be kept, 28 registers of every block)
#pragma unroll
            for (int i = 0; i < WORDS; ++i) asm volatile("" : "+v"(again.w[i]));
            s[tt] = tile_scores(again.w, f8, w_f);
          }
          reduce_scatter(s, rest);
#pragma unroll
          for (int r = 0; r < 4; ++r) sc[0][half][r] += rest[r];
        }
      }
    }
    if (kValuesAfterQK) {
#pragma unroll
      for (int mt = 0; mt < 8; ++mt) issue_vtile(bi, mt);
    }
  };
  auto advance = [&]() {
    // Both sums grow with the number of tokens, their difference (the signal) with its square root: every
    // 16 blocks the centre sum is taken out of the accumulators and starts again from zero.
    if (!kSingle && (done & 15) == 0) {
#pragma unroll
      for (int mt = 0; mt < 8; ++mt) oacc[mt] -= xacc[0];
      xacc = (f4_t){0.f, 0.f, 0.f, 0.f};
    }
    wave_sync();   // the next block's prep overwrites this wave's LDS scratch
    first = false;
    blk = nblk;
    bi = nbi;
  };
  // (The residual slice inside both branches: the loads behind its own are then known to the compiler, which otherwise
  // waits for all of them.  Likewise the blocks inside the one that requests the first, and one way out of their loop, past
  // no load whose use it skips: wherever the compiler sees a path, be it one that is never taken, on which a load has not
  // been waited for, it waits for all of them the next time round.)
  // (A long slice beside a block's registers would leave two workgroups of one block a wave on a compute unit, not three: it
  // comes first.)
  if constexpr (BLOCKS == kOneBlockSlice) {
    start_slice();
    scale_queries();
    count_in();
    attend_slice();
    raise_if_last();
    if (blk < blk1) {
      issue_first();
      set_scales();
      score_block();
      attend_block();
    }
  } else if (blk >= blk1) {
    start_slice();
    scale_queries();
    count_in();
    attend_slice();
    raise_if_last();
  } else {
    start_slice();
    issue_first();
    scale_queries();
    count_in();
    attend_slice();
    raise_if_last();
    loads_left<kBlockLoads>();
    set_scales();
    if constexpr (kEarly) {
      // (the loop's end is between a block's two halves, with the values on their way: 32K tokens 12.9 -> 12.45 us a
      // step, 8 x 32K at 2 bits 34.7 -> 33.6, against a loop that is left in the middle)
      score_block();
      next_page();
      while (has_next) {
        request_next();
        attend_block();
        advance();
        score_block();
        next_page();
      }
      attend_block();
    } else {
      while (true) {
        score_block();
        attend_block();
        next_page();
        if (!has_next) break;
        request_next();
        advance();
      }
    }
  }

  // ---- merge the column groups (groups of 8 heads), then the waves of the workgroup
  //      (cross-wave step of the cooperative softmax)
  l_run = head_sum<COPIES>(l_run);
  z_run = head_sum<COPIES>(z_run);
  if (files)
    *reinterpret_cast<u4_t*>(const_cast<uint16_t*>(tid >= 16 ? a.v_res : hot.k_res) + (unit * kBlock + new_slot) * kD + 8 * (tid & 15)) = filed;
  lds_barrier();   // every wave is done with its WaveLds before the space is reused
  ML& ml = *reinterpret_cast<ML*>(smem_raw);
  // The column groups' shares are added below, by the threads that merge the waves: 12 (4) more LDS reads there for 288 (32)
  // DPP moves and adds of every wave here.  A wave alone on its SIMD issues one instruction every 4 to 5 cycles, and at the
  // end of the kernel nothing hides them: 0.25 us of a launch (32K tokens, 8 units: 12.6 -> 12.35 a step; with the shorter
  // forms of masks and pieces, bd_fmt.h, 12.1).
#pragma unroll
  for (int mt = 0; mt < 8; ++mt) {
    f4_t o;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = kF8 ? oacc[mt][r] - xacc[0] : (oacc[mt][r] - xacc[0]) * kTwo24;
    *reinterpret_cast<f4_t*>(&ml.o[wave][col][16 * mt + 4 * g]) = o;
  }
  if (lane < GQP) {
    ml.m[wave][col] = m_run;
    ml.l[wave][col] = l_run;
    ml.z[wave][col] = z_run;
  }
  lds_barrier();
#pragma unroll
  for (int p = 0; p < HP; ++p) {
    const int h = 4 * p + wave, c0 = 2 * (tid & 63);
    if (h < gq) {
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
          Z += f * ml.z[w][h];
          float2 o = *reinterpret_cast<const float2*>(&ml.o[w][h][c0]);
#pragma unroll
          for (int k = 1; k < COPIES; ++k) {
            const float2 s = *reinterpret_cast<const float2*>(&ml.o[w][GQP * k + h][c0]);
            o.x += s.x;
            o.y += s.y;
          }
          o0 += f * o.x;
          o1 += f * o.y;
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
        if ((tid & 63) == 0) {
          a.part_ml[row * 2] = M;
          a.part_ml[row * 2 + 1] = L;
        }
      }
    }
  }
}
