// What the host decides about an attention launch.  Plain C++, no HIP: tests compile it for the CPU and hold it against the
// kernels as built.
#pragma once

namespace bd {

// Workgroups (four waves, one per SIMD) of a kernel instance that share a compute unit: what the instance is compiled for.
// Groups of 64 and 32: every instance fits 256 registers (two waves per SIMD) but those for groups of 32 with more than 4
// heads per workgroup and 4-bit codes or per-token K, which would spill and run one wave per SIMD instead.
constexpr int grp_waves_per_simd(int bits, int group, int gqp, bool kt) {
  return (bits == 4 || kt) && group == 32 && gqp == 8 ? 1 : 2;
}
// MXFP4: 9 .. 16 heads in pages take 267.
constexpr int mx_waves_per_simd(int gqp, bool paged) { return gqp == 16 && paged ? 1 : 2; }

// The integer kernel in its three forms (BLOCKS), and the workgroups of up to 8 heads of each that share a unit; of 9 .. 16
// heads two do in every form.
constexpr int kManyBlocks = 0, kOneBlock = 1, kOneBlockSlice = 2;
constexpr int kOneBlockWide = 3;   // one block a wave in workgroups of eight (wide_int_kernel)
constexpr int int_waves_per_simd(int gqp, int blocks) { return gqp <= 8 && blocks != kManyBlocks ? 3 : 2; }

constexpr int kResShort = 32;   // residual tokens that a workgroup attends in one round
// Which form a call over `nb` blocks and `res_len` residual tokens a unit in `splits` splits takes, `wgs` workgroups in all.
// One block a wave at most takes half the registers, a residual slice of more than a round beside that block all of them
// again.  Ahead of the block it does not, but is not hidden by the block's way here: better once a unit has two workgroups
// (256 units), most where a third one on it spares a second round.  A step, 4 bits, the slice beside the block / ahead of it:
// 8 heads per KV head 320 workgroups with 36 residual tokens 11.4 / 11.1 us, 512 with 116 14.9 / 14.6, 640 with 45 19.4 / 15.5,
// with 100 21.1 / 17.6; 4 heads 640 with 45 16.5 / 14.0; but 192 with 116 9.9 / 10.3, 264 with 84 11.9 / 12.0.
inline int one_block_instance(int nb, int splits, int res_len, long wgs) {
  if ((nb + splits - 1) / splits > 4) return kManyBlocks;   // (four waves)
  if (res_len <= (kResShort - 2) * splits) return kOneBlock;
  return wgs > 256 ? kOneBlockSlice : kManyBlocks;
}

// Whether a call runs workgroups of eight waves: where four would have two blocks each, eight have one, and a
// second block's first bytes are not waited for.  K by channel, up to 4 heads per KV head, while a unit has one workgroup.  A
// step issued one by one, four waves / eight: 4 bits, 640 tokens, 8 units 7.4 / 6.6 us, 1K 7.5 / 7.0, 256 units of 700 10.5 /
// 10.05, of 1.1K 11.45 / 11.45; 2 bits 1K 7.2 / 6.9.  In several splits until most waves have a second block, and further with
// 2 bits, whose blocks are half the bytes: 8 units, 32 splits 20K 10.7 / 10.1, 24K 10.8 / 10.25, 26K 10.55 / 10.55, 32K 11.06 /
// 11.55; 2 bits 17K 9.9 / 9.6, 32K 10.05 / 9.8.  No more than that: the two waves of a SIMD issue as many instructions as one
// with two blocks does.  Per-token K, whose blocks have fewer: 32K 11.0 / 11.45.
inline bool wide_instance(int nb, int splits, int bits, int gq, bool kt, long wgs) {
  return gq <= 4 && !kt && nb > 4 * splits && nb <= (bits == 4 && splits > 1 ? 6 : 8) * splits && wgs <= 256;
}

// The form of a contiguous call: `splits` workgroups for each of `units`, and one more where the call packs a block behind its
// attention (of which those of eight waves fill a compute unit each, too: 256 attending and 256 packing ones of them are two
// rounds, a step of 32 sequences of 767 tokens, 8 KV heads, 4 bits 19.9 us, in four waves 16.4; 2 bits, 895 tokens 19.4 / 15.3).
inline int contiguous_form(int nb, int splits, int res_len, int bits, int gq, bool kt, long units, bool packs) {
  const long wgs = splits * units;
  return wide_instance(nb, splits, bits, gq, kt, wgs + (packs ? units : 0)) ? kOneBlockWide : one_block_instance(nb, splits, res_len, wgs);
}

// Paged cache: how many sequences of a batch are to be sorted by length (0: left as they are), and how many of them are in
// the second layer, from bit 10 (paged_sequence has the rule and its reasons).  per_seq: workgroups of a sequence; waves: per
// SIMD, of the instance that the launch takes.
inline int sorted_sequences(long per_seq, int batch, int max_wgs, int waves, int blocks_per_split) {
  const long wgs = per_seq * batch;
  if (batch < 2 || batch > 64 || wgs <= 256 || wgs > max_wgs) return 0;
  if (wgs > (blocks_per_split >= 8 ? 512 : 384)) return (wgs - 1) % 256 >= 128 ? 0 : batch;
  if (waves < 2) return batch;
  const long second = (wgs - 256 + per_seq - 1) / per_seq;
  return batch | (int)(second < batch / 2 ? second : batch / 2) << 10;
}
// Which of the n sequences, longest first, is launched z-th, if `second` of them make a second layer.
constexpr int place_by_length(int z, int n, int second) {
  const int first = n - second;
  return second <= 0 ? z : z < second ? first - second + z : z < first ? z - second : n - 1 - (z - first);
}

// A launch of attention over pages: `splits` x `groups` (KV heads x pieces of the query group) workgroups for each of
// `batch` sequences, of which `order` says how they are dealt (sorted_sequences).
struct PagedGrid {
  int x, y, z;
  int order;
  int flush_mode;   // kFlushNone, kFlushAfter, kFlushLast
};
// How a step whose token fills a residual block packs the block in the attention launch (Sec. IV-B(1); DecodeArgs / GrpArgs
// flush_mode): not at all, before it is attended, or while its fp16 rows are, by workgroups of their own: blockIdx.x == 0 of
// every split row, or rows of grid z behind the last sequence's.
constexpr int kFlushNone = 0, kFlushFirst = 1, kFlushAfter = 2, kFlushLast = 3;
// Lazy: one packing workgroup per (sequence, KV head), which ends at once if the sequence's residual is not full.
// - An odd number of splits: behind the attending ones, in rows of grid z of their own, so that the attending ones lie on the
//   chip as if they were alone.  At blockIdx.x == 0 of rows of an even length they all went to the same XCDs and left those
//   without attending ones (one split: half of the chip).  40 sequences of 1K to 3.1K tokens, one split, 2 bits, 8 heads per KV
//   head 40.3 -> 23.0 us a step (eager 23.5); 4 bits 24 of up to 5K, three splits 31.3 -> 26.9, 12 of 4K, five 17.6 -> 14.6.
// - An even one: blockIdx.x == 0.  There the rows go round the XCDs, and the packing ones start first: 4 splits 24 of 4K 25.0
//   us, behind the others 25.9, 8 splits 8 of 5K 16.1 / 16.6, 2 splits 48 of 2K 26.2 / 27.1 (but 32 of 4K 28.1 / 24.2).  They
//   take places as the others do and count as such.
// (Fewer sequences than splits would leave most of a row of grid z without work, and from 2^14 sequences on their number does
// not fit the preloaded arguments: as with an even number.)
inline PagedGrid paged_grid(int splits, int groups, int batch, bool lazy, int max_wgs, int waves, int max_pages) {
  PagedGrid g{splits, groups, batch, 0, kFlushNone};
  const bool last = splits % 2 == 1 && batch >= splits && batch < 1 << 14;
  if (lazy && !last) {
    g.x += 1;
    g.flush_mode = kFlushAfter;
  }
  g.order = sorted_sequences((long)g.x * g.y, batch, max_wgs, waves, max_pages / splits);
  if (lazy && last) {
    g.z += (batch + splits - 1) / splits;
    g.flush_mode = kFlushLast;
  }
  return g;
}
// One split and no merge behind it: the attention launch of a step raises the lengths itself (LengthRaise, bd_device.h) if the
// cache has counters for its workgroups.
constexpr int kRaiseShards = 16;        // counters that share out the workgroups, by sequence: at most (a counter takes some 10 ns a workgroup)
constexpr int kRaiseStride = 16;        // words from one to the next: a line of 64 bytes each
constexpr int kRaiseCountBits = 20;
constexpr int raise_shards(int batch) { return batch < kRaiseShards ? batch : kRaiseShards; }
constexpr long raise_bytes(int batch) { return 4L * kRaiseStride * (raise_shards(batch) + 1); }
// workgroups that count in at shard s, `per_seq` of every sequence
constexpr long raise_arrivals(int s, long per_seq, int batch) { return per_seq * ((batch - s + raise_shards(batch) - 1) / raise_shards(batch)); }
// Whether a launch can, or the lengths are left to a launch of their own.  (More workgroups of a sequence than a counter counts:
// not in use.)
constexpr bool raises_in_launch(long per_seq, int batch, long counter_bytes) {
  return raise_arrivals(0, per_seq, batch) < 1L << kRaiseCountBits && raise_bytes(batch) <= counter_bytes;
}

// The sequence of the packing workgroup at (x, z) of such a grid; `batch` and more: none.
constexpr int packed_sequence(int x, int z, int splits, int batch) { return (z - batch) * splits + x; }

}  // namespace bd
