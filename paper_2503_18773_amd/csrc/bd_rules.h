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

}  // namespace bd
