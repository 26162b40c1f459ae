// Answers questions about the launch rules (bd_rules.h), one per argument group, one line each:
//   grp BITS GROUP GQP KT | mx GQP PAGED | int GQP BLOCKS   waves per SIMD that the launch counts on
//   blocks NB SPLITS RES_LEN WGS             the form of the integer kernel that a contiguous call takes in workgroups of four waves
//   form NB SPLITS RES_LEN BITS GQ KT UNITS PACKS   the form that it takes
//   lazy SPLITS GROUPS BATCH MAX_PAGES        grid x, y, z of a lazy step, its order and flush mode; then the sequence of every
//                                            (x, z) whose workgroups pack
//   raise PER_SEQ BATCH WORKSPACE             the count that each shard of a step in one split reaches, or "no"
//   order PER_SEQ BATCH MAX_WGS WAVES BPS    places by length in launch order, or "as given"; then the second layer's size
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "bd_rules.h"

int main(int argc, char** argv) {
  auto arg = [&](int i) { return i < argc ? atoi(argv[i]) : 0; };
  for (int i = 1; i < argc;) {
    if (!strcmp(argv[i], "grp")) {
      printf("%d\n", bd::grp_waves_per_simd(arg(i + 1), arg(i + 2), arg(i + 3), arg(i + 4) != 0));
      i += 5;
    } else if (!strcmp(argv[i], "mx")) {
      printf("%d\n", bd::mx_waves_per_simd(arg(i + 1), arg(i + 2) != 0));
      i += 3;
    } else if (!strcmp(argv[i], "int")) {
      printf("%d\n", bd::int_waves_per_simd(arg(i + 1), arg(i + 2)));
      i += 3;
    } else if (!strcmp(argv[i], "blocks")) {
      printf("%d\n", bd::one_block_instance(arg(i + 1), arg(i + 2), arg(i + 3), arg(i + 4)));
      i += 5;
    } else if (!strcmp(argv[i], "form")) {
      printf("%d\n", bd::contiguous_form(arg(i + 1), arg(i + 2), arg(i + 3), arg(i + 4), arg(i + 5), arg(i + 6) != 0, arg(i + 7), arg(i + 8) != 0));
      i += 9;
    } else if (!strcmp(argv[i], "raise")) {
      const int batch = arg(i + 2);
      if (!bd::raises_in_launch(arg(i + 1), batch, arg(i + 3))) printf("no");
      else for (int k = 0; k < bd::raise_shards(batch); ++k) printf("%ld ", bd::raise_arrivals(k, arg(i + 1), batch));
      printf("\n");
      i += 4;
    } else if (!strcmp(argv[i], "order")) {
      const int r = bd::sorted_sequences(arg(i + 1), arg(i + 2), arg(i + 3), arg(i + 4), arg(i + 5)), n = r & 255, second = r >> 10;
      if (n == 0) printf("as given");
      for (int z = 0; z < n; ++z) printf("%d ", bd::place_by_length(z, n, second));
      printf("; %d\n", second);
      i += 6;
    } else if (!strcmp(argv[i], "lazy")) {
      const int splits = arg(i + 1), batch = arg(i + 3);
      const bd::PagedGrid g = bd::paged_grid(splits, arg(i + 2), batch, true, 1 << 30, 2, arg(i + 4));
      printf("%d %d %d %d %d ;", g.x, g.y, g.z, g.order, g.flush_mode);
      for (int z = batch; z < g.z && batch < 1000; ++z)
        for (int x = 0; x < g.x; ++x) printf(" %d", bd::packed_sequence(x, z, splits, batch));
      printf("\n");
      i += 5;
    } else {
      return 2;
    }
  }
  return 0;
}
