// The rule of csrc/split_rule.h on lines of "b nbr tokens nnz fullest decode cus": prints the waves, and whether the workgroup
// ids of that launch cover every tile once.
#include <cstdio>
#include <vector>

#include "../paper_2507_03117_amd/csrc/split_rule.h"

using namespace blast_dev;

int main() {
  int b, decode;
  long nbr, tokens, nnz, fullest, cus;
  while (std::scanf("%d %ld %ld %ld %ld %d %ld", &b, &nbr, &tokens, &nnz, &fullest, &decode, &cus) == 7) {
    const int units = (int)(nbr * (b / 64)), groups = (int)((tokens + 63) / 64), stride_log2 = split_stride_log2(units, groups, cus);
    std::vector<int> seen((size_t)units * groups);
    bool once = true;
    for (int id = 0; id < split_workgroups(units, groups, cus); ++id) {
      const SplitTile t = split_tile(id, stride_log2, groups);
      if (t.group < 0 || t.group >= groups || t.unit < 0) once = false;
      else if (t.unit < units) ++seen[(size_t)t.unit * groups + t.group];
    }
    for (int n : seen) once = once && n == 1;
    std::printf("%d %d\n", split_waves(b, nbr, tokens, nnz, fullest, decode != 0, cus), once ? 1 : 0);
  }
}
