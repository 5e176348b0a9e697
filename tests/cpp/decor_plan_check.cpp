// Host check of the loads of the correlation reduction's substitution: for
// every number of rows M that the reduction takes, every row read is one the
// M x M factor has, and the batches cover each block before the diagonal once,
// in order.
#include <cstdio>

#include "../../paper_2007_03847_amd/csrc/decor_plan.hpp"

using namespace fmc;

int main() {
  for (int M = 1; M <= 1024; ++M) {
    const int n_blk = (M + kDcT - 1) / kDcT;
    DcBatch t = dc_first_batch();
    for (int b = 1; b < n_blk; ++b)
      for (int k = 0; k < b; k += kDcBatch) {
        if (t.b != b || t.k != k) return std::printf("M=%d: batch (%d, %d) for (%d, %d)\n", M, t.b, t.k, b, k), 1;
        for (int q = 0; q < kDcBatch; ++q) {
          if (k + q < b && t.block(q) != k + q) return std::printf("M=%d: block\n", M), 1;
          for (int s = 0; s < 4; ++s)
            for (int g = 0; g < 4; ++g)
              if (dc_row(t.block(q), s, g) < 0 || dc_row(t.block(q), s, g) >= M)
                return std::printf("M=%d: row %d\n", M, dc_row(t.block(q), s, g)), 1;
        }
        t = dc_next_batch(t);
      }
    if (t.b < n_blk) return std::printf("M=%d: a batch too many\n", M), 1;
  }
  std::printf("ALL OK\n");
  return 0;
}
