// decor_plan.hpp -- the order in which the substitution of the correlation
// reduction (k_dc_whiten) loads the blocks of the Cholesky factor.  Plain C++,
// so that the rows it reads can be checked on the host.
#pragma once

namespace fmc {

constexpr int kDcT = 16;     // edge of a block of the factor
constexpr int kDcBatch = 4;  // blocks of a row loaded together

// A batch: blocks k .. k + kDcBatch - 1 of block row b, those from b on left out.
// Of a block left out the row's first one is loaded in its place (and not used), so
// b >= 1: block row 0 has nothing before the diagonal and M < 16 no whole block.
struct DcBatch {
  int b, k;
  constexpr int block(int q) const { return k + q < b ? k + q : 0; }
};

// Row of the transposed factor that quarter g of a wave loads in step s of block k.
constexpr int dc_row(int k, int s, int g) { return kDcT * k + 4 * s + g; }
constexpr DcBatch dc_first_batch() { return {1, 0}; }
// The batch after c; its b is n_blk (no such block row) after the last.
constexpr DcBatch dc_next_batch(DcBatch c) {
  return c.k + kDcBatch < c.b ? DcBatch{c.b, c.k + kDcBatch} : DcBatch{c.b + 1, 0};
}

}  // namespace fmc
