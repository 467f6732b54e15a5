// Where a lane's quad of products is read (plain C++: the kernels' arithmetic, also for the host's tests).
#pragma once
#include <cstdint>

namespace spg {

// Where a quad's products come from, in one word: the lane of its entry, how many there are (left: to the entry's end), its first
// product inside the entry.  A lane without a quad has the word 0: no products, at the start of lane 0's entry.
constexpr unsigned pack_quad(int src, int left, int off) {
  const int n = left < 0 ? 0 : (left < 4 ? left : 4);
  return (unsigned)src | ((unsigned)n << 6) | ((unsigned)off << 9);
}
constexpr int quad_src(unsigned w) { return (int)(w & 63u); }
constexpr int quad_count(unsigned w) { return (int)((w >> 6) & 7u); }
constexpr int quad_off(unsigned w) { return (int)(w >> 9); }

// Whether a load of four, wherever in lane `lane`'s entry (the B row of `len` products from bs on) a quad begins, may reach behind the b_nnz
// entries of B.  Lane 0's entry is read also where it has no products: by the lanes without a quad.
constexpr bool quads_leave(int lane, int64_t bs, int len, int64_t b_nnz) {
  return (len > 0 || lane == 0) && bs + (len > 0 ? len : 1) + 3 > b_nnz;
}

}  // namespace spg
