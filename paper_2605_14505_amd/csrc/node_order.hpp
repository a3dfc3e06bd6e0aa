// Order in which the node kernels walk the box: block size, division by the box edge and the
// block-to-node map.  Plain C++ (no HIP), so that the maps are also checked on the host.
#pragma once
#include <stdint.h>

namespace stgv {

// Threads (and nodes) of a node kernel's block: 256, and single wavefronts where the box has
// no more than two of them per CU, so that every CU has some (mean step: 32^3 6.59 -> 5.36 us,
// 16^3 4.94 -> 4.54; 128 threads 6.01 and 4.60; at 40^3 single wavefronts lose, 9.34 -> 10.1).
constexpr int kNodeBlock = 256;
constexpr int node_threads(int n) { return (int64_t)n * n * n <= 2 * 256 * 64 ? 64 : kNodeBlock; }

struct Geometry {
  int n;             // box edge
  int64_t stride;    // elements between population arrays
  uint32_t n3;       // nodes
  uint32_t div_mul;  // i / n = (i div_mul) >> (32 + div_shift) for i < 2^30
  int div_shift;
  int xcd_group;     // consecutive blocks that the x-shifted steps keep on one XCD
};

// Division by n as a multiplication: with 2^(s-1) < n <= 2^s and m = floor(2^(31 + s) / n) + 1
// (< 2^32), m n exceeds 2^(31 + s) by at most n <= 2^s, so i m / 2^(31 + s) exceeds i / n by less
// than 1 / n for every i < 2^31 (n^3 <= 2^30).
constexpr Geometry make_geometry(int n, int64_t stride) {
  Geometry g{};
  g.n = n;
  g.stride = stride;
  g.n3 = (uint32_t)n * n * n;
  int s = 0;
  while ((1 << s) < n) ++s;
  g.div_mul = (uint32_t)((1ull << (31 + s)) / (unsigned)n + 1);
  g.div_shift = s - 1;
  // blocks that make up whole rows (at most 8 of them)
  int rows = n, blk = node_threads(n);
  while (blk > 1 && rows % 2 == 0) { rows /= 2; blk /= 2; }
  g.xcd_group = rows < 8 ? rows : 8;
  return g;
}

// i / n
constexpr uint32_t over_n(uint32_t i, const Geometry& geo) {
  return (uint32_t)((uint64_t)i * geo.div_mul >> 32) >> geo.div_shift;
}

// The hardware hands consecutive workgroups to the 8 XCDs in turn, each with its own L2, so
// neighbouring blocks sit on different XCDs; the steps whose loads or stores are shifted
// along x (odd AA, A-B) share a line at every block seam inside a row, and then fetch it from
// HBM twice (at 512^3 FP16, 15 % more than the algorithmic bytes).  For those steps the
// workgroups are renumbered so that the `xcd_group` consecutive blocks that make up whole
// rows are 8 apart in dispatch order, i.e. on one XCD: workgroup L = 8 (G q + h) + k holds
// block G (8 q + k) + h; the blocks past the last multiple of 8 G keep their places.
constexpr uint32_t block_at(uint32_t b, uint32_t blocks, const Geometry& geo) {
  if (geo.xcd_group > 1) {
    const uint32_t G = (uint32_t)geo.xcd_group, whole = blocks / (8 * G) * (8 * G);
    if (b < whole) {
      const uint32_t k = b & 7, rest = b >> 3;
      b = G * (8 * (rest / G) + k) + rest % G;
    }
  }
  return b;
}

}  // namespace stgv
