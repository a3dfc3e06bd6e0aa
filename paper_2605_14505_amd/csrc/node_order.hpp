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
  // small states: an XCD owns `slab >> 4` consecutive blocks, one more on the first (slab >> 1) & 7
  // XCDs, bit 0 set; else 0.  One word (32 bytes in all): with the kernel arguments on a third
  // 64-byte line, steps of 4 us took 0.15 us longer
  uint32_t slab;
  int64_t stride;    // elements between population arrays
  uint32_t n3;       // nodes
  uint32_t div_mul;  // i / n = (i div_mul) >> (32 + div_shift) for i < 2^30
  int div_shift;
  int xcd_group;     // consecutive blocks that the x-shifted steps keep on one XCD
};
static_assert(sizeof(Geometry) == 32, "two 64-byte lines of kernel arguments");

// Whether a state (`bytes` of populations) is small enough that what a step leaves in the XCDs' L2s
// (8 x 4 MB) matters to the next one: up to twice their size some of it is found there.
constexpr bool near_state(int64_t bytes) { return bytes <= ((int64_t)64 << 20); }

// Division by n as a multiplication: with 2^(s-1) < n <= 2^s and m = floor(2^(31 + s) / n) + 1
// (< 2^32), m n exceeds 2^(31 + s) by at most n <= 2^s, so i m / 2^(31 + s) exceeds i / n by less
// than 1 / n for every i < 2^31 (n^3 <= 2^30).
// near: near_state of the population buffer.
constexpr Geometry make_geometry(int n, int64_t stride, bool near = false) {
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
  const uint32_t blocks = (g.n3 + node_threads(n) - 1) / node_threads(n);
  if (near) {
    g.slab = blocks / 8 << 4 | blocks % 8 << 1 | 1;
    g.xcd_group = 1;
  }
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
//
// A small state (near_state) is another matter: there a step finds what the step before left in its
// XCD's L2, if the same XCD wrote it.  Renumbered in the shifted steps alone, a node moved to
// another XCD every step (19 x 7 FP32 48^3 6.3 -> 9.4 us a step against blocks of 64 x 4 nodes in
// dispatch order).  So every step of a small state gives XCD k the k-th slab of consecutive blocks,
// whose inner neighbours it owns too.  Mean step in us, 64 x 4 blocks / renumbered shifted steps /
// slabs: 27 x 19 FP32 36^3 7.7 / 8.8 / 6.0, 48^3 11.2 / 11.3 / 7.9; FP16 52^3 9.9 / 11.0 / 7.1, 80^3
// (47 MB) 28.1 / 17.8 / 16.4; 19 x 7 FP32 40^3 5.3 / 6.9 / 4.5, 48^3 6.3 / 9.4 / 5.6; where rows are
// whole blocks, which are not renumbered, 27 x 19 FP32 64^3 16.0 / 15.6 / 14.7, 7 x 27 FP16 64^3 7.6 /
// 8.0 / 7.3, FP64 arithmetic 64^3 19.5 / 19.8 / 19.3, 32^3 6.5 / 5.2 / 5.0.  Beyond 64 MB, renumbered /
// slabs: 27 x 19 FP32 72^3 22.4 / 22.2, 19 x 7 88^3 23.1 / 23.1, 27 x 7 96^3 (120 MB) 37.1 / 37.6.
constexpr uint32_t block_at(uint32_t b, uint32_t blocks, const Geometry& geo, bool shifted = true) {
  // without a branch, so that its constants come with the kernel's other scalar loads: a wait more
  // costs 0.2 us of a 4 us step
  const uint32_t on = geo.slab & 1, rest = geo.slab >> 1 & 7, own = b & (7 * on);
  b = own * (geo.slab >> 4) + (own < rest ? own : rest) + (b >> (3 * on));
  if (shifted && geo.xcd_group > 1) {
    const uint32_t G = (uint32_t)geo.xcd_group, whole = blocks / (8 * G) * (8 * G);
    if (b < whole) {
      const uint32_t k = b & 7, rest = b >> 3;
      b = G * (8 * (rest / G) + k) + rest % G;
    }
  }
  return b;
}

}  // namespace stgv
