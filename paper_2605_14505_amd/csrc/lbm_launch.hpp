// Host-side launchers: map run-time choices (stencil pair, forcing, layout mode,
// kernel flags) onto the kernel template instances of one storage type.
#pragma once
#include <hip/hip_runtime.h>

#include "lbm_device.hpp"

namespace stgv {

struct LaunchShape {
  dim3 grid, block;
};

// The stencil pairs (momentum Q_f x scalar Q_g) with kernel instances: those of the
// stencil comparisons of Sections 3.2-3.3 and of the D3Q7-scalar sweep.  X(qf, qg) is applied
// to each.
#define STGV_FOR_EACH_PAIR(X) X(27, 19) X(27, 7) X(19, 7) X(27, 27) X(19, 19) X(19, 15) X(15, 7) X(7, 27)

// Blocks of the plain node kernels (node_threads(n) consecutive nodes each).
inline unsigned node_blocks(int n) {
  return (unsigned)(((int64_t)n * n * n + node_threads(n) - 1) / node_threads(n));
}

// Whether a step's loads and stores go through the caches instead of bypassing them: for a
// state (`bytes` of populations) that stays in the 256 MB last-level cache from step to step.
// Measured on gfx950, mean step in us, bypassing / cached: FP32 27 x 19 56^3 (32 MB) 15.2 / 11.7,
// 72^3 27.0 / 22.9, 90^3 49.7 / 42.8, 104^3 (207 MB) 75.0 / 63.9, 112^3 (258 MB) 96.8 / 78.6,
// 120^3 (318 MB) 115.5 / 117.8, 128^3 124 / 149; FP16 64^3 10.7 / 9.2, 96^3 (BF16) 34.3 / 28.3,
// 128^3 (193 MB) 69.7 / 60.2, 140^3 (252 MB) 100.8 / 79.6, 144^3 (275 MB) 106.6 / 115.8,
// 160^3 141 / 149.  The A-B push always does, FP32 128^3 181 / 154, 200^3 944 / 652, 256^3 1526 / 1220,
// FP16 256^3 730 / 606.
#ifndef STGV_CACHED_BYTES
#define STGV_CACHED_BYTES ((size_t)256 << 20)
#endif
inline bool cached_state(size_t bytes) { return bytes <= STGV_CACHED_BYTES; }

// Rows of the box for the shifted odd step.  Where rows are no whole 128-byte lines, the lines of
// the x-aligned directions are shared by wavefronts too, and everything goes through the caches.
// Mean step in us, bypassing / x-aligned loads cached / stores cached as well: FP32 130^3 148 /
// 145 / 139, 200^3 596 / 575 / 561, 250^3 1220 / 1174 / 1130, 300^3 2094 / 2002 / 1952; FP16
// 150^3 129 / 115 / 115, 250^3 599 / 549 / 543; with whole lines, the first two, FP32 160^3 270 /
// 285, 320^3 2250 / 2338, FP16 320^3 1158 / 1171.
inline int row_kind(int n, size_t elem) {
  return n % 64 == 0 ? ROWS_WAVES : ((size_t)n * elem % 128 == 0 ? ROWS_LINES : ROWS_ANY);
}

// Whether the plain odd step runs row-aligned through an LDS ring (lbm_step_ring_kernel):
// on blocks of whole rows that tile the box or on 256-node blocks holding part of one
// row (n a multiple of 256, from 512); whole rows from n = 128 for 2-byte storage, from
// n = 256 for FP32 (FP32 at 128^3 and 64^3 lost 13 % and 2.5 % with it).  Only for the
// stencil pairs where it measured faster (ring_pair).  Measured on gfx950 (odd step, ms,
// shifted loads and stores -> ring): 256^3 FP32 27x19 1.141 -> 1.090 (2 blocks per CU,
// ring_step_lds), 19x19 0.957 -> 0.871, 7x27 0.819 -> 0.805; FP16 27x19 0.567 -> 0.549,
// 27x7 0.403 -> 0.396; 512^3 27x19 FP32 9.61 -> 9.22, FP16 4.80 and BF16 4.82 against 5.22
// and 9.5 for LDS-staged stores alone.  Slower with the ring, so shifted: FP32 27x27
// (1.377 -> 1.822), 19x15, 15x7, 19x7, 27x7 (within 1 %); FP16 19x7 (0.294 -> 0.308).
template <int QF, int QG>
constexpr bool ring_pair(size_t elem) {
  return elem == 4 ? ((QF == 27 && QG == 19) || (QF == 19 && QG == 19) || (QF == 7 && QG == 27))
                   : ((QF == 27 && QG == 19) || (QF == 27 && QG == 7));
}
inline bool ring_whole(int n, size_t elem) { return n == 256 || (n == 128 && elem != 4); }
inline bool ring_part(int n) { return n >= 512 && n % 256 == 0; }
// Blocks of n x 256 / n nodes (whole rows) or of 256 nodes of one row.
inline LaunchShape ring_launch(int n) {
  LaunchShape s;
  s.block = n < 256 ? dim3(n, 256 / n, 1) : dim3(256, 1, 1);
  s.grid = dim3(n / s.block.x, n / s.block.y, n);
  return s;
}

// Blocks resident per CU for the plain even step (0 = as many as the registers allow), set
// by requesting unused dynamic LDS (160 KiB per CU): FP32 storage for n >= 256, 2-byte
// storage for n >= 512.  The even step keeps every population array of its resident
// wavefronts open at once; past ~70-95 KB of loads in flight per CU more wavefronts only
// add open streams.  Measured on gfx950 (D3Q27 x D3Q19 even step, ms): FP32 at 2 blocks
// instead of 4, 256^3 1.137 -> 1.080, 384^3 4.02 -> 3.84, 512^3 9.26 -> 8.98 (3 blocks:
// 1.131 at 256^3); 2-byte storage at 3 blocks instead of 4, 512^3 FP16 4.67 -> 4.42, BF16
// 5.00 -> 4.92 (before its loads were batched), while 256^3 and 128^3 lose with any cap.  The shifted odd step, whose
// x-shifted lines neighbouring wavefronts share, gains nothing from a cap; the ring odd
// step has its own (ring_step_lds).
// The caps assume a step that issues its loads in two batches; the BF16 even step is made
// to (lbm_step_kernel), and is then best with FP16's caps.
#ifndef STGV_EVEN_CAP_FP32
#define STGV_EVEN_CAP_FP32 2
#endif
#ifndef STGV_EVEN_CAP_2B
#define STGV_EVEN_CAP_2B 3
#endif
// The passes that read the state in natural order without or beside the collision have caps of
// their own: diagnostic step FP32 2 (256^3 1314 -> 1269 us, 384^3 -7 %; 2-byte loses with any);
// fields FP32 2 (256^3 675 -> 645, 512^3 5250 -> 4919), 2-byte 3 (256^3 FP16 367 -> 352); fields and
// partials FP32 3 (256^3 record 722 -> 709, 512^3 5910 -> 5670), 2-byte 4 (436 -> 428).
inline size_t even_step_lds(size_t elem, int n, int flags) {
  int cap = 0;
  if (flags == K_COLLIDE) cap = elem == 4 ? (n >= 256 ? STGV_EVEN_CAP_FP32 : 0) : (n >= 512 ? STGV_EVEN_CAP_2B : 0);
  else if (n >= 256 && flags == (K_COLLIDE | K_FIELDS | K_PARTIALS)) cap = elem == 4 ? 2 : 0;
  else if (n >= 256 && flags == K_FIELDS) cap = elem == 4 ? 2 : 3;
  else if (n >= 256 && flags == (K_FIELDS | K_PARTIALS)) cap = elem == 4 ? 3 : 4;
  if (cap <= 0) return 0;
  // just over a (cap + 1)-th of the CU's LDS, so that cap blocks fit and cap + 1 do not
  size_t b = (160u * 1024u) / (size_t)(cap + 1) + 1024u;
  return b > 65536u ? 65536u : b;
}

// Blocks resident per CU for the ring odd step (0 = as many as registers and its LDS
// allow), counting the kernel's own LDS of `static_lds` bytes: FP32 at 2 (256^3 odd step
// 1.103 -> 1.088 ms, 512^3 9.37 -> 9.22 against no cap; at 3, 1.106); 2-byte storage lost
// with a cap of 2 (256^3 0.553 -> 0.600), gained nothing at 3 or 4 (512^3), and keeps none.
#ifndef STGV_ODD_CAP_FP32
#define STGV_ODD_CAP_FP32 2
#endif
#ifndef STGV_ODD_CAP_2B
#define STGV_ODD_CAP_2B 0
#endif
inline size_t ring_step_lds(size_t elem, size_t static_lds) {
  const int cap = elem == 4 ? STGV_ODD_CAP_FP32 : STGV_ODD_CAP_2B;
  if (cap <= 0) return 0;
  const size_t want = (160u * 1024u) / (size_t)(cap + 1) + 1024u;
  if (want <= static_lds) return 0;
  return want > 65536u ? 65536u - static_lds : want - static_lds;
}

// Every function returns the launch error (hipSuccess when queued).  cached: cached_state of
// the population buffer.
template <typename T, typename C>
hipError_t launch_step(int qf, int qg, int force, int mode, int flags, bool cached, hipStream_t st, T* pop, T* dst,
                       Geometry geo, PhysConsts c, float* fields, double* partials);

template <typename T>
hipError_t launch_init(int qf, int qg, hipStream_t st, T* pop, Geometry geo, double u0, double noise_amp, uint64_t seed);

// Free streaming (lbm_stream_kernel) in layout MODE, from pop into dst.
template <typename T>
hipError_t launch_stream(int qf, int qg, int mode, bool cached, hipStream_t st, T* pop, T* dst, Geometry geo);

template <typename T>
hipError_t launch_canon(int qf, int qg, int mode, hipStream_t st, const T* pop, Geometry geo, float* out);

template <typename T>
hipError_t launch_load(int qf, int qg, hipStream_t st, T* pop, Geometry geo, const float* in);

}  // namespace stgv
