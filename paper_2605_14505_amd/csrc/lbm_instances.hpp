// Template instances of the node kernels for one storage type STGV_T and one
// compute type STGV_C.  Included once per (storage, compute) pair by the
// lbm_*.hip translation units; the layout kernels (init, canonicalise, load)
// are instantiated by the FP32-compute unit of each storage type
// (STGV_LAYOUT_KERNELS).
#pragma once
#include "lbm_kernels.hpp"
#include "lbm_launch.hpp"

namespace stgv {
// Internal linkage: every (storage, compute) translation unit has its own
// helpers, whose template arguments do not name the compute type.
namespace {

template <int QF, int QG, int FORCE, typename T, int MODE, int FLAGS, int ROWS, bool CACHED>
hipError_t go_step(hipStream_t st, T* pop, T* dst, Geometry geo, PhysConsts c, float* fields, double* partials) {
  const size_t lds = MODE == MODE_EVEN ? even_step_lds(sizeof(T), geo.n, FLAGS) : 0;
  hipLaunchKernelGGL((lbm_step_kernel<QF, QG, FORCE, T, STGV_C, MODE, FLAGS, ROWS, CACHED>), dim3(node_blocks(geo.n)),
                     dim3(node_threads(geo.n)), lds, st, pop, dst, geo, c, fields, partials);
  return hipGetLastError();
}

template <int QF, int QG, int FORCE, typename T, bool CACHED>
hipError_t step_mode(int mode, bool diag, hipStream_t st, T* pop, T* dst, Geometry geo, PhysConsts c, float* fields,
                     double* partials) {
  constexpr int STEP = K_COLLIDE;
  constexpr int STEP_DIAG = K_COLLIDE | K_FIELDS | K_PARTIALS;
#define STGV_GO(M, FL, ROWS) return go_step<QF, QG, FORCE, T, M, FL, ROWS, CACHED>(st, pop, dst, geo, c, fields, partials)
  if (mode == MODE_EVEN) { if (diag) STGV_GO(MODE_EVEN, STEP_DIAG, ROWS_ANY); STGV_GO(MODE_EVEN, STEP, ROWS_ANY); }
  if (mode == MODE_AB)      // through the caches whatever the box: every shifted store shares its lines
    return diag ? go_step<QF, QG, FORCE, T, MODE_AB, STEP_DIAG, ROWS_ANY, true>(st, pop, dst, geo, c, fields, partials)
                : go_step<QF, QG, FORCE, T, MODE_AB, STEP, ROWS_ANY, true>(st, pop, dst, geo, c, fields, partials);
  if (mode != MODE_ODD) return hipErrorInvalidValue;
  if (diag) {
    if constexpr (!CACHED) {      // 250^3, a record every step: FP32 1325 -> 1255 us, FP16 793 -> 780
      if (row_kind(geo.n, sizeof(T)) == ROWS_ANY) STGV_GO(MODE_ODD, STEP_DIAG, ROWS_ANY);
    }
    STGV_GO(MODE_ODD, STEP_DIAG, ROWS_LINES);
  }
  if constexpr (sizeof(STGV_C) == 4 && ring_pair<QF, QG>(sizeof(T))) {
    const bool whole = ring_whole(geo.n, sizeof(T));
    if (whole || ring_part(geo.n)) {
      const LaunchShape sh = ring_launch(geo.n);
      const size_t lds = ring_step_lds(sizeof(T), (size_t)(x_moving<QF>() + x_moving<QG>()) * 256 * sizeof(T));
      if (whole)
        hipLaunchKernelGGL((lbm_step_ring_kernel<QF, QG, FORCE, T, STGV_C, false, CACHED && sizeof(T) != 4>), sh.grid,
                           sh.block, lds, st, pop, geo, c);
      else
        hipLaunchKernelGGL((lbm_step_ring_kernel<QF, QG, FORCE, T, STGV_C, true, false>), sh.grid, sh.block, lds, st,
                           pop, geo, c);
      return hipGetLastError();
    }
  }
  const int rows = row_kind(geo.n, sizeof(T));
  if (rows == ROWS_WAVES) STGV_GO(MODE_ODD, STEP, ROWS_WAVES);
  if constexpr (!CACHED && sizeof(T) == 4) {      // 2-byte rows of whole lines are whole wavefronts
    if (rows == ROWS_LINES) STGV_GO(MODE_ODD, STEP, ROWS_LINES);
  }
#undef STGV_GO
  // ragged rows go through the caches in any case; only kLoadsFirst tells large states from small
  return go_step<QF, QG, FORCE, T, MODE_ODD, STEP, ROWS_ANY, CACHED || sizeof(T) != 4 || sizeof(STGV_C) != 4>(st, pop, dst, geo, c, fields, partials);
}

template <int QF, int QG, int FORCE, typename T>
hipError_t step_force(int mode, bool diag, bool cached, hipStream_t st, T* pop, T* dst, Geometry geo, PhysConsts c,
                      float* fields, double* partials) {
  return cached ? step_mode<QF, QG, FORCE, T, true>(mode, diag, st, pop, dst, geo, c, fields, partials)
                : step_mode<QF, QG, FORCE, T, false>(mode, diag, st, pop, dst, geo, c, fields, partials);
}

template <int QF, int QG, typename T>
hipError_t step_pair(int force, int mode, int flags, bool cached, hipStream_t st, T* pop,
                     T* dst, Geometry geo, PhysConsts c, float* fields, double* partials) {
  constexpr int STEP = K_COLLIDE;
  constexpr int STEP_DIAG = K_COLLIDE | K_FIELDS | K_PARTIALS;
  constexpr int SAMPLE = K_FIELDS | K_PARTIALS;
  constexpr int FIELDS = K_FIELDS;
  if (flags == STEP || flags == STEP_DIAG) {
    const bool d = flags == STEP_DIAG;
    switch (force) {
      case FORCE_GUO: return step_force<QF, QG, FORCE_GUO, T>(mode, d, cached, st, pop, dst, geo, c, fields, partials);
      case FORCE_SHIFT: return step_force<QF, QG, FORCE_SHIFT, T>(mode, d, cached, st, pop, dst, geo, c, fields, partials);
      case FORCE_EDM: return step_force<QF, QG, FORCE_EDM, T>(mode, d, cached, st, pop, dst, geo, c, fields, partials);
      case FORCE_HCZ: return step_force<QF, QG, FORCE_HCZ, T>(mode, d, cached, st, pop, dst, geo, c, fields, partials);
      default: return hipErrorInvalidValue;
    }
  }
  // Moment-only passes read the natural layout (MODE_EVEN, also the AB lattice)
  // or the odd AA layout; the physical velocity does not depend on the forcing.  They bypass the
  // caches as in the step of a large box of whole lines, whatever the state: through the caches a
  // record of a state held there would be faster (after an odd number of steps 90^3 FP32 48 -> 36 us,
  // 128^3 FP16 64 -> 50; 64^3 21 -> 18).
#define STGV_GO(M, FL) return go_step<QF, QG, FORCE_GUO, T, M, FL, ROWS_LINES, false>(st, pop, dst, geo, c, fields, partials)
  const int gm = (mode == MODE_ODD) ? MODE_ODD : MODE_EVEN;
  if (flags == SAMPLE) {
    if (gm == MODE_EVEN) STGV_GO(MODE_EVEN, SAMPLE);
    STGV_GO(MODE_ODD, SAMPLE);
  }
  if (flags == FIELDS) {
    if (gm == MODE_EVEN) STGV_GO(MODE_EVEN, FIELDS);
    STGV_GO(MODE_ODD, FIELDS);
  }
#undef STGV_GO
  return hipErrorInvalidValue;
}

}  // namespace

template <>
hipError_t launch_step<STGV_T, STGV_C>(int qf, int qg, int force, int mode, int flags, bool cached,
                               hipStream_t st, STGV_T* pop, STGV_T* dst,
                               Geometry geo, PhysConsts c, float* fields, double* partials) {
#define STGV_STEP_PAIR(A, B) \
  if (qf == A && qg == B) return step_pair<A, B, STGV_T>(force, mode, flags, cached, st, pop, dst, geo, c, fields, partials);
  STGV_FOR_EACH_PAIR(STGV_STEP_PAIR)
#undef STGV_STEP_PAIR
  return hipErrorInvalidValue;
}

#ifdef STGV_LAYOUT_KERNELS
template <>
hipError_t launch_init<STGV_T>(int qf, int qg, hipStream_t st, STGV_T* pop,
                               Geometry geo, double u0, double noise_amp, uint64_t seed) {
#define STGV_INIT(A, B) \
  if (qf == A && qg == B) { \
    hipLaunchKernelGGL((lbm_init_tgv_kernel<A, B, STGV_T>), dim3(node_blocks(geo.n)), dim3(node_threads(geo.n)), 0, st, pop, geo, u0, noise_amp, seed); \
    return hipGetLastError(); }
  STGV_FOR_EACH_PAIR(STGV_INIT)
#undef STGV_INIT
  return hipErrorInvalidValue;
}

template <int A, int B, bool CACHED>
static hipError_t stream_pair(int mode, hipStream_t st, STGV_T* pop, STGV_T* dst, Geometry geo) {
  const dim3 grid(node_blocks(geo.n)), block(node_threads(geo.n));
  if constexpr (ring_pair<A, B>(sizeof(STGV_T))) {
    const bool whole = ring_whole(geo.n, sizeof(STGV_T));
    if (mode == MODE_ODD && (whole || ring_part(geo.n))) {
      const LaunchShape sh = ring_launch(geo.n);
      const size_t lds = ring_step_lds(sizeof(STGV_T), (size_t)(x_moving<A>() + x_moving<B>()) * 256 * sizeof(STGV_T));
      if (whole) hipLaunchKernelGGL((lbm_stream_ring_kernel<A, B, STGV_T, false, CACHED && sizeof(STGV_T) != 4>), sh.grid, sh.block, lds, st, pop, geo);
      else hipLaunchKernelGGL((lbm_stream_ring_kernel<A, B, STGV_T, true, false>), sh.grid, sh.block, lds, st, pop, geo);
      return hipGetLastError();
    }
  }
#define STGV_STREAM_GO(MODE, ROWS, C, LDS) \
  hipLaunchKernelGGL((lbm_stream_kernel<A, B, STGV_T, MODE, ROWS, C>), grid, block, LDS, st, pop, dst, geo)
  if (mode == MODE_EVEN) {
    STGV_STREAM_GO(MODE_EVEN, ROWS_ANY, CACHED, even_step_lds(sizeof(STGV_T), geo.n, K_COLLIDE));
    return hipGetLastError();
  }
  if (mode == MODE_AB) {
    STGV_STREAM_GO(MODE_AB, ROWS_ANY, true, 0);
    return hipGetLastError();
  }
  const int rows = row_kind(geo.n, sizeof(STGV_T));
  if (rows == ROWS_WAVES) {
    STGV_STREAM_GO(MODE_ODD, ROWS_WAVES, CACHED, 0);
    return hipGetLastError();
  }
  if constexpr (!CACHED && sizeof(STGV_T) == 4) {      // 2-byte rows of whole lines are whole wavefronts
    if (rows == ROWS_LINES) {
      STGV_STREAM_GO(MODE_ODD, ROWS_LINES, false, 0);
      return hipGetLastError();
    }
  }
  STGV_STREAM_GO(MODE_ODD, ROWS_ANY, true, 0);
#undef STGV_STREAM_GO
  return hipGetLastError();
}

template <>
hipError_t launch_stream<STGV_T>(int qf, int qg, int mode, bool cached, hipStream_t st, STGV_T* pop, STGV_T* dst,
                                 Geometry geo) {
#define STGV_STREAM(A, B) \
  if (qf == A && qg == B) \
    return cached ? stream_pair<A, B, true>(mode, st, pop, dst, geo) : stream_pair<A, B, false>(mode, st, pop, dst, geo);
  STGV_FOR_EACH_PAIR(STGV_STREAM)
#undef STGV_STREAM
  return hipErrorInvalidValue;
}

// Conversion in natural order (lbm_convert_kernel): four values at a time where every array of the
// natural side starts on 16 bytes and holds a multiple of four values (n even makes n^3 a multiple of
// 8).  Elsewhere four of a 2-byte type all the same, single values of FP32.  Read-back / load in us,
// one thread per node, single values, four at a time: FP16 101^3 75 / 70, 97 / 86, 57 / 60, 251^3
// 1290 / 1230, 1310 / 1110, 757 / 718; FP32 225^3 1115 / 1141, 714 / 675, 798 / 719, 251^3 1678 /
// 1342, 991 / 931, 1096 / 961.
template <bool LOAD>
static hipError_t convert(int arrays, hipStream_t st, STGV_T* pop, Geometry geo, float* natural) {
  constexpr int V = 4, VU = sizeof(STGV_T) == 4 ? 1 : V;
  const bool aligned = geo.n % 2 == 0 && (uintptr_t)natural % 16 == 0;
  const bool cached = cached_state((size_t)arrays * geo.n3 * (LOAD ? sizeof(float) : sizeof(STGV_T)));
  const unsigned chunk = kNodeBlock * kConvertUnroll * (aligned ? V : VU);
  const dim3 grid((geo.n3 + chunk - 1) / chunk, (unsigned)arrays), block(kNodeBlock);
#define STGV_CONVERT(W, ALIGNED, CACHED) \
  hipLaunchKernelGGL((lbm_convert_kernel<STGV_T, W, LOAD, ALIGNED, CACHED>), grid, block, 0, st, pop, geo, natural)
  if (aligned) { if (cached) STGV_CONVERT(V, true, true); else STGV_CONVERT(V, true, false); }
  else { if (cached) STGV_CONVERT(VU, false, true); else STGV_CONVERT(VU, false, false); }
#undef STGV_CONVERT
  return hipGetLastError();
}

template <>
hipError_t launch_canon<STGV_T>(int qf, int qg, int mode, hipStream_t st, const STGV_T* pop, Geometry geo, float* out) {
  if (mode != MODE_ODD) return convert<false>(qf + qg, st, const_cast<STGV_T*>(pop), geo, out);
  const bool lines = geo.n3 % 32 == 0 && (uintptr_t)out % 128 == 0;
  const dim3 grid(node_blocks(geo.n)), block(node_threads(geo.n));
#define STGV_CANON(A, B) \
  if (qf == A && qg == B) { \
    if (lines) hipLaunchKernelGGL((lbm_canon_odd_kernel<A, B, STGV_T, true>), grid, block, 0, st, pop, geo, out); \
    else hipLaunchKernelGGL((lbm_canon_odd_kernel<A, B, STGV_T, false>), grid, block, 0, st, pop, geo, out); \
    return hipGetLastError(); }
  STGV_FOR_EACH_PAIR(STGV_CANON)
#undef STGV_CANON
  return hipErrorInvalidValue;
}

template <>
hipError_t launch_load<STGV_T>(int qf, int qg, hipStream_t st, STGV_T* pop, Geometry geo, const float* in) {
  return convert<true>(qf + qg, st, pop, geo, const_cast<float*>(in));
}
#endif  // STGV_LAYOUT_KERNELS

}  // namespace stgv
