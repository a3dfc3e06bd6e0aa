// Kernels of the DDF lattice Boltzmann step and its diagnostics (gfx950).
#pragma once
#include "lbm_device.hpp"

namespace stgv {

// ---------------------------------------------------------------------------
// Fused stream-collide-force step (optionally with the diagnostic moments)
//
// `pop` is the population array (AA) or the source lattice (AB); `dst` is the AB
// destination and equals `pop` otherwise.
// ---------------------------------------------------------------------------
// Minimum resident 256-thread blocks per CU requested from the register allocator
// (0 = compiler's choice): STGV_EVEN_MIN_BLOCKS for the plain even step with 4-byte
// storage and arithmetic (the instance that fits a tighter register budget without
// spilling), STGV_STEP_MIN_BLOCKS for every other step instance.
#ifndef STGV_STEP_MIN_BLOCKS
#define STGV_STEP_MIN_BLOCKS 0
#endif
#ifndef STGV_EVEN_MIN_BLOCKS
#define STGV_EVEN_MIN_BLOCKS STGV_STEP_MIN_BLOCKS
#endif
template <int MODE, int FLAGS, typename T, typename C>
constexpr int step_min_blocks() {
  const int b = (MODE == MODE_EVEN && FLAGS == K_COLLIDE && sizeof(T) == 4 && sizeof(C) == 4)
                    ? STGV_EVEN_MIN_BLOCKS : STGV_STEP_MIN_BLOCKS;
  return b > 0 ? b : 1;
}
#define STGV_STEP_BOUNDS_FOR(MODE, FLAGS, T, C) __launch_bounds__(256, (step_min_blocks<MODE, FLAGS, T, C>()))
#define STGV_STEP_BOUNDS STGV_STEP_BOUNDS_FOR(MODE_ODD, K_COLLIDE, T, C)

// Nodes of the plain node kernels: block b holds the node_threads(n) consecutive nodes from
// node_threads(n) b of the linear order x + n (y + n z), whatever the box, so that no lane is idle
// and every wavefront's access is one contiguous run.  Against x-y block shapes (128 x 2 for
// 90^3 and 100^3, 32 x 8 for 96^3 and 160^3), mean step in us: 90^3 FP16 27 x 7 35.6 -> 23.8,
// FP32 27 x 19 72.2 -> 50.1; 100^3 FP32 91.7 -> 67.5; 160^3 FP16 215 -> 145; 96^3 FP32
// 60.2 -> 58.5; boxes whose rows are whole wavefronts are unchanged within 1 %.  Blocks are
// taken in the XCD-aware order of block_at.
template <int MODE>
__device__ __forceinline__ uint32_t node_block(const Geometry& geo) {
  return block_at(blockIdx.x, gridDim.x, geo, MODE != MODE_EVEN);
}
template <int MODE>
__device__ __forceinline__ uint32_t node_of(const Geometry& geo) {
  return node_block<MODE>(geo) * blockDim.x + threadIdx.x;
}

// Neighbour offsets of node i.  ROWS_WAVES: n is a multiple of 64, so a wavefront's nodes lie in
// one row and its y and z are scalar.  Even steps address their own node only.
template <int MODE, int ROWS>
__device__ __forceinline__ NodeIndex index_of(uint32_t i, const Geometry& geo) {
  NodeIndex ix{};
  ix.base = i;
  if constexpr (MODE != MODE_EVEN) {
    uint32_t r = over_n(i, geo);
    const uint32_t x = i - r * (uint32_t)geo.n;
    if constexpr (ROWS == ROWS_WAVES) r = (uint32_t)__builtin_amdgcn_readfirstlane((int)r);
    const uint32_t z = over_n(r, geo);
    ix = make_index((int)x, (int)(r - z * (uint32_t)geo.n), (int)z, geo.n);
  }
  return ix;
}

// Block coordinates of the row-aligned kernels, whose blocks are (bx, by) nodes of whole or
// part rows; renumbered as above where rows are split.
struct BlockXYZ { int bx, by, bz; };

__device__ __forceinline__ BlockXYZ ring_block() {
  BlockXYZ b{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z};
  const int gx = (int)gridDim.x, gy = (int)gridDim.y;
  if (gx > 1 && ((gy * (int)gridDim.z) & 7) == 0) {
    const int L = b.bx + gx * (b.by + gy * b.bz);
    const int k = L & 7, rest = L >> 3;
    const int rg = (rest / gx) * 8 + k;
    b.bx = rest % gx;
    b.by = rg % gy;
    b.bz = rg / gy;
  }
  return b;
}

// Left alone, the compiler has the BF16 even step issue all 46 loads before its first
// wait, where the FP16 one issues 32, waits, then the rest; at the occupancy caps of
// even_step_lds that keeps more bytes in flight than the step can use.  An empty asm that
// takes the 27 f values makes the wavefront wait for them before it issues the g loads.  BF16 even step,
// ms: 512^3 4.75 -> 4.50 (at FP16's 3 blocks per CU; with a cap of 2 and all loads first
// 4.59-4.75), 256^3 0.548 -> 0.549.
template <int MODE, int FLAGS, typename T, int QF>
constexpr bool kBatchBf16 = MODE == MODE_EVEN && FLAGS == K_COLLIDE && std::is_same<T, bf16_t>::value && QF == 27;
#define STGV_OPERANDS_27(a) "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]), "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15]), "+v"(a[16]), "+v"(a[17]), "+v"(a[18]), "+v"(a[19]), "+v"(a[20]), "+v"(a[21]), "+v"(a[22]), "+v"(a[23]), "+v"(a[24]), "+v"(a[25]), "+v"(a[26])

// FP32 states that stay in the last-level cache: all loads of the in-place steps ahead of the first
// wait.  Their time is latency, and the compiler left a wait for the first values between two
// batches of the even step's loads and, with Guo forcing, between single loads of the odd step's.
// Mean step in us: 8^3 4.37 -> 4.29, 32^3 5.36 -> 5.26, 64^3 16.05 -> 15.90, 90^3 42.7 -> 42.1,
// 27 x 27 64^3 18.98 -> 18.08.  2-byte storage (BF16 64^3 9.33 -> 9.46), the A-B push (128^3 153.3
// -> 154.9) and larger states (192^3 464 -> 468, 250^3 1116 -> 1120, with Guo forcing 1091 -> 1098) are
// better left alone.
template <int MODE, int FLAGS, typename T, typename C, bool CACHED>
constexpr bool kLoadsFirst = CACHED && MODE != MODE_AB && FLAGS == K_COLLIDE && sizeof(T) == 4 && sizeof(C) == 4;

template <int QF, int QG, int FORCE, typename T, typename C, int MODE, int FLAGS, int ROWS, bool CACHED>
__global__ STGV_STEP_BOUNDS_FOR(MODE, FLAGS, T, C) void lbm_step_kernel(T* pop, T* dst, Geometry geo,
                                                       PhysConsts c, float* __restrict__ fields,
                                                       double* __restrict__ partials) {
  const uint32_t node = node_of<MODE>(geo);
  const bool active = node < geo.n3;
  constexpr bool kPart = (FLAGS & K_PARTIALS) != 0;
  if (!kPart && !active) return;

  double acc[NPART];
#pragma unroll
  for (int k = 0; k < NPART; ++k) acc[k] = 0.0;

  if (active) {
    const NodeIndex ix = index_of<MODE, ROWS>(node, geo);
    C f[QF], g[QG];
    gather<QF, T, MODE, ROWS != ROWS_ANY, CACHED>(f, pop, 0, ix, geo.stride);
    if constexpr (kBatchBf16<MODE, FLAGS, T, QF>) asm volatile("" : STGV_OPERANDS_27(f) :: "memory");
    gather<QG, T, MODE, ROWS != ROWS_ANY, CACHED>(g, pop, QF, ix, geo.stride);
    if constexpr (kLoadsFirst<MODE, FLAGS, T, C, CACHED>) __builtin_amdgcn_sched_barrier(0);
    StepMacro<C> m;
    step_macro<QF, QG, FORCE, sizeof(T) == 4>(f, g, c, m);
    if (FLAGS & (K_FIELDS | K_PARTIALS)) {
      const NodeMacro<C> dm = diag_macro(m);
      if (FLAGS & K_FIELDS) write_fields(dm, fields, node, (int64_t)geo.n3);
      if (kPart) node_partials(dm, c, acc);
    }
    if (FLAGS & K_COLLIDE) {
      step_collide<QF, QG, FORCE, sizeof(T) == 4>(f, g, c, m);
      constexpr bool cached = CACHED || (MODE == MODE_ODD && ROWS == ROWS_ANY);      // row_kind
      scatter<QF, T, MODE, cached>(f, dst, 0, ix, geo.stride);
      scatter<QG, T, MODE, cached>(g, dst, QF, ix, geo.stride);
    }
  }
  if (kPart) {
    block_reduce_store<NPART, (1u << P_UMAX2)>(acc, partials + (int64_t)node_block<MODE>(geo) * NPART);
  }
}

// The plain odd step row-aligned, its x-shift taken through a ring in LDS per block row
// (row_load / row_pick / row_put / row_store), on the shapes of ring_whole and ring_part (blocks of
// whole rows, or 256-node blocks holding part of one row), which tile the box exactly,
// so every lane is active and reaches the barriers.
// PART: blocks holding part of a row, whose x-moving loads and stores use the cache
// policy STGV_RING_PART_NT_XLOAD / STGV_RING_PART_NT_XSTORE (1 = bypass); whole-row
// blocks bypass the caches for every access.  CACHED: every access goes through them
// (cached_state).  A seam lane's load shares its line with
// the neighbouring block's aligned load, which finds it in L2 only if it was loaded
// cached: 512^3 odd step FP16 5.21 -> 4.80 ms, BF16 5.67 -> 4.82 ms with cached x-moving
// loads; cached x-moving stores changed nothing further (4.80 / 4.80) and alone gave
// 4.90 / 4.96.
#ifndef STGV_RING_PART_NT_XLOAD
#define STGV_RING_PART_NT_XLOAD 0
#endif
#ifndef STGV_RING_PART_NT_XSTORE
#define STGV_RING_PART_NT_XSTORE 1
#endif
// All of a ring kernel's loads, issued before the first wait: left to itself the compiler
// wrote each value to the ring as it arrived in some instances and waited for every load by
// itself (BF16 27 x 19 with Guo or HCZ forcing, odd step at 256^3: 1490 us against 555).
template <int QF, int QG, typename T, bool NT0, bool NL, typename C>
__device__ __forceinline__ void ring_loads(C* f, C* g, T (*xs)[256], const T* pop, const NodeIndex& ix, int64_t stride,
                                           const RowLane& l) {
  T rf[QF], rg[QG];
  row_load<QF, T, NT0, NL>(rf, pop, 0, ix, stride, l, std::make_integer_sequence<int, QF>{});
  row_load<QG, T, NT0, NL>(rg, pop, QF, ix, stride, l, std::make_integer_sequence<int, QG>{});
  __builtin_amdgcn_sched_barrier(0);
  row_stage<QF>(f, rf, xs, 0, l, std::make_integer_sequence<int, QF>{});
  row_stage<QG>(g, rg, xs, x_moving<QF>(), l, std::make_integer_sequence<int, QG>{});
}

template <int QF, int QG, int FORCE, typename T, typename C, bool PART, bool CACHED>
__global__ STGV_STEP_BOUNDS void lbm_step_ring_kernel(T* pop, Geometry geo, PhysConsts c) {
  constexpr bool NL = !CACHED && (!PART || STGV_RING_PART_NT_XLOAD), NS = !CACHED && (!PART || STGV_RING_PART_NT_XSTORE);
  constexpr int KF = x_moving<QF>(), KG = x_moving<QG>();
  __shared__ T xs[KF + KG][256];
  const int n = geo.n;
  const BlockXYZ blk = ring_block();
  const int x = blk.bx * blockDim.x + threadIdx.x;
  const int y = blk.by * blockDim.y + threadIdx.y;
  const NodeIndex ix = make_index(x, y, blk.bz, n);
  const RowLane l = make_rowlane(x, n);
  C f[QF], g[QG];
  ring_loads<QF, QG, T, !CACHED, NL>(f, g, xs, pop, ix, geo.stride, l);
  __syncthreads();
  row_pick<QF>(f, (const T(*)[256])xs, 0, l, std::make_integer_sequence<int, QF>{});
  row_pick<QG>(g, (const T(*)[256])xs, KF, l, std::make_integer_sequence<int, QG>{});
  __syncthreads();                      // every lane has taken its values before any put
  StepMacro<C> m;
  step_macro<QF, QG, FORCE, sizeof(T) == 4>(f, g, c, m);
  step_collide<QF, QG, FORCE, sizeof(T) == 4>(f, g, c, m);
  row_put<QF>(f, xs, 0, l, std::make_integer_sequence<int, QF>{});
  row_put<QG>(g, xs, KF, l, std::make_integer_sequence<int, QG>{});
  __syncthreads();
  row_store<QF, T, !CACHED, NS>(f, (const T(*)[256])xs, 0, pop, 0, ix, geo.stride, l, std::make_integer_sequence<int, QF>{});
  row_store<QG, T, !CACHED, NS>(g, (const T(*)[256])xs, KF, pop, QF, ix, geo.stride, l, std::make_integer_sequence<int, QG>{});
}

// ---------------------------------------------------------------------------
// Free streaming: the step's loads, stores, launch shape and block order with the
// identity in place of the collision, so every population moves one link along its
// velocity per call (the streaming half of Eqs. (5) and (11) alone).  Values pass
// through FP32, which holds every FP16 / BF16 value exactly, so a stream is exact in
// every storage type.  It is the ceiling of the step's own access pattern.
// ---------------------------------------------------------------------------
template <int QF, int QG, typename T, int MODE, int ROWS, bool CACHED>
__global__ __launch_bounds__(kNodeBlock) void lbm_stream_kernel(T* pop, T* dst, Geometry geo) {
  const uint32_t node = node_of<MODE>(geo);
  if (node >= geo.n3) return;
  const NodeIndex ix = index_of<MODE, ROWS>(node, geo);
  float f[QF], g[QG];
  gather<QF, T, MODE, ROWS != ROWS_ANY, CACHED>(f, pop, 0, ix, geo.stride);
  gather<QG, T, MODE, ROWS != ROWS_ANY, CACHED>(g, pop, QF, ix, geo.stride);
  scatter<QF, T, MODE, CACHED>(f, dst, 0, ix, geo.stride);
  scatter<QG, T, MODE, CACHED>(g, dst, QF, ix, geo.stride);
}

// The odd free-streaming step row-aligned, on the shapes where the odd step runs
// row-aligned (ring_whole, ring_part; every lane active).
template <int QF, int QG, typename T, bool PART, bool CACHED>
__global__ __launch_bounds__(256) void lbm_stream_ring_kernel(T* pop, Geometry geo) {
  constexpr bool NL = !CACHED && (!PART || STGV_RING_PART_NT_XLOAD), NS = !CACHED && (!PART || STGV_RING_PART_NT_XSTORE);
  constexpr int KF = x_moving<QF>(), KG = x_moving<QG>();
  __shared__ T xs[KF + KG][256];
  const int n = geo.n;
  const BlockXYZ blk = ring_block();
  const int x = blk.bx * blockDim.x + threadIdx.x;
  const int y = blk.by * blockDim.y + threadIdx.y;
  const NodeIndex ix = make_index(x, y, blk.bz, n);
  const RowLane l = make_rowlane(x, n);
  float f[QF], g[QG];
  ring_loads<QF, QG, T, !CACHED, NL>(f, g, xs, pop, ix, geo.stride, l);
  __syncthreads();
  row_pick<QF>(f, (const T(*)[256])xs, 0, l, std::make_integer_sequence<int, QF>{});
  row_pick<QG>(g, (const T(*)[256])xs, KF, l, std::make_integer_sequence<int, QG>{});
  __syncthreads();
  row_put<QF>(f, xs, 0, l, std::make_integer_sequence<int, QF>{});
  row_put<QG>(g, xs, KF, l, std::make_integer_sequence<int, QG>{});
  __syncthreads();
  row_store<QF, T, !CACHED, NS>(f, (const T(*)[256])xs, 0, pop, 0, ix, geo.stride, l, std::make_integer_sequence<int, QF>{});
  row_store<QG, T, !CACHED, NS>(g, (const T(*)[256])xs, KF, pop, QF, ix, geo.stride, l, std::make_integer_sequence<int, QG>{});
}

// ---------------------------------------------------------------------------
// Taylor-Green initial state (Eqs. (20)-(21)) in natural order.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  // one output of SplitMix64 (Steele, Lea & Flood 2014) from state x
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// One rounding of an FP64 value into the storage type.  FP32 rounds directly; FP16 and
// BF16 go through FP32 rounded to odd (truncate, then set the last bit when inexact),
// which carries at least two more significand bits than either, so the final
// round-to-nearest-even of the hardware conversion equals a direct rounding of the
// FP64 value.
__device__ __forceinline__ float round_to_odd_f32(double d) {
  float r = (float)d;
  if ((double)r != d) {
    uint32_t b = __float_as_uint(r);
    if (fabs((double)r) > fabs(d)) b -= 1u;     // step back toward zero (sign-magnitude)
    r = __uint_as_float(b | 1u);
  }
  return r;
}
__device__ __forceinline__ void store_once(float* p, double d) { store_as(p, (float)d); }
__device__ __forceinline__ void store_once(_Float16* p, double d) { store_as(p, round_to_odd_f32(d)); }
__device__ __forceinline__ void store_once(bf16_t* p, double d) { store_as(p, round_to_odd_f32(d)); }

template <int QF, int QG, typename T>
__global__ __launch_bounds__(kNodeBlock) void lbm_init_tgv_kernel(T* pop, Geometry geo, double u0,
                                                           double noise_amp, uint64_t seed) {
  using SF = Stencil<QF>;
  using SG = Stencil<QG>;
  const int n = geo.n;
  const uint32_t node = node_of<MODE_EVEN>(geo);
  if (node >= geo.n3) return;
  const int r = (int)(node / (uint32_t)n), x = (int)node - r * n, z = r / n, y = r - z * n;
  const double h = 2.0 * M_PI / n;
  const double X = h * x, Y = h * y, Z = h * z;
  const double vx = u0 * sin(X) * cos(Y) * cos(Z);
  const double vy = -u0 * cos(X) * sin(Y) * cos(Z);
  const double vz = 0.0;
  const double p0 = u0 * u0 / 16.0 * (cos(2.0 * X) + cos(2.0 * Y)) * (cos(2.0 * Z) + 2.0);
  const double drho = p0 / SF::cs2;
  const double rho = 1.0 + drho;
  const uint64_t ctr = (seed << 40) + (uint64_t)node;
  const double xi = (double)(splitmix64(ctr) >> 11) * 0x1.0p-53;
  const double rho_p = noise_amp * (2.0 * xi - 1.0);
  const double usq = vx * vx + vy * vy + vz * vz;
#pragma unroll
  for (int i = 0; i < QF; ++i) {
    const double eu = SF::ex[i] * vx + SF::ey[i] * vy + SF::ez[i] * vz;
    const double d = SF::w[i] * (drho + rho * (eu / SF::cs2 + eu * eu / (2.0 * SF::cs2 * SF::cs2)
                                               - usq / (2.0 * SF::cs2)));
    store_once(pop + (int64_t)i * geo.stride + node, d);
  }
#pragma unroll
  for (int j = 0; j < QG; ++j) {
    const double eu = SG::ex[j] * vx + SG::ey[j] * vy + SG::ez[j] * vz;
    const double poly = eu / SG::cs2 + eu * eu / (2.0 * SG::cs2 * SG::cs2) - usq / (2.0 * SG::cs2);
    const double d = SG::w[j] * (rho_p + (1.0 + rho_p) * poly);
    store_once(pop + (int64_t)(QF + j) * geo.stride + node, d);
  }
}

// ---------------------------------------------------------------------------
// Layout conversion: current layout -> natural FP32 deviations, and back.
// ---------------------------------------------------------------------------
// Where the array is in natural order (an even number of steps, A-B, a load) a conversion is a
// copy of each population array by itself: block (b, q) converts a contiguous chunk of array
// q, V values at a time (contiguous over a wavefront on both sides: eight of a 2-byte type
// left gaps between the 16-byte stores, 512^3 FP16 read-back 8.81 ms), all loads ahead of the
// stores.  The population arrays start on whole lines, the natural ones on any float (odd boxes,
// the caller's buffer); global memory takes four floats there all the same.  ALIGNED: the natural
// arrays start on 16 bytes; their stores bypass the caches only then.  CACHED: the source may still be
// in the last-level cache (cached_state of its size) and is read through the caches: load and read-back
// in us, bypassing / cached, 64^3 FP32 27.8 / 24.6 and 29.7 / 24.4, 101^3 FP16 60 / 51 and 54 / 53; a source
// of 326 MB (121^3 FP16 load) 91 / 97.
// HBM-bound, 5.7-5.9 TB/s: 512^3 FP16 read-back 7.86 -> 6.26 ms and
// load 7.33 -> 6.26, 256^3 FP32 1171 -> 1081 us and 1144 -> 1088, against one thread per node with
// 46 streams open.
constexpr int kConvertUnroll = 4;

template <typename T, int V> struct Packet { T v[V]; };
template <int BYTES, int ALIGN> struct PacketWord {
  typedef uint32_t type __attribute__((ext_vector_type(BYTES / 4), aligned(ALIGN)));
};
// ALIGN: what the address is a multiple of (4 for single values of any type).  NT: past the caches.
template <int V, int ALIGN, bool NT, typename T>
__device__ __forceinline__ Packet<T, V> load_packet(const T* p) {
  if constexpr (V == 1) return Packet<T, V>{{raw_load<NT>(p)}};
  else return __builtin_bit_cast(Packet<T, V>, get<NT>((const typename PacketWord<sizeof(T) * V, ALIGN>::type*)p));
}
template <int V, int ALIGN, bool NT, typename T>
__device__ __forceinline__ void store_packet(T* p, const Packet<T, V>& v) {
  if constexpr (V == 1) {
    raw_store<NT>(p, v.v[0]);
  } else {
    using Word = typename PacketWord<sizeof(T) * V, ALIGN>::type;
    put<NT>((Word*)p, __builtin_bit_cast(Word, v));
  }
}
template <typename T, int V>
__device__ __forceinline__ Packet<float, V> widened(const Packet<T, V>& t) {
  Packet<float, V> f;
#pragma unroll
  for (int j = 0; j < V; ++j) f.v[j] = load_as<float>(&t.v[j]);
  return f;
}
template <typename T, int V>
__device__ __forceinline__ Packet<T, V> narrowed(const Packet<float, V>& f) {
  Packet<T, V> t;
#pragma unroll
  for (int j = 0; j < V; ++j) t.v[j] = rounded((const T*)nullptr, f.v[j]);
  return t;
}

template <typename T, int V, bool LOAD, bool ALIGNED, bool CACHED>
__global__ __launch_bounds__(kNodeBlock) void lbm_convert_kernel(T* pop, Geometry geo, float* natural) {
  constexpr bool NT = ALIGNED || V == 1;
  T* const a = pop + (int64_t)blockIdx.y * geo.stride;
  float* const b = natural + (int64_t)blockIdx.y * geo.n3;
  const uint32_t e0 = (blockIdx.x * (kNodeBlock * kConvertUnroll) + threadIdx.x) * V, rest = geo.n3 % V, whole = geo.n3 - rest;
  Packet<float, V> f[kConvertUnroll];
#pragma unroll
  for (int k = 0; k < kConvertUnroll; ++k) {
    const uint32_t e = e0 + k * (kNodeBlock * V);
    if (e >= whole) continue;
    if constexpr (LOAD) f[k] = load_packet<V, 4, !CACHED>(b + e);
    else f[k] = widened(load_packet<V, V * sizeof(T), !CACHED>(a + e));
    // each packet of a 2-byte read-back is waited for here, which measures better than all four loads
    // in flight: 256^3 FP16 787 -> 743 us, BF16 780 -> 736, 250^3 796 -> 737 and 789 -> 737
    if constexpr (!LOAD && sizeof(T) == 2) asm volatile("" : "+v"(f[k].v[0]));
  }
#pragma unroll
  for (int k = 0; k < kConvertUnroll; ++k) {
    const uint32_t e = e0 + k * (kNodeBlock * V);
    if (e >= whole) continue;
    if constexpr (LOAD) store_packet<V, V * sizeof(T), true>(a + e, narrowed<T>(f[k]));
    else store_packet<V, 4, NT>(b + e, f[k]);
  }
  if (V > 1 && rest && blockIdx.x == 0 && threadIdx.x < rest) {       // the last values of an odd box
    const uint32_t e = whole + threadIdx.x;
    if constexpr (LOAD) store_packet<1, 4, true>(a + e, narrowed<T>(load_packet<1, 4, !CACHED>(b + e)));
    else store_packet<1, 4, NT>(b + e, widened(load_packet<1, 4, !CACHED>(a + e)));
  }
}

// Read-back of the odd AA layout: one thread per node, x-shifted loads.  The blocks are renumbered as
// in the odd step, and the stores bypass the caches only where every natural array starts on a whole
// line (LINES).  In us, x-y blocks with cached stores / linear order in dispatch order with stores
// that bypass / this: FP16 81^3 39 / 45 / 34, 90^3 45 / 56 / 40, 225^3 773 / 670-877 / 568; FP32 127^3
// 178 / 202 / 170, 251^3 1285 / 1495 / 1240; with whole lines, cached stores / this, FP16 128^3 126 / 81.
template <int QF, int QG, typename T, bool LINES>
__global__ __launch_bounds__(kNodeBlock) void lbm_canon_odd_kernel(const T* pop, Geometry geo,
                                                                   float* __restrict__ out) {
  const uint32_t node = node_of<MODE_ODD>(geo);
  if (node >= geo.n3) return;
  const NodeIndex ix = index_of<MODE_ODD, ROWS_ANY>(node, geo);
  const int64_t n3 = geo.n3;
  float f[QF], g[QG];
  gather<QF, T, MODE_ODD>(f, pop, 0, ix, geo.stride);
  gather<QG, T, MODE_ODD>(g, pop, QF, ix, geo.stride);
#pragma unroll
  for (int i = 0; i < QF; ++i) put<LINES>(out + i * n3 + node, f[i]);
#pragma unroll
  for (int j = 0; j < QG; ++j) put<LINES>(out + (QF + j) * n3 + node, g[j]);
}

}  // namespace stgv
