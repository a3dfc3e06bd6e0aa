// Learned correction of a coarse run: restriction of a fine state, training
// pairs, the network's forward / backward / Adam kernels on BF16 MFMA.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "learned.hpp"
#include "lbm_device.hpp"
#include "mlp_device.hpp"

namespace stgv {
namespace mlp {

__constant__ StepTables kStepTables = make_step_tables();

// ---------------------------------------------------------------------------
// packing: FP32 master parameters (W1 [64][47], b1, W2 [64][64], b2, W3 [41][64],
// b3) and the normalisation (x_mean[47], x_iscale[47], y_scale[41]) -> Packed.
// The time is a few dependent load latencies: 27 us when one 256-thread block walked the
// tables, 5 with one element of every table per thread, 2.9 as below.
// ---------------------------------------------------------------------------
// The tables are divided over the grid's rows (blockIdx.y), so that no thread waits for more
// than two or three loads in turn.
constexpr int kPackBlocks = N_HID * N_HID / 256;      // the largest table, one element per thread
constexpr int kPackRows = 4;

__global__ __launch_bounds__(256) void pack_kernel(const float* __restrict__ theta,
                                                   const float* __restrict__ norm,
                                                   Packed* __restrict__ P) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const float* W1 = theta;
  const float* b1 = W1 + N_HID * N_IN;
  const float* W2 = b1 + N_HID;
  const float* b2 = W2 + N_HID * N_HID;
  const float* W3 = b2 + N_HID;
  const float* b3 = W3 + N_OUT * N_HID;
  const float* y_scale = norm + 2 * N_IN;
  // The fused step's copies (..p) hold logical row k at physical row perm_row(k); their output
  // layer carries y_scale so that its result is the moment correction itself.
  if (blockIdx.y == 0) {
    if (t >= N_HID * K_IN) return;
    const int r = t / K_IN, c = t % K_IN, k = perm_row(r);
    const float w = W1[r * N_IN + min(c, N_IN - 1)], wp = W1[k * N_IN + min(c, N_IN - 1)];
    P->w1[t] = c < N_IN ? bf16_bits(w) : 0;
    P->w1p[t] = c < N_IN ? bf16_bits(wp) : 0;
    P->tab.feat[t] = kStepTables.feat[t];
    P->tab.minv[t] = kStepTables.minv[t];
  } else if (blockIdx.y == 1) {
    const int r = t / N_HID, c = t % N_HID, k = perm_row(r);
    const float w = W2[t], wt = W2[c * N_HID + r], wp = W2[k * N_HID + c];
    P->w2[t] = bf16_bits(w);
    P->w2t[t] = bf16_bits(wt);
    P->w2p[t] = bf16_bits(wp);
  } else if (blockIdx.y == 2) {
    const int r = t / N_HID, c = t % N_HID, k = perm_row(r);     // w3: [output r][hidden c]
    const int h = t / M_OUT, o = t % M_OUT;                      // w3t: [hidden h][output o]
    const int rr = min(r, N_OUT - 1), oo = min(o, N_OUT - 1), kk = min(k, N_OUT - 1);
    const float w = W3[rr * N_HID + c], wt = W3[oo * N_HID + h], wp = y_scale[kk] * W3[kk * N_HID + c];
    P->w3[t] = r < N_OUT ? bf16_bits(w) : 0;
    P->w3t[t] = o < N_OUT ? bf16_bits(wt) : 0;
    P->w3p[t] = k < N_OUT ? bf16_bits(wp) : 0;
  } else if (t < M_OUT) {
    const int k = perm_row(t), o = min(t, N_OUT - 1), ko = min(k, N_OUT - 1), in = min(t, N_IN - 1), ki = min(k, N_IN - 1);
    const float v1 = b1[t], v2 = b2[t], v3 = b3[o], ys = y_scale[o], xm = norm[in], xi = norm[N_IN + in];
    const float p1 = b1[k], p2 = b2[k], p3 = y_scale[ko] * b3[ko], pm = norm[ki], pi = norm[N_IN + ki];
    P->b1[t] = v1;
    P->b2[t] = v2;
    P->b3[t] = t < N_OUT ? v3 : 0.f;
    P->y_scale[t] = t < N_OUT ? ys : 0.f;
    if (t < K_IN) {
      P->x_mean[t] = t < N_IN ? xm : 0.f;
      P->x_iscale[t] = t < N_IN ? xi : 0.f;
    }
    P->b1p[t] = p1;
    P->b2p[t] = p2;
    P->b3p[t] = k < N_OUT ? p3 : 0.f;
    P->x_mean_p[t] = k < N_IN ? pm : 0.f;
    P->x_iscale_p[t] = k < N_IN ? pi : 0.f;
  }
}
static_assert(N_HID == 64 && M_OUT == 64 && N_HID * K_IN <= N_HID * N_HID && M_OUT * N_HID == N_HID * N_HID &&
              64 * K_IN == N_HID * K_IN, "one thread per element of each table");

// V floats read or written at once.
template <int V> struct FloatPiece { typedef float type __attribute__((ext_vector_type(V))); };
template <> struct FloatPiece<1> { typedef float type; };

// A operand of a 32-row tile of W [rows][KW]: all k-steps of the lane's row.
template <int KW>
struct WeightTile {
  bf16x8 v[KW / 16];
  __device__ __forceinline__ void load(const uint16_t* W, int mt, int col, int half) {
#pragma unroll
    for (int ks = 0; ks < KW / 16; ++ks) v[ks] = load8(W + (32 * mt + col) * KW + 16 * ks + 8 * half);
  }
};

// ---------------------------------------------------------------------------
// Batch inference: rows of raw features -> de-normalised moment corrections.
//
// A wavefront takes tiles of 32 rows.  A tile's 6 KB of features are contiguous: they come
// in by 16-byte pieces and go through the wavefront's LDS buffer to the lanes that hold each
// row's MFMA operand; the same buffer then carries the hidden activations from a layer's
// result layout to the next one's operand layout, and last the outputs, stored contiguously
// again.  The weights sit in LDS, once per block.  Bound by VALU issue, most of it the 128
// tanh per row: 262 144 rows 113 -> 31.5 us (one 64-row wavefront per block had read its rows
// one lane per row and run tanhf's two branches per value).
// ---------------------------------------------------------------------------
constexpr int kInferThreads = 256, kInferRows = 32;
constexpr int kInferBlocks = 3 * 256;                  // three resident blocks per CU
constexpr int kInferBuf = kInferRows * N_IN;          // floats per wavefront: 6016 B
static_assert(kInferRows * LDS_PITCH * 2 <= kInferBuf * 4 && kInferRows * N_OUT <= kInferBuf,
              "activations and outputs share the feature buffer");

// Orders the wavefront's own LDS writes before its later reads of other lanes' values.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// `count` (at most MAX) contiguous floats from src to dst, every load ahead of the first
// store, in pieces of V floats; V = 4 wants count = MAX and 16-byte alignment of both ends.
template <int V, int MAX>
__device__ __forceinline__ void wave_copy(float* dst, const float* src, int lane, int count) {
  using Piece = typename FloatPiece<V>::type;
  constexpr int iters = (MAX / V + 63) / 64;
  Piece p[iters];
#pragma unroll
  for (int j = 0; j < iters; ++j) p[j] = *reinterpret_cast<const Piece*>(src + min(V * (lane + 64 * j), count - V));
#pragma unroll
  for (int j = 0; j < iters; ++j) {
    const int e = V * (lane + 64 * j);
    if (e < count) *reinterpret_cast<Piece*>(dst + e) = p[j];
  }
}

template <bool VEC>
__global__ __launch_bounds__(kInferThreads) void forward_kernel(const Packed* __restrict__ P,
                                                                const float* __restrict__ x, int64_t rows,
                                                                float* __restrict__ y) {
  __shared__ __attribute__((aligned(16))) float buf_all[kInferThreads / 64][kInferBuf];
  __shared__ __attribute__((aligned(16))) uint16_t w1[N_HID * K_IN], w2[N_HID * N_HID], w3[M_OUT * N_HID];
  __shared__ float mean[K_IN], iscale[K_IN], b1[N_HID], b2[N_HID], b3[M_OUT], y_scale[M_OUT];
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int e = 8 * tid; e < N_HID * K_IN; e += 8 * kInferThreads) *reinterpret_cast<bf16x8*>(w1 + e) = load8(P->w1 + e);
  for (int e = 8 * tid; e < N_HID * N_HID; e += 8 * kInferThreads) {
    *reinterpret_cast<bf16x8*>(w2 + e) = load8(P->w2 + e);
    *reinterpret_cast<bf16x8*>(w3 + e) = load8(P->w3 + e);
  }
  if (tid < K_IN) { mean[tid] = P->x_mean[tid]; iscale[tid] = P->x_iscale[tid]; }
  if (tid < N_HID) { b1[tid] = P->b1[tid]; b2[tid] = P->b2[tid]; b3[tid] = P->b3[tid]; y_scale[tid] = P->y_scale[tid]; }
  __syncthreads();

  float* const buf = buf_all[wv];
  uint16_t* const act = reinterpret_cast<uint16_t*>(buf);
  const int64_t tiles = (rows + kInferRows - 1) / kInferRows, step = (int64_t)gridDim.x * (kInferThreads / 64);
  for (int64_t t = (int64_t)blockIdx.x * (kInferThreads / 64) + wv; t < tiles; t += step) {
    const int live = (int)(rows - t * kInferRows < kInferRows ? rows - t * kInferRows : kInferRows);
    const bool vec = VEC && live == kInferRows;       // a partial tile goes by single floats
    if (vec) wave_copy<4, kInferBuf>(buf, x + t * kInferBuf, lane, kInferBuf);
    else wave_copy<1, kInferBuf>(buf, x + t * kInferBuf, lane, live * N_IN);
    wave_lds_sync();
    bf16x8 op[4];
    {
      const int r = min(col, live - 1);
#pragma unroll
      for (int ks = 0; ks < K_IN / 16; ++ks) {
        uint4 q;
        uint32_t* w = reinterpret_cast<uint32_t*>(&q);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const int k = 16 * ks + 8 * half + 2 * p;
          const float v0 = (buf[r * N_IN + k] - mean[k]) * iscale[k];
          const float v1 = k + 1 < N_IN ? (buf[r * N_IN + min(k + 1, N_IN - 1)] - mean[k + 1]) * iscale[k + 1] : 0.f;
          w[p] = to_bf16_pair(v0, v1);
        }
        op[ks] = __builtin_bit_cast(bf16x8, q);
      }
    }
    wave_lds_sync();
    // one layer: both 32-row tiles from the operand registers, results handed to emit(mt, j, 4 values)
    auto layer = [&](const uint16_t* W, const float* bias, auto kw, auto emit) {
      constexpr int KW = decltype(kw)::value;
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = bias[32 * mt + d_row(r, lane)];
        WeightTile<KW> w;
        w.load(W, mt, col, half);
#pragma unroll
        for (int ks = 0; ks < KW / 16; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w.v[ks], op[ks], acc, 0, 0, 0);
        emit(mt, acc);
      }
    };
    auto to_act = [&](int mt, const f32x16& acc) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint2 q = {tanh_bf16_pair(acc[4 * j], acc[4 * j + 1]), tanh_bf16_pair(acc[4 * j + 2], acc[4 * j + 3])};
        *reinterpret_cast<uint2*>(act + col * LDS_PITCH + 32 * mt + 8 * j + 4 * half) = q;
      }
    };
    auto from_act = [&] {
      wave_lds_sync();
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) op[ks] = load8(act + col * LDS_PITCH + 16 * ks + 8 * half);
      wave_lds_sync();
    };
    layer(w1, b1, std::integral_constant<int, K_IN>{}, to_act);
    from_act();
    layer(w2, b2, std::integral_constant<int, N_HID>{}, to_act);
    from_act();
    layer(w3, b3, std::integral_constant<int, N_HID>{}, [&](int mt, const f32x16& acc) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 32 * mt + d_row(r, lane);
        if (row < N_OUT) buf[col * N_OUT + row] = acc[r] * y_scale[row];
      }
    });
    wave_lds_sync();
    float* dst = y + t * (kInferRows * N_OUT);
    if (vec) wave_copy<4, kInferRows * N_OUT>(dst, buf, lane, kInferRows * N_OUT);
    else wave_copy<1, kInferRows * N_OUT>(dst, buf, lane, live * N_OUT);
    wave_lds_sync();
  }
}

// ---------------------------------------------------------------------------
// Gradient of the mean squared error over a batch (rows idx[0..batch)): per-block partial
// gradients in the master-parameter order and a partial loss.
//
// A block is 64 samples on four wavefronts; each 64 x 64 product of a layer is four 32 x 32
// MFMA tiles, one per wavefront, with the operands in LDS: activations node-major (the next
// layer's B operand, 16-byte reads) and, for the sums over the samples, also row-major
// ([row][node], so that both operands of an outer product are 16-byte reads).  A wavefront
// keeps its tile's hidden activations in registers for tanh' = 1 - h^2, and loads all its
// weight operands before the first product.  The time is one block's chain (16 384 rows are
// one block per CU), not bandwidth: loads 4.2 us, the two tanh layers 2.0 us each, the output
// layer 1.3, back 0.9, outer products and stores 1.5-2.0.  52 -> 18 us at 16 384 rows (one
// wavefront per block had read its rows per lane and its outer-product operands one 2-byte
// value at a time).
// ---------------------------------------------------------------------------
constexpr int kGradRows = 64, kGradThreads = 256;

// acc + W tile x the 32 nodes at `nt` of a node-major buffer
template <int KW>
__device__ __forceinline__ f32x16 tile_product(const WeightTile<KW>& w, const uint16_t* act, int nt, int col,
                                               int half, f32x16 acc) {
#pragma unroll
  for (int ks = 0; ks < KW / 16; ++ks)
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w.v[ks], load8(act + (32 * nt + col) * LDS_PITCH + 16 * ks + 8 * half),
                                                  acc, 0, 0, 0);
  return acc;
}

// The tile's 16 results of a lane (rows 32 mt + d_row(r), node 32 nt + col) into the
// node-major buffer `act` and the row-major buffer `tr` (either may be null).
__device__ __forceinline__ void put_tile(const uint16_t (&v)[16], uint16_t* act, uint16_t* tr, int mt, int nt,
                                         int col, int half) {
  const int node = 32 * nt + col;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = 32 * mt + 8 * j + 4 * half;
    if (act) {
      const uint2 q = {(uint32_t)v[4 * j] | ((uint32_t)v[4 * j + 1] << 16),
                       (uint32_t)v[4 * j + 2] | ((uint32_t)v[4 * j + 3] << 16)};
      *reinterpret_cast<uint2*>(act + node * LDS_PITCH + row) = q;
    }
    if (tr) {
#pragma unroll
      for (int q = 0; q < 4; ++q) tr[(row + q) * LDS_PITCH + node] = v[4 * j + q];
    }
  }
}

// One 32 x 32 tile of sum_n A[i][n] B[j][n] over the block's samples (row-major buffers).
__device__ __forceinline__ f32x16 outer_tile(const uint16_t* A, const uint16_t* B, int mt, int nt, int col, int half) {
  f32x16 acc = {0};
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(load8(A + (32 * mt + col) * LDS_PITCH + 16 * ks + 8 * half),
                                                  load8(B + (32 * nt + col) * LDS_PITCH + 16 * ks + 8 * half), acc, 0, 0, 0);
  return acc;
}

// Sum over the block's samples of one row of a row-major buffer, in sample order.
__device__ __forceinline__ float row_sum(const uint16_t* row) {
  float s = 0.f;
#pragma unroll
  for (int n = 0; n < kGradRows; n += 8) {
    const bf16x8 v = load8(row + n);
#pragma unroll
    for (int q = 0; q < 8; ++q) s += (float)v[q];
  }
  return s;
}

__global__ __launch_bounds__(kGradThreads) void grad_kernel(const Packed* __restrict__ P,
                                                            const float* __restrict__ x,
                                                            const float* __restrict__ y,
                                                            const int64_t* __restrict__ idx, int64_t batch,
                                                            float* __restrict__ gpart,
                                                            double* __restrict__ lpart) {
  constexpr int BUF = 64 * LDS_PITCH;
  // node-major: X then h2 then delta 1; h1 then delta 0 (and last, row-major, delta 2)
  __shared__ __attribute__((aligned(16))) uint16_t A[BUF], B[BUF];
  // row-major: the input, the hidden activations and the back-propagated deltas
  __shared__ __attribute__((aligned(16))) uint16_t XT[BUF], H1T[BUF], H2T[BUF], D0T[BUF], D1T[BUF];
  uint16_t* const D2T = B;
  __shared__ float yn[kGradRows * N_OUT];       // normalised targets, then the residuals
  __shared__ float lsum[64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int half = lane >> 5, col = lane & 31;
  const int mt = wv >> 1, nt = wv & 1;          // this wavefront's tile of every product
  const int64_t s0 = (int64_t)blockIdx.x * kGradRows;
  const int live = (int)(batch - s0 < kGradRows ? batch - s0 : kGradRows);
  const float inv_count = 1.0f / (float)(batch * N_OUT);

  // A wavefront reads 16 rows, a lane one column of each: the row's address is scalar and the
  // column's normalisation constants are the lane's own.  Every load is unconditional (a
  // padded sample or column reads a valid neighbour and is discarded below): behind a branch
  // each one was waited for by itself (10.7 us for this phase; with per-lane row addresses 6.2).
  constexpr int NR = kGradRows / 4;
  const int r0 = NR * wv;
  const int kx = min(lane, N_IN - 1), ky = min(lane, N_OUT - 1);
  float xv[NR], yv[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    const int64_t row = idx[s0 + min(r0 + j, live - 1)];
    xv[j] = (x + row * N_IN)[kx];
    yv[j] = (y + row * N_OUT)[ky];
  }
  const float mean = P->x_mean[kx], iscale = P->x_iscale[kx], yscale = P->y_scale[ky];
  WeightTile<K_IN> w1;
  WeightTile<N_HID> w2, w3, w2t;
  WeightTile<M_OUT> w3t;
  w1.load(P->w1, mt, col, half);
  w2.load(P->w2, mt, col, half);
  w3.load(P->w3, mt, col, half);
  w3t.load(P->w3t, mt, col, half);
  w2t.load(P->w2t, mt, col, half);
  f32x16 b1, b2, b3;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 32 * mt + d_row(r, lane);
    b1[r] = P->b1[row];
    b2[r] = P->b2[row];
    b3[r] = P->b3[row];
  }
  if (lane < K_IN) {
#pragma unroll
    for (int j = 0; j < NR; j += 2) {
      uint32_t v[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float xr = r0 + j + q < live ? xv[j + q] : 0.f;
        v[q] = lane < N_IN ? to_bf16_bits((xr - mean) * iscale) : 0u;
        A[(r0 + j + q) * LDS_PITCH + lane] = (uint16_t)v[q];
      }
      *reinterpret_cast<uint32_t*>(XT + lane * LDS_PITCH + r0 + j) = v[0] | (v[1] << 16);
    }
  }
  if (lane < N_OUT) {
#pragma unroll
    for (int j = 0; j < NR; ++j) yn[(r0 + j) * N_OUT + lane] = r0 + j < live ? yv[j] / yscale : 0.f;
  }
  __syncthreads();

  // forward; the hidden tiles stay in registers as the BF16 values the next layer sees
  uint16_t h1[16], h2[16], d[16];
  {
    const f32x16 t = tile_product(w1, A, nt, col, half, b1);
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const uint32_t q = tanh_bf16_pair(t[r], t[r + 1]);
      h1[r] = (uint16_t)q;
      h1[r + 1] = (uint16_t)(q >> 16);
    }
    put_tile(h1, B, H1T, mt, nt, col, half);
  }
  __syncthreads();
  {
    const f32x16 t = tile_product(w2, B, nt, col, half, b2);
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const uint32_t q = tanh_bf16_pair(t[r], t[r + 1]);
      h2[r] = (uint16_t)q;
      h2[r + 1] = (uint16_t)(q >> 16);
    }
    put_tile(h2, A, H2T, mt, nt, col, half);
  }
  __syncthreads();
  // output layer and dL/do = 2 (o - y) / (batch * 41); padded samples contribute nothing
  {
    const f32x16 t = tile_product(w3, A, nt, col, half, b3);
    const int node = 32 * nt + col;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = 32 * mt + d_row(r, lane);
      const float res = t[r] - yn[node * N_OUT + min(row, N_OUT - 1)];
      d[r] = row < N_OUT && node < live ? to_bf16_bits(2.f * res * inv_count) : (uint16_t)0;
      if (row < N_OUT) yn[node * N_OUT + row] = res;
    }
    put_tile(d, B, D0T, mt, nt, col, half);
  }
  __syncthreads();
  // back through the hidden layers (transposed weights), tanh' = 1 - h^2
  {
    const f32x16 zero = {0};
    const f32x16 t = tile_product(w3t, B, nt, col, half, zero);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float h = bf16_float(h2[r]);
      d[r] = to_bf16_bits(t[r] * (1.f - h * h));
    }
    put_tile(d, A, D1T, mt, nt, col, half);
  }
  __syncthreads();
  {
    const f32x16 zero = {0};
    const f32x16 t = tile_product(w2t, A, nt, col, half, zero);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float h = bf16_float(h1[r]);
      d[r] = to_bf16_bits(t[r] * (1.f - h * h));
    }
    put_tile(d, nullptr, D2T, mt, nt, col, half);
  }
  __syncthreads();
  // weight gradients: sums over the block's samples of outer products
  float* g = gpart + (int64_t)blockIdx.x * N_PARAMS;
  float* gW1 = g;
  float* gb1 = gW1 + N_HID * N_IN;
  float* gW2 = gb1 + N_HID;
  float* gb2 = gW2 + N_HID * N_HID;
  float* gW3 = gb2 + N_HID;
  float* gb3 = gW3 + N_OUT * N_HID;
  const int j = 32 * nt + col;
  const f32x16 t1 = outer_tile(D2T, XT, mt, nt, col, half);
  const f32x16 t2 = outer_tile(D1T, H1T, mt, nt, col, half);
  const f32x16 t3 = outer_tile(D0T, H2T, mt, nt, col, half);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = 32 * mt + d_row(r, lane);
    if (j < N_IN) gW1[i * N_IN + j] = t1[r];
    gW2[i * N_HID + j] = t2[r];
    if (i < N_OUT) gW3[i * N_HID + j] = t3[r];
  }
  if (wv == 0) {
    // the partial loss: each lane its residuals in tile order, then the lanes in order
    float lacc = 0.f;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = 32 * a + d_row(r, lane), node = 32 * b + col;
          const float res = yn[node * N_OUT + min(row, N_OUT - 1)];
          lacc = row < N_OUT && node < live ? fma_c(res, res, lacc) : lacc;
        }
    lsum[lane] = lacc;
    wave_lds_sync();
    if (lane == 0) {
      double t = 0.0;
#pragma unroll
      for (int n = 0; n < 64; ++n) t += (double)lsum[n];
      lpart[blockIdx.x] = t;
    }
  } else if (wv == 1) {
    gb1[lane] = row_sum(D2T + lane * LDS_PITCH);
  } else if (wv == 2) {
    gb2[lane] = row_sum(D1T + lane * LDS_PITCH);
  } else {
    const float c = row_sum(D0T + lane * LDS_PITCH);
    if (lane < N_OUT) gb3[lane] = c;
  }
}

// Fixed-order FP64 sums of the per-block partials: the gradient and the batch loss.  One
// wavefront's lanes hold 64 neighbouring parameters (a partial row is read in 256-byte runs)
// and the block's 16 wavefronts take every 16th row, eight loads in flight each; their sums
// are added in wavefront order.  One more block sums the losses.  Bound by the latency of a
// few loads and the 10 MB of partials at 16 384 rows (from L2): one thread per parameter
// walking all 256 rows had 39 blocks in flight; 76 -> 4.1 us at 16 384 rows.
constexpr int kReduceSlices = 16;
constexpr int kReduceBlocks = (N_PARAMS + 63) / 64;

__global__ __launch_bounds__(64 * kReduceSlices) void grad_reduce_kernel(const float* __restrict__ gpart,
                                                                         const double* __restrict__ lpart,
                                                                         int64_t nblocks, int64_t batch,
                                                                         float* __restrict__ grad,
                                                                         double* __restrict__ loss) {
  __shared__ double part[kReduceSlices][64];
  const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6;
  double s = 0.0;
  if (blockIdx.x < kReduceBlocks) {
    const int p = blockIdx.x * 64 + lane;
    if (p < N_PARAMS) {
#pragma unroll 8
      for (int64_t b = slice; b < nblocks; b += kReduceSlices) s += (double)gpart[b * N_PARAMS + p];
    }
    part[slice][lane] = s;
    __syncthreads();
    if (slice != 0 || p >= N_PARAMS) return;
    for (int k = 1; k < kReduceSlices; ++k) s += part[k][lane];
    grad[p] = (float)s;
  } else {
#pragma unroll 4
    for (int64_t b = threadIdx.x; b < nblocks; b += 64 * kReduceSlices) s += lpart[b];
    s = wave_reduce<false>(s);
    if (lane == 63) part[slice][0] = s;
    __syncthreads();
    if (threadIdx.x != 0) return;
    s = part[0][0];
    for (int k = 1; k < kReduceSlices; ++k) s += part[k][0];
    *loss = s / ((double)batch * N_OUT);
  }
}

// Adam (Kingma & Ba 2015); c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t).
__global__ __launch_bounds__(256) void adam_kernel(float* __restrict__ theta, float* __restrict__ m,
                                                   float* __restrict__ v, const float* __restrict__ grad,
                                                   float lr, float beta1, float beta2, float omb1,
                                                   float omb2, float eps, float c1, float c2) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N_PARAMS) return;
  const float gr = grad[p];
  const float mm = beta1 * m[p] + omb1 * gr;
  const float vv = beta2 * v[p] + omb2 * gr * gr;
  m[p] = mm;
  v[p] = vv;
  theta[p] -= lr * (mm * c1) / (sqrtf(vv * c2) + eps);
}

// ---------------------------------------------------------------------------
// normalisation: column sums of the features and their squares and of the squared targets
// over all rows, FP64, in two stages.  The features are taken relative to the first row, so a
// constant column sums to exactly zero whatever the order of the sums (without, its variance was a
// rounding residue that came out positive for about half of all constants at 262 144 rows, and
// 1 / std of it some 1e8), and a mean far from zero costs no digits: a row is at most sqrt(rows)
// standard deviations from the mean, so the variance loses no more than the factor `rows` of FP64's
// 1e-16.  The subtraction costs 0.6 us of 65 at 1 048 576 rows.
//
// One pass over the rows, HBM-bound (369 MB at 1 048 576 rows).  V rows of C columns are a
// run of C pieces of V floats; C neighbouring threads take one piece each, so a thread's V
// columns are the same in every run it reads and its sums stay in registers.  (A pass per
// statistic, 135 in all, each with a strided 4-byte load per row, took 2.58 ms there.)
// ---------------------------------------------------------------------------
constexpr int NSTAT = 2 * N_IN + N_OUT;    // sum x, sum x^2, sum y^2
constexpr int kStatsThreads = 1024;

template <int V>
__device__ __forceinline__ float piece_at(const typename FloatPiece<V>::type& p, int j) {
  if constexpr (V == 1) return p;
  else return p[j];
}

// k with V k = 1 (mod C)
constexpr int inverse_mod(int V, int C) {
  for (int k = 1; k < C; ++k)
    if ((V * k) % C == 1) return k;
  return 1;
}

// What a column of the features is taken relative to: its first row, unless that is infinite or NaN.
__device__ __forceinline__ double shift_of(float first) { return isfinite(first) ? (double)first : 0.0; }

// The first row's values of the V columns that a thread sums in a [rows][C] table.
template <int C, int V>
__device__ __forceinline__ void first_row(const float* __restrict__ t, float (&first)[V]) {
#pragma unroll
  for (int j = 0; j < V; ++j) first[j] = t[(V * (int)(threadIdx.x % C) + j) % C];
}

// Column sums of a [rows][C] table: runs [u0, u1) of V rows by this block's threads, the
// per-thread sums left in LDS as [piece element][thread].  FIRST: sums of t - shift_of(first) and
// squares of that, else squares of t alone.
template <int C, int V, bool FIRST>
__device__ __forceinline__ void column_sums(const float* __restrict__ t, int64_t u0, int64_t u1, const float (&first)[V],
                                            double (*sum)[kStatsThreads], double (*sq)[kStatsThreads]) {
  using Piece = typename FloatPiece<V>::type;
  constexpr int G = kStatsThreads / C;
  const int g = threadIdx.x / C, i = threadIdx.x % C;
  double s[V], s2[V], shift[V];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    s[j] = 0.0;
    s2[j] = 0.0;
    shift[j] = FIRST ? shift_of(first[j]) : 0.0;
  }
  if (g < G) {
    const Piece* p = reinterpret_cast<const Piece*>(t);
#pragma unroll 4
    for (int64_t u = u0 + g; u < u1; u += G) {
      const Piece v = p[u * C + i];
#pragma unroll
      for (int j = 0; j < V; ++j) {
        const double d = FIRST ? (double)piece_at<V>(v, j) - shift[j] : (double)piece_at<V>(v, j);
        if (FIRST) s[j] += d;
        s2[j] = fma_c(d, d, s2[j]);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < V; ++j) {
    if (FIRST) sum[j][threadIdx.x] = s[j];
    sq[j][threadIdx.x] = s2[j];
  }
}

// Sum of column c over the block's threads, in a fixed order.
template <int C, int V>
__device__ __forceinline__ double column_total(const double (*part)[kStatsThreads], int c) {
  constexpr int G = kStatsThreads / C, inv = inverse_mod(V, C);
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < V; ++j) {
    const int i = ((c + C - j) * inv) % C;          // the thread whose element j is column c
#pragma unroll
    for (int g = 0; g < G; ++g) s += part[j][g * C + i];
  }
  return s;
}

template <int V>
__global__ __launch_bounds__(kStatsThreads) void stats_kernel(const float* __restrict__ x,
                                                              const float* __restrict__ y, int64_t rows,
                                                              double* __restrict__ part) {
  __shared__ double sx[V][kStatsThreads], sx2[V][kStatsThreads], sy2[V][kStatsThreads];
  const int64_t b = blockIdx.x, nb = gridDim.x, runs = rows / V;
  const int64_t u0 = runs * b / nb, u1 = runs * (b + 1) / nb;
  float first[V];       // on its way while the targets are summed
  first_row<N_IN, V>(x, first);
  column_sums<N_OUT, V, false>(y, u0, u1, first, nullptr, sy2);
  column_sums<N_IN, V, true>(x, u0, u1, first, sx, sx2);
  __syncthreads();
  // one wavefront per statistic; the last block also takes the rows past the last whole run
  const int c = threadIdx.x & 63, which = threadIdx.x >> 6;
  if (which > 2 || c >= (which < 2 ? N_IN : N_OUT)) return;
  double s = which == 0 ? column_total<N_IN, V>(sx, c)
                        : (which == 1 ? column_total<N_IN, V>(sx2, c) : column_total<N_OUT, V>(sy2, c));
  if (b == nb - 1)
    for (int64_t r = runs * V; r < rows; ++r) {
      const double d = which < 2 ? (double)x[r * N_IN + c] - shift_of(x[c]) : (double)y[r * N_OUT + c];
      s += which == 0 ? d : d * d;
    }
  part[(which * N_IN + c) * nb + b] = s;
}

// One wavefront per column: the blocks' partial sums (contiguous per statistic) to the norm.
__global__ __launch_bounds__(64) void norm_kernel(const float* __restrict__ x, const double* __restrict__ part,
                                                  int nblocks, int64_t rows, float* __restrict__ norm) {
  const int c = blockIdx.x, lane = threadIdx.x;
  const float first = x[c < N_IN ? c : 0];
  auto total = [&](int stat) {
    double s = 0.0;
#pragma unroll 4
    for (int b = lane; b < nblocks; b += 64) s += part[stat * nblocks + b];
    return wave_reduce<false>(s);      // in lane 63
  };
  if (c < N_IN) {
    const double s = total(c), s2 = total(N_IN + c);
    const double mean = s / rows;
    const double var = s2 / rows - mean * mean;
    if (lane == 63) {
      norm[c] = (float)(shift_of(first) + mean);
      norm[N_IN + c] = var > 1e-300 ? (float)(1.0 / sqrt(var)) : 0.f;
    }
  } else {
    const double ms = total(N_IN + c) / rows;       // statistic 2 N_IN + (c - N_IN)
    if (lane == 63) norm[N_IN + c] = ms > 1e-300 ? (float)sqrt(ms) : 1.f;
  }
}

// ---------------------------------------------------------------------------
// restriction of a fine D3Q27 x D3Q19 state to the coarse grid (ratio 4)
//
// The filter is separable.  A lane holds one fine x and sums its 5 x 5 rows of a coarse
// (Y, Z) over y and z (the 46 populations and their 46 non-equilibrium parts, in registers);
// the five x of a coarse node are then added through LDS.  Every row is read in whole lines
// and each fine node's equilibria are formed 25 / 16 times, against 125 / 64 strided reads
// and evaluations when a thread walked its coarse node's whole 5^3 stencil.
//
// A block is LANES lanes (256): with n <= LANES whole fine rows of LANES / n neighbouring Y (the
// x sums wrap around in LDS), else the row segment of (LANES - 1) / 4 coarse nodes and the halo
// of two fine nodes on its left and right.
//
// Up to 64^3 that is too few wavefronts for the card and the time is the chain of 25 rows: there a
// block has a wavefront for each of the five planes, added through LDS (64^3 -> 16^3 44.5 -> 21.0
// us, 32^3 38.9 -> 18.7).  Above, the split loses: with two segments a row 46.0 -> 59.6 us at 68^3,
// with 128 lanes, which spill, 48.7.
//
// 256^3 -> 64^3, FP32: 3480 us for the per-node stencil, 816 in this form with loads that
// bypass the caches, 725 with cached ones (of sixteen rows nine are read once, six twice and one four times), 712
// with a run of (Y, Z) per XCD, 659 with tiles of them and both sweeps opposed; 500 us is one
// read of the state.
// ---------------------------------------------------------------------------
constexpr int kRestrictThreads = 256, kRestrictChunk = 23;     // 92 sums go through LDS in four chunks

struct RestrictShape {
  int rows;     // coarse rows (Y) of a block
  int xseg;     // coarse nodes of a block's row segment
  int segs;     // segments of a row
};
template <int LANES>
__host__ __device__ inline RestrictShape restrict_shape(int nc) {
  const int n = 4 * nc;
  if (n <= LANES) return {LANES / n, nc, 1};
  constexpr int X = (LANES - 1) / 4;                             // X coarse nodes need 4 X + 1 fine ones
  return {1, X, (nc + X - 1) / X};
}

template <typename T, int MODE, int LANES, int PLANES>
__global__ __launch_bounds__(LANES * PLANES) void restrict_kernel(const T* __restrict__ fine, Geometry gf,
                                                                    PhysConsts cf, int nc, float sf, float sg,
                                                                    float* __restrict__ out) {
  constexpr int NV = 2 * (27 + 19);
  static_assert(NV % kRestrictChunk == 0, "chunks of equal size");
  static_assert((PLANES == 1 && LANES == kRestrictThreads) || PLANES == 5, "all five planes, or one each");
  __shared__ float xs[kRestrictChunk][LANES * PLANES];
  const int n = gf.n, t = (int)threadIdx.x % LANES, plane = (int)threadIdx.x / LANES;
  const RestrictShape sh = restrict_shape<LANES>(nc);
  const bool ring = sh.segs == 1;
  // consecutive workgroups go to the 8 XCDs in turn: renumbered so that each XCD has a run of
  // neighbouring (Y, Z), whose shared rows its L2 may still hold; in tiles of 8 x 8 of them
  // (about what an XCD has resident) where the box divides into such tiles
  int bx = blockIdx.x, by = blockIdx.y, Z = blockIdx.z;
  const int gx = gridDim.x, gy = gridDim.y, blocks = gx * gy * (int)gridDim.z;
  if ((blocks & 7) == 0) {
    int b = bx + gx * (by + gy * Z);
    b = (b & 7) * (blocks >> 3) + (b >> 3);
    bx = b % gx;
    b /= gx;
    if (((gy | nc) & 7) == 0) {
      const int tile = b >> 6, ty = gy >> 3;
      by = 8 * (tile % ty) + (b & 7);
      Z = 8 * (tile / ty) + ((b >> 3) & 7);
    } else {
      by = b % gy;
      Z = b / gy;
    }
  }
  const int Y0 = by * sh.rows, X0 = bx * sh.xseg;
  const int width = ring ? n : LANES;
  const int yy = t / width, l = t % width;
  const int Y = Y0 + yy;
  int x = ring ? l : 4 * X0 - 2 + l;
  x += x < 0 ? n : 0;
  x -= x >= n ? n : 0;
  auto wf = [](int d) { return (d == -2 || d == 2) ? 0.125f : 0.25f; };   // [1,2,2,2,1] / 8
  auto wrap = [n](int v) { return v < 0 ? v + n : (v >= n ? v - n : v); };
  float a[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) a[k] = 0.f;
  if (yy < sh.rows && Y < nc && (ring || x < n)) {
    // neighbouring Y, and neighbouring Z, sweep in opposite directions, so that the rows they
    // share are read by both at the same time
    const int dir = (Y & 1) ? -1 : 1, dirz = (Z & 1) ? -1 : 1;
#pragma unroll 1
    for (int dzi = PLANES > 1 ? plane - 2 : -2; dzi <= (PLANES > 1 ? plane - 2 : 2); ++dzi)
#pragma unroll 1
      for (int dyi = -2; dyi <= 2; ++dyi) {
        const int dy = dir * dyi, dz = dirz * dzi;
        const float w = wf(dy) * wf(dz);
        const NodeIndex ix = make_index(x, wrap(4 * Y + dy), wrap(4 * Z + dz), n);
        float f[27], g[19];
        gather<27, T, MODE, false, true>(f, fine, 0, ix, gf.stride);
        gather<19, T, MODE, false, true>(g, fine, 27, ix, gf.stride);
        NodeMacro<float> m;
        node_macro<27, 19, FORCE_GUO>(f, g, cf, m);
        m.vx = m.ux; m.vy = m.uy; m.vz = m.uz;           // equilibria at the physical velocity
        const Collision<27, 19, FORCE_GUO, float> col(cf, m);
#pragma unroll
        for (int i = 0; i < 27; ++i) { a[i] += w * f[i]; a[46 + i] += w * (f[i] - col.feq(i)); }
#pragma unroll
        for (int j = 0; j < 19; ++j) { a[27 + j] += w * g[j]; a[73 + j] += w * (g[j] - col.geq(j)); }
      }
  }
  // the five fine x of this thread's coarse node (threads q < rows * xseg)
  const int cy = t / sh.xseg, cx = t % sh.xseg;
  const bool coarse = plane == 0 && cy < sh.rows && Y0 + cy < nc && X0 + cx < nc;
  int at[5];
#pragma unroll
  for (int d = 0; d < 5; ++d) {
    const int p = ring ? wrap(4 * cx + d - 2) : 4 * cx + d;
    at[d] = coarse ? cy * width + p : 0;
  }
  float b[NV];
#pragma unroll
  for (int k0 = 0; k0 < NV; k0 += kRestrictChunk) {
    if (k0) __syncthreads();
#pragma unroll
    for (int k = 0; k < kRestrictChunk; ++k) xs[k][threadIdx.x] = a[k0 + k];
    __syncthreads();
    if constexpr (PLANES > 1) {
      for (int k = plane; k < kRestrictChunk; k += PLANES) {
        float z = xs[k][t];
#pragma unroll
        for (int p = 1; p < PLANES; ++p) z += xs[k][p * LANES + t];
        xs[k][t] = z;
      }
      __syncthreads();
    }
    if (coarse) {
#pragma unroll
      for (int k = 0; k < kRestrictChunk; ++k)
        b[k0 + k] = 0.125f * (xs[k][at[0]] + xs[k][at[4]]) + 0.25f * (xs[k][at[1]] + xs[k][at[2]] + xs[k][at[3]]);
    }
  }
  if (!coarse) return;
  const int64_t nc3 = (int64_t)nc * nc * nc, J = X0 + cx + (int64_t)nc * (Y0 + cy + (int64_t)nc * Z);
  const float *fb = b, *gb = b + 27, *fn = b + 46, *gn = b + 73;
  // non-conserved moments of the filtered non-equilibrium part, rescaled by (s - 1)
  float mf[27], mg[19];
#pragma unroll
  for (int k = 0; k < 27; ++k) mf[k] = k < NCF ? 0.f : (sf - 1.f) * moment<27>(k, fn);
#pragma unroll
  for (int k = 0; k < 19; ++k) mg[k] = k < NCG ? 0.f : (sg - 1.f) * moment<19>(k, gn);
#pragma unroll
  for (int i = 0; i < 27; ++i) {
    float v = fb[i];
#pragma unroll
    for (int k = NCF; k < 27; ++k)
      if (MINV_F.v[i][k] != 0.f) v += MINV_F.v[i][k] * mf[k];
    out[i * nc3 + J] = v;
  }
#pragma unroll
  for (int j = 0; j < 19; ++j) {
    float v = gb[j];
#pragma unroll
    for (int k = NCG; k < 19; ++k)
      if (MINV_G.v[j][k] != 0.f) v += MINV_G.v[j][k] * mg[k];
    out[(27 + j) * nc3 + J] = v;
  }
}

// ---------------------------------------------------------------------------
// training pairs on the coarse grid: features of state a; targets from the
// residual b - c (b: restricted fine state one coarse step later, c: the
// coarse step of a), returned to the source node and projected on the
// non-conserved moments.  a, b, c: natural-order FP32 deviations.
// ---------------------------------------------------------------------------
template <int FORCE>
__global__ __launch_bounds__(256) void pairs_kernel(const float* __restrict__ a,
                                                    const float* __restrict__ b,
                                                    const float* __restrict__ c, int nc,
                                                    PhysConsts pc, float* __restrict__ xo,
                                                    float* __restrict__ yo) {
  using SF = Stencil<27>;
  using SG = Stencil<19>;
  const int64_t nc3 = (int64_t)nc * nc * nc;
  const int64_t J = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (J >= nc3) return;
  const int X = (int)(J % nc), Y = (int)((J / nc) % nc), Z = (int)(J / ((int64_t)nc * nc));
  const NodeIndex ix = make_index(X, Y, Z, nc);
  float f[27], g[19];
#pragma unroll
  for (int i = 0; i < 27; ++i) f[i] = a[i * nc3 + J];
#pragma unroll
  for (int j = 0; j < 19; ++j) g[j] = a[(27 + j) * nc3 + J];
  NodeMacro<float> m;
  node_macro<27, 19, FORCE>(f, g, pc, m);
  const Collision<27, 19, FORCE, float> col(pc, m);
  col.relaxation_increments(f, g);       // f <- f^eq - f, g <- g^eq - g
  float* xr = xo + J * N_IN;
  node_features<FORCE>(f, g, m, (float)pc.tau_f, [&](int k, float v) { xr[k] = v; });
  float rf[27], rg[19];
#pragma unroll
  for (int i = 0; i < 27; ++i) {
    const uint32_t o = ix.at(SF::ex[i], SF::ey[i], SF::ez[i]);
    rf[i] = b[i * nc3 + o] - c[i * nc3 + o];
  }
#pragma unroll
  for (int j = 0; j < 19; ++j) {
    const uint32_t o = ix.at(SG::ex[j], SG::ey[j], SG::ez[j]);
    rg[j] = b[(27 + j) * nc3 + o] - c[(27 + j) * nc3 + o];
  }
  float* yr = yo + J * N_OUT;
#pragma unroll
  for (int k = NCF; k < 27; ++k) yr[k - NCF] = moment<27>(k, rf);
#pragma unroll
  for (int k = NCG; k < 19; ++k) yr[27 - NCF + k - NCG] = moment<19>(k, rg);
}

}  // namespace mlp

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
hipError_t mlp_launch_pack(const float* theta, const float* norm, void* packed, hipStream_t st) {
  hipLaunchKernelGGL(mlp::pack_kernel, dim3(mlp::kPackBlocks, mlp::kPackRows), dim3(256), 0, st, theta, norm, (mlp::Packed*)packed);
  return hipGetLastError();
}

hipError_t mlp_launch_forward(const void* packed, const float* x, int64_t rows, float* y, hipStream_t st) {
  const int64_t tiles = (rows + mlp::kInferRows - 1) / mlp::kInferRows, waves = mlp::kInferThreads / 64;
  const int64_t blocks = std::min<int64_t>((tiles + waves - 1) / waves, mlp::kInferBlocks);
  if (((uintptr_t)x | (uintptr_t)y) % 16 == 0)        // a whole tile of either starts on 16 bytes
    hipLaunchKernelGGL(mlp::forward_kernel<true>, dim3((unsigned)blocks), dim3(mlp::kInferThreads), 0, st,
                       (const mlp::Packed*)packed, x, rows, y);
  else
    hipLaunchKernelGGL(mlp::forward_kernel<false>, dim3((unsigned)blocks), dim3(mlp::kInferThreads), 0, st,
                       (const mlp::Packed*)packed, x, rows, y);
  return hipGetLastError();
}

hipError_t mlp_launch_grad(const void* packed, const float* x, const float* y, const int64_t* idx,
                           int64_t batch, float* gpart, double* lpart, float* grad, double* loss,
                           hipStream_t st) {
  const int64_t blocks = (batch + 63) / 64;
  hipLaunchKernelGGL(mlp::grad_kernel, dim3((unsigned)blocks), dim3(mlp::kGradThreads), 0, st,
                     (const mlp::Packed*)packed, x, y, idx, batch, gpart, lpart);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(mlp::grad_reduce_kernel, dim3(mlp::kReduceBlocks + (loss ? 1 : 0)),
                     dim3(64 * mlp::kReduceSlices), 0, st, gpart, lpart, blocks, batch, grad, loss);
  return hipGetLastError();
}

hipError_t mlp_launch_adam(float* theta, float* m, float* v, const float* grad, float lr, float b1,
                           float b2, float omb1, float omb2, float eps, float c1, float c2, hipStream_t st) {
  hipLaunchKernelGGL(mlp::adam_kernel, dim3((mlp::N_PARAMS + 255) / 256), dim3(256), 0, st, theta,
                     m, v, grad, lr, b1, b2, omb1, omb2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t mlp_launch_norm(const float* x, const float* y, int64_t rows, double* part, int nblocks,
                           float* norm, hipStream_t st) {
  // 16-byte pieces where both tables are so aligned (any row count; a view that starts at an
  // odd row is not), else single floats
  if (((uintptr_t)x | (uintptr_t)y) % 16 == 0)
    hipLaunchKernelGGL(mlp::stats_kernel<4>, dim3(nblocks), dim3(mlp::kStatsThreads), 0, st, x, y, rows, part);
  else
    hipLaunchKernelGGL(mlp::stats_kernel<1>, dim3(nblocks), dim3(mlp::kStatsThreads), 0, st, x, y, rows, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(mlp::norm_kernel, dim3(mlp::N_IN + mlp::N_OUT), dim3(64), 0, st, x, part, nblocks, rows, norm);
  return hipGetLastError();
}

template <typename T, int LANES, int PLANES>
static void restrict_launch(const T* fine, int mode, Geometry gf, PhysConsts cf, int nc, float sf, float sg,
                            float* out, hipStream_t st) {
  const mlp::RestrictShape sh = mlp::restrict_shape<LANES>(nc);
  const dim3 grid((unsigned)sh.segs, (unsigned)((nc + sh.rows - 1) / sh.rows), (unsigned)nc), block(LANES * PLANES);
  if (mode == MODE_ODD)
    hipLaunchKernelGGL((mlp::restrict_kernel<T, MODE_ODD, LANES, PLANES>), grid, block, 0, st, fine, gf, cf, nc, sf, sg, out);
  else
    hipLaunchKernelGGL((mlp::restrict_kernel<T, MODE_EVEN, LANES, PLANES>), grid, block, 0, st, fine, gf, cf, nc, sf, sg, out);
}

template <typename T>
static hipError_t restrict_t(const void* fine, int mode, Geometry gf, PhysConsts cf, int nc, float sf,
                             float sg, float* out, hipStream_t st) {
  if (gf.n <= 64)
    restrict_launch<T, 64, 5>((const T*)fine, mode, gf, cf, nc, sf, sg, out, st);
  else
    restrict_launch<T, mlp::kRestrictThreads, 1>((const T*)fine, mode, gf, cf, nc, sf, sg, out, st);
  return hipGetLastError();
}

hipError_t mlp_launch_restrict(int storage, const void* fine, int mode, Geometry gf, PhysConsts cf,
                               int nc, float sf, float sg, float* out, hipStream_t st) {
  switch (storage) {
    case 0: return restrict_t<float>(fine, mode, gf, cf, nc, sf, sg, out, st);
    case 1: return restrict_t<_Float16>(fine, mode, gf, cf, nc, sf, sg, out, st);
    default: return restrict_t<bf16_t>(fine, mode, gf, cf, nc, sf, sg, out, st);
  }
}

hipError_t mlp_launch_pairs(int forcing, const float* a, const float* b, const float* c, int nc,
                            PhysConsts pc, float* x, float* y, hipStream_t st) {
  const int64_t nc3 = (int64_t)nc * nc * nc;
  const dim3 grid((unsigned)((nc3 + 255) / 256));
  if (forcing == FORCE_GUO)
    hipLaunchKernelGGL((mlp::pairs_kernel<FORCE_GUO>), grid, dim3(256), 0, st, a, b, c, nc, pc, x, y);
  else
    hipLaunchKernelGGL((mlp::pairs_kernel<FORCE_SHIFT>), grid, dim3(256), 0, st, a, b, c, nc, pc, x, y);
  return hipGetLastError();
}

}  // namespace stgv
