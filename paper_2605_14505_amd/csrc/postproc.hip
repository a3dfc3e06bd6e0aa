// Kinetic-energy spectrum: E(k) = sum over the wavevectors with round(|k|) = k of
// |u_hat|^2 / 2, u_hat = FFT(u / u0) / n^3 (Section 3.5, spectra at peak activity).
// The transforms are rocFFT's; the binning is a grid-stride pass over the
// half-spectrum of each component into per-block LDS histograms, reduced over
// the blocks in a fixed order.
#include "postproc.hpp"

#include "lbm_device.hpp"

#include <rocfft/rocfft.h>

#include <cmath>
#include <cstdio>
#include <map>
#include <mutex>

namespace stgv {
namespace {

constexpr int kShellBlocks = 1024;           // at most, a component
constexpr int kShellThreads = 256;
// Components that one transform and one binning launch take: all three up to a size, beyond it one.
// Below, the time is launches (16^3 33.9 -> 16.1 us, 64^3 53.4 -> 30.1) and the tail of each (128^3
// 191 -> 140, 160^3 329 -> 260), and the results are the same; towards the line the gain fades as
// three half spectra and their work space leave the caches.  The line is a table of measurements, not
// a count of bytes: rocFFT takes rows of whole 64-byte pieces without work space, other even boxes
// with one half spectrum of it a component, and odd ones, whose rows it transforms at full length,
// with four.  One by one / at once, us: odd 181^3 1230 / 1135, 191^3 1356 / 1299, 199^3 1551 / 1537
// and, on another day, 1458 / 1467, 225^3 1313 / 1430; even 230^3 1405 / 1350, 238^3 1087 / 1093, 246^3
// 1615 / 1618, 250^3 1156 / 1204; multiples of 16 240^3 978 / 934, 256^3 1119 / 1083, 272^3 1472 / 1529.
inline int components_at_once(int n) {
  const int up_to = n % 16 == 0 ? 256 : (n % 2 == 0 ? 240 : 181);
  return n <= up_to ? 3 : 1;
}
inline int64_t half_spectrum(int n) { return (int64_t)(n / 2 + 1) * n * n; }
inline int shell_blocks(int n) {
  const int64_t b = (half_spectrum(n) + kShellThreads - 1) / kShellThreads;
  return b < kShellBlocks ? (int)b : kShellBlocks;
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// One component's half spectrum c[(n/2 + 1) n n] (kx fastest): the Hermitian twins of
// 0 < kx < n/2 are counted twice.  scale = 1 / (2 n^6 u0^2).  The grid-stride walk carries
// (kx, ky, kz) along by adding the stride's own digits, so no element needs a division, and
// the shell is taken in FP32: |k|^2 is an integer below 2^20, and the values next to a shell's
// edge, (s - 1/2)^2 -+ 1/4 and 3/4, are 1e-4 or more away from it in |k|, twice the rounding.
// Bound by reading c: 256^3 30 -> 20 us a component.  blockIdx.y is the component of a batch; partial
// is [shell][block], so that the reduction reads a shell's partials contiguously.
struct Digits {
  int kx, ky, kz;
};

__global__ __launch_bounds__(kShellThreads) void shell_kernel(const float2* __restrict__ c, int n, int nshell,
                                                              double scale, double* __restrict__ partial,
                                                              int parts, int part0) {
  extern __shared__ double hist[];
  for (int s = threadIdx.x; s < nshell; s += blockDim.x) hist[s] = 0.0;
  __syncthreads();
  const int nh = n / 2 + 1, total = nh * n * n, step = gridDim.x * blockDim.x;
  c += (int64_t)blockIdx.y * total;
  part0 += blockIdx.y * gridDim.x;
  auto digits = [=](int i) { return Digits{i % nh, (i / nh) % n, i / nh / n}; };
  const Digits d = digits(step);
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  Digits k = digits(i);
  for (; i < total; i += step) {
    const float2 v = c[i];
    const int ky = k.ky <= n / 2 ? k.ky : k.ky - n, kz = k.kz <= n / 2 ? k.kz : k.kz - n;
    const int s = (int)(sqrtf((float)(k.kx * k.kx + ky * ky + kz * kz)) + 0.5f);
    const double w = (k.kx == 0 || 2 * k.kx == n) ? scale : 2.0 * scale;
    atomicAdd(&hist[s], w * ((double)v.x * v.x + (double)v.y * v.y));
    k.kx += d.kx;
    k.ky += d.ky;
    k.kz += d.kz;
    if (k.kx >= nh) { k.kx -= nh; ++k.ky; }
    if (k.ky >= n) { k.ky -= n; ++k.kz; }
  }
  __syncthreads();
  for (int s = threadIdx.x; s < nshell; s += blockDim.x) partial[(int64_t)s * parts + part0 + blockIdx.x] = hist[s];
}

// One block per shell; fixed order.  256^3: 720 -> 4 us against one thread per shell walking a
// strided column of 3072 partials.
__global__ __launch_bounds__(256) void shell_reduce_kernel(const double* __restrict__ partial, int nparts,
                                                           double* __restrict__ out) {
  const double* p = partial + (int64_t)blockIdx.x * nparts;
  double acc = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < nparts; b += 256) acc += p[b];
  block_reduce_store<1, 0u>(&acc, out + blockIdx.x);
}

struct Plan {
  rocfft_plan plan = nullptr;
  size_t work = 0;
};
std::mutex g_mutex;
std::map<std::pair<int, int>, Plan> g_plans;      // (n, components at once)
bool g_setup = false;

const Plan* get_plan(int n, int at_once, char* err) {
  std::lock_guard<std::mutex> lock(g_mutex);
  if (!g_setup) {
    if (rocfft_setup() != rocfft_status_success) {
      snprintf(err, 512, "rocfft_setup failed");
      return nullptr;
    }
    g_setup = true;
  }
  auto it = g_plans.find({n, at_once});
  if (it != g_plans.end()) return &it->second;
  Plan p;
  const size_t lengths[3] = {(size_t)n, (size_t)n, (size_t)n};
  if (rocfft_plan_create(&p.plan, rocfft_placement_notinplace, rocfft_transform_type_real_forward,
                         rocfft_precision_single, 3, lengths, at_once, nullptr) != rocfft_status_success) {
    snprintf(err, 512, "rocfft_plan_create failed for %d^3", n);
    return nullptr;
  }
  if (rocfft_plan_get_work_buffer_size(p.plan, &p.work) != rocfft_status_success) {
    snprintf(err, 512, "rocfft_plan_get_work_buffer_size failed");
    rocfft_plan_destroy(p.plan);
    return nullptr;
  }
  return &(g_plans[{n, at_once}] = p);
}

struct Layout {
  size_t complex_off, partial_off, fft_off, total;
};

Layout layout(int n, int at_once, size_t fft_work) {
  Layout l;
  const size_t cbytes = (size_t)half_spectrum(n) * at_once * sizeof(float2);
  l.complex_off = 0;
  l.partial_off = align256(cbytes);
  l.fft_off = l.partial_off + align256((size_t)3 * shell_blocks(n) * spectrum_shells(n) * sizeof(double));
  l.total = l.fft_off + align256(fft_work);
  return l;
}

}  // namespace

int spectrum_shells(int n) { return (int)std::floor(std::sqrt(3.0) * n / 2.0 + 0.5) + 1; }

size_t spectrum_extra_bytes(int n, char* err) {
  const int at_once = components_at_once(n);
  char unused[512];
  if (at_once > 1) get_plan(n, 1, unused);      // a smaller buffer's (spectrum_launch): 0.01 s beside the other's 0.6
  const Plan* p = get_plan(n, at_once, err);
  return p ? layout(n, at_once, p->work).total : 0;
}

hipError_t spectrum_launch(const float* u, int n, double u0, void* work,
                           size_t work_bytes, double* out, hipStream_t st, char* err) {
  int at_once = components_at_once(n);
  const Plan* p = get_plan(n, at_once, err);
  if (!p) return hipErrorUnknown;
  Layout l = layout(n, at_once, p->work);
  if (at_once > 1 && work_bytes < l.total) {      // room for one component's half spectrum may do
    at_once = 1;
    p = get_plan(n, at_once, err);
    if (!p) return hipErrorUnknown;
    l = layout(n, at_once, p->work);
  }
  if (work_bytes < l.total) {
    snprintf(err, 512, "spectrum work buffer has %zu bytes, needs %zu", work_bytes, l.total);
    return hipErrorInvalidValue;
  }
  char* base = static_cast<char*>(work);
  float2* cbuf = reinterpret_cast<float2*>(base + l.complex_off);
  double* partial = reinterpret_cast<double*>(base + l.partial_off);
  rocfft_execution_info info = nullptr;
  if (rocfft_execution_info_create(&info) != rocfft_status_success) {
    snprintf(err, 512, "rocfft_execution_info_create failed");
    return hipErrorUnknown;
  }
  hipError_t e = hipSuccess;
  bool ok = rocfft_execution_info_set_stream(info, st) == rocfft_status_success;
  if (ok && p->work > 0)
    ok = rocfft_execution_info_set_work_buffer(info, base + l.fft_off, p->work) == rocfft_status_success;
  const int nshell = spectrum_shells(n);
  const double scale = 1.0 / (2.0 * std::pow((double)n, 6.0) * u0 * u0);
  const int blocks = shell_blocks(n);
  for (int c = 0; ok && c < 3; c += at_once) {
    void* in[1] = {const_cast<float*>(u + c * (int64_t)n * n * n)};
    void* outp[1] = {cbuf};
    ok = rocfft_execute(p->plan, in, outp, info) == rocfft_status_success;
    if (!ok) break;
    hipLaunchKernelGGL(shell_kernel, dim3(blocks, at_once), dim3(kShellThreads), nshell * sizeof(double), st, cbuf, n,
                       nshell, scale, partial, 3 * blocks, c * blocks);
    e = hipGetLastError();
    if (e != hipSuccess) break;
  }
  rocfft_execution_info_destroy(info);
  if (!ok) {
    snprintf(err, 512, "rocFFT execution failed for %d^3", n);
    return hipErrorUnknown;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(shell_reduce_kernel, dim3(nshell), dim3(256), 0, st, partial, 3 * blocks, out);
  return hipGetLastError();
}

}  // namespace stgv
