// kernels_metrics.hip -- per-round metrics, off the hot path.
//
// Appendix A states the goal as minimising the sum of the private objectives
// at a common point and bounds the distance to consensus by sigma_2(P)^t.
// These kernels report, in fp64 with fixed summation orders:
//   mean_i f_i(w_i), F(w_bar) = (1/n) sum_i f_i(w_bar), ||W - 1 w_bar^T||_F and
//   the mean of all model entries (which a doubly-stochastic reduce keeps).
#include <cmath>
#include <mutex>

#include "asap_launch.h"

namespace asap {
namespace {

// partials: [kMetricColBlocks][4] of the column pass, then [n][chunks][2] of
// the loss pass
constexpr int kColBlocksMax = kMetricColBlocks;
constexpr int64_t kLossBase = 4 * int64_t(kColBlocksMax);

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// fixed-order tree over the 256 threads of a block
__device__ double block_sum_d(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

__device__ __forceinline__ double scale_of(const MetricArgs& a, int i) { return a.scale ? double(a.scale[i]) : 1.0; }

// Column pass: w_bar, and per block the consensus, mean, ||w_bar||^2 and
// ||W||^2 partials.  A block takes 64 columns at a time, a float4 for each of
// 16 lanes, its rows dealt to 16 groups; with R rows to a thread (n <= 16 R)
// they stay in registers between the mean and the distances, so the models are
// read once (64 x 2^20: 124 -> 60 us, and the loss pass no longer reads them
// for their norms); R = 0: any n, read twice.
template <int R>
__global__ __launch_bounds__(256) void cols_kernel(MetricArgs a) {
  __shared__ double sh[256];
  __shared__ double sums[16][64];
  __shared__ double mean[64];
  const int cl = threadIdx.x & 15, rg = threadIdx.x >> 4;
  double cons = 0.0, msum = 0.0, wb2 = 0.0, w2 = 0.0;
  auto entry = [&](int i, int64_t c) { return *reinterpret_cast<const float4*>(a.W + int64_t(i) * a.ld + c); };
  for (int64_t c0 = int64_t(blockIdx.x) * 64; c0 < a.dim; c0 += int64_t(gridDim.x) * 64) {
    const int64_t c = c0 + 4 * cl;
    const bool in = c < a.dim;  // rows are padded to whole float4s; entries past dim are not used
    double m[4] = {0.0, 0.0, 0.0, 0.0};
    float4 x[R ? R : 1];
    if constexpr (R > 0) {
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int i = rg + 16 * k;
        x[k] = in && i < a.n ? entry(i, c) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int i = rg + 16 * k;
        const double si = i < a.n ? scale_of(a, i) : 0.0;
        m[0] += si * double(x[k].x);
        m[1] += si * double(x[k].y);
        m[2] += si * double(x[k].z);
        m[3] += si * double(x[k].w);
      }
    } else if (in) {
      for (int i = rg; i < a.n; i += 16) {
        const float4 v = entry(i, c);
        const double si = scale_of(a, i);
        m[0] += si * double(v.x);
        m[1] += si * double(v.y);
        m[2] += si * double(v.z);
        m[3] += si * double(v.w);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) sums[rg][4 * cl + e] = m[e];
    __syncthreads();
    if (threadIdx.x < 64 && c0 + threadIdx.x < a.dim) {
      double t = 0.0;
      for (int g = 0; g < 16; ++g) t += sums[g][threadIdx.x];
      t /= double(a.n);
      mean[threadIdx.x] = t;
      a.wbar[c0 + threadIdx.x] = t;
      msum += t;
      wb2 += t * t;
    }
    __syncthreads();
    auto distance = [&](const float4& v, double si) {
      const double w[4] = {si * double(v.x), si * double(v.y), si * double(v.z), si * double(v.w)};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (c + e >= a.dim) continue;
        const double d = w[e] - mean[4 * cl + e];
        cons += d * d;
        w2 += w[e] * w[e];
      }
    };
    if (in) {
      if constexpr (R > 0) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
          // opaque: widened again here, not kept in both widths from the mean on
          asm volatile("" : "+v"(x[k].x), "+v"(x[k].y), "+v"(x[k].z), "+v"(x[k].w));
          if (rg + 16 * k < a.n) distance(x[k], scale_of(a, rg + 16 * k));
        }
      } else {
        for (int i = rg; i < a.n; i += 16) distance(entry(i, c), scale_of(a, i));
      }
    }
  }
  cons = block_sum_d(cons, sh);
  msum = block_sum_d(msum, sh);
  wb2 = block_sum_d(wb2, sh);
  w2 = block_sum_d(w2, sh);
  if (threadIdx.x == 0) {
    double* q = a.part + 4 * blockIdx.x;
    q[0] = cons;
    q[1] = msum;
    q[2] = wb2;
    q[3] = w2;
  }
}

// Out of line: inlined, its exp and log1p took the CSR pass from 54 to 82
// registers (5 instead of 8 waves a SIMD).
__device__ __attribute__((noinline)) double loss_of(double ym, int loss) {
  if (loss == 1) return fmax(0.0, 1.0 - ym);
  return fmax(-ym, 0.0) + log1p(exp(-fabs(ym)));  // softplus(-ym)
}

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false),
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false));
}
// sum over the 16 lanes of a DPP row, the same bits in all of them
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_d<0xB1>(v);
  v += dpp_d<0x4E>(v);
  v += dpp_d<0x141>(v);
  v += dpp_d<0x140>(v);
  return v;
}

// Losses of the CSR samples at their workers' own models and at w_bar.  16
// lanes a row (one wave a row left a third of the lanes of rows of 80 nonzeros
// idle), four nonzeros of a lane in flight; lanes 0 and 1 of a row take the two
// losses.  Bound by the random reads of the two models, so the blocks of an XCD
// (blockIdx mod 8) walk one eighth of the samples together, in order: a model
// is read by one XCD, one worker at a time, and stays in its L2; nonzeros,
// read once, are loaded non-temporally.  64 x 2^20, 4096 samples each of 83
// nonzeros, a call: 488 us with samples of a block contiguous, 419 in this
// order, 408 non-temporally, 389 with the loss out of line (above); a pass over
// the samples for each of the two models: 452.
__global__ __launch_bounds__(256, 8) void loss_csr_kernel(MetricArgs a) {
  __shared__ double sh[256];
  const int sub = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const uint32_t parts = gridDim.x % 8u == 0u ? 8u : 1u;
  const int64_t rows = int64_t(a.n) * a.S, part = blockIdx.x % parts, stride = 16 * int64_t(gridDim.x / parts);
  const int64_t g1 = rows * (part + 1) / parts;
  double lsum = 0.0;
  for (int64_t g = rows * part / parts + 16 * int64_t(blockIdx.x / parts) + grp; g < g1; g += stride) {
    const int i = int(g / a.S);
    const float* w = a.W + int64_t(i) * a.ld;
    const int64_t p0 = a.row_ptr[g];
    const int len = int(a.row_ptr[g + 1] - p0);
    const int32_t* cp = a.col + p0;
    const float* vp = a.val + p0;
    double mo = 0.0, mb = 0.0;
    for (int e = sub; e < len; e += 64) {
      int c[4];
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool in = e + 16 * u < len;
        c[u] = in ? __builtin_nontemporal_load(cp + e + 16 * u) : 0;
        v[u] = in ? __builtin_nontemporal_load(vp + e + 16 * u) : 0.f;
      }
      float wo[4];
      double wb[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool in = e + 16 * u < len;
        wo[u] = in ? w[c[u]] : 0.f;
        wb[u] = in ? a.wbar[c[u]] : 0.0;
      }
      const double si = scale_of(a, i);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        mo = fma(double(v[u]), si * double(wo[u]), mo);
        mb = fma(double(v[u]), wb[u], mb);
      }
    }
    mo = row16_sum(mo);
    mb = row16_sum(mb);
    if (sub < 2) lsum += loss_of(double(a.y[g]) * (sub ? mb : mo), a.loss);
  }
  const double lown = block_sum_d(sub == 0 ? lsum : 0.0, sh), lbar = block_sum_d(sub == 1 ? lsum : 0.0, sh);
  if (threadIdx.x == 0) {
    double* q = a.part + kLossBase + 2 * int64_t(blockIdx.x);
    q[0] = lown;
    q[1] = lbar;
  }
}

// The same for dense shards; block (i, ch) takes worker i's samples of chunk ch
// (a contiguous range).  A wave takes four rows at a time, so that the two
// models (4 + 8 bytes a column) are read once for four rows of 4 bytes, and
// the next 256 columns load while these are summed.  16 x 6275, 2504 samples
// each, a call: 374 us with w_bar read a column at a time, 232 by whole groups
// of columns, 218 with the next group loading.
__global__ __launch_bounds__(256, 4) void loss_dense_kernel(MetricArgs a, int nch) {
  __shared__ double sh[256];
  const int i = blockIdx.x / nch, ch = blockIdx.x % nch, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r0 = a.S * ch / nch, r1 = a.S * (ch + 1) / nch;
  const float* w = a.W + int64_t(i) * a.ld;
  const double si = scale_of(a, i);
  struct Cols {
    float4 v[4], w;
    double2 b0, b1;
  };
  double lsum = 0.0;
  for (int64_t r = r0 + 4 * wave; r < r1; r += 16) {
    const float* x = a.X + (int64_t(i) * a.S + r) * a.ldx;
    double mo[4] = {0.0, 0.0, 0.0, 0.0}, mb[4] = {0.0, 0.0, 0.0, 0.0};
    // columns c .. c + 3 of the four rows (past the chunk the first row again);
    // lanes past the last column read column 0 and are masked below.  Rows and
    // w_bar are padded to whole groups of four.
    auto load = [&](Cols& q, int64_t c) {
      if (c >= a.dim) c = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) q.v[k] = *reinterpret_cast<const float4*>(x + (r + k < r1 ? k * a.ldx : 0) + c);
      q.w = *reinterpret_cast<const float4*>(w + c);
      q.b0 = *reinterpret_cast<const double2*>(a.wbar + c);
      q.b1 = *reinterpret_cast<const double2*>(a.wbar + c + 2);
    };
    auto sum = [&](const Cols& q, int64_t c, bool whole) {
      const float we[4] = {q.w.x, q.w.y, q.w.z, q.w.w};
      const double be[4] = {q.b0.x, q.b0.y, q.b1.x, q.b1.y};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (!whole && c + e >= a.dim) continue;  // entries past dim are not used
        const double wo = si * double(we[e]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double xv = e == 0 ? q.v[k].x : e == 1 ? q.v[k].y : e == 2 ? q.v[k].z : q.v[k].w;
          mo[k] = fma(xv, wo, mo[k]);
          mb[k] = fma(xv, be[e], mb[k]);
        }
      }
    };
    Cols q0, q1;
    int64_t c0 = 0;
    load(q0, 4 * lane);
    for (; c0 + 512 <= a.dim; c0 += 512) {
      load(q1, c0 + 256 + 4 * lane);
      sum(q0, c0 + 4 * lane, true);
      load(q0, c0 + 512 + 4 * lane);
      sum(q1, c0 + 256 + 4 * lane, true);
    }
    if (c0 + 256 < a.dim) load(q1, c0 + 256 + 4 * lane);
    if (c0 < a.dim) sum(q0, c0 + 4 * lane, false);
    if (c0 + 256 < a.dim) sum(q1, c0 + 256 + 4 * lane, false);
    // lane k: row k at its own model, lane 4 + k: at w_bar
    double m = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double o = wave_sum_d(mo[k]), b = wave_sum_d(mb[k]);
      m = lane == k ? o : lane == 4 + k ? b : m;
    }
    if (lane < 8 && r + (lane & 3) < r1) lsum += loss_of(double(a.y[int64_t(i) * a.S + r + (lane & 3)]) * m, a.loss);
  }
  const double lown = block_sum_d(lane < 4 ? lsum : 0.0, sh), lbar = block_sum_d(lane >= 4 ? lsum : 0.0, sh);
  if (threadIdx.x == 0) {
    double* q = a.part + kLossBase + 2 * (int64_t(i) * nch + ch);
    q[0] = lown;
    q[1] = lbar;
  }
}

// One block; every sum is linear in the partials, so they are added flat
// (||w_bar||^2 comes from the column pass: one block over w_bar took 1 ms at
// 2^20 columns).  Bound by latency: 1024 threads, so that each has a few loads
// and none waits for another, and one trip through LDS for all six sums (256
// threads and a block sum each: 16 us for 4096 + 2048 partials; now 9).
__global__ __launch_bounds__(1024) void finish_kernel(MetricArgs a, int ncb, int nch) {
  __shared__ double sh[6][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double cons = 0.0, msum = 0.0, wb2 = 0.0, w2 = 0.0, own = 0.0, bar = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < ncb; b += 1024) {
    const double* q = a.part + 4 * b;
    cons += q[0];
    msum += q[1];
    wb2 += q[2];
    w2 += q[3];
  }
  if (a.S > 0)
    for (int64_t b = threadIdx.x; b < int64_t(a.n) * nch; b += 1024) {
      const double* q = a.part + kLossBase + 2 * b;
      own += q[0];
      bar += q[1];
    }
  double v[6] = {cons, msum, wb2, w2, own, bar};
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    v[k] = wave_sum_d(v[k]);
    if (lane == 0) sh[k][wave] = v[k];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      v[k] = 0.0;
      for (int g = 0; g < 16; ++g) v[k] += sh[k][g];
    }
    cons = v[0], msum = v[1], wb2 = v[2], w2 = v[3], own = v[4], bar = v[5];
    const double nan = __longlong_as_double(0x7ff8000000000000ll), samples = double(a.n) * double(a.S);
    a.out[0] = a.S > 0 ? own / samples + 0.5 * double(a.l2) * (w2 / double(a.n)) : nan;
    a.out[1] = a.S > 0 ? bar / samples + 0.5 * double(a.l2) * wb2 : nan;
    a.out[2] = sqrt(cons);
    a.out[3] = msum / double(a.dim);
  }
}

}  // namespace

hipError_t launch_metrics(const MetricArgs& a, hipStream_t s) {
  const int ncb = int(std::min<int64_t>((a.dim + 63) / 64, kColBlocksMax));
  const int nch = metric_chunks(a.n, a.S);
  if (a.n <= 64)
    hipLaunchKernelGGL(cols_kernel<4>, dim3(ncb), dim3(256), 0, s, a);
  else if (a.n <= 256)
    hipLaunchKernelGGL(cols_kernel<16>, dim3(ncb), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(cols_kernel<0>, dim3(ncb), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.S > 0) {
    const dim3 grid(uint32_t(a.n) * uint32_t(nch));
    if (a.row_ptr)
      hipLaunchKernelGGL(loss_csr_kernel, grid, dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL(loss_dense_kernel, grid, dim3(256), 0, s, a, nch);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(1024), 0, s, a, ncb, nch);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Static scratch for callers that cannot allocate (asap_metrics_noalloc):
// w_bar, the partial sums and the four results live in this file-scope
// device array, one copy per GPU, kept until the process ends.  Host code
// never passes the array's name to a kernel or a copy: it uses the device
// address hipGetSymbolAddress returns for the current device.
// ---------------------------------------------------------------------------
namespace {

// n * metric_chunks(n, S) <= max(2048, n), so the partial sums of at most
// kStaticMetricMaxWorkers workers fit in kStaticPartMax bytes
constexpr size_t kStaticWbarBytes = size_t(kStaticMetricMaxDim) * 8;
constexpr size_t kStaticPartMax = (size_t(4 * kMetricColBlocks) + 2 * size_t(kStaticMetricMaxWorkers)) * 8;
constexpr size_t kStaticScratchBytes = kStaticWbarBytes + kStaticPartMax + 256;  // 8.4 MiB

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};

// device address of this GPU's copy of `scratch`, looked up once per device
// with that device current
hipError_t scratch_for_current_device(unsigned char** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_dev[dev] = p;
  }
  *ptr = static_cast<unsigned char*>(g_scratch_dev[dev]);
  return hipSuccess;
}

}  // namespace

hipError_t metrics_static_scratch(MetricArgs a, hipStream_t s, double* out_host) {
  if (a.dim < 1 || a.dim > kStaticMetricMaxDim || a.n < 1 || a.n > kStaticMetricMaxWorkers)
    return hipErrorInvalidValue;
  if (metric_part_doubles(a.n, a.S) * 8 > kStaticPartMax) return hipErrorInvalidValue;
  unsigned char* base = nullptr;
  hipError_t e = scratch_for_current_device(&base);
  if (e != hipSuccess) return e;
  // every word the kernels read is written by them first in this call
  // (w_bar by the column pass, the partials by the column and loss passes,
  // the results by the final pass), so nothing needs clearing
  a.wbar = reinterpret_cast<double*>(base);
  a.part = reinterpret_cast<double*>(base + kStaticWbarBytes);
  a.out = reinterpret_cast<double*>(base + kStaticWbarBytes + kStaticPartMax);
  if ((e = launch_metrics(a, s)) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(out_host, a.out, 4 * sizeof(double), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  return hipStreamSynchronize(s);
}

}  // namespace asap
