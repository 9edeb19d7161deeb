// The reductions of an FP32 CG iteration, accumulated in FP64.  A workgroup takes one
// case (grid row), so that a thread holds 1 + D or 2 + 2 D sums instead of C times as
// many: on small cells the tree over the lanes, once per value, is what a reduction
// takes, on large ones its registers kept loads out of flight.  The column means of z
// come out of the same pass as r.z and r.r (r.(z - m) = r.z - sum_d m_d sum r_d, in FP64),
// instead of a pass of their own before it.  The FP64 solves keep the summation order of
// the kernels in kernels.hip.
// Per iteration at 32^3 (14.5 k nodes): column sums 6.6 + 3.2, p.q 9.6 + 3.8, r.z 8.9 +
// 3.7 us before; 4.1 + 2.9 and 4.7 + 6.0 us so.  512^3 (2.4 GB a vector): 0.42 + 0.80 +
// 0.81 ms before, 0.81 + 0.81 ms so (6.0 TB/s).
#include "common.h"

namespace gmt {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxGroups = 256;  // per case: 6 cases fill 256 CUs six times over

__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}

// this workgroup's sums of NV values per thread to partial[(case, workgroup)][NV]
template <int NV>
__device__ __forceinline__ void store_sums(const double (&v)[NV], double* __restrict__ partial) {
  __shared__ double sh[kThreads / 64][NV];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const double s = wave_sum64(v[k]);
    if (lane == 0) sh[w][k] = s;
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kThreads / 64; ++i) s += sh[i][threadIdx.x];
    partial[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * NV + threadIdx.x] = s;
  }
}

// PAIR = 0: [a.b, D column sums of b]; 1: [a.b, a.a, column sums of b, column sums of a]
template <int D, int PAIR>
__global__ __launch_bounds__(kThreads) void k_case_sums(const float* __restrict__ a, const float* __restrict__ b,
                                                        int n, double* __restrict__ partial) {
  constexpr int NV = PAIR ? 2 + 2 * D : 1 + D;
  constexpr int kAhead = 4;  // nodes whose values a thread loads at once
  a += (size_t)blockIdx.y * n * D;
  b += (size_t)blockIdx.y * n * D;
  double v[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = 0.0;
  const int step = (int)gridDim.x * kThreads;
  for (long long i0 = (long long)blockIdx.x * kThreads + threadIdx.x; i0 < n; i0 += (long long)kAhead * step) {
    float av[kAhead][D], bv[kAhead][D];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const long long i = i0 + (long long)k * step;
      const size_t at = (size_t)(i < n ? i : i0) * D;
#pragma unroll
      for (int q = 0; q < D; ++q) {
        av[k][q] = a[at + q];
        bv[k][q] = b[at + q];
      }
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (i0 + (long long)k * step >= n) break;
#pragma unroll
      for (int q = 0; q < D; ++q) {
        const double x = (double)av[k][q], y = (double)bv[k][q];
        v[0] += x * y;
        if (PAIR) {
          v[1] += x * x;
          v[2 + q] += y;
          v[2 + D + q] += x;
        } else {
          v[1 + q] += y;
        }
      }
    }
  }
  store_sums<NV>(v, partial);
}

// the groups' partials of case c, value threadIdx.x / 64, in every lane 0
__device__ __forceinline__ double group_sum(const double* __restrict__ partial, int groups, int nv, int c) {
  const int lane = threadIdx.x & 63, k = threadIdx.x >> 6;
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < kMaxGroups / 64; ++j) {
    const int g = lane + 64 * j;
    if (g < groups) s += partial[((size_t)c * groups + g) * nv + k];
  }
  return wave_sum64(s);
}

// second stage of p.q and the sums of q (a workgroup per case); r.z of the last
// iteration becomes the previous one (prev = cur)
template <int D>
__global__ __launch_bounds__(64 * (1 + D)) void k_finish_pq(const double* __restrict__ partial, int groups,
                                                            double* __restrict__ pq, double* __restrict__ sums,
                                                            const double* __restrict__ cur, double* __restrict__ prev) {
  const int c = blockIdx.x, k = threadIdx.x >> 6;
  const double s = group_sum(partial, groups, 1 + D, c);
  if ((threadIdx.x & 63) != 0) return;
  if (k == 0) {
    pq[c] = s;
    if (cur) prev[c] = cur[c];
  } else {
    sums[c * D + k - 1] = s;
  }
}

// second stage of r.(z - m), r.r and the sums of z, and the end of an iteration: with
// flags (captured iterations), flags[1] counts the iterations that ran with the flag
// clear, and flags[0] is set once every case meets ||r_m||^2 <= flags[2 + m] or a
// residual is not finite (the host reports that).  m is rounded as the direction update
// rounds it.
template <int D>
__global__ __launch_bounds__(64 * (2 + 2 * D)) void k_finish_rz(const double* __restrict__ partial, int groups, int C,
                                                                double inv_n, double* __restrict__ rz,
                                                                double* __restrict__ rr, double* __restrict__ sums,
                                                                double* __restrict__ flags) {
  constexpr int NV = 2 + 2 * D;
  __shared__ double sh[8][NV];
  const int k = threadIdx.x >> 6;
  for (int c = 0; c < C; ++c) {
    const double s = group_sum(partial, groups, NV, c);
    if ((threadIdx.x & 63) == 0) sh[c][k] = s;
  }
  __syncthreads();
  if ((int)threadIdx.x < C) {
    const int c = threadIdx.x;
    double v = sh[c][0];
#pragma unroll
    for (int q = 0; q < D; ++q) {
      v -= (double)(float)(sh[c][2 + q] * inv_n) * sh[c][2 + D + q];
      sums[c * D + q] = sh[c][2 + q];
    }
    rz[c] = v;
    rr[c] = sh[c][1];
  }
  if (!flags || threadIdx.x != 0 || flags[0] != 0.0) return;
  flags[1] += 1.0;
  bool done = true;
  for (int c = 0; c < C; ++c) {
    if (!isfinite(sh[c][1])) {
      done = true;
      break;
    }
    if (!(sh[c][1] <= flags[2 + c])) done = false;
  }
  if (done) flags[0] = 1.0;
}

int groups_for(int n) {
  const int g = (n + 2 * kThreads - 1) / (2 * kThreads);
  return g < 1 ? 1 : (g > kMaxGroups ? kMaxGroups : g);
}

}  // namespace

size_t case_sums_partials(int C) { return (size_t)C * kMaxGroups * 8; }

void launch_sums_pq(const float* p, const float* q, int n, int C, int D, double* partial, double* pq, double* sums,
                    hipStream_t s, const double* cur, double* prev) {
  const int g = groups_for(n);
  if (D == 3) {
    hipLaunchKernelGGL((k_case_sums<3, 0>), dim3(g, C), dim3(kThreads), 0, s, p, q, n, partial);
    hipLaunchKernelGGL((k_finish_pq<3>), dim3(C), dim3(256), 0, s, partial, g, pq, sums, cur, prev);
  } else if (D == 1) {
    hipLaunchKernelGGL((k_case_sums<1, 0>), dim3(g, C), dim3(kThreads), 0, s, p, q, n, partial);
    hipLaunchKernelGGL((k_finish_pq<1>), dim3(C), dim3(128), 0, s, partial, g, pq, sums, cur, prev);
  } else {
    fail(GMT_E_INVAL, "unsupported d = %d", D);
  }
  GMT_LAUNCH_CHECK();
}

void launch_sums_rz(const float* r, const float* z, double inv_n, int n, int C, int D, double* partial, double* rz,
                    double* rr, double* sums, double* flags, hipStream_t s) {
  if (C > 8) fail(GMT_E_INVAL, "unsupported c = %d", C);
  const int g = groups_for(n);
  if (D == 3) {
    hipLaunchKernelGGL((k_case_sums<3, 1>), dim3(g, C), dim3(kThreads), 0, s, r, z, n, partial);
    hipLaunchKernelGGL((k_finish_rz<3>), dim3(1), dim3(512), 0, s, partial, g, C, inv_n, rz, rr, sums, flags);
  } else if (D == 1) {
    hipLaunchKernelGGL((k_case_sums<1, 1>), dim3(g, C), dim3(kThreads), 0, s, r, z, n, partial);
    hipLaunchKernelGGL((k_finish_rz<1>), dim3(1), dim3(256), 0, s, partial, g, C, inv_n, rz, rr, sums, flags);
  } else {
    fail(GMT_E_INVAL, "unsupported d = %d", D);
  }
  GMT_LAUNCH_CHECK();
}

}  // namespace gmt
