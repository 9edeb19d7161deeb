// Optimality-Criteria update of SIMP inverse homogenization (App. F.3).
#include <algorithm>

#include "common.h"

namespace gmt {
namespace {

constexpr int kBlock = 256;
constexpr int kDepth = 3;                  // bisection steps per pass over the densities
constexpr int kCand = (1 << kDepth) - 1;   // multipliers they may try
constexpr int kMaxSteps = 200;

__device__ __forceinline__ double oc_density(double r, double B, double lam, double move, double eta, double lo) {
  const double cand = r * pow(B / lam, eta);
  return fmin(fmin(1.0, r + move), fmax(cand, fmax(lo, r - move)));
}

// The multipliers that up to three bisection steps from [lo, hi] may try, in heap order
// (the children of k, 2 k + 1 and 2 k + 2, follow hi = lam and lo = lam).
__device__ __forceinline__ void candidates(double lo, double hi, double (&lam)[kCand]) {
  double l[kCand], h[kCand];
  l[0] = lo, h[0] = hi;
#pragma unroll
  for (int k = 0; k < kCand; ++k) {
    lam[k] = 0.5 * (l[k] + h[k]);
    if (2 * k + 2 < kCand) {
      l[2 * k + 1] = l[k], h[2 * k + 1] = lam[k];
      l[2 * k + 2] = lam[k], h[2 * k + 2] = h[k];
    }
  }
}

// Per-block sums of the updated densities for every candidate multiplier.  Bisecting one
// step per pass costs ~76 passes of two launches and a host round trip each (25 us a
// step, whatever n); three steps a pass with the decision on the device cost 7 powers
// per density and no round trip: 64^3 densities 1.9 -> 0.6 ms.  Each sum is the one a
// pass with that multiplier alone forms, bit for bit.
__global__ __launch_bounds__(kBlock) void k_oc_sums(const double* __restrict__ rho, const double* __restrict__ dc,
                                                    size_t n, double move, double eta, double lo,
                                                    const OcState* __restrict__ st, double* __restrict__ partial) {
  __shared__ double sh[kBlock / 64][kCand];
  if (st->done) return;
  double lam[kCand], acc[kCand];
  candidates(st->lo, st->hi, lam);
#pragma unroll
  for (int k = 0; k < kCand; ++k) acc[k] = 0.0;
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) {
    const double r = rho[i];
    const double B = fmax(-dc[i], 0.0);
#pragma unroll
    for (int k = 0; k < kCand; ++k) acc[k] += oc_density(r, B, lam[k], move, eta, lo);
  }
#pragma unroll
  for (int k = 0; k < kCand; ++k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_down(acc[k], o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][k] = acc[k];
  }
  __syncthreads();
  if (threadIdx.x < kCand) {
    double t = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) t += sh[w][threadIdx.x];
    partial[(size_t)blockIdx.x * kCand + threadIdx.x] = t;
  }
}

// Totals (a wave per candidate; lane l sums the partials b = l + 64 q, b + 256, .. for q <
// 4, then a tree) and the bisection steps they decide: vol > target raises lo.
__global__ __launch_bounds__(64 * kCand) void k_oc_step(const double* __restrict__ partial, int nblocks, double target,
                                                        OcState* __restrict__ st) {
  __shared__ double vol[kCand];
  if (st->done) return;
  const int lane = threadIdx.x & 63, k = threadIdx.x >> 6;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 4; ++q)
    for (int b = lane + 64 * q; b < nblocks; b += kBlock) s[q] += partial[(size_t)b * kCand + k];
  double v = (s[0] + s[2]) + (s[1] + s[3]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if (lane == 0) vol[k] = v;
  __syncthreads();
  if (threadIdx.x != 0) return;
  double lo = st->lo, hi = st->hi, lam = st->lam;
  int steps = st->steps, done = 0;
  for (int d = 0, at = 0; d < kDepth && !done; ++d) {
    lam = 0.5 * (lo + hi);
    const bool up = vol[at] > target;
    if (up) lo = lam;
    else hi = lam;
    at = 2 * at + (up ? 2 : 1);
    ++steps;
    done = hi - lo <= 1e-10 * fmax(hi, 1e-30) || steps >= kMaxSteps;
  }
  st->lo = lo;
  st->hi = hi;
  st->lam = lam;
  st->steps = steps;
  st->done = done;
}

__global__ void k_oc_init(OcState* st) {
  st->lo = 0.0;
  st->hi = 1e9;
  st->lam = 1e9;
  st->steps = st->done = 0;
}

__global__ __launch_bounds__(kBlock) void k_oc_write(const double* __restrict__ rho, const double* __restrict__ dc,
                                                     size_t n, double move, double eta, double lo,
                                                     const OcState* __restrict__ st, double* __restrict__ out) {
  const double lam = st->lam;
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock)
    out[i] = oc_density(rho[i], fmax(-dc[i], 0.0), lam, move, eta, lo);
}

unsigned oc_grid(size_t n) { return (unsigned)std::min<size_t>(kRedBlocks, (n + kBlock - 1) / kBlock); }

}  // namespace

size_t oc_partial_doubles() { return (size_t)kRedBlocks * kCand; }

void launch_oc_begin(OcState* st, hipStream_t s) {
  hipLaunchKernelGGL(k_oc_init, dim3(1), dim3(1), 0, s, st);
  GMT_LAUNCH_CHECK();
}

void launch_oc_pass(const double* rho, const double* dc, size_t n, double target, double move, double eta, double lo,
                    OcState* st, double* partial, hipStream_t s) {
  const unsigned g = oc_grid(n);
  hipLaunchKernelGGL(k_oc_sums, dim3(g), dim3(kBlock), 0, s, rho, dc, n, move, eta, lo, st, partial);
  hipLaunchKernelGGL(k_oc_step, dim3(1), dim3(64 * kCand), 0, s, partial, (int)g, target, st);
  GMT_LAUNCH_CHECK();
}

void launch_oc_write(const double* rho, const double* dc, size_t n, double move, double eta, double lo,
                     const OcState* st, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_oc_write, dim3(oc_grid(n)), dim3(kBlock), 0, s, rho, dc, n, move, eta, lo, st, out);
  GMT_LAUNCH_CHECK();
}

}  // namespace gmt
