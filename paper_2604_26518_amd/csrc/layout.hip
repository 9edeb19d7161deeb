// Layout changes between the ABI's [n][C][D] and the solver's [C][n][D].
#include "common.h"

namespace gmt {
namespace {

constexpr int kBlock = 256;
constexpr int kTile = 128;  // nodes per workgroup

// ABI [n][C][D] -> solver [C][n][D].  Bound by HBM.  A node's values are one
// contiguous run of the source, and of C runs of the destination that lie n D
// apart: read in destination order, every 128-byte line of the source is
// fetched by several cases' workgroups long after one another.  So a workgroup
// reads the rows of 128 nodes once, in order, into LDS and writes each case's
// run from there.  8.7 M nodes, 6 cases, FP64 (2.5 GB): 1.30 ms (1.9 TB/s) in
// destination order, 0.37 ms (6.5 TB/s) so.
template <typename Tin, typename Tout, int C, int D>
__global__ __launch_bounds__(kBlock) void k_aos_to_soa(const Tin* __restrict__ a, Tout* __restrict__ b, int n) {
  constexpr int Q = C * D;
  __shared__ Tin s[kTile * Q];
  const size_t i0 = (size_t)blockIdx.x * kTile;
  const int m = (int)min((size_t)kTile, (size_t)n - i0);  // nodes of this tile
#pragma unroll
  for (int k = 0; k < (kTile * Q + kBlock - 1) / kBlock; ++k) {
    const int j = k * kBlock + (int)threadIdx.x;
    if (j < m * Q) s[j] = a[i0 * Q + j];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < (kTile * Q + kBlock - 1) / kBlock; ++k) {
    const int j = k * kBlock + (int)threadIdx.x;
    const int c = j / (kTile * D), r = j % (kTile * D);
    if (c < C && r < m * D) b[((size_t)c * n + i0) * D + r] = (Tout)s[(r / D) * Q + c * D + r % D];
  }
}

// solver [C][n][D] -> ABI [n][C][D]: in destination order (the C source runs are
// read once each: 5.6 TB/s on the vector above)
template <typename Tin, typename Tout, int C, int D>
__global__ __launch_bounds__(kBlock) void k_soa_to_aos(const Tin* __restrict__ a, Tout* __restrict__ b, int n) {
  const size_t idx = (size_t)blockIdx.x * kBlock + threadIdx.x;  // index into b
  if (idx >= (size_t)n * C * D) return;
  const int d = (int)(idx % D);
  const size_t t = idx / D;
  const size_t c = t % C, i = t / C;
  b[idx] = (Tout)a[(c * n + i) * D + d];
}

}  // namespace

template <typename Tin, typename Tout>
void launch_aos_to_soa(const Tin* a, Tout* b, int n, int C, int D, hipStream_t s) {
  if (n <= 0) return;
  const dim3 g((unsigned)((n + kTile - 1) / kTile));
  if (C == 6 && D == 3) hipLaunchKernelGGL((k_aos_to_soa<Tin, Tout, 6, 3>), g, dim3(kBlock), 0, s, a, b, n);
  else if (C == 3 && D == 1) hipLaunchKernelGGL((k_aos_to_soa<Tin, Tout, 3, 1>), g, dim3(kBlock), 0, s, a, b, n);
  else fail(GMT_E_INVAL, "unsupported (c, d)");
  GMT_LAUNCH_CHECK();
}

template <typename Tin, typename Tout>
void launch_soa_to_aos(const Tin* a, Tout* b, int n, int C, int D, hipStream_t s) {
  if (n <= 0) return;
  const dim3 g((unsigned)(((size_t)n * C * D + kBlock - 1) / kBlock));
  if (C == 6 && D == 3) hipLaunchKernelGGL((k_soa_to_aos<Tin, Tout, 6, 3>), g, dim3(kBlock), 0, s, a, b, n);
  else if (C == 3 && D == 1) hipLaunchKernelGGL((k_soa_to_aos<Tin, Tout, 3, 1>), g, dim3(kBlock), 0, s, a, b, n);
  else fail(GMT_E_INVAL, "unsupported (c, d)");
  GMT_LAUNCH_CHECK();
}

#define GMT_LAYOUT(Tin, Tout)                                                              \
  template void launch_aos_to_soa<Tin, Tout>(const Tin*, Tout*, int, int, int, hipStream_t); \
  template void launch_soa_to_aos<Tin, Tout>(const Tin*, Tout*, int, int, int, hipStream_t);
GMT_LAYOUT(float, float)
GMT_LAYOUT(double, double)
GMT_LAYOUT(float, double)
GMT_LAYOUT(double, float)

}  // namespace gmt
