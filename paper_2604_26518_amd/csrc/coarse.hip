// Coarsest level: assembly and inversion of its pinned operator on the GPU.
//
// The coarsest grid has N_L = N / 2^(L-1) voxels per axis, so its matrix has
// 192 (4^3 nodes, elastic) to 2048 rows.  A = L L^T, W = L^-1 and A^-1 = W^T W are
// formed by blocks of 32 columns, two launches each.  Every entry is a sum over
// ascending k whose products and sums are rounded one by one (contraction is
// off in this file), so the blocking does not show in the result: it is the
// textbook column-by-column evaluation bit for bit, whatever the block size.
// Bound: the serial chain of the 32 columns inside a block (an LDS update each)
// and the two launches per block, not the n^3 FP64 operations.  Measured for the
// build of a 112^3 cell (n = 1029): 256 ms with the same sums on one host core,
// 6.4 ms so; for n = 192 the build of a 32^3 cell went from 4.2 to 3.1 ms.
#include "common.h"

#pragma clang fp contract(off)

namespace gmt {
namespace {

constexpr int kB = 32;      // columns per block, and the edge of an update tile
constexpr int kPanel = 64;  // rows (of L) or columns (of W) per panel workgroup

__device__ __forceinline__ int wrap(int v, int N) { return v < 0 ? v + N : (v >= N ? v - N : v); }

// Row block of node i: zero, then the element matrices of its (up to 8) active
// octants added in ascending element order (the 8 corners of an element are
// distinct nodes for N >= 2, so the threads of an element write distinct entries:
// no atomics, fixed order).  Rows and columns of node 0 (pinned) and the padding
// rows n .. np are those of the identity.
template <int D>
__global__ __launch_bounds__(256) void k_coarse_assemble(const int* __restrict__ node_lin,
                                                         const int* __restrict__ node_map,
                                                         const int* __restrict__ elem_map, int N, int n_n,
                                                         const double* __restrict__ Kel, int np,
                                                         double* __restrict__ A) {
  constexpr int M = 8 * D;
  const int i = blockIdx.x;
  const int t = threadIdx.x;
  const bool identity = i == 0 || i >= n_n;
  for (int k = t; k < D * np; k += 256) {
    const int row = i * D + k / np, col = k % np;
    if (row < np) A[(size_t)row * np + col] = identity && row == col ? 1.0 : 0.0;
  }
  if (identity) return;
  const int lin = node_lin[i];
  const int x = lin % N, y = (lin / N) % N, z = lin / (N * N);
  int last = -1;
  for (int step = 0; step < 8; ++step) {
    // the next larger element id among the octants (every thread finds the same)
    int e = -1, k = 0;
    for (int o = 0; o < 8; ++o) {
      const int ex = wrap(x - 1 + (o & 1), N), ey = wrap(y - 1 + ((o >> 1) & 1), N), ez = wrap(z - 1 + (o >> 2), N);
      const int v = elem_map[(ez * N + ey) * N + ex];
      if (v > last && (e < 0 || v < e)) e = v, k = o;
    }
    if (e < 0) return;
    last = e;
    __syncthreads();
    if (t >= D * M) continue;
    const int ex = wrap(x - 1 + (k & 1), N), ey = wrap(y - 1 + ((k >> 1) & 1), N), ez = wrap(z - 1 + (k >> 2), N);
    const int a = 7 - k, di = t / M, b = (t % M) / D, dj = t % D;
    const int j = node_map[(wrap(ez + (b >> 2), N) * N + wrap(ey + ((b >> 1) & 1), N)) * N + wrap(ex + (b & 1), N)];
    if (j > 0)
      A[(size_t)(i * D + di) * np + j * D + dj] += Kel[(size_t)e * M * M + (a * D + di) * M + b * D + dj];
  }
}

// Block k, first half.  Every workgroup factors the 32 x 32 diagonal block in LDS
// (redundantly: the workgroups run side by side); workgroup 0 checks the pivots
// (status[0]: 1 + the first column whose pivot is not above 1e-13 of the largest
// diagonal entry, status[1]: that pivot, status[2]: the entry).  Then the first
// n_lrow workgroups solve for 64 rows of L each below the block (a thread per
// row), the others finish 64 columns of W in the block's rows (a thread per
// column; W holds the sums over earlier blocks).
__global__ __launch_bounds__(256) void k_chol_panel(double* __restrict__ A, double* __restrict__ W, int np, int n,
                                                    int k, int n_lrow, double* __restrict__ status) {
  __shared__ double S[kB][kB + 1];
  __shared__ double red[256];
  const int t = threadIdx.x;
  const int k0 = k * kB;
  const bool first = blockIdx.x == 0;
  double dmax = 0.0;
  if (first) {
    if (k == 0) {
      for (int i = t; i < n; i += 256) dmax = fmax(dmax, A[(size_t)i * np + i]);
      red[t] = dmax;
      __syncthreads();
      for (int o = 128; o > 0; o >>= 1) {
        if (t < o) red[t] = fmax(red[t], red[t + o]);
        __syncthreads();
      }
      dmax = red[0];
      if (t == 0) {
        status[0] = status[1] = 0.0;
        status[2] = dmax;
      }
    } else {
      dmax = status[2];
    }
  }
  const int r = t >> 3, c0 = (t & 7) * 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) S[r][c0 + q] = A[(size_t)(k0 + r) * np + k0 + c0 + q];
  for (int p = 0; p < kB; ++p) {
    __syncthreads();
    const double piv = S[p][p];
    const double l = sqrt(piv);
    if (first && t == 0 && !(piv > 1e-13 * dmax) && status[0] == 0.0) {
      status[0] = k0 + p + 1;
      status[1] = piv;
    }
    __syncthreads();
    if (t == p) S[p][p] = l;
    else if (t > p && t < kB) S[t][p] = S[t][p] / l;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = c0 + q;
      if (c > p && r >= c) S[r][c] = S[r][c] - S[r][p] * S[c][p];
    }
  }
  __syncthreads();
  if ((int)blockIdx.x < n_lrow) {
    if (t < kPanel) {
      const int row = k0 + kB + (int)blockIdx.x * kPanel + t;
      if (row < np) {
        double* a = A + (size_t)row * np + k0;
        double v[kB];
#pragma unroll
        for (int j = 0; j < kB; ++j) v[j] = a[j];
#pragma unroll
        for (int j = 0; j < kB; ++j) {
          double s = v[j];
#pragma unroll
          for (int m = 0; m < j; ++m) s = s - v[m] * S[j][m];
          v[j] = s / S[j][j];
        }
#pragma unroll
        for (int j = 0; j < kB; ++j) a[j] = v[j];
      }
    }
  } else if (t < kPanel) {
    const int c = ((int)blockIdx.x - n_lrow) * kPanel + t;
    if (c < k0 + kB) {
      double w[kB];
#pragma unroll
      for (int i = 0; i < kB; ++i) w[i] = c < k0 ? W[(size_t)(k0 + i) * np + c] : 0.0;
#pragma unroll
      for (int i = 0; i < kB; ++i) {
        double s = w[i];
#pragma unroll
        for (int m = 0; m < i; ++m) s = s + S[i][m] * w[m];
        w[i] = c == k0 + i ? 1.0 / S[i][i] : (c < k0 + i ? -s / S[i][i] : 0.0);
      }
#pragma unroll
      for (int i = 0; i < kB; ++i) W[(size_t)(k0 + i) * np + c] = w[i];
    }
  }
}

// Block k, second half, 32 x 32 tiles (ti, tj) of the rows below the block:
// z = 0: A_ij - sum_k L_ik L_jk for k0 + 32 <= j <= i; z = 1: the sums of W's
// rows, W_ic + sum_k L_ik W_kc for c < k0 + 32 (W starts at zero).
__global__ __launch_bounds__(256) void k_chol_update(double* __restrict__ A, double* __restrict__ W, int np, int k) {
  __shared__ double X[kB][kB + 1], Y[kB][kB + 1];
  const int t = threadIdx.x;
  const int k0 = k * kB;
  const int r = t >> 3, c0 = (t & 7) * 4;
  const int ti = k + 1 + (int)blockIdx.y;
  const bool lower = blockIdx.z == 0;
  const int tj = (int)blockIdx.x + (lower ? k + 1 : 0);
  if (lower ? tj > ti : tj > k) return;
  double* out = lower ? A : W;
  double v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    X[r][c0 + q] = A[(size_t)(ti * kB + r) * np + k0 + c0 + q];  // L_ik
    // Y[m][c]: L_jk transposed, or W_kc
    if (lower) Y[c0 + q][r] = A[(size_t)(tj * kB + r) * np + k0 + c0 + q];
    else Y[r][c0 + q] = W[(size_t)(k0 + r) * np + tj * kB + c0 + q];
    // the first block whose rows of W are finished starts their sums
    v[q] = !lower && tj == k ? 0.0 : out[(size_t)(ti * kB + r) * np + tj * kB + c0 + q];
  }
  __syncthreads();
  if (lower) {
    for (int m = 0; m < kB; ++m) {
      const double x = X[r][m];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = v[q] - x * Y[m][c0 + q];
    }
  } else {
    for (int m = 0; m < kB; ++m) {
      const double x = X[r][m];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = v[q] + x * Y[m][c0 + q];
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) out[(size_t)(ti * kB + r) * np + tj * kB + c0 + q] = v[q];
}

// A^-1 = W^T W, tiles ti >= tj mirrored; rows and columns of the pinned node are zero
__global__ __launch_bounds__(256) void k_chol_inverse(const double* __restrict__ W, int np, int n, int D,
                                                      double* __restrict__ c64, float* __restrict__ c32) {
  const int tj = blockIdx.x, ti = blockIdx.y;
  if (tj > ti) return;
  __shared__ double X[kB][kB + 1], Y[kB][kB + 1];
  const int t = threadIdx.x;
  const int r = t >> 3, c0 = (t & 7) * 4;
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (int kb = ti; kb * kB < np; ++kb) {  // W is zero above its diagonal
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      X[r][c0 + q] = W[(size_t)(kb * kB + r) * np + ti * kB + c0 + q];
      Y[r][c0 + q] = W[(size_t)(kb * kB + r) * np + tj * kB + c0 + q];
    }
    __syncthreads();
#pragma unroll 8
    for (int m = 0; m < kB; ++m) {
      const double x = X[m][r];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = v[q] + x * Y[m][c0 + q];
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = ti * kB + r, j = tj * kB + c0 + q;
    if (i >= n || j > i) continue;
    const double x = j < D || i < D ? 0.0 : v[q];
    c64[(size_t)i * n + j] = c64[(size_t)j * n + i] = x;
    c32[(size_t)i * n + j] = c32[(size_t)j * n + i] = (float)x;
  }
}

}  // namespace

size_t coarse_scratch_doubles(int n) {
  const size_t np = (size_t)(n + kB - 1) / kB * kB;
  return 2 * np * np;
}

// Kel: [n_e][8D][8D] element matrices of the coarsest level; scratch:
// coarse_scratch_doubles(n_n * D) doubles; status: 3 doubles (see k_chol_panel).
void launch_coarse_inverse(const int* node_lin, const int* node_map, const int* elem_map, int N, int n_n, int D,
                           const double* Kel, double* scratch, double* c64, float* c32, double* status,
                           hipStream_t s) {
  const int n = n_n * D, nt = (n + kB - 1) / kB, np = nt * kB;
  double* A = scratch;
  double* W = A + (size_t)np * np;
  const int rows = (np + D - 1) / D;  // node rows, the padding included
  if (D == 3)
    hipLaunchKernelGGL(k_coarse_assemble<3>, dim3(rows), dim3(256), 0, s, node_lin, node_map, elem_map, N, n_n, Kel,
                       np, A);
  else
    hipLaunchKernelGGL(k_coarse_assemble<1>, dim3(rows), dim3(256), 0, s, node_lin, node_map, elem_map, N, n_n, Kel,
                       np, A);
  GMT_LAUNCH_CHECK();
  for (int k = 0; k < nt; ++k) {
    const int below = nt - 1 - k;  // row tiles below the block
    const int n_lrow = below > 0 ? (below * kB + kPanel - 1) / kPanel : 1;
    const int n_wcol = ((k + 1) * kB + kPanel - 1) / kPanel;
    hipLaunchKernelGGL(k_chol_panel, dim3(n_lrow + n_wcol), dim3(256), 0, s, A, W, np, n, k, n_lrow, status);
    if (below > 0)
      hipLaunchKernelGGL(k_chol_update, dim3(nt, below, 2), dim3(256), 0, s, A, W, np, k);
    GMT_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(k_chol_inverse, dim3(nt, nt), dim3(256), 0, s, W, np, n, D, c64, c32);
  GMT_LAUNCH_CHECK();
}

}  // namespace gmt
