// Operator sweeps of the coarse levels from assembled stencils: per node the 27 D x D
// blocks of K^l and its 27 neighbour ids, instead of the 8 element matrices around it
// (64 blocks, found through the dense maps).  Bound by the matrix bytes: 27 D^2 values
// a node (1008 B for D = 3 in FP32, padding included) against 64 D^2 (2304 B), read
// coalesced (a node's coefficients lie n apart in runs of 4), and on the small levels
// by the dependent loads (map -> element -> coefficient -> gather before, id -> gather
// now).  The blocks are summed in FP64 and rounded once, so an FP32 sweep rounds less
// than with the FP32 element matrices.
#include "common.h"

namespace gmt {
namespace {

constexpr int kGroups = 7;  // neighbours in groups of 4: 27 and one of padding
constexpr int kBS = 64;

template <typename T>
struct alignas(16) vec4 {
  T v[4];
};

__device__ __forceinline__ int wrapm(int v, int N) { return v < 0 ? v + N : (v >= N ? v - N : v); }

// XCD k works on the k-th contiguous share of the nodes (kernels.hip: xcd_block)
__device__ __forceinline__ int block_index(int xcd) {
  const int B = (int)gridDim.x, b = (int)blockIdx.x;
  if (!xcd) return b;
  const int x = b & 7, q = B >> 3, r = B & 7;
  return x * q + min(x, r) + (b >> 3);
}

// Coefficients of group g of node i at stc[(g D^2 + k) n + i], k < D^2 (4 values each:
// neighbour 4 g + nb's block row-major at nb D^2 ..), its ids at nbr[g n + i]; an
// absent neighbour and the padding have zero blocks and the node's own id.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_stencil_build(int n, int N, int kind, const int* __restrict__ node_lin,
                                                       const int* __restrict__ node_map,
                                                       const int* __restrict__ elem_map,
                                                       const uint8_t* __restrict__ cmask,
                                                       const double* __restrict__ K, vec4<T>* __restrict__ stc,
                                                       int4* __restrict__ nbr) {
  constexpr int DD = D * D, M = 8 * D;
  const int i = blockIdx.x * 256 + threadIdx.x, g = blockIdx.y;
  if (i >= n) return;
  const int lin = node_lin[i];
  const int x = lin % N, y = (lin / N) % N, z = lin / (N * N);
  double blk[4 * DD];
  int id[4];
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) {
    const int j = 4 * g + nb;
    const int jx = j % 3, jy = j / 3 % 3, jz = j / 9;
#pragma unroll
    for (int e = 0; e < DD; ++e) blk[nb * DD + e] = 0.0;
    id[nb] = i;
    if (j >= 27) continue;
    const int v = node_map[wrapm(x + jx - 1, N) + N * (wrapm(y + jy - 1, N) + N * wrapm(z + jz - 1, N))];
    if (v < 0) continue;
    id[nb] = v;
    for (int k = 0; k < 8; ++k) {
      const int dx = jx - (k & 1), dy = jy - ((k >> 1) & 1), dz = jz - (k >> 2);
      if (dx < 0 || dx > 1 || dy < 0 || dy > 1 || dz < 0 || dz > 1) continue;  // j is not a corner of octant k
      const int el = elem_map[wrapm(x - 1 + (k & 1), N) +
                              N * (wrapm(y - 1 + ((k >> 1) & 1), N) + N * wrapm(z - 1 + (k >> 2), N))];
      if (el < 0) continue;
      const double* Km = K + (size_t)(kind == KIND_TABLE ? (int)cmask[el] : el) * M * M + (7 - k) * D * M +
                         (dx + 2 * dy + 4 * dz) * D;
#pragma unroll
      for (int q = 0; q < D; ++q)
#pragma unroll
        for (int q2 = 0; q2 < D; ++q2) blk[nb * DD + q * D + q2] += Km[q * M + q2];
    }
  }
#pragma unroll
  for (int k = 0; k < DD; ++k) {
    vec4<T> c;
#pragma unroll
    for (int m = 0; m < 4; ++m) c.v[m] = (T)blk[4 * k + m];
    stc[((size_t)g * DD + k) * n + i] = c;
  }
  nbr[(size_t)g * n + i] = make_int4(id[0], id[1], id[2], id[3]);
}

template <typename T, int D, int CB, int EPI>
__global__ __launch_bounds__(kBS) void k_apply_stencil(LevelView<T> L, sweep_input<T, EPI> u, EpiArgs<T> e) {
  constexpr int DD = D * D;
  const int row = block_index(L.xcd) * kBS + threadIdx.x;
  if (row >= (L.list ? L.n_list : L.n_n)) return;
  const size_t i = L.list ? L.list[row] : row;
  const size_t n = (size_t)L.n_n;
  const int c0 = (int)blockIdx.y * CB;
  const vec4<T>* __restrict__ stc = reinterpret_cast<const vec4<T>*>(L.stc);
  const int4* __restrict__ nbr = reinterpret_cast<const int4*>(L.snbr);
  int4 ids[kGroups];
#pragma unroll
  for (int g = 0; g < kGroups; ++g) ids[g] = nbr[(size_t)g * n + i];
  // own values and epilogue inputs: loaded with the first group
  T fv[CB][D], dd[CB][D], us[CB][D], di[D], acc[CB][D];
  constexpr bool kDinv = EPI == EPI_JACOBI || EPI == EPI_GS || EPI == EPI_CHEB || EPI == EPI_CHEB0;
#pragma unroll
  for (int q = 0; q < D; ++q) di[q] = kDinv ? e.dinv[i * D + q] : T(0);
#pragma unroll
  for (int c = 0; c < CB; ++c)
#pragma unroll
    for (int q = 0; q < D; ++q) {
      const size_t idx = ((size_t)(c0 + c) * n + i) * D + q;
      fv[c][q] = EPI != EPI_KU ? e.f[idx] : T(0);
      dd[c][q] = EPI == EPI_CHEB ? e.dvec_in[idx] : T(0);
      us[c][q] = kDinv ? u[idx] : T(0);
      acc[c][q] = T(0);
    }
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    vec4<T> co[DD];
#pragma unroll
    for (int k = 0; k < DD; ++k) co[k] = stc[((size_t)g * DD + k) * n + i];
    const int id[4] = {ids[g].x, ids[g].y, ids[g].z, ids[g].w};
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      if (4 * g + nb >= 27) break;
#pragma unroll
      for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int q2 = 0; q2 < D; ++q2) {
          const T v = u[((size_t)(c0 + c) * n + id[nb]) * D + q2];
#pragma unroll
          for (int q = 0; q < D; ++q) {
            const int k = nb * DD + q * D + q2;
            acc[c][q] = fma(co[k / 4].v[k % 4], v, acc[c][q]);
          }
        }
    }
  }
  T o[CB][D], dn[CB][D];
#pragma unroll
  for (int c = 0; c < CB; ++c)
#pragma unroll
    for (int q = 0; q < D; ++q) {
      dn[c][q] = T(0);
      if constexpr (EPI == EPI_KU) {
        o[c][q] = acc[c][q];
      } else if constexpr (EPI == EPI_RESID) {
        o[c][q] = fv[c][q] - acc[c][q];
      } else if constexpr (EPI == EPI_JACOBI || EPI == EPI_GS) {
        o[c][q] = us[c][q] + e.omega * di[q] * (fv[c][q] - acc[c][q]);
      } else {
        dn[c][q] = e.rho2 * di[q] * (fv[c][q] - acc[c][q]);
        if constexpr (EPI == EPI_CHEB) dn[c][q] = e.rho1 * dd[c][q] + dn[c][q];
        o[c][q] = us[c][q] + dn[c][q];
      }
    }
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    const size_t idx = ((size_t)(c0 + c) * n + i) * D;
    if constexpr (EPI == EPI_CHEB || EPI == EPI_CHEB0) {
#pragma unroll
      for (int q = 0; q < D; ++q) e.dvec[idx + q] = dn[c][q];
    }
#pragma unroll
    for (int q = 0; q < D; ++q) e.out[idx + q] = o[c][q];
  }
}

template <typename T, int D, int CB>
void dispatch_epi(const LevelView<T>& L, int rows, int epi, const T* u, const EpiArgs<T>& e, hipStream_t s) {
  const int n = L.list ? L.n_list : L.n_n;
  if (n <= 0) return;
  const dim3 g((unsigned)((n + kBS - 1) / kBS), (unsigned)rows);
  switch (epi) {
    case EPI_KU: hipLaunchKernelGGL((k_apply_stencil<T, D, CB, EPI_KU>), g, dim3(kBS), 0, s, L, u, e); break;
    case EPI_RESID: hipLaunchKernelGGL((k_apply_stencil<T, D, CB, EPI_RESID>), g, dim3(kBS), 0, s, L, u, e); break;
    case EPI_JACOBI: hipLaunchKernelGGL((k_apply_stencil<T, D, CB, EPI_JACOBI>), g, dim3(kBS), 0, s, L, u, e); break;
    case EPI_GS: hipLaunchKernelGGL((k_apply_stencil<T, D, CB, EPI_GS>), g, dim3(kBS), 0, s, L, u, e); break;
    case EPI_CHEB: hipLaunchKernelGGL((k_apply_stencil<T, D, CB, EPI_CHEB>), g, dim3(kBS), 0, s, L, u, e); break;
    default: hipLaunchKernelGGL((k_apply_stencil<T, D, CB, EPI_CHEB0>), g, dim3(kBS), 0, s, L, u, e); break;
  }
  GMT_LAUNCH_CHECK();
}

}  // namespace

size_t stencil_values(int n, int D) { return (size_t)n * kGroups * 4 * D * D; }
size_t stencil_ids(int n) { return (size_t)n * kGroups * 4; }

template <typename T>
void launch_stencil_build(int n, int N, int D, int kind, const int* node_lin, const int* node_map,
                          const int* elem_map, const uint8_t* cmask, const double* K, T* stc, int* nbr,
                          hipStream_t s) {
  if (n <= 0) return;
  const dim3 g((unsigned)((n + 255) / 256), kGroups);
  if (D == 3)
    hipLaunchKernelGGL((k_stencil_build<T, 3>), g, dim3(256), 0, s, n, N, kind, node_lin, node_map, elem_map, cmask, K,
                       reinterpret_cast<vec4<T>*>(stc), reinterpret_cast<int4*>(nbr));
  else
    hipLaunchKernelGGL((k_stencil_build<T, 1>), g, dim3(256), 0, s, n, N, kind, node_lin, node_map, elem_map, cmask, K,
                       reinterpret_cast<vec4<T>*>(stc), reinterpret_cast<int4*>(nbr));
  GMT_LAUNCH_CHECK();
}

// L.cb: cases per thread, kStencilAll (all), kStencilOne or kStencilTwo (elastic)
template <typename T>
void launch_apply_stencil(const LevelView<T>& L, int D, int C, int epi, const T* u, const EpiArgs<T>& e,
                          hipStream_t s) {
  if (D == 3 && C == 6) {
    if (L.cb == kStencilOne) dispatch_epi<T, 3, 1>(L, 6, epi, u, e, s);
    else if (L.cb == kStencilTwo) dispatch_epi<T, 3, 2>(L, 3, epi, u, e, s);
    else dispatch_epi<T, 3, 6>(L, 1, epi, u, e, s);
  } else if (D == 1 && C == 3) {
    if (L.cb == kStencilOne) dispatch_epi<T, 1, 1>(L, 3, epi, u, e, s);
    else dispatch_epi<T, 1, 3>(L, 1, epi, u, e, s);
  } else {
    fail(GMT_E_INVAL, "unsupported (d, c) = (%d, %d)", D, C);
  }
}

#define GMT_STENCIL(T)                                                                                             \
  template void launch_stencil_build<T>(int, int, int, int, const int*, const int*, const int*, const uint8_t*,    \
                                        const double*, T*, int*, hipStream_t);                                     \
  template void launch_apply_stencil<T>(const LevelView<T>&, int, int, int, const T*, const EpiArgs<T>&, hipStream_t);
GMT_STENCIL(float)
GMT_STENCIL(double)

}  // namespace gmt
