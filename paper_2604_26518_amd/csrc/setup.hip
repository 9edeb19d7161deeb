// Hierarchy construction: compaction of flag fields, the tables of the staged
// interior sweep, connected components, Galerkin element matrices.
#include <algorithm>
#include <climits>
#include <cstdlib>

#include "common.h"

namespace gmt {
namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ int wrapm(int v, int N) { return v < 0 ? v + N : (v >= N ? v - N : v); }

// ---------------------------------------------------------------- scan
// Flags to ids: per-tile sums, their exclusive scan by one workgroup, then the
// map (id or -1) and list of the flagged items in linear order.  Bound by HBM
// (flags read twice, map written); a tile is 256 threads x 16 items.
constexpr int kScanItems = 16;
constexpr int kScanTile = kBlock * kScanItems;

// exclusive scan over NT threads, with the NT / 64 wave sums in the caller's LDS
// (free at the call; it is free again when the function returns)
template <int NT>
__device__ int block_exclusive_scan(int v, int* total, int* wsum) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int tt = __shfl_up(incl, o, 64);
    if (lane >= o) incl += tt;
  }
  if (lane == 63) wsum[wid] = incl;
  __syncthreads();
  int off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    if (w < wid) off += wsum[w];
    tot += wsum[w];
  }
  __syncthreads();
  *total = tot;
  return off + incl - v;
}

__global__ __launch_bounds__(kBlock) void k_scan_reduce(const int* __restrict__ flags, size_t n,
                                                        int* __restrict__ bsum) {
  __shared__ int wsum[kBlock / 64];
  const size_t base = (size_t)blockIdx.x * kScanTile;
  int s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    size_t i = base + (size_t)k * kBlock + threadIdx.x;
    if (i < n) s += flags[i];
  }
  int tot;
  block_exclusive_scan<kBlock>(s, &tot, wsum);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// exclusive scan of nb tile sums by one workgroup, 16 consecutive sums per thread
// and step (a 512^3 field has 32768 tiles: 8 steps); total -> *d_total
__global__ __launch_bounds__(kBlock) void k_scan_top(int* __restrict__ bsum, int nb, int* __restrict__ d_total) {
  __shared__ int wsum[kBlock / 64];
  int carry = 0;
  for (int base = 0; base < nb; base += kScanTile) {
    const int i0 = base + (int)threadIdx.x * kScanItems;
    int v[kScanItems], s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      v[k] = i0 + k < nb ? bsum[i0 + k] : 0;
      s += v[k];
    }
    int tot;
    int off = carry + block_exclusive_scan<kBlock>(s, &tot, wsum);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      if (i0 + k < nb) bsum[i0 + k] = off;
      off += v[k];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) *d_total = carry;
}

// A wave owns 1024 consecutive items and takes them 64 at a time, so that every
// load and store is contiguous; an item's rank is the wave's offset plus the
// flags below it by ballot.
__global__ __launch_bounds__(kBlock) void k_scan_write(const int* __restrict__ flags, size_t n,
                                                       const int* __restrict__ boff, int* __restrict__ map,
                                                       int* __restrict__ lin) {
  __shared__ int wsum[kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)wid * (64 * kScanItems);
  unsigned long long bits[kScanItems];
  int s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const size_t i = base + (size_t)k * 64 + lane;
    bits[k] = __ballot(i < n && flags[i] != 0);
    s += __popcll(bits[k]);
  }
  if (lane == 0) wsum[wid] = s;
  __syncthreads();
  int off = boff[blockIdx.x];
  for (int w = 0; w < wid; ++w) off += wsum[w];
  const unsigned long long below = (1ull << lane) - 1;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const size_t i = base + (size_t)k * 64 + lane;
    const int id = off + __popcll(bits[k] & below);
    const bool set = (bits[k] >> lane) & 1;
    if (i < n) {
      map[i] = set ? id : -1;
      if (set && lin) lin[id] = (int)i;
    }
    off += __popcll(bits[k]);
  }
}

// ---------------------------------------------------------------- staged interior sweep
// Tables of the staged interior sweep, one workgroup per group of NB interior
// nodes: the distinct ids among their 27 NB neighbours are counted (pass 0, every
// group b: cnt[b]) or, for the groups b = blk[g] that the staged sweep takes,
// written out ascending at off[g] together with each node's 27 positions among
// them (pass 1).
//
// The neighbours in one z-plane lie in a short interval of ids (consecutive interior
// nodes have consecutive neighbours, and the x - 1, x, x + 1 neighbours are
// consecutive ids), so the set is a bitmap over the intervals of the group's planes:
// bits set by LDS atomics, positions by popcount against a prefix over the words.
// Groups whose intervals need more than kStageBits bits (at 512^3 those that wrap
// in y) are left to the sorting kernel below (route[b] = 1).  Bound by the node-map lookups (9 per node) and the slot rows.
// 512^3 gyroid, 32.3 M interior nodes: 2 x 29.5 ms with every group sorted,
// 2 x 1.4 ms so (and 2 x 0.7 ms for the groups that are sorted).
constexpr int kStageBits = 1 << 17;
// planes told apart: those before, of and after the group's first node's plane and on;
// the last one takes all further planes (small cells)
constexpr int kStagePlanes = 6;

template <int NB>
__global__ __launch_bounds__(NB) void k_stage_tables(const int* __restrict__ interior, int n_int,
                                                     const int* __restrict__ node_lin,
                                                     const int* __restrict__ node_map, int N, int pass,
                                                     const int* __restrict__ blk, int* __restrict__ cnt,
                                                     const long long* __restrict__ off, int* __restrict__ ids,
                                                     uint16_t* __restrict__ slot, int* __restrict__ route, int max_words) {
  constexpr int kWords = kStageBits / 32;  // >= max_words
  __shared__ unsigned bits[kWords];
  __shared__ uint16_t pre[kWords];
  __shared__ int list[8 * NB];  // pass 1: a staged group has at most 8 NB distinct ids
  constexpr int PL = kStagePlanes;
  __shared__ int lo3[PL], hi3[PL], bias3[PL];
  __shared__ int wstart[PL], wbias[PL], n_words, z_first;
  __shared__ int wsum[NB / 64];
  const int tid = threadIdx.x;
  const int b = pass == 0 ? (int)blockIdx.x : blk[blockIdx.x];
  const int t = b * NB + tid;
  const bool valid = t < n_int;
  int ctr[9], edge[9];
  bool left = false, right = false;  // x - 1 / x + 1 is the id next to ctr (no wrap)
  int plane = 0;                     // of z - 1; z and z + 1 follow
  if (tid < PL) lo3[tid] = INT_MAX, hi3[tid] = -1;
  if (tid == 0) z_first = node_lin[interior[t]] / (N * N);
  __syncthreads();
  int mn[3] = {INT_MAX, INT_MAX, INT_MAX}, mx[3] = {-1, -1, -1};
  if (valid) {
    const int lin = node_lin[interior[t]];
    const int x = lin % N, y = (lin / N) % N, z = lin / (N * N);
    left = x > 0;
    right = x < N - 1;
    plane = z - z_first;
#pragma unroll
    for (int r = 0; r < 9; ++r) {
      const int row = N * (wrapm(y + r % 3 - 1, N) + N * wrapm(z + r / 3 - 1, N));
      ctr[r] = node_map[x + row];
      edge[r] = left && right ? ctr[r] : node_map[(left ? 0 : N - 1) + row];
      mn[r / 3] = min(mn[r / 3], min(left ? ctr[r] - 1 : ctr[r], edge[r]));
      mx[r / 3] = max(mx[r / 3], max(right ? ctr[r] + 1 : ctr[r], edge[r]));
    }
  }
  const int p0 = __shfl(plane, 0, 64);
  if (__all(!valid || plane == p0)) {  // one plane's nodes in the wave: one update per interval
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        mn[k] = min(mn[k], __shfl_xor(mn[k], o, 64));
        mx[k] = max(mx[k], __shfl_xor(mx[k], o, 64));
      }
      if ((tid & 63) == 0) {
        atomicMin(&lo3[min(p0 + k, PL - 1)], mn[k]);
        atomicMax(&hi3[min(p0 + k, PL - 1)], mx[k]);
      }
    }
  } else if (valid) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      atomicMin(&lo3[min(plane + k, PL - 1)], mn[k]);
      atomicMax(&hi3[min(plane + k, PL - 1)], mx[k]);
    }
  }
  __syncthreads();
  if (tid == 0) {
    // intervals in ascending order (empty ones, lo = INT_MAX, last); overlapping ones
    // share their bits
    int o[PL];
    for (int k = 0; k < PL; ++k) {
      int at = k;
      for (; at > 0 && lo3[o[at - 1]] > lo3[k]; --at) o[at] = o[at - 1];
      o[at] = k;
    }
    int words = 0, nw = 0, end = -1;
    for (int k = 0; k < PL; ++k) {
      const int w = o[k];
      if (hi3[w] < 0) break;
      if (nw > 0 && lo3[w] <= end) {
        end = max(end, hi3[w]);
      } else {
        if (nw > 0) words = wstart[nw - 1] + (end - (wbias[nw - 1] + 32 * wstart[nw - 1])) / 32 + 1;
        wstart[nw] = words;
        wbias[nw] = lo3[w] - 32 * words;
        ++nw;
        end = hi3[w];
      }
      bias3[w] = wbias[nw - 1];
    }
    words = wstart[nw - 1] + (end - (wbias[nw - 1] + 32 * wstart[nw - 1])) / 32 + 1;
    for (int k = nw; k < PL; ++k) wstart[k] = INT_MAX;
    n_words = words;
  }
  __syncthreads();
  const int words = n_words;
  if (words > max_words) {
    if (pass == 0 && tid == 0) route[b] = 1;
    return;
  }
  for (int w = tid; w < words; w += NB) bits[w] = 0;
  __syncthreads();
  if (valid) {
#pragma unroll
    for (int r = 0; r < 9; ++r) {
      const int base = ctr[r] - bias3[min(plane + r / 3, PL - 1)] - (left ? 1 : 0);
      const unsigned long long m = (unsigned long long)(left ? (right ? 7u : 3u) : (right ? 3u : 1u)) << (base & 31);
      atomicOr(&bits[base >> 5], (unsigned)m);
      if (m >> 32) atomicOr(&bits[(base >> 5) + 1], (unsigned)(m >> 32));
      if (!left || !right) {
        const int p = edge[r] - bias3[min(plane + r / 3, PL - 1)];
        atomicOr(&bits[p >> 5], 1u << (p & 31));
      }
    }
  }
  __syncthreads();
  const int per = (words + NB - 1) / NB, w0 = tid * per, w1 = min(words, w0 + per);
  int m = 0;
  for (int w = w0; w < w1; ++w) m += __popc(bits[w]);
  int total;
  int pos = block_exclusive_scan<NB>(m, &total, wsum);
  if (pass == 0) {
    if (tid == 0) cnt[b] = total, route[b] = 0;
    return;
  }
  for (int w = w0; w < w1; ++w) {
    pre[w] = (uint16_t)pos;
    int bias = wbias[0];
    for (int k = 1; k < PL && w >= wstart[k]; ++k) bias = wbias[k];
    for (unsigned v = bits[w]; v; v &= v - 1) list[pos++] = 32 * w + __ffs((int)v) - 1 + bias;
  }
  __syncthreads();
  const long long o0 = off[b];
  for (int k = tid; k < total; k += NB) ids[o0 + k] = list[k];
  if (!valid) return;
  auto rank = [&](int id, int bias) {
    const int p = id - bias;
    return (unsigned)pre[p >> 5] + (unsigned)__popc(bits[p >> 5] & ((1u << (p & 31)) - 1));
  };
  uint16_t row[kSlotStride];
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    const unsigned k = rank(ctr[r], bias3[min(plane + r / 3, PL - 1)]);
    const unsigned e = left && right ? 0 : rank(edge[r], bias3[min(plane + r / 3, PL - 1)]);
    row[3 * r] = (uint16_t)(left ? k - 1 : e);
    row[3 * r + 1] = (uint16_t)k;
    row[3 * r + 2] = (uint16_t)(right ? k + 1 : e);
  }
  row[27] = 0;
  static_assert(kSlotStride == 28, "slot rows are written as 7 words of 8 bytes");
  uint2* out = reinterpret_cast<uint2*>(slot + (size_t)t * kSlotStride);
#pragma unroll
  for (int k = 0; k < 7; ++k)
    out[k] = make_uint2(row[4 * k] | (unsigned)row[4 * k + 1] << 16, row[4 * k + 2] | (unsigned)row[4 * k + 3] << 16);
}

// The same for the groups with route[b] = 1: the 27 NB neighbour ids are sorted in
// LDS (bitonic) and a node's positions found by binary search.
template <int NB>
__global__ __launch_bounds__(NB) void k_stage_sort(const int* __restrict__ interior, int n_int,
                                                         const int* __restrict__ node_lin,
                                                         const int* __restrict__ node_map, int N, int pass,
                                                         const int* __restrict__ blk, int* __restrict__ cnt,
                                                         const long long* __restrict__ off, int* __restrict__ ids,
                                                         uint16_t* __restrict__ slot,
                                                         const int* __restrict__ route) {
  constexpr int kStageNodes = NB;
  constexpr int kStageSort = NB == 256 ? 8192 : 16384;  // >= 27 * NB, a power of two
  constexpr int kStageItems = kStageSort / NB;
  static_assert(27 * NB <= kStageSort, "sort buffer too small");
  __shared__ int s[kStageSort];
  const int g = blockIdx.x;
  const int b = pass == 0 ? g : blk[g];
  if (!route[b]) return;
  const int t = b * kStageNodes + (int)threadIdx.x;
  const bool valid = t < n_int;
  int nb[27];
  if (valid) {
    const int lin = node_lin[interior[t]];
    const int x = lin % N, y = (lin / N) % N, z = lin / (N * N);
#pragma unroll
    for (int j = 0; j < 27; ++j)
      nb[j] = node_map[wrapm(x + j % 3 - 1, N) + N * (wrapm(y + j / 3 % 3 - 1, N) + N * wrapm(z + j / 9 - 1, N))];
  }
#pragma unroll
  for (int j = 0; j < 27; ++j) s[(int)threadIdx.x * 27 + j] = valid ? nb[j] : INT_MAX;
  for (int k = 27 * kStageNodes + (int)threadIdx.x; k < kStageSort; k += kStageNodes) s[k] = INT_MAX;
  __syncthreads();
  for (int size = 2; size <= kStageSort; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int p = (int)threadIdx.x; p < kStageSort / 2; p += kStageNodes) {
        const int lo = 2 * p - (p & (stride - 1));  // the partner index lo + stride has that bit set
        const int hi = lo + stride;
        const int a = s[lo], c = s[hi];
        if ((a > c) == ((lo & size) == 0)) {
          s[lo] = c;
          s[hi] = a;
        }
      }
      __syncthreads();
    }
  }
  // distinct values: thread k owns the sorted entries k * kStageItems ..
  int v[kStageItems];
  int m = 0;
  const int base = (int)threadIdx.x * kStageItems;
#pragma unroll
  for (int k = 0; k < kStageItems; ++k) {
    v[k] = s[base + k];
    const int prev = base + k > 0 ? s[base + k - 1] : INT_MIN;
    if (v[k] == INT_MAX || v[k] == prev) v[k] = -1;  // not the first of its value
    m += v[k] >= 0;
  }
  int total;
  __syncthreads();  // every read of s above is done: its first words hold the wave sums
  int pos = block_exclusive_scan<kStageNodes>(m, &total, s);
  if (pass == 0) {
    if (threadIdx.x == 0) cnt[b] = total;
    return;
  }
  const long long o0 = off[b];
#pragma unroll
  for (int k = 0; k < kStageItems; ++k)
    if (v[k] >= 0) {
      s[pos] = v[k];
      ids[o0 + pos] = v[k];
      ++pos;
    }
  __syncthreads();
  if (!valid) return;
  uint16_t* row = slot + (size_t)t * kSlotStride;
#pragma unroll
  for (int j = 0; j < 27; ++j) {
    int lo = 0, hi = total;  // first position with s[pos] >= nb[j]
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (s[mid] < nb[j]) lo = mid + 1;
      else hi = mid;
    }
    row[j] = (uint16_t)lo;
  }
  row[27] = 0;
}

// ---------------------------------------------------------------- connected components
// Union-find over the active elements of level 1 with lock-free hooking (the
// scheme of Jaiganesh and Burtscher's ECL-CC): every element points to an
// element of smaller id in its set (parent[v] <= v), a root to itself; a union
// hooks the larger of the two roots under the smaller one by compare-and-swap
// and retries from the value it found when another thread hooked that root
// first.  Ids only decrease along every chain, so each loop ends.
__device__ __forceinline__ int cc_load(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// root of v's set, shortening the chain on the way (each element is pointed
// past its parent to its grandparent, which is also in the set)
__device__ int cc_root(int* parent, int v) {
  int cur = cc_load(parent + v);
  if (cur != v) {
    int prev = v, next;
    while (cur > (next = cc_load(parent + cur))) {
      __hip_atomic_store(parent + prev, next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      prev = cur;
      cur = next;
    }
  }
  return cur;
}

// Elements are in linear order, so a run of elements along x is a run of ids: an
// element starts under its run's first element (under the last element before its
// wave if the run began there), and only pairs of runs are left to union.
__device__ __forceinline__ bool run_head(const int* __restrict__ elem_lin, int v, int lin, int x) {
  return v == 0 || x == 0 || elem_lin[v - 1] != lin - 1;
}

__global__ __launch_bounds__(kBlock) void k_cc_init(const int* __restrict__ elem_lin, int n_e, int N,
                                                    int* __restrict__ parent, int* __restrict__ count) {
  const int v = blockIdx.x * kBlock + threadIdx.x;
  const int lane = threadIdx.x & 63;
  if (v == 0) *count = 0;
  bool head = false;
  if (v < n_e) {
    const int lin = elem_lin[v];
    head = run_head(elem_lin, v, lin, lin % N);
  }
  const unsigned long long m = __ballot(head) & (~0ull >> (63 - lane));  // heads at or below this lane
  if (v < n_e) parent[v] = v - lane + (m ? 63 - __clzll(m) : -1);
}

__device__ void cc_union(int* parent, int v, int w) {
  int a = cc_root(parent, v), b = cc_root(parent, w);
  while (a != b) {
    if (a < b) {
      const int got = atomicCAS(parent + b, b, a);
      if (got == b) break;
      b = got;  // b was hooked meanwhile: continue from its new parent (smaller)
    } else {
      const int got = atomicCAS(parent + a, a, b);
      if (got == a) break;
      a = got;
    }
  }
}

// Joins v to the active elements among its 26 periodic neighbours (all of them
// share at least one node with v).  Only the rows ahead (dy = 1 in the plane, dy =
// -1..1 in the next one: the others are joined from the other side) and, per row,
// only what the element before v in its run has not joined already: a run head
// sees the runs at x - 1, x, x + 1, another element one that begins at x + 1; the
// periodic ends of the rows are joined apart.  ~1.3 unions per run instead of 26 per
// element; 512^3 gyroid (33.6 M elements): 9 ms with every neighbour pair, 1.3 ms so.
__global__ __launch_bounds__(kBlock) void k_cc_hook(const int* __restrict__ elem_lin, int n_e,
                                                    const int* __restrict__ elem_map, int N, int* parent) {
  const int v = blockIdx.x * kBlock + threadIdx.x;
  if (v >= n_e) return;
  const int lin = elem_lin[v];
  const int x = lin % N, y = (lin / N) % N, z = lin / (N * N);
  const bool head = run_head(elem_lin, v, lin, x);
  const bool inner = x > 0 && x < N - 1;
  if (x == N - 1) {  // the start of its own row
    const int w = elem_map[lin - x];
    if (w >= 0 && w != v) cc_union(parent, v, w);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int dy = r == 0 ? 1 : r - 2, dz = r == 0 ? 0 : 1;
    const int row = N * (wrapm(y + dy, N) + N * wrapm(z + dz, N));
    const int mid = elem_map[x + row];
    if (head && mid >= 0 && mid != v) cc_union(parent, v, mid);
    if (x == 0 || (head && mid < 0)) {
      const int w = elem_map[wrapm(x - 1, N) + row];
      if (w >= 0 && w != v) cc_union(parent, v, w);
    }
    if (!inner || mid < 0) {
      const int w = elem_map[wrapm(x + 1, N) + row];
      if (w >= 0 && w != v) cc_union(parent, v, w);
    }
  }
}

__global__ void k_cc_count(const int* __restrict__ parent, int n_e, int* __restrict__ count) {
  const int v = blockIdx.x * kBlock + threadIdx.x;
  const bool root = v < n_e && parent[v] == v;
  const unsigned long long m = __ballot(root);
  if ((threadIdx.x & 63) == 0 && m) atomicAdd(count, __popcll(m));
}

// ---------------------------------------------------------------- Galerkin operators
// Local Galerkin projection (Sec. 4.6): K_E = sum_{active children c} P_c^T K_c P_c,
// P_c = Ps_c (8x8 trilinear weights) (x) I_D.  One block per coarse element.  Bound by
// the two 8-term products of every entry (LDS), 8 times per element.
template <int D>
__global__ __launch_bounds__(kBlock) void k_galerkin(const int* __restrict__ elem_lin_c, int Nc,
                                                     const int* __restrict__ emap_f,
                                                     const double* __restrict__ Ksrc,
                                                     const double* __restrict__ Ps, double* __restrict__ out64,
                                                     float* __restrict__ out32) {
  constexpr int M = 8 * D;
  __shared__ double Kc[M * M];
  __shared__ double T1[M * M];
  __shared__ double acc[M * M];
  __shared__ double P[64];
  const int e = blockIdx.x;
  const int Nf = 2 * Nc;
  const int lin = elem_lin_c[e];
  const int X = lin % Nc, Y = (lin / Nc) % Nc, Z = lin / (Nc * Nc);
  for (int t = threadIdx.x; t < M * M; t += kBlock) acc[t] = 0.0;
  for (int c = 0; c < 8; ++c) {
    const int fx = 2 * X + (c & 1), fy = 2 * Y + ((c >> 1) & 1), fz = 2 * Z + ((c >> 2) & 1);
    const int fid = emap_f[fx + Nf * (fy + Nf * fz)];
    if (fid < 0) continue;  // uniform across the block
    const double* src = Ksrc + (size_t)fid * M * M;
    __syncthreads();
    for (int t = threadIdx.x; t < M * M; t += kBlock) Kc[t] = src[t];
    if (threadIdx.x < 64) P[threadIdx.x] = Ps[c * 64 + threadIdx.x];
    __syncthreads();
    // T1[(m,i),(p,j)] = sum_n Kc[(m,i),(n,j)] P[n][p]
    for (int t = threadIdx.x; t < M * M; t += kBlock) {
      const int row = t / M, col = t % M;
      const int p = col / D, j = col % D;
      double s = 0.0;
#pragma unroll
      for (int n = 0; n < 8; ++n) s += Kc[row * M + n * D + j] * P[n * 8 + p];
      T1[t] = s;
    }
    __syncthreads();
    // acc[(o,i),(p,j)] += sum_m P[m][o] T1[(m,i),(p,j)]
    for (int t = threadIdx.x; t < M * M; t += kBlock) {
      const int row = t / M, col = t % M;
      const int o = row / D, i = row % D;
      double s = 0.0;
#pragma unroll
      for (int m = 0; m < 8; ++m) s += P[m * 8 + o] * T1[(m * D + i) * M + col];
      acc[t] += s;
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < M * M; t += kBlock) {
    out64[(size_t)e * M * M + t] = acc[t];
    out32[(size_t)e * M * M + t] = (float)acc[t];
  }
}

// Where the children's matrices come from a table of nm (the 256 mask matrices of level 2;
// the voxel's K_e, nm = 1), every term P_c^T K P_c is one of 8 nm: they are formed once
// (k_galerkin_terms, the arithmetic of k_galerkin) and an element is the sum of its
// children's terms, in the same order, each times the child's stiffness scale in a
// density hierarchy.  Bound by reading the terms (37 KB an element, from L2) and writing
// the matrices.  Level 3 of a 512^3 cell (581 k elements): 11.5 ms element by element,
// 2.4 ms so.
template <int D>
__global__ __launch_bounds__(kBlock) void k_galerkin_terms(int nm, const double* __restrict__ Ksrc,
                                                           const double* __restrict__ Ps, double* __restrict__ terms) {
  constexpr int M = 8 * D;
  __shared__ double Kc[M * M];
  __shared__ double T1[M * M];
  __shared__ double P[64];
  const int m = blockIdx.x, c = blockIdx.y;
  for (int t = threadIdx.x; t < M * M; t += kBlock) Kc[t] = Ksrc[(size_t)m * M * M + t];
  if (threadIdx.x < 64) P[threadIdx.x] = Ps[c * 64 + threadIdx.x];
  __syncthreads();
  for (int t = threadIdx.x; t < M * M; t += kBlock) {
    const int row = t / M, col = t % M;
    const int p = col / D, j = col % D;
    double s = 0.0;
#pragma unroll
    for (int n = 0; n < 8; ++n) s += Kc[row * M + n * D + j] * P[n * 8 + p];
    T1[t] = s;
  }
  __syncthreads();
  for (int t = threadIdx.x; t < M * M; t += kBlock) {
    const int row = t / M, col = t % M;
    const int o = row / D, i = row % D;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) s += P[k * 8 + o] * T1[(k * D + i) * M + col];
    terms[((size_t)c * nm + m) * M * M + t] = s;
  }
}

template <int D>
__global__ __launch_bounds__(D == 3 ? 288 : 256) void k_galerkin_sum(const int* __restrict__ elem_lin_c, int n_e, int Nc,
                                                                     const int* __restrict__ emap_f,
                                                                     const uint8_t* __restrict__ mask_f, int nm,
                                                                     const double* __restrict__ terms,
                                                                     const double* __restrict__ fscale,
                                                                     double* __restrict__ out64,
                                                                     float* __restrict__ out32) {
  constexpr int M = 8 * D, H = M * M / 2;  // two entries per thread
  constexpr int EPB = D == 3 ? 1 : 8;      // elements per workgroup
  const int e = blockIdx.x * EPB + (int)threadIdx.x / H;
  if (e >= n_e) return;
  const int t = (int)threadIdx.x % H;
  const int Nf = 2 * Nc;
  const int lin = elem_lin_c[e];
  const int X = lin % Nc, Y = (lin / Nc) % Nc, Z = lin / (Nc * Nc);
  int fid[8], row[8];
#pragma unroll
  for (int c = 0; c < 8; ++c)
    fid[c] = emap_f[2 * X + (c & 1) + Nf * (2 * Y + ((c >> 1) & 1) + Nf * (2 * Z + (c >> 2)))];
#pragma unroll
  for (int c = 0; c < 8; ++c) row[c] = c * nm + (nm > 1 && fid[c] >= 0 ? mask_f[fid[c]] : 0);
  double a0 = 0.0, a1 = 0.0;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    if (fid[c] < 0) continue;
    // pairs of values, for which the allocator's memory need not be aligned: one wide access
    // each all the same
    const double* v = terms + (size_t)row[c] * M * M + 2 * t;
    const double v0 = v[0], v1 = v[1];
    if (fscale) {
      const double sc = fscale[fid[c]];
      a0 = fma(sc, v0, a0);
      a1 = fma(sc, v1, a1);
    } else {
      a0 += v0;
      a1 += v1;
    }
  }
  const size_t at = (size_t)e * M * M + 2 * t;
  out64[at] = a0;
  out64[at + 1] = a1;
  out32[at] = (float)a0;
  out32[at + 1] = (float)a1;
}

inline unsigned blocks_for(size_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

size_t scan_scratch_ints(size_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

int64_t scan_count(const int* flags, size_t n, int* scratch, int* d_total, hipStream_t s) {
  const unsigned nb = (unsigned)((n + kScanTile - 1) / kScanTile);
  hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kBlock), 0, s, flags, n, scratch);
  GMT_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kBlock), 0, s, scratch, (int)nb, d_total);
  GMT_LAUNCH_CHECK();
  int total = 0;
  GMT_HIP(hipMemcpyAsync(&total, d_total, sizeof(int), hipMemcpyDeviceToHost, s));
  GMT_HIP(hipStreamSynchronize(s));
  return total;
}

void scan_write(const int* flags, size_t n, int* map_out, int* lin_out, const int* scratch, hipStream_t s) {
  const unsigned nb = (unsigned)((n + kScanTile - 1) / kScanTile);
  hipLaunchKernelGGL(k_scan_write, dim3(nb), dim3(kBlock), 0, s, flags, n, scratch, map_out, lin_out);
  GMT_LAUNCH_CHECK();
}

void launch_stage_tables(const int* interior, int n_int, const int* node_lin, const int* node_map, int N, int nb,
                         int pass, const int* blk, int n_blk, int* cnt, const long long* off, int* ids, uint16_t* slot,
                         int* route, hipStream_t s) {
  const unsigned grid = pass == 0 ? (unsigned)((n_int + nb - 1) / nb) : (unsigned)n_blk;
  if (!n_int || !grid) return;
  int max_words = kStageBits / 32;
  // GMT_STAGE_WORDS=<k> lowers the bitmap's size (tests of the sorted groups)
  if (const char* e = std::getenv("GMT_STAGE_WORDS"))
    if (*e && std::atoi(e) >= 0) max_words = std::min(max_words, std::atoi(e));
  if (nb == 512) {
    hipLaunchKernelGGL(k_stage_tables<512>, dim3(grid), dim3(512), 0, s, interior, n_int, node_lin, node_map, N, pass,
                       blk, cnt, off, ids, slot, route, max_words);
    hipLaunchKernelGGL(k_stage_sort<512>, dim3(grid), dim3(512), 0, s, interior, n_int, node_lin, node_map, N, pass,
                       blk, cnt, off, ids, slot, route);
  } else {
    hipLaunchKernelGGL(k_stage_tables<256>, dim3(grid), dim3(256), 0, s, interior, n_int, node_lin, node_map, N, pass,
                       blk, cnt, off, ids, slot, route, max_words);
    hipLaunchKernelGGL(k_stage_sort<256>, dim3(grid), dim3(256), 0, s, interior, n_int, node_lin, node_map, N, pass,
                       blk, cnt, off, ids, slot, route);
  }
  GMT_LAUNCH_CHECK();
}

size_t galerkin_term_doubles(int src_kind, int D) {
  return src_kind == KIND_PERELEM ? 0 : (size_t)8 * (src_kind == KIND_TABLE ? 256 : 1) * 64 * D * D;
}

void launch_galerkin(const int* elem_lin_c, int n_e_c, int Nc, const int* emap_f, const uint8_t* cmask_f,
                     const double* Ksrc, int src_kind, int D, const double* Ps, const double* fscale, double* terms,
                     double* out64, float* out32, hipStream_t s) {
  if (!n_e_c) return;
#define GMT_GALERKIN(DD)                                                                                             \
  if (D == DD) {                                                                                                     \
    if (src_kind == KIND_PERELEM) {                                                                                  \
      hipLaunchKernelGGL(k_galerkin<DD>, dim3(n_e_c), dim3(kBlock), 0, s, elem_lin_c, Nc, emap_f, Ksrc, Ps, out64,    \
                         out32);                                                                                     \
    } else {                                                                                                         \
      const int nm = src_kind == KIND_TABLE ? 256 : 1, epb = DD == 3 ? 1 : 8;                                        \
      hipLaunchKernelGGL(k_galerkin_terms<DD>, dim3(nm, 8), dim3(kBlock), 0, s, nm, Ksrc, Ps, terms);                 \
      hipLaunchKernelGGL(k_galerkin_sum<DD>, dim3((unsigned)((n_e_c + epb - 1) / epb)), dim3(DD == 3 ? 288 : 256), 0, \
                         s, elem_lin_c, n_e_c, Nc, emap_f, cmask_f, nm, terms, fscale, out64, out32);                \
    }                                                                                                                \
  }
  GMT_GALERKIN(3)
  GMT_GALERKIN(1)
#undef GMT_GALERKIN
  GMT_LAUNCH_CHECK();
}

int count_components(const int* elem_lin, int n_e, const int* elem_map, int N, int* parent, int* d_count,
                     hipStream_t s) {
  if (n_e <= 0) return 0;
  const unsigned g = blocks_for(n_e);
  hipLaunchKernelGGL(k_cc_init, dim3(g), dim3(kBlock), 0, s, elem_lin, n_e, N, parent, d_count);
  GMT_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_cc_hook, dim3(g), dim3(kBlock), 0, s, elem_lin, n_e, elem_map, N, parent);
  GMT_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_cc_count, dim3(g), dim3(kBlock), 0, s, parent, n_e, d_count);
  GMT_LAUNCH_CHECK();
  int h = 0;
  GMT_HIP(hipMemcpyAsync(&h, d_count, sizeof(int), hipMemcpyDeviceToHost, s));
  GMT_HIP(hipStreamSynchronize(s));
  return h;
}

}  // namespace gmt
