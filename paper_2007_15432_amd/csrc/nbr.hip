// nbr.hip -- neighbour lists as CSR (Section 2.3), neighbour-cluster indices
// and the cluster CSR.
//
// Neighbour pairs (i, j) in original indices arrive unordered from the force
// phase.  CSR: per-row counts, exclusive scan, scatter, then each row is
// sorted ascending (rows are short: <n_b> << 1 in the regime the method is
// meant for).  The result does not depend on the arrival order.
//
// Cluster index (Section 2.3 steps i-iii: the fixed point of "take the
// minimum index over yourself and your neighbours") is the minimum index of
// the particle's connected component.  Computed with a lock-free union-find
// that always hooks the larger root under the smaller one, so every
// component's root is its minimum index; the kernels that find the pairs join
// them as they report them (uf_union), so the parents are complete when the
// evaluation is.
//
// Cluster CSR by counting: members per label, a scan of (cluster, size) over
// the labels, members into their cluster's range, ranges sorted.  Most
// particles are clusters of their own and every cluster starts with its label's
// particle, so only the others take a slot and only clusters of three and more
// need sorting: five short launches.  With the bucket lists of the hard part, a
// radix sort of (label, index) against this: 65,536 particles 96 -> 34 us, 2^20
// 190 -> 75 us.  Where many members share a label (a percolated disk, a caller's
// classes), ordering the members is left to the radix sort after all, whose
// cost does not depend on the cluster sizes (see CL_WORK).
#include <algorithm>

#include "p3t_internal.h"

namespace p3t {

static inline unsigned g1d(int64_t n, int64_t cap = 65536) {
  int64_t b = (n + 255) / 256;
  return (unsigned)(b < 1 ? 1 : (b > cap ? cap : b));
}

// ------------------------------------------------------------------ scan over items in two launches
// What an index contributes: its cluster (bit 32) and members, or its row's
// length.
//   CL_ROOT: label[i] == i marks a cluster of 1 + cnt[i] members
//   CL_ANY:  cnt[i] > 0 members carry the label i
//   CL_ROWS: cnt[i] entries in row i
constexpr int CL_ROOT = 0, CL_ANY = 1, CL_ROWS = 2;
constexpr int CS_T = 256, CS_CHUNK = 4 * CS_T, CS_BLOCKS = 1024;
// words behind c->cl_nc: a label was out of range, members are not in order
constexpr int CL_BAD = 1, CL_UNSORTED = 2;
// Members ascending in every cluster (k_cl_sort): up to CL_SMALL members by the
// cluster's thread in place, larger ones one after another by the wavefront
// that holds their thread, which ranks m members in about m + m^2 / 64 steps.
// Where a wavefront's clusters add up to more than CL_WORK steps, or a cluster
// exceeds CL_LARGE members, the members are sorted by label and index instead
// (members_sorted).  CL_WORK is some ten microseconds, a sixth of that sort's
// launches.  Without the line, 2^20 particles in 512 classes took 212 ms (the
// sort alone: see members_sorted) and 65,536 in clusters of 128 took 1.0 ms.
constexpr int CL_SMALL = 12, CL_WORK = 2048;
constexpr uint32_t CL_LARGE = 320;  // m + m^2 / 64 <= CL_WORK

// The counter of label or row i.  A caller's labels (CL_ANY) are often small
// neighbouring numbers, and atomics on one cache line queue up like those on one
// counter: their counters are dealt to parts of cnt, few of them where the
// labels of a wavefront's particles may as well be neighbours and their atomics
// share a line.  2^20 particles in 512 classes 0 to 511, counting launch: 273 us
// in one part, 165 in 32, 62 in 256 (16 with the tiles below).
constexpr int64_t CC_WAVE_MAX = 1 << 17;  // up to here k_cl_count, above it k_cl_count_tile
constexpr int CNT_PARTS = 256;            // at most

template <int KIND>
__device__ __forceinline__ int64_t counter(int64_t i, int64_t n) {
  if (KIND != CL_ANY) return i;
  const int lg = n <= CC_WAVE_MAX ? 4 : 8;
  return (i & ((1 << lg) - 1)) * ((n + (1 << lg) - 1) >> lg) + (i >> lg);
}

template <int KIND>
__device__ __forceinline__ uint64_t item(const int32_t *__restrict__ label, const int32_t *__restrict__ cnt, int64_t i,
                                         int64_t n) {
  const uint64_t c = (uint32_t)cnt[counter<KIND>(i, n)];
  if (KIND == CL_ROOT) return label[i] == (int32_t)i ? (1ull << 32) + 1ull + c : 0ull;
  if (KIND == CL_ANY) return c > 0 ? (1ull << 32) + c : 0ull;
  return c;
}

// indices per workgroup, a multiple of CS_CHUNK, for at most CS_BLOCKS workgroups
static int64_t scan_tile(int64_t n) {
  const int64_t chunks = (n + CS_CHUNK - 1) / CS_CHUNK;
  return CS_CHUNK * ((chunks + CS_BLOCKS - 1) / CS_BLOCKS);
}

__device__ __forceinline__ uint64_t block_sum(uint64_t v, uint64_t *ws) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & (WAVE - 1)) == 0) ws[threadIdx.x / WAVE] = v;
  __syncthreads();
  uint64_t r = 0;
#pragma unroll
  for (int q = 0; q < CS_T / WAVE; ++q) r += ws[q];
  return r;
}

// (also clears the flag that the launches behind it set, nullable)
template <int KIND>
__global__ __launch_bounds__(CS_T) void k_item_sums(int64_t n, int64_t tile, const int32_t *__restrict__ label,
                                                    const int32_t *__restrict__ cnt, uint64_t *__restrict__ sums,
                                                    int64_t *__restrict__ unsorted) {
  __shared__ uint64_t ws[CS_T / WAVE];
  if (unsorted && blockIdx.x == 0 && threadIdx.x == 0) *unsorted = 0;
  const int64_t a = (int64_t)blockIdx.x * tile, b = a + tile < n ? a + tile : n;
  uint64_t s = 0;
  for (int64_t i = a + threadIdx.x; i < b; i += CS_T) s += item<KIND>(label, cnt, i, n);
  s = block_sum(s, ws);
  if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

// Every workgroup adds the sums before its own itself, then scans its tile.
// Clusters: their first slot into start[] (by label) and cl_ptr[] (by
// cluster), CL_ROOT also the root into its slot; cnt is left cleared; the
// cluster count goes to *out64, clear[0, n_clear) is cleared for the launch
// that buckets the clusters, and a cluster above CL_LARGE members sets
// *unsorted.  Rows: row_ptr.
template <int KIND>
__global__ __launch_bounds__(CS_T) void k_item_place(int64_t n, int64_t tile, const int32_t *__restrict__ label,
                                                     int32_t *__restrict__ cnt, const uint64_t *__restrict__ sums,
                                                     int32_t *__restrict__ start, int32_t *__restrict__ cl_ptr,
                                                     int32_t *__restrict__ members, int64_t *__restrict__ out64,
                                                     int64_t *__restrict__ unsorted, int32_t *__restrict__ clear,
                                                     int n_clear) {
  __shared__ uint64_t ws[CS_T / WAVE];
  const int t = threadIdx.x, lane = t & (WAVE - 1), w = t / WAVE;
  uint64_t run = 0;
  for (int q = t; q < (int)blockIdx.x; q += CS_T) run += sums[q];
  run = block_sum(run, ws);
  if (blockIdx.x == 0 && clear)
    for (int q = t; q < n_clear; q += CS_T) clear[q] = 0;
  const int64_t a = (int64_t)blockIdx.x * tile, b = a + tile < n ? a + tile : n;
  for (int64_t c0 = a; c0 < b; c0 += CS_CHUNK) {
    uint64_t v[4], s = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = c0 + 4 * t + q;
      v[q] = i < b ? item<KIND>(label, cnt, i, n) : 0ull;
      s += v[q];
    }
    uint64_t incl = s;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const uint64_t u = __shfl_up(incl, o, WAVE);
      if (lane >= o) incl += u;
    }
    __syncthreads();
    if (lane == WAVE - 1) ws[w] = incl;
    __syncthreads();
    uint64_t at = run + incl - s, all = 0;
#pragma unroll
    for (int q = 0; q < CS_T / WAVE; ++q) {
      at += q < w ? ws[q] : 0ull;
      all += ws[q];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = c0 + 4 * t + q;
      if (i >= b) break;
      if (KIND == CL_ROWS) {
        out64[i] = (int64_t)at;
      } else if (v[q]) {
        const int32_t o = (int32_t)(uint32_t)at;
        start[i] = o;
        cl_ptr[at >> 32] = o;
        if (KIND == CL_ROOT) members[o] = (int32_t)i;
        if ((uint32_t)v[q] > (KIND == CL_ROOT ? 1u : 0u)) cnt[counter<KIND>(i, n)] = 0;
        if ((uint32_t)v[q] > CL_LARGE) *unsorted = 1;
      }
      at += v[q];
    }
    run += all;
  }
  if (blockIdx.x == gridDim.x - 1 && t == 0) {
    if (KIND == CL_ROWS) {
      out64[n] = (int64_t)run;
    } else {
      *out64 = (int64_t)(run >> 32);
      cl_ptr[run >> 32] = (int32_t)(uint32_t)run;
    }
  }
}

template <int KIND>
static void scan_items(p3t_ctx *c, int64_t n, const int32_t *label, int32_t *cnt, int32_t *cl_ptr, int32_t *members,
                       int64_t *out64, int32_t *clear, int n_clear) {
  const int64_t tile = scan_tile(n);
  const unsigned g = (unsigned)((n + tile - 1) / tile);
  uint64_t *sums = reinterpret_cast<uint64_t *>(c->cl_sums);
  int64_t *unsorted = KIND == CL_ROWS ? nullptr : c->cl_nc + CL_UNSORTED;
  hipLaunchKernelGGL(k_item_sums<KIND>, dim3(g), dim3(CS_T), 0, c->stream, n, tile, label, (const int32_t *)cnt, sums,
                     unsorted);
  hipLaunchKernelGGL(k_item_place<KIND>, dim3(g), dim3(CS_T), 0, c->stream, n, tile, label, cnt, (const uint64_t *)sums,
                     c->cl_start, cl_ptr, members, out64, unsorted, clear, n_clear);
}
int64_t scan_sums_need() { return CS_BLOCKS; }
int64_t label_counters_need(int64_t n_cap) { return n_cap + CNT_PARTS; }

// ------------------------------------------------------------------ neighbour CSR
__global__ void k_pair_count(const int2 *__restrict__ pairs, int64_t np, int32_t *__restrict__ cnt) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += (int64_t)gridDim.x * blockDim.x)
    atomicAdd(&cnt[pairs[p].x], 1);
}

// counts the row's cursor back to zero
__global__ void k_pair_fill(const int2 *__restrict__ pairs, int64_t np, const int64_t *__restrict__ row_ptr,
                            int32_t *__restrict__ cur, int32_t *__restrict__ col) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += (int64_t)gridDim.x * blockDim.x) {
    const int2 e = pairs[p];
    col[row_ptr[e.x] + atomicSub(&cur[e.x], 1) - 1] = e.y;
  }
}

// rows ascending, and the label of every particle (nullable)
__global__ void k_row_sort(int64_t n, const int64_t *__restrict__ row_ptr, int32_t *__restrict__ col, int32_t *uf,
                           int32_t *__restrict__ label) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    if (label) label[i] = uf_find(uf, (int)i);
    const int64_t a = row_ptr[i], b = row_ptr[i + 1];
    for (int64_t k = a + 1; k < b; ++k) {
      const int32_t v = col[k];
      int64_t q = k - 1;
      while (q >= a && col[q] > v) {
        col[q + 1] = col[q];
        --q;
      }
      col[q + 1] = v;
    }
  }
}

hipError_t neighbour_csr(p3t_ctx *c, int64_t n, int64_t np, int64_t *row_ptr, int32_t *col, int32_t *label) {
  hipStream_t s = c->stream;
  if (np > 0) hipLaunchKernelGGL(k_pair_count, dim3(g1d(np)), dim3(256), 0, s, c->pairs, np, c->row_cnt);
  scan_items<CL_ROWS>(c, n, nullptr, c->row_cnt, nullptr, nullptr, row_ptr, nullptr, 0);
  if (np > 0)
    hipLaunchKernelGGL(k_pair_fill, dim3(g1d(np)), dim3(256), 0, s, c->pairs, np, (const int64_t *)row_ptr, c->row_cnt,
                       col);
  hipLaunchKernelGGL(k_row_sort, dim3(g1d(n)), dim3(256), 0, s, n, (const int64_t *)row_ptr, col, c->uf_parent, label);
  return hipGetLastError();
}

// ------------------------------------------------------------------ cluster CSR
// The label of every particle and its slot among those that share it (in any
// order): from the union-find (CL_ROOT, every member but the root takes a slot
// behind it) or the caller's labels (CL_ANY, one outside [0, n) is reported).
// The atomics of one label queue up, 12 ns each, so they are taken for several
// members at once.  Counting launch, one atomic per member against this: 2^20
// particles of one label 12 ms -> 14 us, of distinct labels 46 -> 47.

// label of particle i, -1 where no slot is wanted
template <int KIND>
__device__ __forceinline__ int slot_label(int64_t i, int64_t n, int32_t *uf, int32_t *__restrict__ label,
                                          int64_t *__restrict__ bad) {
  if (i >= n) return -1;
  if (KIND == CL_ROOT) {
    const int r = uf_find(uf, (int)i);
    label[i] = r;
    return r != (int)i ? r : -1;
  }
  const int l = label[i];
  if ((uint32_t)l < (uint64_t)n) return l;
  *bad = 1;
  return -1;
}

// One atomic per label that the wavefront's first lanes share; as soon as the
// first lane left is the only one with its label, the others go one by one:
// many labels, which do not queue up, or few and most of them counted.
template <int KIND>
__global__ __launch_bounds__(CS_T) void k_cl_count(int64_t n, int32_t *uf, int32_t *__restrict__ label,
                                                   int32_t *__restrict__ cnt, int32_t *__restrict__ slot,
                                                   int64_t *__restrict__ bad) {
  const int64_t i = (int64_t)blockIdx.x * CS_T + threadIdx.x;
  const int l = slot_label<KIND>(i, n, uf, label, bad), lane = lane_id();
  int s = 0;
  unsigned long long left = __ballot(l >= 0);
  while (left != 0ull) {  // uniform
    const int lead = __ffsll((long long)left) - 1;
    const unsigned long long same = __ballot(l == uniform_lane(l, lead)) & left;
    const int m = (int)__popcll(same);
    if (m == 1) break;
    int base = 0;
    if (lane == lead) base = atomicAdd(&cnt[counter<KIND>(l, n)], m);
    base = uniform_lane(base, lead);
    if ((same >> lane) & 1ull) s = base + popc_below(same);
    left &= ~same;
  }
  if ((left >> lane) & 1ull) s = atomicAdd(&cnt[counter<KIND>(l, n)], 1);
  if (l >= 0) slot[i] = (KIND == CL_ROOT ? 1 : 0) + s;
}

// The same by tiles of 4096, whose labels a workgroup counts in an LDS table
// (at most half full): 1.2 launches of the former for distinct labels of 2^20
// particles, but 64 labels do not queue up either.
constexpr int CT_T = 1024, CT_I = 4, CT_SLOTS = 2 * CT_T * CT_I;

template <int KIND>
__global__ __launch_bounds__(CT_T) void k_cl_count_tile(int64_t n, int32_t *uf, int32_t *__restrict__ label,
                                                        int32_t *__restrict__ cnt, int32_t *__restrict__ slot,
                                                        int64_t *__restrict__ bad) {
  __shared__ int key[CT_SLOTS], val[CT_SLOTS];
  const int t = threadIdx.x;
  for (int64_t base = (int64_t)blockIdx.x * (CT_T * CT_I); base < n;
       base += (int64_t)gridDim.x * (CT_T * CT_I)) {  // uniform
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2 * CT_I; ++q) {
      key[q * CT_T + t] = -1;
      val[q * CT_T + t] = 0;
    }
    int l[CT_I];
#pragma unroll
    for (int q = 0; q < CT_I; ++q) l[q] = slot_label<KIND>(base + q * CT_T + t, n, uf, label, bad);
    __syncthreads();
    int at[CT_I], rank[CT_I];  // table entry and place among the tile's members
#pragma unroll
    for (int q = 0; q < CT_I; ++q) {
      if (l[q] < 0) continue;
      unsigned h = ((unsigned)l[q] * 2654435761u) / (0xffffffffu / CT_SLOTS + 1u);
      for (;;) {
        const int k = atomicCAS(&key[h], -1, l[q]);
        if (k == -1 || k == l[q]) break;
        h = (h + 1) & (CT_SLOTS - 1);
      }
      at[q] = (int)h;
      rank[q] = atomicAdd(&val[h], 1);
    }
    __syncthreads();
    int k[2 * CT_I], v[2 * CT_I];
#pragma unroll
    for (int q = 0; q < 2 * CT_I; ++q) {
      k[q] = key[q * CT_T + t];
      v[q] = val[q * CT_T + t];
    }
    // (all of them issued before the first is waited for)
#pragma unroll
    for (int q = 0; q < 2 * CT_I; ++q)
      if (k[q] >= 0) v[q] = atomicAdd(&cnt[counter<KIND>(k[q], n)], v[q]);
#pragma unroll
    for (int q = 0; q < 2 * CT_I; ++q) val[q * CT_T + t] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < CT_I; ++q)
      if (l[q] >= 0) slot[base + q * CT_T + t] = (KIND == CL_ROOT ? 1 : 0) + val[at[q]] + rank[q];
  }
}

template <int KIND>
static void count_labels(p3t_ctx *c, int64_t n, int32_t *label) {
  auto go = [&](auto kernel, int64_t g, int t) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)std::min<int64_t>(65536, g)), dim3(t), 0, c->stream, n, c->uf_parent, label,
                       c->cl_cnt, c->cl_slot, c->cl_nc + CL_BAD);
  };
  if (n <= CC_WAVE_MAX)
    go(k_cl_count<KIND>, (n + CS_T - 1) / CS_T, CS_T);
  else
    go(k_cl_count_tile<KIND>, (n + CT_T * CT_I - 1) / (CT_T * CT_I), CT_T);
}

template <int KIND>
__global__ void k_cl_fill(int64_t n, const int32_t *__restrict__ label, const int32_t *__restrict__ start,
                          const int32_t *__restrict__ slot, const int64_t *__restrict__ unsorted,
                          int32_t *__restrict__ members) {
  // (the hard part reads its members before they are in order: CL_ROOT fills them in any case)
  if (KIND == CL_ANY && *unsorted) return;  // uniform: sorted from the labels instead
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int l = label[i];
    if (KIND == CL_ROOT ? l != (int)i : (uint32_t)l < (uint64_t)n) members[start[l] + slot[i]] = (int32_t)i;
  }
}

// members ascending in every cluster (see CL_WORK)
__global__ __launch_bounds__(CS_T) void k_cl_sort(int64_t n, const int64_t *__restrict__ nc_dev,
                                                  const int32_t *__restrict__ cl_ptr, int64_t *unsorted,
                                                  int32_t *__restrict__ members) {
  __shared__ int32_t buf[CS_T / WAVE][CL_LARGE];
  const int lane = threadIdx.x & (WAVE - 1), w = uniform_first((int)threadIdx.x / WAVE);
  // (clusters above CL_LARGE set the flag before this launch)
  if (uniform_first((int)__hip_atomic_load(unsorted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) return;
  // consecutive clusters in the lanes; where they hold more than CL_SMALL
  // members on average, dealt to all wavefronts instead
  const int64_t nc = *nc_dev, nw = (int64_t)gridDim.x * (CS_T / WAVE), gw = (int64_t)blockIdx.x * (CS_T / WAVE) + w;
  const int64_t c = nc * CL_SMALL <= n ? gw + lane * nw : gw * WAVE + lane;
  const int a = c < nc ? cl_ptr[c] : 0, m = c < nc ? cl_ptr[c + 1] - a : 0;
  if (m <= CL_SMALL) {
    for (int k = a + 1; k < a + m; ++k) {
      const int32_t v = members[k];
      int q = k - 1;
      while (q >= a && members[q] > v) {
        members[q + 1] = members[q];
        --q;
      }
      members[q + 1] = v;
    }
  }
  unsigned long long large = __ballot(m > CL_SMALL && m <= (int)CL_LARGE);
  if (large == 0ull) return;  // uniform
  if (wave_sum(m > CL_SMALL ? m + m * m / WAVE : 0) > CL_WORK) {
    if (lane == 0) *unsorted = 1;
    return;
  }
  while (large != 0ull) {
    const int l = __ffsll((long long)large) - 1;
    large &= large - 1ull;
    const int a0 = uniform_lane(a, l), k0 = uniform_lane(m, l);
    for (int k = lane; k < k0; k += WAVE) buf[w][k] = members[a0 + k];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int k = lane; k < k0; k += WAVE) {
      const int32_t v = buf[w][k];
      int r = 0;
#pragma unroll 8
      for (int q = 0; q < k0; ++q) r += buf[w][q] < v ? 1 : 0;
      members[a0 + r] = v;
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// The clusters of the last evaluation: labels, cluster CSR and the cluster
// count (c->cl_nc, on the device).  clear: words to clear on the way (the
// bucket words).  Where c->cl_nc[CL_UNSORTED] ends up set, which the bucket
// words report as HERM_BC_UNSORTED, the members are not in order:
// members_sorted.
hipError_t clusters_pairs(p3t_ctx *c, int64_t n, int32_t *label, int32_t *cl_ptr, int32_t *cl_members,
                          int32_t *clear, int n_clear) {
  hipStream_t s = c->stream;
  count_labels<CL_ROOT>(c, n, label);
  scan_items<CL_ROOT>(c, n, label, c->cl_cnt, cl_ptr, cl_members, c->cl_nc, clear, n_clear);
  hipLaunchKernelGGL(k_cl_fill<CL_ROOT>, dim3(g1d(n)), dim3(256), 0, s, n, (const int32_t *)label,
                     (const int32_t *)c->cl_start, (const int32_t *)c->cl_slot,
                     (const int64_t *)c->cl_nc + CL_UNSORTED, cl_members);
  hipLaunchKernelGGL(k_cl_sort, dim3((unsigned)((n + CS_T - 1) / CS_T)), dim3(CS_T), 0, s, n,
                     (const int64_t *)c->cl_nc, (const int32_t *)cl_ptr, c->cl_nc + CL_UNSORTED, cl_members);
  return hipGetLastError();
}

// ------------------------------------------------------------------ caller's labels
__global__ void k_cl_keys(int64_t n, const int32_t *__restrict__ label, uint64_t *__restrict__ key) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    key[i] = ((uint64_t)(uint32_t)label[i] << 32) | (uint64_t)(uint32_t)i;
}

__global__ void k_cl_flags(int64_t n, const uint64_t *__restrict__ key, int32_t *__restrict__ members,
                           int32_t *__restrict__ flag) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
    members[k] = (int32_t)(key[k] & 0xffffffffull);
    flag[k] = (k == 0 || (key[k] >> 32) != (key[k - 1] >> 32)) ? 1 : 0;
  }
}

__global__ void k_cl_ptr(int64_t n, const int32_t *__restrict__ flag, const int64_t *__restrict__ pos,
                         int32_t *__restrict__ cl_ptr) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
    if (flag[k]) cl_ptr[pos[k]] = (int32_t)k;
  if (blockIdx.x == 0 && threadIdx.x == 0) cl_ptr[pos[n]] = (int32_t)n;
}

// sorted keys (label, index) to members
__global__ void k_cl_members(int64_t n, const uint64_t *__restrict__ key, int32_t *__restrict__ members) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
    members[k] = (int32_t)(key[k] & 0xffffffffull);
}

// (label, index) sorted by the low bits that labels of n particles need, in
// c->cl_keys or c->cl_keys_alt
static hipError_t sort_labels(p3t_ctx *c, int64_t n, const int32_t *label, uint64_t **sorted) {
  hipStream_t s = c->stream;
  hipLaunchKernelGGL(k_cl_keys, dim3(g1d(n)), dim3(256), 0, s, n, label, c->cl_keys);
  int bits = 1;
  while ((int64_t(1) << bits) < n) ++bits;
  // keys start ascending in the particle index, so a stable sort on the
  // label bits alone orders by (label, index)
  uint64_t *k = c->cl_keys, *ka = c->cl_keys_alt;
  int32_t *v = nullptr, *va = nullptr;
  const hipError_t e = radix_sort_pairs(k, v, ka, va, n, 32, 32 + bits, c->radix_hist, c->radix_hist_cap, false, s);
  *sorted = k;
  return e;
}

hipError_t members_sorted(p3t_ctx *c, int64_t n, const int32_t *label, int32_t *cl_members) {
  uint64_t *k = nullptr;
  const hipError_t e = sort_labels(c, n, label, &k);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_cl_members, dim3(g1d(n)), dim3(256), 0, c->stream, n, (const uint64_t *)k, cl_members);
  return hipGetLastError();
}

// Labels outside [0, n) cannot index a count: sorted, neighbours of different
// label split, as such labels were always treated.
static hipError_t clusters_sorted(p3t_ctx *c, int64_t n, const int32_t *label, int32_t *cl_ptr, int32_t *cl_members,
                                  int64_t *n_clusters) {
  hipStream_t s = c->stream;
  hipError_t e;
  uint64_t *k = nullptr;
  if ((e = sort_labels(c, n, label, &k)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_cl_flags, dim3(g1d(n)), dim3(256), 0, s, n, k, cl_members, c->cl_slot);
  if ((e = scan_i32_to_i64(c->cl_slot, c->node_scan, n, c->scan_tmp, c->scan_tmp_cap, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_cl_ptr, dim3(g1d(n)), dim3(256), 0, s, n, c->cl_slot, c->node_scan, cl_ptr);
  int64_t nc = 0;
  if ((e = hipMemcpyAsync(&nc, c->node_scan + n, sizeof(int64_t), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
  *n_clusters = nc;
  return hipSuccess;
}

hipError_t clusters_csr(p3t_ctx *c, int64_t n, const int32_t *label, int32_t *cl_ptr, int32_t *cl_members,
                        int64_t *n_clusters) {
  hipStream_t s = c->stream;
  hipError_t e;
  count_labels<CL_ANY>(c, n, const_cast<int32_t *>(label));  // (read only)
  scan_items<CL_ANY>(c, n, nullptr, c->cl_cnt, cl_ptr, cl_members, c->cl_nc, nullptr, 0);
  hipLaunchKernelGGL(k_cl_fill<CL_ANY>, dim3(g1d(n)), dim3(256), 0, s, n, label, (const int32_t *)c->cl_start,
                     (const int32_t *)c->cl_slot, (const int64_t *)c->cl_nc + CL_UNSORTED, cl_members);
  hipLaunchKernelGGL(k_cl_sort, dim3((unsigned)((n + CS_T - 1) / CS_T)), dim3(CS_T), 0, s, n,
                     (const int64_t *)c->cl_nc, (const int32_t *)cl_ptr, c->cl_nc + CL_UNSORTED, cl_members);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  int64_t *h = c->host_words;
  if ((e = hipMemcpyAsync(h, c->cl_nc, 3 * sizeof(int64_t), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
  *n_clusters = h[0];
  if (h[CL_BAD]) {
    if ((e = fill_i32(reinterpret_cast<int32_t *>(c->cl_nc + CL_BAD), 0, 2, s)) != hipSuccess) return e;
    return clusters_sorted(c, n, label, cl_ptr, cl_members, n_clusters);
  }
  if (!h[CL_UNSORTED]) return hipSuccess;
  if ((e = members_sorted(c, n, label, cl_members)) != hipSuccess) return e;
  return hipStreamSynchronize(s);
}

}  // namespace p3t
