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
// particle, so only the others take an atomic and only clusters of three and
// more need sorting: five short launches, where a radix sort of (label, index)
// took two or three passes of three launches, a flag pass and a scan.  With the
// bucket lists of the hard part: 65,536 particles 96 -> 34 us, 2^20 190 ->
// 75 us; neighbour lists and clusters of 65,536 particles 208 -> 82 us a call.
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

template <int KIND>
__device__ __forceinline__ uint64_t item(const int32_t *__restrict__ label, const int32_t *__restrict__ cnt, int64_t i) {
  const uint64_t c = (uint32_t)cnt[i];
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

template <int KIND>
__global__ __launch_bounds__(CS_T) void k_item_sums(int64_t n, int64_t tile, const int32_t *__restrict__ label,
                                                    const int32_t *__restrict__ cnt, uint64_t *__restrict__ sums) {
  __shared__ uint64_t ws[CS_T / WAVE];
  const int64_t a = (int64_t)blockIdx.x * tile, b = a + tile < n ? a + tile : n;
  uint64_t s = 0;
  for (int64_t i = a + threadIdx.x; i < b; i += CS_T) s += item<KIND>(label, cnt, i);
  s = block_sum(s, ws);
  if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

// Every workgroup adds the sums before its own itself, then scans its tile.
// Clusters: their first slot into start[] (by label) and cl_ptr[] (by
// cluster), CL_ROOT also the root into its slot; cnt is left cleared; the
// cluster count goes to *nc, and clear[0, n_clear) is cleared for the launch
// that buckets the clusters.  Rows: row_ptr.
template <int KIND>
__global__ __launch_bounds__(CS_T) void k_item_place(int64_t n, int64_t tile, const int32_t *__restrict__ label,
                                                     int32_t *__restrict__ cnt, const uint64_t *__restrict__ sums,
                                                     int32_t *__restrict__ start, int32_t *__restrict__ cl_ptr,
                                                     int32_t *__restrict__ members, int64_t *__restrict__ out64,
                                                     int32_t *__restrict__ clear, int n_clear) {
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
      v[q] = i < b ? item<KIND>(label, cnt, i) : 0ull;
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
        if ((uint32_t)v[q] > (KIND == CL_ROOT ? 1u : 0u)) cnt[i] = 0;
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
  hipLaunchKernelGGL(k_item_sums<KIND>, dim3(g), dim3(CS_T), 0, c->stream, n, tile, label, (const int32_t *)cnt, sums);
  hipLaunchKernelGGL(k_item_place<KIND>, dim3(g), dim3(CS_T), 0, c->stream, n, tile, label, cnt, (const uint64_t *)sums,
                     c->cl_start, cl_ptr, members, out64, clear, n_clear);
}
int64_t scan_sums_need() { return CS_BLOCKS; }

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
// labels from the union-find; every member but the root takes a slot behind it
__global__ void k_cl_labels(int64_t n, int32_t *uf, int32_t *__restrict__ label, int32_t *__restrict__ cnt,
                            int32_t *__restrict__ slot) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int r = uf_find(uf, (int)i);
    label[i] = r;
    if (r != (int)i) slot[i] = 1 + atomicAdd(&cnt[r], 1);
  }
}

// caller's labels: a slot per member; a label outside [0, n) is reported
__global__ void k_cl_count(int64_t n, const int32_t *__restrict__ label, int32_t *__restrict__ cnt,
                           int32_t *__restrict__ slot, int64_t *__restrict__ bad) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int l = label[i];
    if ((uint32_t)l < (uint64_t)n)
      slot[i] = atomicAdd(&cnt[l], 1);
    else
      *bad = 1;
  }
}

template <int KIND>
__global__ void k_cl_fill(int64_t n, const int32_t *__restrict__ label, const int32_t *__restrict__ start,
                          const int32_t *__restrict__ slot, int32_t *__restrict__ members) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int l = label[i];
    if (KIND == CL_ROOT ? l != (int)i : (uint32_t)l < (uint64_t)n) members[start[l] + slot[i]] = (int32_t)i;
  }
}

// Members ascending in every cluster.  Up to CL_SMALL members by the
// cluster's thread in place; up to CL_WAVE by one wavefront that ranks them in
// LDS; above that (a percolated graph) by the workgroup, which rereads the
// labels of all particles and compacts those of the cluster.
constexpr int CL_SMALL = 12, CL_WAVE = 1024;

__global__ __launch_bounds__(CS_T) void k_cl_sort(int64_t n, const int64_t *__restrict__ nc_dev,
                                                  const int32_t *__restrict__ cl_ptr,
                                                  const int32_t *__restrict__ label, int32_t *__restrict__ members) {
  __shared__ int32_t buf[CS_T / WAVE][CL_WAVE];
  __shared__ int list[CS_T], n_list;
  __shared__ int wsum[CS_T / WAVE];
  const int t = threadIdx.x, lane = t & (WAVE - 1), w = uniform_first(t / WAVE);
  const int64_t nc = *nc_dev;
  if (t == 0) n_list = 0;
  __syncthreads();
  const int64_t c = (int64_t)blockIdx.x * CS_T + t;
  if (c < nc) {
    const int a = cl_ptr[c], b = cl_ptr[c + 1];
    if (b - a > CL_SMALL) {
      list[atomicAdd(&n_list, 1)] = (int)c;
    } else {
      for (int k = a + 1; k < b; ++k) {
        const int32_t v = members[k];
        int q = k - 1;
        while (q >= a && members[q] > v) {
          members[q + 1] = members[q];
          --q;
        }
        members[q + 1] = v;
      }
    }
  }
  __syncthreads();
  const int nl = n_list;
  for (int e = w; e < nl; e += CS_T / WAVE) {  // uniform per wavefront
    const int a = cl_ptr[list[e]], m = cl_ptr[list[e] + 1] - a;
    if (m > CL_WAVE) continue;
    for (int k = lane; k < m; k += WAVE) buf[w][k] = members[a + k];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int k = lane; k < m; k += WAVE) {
      const int32_t v = buf[w][k];
      int r = 0;
      for (int q = 0; q < m; ++q) r += buf[w][q] < v ? 1 : 0;
      members[a + r] = v;
    }
    __builtin_amdgcn_wave_barrier();
  }
  for (int e = 0; e < nl; ++e) {  // uniform over the workgroup
    const int a = cl_ptr[list[e]], m = cl_ptr[list[e] + 1] - a;
    if (m <= CL_WAVE) continue;
    __syncthreads();  // every thread reads the label before a member is rewritten
    const int l = label[members[a]];
    __syncthreads();
    int at = a;
    for (int64_t i0 = 0; i0 < n; i0 += 4 * CS_T) {
      int own = 0;
      bool in[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t i = i0 + 4 * t + q;
        in[q] = i < n && label[i] == l;
        own += in[q] ? 1 : 0;
      }
      const int incl = wave_incl_scan(own);
      if (lane == WAVE - 1) wsum[w] = incl;
      __syncthreads();
      int o = at + incl - own;
#pragma unroll
      for (int q = 0; q < CS_T / WAVE; ++q) {
        o += q < w ? wsum[q] : 0;
        at += wsum[q];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (in[q]) members[o++] = (int32_t)(i0 + 4 * t + q);
      __syncthreads();
    }
  }
}

// The clusters of the last evaluation: labels, cluster CSR and the cluster
// count (c->cl_nc, on the device).  clear: words to clear on the way (the
// bucket words).
hipError_t clusters_pairs(p3t_ctx *c, int64_t n, int32_t *label, int32_t *cl_ptr, int32_t *cl_members,
                          int32_t *clear, int n_clear) {
  hipStream_t s = c->stream;
  hipLaunchKernelGGL(k_cl_labels, dim3(g1d(n)), dim3(256), 0, s, n, c->uf_parent, label, c->cl_cnt, c->cl_slot);
  scan_items<CL_ROOT>(c, n, label, c->cl_cnt, cl_ptr, cl_members, c->cl_nc, clear, n_clear);
  hipLaunchKernelGGL(k_cl_fill<CL_ROOT>, dim3(g1d(n)), dim3(256), 0, s, n, (const int32_t *)label,
                     (const int32_t *)c->cl_start, (const int32_t *)c->cl_slot, cl_members);
  hipLaunchKernelGGL(k_cl_sort, dim3((unsigned)((n + CS_T - 1) / CS_T)), dim3(CS_T), 0, s, n,
                     (const int64_t *)c->cl_nc, (const int32_t *)cl_ptr, (const int32_t *)label, cl_members);
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

// Labels outside [0, n) cannot index a count: (label, index) sorted by the
// low bits that labels of n particles need, neighbours of different label
// split, as such labels were always treated.
static hipError_t clusters_sorted(p3t_ctx *c, int64_t n, const int32_t *label, int32_t *cl_ptr, int32_t *cl_members,
                                  int64_t *n_clusters) {
  hipStream_t s = c->stream;
  hipError_t e;
  hipLaunchKernelGGL(k_cl_keys, dim3(g1d(n)), dim3(256), 0, s, n, label, c->cl_keys);
  int bits = 1;
  while ((int64_t(1) << bits) < n) ++bits;
  // keys start ascending in the particle index, so a stable sort on the
  // label bits alone orders by (label, index)
  uint64_t *k = c->cl_keys, *ka = c->cl_keys_alt;
  int32_t *v = nullptr, *va = nullptr;
  if ((e = radix_sort_pairs(k, v, ka, va, n, 32, 32 + bits, c->radix_hist, c->radix_hist_cap, false, s)) != hipSuccess)
    return e;
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
  // c->cl_nc[1]: a label was out of range
  hipLaunchKernelGGL(k_cl_count, dim3(g1d(n)), dim3(256), 0, s, n, label, c->cl_cnt, c->cl_slot, c->cl_nc + 1);
  scan_items<CL_ANY>(c, n, nullptr, c->cl_cnt, cl_ptr, cl_members, c->cl_nc, nullptr, 0);
  hipLaunchKernelGGL(k_cl_fill<CL_ANY>, dim3(g1d(n)), dim3(256), 0, s, n, label, (const int32_t *)c->cl_start,
                     (const int32_t *)c->cl_slot, cl_members);
  hipLaunchKernelGGL(k_cl_sort, dim3((unsigned)((n + CS_T - 1) / CS_T)), dim3(CS_T), 0, s, n,
                     (const int64_t *)c->cl_nc, (const int32_t *)cl_ptr, label, cl_members);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  int64_t *h = c->host_words;
  if ((e = hipMemcpyAsync(h, c->cl_nc, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
  if (h[1]) {
    if ((e = fill_i32(reinterpret_cast<int32_t *>(c->cl_nc + 1), 0, 2, s)) != hipSuccess) return e;
    return clusters_sorted(c, n, label, cl_ptr, cl_members, n_clusters);
  }
  *n_clusters = h[0];
  return hipSuccess;
}

}  // namespace p3t
