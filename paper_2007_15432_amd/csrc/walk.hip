// walk.hip -- per-group tree walk producing three interaction lists.
//
// For a group g (a tree node of at most n_group_max particles) and a node c:
//   separated(g, c): the bounding-box distance exceeds max(reach_g, reach_c)
//     (reach = max(r_search, r_out) over the members) with a 1e-12 guard, so
//     no pair between them can be a neighbour candidate or feel K < 1;
//   accepted(g, c): separated, more than one particle, and the opening test
//     l_c < theta * d (l_c the longest edge of c's box, d the distance from
//     c's centre of mass to g's box);
// accepted nodes become multipole CELLS; opened leaves (<= n_leaf_max
// particles) give NEAR particles if not separated, FAR particles otherwise;
// other opened nodes push their two children.  theta = 0 accepts nothing,
// which reduces the tree force to the direct sum.
//
// One wavefront per group, persistent grid.  The wavefront tests up to 64
// nodes of its DFS stack at a time; the stack, the accepted cells and the
// opened leaves (as ranges of particles, expanded only when the finished list
// goes to the shared pool at an atomically reserved offset) live in LDS, with
// per-wavefront device memory behind them for the groups that need more.  Every
// write is bounds-checked; an overflow marks the group (offset -1) and sets a
// status bit so that the host can grow and retry.
//   A group is a chain of about 30 frontiers, each the load of up to 64
// scattered node records and some 200 VALU instructions.  Up to about six
// wavefronts per CU the latency of that chain bounds the walk (2^20 particles,
// with the order of the groups: 757 us with one, 414 with two, 252 with four,
// 220 with six), beyond that the throughput of the node tests: 211 with eight or
// ten, and with half the LDS, so that 22 fit instead of 11, 215 with eight, 209
// with eighteen.  65,536 particles have three groups per CU: the chain alone.
// With the stack and lists in device memory, a store waited for per frontier,
// and the particles written one by one to a scratch list first, 2^20 particles
// took 359 us, 65,536 65, 2048 43; now 199, 31 and 16.
//   The group list is cut into eight parts, a part to the workgroups of one XCD
// (blockIdx mod 8), whose L2 then serves one region of the tree: the list is
// roughly in Morton order (that of the arrival of the workgroups that filled
// it).  A wavefront whose part is done takes groups of the others.
#include "p3t_internal.h"

namespace p3t {

constexpr int GROUP_CLASSES = 128;
constexpr int WALK_STACK = 1536, WALK_CELLS = 768, WALK_NEAR = 256, WALK_FAR = 384;

// Work of a group (its i-particles times its list entries, cells counted
// twice), in classes of half an octave: the force kernels take the groups
// in descending class, so the longest lists start first and the tail of
// the launch is short.  Only the order of the work depends on it.
__device__ __forceinline__ int group_class(int count, int n_cell, int n_near, int n_far) {
  const uint64_t work = (uint64_t)count * (uint64_t)(n_near + n_far + 2 * n_cell) / 64 + 1;
  const int msb = 63 - __clzll((long long)work);
  const int half = msb > 0 ? (int)((work >> (msb - 1)) & 1ull) : 0;
  return min(GROUP_CLASSES - 1, 2 * msb + half);
}

// the ranges of one class, expanded in order to out
__device__ __forceinline__ void expand_ranges(const int2 *lds, int lds_cap, const int32_t *slot, int n_ranges,
                                              int32_t *out, int lane) {
  int base = 0;
  for (int r0 = 0; r0 < n_ranges; r0 += WAVE) {  // uniform
    const int r = r0 + lane;
    int2 v = make_int2(0, 0);
    if (r < n_ranges) v = r < lds_cap ? lds[r] : make_int2(slot[2 * r], slot[2 * r + 1]);
    const int incl = wave_incl_scan(v.y);
    int32_t *o = out + base + incl - v.y;
    for (int q = 0; q < v.y; ++q) o[q] = v.x + q;
    base += uniform_lane(incl, WAVE - 1);
  }
}

__global__ __launch_bounds__(WAVE) void k_walk(const WalkNode *__restrict__ wn, const int32_t *__restrict__ group_node,
                                               DevCounters *cnt, unsigned long long *__restrict__ queues,
                                               GroupList *__restrict__ gl, int32_t *__restrict__ group_cls,
                                               int32_t *__restrict__ pool, int64_t pool_cap,
                                               int32_t *__restrict__ slot_lists, int cap,
                                               int32_t *__restrict__ slot_stack, int stack_cap, double theta2,
                                               int n_leaf) {
  __shared__ int lstk[WALK_STACK], lcell[WALK_CELLS];
  __shared__ int2 lnear[WALK_NEAR], lfar[WALK_FAR];
  const int lane = threadIdx.x;
  // device memory behind the LDS lists: entries (cells, stack) and ranges
  // (two words each) beyond the LDS capacity, at their own index
  int32_t *Lc = slot_lists + (int64_t)blockIdx.x * 3 * cap;
  int32_t *Ln = Lc + cap;
  int32_t *Lf = Ln + cap;
  int32_t *stk = slot_stack + (int64_t)blockIdx.x * stack_cap;
  const int ngroups = uniform_first((int)cnt->n_groups);
  int part = 0;  // parts finished so far
  for (;;) {
    int gi = -1;
    while (part < WALK_PARTS) {  // uniform
      const int s = (blockIdx.x + part) % WALK_PARTS;
      const int g0 = (int)((int64_t)ngroups * s / WALK_PARTS), g1 = (int)((int64_t)ngroups * (s + 1) / WALK_PARTS);
      unsigned long long *q = queues + (int64_t)s * WALK_QUEUE_STRIDE;
      // another part's queue is looked at first: the atomics of every
      // wavefront that finds it empty would queue up behind each other
      if (part > 0 &&
          uniform_first((int)__hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >= g1 - g0) {
        ++part;
        continue;
      }
      const int k = (int)wave_fetch_add(q, 1ull);
      if (k < g1 - g0) {
        gi = g0 + k;
        break;
      }
      ++part;
    }
    if (gi < 0) break;
    const int g = group_node[gi];
    double glo[3], ghi[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      glo[d] = wn[g].lo[d];
      ghi[d] = wn[g].hi[d];
    }
    const double greach = wn[g].reach;
    const int gcount = wn[g].count;
    int top = 1, ncell = 0, nnear = 0, nfar = 0;  // entries, cells, near and far ranges
    int tnear = 0, tfar = 0;                      // this lane's near and far particles
    bool ovf = false;
    __syncthreads();
    if (lane == 0) lstk[0] = 0;  // root
    while (top > 0 && !ovf) {
      __syncthreads();
      const int npop = top < WAVE ? top : WAVE;
      const int p0 = top - npop + lane;
      const int node = lane < npop ? (p0 < WALK_STACK ? lstk[p0] : stk[p0]) : -1;
      top -= npop;
      __syncthreads();
      int outcome = 0;  // 0 none, 1 cell, 2 near leaf, 3 far leaf, 4 open
      int first = 0, count = 0, left = 0, right = 0;
      if (node >= 0) {
        const WalkNode W = wn[node];
        double dbb2 = 0.0, dc2 = 0.0, l = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const double gap = fmax(fmax(W.lo[d] - ghi[d], glo[d] - W.hi[d]), 0.0);
          dbb2 += gap * gap;
          const double cg = fmax(fmax(glo[d] - W.com[d], W.com[d] - ghi[d]), 0.0);
          dc2 += cg * cg;
          l = fmax(l, W.hi[d] - W.lo[d]);
        }
        const double rr = fmax(greach, W.reach) * (1.0 + 1e-12);
        const bool sep = dbb2 > rr * rr;
        const bool accept = sep && W.count > 1 && l * l < theta2 * dc2;
        first = W.first;
        count = W.count;
        left = W.left;
        right = W.right;
        if (accept)
          outcome = 1;
        else if (W.count <= n_leaf || W.left < 0)
          outcome = sep ? 3 : 2;
        else
          outcome = 4;
      }
      const unsigned long long mc = __ballot(outcome == 1), mn = __ballot(outcome == 2), mf = __ballot(outcome == 3),
                               mo = __ballot(outcome == 4);
      if (outcome == 1) {
        const int p = ncell + popc_below(mc);
        if (p < WALK_CELLS)
          lcell[p] = node;
        else if (p < cap)
          Lc[p] = node;
      } else if (outcome == 2) {
        const int p = nnear + popc_below(mn);
        if (p < WALK_NEAR)
          lnear[p] = make_int2(first, count);
        else if (2 * p + 1 < cap)
          Ln[2 * p] = first, Ln[2 * p + 1] = count;
        tnear += count;
      } else if (outcome == 3) {
        const int p = nfar + popc_below(mf);
        if (p < WALK_FAR)
          lfar[p] = make_int2(first, count);
        else if (2 * p + 1 < cap)
          Lf[2 * p] = first, Lf[2 * p + 1] = count;
        tfar += count;
      } else if (outcome == 4) {  // both children
        const int p = top + 2 * popc_below(mo);
        if (p + 1 < WALK_STACK) {
          lstk[p] = left;
          lstk[p + 1] = right;
        } else if (p + 1 < stack_cap) {
          (p < WALK_STACK ? lstk : stk)[p] = left;
          stk[p + 1] = right;
        }
      }
      ncell += (int)__popcll(mc);
      nnear += (int)__popcll(mn);
      nfar += (int)__popcll(mf);
      top += 2 * (int)__popcll(mo);
      if (ncell > cap || 2 * nnear > cap || 2 * nfar > cap || top > stack_cap) ovf = true;
    }
    if (ovf) {
      if (lane == 0) {
        set_flag(cnt, top > stack_cap ? P3T_FLAG_STACK_OVERFLOW : P3T_FLAG_LIST_OVERFLOW);
        GroupList o;
        o.off = -1;
        o.n_cell = o.n_near = o.n_far = 0;
        o.node = g;
        gl[gi] = o;
        group_cls[gi] = 0;
      }
      continue;
    }
    __syncthreads();
    const int np = uniform_first(wave_sum(tnear)), nq = uniform_first(wave_sum(tfar));
    const int total = ncell + np + nq;
    const long long off = (long long)wave_fetch_add(&cnt->pool_cursor, (unsigned long long)total);
    const bool fits = off + total <= pool_cap;
    if (lane == 0) {
      if (!fits) set_flag(cnt, P3T_FLAG_LIST_OVERFLOW);
      GroupList o;
      o.off = fits ? off : -1;
      o.n_cell = fits ? ncell : 0;
      o.n_near = fits ? np : 0;
      o.n_far = fits ? nq : 0;
      o.node = g;
      gl[gi] = o;
      group_cls[gi] = group_class(gcount, o.n_cell, o.n_near, o.n_far);
    }
    if (!fits) continue;
    for (int q = lane; q < ncell; q += WAVE) pool[off + q] = q < WALK_CELLS ? lcell[q] : Lc[q];
    expand_ranges(lnear, WALK_NEAR, Ln, nnear, pool + off + ncell, lane);
    expand_ranges(lfar, WALK_FAR, Lf, nfar, pool + off + ncell + np, lane);
  }
}

// Queue heads and per-evaluation counters; with a new pair list to come, the
// close-pair flags are cleared and every particle becomes its own cluster
// (close nullable).
__global__ void k_reset_queues(DevCounters *cnt, unsigned long long *__restrict__ queues, int64_t n,
                               int32_t *__restrict__ close, int32_t *__restrict__ uf) {
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, ts = (int64_t)gridDim.x * blockDim.x;
  if (close) {
    for (int64_t k = t0; k < (n + 3) / 4; k += ts) close[k] = 0;
    for (int64_t k = t0; k < n; k += ts) uf[k] = (int32_t)k;
  }
  if (t0 < WALK_PARTS) queues[t0 * WALK_QUEUE_STRIDE] = 0;
  if (t0 != 0) return;
  cnt->force_queue = 0;
  cnt->queue = 0;
  for (int k = 0; k < 4; ++k) cnt->force_clk[k] = 0;
  cnt->pool_cursor = 0;
  cnt->n_pairs = 0;
  cnt->n_near = 0;
  cnt->n_far = 0;
  cnt->n_cell = 0;
}

// One workgroup: a counting sort of the groups by class, largest first
// (within a class in any order).  A device count above n_static (the host's
// bound, from the last evaluation) sets P3T_FLAG_GROUP_BOUND: the order and
// the force then cover only the first n_static groups and the host
// evaluates again with the bound n.
__global__ __launch_bounds__(1024) void k_group_order(const int32_t *__restrict__ cls, int n_static, DevCounters *cnt,
                                                      int32_t *__restrict__ order) {
  __shared__ int hist[GROUP_CLASSES];
  const int t = threadIdx.x;
  int ng = (int)cnt->n_groups;
  if (ng > n_static) {
    if (t == 0) atomicOr(&cnt->status, P3T_FLAG_GROUP_BOUND);
    ng = n_static;
  }
  for (int q = t; q < GROUP_CLASSES; q += blockDim.x) hist[q] = 0;
  __syncthreads();
  for (int g = t; g < ng; g += blockDim.x) atomicAdd(&hist[cls[g]], 1);
  __syncthreads();
  if (t == 0) {  // exclusive offsets, largest class first
    int acc = 0;
    for (int q = GROUP_CLASSES - 1; q >= 0; --q) {
      const int h = hist[q];
      hist[q] = acc;
      acc += h;
    }
  }
  __syncthreads();
  for (int g = t; g < ng; g += blockDim.x) order[atomicAdd(&hist[cls[g]], 1)] = g;
}

static void reset(p3t_ctx *c, bool new_pairs) {
  const unsigned g = new_pairs ? (unsigned)std::max<int64_t>(1, std::min<int64_t>(1024, (c->n + 255) / 256)) : 1u;
  hipLaunchKernelGGL(k_reset_queues, dim3(g), dim3(256), 0, c->stream, c->cnt, c->walk_q, c->n,
                     new_pairs ? reinterpret_cast<int32_t *>(c->close_flag) : nullptr, c->uf_parent);
}

hipError_t walk_groups(p3t_ctx *c, int64_t n_groups_max) {
  hipStream_t s = c->stream;
  reset(c, true);
  const double th = c->P.theta;
  // small disks have few groups (about n / 87): no more wavefronts than could find one
  const unsigned g = (unsigned)std::min<int64_t>(c->walk_slots, std::max<int64_t>(64, c->n / 16));
  hipLaunchKernelGGL(k_walk, dim3(g), dim3(WAVE), 0, s, c->wnode, c->group_node, c->cnt, c->walk_q, c->glist,
                     c->group_cls, c->pool, c->pool_cap, c->slot_lists, (int)c->slot_cap_list, c->slot_stack,
                     (int)c->slot_cap_stack, th * th, c->P.n_leaf_max);
  // longest-first order for the force kernels; the device-side group count
  // bounds it, so n_groups_max may be any upper bound (a captured graph
  // passes the particle count)
  const int ns = (int)std::min<int64_t>(n_groups_max, INT32_MAX);
  hipLaunchKernelGGL(k_group_order, dim3(1), dim3(1024), 0, s, c->group_cls, ns, c->cnt, c->group_order);
  return hipGetLastError();
}

// (the frozen-list evaluation keeps the pairs, and the close flags, of the last one)
void reset_queues(p3t_ctx *c) { reset(c, false); }

}  // namespace p3t
