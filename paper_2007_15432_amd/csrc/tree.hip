// tree.hip -- Barnes-Hut tree over the particles (the paper uses the tree of
// its particle framework, Section 2.1.1; its construction is not specified
// there).  Built here for one GPU, fully in parallel:
//   1. bounding box; 48-bit Morton keys on a cube over the box (16 bits/axis,
//      cells of 2^-16 of the box, far below the leaf scale; the thin disk
//      then splits in x/y first and in z only at small scales);
//   2. stable radix sort of (key, index); gather of a Morton-ordered SoA copy;
//   3. binary radix tree over the sorted keys (one thread per internal node,
//      Karras 2012), ties broken by the sorted position;
//      and the lists of interaction groups (nodes with at most n_group_max
//      particles whose parent has more) and of the chunks of step 4;
//   4. bottom-up pass (one thread per lowest node that the walk can reach,
//      second arrival combines): tight bounding box, mass, centre of mass,
//      traceless quadrupole, max reach.
#include "p3t_internal.h"

namespace p3t {

// bit k of v (k < 21) to bit 3k
__device__ __forceinline__ uint64_t spread3(uint32_t v) {
  uint64_t x = v & 0x1fffffu;
  x = (x | (x << 32)) & 0x1f00000000ffffull;
  x = (x | (x << 16)) & 0x1f0000ff0000ffull;
  x = (x | (x << 8)) & 0x100f00f00f00f00full;
  x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
  x = (x | (x << 2)) & 0x1249249249249249ull;
  return x;
}

// bits per axis of the Morton keys: 3 MORTON_BITS = 48 key bits, six 8-bit
// radix passes
constexpr int MORTON_BITS = 16;

// Per-block bounding boxes of the positions.  Also clears the sort's
// histograms and the lists' counters for the launches that follow.
constexpr int BB_T = 256, BB_BLOCKS = 256;

__global__ __launch_bounds__(BB_T) void k_bbox_part(const double *__restrict__ pos, int64_t n, double *__restrict__ part,
                                                    uint32_t *__restrict__ hist, int64_t hist_words,
                                                    p3t::DevCounters *cnt) {
  __shared__ double sh[6][BB_T / p3t::WAVE];
  const int64_t g0 = (int64_t)blockIdx.x * BB_T + threadIdx.x, gs = (int64_t)gridDim.x * BB_T;
  if (g0 == 0) cnt->n_chunks = cnt->n_top = cnt->n_groups = 0;
  for (int64_t q = g0; q < hist_words; q += gs) hist[q] = 0u;
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int64_t k = g0; k < n; k += gs) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double x = pos[c * n + k];
      lo[c] = fmin(lo[c], x);
      hi[c] = fmax(hi[c], x);
    }
  }
  const int t = threadIdx.x;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    lo[c] = p3t::wave_min(lo[c]);
    hi[c] = p3t::wave_max(hi[c]);
    if ((t & (p3t::WAVE - 1)) == 0) {
      sh[c][t / p3t::WAVE] = lo[c];
      sh[3 + c][t / p3t::WAVE] = hi[c];
    }
  }
  __syncthreads();
  if (t < 6) {
    double v = sh[t][0];
    for (int w = 1; w < BB_T / p3t::WAVE; ++w) v = t < 3 ? fmin(v, sh[t][w]) : fmax(v, sh[t][w]);
    part[t * gridDim.x + blockIdx.x] = v;
  }
}

// The caller's rows packed into one 72-B record per particle (coalesced on
// both sides), so that the gather below reads one record per particle where
// it would read nine 8-B elements from nine scattered rows.
constexpr int PACK = 9;

// Morton keys, the tile histogram of their lowest digit for the sort
// (nullable), and the packed rows.  Every block reduces the at most BB_T box partials itself.
__global__ __launch_bounds__(BB_T) void k_morton(int64_t n, const double *__restrict__ pos,
                                                 const double *__restrict__ vel, const double *__restrict__ m,
                                                 const double *__restrict__ ro, const double *__restrict__ rs,
                                                 const double *__restrict__ part, int nb, uint64_t *__restrict__ keys,
                                                 int32_t *__restrict__ perm, double *__restrict__ rec,
                                                 uint32_t *__restrict__ hist, int tile) {
  __shared__ double sh[6][BB_T / p3t::WAVE];
  __shared__ double lrec[PACK * BB_T];
  double box[6];
  {
    const int t = threadIdx.x, w = t / p3t::WAVE;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const double v = t < nb ? part[c * nb + t] : (c < 3 ? INFINITY : -INFINITY);
      const double r = c < 3 ? p3t::wave_min(v) : p3t::wave_max(v);
      if ((t & (p3t::WAVE - 1)) == 0) sh[c][w] = r;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      box[c] = sh[c][0];
      for (int q = 1; q < BB_T / p3t::WAVE; ++q) box[c] = c < 3 ? fmin(box[c], sh[c][q]) : fmax(box[c], sh[c][q]);
    }
  }
  const double lx = box[0], ly = box[1], lz = box[2];
  const double ext = fmax(fmax(box[3] - lx, box[4] - ly), box[5] - lz);
  const double qmax = (double)((1 << MORTON_BITS) - 1);
  const double scale = ext > 0.0 ? qmax / ext : 0.0;
  for (int64_t b0 = (int64_t)blockIdx.x * BB_T; b0 < n; b0 += (int64_t)gridDim.x * BB_T) {
    const int64_t i = b0 + threadIdx.x;
    __syncthreads();
    if (i < n) {
      const double x = pos[i], y = pos[n + i], z = pos[2 * n + i];
      const double q[3] = {(x - lx) * scale, (y - ly) * scale, (z - lz) * scale};
      uint32_t u[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) u[c] = (uint32_t)fmin(fmax(q[c], 0.0), qmax);
      const uint64_t key = (spread3(u[0]) << 2) | (spread3(u[1]) << 1) | spread3(u[2]);
      keys[i] = key;
      perm[i] = (int32_t)i;
      if (hist) p3t::count_entry(hist, (uint32_t)(i / tile) * 256u + (uint32_t)(key & 255u), true);
      // the records through LDS: stored lane by lane, every instruction
      // would leave 64 partial lines
      double *r = lrec + PACK * threadIdx.x;
      r[0] = x;
      r[1] = y;
      r[2] = z;
      r[3] = vel[i];
      r[4] = vel[n + i];
      r[5] = vel[2 * n + i];
      r[6] = m[i];
      r[7] = ro[i];
      r[8] = rs[i];
    }
    __syncthreads();
    const int words = PACK * (int)(n - b0 < BB_T ? n - b0 : BB_T);
    for (int q = threadIdx.x; q < words; q += BB_T) rec[PACK * b0 + q] = lrec[q];
  }
}

// new positions and masses into the sorted arrays of the current order
__global__ void k_regather_xm(int64_t n, const int32_t *__restrict__ sid, const double *__restrict__ pos,
                              const double *__restrict__ m, double *__restrict__ sx, double *__restrict__ sy,
                              double *__restrict__ sz, double *__restrict__ sm) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = sid[k];
    sx[k] = pos[i];
    sy[k] = pos[n + i];
    sz[k] = pos[2 * n + i];
    sm[k] = m[i];
  }
}

// leaves per subtree of the bottom-up moments' first phase (see below)
constexpr int CHUNK = 2048;

// common-prefix length of sorted keys i and j (positions break ties); the
// keys of [lo, lo + GT_KEYS) are in LDS
constexpr int GT_T = 256, GT_TILE = 2 * GT_T, GT_HALO = 768, GT_KEYS = GT_TILE + 2 * GT_HALO;
struct KeyView {
  const uint64_t *k, *lds;
  int n, lo;
  __device__ __forceinline__ uint64_t at(int i) const {
    const unsigned o = (unsigned)(i - lo);
    return o < (unsigned)GT_KEYS ? lds[o] : k[i];
  }
  __device__ __forceinline__ int prefix(int i, uint64_t a, int j) const {
    if (j < 0 || j >= n) return -1;
    const uint64_t b = at(j);
    if (a == b) return 64 + __clz((unsigned)(i ^ j));
    return __clzll(a ^ b);
  }
};

// Into Morton order, and the radix tree over the sorted keys, in one launch
// (position k: sorted particle k and internal node k).
//   The particle's packed record (k_morton) is read once, its rows written.
//   The internal node's key range and split (Karras 2012) go to topo (left,
// right, first, count: 16 B per node, so that every later pass over the
// topology reads coalesced 16-B records).  Each node lists its children that
// are chunk roots of the moments pass (at most CHUNK leaves, the parent more),
// and groups (at most ng leaves, the parent more); a node of more than CHUNK
// leaves lists itself as a top node.  The root is listed by node 0's thread.
// The lists' order does not matter; a workgroup gathers its entries in LDS and
// takes their slots with one atomic per list (one per entry queued up on the
// counter: the flag, scan and compaction launches this replaces were no
// slower at 2^20 particles).  The arrival counter of every internal node is cleared.
//   Latency of the binary searches bounds the tree part, so the keys around
// the tile are in LDS (nearly every search stays within GT_HALO keys); the
// gather is bound by the scattered 72-B records.  2^20 particles: 75 us, the
// two separate kernels 45 + 46 us, and 33 us of flag scan and compaction.
__global__ __launch_bounds__(GT_T) void k_gather_tree(
    int n, int ng, const int32_t *__restrict__ perm, const double *__restrict__ rec, const uint64_t *__restrict__ keys,
    double *__restrict__ sx, double *__restrict__ sy, double *__restrict__ sz, double *__restrict__ svx,
    double *__restrict__ svy, double *__restrict__ svz, double *__restrict__ sm, double *__restrict__ sro,
    double *__restrict__ sinv, double *__restrict__ sreach, double *__restrict__ srs, int32_t *__restrict__ sid,
    int4 *__restrict__ topo, int32_t *__restrict__ parent, int32_t *__restrict__ visit,
    int32_t *__restrict__ chunk_list, int32_t *__restrict__ top_list, int32_t *__restrict__ group_node,
    p3t::DevCounters *cnt) {
  __shared__ uint64_t lk[GT_KEYS];
  // a node lists itself or up to two children per list (the root's thread
  // the root too, but then no child)
  __shared__ int lchunk[2 * GT_TILE], lgroup[2 * GT_TILE], ltop[GT_TILE];
  __shared__ int lcount[3];
  __shared__ unsigned long long lbase[3];
  const int t = threadIdx.x, leaf0 = n - 1;
  for (int base = blockIdx.x * GT_TILE; base < n; base += gridDim.x * GT_TILE) {
    __syncthreads();
    if (t < 3) lcount[t] = 0;
    KeyView K{keys, lk, n, base - GT_HALO};
    for (int q = t; q < GT_KEYS; q += GT_T) {
      const int i = base - GT_HALO + q;
      lk[q] = (i >= 0 && i < n) ? keys[i] : 0ull;
    }
    __syncthreads();
    for (int k = base + t; k < min(n, base + GT_TILE); k += GT_T) {
      {
        const int i = perm[k];
        const double *r = rec + (int64_t)PACK * i;
        sx[k] = r[0];
        sy[k] = r[1];
        sz[k] = r[2];
        svx[k] = r[3];
        svy[k] = r[4];
        svz[k] = r[5];
        sm[k] = r[6];
        const double o = r[7], s = r[8];
        sro[k] = o;
        sinv[k] = p3t::inv_cutoff(o);
        sreach[k] = fmax(o, s);
        srs[k] = s;
        sid[k] = i;
      }
      if (k == 0) {
        parent[0] = -1;  // node 0 is the root (the only particle's record if n = 1) and never a child
        if (n <= CHUNK) lchunk[atomicAdd(&lcount[0], 1)] = 0;
        if (n <= ng) lgroup[atomicAdd(&lcount[1], 1)] = 0;
      }
      if (k >= n - 1) continue;
      const int i = k;
      const uint64_t ki = K.at(i);
      const int d = (K.prefix(i, ki, i + 1) - K.prefix(i, ki, i - 1)) > 0 ? 1 : -1;
      const int dmin = K.prefix(i, ki, i - d);
      int lmax = 2;
      while (K.prefix(i, ki, i + lmax * d) > dmin) lmax <<= 1;
      int l = 0;
      for (int h = lmax >> 1; h >= 1; h >>= 1)
        if (K.prefix(i, ki, i + (l + h) * d) > dmin) l += h;
      const int j = i + l * d;
      const int dnode = K.prefix(i, ki, j);
      int s = 0, h = l;
      do {
        h = (h + 1) >> 1;
        if (K.prefix(i, ki, i + (s + h) * d) > dnode) s += h;
      } while (h > 1);
      const int split = i + s * d + (d < 0 ? -1 : 0);
      const int lo = i < j ? i : j, hi = i < j ? j : i;
      const int left = (lo == split) ? leaf0 + split : split;
      const int right = (hi == split + 1) ? leaf0 + split + 1 : split + 1;
      const int count = hi - lo + 1;
      topo[i] = make_int4(left, right, lo, count);
      parent[left] = i;
      parent[right] = i;
      visit[i] = 0;
      const int cl = split - lo + 1, cr = hi - split;
      if (count > CHUNK) {
        ltop[atomicAdd(&lcount[2], 1)] = i;
        if (cl <= CHUNK) lchunk[atomicAdd(&lcount[0], 1)] = left;
        if (cr <= CHUNK) lchunk[atomicAdd(&lcount[0], 1)] = right;
      }
      if (count > ng) {
        if (cl <= ng) lgroup[atomicAdd(&lcount[1], 1)] = left;
        if (cr <= ng) lgroup[atomicAdd(&lcount[1], 1)] = right;
      }
    }
    __syncthreads();
    if (t < 3 && lcount[t] > 0) {
      unsigned long long *c = t == 0 ? &cnt->n_chunks : t == 1 ? &cnt->n_groups : &cnt->n_top;
      lbase[t] = atomicAdd(c, (unsigned long long)lcount[t]);
    }
    __syncthreads();
    for (int q = t; q < lcount[0]; q += GT_T) chunk_list[lbase[0] + q] = lchunk[q];
    for (int q = t; q < lcount[1]; q += GT_T) group_node[lbase[1] + q] = lgroup[q];
    for (int q = t; q < lcount[2]; q += GT_T) top_list[lbase[2] + q] = ltop[q];
  }
}

// Bottom-up moments in two phases so that every hand-over between threads
// stays inside one workgroup (workgroup-scope fences only; device-scope
// fences would write back and invalidate the L2 of every XCD per level).
//   chunk roots: nodes with <= CHUNK leaves whose parent has more;
//   phase 1: one workgroup per chunk, from its bottom nodes to its root;
//   phase 2: one workgroup from every chunk root to the tree root.
// Bottom nodes: nodes of at most `lim` = min(n_leaf, n_group) particles whose
// parent holds more.  Nothing below them is read by the walk (it stops at
// nodes of at most n_leaf particles; the groups are bottom nodes or above), so
// one thread sums a bottom node over its particles directly and only the
// bottom nodes and those above (one node in eight at 16 leaves) have a record.

// What a parent needs of a child: box, centre of mass, mass, quadrupole,
// reach, range.
struct NodeRec {
  double lo[3], hi[3], com[3];
  double mass, reach;
  double q[6];
  int first, count;
};
static_assert(sizeof(NodeRec) == 144, "NodeRec layout");

__device__ __forceinline__ void quad_shift(double q[6], double m, double dx, double dy, double dz) {
  // add m (3 d d^T - |d|^2 I) for a point mass m at offset d from the new centre
  const double d2 = dx * dx + dy * dy + dz * dz;
  q[0] += m * (3.0 * dx * dx - d2);
  q[1] += m * (3.0 * dy * dy - d2);
  q[2] += m * (3.0 * dz * dz - d2);
  q[3] += m * 3.0 * dx * dy;
  q[4] += m * 3.0 * dx * dz;
  q[5] += m * 3.0 * dy * dz;
}

// Internal node from its two children: tight box, mass, centre of mass,
// traceless quadrupole about the centre of mass (parallel-axis shift of each
// child's moment), max reach.  Fixed order (left, right): deterministic.
__device__ __forceinline__ NodeRec combine_rec(const NodeRec &a, const NodeRec &b) {
  NodeRec o;
  const double M = a.mass + b.mass;
  o.mass = M;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    o.lo[d] = fmin(a.lo[d], b.lo[d]);
    o.hi[d] = fmax(a.hi[d], b.hi[d]);
    o.com[d] = M > 0.0 ? (a.mass * a.com[d] + b.mass * b.com[d]) / M : 0.5 * (o.lo[d] + o.hi[d]);
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) o.q[q] = a.q[q] + b.q[q];
  quad_shift(o.q, a.mass, a.com[0] - o.com[0], a.com[1] - o.com[1], a.com[2] - o.com[2]);
  quad_shift(o.q, b.mass, b.com[0] - o.com[0], b.com[1] - o.com[1], b.com[2] - o.com[2]);
  o.reach = fmax(a.reach, b.reach);
  o.first = a.first;
  o.count = a.count + b.count;
  return o;
}

// The children in the order (left, right), through one copy of the
// arithmetic: whichever of them arrives second, the result has the same bits
// (two inlined copies would be contracted differently).
__device__ __forceinline__ NodeRec combine_pair(const NodeRec &cur, const NodeRec &other, bool cur_left) {
  NodeRec a, b;
  auto pick = [&](auto x, auto y, auto &p, auto &q) {
    p = cur_left ? x : y;
    q = cur_left ? y : x;
  };
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    pick(cur.lo[d], other.lo[d], a.lo[d], b.lo[d]);
    pick(cur.hi[d], other.hi[d], a.hi[d], b.hi[d]);
    pick(cur.com[d], other.com[d], a.com[d], b.com[d]);
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) pick(cur.q[q], other.q[q], a.q[q], b.q[q]);
  pick(cur.mass, other.mass, a.mass, b.mass);
  pick(cur.reach, other.reach, a.reach, b.reach);
  pick(cur.first, other.first, a.first, b.first);
  pick(cur.count, other.count, a.count, b.count);
  return combine_rec(a, b);
}

// Particles [first, first + count) summed in order: sums of m and m x, then
// the quadrupole about the centre of mass.
__device__ __forceinline__ NodeRec bottom_rec(int first, int count, const double *__restrict__ sx,
                                              const double *__restrict__ sy, const double *__restrict__ sz,
                                              const double *__restrict__ sm, const double *__restrict__ sreach) {
  NodeRec o;
  o.first = first;
  o.count = count;
  double p[3] = {sx[first], sy[first], sz[first]};
  o.mass = sm[first];
  o.reach = sreach[first];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    o.lo[d] = o.hi[d] = o.com[d] = p[d];
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) o.q[q] = 0.0;
  if (count == 1) return o;
  double s[3] = {o.mass * p[0], o.mass * p[1], o.mass * p[2]};
#pragma unroll 4
  for (int k = first + 1; k < first + count; ++k) {
    const double x = sx[k], y = sy[k], z = sz[k], m = sm[k];
    o.lo[0] = fmin(o.lo[0], x);
    o.hi[0] = fmax(o.hi[0], x);
    o.lo[1] = fmin(o.lo[1], y);
    o.hi[1] = fmax(o.hi[1], y);
    o.lo[2] = fmin(o.lo[2], z);
    o.hi[2] = fmax(o.hi[2], z);
    o.mass += m;
    s[0] += m * x;
    s[1] += m * y;
    s[2] += m * z;
    o.reach = fmax(o.reach, sreach[k]);
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) o.com[d] = o.mass > 0.0 ? s[d] / o.mass : 0.5 * (o.lo[d] + o.hi[d]);
#pragma unroll 4
  for (int k = first; k < first + count; ++k)
    quad_shift(o.q, sm[k], sx[k] - o.com[0], sy[k] - o.com[1], sz[k] - o.com[2]);
  return o;
}

__device__ __forceinline__ void write_node(p3t::WalkNode *wn, p3t::CellMom *cm, int node, int left, int right,
                                           const NodeRec &o, bool moments) {
  p3t::WalkNode w;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    w.lo[d] = o.lo[d];
    w.hi[d] = o.hi[d];
    w.com[d] = o.com[d];
  }
  w.reach = o.reach;
  w.first = o.first;
  w.count = o.count;
  w.left = left;
  w.right = right;
  wn[node] = w;
  if (!moments) return;
  p3t::CellMom c;
#pragma unroll
  for (int d = 0; d < 3; ++d) c.com[d] = o.com[d];
  c.mass = o.mass;
#pragma unroll
  for (int q = 0; q < 6; ++q) c.q[q] = o.q[q];
  cm[node] = c;
}

__device__ __forceinline__ NodeRec read_node(const p3t::WalkNode *wn, const p3t::CellMom *cm, int node) {
  const p3t::WalkNode w = wn[node];
  const p3t::CellMom c = cm[node];
  NodeRec o;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    o.lo[d] = w.lo[d];
    o.hi[d] = w.hi[d];
    o.com[d] = c.com[d];
  }
  o.mass = c.mass;
  o.reach = w.reach;
#pragma unroll
  for (int q = 0; q < 6; ++q) o.q[q] = c.q[q];
  o.first = w.first;
  o.count = w.count;
  return o;
}

// Phase 1.  A subtree of the radix tree over leaves [first, first + count)
// numbers its count - 1 internal nodes inside [first, first + count), so
// node - first indexes the chunk's slot map.  The chunk's wide nodes (more
// than lim particles) and its internal bottom nodes take one of MOM_SLOTS LDS
// records each (a full chunk of 2048 needs 300-400 at 16 leaves; nodes that
// find none, with smaller leaves, hand over through their device-memory record
// and arrival counter).  A thread takes a bottom node, writes its record and
// climbs: the second arrival at a node combines its children, its own record
// still in registers.
// Bound by latency: the climb is a chain of about ten levels per chunk.  With
// 73 KB of LDS two workgroups share a CU (the earlier climb from every
// particle kept 1024 records, 152 KB).
constexpr int MOM_T = 512, MOM_SLOTS = 384;

__global__ __launch_bounds__(MOM_T) void k_moments_local(int n, int lim, const double *__restrict__ sx,
                                                         const double *__restrict__ sy, const double *__restrict__ sz,
                                                         const double *__restrict__ sm,
                                                         const double *__restrict__ sreach, p3t::WalkNode *wn,
                                                         p3t::CellMom *cm, const int4 *__restrict__ topo,
                                                         const int32_t *__restrict__ parent, int32_t *visit,
                                                         const int32_t *__restrict__ chunk, p3t::DevCounters *cnt) {
  __shared__ NodeRec rec[MOM_SLOTS];
  __shared__ int4 st[MOM_SLOTS];  // wide nodes: left, right, parent, arrivals
  __shared__ short map[CHUNK];    // slot of internal node first + t, or -1
  __shared__ int bot[CHUNK];      // bottom nodes
  __shared__ int n_bot, n_slot;
  const int leaf0 = n - 1, t0 = threadIdx.x;
  const int nch = (int)cnt->n_chunks;
  for (int ci = blockIdx.x; ci < nch; ci += gridDim.x) {
    const int r = chunk[ci];
    const int4 tr = r >= leaf0 ? make_int4(-1, -1, r - leaf0, 1) : topo[r];
    const int first = tr.z, count = min(tr.w, CHUNK);
    __syncthreads();
    if (t0 == 0) {
      n_bot = n_slot = 0;
      if (count <= lim) {
        bot[0] = r;
        n_bot = 1;
      }
    }
    __syncthreads();
    for (int t = t0; t < count && count > lim; t += MOM_T) {
      const int node = first + t;
      map[t] = -1;
      if (node >= leaf0) continue;
      const int4 tp = topo[node];
      // (one index of the range may be a node that reaches outside it)
      if (tp.w <= lim || tp.z < first || tp.z + tp.w > first + count) continue;
      const int s = atomicAdd(&n_slot, 1);
      if (s < MOM_SLOTS) {
        map[t] = (short)s;
        st[s] = make_int4(tp.x, tp.y, parent[node], 0);
      }
      // (a particle's or node's count: only wide nodes look at their children)
      if (tp.x >= leaf0 || topo[tp.x].w <= lim) bot[atomicAdd(&n_bot, 1)] = tp.x;
      if (tp.y >= leaf0 || topo[tp.y].w <= lim) bot[atomicAdd(&n_bot, 1)] = tp.y;
    }
    __syncthreads();
    const int nb = n_bot;
    __syncthreads();
    for (int b = t0; b < nb; b += MOM_T) {
      int child = bot[b];
      NodeRec cur;
      {
        const int4 tp = child >= leaf0 ? make_int4(-1, -1, child - leaf0, 1) : topo[child];
        cur = bottom_rec(tp.z, tp.w, sx, sy, sz, sm, sreach);
        // a particle is no cell: its moments are read only by the top climb
        write_node(wn, cm, child, tp.x, tp.y, cur, tp.w > 1 || child == r);
      }
      if (child == r) break;
      bool in_lds = true;  // the child's record is in LDS (a particle's is read from the arrays)
      if (child < leaf0) {
        const int s = atomicAdd(&n_slot, 1);
        in_lds = s < MOM_SLOTS;
        if (in_lds) rec[s] = cur;
        map[child - first] = (short)(in_lds ? s : -1);
      }
      int node = parent[child];
      for (;;) {
        const unsigned off = (unsigned)(node - first);
        if (off >= (unsigned)count) {  // not a radix subtree: reported, never indexed
          p3t::set_flag(cnt, P3T_FLAG_NAN);
          break;
        }
        const int s = map[off];
        if (in_lds)
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        else
          __threadfence_block();
        // first arrival: the sibling will finish; only the second arrival
        // combines (a third would mean a malformed tree: stop, never loop)
        const int prev = s >= 0 ? atomicAdd(&st[s].w, 1) : atomicAdd(&visit[node], 1);
        if (prev != 1) break;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        int left, right, up;
        if (s >= 0) {
          left = st[s].x;
          right = st[s].y;
          up = st[s].z;
        } else {
          left = topo[node].x;
          right = topo[node].y;
          up = parent[node];
        }
        const int sib = left == child ? right : left;
        NodeRec o;
        if (sib >= leaf0) {
          o = bottom_rec(sib - leaf0, 1, sx, sy, sz, sm, sreach);
        } else {
          const unsigned so = (unsigned)(sib - first);
          if (so >= (unsigned)count) {
            p3t::set_flag(cnt, P3T_FLAG_NAN);
            break;
          }
          const int q = map[so];
          if (q >= 0) {
            o = rec[q];
          } else {
            __threadfence_block();
            o = read_node(wn, cm, sib);
          }
        }
        cur = combine_pair(cur, o, left == child);
        write_node(wn, cm, node, left, right, cur, true);
        if (node == r) break;
        in_lds = s >= 0;
        if (in_lds) rec[s] = cur;
        child = node;
        node = up;
      }
    }
  }
}

constexpr int TOP_SLOTS = 4096;  // power of two
constexpr int TOP_PROBES = 32;   // probes per node before it falls back to device memory
constexpr int TOP_RECS = 768;

// Phase 2: one workgroup climbs from every chunk root to the root.  The top
// nodes' links, arrival counters and finished records are in LDS, found
// through a hash table of `slots` entries (a power of two <= TOP_SLOTS; open
// addressing on the node id), filled before the climb starts.  A top node
// beyond the TOP_RECS records (2^20 particles have about 750), or that finds
// no free entry within TOP_PROBES probes, goes through its record and counter
// in device memory.
__global__ __launch_bounds__(1024) void k_moments_top(p3t::WalkNode *wn, p3t::CellMom *cm,
                                                      const int4 *__restrict__ topo,
                                                      const int32_t *__restrict__ parent, int32_t *visit,
                                                      const int32_t *__restrict__ chunk,
                                                      const int32_t *__restrict__ top_list,
                                                      const p3t::DevCounters *cnt, int slots) {
  __shared__ NodeRec rec[TOP_RECS];
  __shared__ int4 st[TOP_RECS];  // left, right, parent, arrivals
  __shared__ int hkey[TOP_SLOTS];
  __shared__ short hval[TOP_SLOTS];
  const unsigned mask = (unsigned)slots - 1u;
  const int probes = slots < TOP_PROBES ? slots : TOP_PROBES;
  const int ntop = (int)cnt->n_top;
  if (ntop == 0) return;  // the root is a chunk root
  for (int q = threadIdx.x; q < slots; q += blockDim.x) hkey[q] = -1;
  __syncthreads();
  for (int q = threadIdx.x; q < min(ntop, TOP_RECS); q += blockDim.x) {
    const int node = top_list[q];
    const int4 tp = topo[node];
    st[q] = make_int4(tp.x, tp.y, parent[node], 0);
    unsigned h = ((unsigned)node * 2654435761u) & mask;
    for (int probe = 0; probe < probes; ++probe) {
      if (atomicCAS(&hkey[h], -1, node) == -1) {
        hval[h] = (short)q;
        break;
      }
      h = (h + 1) & mask;
    }
  }
  __syncthreads();
  // the record index of a top node, -1 for every other node
  auto find = [&](int node) -> int {
    unsigned h = ((unsigned)node * 2654435761u) & mask;
    for (int probe = 0; probe < probes; ++probe) {
      const int k = hkey[h];
      if (k == node) return hval[h];
      if (k == -1) return -1;
      h = (h + 1) & mask;
    }
    return -1;
  };
  const int nch = (int)cnt->n_chunks;
  for (int ci = threadIdx.x; ci < nch; ci += blockDim.x) {
    int child = chunk[ci];
    NodeRec cur = read_node(wn, cm, child);
    int node = parent[child];
    bool in_lds = true;  // (a chunk root's record was written by the launch before)
    while (node >= 0) {
      const int q = find(node);
      if (in_lds)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      else
        __threadfence_block();
      const int prev = q >= 0 ? atomicAdd(&st[q].w, 1) : atomicAdd(&visit[node], 1);
      if (prev != 1) break;
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
      int left, right, up;
      if (q >= 0) {
        left = st[q].x;
        right = st[q].y;
        up = st[q].z;
      } else {
        left = topo[node].x;
        right = topo[node].y;
        up = parent[node];
      }
      const int sib = left == child ? right : left;
      const int qs = find(sib);
      NodeRec o;
      if (qs >= 0) {
        o = rec[qs];
      } else {  // a chunk root, or a top node without a record in LDS
        __threadfence_block();
        o = read_node(wn, cm, sib);
      }
      cur = combine_pair(cur, o, left == child);
      write_node(wn, cm, node, left, right, cur, true);
      in_lds = q >= 0;
      if (in_lds) rec[q] = cur;
      child = node;
      node = up;
    }
  }
}

static inline unsigned g1d(int64_t n, int64_t cap = 65536) {
  int64_t b = (n + 255) / 256;
  return (unsigned)(b < 1 ? 1 : (b > cap ? cap : b));
}

// Moments and boxes of the current topology (the bottom-up pass; the arrival
// counters are clear).  2^20 particles, 16 leaves: local 63 us, top 38 us
// (climbing from every particle in chunks of 1024: 190 and 80 us); 65,536
// particles: 27 and 12 us (42 and 14).
static hipError_t moments_pass(p3t_ctx *c, int64_t n) {
  hipStream_t s = c->stream;
  hipLaunchKernelGGL(k_moments_local, dim3(c->n_cu * 2), dim3(MOM_T), 0, s, (int)n,
                     std::min(c->P.n_leaf_max, c->P.n_group_max), c->sx, c->sy, c->sz, c->sm, c->sreach, c->wnode,
                     c->cmom, c->topo, c->parent, c->visit, c->chunk_list, c->cnt);
  hipLaunchKernelGGL(k_moments_top, dim3(1), dim3(1024), 0, s, c->wnode, c->cmom, c->topo, c->parent, c->visit,
                     c->chunk_list, c->top_list, c->cnt, c->top_slots);
  return hipGetLastError();
}

hipError_t build_tree(p3t_ctx *c, int64_t n, const double *pos3, const double *vel3, const double *mass,
                      const double *r_out, const double *r_search) {
  hipStream_t s = c->stream;
  hipError_t e;
  const RadixPlan rp = radix_plan(n);
  const int nb = (int)std::min<int64_t>(BB_BLOCKS, (n + BB_T - 1) / BB_T);
  // The node records are rebuilt below, so their storage (96 B per node,
  // 2n - 1 nodes) holds the packed rows until then.
  static_assert(PACK * sizeof(double) <= 2 * sizeof(WalkNode), "packed rows exceed the node storage");
  double *rec = reinterpret_cast<double *>(c->wnode);
  hipLaunchKernelGGL(k_bbox_part, dim3(nb), dim3(BB_T), 0, s, pos3, n, c->bbox_part, c->radix_hist,
                     rp.chain ? (int64_t)RADIX_PASSES * rp.ntiles * 256 : 0, c->cnt);
  hipLaunchKernelGGL(k_morton, dim3(g1d(n)), dim3(BB_T), 0, s, n, pos3, vel3, mass, r_out, r_search, c->bbox_part, nb,
                     c->keys, c->perm, rec, rp.chain ? c->radix_hist : nullptr, rp.tile);
  uint64_t *k = c->keys, *ka = c->keys_alt;
  int32_t *v = c->perm, *va = c->perm_alt;
  ev_record(c, 17);
  static_assert(3 * MORTON_BITS <= 8 * RADIX_PASSES, "more sort passes than histograms");
  if ((e = radix_sort_pairs(k, v, ka, va, n, 0, 3 * MORTON_BITS, c->radix_hist, c->radix_hist_cap, true, s)) !=
      hipSuccess)
    return e;
  ev_record(c, 18);
  hipLaunchKernelGGL(k_gather_tree, dim3((unsigned)((n + GT_TILE - 1) / GT_TILE)), dim3(GT_T), 0, s, (int)n,
                     c->P.n_group_max, v, rec, k, c->sx, c->sy, c->sz, c->svx, c->svy, c->svz, c->sm, c->sro, c->sinv,
                     c->sreach, c->srs, c->sid, c->topo, c->parent, c->visit, c->chunk_list, c->top_list,
                     c->group_node, c->cnt);
  return moments_pass(c, n);
}

// the bottom-up pass over the current topology, its chunks and groups
hipError_t tree_moments(p3t_ctx *c, int64_t n) {
  const hipError_t e = fill_i32(c->visit, 0, n > 1 ? n - 1 : 1, c->stream);
  return e != hipSuccess ? e : moments_pass(c, n);
}

// Same topology, same lists: positions and masses replaced, moments redone.
hipError_t refresh_tree(p3t_ctx *c, const double *pos3, const double *mass) {
  const int64_t n = c->n;
  hipLaunchKernelGGL(k_regather_xm, dim3(g1d(n)), dim3(256), 0, c->stream, n, c->sid, pos3, mass, c->sx, c->sy, c->sz,
                     c->sm);
  return tree_moments(c, n);
}

}  // namespace p3t
