// adjoint.hip -- vector-Jacobian product of the soft kick v' = v + h a(x, m)
// (eq. (HamiltonSol) with the soft force of eq. (softforce)) over the current
// tree, its interaction lists and the pair cut-offs r_out,ij held fixed.
//
// With a_i = sum_{j in P(i)} m_j phi(r_ij) d_ij + sum_{c in C(i)} M_c phi_1(r_ic) e_ic,
//   d_ij = x_j - x_i, e_ic = X_c - x_i, phi = G K(r / R_ij) / r^3, phi_1 = G / r^3,
// and the cotangent lambda of v', the loss L = sum_i lambda_i . a_i has, per
// list entry (i, j) with T_ij = m_j phi lambda_i . d_ij,
//   dT/dx_j = -dT/dx_i = m_j [ phi lambda_i + (phi'/r) (lambda_i . d) d ] =: g_ij,
//   dT/dm_j = phi lambda_i . d,
//   phi'/r = G [ K_y / (R r^4) - 3 K / r^5 ],
// and the same for a monopole cell with (X_c, M_c) in place of (x_j, m_j),
// K = 1.  A cell's centre of mass and mass depend on its members k:
//   dX_c/dx_k = m_k / M_c,  dX_c/dm_k = (x_k - X_c) / M_c,  dM_c/dm_k = 1,
// so the cell adjoints (dL/dX_c, dL/dM_c) are pushed down to every member.
//
// Every list entry is evaluated once: its term goes to both sides, into the
// registers of the i-particle and, travelling round a row of lanes, into the
// sums of the entry (k_adj_groups).  The i-side sums are written once per i,
// the entry's with one atomic add per (group, entry) and component.
// Then per node A_c = dL/dX_c / M_c, B_c = dL/dM_c - X_c . A_c, and per
// particle the sums of A and B over its ancestors:
//   dL/dx_k += m_k sum A,  dL/dm_k += sum B + x_k . sum A.
// Mixed precision (precision = 1, as the forward force): the K = 1 terms
// (far particles and cells) are evaluated in FP32 from offsets d formed in
// FP64 and the cotangent rounded to FP32; every sum stays FP64.  The
// changeover terms (near particles) are FP64 in both modes.
#include "p3t_internal.h"

namespace p3t {

namespace {

struct AdjArgs {
  const double *sx, *sy, *sz, *sm, *sinv;
  const int32_t *sid;
  const WalkNode *wn;
  const CellMom *cm;
  const GroupList *gl;
  const int32_t *order;
  const int32_t *pool;
  const int32_t *parent;
  DevCounters *cnt;
  const double *lam;  // cotangent in sorted order (3n)
  double *own;        // i-side terms, sorted order (3n), written once per particle
  double *g4;         // j-side terms and mass term, sorted order (n records of 4), atomic
  double *c4;         // cell adjoints dL/dX_c, dL/dM_c (n_nodes records of 4), atomic
  int64_t n;
  int n_nodes;
  double G, gamma, inv1mg;
  unsigned long long *queue;
};

// phi lambda + (phi'/r)(lambda . d) d (without the mass) and phi lambda . d
// for one entry; lambda carries the factor g (1 where it holds G already).
// `ok` false (the particle itself, a lane without a particle) gives zeros.
template <bool NEAR>
__device__ __forceinline__ void adj_term(double dx, double dy, double dz, double lx, double ly, double lz, double invR,
                                         bool ok, double g, const AdjArgs &A, double &tx, double &ty, double &tz,
                                         double &s) {
  if (NEAR) {  // (lambda, not the factors: whatever it holds, its product here is zero)
    dx = ok ? dx : 1.0;
    lx = ok ? lx : 0.0;
    ly = ok ? ly : 0.0;
    lz = ok ? lz : 0.0;
  }
  const double r2 = dx * dx + dy * dy + dz * dz;
  const double rinv = rsqrt_pos(r2);
  const double rinv2 = rinv * rinv;
  double phi = g * rinv * rinv2, dphi_r;  // phi, phi'(r) / r
  if (NEAR) {
    const double y = r2 * rinv * invR;
    const double x = fmin(fmax((y - A.gamma) * A.inv1mg, 0.0), 1.0);
    const double x2 = x * x, omx = 1.0 - x;
    const double K = x2 * x2 * (35.0 + x * (-84.0 + x * (70.0 - 20.0 * x)));
    const double Ky = 140.0 * x2 * x * omx * omx * omx * A.inv1mg;
    dphi_r = phi * (Ky * invR - 3.0 * K * rinv) * rinv;
    phi = phi * K;
  } else {
    dphi_r = -3.0 * phi * rinv2;
  }
  const double ld = lx * dx + ly * dy + lz * dz;
  const double c = dphi_r * ld;
  tx = phi * lx + c * dx;
  ty = phi * ly + c * dy;
  tz = phi * lz + c * dz;
  s = phi * ld;
}

// the K = 1 term in FP32: g = m (phi lambda + (phi'/r)(lambda . d) d),
// phi = G / r^3, phi'/r = -3 G / r^5
__device__ __forceinline__ void adj_term_f32(double dx, double dy, double dz, double lx, double ly, double lz,
                                             double mj, float G, double &gx, double &gy, double &gz, double &s) {
  const float fx = (float)dx, fy = (float)dy, fz = (float)dz;
  const float flx = (float)lx, fly = (float)ly, flz = (float)lz;
  const float r2 = fx * fx + fy * fy + fz * fz;
  const float rinv = rsqrtf(r2);
  const float rinv2 = rinv * rinv;
  const float phi = G * rinv * rinv2;
  const float dphi_r = -3.0f * phi * rinv2;
  const float ld = flx * fx + fly * fy + flz * fz;
  const float c = dphi_r * ld;
  const float m = (float)mj;
  gx = (double)(m * (phi * flx + c * fx));
  gy = (double)(m * (phi * fly + c * fy));
  gz = (double)(m * (phi * flz + c * fz));
  s = (double)(phi * ld);
}

__global__ void k_adj_prep(AdjArgs A, const double *__restrict__ lam_v3) {
  const int64_t n = A.n;
  if (blockIdx.x == 0 && threadIdx.x == 0) *A.queue = 0ull;
  double *lam = const_cast<double *>(A.lam);
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
    const int64_t o = A.sid[k];
    lam[k] = lam_v3[o];
    lam[n + k] = lam_v3[n + o];
    lam[2 * n + k] = lam_v3[2 * n + o];
    double2 *g = (double2 *)(A.g4 + 4 * k);
    g[0] = g[1] = make_double2(0.0, 0.0);
  }
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < A.n_nodes;
       c += (int64_t)gridDim.x * blockDim.x) {
    double2 *g = (double2 *)(A.c4 + 4 * c);
    g[0] = g[1] = make_double2(0.0, 0.0);
  }
}

constexpr int ADJ_W = 4;       // wavefronts per group
constexpr int ADJ_BLOCKS = 3;  // workgroups per CU
enum { ADJ_NEAR, ADJ_FAR, ADJ_CELL };

struct AdjTile {  // one wavefront's tile of particles or cells
  double2 xy[WAVE], zm[WAVE];
  double inv[WAVE];
  int id[WAVE];
};
struct AdjLds {
  AdjTile tile[ADJ_W];
  double own[3][ADJ_W][WAVE];
  int gi;
};

// LDS ordering inside one wavefront (its LDS operations execute in order)
__device__ __forceinline__ void adj_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// the value of the next lower lane of the row of 16 (row_ror:1)
__device__ __forceinline__ double row_ror1(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x121, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x121, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}
// a summed over rows 0, 1 (and 2, 3) in rows 0 (and 2), b's in rows 1 (and 3)
__device__ __forceinline__ double row_pair_add(double a, double b) {
  const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
  return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}

// the group's particles of one lane: number 32 s + (lane & 31) for slot s
template <int IPL>
struct AdjI {
  int id[IPL];  // -1: none
  double x[IPL], y[IPL], z[IPL], lx[IPL], ly[IPL], lz[IPL], inv[IPL], ox[IPL], oy[IPL], oz[IPL];
};

// One tile of up to 64 entries (list places t0 .. t0 + nt), 32 at a time: rows
// 0 and 1 hold the group's particles and take the first 16 entries, rows 2 and
// 3 hold the same particles and take the others.  In step s a lane meets entry
// (lane - s) mod 16 of its half; the entry's sums move on one lane per step and
// are home after 16.  The places behind nt repeat the first entry with no mass.
template <int IPL, int KIND, bool MIXED>
__device__ __forceinline__ void adj_tile(const AdjArgs &A, AdjTile &S, const int32_t *L, int nt, int lane,
                                         AdjI<IPL> &I) {
  constexpr bool F32 = MIXED && KIND != ADJ_NEAR;
  const double g = MIXED ? A.G : 1.0;  // (FP64 throughout: lambda holds G)
  {
    const bool in = lane < nt;
    const int j = L[in ? lane : 0];
    double x, y, z, m;
    if (KIND == ADJ_CELL) {
      const CellMom &cm = A.cm[j];
      x = cm.com[0];
      y = cm.com[1];
      z = cm.com[2];
      m = cm.mass;
    } else {
      x = A.sx[j];
      y = A.sy[j];
      z = A.sz[j];
      m = A.sm[j];
    }
    adj_wave_sync();  // the last tile is read
    S.xy[lane] = make_double2(x, y);
    S.zm[lane] = make_double2(z, in ? m : 0.0);
    if (KIND == ADJ_NEAR) S.inv[lane] = A.sinv[j];
    S.id[lane] = j;
    adj_wave_sync();
  }
  const int row = lane >> 4, base = (lane >> 5) << 4;
  for (int u = 0; u < nt; u += 32) {
    double ax = 0.0, ay = 0.0, az = 0.0, am = 0.0;
#pragma unroll 1
    for (int s = 0; s < 16; ++s) {
      const int e = u + base + ((lane - s) & 15);
      const double2 xy = S.xy[e], zm = S.zm[e];
      const double inv = KIND == ADJ_NEAR ? S.inv[e] : 0.0;
      const int jid = KIND == ADJ_NEAR ? S.id[e] : 0;
#pragma unroll
      for (int q = 0; q < IPL; ++q) {
        const double dx = xy.x - I.x[q], dy = xy.y - I.y[q], dz = zm.x - I.z[q];
        double tx, ty, tz, sc;
        if constexpr (F32) {  // (tx, ty, tz hold the mass)
          adj_term_f32(dx, dy, dz, I.lx[q], I.ly[q], I.lz[q], zm.y, (float)A.G, tx, ty, tz, sc);
          I.ox[q] -= tx;
          I.oy[q] -= ty;
          I.oz[q] -= tz;
        } else {
          const bool ok = KIND != ADJ_NEAR || (I.id[q] >= 0 && I.id[q] != jid);
          adj_term<KIND == ADJ_NEAR>(dx, dy, dz, I.lx[q], I.ly[q], I.lz[q],
                                     KIND == ADJ_NEAR ? fmin(I.inv[q], inv) : 0.0, ok, g, A, tx, ty, tz, sc);
          I.ox[q] -= zm.y * tx;
          I.oy[q] -= zm.y * ty;
          I.oz[q] -= zm.y * tz;
        }
        ax += tx;
        ay += ty;
        az += tz;
        am += sc;
      }
      ax = row_ror1(ax);
      ay = row_ror1(ay);
      az = row_ror1(az);
      am = row_ror1(am);
    }
    const int e = u + base + (lane & 15);
    const double m = F32 ? 1.0 : S.zm[e].y;
    // rows 0 and 2 add x and z of their entries, rows 1 and 3 y and the mass term
    const double v0 = row_pair_add(ax, ay), v1 = row_pair_add(az, am);
    if (e < nt) {
      double *o = (KIND == ADJ_CELL ? A.c4 : A.g4) + 4 * (int64_t)S.id[e] + (row & 1);
      unsafeAtomicAdd(o, m * v0);
      unsafeAtomicAdd(o + 2, (row & 1) ? v1 : m * v1);
    }
  }
}

template <int IPL, bool MIXED>
__device__ __forceinline__ void adj_group(const AdjArgs &A, AdjLds &S, const GroupList &Lh, int first, int gcount,
                                          int lane, int w) {
  const long long off = uniform_first64(Lh.off);
  const int n_cell = uniform_first(Lh.n_cell), n_near = uniform_first(Lh.n_near), n_far = uniform_first(Lh.n_far);
  const int64_t n = A.n;
  AdjI<IPL> I;
#pragma unroll
  for (int s = 0; s < IPL; ++s) {
    const int k = (lane & 31) + 32 * s;
    const bool in = k < gcount;
    const int i = in ? first + k : first;
    const double f = MIXED ? 1.0 : A.G;
    I.id[s] = in ? i : -1;
    I.x[s] = A.sx[i];
    I.y[s] = A.sy[i];
    I.z[s] = A.sz[i];
    I.lx[s] = in ? f * A.lam[i] : 0.0;
    I.ly[s] = in ? f * A.lam[n + i] : 0.0;
    I.lz[s] = in ? f * A.lam[2 * n + i] : 0.0;
    I.inv[s] = A.sinv[i];
    I.ox[s] = I.oy[s] = I.oz[s] = 0.0;
  }
  // the tiles of the three lists in turn over the wavefronts
  const int32_t *Lc = A.pool + off, *Ln = Lc + n_cell, *Lf = Ln + n_near;
  const int tn = (n_near + WAVE - 1) / WAVE, tf = (n_far + WAVE - 1) / WAVE, tc = (n_cell + WAVE - 1) / WAVE;
  int t = w;
  for (; t < tn; t += ADJ_W)
    adj_tile<IPL, ADJ_NEAR, MIXED>(A, S.tile[w], Ln + t * WAVE, min(WAVE, n_near - t * WAVE), lane, I);
  for (t -= tn; t < tf; t += ADJ_W)
    adj_tile<IPL, ADJ_FAR, MIXED>(A, S.tile[w], Lf + t * WAVE, min(WAVE, n_far - t * WAVE), lane, I);
  for (t -= tf; t < tc; t += ADJ_W)
    adj_tile<IPL, ADJ_CELL, MIXED>(A, S.tile[w], Lc + t * WAVE, min(WAVE, n_cell - t * WAVE), lane, I);
  // the particles' sums: two copies in each of the wavefronts
#pragma unroll
  for (int s = 0; s < IPL; ++s) {
    S.own[0][w][lane] = I.ox[s];
    S.own[1][w][lane] = I.oy[s];
    S.own[2][w][lane] = I.oz[s];
    __syncthreads();
    const int d = threadIdx.x >> 5, k = (threadIdx.x & 31) + 32 * s;
    if (d < 3 && k < gcount) {
      double v = 0.0;
#pragma unroll
      for (int q = 0; q < ADJ_W; ++q) v += S.own[d][q][threadIdx.x & 31] + S.own[d][q][(threadIdx.x & 31) + 32];
      A.own[d * n + first + k] = v;
    }
    __syncthreads();
  }
}

// One workgroup of four wavefronts per group, from a queue in the order of the
// work.  Bound by FP64 arithmetic: about 40 operations per pair (60 with the
// changeover).  Meeting each entry once with the sums passed along the row
// costs 8 lane moves per step for up to four pairs, where a second loop with
// the entries in lanes evaluated every pair again; rows of 16 leave less of a
// group's 65 to 128 places empty than lanes of 64 do.  262,144 particles,
// monopole cells: 1041 -> 422 us.
template <bool MIXED>
__global__ __launch_bounds__(ADJ_W *WAVE) void k_adj_groups(AdjArgs A) {
  __shared__ AdjLds S;
  const int lane = threadIdx.x & (WAVE - 1), w = uniform_first((int)threadIdx.x / WAVE);
  const int ngroups = uniform_first((int)A.cnt->n_groups);
  for (;;) {
    if (threadIdx.x == 0) S.gi = (int)atomicAdd(A.queue, 1ull);
    __syncthreads();
    const int gi = uniform_first(S.gi);
    __syncthreads();
    if (gi >= ngroups) break;
    const int q = uniform_first(A.order ? A.order[gi] : gi);
    const GroupList Lh = A.gl[q];
    if (uniform_first64(Lh.off) < 0) continue;
    const int node = uniform_first(Lh.node);
    const int first = uniform_first(A.wn[node].first), cnt = uniform_first(A.wn[node].count);
    if (cnt <= 32)
      adj_group<1, MIXED>(A, S, Lh, first, cnt, lane, w);
    else if (cnt <= 64)
      adj_group<2, MIXED>(A, S, Lh, first, cnt, lane, w);
    else if (cnt <= 96)
      adj_group<3, MIXED>(A, S, Lh, first, cnt, lane, w);
    else
      adj_group<4, MIXED>(A, S, Lh, first, cnt, lane, w);
  }
}

// A_c = dL/dX_c / M_c, B_c = dL/dM_c - X_c . A_c (in place)
__global__ void k_adj_cell_coeffs(AdjArgs A) {
  const int64_t nn = A.n_nodes;
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < nn; c += (int64_t)gridDim.x * blockDim.x) {
    double2 *r = (double2 *)(A.c4 + 4 * c);
    const double2 xy = r[0], zm = r[1];
    if (xy.x == 0.0 && xy.y == 0.0 && zm.x == 0.0 && zm.y == 0.0) continue;  // cell never used
    const double M = A.cm[c].mass;  // (the records of nodes no walk reaches are not written)
    const double iM = 1.0 / M;
    const double px = xy.x * iM, py = xy.y * iM, pz = zm.x * iM;
    r[0] = make_double2(px, py);
    r[1] = make_double2(pz, zm.y - (A.cm[c].com[0] * px + A.cm[c].com[1] * py + A.cm[c].com[2] * pz));
  }
}

// per particle: the ancestors' push-down, the three parts summed, scaled by h,
// written in the caller's order
__global__ void k_adj_final(AdjArgs A, double h, double *__restrict__ g_pos3, double *__restrict__ g_mass) {
  const int64_t n = A.n;
  const int leaf0 = (int)n - 1;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
    double sx = 0.0, sy = 0.0, sz = 0.0, sb = 0.0;
    int node = n > 1 ? A.parent[leaf0 + k] : -1;
    while (node >= 0) {
      const double2 *r = (const double2 *)(A.c4 + 4 * (int64_t)node);
      const double2 xy = r[0], zm = r[1];
      node = A.parent[node];
      sx += xy.x;
      sy += xy.y;
      sz += zm.x;
      sb += zm.y;
    }
    const double m = A.sm[k];
    const double2 *g4 = (const double2 *)(A.g4 + 4 * k);
    const double2 xy = g4[0], zm = g4[1];
    const double gx = A.own[k] + xy.x + m * sx;
    const double gy = A.own[n + k] + xy.y + m * sy;
    const double gz = A.own[2 * n + k] + zm.x + m * sz;
    const double gm = zm.y + sb + A.sx[k] * sx + A.sy[k] * sy + A.sz[k] * sz;
    const int64_t o = A.sid[k];
    g_pos3[o] = h * gx;
    g_pos3[n + o] = h * gy;
    g_pos3[2 * n + o] = h * gz;
    g_mass[o] = h * gm;
  }
}

}  // namespace

hipError_t soft_kick_adjoint(p3t_ctx *c, double h, const double *lam_v3, double *g_pos3, double *g_mass) {
  const hipStream_t s = c->stream;
  const int64_t n = c->n;
  AdjArgs A;
  A.sx = c->sx;
  A.sy = c->sy;
  A.sz = c->sz;
  A.sm = c->sm;
  A.sinv = c->sinv;
  A.sid = c->sid;
  A.wn = c->wnode;
  A.cm = c->cmom;
  A.gl = c->glist;
  A.order = c->group_order;
  A.pool = c->pool;
  A.parent = c->parent;
  A.cnt = c->cnt;
  A.lam = c->adj_buf;
  A.own = c->adj_buf + 3 * n;
  A.g4 = c->adj_buf + 6 * n;  // (records of 4 aligned to 16 bytes: 48 n and 80 n bytes in)
  A.n_nodes = (int)(n > 0 ? 2 * n - 1 : 0);
  A.c4 = c->adj_buf + 10 * n;
  A.n = n;
  A.G = c->P.G;
  A.gamma = c->P.gamma;
  A.inv1mg = 1.0 / (1.0 - c->P.gamma);
  A.queue = &c->cnt->queue;
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>((int64_t)c->n_cu * 8, (2 * n + 255) / 256));
  hipLaunchKernelGGL(k_adj_prep, dim3(g), dim3(256), 0, s, A, lam_v3);
  if (c->P.precision == 1)
    hipLaunchKernelGGL(k_adj_groups<true>, dim3(c->n_cu * ADJ_BLOCKS), dim3(ADJ_W * WAVE), 0, s, A);
  else
    hipLaunchKernelGGL(k_adj_groups<false>, dim3(c->n_cu * ADJ_BLOCKS), dim3(ADJ_W * WAVE), 0, s, A);
  hipLaunchKernelGGL(k_adj_cell_coeffs, dim3(g), dim3(256), 0, s, A);
  hipLaunchKernelGGL(k_adj_final, dim3(g), dim3(256), 0, s, A, h, g_pos3, g_mass);
  return hipGetLastError();
}

int64_t adjoint_buf_need(int64_t n_cap) { return 10 * n_cap + 4 * (2 * n_cap); }

}  // namespace p3t
