// cutoff.hip -- per-particle cut-off and search radii (Hill radius of
// Section 2.1.1, eq. (routi2), eq. (rsearch); shared mode eq. (rout1)).
//
// The random velocity of a particle is |v - v_K| with v_K the circular speed
// sqrt(G M_* / |x|) along phi-hat; v_ran,i is the rms of that quantity over
// the particle's bin among `vran_bins` log-spaced bins in cylindrical radius
// (bins with too few members fall back to the rms over all particles).
// Bin sums are formed per block in a fixed order and combined in block order,
// so the result does not depend on scheduling.
#include <algorithm>
#include <cstdio>
#include <mutex>
#include <string>

#include "p3t_internal.h"

// No multiply-add contraction in this file: the staged and the recomputing
// passes then form every per-particle term with the same roundings (the
// compiler would otherwise fuse differently in different kernels), so both
// entry points give the same bits.  The passes are bound by memory, not by
// arithmetic.
#pragma clang fp contract(off)

namespace p3t {

constexpr int CUT_T = 256;
constexpr int CUT_CHUNK = 1024;  // particles per bin-sum slot that the scratch sizes allow for
constexpr int CUT_MAX_BINS = 256;
constexpr int CUT_BLOCKS = 256;       // workgroups of the bin pass at most
constexpr int CUT_CELLS = 64 * CUT_T;  // LDS accumulators of the bin pass (128 KB)
constexpr int CUT_BT = 1024;           // threads of the bin pass

// The caller's particles and the constants of the per-particle terms.
struct CutIn {
  const double *pos, *vel, *m;
  int64_t n;
  double GM, m_star;
  int hill_length;
};

// Per-particle terms: cylindrical radius, squared random velocity |v -
// v_K phi-hat|^2 and the Hill radius (osculating semi-major axis, or |x|).
// The staged path stores them; the allocation-free path recomputes them
// where they are needed, with the same operations (same bits).
__device__ __forceinline__ void cut_terms(const CutIn &I, int64_t i, double &Rc, double &u2, double &rh) {
  const int64_t n = I.n;
  const double x = I.pos[i], y = I.pos[n + i], z = I.pos[2 * n + i];
  const double vx = I.vel[i], vy = I.vel[n + i], vz = I.vel[2 * n + i];
  const double r = sqrt(x * x + y * y + z * z);
  Rc = sqrt(x * x + y * y);
  const double v2 = vx * vx + vy * vy + vz * vz;
  double a;
  if (I.hill_length == 1) {
    a = r;
  } else {
    const double inv_a = 2.0 / r - v2 / I.GM;
    a = inv_a > 0.0 ? 1.0 / inv_a : r;  // unbound: fall back to |x|
  }
  rh = cbrt(I.m[i] / (3.0 * I.m_star)) * a;
  const double vk = sqrt(I.GM / r);
  const double phx = Rc > 0.0 ? -y / Rc : 0.0;
  const double phy = Rc > 0.0 ? x / Rc : 0.0;
  const double ux = vx - vk * phx, uy = vy - vk * phy, uz = vz;
  u2 = ux * ux + uy * uy + uz * uz;
}

// log-spaced bin of cylindrical radius R over [Rmin, Rmax]
__device__ __forceinline__ int cut_bin(double R, double Rmin, double lspan, int nbins) {
  int bb = 0;
  if (lspan > 0.0) {
    const double tt = floor((double)nbins * (log(R / Rmin) / lspan));
    bb = tt < 0.0 ? 0 : (tt > (double)(nbins - 1) ? nbins - 1 : (int)tt);
  }
  return bb;
}

__device__ __forceinline__ double cut_lspan(const double *mm) {
  const double Rmin = mm[0], Rmax = mm[1];
  return (Rmax > Rmin && Rmin > 0.0) ? log(Rmax / Rmin) : 0.0;
}

// STORE: keep R, u2 and the Hill radius per particle for the later passes
// (R_out, u2_out, rh_out); otherwise only the range of R is formed.
template <bool STORE>
__global__ __launch_bounds__(CUT_T) void k_cut_prep(CutIn I, double *__restrict__ R_out, double *__restrict__ u2_out,
                                                    double *__restrict__ rh_out, double *__restrict__ part) {
  __shared__ double sh[2][CUT_T / WAVE];
  double rmin = INFINITY, rmax = -INFINITY;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < I.n; i += (int64_t)gridDim.x * blockDim.x) {
    double Rc, u2, rh;
    cut_terms(I, i, Rc, u2, rh);
    if (STORE) {
      rh_out[i] = rh;
      u2_out[i] = u2;
      R_out[i] = Rc;
    }
    rmin = fmin(rmin, Rc);
    rmax = fmax(rmax, Rc);
  }
  rmin = wave_min(rmin);
  rmax = wave_max(rmax);
  const int t = threadIdx.x;
  if ((t & (WAVE - 1)) == 0) {
    sh[0][t / WAVE] = rmin;
    sh[1][t / WAVE] = rmax;
  }
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < CUT_T / WAVE; ++w) {
      rmin = fmin(rmin, sh[0][w]);
      rmax = fmax(rmax, sh[1][w]);
    }
    part[2 * blockIdx.x] = fmin(sh[0][0], rmin);
    part[2 * blockIdx.x + 1] = fmax(sh[1][0], rmax);
  }
}

// Per workgroup's range of particles: bin index of each particle and, per
// bin, the range's sum of u^2 and member count.  The accumulators are
// [bin][column] in LDS, 256 columns up to 64 bins, fewer above; all threads
// form their particles' bins (a logarithm each), then as many threads as there
// are columns at a time add theirs, each to its own column.  At the end
// threads share a bin and add its columns in order, and their partials are
// added in order: a fixed reduction order, so the result does not depend on
// scheduling.  2^20 particles: 16 us, where each bin's threads scanning
// a chunk's bins for their own took 35.
// The range of R is reduced from the partials by every workgroup itself;
// workgroup 0 also leaves it in mm.
// STORE: R and u2 come from the prep pass, and the bins are kept for the
// last pass; otherwise R and u2 are recomputed here and nothing is kept.
template <bool STORE>
__global__ __launch_bounds__(CUT_BT) void k_cut_bins(CutIn I, const double *__restrict__ R,
                                                    const double *__restrict__ u2, const double *__restrict__ part,
                                                    int nb_part, double *__restrict__ mm, int nbins, int64_t range,
                                                    int32_t *__restrict__ bin_out, double *__restrict__ psum,
                                                    double *__restrict__ pcnt) {
  __shared__ double cell[CUT_CELLS];
  __shared__ int cnt[CUT_MAX_BINS];
  __shared__ double ps[CUT_BT], sh[2][CUT_BT / WAVE];
  const int t = threadIdx.x;
  const int cols = CUT_CELLS / nbins < CUT_T ? CUT_CELLS / nbins : CUT_T;
  {
    double lo = INFINITY, hi = -INFINITY;
    for (int b = t; b < nb_part; b += CUT_BT) {
      lo = fmin(lo, part[2 * b]);
      hi = fmax(hi, part[2 * b + 1]);
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    if ((t & (WAVE - 1)) == 0) {
      sh[0][t / WAVE] = lo;
      sh[1][t / WAVE] = hi;
    }
  }
  for (int q = t; q < nbins * cols; q += CUT_BT) cell[q] = 0.0;
  for (int q = t; q < nbins; q += CUT_BT) cnt[q] = 0;
  __syncthreads();
  double range_mm[2] = {sh[0][0], sh[1][0]};
  for (int w = 1; w < CUT_BT / WAVE; ++w) {
    range_mm[0] = fmin(range_mm[0], sh[0][w]);
    range_mm[1] = fmax(range_mm[1], sh[1][w]);
  }
  if (blockIdx.x == 0 && t < 2) mm[t] = range_mm[t];
  const double Rmin = range_mm[0], lspan = cut_lspan(range_mm);
  const int64_t a = (int64_t)blockIdx.x * range, b = a + range < I.n ? a + range : I.n;
  const int group = t / cols, col = t - group * cols, groups = (CUT_BT + cols - 1) / cols;
  constexpr int PER = 4;
  for (int64_t i0 = a; i0 < b; i0 += PER * CUT_BT) {  // uniform
    int bb[PER];
    double u[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int64_t i = i0 + q * CUT_BT + t;
      bb[q] = -1;
      u[q] = 0.0;
      if (i >= b) continue;
      double Ri;
      if (STORE) {
        Ri = R[i];
        u[q] = u2[i];
      } else {
        double rh;
        cut_terms(I, i, Ri, u[q], rh);
      }
      bb[q] = cut_bin(Ri, Rmin, lspan, nbins);
      if (STORE) bin_out[i] = bb[q];
      atomicAdd(&cnt[bb[q]], 1);
    }
    for (int g = 0; g < groups; ++g) {  // uniform
      if (g == group) {
#pragma unroll
        for (int q = 0; q < PER; ++q)
          if (bb[q] >= 0) cell[bb[q] * cols + col] += u[q];
      }
      __syncthreads();
    }
  }
  // threads per bin, at least four; their partials are added one after another,
  // so no more than 64 (one bin, 1,000 particles: 41 -> 32 us a call)
  const int L = CUT_BT / nbins < WAVE ? CUT_BT / nbins : WAVE;
  const int k = t / L, q0 = t - k * L;
  double s = 0.0;
  if (k < nbins)
    for (int q = q0; q < cols; q += L) s += cell[k * cols + q];
  ps[t] = s;
  __syncthreads();
  if (t < nbins) {
    double ts = 0.0;
    for (int p = 0; p < L; ++p) ts += ps[t * L + p];
    psum[(int64_t)t * gridDim.x + blockIdx.x] = ts;  // [bin][workgroup]
    pcnt[(int64_t)t * gridDim.x + blockIdx.x] = (double)cnt[t];
  }
}

// One block per bin: the bin's partials in a fixed reduction order.
__global__ __launch_bounds__(256) void k_cut_binsum(const double *__restrict__ psum, const double *__restrict__ pcnt,
                                                    int nblk, double *__restrict__ bsum, double *__restrict__ bcnt) {
  __shared__ double shs[256 / WAVE], shc[256 / WAVE];
  const int k = blockIdx.x, t = threadIdx.x;
  double s = 0.0, c = 0.0;
  for (int b = t; b < nblk; b += 256) {
    s += psum[(int64_t)k * nblk + b];
    c += pcnt[(int64_t)k * nblk + b];
  }
  s = wave_sum(s);
  c = wave_sum(c);
  if ((t & (WAVE - 1)) == 0) {
    shs[t / WAVE] = s;
    shc[t / WAVE] = c;
  }
  __syncthreads();
  if (t == 0) {
    double ts = 0.0, tc = 0.0;
    for (int w = 0; w < 256 / WAVE; ++w) {
      ts += shs[w];
      tc += shc[w];
    }
    bsum[k] = ts;
    bcnt[k] = tc;
  }
}

// The radii.  Every workgroup forms the bins' rms itself (and the rms over
// all particles for sparse bins) from the at most 256 bin sums.
// STORE: bins and Hill radii from the earlier passes; otherwise recomputed.
// mxp (shared cut-offs, nullable): per workgroup the largest r_out and
// r_search.
template <bool STORE>
__global__ __launch_bounds__(CUT_T) void k_cut_out(CutIn I, const int32_t *__restrict__ bin,
                                                   const double *__restrict__ rh_in, const double *__restrict__ mm,
                                                   int nbins, int min_count, const double *__restrict__ bsum,
                                                   const double *__restrict__ bcnt, double rc0, double rc1, double rs0,
                                                   double rs1, double dt, double *__restrict__ r_out,
                                                   double *__restrict__ r_search, double *__restrict__ v_ran,
                                                   double *__restrict__ mxp) {
  __shared__ double ssum[CUT_MAX_BINS], scnt[CUT_MAX_BINS], vr_bin[CUT_MAX_BINS];
  __shared__ double vglob, sh[2][CUT_T / WAVE];
  const int t = threadIdx.x;
  if (t < nbins) {
    ssum[t] = bsum[t];
    scnt[t] = bcnt[t];
  }
  __syncthreads();
  if (t == 0) {
    double s = 0.0, c = 0.0;
    for (int q = 0; q < nbins; ++q) {
      s += ssum[q];
      c += scnt[q];
    }
    vglob = c > 0.0 ? sqrt(s / c) : 0.0;
  }
  __syncthreads();
  if (t < nbins) vr_bin[t] = scnt[t] >= (double)min_count ? sqrt(ssum[t] / scnt[t]) : vglob;
  __syncthreads();
  const double Rmin = STORE ? 0.0 : mm[0], lspan = STORE ? 0.0 : cut_lspan(mm);
  double mo = -INFINITY, ms = -INFINITY;
  for (int64_t i = (int64_t)blockIdx.x * CUT_T + t; i < I.n; i += (int64_t)gridDim.x * CUT_T) {
    int b;
    double rh;
    if (STORE) {
      b = bin[i];
      rh = rh_in[i];
    } else {
      double Rc, u2;
      cut_terms(I, i, Rc, u2, rh);
      b = cut_bin(Rc, Rmin, lspan, nbins);
    }
    const double vr = vr_bin[b];
    const double ro = fmax(rc0 * rh, rc1 * vr * dt);
    const double rs = rs0 * ro + rs1 * vr * dt;
    if (mxp) {
      mo = fmax(mo, ro);
      ms = fmax(ms, rs);
    } else {
      r_out[i] = ro;
      r_search[i] = rs;
    }
    if (v_ran) v_ran[i] = vr;
  }
  if (!mxp) return;  // uniform
  mo = wave_max(mo);
  ms = wave_max(ms);
  if ((t & (WAVE - 1)) == 0) {
    sh[0][t / WAVE] = mo;
    sh[1][t / WAVE] = ms;
  }
  __syncthreads();
  if (t < 2) {
    double m = sh[t][0];
    for (int w = 1; w < CUT_T / WAVE; ++w) m = fmax(m, sh[t][w]);
    mxp[2 * blockIdx.x + t] = m;
  }
}

// shared cut-off (eq. (rout1)): every particle takes the maxima over all
// particles, which every workgroup reduces from the nb partials
__global__ __launch_bounds__(CUT_T) void k_cut_shared(int64_t n, const double *__restrict__ mxp, int nb,
                                                      double *__restrict__ r_out, double *__restrict__ r_search) {
  __shared__ double sh[2][CUT_T / WAVE];
  const int t = threadIdx.x;
  double ro = -INFINITY, rs = -INFINITY;
  for (int b = t; b < nb; b += CUT_T) {
    ro = fmax(ro, mxp[2 * b]);
    rs = fmax(rs, mxp[2 * b + 1]);
  }
  ro = wave_max(ro);
  rs = wave_max(rs);
  if ((t & (WAVE - 1)) == 0) {
    sh[0][t / WAVE] = ro;
    sh[1][t / WAVE] = rs;
  }
  __syncthreads();
  ro = sh[0][0];
  rs = sh[1][0];
  for (int w = 1; w < CUT_T / WAVE; ++w) {
    ro = fmax(ro, sh[0][w]);
    rs = fmax(rs, sh[1][w]);
  }
  for (int64_t i = (int64_t)blockIdx.x * CUT_T + t; i < n; i += (int64_t)gridDim.x * CUT_T) {
    r_out[i] = ro;
    r_search[i] = rs;
  }
}

// The passes on stream s.  tmp (3n doubles) and bin (n int32) hold the
// per-particle terms between passes; with tmp == nullptr they are recomputed
// in each pass instead (the allocation-free entry point), with the same
// result.  part: cut_part_need(n) doubles, nothing in it needs clearing.
hipError_t cutoffs_run(const p3t_params &P, int64_t n, const double *pos3, const double *vel3, const double *mass,
                       double *r_out, double *r_search, double *v_ran, double *tmp, int32_t *bin, double *part,
                       hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const bool store = tmp != nullptr;
  double *R = store ? tmp : nullptr, *u2 = store ? tmp + n : nullptr, *rh = store ? tmp + 2 * n : nullptr;
  double *mm = part + 2048;
  double *psum = mm + 8 + CUT_MAX_BINS;
  const int nbins = P.vran_bins;
  const int nb_prep = (int)std::min<int64_t>(1024, (n + CUT_T - 1) / CUT_T);
  const int nblk = (int)std::min<int64_t>(CUT_BLOCKS, (n + CUT_CHUNK - 1) / CUT_CHUNK);
  const int64_t range = (n + nblk - 1) / nblk;
  double *pcnt = psum + (int64_t)nblk * nbins;
  CutIn I;
  I.pos = pos3;
  I.vel = vel3;
  I.m = mass;
  I.n = n;
  I.GM = P.G * P.m_star;
  I.m_star = P.m_star;
  I.hill_length = P.hill_length;
  if (store)
    hipLaunchKernelGGL(k_cut_prep<true>, dim3(nb_prep), dim3(CUT_T), 0, s, I, R, u2, rh, part);
  else
    hipLaunchKernelGGL(k_cut_prep<false>, dim3(nb_prep), dim3(CUT_T), 0, s, I, R, u2, rh, part);
  if (store)
    hipLaunchKernelGGL(k_cut_bins<true>, dim3(nblk), dim3(CUT_BT), 0, s, I, R, u2, part, nb_prep, mm, nbins, range, bin,
                       psum, pcnt);
  else
    hipLaunchKernelGGL(k_cut_bins<false>, dim3(nblk), dim3(CUT_BT), 0, s, I, R, u2, part, nb_prep, mm, nbins, range,
                       bin, psum, pcnt);
  double *bsum = part, *bcnt = part + CUT_MAX_BINS;  // the min/max partials are consumed
  hipLaunchKernelGGL(k_cut_binsum, dim3(nbins), dim3(256), 0, s, psum, pcnt, nblk, bsum, bcnt);
  const bool shared = P.cutoff_mode == 1;
  const int64_t g_max = shared ? CUT_BLOCKS : 2048;
  const unsigned g = (unsigned)std::min<int64_t>(g_max, (n + CUT_T - 1) / CUT_T);
  double *mxp = shared ? part + 2 * CUT_MAX_BINS : nullptr;  // 2 CUT_BLOCKS doubles, behind the bin sums
  static_assert(2 * CUT_MAX_BINS + 2 * CUT_BLOCKS <= 2048, "maxima exceed the range partials' scratch");
  if (store)
    hipLaunchKernelGGL(k_cut_out<true>, dim3(g), dim3(CUT_T), 0, s, I, bin, rh, mm, nbins, P.vran_min_count, bsum, bcnt,
                       P.r_cut0, P.r_cut1, P.r_search0, P.r_search1, P.dt_soft, r_out, r_search, v_ran, mxp);
  else
    hipLaunchKernelGGL(k_cut_out<false>, dim3(g), dim3(CUT_T), 0, s, I, bin, rh, mm, nbins, P.vran_min_count, bsum,
                       bcnt, P.r_cut0, P.r_cut1, P.r_search0, P.r_search1, P.dt_soft, r_out, r_search, v_ran, mxp);
  if (shared)
    // shared cut-off (eq. (rout1)) and shared search radius (Section 2.3)
    hipLaunchKernelGGL(k_cut_shared, dim3((unsigned)std::min<int64_t>(2048, (n + CUT_T - 1) / CUT_T)), dim3(CUT_T), 0,
                       s, n, (const double *)mxp, (int)g, r_out, r_search);
  return hipGetLastError();
}

hipError_t compute_cutoffs(p3t_ctx *c, int64_t n, const double *pos3, const double *vel3, const double *mass,
                           double *r_out, double *r_search, double *v_ran) {
  return cutoffs_run(c->P, n, pos3, vel3, mass, r_out, r_search, v_ran, c->tmp_d, c->cut_bin, c->cut_part, c->stream);
}

int64_t cut_part_need(int64_t n_cap) {
  const int64_t nblk = (n_cap + CUT_CHUNK - 1) / CUT_CHUNK;
  return 2048 + 8 + CUT_MAX_BINS + 2 * nblk * CUT_MAX_BINS + 64;
}

}  // namespace p3t

// ---------------------------------------------------------------- allocation-free entry point
// p3t_compute_cutoffs_noalloc keeps its scratch (the range partials, the
// per-chunk bin sums, the bin values) in this array instead of a context's
// memory: every GPU the library runs on holds one copy until the process
// ends.  In host code `scratch` only names the symbol; its device address is
// looked up per device with hipGetSymbolAddress and used from then on.
constexpr size_t NOALLOC_SCRATCH_BYTES = size_t(8) << 20;  // 8 MiB per GPU
static __device__ __align__(256) double scratch[NOALLOC_SCRATCH_BYTES / sizeof(double)];

namespace {

constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};  // device address of `scratch` per device
thread_local std::string g_noalloc_error;

p3t_status noalloc_fail(p3t_status st, const char *msg) {
  g_noalloc_error = msg;
  return st;
}

// The device address of `scratch` on the current device (looked up once).
hipError_t scratch_ptr(int dev, double **out) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<double *>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace

namespace p3t {
const char *noalloc_last_error() { return g_noalloc_error.c_str(); }
}  // namespace p3t

extern "C" p3t_status p3t_compute_cutoffs_noalloc(const p3t_params *p_host, int64_t n, const double *pos3,
                                                  const double *vel3, const double *mass, double *r_out,
                                                  double *r_search, double *v_ran, void *hip_stream) {
  using namespace p3t;
  if (!p_host) return noalloc_fail(P3T_ERR_ARG, "compute_cutoffs_noalloc: null parameters");
  const char *why = params_error(*p_host);
  if (why) return noalloc_fail(P3T_ERR_ARG, why);
  if (n < 0 || n > (int64_t(1) << 30)) return noalloc_fail(P3T_ERR_ARG, "compute_cutoffs_noalloc: n out of range");
  if (bad_ptr(pos3, n) || bad_ptr(vel3, n) || bad_ptr(mass, n) || bad_ptr(r_out, n) || bad_ptr(r_search, n))
    return noalloc_fail(P3T_ERR_ARG, "compute_cutoffs_noalloc: null pointer");
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= NOALLOC_MAX_DEVICES)
    return noalloc_fail(P3T_ERR_HIP, "compute_cutoffs_noalloc: no usable current device");
  double *part = nullptr;
  hipError_t e = scratch_ptr(dev, &part);
  if (e != hipSuccess) {
    char buf[256];
    snprintf(buf, sizeof(buf), "compute_cutoffs_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(e));
    return noalloc_fail(P3T_ERR_HIP, buf);
  }
  if (n == 0) return P3T_OK;
  // doubles the passes use: range partials, range, bin values, per-chunk bin sums and counts
  const int64_t nblk = (n + CUT_CHUNK - 1) / CUT_CHUNK;
  const int64_t need = 2048 + 8 + CUT_MAX_BINS + 2 * nblk * (int64_t)p_host->vran_bins;
  if (need * (int64_t)sizeof(double) > (int64_t)NOALLOC_SCRATCH_BYTES) {
    char buf[256];
    snprintf(buf, sizeof(buf),
             "compute_cutoffs_noalloc: n = %lld with %d bins needs %lld bytes of scratch, above its %zu",
             (long long)n, p_host->vran_bins, (long long)(need * (int64_t)sizeof(double)), NOALLOC_SCRATCH_BYTES);
    return noalloc_fail(P3T_ERR_CAPACITY, buf);
  }
  e = cutoffs_run(*p_host, n, pos3, vel3, mass, r_out, r_search, v_ran, nullptr, nullptr, part,
                  (hipStream_t)hip_stream);
  if (e != hipSuccess) {
    char buf[256];
    snprintf(buf, sizeof(buf), "compute_cutoffs_noalloc: launch: %s", hipGetErrorString(e));
    return noalloc_fail(P3T_ERR_HIP, buf);
  }
  return P3T_OK;
}

