// force_split.hip -- the soft force (eq. (softforce) with the pair cut-off of
// eq. (rout2); neighbour pairs of Section 2.3) over the groups' lists, an
// alternative to the fused kernel of force.hip.
//
//   k_force_all  one workgroup of W wavefronts per group; the list's tiles of
//            64 entries are dealt to the wavefronts, each class with a loop of
//            its own:
//     near   FP64 with the changeover K (mixed form: the pairs beyond both
//            cut-offs, where K = 1, in FP32 from FP64 offsets, the few
//            inside the changeover in FP64); while it runs, each lane
//            records in a bit mask which j of the current tile are
//            neighbour candidates
//            (r^2 <= max reach^2, with a relative margin that covers the
//            rounding of r^2); after the tile they queue up in LDS for the
//            exact neighbour test of Section 2.3, one per lane, and neighbours
//            go to the pair buffer.  Coincident pairs (r = 0, i != j) are
//            always candidates and are reported there.
//     far    K = 1 particles, FP64 or (mixed) FP32 offsets from the group
//            centre with compensated accumulation.
//     cells  monopole or traceless-quadrupole cells, FP64 or FP32.
//            The wavefronts' sums are added in LDS and written in the caller's
//            order, with the NaN check.
//
// A lane owns one i-particle, or two when the group holds more than 64 (the
// choice is per group, so small groups do not pay for an idle second slot).
// j data are staged 64 at a time in the wavefront's own LDS tile and read back
// as broadcasts; the tile is padded to the unroll width with massless dummies
// placed far from the group.
//
// Bound by VALU issue.  One launch instead of one per class and a scatter:
// the i-particles are read once, the sums written once, and the classes fill
// each other's tails; by itself this took tree + walk + force at 2^20 particles
// from 2069 to 1818 us mixed and 2509 to 2299 us FP64, at 65,536 from 592 to 447
// and 658 to 473.  With what came after, here and in the tree, an evaluation is
// 1.37 ms mixed and 1.69 ms FP64 at 2^20 particles, 0.27 ms mixed at 65,536.
#include "force_common.h"

namespace p3t {

namespace {

// The time of the force phase by class, where it is asked for (A.clk): each
// wavefront's cycles in the near, far and cell loops and in the candidate
// tests, added per workgroup in LDS.  The host divides the launch's time in
// their proportion.
enum { CLK_NEAR, CLK_FAR, CLK_CELL, CLK_CAND, CLK_N };

__device__ __forceinline__ unsigned long long clk_now(const ForceArgs &A) {
  return A.clk ? (unsigned long long)__builtin_readcyclecounter() : 0ull;  // uniform
}

struct GroupHdr {
  long long off;
  int n_cell, n_near, n_far, first, count;
  double cx, cy, cz;
  double px;  // x of the massless entries that pad a tile
};

// Padding lies outside the group's box in x, by a distance that survives
// rounding in any unit of length, so that r > 0 for every particle.  It may lie
// inside a search reach: it is never a neighbour candidate (see near_group).
constexpr double kDummyOffset = 1.0e3;

// Reads the list header of the gi-th group (in work order); every field is
// wave-uniform.  Returns false for a group whose walk overflowed.
__device__ __forceinline__ bool group_header(const ForceArgs &A, int gi, GroupHdr &h) {
  const int q = uniform_first(A.order ? A.order[gi] : gi);
  const GroupList L = A.gl[q];
  h.off = uniform_first64(L.off);
  if (h.off < 0) return false;
  h.n_cell = uniform_first(L.n_cell);
  h.n_near = uniform_first(L.n_near);
  h.n_far = uniform_first(L.n_far);
  const int node = uniform_first(L.node);
  h.first = uniform_first(A.wn[node].first);
  h.count = uniform_first(A.wn[node].count);
  h.cx = 0.5 * (A.wn[node].lo[0] + A.wn[node].hi[0]);
  h.cy = 0.5 * (A.wn[node].lo[1] + A.wn[node].hi[1]);
  h.cz = 0.5 * (A.wn[node].lo[2] + A.wn[node].hi[2]);
  const double hx = A.wn[node].hi[0];
  h.px = hx + kDummyOffset * (1.0 + fabs(hx));
  return true;
}

// LDS ordering inside one wavefront (each wavefront has tiles of its own): a
// wave's LDS operations execute in order, so a compiler fence is enough
// between a write by one lane and a read by another.
__device__ __forceinline__ void tile_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr double kTinyR2 = 1.0e-150;     // floor of r^2 in the near kernel (see there)
// relative margin on reach^2 for neighbour candidates: it covers the rounding
// of r^2 as computed here, so no pair the exact test keeps is missed
constexpr double kCandMargin = 1.0 + 1.0e-12;

// ------------------------------------------------------------------ near
struct NearTile {
  double4 a[WAVE];  // x, y, z, G m
  double2 b[WAVE];  // 1/r_out, reach^2
  float4 f[WAVE];   // MIXED: r_out^2 and reach^2 widened by kMixMargin, G m
  int j[WAVE];      // sorted index (-2: padding)
};

// MIXED screens each pair on the FP32 square of its offset.  Both tests
// take a margin far above the rounding of that square (a few units in
// 2^-24): every pair inside the changeover (y < 1) is flagged, and every
// pair within a search reach is a candidate.  The flagged pairs are then
// evaluated in FP64 (K = 1 for the few beyond the cut-off), and the exact
// test decides the candidates.  The tests compare the bit patterns of
// non-negative floats as integers, which orders them as the floats.
constexpr double kMixMargin = 1.0e-5;

// The FP64 pair term with the changeover for one near pair (r^2 floored,
// see near_group), added to (ax, ay, az).
__device__ __forceinline__ void near_term64(const ForceArgs &A, double dx, double dy, double dz, double r2, double gm,
                                            double invi, double invj, double &ax, double &ay, double &az) {
  // r = 0 (the particle itself, or a coincident pair, which the candidate
  // test reports) gives y ~ 0 < gamma, so K = 0 and the term vanishes
  // exactly: rinv^3 = 1e225 stays finite.  Adding the floor changes no r^2
  // above 1e-134 (it is below half an ulp there) and costs one add instead
  // of a max with operand canonicalisation.
  const double r2s = r2 + kTinyR2;
  const double rinv = rsqrt_pos(r2s);
  const double y = r2s * rinv * fmin(invi, invj);
  const double x = fmin(fmax((y - A.gamma) * A.inv1mg, 0.0), 1.0);
  const double x2 = x * x;
  const double K = x2 * x2 * (35.0 + x * (-84.0 + x * (70.0 - 20.0 * x)));
  const double f = gm * K * rinv * rinv * rinv;
  ax += f * dx;
  ay += f * dy;
  az += f * dz;
}

// MIXED: a pair beyond both cut-offs (y = r / max(r_out) >= 1, so K = 1)
// takes the Newtonian term in FP32 from its FP64 offset, summed per tile in
// FP32 and folded into the FP64 sums; the pairs inside the changeover
// (y < 1, a fraction of a percent of the near lists) are flagged per lane
// and evaluated in FP64 after the tile.  Without MIXED every pair is FP64.
// Neighbour candidates of a wavefront (sorted indices) waiting for the exact
// test of Section 2.3, in LDS.  The tests run 64 at a time, one per lane, as
// soon as that many wait: a candidate costs its lane 18 gathers of 8 bytes, which
// overlap with the pair terms of the CU's other wavefronts.  (A buffer in
// device memory and a launch of its own for the tests were bound by those
// gathers' addresses: 159 us at 2^20 particles, 22 at 65,536; the tests here add
// 60 and 11 us to the force launch.)
struct CandQueue {
  int2 e[2 * WAVE];
};

// tests the first min(n, 64) candidates and reports the neighbours (every
// lane of the wavefront takes part)
__device__ __forceinline__ void test_candidates(const ForceArgs &A, const CandQueue &Q, int n, int lane) {
  bool nb = false;
  int i = 0, j = 0, a = 0, b = 0;
  if (lane < n) {
    i = Q.e[lane].x;
    j = Q.e[lane].y;
    a = A.sid[i];
    b = A.sid[j];
    // a slow member sits at its pre-drift position here; its pairs are
    // tested once its integration has finished
    if (!(A.slow && (A.slow[a] | A.slow[b]))) {
      const double xi = A.sx[i], yi = A.sy[i], zi = A.sz[i], xj = A.sx[j], yj = A.sy[j], zj = A.sz[j];
      if (xi == xj && yi == yj && zi == zj) set_flag(A.cnt, P3T_FLAG_COINCIDENT);
      nb = neighbour_test(xi, yi, zi, A.svx[i], A.svy[i], A.svz[i], A.sm[i], A.sro[i], A.srs[i], xj, yj, zj, A.svx[j],
                          A.svy[j], A.svz[j], A.sm[j], A.sro[j], A.srs[j], A.G, A.rsch2, A.rsch3, A.dt);
    }
  }
  const unsigned long long bal = __ballot(nb);
  if (bal == 0ull) return;  // uniform
  const unsigned long long o0 = wave_fetch_add(&A.cnt->n_pairs, (unsigned long long)__popcll(bal));
  if (nb) {
    mark_close_pair(A, i, j);
    join_pair(A, a, b);
    const unsigned long long q = o0 + popc_below(bal);
    if ((int64_t)q < A.pair_cap)
      A.pairs[q] = make_int2(a, b);
    else
      set_flag(A.cnt, P3T_FLAG_PAIR_OVERFLOW);
  }
}

// How a group's particles lie in the lanes.  Whole: number 64 s + lane in slot
// s, every lane meets every entry of a tile.  Halved (HALF): number 32 s +
// (lane & 31) in both halves of the wavefront, each half meets its half of
// the tile.  Per 64 entries that is 64 evaluations per slot whole and 32
// halved, so 65 to 96 particles cost 3 x 32 halved against 2 x 64 whole, and up
// to 32 cost 32 against 64; two thirds of the groups of a disk hold 65 to
// 96.  Force launch, us, whole -> halved where it is less: 2^20 particles,
// quadrupoles 1325 -> 1175; 200,000, monopoles 225 -> 209; 262,144 281 -> 261.
// Eight wavefronts per group keep the whole layout: those launches wait for
// the longest group, not for arithmetic (2,048 particles: 26.7 whole, 29.4
// halved).  FP64 only: the FP32 sums of the mixed force are formed per tile,
// and splitting a tile would round them differently.
template <bool HALF>
struct Lay {
  static constexpr int STRIDE = HALF ? 32 : WAVE;
  static __device__ __forceinline__ int slot(int lane) { return HALF ? lane & 31 : lane; }
  // entries that each lane loops over in a tile of nt, a multiple of unr
  static __device__ __forceinline__ int span(int nt, int unr) {
    return HALF ? ((nt + 1) / 2 + unr - 1) / unr * unr : min(WAVE, (nt + unr - 1) / unr * unr);
  }
  // entries of the padded tile, and the first one of this lane
  static __device__ __forceinline__ int padded(int span) { return HALF ? 2 * span : span; }
  static __device__ __forceinline__ int first(int lane, int span) { return HALF && lane >= 32 ? span : 0; }
};

// a mask of the lowest k bits (none for k <= 0, all for k >= 32)
__device__ __forceinline__ unsigned low_bits(int k) { return k >= 32 ? ~0u : k <= 0 ? 0u : (1u << k) - 1u; }

// The near terms of the tiles from list position `from` on, every `step`
// positions (multiples of WAVE), added to (ax, ay, az).
template <bool MIXED, int IPL, int UNR, bool HALF>
__device__ __forceinline__ void near_group(const ForceArgs &A, const GroupHdr &h, NearTile &T, int lane, int from,
                                           int step, CandQueue &Q, double *ax, double *ay, double *az,
                                           unsigned long long &cand) {
  int ii[IPL];
  int nq = 0;  // candidates waiting, fewer than 64 between tiles
  double xi[IPL], yi[IPL], zi[IPL], invi[IPL], rch2[IPL];
  int ro2q[IPL], rch2q[IPL];  // MIXED: bit patterns of the widened FP32 squares
#pragma unroll
  for (int s = 0; s < IPL; ++s) {
    const int k = Lay<HALF>::slot(lane) + Lay<HALF>::STRIDE * s;
    ii[s] = k < h.count ? h.first + k : -1;
    const int i = ii[s] >= 0 ? ii[s] : h.first;
    // an empty slot sits beyond the padding entries
    xi[s] = ii[s] >= 0 ? A.sx[i] : 2.0 * h.px - h.cx;
    yi[s] = A.sy[i];
    zi[s] = A.sz[i];
    invi[s] = A.sinv[i];
    rch2[s] = A.sreach[i] * A.sreach[i] * kCandMargin;
    if constexpr (MIXED) {
      const double ro = A.sro[i], r = A.sreach[i];
      ro2q[s] = __float_as_int((float)(ro * ro * (1.0 + kMixMargin)));
      rch2q[s] = __float_as_int((float)(r * r * (1.0 + kMixMargin)));
    }
  }
  const int32_t *Ln = A.pool + h.off + h.n_cell;
  // the next tile's entry of this lane is loaded into registers while the
  // current tile is evaluated (its gathers are the kernel's memory latency)
  double4 na;
  double2 nb;
  float4 nf;
  int nj = -2;
  auto fetch = [&](int t0) {
    const int nt = min(WAVE, h.n_near - t0);
    const int ntp = Lay<HALF>::padded(Lay<HALF>::span(nt, UNR));
    if (lane < nt) {
      const int j = Ln[t0 + lane];
      const double r = A.sreach[j];
      na = make_double4(A.sx[j], A.sy[j], A.sz[j], A.G * A.sm[j]);
      nb = make_double2(A.sinv[j], r * r * kCandMargin);
      if constexpr (MIXED) {
        const double ro = A.sro[j];
        nf = make_float4((float)(ro * ro * (1.0 + kMixMargin)), (float)(r * r * (1.0 + kMixMargin)), (float)na.w, 0.0f);
      }
      nj = j;
    } else if (lane < ntp) {
      // padding: massless, without a reach or a cut-off of its own
      na = make_double4(h.px, h.cy, h.cz, 0.0);
      nb = make_double2(1.0, 0.0);
      nf = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      nj = -2;
    }
  };
  if (h.n_near > from) fetch(from);
  for (int t0 = from; t0 < h.n_near; t0 += step) {
    const int nt = min(WAVE, h.n_near - t0);
    const int span = Lay<HALF>::span(nt, UNR), ntp = Lay<HALF>::padded(span), e0 = Lay<HALF>::first(lane, span);
    tile_sync();
    if (lane < ntp) {
      T.a[lane] = na;
      T.b[lane] = nb;
      if constexpr (MIXED) T.f[lane] = nf;
      T.j[lane] = nj;
    }
    tile_sync();
    if (t0 + step < h.n_near) fetch(t0 + step);
    unsigned cm[2][IPL], chg_m[2][IPL];
    float tx[IPL], ty[IPL], tz[IPL];
#pragma unroll
    for (int s = 0; s < IPL; ++s) tx[s] = ty[s] = tz[s] = 0.0f;
#pragma unroll
    for (int half = 0; half < (HALF ? 1 : 2); ++half) {
#pragma unroll
      for (int s = 0; s < IPL; ++s) cm[half][s] = chg_m[half][s] = 0u;
      const int lo = half * 32, hi = min(span, lo + 32);
      for (int jj = lo; jj < hi; jj += UNR) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const double4 a = T.a[e0 + jj + u];
          const int jidx = T.j[e0 + jj + u];
          const unsigned bit = 1u << ((jj + u) & 31);
          if constexpr (MIXED) {
            const float4 fj = T.f[jj + u];
            const int ro2j = __float_as_int(fj.x), rch2j = __float_as_int(fj.y);
#pragma unroll
            for (int s = 0; s < IPL; ++s) {
              const double dx = a.x - xi[s], dy = a.y - yi[s], dz = a.z - zi[s];
              const float fdx = (float)dx, fdy = (float)dy, fdz = (float)dz;
              const float r2f = fdx * fdx + fdy * fdy + fdz * fdz;
              const int r2q = __float_as_int(r2f);
              // inside the changeover of either side (or r = 0): FP64 below
              const bool chg = (r2q < ro2q[s]) | (r2q < ro2j);
              const float ri = __frsqrt_rn(r2f);
              const float f = chg ? 0.0f : fj.z * ri * ri * ri;
              tx[s] += f * fdx;
              ty[s] += f * fdy;
              tz[s] += f * fdz;
              const bool other = jidx != ii[s];
              chg_m[half][s] |= (chg & other) ? bit : 0u;
              // evaluated without short-circuit, so no branch per pair
              const bool cand = other & ((r2q <= rch2q[s]) | (r2q <= rch2j));
              cm[half][s] |= cand ? bit : 0u;
            }
          } else {
            const double2 b = T.b[e0 + jj + u];
            const long long rch2j = __double_as_longlong(b.y);
#pragma unroll
            for (int s = 0; s < IPL; ++s) {
              const double dx = a.x - xi[s], dy = a.y - yi[s], dz = a.z - zi[s];
              const double r2 = dx * dx + dy * dy + dz * dz;
              near_term64(A, dx, dy, dz, r2, a.w, invi[s], b.x, ax[s], ay[s], az[s]);
              // reach^2 of both sides carry the candidate margin already;
              // compared as bit patterns of non-negative doubles (ordered as
              // the doubles), without short-circuit, so no branch per pair
              const long long r2q = __double_as_longlong(r2);
              const bool cand = (jidx != ii[s]) & ((r2q <= __double_as_longlong(rch2[s])) | (r2q <= rch2j));
              cm[half][s] |= cand ? bit : 0u;
            }
          }
        }
      }
    }
    if constexpr (MIXED) {
      // the changeover pairs of this tile in FP64, then the tile's FP32 sums
#pragma unroll
      for (int s = 0; s < IPL; ++s) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          unsigned m = ii[s] >= 0 ? chg_m[half][s] : 0u;
          while (m != 0u) {
            const int q = 32 * half + __ffs(m) - 1;
            m &= m - 1u;
            const double4 a = T.a[q];
            const double dx = a.x - xi[s], dy = a.y - yi[s], dz = a.z - zi[s];
            const double r2 = dx * dx + dy * dy + dz * dz;
            near_term64(A, dx, dy, dz, r2, a.w, invi[s], T.b[q].x, ax[s], ay[s], az[s]);
          }
        }
        ax[s] += (double)tx[s];
        ay[s] += (double)ty[s];
        az[s] += (double)tz[s];
      }
    }
    // hand this tile's candidates to the exact test: one of each lane a round.
    // The padding behind the lane's entries is masked out: it has no particle
    // index, and a reach of a thousand units of length may cover it.
    if (A.collect) {
      const unsigned real0 = low_bits(nt - e0), real1 = low_bits(nt - e0 - 32);
#pragma unroll
      for (int s = 0; s < IPL; ++s) {
        unsigned m0 = ii[s] >= 0 ? cm[0][s] & real0 : 0u, m1 = !HALF && ii[s] >= 0 ? cm[1][s] & real1 : 0u;
        for (;;) {
          const bool has = (m0 | m1) != 0u;
          const unsigned long long bal = __ballot(has);
          if (bal == 0ull) break;  // uniform
          if (has) {
            const int q = m0 ? __ffs(m0) - 1 : 31 + __ffs(m1);
            if (m0)
              m0 &= m0 - 1u;
            else
              m1 &= m1 - 1u;
            Q.e[nq + popc_below(bal)] = make_int2(ii[s], T.j[e0 + q]);
          }
          nq += (int)__popcll(bal);
          if (nq >= WAVE) {
            tile_sync();
            const unsigned long long c0 = clk_now(A);
            test_candidates(A, Q, WAVE, lane);
            cand += clk_now(A) - c0;
            const int2 rest = Q.e[WAVE + lane];
            tile_sync();
            Q.e[lane] = rest;
            nq -= WAVE;
          }
        }
      }
    }
  }
  if (nq > 0) {
    tile_sync();
    const unsigned long long c0 = clk_now(A);
    test_candidates(A, Q, nq, lane);
    cand += clk_now(A) - c0;
  }
}

// ------------------------------------------------------------------ far
union FarTile {
  double4 d[WAVE];  // x, y, z, G m
  float4 f[WAVE];   // offsets from the group centre, G m
};

template <bool MIXED, int IPL, int UNR, bool HALF>
__device__ __forceinline__ void far_group(const ForceArgs &A, const GroupHdr &h, FarTile &T, int lane, int from,
                                          int step, double *ax, double *ay, double *az) {
  double xi[IPL], yi[IPL], zi[IPL];
#pragma unroll
  for (int s = 0; s < IPL; ++s) {
    const int k = Lay<HALF>::slot(lane) + Lay<HALF>::STRIDE * s;
    const int i = k < h.count ? h.first + k : h.first;
    xi[s] = A.sx[i];
    yi[s] = A.sy[i];
    zi[s] = A.sz[i];
  }
  const int32_t *Lf = A.pool + h.off + h.n_cell + h.n_near;
  if (!MIXED) {
    for (int t0 = from; t0 < h.n_far; t0 += step) {
      const int nt = min(WAVE, h.n_far - t0);
      const int span = Lay<HALF>::span(nt, UNR), ntp = Lay<HALF>::padded(span), e0 = Lay<HALF>::first(lane, span);
      tile_sync();
      if (lane < nt) {
        const int j = Lf[t0 + lane];
        T.d[lane] = make_double4(A.sx[j], A.sy[j], A.sz[j], A.G * A.sm[j]);
      } else if (lane < ntp) {
        T.d[lane] = make_double4(h.px, h.cy, h.cz, 0.0);
      }
      tile_sync();
      for (int jj = 0; jj < span; jj += UNR) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const double4 a = T.d[e0 + jj + u];
#pragma unroll
          for (int s = 0; s < IPL; ++s) {
            const double dx = a.x - xi[s], dy = a.y - yi[s], dz = a.z - zi[s];
            const double r2 = dx * dx + dy * dy + dz * dz;
            const double rinv = rsqrt_pos(r2);  // r > 0: beyond the group's reach
            const double f = a.w * rinv * rinv * rinv;
            ax[s] += f * dx;
            ay[s] += f * dy;
            az[s] += f * dz;
          }
        }
      }
    }
  } else {
    float fxi[IPL], fyi[IPL], fzi[IPL], hx[IPL], hy[IPL], hz[IPL], lx[IPL], ly[IPL], lz[IPL];
#pragma unroll
    for (int s = 0; s < IPL; ++s) {
      fxi[s] = (float)(xi[s] - h.cx);
      fyi[s] = (float)(yi[s] - h.cy);
      fzi[s] = (float)(zi[s] - h.cz);
      hx[s] = hy[s] = hz[s] = lx[s] = ly[s] = lz[s] = 0.0f;
    }
    for (int t0 = from; t0 < h.n_far; t0 += step) {
      const int nt = min(WAVE, h.n_far - t0);
      const int ntp = min(WAVE, (nt + UNR - 1) / UNR * UNR);
      tile_sync();
      if (lane < nt) {
        const int j = Lf[t0 + lane];
        T.f[lane] = make_float4((float)(A.sx[j] - h.cx), (float)(A.sy[j] - h.cy), (float)(A.sz[j] - h.cz),
                                (float)(A.G * A.sm[j]));
      } else if (lane < ntp) {
        T.f[lane] = make_float4((float)(h.px - h.cx), 0.0f, 0.0f, 0.0f);
      }
      tile_sync();
      float tx[IPL], ty[IPL], tz[IPL];
#pragma unroll
      for (int s = 0; s < IPL; ++s) tx[s] = ty[s] = tz[s] = 0.0f;
      for (int jj = 0; jj < ntp; jj += UNR) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const float4 a = T.f[jj + u];
#pragma unroll
          for (int s = 0; s < IPL; ++s) {
            const float dx = a.x - fxi[s], dy = a.y - fyi[s], dz = a.z - fzi[s];
            const float r2 = dx * dx + dy * dy + dz * dz;
            const float rinv = __frsqrt_rn(r2);
            const float f = a.w * rinv * rinv * rinv;
            tx[s] += f * dx;
            ty[s] += f * dy;
            tz[s] += f * dz;
          }
        }
      }
#pragma unroll
      for (int s = 0; s < IPL; ++s) {
        two_sum_acc(hx[s], lx[s], tx[s]);
        two_sum_acc(hy[s], ly[s], ty[s]);
        two_sum_acc(hz[s], lz[s], tz[s]);
      }
    }
#pragma unroll
    for (int s = 0; s < IPL; ++s) {
      ax[s] += (double)hx[s] + (double)lx[s];
      ay[s] += (double)hy[s] + (double)ly[s];
      az[s] += (double)hz[s] + (double)lz[s];
    }
  }
}

// ------------------------------------------------------------------ cells
union CellTile {
  struct {
    double4 a[WAVE];  // centre of mass, G M
    double4 qa[WAVE];  // G q_xx, q_yy, q_zz, q_xy
    double2 qb[WAVE];  // G q_xz, q_yz
  } d;
  struct {
    float4 a[WAVE];
    float4 qa[WAVE];
    float2 qb[WAVE];
  } f;
};

union ForceTile {
  NearTile near;
  FarTile far;
  CellTile cell;
  double sum[3][2 * WAVE];  // a wavefront's sums of the group
};

template <typename R>
__device__ __forceinline__ R fma_r(R a, R b, R c) {
  return __builtin_fma(a, b, c);
}
template <>
__device__ __forceinline__ float fma_r<float>(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}

// The cell term added to (ax, ay, az):
//   a = G [ M d / r^3 - Q d / r^5 + (5/2) (d.Q d) d / r^7 ],  d = X_c - x_i,
// as d (G M / r^3 + (5/2) (d.Q d) / r^7) - Q d / r^5, so that each
// component is two fused multiply-adds onto the running sum.
template <typename R>
__device__ __forceinline__ void cell_acc(R dx, R dy, R dz, R gm, R q0, R q1, R q2, R q3, R q4, R q5, bool quad,
                                         R rinv, R &ax, R &ay, R &az) {
  const R rinv2 = rinv * rinv;
  const R rinv3 = rinv * rinv2;
  if (!quad) {
    const R f = gm * rinv3;
    ax = fma_r(f, dx, ax);
    ay = fma_r(f, dy, ay);
    az = fma_r(f, dz, az);
    return;
  }
  const R qx = fma_r(q4, dz, fma_r(q3, dy, q0 * dx));
  const R qy = fma_r(q5, dz, fma_r(q1, dy, q3 * dx));
  const R qz = fma_r(q2, dz, fma_r(q5, dy, q4 * dx));
  const R dqd = fma_r(dz, qz, fma_r(dy, qy, dx * qx));
  const R rinv5 = rinv3 * rinv2;
  const R f = fma_r(gm, rinv3, R(2.5) * dqd * (rinv5 * rinv2));
  ax = fma_r(-qx, rinv5, fma_r(f, dx, ax));
  ay = fma_r(-qy, rinv5, fma_r(f, dy, ay));
  az = fma_r(-qz, rinv5, fma_r(f, dz, az));
}

template <bool MIXED, bool QUAD, int IPL, int UNR, bool HALF>
__device__ __forceinline__ void cell_group(const ForceArgs &A, const GroupHdr &h, CellTile &T, int lane, int from,
                                           int step, double *ax, double *ay, double *az) {
  double xi[IPL], yi[IPL], zi[IPL];
#pragma unroll
  for (int s = 0; s < IPL; ++s) {
    const int k = Lay<HALF>::slot(lane) + Lay<HALF>::STRIDE * s;
    const int i = k < h.count ? h.first + k : h.first;
    xi[s] = A.sx[i];
    yi[s] = A.sy[i];
    zi[s] = A.sz[i];
  }
  const int32_t *Lc = A.pool + h.off;
  const double G = A.G;
  if (!MIXED) {
    for (int t0 = from; t0 < h.n_cell; t0 += step) {
      const int nt = min(WAVE, h.n_cell - t0);
      const int span = Lay<HALF>::span(nt, UNR), ntp = Lay<HALF>::padded(span), e0 = Lay<HALF>::first(lane, span);
      tile_sync();
      if (lane < nt) {
        const CellMom c = A.cm[Lc[t0 + lane]];
        T.d.a[lane] = make_double4(c.com[0], c.com[1], c.com[2], G * c.mass);
        if (QUAD) {
          T.d.qa[lane] = make_double4(G * c.q[0], G * c.q[1], G * c.q[2], G * c.q[3]);
          T.d.qb[lane] = make_double2(G * c.q[4], G * c.q[5]);
        }
      } else if (lane < ntp) {
        T.d.a[lane] = make_double4(h.px, h.cy, h.cz, 0.0);
        if (QUAD) {
          T.d.qa[lane] = make_double4(0.0, 0.0, 0.0, 0.0);
          T.d.qb[lane] = make_double2(0.0, 0.0);
        }
      }
      tile_sync();
      for (int jj = 0; jj < span; jj += UNR) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const double4 a = T.d.a[e0 + jj + u];
          double4 qa = make_double4(0.0, 0.0, 0.0, 0.0);
          double2 qb = make_double2(0.0, 0.0);
          if (QUAD) {
            qa = T.d.qa[e0 + jj + u];
            qb = T.d.qb[e0 + jj + u];
          }
#pragma unroll
          for (int s = 0; s < IPL; ++s) {
            const double dx = a.x - xi[s], dy = a.y - yi[s], dz = a.z - zi[s];
            const double r2 = dx * dx + dy * dy + dz * dz;
            cell_acc<double>(dx, dy, dz, a.w, qa.x, qa.y, qa.z, qa.w, qb.x, qb.y, QUAD, rsqrt_pos(r2), ax[s], ay[s],
                             az[s]);
          }
        }
      }
    }
  } else {
    float fxi[IPL], fyi[IPL], fzi[IPL], hx[IPL], hy[IPL], hz[IPL], lx[IPL], ly[IPL], lz[IPL];
#pragma unroll
    for (int s = 0; s < IPL; ++s) {
      fxi[s] = (float)(xi[s] - h.cx);
      fyi[s] = (float)(yi[s] - h.cy);
      fzi[s] = (float)(zi[s] - h.cz);
      hx[s] = hy[s] = hz[s] = lx[s] = ly[s] = lz[s] = 0.0f;
    }
    for (int t0 = from; t0 < h.n_cell; t0 += step) {
      const int nt = min(WAVE, h.n_cell - t0);
      const int ntp = min(WAVE, (nt + UNR - 1) / UNR * UNR);
      tile_sync();
      if (lane < nt) {
        const CellMom c = A.cm[Lc[t0 + lane]];
        T.f.a[lane] = make_float4((float)(c.com[0] - h.cx), (float)(c.com[1] - h.cy), (float)(c.com[2] - h.cz),
                                  (float)(G * c.mass));
        if (QUAD) {
          T.f.qa[lane] = make_float4((float)(G * c.q[0]), (float)(G * c.q[1]), (float)(G * c.q[2]),
                                     (float)(G * c.q[3]));
          T.f.qb[lane] = make_float2((float)(G * c.q[4]), (float)(G * c.q[5]));
        }
      } else if (lane < ntp) {
        T.f.a[lane] = make_float4((float)(h.px - h.cx), 0.0f, 0.0f, 0.0f);
        if (QUAD) {
          T.f.qa[lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
          T.f.qb[lane] = make_float2(0.0f, 0.0f);
        }
      }
      tile_sync();
      float tx[IPL], ty[IPL], tz[IPL];
#pragma unroll
      for (int s = 0; s < IPL; ++s) tx[s] = ty[s] = tz[s] = 0.0f;
      for (int jj = 0; jj < ntp; jj += UNR) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const float4 a = T.f.a[jj + u];
          float4 qa = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
          float2 qb = make_float2(0.0f, 0.0f);
          if (QUAD) {
            qa = T.f.qa[jj + u];
            qb = T.f.qb[jj + u];
          }
#pragma unroll
          for (int s = 0; s < IPL; ++s) {
            const float dx = a.x - fxi[s], dy = a.y - fyi[s], dz = a.z - fzi[s];
            const float r2 = dx * dx + dy * dy + dz * dz;
            cell_acc<float>(dx, dy, dz, a.w, qa.x, qa.y, qa.z, qa.w, qb.x, qb.y, QUAD, __frsqrt_rn(r2), tx[s], ty[s],
                            tz[s]);
          }
        }
      }
#pragma unroll
      for (int s = 0; s < IPL; ++s) {
        two_sum_acc(hx[s], lx[s], tx[s]);
        two_sum_acc(hy[s], ly[s], ty[s]);
        two_sum_acc(hz[s], lz[s], tz[s]);
      }
    }
#pragma unroll
    for (int s = 0; s < IPL; ++s) {
      ax[s] += (double)hx[s] + (double)lx[s];
      ay[s] += (double)hy[s] + (double)ly[s];
      az[s] += (double)hz[s] + (double)lz[s];
    }
  }
}

// ------------------------------------------------------------------ one launch, W wavefronts per group
// The three classes of a group's list in one launch: its tiles (near, then
// far, then cells) are dealt round robin to the W wavefronts of a workgroup,
// each with a tile of LDS of its own; the wavefronts' sums are added in
// wavefront order and written in the caller's order.  Deterministic: the same
// tiles in the same wavefronts whatever the grid.
// a + the value of the lane 32 lanes away
__device__ __forceinline__ double other_half_add(double a) {
  const uint64_t u = (uint64_t)__double_as_longlong(a);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
  return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}

template <bool MIXED, bool QUAD, int IPL, int UNR, int W, bool HALF = false>
__device__ __forceinline__ void all_group(const ForceArgs &A, const GroupHdr &h, ForceTile *T, CandQueue *Q,
                                          unsigned long long *clk, int lane, int w) {
  double ax[IPL] = {}, ay[IPL] = {}, az[IPL] = {};
  const int nt = (h.n_near + WAVE - 1) / WAVE, ft = (h.n_far + WAVE - 1) / WAVE;
  // first far / cell tile of wavefront w: the tiles are numbered through
  const int f0 = ((w - nt) % W + W) % W, c0 = ((w - nt - ft) % W + W) % W;
  unsigned long long cand = 0;
  const unsigned long long t0 = clk_now(A);
  near_group<MIXED, IPL, UNR, HALF>(A, h, T[w].near, lane, WAVE * w, WAVE * W, Q[w], ax, ay, az, cand);
  const unsigned long long t1 = clk_now(A);
  far_group<MIXED, IPL, UNR, HALF>(A, h, T[w].far, lane, WAVE * f0, WAVE * W, ax, ay, az);
  const unsigned long long t2 = clk_now(A);
  cell_group<MIXED, QUAD, IPL, UNR, HALF>(A, h, T[w].cell, lane, WAVE * c0, WAVE * W, ax, ay, az);
  if (A.clk && lane == 0) {
    atomicAdd(&clk[CLK_NEAR], t1 - t0 - cand);
    atomicAdd(&clk[CLK_FAR], t2 - t1);
    atomicAdd(&clk[CLK_CELL], clk_now(A) - t2);
    atomicAdd(&clk[CLK_CAND], cand);
  }
  tile_sync();
#pragma unroll
  for (int s = 0; s < IPL; ++s) {
    if (HALF) {
      ax[s] = other_half_add(ax[s]);
      ay[s] = other_half_add(ay[s]);
      az[s] = other_half_add(az[s]);
    }
    const int k = Lay<HALF>::slot(lane) + Lay<HALF>::STRIDE * s;  // (both halves hold the same)
    T[w].sum[0][k] = ax[s];
    T[w].sum[1][k] = ay[s];
    T[w].sum[2][k] = az[s];
  }
  __syncthreads();
  for (int k = WAVE * w + lane; k < h.count; k += WAVE * W) {
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < W; ++q) {
#pragma unroll
      for (int d = 0; d < 3; ++d) v[d] += T[q].sum[d][k];
    }
    const int64_t o = A.sid[h.first + k];
    A.acc[o] = v[0];
    A.acc[A.n + o] = v[1];
    A.acc[2 * A.n + o] = v[2];
    if (!(isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2]))) set_flag(A.cnt, P3T_FLAG_NAN);
  }
}

// wavefronts per SIMD that the registers allow: FP64 with three slots of half
// wavefronts needs 167 (unroll 2), and bounded to the 128 of four wavefronts it
// spilled: 200,000 particles 218 us with four, 209 with three; 2^20 1184 and 1175
constexpr int min_waves(int unr, bool mixed, int w) {
  return unr == 2 && !mixed && w == 4 ? 3 : unr <= 2 ? 4 : unr <= 4 ? 3 : 2;
}

template <bool MIXED, bool QUAD, int UNR, int W>
__global__ __launch_bounds__(WAVE *W, min_waves(UNR, MIXED, W)) void k_force_all(ForceArgs A) {
  __shared__ ForceTile T[W];
  __shared__ CandQueue Q[W];
  __shared__ unsigned long long clk[CLK_N];
  __shared__ int next;
  if (A.clk) {  // uniform
    if (threadIdx.x < CLK_N) clk[threadIdx.x] = 0ull;
    __syncthreads();
  }
  const int lane = threadIdx.x & (WAVE - 1), w = uniform_first(threadIdx.x / WAVE);
  const int ngroups = uniform_first(min((int)A.cnt->n_groups, A.ngroups_bound));
  unsigned long long nn = 0, nf = 0, nc = 0;  // this workgroup's interactions, added once at its end
  for (int iter = 0;; ++iter) {
    int gi;
    if (A.persistent) {
      __syncthreads();  // also: the sums of the last group are read
      if (threadIdx.x == 0) next = (int)atomicAdd(A.queue, 1ull);
      __syncthreads();
      gi = uniform_first(next);
    } else {
      if (iter > 0) __syncthreads();  // the sums of the last group are read
      const long long k = (long long)iter * gridDim.x + blockIdx.x;
      gi = k < ngroups ? (int)k : ngroups;
    }
    if (gi >= ngroups) break;
    GroupHdr h;
    if (!group_header(A, gi, h)) continue;
    if (!MIXED && W == 4 && h.count > WAVE && h.count <= 96)
      all_group<false, QUAD, 3, UNR, W, true>(A, h, T, Q, clk, lane, w);
    else if (!MIXED && W == 4 && h.count <= 32)
      all_group<false, QUAD, 1, UNR, W, true>(A, h, T, Q, clk, lane, w);
    else if (h.count > WAVE)
      all_group<MIXED, QUAD, 2, UNR, W>(A, h, T, Q, clk, lane, w);
    else
      all_group<MIXED, QUAD, 1, UNR, W>(A, h, T, Q, clk, lane, w);
    const unsigned long long ni = (unsigned long long)h.count;
    nn += ni * (unsigned long long)h.n_near - ni;
    nf += ni * (unsigned long long)h.n_far;
    nc += ni * (unsigned long long)h.n_cell;
  }
  if (threadIdx.x == 0) {
    if (nn) atomicAdd(&A.cnt->n_near, nn);
    if (nf) atomicAdd(&A.cnt->n_far, nf);
    if (nc) atomicAdd(&A.cnt->n_cell, nc);
  }
  if (A.clk) {  // uniform
    __syncthreads();
    if (threadIdx.x < CLK_N) atomicAdd(&A.clk[threadIdx.x], clk[threadIdx.x]);
  }
}

// Wavefronts per group.  A group's list holds about a dozen tiles, and a
// wavefront's tile is 64 entries x 64 or 128 particles, so with one wavefront
// per group a disk of 65,536 particles (750 groups) leaves a quarter of the
// 1024 SIMDs idle and the others with one wavefront each.  Measured (tree +
// walk + force, mixed quadrupole, us; groups counted as n / (2/3 n_group_max)):
//   particles   groups   W = 2    4     8    16
//     16,384      190      411   388   370     -
//     65,536      750      503   467   447   478
//    131,072     1500      599   581   594   634
//  1,048,576   12,000     1829  1818  2236  2584
// Above 1200 groups four are as good as any, below eight are.
constexpr int64_t kGroupsWide = 1200;

template <int UNR, int W>
void launch_all(p3t_ctx *c, const ForceArgs &A, unsigned nonpersistent_grid) {
  const bool mixed = c->P.precision == 1, quad = c->P.multipole == 2;
  auto go = [&](auto kernel) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, WAVE * W, 0) != hipSuccess || nb <= 0) nb = 1;
    nb = std::min(nb, std::max(1, c->fcfg.waves_per_cu / W));
    const unsigned g = A.persistent ? (unsigned)(c->n_cu * nb) : nonpersistent_grid;
    hipLaunchKernelGGL(kernel, dim3(g), dim3(WAVE * W), 0, c->stream, A);
  };
  if (mixed && quad)
    go(k_force_all<true, true, UNR, W>);
  else if (mixed)
    go(k_force_all<true, false, UNR, W>);
  else if (quad)
    go(k_force_all<false, true, UNR, W>);
  else
    go(k_force_all<false, false, UNR, W>);
}

template <int UNR>
hipError_t launch_split(p3t_ctx *c, ForceArgs A, unsigned nonpersistent_grid, double *acc3) {
  A.acc = acc3;
  A.queue = &c->cnt->queue;
  A.clk = c->timing ? c->cnt->force_clk : nullptr;
  const int64_t groups = c->n / std::max(1, 2 * c->P.n_group_max / 3);
  // One workgroup per group, without launching the host's bound of n (a
  // replayed evaluation) to find most of them idle: above four times the
  // expected groups a workgroup takes several.  2^19 particles replayed, mixed:
  // 1771 -> 935 us.
  nonpersistent_grid = (unsigned)std::min<int64_t>(nonpersistent_grid, 4 * groups + 1024);
  if (groups < kGroupsWide)
    launch_all<UNR, 8>(c, A, nonpersistent_grid);
  else
    launch_all<UNR, 4>(c, A, nonpersistent_grid);
  ev_record(c, 11);
  return hipGetLastError();
}

}  // namespace

hipError_t soft_force_split(p3t_ctx *c, const ForceArgs &A, unsigned nonpersistent_grid, double *acc3) {
  switch (c->fcfg.unroll) {
    case 1:
      return launch_split<1>(c, A, nonpersistent_grid, acc3);
    case 2:
      return launch_split<2>(c, A, nonpersistent_grid, acc3);
    case 8:
      return launch_split<8>(c, A, nonpersistent_grid, acc3);
    default:
      return launch_split<4>(c, A, nonpersistent_grid, acc3);
  }
}

}  // namespace p3t
