// util.hip -- device-wide building blocks: exclusive scans, a stable LSD radix
// sort of 64-bit keys with 32-bit values, fills and the soft kick.
#include <algorithm>

#include "p3t_internal.h"

namespace p3t {

// ------------------------------------------------------------------ scan
constexpr int SCAN_T = 256;
constexpr int SCAN_I = 16;
constexpr int SCAN_TILE = SCAN_T * SCAN_I;

template <typename Tin>
__global__ __launch_bounds__(SCAN_T) void k_scan_sums(const Tin *__restrict__ in, int64_t n, int64_t *__restrict__ sums) {
  __shared__ int64_t ws[SCAN_T / WAVE];
  const int t = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
  int64_t s = 0;
#pragma unroll
  for (int r = 0; r < SCAN_I; ++r) {
    int64_t k = base + (int64_t)r * SCAN_T + t;
    if (k < n) s += (int64_t)in[k];
  }
  s = wave_sum(s);
  if ((t & (WAVE - 1)) == 0) ws[t / WAVE] = s;
  __syncthreads();
  if (t == 0) {
    int64_t tot = 0;
    for (int w = 0; w < SCAN_T / WAVE; ++w) tot += ws[w];
    sums[blockIdx.x] = tot;
  }
}

// exclusive scan of one tile (+ block offset).  If total_out, out[n] = total.
template <typename Tin, typename Tout>
__global__ __launch_bounds__(SCAN_T) void k_scan_down(const Tin *__restrict__ in, Tout *__restrict__ out, int64_t n,
                                                      const int64_t *__restrict__ offs, int total_out) {
  __shared__ int64_t buf[SCAN_TILE];
  __shared__ int64_t ws[SCAN_T / WAVE];
  const int t = threadIdx.x, w = t / WAVE, l = t & (WAVE - 1);
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
#pragma unroll
  for (int r = 0; r < SCAN_I; ++r) {
    int64_t k = base + (int64_t)r * SCAN_T + t;
    buf[r * SCAN_T + t] = k < n ? (int64_t)in[k] : 0;
  }
  __syncthreads();
  int64_t s = 0;
#pragma unroll
  for (int q = 0; q < SCAN_I; ++q) s += buf[t * SCAN_I + q];
  int64_t incl = s;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    int64_t v = __shfl_up(incl, o, WAVE);
    if (l >= o) incl += v;
  }
  if (l == WAVE - 1) ws[w] = incl;
  __syncthreads();
  int64_t run = (offs ? offs[blockIdx.x] : 0) + incl - s;
  for (int q = 0; q < w; ++q) run += ws[q];
#pragma unroll
  for (int q = 0; q < SCAN_I; ++q) {
    int64_t v = buf[t * SCAN_I + q];
    buf[t * SCAN_I + q] = run;
    run += v;
    // the thread holding element n-1 writes the grand total to out[n]
    if (total_out && base + t * SCAN_I + q == n - 1) out[n] = (Tout)run;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < SCAN_I; ++r) {
    int64_t k = base + (int64_t)r * SCAN_T + t;
    if (k < n) out[k] = (Tout)buf[r * SCAN_T + t];
  }
}

__global__ void k_write_zero_i64(int64_t *p) { *p = 0; }

int64_t scan_tmp_need(int64_t n) {
  int64_t need = 0;
  while (n > SCAN_TILE) {
    n = (n + SCAN_TILE - 1) / SCAN_TILE;
    need += n;
  }
  return need + 16;
}

template <typename Tin, typename Tout>
static hipError_t scan_impl(const Tin *in, Tout *out, int64_t n, int total_out, int64_t *tmp, int64_t tmp_cap,
                            hipStream_t s) {
  if (n <= 0) {
    if (total_out) hipLaunchKernelGGL(k_write_zero_i64, dim3(1), dim3(1), 0, s, (int64_t *)out);
    return hipGetLastError();
  }
  int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
  if (nb == 1) {
    hipLaunchKernelGGL((k_scan_down<Tin, Tout>), dim3(1), dim3(SCAN_T), 0, s, in, out, n, (const int64_t *)nullptr,
                       total_out);
    return hipGetLastError();
  }
  if (tmp_cap < nb) return hipErrorInvalidValue;
  int64_t *sums = tmp;
  hipLaunchKernelGGL((k_scan_sums<Tin>), dim3((unsigned)nb), dim3(SCAN_T), 0, s, in, n, sums);
  hipError_t e = scan_impl<int64_t, int64_t>(sums, sums, nb, 0, tmp + nb, tmp_cap - nb, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_scan_down<Tin, Tout>), dim3((unsigned)nb), dim3(SCAN_T), 0, s, in, out, n,
                     (const int64_t *)sums, total_out);
  return hipGetLastError();
}

hipError_t scan_i32_to_i64(const int32_t *in, int64_t *out, int64_t n, int64_t *tmp, int64_t tmp_cap, hipStream_t s) {
  return scan_impl<int32_t, int64_t>(in, out, n, 1, tmp, tmp_cap, s);
}

// ------------------------------------------------------------------ radix sort
// Stable LSD radix sort, 8-bit digits, one launch per pass.  A workgroup of
// 1024 threads takes a tile of 1024, 2048 or 4096 keys: every wavefront ranks
// its own keys with ballots and counters of its own (no barrier per round),
// the tile is ordered in LDS and written out in runs of equal digits.
// The pass's tile histogram (hist[tile][digit]) is complete when it starts.
// Up to RS_CHAIN keys the pass before, which knows where each key lands, adds
// the key's next digit to it (the first one comes with the keys): one launch
// per pass.  More keys make that an atomic per key too many, and a launch of its
// own counts each tile in LDS.  Up to RS_SELF tiles every workgroup sums the
// histogram's columns itself (256 rows of 1 KB, 3 us); more tiles take one
// launch more per pass that scans the columns.
//   48-bit keys with values, all passes, us: 2,048 keys 34, 65,536 46, 262,144
// 68, 2^20 118 (one histogram, one column or row scan and one scatter per pass of
// 2048-key tiles: 82, 116, 105, 144).  The lines, both sides in us: chained
// against counted 65,537 keys 46 and 50, 98,304 62 and 61, 131,072 60 and 55;
// columns summed against scanned 2^20 118 and 135, 1,250,000 159 and 158, 2^21
// 204 and 187; tiles below.
constexpr int RS_T = 1024, RS_W = RS_T / WAVE;
constexpr int RS_SELF = 256;
constexpr int64_t RS_CHAIN = 3 << 15;

// keys per thread: small tiles while the chip is not full (tiles of 1024, 2048
// and 4096 keys: 131,072 keys 55, 59 and 83 us, 262,144 72, 68 and 80, 2^19 -, 89
// and 93), and at most RS_SELF of them up to 2^20 keys
static int radix_items(int64_t n) { return n <= (1 << 17) ? 1 : n <= (1 << 19) ? 2 : 4; }

RadixPlan radix_plan(int64_t n) {
  RadixPlan p;
  p.tile = RS_T * radix_items(n);
  p.ntiles = (int)((n + p.tile - 1) / p.tile);
  p.chain = n <= RS_CHAIN;
  return p;
}

// one pass's histogram, a workgroup per tile (no clearing before)
__global__ __launch_bounds__(RS_T) void k_radix_tile_hist(const uint64_t *__restrict__ kin, int64_t n, int shift,
                                                          int tile, uint32_t *__restrict__ hist) {
  __shared__ uint32_t h[256];
  const int t = threadIdx.x;
  if (t < 256) h[t] = 0u;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * tile;
#pragma unroll 4
  for (int q = t; q < tile; q += RS_T)
    if (base + q < n) atomicAdd(&h[(unsigned)(kin[base + q] >> shift) & 255u], 1u);
  __syncthreads();
  if (t < 256) hist[(int64_t)blockIdx.x * 256 + t] = h[t];
}

// the first pass's histogram of up to RS_CHAIN keys that come without one (cleared before)
__global__ __launch_bounds__(256) void k_radix_hist(const uint64_t *__restrict__ kin, int64_t n, int shift, int tile,
                                                    uint32_t *__restrict__ hist) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
    count_entry(hist, (uint32_t)(k / tile) * 256u + ((unsigned)(kin[k] >> shift) & 255u), true);
}

// Column d of hist (tile counts of digit d) becomes its exclusive scan, tot[d]
// its total: one wavefront per digit, 64 rows at a time.
__global__ __launch_bounds__(256) void k_radix_colscan(uint32_t *__restrict__ hist, int ntiles,
                                                       uint32_t *__restrict__ tot) {
  const int d = blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE, l = threadIdx.x & (WAVE - 1);
  uint32_t carry = 0;
  for (int r0 = 0; r0 < ntiles; r0 += WAVE) {  // uniform
    const int r = r0 + l;
    const uint32_t v = r < ntiles ? hist[(int64_t)r * 256 + d] : 0u;
    const uint32_t incl = (uint32_t)wave_incl_scan((int)v);
    if (r < ntiles) hist[(int64_t)r * 256 + d] = carry + incl - v;
    carry += (uint32_t)uniform_lane((int)incl, WAVE - 1);
  }
  if (l == 0) tot[d] = carry;
}

// exclusive scan over the 256 values of threads 0..255 (every thread of the
// workgroup calls it; ws: four words)
__device__ __forceinline__ uint32_t scan256(uint32_t v, int t, uint32_t *ws) {
  const uint32_t incl = (uint32_t)wave_incl_scan((int)v);
  if (t < 256 && (t & (WAVE - 1)) == WAVE - 1) ws[t / WAVE] = incl;
  __syncthreads();
  uint32_t base = incl - v;
#pragma unroll
  for (int q = 0; q < 3; ++q) base += q < t / WAVE ? ws[q] : 0u;
  __syncthreads();
  return base;
}

template <int I, bool VALS, bool SELF>
__global__ __launch_bounds__(RS_T) void k_radix_pass(const uint64_t *__restrict__ kin, const int32_t *__restrict__ vin,
                                                     uint64_t *__restrict__ kout, int32_t *__restrict__ vout,
                                                     int64_t n, int ntiles, int shift,
                                                     const uint32_t *__restrict__ hist,
                                                     const uint32_t *__restrict__ tot,
                                                     uint32_t *__restrict__ hist_next) {
  constexpr int TILE = RS_T * I;
  __shared__ uint32_t wc[RS_W][256];  // the column sums, then each wavefront's digit counts
  __shared__ uint32_t gbase[256], lstart[256], ws[4];
  __shared__ uint64_t lk[TILE];
  __shared__ int32_t lv[VALS ? TILE : 1];
  const int t = threadIdx.x, w = t / WAVE, lane = t & (WAVE - 1), d0 = t & 255;
  const int64_t base = (int64_t)blockIdx.x * TILE;
  uint64_t key[I];
  int32_t val[I];
  // wavefront w owns the keys [w 64 I, (w + 1) 64 I) of the tile, in order
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int64_t k = base + w * (WAVE * I) + i * WAVE + lane;
    key[i] = k < n ? kin[k] : 0ull;
    val[i] = VALS && k < n ? vin[k] : 0;
  }
  {
    uint32_t before = 0, all = 0;
    if (SELF) {
      const int b = blockIdx.x;
#pragma unroll 16
      for (int r = t >> 8; r < ntiles; r += RS_T / 256) {
        const uint32_t c = hist[(int64_t)r * 256 + d0];
        all += c;
        before += r < b ? c : 0u;
      }
      wc[t >> 8][d0] = all;
      wc[4 + (t >> 8)][d0] = before;
      __syncthreads();
      if (t < 256) {
        all = wc[0][t] + wc[1][t] + wc[2][t] + wc[3][t];
        before = wc[4][t] + wc[5][t] + wc[6][t] + wc[7][t];
      }
      __syncthreads();
    } else if (t < 256) {
      all = tot[t];
      before = hist[(int64_t)blockIdx.x * 256 + t];
    }
    const uint32_t first = scan256(all, t, ws);
    if (t < 256) gbase[t] = first + before;
  }
#pragma unroll
  for (int q = 0; q < RS_W / 4; ++q) wc[4 * q + (t >> 8)][d0] = 0u;
  __syncthreads();
  uint32_t rank[I];
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const bool valid = base + w * (WAVE * I) + i * WAVE + lane < n;
    const unsigned d = (unsigned)(key[i] >> shift) & 255u;
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1u;
      const unsigned long long bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const int r = popc_below(peers);
    const uint32_t c = wc[w][d];
    rank[i] = c + (uint32_t)r;
    // a wavefront's LDS operations execute in order: every peer has read c
    __builtin_amdgcn_wave_barrier();
    if (valid && r == 0) wc[w][d] = c + (uint32_t)__popcll(peers);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  uint32_t cnt = 0;
  if (t < 256) {
#pragma unroll
    for (int q = 0; q < RS_W; ++q) {
      const uint32_t c = wc[q][t];
      wc[q][t] = cnt;
      cnt += c;
    }
  }
  const uint32_t ls = scan256(cnt, t, ws);
  if (t < 256) lstart[t] = ls;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < I; ++i) {
    if (base + w * (WAVE * I) + i * WAVE + lane >= n) continue;
    const unsigned d = (unsigned)(key[i] >> shift) & 255u;
    const uint32_t p = lstart[d] + wc[w][d] + rank[i];
    lk[p] = key[i];
    if (VALS) lv[p] = val[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int p = i * RS_T + t;
    if (base + p >= n) break;
    const uint64_t k = lk[p];
    const unsigned d = (unsigned)(k >> shift) & 255u;
    const uint32_t off = gbase[d] + (uint32_t)p - lstart[d];
    kout[off] = k;
    if (VALS) vout[off] = lv[p];
    if (hist_next) count_entry(hist_next, (off / TILE) * 256u + ((unsigned)(k >> (shift + 8)) & 255u), true);
  }
}

// histograms of up to RADIX_PASSES passes (one, above RS_CHAIN keys), and the
// digit totals
int64_t radix_hist_need(int64_t n) {
  const int64_t tiles = (n + 4 * RS_T - 1) / (4 * RS_T);
  return std::max<int64_t>(RADIX_PASSES * 128, tiles) * 256 + 256;
}

hipError_t radix_sort_pairs(uint64_t *&keys, int32_t *&vals, uint64_t *&keys_alt, int32_t *&vals_alt, int64_t n,
                            int bit_lo, int bit_hi, uint32_t *hist, int64_t hist_cap, bool hist_ready,
                            hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const RadixPlan p = radix_plan(n);
  const int passes = (bit_hi - bit_lo + 7) / 8;
  const int64_t words = (int64_t)p.ntiles * 256;
  const int64_t used = p.chain ? passes * words : words;  // one histogram per pass, or one for all
  if (passes > RADIX_PASSES || used + 256 > hist_cap) return hipErrorInvalidValue;
  uint32_t *tot = hist + used;
  if (p.chain && !hist_ready) {
    const hipError_t e = fill_i32(reinterpret_cast<int32_t *>(hist), 0, passes * words, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)std::min<int64_t>(65536, (n + 255) / 256)), dim3(256), 0, s, keys,
                       n, bit_lo, p.tile, hist);
  }
  for (int q = 0; q < passes; ++q) {
    uint32_t *h = p.chain ? hist + q * words : hist, *hn = p.chain && q + 1 < passes ? h + words : nullptr;
    const int shift = bit_lo + 8 * q;
    if (!p.chain) hipLaunchKernelGGL(k_radix_tile_hist, dim3(p.ntiles), dim3(RS_T), 0, s, keys, n, shift, p.tile, h);
    const bool self = p.ntiles <= RS_SELF;
    if (!self) hipLaunchKernelGGL(k_radix_colscan, dim3(256 / (256 / WAVE)), dim3(256), 0, s, h, p.ntiles, tot);
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(p.ntiles), dim3(RS_T), 0, s, keys, vals, keys_alt, vals_alt, n, p.ntiles, shift,
                         h, tot, hn);
    };
    if (vals) {
      if (p.tile == RS_T)
        go(k_radix_pass<1, true, true>);
      else if (p.tile == 2 * RS_T)
        go(k_radix_pass<2, true, true>);
      else if (self)
        go(k_radix_pass<4, true, true>);
      else
        go(k_radix_pass<4, true, false>);
    } else {
      if (p.tile == RS_T)
        go(k_radix_pass<1, false, true>);
      else if (p.tile == 2 * RS_T)
        go(k_radix_pass<2, false, true>);
      else if (self)
        go(k_radix_pass<4, false, true>);
      else
        go(k_radix_pass<4, false, false>);
    }
    std::swap(keys, keys_alt);
    std::swap(vals, vals_alt);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------ fills, kick
__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) p[k] = v;
}

static inline unsigned grid_for(int64_t n, int threads = 256, int64_t cap = 65536) {
  int64_t b = (n + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}

__global__ void k_iota_i32(int32_t *p, int64_t n) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
    p[k] = (int32_t)k;
}

__global__ void k_fill_f64(double *p, double v, int64_t n) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) p[k] = v;
}

hipError_t iota_i32(int32_t *p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_iota_i32, dim3(grid_for(n)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t fill_f64(double *p, double v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_f64, dim3(grid_for(n)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

hipError_t fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

__global__ void k_kick(int64_t n3, double h, const double *__restrict__ a, double *__restrict__ v) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n3; k += (int64_t)gridDim.x * blockDim.x)
    v[k] += h * a[k];
}

hipError_t kick(int64_t n, double h, const double *acc3, double *vel3, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_kick, dim3(grid_for(3 * n)), dim3(256), 0, s, 3 * n, h, acc3, vel3);
  return hipGetLastError();
}

}  // namespace p3t
