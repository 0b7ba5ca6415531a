// Common-mode atmosphere subtraction (section 4.3, Eqs. common_mode and
// Sj) and inverse-variance gridding of a brightness-temperature TOD, FP64
// arithmetic on FP32 data.
//
//   eta_z,k   = sum_j B0_jk eta_z,j(PWV_mean) / sum_j B0_jk
//   eta_i     = eta_z,k ^ (1 / sin(theta(t) + theta0 + dtheta_i))
//   M(t, k)   = (1 / N_out) sum_{j off source} T_b,j / (1 - eta_j)
//   T*_i      = T_b,i / eta_i - (1 - eta_i) / eta_i M(t, k)
// with 1 - eta = -expm1(ln eta) so that transparent channels keep their
// relative precision.  Gridding bins T*_i(t, k) of spaxel i at (phi(t) +
// dphi_i, theta(t) + dtheta_i) to the nearest node of an n x n grid; per
// (spaxel, channel, cell) the mean and the variance of the samples give a
// weight m / s^2, and the cells of all spaxels are combined with it.
//
// Kernels: setup (scan table, mean PWV, channel transmission), common (M and,
// without maps, T*), grid (T* and cell sums), combine (one thread per
// (channel, cell)).  The common and grid kernels each stream the TOD once.
//
// The cosecants are tabulated once per call for all channels (where that pays,
// see gtod_reduce); each sample then
// takes one FP64 expm1 (eta = 1 + expm1(ln eta), so 1 - eta keeps its relative
// precision) and a division in either kernel, which is what bounds them.
// (Polynomials in elevation in their place take 2.9 ms in all, but the last bits
// of T* decide the weight of a cell whose few samples nearly coincide.)
//
// Cell sums: the samples of a tile of time, sorted once per spaxel by cell, are
// summed by one thread per run of a cell and added to the block's sums in LDS,
// without atomics except for cells of more than one run.
//
// 49 spaxels x 347 channels x 57600 samples, T* and 31 x 31 maps: 4.00 ms (8.37
// with a sine and a division per spaxel, sample and four channels and two LDS
// atomics per sample, which run at a lane per clock).  Common 0.92 ms (2.2
// before), grid 2.90 (6.1): about 60 FP64 instructions a sample, 1.5 ms of the
// grid's time, beside 3.9 GB read and 4 GB written.  The sort, 70 us, serves all
// channels.  Short series and few channels go without it (gtod_reduce).
#include <hip/hip_runtime.h>

#include <cmath>

#include "gtod_internal.h"
#include "lds_barrier.h"
#include "scan.h"

namespace gtod {

namespace {

constexpr int kRdThreads = 256;

__device__ double block_sum_256(double v, double* s) {
  s[threadIdx.x] = v;
  __syncthreads();
  for (int st = kRdThreads / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) s[threadIdx.x] += s[threadIdx.x + st];
    __syncthreads();
  }
  const double r = s[0];
  __syncthreads();
  return r;
}

__device__ inline int map_cell(const ReduceArgs& a, double x, double y) {
  const double gx = floor((x + a.half) / a.dcell + 0.5);
  const double gy = floor((y + a.half) / a.dcell + 0.5);
  if (!(gx >= 0.0 && gx < (double)a.map_n && gy >= 0.0 && gy < (double)a.map_n))
    return -1;
  return (int)gy * a.map_n + (int)gx;
}

}  // namespace

// Scan offsets, and the cosecants of spaxel blockIdx.y where they are kept.
__global__ __launch_bounds__(kRdThreads) void k_rd_scan(ReduceArgs a) {
  const int64_t t = (int64_t)blockIdx.x * kRdThreads + threadIdx.x;
  if (t >= a.T) return;
  const int p = blockIdx.y;
  double phi, th;
  scan_offsets(a.scan_kind, a.r_petal, a.omega, a.Omega, a.traj, a.t0 + t,
               a.f_s, &phi, &th);
  if (p == 0) {
    a.scan_phi[t] = phi;
    a.scan_th[t] = th;
  }
  if (!a.csc_common) return;
  a.csc_common[p * a.T + t] = 1.0 / sin((th + a.theta0) + a.dtheta[p]);
  if (a.csc_grid) a.csc_grid[p * a.T + t] = 1.0 / sin(th + (a.theta0 + a.dtheta[p]));
}

// Mean zenith PWV (one block, fixed-order sums), then ln eta_z,k (one
// block per channel).
__global__ __launch_bounds__(kRdThreads) void k_rd_pwv_mean(ReduceArgs a) {
  __shared__ double s[kRdThreads];
  double acc = 0.0;
  if (a.pwv) {
    const int64_t n = (int64_t)a.P * a.pwv_len;
    for (int64_t i = threadIdx.x; i < n; i += kRdThreads) {
      const int64_t p = i / a.pwv_len, t = i % a.pwv_len;
      acc += (double)a.pwv[p * a.pwv_ld + t];
    }
  }
  const double tot = block_sum_256(acc, s);
  if (threadIdx.x == 0)
    a.pwv_mean[0] = a.pwv ? tot / ((double)a.P * (double)a.pwv_len) : a.pwv_host;
}

// The same 256 partial sums, term by term in the same order, 64 to a block:
// all 16 waves load a tile of 256 terms of each, the first wave adds up the
// one before from LDS.  49 x 576000 values: 1.4 ms, 54 in one block.
constexpr int kPwvTile = 256, kPwvThreads = 1024;
__global__ __launch_bounds__(kPwvThreads) void k_rd_pwv_parts(ReduceArgs a) {
  __shared__ float buf[2][kPwvTile][64];
  constexpr int kEach = kPwvTile * 64 / kPwvThreads;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t n = (int64_t)a.P * a.pwv_len, c = blockIdx.x * 64 + lane;
  const bool rows = a.pwv_ld != a.pwv_len;
  const int64_t tiles = (n + kPwvTile * 256 - 1) / (kPwvTile * 256);
  float v[kEach];
  auto load = [&](int64_t tile) {
#pragma unroll
    for (int e = 0; e < kEach; ++e) {
      const int64_t i = (tile * kPwvTile + wave + 16 * e) * 256 + c;
      v[e] = 0.f;
      if (i < n) v[e] = a.pwv[rows ? i / a.pwv_len * a.pwv_ld + i % a.pwv_len : i];
    }
  };
  double acc = 0.0;
  load(0);
  for (int64_t tile = 0; tile < tiles; ++tile) {
#pragma unroll
    for (int e = 0; e < kEach; ++e) buf[tile & 1][wave + 16 * e][lane] = v[e];
    lds_barrier();
    if (tile + 1 < tiles) load(tile + 1);
    if (wave == 0) {
      const int64_t left = (n - c + 255) / 256 - tile * kPwvTile;
      const int m = (int)min(left, (int64_t)kPwvTile);
#pragma unroll 16
      for (int j = 0; j < m; ++j) acc += (double)buf[tile & 1][j][lane];
    }
  }
  if (wave == 0) a.pwv_part[c] = acc;
}

__global__ __launch_bounds__(kRdThreads) void k_rd_channel(ReduceArgs a) {
  __shared__ double s[kRdThreads];
  const int k = blockIdx.x;
  double mean;
  if (a.pwv_part && a.pwv)
    mean = block_sum_256(a.pwv_part[threadIdx.x], s) / ((double)a.P * (double)a.pwv_len);
  else
    mean = a.pwv_mean[0];
  double g = (mean - a.pwv0) / a.dpwv;
  g = fmin(fmax(g, 0.0), (double)(a.n_pwv - 1));
  int ci = (int)floor(g);
  if (ci > a.n_pwv - 2) ci = a.n_pwv - 2;
  const double wg = g - ci;
  double num = 0.0, den = 0.0;
  for (int j = threadIdx.x; j < a.F; j += kRdThreads) {
    const double tz = (1.0 - wg) * a.tau64[(int64_t)ci * a.F + j] +
                      wg * a.tau64[(int64_t)(ci + 1) * a.F + j];
    const double b = a.B0[(int64_t)j * a.K + k];
    num += b * exp(-tz);
    den += b;
  }
  const double N = block_sum_256(num, s);
  const double D = block_sum_256(den, s);
  if (threadIdx.x == 0) a.lnz[k] = (D > 0.0) ? log(N / D) : NAN;
}

// Four samples of a row; n < 4 at its end.  Rows start at any multiple of 4 B,
// which is all the vector loads ask for.
typedef float Float4 __attribute__((ext_vector_type(4), aligned(4)));
typedef double Double4 __attribute__((ext_vector_type(4), aligned(8)));
// STREAM: past the caches, for rows that are not read again here
template <typename V, bool STREAM = false, typename T>
__device__ inline void load4(const T* p, int n, T* v) {
  if (n >= 4) {
    V f;
    if constexpr (STREAM) f = __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
    else f = *reinterpret_cast<const V*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = f[i];
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = i < n ? p[i] : T(0);
  }
}
template <typename V, bool STREAM, typename T>
__device__ inline void store4(T* p, int n, const T* v) {
  if (n >= 4) {
    V f;
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = v[i];
    if constexpr (STREAM) __builtin_nontemporal_store(f, reinterpret_cast<V*>(p));
    else *reinterpret_cast<V*>(p) = f;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < n) p[i] = v[i];
  }
}

// One thread per sample and CH channels of the group: kRdChan, or fewer where a
// call has fewer (7 x 1 x 100 samples: 33 us, 38 with 7 slots that repeat the
// channel).
template <int CH>
__global__ __launch_bounds__(kRdThreads) void k_rd_common(ReduceArgs a) {
  const int64_t t = (int64_t)blockIdx.x * kRdThreads + threadIdx.x;
  const int kl0 = blockIdx.y * CH;
  if (t >= a.T) return;
  const int nk = min(CH, a.kg - kl0);
  double lz[CH], sum[CH];
#pragma unroll
  for (int q = 0; q < CH; ++q) {
    lz[q] = a.lnz[a.k0 + min(kl0 + q, a.kg - 1)];    // dead slots repeat the last channel
    sum[q] = 0.0;
  }
  const double th = a.scan_th[t] + a.theta0;
  const int64_t rowK = a.ld;                      // stride between channels
  auto cosecant = [&](int p) {
    return a.csc_common ? a.csc_common[p * a.T + t] : 1.0 / sin(th + a.dtheta[p]);
  };
  auto load = [&](int p, float (&v)[CH]) {
    const float* src = a.tod + ((int64_t)p * a.K + a.k0 + kl0) * rowK + t;
#pragma unroll
    for (int q = 0; q < CH; ++q) v[q] = src[min(q, nk - 1) * rowK];
  };
  // the spaxels off source alone are read, the next one's samples ahead
  auto next = [&](int p) { return p + 1 < a.P ? a.off[p + 1] : a.P; };
  float v[CH], w[CH];
  int p0 = a.off[0], p1 = next(p0);      // there is one
  load(p0, v);
  while (p0 < a.P) {
    if (p1 < a.P) load(p1, w);
    const int p2 = next(p1);
    const double csc = cosecant(p0);
#pragma unroll
    for (int q = 0; q < CH; ++q) sum[q] += (double)v[q] / -expm1(lz[q] * csc);
#pragma unroll
    for (int q = 0; q < CH; ++q) v[q] = w[q];
    p0 = p1;
    p1 = p2;
  }
#pragma unroll
  for (int q = 0; q < CH; ++q) {
    sum[q] /= (double)a.n_out;
    if (q < nk && a.M) a.M[(int64_t)(kl0 + q) * a.T + t] = sum[q];
  }
  if (!a.t_star || a.map_n > 0) return;
  for (int p = 0; p < a.P; ++p) {
    const double csc = cosecant(p);
    load(p, v);
    float* dst = a.t_star + ((int64_t)p * a.K + a.k0 + kl0) * rowK + t;
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const double em = expm1(lz[q] * csc);     // eta - 1
      if (q < nk) dst[q * rowK] = (float)(((double)v[q] + em * sum[q]) / (1.0 + em));
    }
  }
}

// Sorts a tile's samples of a spaxel by cell (bitonic, on cell and sample:
// the order is that of time within a cell) and lists the runs.  Blocks (tile,
// spaxel).
constexpr int kRdSortThreads = 512;
__global__ __launch_bounds__(kRdSortThreads) void k_rd_sort(ReduceArgs a) {
  constexpr uint32_t kNone = 4095;
  __shared__ uint32_t key[kRdTile];
  __shared__ int heads[kRdSortThreads / 64];
  const int tid = threadIdx.x, p = blockIdx.y;
  const int64_t t0 = (int64_t)blockIdx.x * kRdTile;
  for (int i = tid; i < kRdTile; i += kRdSortThreads) {
    int c = -1;
    if (t0 + i < a.T)
      c = map_cell(a, a.scan_phi[t0 + i] + a.dphi[p], a.scan_th[t0 + i] + a.dtheta[p]);
    key[i] = (c < 0 ? kNone : (uint32_t)c) << 11 | (uint32_t)i;
  }
  __syncthreads();
  for (int n = 2; n <= kRdTile; n <<= 1)
    for (int d = n >> 1; d > 0; d >>= 1) {
      for (int i = tid; i < kRdTile / 2; i += kRdSortThreads) {
        const int lo = (i & ~(d - 1)) * 2 + (i & (d - 1)), hi = lo + d;
        const uint32_t x = key[lo], y = key[hi];
        if ((x > y) == ((lo & n) == 0)) {
          key[lo] = y;
          key[hi] = x;
        }
      }
      __syncthreads();
    }
  auto first = [&](uint32_t least) {    // first sorted position with key >= least
    int b = 0;
    for (int st = kRdTile / 2; st > 0; st >>= 1)
      if (key[b + st - 1] < least) b += st;
    return b + (key[b] < least);
  };
  const int64_t tile = (int64_t)p * gridDim.x + blockIdx.x;
  constexpr int kEach = kRdTile / kRdSortThreads;
  uint32_t run[kEach];
  int n = 0;
#pragma unroll
  for (int e = 0; e < kEach; ++e) {
    const int s = tid * kEach + e;
    const uint32_t k = key[s], cell = k >> 11;
    // the word of the tile in LDS: k_rd_map's threads store a column each
    const uint32_t i = k & (kRdTile - 1);
    a.perm[tile * kRdTile + s] = (uint16_t)((i & 3) * (kRdTile / 4) + (i >> 2));
    run[e] = ~0u;
    if (cell == kNone) continue;
    const int b = first(cell << 11);
    if ((s - b) % kRdRun) continue;
    const int end = first((cell + 1) << 11), len = min(end - s, kRdRun);
    run[e] = (uint32_t)s | (uint32_t)(len - 1) << 11 | cell << 16 |
             (uint32_t)(end - b > kRdRun) << 28;
    ++n;
  }
  // ranks of the runs: waves, then lanes
  int before = n;
#pragma unroll
  for (int st = 1; st < 64; st <<= 1) {
    const int v = __shfl_up(before, st);
    if ((tid & 63) >= st) before += v;
  }
  if ((tid & 63) == 63) heads[tid >> 6] = before;
  __syncthreads();
  int at = before - n;
  for (int w = 0; w < (tid >> 6); ++w) at += heads[w];
#pragma unroll
  for (int e = 0; e < kEach; ++e)
    if (run[e] != ~0u) a.runs[tile * kRdTile + at++] = run[e];
  if (tid == kRdSortThreads - 1) a.n_runs[tile] = at;
}

// The square rounded before it is added, as the atomics of k_rd_grid take it.
__device__ inline double add_square(double s, double v) {
  double q = v * v;
  asm("" : "+v"(q));   // not fused into one multiply-add
  return s + q;
}

// One block per (spaxel, kRdMapChan channels).  Per tile of time: T* of 4
// samples a thread, its distance from the channel's first sample to LDS; then
// a run of a cell to a thread, added to the block's cell sums.  The variance is
// (S2 - S1^2 / m) / (m - 1).  When T* is requested with maps, this kernel also
// stores it (for every sample, in or out of the map).
constexpr int kRdMapChan = 2, kRdMapThreads = kRdTile / 4;
__global__ __launch_bounds__(kRdMapThreads, 4) void k_rd_map(ReduceArgs a) {
  extern __shared__ double gsm[];
  const int p = blockIdx.x % a.P, group = blockIdx.x / a.P;   // a group's blocks share M rows
  const int C = a.map_n * a.map_n, tid = threadIdx.x;
  double2* const v = (double2*)gsm;                   // [tile] both channels
  double2* const s1 = v + kRdTile;                    // [C]
  double2* const s2 = s1 + C;                         // [C]
  unsigned* const cnt = (unsigned*)(s2 + C);          // [C]
  uint16_t* const perm = (uint16_t*)(cnt + ((C + 3) & ~3));   // [tile]
  const int kl0 = group * kRdMapChan;
  const int nk = min(kRdMapChan, a.kg - kl0);
  for (int c = tid; c < C; c += kRdMapThreads) {
    cnt[c] = 0u;
    s1[c] = s2[c] = make_double2(0.0, 0.0);
  }
  double lz[kRdMapChan], shift[kRdMapChan];
  const float* row[kRdMapChan];
  const double* Mr[kRdMapChan];
  const double* const csc = a.csc_grid + p * a.T;
  auto t_star = [&](int q, double c, float d, double M) {
    const double em = expm1(lz[q] * c);     // eta - 1
    return ((double)d + em * M) / (1.0 + em);
  };
#pragma unroll
  for (int q = 0; q < kRdMapChan; ++q) {
    const int kq = min(kl0 + q, a.kg - 1), k = a.k0 + kq;   // dead slots repeat the last channel
    lz[q] = a.lnz[k];
    row[q] = a.tod + ((int64_t)p * a.K + k) * a.ld;
    Mr[q] = a.M + (int64_t)kq * a.T;
    shift[q] = t_star(q, csc[0], row[q][0], Mr[q][0]);
  }
  float* const out_ts = a.t_star ? a.t_star + ((int64_t)p * a.K + a.k0 + kl0) * a.ld : nullptr;
  const int tiles = (int)((a.T + kRdTile - 1) / kRdTile);
  float d[kRdMapChan][4];
  double M[kRdMapChan][4], c4[4];
  // a tile's run list: its first 2 runs per thread (what most tiles have),
  // the samples' places, the number of runs
  uint32_t u0, u1;
  uint2 pm;
  int n;
  auto load = [&](int tile) {
    const int64_t list = ((int64_t)p * tiles + tile) * kRdTile;
    pm = reinterpret_cast<const uint2*>(a.perm + list)[tid];
    u0 = a.runs[list + tid];
    u1 = a.runs[list + kRdMapThreads + tid];
    n = a.n_runs[(int64_t)p * tiles + tile];
    const int64_t t = (int64_t)tile * kRdTile + tid * 4;
    const int nt = (int)min(a.T - t, (int64_t)4);
    if (nt <= 0) return;
#pragma unroll
    for (int q = 0; q < kRdMapChan; ++q) {
      load4<Float4, true>(row[q] + t, nt, d[q]);
      load4<Double4>(Mr[q] + t, nt, M[q]);
    }
    load4<Double4>(csc + t, nt, c4);
  };
  load(0);
  __syncthreads();
  for (int tile = 0; tile < tiles; ++tile) {
    const int64_t t = (int64_t)tile * kRdTile + tid * 4;
    const int nt = (int)min(a.T - t, (int64_t)4);
    const int64_t list = ((int64_t)p * tiles + tile) * kRdTile;
    if (nt > 0) {
      float o[kRdMapChan][4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        double ts[kRdMapChan];
#pragma unroll
        for (int q = 0; q < kRdMapChan; ++q) {
          ts[q] = t_star(q, c4[i], d[q][i], M[q][i]);
          o[q][i] = (float)ts[q];
        }
        v[i * kRdMapThreads + tid] = make_double2(ts[0] - shift[0], ts[1] - shift[1]);
      }
      if (out_ts)
#pragma unroll
        for (int q = 0; q < kRdMapChan; ++q)
          if (q < nk) store4<Float4, true>(out_ts + q * a.ld + t, nt, o[q]);
    }
    reinterpret_cast<uint2*>(perm)[tid] = pm;
    const int nr = n;
    uint32_t u = u0, ahead = u1;
    if (tile + 1 < tiles) load(tile + 1);
    lds_barrier();
    for (int r = tid; r < nr; r += kRdMapThreads) {
      const int b = u & 2047, len = (int)(u >> 11 & 31) + 1, c = (int)(u >> 16 & 4095);
      double2 x1 = make_double2(0.0, 0.0), x2 = x1;
      for (int e = 0; e < len; e += 4) {
        double2 y[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) y[g] = v[perm[b + min(e + g, len - 1)]];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          if (e + g >= len) y[g] = make_double2(0.0, 0.0);
          x1.x += y[g].x;
          x1.y += y[g].y;
          x2.x = add_square(x2.x, y[g].x);
          x2.y = add_square(x2.y, y[g].y);
        }
      }
      if (u >> 28) {
        atomicAdd(&s1[c].x, x1.x);
        atomicAdd(&s1[c].y, x1.y);
        atomicAdd(&s2[c].x, x2.x);
        atomicAdd(&s2[c].y, x2.y);
        atomicAdd(&cnt[c], (unsigned)len);
      } else {
        const double2 w1 = s1[c], w2 = s2[c];
        s1[c] = make_double2(w1.x + x1.x, w1.y + x1.y);
        s2[c] = make_double2(w2.x + x2.x, w2.y + x2.y);
        cnt[c] += (unsigned)len;
      }
      u = ahead;
      if (r + 2 * kRdMapThreads < nr) ahead = a.runs[list + r + 2 * kRdMapThreads];
    }
    lds_barrier();
  }
  for (int q = 0; q < nk; ++q) {
    double2* out = a.stats + ((int64_t)p * a.kg + kl0 + q) * C;
    for (int c = tid; c < C; c += kRdMapThreads) {
      const double m = (double)cnt[c];
      double w = 0.0, mean = 0.0;
      if (m >= 2.0) {
        const double S1 = q ? s1[c].y : s1[c].x, S2 = q ? s2[c].y : s2[c].x;
        const double var = (S2 - S1 * S1 / m) / (m - 1.0);
        if (var > 0.0) {
          w = m / var;
          mean = S1 / m + (q ? shift[1] : shift[0]);
        }
      }
      out[c] = make_double2(w, mean);
    }
  }
}

// For short series, and workspaces without room for the runs.
// One block per (spaxel, kRdGridChan channels of the group), spaxel
// fastest so that the blocks sharing those channels' M rows run together.
// The sample's cosecant and cell are evaluated once for all its channels;
// cell count (common to the channels), and per channel the sums of v =
// T* - shift (shift = the channel's first sample) and v^2, accumulate in
// LDS; the variance is (S2 - S1^2 / m) / (m - 1).  When T* is requested
// with maps, this kernel also stores it (for every sample, in or out of
// the map).
__global__ __launch_bounds__(kRdThreads) void k_rd_grid(ReduceArgs a) {
  extern __shared__ double gsm[];
  const int C = a.map_n * a.map_n;
  double* s1 = gsm;                                   // [G][C]
  double* s2 = gsm + kRdGridChan * C;                 // [G][C]
  unsigned* cnt = (unsigned*)(gsm + 2 * kRdGridChan * C);   // [C]
  const int p = blockIdx.x % a.P;
  const int kl0 = (blockIdx.x / a.P) * kRdGridChan;
  const int nk = min(kRdGridChan, a.kg - kl0);
  for (int c = threadIdx.x; c < C; c += kRdThreads) {
    cnt[c] = 0u;
#pragma unroll
    for (int q = 0; q < kRdGridChan; ++q) {
      s1[q * C + c] = 0.0;
      s2[q * C + c] = 0.0;
    }
  }
  const double dth = a.theta0 + a.dtheta[p];
  const double dph = a.dphi[p];
  double lz[kRdGridChan], shift[kRdGridChan];
  const float* row[kRdGridChan];
  const double* Mr[kRdGridChan];
  const double csc0 = 1.0 / sin(a.scan_th[0] + dth);
#pragma unroll
  for (int q = 0; q < kRdGridChan; ++q) {
    const int kq = min(kl0 + q, a.kg - 1);     // dead slots repeat the last channel
    lz[q] = a.lnz[a.k0 + kq];
    row[q] = a.tod + ((int64_t)p * a.K + a.k0 + kq) * a.ld;
    Mr[q] = a.M + (int64_t)kq * a.T;
    const double em = expm1(lz[q] * csc0);
    shift[q] = ((double)row[q][0] + em * Mr[q][0]) / (1.0 + em);
  }
  float* out_ts = a.t_star ? a.t_star + ((int64_t)p * a.K + a.k0 + kl0) * a.ld : nullptr;
  __syncthreads();
  for (int64_t t = threadIdx.x; t < a.T; t += kRdThreads) {
    const double th = a.scan_th[t];
    const int c = map_cell(a, a.scan_phi[t] + dph, th + a.dtheta[p]);
    if (c < 0 && !out_ts) continue;
    const double csc = 1.0 / sin(th + dth);
    if (c >= 0) atomicAdd(&cnt[c], 1u);
#pragma unroll
    for (int q = 0; q < kRdGridChan; ++q) {
      if (q < nk) {
        const double em = expm1(lz[q] * csc);     // eta - 1
        const double ts = ((double)row[q][t] + em * Mr[q][t]) / (1.0 + em);
        if (out_ts) out_ts[q * a.ld + t] = (float)ts;
        if (c >= 0) {
          const double v = ts - shift[q];
          atomicAdd(&s1[q * C + c], v);
          atomicAdd(&s2[q * C + c], v * v);
        }
      }
    }
  }
  __syncthreads();
  for (int q = 0; q < nk; ++q) {
    double2* out = a.stats + ((int64_t)p * a.kg + kl0 + q) * C;
    for (int c = threadIdx.x; c < C; c += kRdThreads) {
      const double m = (double)cnt[c];
      double w = 0.0, mean = 0.0;
      if (m >= 2.0) {
        const double S1 = s1[q * C + c], S2 = s2[q * C + c];
        const double var = (S2 - S1 * S1 / m) / (m - 1.0);
        if (var > 0.0) {
          w = m / var;
          mean = S1 / m + shift[q];
        }
      }
      out[c] = make_double2(w, mean);
    }
  }
}

__global__ __launch_bounds__(kRdThreads) void k_rd_combine(ReduceArgs a) {
  const int C = a.map_n * a.map_n;
  const int c = blockIdx.x * kRdThreads + threadIdx.x;
  const int kl = blockIdx.y;
  if (c >= C) return;
  double ws = 0.0, num = 0.0;
  for (int p = 0; p < a.P; ++p) {
    const double2 st = a.stats[((int64_t)p * a.kg + kl) * C + c];
    if (st.x > 0.0) {
      ws += st.x;
      num += st.x * st.y;
    }
  }
  const int64_t o = (int64_t)(a.k0 + kl) * C + c;
  a.map[o] = ws > 0.0 ? num / ws : NAN;
  a.weight[o] = ws;
}

void launch_reduce_setup(const ReduceArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_rd_scan,
                     dim3((unsigned)((a.T + kRdThreads - 1) / kRdThreads), a.csc_common ? a.P : 1),
                     dim3(kRdThreads), 0, s, a);
  if (a.pwv_part && a.pwv)
    hipLaunchKernelGGL(k_rd_pwv_parts, dim3(4), dim3(kPwvThreads), 0, s, a);
  else
    hipLaunchKernelGGL(k_rd_pwv_mean, dim3(1), dim3(kRdThreads), 0, s, a);
  hipLaunchKernelGGL(k_rd_channel, dim3(a.K), dim3(kRdThreads), 0, s, a);
  if (a.runs)
    hipLaunchKernelGGL(k_rd_sort, dim3((unsigned)((a.T + kRdTile - 1) / kRdTile), a.P),
                       dim3(kRdSortThreads), 0, s, a);
}

void launch_reduce_common(const ReduceArgs& a, hipStream_t s) {
  const int ch = a.kg > 4 ? kRdChan : a.kg > 2 ? 4 : a.kg;
  const auto kernel = ch == 1 ? k_rd_common<1> : ch == 2 ? k_rd_common<2>
                      : ch == 4 ? k_rd_common<4> : k_rd_common<kRdChan>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)((a.T + kRdThreads - 1) / kRdThreads),
                                  (a.kg + ch - 1) / ch),
                     dim3(kRdThreads), 0, s, a);
}

int launch_reduce_grid(const ReduceArgs& a, hipStream_t s) {
  const int C = a.map_n * a.map_n;
  if (a.runs) {
    const size_t lds = (size_t)C * 32 + (size_t)((C + 3) & ~3) * 4 + kRdTile * (16 + 2);
    if (hipFuncSetAttribute((const void*)k_rd_map,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return 1;
    const int groups = (a.kg + kRdMapChan - 1) / kRdMapChan;
    hipLaunchKernelGGL(k_rd_map, dim3((unsigned)(a.P * groups)), dim3(kRdMapThreads), lds, s, a);
    return 0;
  }
  const size_t lds = (size_t)C * (2 * kRdGridChan * sizeof(double) + sizeof(unsigned));
  if (hipFuncSetAttribute((const void*)k_rd_grid,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return 1;
  const int groups = (a.kg + kRdGridChan - 1) / kRdGridChan;
  hipLaunchKernelGGL(k_rd_grid, dim3((unsigned)(a.P * groups)), dim3(kRdThreads), lds, s, a);
  return 0;
}

void launch_reduce_combine(const ReduceArgs& a, hipStream_t s) {
  const int C = a.map_n * a.map_n;
  hipLaunchKernelGGL(k_rd_combine, dim3((C + kRdThreads - 1) / kRdThreads, a.kg),
                     dim3(kRdThreads), 0, s, a);
}

}  // namespace gtod
