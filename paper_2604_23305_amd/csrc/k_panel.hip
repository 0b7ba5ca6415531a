// Panel kernel: per (row, nu) spectral power deviation dP = P - Pref.
//
// Per row (one pixel at one time sample), in FP64 (section 2.4):
//   t = n / f_sample; scan offsets (phi, theta) from the pattern;
//   screen position x = h tan(phi + dphi) + u_w t, y = h tan(theta + dtheta)
//   (Eq. xy_atm) -> bilinear PWV on the screen; table row and weight of
//   that PWV; cosecant of the elevation theta + theta0 + dtheta (Eq.
//   airmass); source cell and weights at the full pointing (zero outside).
// Per (row, nu), in FP32, coalesced along nu:
//   tau_z = (1-w) tau[i][nu] + w tau[i+1][nu]    optical-depth interpolation
//   xi    = -expm1(-csc tau_z)                     1 - eta_z^csc
//   P     = E + xi D + (1 - xi) W P_src            collapsed cascade
//   dP    = P - Pref
// A workgroup handles up to kPanelRows rows; a lane takes four bins at a
// time, so that every table, cube and panel access is a contiguous run along
// nu, and all rows of a pass of 1024 bins before the next pass.
//
// With a source cube, a scan that moves a cell or more per sample makes
// consecutive samples read different cube corners (four spectra of F
// floats each), which then come from beyond the L2 for almost every row.
// The rows of a large chunk are therefore first bucketed by the (coarse)
// cube cell they read, with a counting sort, and the workgroups take them in
// bucket order: rows that share corners run together, and a workgroup keeps
// the corners of its current cell in registers.  Each row's result does not
// depend on the order, only the cache traffic does.
//
// What bounds it: HBM.  A launch of 527k IFU rows writes 6.3 GB of panel and
// fetches 0.89 GB (5.4 GB when a workgroup took 4 rows over all bins at a
// time and read their corners again for the next 4) in 1.30 ms, 5.5 TB/s;
// the five kernels together take 1.41 ms, against 2.37 ms before.  On the
// way there it was bound by its instructions (41 per element with vector
// records and the library's expm1f, 32 now) and by the panel's stores
// displacing the tables from the L2: stored past the caches the sorted
// kernel became a fifth faster.
#include <hip/hip_runtime.h>

#include "gtod_internal.h"
#include "scan.h"

namespace gtod {

namespace {

struct RowInfo {
  int valid;
  int li;          // table row below the PWV
  float lw;        // weight of the row above
  float csc;
  int src;         // pointing inside the source grid
  float w[4];      // weights of corners (el, az), (el, az + 1), (el + 1, az), ...
  int64_t sbase;   // offset of corner (el, az) in the cube
};
static_assert(sizeof(RowInfo) <= kPanelRowInfoBytes, "row record");

__device__ inline void clamp_cell(double g, int64_t n, int64_t* cell,
                                  double* w, bool* clamped) {
  const double gc = fmin(fmax(g, 0.0), (double)(n - 1));
  *clamped = (gc != g);
  int64_t c = (int64_t)floor(gc);
  if (c > n - 2) c = n - 2;
  *cell = c;
  *w = gc - (double)c;
}

// Row quantities of row r (FP64 geometry); *bucket gets the row's sort
// bucket.  first: also write the PWV output and count the range events.
__device__ RowInfo row_info(const PanelArgs& a, int64_t r, uint32_t* bucket, bool first) {
  RowInfo q{};
  *bucket = (uint32_t)(a.n_buckets - 1);
  const int pl = (int)(r / a.Tpad);
  const int tl = (int)(r % a.Tpad);
  q.valid = (pl < a.n_pix) && (tl < a.Tc);
  if (!q.valid) return q;
  const int p = a.p0 + pl;
  const int64_t n = a.t0 + tl;
  const double t = (double)n / a.f_s;
  double phi, th;
  scan_offsets(a.scan_kind, a.r_petal, a.omega, a.Omega, a.traj, n, a.f_s,
               &phi, &th);
  const double x = a.h * tan(phi + a.dphi[p]) + a.wind * t;
  const double y = a.h * tan(th + a.dtheta[p]);
  int64_t cx, cy;
  double wx, wy;
  bool ox, oy;
  clamp_cell(x / a.dx + a.ix0, a.nx, &cx, &wx, &ox);
  clamp_cell(y / a.dy + a.iy0, a.ny, &cy, &wy, &oy);
  const double* s0 = a.scr + cy * a.nx + cx;
  const double pwv = (1.0 - wx) * (1.0 - wy) * s0[0] + wx * (1.0 - wy) * s0[1] +
                     (1.0 - wx) * wy * s0[a.nx] + wx * wy * s0[a.nx + 1];
  if (first && (ox || oy)) atomicAdd(&a.counters[0], 1ull);
  if (first && a.pwv_out) a.pwv_out[(int64_t)p * a.out_ld + (n - a.out_t0)] = (float)pwv;
  int64_t li;
  double lw;
  bool ol;
  clamp_cell((pwv - a.pwv0) / a.dpwv, a.n_pwv, &li, &lw, &ol);
  if (first && ol) atomicAdd(&a.counters[1], 1ull);
  q.li = (int)li;
  q.lw = (float)lw;
  const double el = th + a.theta0 + a.dtheta[p];
  const double se = sin(el);
  // an elevation outside (0, pi) has no airmass (only a user trajectory
  // can reach one: analytic scans are checked before launch)
  if (first && !(se > 0.0)) atomicAdd(&a.counters[2], 1ull);
  q.csc = (float)(1.0 / se);
  q.src = 0;
  if (a.cube) {
    const double az = phi + a.phi0 + a.dphi[p];
    const double ga = (az - a.az0) / a.daz;
    const double ge = (el - a.el0) / a.del;
    if (ga >= 0.0 && ga <= (double)(a.n_az - 1) && ge >= 0.0 &&
        ge <= (double)(a.n_el - 1)) {
      int64_t ca, ce;
      double wa, we;
      bool d0, d1;
      clamp_cell(ga, a.n_az, &ca, &wa, &d0);
      clamp_cell(ge, a.n_el, &ce, &we, &d1);
      q.src = 1;
      const float fa = (float)wa, fe = (float)we;
      q.w[0] = (1.f - fa) * (1.f - fe);
      q.w[1] = fa * (1.f - fe);
      q.w[2] = (1.f - fa) * fe;
      q.w[3] = fa * fe;
      q.sbase = (ce * a.n_az + ca) * a.cube_ld;
      if (a.n_buckets > 1)
        *bucket = (uint32_t)((ce >> a.cell_shift) * a.n_az_coarse + (ca >> a.cell_shift));
    }
  }
  return q;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
// the same with the alignment of a float (a cube's rows may have any pitch)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kTileBins = 4 * 256;   // bins of a workgroup pass, 4 per lane

// 1 - e^-x for x >= 0 to about one ulp: n = rint(-x log2 e), r = -x - n ln 2
// in two parts, e^r - 1 = r + r^2 p(r) with p fitted on |r| <= ln(2) / 2 for
// the relative error of e^r - 1 (2e-9), and 1 - e^-x = (1 - 2^n) - 2^n (e^r -
// 1).  15 instructions where the library's expm1f takes 24; beyond x = 40
// the result is 1 either way.
__device__ __forceinline__ float one_minus_exp(float x) {
  const float y = __builtin_elementwise_minimum(x, 40.f);   // keeps a NaN
  constexpr float kMagic = 12582912.f;   // 1.5 * 2^23: the sum's low bits are n
  const float t = __builtin_fmaf(y, -1.44269504088896341f, kMagic);
  const float n = t - kMagic;
  float r = __builtin_fmaf(n, -0.693145751953125f, -y);
  r = __builtin_fmaf(n, -1.428606765330187045e-6f, r);
  float p = 1.98458888917230070e-4f;
  p = __builtin_fmaf(p, r, 1.39406265225261450e-3f);
  p = __builtin_fmaf(p, r, 8.33338964730501175e-3f);
  p = __builtin_fmaf(p, r, 4.16663624346256256e-2f);
  p = __builtin_fmaf(p, r, 1.66666656732559204e-1f);
  p = __builtin_fmaf(p, r, 0.5f);
  const float q = __builtin_fmaf(r * r, p, r);
  const float s = __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, t) << 23) + 0x3f800000u);
  return __builtin_fmaf(-s, q, 1.f - s);
}

// Counts (range counter 3) the (row, bin) elements whose deviation from
// the reference spectrum exceeds P / 8.  While none does, the terms of
// sum_j |dP_j| B_jk add up to at most P_KID / 8 (B >= 0, P > 0), so the
// 16-bit operands of the split contraction (relative error 2^-17 on each
// term) stay within 1e-6 of P_KID; beyond it the stated tolerance of the
// reference-row contraction is not guaranteed.
// far is the wave's count.
__device__ __forceinline__ void far_from_reference(const PanelArgs& a, uint32_t far) {
  if (far && (threadIdx.x & 63) == 0) atomicAdd(&a.counters[3], (unsigned long long)far);
}

// The bins of one workgroup pass: this lane's 4 bins from j, of which those
// below F exist (the spectra are zero beyond).
struct Bins {
  f32x4 E, D, W, Pr;
  uint32_t j, js;        // first bin; first bin of a cube load
  __device__ Bins(const PanelArgs& a, uint32_t j0) : j(j0) {
    const bool in = j < (uint32_t)a.Fp;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    E = in ? *reinterpret_cast<const f32x4*>(a.E + j) : zero;
    D = in ? *reinterpret_cast<const f32x4*>(a.D + j) : zero;
    W = in ? *reinterpret_cast<const f32x4*>(a.W + j) : zero;
    Pr = in ? *reinterpret_cast<const f32x4*>(a.Pref + j) : zero;
    js = min(j, (uint32_t)max(a.F - 4, 0));
  }
  // p[j .. j + 3], zero past the last bin; p is a row of F floats, of any
  // alignment.  The lane across the end reads the row's last four floats
  // and shifts them.
  __device__ __forceinline__ f32x4 cube(const float* p, int F) const {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (F < 4) {
      for (int k = 0; k < 4; ++k)
        if ((int)j + k < F) v[k] = p[j + k];
      return v;
    }
    v = *reinterpret_cast<const f32x4u*>(p + js);
    if (js != j) {
      const uint32_t s = j - js;
      v[0] = s == 1 ? v[1] : s == 2 ? v[2] : s == 3 ? v[3] : 0.f;
      v[1] = s == 1 ? v[2] : s == 2 ? v[3] : 0.f;
      v[2] = s == 1 ? v[3] : 0.f;
      v[3] = 0.f;
    }
    return v;
  }
};

// dP of a row: t0, t1 the table rows around its PWV, ps the source power.
// ANY_EL: the elevation may be one without airmass (csc negative or infinite;
// only a user trajectory reaches it).  csc is the same in the whole workgroup:
// such a row takes the library's expm1f, which overflows to the infinity it
// should, and leaves the bins of the padding, where 0 times infinity would be
// NaN, at zero.  Other scans do without that branch, which takes 6 registers
// and a wave per SIMD (0.6 us of a 45 us call).
template <bool ANY_EL>
__device__ __forceinline__ f32x4 row_deviation(const Bins& b, int F, f32x4 t0, f32x4 t1,
                                               f32x4 ps, float lw, float csc, bool src,
                                               uint32_t* far) {
  f32x4 dP;
  auto bins = [&](auto opacity, auto padded) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float tz = (1.f - lw) * t0[k] + lw * t1[k];
      const float xi = opacity(csc * tz);
      float P = b.E[k] + xi * b.D[k];
      if (src) P += (1.f - xi) * (b.W[k] * ps[k]);
      dP[k] = P - b.Pr[k];
      if (padded(b.j + k)) dP[k] = P = 0.f;
      *far += (uint32_t)__builtin_popcountll(__ballot(fabsf(dP[k]) > 0.125f * P));
    }
  };
  if (!ANY_EL || __builtin_expect(csc >= 0.f && csc < INFINITY, 1))
    bins([](float x) { return one_minus_exp(x); }, [](uint32_t) { return false; });
  else
    bins([](float x) { return -expm1f(-x); }, [&](uint32_t j) { return j >= (uint32_t)F; });
  return dP;
}

// A wave-uniform value, in a scalar register.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) {
  return __builtin_bit_cast(float, uniform(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ int64_t uniform(int64_t v) {
  return ((int64_t)uniform((int)(v >> 32)) << 32) | (uint32_t)uniform((int)v);
}

// Rows of one workgroup, record(rr) giving the record and panel row of the
// rr-th, over the passes of 1024 bins first, first + stride, ...  Within a
// pass the spectra E, D, W, Pref stay in registers, and the cube corners
// are loaded only where a row's cell is another than the row's before.
// kBatch rows' table values are loaded together, ahead of their arithmetic;
// n_rows is a multiple of it.
// NARROW: up to 512 bins are one or two waves' work, so that each wave, or pair
// of waves, takes every fourth, or second, kBatch of rows (1.14 M rows of 64
// bins: 150 us, 700 with three waves idle).
constexpr int kBatch = 2;
constexpr int kNarrowBins = 512;
template <bool ANY_EL, bool NARROW, class Rec>
__device__ __forceinline__ void panel_rows(const PanelArgs& a, int n_rows, int first,
                                           int stride, Rec record) {
  const int64_t Fp = a.Fp;
  const int64_t ld = a.cube_ld, crow = (int64_t)a.n_az * a.cube_ld;
  // waves of a row, and this wave's first and step among the rows
  const int waves = NARROW && a.Fp <= kNarrowBins / 2 ? 1 : 2;
  const int row0 = NARROW ? uniform((int)threadIdx.x >> 6) / waves * kBatch : 0;
  const int row_step = NARROW ? 4 / waves * kBatch : kBatch;
  const int lane = NARROW ? threadIdx.x & (64 * waves - 1) : threadIdx.x;
  uint32_t far = 0;
  for (int j0 = first * kTileBins; j0 < a.Fp; j0 += stride * kTileBins) {
    const Bins b(a, j0 + 4 * lane);
    const bool in = b.j < (uint32_t)a.Fp;
    const uint32_t jc = in ? b.j : 0;
    int64_t cell = -1;                 // the corners held in c
    f32x4 c[4] = {};
#pragma unroll 1
    for (int rb = row0; rb < n_rows; rb += row_step) {
      RowInfo q[kBatch];
      float* out[kBatch];
      f32x4 t0[kBatch], t1[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        int64_t row;
        q[u] = record(rb + u, &row);
        out[u] = a.panel + row * Fp;
        const float* tr = a.tau + (int64_t)q[u].li * Fp + jc;
        t0[u] = *reinterpret_cast<const f32x4*>(tr);
        t1[u] = *reinterpret_cast<const f32x4*>(tr + Fp);
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const bool src = q[u].valid && q[u].src;
        f32x4 ps = {0.f, 0.f, 0.f, 0.f};
        if (src) {
          if (q[u].sbase != cell) {
            cell = q[u].sbase;
            const float* p = a.cube + cell;
            c[0] = b.cube(p, a.F);
            c[1] = b.cube(p + ld, a.F);
            c[2] = b.cube(p + crow, a.F);
            c[3] = b.cube(p + crow + ld, a.F);
          }
          ps = q[u].w[0] * c[0] + q[u].w[1] * c[1] + q[u].w[2] * c[2] + q[u].w[3] * c[3];
        }
        f32x4 dP = {0.f, 0.f, 0.f, 0.f};
        if (q[u].valid)
          dP = row_deviation<ANY_EL>(b, a.F, t0[u], t1[u], ps, q[u].lw, q[u].csc, src, &far);
        // past the caches: the panel is larger than them, and what it would
        // push out (table rows, cube corners) is read again
        if (in) __builtin_nontemporal_store(dP, reinterpret_cast<f32x4*>(out[u] + b.j));
      }
    }
  }
  far_from_reference(a, far);
}

}  // namespace

// Rows in their own order: workgroup (b, y) computes rows R b .. R b + R - 1
// (one pixel, consecutive samples), R = a.rows_wg, in the bin passes y, y +
// gridDim.y, ...; the first R threads derive the row records.
template <bool ANY_EL, bool NARROW>
__global__ __launch_bounds__(256) void k_panel(PanelArgs a) {
  __shared__ RowInfo ri[kPanelRows];
  const int64_t row0 = (int64_t)blockIdx.x * a.rows_wg;
  if ((int)threadIdx.x < a.rows_wg) {
    uint32_t bucket;
    ri[threadIdx.x] = row_info(a, row0 + threadIdx.x, &bucket, blockIdx.y == 0);
  }
  __syncthreads();
  panel_rows<ANY_EL, NARROW>(a, a.rows_wg, blockIdx.y, gridDim.y, [&](int rr, int64_t* row) {
    *row = row0 + rr;
    RowInfo q = ri[rr];
    q.valid = uniform(q.valid);
    q.src = uniform(q.src);
    q.li = uniform(q.li);
    q.sbase = uniform(q.sbase);
    q.lw = uniform(q.lw);
    q.csc = uniform(q.csc);
    for (int k = 0; k < 4; ++k) q.w[k] = uniform(q.w[k]);
    return q;
  });
}

// hist[bucket] += 1 for every active lane; returns the lane's old value.
// The last bucket (rows without source, padding rows) can hold most rows
// of a chunk, so its lanes add once per wave (ballot, one atomic by the
// first of them, rank within the wave from the mask); other buckets are
// spread over cells and add per lane.
__device__ __forceinline__ uint32_t bucket_add(uint32_t* hist, uint32_t bucket,
                                               uint32_t hot) {
  const int lane = threadIdx.x & 63;
  const uint64_t m = __ballot(bucket == hot);
  if (bucket != hot) return atomicAdd(&hist[bucket], 1u);
  const int leader = __ffsll((unsigned long long)m) - 1;
  const uint32_t rank = (uint32_t)__popcll(m & ((1ull << lane) - 1));
  uint32_t base = 0;
  if (lane == leader) base = atomicAdd(&hist[hot], (uint32_t)__popcll(m));
  base = __shfl(base, leader);
  return base + rank;
}

// Sorted panel, step 1: one thread per row writes its record and bucket
// and counts the bucket.
__global__ __launch_bounds__(256) void k_panel_info(PanelArgs a) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= (int64_t)a.n_pix * a.Tpad) return;
  uint32_t bucket;
  const RowInfo q = row_info(a, r, &bucket, true);
  reinterpret_cast<RowInfo*>(a.rinfo)[r] = q;
  a.key[r] = bucket;
  bucket_add(a.hist, bucket, (uint32_t)(a.n_buckets - 1));
}

// Step 2: exclusive prefix sum of the bucket counts, in place (one
// workgroup of 1024 threads, 1024 buckets per round).
__global__ __launch_bounds__(1024) void k_panel_scan(uint32_t* hist, int n) {
  __shared__ uint32_t sh[1024];
  __shared__ uint32_t carry;
  if (threadIdx.x == 0) carry = 0;
  for (int base = 0; base < n; base += 1024) {
    const int i = base + threadIdx.x;
    const uint32_t v = i < n ? hist[i] : 0u;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      const uint32_t u = threadIdx.x >= off ? sh[threadIdx.x - off] : 0u;
      __syncthreads();
      sh[threadIdx.x] += u;
      __syncthreads();
    }
    if (i < n) hist[i] = carry + sh[threadIdx.x] - v;
    __syncthreads();
    if (threadIdx.x == 1023) carry += sh[1023];
    __syncthreads();
  }
}

// Step 3: scatter the row indices into bucket order.
__global__ __launch_bounds__(256) void k_panel_scatter(PanelArgs a) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= (int64_t)a.n_pix * a.Tpad) return;
  const uint32_t pos = bucket_add(a.hist, a.key[r], (uint32_t)(a.n_buckets - 1));
  a.order[pos] = (uint32_t)r;
}

// Step 4: workgroup (b, y) computes the rows at positions R b .. R b + R -
// 1 of the bucket order.  The order slots and row records are read through
// the constant address space at workgroup-uniform addresses, so they load
// into scalar registers: every address and branch of a row is scalar.
template <bool ANY_EL, bool NARROW>
__global__ __launch_bounds__(256) void k_panel_sorted(PanelArgs a) {
  typedef const __attribute__((address_space(4))) uint32_t* CU32;
  typedef const __attribute__((address_space(4))) RowInfo* CRow;
  const CU32 ord = (CU32)(uintptr_t)(a.order + (int64_t)blockIdx.x * a.rows_wg);
  const CRow rinfo = (CRow)(uintptr_t)a.rinfo;
  panel_rows<ANY_EL, NARROW>(a, a.rows_wg, blockIdx.y, gridDim.y, [&](int rr, int64_t* row) {
    const uint32_t r = ord[rr];
    *row = r;
    RowInfo q;
    q.valid = rinfo[r].valid;
    q.li = rinfo[r].li;
    q.lw = rinfo[r].lw;
    q.csc = rinfo[r].csc;
    q.src = rinfo[r].src;
    for (int k = 0; k < 4; ++k) q.w[k] = rinfo[r].w[k];
    q.sbase = rinfo[r].sbase;
    return q;
  });
}

__global__ void k_fill_u32(uint32_t* p, int n, uint32_t v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

void launch_panel(const PanelArgs& a0, hipStream_t s) {
  PanelArgs a = a0;
  const int64_t rows = (int64_t)a.n_pix * a.Tpad;
  const int passes = (a.Fp + kTileBins - 1) / kTileBins;
  // A workgroup per bin pass and fewer rows in each as long as that spreads the
  // rows more evenly over the card (us at 1750 bins, against 32 rows and all
  // passes in one: 33621 rows 90 / 106, 42000 109 / 119, 56000 135 / 146, 84000
  // 200 / 206; against 8 rows, 3000 bins: 160 rows 11.7 / 20.4, 2800 rows 30.8 /
  // 36.2, at 7600 rows of 1500 bins no longer, 45.6 / 44.2); in longer launches a row's record serves all its passes (526848
  // rows of 3000 bins: 3 % less than with one pass each).
  a.rows_wg = rows < 1024 ? 2 : rows < 4096 ? 4 : rows < 1024 * kPanelRows ? 8
              : rows < 2048 * kPanelRows ? 16 : kPanelRows;
  static_assert(2 % kBatch == 0, "rows per workgroup");
  const dim3 grid((unsigned)(rows / a.rows_wg), rows < 4096 * kPanelRows ? passes : 1);
  // rows enough for more than one wave (with 2 the other kernel is 0.4 us faster)
  const bool any_el = a.scan_kind == 2, narrow = a.Fp <= kNarrowBins && a.rows_wg > kBatch;
  if (a.n_buckets <= 1) {
    const auto kernel = any_el ? (narrow ? k_panel<true, true> : k_panel<true, false>)
                               : (narrow ? k_panel<false, true> : k_panel<false, false>);
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a);
    return;
  }
  const unsigned rb = (unsigned)((rows + 255) / 256);
  hipLaunchKernelGGL(k_fill_u32, dim3((a.n_buckets + 255) / 256), dim3(256), 0, s,
                     a.hist, a.n_buckets, 0u);
  hipLaunchKernelGGL(k_panel_info, dim3(rb), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_panel_scan, dim3(1), dim3(1024), 0, s, a.hist, a.n_buckets);
  hipLaunchKernelGGL(k_panel_scatter, dim3(rb), dim3(256), 0, s, a);
  const auto kernel = any_el ? (narrow ? k_panel_sorted<true, true> : k_panel_sorted<true, false>)
                             : (narrow ? k_panel_sorted<false, true> : k_panel_sorted<false, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a);
}

}  // namespace gtod
