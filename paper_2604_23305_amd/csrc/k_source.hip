// Far field of the aperture from panel polynomials, and the source
// convolution by fast Fourier transform.
//
// Far field: H depends on a direction and a frequency only through
// x = 2 pi rho R / lambda, so H(x) / H(0) is tabulated once, as a polynomial
// of degree 12 on every unit panel of x, and a table entry is one evaluation
// instead of a quadrature.  The integrand's band limit is 1 per unit of x
// (J0(x r / R), r <= R), so interpolation at 13 Chebyshev nodes leaves
// (1/2)^13 / (2^12 13!) = 5e-18 of H(0).
//
// Source: the table is an even kernel in both directions.  With both sides
// zero-padded to powers of two of at least 2 n - 1 the convolution is a
// product of spectra, all in FP64:
//   rows     two rows of a plane to a complex transform; the intensities'
//            half spectrum, and the (real) one of the even-extended table,
//            stored by column
//   columns  in place: transform, times the table's spectrum, inverse
//   inverse  rows, two to a transform; the powers as FP32 planes
// Its error is a few 2^-53 of the product of the 2-norms of intensities and
// table, whatever the output's own size.  An output too small for that to be
// 2^-26 of it (deep nulls around a lone bright node), and all of a plane with
// a value that is not finite, are summed directly in a last pass.
//
// 121 x 121 nodes, 3000 frequencies: 2.56 ms where every output's direct sum
// (643 G multiply-adds) took 180 ms and a quadrature per table entry 31.9 ms.
// Per 512 frequencies: columns 190 us, rows 97, inverse 49, planes 33, table 33,
// last pass 19, output 15.  The transforms are bound by LDS (11 words of 16 B
// per point and four stages) and by their barriers; the rest by memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "gtod_internal.h"

namespace gtod {

namespace {

constexpr double kC = 299792458.0;
constexpr double kPi = 3.14159265358979323846;
constexpr int kThreads = 256;
constexpr int kPoints = 1024;                      // points of a workgroup's transforms

// 16 B elements: one word of padding per 8 spreads the strided stores of the
// first stages over the banks
__device__ inline int slot(int i) { return i + (i >> 3); }
constexpr int kSlotsN = kPoints + kPoints / 8;

__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// kPoints / 2^LOG forward transforms in LDS, in order in and out: radix 4
// (one radix 2 last if LOG is odd), each thread one butterfly per stage.
// Enters and leaves with the workgroup synchronised.
template <int LOG>
__device__ inline void transforms(double2* z, const double2* tw) {
  constexpr int L = 1 << LOG, Q = L / 4;
  const int q = threadIdx.x / Q * L, b = threadIdx.x % Q;
  double2 v[4];
#pragma unroll
  for (int st = 0; st < LOG / 2; ++st) {
    const int ns = 1 << (2 * st), j = b & (ns - 1);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = z[slot(q + b + k * Q)];
    if (st) {
#pragma unroll
      for (int k = 1; k < 4; ++k) v[k] = cmul(v[k], tw[j * k * (Q / ns)]);
    }
    const double2 s0 = cadd(v[0], v[2]), d0 = csub(v[0], v[2]);
    const double2 s1 = cadd(v[1], v[3]), d1 = csub(v[1], v[3]);
    __syncthreads();
    const int o = q + (b - j) * 4 + j;
    z[slot(o)] = cadd(s0, s1);
    z[slot(o + ns)] = make_double2(d0.x + d1.y, d0.y - d1.x);
    z[slot(o + 2 * ns)] = csub(s0, s1);
    z[slot(o + 3 * ns)] = make_double2(d0.x - d1.y, d0.y + d1.x);
    __syncthreads();
  }
  if (LOG & 1) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = q + b + h * Q;
      const double2 u = z[slot(i)], w = cmul(z[slot(i + L / 2)], tw[b + h * Q]);
      z[slot(i)] = cadd(u, w);
      z[slot(i + L / 2)] = csub(u, w);
    }
    __syncthreads();
  }
}

// exp(-2 pi i m / L), m < L
template <int LOG>
__device__ inline void load_twiddles(double2* tw, const double2* all) {
  constexpr int L = 1 << LOG;
  for (int m = threadIdx.x; m < L; m += kThreads) tw[m] = all[m << (kMaxFftLog - LOG)];
}

__device__ inline double block_sum(double v, double* part) {
#pragma unroll
  for (int st = 32; st > 0; st >>= 1) v += __shfl_xor(v, st);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  return (part[0] + part[1]) + (part[2] + part[3]);
}

}  // namespace

// One workgroup (a wave) per panel: H / H(0) at the panel's 13 Chebyshev
// nodes by quadrature, lanes over the quadrature nodes, then the monomial
// coefficients in t = 2 (x - p) - 1.
__global__ __launch_bounds__(64) void k_beam_panels(BeamArgs a) {
  constexpr int N = kBeamTerms;
  const int lane = threadIdx.x;
  double x[N], h[N], h0 = 0.0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    x[i] = blockIdx.x + 0.5 + 0.5 * cospi((i + 0.5) / N);
    h[i] = 0.0;
  }
  for (int n = lane; n < a.n_nodes; n += 64) {
    const double q = a.gl_x[n];
    const double g = a.gl_w[n] * (q >= 1.0 ? 0.0 : exp10(a.t_edge_db * q * q / 20.0)) * q;
    h0 += g;
#pragma unroll
    for (int i = 0; i < N; ++i) h[i] += g * j0(x[i] * q);
  }
#pragma unroll
  for (int st = 32; st > 0; st >>= 1) {
    h0 += __shfl_xor(h0, st);
#pragma unroll
    for (int i = 0; i < N; ++i) h[i] += __shfl_xor(h[i], st);
  }
  __shared__ double c[N];
  if (lane < N) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) s += h[i] / h0 * cospi(lane * (i + 0.5) / N);
    c[lane] = s * (lane ? 2.0 : 1.0) / N;
  }
  __syncthreads();
  // T_k by its recurrence; lane m keeps the coefficient of t^m
  double t0 = lane == 0 ? 1.0 : 0.0, t1 = lane == 1 ? 1.0 : 0.0;
  double m = c[0] * t0 + c[1] * t1;
  for (int k = 2; k < N; ++k) {
    double up = __shfl_up(t1, 1);
    if (lane == 0) up = 0.0;
    const double t2 = 2.0 * up - t0;
    m += c[k] * t2;
    t0 = t1;
    t1 = t2;
  }
  if (lane < N) a.poly[blockIdx.x * N + lane] = m;
}

// One thread per grid node and kEvalF frequencies.
constexpr int kEvalF = 8;
__global__ __launch_bounds__(256) void k_beam_eval(BeamArgs a) {
  const int64_t per = (int64_t)a.n_a * a.n_b;
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (id >= per) return;
  const int ib = (int)(id / a.n_a), ia = (int)(id % a.n_a);
  const double rho = sqrt((ia * a.da) * (ia * a.da) + (ib * a.db) * (ib * a.db));
  const double k = 2.0 * kPi * rho / kC * a.r_tel;
  const int f1 = min((int)(blockIdx.y + 1) * kEvalF, a.F);
  for (int f = blockIdx.y * kEvalF; f < f1; ++f) {
    const double x = k * a.nu[f];
    const int p = min((int)x, a.panels - 1);
    const double t = 2.0 * (x - p) - 1.0;
    const double* c = a.poly + p * kBeamTerms;
    double q = c[kBeamTerms - 1];
#pragma unroll
    for (int m = kBeamTerms - 2; m >= 0; --m) q = fma(q, t, c[m]);
    a.table[f * per + id] = (float)(q * q);
  }
}

__global__ void k_src_twiddles(double2* tw) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= 1 << kMaxFftLog) return;
  double s, c;
  sincospi(-2.0 * m / (1 << kMaxFftLog), &s, &c);
  tw[m] = make_double2(c, s);
}

// Intensities times cos(el) by frequency plane: tiles of 64 nodes x 64
// frequencies through LDS, both sides in whole lines.
__global__ __launch_bounds__(256) void k_src_planes(SrcConvArgs a) {
  __shared__ float t[64][65];
  const int nn = a.n_az * a.n_el, n0 = blockIdx.x * 64, f0 = blockIdx.y * 64;
  const int lane = threadIdx.x & 63;
  for (int r = threadIdx.x >> 6; r < 64; r += 4) {
    const int q = n0 + r;
    if (q < nn && f0 + lane < a.nf)
      t[r][lane] = (float)((double)a.in[(int64_t)q * a.ld_in + a.f0 + f0 + lane] *
                           cos(a.el0 + q / a.n_az * a.del));
  }
  __syncthreads();
  for (int r = threadIdx.x >> 6; r < 64; r += 4)
    if (f0 + r < a.nf && n0 + lane < nn)
      a.planes[(int64_t)(f0 + r) * nn + n0 + lane] = t[lane][r];
}

// The powers' planes back to the caller's order.
__global__ __launch_bounds__(256) void k_src_out(SrcConvArgs a) {
  __shared__ float t[64][65];
  const int nn = a.n_az * a.n_el, n0 = blockIdx.x * 64, f0 = blockIdx.y * 64;
  const int lane = threadIdx.x & 63;
  for (int r = threadIdx.x >> 6; r < 64; r += 4)
    if (f0 + r < a.nf && n0 + lane < nn)
      t[r][lane] = a.powers[(int64_t)(f0 + r) * nn + n0 + lane];
  __syncthreads();
  for (int r = threadIdx.x >> 6; r < 64; r += 4) {
    const int q = n0 + r;
    if (q < nn && f0 + lane < a.nf)
      a.out[(int64_t)q * a.ld_out + a.f0 + f0 + lane] = t[lane][r];
  }
}

// Blocks (row group, frequency, intensities or table).
template <int LOG>
__global__ __launch_bounds__(kThreads) void k_src_rows(SrcConvArgs a) {
  constexpr int L = 1 << LOG, R = 2 * (kPoints / L);
  __shared__ double2 z[kSlotsN];
  __shared__ double2 tw[L];
  __shared__ double part[4];
  const int nx = a.n_az, ny = a.n_el, r0 = blockIdx.x * R, f = blockIdx.y, tid = threadIdx.x;
  const bool table = blockIdx.z != 0;
  load_twiddles<LOG>(tw, a.twiddles);
  const float* plane = (table ? a.table : a.planes) + (int64_t)f * nx * ny;
  double sq = 0.0;
#pragma unroll
  for (int p = tid; p < kPoints; p += kThreads) {
    const int q = p >> LOG, i = p & (L - 1), row = r0 + 2 * q;
    const int x = table ? min(i, L - i) : i;
    double u = 0.0, v = 0.0;
    if (x < nx) {
      if (row < ny) u = plane[row * nx + x];
      if (row + 1 < ny) v = plane[(row + 1) * nx + x];
    }
    z[slot(p)] = make_double2(u, v);
    sq += table && row ? 2.0 * (u * u) : u * u;
    sq += table ? 2.0 * (v * v) : v * v;
  }
  sq = block_sum(sq, part);
  if (tid == 0) a.norms[((int64_t)f * 2 + blockIdx.z) * gridDim.x + blockIdx.x] = sq;
  transforms<LOG>(z, tw);
  for (int p = tid; p < (L / 2 + 1) * R; p += kThreads) {
    const int k = p / R, r = p % R, q = (r >> 1) * L;
    if (r0 + r >= ny) continue;
    const double2 u = z[slot(q + k)];
    const int64_t o = ((int64_t)f * (L / 2 + 1) + k) * ny + r0 + r;
    if (table) {
      a.rows_table[o] = r & 1 ? u.y : u.x;
    } else {
      const double2 w = z[slot(q + ((L - k) & (L - 1)))];
      a.spectrum[o] = r & 1 ? make_double2(0.5 * (u.y + w.y), 0.5 * (w.x - u.x))
                            : make_double2(0.5 * (u.x + w.x), 0.5 * (u.y - w.y));
    }
  }
}

// Blocks (column group, frequency).
template <int LOG>
__global__ __launch_bounds__(kThreads) void k_src_columns(SrcConvArgs a) {
  constexpr int L = 1 << LOG, B = kPoints / L;
  __shared__ double2 z[kSlotsN];
  __shared__ double2 tw[L];
  __shared__ double spec[2 * kPoints];
  const int ny = a.n_el, c0 = blockIdx.x * 2 * B, f = blockIdx.y, tid = threadIdx.x;
  const int cols = (1 << a.log_x) / 2 + 1;
  load_twiddles<LOG>(tw, a.twiddles);
  const int64_t base = ((int64_t)f * cols + c0) * ny;
  const double* const h = a.rows_table + base;
#pragma unroll
  for (int p = tid; p < kPoints; p += kThreads) {
    const int q = p >> LOG, j = p & (L - 1), y = min(j, L - j);
    double u = 0.0, v = 0.0;
    if (y < ny) {
      if (c0 + 2 * q < cols) u = h[2 * q * ny + y];
      if (c0 + 2 * q + 1 < cols) v = h[(2 * q + 1) * ny + y];
    }
    z[slot(p)] = make_double2(u, v);
  }
  __syncthreads();
  transforms<LOG>(z, tw);
  const double norm = a.scale / ((double)L * (1 << a.log_x));
#pragma unroll
  for (int p = tid; p < kPoints; p += kThreads) {
    const int q = p >> LOG, j = p & (L - 1);
    const double2 u = z[slot(p)];
    spec[2 * q * L + j] = norm * u.x;
    spec[(2 * q + 1) * L + j] = norm * u.y;
  }
  for (int half = 0; half < 2; ++half) {
    const int c = half * B;
    if (c0 + c >= cols) break;
    double2* const s = a.spectrum + base + (int64_t)c * ny;
    __syncthreads();
#pragma unroll
    for (int p = tid; p < kPoints; p += kThreads) {
      const int q = p >> LOG, j = p & (L - 1);
      const bool in = j < ny && c0 + c + q < cols;
      z[slot(p)] = in ? s[q * ny + j] : make_double2(0.0, 0.0);
    }
    __syncthreads();
    transforms<LOG>(z, tw);
    // the inverse is the forward transform with real and imaginary parts
    // exchanged before and after
#pragma unroll
    for (int p = tid; p < kPoints; p += kThreads) {
      const double2 u = z[slot(p)];
      const double g = spec[c * L + p];
      z[slot(p)] = make_double2(g * u.y, g * u.x);
    }
    __syncthreads();
    transforms<LOG>(z, tw);
#pragma unroll
    for (int p = tid; p < kPoints; p += kThreads) {
      const int q = p >> LOG, j = p & (L - 1);
      if (j >= ny || c0 + c + q >= cols) continue;
      const double2 u = z[slot(p)];
      s[q * ny + j] = make_double2(u.y, u.x);
    }
  }
}

// Blocks (row group, frequency).  Outputs for the direct pass become NaN.
template <int LOG>
__global__ __launch_bounds__(kThreads) void k_src_inverse(SrcConvArgs a) {
  constexpr int L = 1 << LOG, B = kPoints / L, R = 2 * B;
  __shared__ double2 z[kSlotsN];
  __shared__ double2 tw[L];
  const int nx = a.n_az, ny = a.n_el, r0 = blockIdx.x * R, f = blockIdx.y, tid = threadIdx.x;
  load_twiddles<LOG>(tw, a.twiddles);
  for (int p = tid; p < (L / 2 + 1) * B; p += kThreads) {
    const int k = p / B, q = p % B, row = r0 + 2 * q;
    double2 u = make_double2(0.0, 0.0), v = u;
    const double2* const s = a.spectrum + ((int64_t)f * (L / 2 + 1) + k) * ny + row;
    if (row < ny) u = s[0];
    if (row + 1 < ny) v = s[1];
    if (k == 0 || k == L / 2) u.y = v.y = 0.0;
    // u + i v, exchanged
    z[slot(q * L + k)] = make_double2(u.y + v.x, u.x - v.y);
    if (k && k < L / 2) z[slot(q * L + L - k)] = make_double2(v.x - u.y, u.x + v.y);
  }
  __syncthreads();
  transforms<LOG>(z, tw);
  double n2[2] = {0.0, 0.0};
  const double* const norms = a.norms + (int64_t)f * 2 * gridDim.x;
  for (int i = 0; i < (int)gridDim.x; ++i) {
    n2[0] += norms[i];
    n2[1] += norms[gridDim.x + i];
  }
  const double least = kSrcLeast * a.scale * sqrt(n2[0] * n2[1]);
  float* const out = a.powers + (int64_t)f * nx * ny;
#pragma unroll
  for (int p = tid; p < kPoints; p += kThreads) {
    const int q = p >> LOG, i = p & (L - 1), row = r0 + 2 * q;
    if (i >= nx) continue;
    const double2 u = z[slot(p)];
    if (row < ny) out[row * nx + i] = fabs(u.y) >= least ? (float)u.y : NAN;
    if (row + 1 < ny) out[(row + 1) * nx + i] = fabs(u.x) >= least ? (float)u.x : NAN;
  }
}

// Blocks (frequency, part of the nodes): sums every output that the inverse left
// as NaN over all nodes, two to a thread.  A NaN among the intensities reaches
// every output, and stays.  A workgroup looks at the outputs of its own part
// alone.  Parts enough for one workgroup per CU: a lone node on 200 x 99 at one
// frequency, nearly all of whose outputs come this way, 3.6 ms in one part, 1.2 ms.
constexpr int kRest = 512;
__global__ __launch_bounds__(kRest) void k_src_direct_rest(SrcConvArgs a) {
  extern __shared__ float smem[];
  __shared__ uint16_t queue[3 * kRest];
  __shared__ int count;
  const int nn = a.n_az * a.n_el, tid = threadIdx.x;
  const int part = (nn + gridDim.y - 1) / gridDim.y;
  const int first = min((int)blockIdx.y * part, nn), last = min(first + part, nn);
  float* const out = a.powers + (int64_t)blockIdx.x * nn;
  bool any = false;
  for (int q = first + tid; q < last; q += kRest) any |= isnan(out[q]);
  if (!__syncthreads_or(any)) return;
  float* const sI = smem;
  float* const sF = smem + nn;
  any = false;
  for (int q = tid; q < nn; q += kRest) {
    sI[q] = a.planes[(int64_t)blockIdx.x * nn + q];
    sF[q] = a.table[(int64_t)blockIdx.x * nn + q];
    any |= isnan(sI[q]);
  }
  if (tid == 0) count = 0;
  if (__syncthreads_or(any)) return;
  for (int q0 = first; q0 < last; q0 += kRest) {
    const int q = q0 + tid;
    if (q < last && isnan(out[q])) queue[atomicAdd(&count, 1)] = (uint16_t)q;
    __syncthreads();
    const int n = count;
    __syncthreads();
    if (n < 2 * kRest && q0 + kRest < last) continue;
    for (int b = 0; b < n; b += 2 * kRest) {
      const int o0 = queue[min(b + tid, n - 1)], o1 = queue[min(b + kRest + tid, n - 1)];
      const int i0 = o0 % a.n_az, j0 = o0 / a.n_az, i1 = o1 % a.n_az, j1 = o1 / a.n_az;
      double acc0 = 0.0, acc1 = 0.0;
      for (int jp = 0; jp < a.n_el; ++jp) {
        const float* const rI = sI + jp * a.n_az;
        const float* const r0 = sF + abs(j0 - jp) * a.n_az;
        const float* const r1 = sF + abs(j1 - jp) * a.n_az;
#pragma unroll 4
        for (int ip = 0; ip < a.n_az; ++ip) {
          const double v = rI[ip];
          acc0 = fma(v, (double)r0[abs(i0 - ip)], acc0);
          acc1 = fma(v, (double)r1[abs(i1 - ip)], acc1);
        }
      }
      if (b + tid < n) out[o0] = (float)(a.scale * acc0);
      if (b + kRest + tid < n) out[o1] = (float)(a.scale * acc1);
    }
    __syncthreads();
    if (tid == 0) count = 0;
    __syncthreads();
  }
}

void launch_beam_polynomials(const BeamArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_beam_panels, dim3(a.panels), dim3(64), 0, s, a);
}

void launch_beam_eval(const BeamArgs& a, hipStream_t s) {
  const int64_t per = (int64_t)a.n_a * a.n_b;
  for (int f0 = 0; f0 < a.F; f0 += 65535 * kEvalF) {
    BeamArgs b = a;
    b.F = std::min(a.F - f0, 65535 * kEvalF);
    b.nu += f0;
    b.table += f0 * per;
    hipLaunchKernelGGL(k_beam_eval, dim3((unsigned)((per + 255) / 256), (b.F + kEvalF - 1) / kEvalF),
                       dim3(256), 0, s, b);
  }
}

void launch_src_twiddles(double2* tw, hipStream_t s) {
  hipLaunchKernelGGL(k_src_twiddles, dim3((1 << kMaxFftLog) / 256), dim3(256), 0, s, tw);
}

int src_fft_log(int n) {
  int log = kMinFftLog;
  while ((1 << log) < 2 * n - 1) ++log;
  return log;
}

// doubles of the norms of one frequency
int src_fft_norms(int n_az, int n_el) {
  const int rows = 2 * (kPoints >> src_fft_log(n_az));
  return 2 * ((n_el + rows - 1) / rows);
}

template <int LOG>
static void rows(const SrcConvArgs& a, hipStream_t s, bool inverse) {
  const int per = 2 * (kPoints >> LOG), groups = (a.n_el + per - 1) / per;
  if (inverse) hipLaunchKernelGGL(k_src_inverse<LOG>, dim3(groups, a.nf), dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL(k_src_rows<LOG>, dim3(groups, a.nf, 2), dim3(kThreads), 0, s, a);
}

template <int LOG>
static void columns(const SrcConvArgs& a, hipStream_t s) {
  const int per = 2 * (kPoints >> LOG), cols = (1 << a.log_x) / 2 + 1;
  hipLaunchKernelGGL(k_src_columns<LOG>, dim3((cols + per - 1) / per, a.nf), dim3(kThreads), 0, s,
                     a);
}

int launch_source_fft(const SrcConvArgs& a, hipStream_t s) {
  const int nn = a.n_az * a.n_el;
  const size_t lds = (size_t)2 * nn * sizeof(float);
  if (hipFuncSetAttribute((const void*)k_src_direct_rest,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return 1;
  auto any_rows = [&](bool inverse) {
    switch (a.log_x) {
      case 5: return rows<5>(a, s, inverse);
      case 6: return rows<6>(a, s, inverse);
      case 7: return rows<7>(a, s, inverse);
      case 8: return rows<8>(a, s, inverse);
      default: return rows<9>(a, s, inverse);
    }
  };
  const dim3 tiles((nn + 63) / 64, (a.nf + 63) / 64);
  hipLaunchKernelGGL(k_src_planes, tiles, dim3(256), 0, s, a);
  any_rows(false);
  switch (a.log_y) {
    case 5: columns<5>(a, s); break;
    case 6: columns<6>(a, s); break;
    case 7: columns<7>(a, s); break;
    case 8: columns<8>(a, s); break;
    default: columns<9>(a, s);
  }
  any_rows(true);
  const int parts = std::max(1, std::min(256 / a.nf, (nn + 2 * kRest - 1) / (2 * kRest)));
  hipLaunchKernelGGL(k_src_direct_rest, dim3(a.nf, parts), dim3(kRest), lds, s, a);
  hipLaunchKernelGGL(k_src_out, tiles, dim3(256), 0, s, a);
  return 0;
}

}  // namespace gtod
