// Input preparation (section 2.2): far-field pattern of the Gaussian-tapered
// aperture, source-beam convolution (Eq. convolve_src) and footprint
// smoothing of the PWV screen.
//
// Aperture (Eq. aper_dist): A(r) = 10^(t_edge (r / R)^2 / 20) for r < R.
// Far field: F = |FT{A}|^2 / peak.  For a circularly symmetric field the
// two-dimensional transform is the Hankel transform
//   H(rho) = int_0^R A(r) J0(2 pi rho r / lambda) r dr,   F = (H / H(0))^2,
// evaluated with Gauss-Legendre quadrature on [0, R] (the node count is
// chosen by the runtime from the largest 2 pi rho R / lambda of the grid).
// Source: P(i, j) = A_p daz del sum_{i', j'} I(i', j') cos(el_j') F(rho),
// rho = sqrt(((i - i') daz)^2 + ((j - j') del)^2).  Small and very long grids,
// summed directly here (the others by transforms, in k_source.hip): one block
// per (frequency, 32x32 output tile) holding the frequency's weighted intensity
// plane and its far-field table F[|dj|][|di|] in LDS; each thread sums 2x2
// outputs in FP64.  Screen: weights A(r) normalised to 1 over the cells within R,
// edges clamped; A is a product of a function of x and one of y inside the
// disk, so a row's cells are summed once per row of the footprint (in strips), or
// cell by cell where the footprint or the screen is small.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "gtod_internal.h"
#include "lds_barrier.h"

namespace gtod {

namespace {

constexpr double kC = 299792458.0;
constexpr double kPi = 3.14159265358979323846;

__device__ inline double aperture(double r, double R, double t_edge_db) {
  if (r >= R) return 0.0;
  const double q = r / R;
  return exp10(t_edge_db * q * q / 20.0);
}

}  // namespace

// Gauss-Legendre nodes and weights on [0, 1]: Newton on P_n from the
// Chebyshev-like initial guess, one thread per node.
__global__ void k_gauss_legendre(double* x, double* w, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double z = cos(kPi * (i + 0.75) / (n + 0.5));
  double dp = 1.0;
  for (int it = 0; it < 100; ++it) {
    double p0 = 1.0, p1 = z;
    for (int k = 2; k <= n; ++k) {
      const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
      p0 = p1;
      p1 = p2;
    }
    dp = n * (z * p1 - p0) / (z * z - 1.0);
    const double dz = p1 / dp;
    z -= dz;
    if (fabs(dz) < 1e-16) break;
  }
  x[i] = 0.5 * (1.0 - z);
  w[i] = 1.0 / ((1.0 - z * z) * dp * dp);
}

// One thread per (a, b, frequency), a quadrature each: for calls of few
// entries (the others from polynomials, in k_source.hip).
__global__ __launch_bounds__(256) void k_beam_table(BeamArgs a) {
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t per = (int64_t)a.n_a * a.n_b;
  if (id >= per * a.F) return;
  const int f = (int)(id / per);
  const int rem = (int)(id % per);
  const int ib = rem / a.n_a, ia = rem % a.n_a;
  const double lam = kC / a.nu[f];
  const double rho = sqrt((ia * a.da) * (ia * a.da) + (ib * a.db) * (ib * a.db));
  const double k = 2.0 * kPi * rho / lam;
  double h = 0.0, h0 = 0.0;
  for (int n = 0; n < a.n_nodes; ++n) {
    const double r = a.r_tel * a.gl_x[n];
    const double g = a.gl_w[n] * aperture(r, a.r_tel, a.t_edge_db) * r;
    h0 += g;
    h += g * j0(k * r);
  }
  const double q = h / h0;
  a.table[id] = (float)(q * q);
}

// Block: frequency f0 + blockIdx.y, output tile blockIdx.x (32x32).
__global__ __launch_bounds__(256) void k_source_conv(SrcConvArgs a) {
  extern __shared__ float dyn[];
  const int nn = a.n_az * a.n_el;
  float* sI = dyn;          // [n_el][n_az] I cos(el)
  float* sF = dyn + nn;     // [n_el][n_az] F(|dj|, |di|)
  const int fl = blockIdx.y, f = a.f0 + fl;
  const int tiles_x = (a.n_az + 31) / 32;
  const int ti = (blockIdx.x % tiles_x) * 32, tj = (blockIdx.x / tiles_x) * 32;
  const float* tab = a.table + (int64_t)fl * nn;
  for (int q = threadIdx.x; q < nn; q += 256) {
    const int j = q / a.n_az;
    sI[q] = (float)((double)a.in[(int64_t)q * a.ld_in + f] * cos(a.el0 + j * a.del));
    sF[q] = tab[q];
  }
  __syncthreads();
  const int i0 = ti + (threadIdx.x & 15), j0_ = tj + (threadIdx.x >> 4);
  const int i1 = i0 + 16, j1 = j0_ + 16;
  double acc00 = 0.0, acc01 = 0.0, acc10 = 0.0, acc11 = 0.0;
  for (int jp = 0; jp < a.n_el; ++jp) {
    const float* rI = sI + jp * a.n_az;
    // rows beyond the grid only occur for outputs outside it (not stored);
    // clamping keeps their reads inside the table
    const float* rF0 = sF + min(abs(j0_ - jp), a.n_el - 1) * a.n_az;
    const float* rF1 = sF + min(abs(j1 - jp), a.n_el - 1) * a.n_az;
    for (int ip = 0; ip < a.n_az; ++ip) {
      const double v = rI[ip];
      const int e0 = min(abs(i0 - ip), a.n_az - 1), e1 = min(abs(i1 - ip), a.n_az - 1);
      acc00 = fma(v, (double)rF0[e0], acc00);
      acc01 = fma(v, (double)rF0[e1], acc01);
      acc10 = fma(v, (double)rF1[e0], acc10);
      acc11 = fma(v, (double)rF1[e1], acc11);
    }
  }
  auto put = [&](int i, int j, double acc) {
    if (i < a.n_az && j < a.n_el)
      a.out[((int64_t)j * a.n_az + i) * a.ld_out + f] = (float)(a.scale * acc);
  };
  put(i0, j0_, acc00);
  put(i1, j0_, acc01);
  put(i0, j1, acc10);
  put(i1, j1, acc11);
}

constexpr int kFactorPitch = 64;   // one word per lane

__device__ inline double lane_value(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(u >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Factors of the footprint, one block: A(r) = gx(x) gy(y) for r < R, so row
// dy of the footprint is gy[dy] times the gx-weighted cells up to width[dy]
// on either side (-1: none).  w: gx[0 .. rx], then gy[0 .. ry] with the
// normalisation (the sum of the weights is 1; fixed-order sum), then width,
// each at a pitch of kFactorPitch words.
__global__ __launch_bounds__(64) void k_screen_weights(ScreenConvArgs a) {
  __shared__ double sum[64], gx[64];
  double* gy = a.w + kFactorPitch;
  int* width = reinterpret_cast<int*>(a.w + 2 * kFactorPitch);
  auto factor = [&](double x) {
    const double q = x / a.r_tel;
    return exp10(a.t_edge_db * q * q / 20.0);
  };
  const int d = threadIdx.x;
  gx[d] = d <= a.rx ? factor(d * a.dx) : 0.0;
  a.w[d] = gx[d];
  __syncthreads();
  const double gyd = d <= a.ry ? factor(d * a.dy) : 0.0;
  double acc = 0.0;
  int wd = -1;
  if (d <= a.ry)
    for (int c = 0; c <= a.rx; ++c) {
      const double x = c * a.dx, y = d * a.dy;
      if (!(sqrt(x * x + y * y) < a.r_tel)) break;
      acc += (c ? 2.0 : 1.0) * gx[c];
      wd = c;
    }
  sum[d] = (d ? 2.0 : 1.0) * gyd * acc;
  __syncthreads();
  for (int st = 32; st > 0; st >>= 1) {
    if (d < st) sum[d] += sum[d + st];
    __syncthreads();
  }
  const double g = gyd / sum[0];
  // cells whose weight underflows to zero take no part
  while (wd >= 0 && gx[wd] * g == 0.0) --wd;
  gy[d] = g;
  width[d] = wd;
}

// One workgroup: 256 columns of a strip of rows, a thread per column.  Input
// rows come one at a time through LDS; a thread forms the running sum of its
// gx-weighted cells outwards from the column, keeps every partial sum in a
// column of LDS of its own, takes the row sum of each footprint row from there
// (the partial sum at its width), and adds them to the 2 N + 1 output rows that
// the input row reaches, which it holds in registers and shifts by one as it
// stores the finished one.  That is about 4 N multiplications per cell instead
// of one per cell of the disk, and without a branch; LDS bounds it (4 N words
// read or written per cell).  512 x 65536 cells of 0.2 m under a 5 m dish (1961
// cells of footprint): 19.1 ms when every output summed its whole disk from a
// 2-D tile, 1.46 ms with branches on the widths instead of partial sums in LDS,
// 0.84 ms now; error against the exact sum 3.4e-16 rms (1.1e-15 before).
template <int N>
__global__ __launch_bounds__(256) void k_screen_conv(ScreenConvArgs a) {
  __shared__ double buf[2][256 + 2 * N];
  __shared__ double partial[N + 1][256];
  const int tid = threadIdx.x, lane = tid & 63;
  const double gx = a.w[lane], gy = a.w[kFactorPitch + lane];
  const int wd = reinterpret_cast<const int*>(a.w + 2 * kFactorPitch)[lane];
  const int64_t x0 = (int64_t)blockIdx.x * 256, y0 = (int64_t)blockIdx.y * a.strip;
  const int64_t y1 = min(y0 + a.strip, a.ny);
  auto column = [&](int64_t x) { return x < 0 ? (int64_t)0 : (x >= a.nx ? a.nx - 1 : x); };
  const int64_t xa = column(x0 - N + tid), xb = column(x0 - N + 256 + tid);
  const bool two = tid < 2 * N;
  double va = 0.0, vb = 0.0;
  auto load = [&](int64_t y) {
    const double* row = a.in + (y < 0 ? (int64_t)0 : (y >= a.ny ? a.ny - 1 : y)) * a.nx;
    va = row[xa];
    if (two) vb = row[xb];
  };
  double acc[2 * N + 2];
#pragma unroll
  for (int k = 0; k < 2 * N + 2; ++k) acc[k] = 0.0;
  load(y0 - N);
  for (int64_t y = y0 - N; y < y1 + N; ++y) {
    double* const b = buf[(y - y0) & 1];
    b[tid] = va;
    if (two) b[256 + tid] = vb;
    load(y + 1);
    lds_barrier();
    const double* const s = b + N + tid;
    double h = lane_value(gx, 0) * s[0];
    partial[0][tid] = h;
#pragma unroll
    for (int d = 1; d <= N; ++d) {
      h = fma(lane_value(gx, d), s[-d] + s[d], h);
      partial[d][tid] = h;
    }
    // a thread reads back only what it wrote
    double H[N + 1];
#pragma unroll
    for (int dy = 0; dy <= N; ++dy) {
      const int w = __builtin_amdgcn_readlane(wd, dy);
      H[dy] = partial[max(w, 0)][tid];
      if (w < 0) H[dy] = 0.0;
    }
#pragma unroll
    for (int k = 0; k <= 2 * N; ++k) {
      const int dy = k < N ? N - k : k - N;
      acc[k] = fma(lane_value(gy, dy), H[dy], acc[k + 1]);
    }
    const int64_t o = y - N;
    if (o >= y0 && x0 + tid < a.nx) a.out[o * a.nx + x0 + tid] = acc[0];
  }
}

// Small footprints and narrow screens: 64 x 32 outputs and the cells around them
// in LDS, thread (tx, ty) sums the footprint of rows ty + 4 r of column tx cell by
// cell.  Nothing is serial along the screen, so small calls fill the card.
constexpr int kTileX = 64, kTileY = 32;
static int64_t tile_lds(const ScreenConvArgs& a) {
  return 8 * ((int64_t)(2 * a.rx + 1) * (2 * a.ry + 1) +
              (int64_t)(kTileX + 2 * a.rx) * (kTileY + 2 * a.ry));
}
__global__ __launch_bounds__(256) void k_screen_tile(ScreenConvArgs a) {
  extern __shared__ double dsm[];
  const int wx = 2 * a.rx + 1, wy = 2 * a.ry + 1;
  const int TW = kTileX + 2 * a.rx, TH = kTileY + 2 * a.ry;
  double* const sw = dsm;              // [wy][wx]
  double* const st = dsm + wx * wy;    // [TH][TW]
  const double* const gx = a.w;
  const double* const gy = a.w + kFactorPitch;
  const int* const width = reinterpret_cast<const int*>(a.w + 2 * kFactorPitch);
  const int64_t tiles_x = (a.nx + kTileX - 1) / kTileX;
  const int64_t x0 = (blockIdx.x % tiles_x) * kTileX;
  const int64_t y0 = (blockIdx.x / tiles_x) * kTileY;
  for (int q = threadIdx.x; q < wx * wy; q += 256) {
    const int dx = abs(q % wx - a.rx), dy = abs(q / wx - a.ry);
    sw[q] = dx <= width[dy] ? gx[dx] * gy[dy] : 0.0;
  }
  for (int q = threadIdx.x; q < TW * TH; q += 256) {
    int64_t y = y0 - a.ry + q / TW, x = x0 - a.rx + q % TW;
    y = y < 0 ? 0 : (y >= a.ny ? a.ny - 1 : y);
    x = x < 0 ? 0 : (x >= a.nx ? a.nx - 1 : x);
    st[q] = a.in[y * a.nx + x];
  }
  __syncthreads();
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  double acc[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) acc[r] = 0.0;
  for (int dy = 0; dy < wy; ++dy) {
    for (int dx = 0; dx < wx; ++dx) {
      const double w = sw[dy * wx + dx];
      if (w == 0.0) continue;
      const double* const col = st + (ty + dy) * TW + tx + dx;
#pragma unroll
      for (int r = 0; r < 8; ++r) acc[r] += w * col[4 * r * TW];
    }
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int64_t y = y0 + ty + 4 * r, x = x0 + tx;
    if (y < a.ny && x < a.nx) a.out[y * a.nx + x] = acc[r];
  }
}

void launch_gauss_legendre(double* x, double* w, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_gauss_legendre, dim3((n + 127) / 128), dim3(128), 0, s, x, w, n);
}

void launch_beam_table(const BeamArgs& a, hipStream_t s) {
  const int64_t n = (int64_t)a.n_a * a.n_b * a.F;
  hipLaunchKernelGGL(k_beam_table, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
}

int launch_source_conv(const SrcConvArgs& a, hipStream_t s) {
  const size_t lds = (size_t)2 * a.n_az * a.n_el * sizeof(float);
  if (hipFuncSetAttribute((const void*)k_source_conv,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return 1;
  const int tiles = ((a.n_az + 31) / 32) * ((a.n_el + 31) / 32);
  hipLaunchKernelGGL(k_source_conv, dim3(tiles, a.nf), dim3(256), lds, s, a);
  return 0;
}

void launch_screen_conv(const ScreenConvArgs& a0, hipStream_t s) {
  ScreenConvArgs a = a0;
  hipLaunchKernelGGL(k_screen_weights, dim3(1), dim3(64), 0, s, a);
  const int n = std::max(a.rx, a.ry);
  // the longest strips (their ry extra rows on either side are work done
  // again) that still give every CU the two workgroups it holds: 512 x 65536
  // cells of 0.2 m 0.92 -> 0.84 ms against four workgroups, 300 x 8000 of 0.25 m
  // 299 -> 217 us
  const int64_t cols = (a.nx + 255) / 256;
  const int64_t strips = std::max<int64_t>(1, 512 / cols);
  a.strip = (int)std::max<int64_t>((a.ny + strips - 1) / strips, 16);
  const dim3 grid((unsigned)cols, (unsigned)((a.ny + a.strip - 1) / a.strip));
  if (n <= 16) {
    // Cell by cell or in strips, by the time either takes (us; the constants
    // from screens of 16 x 16 to 512 x 65536 and footprints of 0 to 12 cells):
    // a tile's chain of 0.148 per cell of the footprint, of which a CU overlaps
    // as many as its LDS holds down to 0.0577 each; a strip's rows, each a chain
    // from load to store, one or two strips to a CU.  4 cells, 64 x 64: 19 by
    // tiles, 30 in strips; 512 x 65536: 281 and 298; 8 cells: 44 and 31, 755 and
    // 300; 100000 x 64: 171 and 224.
    const double taps = 0.785 * (2 * a.rx + 1) * (2 * a.ry + 1);
    const int64_t lds = tile_lds(a), resident = std::min<int64_t>(8, (160 << 10) / lds);
    const int64_t tiles = (a.nx + kTileX - 1) / kTileX * ((a.ny + kTileY - 1) / kTileY);
    const int64_t per_cu = (tiles + 255) / 256;
    auto round = [&](int64_t k) { return k ? std::max(0.148, 0.0577 * (double)k) * taps : 0.0; };
    const double by_tiles = 10.0 + (double)(per_cu / resident) * round(resident) +
                            round(per_cu % resident);
    const bool shared = (int64_t)grid.x * grid.y > 256;
    const double per_row = n <= 8 ? (shared ? 1.08 : 0.78) : (shared ? 1.83 : 1.32);
    const double by_strips = 5.0 + (std::min<int64_t>(a.strip, a.ny) + (n <= 8 ? 16 : 32)) * per_row;
    if (by_tiles < by_strips) {
      hipLaunchKernelGGL(k_screen_tile, dim3((unsigned)tiles), dim3(256), lds, s, a);
      return;
    }
  }
  if (n <= 8) hipLaunchKernelGGL(k_screen_conv<8>, grid, dim3(256), 0, s, a);
  else if (n <= 16) hipLaunchKernelGGL(k_screen_conv<16>, grid, dim3(256), 0, s, a);
  else if (n <= 25) hipLaunchKernelGGL(k_screen_conv<25>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_screen_conv<32>, grid, dim3(256), 0, s, a);
}

}  // namespace gtod
