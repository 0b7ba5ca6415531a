// 1/f noise by the method of Timmer and Koenig (section 2.6), added into
// the TOD.
//
// Series (p, k) of N = 2^q samples (first t_total kept): bins j = 1..N/2-1
// get X_j = c_j (z_re + i z_im), c_j = sqrt(A_k f_j^-alpha_k N f_s / 4) / N,
// f_j = j f_s / N, with (z_re, z_im) the Box-Muller pair of Philox counter
// (j, k, p, 1); DC and Nyquist are zero.  x = inverse real DFT of X.
//
// The real inverse transform of length N is done as one complex inverse
// DFT of length M = N/2 on
//   Z_k = (X_k + conj X_{M-k}) + i e^{2 pi i k/N} (X_k - conj X_{M-k}),
// whose output z_m = x_{2m} + i x_{2m+1}.  The complex DFT uses the
// four-step split M = M1 * M2 (M2 <= 4096), k = k1 + M1 k2, m = m1 M2 + m2:
//   pass 1, per (series, column set closed under k -> M-k): the spectrum
//     bins of those columns drawn once, Z built in place, length-M2 DFTs
//     over k2 (the stride costs nothing as nothing is read), times
//     e^{2 pi i k1 m2 / M}, stored contiguous in m2;
//   pass 2, per (series, block of B2 consecutive m2): length-M1 DFTs over
//     k1, read and written as runs of B2 consecutive m2.
// With M1 = 1 pass 1 writes the output directly.
//
// Each DFT runs in LDS as self-sorting (Stockham) passes of radix 16, then
// one of radix 2, 4 or 8 for the remaining factor: a thread loads the R
// inputs j + r L/R of one group into registers, multiplies them by
// e^{2 pi i r (j mod S) / (S R)} (S = product of the radices before),
// does the length-R DFT in registers and stores output s at
// (j div S) S R + (j mod S) + s S.  Input and output are in natural order.
// Pass twiddles come from one table of e^{2 pi i m / 4096} in global
// memory (evaluated with sincospi on exact arguments): a pass loads w, w^2,
// w^4, w^8 for its group and forms the other powers as products of at
// most four of them.  The in-register DFTs use the constants cos, sin(2 pi
// m / 16).  The real-to-complex and four-step twiddles of a thread's 16
// elements are a geometric sequence, taken as w0 times products of at most
// four sincospi factors.  Pass 1 keeps its one or
// two transforms contiguous in LDS with one float2 of padding after every
// 16, so that the stride-16 stores of the first pass hit distinct banks;
// pass 2 interleaves its B2 transforms (element i of transform t at
// i B2 + t, t fastest across lanes), which makes every access consecutive.
// All index arithmetic is shifts and masks (lengths are powers of two).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gtod_internal.h"
#include "philox.h"

namespace gtod {

namespace {

constexpr int kLdsC = 4096;   // complex values per transform set

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) {
  return make_float2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ float2 csub(float2 a, float2 b) {
  return make_float2(a.x - b.x, a.y - b.y);
}

__device__ __forceinline__ float2 twiddle(uint32_t num, int lg_den) {
  // e^{2 pi i num / 2^lg_den}, num < 2^lg_den <= 2^24
  const float x = ldexpf((float)num, 1 - lg_den);  // 2 num / den, exact
  float s, c;
  sincospif(x, &s, &c);
  return make_float2(c, s);
}

// e^{2 pi i (e0 + i d) / 2^lg} for i = 0 .. 15: w0 times the product of the
// factors e^{2 pi i 2^b d / 2^lg} for the set bits b of i, each evaluated
// with sincospi on an exact argument (at most five roundings in all).
struct GeoTwiddle {
  float2 w0, f[4];
  __device__ GeoTwiddle(uint32_t e0, uint32_t d, int lg) {
    const uint32_t mask = (1u << lg) - 1;
    w0 = twiddle(e0 & mask, lg);
#pragma unroll
    for (int b = 0; b < 4; ++b) f[b] = twiddle((d << b) & mask, lg);
  }
  __device__ float2 operator()(int i) const {
    float2 w = w0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if ((i >> b) & 1) w = cmul(w, f[b]);
    return w;
  }
};

// cos and sin of 2 pi m / 16, m = 0 .. 7, rounded to float
__device__ constexpr float kCos16[8] = {
    1.0f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f,
    0.0f, -0.38268343236508977f, -0.70710678118654752f, -0.92387953251128674f};
__device__ constexpr float kSin16[8] = {
    0.0f, 0.38268343236508977f, 0.70710678118654752f, 0.92387953251128674f,
    1.0f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f};

// a e^{2 pi i m / 16}; m is a constant once the callers are unrolled
__device__ __forceinline__ float2 mul_w16(float2 a, int m) {
  if (m == 0) return a;
  if (m == 4) return make_float2(-a.y, a.x);
  return make_float2(a.x * kCos16[m] - a.y * kSin16[m],
                     a.x * kSin16[m] + a.y * kCos16[m]);
}

constexpr int brev_c(int x, int bits) {
  int r = 0;
  for (int b = 0; b < bits; ++b) r |= ((x >> b) & 1) << (bits - 1 - b);
  return r;
}

// In-register inverse DFT of length 2^LGR (<= 16), natural order in and
// out: bit-reversed copy, then radix-2 decimation in time.
template <int LGR>
__device__ __forceinline__ void dft_inv(float2 (&v)[1 << LGR]) {
  constexpr int R = 1 << LGR;
  float2 u[R];
#pragma unroll
  for (int r = 0; r < R; ++r) u[brev_c(r, LGR)] = v[r];
#pragma unroll
  for (int s = 1; s <= LGR; ++s) {
    const int half = 1 << (s - 1);
#pragma unroll
    for (int b = 0; b < R / 2; ++b) {
      const int pos = b & (half - 1);
      const int i = ((b >> (s - 1)) << s) + pos;
      const float2 x = u[i];
      const float2 y = mul_w16(u[i + half], pos << (4 - s));
      u[i] = cadd(x, y);
      u[i + half] = csub(x, y);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = u[r];
}

// v[r] times w^r for w = e^{2 pi i k 2^sh / 4096}: w^1, w^2, w^4, w^8 from the
// table, the other powers as products of at most four of them.
template <int LGR>
__device__ __forceinline__ void twiddle_powers(float2 (&v)[1 << LGR], const float2* __restrict__ tab,
                                               int k, int sh) {
  constexpr int R = 1 << LGR;
  float2 wp[R];
  wp[0] = make_float2(1.f, 0.f);
#pragma unroll
  for (int b = 0; b < LGR; ++b) wp[1 << b] = tab[(k << b) << sh];
#pragma unroll
  for (int r = 3; r < R; ++r)
    if (r & (r - 1)) wp[r] = cmul(wp[r & (r - 1)], wp[r & -r]);
#pragma unroll
  for (int r = 1; r < R; ++r) v[r] = cmul(v[r], wp[r]);
}

// Element i of transform t: pass 1 keeps transforms contiguous with one
// float2 of padding after every 16; pass 2 interleaves them.
struct AddrPadded {
  int lgL;
  __device__ int operator()(int t, int i) const {
    const int x = (t << lgL) + i;
    return x + (x >> 4);
  }
};
struct AddrInterleaved {
  int lgT;
  __device__ int operator()(int t, int i) const { return (i << lgT) + t; }
};

// One Stockham pass of radix 2^LGR over the 2^lgT transforms of length
// 2^lgL in buf, after passes whose radices multiply to 2^lgNs.  EMAX is
// the largest element count of any caller (groups per thread <= EMAX /
// (256 R)).  Transform t and group j of group g: t slowest for contiguous
// transforms (TFAST = false), fastest for interleaved ones.
template <int LGR, int EMAX, bool TFAST, class Addr>
__device__ __forceinline__ void stockham_pass(float2* buf, Addr addr, int lgL, int lgT,
                                              int lgNs, const float2* __restrict__ tab) {
  constexpr int R = 1 << LGR;
  constexpr int GM = (EMAX / 256 / R) > 0 ? EMAX / 256 / R : 1;
  const int lgJ = lgL - LGR;                     // log2 of the groups per transform
  const int nG = 1 << (lgT + lgJ);
  float2 v[GM][R];
#pragma unroll
  for (int gi = 0; gi < GM; ++gi) {
    const int g = threadIdx.x + gi * 256;
    if (g < nG) {
      const int t = TFAST ? (g & ((1 << lgT) - 1)) : (g >> lgJ);
      const int j = TFAST ? (g >> lgT) : (g & ((1 << lgJ) - 1));
#pragma unroll
      for (int r = 0; r < R; ++r) v[gi][r] = buf[addr(t, j + (r << lgJ))];
      if (lgNs > 0) {
        twiddle_powers<LGR>(v[gi], tab, j & ((1 << lgNs) - 1), 12 - lgNs - LGR);
      }
      dft_inv<LGR>(v[gi]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int gi = 0; gi < GM; ++gi) {
    const int g = threadIdx.x + gi * 256;
    if (g < nG) {
      const int t = TFAST ? (g & ((1 << lgT) - 1)) : (g >> lgJ);
      const int j = TFAST ? (g >> lgT) : (g & ((1 << lgJ) - 1));
      const int k = j & ((1 << lgNs) - 1);
      const int d = ((j >> lgNs) << (lgNs + LGR)) + k;
#pragma unroll
      for (int s = 0; s < R; ++s) buf[addr(t, d + (s << lgNs))] = v[gi][s];
    }
  }
  __syncthreads();
}

// In-place inverse DFTs (natural order in and out) of the 2^lgT
// transforms of length 2^lgL (<= 4096) in buf.
template <int EMAX, bool TFAST, class Addr>
__device__ __forceinline__ void fft_inv(float2* buf, Addr addr, int lgL, int lgT,
                                        const float2* __restrict__ tab) {
  int lgNs = 0;
  while (lgL - lgNs >= 4) {
    stockham_pass<4, EMAX, TFAST>(buf, addr, lgL, lgT, lgNs, tab);
    lgNs += 4;
  }
  switch (lgL - lgNs) {
    case 1: stockham_pass<1, EMAX, TFAST>(buf, addr, lgL, lgT, lgNs, tab); break;
    case 2: stockham_pass<2, EMAX, TFAST>(buf, addr, lgL, lgT, lgNs, tab); break;
    case 3: stockham_pass<3, EMAX, TFAST>(buf, addr, lgL, lgT, lgNs, tab); break;
    default: break;
  }
}

// Samples 2m and 2m + 1 of a series: one 8-byte access where the pair is
// 8-byte aligned (even row pitch, aligned output), so that a run of lanes
// covers whole cache lines in one store; else two 4-byte accesses.
__device__ __forceinline__ void store_out(const PinkArgs& a, int64_t series,
                                          int64_t m, float2 z) {
  const int64_t t = 2 * m;
  float* dst = a.tod + series * a.out_ld;
  const bool pairs = ((a.out_ld & 1) == 0) && ((reinterpret_cast<uintptr_t>(a.tod) & 7) == 0);
  if (pairs && t + 1 < a.t_total) {
    float2* d2 = reinterpret_cast<float2*>(dst + t);
    if (a.accumulate) {
      float2 o = *d2;
      o.x += z.x;
      o.y += z.y;
      *d2 = o;
    } else {
      *d2 = z;
    }
    return;
  }
  if (t < a.t_total) {
    if (a.accumulate) dst[t] += z.x; else dst[t] = z.x;
  }
  if (t + 1 < a.t_total) {
    if (a.accumulate) dst[t + 1] += z.y; else dst[t + 1] = z.y;
  }
}

}  // namespace

// Twiddle table: entry m holds e^{2 pi i m / 4096}.
__global__ void k_pink_tables(float2* tab) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m < kLdsC) tab[m] = twiddle((uint32_t)m, 12);
}

// Pass 1 works on a set of columns closed under k -> M - k: column 0,
// column M1/2, or the pair (k1, M1 - k1).  Each spectral bin X_j is drawn
// once; every Z_k is built from X_k and X_{M-k} held in LDS, two at a time
// (e^{2 pi i (M-k)/N} = -conj e^{2 pi i k/N}).
// Dynamic LDS: one or two padded transforms of M2 values; EMAX bounds the
// values per workgroup.  LGM2 > 0, for series of one column, fixes lg M2 at
// compile time, so that the transform's index arithmetic folds into constants;
// LGM2 = 0 takes it from the arguments.  For series of one pass (M <= 2048), and
// of columns longer than 2048 (the others: k_pink_pairs).
template <int EMAX, int LGM2>
__global__ __launch_bounds__(256) void k_pink_pass1(PinkArgs a) {
  extern __shared__ float2 buf[];
  const int lgM2 = LGM2 > 0 ? LGM2 : a.lgM2;
  const AddrPadded at{lgM2};
  const int grp = blockIdx.x;
  const int sl = blockIdx.y;
  const int64_t series = a.s0 + sl;
  const int p = (int)(series / a.K);
  const int k = (int)(series % a.K);
  const float sc = a.scale[k];
  const float halpha = -0.5f * a.alpha[k];
  const float fstep = (float)(a.fs / (double)a.N);
  const int M1 = a.M1, M2 = 1 << lgM2;
  const int lgN = a.lgM1 + lgM2 + 1;
  // columns of this group: kind 0 = {0}, 1 = {M1/2}, 2 = {k1, M1 - k1}
  int kind, col[2], ncol;
  if (grp == 0) { kind = 0; col[0] = 0; ncol = 1; }
  else if (grp == 1) { kind = 1; col[0] = M1 / 2; ncol = 1; }
  else { kind = 2; col[0] = grp - 1; col[1] = M1 - (grp - 1); ncol = 2; }
  col[1] = (ncol == 2) ? col[1] : col[0];

  // draw X for every bin of the group's columns (natural order)
  for (int idx = threadIdx.x; idx < (ncol << lgM2); idx += blockDim.x) {
    const int c = idx >> lgM2, k2 = idx & (M2 - 1);
    const int64_t j = col[c] + (int64_t)M1 * k2;
    float2 x = make_float2(0.f, 0.f);
    if (j > 0 && j < a.M) {
      const u32x4 o = philox10(u32x4{(uint32_t)j, (uint32_t)k, (uint32_t)(a.pix0 + p), 1u},
                               a.key0, a.key1);
      float zc, zs;
      box_muller(o.x, o.y, &zc, &zs);
      // power law from the hardware log2 and exp2 (about one ulp each)
      const float cj = sc * __builtin_amdgcn_exp2f(halpha * __builtin_amdgcn_logf((float)j * fstep));
      x = make_float2(cj * zc, cj * zs);
    }
    buf[at(c, k2)] = x;
  }
  __syncthreads();
  // Z in place, one pair (k, M - k) per work item
  const int U = kind == 0 ? M2 / 2 + 1 : (kind == 1 ? M2 / 2 : M2);
  // e^{2 pi i k / N} at k = col + M1 u, u = threadIdx.x + 256 i
  const GeoTwiddle wz((uint32_t)(col[0] + (int64_t)M1 * threadIdx.x),
                      (uint32_t)((int64_t)M1 * 256), lgN);
  for (int u = threadIdx.x, iu = 0; u < U; u += 256, ++iu) {
    int ca, ra, cb, rb;   // (column slot, row) of k and of M - k
    bool nyq = false;
    if (kind == 0) {
      ca = 0; ra = (u == M2 / 2 && M2 > 1) ? M2 / 2 : u;
      if (u == 0 || M2 == 1) { nyq = true; cb = 0; rb = 0; }
      else { cb = 0; rb = M2 - ra; }
    } else if (kind == 1) {
      ca = 0; ra = u; cb = 0; rb = M2 - 1 - u;
    } else {
      ca = 0; ra = u; cb = 1; rb = M2 - 1 - u;
    }
    const float2 xa = buf[at(ca, ra)];
    const float2 xb = nyq ? make_float2(0.f, 0.f) : buf[at(cb, rb)];
    const float2 w = wz(iu);
    // Z_k = (X_k + conj X_{M-k}) + i w (X_k - conj X_{M-k})
    const float2 ev = make_float2(xa.x + xb.x, xa.y - xb.y);
    const float2 od = make_float2(xa.x - xb.x, xa.y + xb.y);
    const float2 wo = cmul(w, od);
    const float2 za = make_float2(ev.x - wo.y, ev.y + wo.x);
    if (nyq || (ca == cb && ra == rb)) {
      buf[at(ca, ra)] = za;
    } else {
      // Z_{M-k} with twiddle -conj(w): E' = conj(E), O' = -conj(O)
      const float2 wb = make_float2(-w.x, w.y);
      const float2 evb = make_float2(ev.x, -ev.y);
      const float2 odb = make_float2(-od.x, od.y);
      const float2 wob = cmul(wb, odb);
      buf[at(ca, ra)] = za;
      buf[at(cb, rb)] = make_float2(evb.x - wob.y, evb.y + wob.x);
    }
  }
  __syncthreads();
  if constexpr (LGM2 > 0) fft_inv<EMAX, false>(buf, at, LGM2, 0, a.tab);
  else fft_inv<EMAX, false>(buf, at, lgM2, ncol - 1, a.tab);
  const int lgM = a.lgM1 + lgM2;
  for (int c = 0; c < ncol; ++c) {
    const int k1 = col[c];
    if (M1 == 1) {
      for (int m2 = threadIdx.x; m2 < M2; m2 += blockDim.x)
        store_out(a, series, m2, buf[at(c, m2)]);
    } else {
      float2* dst = a.scratch + ((int64_t)sl * M1 + k1) * M2;
      // e^{2 pi i k1 m2 / M} at m2 = threadIdx.x + 256 i
      const GeoTwiddle ws((uint32_t)((uint64_t)k1 * threadIdx.x),
                          (uint32_t)((uint64_t)k1 * 256), lgM);
      for (int m2 = threadIdx.x, im = 0; m2 < M2; m2 += 256, ++im)
        dst[m2] = cmul(buf[at(c, m2)], ws(im));
    }
  }
}

// Pass 1 at lg M2 = 11 and M1 >= 2: a workgroup takes the columns k1 and M1 -
// k1, or 0 and M1 / 2.  A thread draws X_k and X_{M-k} of its 8 pairs and writes their Z to LDS; two passes of radix 16 in
// LDS (thread (t, j) = one group of transform t), then one of radix 8 whose
// outputs, tid + 256 s of both transforms, are stored from registers.  Every
// LDS address is one of three per-thread bases plus a constant, and every
// twiddle but each sequence's first is a constant or uniform:
//   e^{2 pi i k / N}, k = k1 + M1 (tid + 256 i):       first times e^{2 pi i i / 16}
//   e^{2 pi i k1 m2 / M}, m2 = tid + 256 s:            first times e^{2 pi i k1 s / (8 M1)}
// Bound by the vector ALU (39 of its instructions per bin are Philox).  2429
// series of 2^20 samples: 3.81 ms; 6.03 with run-time strides, five sincospi per
// sequence and the bins taken through LDS.
__global__ __launch_bounds__(256) void k_pink_pairs(PinkArgs a) {
  constexpr int kM2 = 1 << kPinkLgM2, kCol = kM2 + (kM2 >> 4), kStep = 256 + 16;
  __shared__ float2 buf[2 * kCol];
  const int tid = threadIdx.x, lane = tid & 63, sl = blockIdx.y;
  const int64_t series = a.s0 + sl;
  const int p = (int)(series / a.K);
  const int k = (int)(series % a.K);
  const float sc = a.scale[k];
  const float halpha = -0.5f * a.alpha[k];
  const float fstep = (float)(a.fs / (double)a.N);
  const int M1 = a.M1, lgM = a.lgM1 + kPinkLgM2;
  const uint32_t M = (uint32_t)a.M, step = (uint32_t)M1 * 256u;
  const int col[2] = {(int)blockIdx.x, blockIdx.x ? M1 - (int)blockIdx.x : M1 / 2};
  auto draw = [&](uint32_t j) {
    const u32x4 o = philox10(u32x4{j, (uint32_t)k, (uint32_t)(a.pix0 + p), 1u}, a.key0, a.key1);
    float zc, zs;
    box_muller(o.x, o.y, &zc, &zs);
    // power law from the hardware log2 and exp2 (about one ulp each)
    const float cj = sc * __builtin_amdgcn_exp2f(halpha * __builtin_amdgcn_logf((float)j * fstep));
    return make_float2(cj * zc, cj * zs);
  };
  // Z_k = (X_k + conj X_{M-k}) + i w (X_k - conj X_{M-k}); Z_{M-k} is
  // conj E - i conj(w O)
  auto pair = [&](uint32_t j, float2 w, float2* zk, float2* zm) {
    const float2 xa = draw(j), xb = draw(M - j);
    const float2 ev = make_float2(xa.x + xb.x, xa.y - xb.y);
    const float2 wo = cmul(w, make_float2(xa.x - xb.x, xa.y + xb.y));
    *zk = make_float2(ev.x - wo.y, ev.y + wo.x);
    *zm = make_float2(ev.x + wo.y, wo.x - ev.y);
  };
  float2* const up = buf + tid + (tid >> 4);
  float2* const down = buf + (255 - tid) + ((255 - tid) >> 4);
  if (blockIdx.x) {
    const uint32_t j0 = (uint32_t)col[0] + (uint32_t)M1 * tid;
    const float2 w0 = twiddle(j0, lgM + 1);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      pair(j0 + step * i, mul_w16(w0, i), up + kStep * i, down + kCol + kStep * (7 - i));
  } else {
    // columns 0 (rows u and 2048 - u) and M1 / 2 (u and 2047 - u), each its
    // own mirror; Z_0 = 0, Z_{M/2} = 2 conj X_{M/2}
    float2* const down0 = buf + (256 - tid) + ((256 - tid) >> 4);
    const uint32_t j0 = (uint32_t)M1 * tid, j1 = j0 + (uint32_t)col[1];
    const float2 w0 = twiddle(j0, lgM + 1), w1 = twiddle(j1, lgM + 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      pair(j1 + step * i, mul_w16(w1, i), up + kCol + kStep * i, down + kCol + kStep * (7 - i));
      if (i || tid) {
        pair(j0 + step * i, mul_w16(w0, i), up + kStep * i, down0 + kStep * (7 - i));
      } else {
        const float2 x = draw(M / 2);
        buf[0] = make_float2(0.f, 0.f);
        buf[4 * kStep] = make_float2(2.f * x.x, -2.f * x.y);
      }
    }
  }
  __syncthreads();
  {
    const int t = tid >> 7, j = tid & 127;
    float2* const in = buf + t * kCol + j + (j >> 4);
    float2 v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = in[(128 + 8) * r];
    dft_inv<4>(v);
    __syncthreads();
    float2* const out = buf + t * kCol + 17 * j;
#pragma unroll
    for (int s = 0; s < 16; ++s) out[s] = v[s];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = in[(128 + 8) * r];
    twiddle_powers<4>(v, a.tab, j & 15, 4);
    dft_inv<4>(v);
    __syncthreads();
    float2* const out2 = buf + t * kCol + (j >> 4) * kStep + (j & 15);
#pragma unroll
    for (int s = 0; s < 16; ++s) out2[17 * s] = v[s];
  }
  __syncthreads();
  // lanes 0 - 15: the uniform factors of the two columns
  const float2 f = twiddle((uint32_t)((lane & 8 ? col[1] : col[0]) * (lane & 7)) &
                               (uint32_t)(8 * M1 - 1),
                           a.lgM1 + 3);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const float2* const in = buf + c * kCol + tid + (tid >> 4);
    float2 v[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = in[kStep * r];
    twiddle_powers<3>(v, a.tab, tid, 1);
    dft_inv<3>(v);
    const float2 w0 = twiddle((uint32_t)((uint64_t)col[c] * tid) & (uint32_t)(a.M - 1), lgM);
    float2* const dst = a.scratch + (((int64_t)sl * M1 + col[c]) << kPinkLgM2) + tid;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      float2 w = w0;
      if (s) {
        const float2 u = make_float2(
            __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, f.x), 8 * c + s)),
            __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, f.y), 8 * c + s)));
        w = cmul(w, u);
      }
      dst[256 * s] = cmul(v[s], w);
    }
  }
}

// Pass 2 for columns of 2048 (lg M2 = 11) and LGM1 <= 8: bound by memory, so
// each thread has its 16 (or M1, if fewer) elements in flight at once, straight
// into the registers of the first radix, and the last radix stores from
// registers; what lies between goes through LDS once, or not at all up to M1 =
// 16.  Columns fastest across lanes, so that every access runs over at least
// 128 B.  2429 series of 2^20 samples (576000 kept): 3.22 ms, 4.66 with both
// sides staged in LDS; 13680 series of 2^14: 0.35 ms, 1.01.
template <int LGM1>
__global__ __launch_bounds__(256) void k_pink_columns(PinkArgs a) {
  constexpr int LG1 = LGM1 < 4 ? LGM1 : 4, LG2 = LGM1 - LG1, R1 = 1 << LG1;
  constexpr int kLgB = 8 - LG2, B = 1 << kLgB;     // columns per workgroup
  const int tid = threadIdx.x, t = tid & (B - 1), j = tid >> kLgB;
  const int64_t m20 = (int64_t)blockIdx.x * B;
  const int64_t series = a.s0 + blockIdx.y;
  const float2* const src = a.scratch + ((int64_t)blockIdx.y << (LGM1 + kPinkLgM2)) + m20 + t +
                            ((int64_t)j << kPinkLgM2);
  float* const dst = a.tod + series * a.out_ld;
  const bool pairs = ((a.out_ld & 1) == 0) && ((reinterpret_cast<uintptr_t>(a.tod) & 7) == 0);
  // element e of v is output m1(e) of column m20 + col(e)
  auto store = [&](const auto& v, auto m1, auto col, int n) {
    if (!pairs) {
#pragma unroll
      for (int e = 0; e < n; ++e)
        store_out(a, series, ((int64_t)m1(e) << kPinkLgM2) + m20 + col(e), v[e]);
      return;
    }
    float2 old[R1];
    if (a.accumulate) {
#pragma unroll
      for (int e = 0; e < n; ++e) {
        const int64_t x = 2 * (((int64_t)m1(e) << kPinkLgM2) + m20 + col(e));
        old[e] = x + 1 < a.t_total ? *reinterpret_cast<const float2*>(dst + x) : make_float2(0.f, 0.f);
      }
    }
#pragma unroll
    for (int e = 0; e < n; ++e) {
      const int64_t x = 2 * (((int64_t)m1(e) << kPinkLgM2) + m20 + col(e));
      if (x + 1 < a.t_total) {
        float2 z = v[e];
        if (a.accumulate) z = cadd(old[e], z);
        *reinterpret_cast<float2*>(dst + x) = z;
      } else if (x < a.t_total) {      // the last sample of an odd length
        if (a.accumulate) dst[x] += v[e].x;
        else dst[x] = v[e].x;
      }
    }
  };
  float2 v[R1];
#pragma unroll
  for (int r = 0; r < R1; ++r) {
    // read once, past the caches: us past / through them for 45, 347 and 2429
    // series of 8 columns 6.7 / 6.7, 14.8 / 14.9, 88 / 111; 32 columns 12 / 12, 54
    // / 54, 377 / 394; 256 columns 56 / 58, 521 / 529, 3507 / 3682.  Not at 16
    // columns, 21 / 7.8, 35 / 26, 199 / 215: what costs the small launches 13 us
    // at this length alone is not known
    const float2* const p = src + ((int64_t)r << (LG2 + kPinkLgM2));
    if constexpr (LGM1 == 4)
      v[r] = *p;
    else
      v[r] = __builtin_bit_cast(float2,
                                __builtin_nontemporal_load(reinterpret_cast<const double*>(p)));
  }
  dft_inv<LG1>(v);
  if constexpr (LG2 == 0) {
    store(v, [](int e) { return e; }, [&](int) { return t; }, R1);
  } else {
    __shared__ float2 buf[1 << 12];
#pragma unroll
    for (int s = 0; s < R1; ++s) buf[(((j << 4) + s) << kLgB) + t] = v[s];
    __syncthreads();
    constexpr int R2 = 1 << LG2, G = 16 / R2;      // transforms of length R2 per thread
    float2 o[16];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int q = tid + 256 * g, c = q & (B - 1), k = q >> kLgB;
      float2 u[R2];
#pragma unroll
      for (int r = 0; r < R2; ++r) u[r] = buf[((k + 16 * r) << kLgB) + c];
      twiddle_powers<LG2>(u, a.tab, k, 8 - LG2);
      dft_inv<LG2>(u);
#pragma unroll
      for (int s = 0; s < R2; ++s) o[g * R2 + s] = u[s];
    }
    store(o, [&](int e) { return ((tid + 256 * (e / R2)) >> kLgB) + 16 * (e % R2); },
          [&](int e) { return (tid + 256 * (e / R2)) & (B - 1); }, 16);
  }
}

// Pass 2 for other lengths: 2^(lgM1 + lgB2) elements per workgroup, held in
// dynamic LDS of exactly that size.
__global__ __launch_bounds__(256) void k_pink_pass2(PinkArgs a) {
  extern __shared__ float2 buf[];
  const int nb = blockIdx.x;
  const int sl = blockIdx.y;
  const int64_t series = a.s0 + sl;
  const int M2 = 1 << a.lgM2, lgB2 = a.lgB2, B2 = 1 << lgB2;
  const int m20 = nb << lgB2;
  const float2* src = a.scratch + ((int64_t)sl << (a.lgM1 + a.lgM2));
  const int n = 1 << (a.lgM1 + lgB2);
  // element k1 of transform bb at k1 B2 + bb: both sides consecutive
  for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
    const int k1 = idx >> lgB2, bb = idx & (B2 - 1);
    buf[idx] = src[(int64_t)k1 * M2 + m20 + bb];
  }
  __syncthreads();
  fft_inv<kLdsC, true>(buf, AddrInterleaved{lgB2}, a.lgM1, lgB2, a.tab);
  for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
    const int m1 = idx >> lgB2, bb = idx & (B2 - 1);
    store_out(a, series, (int64_t)m1 * M2 + m20 + bb, buf[idx]);
  }
}

void launch_pink_tables(float2* tab, hipStream_t s) {
  static_assert(kPinkTable == kLdsC, "table");
  hipLaunchKernelGGL(k_pink_tables, dim3(kPinkTable / 256), dim3(256), 0, s, tab);
}

void launch_pink_pass1(const PinkArgs& a, hipStream_t s) {
  if (a.lgM2 == kPinkLgM2 && a.M1 >= 2) {
    hipLaunchKernelGGL(k_pink_pairs, dim3(a.M1 / 2, a.n_series), dim3(256), 0, s, a);
    return;
  }
  const int groups = a.M1 == 1 ? 1 : a.M1 / 2 + 1;
  const int e = (a.M1 == 1 ? 1 : 2) << a.lgM2;   // values per workgroup
  const size_t lds = (size_t)(e + (e >> 4)) * sizeof(float2);
  const dim3 grid(groups, a.n_series);
  if (a.M1 == 1 && a.lgM2 == kPinkLgM2)
    hipLaunchKernelGGL((k_pink_pass1<kLdsC, kPinkLgM2>), grid, dim3(256), lds, s, a);
  else if (e <= kLdsC)
    hipLaunchKernelGGL((k_pink_pass1<kLdsC, 0>), grid, dim3(256), lds, s, a);
  else
    hipLaunchKernelGGL((k_pink_pass1<2 * kLdsC, 0>), grid, dim3(256), lds, s, a);
}

void launch_pink_pass2(const PinkArgs& a, hipStream_t s) {
  if (a.lgM2 == kPinkLgM2 && a.lgM1 <= 8) {
    const int lg_cols = a.lgM1 <= 4 ? 8 : 12 - a.lgM1;
    const dim3 grid(a.M2 >> lg_cols, a.n_series);
#define GTOD_COLUMNS(L) \
  case L: hipLaunchKernelGGL(k_pink_columns<L>, grid, dim3(256), 0, s, a); return
    switch (a.lgM1) {
      GTOD_COLUMNS(1);
      GTOD_COLUMNS(2);
      GTOD_COLUMNS(3);
      GTOD_COLUMNS(4);
      GTOD_COLUMNS(5);
      GTOD_COLUMNS(6);
      GTOD_COLUMNS(7);
      GTOD_COLUMNS(8);
    }
#undef GTOD_COLUMNS
  }
  const size_t lds = sizeof(float2) << (a.lgM1 + a.lgB2);
  hipLaunchKernelGGL(k_pink_pass2, dim3(a.M2 >> a.lgB2, a.n_series), dim3(256), lds, s, a);
}

__global__ void k_philox(const uint32_t* ctr, uint32_t* out, int64_t n,
                         uint32_t k0, uint32_t k1) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const u32x4 o = philox10(u32x4{ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2],
                                 ctr[4 * i + 3]}, k0, k1);
  out[4 * i] = o.x;
  out[4 * i + 1] = o.y;
  out[4 * i + 2] = o.z;
  out[4 * i + 3] = o.w;
}

void launch_philox(const uint32_t* ctr, uint32_t* out, int64_t n, uint32_t k0,
                   uint32_t k1, hipStream_t s) {
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(k_philox, dim3((unsigned)blocks), dim3(256), 0, s, ctr, out,
                     n, k0, k1);
}

}  // namespace gtod
