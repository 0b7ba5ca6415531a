// Epilogue of the contraction kernels: reference terms, photon-noise sigma,
// Philox white noise and the store into [pixel][channel][time].
//
// Each wave owns NI x NJ accumulator tiles of 32 channels x 32 samples of
// C0 (P_KID) and C1 (NEP^2, with the dP^2 B2 term already in it); tile
// (i, j) starts at channel ch_base + 32 i and row row_base + 32 j.  The
// accumulators of channel k are in units of unit0[k] (W) and unit1[k]
// (W^2/Hz), powers of two.  Per row tile, the wave's accumulators go to its
// own LDS slice (epi_wave_bytes at lds, distinct for each wave) with static
// register indices and are read back by a compact loop in which lane l
// handles sample (l mod 32) of channel rows 2s + l/32: stores are runs of
// 32 consecutive samples.  The slice belongs to one wave, whose LDS
// accesses complete in order, so the waves of a workgroup go through the
// epilogue without barriers (the kernel has one before it, after the last
// read of its operand ring).
//
// The kernel runs one wave per SIMD and nothing overlaps its epilogue, so
// its latencies count in full.  The channel constants are read from global
// memory once per wave, into the slice.  The TOD values that a job adds to
// come by direct-to-LDS loads, one unit of work (a row tile and up to two
// channel tiles) ahead: as ordinary loads they put a wait for every earlier
// store before each store.  The loop takes four samples at a time, part by
// part, so that their instructions interleave.  The draw is Philox4x32-10
// under counter (t, k, p, 0) with the products that depend on t alone taken
// once per row and those that depend on k and p alone once per channel: 14
// of its 20 wide multiplications remain per sample.
#pragma once

#include <hip/hip_runtime.h>

#include "gtod_internal.h"
#include "philox.h"

namespace gtod {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Channel constants, in LDS.
struct EpiChannel {
  double c0, u0, c1, u1;   // reference terms and accumulator units
  double kel_a, kel_ib;    // Kelvin scale
  uint2 m;                 // M0 x1 of the white-noise draw (lo, hi)
};

constexpr int kEpiPitch = 33;
constexpr int kEpiTileBytes = 2 * 32 * kEpiPitch * 4;   // C0 and C1 of a tile
constexpr int kEpiPrevBytes = 32 * 32 * 4;              // TOD values of a tile
// LDS of one wave: the constants of its channels, the tiles of one unit and
// the TOD values of two
constexpr int epi_unit(int ni) { return ni > 1 ? 2 : 1; }
constexpr int epi_wave_bytes(int ni) {
  return ni * 32 * (int)sizeof(EpiChannel) +
         epi_unit(ni) * (kEpiTileBytes + 2 * kEpiPrevBytes);
}

// One wave-wide direct-to-LDS load of 4 bytes per lane: lane i moves the
// word at p to LDS byte address m0 + 4 i (see dma16 of the contraction).
__device__ __forceinline__ void dma4(const float* p, uint32_t m0) {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
               :: "s"(m0), "v"(p) : "memory", "m0");
#pragma clang diagnostic pop
}

// Units of the accumulators: per channel (arrays), or one value for all.
struct EpiUnits {
  const double* unit0;
  const double* unit1;
  double same;
};

// store[i][j]: whether this lane's row of tile (i, j) is written.
template <int NI, int NJ>
__device__ __forceinline__ void contraction_epilogue(
    const GemmArgs& a, f32x16 (&acc)[2][NI][NJ], char* lds,
    int64_t row_base, int ch_base, int n_live, const bool (&store)[NI][NJ],
    const EpiUnits& units) {
  constexpr int NU = epi_unit(NI), kUnits = NI / NU;   // channel tiles per unit, units per row tile
  const int lane = threadIdx.x & 63;
  const int h = lane >> 5, c = lane & 31;
  EpiChannel* const kc = reinterpret_cast<EpiChannel*>(lds);
  char* const tile = lds + NI * 32 * (int)sizeof(EpiChannel);
  char* const prev = tile + NU * kEpiTileBytes;
  const uint32_t prev_m0 = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)prev);
  const int n_ch = min(32 * n_live, a.K - ch_base);   // channels stored
  for (int k = lane; k < n_ch; k += 64) {
    const int ch = ch_base + k;
    EpiChannel e;
    e.c0 = a.c0[ch];
    e.c1 = a.c1[ch];
    e.u0 = units.unit0 ? units.unit0[ch] : units.same;
    e.u1 = units.unit1 ? units.unit1[ch] : units.same;
    e.kel_a = a.kelvin ? a.kel_a[ch] : 0.0;
    e.kel_ib = a.kelvin ? a.kel_ib[ch] : 1.0;
    e.m = make_uint2(0u, 0u);
    kc[k] = e;
  }
  // row tile j: its pixel and this lane's sample (clamped into the job's)
  auto pixel = [&](int j) { return (int)((row_base + j * 32) / a.Tpad); };
  auto sample = [&](int j) { return (int)((row_base + j * 32) % a.Tpad) + c; };
  auto offset = [&](int j, int tl) {
    return ((int64_t)(a.p0 + pixel(j)) * a.K + ch_base) * a.out_ld +
           (a.t0 + tl - a.out_t0);
  };
  // channels of unit u: [32 NU (u mod kUnits), + n_unit(u)), this lane's k
  // of pair q is 2 q + h
  auto n_unit = [&](int u) { return min(32 * NU, n_ch - 32 * NU * (u % kUnits)); };
  auto fetch_prev = [&](int u) {
    const int j = u / kUnits, n = n_unit(u);
    if (!a.accumulate || n <= 0 || pixel(j) >= a.n_pix) return;
    const int64_t o = offset(j, min(sample(j), a.Tc - 1)) + 32 * NU * (u % kUnits) * a.out_ld;
    const uint32_t m0 = prev_m0 + (u & 1) * (NU * kEpiPrevBytes);
    for (int q = 0; 2 * q < n; ++q)
      dma4(a.tod + o + min(2 * q + h, n - 1) * a.out_ld, m0 + q * 256);
  };
  fetch_prev(0);
#pragma unroll
  for (int u = 0; u < NJ * kUnits; ++u) {
    const int j = u / kUnits, i0 = NU * (u % kUnits), n = n_unit(u);
    // this unit's TOD values have landed
    __builtin_amdgcn_s_waitcnt(0x3f70);
    if (u + 1 < NJ * kUnits) fetch_prev(u + 1);
    if (n <= 0) continue;
    const int pl = pixel(j), tl = sample(j);
    const bool store0 = store[i0][j], store1 = store[i0 + NU - 1][j];
    const bool valid = (store0 || store1) && pl < a.n_pix && tl < a.Tc;
    const uint32_t t = (uint32_t)(a.t0 + tl), p = (uint32_t)(a.pix0 + a.p0 + pl);
    const PhiloxRow pr(t, p, a.key0, a.key1);
    __builtin_amdgcn_wave_barrier();
    if (a.photon && i0 == 0)
      for (int k = lane; k < n_ch; k += 64)
        kc[k].m = philox_channel((uint32_t)(ch_base + k), p, a.key0);
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      float* const sn = reinterpret_cast<float*>(tile + i * kEpiTileBytes);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int chl = 8 * (e >> 2) + 4 * h + (e & 3);
        sn[chl * kEpiPitch + c] = acc[0][i0 + i][j][e];
        sn[(32 + chl) * kEpiPitch + c] = acc[1][i0 + i][j][e];
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (!valid) continue;
    // Channel k of the unit is 2 q + h: the lane's part (h) of every address
    // is taken here, the pair's (q) is wave-uniform.  kU pairs at a time,
    // each part for all of them before the next; the last ones may run past
    // the unit's channels, onto other words of the slice, and store nothing.
    constexpr int kU = 4;
    const int64_t off_u = offset(j, tl) + (32 * i0 + h) * a.out_ld;
    const EpiChannel* const kh = kc + 32 * i0 + h;
    const float* const th = reinterpret_cast<const float*>(tile) + h * kEpiPitch + c;
    const float* const pv = reinterpret_cast<const float*>(
        prev + (u & 1) * (NU * kEpiPrevBytes)) + lane;
    for (int q0 = 0; 2 * q0 < n; q0 += kU) {
      if (!(q0 < 16 ? store0 : store1)) continue;
      const EpiChannel* const e = kh + 2 * q0;
      const float* const sn = th + (q0 >> 4) * (kEpiTileBytes / 4) + (q0 & 15) * 2 * kEpiPitch;
      double pkd[kU];
      float pk[kU], sg[kU], v[kU];
#pragma unroll
      for (int q = 0; q < kU; ++q) {
        // P_KID and NEP^2 in FP64: NEP^2 lies below the FP32 normal range
        pkd[q] = e[2 * q].c0 + (double)sn[2 * q * kEpiPitch] * e[2 * q].u0;
        pk[q] = (float)pkd[q];
        const double n2 = e[2 * q].c1 + (double)sn[(32 + 2 * q) * kEpiPitch] * e[2 * q].u1;
        // sigma to FP32 rounding (its tolerance is 1e-5); its square times
        // 2^40, as that of a faint channel is below the normal range
        sg[q] = 0x1p-20f * sqrtf((float)(fmax(n2, 0.0) * ((double)a.fs_half * 0x1p40)));
        v[q] = 0.f;
      }
      if (a.photon) {
        uint2 o[kU];
#pragma unroll
        for (int q = 0; q < kU; ++q) o[q] = pr.draw(e[2 * q].m);
#pragma unroll
        for (int q = 0; q < kU; ++q) v[q] = sg[q] * box_muller_cos(o[q].x, o[q].y);
      }
      if (a.kelvin) {
        // (P - a_k) / b_k with the offset taken in FP64
#pragma unroll
        for (int q = 0; q < kU; ++q)
          v[q] = (float)(((pkd[q] - e[2 * q].kel_a) + (double)v[q]) * e[2 * q].kel_ib);
      } else {
#pragma unroll
        for (int q = 0; q < kU; ++q) v[q] = pk[q] + v[q];
      }
#pragma unroll
      for (int q = 0; q < kU; ++q)
        if (a.accumulate) v[q] = pv[(q0 + q) * 64] + v[q];
      auto put = [&](float* out, const float (&x)[kU]) {
        float* o = out + off_u + 2 * q0 * a.out_ld;
        if (2 * (q0 + kU) <= n) {
#pragma unroll
          for (int q = 0; q < kU; ++q) o[2 * q * a.out_ld] = x[q];
        } else {
#pragma unroll
          for (int q = 0; q < kU; ++q)
            if (2 * (q0 + q) + h < n) o[2 * q * a.out_ld] = x[q];
        }
      };
      put(a.tod, v);
      if (a.p_kid) put(a.p_kid, pk);
      if (a.sigma) put(a.sigma, sg);
    }
  }
}

}  // namespace gtod
