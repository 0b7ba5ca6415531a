// Filterbank contraction on the 16-bit matrix cores with split operands and
// FP32 accumulation (v_mfma_f32_32x32x16_{f16,bf16}), with the photon-noise
// epilogue (sections 2.5-2.7).
//
// Per row (one sample of one pixel) and channel, over the frequency axis,
//   C0 = x B0,   C1 = x B1' + x^2 B2,   P_KID = c0 + C0,  NEP^2 = c1 + C1,
// x the deviation dP from the reference spectrum.
//
// FP32 jobs (F16 = true): every FP32 operand is carried as two FP16 halves,
// h = f16(v) and l = f16(v - h) (round to nearest even): 22 bits, and three
// products (l h, h l, h h) for each of x B0, x B1' and x^2 B2.  The panel
// holds x scaled per bin so that the reference power of every bin lies in
// [2, 4) (down to 2^-123 W/Hz; a fainter bin's is scaled by 2^124), and each
// response channel is scaled to a maximum in [2^13, 2^14), all by powers of two
// that cancel or are undone in the epilogue.  The halves of x are off by at
// most max(2^-25, 2^-23 |x|): near the reference (|x| < 1/2) that is 2^-26 of
// the bin's power, below the FP32 rounding of the panel itself, far from it up
// to twice the FP32 rounding of x.  Rows beyond
// the FP16 range (|x| > 255, i.e. a deviation of 64 to 128 times the
// reference power, and infinities or NaN) make their accumulators non-finite,
// and so does a response that is not finite itself; the wave then recomputes
// its tile with FP32 MFMAs on FP32 operands (x with its bin's scale taken out
// again, and the unscaled responses) and stores the rows of 32 channels with
// such an accumulator from there.  32 channels are a tile in every shape, so
// the choice depends on the row and the setup alone.
// Why: the FP32 matrix rate is 1/16 of the 16-bit one and nine 16-bit
// products replace three FP32 ones.
//
// Split jobs (F16 = false): two BF16 halves (16 bits), three products for x
// B0 and x B1' and one for x^2 B2.
//
// Workgroup: 4 waves, WR along rows x WC along channels, one per SIMD; a
// wave owns NJ row tiles x NI channel tiles of 32 x 32, two accumulators
// each.  The large shape has 256 rows x 128 channels, WR = 4, NI = 4, NJ =
// 2: 256 accumulator registers of the 512 a lone wave has, every panel row
// read and split by one wave only (with WC = 2, NJ = 4 by two: 50.5 against
// 47.4 ms in six minutes of the IFU), and 72 (BF16: 56) MFMAs per step.
//
// What bounds it: the power of the matrix cores, and what still stands
// between two MFMAs.  Registers-only MFMAs on random operands run at 1.6
// (FP16) and 1.75 PFLOP/s on this card, where zeros reach 2.46; the large
// shape executes 1.2 (FP16).  Per workgroup and 3008 bins 0.57 M cycles go
// to the steps (0.41 M of MFMAs) and 0.096 M to the epilogue.
//
// Operand staging: steps of 16 bins (one MFMA depth) go from global memory
// into an LDS ring of STAGES stages with global_load_lds_dwordx4, STAGES -
// 1 steps ahead.  A stage is the panel [MT][16] FP32 in 64-byte rows
// (16-byte slot of bin quad q in row r at q ^ swz(r)) and, per group of 64
// channels, the response planes [64][16] of 16-bit values in 32-byte rows
// (16-byte half h of row r at h ^ swb(r)); both put the 16-byte reads of
// each group of 16 lanes on distinct banks of the 256-byte-wide LDS.  The
// responses are stored in that layout by the setup (k_tile_responses), so
// their DMAs move 1 KB of consecutive bytes.
//
// Schedule: a step is a list of slots of one MFMA each, in program order.
// Between the MFMAs of step s the wave issues the DMAs of step s + STAGES -
// 1, the LDS reads of the responses two planes ahead and of the panel of
// step s + 1, and the split of that panel, so that neither LDS latency nor
// the split stands between two MFMAs.  One barrier per step: before it each
// wave has waited for its DMAs of step s + 1; after it stages s and s + 1
// are visible and no wave reads stage s - 1 any more.
//
// Every accumulator is summed over the steps in order, with the products of
// a step in a fixed order, in every shape below: the bits of a row do not
// depend on the launch it is in.
//
// Tile index -> workgroup mapping: block b runs on XCD b mod 8, so the
// channel groups of one row tile are given blocks of the same XCD and can
// share the panel tile in its L2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "gtod_internal.h"
#include "gemm_epilogue.h"
#include "philox.h"

namespace gtod {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int KC = 16;       // bins per stage = one MFMA step
constexpr int kGroup = 64;   // channels per tiled response group
constexpr int kPlaneBytes = kGroup * KC * 2;

// panel rows (64 bytes, four 16-byte slots)
__device__ __forceinline__ int swz(int row) { return ((row >> 1) ^ (row >> 2)) & 3; }
// response rows (32 bytes, two 16-byte halves): rows r and r + 8 lie 256
// bytes apart, on the same banks, so their halves are swapped
__device__ __forceinline__ int swb(int row) { return (row >> 3) & 1; }

__device__ __forceinline__ uint32_t lds_addr(void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)p;
}

// One wave-wide direct-to-LDS load: lane i moves the 16 bytes at base +
// voff (base wave-uniform, in scalar registers; voff the lane's byte
// offset) to LDS byte address m0 + 16 i (m0 uniform).  Advancing base is
// scalar arithmetic.  M0 is a reserved register the compiler does not
// save around inline assembly; no other code in this kernel uses it.  The
// s_nop covers the M0 write -> LDS DMA hazard.
__device__ __forceinline__ void dma16(const void* base, uint32_t voff, uint32_t m0) {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(m0), "v"(voff), "s"(base) : "memory", "m0");
#pragma clang diagnostic pop
}

// s_waitcnt with vmcnt = N (< 64) and the other counters left free.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
  __builtin_amdgcn_s_waitcnt(0x3f70 | (N & 15) | ((N >> 4) << 14));
}

template <bool F16>
struct Half {
  typedef f16x8 v8;
  static constexpr int kPlanes = 6;   // B0l B0h B1l B1h B2l B2h
  static constexpr int kOps = 4;      // xh xl qh ql, q = x^2
  __device__ static f32x16 mfma(v8 b, v8 x, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(b, x, c, 0, 0, 0);
  }
};
template <>
struct Half<false> {
  typedef bf16x8 v8;
  static constexpr int kPlanes = 5;   // B0l B0h B1l B1h B2h
  static constexpr int kOps = 3;      // xh xl qh
  __device__ static f32x16 mfma(v8 b, v8 x, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, x, c, 0, 0, 0);
  }
};

// Products of plane p, in order: how many, the accumulator and the operand
// of product m (small terms first).  Planes 0, 2, 4 are low halves, except
// that BF16 has only the high half of B2 in plane 4.
template <bool F16>
constexpr int n_products(int p) { return (p & 1) ? 2 : 1; }
constexpr int acc_of(int p) { return p < 2 ? 0 : 1; }
constexpr int op_of(int p, int m) {
  const int base = p < 4 ? 0 : 2;            // x or q
  return (p & 1) ? base + 1 - m : base;      // high plane: l then h; low plane: h
}
template <bool F16>
constexpr int first_slot(int p) {
  int t = 0;
  for (int r = 0; r < p; ++r) t += n_products<F16>(r);
  return t;
}

// f16(a b - h) for the two halves of h, each rounded once, as one
// v_fma_mix{lo,hi}_f16 per half (the compiler makes three instructions of
// it).  No MFMA reads the result within two wait states of it.
__device__ __forceinline__ f16x2 rest(f32x2 a, f32x2 b, f16x2 h) {
  uint32_t r;
  const uint32_t hu = __builtin_bit_cast(uint32_t, h);
  asm("v_fma_mixlo_f16 %0, %1, %2, -%3 op_sel_hi:[0,0,1]"
      : "=v"(r) : "v"(a[0]), "v"(b[0]), "v"(hu));
  asm("v_fma_mixhi_f16 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]"
      : "+v"(r) : "v"(a[1]), "v"(b[1]), "v"(hu));
  return __builtin_bit_cast(f16x2, r);
}

// Splits bins e, e + 1 of x into the operands o (see Half::kOps); one is
// 1.0 in a register.
__device__ __forceinline__ void split_pair(f32x2 x, int e, float one, f16x8 (&o)[4]) {
  const f16x2 h = __builtin_convertvector(x, f16x2);
  const f16x2 q = __builtin_convertvector(x * x, f16x2);
  const f16x2 hl = rest(x, f32x2{one, one}, h), ql = rest(x, x, q);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    o[0][e + k] = h[k];
    o[1][e + k] = hl[k];
    o[2][e + k] = q[k];
    o[3][e + k] = ql[k];
  }
}
__device__ __forceinline__ void split_pair(f32x2 x, int e, float, bf16x8 (&o)[3]) {
  const bf16x2 hi = __builtin_convertvector(x, bf16x2);
  const uint32_t hb = __builtin_bit_cast(uint32_t, hi);
  const f32x2 hf = {__builtin_bit_cast(float, hb << 16),
                    __builtin_bit_cast(float, hb & 0xffff0000u)};
  const bf16x2 lo = __builtin_convertvector(x - hf, bf16x2);
  const bf16x2 sq = __builtin_convertvector(x * x, bf16x2);
  o[0][e] = hi[0];
  o[0][e + 1] = hi[1];
  o[1][e] = lo[0];
  o[1][e + 1] = lo[1];
  o[2][e] = sq[0];
  o[2][e + 1] = sq[1];
}

}  // namespace

// ---------------------------------------------------------------------------
// Response planes (setup)
// ---------------------------------------------------------------------------

size_t tiled_response_bytes(int Kp, int Fp, bool f16) {
  const size_t groups = (size_t)(Kp + kGroup - 1) / kGroup;
  return groups * (size_t)(Fp / KC) * (f16 ? 6 : 5) * kPlaneBytes;
}

// Power-of-two scale of channel k's FP16 responses: the largest |B0| 2^-d and
// the largest of |B1'| 2^-d, |B2| 2^(-2 d - p) come to [2^13, 2^14).  unit0, unit1 are
// what one accumulator unit is worth; a channel without response, or with
// a non-finite one, is left unscaled.
__global__ __launch_bounds__(256) void k_response_units(const float* __restrict__ B,
                                                        const int* __restrict__ d, int Kp,
                                                        int Fp, int pexp, int* e0, int* e1,
                                                        double* unit0, double* unit1) {
  __shared__ double m0[256], m1[256];
  const int k = blockIdx.x;
  const int64_t KF = (int64_t)Kp * Fp;
  const float* b = B + (int64_t)k * Fp;
  double x0 = 0.0, x1 = 0.0;
  for (int j = threadIdx.x; j < Fp; j += 256) {
    x0 = fmax(x0, ldexp(fabs((double)b[j]), -d[j]));
    x1 = fmax(x1, fmax(ldexp(fabs((double)b[KF + j]), -d[j]),
                       ldexp(fabs((double)b[2 * KF + j]), -2 * d[j] - pexp)));
  }
  m0[threadIdx.x] = x0;
  m1[threadIdx.x] = x1;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      m0[threadIdx.x] = fmax(m0[threadIdx.x], m0[threadIdx.x + st]);
      m1[threadIdx.x] = fmax(m1[threadIdx.x], m1[threadIdx.x + st]);
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  auto exponent = [](double m) { return (m > 0.0 && isfinite(m)) ? 13 - ilogb(m) : 0; };
  e0[k] = exponent(m0[0]);
  e1[k] = exponent(m1[0]);
  unit0[k] = ldexp(1.0, -pexp - e0[k]);
  unit1[k] = ldexp(1.0, -pexp - e1[k]);
}

// Tiled split responses: for channel group g (64 channels) and step s (16
// bins), plane m as [64][16] 16-bit rows with the in-row swizzle applied,
// i.e. the LDS image of the stage, contiguous:
// T[g][s][m][r][slot] = B_m[64 g + r][16 s + 8 (slot ^ swb(r)) .. + 7],
// zero for channels past the padded matrix.  The B2 planes are taken times
// 2^-p, so that x^2 B2 adds straight into C1; the FP16 halves' scales (the
// channel's, the bin's) go into the same exponent, so that none of them
// underflows by itself.
template <bool F16>
__global__ void k_tile_responses(const float* __restrict__ B, const int* __restrict__ d,
                                 const int* __restrict__ e0, const int* __restrict__ e1, 
                                 uint16_t* __restrict__ T, int Kp, int Fp, int pexp, int64_t n_slots) {
  constexpr int NPL = Half<F16>::kPlanes;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_slots) return;
  const int slot = (int)(i & 1);
  const int r = (int)((i >> 1) % kGroup);
  const int64_t q = (i >> 1) / kGroup;
  const int m = (int)(q % NPL);
  const int64_t gs = q / NPL;
  const int n_steps = Fp / KC;
  const int s = (int)(gs % n_steps);
  const int ch = (int)(gs / n_steps) * kGroup + r;
  const int mat = m >> 1;
  const bool low = !(m & 1) && (F16 || m < 4);
  uint16_t v[8] = {};
  if (ch < Kp) {
    const int j = s * KC + 8 * (slot ^ swb(r));
    const float* src = B + ((int64_t)mat * Kp + ch) * Fp + j;
    const int e = (F16 ? (mat == 0 ? e0[ch] : e1[ch]) : 0) - (mat == 2 ? pexp : 0);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float x = ldexpf(src[k], F16 ? e - (mat == 2 ? 2 : 1) * d[j + k] : e);
      if constexpr (F16) {
        const _Float16 h = (_Float16)x;
        const _Float16 o = low ? (_Float16)(x - (float)h) : h;
        v[k] = __builtin_bit_cast(uint16_t, o);
      } else {
        const __bf16 h = (__bf16)x;
        const __bf16 o = low ? (__bf16)(x - (float)h) : h;
        v[k] = __builtin_bit_cast(uint16_t, o);
      }
    }
  }
  uint4 w;
  w.x = v[0] | ((uint32_t)v[1] << 16);
  w.y = v[2] | ((uint32_t)v[3] << 16);
  w.z = v[4] | ((uint32_t)v[5] << 16);
  w.w = v[6] | ((uint32_t)v[7] << 16);
  reinterpret_cast<uint4*>(T)[i] = w;
}

void launch_tile_responses(const float* B, const int* d, int* e0, int* e1, double* unit0,
                           double* unit1, uint16_t* Tb, uint16_t* Th, int Kp, int Fp, int pexp,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_response_units, dim3(Kp), dim3(256), 0, s, B, d, Kp, Fp, pexp, e0,
                     e1, unit0, unit1);
  const int64_t nb = (int64_t)(tiled_response_bytes(Kp, Fp, false) / 16);
  const int64_t nh = (int64_t)(tiled_response_bytes(Kp, Fp, true) / 16);
  hipLaunchKernelGGL(k_tile_responses<false>, dim3((unsigned)((nb + 255) / 256)), dim3(256),
                     0, s, B, d, e0, e1, Tb, Kp, Fp, pexp, nb);
  hipLaunchKernelGGL(k_tile_responses<true>, dim3((unsigned)((nh + 255) / 256)), dim3(256),
                     0, s, B, d, e0, e1, Th, Kp, Fp, pexp, nh);
}

// ---------------------------------------------------------------------------
// Contraction
// ---------------------------------------------------------------------------

// SPL = 2: two waves per 32 x 32 tile, one for each accumulator (C0; C1 with
// C2).  Where a launch leaves most CUs idle its time is a wave's chain of LDS
// reads, splits and MFMAs per step: 160 rows x 347 channels x 3000 bins take 50
// us in 64 x 32 tiles so (57 with one wave per tile, 62 in 64 x 64 tiles; 32 x
// 32 tiles and 16 stages are no faster).  The sums are the same.
template <bool F16, int WR, int WC, int NI, int NJ, int STAGES, int SPL = 1>
__global__ __launch_bounds__(64 * WR * WC * SPL, 1) void k_contract(GemmArgs a) {
  typedef Half<F16> H;
  typedef typename H::v8 v8;
  constexpr int NPL = H::kPlanes, ND = H::kOps;
  constexpr int MT = WR * 32 * NJ, NT = WC * 32 * NI, NG = NT < kGroup ? 1 : NT / kGroup;
  constexpr int kPanelBytes = MT * KC * 4;
  constexpr int kGroupBytes = NPL * kPlaneBytes;
  // a tile of 32 channels takes half of each plane of its group
  constexpr int kPlane = NT < kGroup ? kPlaneBytes / 2 : kPlaneBytes;
  constexpr int kStageBytes = kPanelBytes + NG * NPL * kPlane;
  constexpr int kDma = kStageBytes / 1024;         // 1 KB DMAs of a stage
  constexpr int kTiles = WR * WC, NW = kTiles * SPL;
  constexpr int kPanelQ = MT / 16 / 4;             // panel DMAs per wave (SPL = 1)
  constexpr int Q = (kDma + NW - 1) / NW;          // DMAs per wave (some one less)
  static_assert(SPL > 1 || (kTiles == 4 && NT % kGroup == 0 && (MT / 16) % 4 == 0), "shape");
  static_assert((STAGES & (STAGES - 1)) == 0 && STAGES >= 4, "stage index by mask");
    // the ring, then the epilogue's slices
  constexpr int kLds = STAGES * kStageBytes > kTiles * epi_wave_bytes(NI)
                           ? STAGES * kStageBytes : kTiles * epi_wave_bytes(NI);
  static_assert(kLds <= 160 * 1024, "LDS");

  const int b = blockIdx.x;
  const int xcd = b & 7;
  const int l = b >> 3;
  // Tile order: the workgroups of a partial last channel group take less
  // time per step than the others, so they come last, after all full groups
  // of all row tiles.  Workgroups that run together then advance along the
  // frequency axis together and share what they read in the L2.
  const int n_same = a.K % NT ? max(1, a.n_cg - 1) : a.n_cg;
  const int n_tt8 = gridDim.x / (8 * a.n_cg);
  int tt, cg;
  if (l < n_tt8 * n_same) {
    tt = (l / n_same) * 8 + xcd;
    cg = l % n_same;
  } else {
    tt = (l - n_tt8 * n_same) * 8 + xcd;
    cg = n_same;
  }
  // rows of the chunk's panel; a last tile reads rows past them from
  // clamped addresses and stores none of them
  const int64_t n_rows = (int64_t)a.n_pix * a.Tpad;
  const int64_t row0 = (int64_t)tt * MT;
  if (row0 >= n_rows) return;
  // a tile of padding rows only has nothing to store
  const int tl0 = (int)(row0 % a.Tpad);
  if (tl0 >= a.Tc && tl0 + MT <= a.Tpad) return;
  const int ch0 = cg * NT;

  __shared__ __attribute__((aligned(16))) char ring[kLds];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int h = lane >> 5, c = lane & 31;
  const int part = wave / kTiles;        // accumulator of this wave (SPL = 2)
  const int rw = wave % WR, cw = wave % kTiles / WR;

  const int64_t Fp = a.Fp;
  const int n_steps = a.Fp / KC;

  // DMA sources are a wave-uniform base plus a 32-bit lane offset (the
  // spectral setup keeps 256 panel rows below 4 GiB).  Wave w moves the
  // 1 KB blocks w + 4 q of a stage; a panel block is 16 rows, lane taking
  // bin quad (lane % 4) ^ swz(row) of row lane / 4.
  const char* const gp = reinterpret_cast<const char*>(a.panel + row0 * Fp);
  const int n_g = (a.Kp + kGroup - 1) / kGroup;
  auto panel_offset = [&](int block) {
    const int r = block * 16 + (lane >> 2);
    const int64_t gr = min(row0 + r, n_rows - 1);
    return (uint32_t)(4 * ((gr - row0) * Fp + 4 * ((lane & 3) ^ swz(r))));
  };
  auto response = [&](int block) {
    if constexpr (NT < kGroup)
      return reinterpret_cast<const char*>(F16 ? a.Th : a.Tb) +
             (size_t)(ch0 / kGroup) * n_steps * kGroupBytes + min(block, NPL - 1) * kPlaneBytes +
             ch0 % kGroup * (KC * 2);
    const int e = min(block, NG * NPL * 2 - 1);
    const int gr = min(ch0 / kGroup + e / (NPL * 2), n_g - 1);   // past the last: unused data
    return reinterpret_cast<const char*>(F16 ? a.Th : a.Tb) +
           (size_t)gr * n_steps * kGroupBytes + (e % (NPL * 2)) * 1024;
  };
  // lane offset, source and advance per step of the wave's DMAs: the panel's
  // first kPanelQ of each wave, or with SPL = 2 the first of the first waves
  uint32_t vo[Q];
  const char* src[Q];
  uint32_t advance[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int block = wave + NW * q;
    const bool panel = SPL == 1 ? q < kPanelQ : block < MT / 16;
    vo[q] = panel ? panel_offset(block) : (uint32_t)lane * 16u;
    src[q] = panel ? gp : response(block - MT / 16);
    advance[q] = panel ? KC * 4 : kGroupBytes;
  }
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(ring));
  const bool all_q = kDma % NW == 0 || wave < kDma % NW;   // this wave issues Q DMAs
  // DMA q of step st
  auto issue = [&](int st, int q) {
    const uint32_t dst = lds0 + (uint32_t)((st & (STAGES - 1)) * kStageBytes + (wave + NW * q) * 1024);
    if (q + 1 < Q || all_q) dma16(src[q] + (size_t)st * advance[q], vo[q], dst);
  };
  // wait until at most the wave's DMAs of STAGE_N stages are in flight
  auto wait_stages = [&](auto stage_n) {
    constexpr int n = decltype(stage_n)::value;
    if (all_q) wait_vm<n * Q>(); else wait_vm<n * (Q - 1)>();
  };

  // live 32-channel tiles of this wave
  const int ch_w = ch0 + cw * 32 * NI;
  const int n_live = max(0, min(NI, (a.K - ch_w + 31) / 32));

  f32x16 acc[2][NI][NJ];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[m][i][j][e] = 0.f;

  float one;
  asm("s_mov_b32 %0, 1.0" : "=s"(one));

  // LDS byte offsets inside a stage
  const int oP = (rw * 32 * NJ + c) * (KC * 4) + 16 * ((2 * h) ^ swz(c));
  const int rb = (cw * 32 * NI) % kGroup + c;
  const int oB = kPanelBytes + (cw * 32 * NI) / kGroup * kGroupBytes + rb * (KC * 2) +
                 16 * (h ^ swb(rb));

  for (int s = 0; s < STAGES - 1 && s < n_steps; ++s)
#pragma unroll
    for (int q = 0; q < Q; ++q) issue(s, q);
  if (n_steps >= STAGES - 1) wait_stages(std::integral_constant<int, STAGES - 2>{});
  else wait_vm<0>();
  __builtin_amdgcn_s_barrier();

  auto run = [&](auto nl_c, auto part_c) {
    constexpr int NL = decltype(nl_c)::value;
    // planes of this wave
    constexpr int P0 = SPL == 1 ? 0 : (decltype(part_c)::value ? 2 : 0);
    constexpr int P1 = SPL == 1 ? NPL : (decltype(part_c)::value ? NPL : 2);
    constexpr int kSlots = first_slot<F16>(P1) - first_slot<F16>(P0);
    if constexpr (NL == 0) {
      // no live channel: this wave only moves its part of the operands
      for (int s = 0; s < n_steps; ++s) {
        if (s + STAGES - 2 < n_steps) wait_stages(std::integral_constant<int, STAGES - 3>{});
        else wait_vm<0>();
        __builtin_amdgcn_s_barrier();
        if (s + STAGES - 1 < n_steps) {
#pragma unroll
          for (int q = 0; q < Q; ++q) issue(s + STAGES - 1, q);
        }
      }
    } else {
      constexpr int NM = kSlots * NL * NJ;             // slots of a step
      constexpr int kConv0 = NM / 5 > 3 ? NM / 5 : 3;  // first split slot
      constexpr int kConvS = (NM - kConv0) / (4 * NJ) > 0 ? (NM - kConv0) / (4 * NJ) : 1;
      typedef v8 Ops[NJ][ND];
      v8 pf[2][NL];           // the first two response planes of the coming step
      float4 raw[NJ][2];
      auto read_x = [&](const char* st, int r) {
        raw[r >> 1][r & 1] = *reinterpret_cast<const float4*>(
            st + (oP ^ (16 * (r & 1))) + (r >> 1) * 32 * KC * 4);
      };
      auto read_b = [&](const char* st, int p, int i) {
        return *reinterpret_cast<const v8*>(st + oB + (i >> 1) * kGroupBytes + p * kPlane +
                                            (i & 1) * 32 * KC * 2);
      };
      // pair k of the 4 NJ pairs: row tile k / 4, bins 2 (k % 4), + 1
      auto split = [&](int k, Ops& o) {
        const int j = k >> 2, e = 2 * (k & 3);
        const f32x2 x = {raw[j][e >> 2][e & 3], raw[j][e >> 2][(e & 3) + 1]};
        split_pair(x, e, one, o[j]);
      };
      auto step = [&](int s, Ops& cur, Ops& nxt, auto main_c) {
        constexpr bool kMain = decltype(main_c)::value;   // step s + STAGES - 1 exists
        if (kMain || s + STAGES - 2 < n_steps)
          wait_stages(std::integral_constant<int, STAGES - 3>{});
        else wait_vm<0>();
        __builtin_amdgcn_s_barrier();
        const char* st = ring + (s & (STAGES - 1)) * kStageBytes;
        // the last step reads a stage that holds older data, and drops it
        const char* sn = ring + ((s + 1) & (STAGES - 1)) * kStageBytes;
        if (!kMain && s + STAGES - 1 < n_steps) {
#pragma unroll
          for (int q = 0; q < Q; ++q) issue(s + STAGES - 1, q);
        }
        v8 bp[NPL + 2][NL];
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int i = 0; i < NL; ++i) bp[P0 + p][i] = pf[p][i];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = P0; p < P1; ++p)
#pragma unroll
          for (int m = 0; m < n_products<F16>(p); ++m)
#pragma unroll
            for (int i = 0; i < NL; ++i)
#pragma unroll
              for (int j = 0; j < NJ; ++j) {
                const int u = (m * NL + i) * NJ + j;
                const int t = (first_slot<F16>(p) - first_slot<F16>(P0)) * NL * NJ + u;
                f32x16& d = acc[acc_of(p)][i][j];
                d = H::mfma(bp[p][i], cur[j][op_of(p, m)], d);
                // responses two planes ahead
                if (u < NL) {
                  if (p + 2 < P1) bp[p + 2][u] = read_b(st, p + 2, u);
                  else bp[p + 2][u] = read_b(sn, p + 2 - P1 + P0, u);
                }
                if (t < 2 * NJ) read_x(sn, t);
                if (kMain && t < Q) issue(s + STAGES - 1, t);
                if (t >= kConv0 && (t - kConv0) % kConvS == 0 && (t - kConv0) / kConvS < 4 * NJ)
                  split((t - kConv0) / kConvS, nxt);
                __builtin_amdgcn_sched_barrier(0);
              }
        // pairs that found no slot
#pragma unroll
        for (int k = (NM - 1 - kConv0) / kConvS + 1; k < 4 * NJ; ++k) split(k, nxt);
#pragma unroll
        for (int q = NM; q < Q; ++q)
          if (kMain) issue(s + STAGES - 1, q);
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int i = 0; i < NL; ++i) pf[p][i] = bp[P1 + p][i];
      };
      Ops xa, xb;
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int i = 0; i < NL; ++i) pf[p][i] = read_b(ring, P0 + p, i);
#pragma unroll
      for (int r = 0; r < 2 * NJ; ++r) read_x(ring, r);
#pragma unroll
      for (int k = 0; k < 4 * NJ; ++k) split(k, xa);
      // the frequency axis is padded to an even number of steps
      const int n_main = max(0, n_steps - (STAGES - 1)) & ~1;
      int s = 0;
      for (; s < n_main; s += 2) {
        step(s, xa, xb, std::true_type{});
        step(s + 1, xb, xa, std::true_type{});
      }
      for (; s < n_steps; s += 2) {
        step(s, xa, xb, std::false_type{});
        step(s + 1, xb, xa, std::false_type{});
      }
    }
  };
  auto run_part = [&](auto part_c) {
    if (NI >= 4 && n_live == 4) run(std::integral_constant<int, NI >= 4 ? 4 : 1>{}, part_c);
    else if (NI >= 4 && n_live == 3) run(std::integral_constant<int, NI >= 4 ? 3 : 1>{}, part_c);
    else if (NI >= 2 && n_live == 2) run(std::integral_constant<int, NI >= 2 ? 2 : 1>{}, part_c);
    else if (WC == 1 || n_live >= 1) run(std::integral_constant<int, 1>{}, part_c);
    else run(std::integral_constant<int, 0>{}, part_c);
  };
  if (SPL == 1 || part == 0) run_part(std::integral_constant<int, 0>{});
  else run_part(std::integral_constant<int, SPL - 1>{});
  __syncthreads();   // every wave is done with the ring before the epilogue reuses it
  if constexpr (SPL > 1) {
    // C1 to the wave that has C0, past the epilogue's slices
    static_assert(NI * NJ == 1 && kTiles * (epi_wave_bytes(NI) + 4096) <= kLds, "exchange");
    float* const x = reinterpret_cast<float*>(ring + kLds - kTiles * 4096) +
                     wave % kTiles * 1024 + lane;
    if (part) {
#pragma unroll
      for (int e = 0; e < 16; ++e) x[e * 64] = acc[1][0][0][e];
    }
    __syncthreads();
    if (part) return;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[1][0][0][e] = x[e * 64];
  }
  if (n_live == 0) return;
  char* const spk = ring + wave * epi_wave_bytes(NI);
  const int64_t row_w = row0 + rw * 32 * NJ;
  bool store[NI][NJ];
  if constexpr (!F16) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) store[i][j] = true;
    contraction_epilogue<NI, NJ>(a, acc, spk, row_w, ch_w, n_live, store,
                                 EpiUnits{nullptr, nullptr, a.pinv});
  } else {
    // rows of a channel tile with a non-finite accumulator (0 x finite = 0,
    // else NaN); both lane halves of a row take part
    bool again = false;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float z = 0.f;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int e = 0; e < 16; ++e) z = __builtin_fmaf(acc[m][i][j][e], 0.f, z);
        const int bad = !(z == 0.f);
        store[i][j] = !(bad | __shfl_xor(bad, 32));
        again |= !store[i][j];
      }
    contraction_epilogue<NI, NJ>(a, acc, spk, row_w, ch_w, n_live, store,
                                 EpiUnits{a.unit0, a.unit1, 0.0});
    if (!__any(again)) return;
    // FP32 matrix products for the rows left out above
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[m][i][j][e] = 0.f;
    const int64_t KF = (int64_t)a.Kp * Fp;
    const float* xr[NJ];
    const float* br[NI];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      xr[j] = a.panel + min(row_w + j * 32 + c, n_rows - 1) * Fp + 4 * h;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      br[i] = a.B + (int64_t)min(ch_w + i * 32 + c, a.Kp - 1) * Fp + 4 * h;
    for (int k0 = 0; k0 < a.Fp; k0 += 8) {
      float4 x[NJ], v[NI][3];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        x[j] = *reinterpret_cast<const float4*>(xr[j] + k0);
        const float4 u = *reinterpret_cast<const float4*>(a.unscale + 4 * h + k0);
        for (int e = 0; e < 4; ++e) x[j][e] *= u[e];
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int m = 0; m < 3; ++m)
          v[i][m] = *reinterpret_cast<const float4*>(br[i] + m * KF + k0);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const float q = x[j][e] * x[j][e] * a.pinv_f;
#pragma unroll
          for (int i = 0; i < NI; ++i) {
            acc[0][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[i][0][e], x[j][e], acc[0][i][j], 0, 0, 0);
            acc[1][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[i][1][e], x[j][e], acc[1][i][j], 0, 0, 0);
            acc[1][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[i][2][e], q, acc[1][i][j], 0, 0, 0);
          }
        }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) store[i][j] = !store[i][j];
    contraction_epilogue<NI, NJ>(a, acc, spk, row_w, ch_w, n_live, store,
                                 EpiUnits{nullptr, nullptr, a.pinv});
  }
}

namespace {

template <bool F16, int WR, int WC, int NI, int NJ, int STAGES, int SPL = 1>
void launch_shape(GemmArgs a, hipStream_t s) {
  constexpr int MT = WR * 32 * NJ, NT = WC * 32 * NI;
  const int64_t n_tt = ((int64_t)a.n_pix * a.Tpad + MT - 1) / MT;
  a.n_cg = (a.K + NT - 1) / NT;
  hipLaunchKernelGGL((k_contract<F16, WR, WC, NI, NJ, STAGES, SPL>),
                     dim3((unsigned)(round_up(n_tt, 8) * a.n_cg)), dim3(64 * WR * WC * SPL), 0, s, a);
}

// One workgroup of a shape runs on a CU at a time, so a launch takes about
// the rounds of 256 workgroups times the time of one, which these weights
// give: microseconds at 3000 bins, measured with one round on an idle card
// (FP16 halves; BF16).  A CU holds two of the 128 x 64 one, but they take
// nearly twice as long as one (256 of them 143 us, 512 253), so it counts by
// rounds of 256 too.  In launches of many rounds the time goes with the tiles
// rather than the rounds; the rule charges whole rounds there as well, which by
// these weights may cost up to 10 % (96000 rows x 347 channels).  There 256 x
// 128 is the fastest per output: 43.2 ms of contractions in six minutes of the
// 49-pixel, 347-channel IFU, against 47.4 with 256 x 64 and 48.2 with 128 x 64;
// a launch of 160 rows takes 62 us with 64 x 64 tiles
// against 261 with 256 x 128, and 50 with 64 x 32; but 198 workgroups of 64 x 32
// take 78 where 108 of 64 x 64 take 65 (operands from beyond the L2), so they
// count by rounds of 128.  Up to 64 channels half of a 256 x 128 tile
// would be dead.
struct Shape {
  int rows, channels, round;
  float f16_us, bf16_us;
};
constexpr int kNShapes = 5;
constexpr Shape kShapes[kNShapes] = {{256, 128, 256, 270.f, 210.f}, {256, 64, 256, 150.f, 127.f},
                                     {128, 64, 256, 92.f, 85.f},    {64, 64, 256, 58.f, 58.f},
                                     {64, 32, 128, 46.f, 41.f}};

int best_shape(bool f16, int64_t rows, int K) {
  int best = -1;
  float least = 0.f;
  for (int q = K <= 64 ? 1 : 0; q < kNShapes; ++q) {
    const Shape& h = kShapes[q];
    const int64_t wgs = (rows + h.rows - 1) / h.rows * ((K + h.channels - 1) / h.channels);
    const float us = (float)((wgs + h.round - 1) / h.round) * (f16 ? h.f16_us : h.bf16_us);
    if (best < 0 || us < least) {
      best = q;
      least = us;
    }
  }
  return best;
}

template <bool F16>
void launch_contract(const GemmArgs& a, hipStream_t s) {
  switch (best_shape(F16, (int64_t)a.n_pix * a.Tpad, a.K)) {
    case 0: launch_shape<F16, 4, 1, 4, 2, 4>(a, s); break;
    case 1: launch_shape<F16, 4, 1, 2, 2, 4>(a, s); break;
    case 2: launch_shape<F16, 2, 2, 1, 2, 4>(a, s); break;
    case 3: launch_shape<F16, 2, 2, 1, 1, 8>(a, s); break;
    default: launch_shape<F16, 2, 1, 1, 1, 8, 2>(a, s); break;
  }
}

}  // namespace

void contraction_tile(bool f16, int64_t rows, int K, int32_t tile[2]) {
  const Shape& h = kShapes[best_shape(f16, rows, K)];
  tile[0] = h.rows;
  tile[1] = h.channels;
}

void launch_gemm_f32(const GemmArgs& a, hipStream_t s) { launch_contract<true>(a, s); }
void launch_gemm_bf16(const GemmArgs& a, hipStream_t s) { launch_contract<false>(a, s); }

}  // namespace gtod
