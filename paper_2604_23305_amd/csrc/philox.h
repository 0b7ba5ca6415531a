// Device-side Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) and the
// uniform / Box-Muller maps the noise kernels use.
//
// One round maps (x0, x1, x2, x3) under key (k0, k1) to
//   (hi(M1*x2) ^ x1 ^ k0, lo(M1*x2), hi(M0*x0) ^ x3 ^ k1, lo(M0*x0))
// and the key advances by the Weyl constants between rounds.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gtod {

struct u32x4 {
  uint32_t x, y, z, w;
};

// a ^ b ^ c in one instruction (the truth table of a three-input xor)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ u32x4 philox10(u32x4 c, uint32_t k0, uint32_t k1) {
  constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u;
  constexpr uint32_t kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;
  // each 64-bit product gives both halves in one v_mad_u64_u32 (separate
  // high and low 32-bit multiplies would take two instructions)
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)kM0 * c.x;
    const uint64_t p1 = (uint64_t)kM1 * c.z;
    c = u32x4{xor3((uint32_t)(p1 >> 32), c.y, k0), (uint32_t)p1,
              xor3((uint32_t)(p0 >> 32), c.w, k1), (uint32_t)p0};
    k0 += kW0;
    k1 += kW1;
  }
  return c;
}

// The first two words of philox10 under counter (t, k, p, 0) for many k at
// one t and p.  Writing x, y, z, w for the state after a round: round 1
// multiplies t and p; x then depends on p and k alone, z on t alone, so
// round 2's products M0 x and M1 z, and round 3's M0 x (x from M1 z and the
// low half of M1 p), do not mix t and k.  philox_channel gives round 2's M0
// x for a channel, PhiloxRow holds what depends on t and p.
__device__ __forceinline__ uint2 philox_channel(uint32_t k, uint32_t p, uint32_t key0) {
  const uint32_t x1 = (uint32_t)(((uint64_t)0xCD9E8D57u * p) >> 32) ^ k ^ key0;
  const uint64_t m = (uint64_t)0xD2511F53u * x1;
  return make_uint2((uint32_t)m, (uint32_t)(m >> 32));
}

struct PhiloxRow {
  uint32_t w1, y2, px, pxh, key0, key1;
  __device__ __forceinline__ PhiloxRow(uint32_t t, uint32_t p, uint32_t k0, uint32_t k1)
      : key0(k0), key1(k1) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * t, p1 = (uint64_t)0xCD9E8D57u * p;
    const uint32_t z1 = (uint32_t)(p0 >> 32) ^ k1;
    w1 = (uint32_t)p0;
    const uint64_t q1 = (uint64_t)0xCD9E8D57u * z1;             // round 2, M1 z
    y2 = (uint32_t)q1;
    const uint32_t x2 = (uint32_t)(q1 >> 32) ^ (uint32_t)p1 ^ (k0 + 0x9E3779B9u);
    const uint64_t r0 = (uint64_t)0xD2511F53u * x2;             // round 3, M0 x
    px = (uint32_t)r0;
    pxh = (uint32_t)(r0 >> 32);
  }
  // m = philox_channel of the channel
  __device__ __forceinline__ uint2 draw(uint2 m) const {
    constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u;
    constexpr uint32_t kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;
    const uint32_t z2 = xor3(m.y, w1, key1 + kW1);
    // round 3
    const uint64_t q = (uint64_t)kM1 * z2;
    u32x4 c{xor3((uint32_t)(q >> 32), y2, key0 + 2 * kW0), (uint32_t)q,
            xor3(pxh, m.x, key1 + 2 * kW1), px};
#pragma unroll
    for (uint32_t r = 3; r < 10; ++r) {
      const uint64_t p0 = (uint64_t)kM0 * c.x;
      const uint64_t p1 = (uint64_t)kM1 * c.z;
      c = u32x4{xor3((uint32_t)(p1 >> 32), c.y, key0 + r * kW0), (uint32_t)p1,
                xor3((uint32_t)(p0 >> 32), c.w, key1 + r * kW1), (uint32_t)p0};
    }
    return make_uint2(c.x, c.y);
  }
};

// ((o >> 9) + 1/2) * 2^-23: exact in FP32, strictly inside (0, 1).
__device__ __forceinline__ float u01(uint32_t o) {
  return (float)(o >> 9) * 1.1920928955078125e-07f + 5.9604644775390625e-08f;
}

// Box-Muller from the hardware transcendentals (about one ulp each): log2
// of u0 (normal, inside (0, 1)), the square root of -2 ln u0 (inside
// (0, 34]) and the cosine and sine of u1 revolutions, i.e. of the angle
// 2 pi u1.  The noise tolerances (the photon-noise term is about 4e-4 of
// the power; the 1/f series is held to 1e-5 of its rms) are orders of
// magnitude above these errors.
__device__ __forceinline__ float bm_radius(uint32_t o0) {
  // -2 ln u = -2 ln(2) log2(u)
  return __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u01(o0)));
}

// (r cos 2 pi u1, r sin 2 pi u1)
__device__ __forceinline__ void box_muller(uint32_t o0, uint32_t o1,
                                           float* zc, float* zs) {
  const float r = bm_radius(o0);
  const float u1 = u01(o1);
  *zc = r * __builtin_amdgcn_cosf(u1);
  *zs = r * __builtin_amdgcn_sinf(u1);
}

// r cos 2 pi u1 only (the white noise)
__device__ __forceinline__ float box_muller_cos(uint32_t o0, uint32_t o1) {
  return bm_radius(o0) * __builtin_amdgcn_cosf(u01(o1));
}

}  // namespace gtod
