// Base conversion of more than 8 source limbs (ModUp and ModDown with few digits), from and to coefficient form, on the matrix
// cores: bytes of the sources times bytes of the constants as in convert.hip.h, four targets to a product of 32 rows.
//
// A workgroup takes 512 positions, one a lane, with all their sources in registers (two each), and walks over the targets in
// groups of four, whose matrices (1 KB per 4 sources) it copies into LDS one group ahead. v_mfma_i32_32x32x32_i8 gives lane half h the
// eight sums of targets h and 2 + h at the 32 positions of one half-wave; two products, one per half of the positions, and a
// swap of half-waves give every lane all four targets at its own position.
//
// What bounds it: memory (sources read once, targets written once), 4.1 TB/s at 12 sources and 3.3 at 25, where the matrix products
// are 0.4 of the time by their count and the sources leave registers for two workgroups. From 25 sources on some scalar registers of
// the prologue spill (the rows' addresses). On the vector units a term took 4 multiply-adds. N = 2^16, both conversions of a key
// switch: 8 rotations of 24 + 12 limbs in 2 digits 216 -> 147 us, 15 of 23 + 25 limbs in one digit 901 -> 344, 2 of 30 + 30 limbs
// 86 (107 with matrices that waited for a private array in LDS, see below); 12 products of 18 + 9 limbs at 2^15 127 -> 89.
#pragma once
#include "convert.hip.h"

#define WIDE_THREADS 512

struct WideArgs {
  const u64* src;            // canonical residues, coefficient form
  u64* dst;
  u64 src_poly_stride, dst_poly_stride;   // elements between the source rows of consecutive b, between destination polynomials b * beta + j
  // [beta][(ntarget + 3) / 4][groups of 4 sources g][64][16] bytes: lane (h, n) = (l / 32, l % 32), n = 8 b + 4 c + r, has, for
  // sources 4g + 2h and 4g + 2h + 1, byte 4 (b % 2) + r of every C_ki of target 2 (b / 2) + c of the four
  const uint4* pieces;
  const ConvReduction* red;  // [nm]: sh = e - 48 and mu = -2^(64 + sh) / m for 2^50 <= m < 2^e, read on those targets
  const ModInfo* mods;
  const ulonglong2* inv;     // != null: [beta][alpha] Shoup pairs the sources are multiplied by first
  u32 logN, src_slot0, src_id0, src_nlimbs, alpha, beta, skip_own, ntarget;   // as in ConvArgs
  u32 main, special;         // target t: modulus t below main, t - main + special from there on
};
// The sums of one target put together: V = lo + mid 2^32 + top 2^48 (mod m).
__device__ __forceinline__ void wide_join(u32& lo, u32& mid, u32& top, int s0, int s1, int s2, int s3, int s4, int s5, int s6, int s7) {
  const int a0 = s0 + (s1 << 8), a1 = s2 + (s3 << 8), a2 = s4 + (s5 << 8), a3 = s6 + (s7 << 8);
  const long long l = conv_mad(a1, conv_opaque(65536), a0);
  lo = (u32)l;
  mid = (u32)a2 + (u32)(l >> 32);
  top = (u32)a3;
}
// V mod m, canonical. At most 48 sources: |V| <= 48 * 8 * 128 m / 2 < 2^14.6 m, so that hi = V / 2^32 fits 31 bits after a shift by sh
// and the quotient is off by 1.3 at most (see conv_settle).
__device__ __forceinline__ u64 wide_settle(u32 lo, u32 mid, u32 top, const ConvTarget& tg) {
  if ((tg.m >> 50) == 0) {
    const double h = __builtin_fma((double)(int)top, 65536.0, (double)(int)mid), l = (double)lo;
    const double c = __builtin_rint(__builtin_fma(l, tg.qinv, h * (tg.qinv * 4294967296.0)));
    return d2u_canon(__builtin_fma(__builtin_fma(-c, tg.qd * (1.0 / 4294967296.0), h), 4294967296.0, l), tg.qd);
  }
  const u64 v = conv_settle(lo, conv_mad((int)top, conv_opaque(65536), (int)mid), tg);
  return csub(csub(v, tg.m), tg.m);
}

// grid = (N / 512, digits, polynomials b)
template <int G>
__global__ void __launch_bounds__(WIDE_THREADS) conv_wide_kernel(WideArgs a) {
  __shared__ __attribute__((aligned(16))) uint4 image[2][G * 64];
  const size_t N = (size_t)1 << a.logN;
  const u32 t = threadIdx.x, n = blockIdx.x * WIDE_THREADS + t, j = blockIdx.y;
  const u32 lo = j * a.alpha, len = min(a.alpha, a.src_nlimbs - lo);
  const u64* src = a.src + (size_t)blockIdx.z * a.src_poly_stride + (size_t)(a.src_slot0 + lo) * N + n;
  u64* dst = a.dst + ((size_t)blockIdx.z * a.beta + j) * a.dst_poly_stride + n;
  // The matrices of a group of four targets: through a register where a request a lane is enough, beyond that straight into LDS, 1 KB
  // a wave and request. (Two requests a lane were an array that the compiler kept in 16 KB of LDS: every word waited for at once and
  // copied twice; two rotations of 30 + 30 limbs in one digit 324 -> 306 us. With one, straight into LDS is no faster: 8 rotations of
  // 24 + 12 limbs 727 -> 737, 12 products of 18 + 9 at 2^15 468 -> 475.)
  constexpr bool DIRECT = G * 64 > WIDE_THREADS;
  const u32 quads = (a.ntarget + 3) / 4, wave = conv_uniform(t >> 6);
  const __amdgpu_buffer_rsrc_t pieces = __builtin_amdgcn_make_buffer_rsrc((void*)a.pieces, 0, (int)(a.beta * quads * G * 1024), 0x00020000);
  uint4 ahead;
  auto request = [&](u32 quad, u32 buffer) {
    const u32 first = (j * quads + quad) * G;
    if (DIRECT) {
#pragma unroll
      for (u32 g0 = 0; g0 < G; g0 += WIDE_THREADS / 64)
        if (g0 + wave < G)   // uniform
          __builtin_amdgcn_raw_ptr_buffer_load_lds(pieces, (lds_void_ptr)&image[buffer][(g0 + wave) * 64], 16, (int)((t & 63) * 16),
                                                   (int)((first + g0 + wave) * 1024), 0, 0);
    } else {
      ahead = a.pieces[(size_t)first * 64 + min(t, G * 64u - 1)];
    }
  };
  auto arrived = [&](u32 buffer) {
    if (DIRECT) conv_wait_vector_memory();
    else if (t < G * 64) image[buffer][t] = ahead;
  };
  // the next group with a target that is not one of the digit's own limbs
  auto skip = [&](u32 quad) {
    if (a.skip_own)
      while (quad < quads && 4 * quad >= lo && min(4 * quad + 4, a.ntarget) <= lo + len) quad++;
    return quad;
  };
  u32 quad = skip(0);
  request(min(quad, quads - 1), 0);
  u64 y[4 * G];
#pragma unroll
  for (int k = 0; k < 4 * G; k++) y[k] = src[(size_t)min((u32)k, len - 1) * N];
  asm volatile("" ::: "memory");   // all of them requested here, not each where it is used
#pragma unroll
  for (int k = 0; k < 4 * G; k++) {
    const u32 i = min((u32)k, len - 1);   // uniform
    const u64 m = scalar_words(a.mods + a.src_id0 + lo + i)[offsetof(ModInfo, m) / 8], h = m >> 1;
    u64 v = y[k];
    if (a.inv) {
      const const_u64_ptr w = scalar_words(a.inv + (size_t)j * a.alpha + i);
      v = shoup(v, w[0], w[1], m);
    }
    y[k] = (u32)k < len ? conv_cut(csub(v + h, m), 0x8080808080808080ull - h) : 0;
  }
  conv_i32x4 b[2][G];
#pragma unroll
  for (int g = 0; g < G; g++) {
    u32 p[2][4];
#pragma unroll
    for (int f = 0; f < 2; f++)
#pragma unroll
      for (int k = 0; k < 2; k++) p[f][2 * k] = (u32)y[4 * g + 2 * f + k], p[f][2 * k + 1] = (u32)(y[4 * g + 2 * f + k] >> 32);
#pragma unroll
    for (int w = 0; w < 4; w++) conv_swap32(p[0][w], p[1][w]);
#pragma unroll
    for (int f = 0; f < 2; f++) b[f][g] = conv_i32x4{(int)p[f][0], (int)p[f][1], (int)p[f][2], (int)p[f][3]};
  }
  arrived(0);
  lds_barrier();
  for (u32 buffer = 0; quad < quads; buffer ^= 1) {
    const u32 next = skip(quad + 1);
    request(min(next, quads - 1), buffer ^ 1);   // read last before the barrier that ended the turn before
    conv_i32x16 d[2] = {};
#pragma unroll
    for (int g = 0; g < G; g++) {
      const conv_i32x4 rows = *(const conv_i32x4*)&image[buffer][g * 64 + (t & 63)];
#pragma unroll
      for (int f = 0; f < 2; f++) d[f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(rows, b[f][g], d[f], 0, 0, 0);
    }
    auto wanted = [&](u32 slot) { return slot < a.ntarget && !(a.skip_own && slot >= lo && slot < lo + len); };   // uniform
    u64 r[4];
#pragma unroll
    for (int p = 0; p < 2; p++) {
      u32 w[2][3];
#pragma unroll
      for (int f = 0; f < 2; f++) {
        const int o = 8 * p;
        wide_join(w[f][0], w[f][1], w[f][2], d[f][o], d[f][o + 1], d[f][o + 2], d[f][o + 3], d[f][o + 4], d[f][o + 5], d[f][o + 6],
                  d[f][o + 7]);
      }
#pragma unroll
      for (int k = 0; k < 3; k++) conv_swap32(w[0][k], w[1][k]);
#pragma unroll
      for (int c = 0; c < 2; c++) {
        const u32 slot = 4 * quad + 2 * p + c;
        if (!wanted(slot)) continue;
        ConvTarget tg;
        tg.fetch(a.mods, a.red, slot, slot < a.main ? slot : slot - a.main + a.special);
        r[2 * p + c] = wide_settle(w[c][0], w[c][1], w[c][2], tg);
        if (!DIRECT) dst[(size_t)slot * N] = r[2 * p + c];
      }
    }
    if (DIRECT) __builtin_amdgcn_sched_barrier(0);
    arrived(buffer ^ 1);
    if (DIRECT) {   // only now: waiting for the request would be waiting for this turn's stores too
#pragma unroll
      for (int c = 0; c < 4; c++)
        if (wanted(4 * quad + c)) dst[(size_t)(4 * quad + c) * N] = r[c];
    }
    lds_barrier();
    quad = next;
  }
}
