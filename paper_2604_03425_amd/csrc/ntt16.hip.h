// Two-pass negacyclic NTT for N = 2^13 .. 2^16 on gfx950. A limb is viewed as R = N / 256 rows of 256 elements; each pass
// works on 4096-element tiles held as 16 registers per lane (256 lanes), as in-register radix-16 rounds with one LDS
// transpose between them. Pass "row" does the first log2 R stages (stride-256 butterflies) on all R rows x 4096 / R
// adjacent columns; pass "blk" does the last 8 stages on 16 contiguous 256-element blocks. Global loads and stores
// always have 16 adjacent lanes on 128 contiguous bytes. The block bodies take R at run time (block h of R takes its
// stage-s twiddles from R << s onward, so R only shifts an index); the row bodies are instantiated per LOGR = log2 R,
// which fixes how many of the second round's stages exist: a lane then holds 16 / (R / 16) columns of that round.
//
// Lazy ranges. Every twiddle product is the approximate shoup_lazy4 (below 4q), and the lazy constant the bodies
// pass around is 4q. SMALL primes (q < 2^52): forward butterflies never correct, values grow by 4q per
// stage (< 65q < 2^59 after 16 stages from canonical input) and are reduced once at the end; inverse
// butterflies let sums double for the 8 stages of a pass (inputs < 4q -> < 1024q). BIG primes (q < 2^60)
// use Harvey's butterflies: 16q fits 64 bits, so forward values are kept in [0,16q) with a correction by 8q in every other stage
// (the first of a round; below 12q after it, 16q after the next), inverse ones in [0,8q).
#pragma once
#include "modarith.hip.h"

#define NTT16_THREADS 256
#define NTT16_LDS_BYTES (16 * 272 * 8)

// ---- butterflies ----
template <bool BIG>
__device__ __forceinline__ u64 lazy_const(u64 q) { return 4 * q; }
// Forward (Cooley-Tukey), q2 = 4q. SMALL: values grow by 4q per stage. BIG: CORRECT takes inputs below 16q to outputs below 12q,
// without it inputs below 12q go to outputs below 16q. X + T is formed in the product's own multiply-add chain. Correcting every
// other stage and adding there: 18 vector instructions on average instead of 22; 4 products of
// 12 + 4 60-bit limbs at 2^16 322 -> 314 us, 12 rotations of 6 + 2 limbs at 2^14 99 -> 97.
template <bool BIG, bool CORRECT>
__device__ __forceinline__ void bf_fwd(u64& X, u64& Y, ulonglong2 w, u64 q, u64 q2) {
  if (BIG && CORRECT) X = csub_neg(X, 2 * q2);
  const u64 s = shoup_lazy4_add(X, Y, w.x, w.y, neg_opaque(q));
  Y = (X << 1) + q2 - s;
  X = s;
}
// The stages of a round are corrected alternately, from the first one (s = 0) on.
template <bool BIG>
__device__ __forceinline__ void bf_fwd(u64& X, u64& Y, ulonglong2 w, u64 q, u64 q2, int s) {
  if (s & 1) bf_fwd<BIG, false>(X, Y, w, q, q2);
  else bf_fwd<BIG, true>(X, Y, w, q, q2);
}
// Inverse (Gentleman-Sande). BIG: c = 4q, inputs and outputs in [0,8q); PRODUCTS: both inputs are products of the stage
// before, below 4q, whose sum needs no correction. SMALL: inputs < c (a multiple of q, at least 4q), X' < 2c, Y' < 4q.
template <bool BIG, bool PRODUCTS = false>
__device__ __forceinline__ void bf_inv(u64& X, u64& Y, ulonglong2 w, u64 q, u64 c) {
  u64 S = X + Y;
  u64 D = X + (BIG && !PRODUCTS ? 2 * c : c) - Y;
  if (BIG && !PRODUCTS) S = csub_neg(S, 2 * c);
  X = S;
  Y = shoup_lazy4(D, w.x, w.y, q);
}

// Pair p of a stage whose pairs are `half` registers apart: of the stage before, half / 2 apart, it holds two sums or, every
// other half / 2 of them, two products. Half the corrections of all but a round's first stage fall away.
template <bool BIG>
__device__ __forceinline__ void bf_inv_pair(u64& X, u64& Y, ulonglong2 w, u64 q, u64 c, int half, int p) {
  if (p & (half >> 1)) bf_inv<BIG, true>(X, Y, w, q, c);
  else bf_inv<BIG>(X, Y, w, q, c);
}

// Four forward stages on 16 registers: stage s pairs (a, a + (8>>s)); tw(s, g) is the twiddle of group g.
template <bool BIG, class TW>
__device__ __forceinline__ void radix16_fwd(u64 (&x)[16], u64 q, u64 q2, TW tw) {
#pragma unroll
  for (int s = 0; s < 4; s++) {
    const int half = 8 >> s;
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      ulonglong2 w = tw(s, g);
#pragma unroll
      for (int p = 0; p < half; p++) bf_fwd<BIG>(x[g * 2 * half + p], x[g * 2 * half + p + half], w, q, q2, s);
    }
  }
}
// Four inverse stages, in the reverse order (s = 3..0). c0 = bound of the inputs (SMALL) or 4q (BIG).
template <bool BIG, class TW>
__device__ __forceinline__ void radix16_inv(u64 (&x)[16], u64 q, u64 c0, TW tw) {
  u64 c = c0;
#pragma unroll
  for (int s = 3; s >= 0; s--) {
    const int half = 8 >> s;
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      ulonglong2 w = tw(s, g);
#pragma unroll
      for (int p = 0; p < half; p++) bf_inv_pair<BIG>(x[g * 2 * half + p], x[g * 2 * half + p + half], w, q, c, half, p);
    }
    if (!BIG) c <<= 1;
  }
}

// The same rounds with a hook after every stage: a pass uses it to request the next round's twiddles as this round's
// die, so that no twiddle is waited for right after it was requested (15 twiddle pairs are 60 registers: two rounds'
// worth do not fit beside the data).
template <bool BIG, class TW, class AFTER>
__device__ __forceinline__ void radix16_fwd_staged(u64 (&x)[16], u64 q, u64 q2, TW tw, AFTER after) {
#pragma unroll
  for (int s = 0; s < 4; s++) {
    const int half = 8 >> s;
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      ulonglong2 w = tw(s, g);
#pragma unroll
      for (int p = 0; p < half; p++) bf_fwd<BIG>(x[g * 2 * half + p], x[g * 2 * half + p + half], w, q, q2, s);
    }
    after(s);
  }
}
template <bool BIG, class TW, class AFTER>
__device__ __forceinline__ void radix16_inv_staged(u64 (&x)[16], u64 q, u64 c0, TW tw, AFTER after) {
  u64 c = c0;
#pragma unroll
  for (int s = 3; s >= 0; s--) {
    const int half = 8 >> s;
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      ulonglong2 w = tw(s, g);
#pragma unroll
      for (int p = 0; p < half; p++) bf_inv_pair<BIG>(x[g * 2 * half + p], x[g * 2 * half + p + half], w, q, c, half, p);
    }
    if (!BIG) c <<= 1;
    after(s);
  }
}
// The first LG stages only, on the 16 >> LG groups of 2^LG adjacent registers (the second round of a row pass over R =
// 2^(4 + LG) rows): all groups share the twiddles.
template <bool BIG, int LG, class TW>
__device__ __forceinline__ void radix_groups_fwd(u64 (&x)[16], u64 q, u64 q2, TW tw) {
#pragma unroll
  for (int s = 0; s < LG; s++) {
    const int half = (1 << LG) >> (s + 1);
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      ulonglong2 w = tw(s, g);
#pragma unroll
      for (int k = 0; k < 16; k += 1 << LG)
#pragma unroll
        for (int p = 0; p < half; p++) bf_fwd<BIG>(x[k + g * 2 * half + p], x[k + g * 2 * half + p + half], w, q, q2, s);
    }
  }
}
template <bool BIG, int LG, class TW>
__device__ __forceinline__ void radix_groups_inv(u64 (&x)[16], u64 q, u64 c0, TW tw) {
  u64 c = c0;
#pragma unroll
  for (int s = LG - 1; s >= 0; s--) {
    const int half = (1 << LG) >> (s + 1);
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      ulonglong2 w = tw(s, g);
#pragma unroll
      for (int k = 0; k < 16; k += 1 << LG)
#pragma unroll
        for (int p = 0; p < half; p++) bf_inv_pair<BIG>(x[k + g * 2 * half + p], x[k + g * 2 * half + p + half], w, q, c, half, p);
    }
    if (!BIG) c <<= 1;
  }
}
// Slot of the twiddle pair of stage s, group g in a round's table of 15.
#define NTT16_TW_INDEX(s, g) ((1 << (s)) - 1 + (g))
// The 2^s twiddle pairs of stage s, from `src`, into their slots of a round's table. Written out per stage so that
// every index is a constant and the table stays in registers.
__device__ __forceinline__ void ntt16_load_stage(ulonglong2 (&t)[15], const ulonglong2* __restrict__ src, int s) {
  if (s == 0) {
    t[0] = src[0];
  } else if (s == 1) {
    t[1] = src[0], t[2] = src[1];
  } else if (s == 2) {
    t[3] = src[0], t[4] = src[1], t[5] = src[2], t[6] = src[3];
  } else {
    t[7] = src[0], t[8] = src[1], t[9] = src[2], t[10] = src[3];
    t[11] = src[4], t[12] = src[5], t[13] = src[6], t[14] = src[7];
  }
}

__device__ __forceinline__ u64 barrett_lazy(u64 v, u64 mu, u64 q) { return v - mul_hi64(v, mu) * q; }  // [0,2q)
// The end of a forward transform: below 2q.
template <bool BIG>
__device__ __forceinline__ u64 fwd_settle(u64 v, u64 mu, u64 q) {
  return BIG ? csub_neg(csub_neg(csub_neg(v, 8 * q), 4 * q), 2 * q) : barrett_lazy(v, mu, q);
}

// ---- pass bodies. `base` points at one limb-vector of N words, `tw` at that modulus' table. ----

// Lane layouts of a row pass over R = 2^LOGR rows (NC = 4096 / R columns per tile, J = R / 16). First round: lane
// (r0 = t / NC, col = t % NC) holds rows i*J + r0 (i = 0..15) of column col0 + col. Second round: lane (i0 = t >> 4,
// c = t & 15) holds rows i0*J + j (j < J) of the columns col0 + c + 16*k (k < 16 / J) in register k*J + j.
template <int LOGR>
struct RowTile {
  static constexpr int LG = LOGR - 4, J = 1 << LG, NC = 4096 >> LOGR;
  // offset of register i of a lane inside the limb, first round / second round
  static __device__ __forceinline__ u32 first(u32 i, u32 t, u32 tile) { return ((i << LG) + t / NC) * 256 + tile * NC + t % NC; }
  static __device__ __forceinline__ u32 second(u32 r, u32 t, u32 tile) {
    return (((t >> 4) << LG) + (r & (J - 1))) * 256 + tile * NC + (t & 15) + 16 * (r >> LG);
  }
  // the same inside the LDS tile [R][NC]; the first round's layout is i * 256 + t
  static __device__ __forceinline__ u32 lds_second(u32 r, u32 t) {
    return (((t >> 4) << LG) + (r & (J - 1))) * NC + (t & 15) + 16 * (r >> LG);
  }
};

// Forward, stages 0..LOGR-1. In: canonical (or < 2q). Out: SMALL < 33q (+in), BIG < 16q. `x` holds the first round's layout.
template <bool BIG, int LOGR>
__device__ __forceinline__ void ntt16_fwd_rows_loaded(u64 (&x)[16], u64* __restrict__ dst, const ulonglong2* __restrict__ tw,
                                                      u64 q, u32 tile, u64* sm) {
  typedef RowTile<LOGR> T;
  const u32 t = threadIdx.x, i0 = t >> 4;
  const u64 q2 = lazy_const<BIG>(q);
  // the second round's twiddles (one set per 16-lane group) are requested here, next to the data loads, and arrive
  // during the first round, whose own twiddles are wave-uniform scalar loads
  ulonglong2 twb[15];
#pragma unroll
  for (int s = 0; s < T::LG; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) twb[NTT16_TW_INDEX(s, g)] = tw[(16 << s) + (i0 << s) + g];
  __builtin_amdgcn_sched_barrier(0);
  radix16_fwd<BIG>(x, q, q2, [&](int s, int g) { return tw[(1 << s) + g]; });
#pragma unroll
  for (int i = 0; i < 16; i++) sm[i * 256 + t] = x[i];
  lds_barrier();
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = sm[T::lds_second(r, t)];
  radix_groups_fwd<BIG, T::LG>(x, q, q2, [&](int s, int g) { return twb[NTT16_TW_INDEX(s, g)]; });
#pragma unroll
  for (int r = 0; r < 16; r++) dst[T::second(r, t, tile)] = x[r];
}
template <bool BIG, int LOGR>
__device__ __forceinline__ void ntt16_fwd_rows(const u64* __restrict__ src, u64* __restrict__ dst, const ulonglong2* __restrict__ tw,
                                               u64 q, u32 tile, u64* sm) {
  u64 x[16];
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = src[RowTile<LOGR>::first(i, threadIdx.x, tile)];
  ntt16_fwd_rows_loaded<BIG, LOGR>(x, dst, tw, q, tile, sm);
}

// Forward, the last 8 stages of a limb of R blocks, then canonical (CANON) or lazy (BIG: < 8q, SMALL: < 67q). `x` is left holding, for lane (hb = t>>4, j0 = t&15), the 16 values at
// block h = tile*16 + hb, positions i*16 + j0 (i = 0..15), ready for a coalesced store or a fused epilogue.
template <bool BIG, bool CANON = true>
__device__ __forceinline__ void ntt16_fwd_blocks_loaded(u64 (&x)[16], const ulonglong2* __restrict__ tw, u64 q, u64 mu,
                                                        u32 tile, u32 R, u64* sm) {
  const u32 t = threadIdx.x, j0 = t & 15, hb = t >> 4, h = tile * 16 + hb;
  const u64 q2 = lazy_const<BIG>(q);
  const u32 i0 = j0;
  // first round's twiddles (one set per group) requested here, next to the caller's data loads; the second round's
  // (one set per lane) take their registers over stage by stage
  ulonglong2 twa[15], twb[15];
#pragma unroll
  for (int s = 0; s < 4; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) twa[NTT16_TW_INDEX(s, g)] = tw[(R << s) + (h << s) + g];
  __builtin_amdgcn_sched_barrier(0);
  radix16_fwd_staged<BIG>(
      x, q, q2, [&](int s, int g) { return twa[NTT16_TW_INDEX(s, g)]; },
      [&](int s) {
        __builtin_amdgcn_sched_barrier(0);
        ntt16_load_stage(twb, tw + (R << (4 + s)) + (h << (4 + s)) + (i0 << s), s);
        __builtin_amdgcn_sched_barrier(0);
      });
#pragma unroll
  for (int i = 0; i < 16; i++) sm[hb * 272 + i * 17 + j0] = x[i];
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) x[j] = sm[hb * 272 + i0 * 17 + j];
  radix16_fwd<BIG>(x, q, q2, [&](int s, int g) { return twb[NTT16_TW_INDEX(s, g)]; });
#pragma unroll
  for (int j = 0; j < 16; j++) {
    if (CANON) x[j] = csub(fwd_settle<BIG>(x[j], mu, q), q);
    else if (BIG) x[j] = csub_neg(x[j], 8 * q);
  }
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) sm[hb * 272 + i0 * 17 + j] = x[j];
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = sm[hb * 272 + i * 17 + j0];
}

template <bool BIG, bool CANON = true>
__device__ __forceinline__ void ntt16_fwd_blocks(u64 (&x)[16], const u64* __restrict__ src, const ulonglong2* __restrict__ tw,
                                                 u64 q, u64 mu, u32 tile, u32 R, u64* sm) {
  const u32 t = threadIdx.x, j0 = t & 15, h = tile * 16 + (t >> 4);
  const u64* blk = src + (size_t)h * 256;
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = blk[i * 16 + j0];
  ntt16_fwd_blocks_loaded<BIG, CANON>(x, tw, q, mu, tile, R, sm);
}

// Forward, the last 8 stages of one 256-element block h of R by 32 adjacent lanes with 8 values each (radix-8, exchange, radix-8, exchange, radix-4; LDS rows of pitch 35 words per 32 elements,
// all exchanges inside the half-wave). In: x[i] = element i*32 + l, lazy (BIG: < 16q). Out: x[c] = element
// (l >> 2)*32 + (l & 3)*8 + c, lazy (BIG: < 16q, SMALL: < 65q). `between` runs after the first exchange has been written.
#define NTT8_PITCH_I 35
#define NTT8_BLOCK_LDS_I (8 * NTT8_PITCH_I)
// (the second of two radix-8 rounds: three stages came before, the first of these is not corrected)
template <bool BIG, class TW>
__device__ __forceinline__ void radix8_fwd(u64 (&x)[8], u64 q, u64 q2, TW tw) {
#pragma unroll
  for (int s = 0; s < 3; s++) {
    const int half = 4 >> s;
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      const ulonglong2 w = tw(s, g);
#pragma unroll
      for (int p = 0; p < half; p++) bf_fwd<BIG>(x[g * 2 * half + p], x[g * 2 * half + p + half], w, q, q2, s + 1);
    }
  }
}
template <bool BIG, class TW, class AFTER>
__device__ __forceinline__ void radix8_fwd_staged(u64 (&x)[8], u64 q, u64 q2, TW tw, AFTER after) {
#pragma unroll
  for (int s = 0; s < 3; s++) {
    const int half = 4 >> s;
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      const ulonglong2 w = tw(s, g);
#pragma unroll
      for (int p = 0; p < half; p++) bf_fwd<BIG>(x[g * 2 * half + p], x[g * 2 * half + p + half], w, q, q2, s);
    }
    after(s);
  }
}
template <bool BIG, class BETWEEN>
__device__ __forceinline__ void ntt256_fwd_blocks_int8(u64 (&x)[8], const ulonglong2* __restrict__ tw, u64 q, u32 h,
                                                       u32 R, u32 l, u64* smb, BETWEEN between) {
  const u32 a = l >> 2, b = l & 3;
  const u64 q2 = lazy_const<BIG>(q);
  // The first two rounds' twiddles are requested before `between` runs: the first round's here, the second round's
  // stage by stage as the first round's registers die. Whatever `between` requests is then younger than all of them,
  // so the second round never waits for it. The last two stages' twiddles follow once the second round's registers
  // are free; by then the caller needs what `between` requested anyway.
  ulonglong2 t1[7], t2[7], t3[6];
#pragma unroll
  for (int s = 0; s < 3; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) t1[(1 << s) - 1 + g] = tw[(R << s) + (h << s) + g];
  __builtin_amdgcn_sched_barrier(0);
  radix8_fwd_staged<BIG>(
      x, q, q2, [&](int s, int g) { return t1[(1 << s) - 1 + g]; },
      [&](int s) {
        __builtin_amdgcn_sched_barrier(0);
        const ulonglong2* ts = tw + (R << (3 + s)) + (h << (3 + s)) + (a << s);
        if (s == 0) {
          t2[0] = ts[0];
        } else if (s == 1) {
          t2[1] = ts[0], t2[2] = ts[1];
        } else {
          t2[3] = ts[0], t2[4] = ts[1], t2[5] = ts[2], t2[6] = ts[3];
        }
        __builtin_amdgcn_sched_barrier(0);
      });
#pragma unroll
  for (int i = 0; i < 8; i++) smb[i * NTT8_PITCH_I + l] = x[i];
  between();
  __builtin_amdgcn_sched_barrier(0);
  wave_lds_sync();
#pragma unroll
  for (int r = 0; r < 8; r++) x[r] = smb[a * NTT8_PITCH_I + r * 4 + b];
  radix8_fwd<BIG>(x, q, q2, [&](int s, int g) { return t2[(1 << s) - 1 + g]; });
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < 2; u++) t3[u] = tw[(R << 6) + (h << 6) + (a << 3) + (b << 1) + u];
#pragma unroll
  for (int k = 0; k < 4; k++) t3[2 + k] = tw[(R << 7) + (h << 7) + (a << 4) + (b << 2) + k];
  __builtin_amdgcn_sched_barrier(0);
  wave_lds_sync();
#pragma unroll
  for (int r = 0; r < 8; r++) smb[a * NTT8_PITCH_I + r * 4 + b] = x[r];
  wave_lds_sync();
#pragma unroll
  for (int c = 0; c < 8; c++) x[c] = smb[a * NTT8_PITCH_I + b * 8 + c];
#pragma unroll
  for (int u = 0; u < 2; u++) {   // stage 14: pairs (c, c + 2) inside each half
#pragma unroll
    for (int p = 0; p < 2; p++) bf_fwd<BIG, true>(x[u * 4 + p], x[u * 4 + p + 2], t3[u], q, q2);
  }
#pragma unroll
  for (int k = 0; k < 4; k++) bf_fwd<BIG, false>(x[2 * k], x[2 * k + 1], t3[2 + k], q, q2);   // stage 15: pairs (2k, 2k + 1)
}

// The way back for two polynomials at once, which share the twiddles: the first 8 inverse stages of block h. In: x[k][c] = element
// (l >> 2)*32 + (l & 3)*8 + c, below 2q. Out: x[k][i] = element i*32 + l, below 2q (BIG: 8q).
template <bool BIG, class TW>
__device__ __forceinline__ void radix8_inv(u64 (&x)[8], u64 q, u64 c0, TW tw) {
  u64 c = c0;
#pragma unroll
  for (int s = 2; s >= 0; s--) {
    const int half = 4 >> s;
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      const ulonglong2 w = tw(s, g);
#pragma unroll
      for (int p = 0; p < half; p++) bf_inv_pair<BIG>(x[g * 2 * half + p], x[g * 2 * half + p + half], w, q, c, half, p);
    }
    if (!BIG) c <<= 1;
  }
}
template <bool BIG>
__device__ __forceinline__ void ntt256_inv_blocks_int8(u64 (&x)[2][8], const ulonglong2* __restrict__ twi, u64 q, u64 mu, u32 h, u32 R,
                                                       u32 l, u64* smb) {
  const u32 a = l >> 2, b = l & 3;
  const u64 q2 = lazy_const<BIG>(q);
  ulonglong2 t1[7], t2[7], t3[6];
#pragma unroll
  for (int u = 0; u < 2; u++) t3[u] = twi[(R << 6) + (h << 6) + (a << 3) + (b << 1) + u];
#pragma unroll
  for (int k = 0; k < 4; k++) t3[2 + k] = twi[(R << 7) + (h << 7) + (a << 4) + (b << 2) + k];
#pragma unroll
  for (int s = 0; s < 3; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) t2[(1 << s) - 1 + g] = twi[(R << (3 + s)) + (h << (3 + s)) + (a << s) + g];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int e = 0; e < 2; e++) {
#pragma unroll
    for (int k = 0; k < 4; k++) bf_inv<BIG>(x[e][2 * k], x[e][2 * k + 1], t3[2 + k], q, q2);
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
      for (int p = 0; p < 2; p++) bf_inv_pair<BIG>(x[e][u * 4 + p], x[e][u * 4 + p + 2], t3[u], q, BIG ? q2 : q2 << 1, 2, p);
  }
#pragma unroll
  for (int s = 0; s < 3; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) t1[(1 << s) - 1 + g] = twi[(R << s) + (h << s) + g];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int e = 0; e < 2; e++) {
    wave_lds_sync();
#pragma unroll
    for (int c = 0; c < 8; c++) smb[a * NTT8_PITCH_I + b * 8 + c] = x[e][c];
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 8; r++) x[e][r] = smb[a * NTT8_PITCH_I + r * 4 + b];
    radix8_inv<BIG>(x[e], q, BIG ? q2 : q2 << 2, [&](int s, int g) { return t2[(1 << s) - 1 + g]; });
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 8; r++) smb[a * NTT8_PITCH_I + r * 4 + b] = x[e][r];
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < 8; i++) x[e][i] = smb[i * NTT8_PITCH_I + l];
    radix8_inv<BIG>(x[e], q, BIG ? q2 : q2 << 5, [&](int s, int g) { return t1[(1 << s) - 1 + g]; });
    if (!BIG) {
#pragma unroll
      for (int i = 0; i < 8; i++) x[e][i] = barrett_lazy(x[e][i], mu, q);
    }
  }
}

// Inverse, the first 8 stages, on contiguous blocks. In: x holds, for lane (hb, j0), the values at positions i*16 + j0
// of block h (any value < 2q). Out: < 2q (BIG: < 8q), same lane layout, ready for a coalesced store.
template <bool BIG>
__device__ __forceinline__ void ntt16_inv_blocks(u64 (&x)[16], const ulonglong2* __restrict__ twi, u64 q, u64 mu, u32 tile,
                                                 u32 R, u64* sm) {
  const u32 t = threadIdx.x, j0 = t & 15, hb = t >> 4, h = tile * 16 + hb;
  const u64 q2 = lazy_const<BIG>(q);
  const u32 i0 = j0;
  // first round's twiddles (one set per lane): requested before the transpose; the second round's (one set per
  // group) take their registers over stage by stage
  ulonglong2 twa[15];
#pragma unroll
  for (int s = 0; s < 4; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) twa[NTT16_TW_INDEX(s, g)] = twi[(R << (4 + s)) + (h << (4 + s)) + (i0 << s) + g];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 16; i++) sm[hb * 272 + i * 17 + j0] = x[i];
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) x[j] = sm[hb * 272 + i0 * 17 + j];
  ulonglong2 twb[15];
  radix16_inv_staged<BIG>(
      x, q, q2, [&](int s, int g) { return twa[NTT16_TW_INDEX(s, g)]; },
      [&](int s) {
        __builtin_amdgcn_sched_barrier(0);
        ntt16_load_stage(twb, twi + (R << s) + (h << s), s);
        __builtin_amdgcn_sched_barrier(0);
      });
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) sm[hb * 272 + i0 * 17 + j] = x[j];
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = sm[hb * 272 + i * 17 + j0];
  radix16_inv<BIG>(x, q, BIG ? q2 : (q2 << 4), [&](int s, int g) { return twb[NTT16_TW_INDEX(s, g)]; });
  if (!BIG) {
#pragma unroll
    for (int i = 0; i < 16; i++) x[i] = barrett_lazy(x[i], mu, q);
  }
}

// Inverse, stages LOGR-1..0 on R rows x NC columns, then multiplication by the constant (sc, scs) (N^-1, possibly
// merged with another per-limb constant) and canonical output. In: < 2q (BIG: < 8q). x receives the first round's layout
// of the row tile.
template <bool BIG, int LOGR>
__device__ __forceinline__ void ntt16_inv_rows(u64 (&x)[16], const u64* __restrict__ src, const ulonglong2* __restrict__ twi,
                                               u64 q, u64 sc, u64 scs, u32 tile, u64* sm) {
  typedef RowTile<LOGR> T;
  const u32 t = threadIdx.x, i0 = t >> 4;
  const u64 q2 = lazy_const<BIG>(q);
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = src[T::second(r, t, tile)];
  // first round's twiddles (one set per group) travel with the data; the second round's are scalar loads
  ulonglong2 twa[15];
#pragma unroll
  for (int s = 0; s < T::LG; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) twa[NTT16_TW_INDEX(s, g)] = twi[(16 << s) + (i0 << s) + g];
  __builtin_amdgcn_sched_barrier(0);
  radix_groups_inv<BIG, T::LG>(x, q, q2, [&](int s, int g) { return twa[NTT16_TW_INDEX(s, g)]; });
#pragma unroll
  for (int r = 0; r < 16; r++) sm[T::lds_second(r, t)] = x[r];
  lds_barrier();
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = sm[i * 256 + t];
  radix16_inv<BIG>(x, q, BIG ? q2 : (q2 << T::LG), [&](int s, int g) { return twi[(1 << s) + g]; });
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = shoup(x[i], sc, scs, q);
}

// Workgroup -> (poly, tile, slot). mode 0: dispatch order is polynomial-fastest; 1: same, made XCD-contiguous;
// 2: tile-fastest; 3: tile-fastest, XCD-contiguous; 4: all polynomials of one (tile, slot) group run on one XCD
// (they share that group's twiddles and key slices in its L2) while eight consecutive groups, one per XCD, are in
// flight together, which keeps the XCDs evenly loaded (groups beyond the last multiple of 8 are dealt out in order).
__device__ __forceinline__ void ntt16_map(u32 mode, u32& poly, u32& tile, u32& slot) {
  const u32 lin0 = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  if (mode == 4) {
    const u32 whole = (gridDim.y * gridDim.z) & ~7u;
    u32 group;
    if (lin0 < whole * gridDim.x) {
      const u32 x = lin0 & 7, rest = lin0 >> 3;
      poly = rest % gridDim.x;
      group = x + 8 * (rest / gridDim.x);
    } else {
      const u32 rest = lin0 - whole * gridDim.x;
      poly = rest % gridDim.x;
      group = whole + rest / gridDim.x;
    }
    tile = group % gridDim.y;
    slot = group / gridDim.y;
    return;
  }
  const u32 lin = (mode & 1) ? xcd_swizzled_linear_id() : lin0;
  if (mode & 2) {
    tile = lin % gridDim.y;
    poly = (lin / gridDim.y) % gridDim.x;
  } else {
    poly = lin % gridDim.x;
    tile = (lin / gridDim.x) % gridDim.y;
  }
  slot = lin / (gridDim.x * gridDim.y);
}
