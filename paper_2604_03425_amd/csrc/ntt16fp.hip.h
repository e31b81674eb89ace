// Double-precision variants of the two-pass bodies of ntt16.hip.h, for primes q < 2^50.
// On gfx950 the vector FP64 units run at full rate, and a modular multiply by a constant is 6 FP64
// instructions (against ~23 integer instructions for the 64-bit Shoup form), exact because every value is an
// integer below 2^53. Same tiles, lane layouts and LDS transposes as the integer bodies.
//
// Twiddles are single doubles (the quotient estimate uses the rounded product and 1/q, so no companion constant
// is stored) in [-q/2, q/2]. Ranges (in units of q): a multiply by one returns at most 0.5 + 0.1875 |y|, so a forward stage takes
// A to 1.1875 A + 0.5: from 0.5 seven stages stay below 7.88 < 8, from 1 and from 1.5 six and five, from 2.64 (where three
// stages from 0.5 end) four. A radix-16 round takes at most 2.64 and ends with bringing all values back to 0.5. An inverse stage
// doubles the sums and leaves the differences at 0.5 + 0.1875 times theirs: from 0.5 four stages end at 8 (which is below
// 2^53, q being below 2^50), from 1 they do if the two sums of eight values are brought back first; every round ends with all
// values at 0.5. Between the two passes of a transform the data lives in global memory as doubles of at most 2.64 (forward,
// from the conversions), 0.5 (otherwise).
#pragma once
#include "ntt16.hip.h"

template <bool REDUCE = true, class TW>
__device__ __forceinline__ void radix16_fwd_fp(double (&x)[16], double q, double qinv, TW tw) {
#pragma unroll
  for (int s = 0; s < 4; s++) {
    const int half = 8 >> s;
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      const double w = tw(s, g);
#pragma unroll
      for (int p = 0; p < half; p++) {
        double& X = x[g * 2 * half + p];
        double& Y = x[g * 2 * half + p + half];
        const double T = fp_mulmod_var(Y, w, qinv, q);
        Y = X - T;
        X = X + T;
      }
    }
  }
  if (REDUCE) {
#pragma unroll
    for (int i = 0; i < 16; i++) x[i] = fp_reduce(x[i], qinv, q);
  }
}
template <class TW>
__device__ __forceinline__ void radix16_inv_fp(double (&x)[16], double q, double qinv, TW tw) {
#pragma unroll
  for (int s = 3; s >= 0; s--) {
    const int half = 8 >> s;
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      const double w = tw(s, g);
#pragma unroll
      for (int p = 0; p < half; p++) {
        double& X = x[g * 2 * half + p];
        double& Y = x[g * 2 * half + p + half];
        const double D = X - Y;
        X = X + Y;
        Y = fp_mulmod_var(D, w, qinv, q);
      }
    }
    if (s == 1) x[0] = fp_reduce(x[0], qinv, q), x[8] = fp_reduce(x[8], qinv, q);
  }
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = fp_reduce(x[i], qinv, q);
}

// The first LG stages only, on 16 >> LG groups of 2^LG adjacent registers sharing the twiddles; reduced at the end. The
// inverse takes |x| <= 0.5.
template <int LG, class TW>
__device__ __forceinline__ void radix_groups_fwd_fp(double (&x)[16], double q, double qinv, TW tw) {
#pragma unroll
  for (int s = 0; s < LG; s++) {
    const int half = (1 << LG) >> (s + 1);
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      const double w = tw(s, g);
#pragma unroll
      for (int k = 0; k < 16; k += 1 << LG)
#pragma unroll
        for (int p = 0; p < half; p++) {
          double& X = x[k + g * 2 * half + p];
          double& Y = x[k + g * 2 * half + p + half];
          const double T = fp_mulmod_var(Y, w, qinv, q);
          Y = X - T;
          X = X + T;
        }
    }
  }
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = fp_reduce(x[i], qinv, q);
}
template <int LG, class TW>
__device__ __forceinline__ void radix_groups_inv_fp(double (&x)[16], double q, double qinv, TW tw) {
#pragma unroll
  for (int s = LG - 1; s >= 0; s--) {
    const int half = (1 << LG) >> (s + 1);
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      const double w = tw(s, g);
#pragma unroll
      for (int k = 0; k < 16; k += 1 << LG)
#pragma unroll
        for (int p = 0; p < half; p++) {
          double& X = x[k + g * 2 * half + p];
          double& Y = x[k + g * 2 * half + p + half];
          const double D = X - Y;
          X = X + Y;
          Y = fp_mulmod_var(D, w, qinv, q);
        }
    }
  }
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = fp_reduce(x[i], qinv, q);
}

// Forward, stages 0..LOGR-1. `x` holds integers of magnitude at most q (residues as doubles) in the first round's layout
// of the row tile (RowTile); dst receives reduced doubles.
template <int LOGR>
__device__ __forceinline__ void ntt16_fwd_rows_fp_loaded(double (&x)[16], double* __restrict__ dst,
                                                         const double* __restrict__ tw, double q, double qinv, u32 tile,
                                                         double* sm) {
  typedef RowTile<LOGR> T;
  const u32 t = threadIdx.x, i0 = t >> 4;
  double twb[15];  // second-round twiddles, requested before the first round
#pragma unroll
  for (int s = 0; s < T::LG; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) twb[(1 << s) - 1 + g] = tw[(16 << s) + (i0 << s) + g];
  radix16_fwd_fp(x, q, qinv, [&](int s, int g) { return tw[(1 << s) + g]; });
#pragma unroll
  for (int i = 0; i < 16; i++) sm[i * 256 + t] = x[i];
  lds_barrier();
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = sm[T::lds_second(r, t)];
  radix_groups_fwd_fp<T::LG>(x, q, qinv, [&](int s, int g) { return twb[(1 << s) - 1 + g]; });
#pragma unroll
  for (int r = 0; r < 16; r++) dst[T::second(r, t, tile)] = x[r];
}
// The same from canonical residues (uint64) in memory.
template <int LOGR>
__device__ __forceinline__ void ntt16_fwd_rows_fp(const u64* __restrict__ src, double* __restrict__ dst,
                                                  const double* __restrict__ tw, double q, double qinv, u32 tile, double* sm) {
  double x[16];
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = u2d(src[RowTile<LOGR>::first(i, threadIdx.x, tile)]);
  ntt16_fwd_rows_fp_loaded<LOGR>(x, dst, tw, q, qinv, tile, sm);
}

// Forward, the last 8 stages of a limb of R blocks, on doubles of at most 2.64 q. Leaves x (|x| <= q/2) in the i-layout of ntt16_fwd_blocks.
// `x` must already hold the tile in the i-layout (lane (hb, j0) holds positions i*16 + j0 of block h).
// `between` runs after the first round (its twiddles are dead by then), e.g. to request data the caller needs
// after the transform.
template <class BETWEEN>
__device__ __forceinline__ void ntt16_fwd_blocks_fp_loaded(double (&x)[16], const double* __restrict__ tw, double q,
                                                           double qinv, u32 tile, u32 R, double* sm, BETWEEN between) {
  const u32 t = threadIdx.x, j0 = t & 15, hb = t >> 4, h = tile * 16 + hb;
  const u32 i0 = j0;
  // the second round's 15 twiddles are requested up front so they arrive during the first round
  double twb[15];
#pragma unroll
  for (int s = 0; s < 4; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) twb[(1 << s) - 1 + g] = tw[(R << (4 + s)) + (h << (4 + s)) + (i0 << s) + g];
  radix16_fwd_fp(x, q, qinv, [&](int s, int g) { return tw[(R << s) + (h << s) + g]; });
#pragma unroll
  for (int i = 0; i < 16; i++) sm[hb * 272 + i * 17 + j0] = x[i];
  between();
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) x[j] = sm[hb * 272 + i0 * 17 + j];
  radix16_fwd_fp(x, q, qinv, [&](int s, int g) { return twb[(1 << s) - 1 + g]; });
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) sm[hb * 272 + i0 * 17 + j] = x[j];
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = sm[hb * 272 + i * 17 + j0];
}
__device__ __forceinline__ void ntt16_fwd_blocks_fp_loaded(double (&x)[16], const double* __restrict__ tw, double q,
                                                           double qinv, u32 tile, u32 R, double* sm) {
  ntt16_fwd_blocks_fp_loaded(x, tw, q, qinv, tile, R, sm, [] {});
}

// The same block pass with its 16 x 16 transposes done in two halves, low words then high words, through a tile of
// 4-byte words (16 groups x 272 words = 17 KB instead of 34 KB): a kernel that wants the rest of its LDS share for
// something else (the prefetched input tiles of ntt16_fwd_blocks_inner_c_kernel) uses this one. `ex` is the
// workgroup's word tile; exchanges stay inside 16-lane groups, so waiting for the wave's own LDS operations orders them.
__device__ __forceinline__ void fp_transpose16_words(double (&x)[16], u32* row_major, u32 wr_stride, u32 wr_lane,
                                                     u32 rd_stride, u32 rd_lane) {
  u32 lo[16], hi[16];
#pragma unroll
  for (int i = 0; i < 16; i++) row_major[i * wr_stride + wr_lane] = (u32)__double2loint(x[i]);
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) lo[j] = row_major[j * rd_stride + rd_lane];
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < 16; i++) row_major[i * wr_stride + wr_lane] = (u32)__double2hiint(x[i]);
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) hi[j] = row_major[j * rd_stride + rd_lane];
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) x[j] = __hiloint2double((int)hi[j], (int)lo[j]);
}
// `loaded` runs once the loads of all 30 twiddles have been issued and before anything waits for them: memory
// requests a caller starts there are younger than every load the two rounds wait for, so those waits leave them in
// flight. `between` runs after the first round.
// The first round's 15 twiddles are the same for the 16 lanes of a group and for every tile the workgroup transforms:
// `twl` holds them in LDS (group hb at twl + hb * NTT16_TWL_PITCH, filled by ntt16_fwd_blocks_fp_words_twl), so a
// transform starts on a short LDS read instead of a trip to the L2.
#define NTT16_TWL_PITCH 18
// Filling it is split in two so that a caller can put other work between the request and the use of the value:
// wave w fills the rows of its own four groups, lane L < 60 moving twiddle L % 15 of group 4w + L / 15.
__device__ __forceinline__ double ntt16_twl_fetch(const double* __restrict__ tw, u32 tile, u32 R) {
  const u32 t = threadIdx.x, L = min(t & 63, 59u);
  const u32 hb = (t >> 6) * 4 + L / 15, k = L % 15, h = tile * 16 + hb;
  const u32 s = k >= 7 ? 3 : k >= 3 ? 2 : k >= 1 ? 1 : 0, g = k + 1 - (1u << s);
  return tw[(R << s) + (h << s) + g];
}
__device__ __forceinline__ void ntt16_twl_store(double v, double* twl) {
  const u32 t = threadIdx.x, L = t & 63;
  if (L < 60) twl[((t >> 6) * 4 + L / 15) * NTT16_TWL_PITCH + L % 15] = v;
}
template <bool REDUCE, class LOADED, class BETWEEN>   // without REDUCE: out at most 3.64 q
__device__ __forceinline__ void ntt16_fwd_blocks_fp_words(double (&x)[16], const double* __restrict__ tw, double q,
                                                          double qinv, u32 tile, u32 R, u32* ex, const double* twl, LOADED loaded,
                                                          BETWEEN between) {
  const u32 t = threadIdx.x, j0 = t & 15, hb = t >> 4, h = tile * 16 + hb;
  const u32 i0 = j0;
  u32* grp = ex + hb * 272;
  double twa[15], twb[15];
#pragma unroll
  for (int s = 0; s < 4; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) twb[(1 << s) - 1 + g] = tw[(R << (4 + s)) + (h << (4 + s)) + (i0 << s) + g];
#pragma unroll
  for (int k = 0; k < 15; k++) twa[k] = twl[hb * NTT16_TWL_PITCH + k];
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  loaded();
  __builtin_amdgcn_sched_barrier(0);
  radix16_fwd_fp(x, q, qinv, [&](int s, int g) { return twa[(1 << s) - 1 + g]; });
  // element (i, j0) -> lane i0 = i holds (i0, j): written at i*17 + j0, read at i0*17 + j
  fp_transpose16_words(x, grp, 17, j0, 1, i0 * 17);
  between();
  radix16_fwd_fp<REDUCE>(x, q, qinv, [&](int s, int g) { return twb[(1 << s) - 1 + g]; });
  // and back: written at i0*17 + j, read at i*17 + j0
  fp_transpose16_words(x, grp, 1, i0 * 17, 17, j0);
}

// Inverse, the first 8 stages. In: x = canonical residues as doubles, i-layout. Out: reduced doubles, i-layout.
__device__ __forceinline__ void ntt16_inv_blocks_fp(double (&x)[16], const double* __restrict__ twi, double q, double qinv,
                                                    u32 tile, u32 R, double* sm) {
  const u32 t = threadIdx.x, j0 = t & 15, hb = t >> 4, h = tile * 16 + hb;
  const u32 i0 = j0;
  double twa[15], twb[15];  // both rounds' twiddles, requested before the first transpose
#pragma unroll
  for (int s = 0; s < 4; s++)
#pragma unroll
    for (int g = 0; g < (1 << s); g++) {
      twa[(1 << s) - 1 + g] = twi[(R << (4 + s)) + (h << (4 + s)) + (i0 << s) + g];
      twb[(1 << s) - 1 + g] = twi[(R << s) + (h << s) + g];
    }
#pragma unroll
  for (int i = 0; i < 16; i++) sm[hb * 272 + i * 17 + j0] = x[i];
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) x[j] = sm[hb * 272 + i0 * 17 + j];
  radix16_inv_fp(x, q, qinv, [&](int s, int g) { return twa[(1 << s) - 1 + g]; });
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 16; j++) sm[hb * 272 + i0 * 17 + j] = x[j];
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = sm[hb * 272 + i * 17 + j0];
  radix16_inv_fp(x, q, qinv, [&](int s, int g) { return twb[(1 << s) - 1 + g]; });
}

// Inverse, stages LOGR-1..0, then multiplication by (sc, sc/q); out receives canonical residues (uint64) in the first
// round's layout of the row tile.
template <int LOGR>
__device__ __forceinline__ void ntt16_inv_rows_fp(u64 (&out)[16], const double* __restrict__ src, const double* __restrict__ twi,
                                                  double q, double qinv, double sc, double scq, u32 tile, double* sm) {
  typedef RowTile<LOGR> T;
  const u32 t = threadIdx.x, i0 = t >> 4;
  double x[16];
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = src[T::second(r, t, tile)];
  radix_groups_inv_fp<T::LG>(x, q, qinv, [&](int s, int g) { return twi[(16 << s) + (i0 << s) + g]; });
#pragma unroll
  for (int r = 0; r < 16; r++) sm[T::lds_second(r, t)] = x[r];
  lds_barrier();
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = sm[i * 256 + t];
  radix16_inv_fp(x, q, qinv, [&](int s, int g) { return twi[(1 << s) + g]; });
#pragma unroll
  for (int i = 0; i < 16; i++) out[i] = d2u_canon(fp_mulmod_const(x[i], sc, scq, q), q);
}

__device__ __forceinline__ void ntt16_fwd_blocks_fp(double (&x)[16], const double* __restrict__ src,
                                                    const double* __restrict__ tw, double q, double qinv, u32 tile, u32 R, double* sm) {
  const u32 t = threadIdx.x, j0 = t & 15, h = tile * 16 + (t >> 4);
  const double* blk = src + (size_t)h * 256;
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = blk[i * 16 + j0];
  ntt16_fwd_blocks_fp_loaded(x, tw, q, qinv, tile, R, sm);
}
