// Radix-4 rounds on four values per lane, and the transform of a 2^12 limb by 1024 lanes built from them. Four values per
// lane instead of sixteen leave room in the registers for what a fused kernel keeps beside the transform, give a lone
// workgroup 16 waves to hide latency with, and make the straight-line code a quarter as long: with few workgroups in
// flight, fetching instructions is a large part of a kernel's time.
#pragma once
#include "ntt16fp.hip.h"

__device__ __forceinline__ void reduce4(double (&x)[4], double q, double qinv) {
#pragma unroll
  for (int i = 0; i < 4; i++) x[i] = fp_reduce(x[i], qinv, q);
}
// Two forward stages: (0,2),(1,3) by w[0], then (0,1) by w[1] and (2,3) by w[2]; reduced between them if BETWEEN. Ranges as
// for radix16_fwd(_fp).
template <bool BETWEEN = false>
__device__ __forceinline__ void radix4_fwd(double (&x)[4], const double (&w)[3], double q, double qinv) {
#pragma unroll
  for (int s = 0; s < 2; s++) {
    if (BETWEEN && s == 1) reduce4(x, q, qinv);
#pragma unroll
    for (int p = 0; p < 2; p++) {
      double& X = x[s == 0 ? p : 2 * p];
      double& Y = x[s == 0 ? p + 2 : 2 * p + 1];
      const double T = fp_mulmod_var(Y, s == 0 ? w[0] : w[1 + p], qinv, q);
      Y = X - T;
      X = X + T;
    }
  }
}
// Two inverse stages in the reverse order.
__device__ __forceinline__ void radix4_inv(double (&x)[4], const double (&w)[3], double q, double qinv) {
#pragma unroll
  for (int s = 1; s >= 0; s--)
#pragma unroll
    for (int p = 0; p < 2; p++) {
      double& X = x[s == 0 ? p : 2 * p];
      double& Y = x[s == 0 ? p + 2 : 2 * p + 1];
      const double D = X - Y;
      X = X + Y;
      Y = fp_mulmod_var(D, s == 0 ? w[0] : w[1 + p], qinv, q);
    }
}
template <bool BIG>
__device__ __forceinline__ void radix4_fwd(u64 (&x)[4], const ulonglong2 (&w)[3], u64 q, u64 q2) {
#pragma unroll
  for (int s = 0; s < 2; s++)
#pragma unroll
    for (int p = 0; p < 2; p++) bf_fwd<BIG>(x[s == 0 ? p : 2 * p], x[s == 0 ? p + 2 : 2 * p + 1], s == 0 ? w[0] : w[1 + p], q, q2, s);
}
// c: bound of the inputs (BIG: 4q, inputs and outputs below 8q). SMALL: outputs below 4c.
template <bool BIG>
__device__ __forceinline__ void radix4_inv(u64 (&x)[4], const ulonglong2 (&w)[3], u64 q, u64 c) {
#pragma unroll
  for (int s = 1; s >= 0; s--) {
#pragma unroll
    for (int p = 0; p < 2; p++) {
      if (s == 0) bf_inv_pair<BIG>(x[p], x[p + 2], w[0], q, c, 2, p);
      else bf_inv<BIG>(x[2 * p], x[2 * p + 1], w[1 + p], q, c);
    }
    if (!BIG) c <<= 1;
  }
}

// ---- a limb of 4096 values in 1024 lanes ----
// Round K (stages 2K, 2K+1) holds, in lane t, the elements (t / S) * 4S + i * S + t % S, S = 1024 >> 2K. From round 2 on a
// wave holds 256 consecutive elements, so only the exchanges between rounds 0, 1 and 2 cross waves. Memory is read and
// written in the layouts of round 0 and of round 2 (64 consecutive elements per wave and register in both).
#define WL_THREADS 1024
#define WL_LDS_WORDS 8192   // two tiles: consecutive workgroup-wide exchanges alternate, which saves a barrier each
__device__ __forceinline__ u32 wl_elem(int K, u32 i) {
  const u32 t = threadIdx.x, s = 10 - 2 * K;
  return ((t >> s) << (s + 2)) + (i << s) + (t & ((1u << s) - 1));
}
// LDS word of element e. The 32 lanes of a half-wave differ in bits 0..4 of e in rounds 0..2, in bits 0..3 and 6 in
// round 3, 0, 1, 4, 5, 6 in round 4 and 2..6 in round 5: folding bit 5 into bits 0 and 2, bit 6 into bits 1, 3 and 4
// spreads each of these sets over all 32 pairs of banks.
__device__ __forceinline__ u32 wl_word(u32 e) { return e ^ (((e >> 5) & 1) * 5) ^ (((e >> 6) & 1) * 26); }
template <int FROM, int TO, class T>
__device__ __forceinline__ void wl_exchange(T (&x)[4], T* sm) {
  constexpr bool in_wave = FROM >= 2 && TO >= 2;
  T* tile = sm + ((FROM == 0 || TO == 0) ? 0 : 4096);
#pragma unroll
  for (int i = 0; i < 4; i++) tile[wl_word(wl_elem(FROM, i))] = x[i];
  if (in_wave) wave_lds_sync();
  else lds_barrier();
#pragma unroll
  for (int i = 0; i < 4; i++) x[i] = tile[wl_word(wl_elem(TO, i))];
  if (in_wave) wave_lds_sync();
}
// Twiddles of round K; rounds 0..2 have the same ones in all lanes of a wave.
template <class TW>
__device__ __forceinline__ void wl_twiddles(TW (&w)[3], const TW* __restrict__ tw, int K) {
  u32 blk = threadIdx.x >> (10 - 2 * K);
  if (K <= 2) {
    blk = __builtin_amdgcn_readfirstlane(blk);
    scalar_fetch(w[0], tw, (1u << (2 * K)) + blk);
    scalar_fetch(w[1], tw, (2u << (2 * K)) + 2 * blk);
    scalar_fetch(w[2], tw, (2u << (2 * K)) + 2 * blk + 1);
    return;
  }
  w[0] = tw[(1u << (2 * K)) + blk];
  w[1] = tw[(2u << (2 * K)) + 2 * blk];
  w[2] = tw[(2u << (2 * K)) + 2 * blk + 1];
}
template <class TW>
struct WlTwiddles {
  TW w[6][3];
  __device__ __forceinline__ void load(const TW* __restrict__ tw) {
#pragma unroll
    for (int K = 0; K < 6; K++) wl_twiddles(w[K], tw, K);
  }
};

// Round-0 layout, |x| <= q  ->  round-2 layout, |x| <= q/2. Six stages between reductions.
__device__ __forceinline__ void wl_fwd(double (&x)[4], const WlTwiddles<double>& w, double q, double qinv, double* sm) {
  radix4_fwd(x, w.w[0], q, qinv);
  wl_exchange<0, 1>(x, sm);
  radix4_fwd(x, w.w[1], q, qinv);
  wl_exchange<1, 2>(x, sm);
  radix4_fwd(x, w.w[2], q, qinv);
  reduce4(x, q, qinv);
  wl_exchange<2, 3>(x, sm);
  radix4_fwd(x, w.w[3], q, qinv);
  wl_exchange<3, 4>(x, sm);
  radix4_fwd(x, w.w[4], q, qinv);
  wl_exchange<4, 5>(x, sm);
  radix4_fwd(x, w.w[5], q, qinv);
  reduce4(x, q, qinv);
  wl_exchange<5, 2>(x, sm);
}
// Round-2 layout, |x| <= q  ->  round-0 layout, times sc, in (-q, q). Two stages to the first reduction, four between others.
__device__ __forceinline__ void wl_inv(double (&x)[4], const WlTwiddles<double>& w, double q, double qinv, double sc, double scq,
                                       double* sm) {
  wl_exchange<2, 5>(x, sm);
  radix4_inv(x, w.w[5], q, qinv);
  reduce4(x, q, qinv);
  wl_exchange<5, 4>(x, sm);
  radix4_inv(x, w.w[4], q, qinv);
  wl_exchange<4, 3>(x, sm);
  radix4_inv(x, w.w[3], q, qinv);
  reduce4(x, q, qinv);
  wl_exchange<3, 2>(x, sm);
  radix4_inv(x, w.w[2], q, qinv);
  wl_exchange<2, 1>(x, sm);
  radix4_inv(x, w.w[1], q, qinv);
  reduce4(x, q, qinv);
  wl_exchange<1, 0>(x, sm);
  radix4_inv(x, w.w[0], q, qinv);
  reduce4(x, q, qinv);
#pragma unroll
  for (int i = 0; i < 4; i++) x[i] = fp_mulmod_const(x[i], sc, scq, q);
}
// Integer classes: canonical in, canonical out.
template <bool BIG>
__device__ __forceinline__ void wl_fwd(u64 (&x)[4], const WlTwiddles<ulonglong2>& w, u64 q, u64 mu, u64* sm) {
  const u64 q2 = lazy_const<BIG>(q);
  radix4_fwd<BIG>(x, w.w[0], q, q2);
  wl_exchange<0, 1>(x, sm);
  radix4_fwd<BIG>(x, w.w[1], q, q2);
  wl_exchange<1, 2>(x, sm);
  radix4_fwd<BIG>(x, w.w[2], q, q2);
  wl_exchange<2, 3>(x, sm);
  radix4_fwd<BIG>(x, w.w[3], q, q2);
  wl_exchange<3, 4>(x, sm);
  radix4_fwd<BIG>(x, w.w[4], q, q2);
  wl_exchange<4, 5>(x, sm);
  radix4_fwd<BIG>(x, w.w[5], q, q2);
#pragma unroll
  for (int i = 0; i < 4; i++) x[i] = csub(fwd_settle<BIG>(x[i], mu, q), q);
  wl_exchange<5, 2>(x, sm);
}
template <bool BIG>
__device__ __forceinline__ void wl_inv(u64 (&x)[4], const WlTwiddles<ulonglong2>& w, u64 q, u64 mu, u64 sc, u64 scs, u64* sm) {
  const u64 q2 = lazy_const<BIG>(q);
  wl_exchange<2, 5>(x, sm);
  radix4_inv<BIG>(x, w.w[5], q, q2);
  wl_exchange<5, 4>(x, sm);
  radix4_inv<BIG>(x, w.w[4], q, BIG ? q2 : q2 << 2);
  wl_exchange<4, 3>(x, sm);
  radix4_inv<BIG>(x, w.w[3], q, BIG ? q2 : q2 << 4);
  wl_exchange<3, 2>(x, sm);
  radix4_inv<BIG>(x, w.w[2], q, BIG ? q2 : q2 << 6);
  if (!BIG) {   // eight stages of doubling sums: back below 2q
#pragma unroll
    for (int i = 0; i < 4; i++) x[i] = barrett_lazy(x[i], mu, q);
  }
  wl_exchange<2, 1>(x, sm);
  radix4_inv<BIG>(x, w.w[1], q, q2);
  wl_exchange<1, 0>(x, sm);
  radix4_inv<BIG>(x, w.w[0], q, BIG ? q2 : q2 << 2);
#pragma unroll
  for (int i = 0; i < 4; i++) x[i] = shoup(x[i], sc, scs, q);
}
