// Single-pass negacyclic NTT for N = 2^10 .. 2^14 on gfx950: one workgroup holds a whole limb, 16 residues in each of N / 16
// lanes, and takes it through all stages; the limb is read and written once. Rounds of radix 16 in registers, what is left of
// log2 N (LAST = 0 .. 3 stages) in a last round on 16 >> LAST groups of 2^LAST adjacent elements, exchanges through LDS between
// them. Same butterflies, lazy ranges and modulus classes as the two-pass bodies (ntt16.hip.h, ntt16fp.hip.h): double precision
// for q < 2^50, uncorrected integer butterflies for q < 2^52, Harvey butterflies for q < 2^60.
//
// Layouts. Round k < F (stages 4k .. 4k + 3, s = log2 N - 4 (k + 1)): lane t holds elements (t >> s) << (s + 4) | i << s | t mod 2^s.
// From round 1 on a wave holds 1024 consecutive elements, so only the exchange between rounds 0 and 1 crosses waves. Last round:
// lane l of a wave holds, in register g << LAST | c, element ((64 g + l) << LAST) + c of the wave's 1024; memory is touched in the
// layout of round 0 and in the same layout for LAST = 0 (64 consecutive elements per register), or for LAST = 1 (128
// consecutive elements per pair of registers).
// LDS word of element e: 2^LAST words of padding after every 2^(LAST + 4) keep the 32 lanes of an access on different banks in the
// rounds of radix 16.
//
// What bounds it: at a few hundred limbs the latency of a lone workgroup, at thousands memory (one read and one write of a limb,
// where the two-pass kernels take two of each and a launch per pass and arithmetic kind). 37 polynomials of 4 limbs at 2^13, both
// ways: 51.4 -> 27.7 us. Other numbers of values a lane were not built. At 128 registers (4 waves per SIMD; 1024 lanes at 2^14 take
// no more) four integer bodies spill: 14 registers in the inverse of 2^14, 2 or 3 in its forward and the inverses of 2^10 and 2^11.
#pragma once
#include "ntt16fp.hip.h"

template <int LOGN>
struct Limb {
  static constexpr int F = LOGN >= 12 ? 3 : 2, LAST = LOGN - 4 * F, THREADS = 1 << (LOGN - 4), GROUPS = 16 >> LAST;
  static constexpr int WORDS = (1 << LOGN) + (1 << (LOGN - 4));
  static constexpr int COALESCED = F + 1;   // layout index; F: the last round
  static __device__ __forceinline__ u32 stride(int k) { return LOGN - 4 * (k + 1); }
  static __device__ __forceinline__ constexpr u32 word(u32 e) { return e + ((e >> (LAST + 4)) << LAST); }
  // element of register r (the lane's part, and what r adds: both to the element and, by word(), to the LDS word)
  static __device__ __forceinline__ u32 base(int k) {
    const u32 t = threadIdx.x, s = stride(k);
    if (k < F) return ((t >> s) << (s + 4)) + (t & ((1u << s) - 1));
    return (t >> 6) * 1024 + ((t & 63) << (k == F ? LAST : 0));
  }
  static __device__ __forceinline__ constexpr u32 step(int k, u32 r) {
    return k < F ? r << (LOGN - 4 * (k + 1)) : k == F ? ((r >> LAST) << (6 + LAST)) + (r & ((1u << LAST) - 1)) : r * 64;
  }
  static __device__ __forceinline__ u32 elem(int k, u32 r) { return base(k) + step(k, r); }
};
template <int LOGN, int FROM, int TO, class T>
__device__ __forceinline__ void limb_exchange(T (&x)[16], T* sm) {
  typedef Limb<LOGN> L;
  constexpr bool in_wave = FROM != 0 && TO != 0;
  const u32 from = L::word(L::base(FROM)), to = L::word(L::base(TO));
#pragma unroll
  for (int r = 0; r < 16; r++) sm[from + L::word(L::step(FROM, r))] = x[r];
  if (in_wave) wave_lds_sync();
  else lds_barrier();
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = sm[to + L::word(L::step(TO, r))];
  if (in_wave) wave_lds_sync();
}
// Twiddles of round k, stage s: 2^s from here on.
template <int LOGN, class TW>
__device__ __forceinline__ const TW* limb_stage(const TW* __restrict__ tw, int k, int s) {
  return tw + (1u << (4 * k + s)) + ((threadIdx.x >> Limb<LOGN>::stride(k)) << s);
}
template <int LOGN>
__device__ __forceinline__ void limb_twiddles(double (&w)[15], const double* __restrict__ tw, int k) {
#pragma unroll
  for (int s = 0; s < 4; s++) {
    const double* p = limb_stage<LOGN>(tw, k, s);
#pragma unroll
    for (int g = 0; g < (1 << s); g++) w[NTT16_TW_INDEX(s, g)] = p[g];
  }
}
// The last round: f(register of X, of Y, twiddle, stage, distance, pair) for each butterfly of its stages. All its twiddles are
// requested together.
template <int LOGN, int S, class TW, class BF>
__device__ __forceinline__ void limb_last_stage(const TW (&w)[16], BF& f) {
  typedef Limb<LOGN> L;
  constexpr int half = (1 << L::LAST) >> (S + 1), per = (1 << L::LAST) - 1;
#pragma unroll
  for (int g = 0; g < L::GROUPS; g++)
#pragma unroll
    for (int c = 0; c < (1 << S); c++)
#pragma unroll
      for (int p = 0; p < half; p++) {
        const int X = (g << L::LAST) + c * 2 * half + p;
        f(X, X + half, w[g * per + (1 << S) - 1 + c], S, half, p);
      }
}
template <int LOGN, bool INV, class TW, class BF>
__device__ __forceinline__ void limb_last(const TW* __restrict__ tw, BF f) {
  typedef Limb<LOGN> L;
  constexpr int per = (1 << L::LAST) - 1;   // twiddles of a group
  if constexpr (L::LAST > 0) {
    const u32 block = (threadIdx.x >> 6) * (1024u >> L::LAST) + (threadIdx.x & 63);
    TW w[16];
#pragma unroll
    for (int g = 0; g < L::GROUPS; g++)
#pragma unroll
      for (int k = 0; k < per; k++) {
        const int s = k >= 3 ? 2 : k >= 1 ? 1 : 0;
        w[g * per + k] = tw[(1u << (LOGN - L::LAST + s)) + ((block + 64 * g) << s) + (k + 1 - (1 << s))];
      }
    if constexpr (!INV) limb_last_stage<LOGN, 0>(w, f);
    if constexpr (L::LAST > 1 && !INV) limb_last_stage<LOGN, 1>(w, f);
    if constexpr (L::LAST > 2) limb_last_stage<LOGN, 2>(w, f);
    if constexpr (L::LAST > 1 && INV) limb_last_stage<LOGN, 1>(w, f);
    if constexpr (INV) limb_last_stage<LOGN, 0>(w, f);
  }
}
// Between memory and the layout next to the last round (with all 16 lanes' rows for LAST >= 2 gathered through LDS). Words of
// LAST = 1 go in pairs, which need the alignment of one word only.
typedef u64 limb_pair __attribute__((ext_vector_type(2), aligned(8)));
template <int LOGN>
__device__ __forceinline__ void limb_store(u64* __restrict__ dst, const u64 (&x)[16]) {
  typedef Limb<LOGN> L;
  if (L::LAST == 1) {
#pragma unroll
    for (int g = 0; g < 8; g++) *(limb_pair*)(dst + L::elem(L::F, 2 * g)) = limb_pair{x[2 * g], x[2 * g + 1]};
  } else {
#pragma unroll
    for (int r = 0; r < 16; r++) dst[L::elem(L::COALESCED, r)] = x[r];
  }
}
template <int LOGN>
__device__ __forceinline__ void limb_load(u64 (&x)[16], const u64* __restrict__ src) {
  typedef Limb<LOGN> L;
  if (L::LAST == 1) {
#pragma unroll
    for (int g = 0; g < 8; g++) {
      const limb_pair v = *(const limb_pair*)(src + L::elem(L::F, 2 * g));
      x[2 * g] = v.x;
      x[2 * g + 1] = v.y;
    }
  } else {
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = src[L::elem(L::COALESCED, r)];
  }
}

// ---- double precision: canonical in, canonical out ----
template <int LOGN>
__device__ __forceinline__ void limb_fwd(const u64* __restrict__ src, u64* __restrict__ dst, const double* __restrict__ tw, double q,
                                         double qinv, double* sm) {
  typedef Limb<LOGN> L;
  double x[16], wa[15], wb[15];
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = u2d(src[L::elem(0, r)]);
  limb_twiddles<LOGN>(wa, tw, 1);
  radix16_fwd_fp(x, q, qinv, [&](int s, int g) { return tw[(1 << s) + g]; });
  limb_exchange<LOGN, 0, 1>(x, sm);
  radix16_fwd_fp(x, q, qinv, [&](int s, int g) { return wa[NTT16_TW_INDEX(s, g)]; });
  if (L::F == 3) {
    // Only now: lanes read them 64 bytes apart, the most lines of any request here, and where two workgroups share a compute unit they
    // would be in the way of its data (2^12, forward, with the ending below: 300 limbs 9.57 -> 9.19 us, 600 12.8 -> 12.2).
    __builtin_amdgcn_sched_barrier(0);
    limb_twiddles<LOGN>(wb, tw, 2);
    __builtin_amdgcn_sched_barrier(0);
    limb_exchange<LOGN, 1, L::F - 1>(x, sm);
    radix16_fwd_fp(x, q, qinv, [&](int s, int g) { return wb[NTT16_TW_INDEX(s, g)]; });
  }
  if (L::LAST == 0) {   // the residues leave as they are read back
    const u32 from = L::word(L::base(L::F - 1)), to = L::word(L::base(L::F));
#pragma unroll
    for (int r = 0; r < 16; r++) sm[from + L::word(L::step(L::F - 1, r))] = x[r];
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 16; r++) dst[L::elem(L::F, r)] = d2u_canon(sm[to + L::word(L::step(L::F, r))], q);
    return;
  }
  limb_exchange<LOGN, L::F - 1, L::F>(x, sm);
  limb_last<LOGN, false>(tw, [&](int X, int Y, double w, int, int, int) {
    const double T = fp_mulmod_var(x[Y], w, qinv, q);
    x[Y] = x[X] - T;
    x[X] = x[X] + T;
  });
  if (L::LAST) {
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = fp_reduce(x[r], qinv, q);
  }
  if (L::LAST > 1) limb_exchange<LOGN, L::F, L::COALESCED>(x, sm);
  u64 y[16];
#pragma unroll
  for (int r = 0; r < 16; r++) y[r] = d2u_canon(x[r], q);
  limb_store<LOGN>(dst, y);
}
template <int LOGN>
__device__ __forceinline__ void limb_inv(const u64* __restrict__ src, u64* __restrict__ dst, const double* __restrict__ twi, double q,
                                         double qinv, double sc, double scq, double* sm) {
  typedef Limb<LOGN> L;
  double x[16], wa[15], wb[15];
  u64 y[16];
  limb_load<LOGN>(y, src);
  if (L::F == 3) limb_twiddles<LOGN>(wb, twi, 2);
  limb_twiddles<LOGN>(wa, twi, 1);
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = u2d(y[r]);
  if (L::LAST > 1) limb_exchange<LOGN, L::COALESCED, L::F>(x, sm);
  limb_last<LOGN, true>(twi, [&](int X, int Y, double w, int, int, int) {   // from residues: sums of at most 8
    const double D = x[X] - x[Y];
    x[X] = x[X] + x[Y];
    x[Y] = fp_mulmod_var(D, w, qinv, q);
  });
  if (L::LAST) {
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = fp_reduce(x[r], qinv, q);
  }
  limb_exchange<LOGN, L::F, L::F - 1>(x, sm);
  if (L::F == 3) {
    radix16_inv_fp(x, q, qinv, [&](int s, int g) { return wb[NTT16_TW_INDEX(s, g)]; });
    limb_exchange<LOGN, L::F - 1, 1>(x, sm);
  }
  radix16_inv_fp(x, q, qinv, [&](int s, int g) { return wa[NTT16_TW_INDEX(s, g)]; });
  limb_exchange<LOGN, 1, 0>(x, sm);
  radix16_inv_fp(x, q, qinv, [&](int s, int g) { return twi[(1 << s) + g]; });
#pragma unroll
  for (int r = 0; r < 16; r++) dst[L::elem(0, r)] = d2u_canon(fp_mulmod_const(x[r], sc, scq, q), q);
}

// ---- integer classes: canonical in, canonical out. A round's twiddle pairs (60 registers) take over those of the round before
// stage by stage, as in the two-pass block bodies. ----
template <bool BIG, int LOGN>
__device__ __forceinline__ void limb_fwd(const u64* __restrict__ src, u64* __restrict__ dst, const ulonglong2* __restrict__ tw, u64 q,
                                         u64 mu, u64* sm) {
  typedef Limb<LOGN> L;
  const u64 q2 = lazy_const<BIG>(q);
  u64 x[16];
  ulonglong2 wa[15], wb[15];
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = src[L::elem(0, r)];
#pragma unroll
  for (int s = 0; s < 3; s++) ntt16_load_stage(wa, limb_stage<LOGN>(tw, 1, s), s);
  __builtin_amdgcn_sched_barrier(0);
  radix16_fwd<BIG>(x, q, q2, [&](int s, int g) { return tw[(1 << s) + g]; });
  __builtin_amdgcn_sched_barrier(0);
  ntt16_load_stage(wa, limb_stage<LOGN>(tw, 1, 3), 3);
  limb_exchange<LOGN, 0, 1>(x, sm);
  radix16_fwd_staged<BIG>(
      x, q, q2, [&](int s, int g) { return wa[NTT16_TW_INDEX(s, g)]; },
      [&](int s) {
        if (L::F == 2) return;
        __builtin_amdgcn_sched_barrier(0);
        ntt16_load_stage(wb, limb_stage<LOGN>(tw, 2, s), s);
        __builtin_amdgcn_sched_barrier(0);
      });
  if (L::F == 3) {
    limb_exchange<LOGN, 1, L::F - 1>(x, sm);
    radix16_fwd<BIG>(x, q, q2, [&](int s, int g) { return wb[NTT16_TW_INDEX(s, g)]; });
  }
  __builtin_amdgcn_sched_barrier(0);
  limb_exchange<LOGN, L::F - 1, L::F>(x, sm);
  limb_last<LOGN, false>(tw, [&](int X, int Y, ulonglong2 w, int s, int, int) { bf_fwd<BIG>(x[X], x[Y], w, q, q2, s); });
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = csub(fwd_settle<BIG>(x[r], mu, q), q);
  if (L::LAST > 1) limb_exchange<LOGN, L::F, L::COALESCED>(x, sm);
  limb_store<LOGN>(dst, x);
}
template <bool BIG, int LOGN>
__device__ __forceinline__ void limb_inv(const u64* __restrict__ src, u64* __restrict__ dst, const ulonglong2* __restrict__ twi, u64 q,
                                         u64 mu, u64 sc, u64 scs, u64* sm) {
  typedef Limb<LOGN> L;
  const u64 q2 = lazy_const<BIG>(q);
  u64 x[16];
  ulonglong2 wa[15], wb[15];
  limb_load<LOGN>(x, src);
  if (L::LAST > 1) limb_exchange<LOGN, L::COALESCED, L::F>(x, sm);
  limb_last<LOGN, true>(twi, [&](int X, int Y, ulonglong2 w, int s, int half, int p) {   // SMALL: sums of at most 8 residues
    bf_inv_pair<BIG>(x[X], x[Y], w, q, BIG ? q2 : q2 << (L::LAST - 1 - s), half, p);
  });
  if (!BIG && L::LAST) {
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = barrett_lazy(x[r], mu, q);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 3; s >= 0; s--) ntt16_load_stage(wb, limb_stage<LOGN>(twi, L::F - 1, s), s);
  __builtin_amdgcn_sched_barrier(0);
  limb_exchange<LOGN, L::F, L::F - 1>(x, sm);
  radix16_inv_staged<BIG>(
      x, q, q2, [&](int s, int g) { return wb[NTT16_TW_INDEX(s, g)]; },
      [&](int s) {
        if (L::F == 2) return;
        __builtin_amdgcn_sched_barrier(0);
        ntt16_load_stage(wa, limb_stage<LOGN>(twi, 1, s), s);
        __builtin_amdgcn_sched_barrier(0);
      });
  if (L::F == 3) {
    limb_exchange<LOGN, L::F - 1, 1>(x, sm);
    radix16_inv<BIG>(x, q, BIG ? q2 : q2 << 4, [&](int s, int g) { return wa[NTT16_TW_INDEX(s, g)]; });
  }
  if (!BIG) {   // four or eight stages of doubling sums: back below 2q before the last four
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = barrett_lazy(x[r], mu, q);
  }
  limb_exchange<LOGN, 1, 0>(x, sm);
  radix16_inv<BIG>(x, q, q2, [&](int s, int g) { return twi[(1 << s) + g]; });
#pragma unroll
  for (int r = 0; r < 16; r++) dst[L::elem(0, r)] = shoup(x[r], sc, scs, q);
}

// grid = (polynomials, limb slots). Slot `s` of polynomial `p` is at + p * poly_stride + s * N in src and dst (src == dst
// transforms in place: every lane has read its words before any lane writes, across the barrier).
struct LimbArgs {
  const u64* src;
  u64* dst;
  const ulonglong2* tw;     // integer table (forward or inverse), [nm][N]
  const double* twfp;       // double table, same indexing (rows of moduli >= 2^50 unused)
  const ModInfo* mods;
  u64 src_poly_stride, dst_poly_stride;
  u32 skip_beta, skip_alpha, skip_nq;   // digit p % skip_beta leaves its own limbs alone (ModUp'ed digits)
  u32 fp_on;                            // 0: integer bodies for every modulus
  unsigned char id[128];                // slot -> modulus id
};

// Both arithmetic kinds share a launch (the kind is uniform per workgroup). 4 waves per SIMD: what the LDS leaves at 2^13, what
// 1024 lanes need at 2^14, and without which the inverses of 2^10 and 2^11 take 132 registers (2000 limbs of 2^11 16.3 -> 18.8 us).
// Left to itself 2^12 takes 123 and is faster (300 limbs: 50-bit inverses 10.05 -> 9.52 us, 60-bit forward 13.0 -> 12.6).
template <int LOGN, bool INV>
__global__ void __launch_bounds__(Limb<LOGN>::THREADS) __attribute__((amdgpu_waves_per_eu(LOGN == 12 ? 1 : 4))) ntt_limb_kernel(LimbArgs a) {
  __shared__ __attribute__((aligned(16))) u64 sm[Limb<LOGN>::WORDS];
  const u32 poly = blockIdx.x, slot = blockIdx.y;
  if (a.skip_beta) {
    const u32 j = poly % a.skip_beta, lo = j * a.skip_alpha, hi = min(lo + a.skip_alpha, a.skip_nq);
    if (slot >= lo && slot < hi) return;
  }
  const u32 id = a.id[slot];
  const ModInfo mi = a.mods[id];
  const u64* src = a.src + (size_t)poly * a.src_poly_stride + ((size_t)slot << LOGN);
  u64* dst = a.dst + (size_t)poly * a.dst_poly_stride + ((size_t)slot << LOGN);
  const ulonglong2* tw = a.tw + ((size_t)id << LOGN);
  const int cls = mod_class(mi.m, a.fp_on);   // uniform per workgroup
  if (cls == 0) {
    const double* twfp = a.twfp + ((size_t)id << LOGN);
    if (INV) limb_inv<LOGN>(src, dst, twfp, mi.qd, mi.qinv, mi.ninvd, mi.ninvq, (double*)sm);
    else limb_fwd<LOGN>(src, dst, twfp, mi.qd, mi.qinv, (double*)sm);
  } else if (cls == 2) {
    if (INV) limb_inv<true, LOGN>(src, dst, tw, mi.m, mi.mu64, mi.ninv, mi.ninvs, sm);
    else limb_fwd<true, LOGN>(src, dst, tw, mi.m, mi.mu64, sm);
  } else {
    if (INV) limb_inv<false, LOGN>(src, dst, tw, mi.m, mi.mu64, mi.ninv, mi.ninvs, sm);
    else limb_fwd<false, LOGN>(src, dst, tw, mi.m, mi.mu64, sm);
  }
}
