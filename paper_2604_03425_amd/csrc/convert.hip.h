// Base conversion fused with the transform passes on both sides of it (ModUp and ModDown, N = 2^13 .. 2^16, at most 8
// source limbs): second inverse pass of the sources, conversion, first forward pass of every target. Only the sources are
// read and only the targets, after their row pass, are written; as separate kernels the same step moved the sources three
// times more and the targets two times more. Where several workgroups share the targets of a tile, the inverse pass may be a
// kernel of its own before this one (READY, chosen in conv_plan).
//
// A conversion needs all sources of a position in one lane and a row pass all rows of a column in one workgroup. A workgroup
// of 512 lanes takes R rows x NC = 2048 / R columns, four positions per lane, and keeps the converted form of all sources
// (8 x 4 words = 64 registers) there while it walks over the targets (integer sources that are transformed here: a quarter
// of the words in scratch memory, stored once and reloaded once per target list; the compiler does not promote them). Four positions per lane is what makes the sources fit
// beside a transform at 4 waves per SIMD; the row pass is then radix-4 rounds with up to three exchanges through LDS (two
// of them across waves), whose two tiles alternate so that an exchange costs one barrier. Two workgroups share a compute
// unit, so one computes while the other waits.
//
// Element e = row * NC + column of the tile; round K (stages 2K, 2K+1) holds, in lane t, the elements
// (t >> s) << (s + 2) | i << s | (t mod 2^s), s = 9 - 2K: the linear layout of a radix-4 transform of 2048 values of which
// only the first LOGR stages are done. The last round has s = 11 - LOGR, a lane then holds four adjacent rows of a column;
// for odd LOGR only the second of its two stages is left to do.
//
// What bounds it: instruction issue (0.62 of the vector peak by executed instructions at 2.3 TB/s). Per target and position the conversion
// of 8 double-precision sources costs 38 FP64 instructions (see convert_fp), its row pass 35; an integer target about
// twice that. N = 2^16, 64 ciphertexts of 24 limbs, 3 digits of 8, 8 special primes: inverse row pass, ModUp and row passes as
// four kernels 2030 us, here 1476 (1551 with canonical results of the integer sums, 9 instructions at the end of a
// double-precision one and two reductions a row pass); the same for ModDown's three 1440 and 1090 (1148). One such ciphertext: 62 ->
// 46 and 49 -> 34 us.
#pragma once
#include "radix4.hip.h"
#include "ntt16_kernels.hip.h"

#include <cstddef>
#include <type_traits>
#include <utility>

#define CONV_THREADS 512
#define CONV_TILE 2048
#define CONV_MAX_SRC 8

struct ConvArgs {
  const u64* src;            // sources after the inverse block pass (reduced doubles / lazy integers, by class)
  u64* dst;                  // targets after the row pass
  u64 src_poly_stride;       // elements between the source rows of consecutive (p / beta)
  u64 dst_poly_stride;       // elements between consecutive destination polynomials p
  u32 src_slot0, src_id0;    // limb index inside a source row, and modulus id, of the first source of digit 0
  u32 src_nlimbs, alpha, beta;  // digit j = p % beta owns sources j*alpha .. j*alpha + len - 1
  u32 skip_own;              // != 0: target slots j*alpha .. j*alpha + len - 1 are the digit's own limbs: left alone
  u32 ntarget;               // targets of a digit in the constant tables
  u32 nfp, nint;             // targets by arithmetic kind: tslot[0 .. nfp), tslot[nfp .. nfp + nint)
  u32 nsplit;                // workgroups that share the targets of a (polynomial, tile)
  u32 pitch;                 // constants per target in mat
  // integer conversion: [beta][ntarget][pitch] constants (C/c_k) mod m_t and [beta][ntarget] the offset of the shifted sources,
  // scaled by 2^60 under NARROW (by 2^64 otherwise): LevelTables::up_conv, dn_conv and their _off, not up_mat, dn_mat_plain
  const u64 *mat, *off;
  const double* matd;        // [beta][ntarget][pitch - 1] centred constants (double-precision sources and targets)
  const ulonglong2* scale;   // [src_nlimbs] per source (Q_j/q_i)^-1 / N, in the form of its class
  const ulonglong2 *tw, *twi;
  const double *twfp, *twifp;
  const ModInfo* mods;
  u32 target[128];           // list index -> target slot | modulus id << 8
};

// a value that is the same in all lanes, said so: what is derived from it then stays in scalar registers
__device__ __forceinline__ u32 conv_uniform(u32 v) { return __builtin_amdgcn_readfirstlane(v); }

// Tables read at wave-uniform places go through the constant address space: between the barriers and stores of the target
// loop the compiler would otherwise not use scalar loads for them.
typedef const __attribute__((address_space(4))) u64* const_u64_ptr;
__device__ __forceinline__ const_u64_ptr conv_const(const void* p) { return (const_u64_ptr)p; }
__device__ __forceinline__ double conv_const_double(const_u64_ptr p) { return __longlong_as_double((long long)*p); }
__device__ __forceinline__ ModInfo conv_mod(const ModInfo* mods, u32 id) {
  const_u64_ptr p = conv_const(mods + id);
  ModInfo m = {};
#define CONV_WORD(FIELD) p[offsetof(ModInfo, FIELD) / 8]
  m.m = CONV_WORD(m);
  m.minv = CONV_WORD(minv);
  m.qd = __longlong_as_double((long long)CONV_WORD(qd));
  m.qinv = __longlong_as_double((long long)CONV_WORD(qinv));
#undef CONV_WORD
  return m;
}
__device__ __forceinline__ void conv_fetch(double& w, const double* tw, u32 i) { w = conv_const_double(conv_const(tw) + i); }
__device__ __forceinline__ void conv_fetch(ulonglong2& w, const ulonglong2* tw, u32 i) {
  const_u64_ptr p = conv_const(tw) + 2 * (size_t)i;
  w = ulonglong2{p[0], p[1]};
}

// ---- layouts ----
__device__ __forceinline__ u32 conv_elem(int s, u32 i) {
  const u32 t = threadIdx.x;
  return ((t >> s) << (s + 2)) + (i << s) + (t & ((1u << s) - 1));
}
// LDS word of element e: 8 words of padding after every 32. The lanes of a half-wave are 32 consecutive elements (s >= 5), two
// runs of 16 64 apart (s = 4) or four runs of 8 32 apart (s = 3): no bank is met twice, and a lane's four words are at
// constant distances in every layout.
#define CONV_TILE_WORDS (CONV_TILE / 4 * 5)
__device__ __forceinline__ u32 conv_word(int s, u32 i) {
  const u32 e0 = conv_elem(s, 0), step = (i << s) + 8 * ((i << s) >> 5);   // (i << s) carries into e0 >> 5 for no i
  return e0 + 8 * (e0 >> 5) + step;
}
template <int FROM, int TO, class T>
__device__ __forceinline__ void conv_exchange(T (&x)[4], T* sm) {
  constexpr bool in_wave = FROM <= 6 && TO <= 6;   // both layouts give a wave 256 consecutive elements
  T* tile = sm + ((FROM == 9 || TO == 9) ? 0 : CONV_TILE_WORDS);
#pragma unroll
  for (int i = 0; i < 4; i++) tile[conv_word(FROM, i)] = x[i];
  if (in_wave) wave_lds_sync();
  else lds_barrier();
#pragma unroll
  for (int i = 0; i < 4; i++) x[i] = tile[conv_word(TO, i)];
  if (in_wave) wave_lds_sync();
}
// Twiddles of the round with stride 2^s whose first stage is stage 2K: rounds 0 and 1 have the same in a whole wave.
template <class TW>
__device__ __forceinline__ void conv_twiddles(TW (&w)[3], const TW* __restrict__ tw, int K) {
  const int s = 9 - 2 * K;
  u32 blk = threadIdx.x >> s;
  if (s >= 6) {
    blk = conv_uniform(blk);
    conv_fetch(w[0], tw, (1u << (2 * K)) + blk);
    conv_fetch(w[1], tw, (2u << (2 * K)) + 2 * blk);
    conv_fetch(w[2], tw, (2u << (2 * K)) + 2 * blk + 1);
    return;
  }
  w[0] = tw[(1u << (2 * K)) + blk];
  w[1] = tw[(2u << (2 * K)) + 2 * blk];
  w[2] = tw[(2u << (2 * K)) + 2 * blk + 1];
}
// The lone last stage of odd LOGR: pairs (0,1) and (2,3).
template <int LOGR, class TW>
__device__ __forceinline__ void conv_twiddles_last(TW (&w)[2], const TW* __restrict__ tw) {
  u32 blk = threadIdx.x >> (11 - LOGR);
  if (11 - LOGR >= 6) {
    blk = conv_uniform(blk);
    conv_fetch(w[0], tw, (1u << (LOGR - 1)) + 2 * blk);
    conv_fetch(w[1], tw, (1u << (LOGR - 1)) + 2 * blk + 1);
    return;
  }
  w[0] = tw[(1u << (LOGR - 1)) + 2 * blk];
  w[1] = tw[(1u << (LOGR - 1)) + 2 * blk + 1];
}

// ---- double precision: forward and inverse row passes ----
// A forward pass gets its first rounds' twiddles (ConvTwiddles) from the caller, who requests them ahead of the conversion;
// the later ones' are requested as the registers for them become free. In: |x| <= 1.5 q. Out: at most 2.64 q (three stages
// from a reduced value), which the block passes take: one reduction, after four or five stages.
template <class TW>
struct ConvTwiddles {
  TW w0[3], w1[3];
  __device__ __forceinline__ void load(const TW* __restrict__ tw) {
    conv_twiddles(w0, tw, 0);
    conv_twiddles(w1, tw, 1);
  }
};
template <int LOGR>
__device__ __forceinline__ void conv_fwd_rows(double (&x)[4], const ConvTwiddles<double>& w, const double* __restrict__ tw,
                                              double q, double qinv, double* sm) {
  constexpr int L = 11 - LOGR;
  double w2[3], w3[3], wl[2];
  if (LOGR >= 6) conv_twiddles(w2, tw, 2);
  radix4_fwd(x, w.w0, q, qinv);
  conv_exchange<9, 7>(x, sm);
  if (LOGR == 8) conv_twiddles(w3, tw, 3);
  if (LOGR & 1) conv_twiddles_last<LOGR>(wl, tw);
  radix4_fwd(x, w.w1, q, qinv);
  if (LOGR < 8) reduce4(x, q, qinv);
  if (LOGR >= 6) {
    conv_exchange<7, 5>(x, sm);
    radix4_fwd<LOGR == 8>(x, w2, q, qinv);
  }
  if (LOGR != 6) conv_exchange<(LOGR >= 6 ? 5 : 7), L>(x, sm);
  if (LOGR == 8) radix4_fwd(x, w3, q, qinv);
  if (LOGR & 1) {
#pragma unroll
    for (int p = 0; p < 2; p++) {
      const double T = fp_mulmod_var(x[2 * p + 1], wl[p], qinv, q);
      x[2 * p + 1] = x[2 * p] - T;
      x[2 * p] = x[2 * p] + T;
    }
  }
}
// In and out: |x| <= q/2; at most four stages between reductions.
template <int LOGR>
__device__ __forceinline__ void conv_inv_rows(double (&x)[4], const double* __restrict__ twi, double q, double qinv, double* sm) {
  constexpr int L = 11 - LOGR;
  double w0[3], w1[3], w2[3], w3[3], wl[2];
  if (LOGR & 1) conv_twiddles_last<LOGR>(wl, twi);
  if (LOGR == 8) conv_twiddles(w3, twi, 3);
  if (LOGR >= 6) conv_twiddles(w2, twi, 2);
  conv_twiddles(w1, twi, 1);
  conv_twiddles(w0, twi, 0);
  if (LOGR & 1) {
#pragma unroll
    for (int p = 0; p < 2; p++) {
      const double D = x[2 * p] - x[2 * p + 1];
      x[2 * p] = x[2 * p] + x[2 * p + 1];
      x[2 * p + 1] = fp_mulmod_var(D, wl[p], qinv, q);
    }
  }
  if (LOGR == 8) radix4_inv(x, w3, q, qinv);
  if (LOGR != 6) conv_exchange<L, (LOGR >= 6 ? 5 : 7)>(x, sm);
  if (LOGR >= 6) {
    radix4_inv(x, w2, q, qinv);
    if (LOGR >= 7) reduce4(x, q, qinv);
    conv_exchange<5, 7>(x, sm);
  }
  radix4_inv(x, w1, q, qinv);
  if (LOGR <= 6) reduce4(x, q, qinv);
  conv_exchange<7, 9>(x, sm);
  radix4_inv(x, w0, q, qinv);
  reduce4(x, q, qinv);
}
// ---- integer classes, Harvey's ranges for every prime below 2^60: [0,16q) forward, [0,8q) inverse ----
template <int LOGR>
__device__ __forceinline__ void conv_fwd_rows(u64 (&x)[4], const ConvTwiddles<ulonglong2>& w,
                                              const ulonglong2* __restrict__ tw, u64 q, u64* sm) {
  constexpr int L = 11 - LOGR;
  const u64 q2 = lazy_const<true>(q);
  ulonglong2 w2[3], w3[3], wl[2];
  radix4_fwd<true>(x, w.w0, q, q2);
  conv_exchange<9, 7>(x, sm);
  if (LOGR >= 6) conv_twiddles(w2, tw, 2);
  radix4_fwd<true>(x, w.w1, q, q2);
  if (LOGR & 1) conv_twiddles_last<LOGR>(wl, tw);
  if (LOGR >= 6) {
    conv_exchange<7, 5>(x, sm);
    if (LOGR == 8) conv_twiddles(w3, tw, 3);
    radix4_fwd<true>(x, w2, q, q2);
  }
  if (LOGR != 6) conv_exchange<(LOGR >= 6 ? 5 : 7), L>(x, sm);
  if (LOGR == 8) radix4_fwd<true>(x, w3, q, q2);
  if (LOGR & 1) {
#pragma unroll
    for (int p = 0; p < 2; p++) bf_fwd<true, true>(x[2 * p], x[2 * p + 1], wl[p], q, q2);
  }
}
template <int LOGR>
__device__ __forceinline__ void conv_inv_rows(u64 (&x)[4], const ulonglong2* __restrict__ twi, u64 q, u64* sm) {
  constexpr int L = 11 - LOGR;
  const u64 q2 = lazy_const<true>(q);
  ulonglong2 w0[3], w1[3], w2[3], w3[3], wl[2];
  if (LOGR & 1) conv_twiddles_last<LOGR>(wl, twi);
  if (LOGR == 8) conv_twiddles(w3, twi, 3);
  conv_twiddles(w1, twi, 1);
  conv_twiddles(w0, twi, 0);
  if (LOGR & 1) {
#pragma unroll
    for (int p = 0; p < 2; p++) bf_inv<true>(x[2 * p], x[2 * p + 1], wl[p], q, q2);
  }
  if (LOGR == 8) radix4_inv<true>(x, w3, q, q2);
  if (LOGR >= 6) conv_twiddles(w2, twi, 2);
  if (LOGR != 6) conv_exchange<L, (LOGR >= 6 ? 5 : 7)>(x, sm);
  if (LOGR >= 6) {
    radix4_inv<true>(x, w2, q, q2);
    conv_exchange<5, 7>(x, sm);
  }
  radix4_inv<true>(x, w1, q, q2);
  conv_exchange<7, 9>(x, sm);
  radix4_inv<true>(x, w0, q, q2);
}

// ---- conversions at the lane's four positions ----
// What is uniform about a target: its modulus and row of constants (zero beyond the digit's length). Fetched one target
// ahead, its place in the list two ahead, so that no target starts by waiting for a chain of scalar loads.
template <int MAXLEN>
struct ConvTarget {
  u32 slot, id;
  u64 m, minv, off, c[MAXLEN];
  double qd, qinv;
  template <bool CHAIN>   // the constants of convert_fp
  __device__ __forceinline__ void fetch(const ConvArgs& a, u32 target, u32 j) {
    slot = target & 255;
    id = target >> 8;
    const ModInfo mi = conv_mod(a.mods, id);
    m = mi.m, minv = mi.minv, qd = mi.qd, qinv = mi.qinv;
    const size_t row = (size_t)j * a.ntarget + slot;
    const_u64_ptr p = CHAIN ? conv_const(a.matd + row * (a.pitch - 1)) : conv_const(a.mat + row * a.pitch);
#pragma unroll
    for (int k = 0; k < MAXLEN; k++) c[k] = p[k];
    off = CHAIN ? 0 : *conv_const(a.off + row);
  }
};
// A source at one position: the centred double, or the 30-bit halves of (y + (q-1)/2) mod q that the integer conversion
// reads; zero beyond the digit's length.
struct ConvWord {
  u32 lo, hi;
  __device__ __forceinline__ void set(double v) { lo = (u32)__double2loint(v), hi = (u32)__double2hiint(v); }
  __device__ __forceinline__ double value() const { return __hiloint2double((int)hi, (int)lo); }
  __device__ __forceinline__ void split(u64 v) { lo = (u32)v & BCONV_M30, hi = (u32)(v >> 30); }
};
// acc += y * c for a constant c that is the same in all lanes. As an instruction: written as a 64-bit product the widened y
// is hoisted out of the target loop, which doubles the registers of the sources.
__device__ __forceinline__ void conv_mad(u64& acc, u32 y, u32 c) {
  asm("v_mad_u64_u32 %0, vcc, %1, %2, %0" : "+v"(acc) : "v"(y), "s"(c) : "vcc");
}
// Double-precision sources (centred integers, |y| < 2^49) to a double-precision target with centred constants |c| < 2^49:
// the products are summed exactly as H + L. H starts at 1.5 * 2^102, in whose binade adding a product rounds it to a
// multiple of 2^50; what that adds to H is exact (both lie in the binade: at most 8 products of 2^98), and so is the rest of
// the product, an integer of magnitude at most 2^49, which goes to L (at most 2^52). Then H - 1.5 * 2^102 + L = c q + x with the
// quotient off by at most 1.25, so that H - 1.5 * 2^102 - c q = x - L stays below 2^53. 4 FP64 instructions a term and 6 at the
// end, against 4 multiply-adds a term and 19 for the sum of 30-bit pieces. Out: |x| <= 1.3 q.
template <int MAXLEN>
__device__ __forceinline__ void convert_fp(double (&x)[4], const ConvWord (&y)[MAXLEN][4], const ConvTarget<MAXLEN>& tg) {
  static_assert(MAXLEN <= 8, "more products leave the binade of H");
  const double q = tg.qd, qinv = tg.qinv;
  constexpr double M = 1.5 * 5070602400912917605986812821504.0;   // 1.5 * 2^102
  double H[4], L[4];
#pragma unroll
  for (int i = 0; i < 4; i++) H[i] = M, L[i] = 0.0;
#pragma unroll
  for (int k = 0; k < MAXLEN; k++) {
    const double ck = __longlong_as_double((long long)tg.c[k]);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const double yk = y[k][i].value(), Hn = __builtin_fma(yk, ck, H[i]);
      const double h = Hn - H[i];
      L[i] += __builtin_fma(yk, ck, -h);
      H[i] = Hn;
    }
  }
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const double h = H[i] - M;
    x[i] = __builtin_fma(-__builtin_rint(__builtin_fma(L[i], qinv, h * qinv)), q, h) + L[i];
  }
}
// Split-form sources to any target. NARROW: below 9m, plus `bias`: 0, or 2^62 less a multiple of m, which leaves the residue to a
// caller that takes 2^62 away again. Otherwise canonical.
template <int MAXLEN, bool NARROW>
__device__ __forceinline__ void convert_int(u64 (&x)[4], const ConvWord (&y)[MAXLEN][4], const ConvTarget<MAXLEN>& tg, u64 bias) {
  static_assert(MAXLEN <= 8, "the transforms that follow take values below 9m");
  Dot30N n[4];
  Dot30 g[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    n[i].a = g[i].s00 = (u32)tg.off & BCONV_M30;
    n[i].b = g[i].s01 = tg.off >> 30;
    g[i].s10 = g[i].s11 = 0;
    n[i].c = bias;
  }
#pragma unroll
  for (int k = 0; k < MAXLEN; k++) {
    const u32 c0 = (u32)tg.c[k] & BCONV_M30, c1 = (u32)(tg.c[k] >> 30);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      conv_mad(NARROW ? n[i].a : g[i].s00, y[k][i].lo, c0);
      conv_mad(NARROW ? n[i].b : g[i].s01, y[k][i].lo, c1);
      conv_mad(NARROW ? n[i].b : g[i].s10, y[k][i].hi, c0);
      conv_mad(NARROW ? n[i].c : g[i].s11, y[k][i].hi, c1);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; i++) {   // one position at a time: folding all four side by side would spill
    x[i] = NARROW ? dot30n_redc60(n[i], tg.m, tg.minv) : csub(redc(dot30_value(g[i]), tg.m, tg.minv), tg.m);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// f(0), .., f(N - 1) with constant indices: unrolled before the optimiser sees it, so that an array indexed in f can stay in
// registers (with an unrolled loop of this size all of it went to scratch memory).
template <class F, int... K>
__device__ __forceinline__ void conv_each_of(F f, std::integer_sequence<int, K...>) {
  (f(std::integral_constant<int, K>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void conv_each(F f) {
  conv_each_of(f, std::make_integer_sequence<int, N>{});
}

// One workgroup per (polynomial, tile, share of the targets), tiles fastest. The 64-byte row pieces of two adjacent tiles
// (N = 2^16) make one line: the XCD-contiguous order keeps them on one L2.
// READY: src holds what the inverse row pass makes of the sources (canonical residues, scaled).
template <int LOGR, int MAXLEN, bool SRC_FP, bool NARROW, bool READY>
__global__ void __launch_bounds__(CONV_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4))) conv_rows_kernel(ConvArgs a) {
  __shared__ u64 sm[2 * CONV_TILE_WORDS];
  constexpr int L = 11 - LOGR, LOGN = LOGR + 8;
  constexpr u32 TILES = 1u << (LOGN - 11);
  const u32 lin = xcd_swizzled_linear_id();
  const u32 tile = lin % TILES, share = conv_uniform((lin / TILES) % a.nsplit), poly = conv_uniform(lin / TILES / a.nsplit);
  const u32 j = conv_uniform(poly % a.beta), lo = j * a.alpha, len = min(a.alpha, a.src_nlimbs - lo);
  // offset inside a limb of the lane's first position in the last round's layout; its rows follow 256 words apart
  const u32 e0 = conv_elem(L, 0), pos = (e0 >> L) * 256 + (tile << L) + (e0 & ((1u << L) - 1));
  const u64* src = a.src + (size_t)(poly / a.beta) * a.src_poly_stride + ((size_t)(a.src_slot0 + lo) << LOGN);
  u64* dst = a.dst + (size_t)poly * a.dst_poly_stride;
  // the sources' positions: READY in the first round's layout, in which the targets start
  const u32 from = READY ? (threadIdx.x >> L) * 256 + (tile << L) + (threadIdx.x & ((1u << L) - 1)) : pos;
  constexpr u32 step = READY ? (CONV_THREADS >> L) * 256 : 256;
  ConvWord y[MAXLEN][4];   // doubles from double-precision sources, until the integer targets
  u64 ahead[4];   // the next source's words are requested before the current one is transformed
#pragma unroll
  for (int i = 0; i < 4; i++) ahead[i] = src[from + i * step];
  conv_each<MAXLEN>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    if ((u32)k >= len) {   // uniform
#pragma unroll
      for (int i = 0; i < 4; i++) y[k][i].lo = y[k][i].hi = 0;
      return;
    }
    const u32 id = a.src_id0 + lo + k;
    const ModInfo mi = conv_mod(a.mods, id);
    ulonglong2 sc;
    if (!READY) conv_fetch(sc, a.scale, lo + k);
    const u64* s = src + ((size_t)min((u32)k + 1, len - 1) << LOGN) + from;
    u64 now[4];
#pragma unroll
    for (int i = 0; i < 4; i++) now[i] = ahead[i];
#pragma unroll
    for (int i = 0; i < 4; i++) ahead[i] = s[i * step];
    if (SRC_FP) {
      double x[4];
      if (READY) {
#pragma unroll
        for (int i = 0; i < 4; i++) x[i] = u2d(now[i]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; i++) x[i] = __longlong_as_double((long long)now[i]);
        conv_inv_rows<LOGR>(x, a.twifp + ((size_t)id << LOGN), mi.qd, mi.qinv, (double*)sm);
#pragma unroll
        for (int i = 0; i < 4; i++)
          x[i] = fp_mulmod_const(x[i], __longlong_as_double((long long)sc.x), __longlong_as_double((long long)sc.y), mi.qd);
      }
      // |x| <= q, and (q + 1) / 2 is 2^-51 or more away from q/2 in units of q: no rounding of x / q can pass one half
#pragma unroll
      for (int i = 0; i < 4; i++) y[k][i].set(fp_reduce(x[i], mi.qinv, mi.qd));
    } else {
      u64 x[4];
#pragma unroll
      for (int i = 0; i < 4; i++) x[i] = now[i];
      if (!READY) {
        conv_inv_rows<LOGR>(x, a.twi + ((size_t)id << LOGN), mi.m, sm);
#pragma unroll
        for (int i = 0; i < 4; i++) x[i] = shoup(x[i], sc.x, sc.y, mi.m);
      }
#pragma unroll
      for (int i = 0; i < 4; i++) y[k][i].split(csub(x[i] + (mi.m >> 1), mi.m));
    }
  });
  lds_barrier();   // the last inverse exchange has been read everywhere
  // targets n, n + nsplit, .. of list [first, first + count) less the digit's own limbs, which stand together in the list of
  // their kind (lists are in the order of the slots): `body` does one
  auto walk = [&](u32 first, u32 count, bool own_kind, u32 n, auto chain, auto body) {
    const u32 skip = own_kind && a.skip_own ? len : 0;
    count -= skip;
    if (n >= count) return;
    auto at = [&](u32 i) {
      i = min(i, count - 1);
      return a.target[first + i + (i >= lo ? skip : 0)];
    };
    ConvTarget<MAXLEN> cur, next;
    cur.template fetch<decltype(chain)::value>(a, at(n), j);
    u32 info = at(n + a.nsplit);
#pragma nounroll
    for (; n < count; n += a.nsplit) {
      next.template fetch<decltype(chain)::value>(a, info, j);
      info = at(n + 2 * a.nsplit);
      body(cur);
      cur = next;
    }
  };
  auto fp_target = [&](const ConvTarget<MAXLEN>& tg) {
    const double* tw = a.twfp + ((size_t)tg.id << LOGN);
    ConvTwiddles<double> w;
    w.load(tw);
    __builtin_amdgcn_sched_barrier(0);
    double x[4];
    if (SRC_FP) {
      convert_fp<MAXLEN>(x, y, tg);
    } else {
      u64 v[4];   // in [-4m, 5m), below 2^53 in magnitude, as an offset from 2^62
      convert_int<MAXLEN, NARROW>(v, y, tg, (1ull << 62) - 4 * tg.m);
#pragma unroll
      for (int i = 0; i < 4; i++) x[i] = NARROW ? fp_reduce(u2d_biased62(v[i]), tg.qinv, tg.qd) : u2d(v[i]);
    }
    conv_fwd_rows<LOGR>(x, w, tw, tg.qd, tg.qinv, (double*)sm);
    double* d = (double*)dst + ((size_t)tg.slot << LOGN) + pos;
#pragma unroll
    for (int i = 0; i < 4; i++) d[i * 256] = x[i];
  };
  if (SRC_FP) walk(0, a.nfp, true, share, std::true_type{}, fp_target);
  else walk(0, a.nfp, false, share, std::false_type{}, fp_target);
  if (a.nint == 0) return;
  if (SRC_FP) {
    conv_each<MAXLEN>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      const double h = (u32)k < len ? (conv_mod(a.mods, a.src_id0 + lo + min((u32)k, len - 1)).qd - 1.0) * 0.5 : 0.0;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        y[k][i].split((u64)__double_as_longlong(y[k][i].value() + h + 4503599627370496.0) & 0x000FFFFFFFFFFFFFull);
      }
    });
  }
  // the shares that got one double-precision target more are the last to get an integer one
  walk(a.nfp, a.nint, !SRC_FP, a.nsplit - 1 - share, std::false_type{}, [&](const ConvTarget<MAXLEN>& tg) {
    const ulonglong2* tw = a.tw + ((size_t)tg.id << LOGN);
    ConvTwiddles<ulonglong2> w;
    w.load(tw);
    __builtin_amdgcn_sched_barrier(0);
    u64 x[4];
    convert_int<MAXLEN, NARROW>(x, y, tg, 0);
    conv_fwd_rows<LOGR>(x, w, tw, tg.m, sm);
    u64* d = dst + ((size_t)tg.slot << LOGN) + pos;
#pragma unroll
    for (int i = 0; i < 4; i++) d[i * 256] = x[i];
  });
}
