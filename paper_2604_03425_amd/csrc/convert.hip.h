// Base conversion fused with the transform passes on both sides of it (ModUp and ModDown, N = 2^13 .. 2^16, at most 8
// source limbs): second inverse pass of the sources, conversion, first forward pass of every target. Only the sources are
// read and only the targets, after their row pass, are written; as separate kernels the same step moved the sources three
// times more and the targets two times more. Where several workgroups share the targets of a tile, the inverse pass may be a
// kernel of its own before this one (READY, chosen in conv_plan).
//
// A conversion needs all sources of a position and a row pass all rows of a column in one workgroup. A workgroup of 512 lanes
// takes R rows x NC = 2048 / R columns, four positions per lane, and keeps all sources (8 x 4 words = 64 registers) while it walks
// over the targets. The conversion is a product of small integers on the matrix cores (see below), for two targets at a time: the
// second one's values wait in LDS (registers where there are four sources or fewer) while the first is transformed. Four positions
// per lane is what makes the sources fit beside a transform at 4 waves per SIMD; the row pass is then radix-4 rounds with up to
// three exchanges through LDS (two of them across waves), whose two tiles alternate so that an exchange costs one barrier. Two
// workgroups share a compute unit, so one computes while the other waits.
//
// Element e = row * NC + column of the tile; round K (stages 2K, 2K+1) holds, in lane t, the elements
// (t >> s) << (s + 2) | i << s | (t mod 2^s), s = 9 - 2K: the linear layout of a radix-4 transform of 2048 values of which
// only the first LOGR stages are done. The last round has s = 11 - LOGR, a lane then holds four adjacent rows of a column;
// for odd LOGR only the second of its two stages is left to do.
//
// What bounds it: instruction issue, at a clock rate that falls with the power the instructions take (1.65 - 1.75 GHz here).
// Vector instructions per target and position: 17 for the conversion (20 to an integer target), 38 and 74 for the row pass, LDS
// addresses included; on the vector units alone the conversion of 8 sources took 38 (double precision on both sides), 56 (integer
// sources) and 50 (integer targets). N = 2^16, 64 ciphertexts of 24 limbs, 3 digits of 8, 8 special primes: ModUp 1325 -> 1230 us,
// ModDown 989 -> 846; one such ciphertext 34.6 -> 30.9 and 23.6 -> 21.7 (inverse pass apart). The conversion, row passes and
// inverse pass as kernels of their own took 2030 and 1440 us.
#pragma once
#include "radix4.hip.h"
#include "ntt16_kernels.hip.h"

#include <cstddef>
#include <type_traits>
#include <utility>

#define CONV_THREADS 512
#define CONV_TILE 2048
#define CONV_MAX_SRC 8

// Reduction constants of an integer target m < 2^e: sh = max(0, e - 51), mu = -2^(64 + sh) / m to the nearest integer.
#define CONV_INT_MIN_BITS 36   // integer targets have more bits
struct ConvReduction {
  u32 sh;
  int mu;
};

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
  const uint4* pieces;       // [beta][ntarget] matrices of bytes of the constants (layout: conv_request_rows)
  // != null, double precision on both sides and at most CONV_DIRECT_SRC sources: [beta][ntarget][CONV_MAX_SRC] centred constants
  // (C/c_k) mod m_t for the conversion on the vector units
  const double* direct = nullptr;
  const ConvReduction* red;     // [nm] per modulus id, read on integer targets
  const ulonglong2* scale;   // [src_nlimbs] per source (Q_j/q_i)^-1 / N, in the form of its class
  const ulonglong2 *tw, *twi;
  const double *twfp, *twifp;
  const ModInfo* mods;
  u32 target[128];           // list index -> target slot | modulus id << 8
};

// a value that is the same in all lanes, said so: what is derived from it then stays in scalar registers
__device__ __forceinline__ u32 conv_uniform(u32 v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ ModInfo conv_mod(const ModInfo* mods, u32 id) {
  const_u64_ptr p = scalar_words(mods + id);
  ModInfo m = {};
#define CONV_WORD(FIELD) p[offsetof(ModInfo, FIELD) / 8]
  m.m = CONV_WORD(m);
  m.minv = CONV_WORD(minv);
  m.qd = __longlong_as_double((long long)CONV_WORD(qd));
  m.qinv = __longlong_as_double((long long)CONV_WORD(qinv));
#undef CONV_WORD
  return m;
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
    scalar_fetch(w[0], tw, (1u << (2 * K)) + blk);
    scalar_fetch(w[1], tw, (2u << (2 * K)) + 2 * blk);
    scalar_fetch(w[2], tw, (2u << (2 * K)) + 2 * blk + 1);
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
    scalar_fetch(w[0], tw, (1u << (LOGR - 1)) + 2 * blk);
    scalar_fetch(w[1], tw, (1u << (LOGR - 1)) + 2 * blk + 1);
    return;
  }
  w[0] = tw[(1u << (LOGR - 1)) + 2 * blk];
  w[1] = tw[(1u << (LOGR - 1)) + 2 * blk + 1];
}

// ---- double precision: forward and inverse row passes ----
// A forward pass gets its first rounds' twiddles (ConvTwiddles) from the caller, who requests them ahead of the conversion;
// the later ones' are requested as the registers for them become free. `freed` runs when the first
// ones are dead. In: |x| <= 1.5 q. Out: at most 2.64 q (three stages
// from a reduced value), which the block passes take: one reduction, after four or five stages.
template <class TW>
struct ConvTwiddles {
  TW w0[3], w1[3];
  __device__ __forceinline__ void load(const TW* __restrict__ tw) {
    conv_twiddles(w0, tw, 0);
    conv_twiddles(w1, tw, 1);
  }
};
template <int LOGR, class FREED>
__device__ __forceinline__ void conv_fwd_rows(double (&x)[4], const ConvTwiddles<double>& w, const double* __restrict__ tw,
                                              double q, double qinv, double* sm, FREED freed) {
  constexpr int L = 11 - LOGR;
  double w2[3], w3[3], wl[2];
  if (LOGR >= 6) conv_twiddles(w2, tw, 2);
  radix4_fwd(x, w.w0, q, qinv);
  conv_exchange<9, 7>(x, sm);
  if (LOGR == 8) conv_twiddles(w3, tw, 3);
  if (LOGR & 1) conv_twiddles_last<LOGR>(wl, tw);
  radix4_fwd(x, w.w1, q, qinv);
  freed();
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
template <int LOGR, class FREED>
__device__ __forceinline__ void conv_fwd_rows(u64 (&x)[4], const ConvTwiddles<ulonglong2>& w,
                                              const ulonglong2* __restrict__ tw, u64 q, u64* sm, FREED freed) {
  constexpr int L = 11 - LOGR;
  const u64 q2 = lazy_const<true>(q);
  ulonglong2 w2[3], w3[3], wl[2];
  radix4_fwd<true>(x, w.w0, q, q2);
  conv_exchange<9, 7>(x, sm);
  if (LOGR >= 6) conv_twiddles(w2, tw, 2);
  radix4_fwd<true>(x, w.w1, q, q2);
  freed();
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

// ---- conversions on the matrix cores ----
// A source y (centred, below 2^60 in magnitude) is cut into 8 bytes y = sum_i y_i 2^(8 i), each in [-128, 127]; on the other
// side stand the bytes of C_ki = c_k 2^(8 i) mod m, centred. Then
//   sum_k y_k c_k  =  sum_p 2^(8 p) S_p  (mod m),   S_p = sum_(k,i) y_ki (byte p of C_ki),
// a product of an 8-row matrix of bytes per target with 8 bytes per source and position: at most 64 products of 2^14 to a sum,
// exact in 32 bits. What is left for the vector units is to put eight sums together, modulo m: the whole is below 2^12 m.
// v_mfma_i32_32x32x32_i8 takes four sources: lane (h, n) = (lane / 32, lane % 32) supplies 16 bytes, sources 2h and 2h + 1 of
// position n in the second operand, of row n in the first, and receives rows 8b + 4h + r of column n. Rows are dealt so that lane
// half h gets the 8 sums (b, r) = (p / 4, p % 4) of target h of a pair; the upper 16 rows of the product are not used (a full
// one would serve four targets, whose results do not fit the registers; the matrix cores are busy an eighth of the time, by their
// counter). A lane's four positions of all sources become the operands of 2 x 4 products by swaps of half-waves, in place.
typedef int conv_i32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) u32* lds_const_ptr;
typedef int conv_i32x16 __attribute__((ext_vector_type(16)));
#define CONV_PIECES 8   // bytes of a constant, and of a source

// A source at one position: its 8 bytes, as a word.
// |v| < 2^49, an integer. 1.5 * 2^52 + v + 0x808080808080: the low 48 bits are the lower six bytes plus 128 each, the four above
// them the next byte (what is left there after taking away the exponent and 2^51); byte 7 meets zeros.
__device__ __forceinline__ u64 conv_cut(double v) {
  const double t = v + (6755399441055744.0 + 141289400074368.0);
  const u32 lo = (u32)__double2loint(t) ^ 0x80808080u, hi = ((u32)__double2hiint(t) ^ 0x8080u) - 0x43380000u;
  return (u64)hi << 32 | lo;
}
// shifted = v + h in [0, 2^60); off8 = 0x8080808080808080 - h
__device__ __forceinline__ u64 conv_cut(u64 shifted, u64 off8) { return (shifted + off8) ^ 0x8080808080808080ull; }
// Swaps the upper half-wave of x with the lower one of y.
__device__ __forceinline__ void conv_swap32(u32& x, u32& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
  x = r[0];
  y = r[1];
}
// a * b + c in 64 bits, one instruction. (Not as an asm statement: next to matrix instructions the compiler has to see what
// writes a register, or it gives out one that a product in flight has yet to write.)
__device__ __forceinline__ long long conv_mad(int a, int b, long long c) { return (long long)a * b + c; }
// b, hidden from the compiler, which would make shifts of a product by a power of two
__device__ __forceinline__ int conv_opaque(int b) {
  asm("" : "+s"(b));
  return b;
}
// What is uniform about a target. Fetched one pair of targets ahead, its place in the list two ahead, so that no target starts
// by waiting for a chain of scalar loads.
struct ConvTarget {
  u32 slot, id, sh;
  int mu;
  u64 m;
  double qd, qinv;
  __device__ __forceinline__ void fetch(const ModInfo* mods, const ConvReduction* red, u32 slot_, u32 id_) {
    slot = slot_;
    id = id_;
    const ModInfo mi = conv_mod(mods, id);
    m = mi.m, qd = mi.qd, qinv = mi.qinv;
    const u64 r = scalar_words(red)[id];
    sh = (u32)r;
    mu = (int)(r >> 32);
  }
  __device__ __forceinline__ void fetch(const ConvArgs& a, u32 target) { fetch(a.mods, a.red, target & 255, target >> 8); }
};
// The lanes' rows of a pair of targets: lane (h, n) has bytes of sources 4g + 2h and 4g + 2h + 1 (byte p of every C_ki, i
// ascending), p = 4 * bit 3 of n + the two lowest bits of n, of target bit 2 of n. Wave g < MAXLEN / 4 copies the rows of group g
// straight into LDS, 16 bytes a lane.
#define CONV_ROWS_WORDS(MAXLEN) ((MAXLEN) / 4 * 256)
template <int MAXLEN>
__device__ __forceinline__ void conv_request_rows(const ConvArgs& a, u32 first_row, u32 slot0, u32 slot1, u32* image) {
  const u32 g = conv_uniform(threadIdx.x >> 6);
  if (g >= MAXLEN / 4) return;
  u32 l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  const u32 h = l >> 5, p = (l & 3) + 4 * ((l >> 3) & 1), row = first_row + ((l & 4) ? slot1 : slot0);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)a.pieces, 0, (int)(a.beta * a.ntarget * (MAXLEN / 4) * 2 * CONV_PIECES * 16), 0x00020000);
  // (beyond the table, so read as zeros, for the unused rows: they would cost power, which is what the clock rate depends on)
  const int at = (l & 16) ? 0x7FFFFFF0 : (int)((((row * (MAXLEN / 4) + g) * 2 + h) * CONV_PIECES + p) * 16);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(image + g * 256), 16, at, 0, 0, 0);
}
// All vector memory requests of the wave are back, said so that the compiler knows.
__device__ __forceinline__ void conv_wait_vector_memory() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  asm volatile("" ::: "memory");
}
template <int MAXLEN>
struct ConvRows {
  conv_i32x4 a[MAXLEN / 4];
  // As an asm statement with its own wait: the compiler, which does not see the barriers that order it after the copy, would wait
  // for everything requested since, stores included. (No product is in flight here whose registers it could be given.)
  __device__ __forceinline__ void take(const u32* image) {
    const u32 at = (u32)(size_t)(lds_const_ptr)image + (threadIdx.x & 63) * 16;
    if (MAXLEN == 4) asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(a[0]) : "v"(at) : "memory");
    else
      asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:1024\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(a[0]), "=&v"(a[MAXLEN / 4 - 1]) : "v"(at) : "memory");
  }
};
// The eight sums of a target at the lane's column, put together: lo + hi 2^32 (mod m), lo < 2^32.
__device__ __forceinline__ void conv_join(u32& lo, long long& hi, const conv_i32x16& d) {
  const int a0 = d[0] + (d[1] << 8), a1 = d[2] + (d[3] << 8), a2 = d[4] + (d[5] << 8), a3 = d[6] + (d[7] << 8);
  const int w = conv_opaque(65536);
  const long long l = conv_mad(a1, w, a0), h = conv_mad(a3, w, a2);
  lo = (u32)l;
  hi = h + (l >> 32);
}
// The same where the whole is below 2^62 (m < 2^50), so that hi fits 32 bits.
__device__ __forceinline__ void conv_join(u32& lo, int& hi, const conv_i32x16& d) {
  const int a0 = d[0] + (d[1] << 8), a1 = d[2] + (d[3] << 8), a2 = d[4] + (d[5] << 8), a3 = d[6] + (d[7] << 8);
  const long long l = conv_mad(a1, conv_opaque(65536), a0);
  lo = (u32)l;
  hi = (int)((u32)(l >> 32) + (u32)a2 + ((u32)a3 << 16));
}
// |x| <= q / 2 (and a rounding): lo + hi 2^32 less its nearest multiple of q; the difference before lo is added is below 2^53.
__device__ __forceinline__ double conv_settle(u32 lo, int hi, double q, double qinv) {
  const double l = (double)lo, h = (double)hi;
  const double c = __builtin_rint(__builtin_fma(l, qinv, h * (qinv * 4294967296.0)));
  return __builtin_fma(__builtin_fma(-c, q * (1.0 / 4294967296.0), h), 4294967296.0, l);
}
// V = lo + hi 2^32, |V| <= 2^12 m: V + s m with s = 2 + floor((hi >> sh) mu / 2^32), which is within [-V / m + 0.75, -V / m + 2.33] (mu
// is off by a half, hi >> sh below 2^31 by one): in [0.75 m, 2.33 m]. Needs 2^36 <= m < 2^60.
__device__ __forceinline__ u64 conv_settle(u32 lo, long long hi, const ConvTarget& tg) {
  const int t = (int)__builtin_amdgcn_alignbit((u32)(hi >> 32), (u32)hi, tg.sh);
  const int s = __mulhi(t, tg.mu) + 2;
  const int m0 = (int)(u32)tg.m;
  const u32 m1 = (u32)(tg.m >> 32) + ((u32)tg.m >> 31);
  const u64 v = (u64)conv_mad(s, m0, (long long)((u64)(u32)hi << 32 | lo));
  return (u64)((u32)(v >> 32) + (u32)s * m1) << 32 | (u32)v;
}
// ---- double precision on both sides, few sources: on the vector units ----
// The matrix products of a pair of targets cost what four or eight sources cost, whatever their number, and a lone workgroup's start
// waits for its matrices; up to 6 sources the sums below are fewer instructions. 460 calls with 1 to 8 sources, every prime below
// 2^50, all two-pass rings: 2 to 4 % faster this way up to 6 sources, even at 8 (not built for 7). us, matrix cores | here: one
// rotation of 5 + 5 limbs in one digit at 2^13 45.3 | 42.5, 24 of them 75.9 | 70.6; 24 of 2 + 2 limbs at 2^16 155 | 150; 24 of 3 + 1 limbs
// in 3 digits at 2^15 131.6 | 126.2.
#define CONV_DIRECT_SRC 6
template <int MAXLEN>
struct ConvFpTarget {
  u32 slot, id;
  double q, qinv, c[MAXLEN];
  __device__ __forceinline__ void fetch(const ConvArgs& a, u32 target, u32 j) {
    slot = target & 255;
    id = target >> 8;
    const ModInfo mi = conv_mod(a.mods, id);
    q = mi.qd, qinv = mi.qinv;
    const const_u64_ptr p = scalar_words(a.direct + ((size_t)j * a.ntarget + slot) * CONV_MAX_SRC);
#pragma unroll
    for (int k = 0; k < MAXLEN; k++) c[k] = scalar_double(p + k);
  }
};
// Sources y (centred integers, |y| < 2^49, doubles kept as words) times constants |c| < 2^49, summed exactly as H + L. H starts at
// 1.5 * 2^102, in whose binade adding a product rounds it to a multiple of 2^50; what that adds to H is exact (both lie in the binade:
// at most 8 products of 2^98), and so is the rest of the product, an integer of magnitude at most 2^49, which goes to L (at most
// 2^52). Then H - 1.5 * 2^102 + L = t q + x with the quotient off by at most 1.25, so that H - 1.5 * 2^102 - t q stays below 2^53.
// 4 instructions a term and 6 at the end. Out: |x| <= 1.3 q.
template <int MAXLEN>
__device__ __forceinline__ void convert_fp(double (&x)[4], const u64 (&y)[CONV_DIRECT_SRC][4], const ConvFpTarget<MAXLEN>& tg) {
  static_assert(MAXLEN <= CONV_DIRECT_SRC && CONV_DIRECT_SRC <= 8, "more products leave the binade of H");
  constexpr double M = 1.5 * 5070602400912917605986812821504.0;   // 1.5 * 2^102
  double H[4], L[4];
#pragma unroll
  for (int i = 0; i < 4; i++) H[i] = M, L[i] = 0.0;
#pragma unroll
  for (int k = 0; k < MAXLEN; k++)
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const double yk = __longlong_as_double((long long)y[k][i]), Hn = __builtin_fma(yk, tg.c[k], H[i]), h = Hn - H[i];
      L[i] += __builtin_fma(yk, tg.c[k], -h);
      H[i] = Hn;
    }
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const double h = H[i] - M;
    x[i] = __builtin_fma(-__builtin_rint(__builtin_fma(L[i], tg.qinv, h * tg.qinv)), tg.q, h) + L[i];
  }
}
// Targets share, share + nsplit, .. less the digit's own limbs, which stand together in the list. What is uniform about one is fetched
// one target ahead, its place in the list two ahead.
template <int LOGR, int MAXLEN>
__device__ __forceinline__ void conv_direct_targets(const ConvArgs& a, const u64 (&y)[CONV_DIRECT_SRC][4], u32 j, u32 lo, u32 len, u32 share,
                                                    u32 pos, u64* dst, u64* sm) {
  constexpr int LOGN = LOGR + 8;
  const u32 skip = a.skip_own ? len : 0, count = a.nfp - skip;
  if (share >= count) return;   // uniform
  auto at = [&](u32 i) {
    i = min(i, count - 1);
    return a.target[i + (i >= lo ? skip : 0)];
  };
  ConvFpTarget<MAXLEN> tg, next;
  next.fetch(a, at(share), j);
  u32 info = at(share + a.nsplit);
  lds_barrier();   // the last inverse exchange has been read everywhere
#pragma nounroll
  for (u32 n = share; n < count; n += a.nsplit) {
    tg = next;
    next.fetch(a, info, j);
    info = at(n + 2 * a.nsplit);
    const double* tw = a.twfp + ((size_t)tg.id << LOGN);
    ConvTwiddles<double> w;
    w.load(tw);
    __builtin_amdgcn_sched_barrier(0);
    double x[4];
    convert_fp<MAXLEN>(x, y, tg);
    conv_fwd_rows<LOGR>(x, w, tw, tg.q, tg.qinv, (double*)sm, [] {});
    double* d = (double*)dst + ((size_t)tg.slot << LOGN) + pos;
#pragma unroll
    for (int i = 0; i < 4; i++) d[i * 256] = x[i];
  }
}
// All sources at the lane's four positions as operands: y[i][f][g], columns = positions i of lane half f, sources 4g .. 4g + 3.
template <int MAXLEN>
struct ConvSources {
  conv_i32x4 y[4][2][MAXLEN / 4];
};
template <int MAXLEN>
__device__ __forceinline__ conv_i32x16 conv_product(const ConvRows<MAXLEN>& r, const conv_i32x4 (&y)[MAXLEN / 4]) {
  conv_i32x16 d = {};
#pragma unroll
  for (int g = 0; g < MAXLEN / 4; g++) d = __builtin_amdgcn_mfma_i32_32x32x32_i8(r.a[g], y[g], d, 0, 0, 0);
  return d;
}
// A pair of double-precision targets at the lane's four positions: |x| <= q / 2. x1 takes the second one's.
template <int MAXLEN, class X1>
__device__ __forceinline__ void convert(double (&x0)[4], X1 x1, const ConvSources<MAXLEN>& y, const ConvRows<MAXLEN>& r,
                                        const ConvTarget& t0, const ConvTarget& t1) {
#pragma unroll
  for (int i = 0; i < 4; i++) {
    u32 lo[2], hi[2];
#pragma unroll
    for (int f = 0; f < 2; f++) {
      int h;
      conv_join(lo[f], h, conv_product<MAXLEN>(r, y.y[i][f]));
      hi[f] = (u32)h;
    }
    conv_swap32(lo[0], lo[1]);
    conv_swap32(hi[0], hi[1]);
    x0[i] = conv_settle(lo[0], (int)hi[0], t0.qd, t0.qinv);
    x1(i, conv_settle(lo[1], (int)hi[1], t1.qd, t1.qinv));
  }
}
// A pair of integer targets: below 2.34 m.
template <int MAXLEN, class X1>
__device__ __forceinline__ void convert(u64 (&x0)[4], X1 x1, const ConvSources<MAXLEN>& y, const ConvRows<MAXLEN>& r,
                                        const ConvTarget& t0, const ConvTarget& t1) {
#pragma unroll
  for (int i = 0; i < 4; i++) {
    u32 lo[2], mid[2], hi[2];
#pragma unroll
    for (int f = 0; f < 2; f++) {
      long long h;
      conv_join(lo[f], h, conv_product<MAXLEN>(r, y.y[i][f]));
      mid[f] = (u32)h;
      hi[f] = (u32)(h >> 32);
    }
    conv_swap32(lo[0], lo[1]);
    conv_swap32(mid[0], mid[1]);
    conv_swap32(hi[0], hi[1]);
    x0[i] = conv_settle(lo[0], (long long)((u64)hi[0] << 32 | mid[0]), t0);
    x1(i, conv_settle(lo[1], (long long)((u64)hi[1] << 32 | mid[1]), t1));
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
// DIRECT: double precision on both sides, on the vector units (a.direct).
template <int LOGR, int MAXLEN, bool SRC_FP, bool READY, bool DIRECT = false>
__global__ void __launch_bounds__(CONV_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4))) conv_rows_kernel(ConvArgs a) {
  __shared__ u64 sm[2 * CONV_TILE_WORDS];
  __shared__ u64 second[MAXLEN == 4 ? 1 : CONV_TILE];
  __shared__ __attribute__((aligned(16))) u32 rows_image[2 * CONV_ROWS_WORDS(MAXLEN)];
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
  u64 y[DIRECT ? CONV_DIRECT_SRC : MAXLEN][4];   // (with four rows of DIRECT the compiler makes one register tuple of it, and copies of that)
  u64 ahead[4];   // the next source's words are requested before the current one is transformed
#pragma unroll
  for (int i = 0; i < 4; i++) ahead[i] = src[from + i * step];
  conv_each<MAXLEN>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    if ((u32)k >= len) {   // uniform
#pragma unroll
      for (int i = 0; i < 4; i++) y[k][i] = 0;
      return;
    }
    const u32 id = a.src_id0 + lo + k;
    const ModInfo mi = conv_mod(a.mods, id);
    ulonglong2 sc;
    if (!READY) scalar_fetch(sc, a.scale, lo + k);
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
      for (int i = 0; i < 4; i++) {
        const double v = fp_reduce(x[i], mi.qinv, mi.qd);
        y[k][i] = DIRECT ? (u64)__double_as_longlong(v) : conv_cut(v);
      }
    } else {
      u64 x[4];
#pragma unroll
      for (int i = 0; i < 4; i++) x[i] = now[i];
      if (!READY) {
        conv_inv_rows<LOGR>(x, a.twi + ((size_t)id << LOGN), mi.m, sm);
#pragma unroll
        for (int i = 0; i < 4; i++) x[i] = shoup(x[i], sc.x, sc.y, mi.m);
      }
      const u64 h = mi.m >> 1, off8 = 0x8080808080808080ull - h;
#pragma unroll
      for (int i = 0; i < 4; i++) y[k][i] = conv_cut(csub(x[i] + h, mi.m), off8);
    }
  });
  if constexpr (DIRECT) return conv_direct_targets<LOGR, MAXLEN>(a, y, j, lo, len, share, pos, dst, sm);
  ConvSources<MAXLEN> ys;
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int g = 0; g < MAXLEN / 4; g++) {
      u32 p[2][4];
#pragma unroll
      for (int f = 0; f < 2; f++)
#pragma unroll
        for (int k = 0; k < 2; k++) p[f][2 * k] = (u32)y[4 * g + 2 * f + k][i], p[f][2 * k + 1] = (u32)(y[4 * g + 2 * f + k][i] >> 32);
#pragma unroll
      for (int w = 0; w < 4; w++) conv_swap32(p[0][w], p[1][w]);
#pragma unroll
      for (int f = 0; f < 2; f++) ys.y[i][f][g] = conv_i32x4{(int)p[f][0], (int)p[f][1], (int)p[f][2], (int)p[f][3]};
    }
  // Targets n, n + nsplit, .. of list [first, first + count) less the digit's own limbs, which stand together in the list of
  // their kind (lists are in the order of the slots), in pairs. `zero`: of the type of their values.
  auto walk = [&](u32 first, u32 count, bool own_kind, u32 n, auto* tables, auto zero, auto transform) {
    typedef decltype(zero) V;
    typedef std::remove_const_t<std::remove_pointer_t<decltype(tables)>> TW;
    const u32 skip = own_kind && a.skip_own ? len : 0;
    count -= skip;
    if (n >= count) return;
    auto at = [&](u32 i) {
      i = min(i, count - 1);
      return a.target[first + i + (i >= lo ? skip : 0)];
    };
    u32 i0 = at(n), i1 = at(n + a.nsplit), buffer = 0;
    ConvTarget t0, t1, n0, n1;
    conv_request_rows<MAXLEN>(a, j * a.ntarget, i0 & 255, i1 & 255, rows_image);
    n0.fetch(a, i0);
    n1.fetch(a, i1);
    i0 = at(n + 2 * a.nsplit);
    i1 = at(n + 3 * a.nsplit);
    conv_wait_vector_memory();
    lds_barrier();   // (the last inverse exchange has been read everywhere, too)
#pragma nounroll
    for (; n < count; n += 2 * a.nsplit) {
      t0 = n0, t1 = n1;
      ConvTwiddles<TW> w;
      w.load(tables + ((size_t)t0.id << LOGN));
      __builtin_amdgcn_sched_barrier(0);
      V x[4], y1[4], *later = (V*)second + threadIdx.x;   // the second target's values wait in LDS
      {
        ConvRows<MAXLEN> rows;
        rows.take(rows_image + buffer);
        convert<MAXLEN>(x, [&](int i, V v) { if (MAXLEN == 4) y1[i] = v; else later[i * CONV_THREADS] = v; }, ys, rows, t0, t1);
      }
      buffer ^= CONV_ROWS_WORDS(MAXLEN);
      // Into the image that the pair before was read from, ahead of its barriers. Wave 0 or 1 waits for them before the first
      // target's stores (everything requested later has been waited for by then); the second's barriers show them to all.
      conv_request_rows<MAXLEN>(a, j * a.ntarget, i0 & 255, i1 & 255, rows_image + buffer);
      ConvTwiddles<TW> w1;
      transform(x, t0, w, [&] {
        w1.load(tables + ((size_t)t1.id << LOGN));
        n0.fetch(a, i0);
        n1.fetch(a, i1);
        i0 = at(n + 4 * a.nsplit);
        i1 = at(n + 5 * a.nsplit);
        __builtin_amdgcn_sched_barrier(0);
      });
      conv_wait_vector_memory();
      auto store = [&](u32 slot) {
        V* d = (V*)dst + ((size_t)slot << LOGN) + pos;
#pragma unroll
        for (int i = 0; i < 4; i++) d[i * 256] = x[i];
      };
      store(t0.slot);
      if (n + a.nsplit >= count) return;
#pragma unroll
      for (int i = 0; i < 4; i++) x[i] = MAXLEN == 4 ? y1[i] : later[i * CONV_THREADS];
      transform(x, t1, w1, [] {});
      store(t1.slot);
    }
  };
  walk(0, a.nfp, SRC_FP, share, a.twfp, 0.0, [&](double (&x)[4], const ConvTarget& tg, const ConvTwiddles<double>& w, auto freed) {
    conv_fwd_rows<LOGR>(x, w, a.twfp + ((size_t)tg.id << LOGN), tg.qd, tg.qinv, (double*)sm, freed);
  });
  // the shares that got one double-precision target more are the last to get an integer one
  walk(a.nfp, a.nint, !SRC_FP, a.nsplit - 1 - share, a.tw, (u64)0,
       [&](u64 (&x)[4], const ConvTarget& tg, const ConvTwiddles<ulonglong2>& w, auto freed) {
         conv_fwd_rows<LOGR>(x, w, a.tw + ((size_t)tg.id << LOGN), tg.m, sm, freed);
       });
}
