// Key switch of the ring N = 2^12 in four kernels. A limb is 32 KB, so a workgroup holds it whole (four values in each of
// 1024 lanes, radix4.hip.h) and everything between two exchanges of data across limbs happens in its registers:
//   front:   what is switched, read through the Galois map or formed as a product of two ciphertexts, to coefficient form;
//   digits:  per digit and extended limb, conversion and forward transform;
//   special: per key component and special limb, inner product with the key and inverse transform;
//   final:   per output limb, ModDown's conversion and transform, inner product, (sum - correction) / P, addends.
// What bounds it: at the batches this ring is used with (tens of ciphertexts of a few limbs) nothing but the number of
// dependent launches and the latency inside each, so a kernel holds one transform per workgroup and no more: with a
// workgroup taking all digits of a limb in line (three kernels) 8 rotations of 5 limbs, 3 digits, took 88 us, 46 us
// this way. Coefficient-domain limbs travel in the split form of ntt16_bconv_rows_kernel: (y + (q-1)/2) mod q as two
// 30-bit halves, which makes the centred conversion a dot product plus a constant per target.
#pragma once
#include "radix4.hip.h"
#include "ntt16_kernels.hip.h"

struct Ks12Args {
  const u64* d;            // polynomial to switch, eval domain: limb-vector (b, i) at d + b*d_stride + i*4096
  u64 d_stride;
  const u64 *pa, *pb;      // != null: d is the product of the second components of pa and pb, [B][2][nlimbs][4096], and the
                           // other two terms of the product are the addends
  u64* dcoef;              // [B][nlimbs][4096] split form
  u64* ext;                // [B][beta][next][4096]: converted digits, eval domain (doubles on double-precision moduli)
  u64* acc;                // [B][2][next][4096]: special limbs only, split form
  u64* out;                // [B][2][nlimbs][4096]
  const u64* evk;          // [dnum][2][nm][4096]
  const u64 *add2, *add_src;   // addends as in FwdFinalArgs
  const ulonglong2 *tw, *twi;
  const double *twfp, *twifp;
  const ModInfo* mods;
  const ulonglong2 *up_scale, *dn_scale, *pinv;
  const u64 *up_mat, *up_off, *dn_mat, *dn_off;
  u32 up_pitch, dn_pitch;
  u32 nlimbs, nq, nm, alpha, beta, next, fp_on;
  u32 fp_mask[4];          // bit id: modulus id is of double-precision class
  u32 mode0, mode1, add2_three;
  u32 d_galois, add_galois;
  u32 multi;               // != 0: ciphertext b uses galois_pc[b] and evk_pc[b]
  u32 galois_pc[KS_MULTI_MAX];
  const u64* evk_pc[KS_MULTI_MAX];
};

// The constants of a modulus, by scalar loads also where the compiler moves them behind stores and barriers.
__device__ __forceinline__ ModInfo ks12_mod(const ModInfo* mods, u32 id) {
  const const_u64_ptr p = scalar_words(mods + id);
  ModInfo m;
  m.m = p[0], m.mu64 = p[1], m.c64 = p[2], m.c64s = p[3], m.ninv = p[4], m.ninvs = p[5], m.minv = p[6], m.pmod = p[7];
  m.qd = __longlong_as_double((long long)p[8]), m.qinv = __longlong_as_double((long long)p[9]);
  m.ninvd = __longlong_as_double((long long)p[10]), m.ninvq = __longlong_as_double((long long)p[11]);
  return m;
}
static_assert(sizeof(ModInfo) == 12 * 8, "ks12_mod lists the words");
// One modulus of double-precision (FP) or integer class with its transforms. Values are doubles or residues.
template <bool FP>
struct Ks12Mod;
template <>
struct Ks12Mod<true> {
  typedef double V;
  const ModInfo mi;
  __device__ __forceinline__ explicit Ks12Mod(const ModInfo& m) : mi(m) {}
  __device__ __forceinline__ V load(u64 v) const { return u2d(v); }
  __device__ __forceinline__ V mul(u64 a, u64 b) const { return fp_mulmod_var(u2d(a), u2d(b), mi.qinv, mi.qd); }   // <= 0.9 q
  __device__ __forceinline__ void forward(V (&x)[4], const WlTwiddles<double>& w, u64* sm) const {
    wl_fwd(x, w, mi.qd, mi.qinv, (double*)sm);
  }
  __device__ __forceinline__ void inverse(u64 (&y)[4], V (&x)[4], const WlTwiddles<double>& w, ulonglong2 sc, u64* sm) const {
    wl_inv(x, w, mi.qd, mi.qinv, __longlong_as_double((long long)sc.x), __longlong_as_double((long long)sc.y), (double*)sm);
#pragma unroll
    for (int i = 0; i < 4; i++) y[i] = d2u_canon(x[i], mi.qd);
  }
  // s += x * e; at most four products (below 0.9 q each) are added between folds
  __device__ __forceinline__ V mac(V s, V x, u64 e, u32 j) const {
    s += fp_mulmod_var(x, u2d(e), mi.qinv, mi.qd);
    return (j & 3) == 3 ? fp_reduce(s, mi.qinv, mi.qd) : s;
  }
  __device__ __forceinline__ V settle(V s) const { return fp_reduce(s, mi.qinv, mi.qd); }
  __device__ __forceinline__ V finish(V acc, V x, ulonglong2 pv) const {   // <= 0.75 q
    return fp_mulmod_const(acc - x, __longlong_as_double((long long)pv.x), __longlong_as_double((long long)pv.y), mi.qd);
  }
  __device__ __forceinline__ V add(V a, u64 b) const { return a + u2d(b); }
  __device__ __forceinline__ V add_product(V r, u64 a0, u64 b0) const { return r + mul(a0, b0); }
  __device__ __forceinline__ u64 result(V r) const { return d2u_canon(fp_reduce(r, mi.qinv, mi.qd), mi.qd); }
};
template <>
struct Ks12Mod<false> {
  typedef u64 V;
  const ModInfo mi;
  const bool big;   // uniform: Harvey butterflies (q >= 2^52)
  __device__ __forceinline__ explicit Ks12Mod(const ModInfo& m) : mi(m), big((m.m >> 52) != 0) {}
  __device__ __forceinline__ V load(u64 v) const { return v; }
  __device__ __forceinline__ V mul(u64 a, u64 b) const { return mulmod(a, b, mi); }
  __device__ __forceinline__ void forward(V (&x)[4], const WlTwiddles<ulonglong2>& w, u64* sm) const {
    if (big) wl_fwd<true>(x, w, mi.m, mi.mu64, sm);
    else wl_fwd<false>(x, w, mi.m, mi.mu64, sm);
  }
  __device__ __forceinline__ void inverse(u64 (&y)[4], V (&x)[4], const WlTwiddles<ulonglong2>& w, ulonglong2 sc, u64* sm) const {
    if (big) wl_inv<true>(x, w, mi.m, mi.mu64, sc.x, sc.y, sm);
    else wl_inv<false>(x, w, mi.m, mi.mu64, sc.x, sc.y, sm);
#pragma unroll
    for (int i = 0; i < 4; i++) y[i] = x[i];
  }
  // products carry the factor 2^-64, which dn_scale, dn_mat and pinv absorb; s stays below 2q
  __device__ __forceinline__ V mac(V s, V x, u64 e, u32) const {
    const Acc128 p = {x * e, mul_hi64(x, e)};
    return csub(s + redc(p, mi.m, mi.minv), 2 * mi.m);
  }
  __device__ __forceinline__ V settle(V s) const { return csub(s, mi.m); }
  __device__ __forceinline__ V finish(V acc, V x, ulonglong2 pv) const { return shoup(acc + mi.m - x, pv.x, pv.y, mi.m); }
  __device__ __forceinline__ V add(V a, u64 b) const { return addmod(a, b, mi.m); }
  __device__ __forceinline__ V add_product(V r, u64 a0, u64 b0) const { return addmod(r, mulmod(a0, b0, mi), mi.m); }
  __device__ __forceinline__ u64 result(V r) const { return r; }
};
template <bool FP>
struct Ks12Tables;
template <>
struct Ks12Tables<true> {
  typedef WlTwiddles<double> W;
  static __device__ __forceinline__ const double* fwd(const Ks12Args& a, u32 id) { return a.twfp + (size_t)id * 4096; }
  static __device__ __forceinline__ const double* inv(const Ks12Args& a, u32 id) { return a.twifp + (size_t)id * 4096; }
};
template <>
struct Ks12Tables<false> {
  typedef WlTwiddles<ulonglong2> W;
  static __device__ __forceinline__ const ulonglong2* fwd(const Ks12Args& a, u32 id) { return a.tw + (size_t)id * 4096; }
  static __device__ __forceinline__ const ulonglong2* inv(const Ks12Args& a, u32 id) { return a.twi + (size_t)id * 4096; }
};

__device__ __forceinline__ u64 ks12_split(u64 y, u64 m) {
  y = csub(y + (m >> 1), m);
  return (y & 0x3FFFFFFFull) | ((y >> 30) << 32);
}
// What is switched at limb i, round-2 layout.
template <bool FP>
__device__ __forceinline__ void ks12_load_d(typename Ks12Mod<FP>::V (&x)[4], const Ks12Args& a, u32 b, u32 i,
                                            const Ks12Mod<FP>& md) {
  if (a.pa) {
    const size_t o = (((size_t)b * 2 + 1) * a.nlimbs + i) * 4096;
#pragma unroll
    for (int k = 0; k < 4; k++) x[k] = md.mul(a.pa[o + wl_elem(2, k)], a.pb[o + wl_elem(2, k)]);
    return;
  }
  const u64* src = a.d + (size_t)b * a.d_stride + (size_t)i * 4096;
  const u32 g = a.multi ? a.galois_pc[__builtin_amdgcn_readfirstlane(b)] : a.d_galois;
#pragma unroll
  for (int k = 0; k < 4; k++) x[k] = md.load(src[g ? galois_src_index(wl_elem(2, k), g, 12) : wl_elem(2, k)]);
}
// Base conversion of `len` split limbs to modulus mi in the round-0 layout, canonical. The constants come by scalar loads, said so:
// of a kernel's two bodies only the first would get them, since the compiler takes its stores for writes that the second may read
// (integer bodies second, with vector loads: a matrix product with 18 rotations of one 55-bit limb 696 -> 692 us, 2 rotations of 4
// 60-bit limbs 46.3 -> 46.0, 8 products of 5 55-bit limbs 56.9 -> 56.4).
template <bool NARROW>
__device__ __forceinline__ void ks12_convert(u64 (&x)[4], const u64* __restrict__ src, u32 len, const_u64_ptr crow,
                                             u64 offc, const ModInfo& mi) {
  BconvAcc<4, NARROW> acc;
  acc.init(offc);
  u64 w[4], wn[4];
#pragma unroll
  for (int i = 0; i < 4; i++) wn[i] = src[wl_elem(0, i)];
  for (u32 k = 0; k < len; k++) {
#pragma unroll
    for (int i = 0; i < 4; i++) w[i] = wn[i];
    const u64* next = src + (size_t)min(k + 1, len - 1) * 4096;
#pragma unroll
    for (int i = 0; i < 4; i++) wn[i] = next[wl_elem(0, i)];
    acc.mac(w, crow[k], k + 1 < len, mi.m, mi.minv);
  }
  acc.fold(mi.m, mi.minv);
#pragma unroll
  for (int i = 0; i < 4; i++)   // at most three chunks (45 sources): the sum of the parts is below 6m
    x[i] = csub(csub(csub(acc.r[i], 4 * mi.m), 2 * mi.m), mi.m);
}

// grid = (B, nlimbs)
template <bool FP>
__device__ __forceinline__ void ks12_front(const Ks12Args& a, u64* sm) {
  const u32 b = blockIdx.x, i = blockIdx.y;
  const Ks12Mod<FP> md(ks12_mod(a.mods, i));
  typename Ks12Tables<FP>::W w;
  w.load(Ks12Tables<FP>::inv(a, i));
  typename Ks12Mod<FP>::V x[4];
  ks12_load_d<FP>(x, a, b, i, md);
  u64 y[4];
  ulonglong2 sc;
  scalar_fetch(sc, a.up_scale, i);
  md.inverse(y, x, w, sc, sm);
  u64* dst = a.dcoef + ((size_t)b * a.nlimbs + i) * 4096;
#pragma unroll
  for (int k = 0; k < 4; k++) dst[wl_elem(0, k)] = ks12_split(y[k], md.mi.m);
}

// grid = (B * beta, next)
template <bool FP, bool NARROW>
__device__ __forceinline__ void ks12_digits(const Ks12Args& a, u64* sm) {
  const u32 b = blockIdx.x / a.beta, j = blockIdx.x % a.beta, t = blockIdx.y;
  const u32 lo = j * a.alpha, hi = min(lo + a.alpha, a.nlimbs);
  if (t >= lo && t < hi) return;   // the digit's own limbs stay as they are
  const u32 id = t < a.nlimbs ? t : t - a.nlimbs + a.nq;
  const Ks12Mod<FP> md(a.mods[id]);
  typename Ks12Tables<FP>::W w;
  w.load(Ks12Tables<FP>::fwd(a, id));
  const size_t row = (size_t)j * a.next + t;
  u64 y[4];
  ks12_convert<NARROW>(y, a.dcoef + ((size_t)b * a.nlimbs + lo) * 4096, hi - lo, scalar_words(a.up_mat + row * a.up_pitch),
                       *scalar_words(a.up_off + row), md.mi);
  typename Ks12Mod<FP>::V x[4];
#pragma unroll
  for (int k = 0; k < 4; k++) x[k] = md.load(y[k]);
  md.forward(x, w, sm);
  typename Ks12Mod<FP>::V* dst = (typename Ks12Mod<FP>::V*)a.ext + ((size_t)blockIdx.x * a.next + t) * 4096;
#pragma unroll
  for (int k = 0; k < 4; k++) dst[wl_elem(2, k)] = x[k];
}

// Inner product of ciphertext b's digits with key component c at extended limb t (modulus id), round-2 layout.
template <bool FP>
__device__ __forceinline__ void ks12_inner(typename Ks12Mod<FP>::V (&s)[4], const Ks12Args& a, u32 b, u32 c, u32 t, u32 id,
                                           const Ks12Mod<FP>& md) {
  const u64* evk = uniform_ptr(a.multi ? a.evk_pc[__builtin_amdgcn_readfirstlane(b)] : a.evk) + ((size_t)c * a.nm + id) * 4096;
#pragma unroll
  for (int k = 0; k < 4; k++) s[k] = 0;
  for (u32 j = 0; j < a.beta; j++) {
    const global_u64_ptr key = (global_u64_ptr)(evk + (size_t)j * 2 * a.nm * 4096);
    typename Ks12Mod<FP>::V x[4];
    if (t < a.nlimbs && t / a.alpha == j) {
      ks12_load_d<FP>(x, a, b, t, md);
    } else {
      const typename Ks12Mod<FP>::V* src = (const typename Ks12Mod<FP>::V*)a.ext + (((size_t)b * a.beta + j) * a.next + t) * 4096;
#pragma unroll
      for (int k = 0; k < 4; k++) x[k] = src[wl_elem(2, k)];
    }
#pragma unroll
    for (int k = 0; k < 4; k++) s[k] = md.mac(s[k], x[k], key[wl_elem(2, k)], j);
  }
#pragma unroll
  for (int k = 0; k < 4; k++) s[k] = md.settle(s[k]);
}

// grid = (2B, special limbs): back to coefficient form, scaled by (P/p_k)^-1 / N (times 2^64 on integer classes)
template <bool FP>
__device__ __forceinline__ void ks12_special(const Ks12Args& a, u64* sm) {
  const u32 bc = blockIdx.x, t = a.nlimbs + blockIdx.y, id = t - a.nlimbs + a.nq;
  const Ks12Mod<FP> md(ks12_mod(a.mods, id));
  typename Ks12Tables<FP>::W w;
  w.load(Ks12Tables<FP>::inv(a, id));
  typename Ks12Mod<FP>::V s[4];
  ks12_inner<FP>(s, a, bc >> 1, bc & 1, t, id, md);
  u64 y[4];
  ulonglong2 sc;
  scalar_fetch(sc, a.dn_scale, t - a.nlimbs);
  md.inverse(y, s, w, sc, sm);
  u64* o = a.acc + ((size_t)bc * a.next + t) * 4096;
#pragma unroll
  for (int k = 0; k < 4; k++) o[wl_elem(0, k)] = ks12_split(y[k], md.mi.m);
}

// grid = (2B, nlimbs)
template <bool FP, bool NARROW>
__device__ __forceinline__ void ks12_final(const Ks12Args& a, u64* sm) {
  const u32 bc = blockIdx.x, i = blockIdx.y, b = bc >> 1, c = bc & 1;
  const Ks12Mod<FP> md(ks12_mod(a.mods, i));
  typename Ks12Tables<FP>::W w;
  w.load(Ks12Tables<FP>::fwd(a, i));
  const size_t pl = (size_t)a.nlimbs * 4096, lo = (size_t)i * 4096;
  const u32 mode = c ? a.mode1 : a.mode0;
  const u32 g = a.multi ? a.galois_pc[__builtin_amdgcn_readfirstlane(b)] : a.add_galois;
  const u64* a2 = a.add2 + (a.add2_three ? (size_t)b * 3 + c : (size_t)bc) * pl + lo;
  const u64* as = a.add_src + (size_t)bc * pl + lo;
  u64 ev[4], ew[4];   // requested ahead of the transform
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const u32 n = wl_elem(2, k);
    if (mode & 1) ev[k] = a2[n];
    if (mode & 2) ew[k] = as[galois_src_index(n, g, 12)];
  }
  u64 y[4];
  ks12_convert<NARROW>(y, a.acc + ((size_t)bc * a.next + a.nlimbs) * 4096, a.next - a.nlimbs,
                       scalar_words(a.dn_mat + (size_t)i * a.dn_pitch), *scalar_words(a.dn_off + i), md.mi);
  typename Ks12Mod<FP>::V x[4];
#pragma unroll
  for (int k = 0; k < 4; k++) x[k] = md.load(y[k]);
  md.forward(x, w, sm);
  typename Ks12Mod<FP>::V s[4];
  ks12_inner<FP>(s, a, b, c, i, i, md);
  ulonglong2 pv;
  scalar_fetch(pv, a.pinv, i);
  const size_t o0 = (size_t)b * 2 * pl + lo, o1 = o0 + pl;
  u64* o = a.out + (size_t)bc * pl + lo;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const u32 n = wl_elem(2, k);
    typename Ks12Mod<FP>::V r = md.finish(s[k], x[k], pv);
    if (mode & 1) r = md.add(r, ev[k]);
    if (mode & 2) r = md.add(r, ew[k]);
    if (a.pa) {
      r = md.add_product(r, a.pa[o0 + n], c == 0 ? a.pb[o0 + n] : a.pb[o1 + n]);
      if (c) r = md.add_product(r, a.pa[o1 + n], a.pb[o0 + n]);
    }
    o[n] = md.result(r);
  }
}

// Both arithmetic kinds share a launch (the kind is uniform per workgroup): a second launch would cost more than the
// registers that the double-precision workgroups do not need. The kind comes with the arguments, not from the modulus: a trip to
// memory less before everything else can be requested (8 rotations of 4 limbs with their own keys 36.9 -> 35.2 us); but for the
// digits, whose integer workgroups start with the scalar loads of a conversion anyway (687 us that way, 693 this way in a
// matrix product with 18 rotations of one 55-bit limb; nothing between them in the others).
#define KS12_KERNEL(NAME, IS_FP, FP_BODY, INT_BODY)                           \
  __global__ void __launch_bounds__(WL_THREADS) NAME(Ks12Args a) {            \
    __shared__ u64 sm[WL_LDS_WORDS];                                          \
    if (IS_FP) FP_BODY(a, sm);                                                \
    else INT_BODY(a, sm);                                                     \
  }
__device__ __forceinline__ bool ks12_fp(const Ks12Args& a, u32 id) { return (a.fp_mask[id >> 5] >> (id & 31)) & 1; }
KS12_KERNEL(ks12_front_kernel, ks12_fp(a, blockIdx.y), ks12_front<true>, ks12_front<false>)
template <bool NARROW>
KS12_KERNEL(ks12_digits_kernel,
            mod_class(a.mods[blockIdx.y < a.nlimbs ? blockIdx.y : blockIdx.y - a.nlimbs + a.nq].m, a.fp_on) == 0,
            (ks12_digits<true, NARROW>), (ks12_digits<false, NARROW>))
KS12_KERNEL(ks12_special_kernel, ks12_fp(a, a.nq + blockIdx.y), ks12_special<true>, ks12_special<false>)
template <bool NARROW>
KS12_KERNEL(ks12_final_kernel, ks12_fp(a, blockIdx.y), (ks12_final<true, NARROW>), (ks12_final<false, NARROW>))
