// Host side of libckks_mi355: context tables, argument checks, launch sequences.
#include "../../include/ckks_mi355.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "kernels.hip.h"
#include "convert.hip.h"
#include "convert_wide.hip.h"
#include "ks12.hip.h"
#include "ntt16_kernels.hip.h"
#include "ntt_limb.hip.h"

typedef unsigned __int128 u128;

// Workspace of ckks_hrot_noalloc, the entry point for callers that cannot allocate: a fixed array in the library's
// own device image (one copy per GPU, held until the process ends). Host code never passes the array's name to a
// kernel or a copy: it uses the per-device address that hipGetSymbolAddress returns (ckks_ctx::scratch_ptr).
#define CKKS_NOALLOC_SCRATCH_BYTES (128ull << 20)
static __device__ __align__(256) unsigned char scratch[CKKS_NOALLOC_SCRATCH_BYTES];

namespace {

thread_local std::string g_err;

int fail(int code, const std::string& msg) {
  g_err = msg;
  return code;
}
#define HIP_TRY(expr)                                                                            \
  do {                                                                                           \
    hipError_t e_ = (expr);                                                                      \
    if (e_ != hipSuccess) return fail(CKKS_EHIP, std::string(#expr ": ") + hipGetErrorString(e_)); \
  } while (0)

// ---- host modular arithmetic (table generation only) ----
inline u64 h_mul(u64 a, u64 b, u64 m) { return (u64)((u128)a * b % m); }
u64 h_pow(u64 a, u64 e, u64 m) {
  u64 r = 1;
  a %= m;
  for (; e; e >>= 1) {
    if (e & 1) r = h_mul(r, a, m);
    a = h_mul(a, a, m);
  }
  return r;
}
inline u64 h_inv(u64 a, u64 m) { return h_pow(a, m - 2, m); }
inline u64 h_shoup(u64 w, u64 m) { return (u64)(((u128)w << 64) / m); }
inline u64 h_mont(u64 v, u64 m) { return (u64)(((u128)v << 64) % m); }  // v * 2^64 mod m
inline u64 h_mont90(u64 v, u64 m) { return h_mul(h_mont(v, m), (u64)(1ull << 26) % m, m); }  // v * 2^90 mod m
inline u32 h_bits(u64 v) {
  u32 b = 0;
  while (v) v >>= 1, b++;
  return b;
}
// Whether a base conversion with at most `n` sources below 2^bs into targets below 2^bt may use the three-sum
// accumulation and the base-2^30 reduction (dot30n_*): none of the three sums, including what the reduction adds
// to them, may reach 2^64.
inline bool bconv_narrow_ok(u32 n, u32 bs, u32 bt, u32 bt_min) {
  if (bs > 60 || bt > 60 || bt_min < 36) return false;  // the result is below m + 2^34 and gets one correction
  if (n > 15) n = 15;  // chunks of 15 terms are reduced separately
  const u128 one = 1, w = (one << 30) - 1;
  const u128 y1 = one << (bs > 30 ? bs - 30 : 0), c1 = one << (bt > 30 ? bt - 30 : 0);
  const u128 amax = (u128)n * w * w + (u128)n * w + w * w;
  const u128 bmax = (u128)n * (w * c1 + y1 * w) + (u128)n * c1 + (one << 34) + w * c1 + w * w;
  const u128 cmax = (u128)n * y1 * c1 + (one << 34) + w * c1 + w * w;
  const u128 lim = one << 64;
  return amax < lim && bmax < lim && cmax < lim;
}
bool h_is_prime(u64 n) {
  if (n < 2) return false;
  const u64 bases[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
  for (u64 b : bases)
    if (n % b == 0) return n == b;
  u64 d = n - 1;
  int r = 0;
  while (!(d & 1)) d >>= 1, r++;
  for (u64 a : bases) {
    u64 x = h_pow(a, d, n);
    if (x == 1 || x == n - 1) continue;
    bool composite = true;
    for (int i = 1; i < r && composite; i++) {
      x = h_mul(x, x, n);
      if (x == n - 1) composite = false;
    }
    if (composite) return false;
  }
  return true;
}
inline u32 h_brev(u32 x, u32 bits) {
  u32 r = 0;
  for (u32 i = 0; i < bits; i++) r |= ((x >> i) & 1) << (bits - 1 - i);
  return r;
}

// Rows of constants per target in up_mat / dn_mat (the smallest of these that covers n): what the kernels that read them are
// instantiated for (4, 8) or walk over.
inline u32 bconv_rows(u32 n) { return n <= 4 ? 4 : n <= 8 ? 8 : n <= 15 ? 15 : n <= 24 ? 24 : n <= 36 ? 36 : 45; }

// Base-conversion constants for ciphertexts at one limb count.
struct LevelTables {
  u32 nlimbs = 0, beta = 0, next = 0;
  bool narrow_up = false, narrow_dn = false, narrow_rs = false;  // which reduction the constants are scaled for
  ulonglong2* up_inv = nullptr;  // [beta][alpha]
  u64* up_mat = nullptr;         // [beta][alpha+1][next]
  ulonglong2* dn_inv = nullptr;  // [K]
  u64* dn_mat = nullptr;         // [K+1][nlimbs]
  ulonglong2* pinv = nullptr;    // [nlimbs]
  // two-pass path
  ulonglong2* up_scale = nullptr;  // [nlimbs]  (Q_j/q_i)^-1 / N mod q_i
  ulonglong2* dn_scale = nullptr;  // [K]       2^64 (P/p_k)^-1 / N mod p_k
  u64* dn_mat_plain = nullptr;     // dn_mat without the Montgomery factor
  // matrices of bytes of (Q_j/q_i) mod m_t ([beta][next]) and (P/p_k) mod q_i ([nlimbs]; on two-pass rings with 2^-64 on
  // integer-class targets), for conv_rows_kernel (at most 8 sources) or conv_wide_kernel
  uint4 *up_pieces = nullptr, *dn_pieces = nullptr;
  double *up_direct = nullptr, *dn_direct = nullptr;   // ConvArgs::direct: two-pass rings with every prime below 2^50
  u64* up_off = nullptr;           // [beta][next] -sum_i ((q_i-1)/2) (Q_j/q_i) mod m_t, scaled like up_mat
  u64* dn_off = nullptr;           // [nlimbs]     -sum_k ((p_k-1)/2) (P/p_k) mod q_i, scaled like dn_mat_plain
  u32 up_pitch = 0, dn_pitch = 0;  // constants per target in up_mat / dn_mat_plain
  ulonglong2* pinv2 = nullptr;     // [nlimbs]  2^64 / P mod q_i
  // rescale from this limb count: drop q_{nlimbs-1}
  uint4* rs_pieces = nullptr;      // [nlimbs-1] matrices of bytes of 1, for conv_rows_kernel
  ulonglong2* rs_scale = nullptr;  // [1]          1 / N mod q_last, in the form of its class
  ulonglong2* rs_one = nullptr;    // [1]          Shoup pair of 1 (the single source needs no pre-scaling)
  u64* rs_mat = nullptr;           // [nlimbs-1][5] row i = (1, 0, 0, 0, -q_last) mod q_i, Montgomery form
  ulonglong2* rs_qinv = nullptr;   // [nlimbs-1]   q_last^-1 mod q_i, Shoup pair
  ulonglong2* rs_qinv16 = nullptr; // same for the two-pass kernels: (c, c/q) doubles on double-precision moduli
};

}  // namespace

enum ProfKind {
  PK_NTT_FWD = 0, PK_NTT_INV,
  // two-pass kernels: three consecutive kinds each, one per modulus class (the kernel's template argument)
  PK_FWD_ROWS, PK_FWD_BLOCKS = PK_FWD_ROWS + 3, PK_INV_BLOCKS = PK_FWD_BLOCKS + 3, PK_INV_ROWS = PK_INV_BLOCKS + 3,
  PK_FWD_FINAL = PK_INV_ROWS + 3,
  PK_AUTOMORPH = PK_FWD_FINAL + 3, PK_MODUP, PK_INNER, PK_INNER16, PK_INNER16_INT, PK_INNER_C, PK_INNER8, PK_INNER8_BIG, PK_BCONV_ROWS, PK_MODDOWN = PK_BCONV_ROWS + 3, PK_FINAL, PK_TENSOR, PK_PMACC, PK_PMACC_FP, PK_ADD,
  PK_KS12_FRONT, PK_KS12_DIGITS, PK_KS12_SPECIAL, PK_KS12_FINAL, PK_CONV_ROWS, PK_COPY, PK_PMACC_STAGED, PK_PMACC_FP_STAGED, PK_COUNT
};
static const char* const kProfNames[PK_COUNT] = {
    "ntt_fwd_pass", "ntt_inv_pass",
    "ntt16_fwd_rows_kernel<0>", "ntt16_fwd_rows_kernel<1>", "ntt16_fwd_rows_kernel<2>",
    "ntt16_fwd_blocks_kernel<0>", "ntt16_fwd_blocks_kernel<1>", "ntt16_fwd_blocks_kernel<2>",
    "ntt16_inv_blocks_kernel<0>", "ntt16_inv_blocks_kernel<1>", "ntt16_inv_blocks_kernel<2>",
    "ntt16_inv_rows_kernel<0>", "ntt16_inv_rows_kernel<1>", "ntt16_inv_rows_kernel<2>",
    "ntt16_fwd_blocks_final_kernel<0>", "ntt16_fwd_blocks_final_kernel<1>", "ntt16_fwd_blocks_final_kernel<2>",
    "automorph_kernel", "modup_kernel", "inner_kernel", "inner16_fp_kernel", "inner16_int_kernel", "ntt16_fwd_blocks_inner_c_kernel", "ntt16_fwd_blocks_inner8_kernel<1>", "ntt16_fwd_blocks_inner8_kernel<2>",
    "ntt16_bconv_rows_kernel<0>", "ntt16_bconv_rows_kernel<1>", "ntt16_bconv_rows_kernel<2>", "moddown_kernel", "ks_final_kernel", "tensor_kernel",
    "pmacc_int_kernel", "pmacc_fp_kernel", "addto_kernel",
    "ks12_front_kernel", "ks12_digits_kernel", "ks12_special_kernel", "ks12_final_kernel", "conv_rows_kernel", "copy",
    "pmacc_int_staged_kernel", "pmacc_fp_staged_kernel"};
struct ProfRec {
  int kind;
  hipEvent_t start, stop;
};

struct ckks_ctx {
  // Tuning knobs (ckks_tune_set; meanings in the public header). 0: workgroup mapping of the two-pass kernels (-1: per
  // kernel); 1: integer bodies everywhere; 2: base conversions with the row passes on both sides of them (0, where they fit),
  // inside the following one (1) or kernels of their own (2); 3: 2 = inner product fused with the final assembly on
  // main limbs, 1 = separate kernels; 4: 0 = fork a row pass that is a kernel of its own onto the second
  // stream; 5: general base-conversion reduction; 6: integer PCMM inner sums; 7: cap on giant steps per pass.
  int tune[8] = {-1, 0, 0, 2, 1, 0, 0, 0};
  bool prof_on = false;
  std::vector<ProfRec> prof_recs;
  std::vector<hipEvent_t> prof_pool;
  double prof_ms[PK_COUNT] = {0};
  uint64_t prof_n[PK_COUNT] = {0};
  int device = 0;
  u32 logN = 0, N = 0, nq = 0, np = 0, nm = 0, dnum = 0, alpha = 0;
  std::vector<u64> mod, psi;
  ModInfo* d_mods = nullptr;
  ulonglong2* d_tw_fwd = nullptr;
  ulonglong2* d_tw_inv = nullptr;
  double* d_twfp_fwd = nullptr;  // N = 2^10 .. 2^16: the twiddles as doubles in [-q/2, q/2] for moduli < 2^50
  double* d_twfp_inv = nullptr;
  hipStream_t side = nullptr;       // second stream for the fork/join inside a key switch (default priority)
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  // Base-conversion constants of every limb count 1..nq, built when the context is created (and again when knob 1
  // or 5 changes): levels[nlimbs] points into one device allocation, d_levels.
  std::vector<LevelTables> levels;
  char* d_levels = nullptr;
  ConvReduction *d_conv_red = nullptr, *d_wide_red = nullptr;   // [nm] each, inside d_levels
  void* scratch_ptr = nullptr;  // this device's address of `scratch` (hipGetSymbolAddress at context creation)
};

namespace {

template <class T>
int upload(T** dst, const std::vector<T>& src) {
  HIP_TRY(hipMalloc((void**)dst, std::max<size_t>(1, src.size()) * sizeof(T)));
  if (!src.empty()) HIP_TRY(hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice));
  return CKKS_OK;
}

struct DeviceGuard {
  int prev = -1;
  bool ok = false;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) == hipSuccess && hipSetDevice(dev) == hipSuccess) ok = true;
  }
  ~DeviceGuard() {
    if (prev >= 0) (void)hipSetDevice(prev);
  }
};

// Brackets the launches made during its lifetime with two events on their stream (only when profiling is on).
struct ProfScope {
  ckks_ctx* c;
  hipStream_t st;
  ProfRec rec;
  bool active = false;
  ProfScope(const ckks_ctx* cc, int kind, hipStream_t s) : c(const_cast<ckks_ctx*>(cc)), st(s) {
    if (!c->prof_on) return;
    auto get = [&](hipEvent_t* e) {
      if (!c->prof_pool.empty()) {
        *e = c->prof_pool.back();
        c->prof_pool.pop_back();
        return true;
      }
      return hipEventCreate(e) == hipSuccess;
    };
    rec.kind = kind;
    if (!get(&rec.start)) return;
    if (!get(&rec.stop)) {
      c->prof_pool.push_back(rec.start);
      return;
    }
    active = hipEventRecord(rec.start, st) == hipSuccess;
  }
  ~ProfScope() {
    if (!active) return;
    (void)hipEventRecord(rec.stop, st);
    c->prof_recs.push_back(rec);
  }
};

// Host image of the device allocation that holds the level tables: every table starts on a 256-byte boundary; the
// LevelTables pointers hold offsets until the image has been uploaded.
struct LevelArena {
  std::vector<char> host;
  template <class T>
  T* add(const std::vector<T>& v) {
    const size_t off = (host.size() + 255) & ~(size_t)255;
    host.resize(off + std::max<size_t>(1, v.size()) * sizeof(T));
    if (!v.empty()) memcpy(host.data() + off, v.data(), v.size() * sizeof(T));
    return (T*)off;
  }
};

// The rows of one target in conv_rows_kernel's matrix of bytes (layout: ConvRows), for sources with constants c[0 .. n)
// that have `bytes` bytes (double-precision ones 7: the kernel leaves their signs in the eighth).
void conv_rows_of(std::vector<unsigned char>& out, size_t row, u32 groups, const u64* c, u32 n, u32 bytes, u64 m) {
  for (u32 k = 0; k < n; k++) {
    u64 v = c[k];
    for (u32 i = 0; i < bytes; i++) {
      const u64 w = ((v > m / 2 ? v - m : v) + 0x8080808080808080ull) ^ 0x8080808080808080ull;   // bytes in [-128, 127]
      for (u32 p = 0; p < CONV_PIECES; p++)
        out[(((row * groups + k / 4) * 2 + k / 2 % 2) * CONV_PIECES + p) * 16 + k % 2 * 8 + i] = (unsigned char)(w >> (8 * p));
      v = h_mul(v, 256, m);
    }
  }
}
// The same for target `slot` of digit j in conv_wide_kernel's matrices (layout there).
void wide_rows_of(std::vector<unsigned char>& out, u32 j, u32 slot, u32 quads, u32 groups, const u64* c, u32 n, u64 m) {
  for (u32 k = 0; k < n; k++) {
    u64 v = c[k];
    const size_t at = (((size_t)j * quads + slot / 4) * groups + k / 4) * 64 + k / 2 % 2 * 32;
    for (u32 i = 0; i < CONV_PIECES; i++) {
      const u64 w = ((v > m / 2 ? v - m : v) + 0x8080808080808080ull) ^ 0x8080808080808080ull;
      for (u32 p = 0; p < CONV_PIECES; p++)
        out[(at + (slot / 2 % 2 * 2 + p / 4) * 8 + slot % 2 * 4 + p % 4) * 16 + k % 2 * 8 + i] = (unsigned char)(w >> (8 * p));
      v = h_mul(v, 256, m);
    }
  }
}
// Groups of 4 sources that a conversion of n of them is done for: by conv_rows_kernel up to 8, by conv_wide_kernel beyond.
inline u32 conv_groups(u32 n) { return n <= 4 ? 1 : n <= CONV_MAX_SRC ? 2 : n <= 12 ? 3 : n <= 16 ? 4 : n <= 24 ? 6 : n <= 36 ? 9 : 12; }

// Constants for ciphertexts at `nlimbs` limbs, appended to the arena (pointers are offsets into it).
LevelTables build_level(const ckks_ctx* c, u32 nlimbs, LevelArena& arena) {
  const bool fp_on = c->tune[1] == 0;
  auto is_fp = [&](u64 m) { return fp_on && (m >> 50) == 0; };
  LevelTables t;
  t.nlimbs = nlimbs;
  t.beta = (nlimbs + c->alpha - 1) / c->alpha;
  t.next = nlimbs + c->np;
  const u32 alpha = c->alpha, K = c->np, next = t.next;
  auto ext_mod = [&](u32 s) { return s < nlimbs ? c->mod[s] : c->mod[c->nq + (s - nlimbs)]; };

  // constants of one output are contiguous: [digit][target][R+1], rows >= digit length are zero, row R = -Q_j
  const u32 R = bconv_rows(alpha), RK = bconv_rows(K);
  u32 bq = 0, bq_min = 64, bp = 0, bp_min = 64;
  for (u32 i = 0; i < nlimbs; i++) bq = std::max(bq, h_bits(c->mod[i])), bq_min = std::min(bq_min, h_bits(c->mod[i]));
  for (u32 k = 0; k < K; k++)
    bp = std::max(bp, h_bits(c->mod[c->nq + k])), bp_min = std::min(bp_min, h_bits(c->mod[c->nq + k]));
  t.narrow_up = c->tune[5] == 0 && bconv_narrow_ok(std::min(alpha, nlimbs), bq, std::max(bq, bp), std::min(bq_min, bp_min));
  t.narrow_dn = c->tune[5] == 0 && bconv_narrow_ok(K, bp, bq, bq_min);
  t.narrow_rs = c->tune[5] == 0 && bconv_narrow_ok(1, bq, bq, bq_min);
  auto mont_up = [&](u64 v, u64 m) { return t.narrow_up ? h_mont90(v, m) : h_mont(v, m); };
  auto mont_dn = [&](u64 v, u64 m) { return t.narrow_dn ? h_mont90(v, m) : h_mont(v, m); };
  auto mont_rs = [&](u64 v, u64 m) { return t.narrow_rs ? h_mont90(v, m) : h_mont(v, m); };
  std::vector<ulonglong2> up_inv((size_t)t.beta * alpha, ulonglong2{0, 0});
  std::vector<u64> up_mat((size_t)t.beta * next * (R + 1), 0), up_off((size_t)t.beta * next, 0);
  const u32 up_groups = conv_groups(alpha), dn_groups = conv_groups(K);
  const bool up_wide = alpha > CONV_MAX_SRC, dn_wide = K > CONV_MAX_SRC;
  auto pieces_bytes = [](u32 digits, u32 targets, u32 groups, bool wide) {
    return wide ? (size_t)digits * ((targets + 3) / 4) * groups * 1024 : (size_t)digits * targets * groups * 2 * CONV_PIECES * 16;
  };
  std::vector<unsigned char> up_pieces(pieces_bytes(t.beta, next, up_groups, up_wide), 0);
  std::vector<unsigned char> dn_pieces(pieces_bytes(1, nlimbs, dn_groups, dn_wide), 0);
  const bool all_fp = c->logN >= 13 && c->logN <= 16 && std::all_of(c->mod.begin(), c->mod.begin() + c->nm, is_fp);
  const bool up_vec = all_fp && alpha <= CONV_DIRECT_SRC, dn_vec = all_fp && K <= CONV_DIRECT_SRC;
  std::vector<double> up_direct(up_vec ? (size_t)t.beta * next * CONV_MAX_SRC : 0, 0.0);
  std::vector<double> dn_direct(dn_vec ? (size_t)nlimbs * CONV_MAX_SRC : 0, 0.0);
  auto centred = [](u64 v, u64 m) { return v > m / 2 ? -(double)(m - v) : (double)v; };
  std::vector<u64> up_plain((size_t)next * alpha), dn_plain((size_t)nlimbs * K);   // (Q_j/q_i) mod m_t of one digit, (P/p_k) mod q_i
  t.up_pitch = R + 1;
  t.dn_pitch = RK + 1;
  for (u32 j = 0; j < t.beta; j++) {
    u32 lo = j * alpha, hi = std::min(lo + alpha, nlimbs);
    for (u32 i = lo; i < hi; i++) {
      u64 qi = c->mod[i], h = 1;
      for (u32 k = lo; k < hi; k++)
        if (k != i) h = h_mul(h, c->mod[k] % qi, qi);
      u64 inv = h_inv(h, qi);
      up_inv[(size_t)j * alpha + (i - lo)] = ulonglong2{inv, h_shoup(inv, qi)};
      for (u32 s = 0; s < next; s++) {
        u64 m = ext_mod(s), v = 1;
        for (u32 k = lo; k < hi; k++)
          if (k != i) v = h_mul(v, c->mod[k] % m, m);
        up_plain[(size_t)s * alpha + (i - lo)] = v;
        if (up_vec) up_direct[((size_t)j * next + s) * CONV_MAX_SRC + (i - lo)] = centred(v, m);
        up_mat[((size_t)j * next + s) * (R + 1) + (i - lo)] = mont_up(v, m);
      }
    }
    for (u32 s = 0; s < next; s++) {
      const u64* plain = &up_plain[(size_t)s * alpha];
      if (up_wide) wide_rows_of(up_pieces, j, s, (next + 3) / 4, up_groups, plain, hi - lo, ext_mod(s));
      else conv_rows_of(up_pieces, (size_t)j * next + s, up_groups, plain, hi - lo, is_fp(c->mod[lo]) ? 7 : CONV_PIECES, ext_mod(s));
    }
    for (u32 s = 0; s < next; s++) {
      u64 m = ext_mod(s), v = 1;
      for (u32 k = lo; k < hi; k++) v = h_mul(v, c->mod[k] % m, m);
      up_mat[((size_t)j * next + s) * (R + 1) + R] = mont_up(v ? m - v : 0, m);
      // offset of the shifted-residue form: -sum_i h_i (Q_j/q_i), h_i = (q_i - 1) / 2
      u64 sum = 0;
      for (u32 i = lo; i < hi; i++)
        sum = (u64)(((u128)sum + h_mul(up_plain[(size_t)s * alpha + (i - lo)], ((c->mod[i] - 1) / 2) % m, m)) % m);
      up_off[(size_t)j * next + s] = mont_up(sum ? m - sum : 0, m);
    }
  }
  std::vector<ulonglong2> dn_inv(K), pinv(nlimbs);
  std::vector<u64> dn_mat((size_t)nlimbs * (RK + 1), 0);
  for (u32 k = 0; k < K; k++) {
    u64 pk = c->mod[c->nq + k], h = 1;
    for (u32 r = 0; r < K; r++)
      if (r != k) h = h_mul(h, c->mod[c->nq + r] % pk, pk);
    u64 inv = h_inv(h, pk);
    dn_inv[k] = ulonglong2{inv, h_shoup(inv, pk)};
    for (u32 i = 0; i < nlimbs; i++) {
      u64 m = c->mod[i], v = 1;
      for (u32 r = 0; r < K; r++)
        if (r != k) v = h_mul(v, c->mod[c->nq + r] % m, m);
      dn_plain[(size_t)i * K + k] = v;
      if (dn_vec) dn_direct[(size_t)i * CONV_MAX_SRC + k] = centred(v, m);
      dn_mat[(size_t)i * (RK + 1) + k] = mont_dn(v, m);
    }
  }
  for (u32 i = 0; i < nlimbs; i++) {
    u64 m = c->mod[i], v = 1;
    for (u32 r = 0; r < K; r++) v = h_mul(v, c->mod[c->nq + r] % m, m);
    dn_mat[(size_t)i * (RK + 1) + RK] = mont_dn(v ? m - v : 0, m);
    u64 inv = h_inv(v, m);
    pinv[i] = ulonglong2{inv, h_shoup(inv, m)};
  }
  // Constants of the two-pass path. 16-byte slots hold a Shoup pair (integer-class modulus) or the doubles
  // (c, c/q) (double-precision class). Integer-class accumulators carry a factor 2^-64 (Montgomery products), which
  // dn_scale and pinv2 undo; double-precision accumulators are plain.
  std::vector<ulonglong2> up_scale(nlimbs), dn_scale(K), pinv2(nlimbs);
  std::vector<u64> dn_mat_plain(dn_mat.size(), 0), dn_off(nlimbs, 0);
  auto as_fp = [](u64 v, u64 m) {
    double2 d{(double)v, (double)v / (double)m};
    ulonglong2 r;
    memcpy(&r, &d, sizeof(r));
    return r;
  };
  for (u32 i = 0; i < nlimbs; i++) {
    u64 m = c->mod[i], ninv = h_inv(c->N % m, m);
    u64 v = h_mul(up_inv[(size_t)(i / alpha) * alpha + (i % alpha)].x, ninv, m);
    u64 r64_inv = h_inv(h_mont(1, m), m);
    {
      u64 sum = 0;   // -sum_k h_k (P/p_k) mod m, then scaled like the row of constants below
      for (u32 k = 0; k < K; k++)
        sum = (u64)(((u128)sum + h_mul(dn_plain[(size_t)i * K + k], ((c->mod[c->nq + k] - 1) / 2) % m, m)) % m);
      const u64 neg = mont_dn(sum ? m - sum : 0, m);
      dn_off[i] = is_fp(m) ? neg : h_mul(neg, r64_inv, m);
    }
    if (is_fp(m)) {
      up_scale[i] = as_fp(v, m);
      pinv2[i] = as_fp(pinv[i].x, m);
      for (u32 k = 0; k <= RK; k++) dn_mat_plain[(size_t)i * (RK + 1) + k] = dn_mat[(size_t)i * (RK + 1) + k];
    } else {
      up_scale[i] = ulonglong2{v, h_shoup(v, m)};
      u64 w = h_mont(pinv[i].x, m);
      pinv2[i] = ulonglong2{w, h_shoup(w, m)};
      // stored constants are c * 2^64; multiply by 2^-64 so the Montgomery reduction leaves t * 2^-64
      for (u32 k = 0; k <= RK; k++)
        dn_mat_plain[(size_t)i * (RK + 1) + k] = h_mul(dn_mat[(size_t)i * (RK + 1) + k], r64_inv, m);
    }
  }
  for (u32 k = 0; k < K; k++) {
    u64 m = c->mod[c->nq + k], ninv = h_inv(c->N % m, m);
    u64 v = h_mul(dn_inv[k].x, ninv, m);
    if (is_fp(m)) {
      dn_scale[k] = as_fp(v, m);
    } else {
      u64 w = h_mont(v, m);
      dn_scale[k] = ulonglong2{w, h_shoup(w, m)};
    }
  }
  for (u32 i = 0; i < nlimbs; i++) {
    const u64 m = c->mod[i];
    u64* plain = &dn_plain[(size_t)i * K];
    if (!is_fp(m) && c->logN >= 13 && c->logN <= 16)
      for (u32 k = 0; k < K; k++) plain[k] = h_mul(plain[k], h_inv(h_mont(1, m), m), m);
    if (dn_wide) wide_rows_of(dn_pieces, 0, i, (nlimbs + 3) / 4, dn_groups, plain, K, m);
    else if (K) conv_rows_of(dn_pieces, i, dn_groups, plain, K, is_fp(c->mod[c->nq]) ? 7 : CONV_PIECES, m);
  }
  std::vector<ulonglong2> rs_one(1), rs_qinv(nlimbs > 1 ? nlimbs - 1 : 0), rs_qinv16(rs_qinv.size());
  std::vector<u64> rs_mat(rs_qinv.size() * 5, 0);
  rs_one[0] = ulonglong2{1, 0};  // floor(1 * 2^64 / q) is filled per use below; with x < q the product x*1 needs no reduction
  if (nlimbs > 1) {
    const u64 qL = c->mod[nlimbs - 1];
    rs_one[0] = ulonglong2{1, h_shoup(1, qL)};
    for (u32 i = 0; i + 1 < nlimbs; i++) {
      u64 m = c->mod[i], ql = qL % m, inv = h_inv(ql, m);
      rs_mat[(size_t)i * 5 + 0] = mont_rs(1, m);
      rs_mat[(size_t)i * 5 + 4] = mont_rs(ql ? m - ql : 0, m);
      rs_qinv[i] = ulonglong2{inv, h_shoup(inv, m)};
      rs_qinv16[i] = is_fp(m) ? as_fp(inv, m) : rs_qinv[i];
    }
  }
  std::vector<unsigned char> rs_pieces(pieces_bytes(1, nlimbs - 1, 1, false), 0);
  const u64 q_last = c->mod[nlimbs - 1], n_inv = h_inv(c->N % q_last, q_last), one = 1;
  for (u32 i = 0; i + 1 < nlimbs; i++) conv_rows_of(rs_pieces, i, 1, &one, 1, is_fp(q_last) ? 7 : CONV_PIECES, c->mod[i]);
  std::vector<ulonglong2> rs_scale(1, is_fp(q_last) ? as_fp(n_inv, q_last) : ulonglong2{n_inv, h_shoup(n_inv, q_last)});
  t.rs_pieces = (uint4*)arena.add(rs_pieces);
  t.rs_scale = arena.add(rs_scale);
  t.rs_one = arena.add(rs_one);
  t.rs_mat = arena.add(rs_mat);
  t.rs_qinv = arena.add(rs_qinv);
  t.rs_qinv16 = arena.add(rs_qinv16);
  t.up_scale = arena.add(up_scale);
  t.dn_scale = arena.add(dn_scale);
  t.dn_mat_plain = arena.add(dn_mat_plain);
  t.up_pieces = (uint4*)arena.add(up_pieces);
  t.dn_pieces = (uint4*)arena.add(dn_pieces);
  if (up_vec) t.up_direct = arena.add(up_direct);
  if (dn_vec) t.dn_direct = arena.add(dn_direct);
  t.up_off = arena.add(up_off);
  t.dn_off = arena.add(dn_off);
  t.pinv2 = arena.add(pinv2);
  t.up_inv = arena.add(up_inv);
  t.up_mat = arena.add(up_mat);
  t.dn_inv = arena.add(dn_inv);
  t.dn_mat = arena.add(dn_mat);
  t.pinv = arena.add(pinv);
  return t;
}

// (Re)build the tables of all limb counts under the current knobs 1 and 5: one allocation, one copy. Called from
// ckks_ctx_create and from ckks_tune_set, never from a call that enqueues work.
int build_levels(ckks_ctx* c) {
  LevelArena arena;
  std::vector<LevelTables> lv(c->nq + 1);
  for (u32 nl = 1; nl <= c->nq; nl++) lv[nl] = build_level(c, nl, arena);
  std::vector<ConvReduction> red(c->nm), wide(c->nm);   // (read on integer targets of 2^36, 2^50 or more)
  for (u32 i = 0; i < c->nm; i++) {
    const u64 m = c->mod[i];
    const u32 e = h_bits(m), sh = e > 51 ? e - 51 : 0;
    red[i] = ConvReduction{sh, e > CONV_INT_MIN_BITS ? -(int)((((u128)1 << (64 + sh)) + m / 2) / m) : 0};
  }
  for (u32 i = 0; i < c->nm; i++) {
    const u64 m = c->mod[i];
    const u32 e = h_bits(m), sh = e > 50 ? e - 48 : 0;
    wide[i] = ConvReduction{sh, e > 50 ? -(int)((((u128)1 << (64 + sh)) + m / 2) / m) : 0};
  }
  ConvReduction *d_red = arena.add(red), *d_wide = arena.add(wide);
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  char* dev = nullptr;
  HIP_TRY(hipMalloc((void**)&dev, arena.host.size()));
  hipError_t e = hipMemcpy(dev, arena.host.data(), arena.host.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(dev);
    return fail(CKKS_EHIP, std::string("uploading the level tables: ") + hipGetErrorString(e));
  }
  auto rebase = [&](auto*& ptr) { ptr = (std::remove_reference_t<decltype(ptr)>)(dev + (size_t)ptr); };
  for (u32 nl = 1; nl <= c->nq; nl++) {
    LevelTables& t = lv[nl];
    rebase(t.up_inv); rebase(t.up_mat); rebase(t.dn_inv); rebase(t.dn_mat); rebase(t.pinv);
    rebase(t.up_scale); rebase(t.dn_scale); rebase(t.dn_mat_plain); rebase(t.pinv2);
    rebase(t.up_pieces); rebase(t.dn_pieces); rebase(t.up_off); rebase(t.dn_off);
    if (t.up_direct) rebase(t.up_direct);
    if (t.dn_direct) rebase(t.dn_direct);
    rebase(t.rs_pieces); rebase(t.rs_scale); rebase(t.rs_one); rebase(t.rs_mat); rebase(t.rs_qinv); rebase(t.rs_qinv16);
  }
  if (c->d_levels) {
    // a knob changed: nothing may still be reading the old tables
    HIP_TRY(hipDeviceSynchronize());
    (void)hipFree(c->d_levels);
  }
  c->d_levels = dev;
  c->d_conv_red = (ConvReduction*)(dev + (size_t)d_red);
  c->d_wide_red = (ConvReduction*)(dev + (size_t)d_wide);
  c->levels.swap(lv);
  return CKKS_OK;
}

// Table look-up only: no allocation, no copy, no synchronisation.
int get_level(const ckks_ctx* c, u32 nlimbs, const LevelTables** out) {
  if (nlimbs == 0 || nlimbs >= c->levels.size()) return fail(CKKS_ESHAPE, "nlimbs must be in [1, L+1]");
  *out = &c->levels[nlimbs];
  return CKKS_OK;
}

LimbMap identity_map(u32 n) {
  LimbMap m;
  for (u32 i = 0; i < CKKS_MAX_SLOTS; i++) m.id[i] = (unsigned char)(i < n ? i : 0);
  return m;
}
// slots 0..nlimbs-1 -> q ids, then the K special primes
LimbMap ext_map(const ckks_ctx* c, u32 nlimbs) {
  LimbMap m = identity_map(nlimbs);
  for (u32 k = 0; k < c->np; k++) m.id[nlimbs + k] = (unsigned char)(c->nq + k);
  return m;
}

// Modulus class (must match mod_class() on the device).
inline int host_class(const ckks_ctx* c, u64 m) {
  if (c->tune[1] == 0 && (m >> 50) == 0) return 0;
  return (m >> 52) == 0 ? 1 : 2;
}
// Workgroup-to-tile mapping of the two-pass kernels (ntt16_map). Knob 0 >= 0 forces one mode everywhere; by default
// the transform passes and the final assembly, which share nothing but twiddles across polynomials, take the
// XCD-swizzled tile-major order (measured best for them), and the kernels that read the key take the
// group-per-XCD order when the batch shares one key (its slices then stay in that XCD's L2) and the plain
// tile-major order when every ciphertext has its own.
inline u32 map_mode_pass(const ckks_ctx* c) { return c->tune[0] >= 0 ? (u32)c->tune[0] : 3u; }
inline u32 map_mode_inner(const ckks_ctx* c, bool shared_key) {
  return c->tune[0] >= 0 ? (u32)c->tune[0] : shared_key ? 4u : 2u;
}
// The two-pass transforms and the kernels fused with them serve N = 2^13 .. 2^16. Below 2^13 a row pass would have fewer
// rows than one radix-16 round; 2^17 needs 512 rows, more than a 4096-element tile with whole 128-byte lines holds. What
// they replaced on 2^13 .. 2^15 was the stage-by-stage ntt_pass_kernel with one kernel per step of a key switch (a
// butterfly's operands through LDS every stage, integer arithmetic throughout): 12 rotations at 2^14 (5 limbs) 287 -> 117 us,
// 8 products at 2^15 (13 limbs) 833 -> 348 us. Whole transforms of 2^13 and most of 2^14 hold a limb per workgroup instead (limb_whole).
inline bool two_pass(const ckks_ctx* c) { return c->logN >= 13 && c->logN <= 16; }
// Ring 2^12: a key switch in four kernels that hold a whole limb per workgroup (ks12.hip.h). 8 rotations with their own
// keys (4 limbs, 2 digits), which took ten launches each: 322 -> 37 us; 8 rotations of one key (5 limbs, 3 digits) 60 -> 46 us.
// A target rereads all sources of its conversion there, so large batches of many limbs are left to one kernel per step, which
// reads a source once: from 100 MB of converted digits on (what the caches no longer hold) where a workgroup rereads two limbs or
// more on average. One key, us, this way | by steps: 16 + 4 limbs, 4 digits, batch 32 162 | 176, 64 350 | 333, 512 2971 | 2386;
// products of it at 64 380 | 348; 16 + 8 60-bit limbs, 2 digits, batch 64 335 | 334, 128 740 | 629; 8 + 8 limbs, 1 digit, 128
// 295 | 311, 512 1291 | 1117; 8 + 2 limbs, 4 digits (1.6 limbs reread) 512 1212 | 1215, products of it (2.1) 1327 | 1299; 5 + 2
// limbs, 3 digits (1.3) 512 695 | 714. A key per ciphertext always goes this way: by steps it is one sequence per ciphertext.
bool whole_limb(const ckks_ctx* c, u32 B, u32 nlimbs, bool product) {
  if (c->logN != 12) return false;
  const u32 beta = (nlimbs + c->alpha - 1) / c->alpha, next = nlimbs + c->np, workgroups = (beta + 2) * next;
  u32 reread = 2 * nlimbs * c->np + (product ? 4 * nlimbs : 0);
  for (u32 lo = 0; lo < nlimbs; lo += c->alpha) {
    const u32 len = std::min(c->alpha, nlimbs - lo);
    reread += len * (next - len);
  }
  return (u64)B * beta * next < 3072 || reread < 2 * workgroups;
}
// Both kinds read what they switch through the Galois map and take separate addends and per-ciphertext keys.
bool gathers(const ckks_ctx* c, u32 B, u32 nlimbs) { return two_pass(c) || whole_limb(c, B, nlimbs, false); }
inline u32 pass_tiles(const ckks_ctx* c) { return c->N >> 12; }   // 4096-element tiles of a limb

// One launch per modulus class present among `nslots` slots, a.slots listing that class's slots: launch(cls, grid).
// class_of_slot(slot) < 0 leaves a slot out.
template <class Args, class ClassOf, class Launch>
void launch_by_class(const ckks_ctx* c, int kind_base, Args& a, u32 nx, u32 nslots, ClassOf class_of_slot, hipStream_t st,
                     Launch launch) {
  for (int cls = 0; cls < 3; cls++) {
    u32 cnt = 0;
    for (u32 s = 0; s < nslots; s++)
      if (class_of_slot(s) == cls) a.slots[cnt++] = (unsigned char)s;
    if (!cnt) continue;
    ProfScope ps(c, kind_base + cls, st);
    launch(cls, dim3(nx, pass_tiles(c), cnt));
  }
}
#define LAUNCH_CLASS_KERNEL(KERNEL, CLS, GRID, STREAM, ARGS)                                             \
  do {                                                                                                   \
    if ((CLS) == 0) hipLaunchKernelGGL((KERNEL<0>), GRID, dim3(NTT16_THREADS), 0, STREAM, ARGS);         \
    else if ((CLS) == 1) hipLaunchKernelGGL((KERNEL<1>), GRID, dim3(NTT16_THREADS), 0, STREAM, ARGS);    \
    else hipLaunchKernelGGL((KERNEL<2>), GRID, dim3(NTT16_THREADS), 0, STREAM, ARGS);                    \
  } while (0)
// the row passes are instantiated per number of rows, N / 256
template <int LOGR>
void launch_rows_of(bool inverse, int cls, dim3 grid, hipStream_t st, const Ntt16Args& a) {
  const dim3 block(NTT16_THREADS);
  if (inverse) {
    if (cls == 0) hipLaunchKernelGGL((ntt16_inv_rows_kernel<0, LOGR>), grid, block, 0, st, a);
    else if (cls == 1) hipLaunchKernelGGL((ntt16_inv_rows_kernel<1, LOGR>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((ntt16_inv_rows_kernel<2, LOGR>), grid, block, 0, st, a);
  } else {
    if (cls == 0) hipLaunchKernelGGL((ntt16_fwd_rows_kernel<0, LOGR>), grid, block, 0, st, a);
    else if (cls == 1) hipLaunchKernelGGL((ntt16_fwd_rows_kernel<1, LOGR>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((ntt16_fwd_rows_kernel<2, LOGR>), grid, block, 0, st, a);
  }
}
void launch_rows(u32 logN, bool inverse, int cls, dim3 grid, hipStream_t st, const Ntt16Args& a) {
  switch (logN) {
    case 13: launch_rows_of<5>(inverse, cls, grid, st, a); break;
    case 14: launch_rows_of<6>(inverse, cls, grid, st, a); break;
    case 15: launch_rows_of<7>(inverse, cls, grid, st, a); break;
    default: launch_rows_of<8>(inverse, cls, grid, st, a); break;
  }
}

struct NttOpts {
  u32 galois = 0;                     // two-pass inverse only: read src through the eval-domain Galois map
  const u64* src_b = nullptr;         // two-pass inverse only: transform the products of src and src_b
  const u32* galois_pc = nullptr;     // same, one element per polynomial (host array, npoly <= KS_MULTI_MAX entries)
  const ulonglong2* scale = nullptr;  // two-pass inverse only: per-slot constants (from slot0) replacing N^-1
  bool split_out = false;             // N = 2^16 inverse only: write the shifted, split form the fused base conversion reads
  bool rows_only = false;             // two-pass only: only the row pass (forward: a fused kernel does the rest; inverse: one did the block pass)
  bool blocks_only = false;           // two-pass only: only the block pass (forward: in place on dst)
  bool raw_out = false;               // with blocks_only: leave reduced doubles on double-precision moduli
  int only_class = -1;                // >= 0: touch only the slots of this modulus class
  int exclude_class = -1;             // >= 0: leave the slots of this modulus class alone
  // a whole transform of all slots, canonical residues in and out
  bool plain() const {
    return !galois && !src_b && !galois_pc && !scale && !split_out && !rows_only && !blocks_only && !raw_out && only_class < 0 &&
           exclude_class < 0;
  }
};
// Whether a whole transform holds a limb per workgroup (ntt_limb.hip.h): always up to 2^13. A limb of 2^14 takes a compute unit's
// LDS, so a round is 256 limbs, and one that is not half full leaves units idle that the two-pass kernels, four workgroups a limb,
// would use. us for n limbs of one arithmetic kind, both forms in turn (two-pass | whole), forward: 50-bit primes n = 32 11.4 | 16.0, 128
// 17.7 | 17.7, 144 19.8 | 17.3, 288 29.0 | 33.3, 400 41.0 | 35.1, 544 49.8 | 52.7, 656 57.8 | 54.7; 60-bit ones 32 13.5 | 21.2, 144
// 25.1 | 22.9, 656 70.8 | 68.8, 900 93.3 | 91.7 (51-bit ones 88.8 | 91.2). Their inverses gain later: 60-bit ones 144 26.9 | 25.7, 656 76.6 | 78.5, 720 82.8 | 80.2.
// With the rounds the gain shrinks, since loads and stores of a unit's only workgroup do not overlap with its stages, and where those
// take longer (inverses, and the spills of integer ones) it turns: 50-bit inverses 1024 87.9 | 85.1, 1450 117 | 120; 51-bit primes
// forward 1024 97.2 | 94.7, 1450 133 | 137, inverse 512 60.1 | 55.9, 700 78.8 | 80.7, 1200 120 | 134; 60-bit inverses 768 85.2 | 83.3, 1024
// 108 | 109, 1200 124 | 134. From eight rounds on (256 MB, what the last-level cache holds) a pass over memory less decides: 2100
// limbs forward 188 | 158, 60-bit ones 228 | 197, inverse 190 | 177; integer inverses 2100 231 | 234, 2304 261 | 251. Limbs of two kinds are
// two launches a pass for the two-pass kernels: 4 limbs 22.5 | 20.1 us, 256 36.0 | 24.0, 1280 119 | 103.
#define LIMB_MAX_LOGN 14
bool limb_whole(const ckks_ctx* c, bool inverse, u32 npoly, u32 nslots, const LimbMap& ids) {
  if (c->logN < LIMB_MAX_LOGN) return true;
  if (c->logN > LIMB_MAX_LOGN) return false;
  const int cls = host_class(c, c->mod[ids.id[0]]);
  for (u32 s = 1; s < nslots; s++)
    if (host_class(c, c->mod[ids.id[s]]) != cls) return true;
  const u64 limbs = (u64)npoly * nslots, full = (limbs - 1) / 256, last = limbs - full * 256;
  if (full >= 8) return !inverse || cls == 0 || full > 8 || last > 128;
  static const u32 rounds[2][3] = {{8, 4, 8}, {4, 2, 3}};   // [inverse][class] that the whole form is ahead for
  return full < rounds[inverse][cls] && last > (full < 2 || cls == 0 || (cls == 2 && !inverse) ? 128 : 192);
}
template <int LOGN>
void launch_limb_kernel(bool inverse, dim3 grid, hipStream_t st, const LimbArgs& a) {
  if (inverse) hipLaunchKernelGGL((ntt_limb_kernel<LOGN, true>), grid, dim3(Limb<LOGN>::THREADS), 0, st, a);
  else hipLaunchKernelGGL((ntt_limb_kernel<LOGN, false>), grid, dim3(Limb<LOGN>::THREADS), 0, st, a);
}
int launch_limbs(const ckks_ctx* c, bool inverse, const u64* src, u64 src_stride, u64* dst, u64 dst_stride, u32 npoly, u32 slot0,
                 u32 nslots, const LimbMap& ids_from_slot0, u32 skip_beta, u32 skip_nq, hipStream_t st) {
  LimbArgs a;
  a.src = src + (size_t)slot0 * c->N;
  a.dst = dst + (size_t)slot0 * c->N;
  a.tw = inverse ? c->d_tw_inv : c->d_tw_fwd;
  a.twfp = inverse ? c->d_twfp_inv : c->d_twfp_fwd;
  a.mods = c->d_mods;
  a.src_poly_stride = src_stride;
  a.dst_poly_stride = dst_stride;
  a.skip_beta = skip_beta;
  a.skip_alpha = c->alpha;
  a.skip_nq = skip_nq;
  a.fp_on = c->tune[1] == 0 ? 1u : 0u;
  for (u32 i = 0; i < 128; i++) a.id[i] = ids_from_slot0.id[i];
  const u32 chunk = 65535 - (skip_beta ? 65535 % skip_beta : 0);   // whole digit groups
  for (u32 p0 = 0; p0 < npoly; p0 += chunk) {
    LimbArgs b = a;
    b.src += (size_t)p0 * src_stride;
    b.dst += (size_t)p0 * dst_stride;
    const dim3 grid(std::min<u32>(chunk, npoly - p0), nslots);
    ProfScope ps(c, inverse ? PK_NTT_INV : PK_NTT_FWD, st);
    switch (c->logN) {
      case 10: launch_limb_kernel<10>(inverse, grid, st, b); break;
      case 11: launch_limb_kernel<11>(inverse, grid, st, b); break;
      case 12: launch_limb_kernel<12>(inverse, grid, st, b); break;
      case 13: launch_limb_kernel<13>(inverse, grid, st, b); break;
      default: launch_limb_kernel<14>(inverse, grid, st, b); break;
    }
  }
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}
// Enqueue a transform of npoly polynomials x slots [slot0, slot0+nslots): reads src, writes dst (src == dst for an
// in-place transform). Rows are *_stride elements apart.
int launch_ntt(const ckks_ctx* c, bool inverse, const u64* src, u64 src_stride, u64* dst, u64 dst_stride, u32 npoly,
               u32 slot0, u32 nslots, const LimbMap& ids_from_slot0, u32 skip_beta, u32 skip_nq, hipStream_t st,
               const NttOpts& opt = NttOpts()) {
  if (npoly == 0 || nslots == 0) return CKKS_OK;
  const int kind = inverse ? PK_NTT_INV : PK_NTT_FWD;
  if (opt.plain() && limb_whole(c, inverse, npoly, nslots, ids_from_slot0))
    return launch_limbs(c, inverse, src, src_stride, dst, dst_stride, npoly, slot0, nslots, ids_from_slot0, skip_beta, skip_nq, st);
  if (two_pass(c)) {
    Ntt16Args a;
    a.logN = c->logN;
    a.src = src + (size_t)slot0 * c->N;
    a.src_b = opt.src_b ? opt.src_b + (size_t)slot0 * c->N : nullptr;
    a.dst = dst + (size_t)slot0 * c->N;
    a.tw = inverse ? c->d_tw_inv : c->d_tw_fwd;
    a.twfp = inverse ? c->d_twfp_inv : c->d_twfp_fwd;
    a.mods = c->d_mods;
    a.src_poly_stride = src_stride;
    a.dst_poly_stride = dst_stride;
    a.skip_beta = skip_beta;
    a.skip_alpha = c->alpha;
    a.skip_nq = skip_nq;
    for (u32 i = 0; i < 128; i++) a.id[i] = ids_from_slot0.id[i];
    a.map_mode = map_mode_pass(c);
    a.galois = opt.galois;
    if (opt.galois_pc) {
      if (npoly > KS_MULTI_MAX) return fail(CKKS_ESHAPE, "internal: per-polynomial Galois elements for too many polynomials");
      a.multi = 1;
      for (u32 i = 0; i < npoly; i++) a.galois_pc[i] = opt.galois_pc[i];
    }
    a.scale = opt.scale;
    a.raw_out = opt.raw_out ? 1 : 0;
    a.split_out = opt.split_out ? 1 : 0;
    Ntt16Args b = a;  // second pass: in place on dst
    b.src = a.dst;
    b.src_poly_stride = dst_stride;
    auto cls_of = [&](u32 s) {
      int k = host_class(c, c->mod[ids_from_slot0.id[s]]);
      if (opt.only_class >= 0 && k != opt.only_class) return -1;
      if (opt.exclude_class >= 0 && k == opt.exclude_class) return -1;
      return k;
    };
    auto rows = [&](Ntt16Args& r, int kind_base) {
      launch_by_class(c, kind_base, r, npoly, nslots, cls_of, st,
                      [&](int cls, dim3 grid) { launch_rows(c->logN, inverse, cls, grid, st, r); });
    };
    if (!inverse) {
      if (!opt.blocks_only) rows(a, PK_FWD_ROWS);
      if (!opt.rows_only)
        launch_by_class(c, PK_FWD_BLOCKS, b, npoly, nslots, cls_of, st,
                        [&](int cls, dim3 grid) { LAUNCH_CLASS_KERNEL(ntt16_fwd_blocks_kernel, cls, grid, st, b); });
    } else {
      if (!opt.rows_only)
        launch_by_class(c, PK_INV_BLOCKS, a, npoly, nslots, cls_of, st,
                        [&](int cls, dim3 grid) {
                          if (cls == 1 && a.src_b) hipLaunchKernelGGL((ntt16_inv_blocks_kernel<1, true>), grid, dim3(NTT16_THREADS), 0, st, a);
                          else if (cls == 2 && a.src_b) hipLaunchKernelGGL((ntt16_inv_blocks_kernel<2, true>), grid, dim3(NTT16_THREADS), 0, st, a);
                          else LAUNCH_CLASS_KERNEL(ntt16_inv_blocks_kernel, cls, grid, st, a);
                        });
      if (!opt.blocks_only) rows(b, PK_INV_ROWS);
    }
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
  }
  // 2^17: stages 0 .. 8 and 9 .. 16 on tiles of 4096 elements
  if (!opt.plain()) return fail(CKKS_EINVAL, "internal: a part of a transform on a ring that has only whole ones");
  if (src != dst) {
    ProfScope ps(c, PK_COPY, st);
    // in place: copy the slots first (rows may be strided)
    HIP_TRY(hipMemcpy2DAsync(dst + (size_t)slot0 * c->N, dst_stride * 8, src + (size_t)slot0 * c->N, src_stride * 8,
                             (size_t)nslots * c->N * 8, npoly, hipMemcpyDeviceToDevice, st));
  }
  NttArgs a;
  a.data = dst + (size_t)slot0 * c->N;
  a.tw = inverse ? c->d_tw_inv : c->d_tw_fwd;
  a.mods = c->d_mods;
  a.poly_stride = dst_stride;
  a.logN = c->logN;
  a.skip_beta = skip_beta;
  a.skip_alpha = c->alpha;
  a.skip_nq = skip_nq;
  a.ids = ids_from_slot0;
  a.tile_log = 12;
  for (int pass = 0; pass < 2; pass++) {
    const bool first = inverse ? pass == 1 : pass == 0;
    a.s0 = first ? 0 : 9;
    a.k = first ? 9 : 8;
    a.logC = first ? 3 : 0;
    dim3 grid(npoly, c->N >> a.tile_log, nslots);
    size_t lds = sizeof(u64) << a.tile_log;
    ProfScope ps(c, kind, st);
    if (inverse)
      hipLaunchKernelGGL(ntt_pass_kernel<true>, grid, dim3(NTT_THREADS), lds, st, a);
    else
      hipLaunchKernelGGL(ntt_pass_kernel<false>, grid, dim3(NTT_THREADS), lds, st, a);
  }
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}

u32 inv_mod_pow2(u32 g, u32 bits) {  // inverse of odd g modulo 2^bits
  u32 x = 1;
  for (int i = 0; i < 6; i++) x *= 2 - g * x;
  return x & ((bits >= 32) ? 0xFFFFFFFFu : ((1u << bits) - 1));
}

int launch_automorph(const ckks_ctx* c, u64* out, u64 out_stride, const u64* in, u64 in_stride, u32 npoly, u32 nslots,
                     const LimbMap& ids, u32 g, bool eval_domain, hipStream_t st) {
  if (npoly == 0 || nslots == 0) return CKKS_OK;
  AutoArgs a;
  a.out = out;
  a.in = in;
  a.mods = c->d_mods;
  a.out_poly_stride = out_stride;
  a.in_poly_stride = in_stride;
  a.logN = c->logN;
  a.g = g;
  a.g_inv = inv_mod_pow2(g, c->logN + 1);
  a.eval_domain = eval_domain ? 1 : 0;
  a.ids = ids;
  ProfScope ps(c, PK_AUTOMORPH, st);
  hipLaunchKernelGGL(automorph_kernel, dim3(c->N / 256, nslots, npoly), dim3(256), 0, st, a);
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct KsLayout {
  size_t dcoef, ext, acc, tq, total;
};
KsLayout ks_layout(const ckks_ctx* c, u32 B, u32 nlimbs) {
  const size_t N = c->N, next = nlimbs + c->np, beta = (nlimbs + c->alpha - 1) / c->alpha;
  KsLayout L;
  size_t off = 0;
  L.dcoef = off; off += align256((size_t)B * nlimbs * N * 8);
  L.ext = off;   off += align256((size_t)B * beta * next * N * 8);
  L.acc = off;   off += align256((size_t)B * 2 * next * N * 8);
  L.tq = off;    off += align256((size_t)B * 2 * nlimbs * N * 8);
  L.total = off;
  return L;
}

// Base-conversion launches, two adjacent coefficients per lane.
template <bool PRESCALED, bool NARROW>
void launch_modup_n(const ckks_ctx* c, const ModUpArgs& a, u32 beta, u32 B, hipStream_t st) {
  dim3 block(BCONV_THREADS), grid(c->N / BCONV_THREADS / 2, beta, B);
  if (c->alpha <= 4) hipLaunchKernelGGL((modup_kernel<4, PRESCALED, NARROW>), grid, block, 0, st, a, a.dcoef, a.ext, a.mods, a.mat);
  else hipLaunchKernelGGL((modup_kernel<8, PRESCALED, NARROW>), grid, block, 0, st, a, a.dcoef, a.ext, a.mods, a.mat);
}
// Conversions of more than 8 sources, on the matrix cores.
void launch_wide(const WideArgs& a, u32 digits, u32 npoly, hipStream_t st) {
  const dim3 block(WIDE_THREADS), grid(std::max(1u, (1u << a.logN) / WIDE_THREADS), digits, npoly);
  switch (conv_groups(a.alpha)) {
    case 3: hipLaunchKernelGGL(conv_wide_kernel<3>, grid, block, 0, st, a); break;
    case 4: hipLaunchKernelGGL(conv_wide_kernel<4>, grid, block, 0, st, a); break;
    case 6: hipLaunchKernelGGL(conv_wide_kernel<6>, grid, block, 0, st, a); break;
    case 9: hipLaunchKernelGGL(conv_wide_kernel<9>, grid, block, 0, st, a); break;
    default: hipLaunchKernelGGL(conv_wide_kernel<12>, grid, block, 0, st, a); break;
  }
}
template <bool PRESCALED>
void launch_modup(const ckks_ctx* c, const LevelTables* lt, const ModUpArgs& a, u32 beta, u32 B, hipStream_t st) {
  const bool narrow = lt->narrow_up;
  if (c->alpha > CONV_MAX_SRC) {
    WideArgs w;
    w.src = a.dcoef;
    w.dst = a.ext;
    w.src_poly_stride = (u64)a.nlimbs << a.logN;
    w.dst_poly_stride = (u64)a.next << a.logN;
    w.pieces = lt->up_pieces;
    w.red = c->d_wide_red;
    w.mods = c->d_mods;
    w.inv = PRESCALED ? nullptr : lt->up_inv;
    w.logN = a.logN;
    w.src_slot0 = w.src_id0 = 0;
    w.src_nlimbs = a.nlimbs;
    w.alpha = c->alpha;
    w.beta = beta;
    w.skip_own = 1;
    w.ntarget = a.next;
    w.main = a.nlimbs;
    w.special = c->nq;
    return launch_wide(w, beta, B, st);
  }
  if (narrow) launch_modup_n<PRESCALED, true>(c, a, beta, B, st);
  else launch_modup_n<PRESCALED, false>(c, a, beta, B, st);
}
template <bool PRESCALED, bool NARROW>
void launch_moddown_n(const ckks_ctx* c, const ModDownArgs& a, u32 B2, hipStream_t st) {
  dim3 block(BCONV_THREADS), grid(c->N / BCONV_THREADS / 2, B2);
  if (a.K <= 4) hipLaunchKernelGGL((moddown_kernel<4, PRESCALED, NARROW>), grid, block, 0, st, a, a.acc, a.tq, a.mods, a.mat);
  else hipLaunchKernelGGL((moddown_kernel<8, PRESCALED, NARROW>), grid, block, 0, st, a, a.acc, a.tq, a.mods, a.mat);
}
template <bool PRESCALED>
void launch_moddown(const ckks_ctx* c, const LevelTables* lt, const ModDownArgs& a, u32 B2, bool narrow, hipStream_t st) {
  if (a.K > CONV_MAX_SRC) {
    WideArgs w;
    w.src = a.acc;
    w.dst = a.tq;
    w.src_poly_stride = (u64)a.next << a.logN;
    w.dst_poly_stride = (u64)a.nlimbs << a.logN;
    w.pieces = lt->dn_pieces;
    w.red = c->d_wide_red;
    w.mods = c->d_mods;
    w.inv = PRESCALED ? nullptr : lt->dn_inv;
    w.logN = a.logN;
    w.src_slot0 = a.src_slot;
    w.src_id0 = a.src_id0;
    w.src_nlimbs = w.alpha = a.K;
    w.beta = 1;
    w.skip_own = 0;
    w.ntarget = w.main = a.nlimbs;
    w.special = 0;
    return launch_wide(w, 1, B2, st);
  }
  if (narrow) launch_moddown_n<PRESCALED, true>(c, a, B2, st);
  else launch_moddown_n<PRESCALED, false>(c, a, B2, st);
}

// What a key switch reads and how its result is assembled.
struct KsIo {
  const u64* d;          // polynomial to switch, eval domain; limb-vector (b, i) at d + b*d_stride + i*N
  u64 d_stride;
  u32 d_galois;          // != 0: d is read through the eval-domain Galois map (HRot's sigma(c1)); two-pass path only
  u64* out;              // [B][2][nlimbs][N]
  u32 mode[2];           // per component: bit 0: + add2 (out itself when null); bit 1: + sigma_g(add_src) (two-pass path only)
  const u64* add_src;    // [B][2][nlimbs][N]
  u32 add_galois;
  // two-pass path, B <= KS_MULTI_MAX: ciphertext b uses galois_pc[b] (for d and add_src) and the key evk_pc[b]
  const u32* galois_pc = nullptr;
  const u64* const* evk_pc = nullptr;
  const u64* add2 = nullptr;   // [B][2][nlimbs][N] plain addend of mode bit 0 (two-pass path); null = out, in place
  bool add2_three = false;     // add2 is [B][3][nlimbs][N]; its first two components are the addends
  // ring 2^12, and two-pass rings with knob 3 at its default (mode {4, 4}): d is the product of the second components of two
  // ciphertexts [B][2][nlimbs][N], whose other two product terms are the addends
  const u64 *prod_a = nullptr, *prod_b = nullptr;
  bool steps = false;          // ring 2^12: one kernel per step (whole_limb said no)
};

// Base conversion fused with the first forward pass (ntt16_bconv_rows_kernel): one launch per modulus class among
// the `ntarget` target slots. class_of_slot(slot) < 0 leaves a slot out.
template <class ClassOf>
int launch_bconv_rows(const ckks_ctx* c, BconvRowsArgs a, u32 npoly, bool narrow, ClassOf class_of_slot, hipStream_t st) {
  if (npoly > 65535) return fail(CKKS_ESHAPE, "batch too large for one launch");
  a.tw = c->d_tw_fwd;
  a.twfp = c->d_twfp_fwd;
  a.mods = c->d_mods;
  // the targets of a polynomial on one XCD, whose L2 then serves the shared source tiles, tiles fastest
  a.map_mode = c->tune[0] >= 0 ? (u32)c->tune[0] : 5u;
  a.npoly = npoly;
  const u32 grid_poly = a.map_mode == 5 ? (npoly + 7) / 8 * 8 : npoly;
  for (int cls = 0; cls < 3; cls++) {
    u32 cnt = 0;
    for (u32 s = 0; s < a.ntarget; s++)
      if (class_of_slot(s) == cls) a.slots[cnt++] = (unsigned char)s;
    if (!cnt) continue;
    const dim3 grid(cnt, 16, grid_poly), block(NTT16_THREADS);
    ProfScope ps(c, PK_BCONV_ROWS + cls, st);
#define LAUNCH_BCONV(CLS)                                                                              \
  if (narrow) hipLaunchKernelGGL((ntt16_bconv_rows_kernel<CLS, true>), grid, block, 0, st, a);         \
  else hipLaunchKernelGGL((ntt16_bconv_rows_kernel<CLS, false>), grid, block, 0, st, a)
    if (cls == 0) { LAUNCH_BCONV(0); }
    else if (cls == 1) { LAUNCH_BCONV(1); }
    else { LAUNCH_BCONV(2); }
#undef LAUNCH_BCONV
  }
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}

// Whether the conversion of digits of `alpha` limbs with modulus ids [id0, id0 + n) runs inside the transform passes around it
// (conv_rows_kernel): the kernel keeps up to 8 sources per position, all of one arithmetic kind. Knob 2 = 0 (the default) allows it. One prime of
// another kind among the main limbs leaves the whole polynomial to the separate kernels, also its digits of one kind. So does an
// integer target below 2^36 (only where knob 1 makes it one), which the reduction of the sums does not take.
bool conv_fits(const ckks_ctx* c, u32 id0, u32 n, u32 alpha) {
  if (c->tune[2] != 0 || alpha > CONV_MAX_SRC) return false;
  const bool fp = host_class(c, c->mod[id0]) == 0;
  for (u32 i = 1; i < n; i++)
    if ((host_class(c, c->mod[id0 + i]) == 0) != fp) return false;
  for (u32 i = 0; i < c->nm; i++)
    if (host_class(c, c->mod[i]) != 0 && h_bits(c->mod[i]) <= CONV_INT_MIN_BITS) return false;
  return true;
}
// A fused conversion about to be launched. READY: the sources' inverse row pass runs in a kernel of its own before it.
struct ConvJob {
  ConvArgs a;
  u32 npoly;
  bool fp, ready;
};
template <int LOGR>
void launch_conv_direct(const ConvJob& j, dim3 grid, hipStream_t st) {
  const dim3 block(CONV_THREADS);
  if (j.a.alpha <= 4) hipLaunchKernelGGL((conv_rows_kernel<LOGR, 4, true, false, true>), grid, block, 0, st, j.a);
  else if (j.ready) hipLaunchKernelGGL((conv_rows_kernel<LOGR, CONV_DIRECT_SRC, true, true, true>), grid, block, 0, st, j.a);
  else hipLaunchKernelGGL((conv_rows_kernel<LOGR, CONV_DIRECT_SRC, true, false, true>), grid, block, 0, st, j.a);
}
template <int LOGR, int MAXLEN, bool READY>
void launch_conv_len(const ConvJob& j, dim3 grid, hipStream_t st) {
  const dim3 block(CONV_THREADS);
  if (j.fp) hipLaunchKernelGGL((conv_rows_kernel<LOGR, MAXLEN, true, READY>), grid, block, 0, st, j.a);
  else hipLaunchKernelGGL((conv_rows_kernel<LOGR, MAXLEN, false, READY>), grid, block, 0, st, j.a);
}
#define CONV_READY_MIN_SRC 6
template <int LOGR>
void launch_conv_of(const ConvJob& j, dim3 grid, hipStream_t st) {
  if (j.a.direct) launch_conv_direct<LOGR>(j, grid, st);
  else if (j.a.alpha <= 4) launch_conv_len<LOGR, 4, false>(j, grid, st);
  else if (j.ready) launch_conv_len<LOGR, 8, true>(j, grid, st);
  else launch_conv_len<LOGR, 8, false>(j, grid, st);
}
// Modelled time of a conversion whose targets are dealt to n workgroups (shares) per (polynomial, tile): two fit a compute unit, and
// a lone one runs at two thirds of their joint rate. Every share repeats what is done for the sources (wsrc). Weights are
// relative numbers of instructions per limb: a target 4 (217 vector instructions a lane) or, integer, 7 (384), a source 4 or 6.
inline u64 conv_cost(u64 groups, u32 wsrc, u32 wtargets, u32 n) {
  const u64 per_cu = (groups * n + 255) / 256;
  return (per_cu / 2 * 8 + per_cu % 2 * 6) * (wsrc + (wtargets + n - 1) / n);
}
// The number of shares: a call on few ciphertexts needs several to fill the chip. What the shares repeat costs a caller nothing
// while the chip is his alone, but costs the others when several calls are in flight: the fewest shares within a
// quarter of the best time that leave no round of workgroups under three quarters full, one share within 10 % (the best, for
// calls that occupy under a quarter of the chip anyway).
u32 conv_shares(u64 groups, u32 wsrc, u32 wtargets, u32 targets) {
  u64 best = ~0ull;
  u32 at = 1;
  for (u32 n = 1; n <= targets; n++) {
    const u64 cost = conv_cost(groups, wsrc, wtargets, n);
    if (cost < best) best = cost, at = n;
  }
  if (groups <= 64) return at;
  if (conv_cost(groups, wsrc, wtargets, 1) * 100 <= best * 110) return 1;
  for (u32 n = 2; n < at; n++) {
    const u64 rounds = (groups * n + 255) / 256;
    if (conv_cost(groups, wsrc, wtargets, n) * 100 <= best * 125 && groups * n * 4 >= rounds * 256 * 3) return n;
  }
  return at;
}
// job.a: everything but the tables of the ring, the target lists and nsplit; target_id(slot) = modulus id of a target slot.
template <class TargetId>
void conv_plan(const ckks_ctx* c, ConvJob& job, TargetId target_id) {
  ConvArgs& a = job.a;
  a.tw = c->d_tw_fwd;
  a.twi = c->d_tw_inv;
  a.twfp = c->d_twfp_fwd;
  a.twifp = c->d_twfp_inv;
  a.mods = c->d_mods;
  a.red = c->d_conv_red;
  a.nfp = a.nint = 0;
  for (int fp = 1; fp >= 0; fp--)
    for (u32 s = 0; s < a.ntarget; s++) {
      const u32 id = target_id(s);
      if ((host_class(c, c->mod[id]) == 0) != (fp == 1)) continue;
      const u32 n = a.nfp + a.nint;
      a.target[n] = s | id << 8;
      if (fp) a.nfp++;
      else a.nint++;
    }
  job.fp = host_class(c, c->mod[a.src_id0]) == 0;
  const u32 len = std::min(a.alpha, a.src_nlimbs), own = a.skip_own ? len : 0;   // own limbs: of the sources' kind, not converted
  const u32 targets = a.nfp + a.nint - own, wtargets = (a.nfp - (job.fp ? own : 0)) * 4 + (a.nint - (job.fp ? 0 : own)) * 7;
  const u64 groups = (u64)job.npoly * (c->N / CONV_TILE);
  // From 6 sources on, and where one share would take over a tenth longer than several (a quarter with double-precision sources,
  // whose inverse pass is cheaper), the sources' inverse row pass runs by itself before the shares instead of in each of them
  // (else its launch costs more than the repeats). us, the inverse pass in every share and the best number of them | this: one
  // rotation of 24 limbs, 3 digits, 8 special primes 138.7 | 133.4, four 364.4 | 358.2, one of 16 + 8 60-bit limbs 120.5 | 107.7.
  const u32 wsrc = len * (job.fp ? 4 : 6);
  u32 n = conv_shares(groups, wsrc, wtargets, targets);
  const u64 one = conv_cost(groups, wsrc, wtargets, 1), several = conv_cost(groups, wsrc, wtargets, n);
  job.ready = len >= CONV_READY_MIN_SRC && one * 100 > several * (job.fp ? 125 : 110);
  if (job.ready) n = conv_shares(groups, len, wtargets, targets);
  a.nsplit = n;
}
int launch_conv_rows(const ckks_ctx* c, const ConvJob& job, hipStream_t st) {
  const u64 blocks = (u64)job.npoly * (c->N / CONV_TILE) * job.a.nsplit;
  if (blocks > 0x7FFFFFFFull) return fail(CKKS_ESHAPE, "batch too large for one launch");
  const dim3 grid((u32)blocks);
  ProfScope ps(c, PK_CONV_ROWS, st);
  switch (c->logN) {
    case 13: launch_conv_of<5>(job, grid, st); break;
    case 14: launch_conv_of<6>(job, grid, st); break;
    case 15: launch_conv_of<7>(job, grid, st); break;
    default: launch_conv_of<8>(job, grid, st); break;
  }
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}
// ModUp on the two-pass path, from the inverse block pass of the polynomial (in dcoef; its row pass too if the plan says ready)
// to ext after the row pass.
ConvJob conv_up_job(const ckks_ctx* c, const LevelTables* lt, const u64* dcoef, u64* ext, u32 B, u32 nlimbs) {
  ConvJob job;
  ConvArgs& a = job.a;
  a.src = dcoef;
  a.dst = ext;
  a.src_poly_stride = (u64)nlimbs * c->N;
  a.dst_poly_stride = (u64)lt->next * c->N;
  a.src_slot0 = a.src_id0 = 0;
  a.src_nlimbs = nlimbs;
  a.alpha = c->alpha;
  a.beta = lt->beta;
  a.skip_own = 1;
  a.ntarget = lt->next;
  a.pieces = lt->up_pieces;
  a.direct = lt->up_direct;
  a.scale = lt->up_scale;
  job.npoly = B * lt->beta;
  conv_plan(c, job, [&](u32 s) { return s < nlimbs ? s : s - nlimbs + c->nq; });
  return job;
}
// ModDown: both accumulators' special limbs to tq.
ConvJob conv_down_job(const ckks_ctx* c, const LevelTables* lt, const u64* acc, u64* tq, u32 B, u32 nlimbs) {
  ConvJob job;
  ConvArgs& a = job.a;
  a.src = acc;
  a.dst = tq;
  a.src_poly_stride = (u64)lt->next * c->N;
  a.dst_poly_stride = (u64)nlimbs * c->N;
  a.src_slot0 = nlimbs;
  a.src_id0 = c->nq;
  a.src_nlimbs = a.alpha = c->np;
  a.beta = 1;
  a.skip_own = 0;
  a.ntarget = nlimbs;
  a.pieces = lt->dn_pieces;
  a.direct = lt->dn_direct;
  a.scale = lt->dn_scale;
  job.npoly = B * 2;
  conv_plan(c, job, [](u32 s) { return s; });
  return job;
}

// ModDown's conversion and the first forward pass of its result on the two-pass path: the special limbs of both
// accumulators back to coefficient form (scaled by (P/p_k)^-1 / N), P -> Q_l, stages 0..7; tq receives the converted
// limbs in row-pass form. Knob 2 = 1 does the conversion inside the row pass (ntt16_bconv_rows_kernel).
// int_blocks_done: the integer-class special limbs have been through their inverse block pass.
int ks16_moddown_rows(ckks_ctx* c, const LevelTables* lt, u32 B, u32 nlimbs, u64* acc, u64* tq, hipStream_t st,
                      bool int_blocks_done = false) {
  int rc;
  const u32 N = c->N, next = lt->next, K = c->np;
  const bool fused = c->tune[2] == 1 && c->logN == 16;
  const bool conv = conv_fits(c, c->nq, K, K);
  LimbMap pmap;
  for (u32 k = 0; k < CKKS_MAX_SLOTS; k++) pmap.id[k] = (unsigned char)(k < K ? c->nq + k : 0);
  NttOpts o3;
  o3.scale = lt->dn_scale;
  o3.split_out = fused;
  ConvJob job;
  if (conv) {
    job = conv_down_job(c, lt, acc, tq, B, nlimbs);
    o3.blocks_only = !job.ready;
  }
  auto inverse = [&](const NttOpts& o) {
    return launch_ntt(c, true, acc, (u64)next * N, acc, (u64)next * N, B * 2, nlimbs, K, pmap, 0, 0, st, o);
  };
  if (int_blocks_done) {
    NttOpts blocks = o3, rows = o3;
    blocks.blocks_only = true;
    blocks.only_class = 0;
    rows.rows_only = true;
    if ((rc = inverse(blocks))) return rc;
    if (!o3.blocks_only && (rc = inverse(rows))) return rc;
  } else if ((rc = inverse(o3))) {
    return rc;
  }
  if (conv) return launch_conv_rows(c, job, st);
  if (!fused) {
    {
      ModDownArgs a{acc, tq, c->d_mods, lt->dn_inv, lt->dn_mat_plain, c->logN, nlimbs, c->nq, K, next, nlimbs, c->nq};
      ProfScope ps(c, PK_MODDOWN, st);
      launch_moddown<true>(c, lt, a, B * 2, lt->narrow_dn, st);
      HIP_TRY(hipGetLastError());
    }
    NttOpts o2;
    o2.rows_only = true;
    return launch_ntt(c, false, tq, (u64)nlimbs * N, tq, (u64)nlimbs * N, B * 2, 0, nlimbs, identity_map(nlimbs), 0, 0, st, o2);
  }
  BconvRowsArgs a;
  a.src = acc;
  a.dst = tq;
  a.mat = lt->dn_mat_plain;
  a.off = lt->dn_off;
  a.src_poly_stride = (u64)next * N;
  a.dst_poly_stride = (u64)nlimbs * N;
  a.src_slot0 = nlimbs;
  a.src_nlimbs = K;
  a.alpha = K;
  a.beta = 1;
  a.skip_own = 0;
  a.ntarget = nlimbs;
  a.pitch = lt->dn_pitch;
  for (u32 i = 0; i < 128; i++) a.id[i] = (unsigned char)(i < nlimbs ? i : 0);
  return launch_bconv_rows(c, a, B * 2, lt->narrow_dn, [&](u32 s) { return host_class(c, c->mod[s]); }, st);
}

// Last kernel of a key switch on the two-pass path: block pass of tq fused with (acc - tq) / P and the addends.
// int_only leaves the double-precision limbs to another kernel.
int ks16_assemble(ckks_ctx* c, const LevelTables* lt, const KsIo& io, u32 B, u32 nlimbs, const u64* acc, const u64* tq,
                  hipStream_t st, bool int_only = false) {
  FwdFinalArgs a;
  a.tq = tq;
  a.acc = acc;
  a.out = io.out;
  a.add_src = io.add_src;
  a.add2 = io.add2 ? io.add2 : io.out;
  a.add2_three = io.add2 && io.add2_three ? 1u : 0u;
  a.tw = c->d_tw_fwd;
  a.twfp = c->d_twfp_fwd;
  a.mods = c->d_mods;
  a.pinv = lt->pinv2;
  a.logN = c->logN;
  a.nlimbs = nlimbs;
  a.next = lt->next;
  a.mode0 = io.mode[0];
  a.mode1 = io.mode[1];
  a.galois = io.add_galois;
  if (io.galois_pc) {
    a.multi = 1;
    for (u32 i = 0; i < B; i++) a.galois_pc[i] = io.galois_pc[i];
  }
  a.map_mode = map_mode_pass(c);
  auto cls_of = [&](u32 s) {
    const int k = host_class(c, c->mod[s]);
    return int_only && k == 0 ? -1 : k;
  };
  launch_by_class(c, PK_FWD_FINAL, a, B * 2, nlimbs, cls_of, st,
                  [&](int cls, dim3 grid) { LAUNCH_CLASS_KERNEL(ntt16_fwd_blocks_final_kernel, cls, grid, st, a); });
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}

// Second half of a key switch on the two-pass path: from the accumulators (all slots) to the assembled output.
// acc_in: accumulators held outside the workspace ([B][2][next][N]; their special-prime slots are overwritten).
int ks16_finish(ckks_ctx* c, const LevelTables* lt, const KsIo& io, u32 B, u32 nlimbs, char* ws, hipStream_t st,
                u64* acc_in = nullptr) {
  int rc;
  KsLayout L = ks_layout(c, B, nlimbs);
  u64* acc = acc_in ? acc_in : (u64*)(ws + L.acc);
  u64* tq = (u64*)(ws + L.tq);
  if ((rc = ks16_moddown_rows(c, lt, B, nlimbs, acc, tq, st))) return rc;
  return ks16_assemble(c, lt, io, B, nlimbs, acc, tq, st);
}

void launch_inner_c(const ckks_ctx* c, u32 B, u32 nslots, const FwdInnerArgs& a, hipStream_t st) {
  const dim3 grid(B * 2, pass_tiles(c), nslots), block(NTT16_THREADS);
  switch (c->logN) {
    case 13: hipLaunchKernelGGL(ntt16_fwd_blocks_inner_c_kernel<13>, grid, block, 0, st, a); break;
    case 14: hipLaunchKernelGGL(ntt16_fwd_blocks_inner_c_kernel<14>, grid, block, 0, st, a); break;
    case 15: hipLaunchKernelGGL(ntt16_fwd_blocks_inner_c_kernel<15>, grid, block, 0, st, a); break;
    default: hipLaunchKernelGGL(ntt16_fwd_blocks_inner_c_kernel<16>, grid, block, 0, st, a); break;
  }
}

// Whether the integer-class main limbs store their sums beside the special limbs' (step 3) and are assembled from there, instead of
// taking all digits and both corrections in line at the end of the call (step 5). The former costs a write and a read of the sums;
// it is faster where the workgroups of both are one round and the digits are many, so that a lone limb's chain is what the call
// ends with. us, in line | stored: 4 rotations at 2^13, one 60-bit limb and four smaller in 5 digits 114.0 | 107.3; one at 2^15, 1 + 12
// limbs in 5 digits 137.2 | 131.1, at 2^16, 1 + 23 in 4 digits 208.8 | 204.8; 4 at 2^14, 6 60-bit limbs in 6 digits 85.7 | 74.6. With
// two digits (4 of 1 + 3 limbs at 2^13) 85.4 | 88.0, with four and no double-precision limb (16 of 4 limbs at 2^13) 73.9 | 74.7, beyond
// a round (one of 14 60-bit limbs in 5 digits at 2^16, 544 workgroups) 129.0 | 130.4; at 512 (16 of 1 + 3 limbs at 2^15) 187.7 | 188.0.
// A product also needs the kernel that forms its three terms then, which reads and writes whole limbs: up to 2^20 words of a batch's
// polynomial (one of 2 + 12 limbs at 2^16, 2^19.8 words, 163.6 | 159.6; 2 of 1 + 14, 2^20.9, 251 | 256).
bool int_sums_stored(const ckks_ctx* c, u32 B, u32 nlimbs, bool product) {
  u32 mains = 0, specials = 0;
  for (u32 i = 0; i < nlimbs; i++) mains += host_class(c, c->mod[i]) != 0;
  for (u32 k = 0; k < c->np; k++) specials += host_class(c, c->mod[c->nq + k]) != 0;
  const u32 beta = (nlimbs + c->alpha - 1) / c->alpha;
  return mains && beta >= (mains < nlimbs ? 4 : 5) && (u64)B * (c->N / 2048) * (mains + specials) <= 512 &&
         (!product || (u64)B * nlimbs * c->N <= 1u << 20);
}

// Two-pass path: transforms fused with their neighbours.
//   1. INTT(d) with (Q_j/q_i)^-1 / N folded in
//   2. ModUp conversion and row pass of every slot a digit does not own
//      (1's row pass and 2 are one kernel where conv_fits; else kernels of their own, knob 2 = 1: one fused kernel for 2)
//   3. integer-class slots (the special primes): [block pass + evk inner product] (x 2^-64 from the Montgomery products)
//   4. INTT of the special limbs with 2^64 (P/p_k)^-1 / N folded in (of the integer-class ones step 3 has done the block pass, in
//      the registers that hold the sums: one launch and a write and read of both accumulators less; 64 rotations with their own
//      keys 5623 -> 5383 us, one rotation 147 -> 139); ModDown conversion and row pass (as step 2)
//   5. double-precision main limbs: [block pass of the digits + evk inner product + block pass of the ModDown
//      correction + (sum - correction) / P + addends] in one kernel, so their accumulators never reach memory;
//      integer-class main limbs the same in theirs (the kernel of step 3, carried to the end), or by the assembly kernel from sums
//      that step 3 stored (int_sums_stored).
// With knob 3 = 1 the main limbs' accumulators are stored (integer-class ones by step 3, double-precision ones by a plain block
// pass and a streaming product) and the assembly kernel replaces step 5. With knob 4 = 0 the double-precision row pass of step 2,
// where it is a kernel of its own, runs on the context's second stream beside the integer-class kernels of step 3 and step 4, which
// do not depend on it, and is joined before the first kernel that reads what it leaves: step 5's, or with knob 3 = 1 the block
// pass of step 3.
// acc_add != null (knob 3 at its default only): the sequence stops before ModDown and ADDS the two accumulators, plus
// P * sigma(io.add_src component 0) on the main primes of the first, to acc_add ([B][2][next][N]).
int keyswitch_fused16(ckks_ctx* c, const LevelTables* lt, const KsIo& io, u32 B, u32 nlimbs, const u64* evk, char* ws,
                      hipStream_t st, u64* acc_add = nullptr) {
  int rc;
  const u32 N = c->N, next = lt->next, beta = lt->beta;
  KsLayout L = ks_layout(c, B, nlimbs);
  u64* dcoef = (u64*)(ws + L.dcoef);
  u64* ext = (u64*)(ws + L.ext);
  u64* acc = (u64*)(ws + L.acc);
  u64* tq = (u64*)(ws + L.tq);
  const LimbMap qmap = identity_map(nlimbs), emap = ext_map(c, nlimbs);
  if (io.galois_pc && B > KS_MULTI_MAX) return fail(CKKS_ESHAPE, "internal: per-ciphertext keys for too many ciphertexts");
  const bool fused_fp = c->tune[3] != 1;
  if (acc_add && !fused_fp) return fail(CKKS_EINVAL, "internal: accumulation needs the default inner kernels");
  auto ext_class = [&](u32 s) { return host_class(c, c->mod[emap.id[s]]); };
  bool any_fp = false, any_int = false, special_fp = false;
  for (u32 s_ = 0; s_ < next; s_++) {
    const bool fp = ext_class(s_) == 0;
    any_fp |= fp;
    any_int |= !fp;
    if (s_ >= nlimbs) special_fp |= fp;
  }
  const bool fused_up = c->tune[2] == 1 && c->logN == 16;
  const bool conv_up = conv_fits(c, 0, nlimbs, c->alpha);
  // 1.
  NttOpts o1;
  o1.galois = io.d_galois;
  o1.galois_pc = io.galois_pc;
  o1.scale = lt->up_scale;
  o1.split_out = fused_up;
  ConvJob up;
  if (conv_up) {
    up = conv_up_job(c, lt, dcoef, ext, B, nlimbs);
    o1.blocks_only = !up.ready;
  }
  const u64 polyN = (u64)nlimbs * N;
  if (io.prod_a) o1.src_b = io.prod_b + polyN;
  if ((rc = launch_ntt(c, true, io.prod_a ? io.prod_a + polyN : io.d, io.prod_a ? 2 * polyN : io.d_stride, dcoef, polyN, B, 0,
                       nlimbs, qmap, 0, 0, st, o1)))
    return rc;
  // 2. The double-precision part of the row pass (memory-bound) may run on the second stream beside the
  // integer-class chain of steps 2-4 (arithmetic-bound), which does not depend on it.
  const bool fork = any_fp && any_int && !special_fp && !acc_add && !conv_up && c->tune[4] == 0;
  hipStream_t sb = st;
  if (conv_up) {
    if ((rc = launch_conv_rows(c, up, st))) return rc;
  } else if (!fused_up) {
    ModUpArgs a{dcoef, ext, c->d_mods, lt->up_inv, lt->up_mat, c->logN, nlimbs, c->nq, c->alpha, beta, next};
    ProfScope ps(c, PK_MODUP, st);
    launch_modup<true>(c, lt, a, beta, B, st);
    HIP_TRY(hipGetLastError());
  }
  if (fork) {
    sb = c->side;
    HIP_TRY(hipEventRecord(c->ev_fork, st));
    HIP_TRY(hipStreamWaitEvent(sb, c->ev_fork, 0));
  }
  if (!conv_up && !fused_up) {
    NttOpts o2;
    o2.rows_only = true;
    if (any_fp) {
      NttOpts o = o2;
      o.only_class = 0;
      if ((rc = launch_ntt(c, false, ext, (u64)next * N, ext, (u64)next * N, B * beta, 0, next, emap, beta, nlimbs, sb, o)))
        return rc;
    }
    if (any_int) {
      NttOpts o = o2;
      o.exclude_class = 0;
      if ((rc = launch_ntt(c, false, ext, (u64)next * N, ext, (u64)next * N, B * beta, 0, next, emap, beta, nlimbs, st, o)))
        return rc;
    }
  } else if (fused_up) {
    BconvRowsArgs up;
    up.src = dcoef;
    up.dst = ext;
    up.mat = lt->up_mat;
    up.off = lt->up_off;
    up.src_poly_stride = (u64)nlimbs * N;
    up.dst_poly_stride = (u64)next * N;
    up.src_slot0 = 0;
    up.src_nlimbs = nlimbs;
    up.alpha = c->alpha;
    up.beta = beta;
    up.skip_own = 1;
    up.ntarget = next;
    up.pitch = lt->up_pitch;
    for (u32 i = 0; i < 128; i++) up.id[i] = emap.id[i];
    if (any_fp &&
        (rc = launch_bconv_rows(c, up, B * beta, lt->narrow_up, [&](u32 s) { return ext_class(s) == 0 ? 0 : -1; }, sb)))
      return rc;
    if (any_int &&
        (rc = launch_bconv_rows(c, up, B * beta, lt->narrow_up, [&](u32 s) { return ext_class(s) == 0 ? -1 : ext_class(s); }, st)))
      return rc;
  }
  if (fork) HIP_TRY(hipEventRecord(c->ev_join, sb));
  FwdInnerArgs ia;
  ia.ext = ext;
  ia.d = io.d;
  ia.d_poly_stride = io.d_stride;
  ia.evk = evk;
  ia.acc = acc;
  ia.tw = c->d_tw_fwd;
  ia.twfp = c->d_twfp_fwd;
  ia.mods = c->d_mods;
  ia.logN = c->logN;
  ia.nlimbs = nlimbs;
  ia.nq = c->nq;
  ia.nm = c->nm;
  ia.alpha = c->alpha;
  ia.beta = beta;
  ia.next = next;
  ia.map_mode = map_mode_inner(c, io.galois_pc == nullptr);
  ia.galois = io.d_galois;
  ia.ext_galois = 0;
  if (io.galois_pc) {
    ia.multi = 1;
    for (u32 i = 0; i < B; i++) ia.galois_pc[i] = io.galois_pc[i], ia.evk_pc[i] = io.evk_pc[i];
  }
  if (acc_add) {
    ia.acc = acc_add;
    ia.accumulate = 1;
    ia.c0 = io.add_src;
    ia.c0_poly_stride = 2 * (u64)nlimbs * N;
  }
  // 3. integer-class slots, 8 values per lane (grid.y = tiles of 8 blocks): the special ones, which go on through their inverse
  // block pass, and the main ones where their accumulators are needed in memory
  if (!acc_add) ia.twi = c->d_tw_inv;
  auto launch_inner8 = [&](FwdInnerArgs a, bool special, bool main_slots, bool fin) {
    for (int cls = 1; cls <= 2; cls++) {
      u32 cnt = 0;
      for (u32 s_ = 0; s_ < next; s_++)
        if (ext_class(s_) == cls && (s_ >= nlimbs ? special : main_slots)) a.slots[cnt++] = (unsigned char)s_;
      if (!cnt) continue;
      ProfScope ps(c, PK_INNER8 + cls - 1, st);
      const dim3 grid(B, N / 2048, cnt), block(256);
      if (fin && cls == 1) hipLaunchKernelGGL((ntt16_fwd_blocks_inner8_kernel<1, true>), grid, block, 0, st, a);
      else if (fin) hipLaunchKernelGGL((ntt16_fwd_blocks_inner8_kernel<2, true>), grid, block, 0, st, a);
      else if (cls == 1) hipLaunchKernelGGL((ntt16_fwd_blocks_inner8_kernel<1, false>), grid, block, 0, st, a);
      else hipLaunchKernelGGL((ntt16_fwd_blocks_inner8_kernel<2, false>), grid, block, 0, st, a);
    }
  };
  const bool stored = fused_fp && !acc_add && !io.prod_a && int_sums_stored(c, B, nlimbs, false);
  launch_inner8(ia, true, acc_add || !fused_fp || stored, false);
  HIP_TRY(hipGetLastError());
  // double-precision slots whose accumulators are needed in memory: the special ones always (ModDown reads them),
  // the main ones when the result is accumulated or when the fusion of step 5 is switched off
  auto launch_inner_fp = [&](bool special, bool main_slots, hipStream_t s) -> int {
    FwdInnerArgs a = ia;
    u32 cnt = 0;
    for (u32 s_ = 0; s_ < next; s_++)
      if (ext_class(s_) == 0 && (s_ >= nlimbs ? special : main_slots)) a.slots[cnt++] = (unsigned char)s_;
    if (!cnt) return CKKS_OK;
    if (fused_fp) {
      ProfScope ps(c, PK_INNER_C, s);
      launch_inner_c(c, B, cnt, a, s);
    } else {
      // plain block pass of every converted double-precision slot (own limbs are skipped), then a streaming product
      NttOpts o;
      o.blocks_only = true;
      o.raw_out = true;
      o.only_class = 0;
      int r2 = launch_ntt(c, false, ext, (u64)next * N, ext, (u64)next * N, B * beta, 0, next, emap, beta, nlimbs, s, o);
      if (r2) return r2;
      ProfScope ps(c, PK_INNER16, s);
      hipLaunchKernelGGL(inner16_fp_kernel, dim3(B, N / 512, cnt), dim3(256), 0, s, a);
    }
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
  };
  if (special_fp || acc_add || !fused_fp) {
    if (fork) HIP_TRY(hipStreamWaitEvent(st, c->ev_join, 0));   // (only with knob 3 = 1: no fork with the other two)
    if ((rc = launch_inner_fp(true, acc_add || !fused_fp, st))) return rc;
  }
  if (acc_add) return CKKS_OK;
  // 4.
  if ((rc = ks16_moddown_rows(c, lt, B, nlimbs, acc, tq, st, true))) return rc;
  if (fork && fused_fp) HIP_TRY(hipStreamWaitEvent(st, c->ev_join, 0));
  // 5.
  if (!fused_fp) return ks16_assemble(c, lt, io, B, nlimbs, acc, tq, st);
  FwdInnerArgs a = ia;
  a.fin_tq = tq;
  a.fin_out = io.out;
  a.fin_add_src = io.add_src;
  a.fin_add2 = io.add2 ? io.add2 : io.out;
  a.fin_add2_three = io.add2 && io.add2_three ? 1u : 0u;
  a.fin_pinv = lt->pinv2;
  a.fin_mode0 = io.mode[0];
  a.fin_mode1 = io.mode[1];
  a.fin_galois = io.add_galois;
  a.prod_a = io.prod_a;
  a.prod_b = io.prod_b;
  u32 cnt = 0;
  for (u32 s_ = 0; s_ < nlimbs; s_++)
    if (ext_class(s_) == 0) a.slots[cnt++] = (unsigned char)s_;
  if (cnt) {
    ProfScope ps(c, PK_INNER_C, st);
    launch_inner_c(c, B, cnt, a, st);
  }
  if (stored) return ks16_assemble(c, lt, io, B, nlimbs, acc, tq, st, true);
  launch_inner8(a, false, true, true);
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}

// Shared front of the hoisted rotations: inverse transform, ModUp and forward transform of c1 of ct_in
// ([B][2][nlimbs][N]) into the workspace, and the arguments of the streaming inner-product kernels that read them
// (accumulators default to the workspace's own).
static int hoist_front16(ckks_ctx* c, const LevelTables* lt, const u64* ct_in, u32 B, u32 nlimbs, char* ws, hipStream_t st,
                         FwdInnerArgs& ia) {
  int rc;
  const u32 N = c->N, next = lt->next, beta = lt->beta;
  const u64 polyN = (u64)nlimbs * N;
  KsLayout L = ks_layout(c, B, nlimbs);
  u64* dcoef = (u64*)(ws + L.dcoef);
  u64* ext = (u64*)(ws + L.ext);
  u64* acc = (u64*)(ws + L.acc);
  const LimbMap qmap = identity_map(nlimbs), emap = ext_map(c, nlimbs);
  const u64* c1 = ct_in + polyN;
  NttOpts o1, of;
  o1.scale = lt->up_scale;
  of.blocks_only = conv_fits(c, 0, nlimbs, c->alpha);
  ConvJob up;
  if (of.blocks_only) {
    up = conv_up_job(c, lt, dcoef, ext, B, nlimbs);
    o1.blocks_only = !up.ready;
  }
  if ((rc = launch_ntt(c, true, c1, 2 * polyN, dcoef, polyN, B, 0, nlimbs, qmap, 0, 0, st, o1))) return rc;
  if (of.blocks_only) {
    if ((rc = launch_conv_rows(c, up, st))) return rc;
  } else {
    ModUpArgs a{dcoef, ext, c->d_mods, lt->up_inv, lt->up_mat, c->logN, nlimbs, c->nq, c->alpha, beta, next};
    ProfScope ps(c, PK_MODUP, st);
    launch_modup<true>(c, lt, a, beta, B, st);
    HIP_TRY(hipGetLastError());
  }
  of.raw_out = true;  // reduced doubles on double-precision moduli, canonical residues elsewhere
  if ((rc = launch_ntt(c, false, ext, (u64)next * N, ext, (u64)next * N, B * beta, 0, next, emap, beta, nlimbs, st, of)))
    return rc;
  ia.ext = ext;
  ia.d = c1;
  ia.d_poly_stride = 2 * polyN;
  ia.acc = acc;
  ia.tw = c->d_tw_fwd;
  ia.twfp = c->d_twfp_fwd;
  ia.mods = c->d_mods;
  ia.logN = c->logN;
  ia.nlimbs = nlimbs;
  ia.nq = c->nq;
  ia.nm = c->nm;
  ia.alpha = c->alpha;
  ia.beta = beta;
  ia.next = next;
  ia.map_mode = map_mode_inner(c, true);
  return CKKS_OK;
}

// Hoisted rotations: out[r] = HRot_{g_r}(ct_in) for r < R. The Galois map commutes exactly with the
// centred base conversion (it permutes coefficients up to sign, and the conversion is odd), so INTT, ModUp and the
// forward transform of c1 are done once on the un-rotated polynomial; each rotation then reads the transformed
// digits through its own index map in the streaming inner product and finishes as usual.
// acc_base != null: rotation r stops before ModDown and leaves its accumulators, with P * sigma(c0) added to the
// first one, at acc_base + r * acc_stride (rotations kept in the extended basis), or adds them to what is there
// (acc_add); out_base is not used then. scratch != null (ordinary rotations): room for the accumulators
// ([B][2][next][N] each) of scratch_rots rotations, which are then computed that many at a time in one pass over the
// digits before each is finished.
int hrot_hoisted16(ckks_ctx* c, u64* out_base, u64 out_stride, const u64* ct_in, u32 B, u32 nlimbs, const u32* galois,
                   const u64* const* evks, u32 R, char* ws, hipStream_t st, u64* acc_base = nullptr, u64 acc_stride = 0,
                   bool acc_add = false, u64* scratch = nullptr, u32 scratch_rots = 0) {
  const LevelTables* lt;
  int rc = get_level(c, nlimbs, &lt);
  if (rc) return rc;
  const u32 N = c->N, next = lt->next, beta = lt->beta;
  const u64 polyN = (u64)nlimbs * N;
  const LimbMap emap = ext_map(c, nlimbs);
  const u64* c1 = ct_in + polyN;
  FwdInnerArgs ia;
  if ((rc = hoist_front16(c, lt, ct_in, B, nlimbs, ws, st, ia))) return rc;
  if (acc_base) {
    ia.c0 = ct_in;
    ia.c0_poly_stride = 2 * polyN;
    ia.accumulate = acc_add ? 1u : 0u;
  }
  // several rotations per pass over the digits (at most KS_MULTI_MAX): accumulators of rotations r0 .. r0+nr-1 to
  // dst + k * stride
  auto launch_rot = [&](u32 r0, u32 nr, u64* dst, u64 stride) -> int {
      ia.acc = dst;
      ia.acc_rot_stride = stride;
      ia.nrot = nr;
      for (u32 r = 0; r < nr; r++) {
        ia.galois_pc[r] = inv_mod_pow2(galois[r0 + r], c->logN + 1);
        ia.evk_pc[r] = evks[r0 + r];
      }
      for (int fp = 1; fp >= 0; fp--) {
        FwdInnerArgs a = ia;
        u32 cnt = 0;
        for (u32 s_ = 0; s_ < next; s_++)
          if ((host_class(c, c->mod[emap.id[s_]]) == 0) == (fp == 1)) a.slots[cnt++] = (unsigned char)s_;
        if (!cnt) continue;
        ProfScope ps(c, fp ? PK_INNER16 : PK_INNER16_INT, st);
        const u32 cb = fp ? INNER16_ROT_CB_FP : INNER16_ROT_CB;
        const dim3 grid((B + cb - 1) / cb, N / 256, cnt);
        if (fp && beta == 1) hipLaunchKernelGGL((inner16_rot_fp_kernel<1, true>), grid, dim3(256), 0, st, a, B);
        else if (fp && beta == 2) hipLaunchKernelGGL((inner16_rot_fp_kernel<2, true>), grid, dim3(256), 0, st, a, B);
        else if (fp && beta == 3) hipLaunchKernelGGL((inner16_rot_fp_kernel<3, true>), grid, dim3(256), 0, st, a, B);
        else if (fp && beta == 4) hipLaunchKernelGGL((inner16_rot_fp_kernel<4, true>), grid, dim3(256), 0, st, a, B);
        else if (fp) hipLaunchKernelGGL((inner16_rot_fp_kernel<INNER16_ROT_MAX_BETA, false>), grid, dim3(256), 0, st, a, B);
        else if (beta <= 4) hipLaunchKernelGGL(inner16_rot_int_kernel<4>, grid, dim3(256), 0, st, a, B);
        else hipLaunchKernelGGL(inner16_rot_int_kernel<INNER16_ROT_MAX_BETA>, grid, dim3(256), 0, st, a, B);
      }
      HIP_TRY(hipGetLastError());
      return CKKS_OK;
  };
  if (acc_base && !acc_add && beta <= INNER16_ROT_MAX_BETA) {
    for (u32 r0 = 0; r0 < R; r0 += KS_MULTI_MAX) {
      const u32 nr = std::min<u32>(KS_MULTI_MAX, R - r0);
      if ((rc = launch_rot(r0, nr, acc_base + (size_t)r0 * acc_stride, acc_stride))) return rc;
    }
    return CKKS_OK;
  }
  if (!acc_base && scratch && scratch_rots >= 2 && R >= 2 && beta <= INNER16_ROT_MAX_BETA) {
    const u64 one = (u64)B * 2 * next * N;
    const u32 per_pass = std::min<u32>(scratch_rots, KS_MULTI_MAX);
    for (u32 r0 = 0; r0 < R; r0 += per_pass) {
      const u32 nr = std::min<u32>(per_pass, R - r0);
      if ((rc = launch_rot(r0, nr, scratch, one))) return rc;
      for (u32 k = 0; k < nr; k++) {
        const u32 r = r0 + k;
        KsIo io{c1, 2 * polyN, galois[r], out_base + (size_t)r * out_stride, {2, 0}, ct_in, galois[r]};
        if ((rc = ks16_finish(c, lt, io, B, nlimbs, ws, st, scratch + (size_t)k * one))) return rc;
      }
    }
    return CKKS_OK;
  }
  for (u32 r = 0; r < R; r++) {
    ia.evk = evks[r];
    ia.galois = galois[r];
    ia.ext_galois = galois[r];
    if (acc_base) ia.acc = acc_base + (size_t)r * acc_stride;
    for (int fp = 1; fp >= 0; fp--) {
      FwdInnerArgs a = ia;
      u32 cnt = 0;
      for (u32 s_ = 0; s_ < next; s_++)
        if ((host_class(c, c->mod[emap.id[s_]]) == 0) == (fp == 1)) a.slots[cnt++] = (unsigned char)s_;
      if (!cnt) continue;
      ProfScope ps(c, fp ? PK_INNER16 : PK_INNER16_INT, st);
      if (fp) hipLaunchKernelGGL(inner16_fp_kernel, dim3(B, N / 512, cnt), dim3(256), 0, st, a);
      else hipLaunchKernelGGL(inner16_int_kernel, dim3(B, N / 512, cnt), dim3(256), 0, st, a);
    }
    HIP_TRY(hipGetLastError());
    if (acc_base) continue;
    KsIo io{c1, 2 * polyN, galois[r], out_base + (size_t)r * out_stride, {2, 0}, ct_in, galois[r]};
    if ((rc = ks16_finish(c, lt, io, B, nlimbs, ws, st))) return rc;
  }
  return CKKS_OK;
}

// Ring 2^12: front, digits, special, final (ks12.hip.h).
int keyswitch_whole12(ckks_ctx* c, const LevelTables* lt, const KsIo& io, u32 B, u32 nlimbs, const u64* evk, char* ws,
                      hipStream_t st) {
  if (io.galois_pc && B > KS_MULTI_MAX) return fail(CKKS_ESHAPE, "internal: per-ciphertext keys for too many ciphertexts");
  const KsLayout L = ks_layout(c, B, nlimbs);
  Ks12Args a;
  a.d = io.d;
  a.d_stride = io.d_stride;
  a.pa = io.prod_a;
  a.pb = io.prod_b;
  a.dcoef = (u64*)(ws + L.dcoef);
  a.ext = (u64*)(ws + L.ext);
  a.acc = (u64*)(ws + L.acc);
  a.out = io.out;
  a.evk = evk;
  a.add2 = io.add2 ? io.add2 : io.out;
  a.add_src = io.add_src;
  a.add2_three = io.add2 && io.add2_three ? 1u : 0u;
  a.tw = c->d_tw_fwd;
  a.twi = c->d_tw_inv;
  a.twfp = c->d_twfp_fwd;
  a.twifp = c->d_twfp_inv;
  a.mods = c->d_mods;
  a.up_scale = lt->up_scale;
  a.dn_scale = lt->dn_scale;
  a.pinv = lt->pinv2;
  a.up_mat = lt->up_mat;
  a.up_off = lt->up_off;
  a.dn_mat = lt->dn_mat_plain;
  a.dn_off = lt->dn_off;
  a.up_pitch = lt->up_pitch;
  a.dn_pitch = lt->dn_pitch;
  a.nlimbs = nlimbs;
  a.nq = c->nq;
  a.nm = c->nm;
  a.alpha = c->alpha;
  a.beta = lt->beta;
  a.next = lt->next;
  a.fp_on = c->tune[1] == 0 ? 1u : 0u;
  for (u32& w : a.fp_mask) w = 0;
  for (u32 i = 0; i < c->nm; i++)
    if (host_class(c, c->mod[i]) == 0) a.fp_mask[i >> 5] |= 1u << (i & 31);
  a.mode0 = io.mode[0];
  a.mode1 = io.mode[1];
  a.d_galois = io.d_galois;
  a.add_galois = io.add_galois;
  a.multi = io.galois_pc ? 1u : 0u;
  if (io.galois_pc)
    for (u32 i = 0; i < B; i++) a.galois_pc[i] = io.galois_pc[i], a.evk_pc[i] = io.evk_pc[i];
  const dim3 block(WL_THREADS);
  {
    ProfScope ps(c, PK_KS12_FRONT, st);
    hipLaunchKernelGGL(ks12_front_kernel, dim3(B, nlimbs), block, 0, st, a);
  }
  {
    ProfScope ps(c, PK_KS12_DIGITS, st);
    const dim3 grid(B * lt->beta, lt->next);
    if (lt->narrow_up) hipLaunchKernelGGL(ks12_digits_kernel<true>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(ks12_digits_kernel<false>, grid, block, 0, st, a);
  }
  {
    ProfScope ps(c, PK_KS12_SPECIAL, st);
    hipLaunchKernelGGL(ks12_special_kernel, dim3(2 * B, c->np), block, 0, st, a);
  }
  {
    ProfScope ps(c, PK_KS12_FINAL, st);
    const dim3 grid(2 * B, nlimbs);
    if (lt->narrow_dn) hipLaunchKernelGGL(ks12_final_kernel<true>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(ks12_final_kernel<false>, grid, block, 0, st, a);
  }
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}

// Key switch of io.d with evk into io.out (see KsIo). Other ring degrees, and io.steps: one kernel per step.
int keyswitch_impl(ckks_ctx* c, const KsIo& io, u32 B, u32 nlimbs, const u64* evk, char* ws, hipStream_t st) {
  const LevelTables* lt;
  int rc = get_level(c, nlimbs, &lt);
  if (rc) return rc;
  if (two_pass(c)) return keyswitch_fused16(c, lt, io, B, nlimbs, evk, ws, st);
  if (c->logN == 12 && !io.steps) return keyswitch_whole12(c, lt, io, B, nlimbs, evk, ws, st);
  if (io.d_galois || io.mode[0] >= 2 || io.mode[1] >= 2 || io.add2)
    return fail(CKKS_EINVAL, "internal: gather modes and separate addends need the fused paths");
  const u64* d = io.d;
  u64* out = io.out;
  const u32 add_mask = (io.mode[0] ? 1u : 0u) | (io.mode[1] ? 2u : 0u);
  const u32 N = c->N, next = lt->next, beta = lt->beta, K = c->np;
  KsLayout L = ks_layout(c, B, nlimbs);
  u64* dcoef = (u64*)(ws + L.dcoef);
  u64* ext = (u64*)(ws + L.ext);
  u64* acc = (u64*)(ws + L.acc);
  u64* tq = (u64*)(ws + L.tq);
  const LimbMap qmap = identity_map(nlimbs), emap = ext_map(c, nlimbs);

  // 1. coefficient form of d
  if ((rc = launch_ntt(c, true, d, io.d_stride, dcoef, (u64)nlimbs * N, B, 0, nlimbs, qmap, 0, 0, st))) return rc;
  // 2. ModUp every digit to the slots it does not own
  {
    ModUpArgs a{dcoef, ext, c->d_mods, lt->up_inv, lt->up_mat, c->logN, nlimbs, c->nq, c->alpha, beta, next};
    ProfScope ps(c, PK_MODUP, st);
    launch_modup<false>(c, lt, a, beta, B, st);
    HIP_TRY(hipGetLastError());
  }
  // 3. forward transform of the converted slots
  if ((rc = launch_ntt(c, false, ext, (u64)next * N, ext, (u64)next * N, B * beta, 0, next, emap, beta, nlimbs, st))) return rc;
  // 4. inner product with the key
  {
    InnerArgs a{d, ext, evk, acc, c->d_mods, c->logN, nlimbs, c->nq, c->nm, c->alpha, beta, next, io.d_stride};
    ProfScope ps(c, PK_INNER, st);
    hipLaunchKernelGGL(inner_kernel, dim3(B, N / 256, next), dim3(256), 0, st, a);
    HIP_TRY(hipGetLastError());
  }
  // 5. special limbs of both accumulators back to coefficient form
  {
    LimbMap pmap;
    for (u32 k = 0; k < CKKS_MAX_SLOTS; k++) pmap.id[k] = (unsigned char)(k < K ? c->nq + k : 0);
    if ((rc = launch_ntt(c, true, acc, (u64)next * N, acc, (u64)next * N, B * 2, nlimbs, K, pmap, 0, 0, st))) return rc;
  }
  // 6. ModDown base conversion P -> Q_l
  {
    ModDownArgs a{acc, tq, c->d_mods, lt->dn_inv, lt->dn_mat, c->logN, nlimbs, c->nq, K, next, nlimbs, c->nq};
    ProfScope ps(c, PK_MODDOWN, st);
    launch_moddown<false>(c, lt, a, B * 2, lt->narrow_dn, st);
    HIP_TRY(hipGetLastError());
  }
  // 7. its forward transform, 8. subtract, scale by P^-1, assemble
  if ((rc = launch_ntt(c, false, tq, (u64)nlimbs * N, tq, (u64)nlimbs * N, B * 2, 0, nlimbs, qmap, 0, 0, st))) return rc;
  {
    FinalArgs a{acc, tq, out, c->d_mods, lt->pinv, c->logN, nlimbs, next, add_mask};
    ProfScope ps(c, PK_FINAL, st);
    hipLaunchKernelGGL(ks_final_kernel, dim3(N / 256, nlimbs, B * 2), dim3(256), 0, st, a);
    HIP_TRY(hipGetLastError());
  }
  return CKKS_OK;
}

// Hoisted sums on double-precision slots. The kernel for several ciphertexts per lane is instantiated for up to 4 digits and
// for any number.
template <int CB>
void launch_inner_sum_fp_of(u32 b0, u32 groups, u32 blocks, u32 slots, const FwdInnerArgs& a, u32 B, hipStream_t st) {
  const dim3 grid(groups, blocks, slots), block(256);
  switch (a.beta) {
    case 1: hipLaunchKernelGGL((inner16_sum_fp_kernel<CB, 1>), grid, block, 0, st, a, B, b0); break;
    case 2: hipLaunchKernelGGL((inner16_sum_fp_kernel<CB, 2>), grid, block, 0, st, a, B, b0); break;
    case 3: hipLaunchKernelGGL((inner16_sum_fp_kernel<CB, 3>), grid, block, 0, st, a, B, b0); break;
    case 4: hipLaunchKernelGGL((inner16_sum_fp_kernel<CB, 4>), grid, block, 0, st, a, B, b0); break;
    default: hipLaunchKernelGGL((inner16_sum_fp_kernel<CB, 0>), grid, block, 0, st, a, B, b0); break;
  }
}
// Ciphertexts go to lanes in as few groups of at most four as hold them, as even as possible: a lone remainder costs nearly
// what a whole group does (5 ciphertexts of 20 limbs, 4 digits, 7 rotations: four and one 405 us, three and two 350; 9: fours
// and one 613, threes 586). The kernel for one ciphertext and two positions per lane is left what it does better: one rotation,
// one ciphertext of more than 4 digits (134 us against 128) and 5 ciphertexts with a few rotations (2 digits, 2: 104 and 93).
void launch_inner_sum_fp(u32 B, u32 N, u32 slots, const FwdInnerArgs& a, hipStream_t st) {
  if (a.nrot <= 1 || (B == 1 && a.beta > 4) || (B == 5 && a.nrot < 4)) {
    hipLaunchKernelGGL(inner16_sum_pair_fp_kernel, dim3(B, N / 512, slots), dim3(256), 0, st, a);
    return;
  }
  if (B <= 2) {
    if (B == 1) launch_inner_sum_fp_of<1>(0, 1, N / 256, slots, a, B, st);
    else launch_inner_sum_fp_of<2>(0, 1, N / 256, slots, a, B, st);
    return;
  }
  const u32 groups = (B + 3) / 4, fours = B > 3 * groups ? B - 3 * groups : 0;   // B = 5: two threes, one place empty
  if (fours) launch_inner_sum_fp_of<4>(0, fours, N / 256, slots, a, B, st);
  if (groups > fours) launch_inner_sum_fp_of<3>(4 * fours, groups - fours, N / 256, slots, a, B, st);
}

int check_common(const ckks_ctx* c, u32 B, u32 nlimbs) {
  if (!c) return fail(CKKS_EINVAL, "null context");
  if (nlimbs == 0 || nlimbs > c->nq) return fail(CKKS_ESHAPE, "nlimbs must be in [1, L+1]");
  if (B == 0 || B > 32767) return fail(CKKS_ESHAPE, "batch must be in [1, 32767]");
  if (c->np == 0) return fail(CKKS_ESHAPE, "key switching needs at least one special prime");
  return CKKS_OK;
}
int check_ws(const ckks_ctx* c, int op, u32 B, u32 nlimbs, u32 n1, const void* ws, size_t ws_bytes) {
  if (!ws || ((uintptr_t)ws & 255)) return fail(CKKS_EWORKSPACE, "workspace is null or not 256-byte aligned");
  size_t need = ckks_workspace_bytes(c, op, B, nlimbs, n1);
  if (ws_bytes < need)
    return fail(CKKS_EWORKSPACE, "workspace too small: need " + std::to_string(need) + " bytes, got " + std::to_string(ws_bytes));
  return CKKS_OK;
}
bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb && y < x + na;
}

int check_ids(const ckks_ctx* c, const uint32_t* ids, u32 n, LimbMap* out) {
  if (!ids) return fail(CKKS_EINVAL, "null limb_ids");
  if (n == 0 || n > CKKS_MAX_SLOTS) return fail(CKKS_ESHAPE, "nlimbs must be in [1, 128]");
  for (u32 i = 0; i < CKKS_MAX_SLOTS; i++) out->id[i] = 0;
  for (u32 i = 0; i < n; i++) {
    if (ids[i] >= c->nm) return fail(CKKS_EINVAL, "limb id out of range");
    out->id[i] = (unsigned char)ids[i];
  }
  return CKKS_OK;
}

// Launch forms of a matrix product's inner sums and what a launch takes, in us, for the choice between them:
//   4 + wait * n1 + limbs * N / 65536 * (issue^4 + traffic^4)^(1/4)
//   issue = groups * (tiles * tile + count * giant) * (n1 + rest), traffic = word * (n1 * (2B + count) + 2B * count)
// for `count` giant steps in tiles of `giants` and 2B polynomials in groups of `polys`: instructions or, where one group shares
// nothing with another, each word once (5.6 TB/s in register tiles, 4.9 staged). Each form was timed alone, 1 .. 64 baby steps and
// 4 .. 32 ciphertexts; the constants fit 24 and 4 limbs at 2^16 (rms 4 .. 6 %, lone tiles of 1 .. 4 giant steps 9 .. 14 %), `wait`, a
// lone workgroup's time a step, 2^12 .. 2^14. Why a choice and not a size: a staged tile costs the most of a whole one when it is
// short, and half as much again beyond its baby steps, while the register-tiled kernels pay for a tile of 4, 3, 2 or 1 giant steps
// most of what one of 6 (integer limbs 3) costs and read the baby steps again for each launch. 24 limbs at 2^16, in register tiles
// and staged, us: 8 ciphertexts, 12 giant x 64 baby steps 6582 and 6205 (integer limbs 8614 and 6306), 12 x 1 549 and 699, 7 x 8
// 1052 and 820, 18 x 8 1713 and 2090; 5 ciphertexts 9 x 8 882 and 956 (integer limbs 840 and 1068). The launches chosen take 0.5 %
// more than the best of the forms on average over 14 counts of giant steps at each of those sizes, 12 % less than register tiles.
struct SumForm {
  u32 giants, polys;
  double tile, giant, rest, word, wait;
};
struct SumForms {
  SumForm tiled[5];    // pmacc_*_kernel: whole tiles only, largest first down to 1, as many of each as fit
  SumForm staged[2];   // pmacc_*_staged_kernel
};
constexpr SumForms kSumsFp = {{{6, PMACC_FP_P, .89, 0, 3.6, .093, .72}, {4, PMACC_FP_P, .73, 0, .6, .093, .48},
                               {3, PMACC_FP_P, .65, 0, .3, .093, .36}, {2, PMACC_FP_P, .63, 0, 0, .093, .24},
                               {1, PMACC_FP_P, .56, 0, 0, .093, .12}},
                              {{12, 8, 1.28, .026, 5.6, .108, .25}, {8, 8, .89, .024, 5.4, .108, .25}}};
constexpr SumForms kSumsInt = {{{3, PMACC_INT_P, .29, 0, 5.8, .093, .36}, {2, PMACC_INT_P, .33, 0, 2.5, .093, .24},
                                {1, PMACC_INT_P, .25, 0, 0, .093, .12}},
                               {{6, 8, .55, .039, 8.7, .108, .25}, {8, 8, .99, .032, 8.0, .108, .25}}};
struct SumPlan {
  double us;
  int staged;   // what the next launch is: a staged form, or -1 for register tiles to the end
  u32 count;    // giant steps it covers
};
// The next launch for `left` giant steps of `work` = limbs * N / 65536: everything left in register tiles, everything in staged
// tiles of either size (the last one short), or 12 steps in the large ones and then the best for the others. Up to 6 steps and
// below 4 ciphertexts register tiles, against which the staged kernels were not measured.
SumPlan sum_plan(const SumForms& f, u32 left, u32 B, u32 n1, double work) {
  auto us = [&](const SumForm& m, u32 count) {
    const u32 groups = (2 * B + m.polys - 1) / m.polys, tiles = (count + m.giants - 1) / m.giants;
    const double issue = groups * (tiles * m.tile + count * m.giant) * (n1 + m.rest);
    const double traffic = m.word * ((double)n1 * (2 * B + count) + 2.0 * B * count);
    return 4 + m.wait * n1 + work * std::sqrt(std::hypot(issue * issue, traffic * traffic));
  };
  SumPlan best{0, -1, left};
  u32 rest = left;
  for (u32 i = 0; rest; rest %= f.tiled[i++].giants)
    if (rest >= f.tiled[i].giants) best.us += us(f.tiled[i], rest / f.tiled[i].giants * f.tiled[i].giants);
  if (left < 7 || B < 4) return best;
  auto consider = [&](double t, int staged, u32 count) {
    if (t < best.us) best = {t, staged, count};
  };
  for (int i = 0; i < 2; i++) consider(us(f.staged[i], left), i, left);
  if (left > 12) consider(us(f.staged[0], 12) + sum_plan(f, left - 12, B, n1, work).us, 0, 12);
  return best;
}
}  // namespace

extern "C" {

const char* ckks_last_error(void) { return g_err.c_str(); }

int ckks_ctx_create(ckks_ctx** out, uint32_t logN, const uint64_t* q, uint32_t nq, const uint64_t* p, uint32_t np,
                    uint32_t dnum, const uint64_t* psi, int device) {
  if (!out || !q || !psi || (np && !p)) return fail(CKKS_EINVAL, "null argument");
  if (logN < 10 || logN > 17) return fail(CKKS_ESHAPE, "logN must be in [10, 17]");
  if (nq == 0 || dnum == 0 || dnum > nq || nq + np > CKKS_MAX_SLOTS || nq > 45 || np > 45)
    return fail(CKKS_ESHAPE, "bad prime or digit count (at most 45 main and 45 special primes)");
  int ndev = 0;
  HIP_TRY(hipGetDeviceCount(&ndev));
  if (device < 0 || device >= ndev) return fail(CKKS_EINVAL, "no such device");
  ckks_ctx* c = new ckks_ctx;
  c->device = device;
  c->logN = logN;
  c->N = 1u << logN;
  c->nq = nq;
  c->np = np;
  c->nm = nq + np;
  c->dnum = dnum;
  c->alpha = (nq + dnum - 1) / dnum;
  for (u32 i = 0; i < nq; i++) c->mod.push_back(q[i]);
  for (u32 i = 0; i < np; i++) c->mod.push_back(p[i]);
  c->psi.assign(psi, psi + c->nm);
  const u64 N = c->N;
  for (u32 i = 0; i < c->nm; i++) {
    u64 m = c->mod[i];
    bool ok = m < (1ull << 60) && m > 2 * N && (m - 1) % (2 * N) == 0 && h_is_prime(m) && c->psi[i] < m &&
              h_pow(c->psi[i], N, m) == m - 1;
    for (u32 k = 0; k < i && ok; k++) ok = c->mod[k] != m;
    if (!ok) {
      delete c;
      return fail(CKKS_EINVAL, "modulus " + std::to_string(i) +
                                   " must be a distinct prime < 2^60, = 1 mod 2N, with psi^N = -1");
    }
  }
  // tables
  std::vector<ModInfo> mods(c->nm);
  std::vector<ulonglong2> fwd((size_t)c->nm * N), inv((size_t)c->nm * N);
  std::vector<double> fwdfp, invfp;
  if (logN <= 16) {   // the rings with double-precision bodies
    fwdfp.assign((size_t)c->nm * N, 0.0);
    invfp.assign((size_t)c->nm * N, 0.0);
  }
  std::vector<u64> pw(N);
  for (u32 i = 0; i < c->nm; i++) {
    u64 m = c->mod[i];
    ModInfo& mi = mods[i];
    mi.m = m;
    mi.mu64 = (u64)((((u128)1) << 64) / m);
    mi.c64 = (u64)((((u128)1) << 64) % m);
    mi.c64s = h_shoup(mi.c64, m);
    mi.ninv = h_inv(N % m, m);
    mi.ninvs = h_shoup(mi.ninv, m);
    {
      u64 x = 1;  // Newton iteration for m^-1 mod 2^64 (m odd)
      for (int it = 0; it < 6; it++) x *= 2 - m * x;
      mi.minv = (u64)0 - x;
      mi.pmod = 0;
      if (i < c->nq) {
        mi.pmod = 1;
        for (u32 k = 0; k < c->np; k++) mi.pmod = h_mul(mi.pmod, c->mod[c->nq + k] % m, m);
      }
    }
    mi.qd = (double)m;
    mi.qinv = 1.0 / (double)m;
    mi.ninvd = (double)mi.ninv;
    mi.ninvq = (double)mi.ninv / (double)m;
    auto centred = [m](u64 v) { return v > m / 2 ? -(double)(m - v) : (double)v; };
    pw[0] = 1;
    for (u64 k = 1; k < N; k++) pw[k] = h_mul(pw[k - 1], c->psi[i], m);
    for (u32 k = 0; k < N; k++) {
      u64 w = pw[h_brev(k, logN)];
      fwd[(size_t)i * N + k] = ulonglong2{w, h_shoup(w, m)};
      // psi^-e = -psi^(N-e)
      u32 e = h_brev(k, logN);
      u64 wi = e == 0 ? 1 : m - pw[N - e];
      inv[(size_t)i * N + k] = ulonglong2{wi, h_shoup(wi, m)};
      if (!fwdfp.empty() && (m >> 50) == 0) {
        fwdfp[(size_t)i * N + k] = centred(w);
        invfp[(size_t)i * N + k] = centred(wi);
      }
    }
  }
  DeviceGuard guard(device);
  int rc = guard.ok ? CKKS_OK : fail(CKKS_EHIP, "cannot select device");
  if (!rc) rc = upload(&c->d_mods, mods);
  if (!rc) rc = upload(&c->d_tw_fwd, fwd);
  if (!rc) rc = upload(&c->d_tw_inv, inv);
  if (!rc) rc = upload(&c->d_twfp_fwd, fwdfp);
  if (!rc) rc = upload(&c->d_twfp_inv, invfp);
  if (!rc) rc = build_levels(c);
  if (!rc) {
    // device current = the context's: every GPU holds its own copy of the array at its own address
    hipError_t e = hipGetSymbolAddress(&c->scratch_ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !c->scratch_ptr)
      rc = fail(CKKS_EHIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
  }
  // the second stream and the events of the fork/join inside a key switch (knob 4) exist from the start, so that
  // no call that enqueues work has to create them
  if (!rc && hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking) != hipSuccess) rc = fail(CKKS_EHIP, "hipStreamCreate");
  if (!rc && hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming) != hipSuccess) rc = fail(CKKS_EHIP, "hipEventCreate");
  if (!rc && hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming) != hipSuccess) rc = fail(CKKS_EHIP, "hipEventCreate");
  if (rc) {
    ckks_ctx_destroy(c);
    return rc;
  }
  *out = c;
  return CKKS_OK;
}

int ckks_ctx_destroy(ckks_ctx* c) {
  if (!c) return CKKS_OK;
  DeviceGuard guard(c->device);
  (void)hipFree(c->d_mods);
  (void)hipFree(c->d_tw_fwd);
  (void)hipFree(c->d_tw_inv);
  (void)hipFree(c->d_twfp_fwd);
  (void)hipFree(c->d_twfp_inv);
  if (c->side) (void)hipStreamSynchronize(c->side), (void)hipStreamDestroy(c->side);
  if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
  if (c->ev_join) (void)hipEventDestroy(c->ev_join);
  for (auto& r : c->prof_recs) {
    (void)hipEventDestroy(r.start);
    (void)hipEventDestroy(r.stop);
  }
  for (auto& e : c->prof_pool) (void)hipEventDestroy(e);
  (void)hipFree(c->d_levels);
  delete c;
  return CKKS_OK;
}

int ckks_tune_set(ckks_ctx* c, int knob, int value) {
  if (!c || knob < 0 || knob >= 8) return fail(CKKS_EINVAL, "bad knob");
  const int old = c->tune[knob];
  c->tune[knob] = value;
  // knobs 1 and 5 select the arithmetic the level tables are scaled for: rebuild them (waits for the device)
  if ((knob == 1 || knob == 5) && (old != 0) != (value != 0)) return build_levels(c);
  return CKKS_OK;
}
int ckks_prof_enable(ckks_ctx* c, int on) {
  if (!c) return fail(CKKS_EINVAL, "null context");
  c->prof_on = on != 0;
  return CKKS_OK;
}
int ckks_prof_copy(ckks_ctx* c, void* dst, const void* src, size_t bytes, void* stream) {
  if (!c || !dst || !src) return fail(CKKS_EINVAL, "null argument");
  if (bytes == 0 || (bytes & 15) || ((uintptr_t)dst & 15) || ((uintptr_t)src & 15) || bytes / 16 / 256 >= (1ull << 31))
    return fail(CKKS_ESHAPE, "ckks_prof_copy: size and addresses must be multiples of 16 bytes");
  if (overlap(dst, bytes, src, bytes)) return fail(CKKS_EINVAL, "dst overlaps src");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  const size_t n = bytes / 16;
  ProfScope ps(c, PK_COPY, (hipStream_t)stream);
  hipLaunchKernelGGL(ckks_prof_copy_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                     (const ulonglong2*)src, (ulonglong2*)dst, n);
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}
int ckks_prof_num_kinds(void) { return PK_COUNT; }
const char* ckks_prof_kind_name(int kind) { return kind >= 0 && kind < PK_COUNT ? kProfNames[kind] : ""; }
int ckks_prof_collect(ckks_ctx* c) {
  if (!c) return fail(CKKS_EINVAL, "null context");
  DeviceGuard guard(c->device);
  for (auto& r : c->prof_recs) {
    HIP_TRY(hipEventSynchronize(r.stop));
    float ms = 0;
    HIP_TRY(hipEventElapsedTime(&ms, r.start, r.stop));
    c->prof_ms[r.kind] += ms;
    c->prof_n[r.kind] += 1;
    c->prof_pool.push_back(r.start);
    c->prof_pool.push_back(r.stop);
  }
  c->prof_recs.clear();
  return CKKS_OK;
}
int ckks_prof_read(ckks_ctx* c, int kind, double* total_ms, uint64_t* launches) {
  if (!c || kind < 0 || kind >= PK_COUNT || !total_ms || !launches) return fail(CKKS_EINVAL, "bad argument");
  *total_ms = c->prof_ms[kind];
  *launches = c->prof_n[kind];
  return CKKS_OK;
}
int ckks_prof_reset(ckks_ctx* c) {
  if (!c) return fail(CKKS_EINVAL, "null context");
  int rc = ckks_prof_collect(c);
  for (int k = 0; k < PK_COUNT; k++) c->prof_ms[k] = 0, c->prof_n[k] = 0;
  return rc;
}

size_t ckks_workspace_bytes(const ckks_ctx* c, int op, uint32_t B, uint32_t nlimbs, uint32_t n1) {
  if (!c || B == 0 || nlimbs == 0 || nlimbs > c->nq) return 0;
  const size_t ks = ks_layout(c, B, nlimbs).total;
  const size_t poly = align256((size_t)B * nlimbs * c->N * 8);
  switch (op) {
    case CKKS_OP_KEYSWITCH: return ks;
    case CKKS_OP_HROT: return ks + poly;
    case CKKS_OP_HMULT_RELIN: return ks + poly;
    case CKKS_OP_RESCALE:
      // coefficient form of the dropped limb, its image on the remaining limbs
      return nlimbs < 2 ? 0 : align256((size_t)B * 2 * c->N * 8) + align256((size_t)B * 2 * (nlimbs - 1) * c->N * 8);
    case CKKS_OP_PCMM_BSGS:
      if (n1 == 0) return 0;
      // baby steps 1..n1-1, PMACC_TILE inner sums, rotated inner sum, HRot workspace
      return (size_t)(n1 - 1) * 2 * poly + (size_t)PMACC_TILE * 2 * poly + 2 * poly + ks + poly;
    case CKKS_OP_HROT_SUM:
      // hoisted digits and ModDown scratch, plus the running sum in the extended basis
      return ks + poly + 2 * align256((size_t)B * (nlimbs + c->np) * c->N * 8);
    case CKKS_OP_PCMM_BSGS_DH: {
      if (n1 == 0) return 0;
      // n1 baby steps, PMACC_TILE inner sums and the sum over giant steps in the extended basis, one inner sum
      // after ModDown, HRot workspace
      const size_t ext_poly = align256((size_t)B * (nlimbs + c->np) * c->N * 8);
      return (size_t)(n1 + PMACC_TILE + 1) * 2 * ext_poly + 2 * poly + ks + poly;
    }
    default: return 0;
  }
}

static int transform_entry(ckks_ctx* c, bool inverse, uint64_t* data, uint32_t npoly, const uint32_t* limb_ids,
                           uint32_t nlimbs, void* stream) {
  if (!c || !data) return fail(CKKS_EINVAL, "null argument");
  LimbMap ids;
  int rc = check_ids(c, limb_ids, nlimbs, &ids);
  if (rc) return rc;
  if (npoly == 0) return CKKS_OK;
  if (npoly > 65535 * 16) return fail(CKKS_ESHAPE, "too many polynomials in one call");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  // grid.x carries the polynomial index; split very large batches
  const u32 chunk = 32768;
  for (u32 p0 = 0; p0 < npoly; p0 += chunk) {
    u32 n = std::min(chunk, npoly - p0);
    u64* base = (u64*)data + (size_t)p0 * nlimbs * c->N;
    rc = launch_ntt(c, inverse, base, (u64)nlimbs * c->N, base, (u64)nlimbs * c->N, n, 0, nlimbs, ids, 0, 0,
                    (hipStream_t)stream);
    if (rc) return rc;
  }
  return CKKS_OK;
}

int ckks_ntt(ckks_ctx* c, uint64_t* data, uint32_t npoly, const uint32_t* limb_ids, uint32_t nlimbs, void* stream) {
  return transform_entry(c, false, data, npoly, limb_ids, nlimbs, stream);
}
int ckks_intt(ckks_ctx* c, uint64_t* data, uint32_t npoly, const uint32_t* limb_ids, uint32_t nlimbs, void* stream) {
  return transform_entry(c, true, data, npoly, limb_ids, nlimbs, stream);
}

int ckks_automorph(ckks_ctx* c, uint64_t* out, const uint64_t* in, uint32_t npoly, const uint32_t* limb_ids,
                   uint32_t nlimbs, uint32_t g, int eval_domain, void* stream) {
  if (!c || !out || !in) return fail(CKKS_EINVAL, "null argument");
  LimbMap ids;
  int rc = check_ids(c, limb_ids, nlimbs, &ids);
  if (rc) return rc;
  if (!(g & 1) || g >= 2 * c->N) return fail(CKKS_EINVAL, "galois_elt must be odd and < 2N");
  if (npoly == 0) return CKKS_OK;
  if (npoly > 65535) return fail(CKKS_ESHAPE, "too many polynomials in one call");
  size_t bytes = (size_t)npoly * nlimbs * c->N * 8;
  if (overlap(out, bytes, in, bytes)) return fail(CKKS_EINVAL, "out overlaps in");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  return launch_automorph(c, (u64*)out, (u64)nlimbs * c->N, (const u64*)in, (u64)nlimbs * c->N, npoly, nlimbs, ids, g,
                          eval_domain != 0, (hipStream_t)stream);
}

int ckks_keyswitch(ckks_ctx* c, uint64_t* ks_out, const uint64_t* d, uint32_t B, uint32_t nlimbs, const uint64_t* evk,
                   uint32_t galois_elt, uint32_t dnum, void* ws, size_t ws_bytes, void* stream) {
  (void)galois_elt;
  int rc = check_common(c, B, nlimbs);
  if (rc) return rc;
  if (!ks_out || !d || !evk) return fail(CKKS_EINVAL, "null argument");
  if (dnum != c->dnum) return fail(CKKS_ESHAPE, "dnum does not match the context");
  if ((rc = check_ws(c, CKKS_OP_KEYSWITCH, B, nlimbs, 0, ws, ws_bytes))) return rc;
  size_t poly = (size_t)B * nlimbs * c->N * 8;
  if (overlap(ks_out, 2 * poly, d, poly)) return fail(CKKS_EINVAL, "ks_out overlaps d");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  KsIo io{(const u64*)d, (u64)nlimbs * c->N, 0, (u64*)ks_out, {0, 0}, nullptr, 0};
  io.steps = !whole_limb(c, B, nlimbs, false);
  return keyswitch_impl(c, io, B, nlimbs, (const u64*)evk, (char*)ws, (hipStream_t)stream);
}

static int hrot_impl(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs, uint32_t g,
                     const uint64_t* evk, void* ws, size_t ws_bytes, void* stream, const uint64_t* ct_add);
int ckks_hrot(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs, uint32_t g,
              const uint64_t* evk, void* ws, size_t ws_bytes, void* stream) {
  return hrot_impl(c, ct_out, ct_in, B, nlimbs, g, evk, ws, ws_bytes, stream, nullptr);
}
// ct_add != null: ct_out = ct_add + HRot(ct_in); ct_add == ct_out accumulates in place (fused paths only).
static int hrot_impl(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs, uint32_t g,
                     const uint64_t* evk, void* ws, size_t ws_bytes, void* stream, const uint64_t* ct_add) {
  int rc = check_common(c, B, nlimbs);
  if (rc) return rc;
  if (!ct_out || !ct_in || !evk) return fail(CKKS_EINVAL, "null argument");
  if (!(g & 1) || g >= 2 * c->N) return fail(CKKS_EINVAL, "galois_elt must be odd and < 2N");
  if ((rc = check_ws(c, CKKS_OP_HROT, B, nlimbs, 0, ws, ws_bytes))) return rc;
  const size_t polyN = (size_t)nlimbs * c->N, ct_bytes = (size_t)B * 2 * polyN * 8;
  if (overlap(ct_out, ct_bytes, ct_in, ct_bytes)) return fail(CKKS_EINVAL, "ct_out overlaps ct_in");
  if (ct_add && ct_add != ct_out && overlap(ct_out, ct_bytes, ct_add, ct_bytes))
    return fail(CKKS_EINVAL, "ct_add must be ct_out itself or not overlap it");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  hipStream_t st = (hipStream_t)stream;
  if (gathers(c, B, nlimbs)) {
    // the permutation is applied where the ciphertext is read: by the first inverse pass and the fused inner product
    // (sigma(c1)) and by the final assembly (sigma(c0)), which also adds ct_add
    KsIo io{(const u64*)ct_in + polyN, 2 * polyN, g, (u64*)ct_out, {ct_add ? 3u : 2u, ct_add ? 1u : 0u},
            (const u64*)ct_in, g};
    io.add2 = (const u64*)ct_add;
    return keyswitch_impl(c, io, B, nlimbs, (const u64*)evk, (char*)ws, st);
  }
  if (ct_add && ct_add == ct_out) return fail(CKKS_EINVAL, "internal: accumulating in place needs the fused paths");
  const size_t ks = ks_layout(c, B, nlimbs).total;
  u64* d = (u64*)((char*)ws + ks);
  const LimbMap qmap = identity_map(nlimbs);
  // sigma(c0) -> out[.,0]; sigma(c1) -> d
  if ((rc = launch_automorph(c, (u64*)ct_out, 2 * polyN, (const u64*)ct_in, 2 * polyN, B, nlimbs, qmap, g, true, st)))
    return rc;
  if ((rc = launch_automorph(c, d, polyN, (const u64*)ct_in + polyN, 2 * polyN, B, nlimbs, qmap, g, true, st))) return rc;
  KsIo io{d, polyN, 0, (u64*)ct_out, {1, 0}, nullptr, 0};
  io.steps = true;
  if ((rc = keyswitch_impl(c, io, B, nlimbs, (const u64*)evk, (char*)ws, st))) return rc;
  if (ct_add) {
    AddArgs ad{(u64*)ct_out, (const u64*)ct_add, c->d_mods, c->logN, nlimbs};
    ProfScope ps(c, PK_ADD, st);
    hipLaunchKernelGGL(addto_kernel, dim3(c->N / 256, nlimbs, 2 * B), dim3(256), 0, st, ad);
    HIP_TRY(hipGetLastError());
  }
  return CKKS_OK;
}

size_t ckks_noalloc_scratch_bytes(void) { return (size_t)CKKS_NOALLOC_SCRATCH_BYTES; }

// ckks_hrot with the library's fixed scratch array as its workspace: no hipMalloc/hipFree here or below (the level
// tables, the second stream and its events exist since ckks_ctx_create). Every region of the workspace is written
// by a kernel of the call before a later kernel reads it, so nothing has to be cleared between calls.
int ckks_hrot_noalloc(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs, uint32_t g,
                      const uint64_t* evk, void* stream) {
  int rc = check_common(c, B, nlimbs);
  if (rc) return rc;
  if (c->prof_on) return fail(CKKS_EINVAL, "ckks_hrot_noalloc: per-kernel timing creates events; disable it first");
  const size_t need = ckks_workspace_bytes(c, CKKS_OP_HROT, B, nlimbs, 0);
  if (need == 0 || need > (size_t)CKKS_NOALLOC_SCRATCH_BYTES)
    return fail(CKKS_EWORKSPACE, "ckks_hrot_noalloc: this batch needs " + std::to_string(need) +
                                     " bytes of workspace, the fixed scratch array holds " +
                                     std::to_string((size_t)CKKS_NOALLOC_SCRATCH_BYTES));
  return hrot_impl(c, ct_out, ct_in, B, nlimbs, g, evk, c->scratch_ptr, (size_t)CKKS_NOALLOC_SCRATCH_BYTES, stream, nullptr);
}

int ckks_hrot_add(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, const uint64_t* ct_add, uint32_t B, uint32_t nlimbs,
                  uint32_t g, const uint64_t* evk, void* ws, size_t ws_bytes, void* stream) {
  if (!ct_add) return fail(CKKS_EINVAL, "null argument");
  if (c && c->logN != 16 && ct_add == ct_out) return fail(CKKS_EINVAL, "ct_add == ct_out needs N = 2^16");
  return hrot_impl(c, ct_out, ct_in, B, nlimbs, g, evk, ws, ws_bytes, stream, ct_add);
}

int ckks_hrot_multi(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs,
                    const uint32_t* galois_elts, const uint64_t* const* evks, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_common(c, B, nlimbs);
  if (rc) return rc;
  if (!ct_out || !ct_in || !galois_elts || !evks) return fail(CKKS_EINVAL, "null argument");
  for (u32 b = 0; b < B; b++) {
    if (!evks[b]) return fail(CKKS_EINVAL, "null key");
    if (!(galois_elts[b] & 1) || galois_elts[b] >= 2 * c->N) return fail(CKKS_EINVAL, "galois_elt must be odd and < 2N");
  }
  if ((rc = check_ws(c, CKKS_OP_HROT, B, nlimbs, 0, ws, ws_bytes))) return rc;
  const size_t polyN = (size_t)nlimbs * c->N, ct_bytes = (size_t)B * 2 * polyN * 8;
  if (overlap(ct_out, ct_bytes, ct_in, ct_bytes)) return fail(CKKS_EINVAL, "ct_out overlaps ct_in");
  if (!two_pass(c) && c->logN != 12) {
    // other ring sizes: one rotation at a time through the general path
    for (u32 b = 0; b < B; b++)
      if ((rc = hrot_impl(c, ct_out + b * 2 * polyN, ct_in + b * 2 * polyN, 1, nlimbs, galois_elts[b], evks[b], ws, ws_bytes,
                          stream, nullptr)))
        return rc;
    return CKKS_OK;
  }
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  hipStream_t st = (hipStream_t)stream;
  // the kernels carry the per-ciphertext elements and key pointers in their arguments, KS_MULTI_MAX at a time
  for (u32 b0 = 0; b0 < B; b0 += KS_MULTI_MAX) {
    const u32 nb = std::min<u32>(KS_MULTI_MAX, B - b0);
    const u64* in = (const u64*)ct_in + (size_t)b0 * 2 * polyN;
    KsIo io{in + polyN, 2 * polyN, 0, (u64*)ct_out + (size_t)b0 * 2 * polyN, {2u, 0u}, in, 0};
    io.galois_pc = galois_elts + b0;
    io.evk_pc = (const u64* const*)evks + b0;
    if ((rc = keyswitch_impl(c, io, nb, nlimbs, nullptr, (char*)ws, st))) return rc;
  }
  return CKKS_OK;
}

int ckks_hmult_relin(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_a, const uint64_t* ct_b, uint32_t B,
                     uint32_t nlimbs, const uint64_t* evk, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_common(c, B, nlimbs);
  if (rc) return rc;
  if (!ct_out || !ct_a || !ct_b || !evk) return fail(CKKS_EINVAL, "null argument");
  if ((rc = check_ws(c, CKKS_OP_HMULT_RELIN, B, nlimbs, 0, ws, ws_bytes))) return rc;
  const size_t ct_bytes = (size_t)B * 2 * nlimbs * c->N * 8;
  if (overlap(ct_out, ct_bytes, ct_a, ct_bytes) || overlap(ct_out, ct_bytes, ct_b, ct_bytes))
    return fail(CKKS_EINVAL, "ct_out overlaps an input");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  hipStream_t st = (hipStream_t)stream;
  if (whole_limb(c, B, nlimbs, true)) {
    KsIo io{nullptr, 0, 0, (u64*)ct_out, {0, 0}, nullptr, 0};
    io.prod_a = (const u64*)ct_a;
    io.prod_b = (const u64*)ct_b;
    return keyswitch_impl(c, io, B, nlimbs, (const u64*)evk, (char*)ws, st);
  }
  // Two-pass rings: the products are formed where they are read (first inverse pass, own digits, assembly), which takes 6 passes
  // over a limb vector where a product kernel of its own and the reads of its results took 11: 32 products of 24 limbs at
  // 2^16 3328 -> 3099 us, 3 of 11 limbs 230 -> 216, 8 of 13 limbs at 2^15 308 -> 293.
  if (two_pass(c) && c->tune[3] != 1 && !int_sums_stored(c, B, nlimbs, true)) {
    KsIo io{nullptr, 0, 0, (u64*)ct_out, {4, 4}, nullptr, 0};
    io.prod_a = (const u64*)ct_a;
    io.prod_b = (const u64*)ct_b;
    return keyswitch_impl(c, io, B, nlimbs, (const u64*)evk, (char*)ws, st);
  }
  const size_t ks = ks_layout(c, B, nlimbs).total;
  u64* d2 = (u64*)((char*)ws + ks);
  TensorArgs a{(const u64*)ct_a, (const u64*)ct_b, (u64*)ct_out, d2, c->d_mods, c->logN, nlimbs};
  {
    ProfScope ps(c, PK_TENSOR, st);
    hipLaunchKernelGGL(tensor_kernel, dim3(c->N / 256, nlimbs, B), dim3(256), 0, st, a);
  }
  HIP_TRY(hipGetLastError());
  KsIo io{d2, (u64)nlimbs * c->N, 0, (u64*)ct_out, {1, 1}, nullptr, 0};
  io.steps = true;
  return keyswitch_impl(c, io, B, nlimbs, (const u64*)evk, (char*)ws, st);
}

int ckks_tensor_acc(ckks_ctx* c, uint64_t* d_out, const uint64_t* ct_a, const uint64_t* ct_b, const uint64_t* d_acc,
                    uint32_t B, uint32_t nlimbs, void* stream) {
  int rc = check_common(c, B, nlimbs);
  if (rc) return rc;
  if (!d_out || !ct_a || !ct_b) return fail(CKKS_EINVAL, "null argument");
  const size_t ct_bytes = (size_t)B * 2 * nlimbs * c->N * 8, d_bytes = ct_bytes / 2 * 3;
  if (overlap(d_out, d_bytes, ct_a, ct_bytes) || overlap(d_out, d_bytes, ct_b, ct_bytes))
    return fail(CKKS_EINVAL, "d_out overlaps an input ciphertext");
  if (d_acc && d_acc != d_out && overlap(d_out, d_bytes, d_acc, d_bytes))
    return fail(CKKS_EINVAL, "d_acc overlaps d_out without being d_out");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  hipStream_t st = (hipStream_t)stream;
  TensorAccArgs a{(const u64*)ct_a, (const u64*)ct_b, (const u64*)d_acc, (u64*)d_out, c->d_mods, c->logN, nlimbs};
  {
    ProfScope ps(c, PK_TENSOR, st);
    hipLaunchKernelGGL(tensor_acc_kernel, dim3(c->N / 256, nlimbs, B), dim3(256), 0, st, a);
  }
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}

int ckks_relin(ckks_ctx* c, uint64_t* ct_out, const uint64_t* d_in, uint32_t B, uint32_t nlimbs, const uint64_t* evk,
               void* ws, size_t ws_bytes, void* stream) {
  int rc = check_common(c, B, nlimbs);
  if (rc) return rc;
  if (!ct_out || !d_in || !evk) return fail(CKKS_EINVAL, "null argument");
  if ((rc = check_ws(c, CKKS_OP_KEYSWITCH, B, nlimbs, 0, ws, ws_bytes))) return rc;
  const size_t polyN = (size_t)nlimbs * c->N;
  if (overlap(ct_out, (size_t)B * 2 * polyN * 8, d_in, (size_t)B * 3 * polyN * 8))
    return fail(CKKS_EINVAL, "ct_out overlaps d_in");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  hipStream_t st = (hipStream_t)stream;
  const u64* d = (const u64*)d_in;
  KsIo io{d + 2 * polyN, 3 * (u64)polyN, 0, (u64*)ct_out, {1, 1}, nullptr, 0};
  if (gathers(c, B, nlimbs)) {
    // the last kernel of the key switch reads d0 and d1 in place
    io.add2 = d;
    io.add2_three = true;
  } else {
    // general path: d0, d1 are copied into ct_out and the key switch adds to them in place
    io.steps = true;
    const size_t pl2 = polyN / 2;
    ProfScope ps(c, PK_ADD, st);
    hipLaunchKernelGGL(first_two_components_kernel, dim3((unsigned)((2 * pl2 + 255) / 256), B), dim3(256), 0, st,
                       (const ulonglong2*)d, (ulonglong2*)ct_out, pl2);
    HIP_TRY(hipGetLastError());
  }
  return keyswitch_impl(c, io, B, nlimbs, (const u64*)evk, (char*)ws, st);
}

static int pcmm_impl(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs,
                     const uint64_t* pt, uint32_t n1, uint32_t n2, uint32_t stride, const uint64_t* const* evk_baby,
                     const uint64_t* const* evk_giant, void* ws, size_t ws_bytes, void* stream, int mode);
int ckks_pcmm_bsgs(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs,
                   const uint64_t* pt, uint32_t n1, uint32_t n2, uint32_t stride, const uint64_t* const* evk_baby,
                   const uint64_t* const* evk_giant, void* ws, size_t ws_bytes, void* stream) {
  return pcmm_impl(c, ct_out, ct_in, B, nlimbs, pt, n1, n2, stride, evk_baby, evk_giant, ws, ws_bytes, stream, 0);
}
int ckks_pcmm_bsgs_hoisted(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs,
                           const uint64_t* pt, uint32_t n1, uint32_t n2, uint32_t stride,
                           const uint64_t* const* evk_baby, const uint64_t* const* evk_giant, void* ws, size_t ws_bytes,
                           void* stream) {
  return pcmm_impl(c, ct_out, ct_in, B, nlimbs, pt, n1, n2, stride, evk_baby, evk_giant, ws, ws_bytes, stream, 1);
}
int ckks_pcmm_bsgs_double_hoisted(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs,
                                  const uint64_t* pt_ext, uint32_t n1, uint32_t n2, uint32_t stride,
                                  const uint64_t* const* evk_baby, const uint64_t* const* evk_giant, void* ws,
                                  size_t ws_bytes, void* stream) {
  if (c && c->logN != 16) return fail(CKKS_ESHAPE, "the double-hoisted schedule is built for N = 2^16 only");
  return pcmm_impl(c, ct_out, ct_in, B, nlimbs, pt_ext, n1, n2, stride, evk_baby, evk_giant, ws, ws_bytes, stream, 2);
}
int ckks_hrot_hoisted(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs,
                      const uint32_t* galois_elts, const uint64_t* const* evks, uint32_t R, void* ws, size_t ws_bytes,
                      void* stream) {
  int rc = check_common(c, B, nlimbs);
  if (rc) return rc;
  if (!ct_out || !ct_in || !galois_elts || !evks) return fail(CKKS_EINVAL, "null argument");
  if (R == 0) return CKKS_OK;
  for (u32 r = 0; r < R; r++) {
    if (!evks[r]) return fail(CKKS_EINVAL, "null key");
    if (!(galois_elts[r] & 1) || galois_elts[r] >= 2 * c->N) return fail(CKKS_EINVAL, "galois_elt must be odd and < 2N");
  }
  if ((rc = check_ws(c, CKKS_OP_HROT, B, nlimbs, 0, ws, ws_bytes))) return rc;
  const size_t ct_elems = (size_t)B * 2 * nlimbs * c->N;
  if (overlap(ct_out, (size_t)R * ct_elems * 8, ct_in, ct_elems * 8)) return fail(CKKS_EINVAL, "ct_out overlaps ct_in");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  if (two_pass(c)) {
    // workspace beyond the required size holds accumulators of rotations that then share a pass over the digits
    const size_t need = ckks_workspace_bytes(c, CKKS_OP_HROT, B, nlimbs, 0);
    const size_t one = (size_t)B * 2 * (nlimbs + c->np) * c->N * 8;
    const u32 fit = (u32)std::min<size_t>((ws_bytes - need) / one, 1u << 20);
    return hrot_hoisted16(c, (u64*)ct_out, ct_elems, (const u64*)ct_in, B, nlimbs, galois_elts, (const u64* const*)evks, R,
                          (char*)ws, (hipStream_t)stream, nullptr, 0, false, (u64*)((char*)ws + need), fit);
  }
  for (u32 r = 0; r < R; r++)  // other ring degrees: the same result, one rotation at a time
    if ((rc = ckks_hrot(c, ct_out + (size_t)r * ct_elems, ct_in, B, nlimbs, galois_elts[r], evks[r], ws, ws_bytes, stream)))
      return rc;
  return CKKS_OK;
}
int ckks_hrot_sum(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs,
                  const uint32_t* galois_elts, const uint64_t* const* evks, uint32_t R, void* ws, size_t ws_bytes,
                  void* stream) {
  int rc = check_common(c, B, nlimbs);
  if (rc) return rc;
  if (c->logN != 16) return fail(CKKS_ESHAPE, "the hoisted rotate-and-sum is built for N = 2^16 only");
  if (!ct_out || !ct_in || (R && (!galois_elts || !evks))) return fail(CKKS_EINVAL, "null argument");
  if (2 * B > 65535) return fail(CKKS_ESHAPE, "batch too large for one call");
  for (u32 r = 0; r < R; r++) {
    if (!evks[r]) return fail(CKKS_EINVAL, "null key");
    if (!(galois_elts[r] & 1) || galois_elts[r] >= 2 * c->N) return fail(CKKS_EINVAL, "galois_elt must be odd and < 2N");
  }
  if ((rc = check_ws(c, CKKS_OP_HROT_SUM, B, nlimbs, 0, ws, ws_bytes))) return rc;
  const size_t N = c->N, ct_bytes = (size_t)B * 2 * nlimbs * N * 8;
  if (overlap(ct_out, ct_bytes, ct_in, ct_bytes)) return fail(CKKS_EINVAL, "ct_out overlaps ct_in");
  const LevelTables* lt;
  if ((rc = get_level(c, nlimbs, &lt))) return rc;
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  hipStream_t st = (hipStream_t)stream;
  const u32 next = nlimbs + c->np;
  char* hws = (char*)ws;
  u64* total = (u64*)(hws + ckks_workspace_bytes(c, CKKS_OP_HROT, B, nlimbs, 0));
  FwdInnerArgs ia;
  if ((rc = hoist_front16(c, lt, (const u64*)ct_in, B, nlimbs, hws, st, ia))) return rc;
  ia.acc = total;
  ia.c0 = (const u64*)ct_in;
  ia.c0_poly_stride = 2 * (u64)nlimbs * N;
  const LimbMap emap = ext_map(c, nlimbs);
  // up to KS_MULTI_MAX rotations per launch; the first launch starts from P * ct, later ones add to the sum
  for (u32 r0 = 0; r0 == 0 || r0 < R; r0 += KS_MULTI_MAX) {
    const u32 nr = std::min<u32>(KS_MULTI_MAX, R - r0);
    ia.nrot = nr;
    ia.accumulate = r0 ? 1u : 0u;
    for (u32 r = 0; r < nr; r++) {
      ia.galois_pc[r] = galois_elts[r0 + r];
      ia.evk_pc[r] = (const u64*)evks[r0 + r];
    }
    for (int fp = 1; fp >= 0; fp--) {
      FwdInnerArgs a = ia;
      u32 cnt = 0;
      for (u32 s_ = 0; s_ < next; s_++)
        if ((host_class(c, c->mod[emap.id[s_]]) == 0) == (fp == 1)) a.slots[cnt++] = (unsigned char)s_;
      if (!cnt) continue;
      ProfScope ps(c, fp ? PK_INNER16 : PK_INNER16_INT, st);
      const dim3 grid(B, N / 512, cnt);
      if (fp) launch_inner_sum_fp(B, (u32)N, cnt, a, st);
      else if (nr * a.beta >= 16) hipLaunchKernelGGL(inner16_sum_int_kernel<true>, grid, dim3(256), 0, st, a);
      else hipLaunchKernelGGL(inner16_sum_int_kernel<false>, grid, dim3(256), 0, st, a);
    }
    HIP_TRY(hipGetLastError());
  }
  KsIo io{nullptr, 0, 0, (u64*)ct_out, {0, 0}, nullptr, 0};
  return ks16_finish(c, lt, io, B, nlimbs, hws, st, total);
}

static int pcmm_impl(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs,
                     const uint64_t* pt, uint32_t n1, uint32_t n2, uint32_t stride, const uint64_t* const* evk_baby,
                     const uint64_t* const* evk_giant, void* ws, size_t ws_bytes, void* stream, int mode) {
  // mode 0: one rotation at a time; 1: hoisted baby steps; 2: baby steps kept in the extended basis (pt holds the
  // plaintexts in that basis), one ModDown per giant step
  const bool hoisted = mode == 1, dh = mode == 2;
  int rc = check_common(c, B, nlimbs);
  if (rc) return rc;
  if (!ct_out || !ct_in || !pt) return fail(CKKS_EINVAL, "null argument");
  if (n1 == 0 || n2 == 0 || stride == 0) return fail(CKKS_ESHAPE, "n1, n2 and stride must be positive");
  if ((n1 > 1 && !evk_baby) || (n2 > 1 && !evk_giant)) return fail(CKKS_EINVAL, "null key array");
  for (u32 b = 1; b < n1; b++)
    if (!evk_baby[b - 1]) return fail(CKKS_EINVAL, "null baby-step key");
  for (u32 g = 1; g < n2; g++)
    if (!evk_giant[g - 1]) return fail(CKKS_EINVAL, "null giant-step key");
  if (2 * B > 65535) return fail(CKKS_ESHAPE, "batch too large for one call");
  if ((rc = check_ws(c, dh ? CKKS_OP_PCMM_BSGS_DH : CKKS_OP_PCMM_BSGS, B, nlimbs, n1, ws, ws_bytes))) return rc;
  const size_t N = c->N, polyN = (size_t)nlimbs * N, ct_bytes = (size_t)B * 2 * polyN * 8;
  if (overlap(ct_out, ct_bytes, ct_in, ct_bytes)) return fail(CKKS_EINVAL, "ct_out overlaps ct_in");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  hipStream_t st = (hipStream_t)stream;
  const size_t ct_al = 2 * align256((size_t)B * polyN * 8);
  // polynomials the inner sums work on: nlimbs limbs, or the nlimbs + K slots of the extended basis
  const u32 pl_limbs = dh ? nlimbs + c->np : nlimbs;
  const size_t sum_al = dh ? 2 * align256((size_t)B * pl_limbs * N * 8) : ct_al;
  char* w = (char*)ws;
  u64* first = nullptr;                 // double-hoisted: (P c0, P c1), the term of baby step 0
  u64* total = nullptr;                 // double-hoisted: sum over giant steps, extended basis
  if (dh) { first = (u64*)w;            w += sum_al; }
  if (dh) { total = (u64*)w;            w += sum_al; }
  u64* baby = (u64*)w;                  w += (size_t)(n1 - 1) * sum_al;
  u64* inner = (u64*)w;                 w += (size_t)PMACC_TILE * sum_al;   // inner sums of one tile of giant steps
  u64* rot = (u64*)w;                   w += ct_al;
  char* hws = w;
  const size_t hws_bytes = ckks_workspace_bytes(c, CKKS_OP_HROT, B, nlimbs, 0);
  const u64 twoN = 2 * N;
  auto galois = [&](u64 r) {  // 5^r mod 2N
    u64 g = 1, b = 5;
    for (; r; r >>= 1) {
      if (r & 1) g = g * b % twoN;
      b = b * b % twoN;
    }
    return (u32)g;
  };
  const size_t ct_elems = ct_al / 8;  // == B*2*nlimbs*N: a limb-vector is a multiple of 256 bytes
  const size_t sum_elems = sum_al / 8;
  const LevelTables* lt = nullptr;
  if (dh) {
    if ((rc = get_level(c, nlimbs, &lt))) return rc;
    LiftArgs la{(const u64*)ct_in, first, c->d_mods, c->logN, nlimbs, pl_limbs, {}};
    for (u32 i = 0; i < nlimbs; i++) la.fp[i] = host_class(c, c->mod[i]) == 0 ? 1 : 0;
    {
      ProfScope ps(c, PK_ADD, st);
      hipLaunchKernelGGL(lift_qp_kernel, dim3(N / 512, pl_limbs, 2 * B), dim3(256), 0, st, la);
    }
    HIP_TRY(hipGetLastError());
    if (n1 > 1) {
      std::vector<u32> gs(n1 - 1);
      for (u32 b = 1; b < n1; b++) gs[b - 1] = galois((u64)b * stride);
      if ((rc = hrot_hoisted16(c, nullptr, 0, (const u64*)ct_in, B, nlimbs, gs.data(), (const u64* const*)evk_baby, n1 - 1,
                               hws, st, baby, sum_elems)))
        return rc;
    }
  } else if (hoisted && n1 > 1) {
    std::vector<u32> gs(n1 - 1);
    for (u32 b = 1; b < n1; b++) gs[b - 1] = galois((u64)b * stride);
    if (two_pass(c)) {
      // the region of the inner sums is free until the baby steps are done: it holds the accumulators of as many
      // rotations as fit, which then share one pass over the hoisted digits
      const size_t one = (size_t)B * 2 * (nlimbs + c->np) * N * 8;
      const u32 fit = (u32)std::min<size_t>((size_t)PMACC_TILE * ct_al / one, 1u << 20);
      rc = hrot_hoisted16(c, baby, ct_elems, (const u64*)ct_in, B, nlimbs, gs.data(), (const u64* const*)evk_baby, n1 - 1,
                          hws, st, nullptr, 0, false, inner, fit);
    } else {
      rc = ckks_hrot_hoisted(c, (uint64_t*)baby, ct_in, B, nlimbs, gs.data(), evk_baby, n1 - 1, hws, hws_bytes, stream);
    }
    if (rc) return rc;
  } else {
    for (u32 b = 1; b < n1; b++) {
      rc = ckks_hrot(c, (uint64_t*)(baby + (size_t)(b - 1) * ct_elems), ct_in, B, nlimbs, galois((u64)b * stride),
                     evk_baby[b - 1], hws, hws_bytes, stream);
      if (rc) return rc;
    }
  }
  // limbs by arithmetic kind: each has kernels of its own. In register tiles the double-precision ones take up to 6 giant
  // steps x 8 polynomials per pass over the baby-step ciphertexts, the integer ones up to 3 x 4
  PmaccArgs fa, ia;
  u32 nfp = 0, nint = 0;
  for (u32 i = 0; i < pl_limbs; i++) {
    const u32 id = i < nlimbs ? i : c->nq + (i - nlimbs);
    if (host_class(c, c->mod[id]) == 0 && c->tune[6] == 0) {
      fa.mod_ids[nfp] = (unsigned char)id;
      fa.limbs[nfp++] = (unsigned char)i;
    } else {
      ia.mod_ids[nint] = (unsigned char)id;
      ia.limbs[nint++] = (unsigned char)i;
    }
  }
  const u32 tile_max = c->tune[7] > 0 ? std::min<u32>(PMACC_TILE, (u32)c->tune[7]) : PMACC_TILE;
  for (u32 g0 = 0; g0 < n2;) {
    const u32 ng = std::min<u32>(tile_max, n2 - g0);
    // giant step 0 needs no rotation: its inner sum is written straight into the output
    auto fill = [&](PmaccArgs& a, u32 first_g, u32 count) {
      a.ct_in = dh ? first : (const u64*)ct_in;
      a.baby = baby;
      a.pt = (const u64*)pt;
      a.out0 = first_g == 0 ? (dh ? total : (u64*)ct_out) : inner + (size_t)(first_g - g0) * sum_elems;
      a.out_rest = inner + (size_t)(first_g - g0 + 1) * sum_elems;
      a.mods = c->d_mods;
      a.logN = c->logN;
      a.nlimbs = pl_limbs;
      a.n1 = n1;
      a.B = B;
      a.g0 = first_g;
      a.ng = count;
    };
    // the kernels that stage their words through LDS copy 16 bytes a lane
    const bool staged_ok = (((uintptr_t)pt | (uintptr_t)baby | (uintptr_t)(dh ? first : (const u64*)ct_in)) & 15) == 0;
    auto plan = [&](const SumForms& f, u32 h0, u32 limbs) {
      return staged_ok ? sum_plan(f, g0 + ng - h0, B, n1, (double)limbs * N / 65536) : SumPlan{0, -1, g0 + ng - h0};
    };
    // (2^32 lanes, which a grid may not pass, take a workspace larger than the memory)
    auto staged_tiles = [&](PmaccArgs& a, u32 h0, const SumPlan& p, const SumForm& m, u32 limbs) {
      fill(a, h0, p.count);
      a.ngt = (p.count + m.giants - 1) / m.giants;
      return dim3((2 * B + m.polys - 1) / m.polys * a.ngt * (N / 64) * limbs);
    };
    for (u32 h0 = g0; nfp && h0 < g0 + ng;) {
      const SumPlan next = plan(kSumsFp, h0, nfp);
      if (next.staged >= 0) {
        const dim3 grid = staged_tiles(fa, h0, next, kSumsFp.staged[next.staged], nfp);
        ProfScope ps(c, PK_PMACC_FP_STAGED, st);
        if (next.staged == 0) hipLaunchKernelGGL((pmacc_fp_staged_kernel<4, 6, 2, 2>), grid, dim3(256), 0, st, fa);
        else hipLaunchKernelGGL((pmacc_fp_staged_kernel<4, 4, 2, 2>), grid, dim3(256), 0, st, fa);
        HIP_TRY(hipGetLastError());
        h0 += fa.ng;
        continue;
      }
      static const u32 kSizes[] = {6, 4, 3, 2, 1};
      u32 cnt = 1;
      for (u32 sz : kSizes)
        if (sz <= g0 + ng - h0) {
          cnt = sz;
          break;
        }
      const u32 ngt = (g0 + ng - h0) / cnt;   // as many whole tiles of this size as remain, in one launch
      fill(fa, h0, cnt);
      fa.ngt = ngt;
      ProfScope ps(c, PK_PMACC_FP, st);
      dim3 grid((2 * B + PMACC_FP_P - 1) / PMACC_FP_P * ngt, N / 256, nfp), block(256);
      switch (cnt) {
        case 6: hipLaunchKernelGGL(pmacc_fp_kernel<6>, grid, block, 0, st, fa); break;
        case 4: hipLaunchKernelGGL(pmacc_fp_kernel<4>, grid, block, 0, st, fa); break;
        case 3: hipLaunchKernelGGL(pmacc_fp_kernel<3>, grid, block, 0, st, fa); break;
        case 2: hipLaunchKernelGGL(pmacc_fp_kernel<2>, grid, block, 0, st, fa); break;
        default: hipLaunchKernelGGL(pmacc_fp_kernel<1>, grid, block, 0, st, fa); break;
      }
      HIP_TRY(hipGetLastError());
      h0 += cnt * ngt;
    }
    for (u32 h0 = g0; nint && h0 < g0 + ng;) {
      const SumPlan next = plan(kSumsInt, h0, nint);
      if (next.staged >= 0) {
        const dim3 grid = staged_tiles(ia, h0, next, kSumsInt.staged[next.staged], nint);
        ProfScope ps(c, PK_PMACC_STAGED, st);
        if (next.staged == 0) hipLaunchKernelGGL((pmacc_int_staged_kernel<4, 3, 2, 2>), grid, dim3(256), 0, st, ia);
        else hipLaunchKernelGGL((pmacc_int_staged_kernel<4, 2, 2, 4>), grid, dim3(512), 0, st, ia);
        HIP_TRY(hipGetLastError());
        h0 += ia.ng;
        continue;
      }
      static const u32 kSizes[] = {3, 2, 1};
      u32 cnt = 1;
      for (u32 sz : kSizes)
        if (sz <= g0 + ng - h0) {
          cnt = sz;
          break;
        }
      const u32 ngt = (g0 + ng - h0) / cnt;
      fill(ia, h0, cnt);
      ia.ngt = ngt;
      ProfScope ps(c, PK_PMACC, st);
      dim3 grid((2 * B + PMACC_INT_P - 1) / PMACC_INT_P * ngt, N / 256, nint), block(256);
      switch (cnt) {
        case 3: hipLaunchKernelGGL(pmacc_int_kernel<3>, grid, block, 0, st, ia); break;
        case 2: hipLaunchKernelGGL(pmacc_int_kernel<2>, grid, block, 0, st, ia); break;
        default: hipLaunchKernelGGL(pmacc_int_kernel<1>, grid, block, 0, st, ia); break;
      }
      HIP_TRY(hipGetLastError());
      h0 += cnt * ngt;
    }
    for (u32 k = 0; k < ng; k++) {
      const u32 g = g0 + k;
      if (dh) {
        // giant step 0 is already in `total`; the others: ModDown of the inner sum into `rot`, then its rotation
        // (one hoisted rotation that stops before ModDown) added to `total`
        if (g == 0) continue;
        KsIo io{nullptr, 0, 0, rot, {0, 0}, nullptr, 0};
        if ((rc = ks16_finish(c, lt, io, B, nlimbs, hws, st, inner + (size_t)k * sum_elems))) return rc;
        const u32 gg = galois((u64)g * n1 * stride);
        const u64* key = (const u64*)evk_giant[g - 1];
        if (c->tune[3] != 1) {
          // the usual fused sequence of a rotation (c1 read through the Galois map), stopped before ModDown
          KsIo gio{rot + polyN, 2 * (u64)polyN, gg, nullptr, {0, 0}, rot, gg};
          rc = keyswitch_fused16(c, lt, gio, B, nlimbs, key, hws, st, total);
        } else {
          rc = hrot_hoisted16(c, nullptr, 0, rot, B, nlimbs, &gg, &key, 1, hws, st, total, 0, /*acc_add=*/true);
        }
        if (rc) return rc;
        continue;
      }
      if (g == 0) continue;
      const u64* src = inner + (size_t)k * ct_elems;
      if (gathers(c, B, nlimbs)) {
        rc = hrot_impl(c, ct_out, (const uint64_t*)src, B, nlimbs, galois((u64)g * n1 * stride), evk_giant[g - 1], hws,
                       hws_bytes, stream, /*ct_add=*/ct_out);
        if (rc) return rc;
      } else {
        rc = ckks_hrot(c, (uint64_t*)rot, (const uint64_t*)src, B, nlimbs, galois((u64)g * n1 * stride), evk_giant[g - 1], hws,
                       hws_bytes, stream);
        if (rc) return rc;
        AddArgs ad{(u64*)ct_out, rot, c->d_mods, c->logN, nlimbs};
        ProfScope ps(c, PK_ADD, st);
        hipLaunchKernelGGL(addto_kernel, dim3(N / 256, nlimbs, 2 * B), dim3(256), 0, st, ad);
        HIP_TRY(hipGetLastError());
      }
    }
    g0 += ng;
  }
  if (dh) {   // one ModDown of the sum over giant steps
    KsIo io{nullptr, 0, 0, (u64*)ct_out, {0, 0}, nullptr, 0};
    if ((rc = ks16_finish(c, lt, io, B, nlimbs, hws, st, total))) return rc;
  }
  return CKKS_OK;
}

int ckks_rescale(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, uint32_t B, uint32_t nlimbs, void* ws,
                 size_t ws_bytes, void* stream) {
  if (!c || !ct_out || !ct_in) return fail(CKKS_EINVAL, "null argument");
  if (nlimbs < 2 || nlimbs > c->nq) return fail(CKKS_ESHAPE, "rescale needs 2..L+1 limbs");
  if (B == 0 || B > 32767) return fail(CKKS_ESHAPE, "batch must be in [1, 32767]");
  int rc = check_ws(c, CKKS_OP_RESCALE, B, nlimbs, 0, ws, ws_bytes);
  if (rc) return rc;
  const u32 N = c->N, nl1 = nlimbs - 1;
  if (overlap(ct_out, (size_t)B * 2 * nl1 * N * 8, ct_in, (size_t)B * 2 * nlimbs * N * 8))
    return fail(CKKS_EINVAL, "ct_out overlaps ct_in");
  const LevelTables* lt;
  if ((rc = get_level(c, nlimbs, &lt))) return rc;
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  hipStream_t st = (hipStream_t)stream;
  u64* last = (u64*)ws;
  u64* tq = (u64*)((char*)ws + align256((size_t)B * 2 * N * 8));
  // 1. coefficient form of the last limb of every polynomial (rows of ct_in are nlimbs*N apart)
  LimbMap lmap = identity_map(0);
  lmap.id[0] = (unsigned char)nl1;
  // 2. its centred representative on the remaining limbs (a one-source base conversion), on two-pass rings with the row passes on
  // both sides of it: as three kernels 8 ciphertexts of 20 limbs took 207 us, this way 176, and one ciphertext 37 instead of 55
  const bool conv = two_pass(c) && conv_fits(c, nl1, 1, 1);
  NttOpts o1;
  o1.blocks_only = conv;
  if ((rc = launch_ntt(c, true, (const u64*)ct_in + (size_t)nl1 * N, (u64)nlimbs * N, last, (u64)N, B * 2, 0, 1, lmap, 0, 0, st, o1)))
    return rc;
  if (conv) {
    ConvJob job;
    ConvArgs& a = job.a;
    a.src = last;
    a.dst = tq;
    a.src_poly_stride = N;
    a.dst_poly_stride = (u64)nl1 * N;
    a.src_slot0 = 0;
    a.src_id0 = nl1;
    a.src_nlimbs = a.alpha = a.beta = 1;
    a.skip_own = 0;
    a.ntarget = nl1;
    a.pieces = lt->rs_pieces;
    a.scale = lt->rs_scale;
    job.npoly = B * 2;
    conv_plan(c, job, [](u32 s) { return s; });
    if ((rc = launch_conv_rows(c, job, st))) return rc;
  } else {
    ModDownArgs a{last, tq, c->d_mods, lt->rs_one, lt->rs_mat, c->logN, nl1, c->nq, 1, 1, 0, nl1};
    ProfScope ps(c, PK_MODDOWN, st);
    launch_moddown<true>(c, lt, a, B * 2, lt->narrow_rs, st);
    HIP_TRY(hipGetLastError());
  }
  // 3. back to the evaluation domain, subtract, divide by q_last
  const LimbMap qmap = identity_map(nl1);
  if (two_pass(c)) {
    NttOpts o;
    o.rows_only = true;
    if (!conv && (rc = launch_ntt(c, false, tq, (u64)nl1 * N, tq, (u64)nl1 * N, B * 2, 0, nl1, qmap, 0, 0, st, o))) return rc;
    FwdFinalArgs a;
    a.tq = tq;
    a.acc = (const u64*)ct_in;
    a.out = (u64*)ct_out;
    a.add_src = nullptr;
    a.add2 = nullptr;
    a.tw = c->d_tw_fwd;
    a.twfp = c->d_twfp_fwd;
    a.mods = c->d_mods;
    a.pinv = lt->rs_qinv16;
    a.logN = c->logN;
    a.nlimbs = nl1;
    a.next = nlimbs;
    a.mode0 = a.mode1 = 0;
    a.galois = 0;
    a.map_mode = map_mode_pass(c);
    auto cls_of = [&](u32 s) { return host_class(c, c->mod[s]); };
    launch_by_class(c, PK_FWD_FINAL, a, B * 2, nl1, cls_of, st,
                    [&](int cls, dim3 grid) { LAUNCH_CLASS_KERNEL(ntt16_fwd_blocks_final_kernel, cls, grid, st, a); });
    HIP_TRY(hipGetLastError());
    return CKKS_OK;
  }
  if ((rc = launch_ntt(c, false, tq, (u64)nl1 * N, tq, (u64)nl1 * N, B * 2, 0, nl1, qmap, 0, 0, st))) return rc;
  FinalArgs a{(const u64*)ct_in, tq, (u64*)ct_out, c->d_mods, lt->rs_qinv, c->logN, nl1, nlimbs, 0};
  ProfScope ps(c, PK_FINAL, st);
  hipLaunchKernelGGL(ks_final_kernel, dim3(N / 256, nl1, B * 2), dim3(256), 0, st, a);
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}

static int pointwise_entry(ckks_ctx* c, bool mul, uint64_t* out, const uint64_t* a, const uint64_t* b, uint32_t npoly,
                           uint32_t nlimbs, bool broadcast, void* stream) {
  if (!c || !out || !a || !b) return fail(CKKS_EINVAL, "null argument");
  if (nlimbs == 0 || nlimbs > c->nq) return fail(CKKS_ESHAPE, "nlimbs must be in [1, L+1]");
  if (npoly == 0) return CKKS_OK;
  if (npoly > 65535) return fail(CKKS_ESHAPE, "too many polynomials in one call");
  DeviceGuard guard(c->device);
  if (!guard.ok) return fail(CKKS_EHIP, "cannot select the context's device");
  PointwiseArgs pa{(u64*)out, (const u64*)a, (const u64*)b, c->d_mods, c->logN, nlimbs, broadcast ? 1u : 0u};
  ProfScope ps(c, mul ? PK_TENSOR : PK_ADD, (hipStream_t)stream);
  dim3 grid(c->N / 512, nlimbs, npoly), block(256);
  if (mul) hipLaunchKernelGGL(pmult_kernel, grid, block, 0, (hipStream_t)stream, pa);
  else hipLaunchKernelGGL(add_kernel, grid, block, 0, (hipStream_t)stream, pa);
  HIP_TRY(hipGetLastError());
  return CKKS_OK;
}
int ckks_pmult(ckks_ctx* c, uint64_t* ct_out, const uint64_t* ct_in, const uint64_t* pt, uint32_t B, uint32_t nlimbs,
               void* stream) {
  if (B > 32767) return fail(CKKS_ESHAPE, "batch must be in [1, 32767]");
  return pointwise_entry(c, true, ct_out, ct_in, pt, B * 2, nlimbs, true, stream);
}
int ckks_add(ckks_ctx* c, uint64_t* out, const uint64_t* a, const uint64_t* b, uint32_t npoly, uint32_t nlimbs,
             void* stream) {
  return pointwise_entry(c, false, out, a, b, npoly, nlimbs, false, stream);
}

}  // extern "C"
