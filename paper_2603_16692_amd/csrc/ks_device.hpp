// Device-side data structures, modular arithmetic and NTT building blocks.
//
// Two arithmetics share the transform code:
//  * ArF, for the Q primes (q < 2^50): residues are held as integer-valued
//    doubles and multiplied with FP64 FMA. For a product p = a*b,
//    h = fl(a*b), l = fma(a, b, -h) gives p = h + l exactly; k = rint(h * fl(1/q))
//    is within 1/2 + 1.5*2^-52*|p|/q of p/q, and r = fma(-k, q, h) + l = p - k*q
//    exactly whenever |p| <= 2^103. So |r| <= q/2 + 1.5*2^-52*|p|. The
//    transform keeps every value within 8q < 2^53 (see ArF), where products of a
//    value and a balanced twiddle (|w| <= q/2) stay below 2^102. MI355X runs FP64
//    FMA at the full vector rate: such a product takes 6 instructions, one of a P
//    prime by a constant 13 and of two variables 17.
//  * ArI, for the P primes: uint64 residues, lazily reduced up to 2^64. The P
//    primes are the largest p = 2^60 - delta = 1 (mod 2N), and delta < 2^29 for
//    every N and count the library takes (the host checks it), so a value folds
//    at bit 60 with one 32-bit multiply-add (p_red), and a product of two
//    variables is a 128-bit product folded twice (p_mul). Products by fixed
//    constants use Shoup's method (w' = floor(w * 2^64 / q)) with the low partial
//    product of the quotient left out. A 32-bit multiply or multiply-add issues
//    in 4.3 to 4.8 cycles per wavefront here, like any other vector instruction
//    of this code, so what counts is the number of instructions.
// At the boundary every limb is canonical uint64 residues. Between the two
// passes of a transform (the workspace arrays t1, ext1 and t2, and the caller's
// array between the passes of ks_ntt / ks_intt) Q-limb words are "raw": the bits
// of the integer-valued double as the pass left it, within 6q, which saves the
// canonical reduction at the store (8 instructions) and the conversion at the
// load (2) of every word. P-limb words there are in the lazy integer ranges
// stated at each kernel.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace ks {

// Per-limb constants (one entry per prime of the extended basis).
struct LimbC {
  uint64_t q;
  uint64_t nq;         // 2^64 - q
  uint64_t delta;      // 2^60 - q (P primes; below 2^29)
  uint64_t ninv, ninv_s;
  uint64_t red_s;      // floor(2^64 / q): Shoup companion of 1
  double qd;           // q as a double (exact for the Q primes)
  double qinv;         // fl(1 / q)
  double ninv_d;       // balanced N^-1 mod q (Q primes)
  // Recombination of the int8-MFMA base conversion (see mx_fold_q, mx_fold_p):
  double qinv32, q32;  // 2^32 fl(1 / q), 2^-32 q (exact scalings; Q primes)
  uint64_t cadj;       // (-2^51 - 2^83) mod q - 0x433 * 2^52 - 0x33 * 2^24 * (2^60 - q), mod 2^64 (P primes)
};

// Every table of one parameter set. Pointers are device addresses after
// upload (offsets into the host blob before it).
struct DevTables {
  int log_n, ell, k, nl, alpha, ndig;
  const LimbC* limb;        // [nl]
  const uint64_t* twf;      // [nl][N][2]: (psi^brv(i), Shoup) for i in [1, N)
  const uint64_t* twi;      // [nl][N][2]: (psi^-brv(i), Shoup)
  const double* twf_d;      // [ell][N]: balanced psi^brv(i) (Q primes)
  const double* twi_d;      // [ell][N]: balanced psi^-brv(i)
  const uint64_t* up_pre;   // [ell][2]: N^-1 * [(D_j/q_i)^-1]_{q_i}, Shoup (j = digit of i)
  const double* up_pre_d;   // [ell]: the same, balanced double
  const uint64_t* up_mat;   // [ell][nl][2]: [D_j/q_i]_t with its Shoup companion mod t
  const double* up_mat_d;   // [ell][ell]: [D_j/q_i]_{q_t}, balanced double (Q targets)
  const uint64_t* dn_pre;   // [k][2]: N^-1 * [(P/p_m)^-1]_{p_m}, Shoup
  const uint64_t* dn_mat;   // [k][ell][2]: [P/p_m]_{q_i}, Shoup mod q_i
  const double* dn_mat_d;   // [k][ell][2]: balanced [2^30 * P/p_m]_{q_i}, [P/p_m]_{q_i}
  const uint64_t* dn_pinv;  // [ell][2]: [P^-1]_{q_i}, Shoup
  const double* dn_pinv_d;  // [ell]: balanced [P^-1]_{q_i}
  const uint64_t* up_hinv;  // [ell][2]: [(D_j/q_i)^-1]_{q_i}, Shoup (no N^-1)
  const uint64_t* dn_hinv;  // [k][2]: [(P/p_m)^-1]_{p_m}, Shoup (no N^-1)
  // Constant operands of the int8-MFMA base conversion: per 4-target group
  // and MFMA step, 16 bytes per lane (see k_modup_cols_mx for the layout).
  const uint64_t* up_mx;    // [ndig][up_ng][up_nm][64][2]
  const uint64_t* dn_mx;    // [dn_ng][dn_nm][64][2]
  int up_ng, up_nm, dn_ng, dn_nm;
  // Rows of the evaluation key [ndig][2][evk_nl][N]: limb t < ell is row t,
  // P limb ell + m is row evk_p0 + m. At the top level evk_nl = nl and
  // evk_p0 = ell; at a lower level the key of the top level is read as is.
  int evk_nl, evk_p0;
};

// Row of limb t of the extended basis in one (digit, component) slice of the key.
__device__ __forceinline__ size_t key_row(const DevTables& tb, int j, int c, int t) {
  return ((size_t)j * 2 + c) * tb.evk_nl + (t < tb.ell ? t : tb.evk_p0 + (t - tb.ell));
}

// ------------------------------------------------------------ integers

__device__ __forceinline__ uint64_t mul_shoup(uint64_t a, uint64_t w, uint64_t ws, uint64_t q) {
  // a < 2^64, w < q: returns a*w mod q in [0, 2q).
  const uint64_t hi = __umul64hi(a, ws);
  return a * w - hi * q;
}

// The same with the quotient's low partial product and carries left out (nq =
// 2^64 - q): three fractions below 1 are dropped (of a1 s0, a0 s1 and a0 s0), whose sum
// is below 3, so the quotient is at most 2 below Shoup's, which is at most 1 below the true
// one, and the result is a*w mod q plus a multiple of q, in [0, 4q).
// 13 multiplies and additions against 18.
__device__ __forceinline__ uint64_t mul_shoup_lazy(uint64_t a, uint64_t w, uint64_t ws, uint64_t nq) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
  const uint32_t s0 = (uint32_t)ws, s1 = (uint32_t)(ws >> 32);
  const uint64_t h = (uint64_t)a1 * s1 + __umulhi(a1, s0) + __umulhi(a0, s1);
  return a * w + h * nq;
}

__device__ __forceinline__ uint64_t reduce2(uint64_t x, uint64_t q) { return x >= q ? x - q : x; }

// ---- P primes p = 2^60 - delta: 2^60 = delta (mod p)

constexpr uint64_t P_MASK = ((uint64_t)1 << 60) - 1;

// Any x < 2^64 to below 2^60 + 2^33 (within p (1 + 2^-26)).
__device__ __forceinline__ uint64_t p_red(uint64_t x, uint32_t delta) {
  return (x & P_MASK) + (uint64_t)(uint32_t)(x >> 60) * delta;
}
// Any x < 2^64 to its canonical residue.
__device__ __forceinline__ uint64_t p_canon(uint64_t x, uint64_t q, uint32_t delta) {
  return reduce2(p_red(x, delta), q);
}
// a*b mod p for a, b < 2^60 + 2^33, below 1.5 * 2^60: the product's bits from 60
// up times delta are below 2^89.1, and theirs below 2^58.6.
__device__ __forceinline__ uint64_t p_mul(uint64_t a, uint64_t b, uint32_t delta) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32), b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
  const uint64_t lo = (uint64_t)a0 * b0;
  uint64_t mid = (uint64_t)a0 * b1 + (lo >> 32);  // a1, b1 <= 2^28 + 2: no overflow
  mid += (uint64_t)a1 * b0;
  const uint64_t hi = (uint64_t)a1 * b1 + (mid >> 32);
  const uint32_t h0 = __builtin_amdgcn_alignbit((uint32_t)hi, (uint32_t)mid, 28);
  const uint32_t h1 = __builtin_amdgcn_alignbit((uint32_t)(hi >> 32), (uint32_t)hi, 28);
  const uint64_t t = (((uint64_t)((uint32_t)mid & 0x0FFFFFFFu) << 32) | (uint32_t)lo) + (uint64_t)h0 * delta;
  const uint64_t u = (uint64_t)h1 * delta + (t >> 32);
  const uint64_t low = ((uint64_t)((uint32_t)u & 0x0FFFFFFFu) << 32) | (uint32_t)t;
  return low + (uint64_t)(uint32_t)(u >> 28) * delta;
}

// --------------------------------------------------------------- FP64

// a*b mod q as an integer-valued double with |r| <= q/2 + 1.5*2^-52*|a*b|,
// for |a*b| <= 2^103 (see the header comment).
__device__ __forceinline__ double f_mul(double a, double b, double q, double qinv) {
  const double h = a * b;
  const double l = __fma_rn(a, b, -h);
  const double k = __builtin_rint(h * qinv);
  const double r = __fma_rn(-k, q, h);
  return r + l;
}

// x mod q into [-q/2 - 1, q/2 + 1], for integer-valued |x| < 2^53.
__device__ __forceinline__ double f_red(double x, double q, double qinv) {
  return __fma_rn(-__builtin_rint(x * qinv), q, x);
}

// Exact conversion of an integer 0 <= v < 2^53: its bits are those of the subnormal
// (or, from 2^52 on, smallest normal) double v 2^-1074. One instruction; an or and
// an addition through 2^52 are 1.6 (a 32-bit logic operation issues in 2.4 cycles a
// wavefront, any other in 4.2).
__device__ __forceinline__ double u2d(uint64_t v) {
  return __builtin_ldexp(__longlong_as_double((long long)v), 1074);
}

// Exact conversion of an integer-valued double in [0, 2^53).
__device__ __forceinline__ uint64_t d2u(double v) {
  return (uint64_t)__double_as_longlong(__builtin_ldexp(v, -1074));
}

// Canonical residue in [0, q) of an integer-valued |x| <= 1.9q, as a double.
// (x + 1/2)/q stays at least 1/(2q) > 2^-51 away from every integer, and for a
// magnitude below 2 its computed value is off by at most 2^-53 (the rounding of
// the fma) + 1.9 * 2^-53 (that of qinv) < 2^-51, so the floor is exact.
__device__ __forceinline__ double f_canon_d(double x, double q, double qinv) {
  return __fma_rn(-__builtin_floor(__fma_rn(x, qinv, 0.5 * qinv)), q, x);
}

// The same for an integer-valued |x| < 2^53.
__device__ __forceinline__ double f_canon_wide_d(double x, double q, double qinv) {
  return f_canon_d(f_red(x, q, qinv), q, qinv);
}

// Canonical residue as uint64, of |x| <= 1.9q and of |x| < 2^53.
__device__ __forceinline__ uint64_t f_canon(double x, double q, double qinv) { return d2u(f_canon_d(x, q, qinv)); }
__device__ __forceinline__ uint64_t f_canon_wide(double x, double q, double qinv) {
  return d2u(f_canon_wide_d(x, q, qinv));
}

// Raw words of Q-limb intermediates.
__device__ __forceinline__ double raw2d(uint64_t v) { return __longlong_as_double((long long)v); }
__device__ __forceinline__ uint64_t d2raw(double v) { return (uint64_t)__double_as_longlong(v); }

// ------------------------------------------------------ arithmetics

// Read-only table loads through the constant address space: when the
// address is the same for the whole wavefront (column-pass twiddles, BConv
// constants) they become scalar loads into SGPRs, sparing vector registers;
// otherwise they are ordinary vector loads.
template <class T>
__device__ __forceinline__ T ldc(const T* p) {
  return *(const __attribute__((address_space(4))) T*)(p);
}

struct Tw {
  uint64_t w, ws;
};

// UNI: idx is the same for the whole wavefront (a scalar load).
template <bool UNI>
__device__ __forceinline__ Tw load_tw(const uint64_t* table, uint32_t idx) {
  if constexpr (UNI) return Tw{ldc(table + 2 * (size_t)idx), ldc(table + 2 * (size_t)idx + 1)};
  const ulonglong2 v = reinterpret_cast<const ulonglong2*>(table)[idx];
  return Tw{v.x, v.y};
}

// Integer arithmetic of one P limb; `tw` is its (w, Shoup) table. Twiddle products
// are in [0, 4q) for any 64-bit operand, so a forward stage adds 4q to the bound
// of its inputs. sub_fwd reduces X (p_red, 3 instructions) in stages 0, 3, 6, ...
// of a group: a group of any raw input (< 2^64) leaves at most 13q + 2^33, and a
// column pass that starts from values below 2.2 * 2^60 skips the first reduction
// (6.2, 10.2, 14.2, then reduced: 5, 9 for up to 5 stages).
// An inverse stage maps inputs within 4q to a lazy sum within 8q and a product
// in [0, 4q), and those to a reduced sum; exits are within 4q.
// With conditional subtractions in every stage and the exact Shoup quotient a
// butterfly was 27 instructions against 19, and a key product by Montgomery's
// reduction 39 against 17 (p_mul): (4, 2^16, 32), batch 8, 946 us then and 863
// with this; (2, 2^13, 6), one ciphertext, 30.6 and 27.1.
struct ArI {
  using T = uint64_t;
  uint64_t q, nq;
  uint32_t delta;
  const uint64_t* tw;
  using TwT = Tw;
  template <bool UNI>
  __device__ __forceinline__ TwT twiddle(uint32_t idx) const {
    return load_tw<UNI>(tw, idx);
  }
  template <bool RED>
  __device__ __forceinline__ void fwd(T& X, T& Y, const TwT& t) const {
    const uint64_t x = RED ? p_red(X, delta) : X;
    const uint64_t v = mul_shoup_lazy(Y, t.w, t.ws, nq);
    X = x + v;
    Y = x + 4 * q - v;
  }
  template <bool RED>
  __device__ __forceinline__ void inv(T& X, T& Y, const TwT& t) const {
    const uint64_t s = X + Y, d = X + 8 * q - Y;
    X = RED ? p_red(s, delta) : s;
    Y = mul_shoup_lazy(d, t.w, t.ws, nq);
  }
  __device__ static constexpr bool fwd_red(int rho, bool red0) { return rho % 3 == 0 && (rho > 0 || red0); }
  __device__ static constexpr bool inv_red(int rho, int k) { return rho == 0 || ((k - 1 - rho) & 1); }
};

// FP64 arithmetic of one Q limb; `tw` is its balanced twiddle table. Values stay
// below 8q < 2^53 in magnitude, where sums are exact and products with a
// balanced twiddle (|w| <= q/2) below 2^102.
//
// Bounds in units of q: a product of |a| <= A and a balanced twiddle is within
// 0.5 + 0.1875 A (1.5 * 2^-52 * q/2 < 0.1875). A forward stage that reduces X maps
// inputs within B to outputs within 1 + 0.1875 B, a lazy one to 0.5 + 1.1875 B.
// sub_fwd reduces in its first stage only: a group of K <= 4 stages then maps
// B <= 8 to at most 2.51 + 0.27 B (K = 3) or 3.48 + 0.32 B (K = 4, less for K < 3), so
// a block pass of a raw input within 6 stays within 5.4 (E = 16; 4.1 with E <= 8)
// and leaves 5.2 (3.6). A column pass starts from reduced values (within 1) and
// skips even that reduction: 1 -> 1.69 -> 2.51 -> 3.48 -> 4.63 -> 5.99 for up to
// 5 stages. The transforms are bound by the instructions they issue: reducing in
// every other stage (one more of 9 per butterfly at E = 8) with canonical words
// between the passes ran 973 us at (4, 2^16, 32), batch 8, against 946 us, and
// 1334 against 1279 us at (8, 2^17, 56), batch 2.
// An inverse stage maps B to X + Y within 2B and W*(X - Y) within 0.5 + 0.375 B:
// from B <= 2 one lazy stage gives 4, and a reducing one (sums up to 8) returns to 2.
struct ArF {
  using T = double;
  double q, qinv;
  const double* tw;   // the table, or a block's staged copy of it
  const double* ctw;  // the table, read where the whole wavefront takes one twiddle (UNI)
  using TwT = double;
  template <bool UNI>
  __device__ __forceinline__ TwT twiddle(uint32_t idx) const {
    if constexpr (UNI) return ldc(ctw + idx);
    return tw[idx];
  }
  // RED: X is first reduced to |X| <= q/2 + 2.
  template <bool RED>
  __device__ __forceinline__ void fwd(T& X, T& Y, TwT w) const {
    const double x = RED ? f_red(X, q, qinv) : X;
    const double v = f_mul(Y, w, q, qinv);
    X = x + v;
    Y = x - v;
  }
  // RED: the sum is reduced.
  template <bool RED>
  __device__ __forceinline__ void inv(T& X, T& Y, TwT w) const {
    const double s = X + Y, d = X - Y;
    X = RED ? f_red(s, q, qinv) : s;
    Y = f_mul(d, w, q, qinv);
  }
  __device__ static constexpr bool fwd_red(int rho, bool red0) { return rho == 0 && red0; }
  // stage rho of a group of k inverse stages (executed from rho = k - 1 down to 0)
  __device__ static constexpr bool inv_red(int rho, int k) { return rho == 0 || ((k - 1 - rho) & 1); }
};

// One subproblem of 2^K elements in registers. Local stage rho pairs
// elements at distance 2^(K-1-rho); the twiddle of local group g is entry
// (base << rho) + g of the bit-reversed table, where `base` is the table
// index of the subproblem at its first stage (the butterfly tree of the
// transform numbers node u's children 2u and 2u+1).
// Which stages reduce their running sums is the arithmetic's choice (fwd_red,
// inv_red); RED0 = false tells it that the inputs are already reduced.
//
// PS >= 0: the table is a block's staged copy (base = 2^PS + p) whose stages
// PS.. are stored group-major, entry (p << rho) + g of stage PS + rho at
// 2^(PS + rho) + (g << PS) + p, so that the lanes of a wave (consecutive p)
// read consecutive words.
//
// The stages themselves, the twiddle of stage rho and group g given by tw(rho, g):
template <int K, bool RED0 = true, class Ar, class F>
__device__ __forceinline__ void sub_fwd_by(const Ar& A, typename Ar::T* x, F tw) {
#pragma unroll
  for (int rho = 0; rho < K; ++rho) {
    const int dist = 1 << (K - 1 - rho);
#pragma unroll
    for (int j = 0; j < (1 << K); ++j) {
      if (j & dist) continue;
      const typename Ar::TwT w = tw(rho, (uint32_t)(j >> (K - rho)));
      if (Ar::fwd_red(rho, RED0))
        A.template fwd<true>(x[j], x[j + dist], w);
      else
        A.template fwd<false>(x[j], x[j + dist], w);
    }
  }
}
template <int K, class Ar, class F>
__device__ __forceinline__ void sub_inv_by(const Ar& A, typename Ar::T* x, F tw) {
#pragma unroll
  for (int rho = K - 1; rho >= 0; --rho) {
    const int dist = 1 << (K - 1 - rho);
#pragma unroll
    for (int j = 0; j < (1 << K); ++j) {
      if (j & dist) continue;
      const typename Ar::TwT w = tw(rho, (uint32_t)(j >> (K - rho)));
      if (Ar::inv_red(rho, K))
        A.template inv<true>(x[j], x[j + dist], w);
      else
        A.template inv<false>(x[j], x[j + dist], w);
    }
  }
}

// With the twiddles read from the table where they are used.
template <int K, int PS = -1, bool RED0 = true, bool UNI = false, class Ar>
__device__ __forceinline__ void sub_fwd(const Ar& A, typename Ar::T* x, uint32_t base) {
  sub_fwd_by<K, RED0>(A, x, [&](int rho, uint32_t g) {
    return A.template twiddle<UNI>(PS < 0 ? (base << rho) + g
                                          : base + ((1u << (PS + rho)) - (1u << PS)) + (g << (PS < 0 ? 0 : PS)));
  });
}
template <int K, bool UNI = false, class Ar>
__device__ __forceinline__ void sub_inv(const Ar& A, typename Ar::T* x, uint32_t base) {
  sub_inv_by<K>(A, x, [&](int rho, uint32_t g) { return A.template twiddle<UNI>((base << rho) + g); });
}

// The 2^K - 1 twiddles of one subproblem, loaded ahead of use.
template <int K, class Ar>
__device__ __forceinline__ void load_sub_tw(const Ar& A, typename Ar::TwT (&w)[(1 << K) - 1], uint32_t base) {
#pragma unroll
  for (int rho = 0; rho < K; ++rho)
#pragma unroll
    for (int g = 0; g < (1 << rho); ++g) w[(1 << rho) - 1 + g] = A.template twiddle<false>((base << rho) + (uint32_t)g);
}

// Operands of HMUL or HROT folded into a fused KeySwitch (a == nullptr: a
// plain KeySwitch). HMUL: ciphertexts a and b [items][2][ell][N], galois 0.
// HROT: a the ciphertext to rotate, b unused, galois the Galois element.
struct EvalIn {
  const uint64_t* a;
  const uint64_t* b;
  uint32_t galois;
};

// Slot of the input that slot t of sigma_g(x) takes in NTT form (slot t holds
// the evaluation at psi^(2 brv(t) + 1)): 2 brv(t') + 1 = g (2 brv(t) + 1) mod 2N.
__device__ __forceinline__ uint32_t galois_src(uint32_t t, uint32_t g, int log_n) {
  const uint32_t e = 2u * (__brev(t) >> (32 - log_n)) + 1u;
  const uint32_t e2 = (uint32_t)(((uint64_t)g * e) & ((2u << log_n) - 1u));
  return __brev((e2 - 1u) >> 1) >> (32 - log_n);
}

// LDS word of element x: one pad word after every 16, so that the strided
// round layouts hit distinct banks.
__device__ __forceinline__ int lds_pad(int x) { return x + (int)((unsigned)x >> 4); }

// lds_pad(x0 + d) = lds_pad(x0) + d + (d >> 4) for the strides d = j*L of a
// round layout (L a power of two, x0 = pos(r, tid, u, 0)): x0 mod 16 plus
// d mod 16 never reaches 16, since either 16 divides d, or x0 mod 16 < L and
// d mod 16 <= 16 - L, or the whole group of 2^k*L <= 16 elements shares its
// 16-word line. The per-register offsets are then compile-time constants.
__device__ constexpr int pad_step(int d) { return d + (d >> 4); }

// Orders this wavefront's memory accesses before this point against those after
// it. Its LDS accesses execute in order, so that no instruction is needed: it keeps
// the compiler from moving one past another of a different type or lane.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Transform stages log_r .. log_n-1 (forward) of one contiguous block of
// M = 2^LOGM elements, block index b in [0, R). T = M / E threads, E = 2^LOGE
// elements per thread, done in rounds of LOGE stages (the first round takes
// the remainder). Between rounds the block goes through LDS.
//
// Register layouts ("positions"): in round r with first local stage s0 and
// size k, register u*2^k + j of thread tid holds element
//   x = hi * (M >> s0) + lo + j * L,  L = M >> (s0 + k),  p = tid + u*T,
//   lo = p mod L, hi = p / L.
// "FR" is the first round's layout (x = p + j*(M >> K1)); "CL" is the
// coalesced layout: wave w owns elements [64E w, 64E (w + 1)), its lane l holds
// x = 64E w + 64 i + l in register i (x = tid + i*T for a block of at most 64
// threads). Forward transforms take FR and return CL; inverse transforms take
// CL and return FR. Both layouts give the lanes of a wave consecutive addresses
// for every register, so global loads and stores at either end are coalesced;
// the last round's own layout (x = tid*E + j) is transposed through LDS, and as
// it holds the same elements in each wave as CL, without a workgroup barrier.
template <int LOGM, int LOGE>
struct BlockNtt {
  static constexpr int M = 1 << LOGM;
  static constexpr int E = 1 << LOGE;
  static constexpr int LOGT = LOGM - LOGE;
  static constexpr int T = M / E;
  static constexpr int NR = (LOGM + LOGE - 1) / LOGE;
  static constexpr int K1 = LOGM - LOGE * (NR - 1);
  static constexpr int LDS_WORDS = M + (M >> 4);
  static_assert(NR >= 2, "a block needs at least two rounds");

  __device__ static constexpr int round_s0(int r) { return r == 0 ? 0 : K1 + (r - 1) * LOGE; }
  __device__ static constexpr int round_k(int r) { return r == 0 ? K1 : LOGE; }

  __device__ static __forceinline__ int pos(int r, int tid, int u, int j) {
    const int s0 = round_s0(r), k = round_k(r);
    const int p = tid + u * T;
    const int L = M >> (s0 + k);
    const int lo = p & (L - 1);
    const int hi = p / L;
    return hi * (M >> s0) + lo + j * L;
  }
  // Rounds whose butterfly groups are at least a wavefront wide: all lanes of a
  // wave take the same twiddles, which come by scalar loads from the table (the
  // first two of four rounds at blocks of 2^12 with E = 8: 14 of 28 twiddle reads
  // of a thread, and the registers they took; (4, 2^16, 32), batch 8, 815 -> 809 us).
  // With 4 elements a thread only the first round does: a scalar load is waited
  // for together with all outstanding LDS accesses, which costs the latency variants
  // more (one ciphertext of (2, 2^15, 10) from a graph 52.0 -> 54.1 us).
  __device__ static constexpr bool uniform(int r) {
    return r == 0 || (LOGE >= 3 && (M >> (round_s0(r) + round_k(r))) >= W);
  }
  __device__ static __forceinline__ uint32_t base(int r, int tid, int u, uint32_t B0) {
    const int s0 = round_s0(r), k = round_k(r);
    if (uniform(r)) tid = __builtin_amdgcn_readfirstlane(tid / W * W);
    const int p = tid + u * T;
    const int L = M >> (s0 + k);
    return (B0 << s0) + (uint32_t)(p / L);
  }
  // Element of register i: a per-thread base plus a constant.
  static constexpr int W = T < 64 ? T : 64;
  __device__ static constexpr int fr_step(int i) { return (i >> K1) * T + (i & ((1 << K1) - 1)) * (M >> K1); }
  __device__ static constexpr int cl_step(int i) { return i * W; }
  __device__ static __forceinline__ int fr_base(int tid) { return tid; }
  __device__ static __forceinline__ int cl_base(int tid) { return (tid / W) * (W * E) + (tid % W); }
  __device__ static __forceinline__ int fr_pos(int tid, int i) { return fr_base(tid) + fr_step(i); }
  __device__ static __forceinline__ int cl_pos(int tid, int i) { return cl_base(tid) + cl_step(i); }

  // The twiddles of a round that is not uniform (LOGE stages, one subproblem a
  // thread), loaded before the exchange that precedes it. All rounds' together at
  // the start of the transform, where they fit the registers, measured the same.
  // (AHEAD false: read where they are used, for a kernel that has no registers for them.)
  template <class Ar>
  struct TwRegs {
    typename Ar::TwT w[E - 1];
  };
  template <class Ar>
  __device__ static __forceinline__ void load_round_tw(const Ar& A, TwRegs<Ar>& t, int r, int tid, uint32_t G0) {
    load_sub_tw<LOGE>(A, t.w, base(r, tid, 0, G0));
  }

  // Round 0 of K1 stages is uniform: its groups are M >> K1 >= T elements wide.
  template <class Ar>
  __device__ static __forceinline__ void round0_fwd(const Ar& A, typename Ar::T* x, int tid, uint32_t G0) {
    static_assert(uniform(0), "");
#pragma unroll
    for (int u = 0; u < (E >> K1); ++u) sub_fwd<K1, -1, true, true>(A, x + u * (1 << K1), base(0, tid, u, G0));
  }
  template <class Ar>
  __device__ static __forceinline__ void round0_inv(const Ar& A, typename Ar::T* x, int tid, uint32_t G0) {
#pragma unroll
    for (int u = 0; u < (E >> K1); ++u) sub_inv<K1, true>(A, x + u * (1 << K1), base(0, tid, u, G0));
  }
  // First stage of the last round, where every thread has its own twiddles.
  static constexpr int LAST_S0 = LOGM - LOGE;
  __device__ static constexpr int round_l(int r) { return M >> (round_s0(r) + round_k(r)); }
  template <int K, class V>
  __device__ static __forceinline__ void to_lds(const V* x, V* lds, int r, int tid) {
#pragma unroll
    for (int u = 0; u < (E >> K); ++u) {
      V* b = lds + lds_pad(pos(r, tid, u, 0));
#pragma unroll
      for (int j = 0; j < (1 << K); ++j) b[pad_step(j * round_l(r))] = x[u * (1 << K) + j];
    }
  }
  template <int K, class V>
  __device__ static __forceinline__ void from_lds(V* x, const V* lds, int r, int tid) {
#pragma unroll
    for (int u = 0; u < (E >> K); ++u) {
      const V* b = lds + lds_pad(pos(r, tid, u, 0));
#pragma unroll
      for (int j = 0; j < (1 << K); ++j) x[u * (1 << K) + j] = b[pad_step(j * round_l(r))];
    }
  }

  // Whether the layout of round q and the next one hold the same elements in
  // each wavefront. In a round whose groups are at most 64 elements apart
  // (L <= 64) with one register subproblem per thread, the 64 threads of wave
  // w hold exactly elements [64E w, 64E (w + 1)), and so in every later
  // round: the exchange between such rounds touches only the wave's own LDS
  // words, and a wave-local ordering point replaces the workgroup barrier.
  __device__ static constexpr bool wave_local(int q) {
    return T <= 64 || ((q >= 1 || K1 == LOGE) && round_l(q) <= 64);
  }
  // Orders the LDS stores before this point against the loads after it: for
  // the whole workgroup, or (local) for this wavefront.
  __device__ static __forceinline__ void exchange_sync(bool local) {
    if (local)
      wave_sync();
    else
      __syncthreads();
  }

  // Forward: x enters in FR, leaves in CL. G0 = R + b. REUSE: a previous call
  // read the LDS block, so a barrier precedes the first store. STAGED: A.tw is a
  // staged copy of the block's twiddles with the last round's stages stored
  // group-major (sub_fwd with PS = LAST_S0), read where they are used. `between(r)`
  // runs before the exchange that precedes round r: loads that a kernel needs after
  // the transform, spread over it.
  struct Nothing {
    __device__ __forceinline__ void operator()(int) const {}
  };
  template <bool STAGED = false, bool REUSE = false, bool AHEAD = true, class Ar, class H = Nothing>
  __device__ static __forceinline__ void fwd(const Ar& A, typename Ar::T* x, typename Ar::T* lds, int tid, uint32_t G0,
                                             H between = H()) {
    round0_fwd(A, x, tid, G0);
    if (REUSE) __syncthreads();
    to_lds<K1>(x, lds, 0, tid);
#pragma unroll
    for (int r = 1; r < NR; ++r) {
      TwRegs<Ar> t;
      if (AHEAD && !STAGED && !uniform(r)) load_round_tw(A, t, r, tid, G0);
      between(r);
      exchange_sync(wave_local(r - 1));
      from_lds<LOGE>(x, lds, r, tid);
      if (uniform(r))
        sub_fwd<LOGE, -1, true, true>(A, x, base(r, tid, 0, G0));
      else if (STAGED && r == NR - 1)
        sub_fwd<LOGE, LAST_S0>(A, x, base(r, tid, 0, 1u));
      else if (STAGED)
        sub_fwd<LOGE>(A, x, base(r, tid, 0, 1u));
      else if (!AHEAD)
        sub_fwd<LOGE>(A, x, base(r, tid, 0, G0));
      else
        sub_fwd_by<LOGE>(A, x, [&](int rho, uint32_t g) { return t.w[(1 << rho) - 1 + g]; });
      to_lds<LOGE>(x, lds, r, tid);
    }
    exchange_sync(true);
    const typename Ar::T* c = lds + lds_pad(cl_base(tid));
#pragma unroll
    for (int i = 0; i < E; ++i) x[i] = c[pad_step(cl_step(i))];
  }

  // Inverse: x enters in CL, leaves in FR. REUSE as in fwd.
  template <bool REUSE = false, bool AHEAD = true, class Ar>
  __device__ static void inv(const Ar& A, typename Ar::T* x, typename Ar::T* lds, int tid, uint32_t G0) {
    if (REUSE) __syncthreads();
    typename Ar::T* c = lds + lds_pad(cl_base(tid));
#pragma unroll
    for (int i = 0; i < E; ++i) c[pad_step(cl_step(i))] = x[i];
#pragma unroll
    for (int r = NR - 1; r >= 1; --r) {
      TwRegs<Ar> t;
      if (AHEAD && !uniform(r)) load_round_tw(A, t, r, tid, G0);
      exchange_sync(r == NR - 1 || wave_local(r));  // the first read follows the CL stores
      from_lds<LOGE>(x, lds, r, tid);
      if (uniform(r))
        sub_inv<LOGE, true>(A, x, base(r, tid, 0, G0));
      else if (!AHEAD)
        sub_inv<LOGE>(A, x, base(r, tid, 0, G0));
      else
        sub_inv_by<LOGE>(A, x, [&](int rho, uint32_t g) { return t.w[(1 << rho) - 1 + g]; });
      to_lds<LOGE>(x, lds, r, tid);
    }
    exchange_sync(wave_local(0));
    from_lds<K1>(x, lds, 0, tid);
    round0_inv(A, x, tid, G0);
  }
};

}  // namespace ks
