// HIP kernels of the KeySwitch path for gfx950, and their host launchers.
//
// A limb of N = R * M coefficients is transformed in two passes:
//   * a column pass: thread c owns the R coefficients c, c + M, ..., and runs
//     the first log R stages of the forward transform (or the last log R of the
//     inverse) in registers; consecutive threads touch consecutive addresses;
//   * a block pass: a workgroup owns M consecutive coefficients and runs the
//     remaining log M stages through LDS (BlockNtt), with coalesced global
//     loads and stores at both ends.
// ModUp's BConv sits between the inverse column pass and the forward column
// pass of the new limbs (same columns, all in registers), KeyMult follows the
// forward block pass, and ModDown repeats the pattern. Q limbs (q < 2^50) run
// on FP64 arithmetic (ArF), P limbs (p < 2^60) on 64-bit integers (ArI); the
// choice is made per workgroup, since a workgroup works on a single limb.
// Every kernel states the ranges of the values it reads and writes.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "ks_device.hpp"
#include "ks_kernels.hpp"

namespace ks {

namespace {

constexpr int TC = 64;  // threads of a column-pass workgroup

__device__ __forceinline__ size_t lane_col() { return (size_t)blockIdx.x * TC + threadIdx.x; }

__device__ __forceinline__ ArF arf(const DevTables& tb, const LimbC& L, int limb, bool inverse) {
  const size_t N = (size_t)1 << tb.log_n;
  const double* tw = (inverse ? tb.twi_d : tb.twf_d) + (size_t)limb * N;
  return ArF{L.qd, L.qinv, tw, tw};
}
__device__ __forceinline__ ArI ari(const DevTables& tb, const LimbC& L, int limb, bool inverse) {
  const size_t N = (size_t)1 << tb.log_n;
  return ArI{L.q, L.nq, (uint32_t)L.delta, (inverse ? tb.twi : tb.twf) + (size_t)limb * N * 2};
}

// XCD-aware placement of block-pass workgroups. MI355X dispatches workgroup
// w to XCD w mod 8, and each XCD has its own 4 MB L2. A block-pass "tile" is
// one (limb, block) pair; the batch items of a tile read the same twiddles
// and, in KeyMult, the same key blocks. The mapping below puts all items of a
// tile on one XCD at consecutive dispatch slots, so those shared reads are
// served by that XCD's L2 instead of going to HBM once per item.
// Grid: 8 * ceil(ntiles / 8) * items workgroups (1-D).
struct Tile {
  int tile, item;
  bool valid;
};
__device__ __forceinline__ Tile xcd_tile(int ntiles, int items) {
  const int w = blockIdx.x;
  const int xcd = w & 7, local = w >> 3;
  const int item = local % items, unit = local / items;
  const int tile = unit * 8 + xcd;
  return Tile{tile, item, tile < ntiles};
}
inline unsigned xcd_grid(int ntiles, int items) { return (unsigned)(((ntiles + 7) / 8) * 8 * items); }

// BlockNtt::fwd with the thread index hidden from the optimiser: a kernel that
// runs several transforms would otherwise keep every LDS and twiddle address
// of all rounds live from the first transform to the last, which costs more
// registers than recomputing them.
template <class B, bool STAGED = false, bool REUSE = true, bool AHEAD = true, class Ar, class H = typename B::Nothing>
__device__ __forceinline__ void fwd_opaque(const Ar& A, typename Ar::T* v, typename Ar::T* ld, int tid, uint32_t B0,
                                           H between = H()) {
  int t = tid;
  asm volatile("" : "+v"(t));
  B::template fwd<STAGED, REUSE, AHEAD>(A, v, ld, t, B0, between);
}
template <class B, bool REUSE = true, bool AHEAD = true, class Ar>
__device__ __forceinline__ void inv_opaque(const Ar& A, typename Ar::T* v, typename Ar::T* ld, int tid,
                                           uint32_t B0) {
  int t = tid;
  asm volatile("" : "+v"(t));
  B::template inv<REUSE, AHEAD>(A, v, ld, t, B0);
}

// A word of an intermediate of the KeySwitch that one workgroup reads, once: a
// non-temporal load, first to leave the L2, so that what is read again (the key for
// the items of a tile, tables) and what the kernel before wrote for the next one stays.
// (4, 2^16, 32), one ciphertext, 154 -> 142 us, batch 8, 783 -> 770; (2, 2^15, 10),
// batch 32, 424 -> 411. Not for the key: level 13 of (4, 2^16, 32), batch 3, 151 -> 158;
// nor for d and the transforms in place, 2% of (2, 2^15, 10), batch 32.
__device__ __forceinline__ uint64_t ld_once(const uint64_t* p) { return __builtin_nontemporal_load(p); }

// Column kernels with ONCE false are for a launch over a chunk of the targets, which
// leaves the sources in the caches for the next chunk's launch: (2, 2^15, 10), batch 8,
// DPOC with 4 chunks, 241 us, with non-temporal loads 247. (A branch in the kernel
// costs the others 1%.) Where a small launch shares a tile between workgroups (mx_parts) they
// load the same words at about the same time, and either kind of load takes the same time:
// (4, 2^16, 32), one ciphertext, with ordinary loads 153.2 us, with these 153.4; 40 shared
// launches of N = 2^10 to 2^16 within 1% both ways.
template <bool ONCE>
__device__ __forceinline__ uint64_t ld_col(const uint64_t* p) {
  if constexpr (ONCE)
    return ld_once(p);
  else
    return *p;
}

// The E words of a thread of a block of M words at `src`, in the FR or CL
// layout, as they are in memory: kernels that load ahead of use convert them
// where they use them, since a conversion at the load would wait for it. Buffer
// loads keep every address but one 32-bit offset in scalar registers, and that
// offset is recomputed for each call (the hidden thread index) instead of being
// held through the transforms. Words in the FR layout are an intermediate's, read
// this once (see ld_once); the key, the twiddles and d are read by several workgroups.
template <class B>
__device__ __forceinline__ void load_words(const uint64_t* src, bool cl, int tid, uint64_t (&w)[B::E]) {
  typedef unsigned int v2u __attribute__((ext_vector_type(2)));
  int t = tid;
  asm volatile("" : "+v"(t));
  const int base = 8 * (cl ? B::cl_base(t) : B::fr_base(t));
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t*>(src), 0, B::M * 8, 0x00027000);
#pragma unroll
  for (int i = 0; i < B::E; ++i) {
    v2u v;
    if (cl)
      v = __builtin_amdgcn_raw_buffer_load_b64(rs, base, 8 * B::cl_step(i), 0);
    else
      v = __builtin_amdgcn_raw_buffer_load_b64(rs, base, 8 * B::fr_step(i), 2);  // non-temporal
    w[i] = ((uint64_t)v.y << 32) | v.x;
  }
}

// ------------------------------------------------------- standalone passes

// Column pass of ks_ntt / ks_intt on x [items][nlimbs][N] (limb r uses prime
// first + r). Q limbs: forward canonical in, raw out; inverse raw in, canonical
// out. P limbs: forward canonical in, below 2^64 out; inverse [0, 4q] in,
// canonical out. The inverse includes N^-1.
template <int LOGR, bool INV>
__global__ __launch_bounds__(TC) void k_cols(DevTables tb, uint64_t* x, int first, int nlimbs, int log_m) {
  constexpr int R = 1 << LOGR;
  const int M = 1 << log_m;
  const size_t c = lane_col();
  if (c >= (size_t)M) return;
  const int limb = first + blockIdx.y;
  const LimbC L = tb.limb[limb];
  const size_t N = (size_t)M * R;
  uint64_t* a = x + ((size_t)blockIdx.z * nlimbs + blockIdx.y) * N;
  if (limb < tb.ell) {
    const ArF A = arf(tb, L, limb, INV);
    double v[R];
    if (!INV) {
#pragma unroll
      for (int i = 0; i < R; ++i) v[i] = u2d(a[c + (size_t)i * M]);
      sub_fwd<LOGR, -1, false>(A, v, 1u);
#pragma unroll
      for (int i = 0; i < R; ++i) a[c + (size_t)i * M] = d2raw(v[i]);
    } else {
#pragma unroll
      for (int i = 0; i < R; ++i) v[i] = raw2d(a[c + (size_t)i * M]);
      sub_inv<LOGR>(A, v, 1u);
#pragma unroll
      for (int i = 0; i < R; ++i)  // |v| <= 2q: the product is within 0.88q
        a[c + (size_t)i * M] = f_canon(f_mul(v[i], L.ninv_d, L.qd, L.qinv), L.qd, L.qinv);
    }
  } else {
    const ArI A = ari(tb, L, limb, INV);
    uint64_t v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = a[c + (size_t)i * M];
    if (!INV) {
      sub_fwd<LOGR, -1, false>(A, v, 1u);
    } else {
      sub_inv<LOGR>(A, v, 1u);
#pragma unroll
      for (int i = 0; i < R; ++i) v[i] = p_canon(mul_shoup_lazy(v[i], L.ninv, L.ninv_s, L.nq), L.q, L.delta);
    }
#pragma unroll
    for (int i = 0; i < R; ++i) a[c + (size_t)i * M] = v[i];
  }
}

// Block pass of ks_ntt / ks_intt (and of d at the start of ModUp): one block
// of one limb (first + l) of one item per workgroup (placed by xcd_tile),
// src -> dst (may alias). `whole`: the pass is the whole transform (no column
// pass), with canonical words at both ends and, in the inverse, times N^-1.
// Otherwise forward: Q raw in, P below 2^64 in, canonical out; inverse: canonical
// in, out Q raw (within 2q), P [0, 4q].
template <int LOGM, int LOGE, bool INV>
__global__ __launch_bounds__((1 << (LOGM - LOGE)), LOGM >= 12 ? 4 : 1) void k_blocks(DevTables tb, const uint64_t* src, uint64_t* dst,
                                                                 int first, int nlimbs, int items, int whole) {
  using B = BlockNtt<LOGM, LOGE>;
  extern __shared__ uint64_t lds[];
  const size_t N = (size_t)1 << tb.log_n;
  const int R = (int)(N >> LOGM);
  const Tile tl = xcd_tile(R * nlimbs, items);
  if (!tl.valid) return;
  const int tid = threadIdx.x, b = tl.tile % R, lrel = tl.tile / R;
  const int limb = first + lrel;
  const LimbC L = tb.limb[limb];
  const uint32_t B0 = (uint32_t)R + b;
  const size_t off = ((size_t)tl.item * nlimbs + lrel) * N + (size_t)b * B::M;
  const uint64_t* s = src + off;
  uint64_t* d = dst + off;
  if (limb < tb.ell) {
    const ArF A = arf(tb, L, limb, INV);
    double* ld = reinterpret_cast<double*>(lds);
    double v[B::E];
    if (!INV) {
      if (whole) {
#pragma unroll
        for (int i = 0; i < B::E; ++i) v[i] = u2d(s[B::fr_pos(tid, i)]);
      } else {
#pragma unroll
        for (int i = 0; i < B::E; ++i) v[i] = raw2d(s[B::fr_pos(tid, i)]);
      }
      B::fwd(A, v, ld, tid, B0);
#pragma unroll
      for (int i = 0; i < B::E; ++i) d[B::cl_pos(tid, i)] = f_canon_wide(v[i], L.qd, L.qinv);
    } else {
#pragma unroll
      for (int i = 0; i < B::E; ++i) v[i] = u2d(s[B::cl_pos(tid, i)]);
      B::inv(A, v, ld, tid, B0);
      if (whole) {
#pragma unroll
        for (int i = 0; i < B::E; ++i)
          d[B::fr_pos(tid, i)] = f_canon(f_mul(v[i], L.ninv_d, L.qd, L.qinv), L.qd, L.qinv);
      } else {
#pragma unroll
        for (int i = 0; i < B::E; ++i) d[B::fr_pos(tid, i)] = d2raw(v[i]);
      }
    }
  } else {
    const ArI A = ari(tb, L, limb, INV);
    uint64_t v[B::E];
    if (!INV) {
#pragma unroll
      for (int i = 0; i < B::E; ++i) v[i] = s[B::fr_pos(tid, i)];
      B::fwd(A, v, lds, tid, B0);
#pragma unroll
      for (int i = 0; i < B::E; ++i) d[B::cl_pos(tid, i)] = p_canon(v[i], L.q, L.delta);
    } else {
#pragma unroll
      for (int i = 0; i < B::E; ++i) v[i] = s[B::cl_pos(tid, i)];
      B::inv(A, v, lds, tid, B0);
      if (whole) {
#pragma unroll
        for (int i = 0; i < B::E; ++i)
          v[i] = p_canon(mul_shoup_lazy(v[i], L.ninv, L.ninv_s, L.nq), L.q, L.delta);
      }
#pragma unroll
      for (int i = 0; i < B::E; ++i) d[B::fr_pos(tid, i)] = v[i];
    }
  }
}

// The first pass of a fused HMUL or HROT (in place of the inverse block pass
// of d): one block of one Q limb of one item per workgroup computes d = a1 b1
// (HMUL) or d = sigma_g(c1) (HROT, a gather in NTT form), stores it (the
// digit-parallel last pass reads it as its own digit) and runs the inverse
// block pass into t1, as k_blocks<INV> does for d.
template <int LOGM, int LOGE>
__global__ __launch_bounds__((1 << (LOGM - LOGE)), LOGM >= 12 ? 4 : 1) void k_eval_blocks(
    DevTables tb, EvalIn ev, uint64_t* d2, uint64_t* t1, int items) {
  using B = BlockNtt<LOGM, LOGE>;
  extern __shared__ uint64_t lds[];
  const size_t N = (size_t)1 << tb.log_n;
  const int R = (int)(N >> LOGM), ell = tb.ell;
  const Tile tl = xcd_tile(R * ell, items);
  if (!tl.valid) return;
  const int tid = threadIdx.x, blk = tl.tile % R, i = tl.tile / R;
  const LimbC L = tb.limb[i];
  const size_t boff = (size_t)blk * B::M;
  const uint64_t* a1 = ev.a + (((size_t)tl.item * 2 + 1) * ell + i) * N;  // the limb's component 1
  const size_t off = ((size_t)tl.item * ell + i) * N + boff;
  double v[B::E];
  if (ev.galois) {
#pragma unroll
    for (int e = 0; e < B::E; ++e) {
      const int x = B::cl_pos(tid, e);
      const uint64_t c = a1[galois_src((uint32_t)(boff + x), ev.galois, tb.log_n)];
      d2[off + x] = c;
      v[e] = u2d(c);
    }
  } else {
    const uint64_t* b1 = ev.b + (((size_t)tl.item * 2 + 1) * ell + i) * N;
#pragma unroll
    for (int e = 0; e < B::E; ++e) {
      const int x = B::cl_pos(tid, e);
      const uint64_t c = f_canon(f_mul(u2d(a1[boff + x]), u2d(b1[boff + x]), L.qd, L.qinv), L.qd, L.qinv);
      d2[off + x] = c;
      v[e] = u2d(c);
    }
  }
  B::inv(arf(tb, L, i, true), v, reinterpret_cast<double*>(lds), tid, (uint32_t)(R + blk));
#pragma unroll
  for (int e = 0; e < B::E; ++e) t1[off + B::fr_pos(tid, e)] = d2raw(v[e]);
}

// The HMUL or HROT part of a thread's outputs of one block of limb i, added to
// ModDown's (o0, o1) before their final reduction: (a0 b0, a0 b1 + a1 b0) or
// (sigma_g(c0), 0). r0 / r1 are the words of component 0 / 1 where the item's
// block of limb i starts, boff the block's first slot in the limb. All operand
// words are loaded before the first use.
template <class B>
__device__ __forceinline__ void add_eval(const LimbC& L, EvalIn ev, size_t r0, size_t r1, uint32_t boff,
                                         int tid, int log_n, double (&o0)[B::E], double (&o1)[B::E]) {
  if (ev.galois) {
    const uint64_t* c0 = ev.a + r0 - boff;
    uint64_t w[B::E];
#pragma unroll
    for (int e = 0; e < B::E; ++e) w[e] = c0[galois_src(boff + (uint32_t)B::cl_pos(tid, e), ev.galois, log_n)];
#pragma unroll
    for (int e = 0; e < B::E; ++e) o0[e] += u2d(w[e]);
    return;
  }
  uint64_t a0[B::E], a1[B::E], b0[B::E], b1[B::E];
  load_words<B>(ev.a + r0, true, tid, a0);
  load_words<B>(ev.b + r0, true, tid, b0);
  load_words<B>(ev.b + r1, true, tid, b1);
  load_words<B>(ev.a + r1, true, tid, a1);
  // both branches end with o0: stores of different arrays at the end of the two
  // would be merged into one through a selected address, which needs scratch memory
#pragma unroll
  for (int e = 0; e < B::E; ++e)
    o1[e] += f_mul(u2d(a0[e]), u2d(b1[e]), L.qd, L.qinv) + f_mul(u2d(a1[e]), u2d(b0[e]), L.qd, L.qinv);
#pragma unroll
  for (int e = 0; e < B::E; ++e) o0[e] += f_mul(u2d(a0[e]), u2d(b0[e]), L.qd, L.qinv);
}

// ------------------------------------------------------------ ModUp (K2)

// A column-pass workgroup: 8 waves over the same 64 columns (the 64 lanes).
// Sources are converted once into LDS (wave w takes sources w, w+8, ...);
// after a barrier the waves split the target limbs the same way, so the
// registers a thread needs do not grow with the number of sources.
constexpr int CW = 8;               // waves per column workgroup
constexpr int CT = CW * TC;         // threads per column workgroup

// Digit j = j0 + blockIdx.y of item blockIdx.z, columns blockIdx.x*64 + lane:
// inverse column pass of the digit's limbs of t1 (the block-pass output of d,
// raw), times N^-1 [(D_j/q_i)^-1]_{q_i}, giving canonical y_i (in LDS,
// [alpha][R][64] doubles); then for every target limb t in [tgt0, tgt1)
// outside D_j: z_t = sum_i y_i [D_j/q_i]_t, forward column pass, store into
// ext1 [items][nslots][nl][N] at slot (slot_stride ? j : 0). Q targets are
// stored raw, P targets below 2^64.
template <int LOGR>
__global__ __launch_bounds__(CT, LOGR <= 4 ? 4 : 2) void k_modup_cols(DevTables tb, const uint64_t* t1, uint64_t* ext1, int j0,
                                                   int nslots, int slot_stride, int tgt0, int tgt1, int log_m) {
  constexpr int R = 1 << LOGR;
  extern __shared__ double ys[];
  const int M = 1 << log_m;
  const size_t N = (size_t)M * R;
  const int lane = threadIdx.x & (TC - 1), wv = threadIdx.x / TC;
  const size_t c = (size_t)blockIdx.x * TC + lane;
  const bool live = c < (size_t)M;
  const int j = j0 + blockIdx.y;
  const int item = blockIdx.z;
  const int ell = tb.ell, nl = tb.nl;
  const int lo = j * tb.alpha;
  const int na = min(lo + tb.alpha, ell) - lo;
  if (live) {
    for (int s = wv; s < na; s += CW) {
      const int i = lo + s;
      const LimbC L = tb.limb[i];
      const uint64_t* a = t1 + ((size_t)item * ell + i) * N;
      double v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = raw2d(a[c + (size_t)r * M]);
      sub_inv<LOGR>(arf(tb, L, i, true), v, 1u);
      const double w = tb.up_pre_d[i];
#pragma unroll
      for (int r = 0; r < R; ++r) ys[(s * R + r) * TC + lane] = f_canon_d(f_mul(v[r], w, L.qd, L.qinv), L.qd, L.qinv);
    }
  }
  __syncthreads();
  if (!live) return;
  const int slot = slot_stride ? j : 0;
  uint64_t* e = ext1 + ((size_t)item * nslots + slot) * (size_t)nl * N;
  int u = 0;  // index of the target among those outside D_j
  for (int t = tgt0; t < tgt1; ++t) {
    if (t >= lo && t < lo + na) continue;
    if ((u++ % CW) != wv) continue;
    const LimbC L = tb.limb[t];
    uint64_t* o = e + (size_t)t * N;
    if (t < ell) {
      // |y * c| <= 2^50 * 2^49: each product is within 0.69q; fold every 8
      double z[R];
#pragma unroll
      for (int r = 0; r < R; ++r) z[r] = 0.0;
      for (int s = 0; s < na; ++s) {
        const double cst = ldc(tb.up_mat_d + (size_t)(lo + s) * ell + t);
#pragma unroll
        for (int r = 0; r < R; ++r) z[r] += f_mul(ys[(s * R + r) * TC + lane], cst, L.qd, L.qinv);
        if ((s & 7) == 7) {
#pragma unroll
          for (int r = 0; r < R; ++r) z[r] = f_red(z[r], L.qd, L.qinv);
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) z[r] = f_red(z[r], L.qd, L.qinv);
      sub_fwd<LOGR, -1, false>(arf(tb, L, t, false), z, 1u);
#pragma unroll
      for (int r = 0; r < R; ++r) o[c + (size_t)r * M] = d2raw(z[r]);
    } else {
      uint64_t z[R];
#pragma unroll
      for (int r = 0; r < R; ++r) z[r] = 0;
      for (int s = 0; s < na; ++s) {
        const size_t ci = 2 * ((size_t)(lo + s) * nl + t);
        const uint64_t w = ldc(tb.up_mat + ci), ws = ldc(tb.up_mat + ci + 1);
#pragma unroll
        for (int r = 0; r < R; ++r) z[r] += mul_shoup_lazy(d2u(ys[(s * R + r) * TC + lane]), w, ws, L.nq);
        if (s % 3 == 2) {  // keep the sum below 2^60 + 2^33 + 3 * 4q
#pragma unroll
          for (int r = 0; r < R; ++r) z[r] = p_red(z[r], L.delta);
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) z[r] = p_red(z[r], L.delta);
      sub_fwd<LOGR, -1, false>(ari(tb, L, t, false), z, 1u);
#pragma unroll
      for (int r = 0; r < R; ++r) o[c + (size_t)r * M] = z[r];
    }
  }
}

// ------------------------------------------- int8-MFMA base conversion

// BConv as an exact integer contraction on the matrix cores. Each residue
// y < 2^60 is written in balanced base-256 digits y = sum_a d_a 256^a
// (d_a in [-128, 127], signed bytes), and each constant c_{s,t} is folded
// with the digit weight, c'_{s,a,t} = [c_{s,t} 256^a]_t, and split the same
// way into bytes e_{s,a,t,b}. Then
//   sum_s y_s c_{s,t} = sum_b 256^b C_b  (mod t),  C_b = sum_{s,a} d_{s,a} e_{s,a,t,b},
// and every C_b is one entry of an int8 x int8 -> int32 matrix product with
// K = 8 * (number of sources): rows (t, b) come from the constant table,
// columns are coefficients. |C_b| <= 8 * 32 * 128 * 128 = 2^22 for up to 32
// sources. A 32-row tile covers four targets; the host's row order puts all
// eight C_b of targets 2h and 2h+1 in the accumulators of lane half h
// (accumulator i = byte i % 8 of target 2h + i / 8).
// MFMA v_mfma_i32_32x32x32_i8: lane l supplies 16 bytes of row (or column)
// l % 32 at K offsets 16 * (l / 32) .. +15, i.e. sources 4m + 2(l/32) + {0, 1}
// of step m, eight digit bytes each.
typedef int mx_v4i __attribute__((ext_vector_type(4)));
typedef int mx_v16i __attribute__((ext_vector_type(16)));

// mx_pack of a canonical Q residue held as a double (v < 2^50): bytes 0..5
// balanced, byte 6 = the rest, in [0, 4]. The 128 of each byte is added together
// with the 2^52 that moves the integer into the mantissa (exact: the sum stays
// below 2^52 + 2^51), and one exclusive or removes both.
__device__ __forceinline__ uint64_t mx_pack_q(double v) {
  return (uint64_t)__double_as_longlong(v + (4503599627370496.0 + 141289400074368.0)) ^ 0x4330808080808080ull;
}

// Signed bytes of the balanced digits of v < 2^60 (byte 7 is below 18):
// adding 128 to each of the seven low bytes makes them the unsigned bytes of
// v + 0x0080...80; flipping their top bit subtracts the 128 again modulo 256.
__device__ __forceinline__ uint64_t mx_pack(uint64_t v) {
  return (v + 0x0080808080808080ull) ^ 0x0080808080808080ull;
}

__device__ __forceinline__ mx_v16i mx_step(const ulonglong2& a, const ulonglong2& b, const mx_v16i& acc) {
  const mx_v4i av = {(int)(uint32_t)a.x, (int)(uint32_t)(a.x >> 32), (int)(uint32_t)a.y, (int)(uint32_t)(a.y >> 32)};
  const mx_v4i bv = {(int)(uint32_t)b.x, (int)(uint32_t)(b.x >> 32), (int)(uint32_t)b.y, (int)(uint32_t)(b.y >> 32)};
  return __builtin_amdgcn_mfma_i32_32x32x32_i8(av, bv, acc, 0, 0, 0);
}

// The target whose partial sums start at accumulator BASE (0 or 8), as
// lo = C0 + 2^8 C1 + 2^16 C2 + 2^24 C3 and hi = C4 + ... + 2^24 C7, exact
// doubles (each pair C + 2^8 C' below 2^30.1) below 2^46.1 in magnitude (the sum is
// lo + 2^32 hi). QG: a Q target, whose constants are below 2^50, so that C7 is 0.
template <int BASE, bool QG>
__device__ __forceinline__ void mx_halves(const mx_v16i& acc, double& lo, double& hi) {
  const int a0 = acc[BASE + 0] + acc[BASE + 1] * 256, a1 = acc[BASE + 2] + acc[BASE + 3] * 256;
  const int b0 = acc[BASE + 4] + acc[BASE + 5] * 256, b1 = QG ? acc[BASE + 6] : acc[BASE + 6] + acc[BASE + 7] * 256;
  lo = __fma_rn((double)a1, 65536.0, (double)a0);
  hi = __fma_rn((double)b1, 65536.0, (double)b0);
}

// lo + 2^32 hi mod q for a Q prime, |result| <= 0.6q: k = rint(2^32 hi / q) (below
// 2^30), and hi - k (q / 2^32) is a multiple of 2^-32 within (q/2 + 1) / 2^32, so
// exact; |lo| < 2^46.1 < 0.07q. 4 instructions (a product with 2^32 mod q took 7;
// (8, 2^17, 56), batch 2, 1126 us with it, 1108 without).
__device__ __forceinline__ double mx_fold_q(double lo, double hi, double q32, double qinv32) {
  return __fma_rn(__fma_rn(-__builtin_rint(hi * qinv32), q32, hi), 4294967296.0, lo);
}

// lo + 2^32 hi mod p for a P prime, below 2.1 * 2^60: with u = x + 2^51 >= 0 in the
// mantissa of x + 1.5 * 2^52, the value is u_lo + 2^32 u_hi - 2^51 - 2^83, and the bits
// of u_hi from 28 up fold at 2^60. The exponent bits stay in both words (0x433 in
// the top 12 bits of u_lo's, 0x33 in the top 8 of the 32 bits taken from u_hi's): cadj
// takes them out with the constant.
__device__ __forceinline__ uint64_t mx_fold_p(double lo, double hi, const LimbC& L) {
  const uint64_t ul = (uint64_t)__double_as_longlong(lo + 6755399441055744.0);
  const uint64_t uh = (uint64_t)__double_as_longlong(hi + 6755399441055744.0);
  const uint32_t top = __builtin_amdgcn_alignbit((uint32_t)(uh >> 32), (uint32_t)uh, 28);
  return ul + (uint64_t)top * (uint32_t)L.delta + ((uint64_t)((uint32_t)uh & 0x0FFFFFFFu) << 32) + L.cadj;
}

// Columns of a workgroup: 64 (two column halves of 32, one per wave parity), or
// 32 where the packed digits of 64 columns (2 KB nm R) would leave room for only
// one workgroup of 8 waves on a CU. With 32 rows the registers do that anyway (built
// for two workgroups they spill: ModUp of (4, 2^16, 32), batch 8, 229 -> 298 us), and
// it is 64 columns as long as they fit.
constexpr int mx_cols(int logr, int nm) { return (nm << logr) <= (logr == 5 ? 64 : 40) ? 64 : 32; }
// From 16 rows on, the first R twiddles of a group's four targets go through the
// wave's own part of the LDS: one or two loads a lane, in flight with the constants
// and stored when the rows are done. Read where each stage uses them, from two
// addresses a wave, they took the registers that the rows need and a latency a
// stage (ModUp of (4, 2^16, 32), batch 8, 181 -> 168 us; 4 of its registers still spill, 10
// with 3 steps and 12 with 4); with 8 rows (7 twiddles) the detour costs 2% of
// (2, 2^15, 10), batch 32.
constexpr bool mx_twl(int logr) { return logr >= 4; }
constexpr int mx_nt(int logr) { return mx_twl(logr) ? (4 << logr) / 64 : 1; }
// LDS: the packed digits, and that part for each wave (16 bytes each, for P targets).
constexpr int mx_lds(int logr, int nm) {
  return (nm << logr) * mx_cols(logr, nm) * 32 + (mx_twl(logr) ? CW * 4 * (16 << logr) : 0);
}

// The other half of the lanes' registers: a keeps its lower 32 lanes and takes b's
// lower into its upper ones, b keeps its upper and takes a's upper into its lower.
__device__ __forceinline__ void swap32(uint64_t& a, uint64_t& b) {
  typedef unsigned v2 __attribute__((ext_vector_type(2)));
  const v2 lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
  const v2 hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
  a = ((uint64_t)hi.x << 32) | lo.x;
  b = ((uint64_t)hi.y << 32) | lo.y;
}
__device__ __forceinline__ void swap32(double& a, double& b) {
  uint64_t x = d2raw(a), y = d2raw(b);
  swap32(x, y);
  a = raw2d(x);
  b = raw2d(y);
}

// Inverse column pass of one source by one wave. With 64 columns a lane holds the R
// rows of its column. With 32 lane half h loads rows h R/2 .. (v[i] is row i + h R/2),
// and after the stages within a half the halves exchange R/4 registers, so that the
// last stage's pairs (row r, row r + R/2) meet in one lane: v[i] is then row
// i + h R/4 and v[i + R/4] row R/2 + i + h R/4, i < R/4 (mx_row).
template <int LOGR, int C>
constexpr int mx_rows() { return C == 64 ? 1 << LOGR : (1 << LOGR) / 2; }
template <int LOGR, int C>
__device__ __forceinline__ int mx_row(int i, int h) {
  constexpr int R = 1 << LOGR;
  return C == 64 ? i : (i < R / 4 ? i + h * (R / 4) : R / 2 + (i - R / 4) + h * (R / 4));
}
template <int LOGR, int C, class Ar>
__device__ __forceinline__ void mx_inv(const Ar& A, typename Ar::T (&v)[mx_rows<LOGR, C>()], int h) {
  if constexpr (C == 64) {
    sub_inv<LOGR>(A, v, 1u);
  } else {
    constexpr int Q = (1 << LOGR) / 4;
    sub_inv<LOGR - 1>(A, v, 2u + (uint32_t)h);
    const typename Ar::TwT w = A.template twiddle<false>(1u);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      swap32(v[i], v[i + Q]);
      A.template inv<true>(v[i], v[i + Q], w);
    }
  }
}

// Phase 2 of the MFMA column kernels for one target group. A lane in half h
// holds the partial sums of targets 2h and 2h + 1 of the group; each is
// finished in its own pass (PASS 0: accumulators 0..7, PASS 1: 8..15), which
// runs the nm MFMA steps of every row r over the packed digits yp
// ([pairs][R][columns] x 16 bytes) again, so that only one target's R values are
// live: for each row the fold mod t, then the forward column pass and, if
// `st`, the store of the R rows. Up to 8 rows both targets' values fit and PASS 2
// finishes both from one run of the MFMA steps. Q groups store raw words, P groups
// values below 2^64. The raised digits (and ModDown's t2) outgrow the caches,
// so the stores are non-temporal (measured: 5% off the ModUp column kernel).
template <bool QG>
using mx_val = typename std::conditional<QG, double, uint64_t>::type;
// (w, Shoup) as a vector type: an array of HIP's ulonglong2 structs with more than one entry
// stays in scratch memory (48 bytes a lane at 32 rows; the times are within noise:
// (8, 2^17, 56), batch 2, 1049 -> 1046 us).
typedef uint64_t mx_v2u __attribute__((ext_vector_type(2)));
template <bool QG>
using mx_tw = typename std::conditional<QG, double, mx_v2u>::type;

// CONV: the conversion alone (ks_bconv): no transform, canonical words.
template <int LOGR, bool QG, bool CONV>
__device__ __forceinline__ void mx_finish(const LimbC& L, const mx_tw<QG>* tw, mx_val<QG> (&z)[1 << LOGR], bool st,
                                          uint64_t* o, size_t cc, int M) {
  constexpr int R = 1 << LOGR;
  if constexpr (CONV) {
    if (st) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if constexpr (QG)
          o[cc + (size_t)r * M] = f_canon(z[r], L.qd, L.qinv);
        else
          o[cc + (size_t)r * M] = p_canon(z[r], L.q, (uint32_t)L.delta);
      }
    }
    return;
  }
  if constexpr (QG)
    sub_fwd<LOGR, -1, false>(ArF{L.qd, L.qinv, tw, tw}, z, 1u);
  else
    sub_fwd<LOGR, -1, false>(ArI{L.q, L.nq, (uint32_t)L.delta, reinterpret_cast<const uint64_t*>(tw)}, z, 1u);
  if (st) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      uint64_t w;
      if constexpr (QG)
        w = d2raw(z[r]);
      else
        w = z[r];
      __builtin_nontemporal_store(w, o + cc + (size_t)r * M);
    }
  }
}

template <int LOGR, bool QG, int NM, int PASS, bool CONV>
__device__ __forceinline__ void mx_target(const DevTables& tb, const ulonglong2* yp, mx_tw<QG>* tw,
                                          const mx_tw<QG> (&wl)[mx_nt(LOGR)], const ulonglong2 (&cst)[NM], int ta0, int ta1, int tb0, int tb1, bool sa, bool sb, uint64_t* oa,
                                          uint64_t* ob, size_t cc, int M) {
  constexpr int R = 1 << LOGR, C = mx_cols(LOGR, NM);
  const int lane = threadIdx.x & (TC - 1), h = lane >> 5;
  const int ycol = (C == 64 ? ((threadIdx.x / TC) & 1) * 32 : 0) + (lane & 31);
  const int ta = h ? ta1 : ta0, tc = h ? tb1 : tb0;
  const LimbC& LA = tb.limb[ta];
  const LimbC& LB = tb.limb[tc];
  using T = mx_val<QG>;
  T za[R], zb[R];
  const double qa = LA.q32, qia = LA.qinv32, qb = LB.q32, qib = LB.qinv32;
  int yo = h * R * C + ycol;  // digit words of row r of step m: yp[yo + (2 m R + r) C]
#pragma unroll
  for (int r = 0; r < R; ++r) {
    mx_v16i acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int m = 0; m < NM; ++m) acc = mx_step(cst[m], yp[yo + (2 * m * R + r) * C], acc);
    double lo, hi;
    if constexpr (PASS != 1) {
      mx_halves<0, QG>(acc, lo, hi);
      if constexpr (QG)
        za[r] = mx_fold_q(lo, hi, qa, qia);
      else
        za[r] = mx_fold_p(lo, hi, LA);
    }
    if constexpr (PASS != 0) {
      mx_halves<8, QG>(acc, lo, hi);
      if constexpr (QG)
        zb[r] = mx_fold_q(lo, hi, qb, qib);
      else
        zb[r] = mx_fold_p(lo, hi, LB);
    }
    // One row at a time: this row's result is materialised here (the compiler
    // would otherwise sink the folds below the loop and keep every row's
    // accumulators live), and the next row's digit loads wait for it.
    if constexpr (PASS == 0)
      asm volatile("" : "+v"(za[r]), "+v"(yo));
    else if constexpr (PASS == 1)
      asm volatile("" : "+v"(zb[r]), "+v"(yo));
    else
      asm volatile("" : "+v"(za[r]), "+v"(zb[r]), "+v"(yo));
  }
  const mx_tw<QG>*wa, *wb;
  if constexpr (mx_twl(LOGR)) {
    if constexpr (!CONV && PASS != 1) {
      // the words hold the twiddles of the wave's group before, of another type if that
      // was the last Q group: its reads come first
      wave_sync();
#pragma unroll
      for (int n = 0; n < mx_nt(LOGR); ++n) tw[lane + 64 * n] = wl[n];
      wave_sync();
    }
    wa = tw + (size_t)(2 * h) * R;
    wb = tw + (size_t)(2 * h + 1) * R;
  } else {
    const mx_tw<QG>* tab;
    if constexpr (QG)
      tab = tb.twf_d;
    else
      tab = reinterpret_cast<const mx_v2u*>(tb.twf);
    wa = tab + ((size_t)ta << tb.log_n);
    wb = tab + ((size_t)tc << tb.log_n);
  }
  if constexpr (PASS != 1) mx_finish<LOGR, QG, CONV>(LA, wa, za, sa, oa, cc, M);
  if constexpr (PASS != 0) mx_finish<LOGR, QG, CONV>(LB, wb, zb, sb, ob, cc, M);
}

// lt[4]: the group's four limbs (padding slots replaced by a stand-in limb,
// wave-uniform); lane half h finishes targets lt[2h] (stored if sa, at oa)
// and lt[2h + 1] (if sb, at ob).
template <int LOGR, bool QG, int NM, bool CONV = false, int C = mx_cols(LOGR, NM)>
__device__ __forceinline__ void mx_group(const DevTables& tb, const ulonglong2* yp, const ulonglong2* cst_g,
                                         const int (&lt)[4], bool sa, bool sb, uint64_t* oa, uint64_t* ob,
                                         size_t cc, int M) {
  const int lane = threadIdx.x & (TC - 1);
  constexpr int R = 1 << LOGR;
  using TW = mx_tw<QG>;
  TW* tw = reinterpret_cast<TW*>(const_cast<ulonglong2*>(yp) + NM * R * C * 2) +
           (size_t)(threadIdx.x / TC) * (4 * R) * (QG ? 2 : 1);
  TW wl[mx_nt(LOGR)];
  if constexpr (!CONV && mx_twl(LOGR)) {
    const int l0 = lt[0], l1 = lt[1], l2 = lt[2], l3 = lt[3];
#pragma unroll
    for (int n = 0; n < mx_nt(LOGR); ++n) {
      const int e = lane + 64 * n, slot = e >> LOGR;
      const int t = slot == 0 ? l0 : slot == 1 ? l1 : slot == 2 ? l2 : l3;
      const size_t x = ((size_t)t << tb.log_n) + (size_t)(e & (R - 1));
      if constexpr (QG)
        wl[n] = tb.twf_d[x];
      else
        wl[n] = reinterpret_cast<const mx_v2u*>(tb.twf)[x];
    }
  }
  ulonglong2 cst[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) cst[m] = cst_g[m * 64 + lane];
  if constexpr (LOGR <= 3) {
    mx_target<LOGR, QG, NM, 2, CONV>(tb, yp, tw, wl, cst, lt[0], lt[2], lt[1], lt[3], sa, sb, oa, ob, cc, M);
  } else {
    mx_target<LOGR, QG, NM, 0, CONV>(tb, yp, tw, wl, cst, lt[0], lt[2], lt[1], lt[3], sa, sb, oa, ob, cc, M);
    mx_target<LOGR, QG, NM, 1, CONV>(tb, yp, tw, wl, cst, lt[0], lt[2], lt[1], lt[3], sa, sb, oa, ob, cc, M);
  }
}

// Waves per SIMD the MFMA column kernels are built for: 4 where the LDS holds two
// workgroups and a lane's rows fit 128 registers.
constexpr int mx_waves(int logr, int nm) { return logr <= 4 && mx_lds(logr, nm) <= 80 * 1024 ? 4 : 2; }

// ModUp columns with the int8-MFMA BConv: same arguments and output as
// k_modup_cols. Phase 1: inverse column pass and pre-scale as in k_modup_cols,
// canonical y packed into LDS as [pair][R][columns] x 16 bytes (pair p = sources
// 2p, 2p + 1; zero past the digit's sources and for columns past M); a wave takes
// one source at a time (mx_inv).
// Phase 2: with 64 columns wave w takes the column half w % 2 (lane l works on
// column (w % 2) * 32 + l % 32 of the workgroup) and the target groups w/2,
// w/2 + 4, ...; with 32 the groups w, w + 8, ...: per digit the Q targets outside
// D_j in groups of four (in basis order), then the P targets. With `parts` > 1 that
// many workgroups share a tile's groups, each with its own phase 1 (mx_parts).
template <int LOGR, int NM, bool ONCE>
__global__ __launch_bounds__(CT, mx_waves(LOGR, NM)) void k_modup_cols_mx(DevTables tb, const uint64_t* t1, uint64_t* ext1, int j0,
                                                     int nslots, int slot_stride, int tgt0, int tgt1, int log_m,
                                                     int parts) {
  constexpr int R = 1 << LOGR, C = mx_cols(LOGR, NM), RL = mx_rows<LOGR, C>();  // RL: rows of a lane in phase 1
  extern __shared__ ulonglong2 yp[];
  const int M = 1 << log_m;
  const size_t N = (size_t)M * R;
  const int lane = threadIdx.x & (TC - 1), wv = threadIdx.x / TC;
  const int col = lane & (C - 1);
  const int tile = blockIdx.x / parts, part = blockIdx.x % parts;
  const size_t c = (size_t)tile * C + col;
  const bool live = c < (size_t)M;
  const int j = j0 + blockIdx.y;
  const int item = blockIdx.z;
  const int ell = tb.ell, nl = tb.nl, k = tb.k;
  const int lo = j * tb.alpha;
  const int na = min(lo + tb.alpha, ell) - lo;
  constexpr int nm = NM;  // = tb.up_nm
  uint64_t* yw = reinterpret_cast<uint64_t*>(yp);
  const int ph = C == 64 ? 0 : lane >> 5;  // row half of phase 1
  for (int s = wv; s < 4 * nm; s += CW) {
    uint64_t* yr = yw + (size_t)(s >> 1) * R * C * 2 + 2 * col + (s & 1);  // row r at yr[2 r C]
    if (s < na && (C == 32 || live)) {  // with 32 columns uniform: those past M read the last one's words
      const int i = lo + s;
      const LimbC L = tb.limb[i];
      const uint64_t* a = t1 + ((size_t)item * ell + i) * N + (C == 64 || live ? c : M - 1) + (size_t)(ph * RL) * M;
      double v[RL];
#pragma unroll
      for (int r = 0; r < RL; ++r) v[r] = raw2d(ld_col<ONCE>(a + (size_t)r * M));
      mx_inv<LOGR, C>(arf(tb, L, i, true), v, ph);
      const double w = tb.up_pre_d[i];
#pragma unroll
      for (int r = 0; r < RL; ++r)
        yr[2 * C * mx_row<LOGR, C>(r, ph)] =
            C == 64 || live ? mx_pack_q(f_canon_d(f_mul(v[r], w, L.qd, L.qinv), L.qd, L.qinv)) : 0;
    } else {
#pragma unroll
      for (int r = 0; r < RL; ++r) yr[2 * C * mx_row<LOGR, C>(r, ph)] = 0;
    }
  }
  __syncthreads();
  const int h = lane >> 5;
  const size_t cc = (size_t)tile * C + (C == 64 ? (wv & 1) * 32 : 0) + (lane & 31);
  const bool clive = cc < (size_t)M;
  const int slot = slot_stride ? j : 0;
  uint64_t* e = ext1 + ((size_t)item * nslots + slot) * (size_t)nl * N;
  const int nq = ell - na, nqg = (nq + 3) >> 2, ng = nqg + ((k + 3) >> 2);
  const ulonglong2* cst_j = reinterpret_cast<const ulonglong2*>(tb.up_mx) + (size_t)j * tb.up_ng * nm * 64;
  for (int g = (wv / (C / 32)) * parts + part; g < ng; g += (CW / (C / 32)) * parts) {
    const bool qg = g < nqg;
    int tg[4];
    bool any = false;
#pragma unroll
    for (int tau = 0; tau < 4; ++tau) {
      int t = -1;
      if (qg) {
        const int u = 4 * g + tau;
        if (u < nq) t = u < lo ? u : u + na;
      } else {
        const int v = 4 * (g - nqg) + tau;
        if (v < k) t = ell + v;
      }
      tg[tau] = t;
      any = any || (t >= tgt0 && t < tgt1);
    }
    if (!any) continue;
    const int ta = tg[2 * h], tb2 = tg[2 * h + 1];
    const bool sa = clive && ta >= tgt0 && ta < tgt1;
    const bool sb = clive && tb2 >= tgt0 && tb2 < tgt1;
    const int pad = qg ? 0 : ell;  // stand-in limb for padding slots (never stored)
    int lt[4];
#pragma unroll
    for (int tau = 0; tau < 4; ++tau) lt[tau] = tg[tau] >= 0 ? tg[tau] : pad;
    uint64_t* oa = e + (size_t)lt[2 * h] * N;
    uint64_t* ob = e + (size_t)lt[2 * h + 1] * N;
    if (qg)
      mx_group<LOGR, true, NM>(tb, yp, cst_j + (size_t)g * nm * 64, lt, sa, sb, oa, ob, cc, M);
    else
      mx_group<LOGR, false, NM>(tb, yp, cst_j + (size_t)g * nm * 64, lt, sa, sb, oa, ob, cc, M);
  }
}

// ---------------------------------------------------------- KeyMult (K3)

// One block b of one target limb t in [tgt0, tgt0 + ntgt) of one item per
// workgroup (placed by xcd_tile): for every
// digit j in [j0, j1): ext_j = (t in D_j) ? d : forward block pass of ext1;
// s_c += ext_j * evk[j][c]. Then v_c = s_c (+ the previous acc if
// `accumulate`), stored canonical. With `finalize` and t a P limb, the inverse
// block pass of ModDown runs on v_c and leaves [0, 4q] in acc.
// QPATH selects the Q-limb (FP64) or the P-limb (integer) body; the two are
// separate kernels so that each gets its own register allocation.
// With 8 elements per thread at M >= 2^12 the kernel fits 128 registers,
// which lets four waves share each SIMD.
template <int LOGM, int LOGE, bool QPATH>
__global__ __launch_bounds__((1 << (LOGM - LOGE)), (LOGE == 3 && LOGM >= 12) ? 4 : 1) void k_keymult_blocks(
    DevTables tb, const uint64_t* d, const uint64_t* ext1, const uint64_t* evk, uint64_t* acc, int j0, int j1,
    int nslots, int slot_stride, int tgt0, int ntgt, int items, int accumulate, int finalize) {
  using B = BlockNtt<LOGM, LOGE>;
  extern __shared__ uint64_t lds[];
  const size_t N = (size_t)1 << tb.log_n;
  const int R = (int)(N >> LOGM);
  const Tile tl = xcd_tile(R * ntgt, items);
  if (!tl.valid) return;
  const int tid = threadIdx.x, b = tl.tile % R;
  const int t = tgt0 + tl.tile / R;
  const int item = tl.item;
  const LimbC L = tb.limb[t];
  const uint32_t B0 = (uint32_t)R + b;
  const int nl = tb.nl;
  const size_t boff = (size_t)b * B::M;
  uint64_t* a0 = acc + (((size_t)item * 2 + 0) * nl + t) * N + boff;
  uint64_t* a1 = acc + (((size_t)item * 2 + 1) * nl + t) * N + boff;
  // At blocks of 2^14 the 16 elements of both sums and of the transform fill the 128 registers of
  // 1024 threads: the next input (P limbs) and a round's twiddles loaded ahead of use went to
  // scratch memory (296 bytes a lane, now 96; (2, 2^17, 44), one ciphertext, 180 us, now 153).
  constexpr bool AHEAD = LOGM <= 13;
  if constexpr (QPATH) {
    const ArF A = arf(tb, L, t, false);
    double* ld = reinterpret_cast<double*>(lds);
    constexpr int FOLD = LOGE >= 4 ? 3 : 4;
    double s0[B::E], s1[B::E], v[B::E];
#pragma unroll
    for (int i = 0; i < B::E; ++i) s0[i] = s1[i] = 0.0;
    for (int j = j0; j < j1; ++j) {
      const int lo = j * tb.alpha;
      if (t >= lo && t < lo + tb.alpha) {
        const uint64_t* src = d + ((size_t)item * tb.ell + t) * N + boff;
#pragma unroll
        for (int i = 0; i < B::E; ++i) v[i] = u2d(src[B::cl_pos(tid, i)]);
      } else {
        const int slot = slot_stride ? j : 0;
        const uint64_t* src = ext1 + (((size_t)item * nslots + slot) * nl + t) * N + boff;
#pragma unroll
        for (int i = 0; i < B::E; ++i) v[i] = raw2d(src[B::fr_pos(tid, i)]);
        fwd_opaque<B, false, true, AHEAD>(A, v, ld, tid, B0);
      }
      const uint64_t* k0 = evk + key_row(tb, j, 0, t) * N + boff;
      const uint64_t* k1 = evk + key_row(tb, j, 1, t) * N + boff;
      // |v| <= 3.6q (5.2q for E = 16), key < q: each product is within 1.85q
      // (2.45q), so the sums stay below 8q when folded every FOLD digits
#pragma unroll
      for (int i = 0; i < B::E; ++i) {
        const int x = B::cl_pos(tid, i);
        s0[i] += f_mul(v[i], u2d(k0[x]), L.qd, L.qinv);
        s1[i] += f_mul(v[i], u2d(k1[x]), L.qd, L.qinv);
      }
      if ((j - j0) % FOLD == FOLD - 1) {
#pragma unroll
        for (int i = 0; i < B::E; ++i) {
          s0[i] = f_red(s0[i], L.qd, L.qinv);
          s1[i] = f_red(s1[i], L.qd, L.qinv);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < B::E; ++i) {
      const int x = B::cl_pos(tid, i);
      double u0 = f_red(s0[i], L.qd, L.qinv), u1 = f_red(s1[i], L.qd, L.qinv);
      if (accumulate) {
        u0 += u2d(a0[x]);
        u1 += u2d(a1[x]);
      }
      a0[x] = f_canon(u0, L.qd, L.qinv);
      a1[x] = f_canon(u1, L.qd, L.qinv);
    }
  } else {
  const ArI A = ari(tb, L, t, false);
  const uint32_t delta = (uint32_t)L.delta;
  uint64_t s0[B::E], s1[B::E], v[B::E];
#pragma unroll
  for (int i = 0; i < B::E; ++i) s0[i] = s1[i] = 0;
  // the next digit's input is loaded before a digit's transform (with K3 waiting for
  // it after the products, (4, 2^16, 32), batch 8, was 828 us, now 809); the key
  // blocks, L2 hits for all but one item, after it: one of them ahead as well
  // takes the registers past 128
  auto load_digit = [&](int j, uint64_t (&w)[B::E]) {
    load_words<B>(ext1 + (((size_t)item * nslots + (slot_stride ? j : 0)) * nl + t) * N + boff, false, tid, w);
  };
  uint64_t nxt[AHEAD ? B::E : 1];
  if constexpr (AHEAD) {
    if (j0 < j1) load_digit(j0, nxt);
  }
  for (int j = j0; j < j1; ++j) {
    uint64_t w0[B::E], w1[B::E];
    if constexpr (AHEAD) {
#pragma unroll
      for (int i = 0; i < B::E; ++i) v[i] = nxt[i];
      if (j + 1 < j1) load_digit(j + 1, nxt);
    } else {
      load_digit(j, v);
    }
    fwd_opaque<B, false, true, AHEAD>(A, v, lds, tid, B0);
    load_words<B>(evk + key_row(tb, j, 0, t) * N + boff, true, tid, w0);
    load_words<B>(evk + key_row(tb, j, 1, t) * N + boff, true, tid, w1);
    // each product is below 1.5 * 2^60: folded every 8 digits, the sums stay below 2^64
#pragma unroll
    for (int i = 0; i < B::E; ++i) {
      v[i] = p_red(v[i], delta);
      s0[i] += p_mul(v[i], w0[i], delta);
    }
#pragma unroll
    for (int i = 0; i < B::E; ++i) s1[i] += p_mul(v[i], w1[i], delta);
    if (((j - j0) & 7) == 7) {
#pragma unroll
      for (int i = 0; i < B::E; ++i) {
        s0[i] = p_red(s0[i], delta);
        s1[i] = p_red(s1[i], delta);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < B::E; ++i) {
    s0[i] = p_red(s0[i], delta);
    s1[i] = p_red(s1[i], delta);
  }
  if (accumulate) {
#pragma unroll
    for (int i = 0; i < B::E; ++i) {
      const int x = B::cl_pos(tid, i);
      s0[i] += a0[x];
      s1[i] += a1[x];
    }
  }
  if (finalize) {
    const ArI Ai = ari(tb, L, t, true);
    inv_opaque<B, true, AHEAD>(Ai, s0, lds, tid, B0);
#pragma unroll
    for (int i = 0; i < B::E; ++i) a0[B::fr_pos(tid, i)] = s0[i];
    inv_opaque<B, true, AHEAD>(Ai, s1, lds, tid, B0);
#pragma unroll
    for (int i = 0; i < B::E; ++i) a1[B::fr_pos(tid, i)] = s1[i];
  } else {
#pragma unroll
    for (int i = 0; i < B::E; ++i) {
      const int x = B::cl_pos(tid, i);
      a0[x] = p_canon(s0[i], L.q, delta);
      a1[x] = p_canon(s1[i], L.q, delta);
    }
  }
  }
}

// ---------------------------------------------------------- ModDown (K4)

// Component blockIdx.y of item blockIdx.z, columns blockIdx.x*64 + lane:
// inverse column pass of the k P limbs (accp [items][2][nl][N] at limbs ell..,
// values in [0, 4q]), times N^-1 [(P/p_m)^-1]: canonical y_m < 2^60 in LDS
// ([k][R][64] uint64). Then for Q limbs i in [tgt0, tgt1), split over the
// waves: z_i = sum_m y_m [P/p_m]_{q_i}, computed in FP64 as
// y_hi [2^30 P/p_m] + y_lo [P/p_m] with y_m = y_hi 2^30 + y_lo; forward column
// pass; t2 [items][2][ell][N] raw.
template <int LOGR>
__global__ __launch_bounds__(CT, LOGR <= 4 ? 4 : 2) void k_moddown_cols(DevTables tb, const uint64_t* accp, uint64_t* t2, int tgt0,
                                                     int tgt1, int log_m) {
  constexpr int R = 1 << LOGR;
  extern __shared__ uint64_t yl[];
  const int M = 1 << log_m;
  const size_t N = (size_t)M * R;
  const int lane = threadIdx.x & (TC - 1), wv = threadIdx.x / TC;
  const size_t c = (size_t)blockIdx.x * TC + lane;
  const bool live = c < (size_t)M;
  const int comp = blockIdx.y, item = blockIdx.z;
  const int ell = tb.ell, nl = tb.nl, k = tb.k;
  if (live) {
    for (int m = wv; m < k; m += CW) {
      const LimbC L = tb.limb[ell + m];
      const uint64_t* a = accp + (((size_t)item * 2 + comp) * nl + ell + m) * N;
      uint64_t v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = a[c + (size_t)r * M];
      sub_inv<LOGR>(ari(tb, L, ell + m, true), v, 1u);
      const uint64_t w = tb.dn_pre[2 * m], ws = tb.dn_pre[2 * m + 1];
#pragma unroll
      for (int r = 0; r < R; ++r) yl[(m * R + r) * TC + lane] = p_canon(mul_shoup_lazy(v[r], w, ws, L.nq), L.q, L.delta);
    }
  }
  __syncthreads();
  if (!live) return;
  for (int i = tgt0 + wv; i < tgt1; i += CW) {
    const LimbC L = tb.limb[i];
    double z[R];
#pragma unroll
    for (int r = 0; r < R; ++r) z[r] = 0.0;
    for (int m = 0; m < k; ++m) {
      const double ch = tb.dn_mat_d[2 * ((size_t)m * ell + i)];
      const double cl = tb.dn_mat_d[2 * ((size_t)m * ell + i) + 1];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        // |y_hi * c|, |y_lo * c| <= 2^79: each product is within q/2 + 1
        const uint64_t yv = yl[(m * R + r) * TC + lane];
        const double yh = (double)(uint32_t)(yv >> 30);
        const double ylo = (double)(uint32_t)(yv & 0x3FFFFFFFull);
        z[r] += f_mul(yh, ch, L.qd, L.qinv) + f_mul(ylo, cl, L.qd, L.qinv);
      }
      if ((m & 3) == 3) {
#pragma unroll
        for (int r = 0; r < R; ++r) z[r] = f_red(z[r], L.qd, L.qinv);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) z[r] = f_red(z[r], L.qd, L.qinv);
    sub_fwd<LOGR, -1, false>(arf(tb, L, i, false), z, 1u);
    uint64_t* o = t2 + (((size_t)item * 2 + comp) * ell + i) * N;
#pragma unroll
    for (int r = 0; r < R; ++r) o[c + (size_t)r * M] = d2raw(z[r]);
  }
}

// ModDown columns with the int8-MFMA BConv: same arguments and output as
// k_moddown_cols. Phase 1 (the P limbs in the place of k_modup_cols_mx's sources):
// inverse column pass of acc_P and the scale by N^-1 [(P/p_m)^-1]_{p_m} as in
// k_moddown_cols, canonical y packed into LDS ([pair][R][columns] x 16 bytes,
// zero past the k sources and for columns past M). Phase 2: the groups of four Q
// limbs that meet [tgt0, tgt1), shared out as in k_modup_cols_mx; output t2 raw.
template <int LOGR, int NM, bool ONCE>
__global__ __launch_bounds__(CT, mx_waves(LOGR, NM)) void k_moddown_cols_mx(DevTables tb, const uint64_t* accp, uint64_t* t2, int tgt0,
                                                       int tgt1, int log_m, int parts) {
  constexpr int R = 1 << LOGR, C = mx_cols(LOGR, NM), RL = mx_rows<LOGR, C>();
  extern __shared__ ulonglong2 yp[];
  const int M = 1 << log_m;
  const size_t N = (size_t)M * R;
  const int lane = threadIdx.x & (TC - 1), wv = threadIdx.x / TC;
  const int col = lane & (C - 1);
  const int tile = blockIdx.x / parts, part = blockIdx.x % parts;
  const size_t c = (size_t)tile * C + col;
  const bool live = c < (size_t)M;
  const int comp = blockIdx.y, item = blockIdx.z;
  const int ell = tb.ell, nl = tb.nl, k = tb.k;
  constexpr int nm = NM;  // = tb.dn_nm
  uint64_t* yw = reinterpret_cast<uint64_t*>(yp);
  const int ph = C == 64 ? 0 : lane >> 5;
  for (int m = wv; m < 4 * nm; m += CW) {
    uint64_t* yr = yw + (size_t)(m >> 1) * R * C * 2 + 2 * col + (m & 1);
    if (m < k && (C == 32 || live)) {
      const LimbC L = tb.limb[ell + m];
      const uint64_t* a =
          accp + (((size_t)item * 2 + comp) * nl + ell + m) * N + (C == 64 || live ? c : M - 1) + (size_t)(ph * RL) * M;
      uint64_t v[RL];
#pragma unroll
      for (int r = 0; r < RL; ++r) v[r] = ld_col<ONCE>(a + (size_t)r * M);
      mx_inv<LOGR, C>(ari(tb, L, ell + m, true), v, ph);
      const uint64_t w = tb.dn_pre[2 * m], ws = tb.dn_pre[2 * m + 1];
#pragma unroll
      for (int r = 0; r < RL; ++r)
        yr[2 * C * mx_row<LOGR, C>(r, ph)] =
            C == 64 || live ? mx_pack(p_canon(mul_shoup_lazy(v[r], w, ws, L.nq), L.q, L.delta)) : 0;
    } else {
#pragma unroll
      for (int r = 0; r < RL; ++r) yr[2 * C * mx_row<LOGR, C>(r, ph)] = 0;
    }
  }
  __syncthreads();
  const int h = lane >> 5;
  const size_t cc = (size_t)tile * C + (C == 64 ? (wv & 1) * 32 : 0) + (lane & 31);
  const bool clive = cc < (size_t)M;
  uint64_t* o = t2 + ((size_t)item * 2 + comp) * ell * N;
  const ulonglong2* cst = reinterpret_cast<const ulonglong2*>(tb.dn_mx);
  for (int g = (tgt0 >> 2) + (wv / (C / 32)) * parts + part; 4 * g < tgt1; g += (CW / (C / 32)) * parts) {
    const int ta = 4 * g + 2 * h, tb2 = ta + 1;
    const bool sa = clive && ta >= tgt0 && ta < tgt1;
    const bool sb = clive && tb2 >= tgt0 && tb2 < tgt1;
    int lt[4];
#pragma unroll
    for (int tau = 0; tau < 4; ++tau) lt[tau] = 4 * g + tau < ell ? 4 * g + tau : 0;
    mx_group<LOGR, true, NM>(tb, yp, cst + (size_t)g * nm * 64, lt, sa, sb, o + (size_t)lt[2 * h] * N,
                             o + (size_t)lt[2 * h + 1] * N, cc, M);
  }
}

// ---------------------------------------------------------- ModDown (K5)

// One block b of one Q limb i in [tgt0, tgt0 + ntgt) of one (item, component)
// pair ic = item*2 + c per workgroup (placed by xcd_tile):
// forward block pass of t2 (raw), then out = (acc_Q - v) * P^-1 (canonical).
template <int LOGM, int LOGE>
__global__ __launch_bounds__((1 << (LOGM - LOGE))) void k_moddown_blocks(DevTables tb, const uint64_t* t2,
                                                                         const uint64_t* acc, uint64_t* out,
                                                                         int tgt0, int ntgt, int ics,
                                                                         EvalIn ev) {
  using B = BlockNtt<LOGM, LOGE>;
  extern __shared__ uint64_t lds[];
  const size_t N = (size_t)1 << tb.log_n;
  const int R = (int)(N >> LOGM);
  const Tile tl = xcd_tile(R * ntgt, ics);
  if (!tl.valid) return;
  const int tid = threadIdx.x, b = tl.tile % R;
  const int i = tgt0 + tl.tile / R;
  const int ic = tl.item;
  const LimbC L = tb.limb[i];
  const uint32_t B0 = (uint32_t)R + b;
  const size_t boff = (size_t)b * B::M;
  const uint64_t* src = t2 + ((size_t)ic * tb.ell + i) * N + boff;
  double v[B::E];
#pragma unroll
  for (int e = 0; e < B::E; ++e) v[e] = raw2d(ld_once(src + B::fr_pos(tid, e)));
  B::fwd(arf(tb, L, i, false), v, reinterpret_cast<double*>(lds), tid, B0);
  const uint64_t* a = acc + ((size_t)ic * tb.nl + i) * N + boff;
  uint64_t* o = out + ((size_t)ic * tb.ell + i) * N + boff;
  const double pinv = tb.dn_pinv_d[i];
  const int item = ic >> 1, comp = ic & 1;
  const size_t r0 = ((size_t)item * 2 * tb.ell + i) * N + boff, r1 = r0 + (size_t)tb.ell * N;
  // MODE 0: plain KeySwitch, 1: HMUL, 2: HROT (chosen once per workgroup)
  auto finish = [&](auto mode) {
    constexpr int MODE = decltype(mode)::value;
#pragma unroll
    for (int e = 0; e < B::E; ++e) {
      const int x = B::cl_pos(tid, e);
      // |acc - v| <= 6.2q, |P^-1| <= q/2: the product is within 1.67q
      double w = f_mul(u2d(a[x]) - v[e], pinv, L.qd, L.qinv);
      if constexpr (MODE == 2) {  // HROT: sigma_g(c0) in component 0
        if (comp == 0) w += u2d(ev.a[r0 + galois_src((uint32_t)(boff + x), ev.galois, tb.log_n) - boff]);
      } else if constexpr (MODE == 1) {  // HMUL: this component's tensor term, a0 b0 or a0 b1 + a1 b0
        const double a0 = u2d(ev.a[r0 + x]);
        if (comp == 0)
          w += f_mul(a0, u2d(ev.b[r0 + x]), L.qd, L.qinv);
        else
          w += f_mul(a0, u2d(ev.b[r1 + x]), L.qd, L.qinv) + f_mul(u2d(ev.a[r1 + x]), u2d(ev.b[r0 + x]), L.qd, L.qinv);
      }
      o[x] = MODE == 0 ? f_canon(w, L.qd, L.qinv) : f_canon_wide(w, L.qd, L.qinv);
    }
  };
  if (!ev.a)
    finish(std::integral_constant<int, 0>{});
  else if (!ev.galois)
    finish(std::integral_constant<int, 1>{});
  else
    finish(std::integral_constant<int, 2>{});
}

// The twiddles one block pass reads, staged in LDS: entry x in [1, M) is
// table entry ((R + b) << s) + x - 2^s with s = floor(log2 x), the twiddle of
// local stage s and group x - 2^s of block b. Stages s >= PS (the last round
// of the forward pass) are stored group-major: group (p << (s - PS)) + g at
// 2^s + (g << PS) + p. BlockNtt::fwd<true> with this table
// computes what BlockNtt::fwd computes with the global table.
// Thread tid moves entries tid + k T: past the first of them the stage is the
// same for all threads. The loads and the stores are separate steps, so that all
// loads of a thread are in flight together (one at a time, they were 5 us of
// latency at the start of every workgroup).
template <class B, class T>
__device__ __forceinline__ void load_twiddles(T (&w)[B::E], const T* table, uint32_t B0, int tid) {
  static_assert(B::E >= 2, "");
  const int s0 = tid ? 31 - __clz(tid) : 0;
  w[0] = table[(B0 << s0) + (uint32_t)(tid ? tid - (1 << s0) : 0)];  // entry 0 is not used
#pragma unroll
  for (int k = 1; k < B::E; ++k) {
    const int s = B::LOGT + 31 - __builtin_clz(k);
    w[k] = table[(B0 << s) + (uint32_t)(k * B::T - (1 << s)) + (uint32_t)tid];
  }
}
template <class B, class T>
__device__ __forceinline__ void store_twiddles(const T (&w)[B::E], T* tw, int tid) {
  constexpr int PS = B::LAST_S0;
#pragma unroll
  for (int k = 0; k < B::E; ++k) {
    const uint32_t x = (uint32_t)(tid + k * B::T);
    const int s = k ? B::LOGT + 31 - __builtin_clz(k) : (tid ? 31 - __clz(tid) : 0);
    uint32_t pos = x;
    if (s >= PS) {  // grp = (p << rho) + g
      const int rho = s - PS;
      const uint32_t grp = x - (1u << s);
      pos = (1u << s) + ((grp & ((1u << rho) - 1)) << PS) + (grp >> rho);
    }
    tw[x ? pos : 0] = w[k];
  }
}

// ModDown's last block pass with the Q-limb KeyMult of digit-parallel plans
// folded in. One block b of one Q limb i in [tgt0, tgt0 + ntgt) of one item
// per workgroup (placed by xcd_tile), all five forward block passes of the
// limb share its twiddles, staged once in LDS:
//   s_c = -NTT(t2_c) + sum_{j in [j0, j1)} ext_j * evk[j][c],
//   ext_j = d (i in D_j) or the forward block pass of ext1 slot j,
//   out_c = s_c * P^-1 (canonical).
// t2 and ext1 raw in, |values| <= 5.4q inside. Inputs and key blocks are
// loaded before the transform that precedes their use, so that their latency
// overlaps it. That holds only while nothing waits for them early: words are kept
// as loaded and converted at their use (a conversion or a register spill after the
// loads waited for all of them), and 128 registers must hold the sums, the
// current block, the next one and both key blocks (buffer loads, whose addresses
// are scalar). With the waits where they belong, the twiddles staged with all loads
// in flight and 6 barriers instead of 10, (4, 2^16, 32), batch 8, went from 863 to
// 803 us and level 13 of it, batch 3, from 211 to 194.
template <int LOGM, int LOGE>
__global__ __launch_bounds__((1 << (LOGM - LOGE)), (LOGE == 3 && LOGM <= 12) ? 4 : 1) void k_moddown_km_blocks(
    DevTables tb, const uint64_t* d, const uint64_t* ext1, const uint64_t* evk, const uint64_t* t2, uint64_t* out,
    int j0, int j1, int nslots, int slot_stride, int tgt0, int ntgt, int items, EvalIn ev) {
  using B = BlockNtt<LOGM, LOGE>;
  extern __shared__ uint64_t lds[];
  double* ld = reinterpret_cast<double*>(lds);
  // Staged twiddles up to blocks of 2^12 (beyond, the extra LDS would leave
  // one workgroup per CU, which costs more than the table reads it saves).
  constexpr bool TWL = LOGM <= 12;
  double* tw = ld + B::LDS_WORDS;
  const size_t N = (size_t)1 << tb.log_n;
  const int R = (int)(N >> LOGM);
  const Tile tl = xcd_tile(R * ntgt, items);
  if (!tl.valid) return;
  const int tid = threadIdx.x, b = tl.tile % R;
  const int i = tgt0 + tl.tile / R;
  const int item = tl.item;
  const LimbC L = tb.limb[i];
  const int nl = tb.nl, ell = tb.ell;
  const size_t boff = (size_t)b * B::M;
  const double* twg = tb.twf_d + (size_t)i * N;
  const ArF A{L.qd, L.qinv, TWL ? tw : twg, twg};
  const uint32_t G0 = (uint32_t)(R + b);
  const int own = i / tb.alpha;  // the digit whose limbs include i: its input is d, already in NTT form
  // Loads ahead of use (words as they are in memory, converted where they are
  // used): always the second t2 component and the first key component of a
  // digit; with DEEP also the next digit's input and the second key component
  // (registers allow it up to blocks of 2^12).
  constexpr bool DEEP = LOGM <= 12;
  // input of digit j: d (CL layout) for the own digit, else ext1 (FR layout)
  auto load_digit = [&](int j, uint64_t (&w)[B::E]) {
    const uint64_t* src = j == own ? d + ((size_t)item * ell + i) * N + boff
                                   : ext1 + (((size_t)item * nslots + (slot_stride ? j : 0)) * nl + i) * N + boff;
    load_words<B>(src, j == own, tid, w);
  };
  // Sums: within q/2 after a fold, plus at most 1.85q a product (2.45q for E = 16)
  constexpr int FOLD = LOGE >= 4 ? 3 : 4;
  const double pinv = ldc(tb.dn_pinv_d + i);
  double s0[B::E], s1[B::E], cur[B::E];
  uint64_t nxt[B::E];
  load_words<B>(t2 + (((size_t)item * 2 + 0) * ell + i) * N + boff, false, tid, nxt);
  double twr[B::E];
  if constexpr (TWL) load_twiddles<B>(twr, twg, G0, tid);
#pragma unroll
  for (int e = 0; e < B::E; ++e) cur[e] = raw2d(nxt[e]);
  load_words<B>(t2 + (((size_t)item * 2 + 1) * ell + i) * N + boff, false, tid, nxt);
  if constexpr (TWL) {
    store_twiddles<B>(twr, tw, tid);
    __syncthreads();
  }
  fwd_opaque<B, TWL, false>(A, cur, ld, tid, G0);
#pragma unroll
  for (int e = 0; e < B::E; ++e) {
    s0[e] = -f_red(cur[e], L.qd, L.qinv);
    cur[e] = raw2d(nxt[e]);
  }
  if (DEEP && j0 < j1) load_digit(j0, nxt);
  fwd_opaque<B, TWL>(A, cur, ld, tid, G0);
#pragma unroll
  for (int e = 0; e < B::E; ++e) s1[e] = -f_red(cur[e], L.qd, L.qinv);
  for (int j = j0; j < j1; ++j) {
    const uint64_t* k0 = evk + key_row(tb, j, 0, i) * N + boff;
    const uint64_t* k1 = evk + key_row(tb, j, 1, i) * N + boff;
    uint64_t in[B::E], w0[B::E], w1[B::E];
    if constexpr (DEEP) {
#pragma unroll
      for (int e = 0; e < B::E; ++e) in[e] = nxt[e];
    }
    // The next input goes out before the transform, the key blocks before its last two
    // exchanges: all 24 loads of a thread at once hold a wave at their issue (the key
    // blocks, L2 hits, were 51 of the kernel's 352 us at (4, 2^16, 32), batch 8). The
    // call: 762 -> 754 us; (8, 2^17, 56), batch 2, 1063 -> 1046.
    if constexpr (DEEP) {
      if (j + 1 < j1) load_digit(j + 1, nxt);
    } else {
      load_words<B>(k0, true, tid, w0);
      load_digit(j, in);
    }
    if (j == own) {
      if constexpr (DEEP) {
        load_words<B>(k0, true, tid, w0);
        load_words<B>(k1, true, tid, w1);
      }
#pragma unroll
      for (int e = 0; e < B::E; ++e) cur[e] = u2d(in[e]);
    } else {
#pragma unroll
      for (int e = 0; e < B::E; ++e) cur[e] = raw2d(in[e]);
      fwd_opaque<B, TWL>(A, cur, ld, tid, G0, [&](int r) {
        if constexpr (DEEP) {
          if (r == (B::NR > 2 ? B::NR - 2 : 1)) load_words<B>(k0, true, tid, w0);
          if (r == B::NR - 1) load_words<B>(k1, true, tid, w1);
        }
      });
    }
    if constexpr (!DEEP) load_words<B>(k1, true, tid, w1);
#pragma unroll
    for (int e = 0; e < B::E; ++e) {
      s0[e] += f_mul(cur[e], u2d(w0[e]), L.qd, L.qinv);
      s1[e] += f_mul(cur[e], u2d(w1[e]), L.qd, L.qinv);
    }
    if ((j - j0) % FOLD == FOLD - 1) {
#pragma unroll
      for (int e = 0; e < B::E; ++e) {
        s0[e] = f_red(s0[e], L.qd, L.qinv);
        s1[e] = f_red(s1[e], L.qd, L.qinv);
      }
    }
  }
  const size_t r0 = (((size_t)item * 2 + 0) * ell + i) * N + boff, r1 = (((size_t)item * 2 + 1) * ell + i) * N + boff;
  // |s| <= 6.1q, |P^-1| <= q/2: the products are within 1.65q
#pragma unroll
  for (int e = 0; e < B::E; ++e) {
    s0[e] = f_mul(s0[e], pinv, L.qd, L.qinv);
    s1[e] = f_mul(s1[e], pinv, L.qd, L.qinv);
  }
  if (ev.a) {  // HMUL or HROT (chosen once per workgroup); |s| stays below 4q
    add_eval<B>(L, ev, r0, r1, (uint32_t)boff, tid, tb.log_n, s0, s1);
#pragma unroll
    for (int e = 0; e < B::E; ++e) {
      s0[e] = f_red(s0[e], L.qd, L.qinv);
      s1[e] = f_red(s1[e], L.qd, L.qinv);
    }
  }
#pragma unroll
  for (int e = 0; e < B::E; ++e) {
    const uint32_t x = (uint32_t)B::cl_pos(tid, e);
    __builtin_nontemporal_store(f_canon(s0[e], L.qd, L.qinv), out + r0 + x);  // the result is not read again here
    __builtin_nontemporal_store(f_canon(s1[e], L.qd, L.qinv), out + r1 + x);
  }
}

// --------------------------------- hoisted forward passes (KS_PLAN_HOIST_FWD)

// The digit-parallel KeyMult and ModDown tail when the raised digits are
// already forward-transformed (k_ext_blocks ran on ext1 in place, canonical
// residues in natural order): every workgroup then handles one component of
// one (limb, block, item) and runs at most one transform, so a launch has
// twice the workgroups of K3 / K5 and a quarter to a third of their serial
// chain, which is what a single small ciphertext needs.

// P limbs: acc_c[t] = sum_j ext1[j][t] * evk[j][c][t] (folded products below
// 1.5 * 2^60), then the inverse block pass; stored like K3's
// finalize (accp in [0, 4q], first-round layout). Tile (P limb, block),
// item (item, component).
template <int LOGM, int LOGE>
__global__ __launch_bounds__((1 << (LOGM - LOGE))) void k_keymult_pre(DevTables tb, const uint64_t* ext1,
                                                                      const uint64_t* evk, uint64_t* acc, int items2) {
  using B = BlockNtt<LOGM, LOGE>;
  extern __shared__ uint64_t lds[];
  const size_t N = (size_t)1 << tb.log_n;
  const int R = (int)(N >> LOGM);
  const Tile tl = xcd_tile(R * tb.k, items2);
  if (!tl.valid) return;
  const int tid = threadIdx.x, b = tl.tile % R;
  const int t = tb.ell + tl.tile / R;
  const int item = tl.item >> 1, c = tl.item & 1;
  const LimbC L = tb.limb[t];
  const int nl = tb.nl;
  const size_t boff = (size_t)b * B::M;
  const uint32_t delta = (uint32_t)L.delta;
  uint64_t s[B::E];
#pragma unroll
  for (int i = 0; i < B::E; ++i) s[i] = 0;
  for (int j = 0; j < tb.ndig; ++j) {
    const uint64_t* src = ext1 + (((size_t)item * tb.ndig + j) * nl + t) * N + boff;
    const uint64_t* key = evk + key_row(tb, j, c, t) * N + boff;
#pragma unroll
    for (int i = 0; i < B::E; ++i) {
      const int x = B::cl_pos(tid, i);
      s[i] += p_mul(src[x], key[x], delta);
    }
    if ((j & 7) == 7) {
#pragma unroll
      for (int i = 0; i < B::E; ++i) s[i] = p_red(s[i], delta);
    }
  }
#pragma unroll
  for (int i = 0; i < B::E; ++i) s[i] = p_red(s[i], delta);
  B::inv(ari(tb, L, t, true), s, lds, tid, (uint32_t)R + b);
  uint64_t* a = acc + (((size_t)item * 2 + c) * nl + t) * N + boff;
#pragma unroll
  for (int i = 0; i < B::E; ++i) a[B::fr_pos(tid, i)] = s[i];
}

// Q limbs: out_c[i] = (sum_j ext_j[i] * evk[j][c][i] - NTT(t2_c)[i]) * P^-1
// with ext_j = d for the digit that owns limb i (d, or a1 b1 / sigma(c1) for
// HMUL / HROT, natural order) and the pre-transformed ext1 slot otherwise;
// HMUL / HROT add their other terms of component c. Tile (Q limb, block),
// item (item, component).
template <int LOGM, int LOGE>
__global__ __launch_bounds__((1 << (LOGM - LOGE))) void k_moddown_pre(DevTables tb, const uint64_t* d,
                                                                      const uint64_t* ext1, const uint64_t* evk,
                                                                      const uint64_t* t2, uint64_t* out, int items2,
                                                                      EvalIn ev) {
  using B = BlockNtt<LOGM, LOGE>;
  extern __shared__ uint64_t lds[];
  const size_t N = (size_t)1 << tb.log_n;
  const int R = (int)(N >> LOGM);
  const Tile tl = xcd_tile(R * tb.ell, items2);
  if (!tl.valid) return;
  const int tid = threadIdx.x, b = tl.tile % R;
  const int i = tl.tile / R;
  const int item = tl.item >> 1, c = tl.item & 1;
  const LimbC L = tb.limb[i];
  const int nl = tb.nl, ell = tb.ell;
  const size_t boff = (size_t)b * B::M;
  const int own = i / tb.alpha;
  double v[B::E];
  {
    const uint64_t* src = t2 + (((size_t)item * 2 + c) * ell + i) * N + boff;
#pragma unroll
    for (int e = 0; e < B::E; ++e) v[e] = raw2d(ld_once(src + B::fr_pos(tid, e)));
  }
  B::fwd(arf(tb, L, i, false), v, reinterpret_cast<double*>(lds), tid, (uint32_t)R + b);
  double sum[B::E];
#pragma unroll
  for (int e = 0; e < B::E; ++e) sum[e] = -f_red(v[e], L.qd, L.qinv);
  for (int j = 0; j < tb.ndig; ++j) {
    const uint64_t* src = j == own ? d + ((size_t)item * ell + i) * N + boff
                                   : ext1 + (((size_t)item * tb.ndig + j) * nl + i) * N + boff;
    const uint64_t* key = evk + key_row(tb, j, c, i) * N + boff;
#pragma unroll
    for (int e = 0; e < B::E; ++e) {
      const int x = B::cl_pos(tid, e);
      sum[e] += f_mul(u2d(src[x]), u2d(key[x]), L.qd, L.qinv);  // canonical operands: within 0.875q
    }
    if ((j & 7) == 7) {  // q/2 + 8 * 0.875q stays below 8q < 2^53
#pragma unroll
      for (int e = 0; e < B::E; ++e) sum[e] = f_red(sum[e], L.qd, L.qinv);
    }
  }
  const double pinv = tb.dn_pinv_d[i];
  const size_t r0 = (((size_t)item * 2 + 0) * ell + i) * N + boff, r1 = (((size_t)item * 2 + 1) * ell + i) * N + boff;
  const size_t rc = c ? r1 : r0;
#pragma unroll
  for (int e = 0; e < B::E; ++e) {
    const int x = B::cl_pos(tid, e);
    double o = f_mul(sum[e], pinv, L.qd, L.qinv);  // |sum| <= 6.7q: within 1.76q
    if (ev.a) {
      if (ev.galois) {  // HROT: sigma(c0) joins component 0
        if (c == 0) o += u2d(ev.a[r0 + x - (boff + x) + galois_src((uint32_t)(boff + x), ev.galois, tb.log_n)]);
      } else {  // HMUL: a0 b0 to component 0, a0 b1 + a1 b0 to component 1
        const double a0 = u2d(ev.a[r0 + x]);
        if (c == 0)
          o += f_mul(a0, u2d(ev.b[r0 + x]), L.qd, L.qinv);
        else
          o += f_mul(a0, u2d(ev.b[r1 + x]), L.qd, L.qinv) + f_mul(u2d(ev.a[r1 + x]), u2d(ev.b[r0 + x]), L.qd, L.qinv);
      }
      o = f_red(o, L.qd, L.qinv);
    }
    __builtin_nontemporal_store(f_canon(o, L.qd, L.qinv), out + rc + x);
  }
}

// ------------------------------------------------------ standalone kernels

// ks_modup: forward block pass of every non-digit limb of ext (in place; Q raw
// in, P below 2^64 in, canonical out).
template <int LOGM, int LOGE>
__global__ __launch_bounds__((1 << (LOGM - LOGE))) void k_ext_blocks(DevTables tb, uint64_t* ext) {
  using B = BlockNtt<LOGM, LOGE>;
  extern __shared__ uint64_t lds[];
  const int tid = threadIdx.x, b = blockIdx.x;
  const int t = blockIdx.y;
  const int j = blockIdx.z % tb.ndig;
  const int lo = j * tb.alpha;
  if (t >= lo && t < lo + tb.alpha && t < tb.ell) return;  // uniform over the workgroup
  const LimbC L = tb.limb[t];
  const size_t N = (size_t)1 << tb.log_n;
  const uint32_t B0 = (uint32_t)(N >> LOGM) + b;
  uint64_t* a = ext + ((size_t)blockIdx.z * tb.nl + t) * N + (size_t)b * B::M;
  if (t < tb.ell) {
    double v[B::E];
#pragma unroll
    for (int e = 0; e < B::E; ++e) v[e] = raw2d(a[B::fr_pos(tid, e)]);
    B::fwd(arf(tb, L, t, false), v, reinterpret_cast<double*>(lds), tid, B0);
#pragma unroll
    for (int e = 0; e < B::E; ++e) a[B::cl_pos(tid, e)] = f_canon_wide(v[e], L.qd, L.qinv);
  } else {
    uint64_t v[B::E];
#pragma unroll
    for (int e = 0; e < B::E; ++e) v[e] = a[B::fr_pos(tid, e)];
    B::fwd(ari(tb, L, t, false), v, lds, tid, B0);
#pragma unroll
    for (int e = 0; e < B::E; ++e) a[B::cl_pos(tid, e)] = p_canon(v[e], L.q, L.delta);
  }
}

// ext[item][j][t] = d[item][t] for t in D_j.
__global__ void k_copy_digits(DevTables tb, const uint64_t* d, uint64_t* ext) {
  const size_t N = (size_t)1 << tb.log_n;
  const size_t x = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= N) return;
  const int t = blockIdx.y, item = blockIdx.z;
  const int j = t / tb.alpha;
  ext[(((size_t)item * tb.ndig + j) * tb.nl + t) * N + x] = d[((size_t)item * tb.ell + t) * N + x];
}

// ks_bconv: coefficient-form conversion of one source set, one thread per
// coefficient, integer arithmetic. src [items][ns][N], dst [items][nd][N].
__global__ void k_bconv(DevTables tb, const uint64_t* src, uint64_t* dst, int set) {
  const size_t N = (size_t)1 << tb.log_n;
  const size_t x = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= N) return;
  const int u = blockIdx.y, item = blockIdx.z;
  int lo, hi, t;
  if (set < 0) {
    lo = tb.ell;
    hi = tb.nl;
    t = u;
  } else {
    lo = set * tb.alpha;
    hi = min(lo + tb.alpha, tb.ell);
    t = u < lo ? u : u + (hi - lo);
  }
  const int ns = hi - lo;
  const int nd = tb.nl - ns;
  const LimbC L = tb.limb[t];
  uint64_t z = 0;
  for (int s = 0; s < ns; ++s) {
    const int i = lo + s;
    const LimbC S = tb.limb[i];
    // y_i = x_i * [(S/s_i)^-1]_{s_i}, canonical
    const uint64_t* hinv = set < 0 ? tb.dn_hinv + 2 * s : tb.up_hinv + 2 * i;
    const uint64_t xi = src[((size_t)item * ns + s) * N + x];
    const uint64_t y = reduce2(mul_shoup(xi, hinv[0], hinv[1], S.q), S.q);
    const uint64_t* cst = set < 0 ? tb.dn_mat + 2 * ((size_t)s * tb.ell + t) : tb.up_mat + 2 * ((size_t)i * tb.nl + t);
    z += reduce2(mul_shoup(y, cst[0], cst[1], L.q), L.q);
    if ((s & 7) == 7) z = reduce2(mul_shoup(z, 1, L.red_s, L.q), L.q);
  }
  dst[((size_t)item * nd + u) * N + x] = reduce2(mul_shoup(z, 1, L.red_s, L.q), L.q);
}

// ks_bconv on the matrix cores, for the numbers of sources the column kernels take
// them for: a workgroup converts BC_R rows of 64 (32 from 6 steps on) of the N
// coefficients (rows N / BC_R apart, which keeps every access to consecutive
// words) to the target groups g with g mod gridDim.z = blockIdx.z. Phase 1 scales
// each source word once and packs its digits; the scalar kernel does that again for
// every target (114 us for 8 sources to 32 targets of 4 x 2^16 coefficients).
constexpr int BC_LOGR = 3, BC_R = 1 << BC_LOGR;

template <int NM>
__global__ __launch_bounds__(CT, mx_waves(BC_LOGR, NM)) void k_bconv_mx(DevTables tb, const uint64_t* src,
                                                                        uint64_t* dst, int set) {
  constexpr int C = mx_cols(BC_LOGR, NM), SPW = TC / C;
  extern __shared__ ulonglong2 yp[];
  const int M = 1 << (tb.log_n - BC_LOGR);
  const size_t N = (size_t)M * BC_R;
  const int lane = threadIdx.x & (TC - 1), wv = threadIdx.x / TC, col = lane & (C - 1);
  const size_t c = (size_t)blockIdx.x * C + col;
  const bool live = c < (size_t)M;
  const int item = blockIdx.y, ell = tb.ell, k = tb.k;
  const int lo = set < 0 ? ell : set * tb.alpha;
  const int ns = (set < 0 ? tb.nl : min(lo + tb.alpha, ell)) - lo;
  uint64_t* yw = reinterpret_cast<uint64_t*>(yp);
  for (int s = wv * SPW + lane / C; s < 4 * NM; s += CW * SPW) {
    uint64_t y[BC_R];
#pragma unroll
    for (int r = 0; r < BC_R; ++r) y[r] = 0;
    if (live && s < ns) {
      const uint64_t q = tb.limb[lo + s].q;
      const uint64_t* hinv = set < 0 ? tb.dn_hinv + 2 * s : tb.up_hinv + 2 * (lo + s);
      const uint64_t w = hinv[0], ws = hinv[1];
      const uint64_t* a = src + ((size_t)item * ns + s) * N + c;
#pragma unroll
      for (int r = 0; r < BC_R; ++r) y[r] = a[(size_t)r * M];
#pragma unroll
      for (int r = 0; r < BC_R; ++r) y[r] = mx_pack(reduce2(mul_shoup(y[r], w, ws, q), q));
    }
#pragma unroll
    for (int r = 0; r < BC_R; ++r) yw[((size_t)((s >> 1) * BC_R + r) * C + col) * 2 + (s & 1)] = y[r];
  }
  __syncthreads();
  const int h = lane >> 5;
  const size_t cc = (size_t)blockIdx.x * C + (C == 64 ? (wv & 1) * 32 : 0) + (lane & 31);
  const bool clive = cc < (size_t)M;
  const int nq = set < 0 ? ell : ell - ns, nqg = (nq + 3) >> 2, ng = nqg + (set < 0 ? 0 : (k + 3) >> 2);
  uint64_t* o = dst + (size_t)item * (set < 0 ? ell : tb.nl - ns) * N;
  const ulonglong2* cst = set < 0 ? reinterpret_cast<const ulonglong2*>(tb.dn_mx)
                                  : reinterpret_cast<const ulonglong2*>(tb.up_mx) + (size_t)set * tb.up_ng * NM * 64;
  for (int g = (wv / (C / 32)) * gridDim.z + blockIdx.z; g < ng; g += (CW / (C / 32)) * gridDim.z) {
    const bool qg = g < nqg;
    // target tau of the group is output row u; the last group of each kind may be short
    const int u0 = qg ? 4 * g : nq + 4 * (g - nqg), cnt = min(4, qg ? nq - 4 * g : k - 4 * (g - nqg));
    int lt[4];
#pragma unroll
    for (int tau = 0; tau < 4; ++tau) {
      const int u = u0 + min(tau, cnt - 1);
      lt[tau] = set < 0 || u < lo ? u : u + ns;
    }
    const bool sa = clive && 2 * h < cnt, sb = clive && 2 * h + 1 < cnt;
    uint64_t* oa = o + (size_t)(u0 + (sa ? 2 * h : 0)) * N;
    uint64_t* ob = o + (size_t)(u0 + (sb ? 2 * h + 1 : 0)) * N;
    if (qg)
      mx_group<BC_LOGR, true, NM, true>(tb, yp, cst + (size_t)g * NM * 64, lt, sa, sb, oa, ob, cc, M);
    else
      mx_group<BC_LOGR, false, NM, true>(tb, yp, cst + (size_t)g * NM * 64, lt, sa, sb, oa, ob, cc, M);
  }
}

// ------------------------------------------------- HMUL and HROT (element-wise)

// HMUL's tensor product over the Q limbs: for ciphertexts a, b
// [items][2][ell][N] (canonical, NTT form): t01 [items][2][ell][N] gets
// (a0 b0, a0 b1 + a1 b0) and d2 [items][ell][N] gets a1 b1, canonical.
// Grid: (ceil(N / 256), ell, items).
__global__ __launch_bounds__(256) void k_tensor(DevTables tb, const uint64_t* a, const uint64_t* b, uint64_t* t01,
                                                uint64_t* d2) {
  const size_t N = (size_t)1 << tb.log_n;
  const size_t x = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (x >= N) return;
  const int i = blockIdx.y, item = blockIdx.z, ell = tb.ell;
  const LimbC L = tb.limb[i];
  const size_t r0 = (((size_t)item * 2 + 0) * ell + i) * N + x, r1 = (((size_t)item * 2 + 1) * ell + i) * N + x;
  const double a0 = u2d(a[r0]), a1 = u2d(a[r1]), b0 = u2d(b[r0]), b1 = u2d(b[r1]);
  t01[r0] = f_canon(f_mul(a0, b0, L.qd, L.qinv), L.qd, L.qinv);
  t01[r1] = f_canon(f_mul(a0, b1, L.qd, L.qinv) + f_mul(a1, b0, L.qd, L.qinv), L.qd, L.qinv);
  d2[((size_t)item * ell + i) * N + x] = f_canon(f_mul(a1, b1, L.qd, L.qinv), L.qd, L.qinv);
}

// The Galois automorphism x -> x^g on NTT-form limbs: slot t holds the value at
// psi^(2 brv(t) + 1), so slot t of the image is slot t' of the input with
// 2 brv(t') + 1 = g (2 brv(t) + 1) mod 2N. src and dst [rows][N] (rows =
// gridDim.y * gridDim.z, any limbs), dst must not alias src.
// Grid: (ceil(N / 256), rows per item, items).
__global__ __launch_bounds__(256) void k_automorph(int log_n, const uint64_t* src, uint64_t* dst, uint32_t g,
                                                   size_t src_item_stride, size_t dst_item_stride) {
  const uint32_t N = 1u << log_n;
  const uint32_t t = blockIdx.x * 256 + threadIdx.x;
  if (t >= N) return;
  const uint32_t e = 2u * (__brev(t) >> (32 - log_n)) + 1u;
  const uint32_t e2 = (uint32_t)(((uint64_t)g * e) & (2u * N - 1u));
  const uint32_t t2 = __brev((e2 - 1u) >> 1) >> (32 - log_n);
  const size_t row = blockIdx.y;
  dst[(size_t)blockIdx.z * dst_item_stride + row * N + t] = src[(size_t)blockIdx.z * src_item_stride + row * N + t2];
}

// out[item][c][i] += add[item][c][i] mod q_i for c < ncomp (both canonical).
// Grid: (ceil(N / 256), ncomp * ell, items).
__global__ __launch_bounds__(256) void k_add_q(DevTables tb, uint64_t* out, const uint64_t* add) {
  const size_t N = (size_t)1 << tb.log_n;
  const size_t x = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (x >= N) return;
  const int ell = tb.ell;
  const int c = blockIdx.y / ell, i = blockIdx.y % ell, item = blockIdx.z;
  const uint64_t q = tb.limb[i].q;
  const size_t r = (((size_t)item * 2 + c) * ell + i) * N + x;
  const uint64_t v = out[r] + add[r];
  out[r] = v >= q ? v - q : v;
}

// ks_keymult: element-wise over acc [items][2][nl][N]. A thread takes E elements
// (256 apart) of one limb for IT items and both components, so that ext is read
// once and a key word once for IT items: it is bound by those bytes (420 MB for
// two items of (4, 2^16, 32); one item and component a thread read 588 MB). Q limbs
// on FP64 (canonical operands: each product within 0.88q), P limbs with p_mul.
// Small calls are bound by a thread's chain over the digits instead, and take E = IT = 1
// (see launch_keymult); there the next digit's loads go out with the current one's.
// Grid: (ceil(N / (256 E)), nl, ceil(items / IT)).
template <int IT, int E>
__global__ __launch_bounds__(256) void k_keymult(DevTables tb, const uint64_t* ext, const uint64_t* evk,
                                                 uint64_t* acc, int items) {
  constexpr int UNROLL = IT * E == 1 ? 2 : 1;
  const size_t N = (size_t)1 << tb.log_n;
  const size_t x0 = (size_t)blockIdx.x * (256 * E) + threadIdx.x;
  const int t = blockIdx.y, i0 = blockIdx.z * IT, nl = tb.nl, ndig = tb.ndig;
  const LimbC L = tb.limb[t];
  const uint32_t delta = (uint32_t)L.delta;
  // words past the end of a small limb or batch are read from its first word or item, and not stored
  size_t x[E];
#pragma unroll
  for (int e = 0; e < E; ++e) x[e] = x0 + 256 * e < N ? x0 + 256 * e : 0;
  const bool isq = t < tb.ell;
  double sq[IT][2][E];
  uint64_t sp[IT][2][E];
#pragma unroll
  for (int i = 0; i < IT; ++i)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      sq[i][0][e] = sq[i][1][e] = 0.0;
      sp[i][0][e] = sp[i][1][e] = 0;
    }
  auto load = [&](int j, uint64_t (&kw)[2][E], uint64_t (&w)[IT][E]) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const uint64_t* key = evk + key_row(tb, j, c, t) * N;
#pragma unroll
      for (int e = 0; e < E; ++e) kw[c][e] = key[x[e]];
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const uint64_t* a = ext + (((size_t)(i0 + i < items ? i0 + i : i0) * ndig + j) * nl + t) * N;
#pragma unroll
      for (int e = 0; e < E; ++e) w[i][e] = a[x[e]];
    }
  };
  uint64_t kw[2][E], w[IT][E];
  if (isq) {
#pragma unroll UNROLL
    for (int j = 0; j < ndig; ++j) {
      load(j, kw, w);
#pragma unroll
      for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int e = 0; e < E; ++e) {
            sq[i][c][e] += f_mul(u2d(w[i][e]), u2d(kw[c][e]), L.qd, L.qinv);
            if ((j & 7) == 7) sq[i][c][e] = f_red(sq[i][c][e], L.qd, L.qinv);
          }
    }
  } else {
#pragma unroll UNROLL
    for (int j = 0; j < ndig; ++j) {
      load(j, kw, w);
#pragma unroll
      for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int e = 0; e < E; ++e) {
            sp[i][c][e] += p_mul(w[i][e], kw[c][e], delta);
            if ((j & 7) == 7) sp[i][c][e] = p_red(sp[i][c][e], delta);
          }
    }
  }
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    if (i0 + i >= items) break;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      uint64_t* a = acc + (((size_t)(i0 + i) * 2 + c) * nl + t) * N;
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (x0 + 256 * e < N)
          a[x[e]] = isq ? f_canon_wide(sq[i][c][e], L.qd, L.qinv) : p_canon(sp[i][c][e], L.q, delta);
    }
  }
}

// ks_moddown, first step: inverse block pass of the P limbs of acc
// (canonical) into the work buffer accp (same layout), values in [0, 4q].
template <int LOGM, int LOGE>
__global__ __launch_bounds__((1 << (LOGM - LOGE))) void k_pblocks_inv(DevTables tb, const uint64_t* acc,
                                                                      uint64_t* accp) {
  using B = BlockNtt<LOGM, LOGE>;
  extern __shared__ uint64_t lds[];
  const int tid = threadIdx.x, b = blockIdx.x;
  const int t = tb.ell + blockIdx.y;
  const int ic = blockIdx.z;
  const LimbC L = tb.limb[t];
  const size_t N = (size_t)1 << tb.log_n;
  const uint32_t B0 = (uint32_t)(N >> LOGM) + b;
  const size_t off = ((size_t)ic * tb.nl + t) * N + (size_t)b * B::M;
  uint64_t v[B::E];
#pragma unroll
  for (int e = 0; e < B::E; ++e) v[e] = acc[off + B::cl_pos(tid, e)];
  B::inv(ari(tb, L, t, true), v, lds, tid, B0);
#pragma unroll
  for (int e = 0; e < B::E; ++e) accp[off + B::fr_pos(tid, e)] = v[e];
}

// ------------------------------------------------------------ dispatching


template <template <int> class F, typename... A>
hipError_t by_logr(int log_r, A... a) {
  switch (log_r) {
    case 0: return F<0>::run(a...);
    case 1: return F<1>::run(a...);
    case 2: return F<2>::run(a...);
    case 3: return F<3>::run(a...);
    case 4: return F<4>::run(a...);
    case 5: return F<5>::run(a...);
    default: return hipErrorInvalidValue;
  }
}

// Elements per thread of the plain block passes: 8 up to blocks of 2^12 (twice the
// threads per block that 16 give, which small transforms need to fill the chip: -22%
// on (2, 2^13, 6) with one ciphertext; at 2^12, -2% on modup + keymult + moddown and
// on HMUL of (4, 2^16, 32)) and 16 beyond. `lean`, the passes that read and write little
// beside their block (the plain inverse ones, k_keymult_pre and k_moddown_pre), take 16 at
// 2^12 too: one LDS exchange less, 2% of (2, 2^15, 10), batch 32.
constexpr int loge_for(int logm, bool lean) {
  return logm >= (lean ? 12 : 13) ? 4 : (logm >= 6 ? 3 : (logm >= 4 ? 2 : 1));
}

// Latency variant of a block pass: 4 elements per thread (8 at blocks of
// 2^13), so that a block of 2^11 to 2^13 coefficients runs on 512 to 1024
// threads. A launch whose default configuration would leave the chip short of
// threads (a single small ciphertext) is bound by the serial chain of each
// thread and by latencies that its few waves cannot hide; halving or
// quartering the elements per thread shortens the chain and puts up to four
// waves on every SIMD that runs a block.
constexpr int loge_lat(int logm) { return logm >= 13 ? 3 : 2; }

// Whether a launch of `wgs` workgroups of blocks of 2^logm with 2^loge
// elements per thread has fewer than 2^18 threads (4 waves per SIMD over the
// 1024 SIMDs): then its latency variant runs instead.
inline bool use_lat(int logm, int loge, long wgs) {
  return logm >= 8 && logm <= 13 && loge_lat(logm) < loge && wgs * (1L << (logm - loge)) < (1L << 18);
}

template <template <int, int> class F, bool LEAN = false, typename... A>
hipError_t by_logm(int log_m, long wgs, A... a) {
  switch (log_m) {
#define KS_CASE(m) \
  case m:                                                                             \
    return use_lat(m, loge_for(m, LEAN), wgs) ? F<m, loge_lat(m)>::run(a...) \
                                                   : F<m, loge_for(m, LEAN)>::run(a...);
    KS_CASE(3) KS_CASE(4) KS_CASE(5) KS_CASE(6) KS_CASE(7) KS_CASE(8) KS_CASE(9) KS_CASE(10) KS_CASE(11)
    KS_CASE(12) KS_CASE(13) KS_CASE(14)
#undef KS_CASE
    default: return hipErrorInvalidValue;
  }
}

// KeyMult keeps two accumulators per element across the digits, so its block
// passes run with 8 elements per thread up to M = 2^13 (1024 threads at 2^13)
// and 16 beyond. K5 also holds its prefetched inputs and key blocks: 8
// elements per thread up to 2^12, 16 from 2^13 on (at 1024 threads it would
// spill).
constexpr int loge_k3(int logm) { return logm >= 14 ? 4 : (logm >= 6 ? 3 : (logm >= 4 ? 2 : 1)); }
constexpr int loge_k5(int logm) { return logm >= 13 ? 4 : loge_k3(logm); }

template <template <int, int> class F, bool K5 = false, typename... A>
hipError_t by_logm_k3(int log_m, long wgs, A... a) {
  switch (log_m) {
#define KS_CASE(m)                                                                   \
  case m:                                                                            \
    return use_lat(m, K5 ? loge_k5(m) : loge_k3(m), wgs) ? F<m, loge_lat(m)>::run(a...) \
                                                         : F<m, K5 ? loge_k5(m) : loge_k3(m)>::run(a...);
    KS_CASE(3) KS_CASE(4) KS_CASE(5) KS_CASE(6) KS_CASE(7) KS_CASE(8) KS_CASE(9) KS_CASE(10) KS_CASE(11)
    KS_CASE(12) KS_CASE(13) KS_CASE(14)
#undef KS_CASE
    default: return hipErrorInvalidValue;
  }
}

dim3 col_grid(int log_m, int y, int z, int cols = TC) {
  return dim3((unsigned)(((1 << log_m) + cols - 1) / cols), (unsigned)y, (unsigned)z);
}

template <int LOGM, int LOGE>
size_t block_lds() {
  return sizeof(uint64_t) * BlockNtt<LOGM, LOGE>::LDS_WORDS;
}

// Lets a kernel take up to the whole 160 KB of LDS as dynamic shared memory
// (done once per kernel instantiation).
template <auto Kernel>
void allow_lds() {
  static const hipError_t once = hipFuncSetAttribute(reinterpret_cast<const void*>(Kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  (void)once;
}

template <int LOGR>
struct ColsFwd {
  static hipError_t run(const DevTables& tb, uint64_t* x, int first, int nl, int items, int log_m, hipStream_t s) {
    k_cols<LOGR, false><<<col_grid(log_m, nl, items), dim3(TC), 0, s>>>(tb, x, first, nl, log_m);
    return hipGetLastError();
  }
};
template <int LOGR>
struct ColsInv {
  static hipError_t run(const DevTables& tb, uint64_t* x, int first, int nl, int items, int log_m, hipStream_t s) {
    k_cols<LOGR, true><<<col_grid(log_m, nl, items), dim3(TC), 0, s>>>(tb, x, first, nl, log_m);
    return hipGetLastError();
  }
};
template <int LOGM, int LOGE>
struct BlocksFwd {
  static hipError_t run(const DevTables& tb, const uint64_t* src, uint64_t* dst, int first, int nl, int items,
                        int whole, hipStream_t s) {
    using B = BlockNtt<LOGM, LOGE>;
    allow_lds<k_blocks<LOGM, LOGE, false>>();
    k_blocks<LOGM, LOGE, false><<<dim3(xcd_grid(nl << (tb.log_n - LOGM), items)), dim3(B::T),
                                  block_lds<LOGM, LOGE>(), s>>>(tb, src, dst, first, nl, items, whole);
    return hipGetLastError();
  }
};
template <int LOGM, int LOGE>
struct BlocksInv {
  static hipError_t run(const DevTables& tb, const uint64_t* src, uint64_t* dst, int first, int nl, int items,
                        int whole, hipStream_t s) {
    using B = BlockNtt<LOGM, LOGE>;
    allow_lds<k_blocks<LOGM, LOGE, true>>();
    k_blocks<LOGM, LOGE, true><<<dim3(xcd_grid(nl << (tb.log_n - LOGM), items)), dim3(B::T),
                                 block_lds<LOGM, LOGE>(), s>>>(tb, src, dst, first, nl, items, whole);
    return hipGetLastError();
  }
};
template <int LOGR>
struct ModupCols {
  static hipError_t run(const DevTables& tb, const uint64_t* t1, uint64_t* ext1, int j0, int nj, int nslots,
                        int slot_stride, int tgt0, int tgt1, int items, int log_m, hipStream_t s) {
    allow_lds<k_modup_cols<LOGR>>();
    const size_t lds = sizeof(double) * (size_t)tb.alpha * (1 << LOGR) * TC;
    k_modup_cols<LOGR><<<col_grid(log_m, nj, items), dim3(CT), lds, s>>>(tb, t1, ext1, j0, nslots, slot_stride, tgt0,
                                                                         tgt1, log_m);
    return hipGetLastError();
  }
};
// Steps (of four sources) an MFMA column kernel is built for: 8, or fewer at the row
// counts for which a plan is accepted with fewer sources only (stage_cap: at most 320 / 2^logr).
constexpr int mx_max_nm(int logr) { return logr <= 3 ? 8 : (logr == 4 ? 5 : 3); }

// F<LOGR, nm>::run for a runtime nm.
template <template <int, int> class F, int LOGR, int NM = 1, typename... A>
hipError_t by_nm(int nm, A... a) {
  if constexpr (NM > mx_max_nm(LOGR))
    return hipErrorInvalidValue;
  else
    return nm == NM ? F<LOGR, NM>::run(a...) : by_nm<F, LOGR, NM + 1>(nm, a...);
}
// Workgroups that share the target groups of one column tile: doubled while a launch
// has fewer than one workgroup for each CU and every wave still gets a group. One
// ciphertext of (4, 2^16, 32) has 128 tiles in ModDown with two groups a wave: 28 us
// there, 22 with two parts. With a workgroup on every CU the repeated phase 1 takes
// what the shorter phase 2 gives (ModUp of the same call, 256 tiles: 37 and 38 us).
inline int mx_parts(long tiles, int groups, int cols) {
  int parts = 1;
  while (tiles * parts < 256 && groups > (CW / (cols / 32)) * parts) parts *= 2;
  return parts;
}

template <int LOGR, int NM>
struct ModupColsMxN {
  static hipError_t run(const DevTables& tb, const uint64_t* t1, uint64_t* ext1, int j0, int nj, int nslots,
                        int slot_stride, int tgt0, int tgt1, int items, int log_m, hipStream_t s) {
    const auto kernel = tgt0 == 0 && tgt1 == tb.nl ? k_modup_cols_mx<LOGR, NM, true> : k_modup_cols_mx<LOGR, NM, false>;
    allow_lds<k_modup_cols_mx<LOGR, NM, true>>();
    allow_lds<k_modup_cols_mx<LOGR, NM, false>>();
    dim3 g = col_grid(log_m, nj, items, mx_cols(LOGR, NM));
    const int na = tb.alpha < tb.ell ? tb.alpha : tb.ell;
    // All the groups of a digit, also for a launch over a chunk of the targets, which may then have
    // workgroups with one group or none: they run on CUs that are idle. With the chunk's
    // groups: (4, 2^16, 32), DSOC, one ciphertext, 4 chunks, 523 -> 537 us, and batch 2,
    // 8 chunks, 1005 -> 983; 100 other chunked calls within 1.5% both ways.
    const int parts = mx_parts((long)g.x * g.y * g.z, (tb.ell - na + 3) / 4 + (tb.k + 3) / 4, mx_cols(LOGR, NM));
    g.x *= parts;
    kernel<<<g, dim3(CT), mx_lds(LOGR, NM), s>>>(tb, t1, ext1, j0, nslots, slot_stride, tgt0, tgt1, log_m, parts);
    return hipGetLastError();
  }
};
template <int LOGR>
struct ModupColsMx {
  template <typename... A>
  static hipError_t run(const DevTables& tb, A... a) {
    return by_nm<ModupColsMxN, LOGR>(tb.up_nm, tb, a...);
  }
};
template <int LOGM, int LOGE>
struct KeymultBlocks {
  static hipError_t run(const DevTables& tb, const uint64_t* d, const uint64_t* ext1, const uint64_t* evk,
                        uint64_t* acc, int j0, int j1, int nslots, int slot_stride, int tgt0, int tgt1, int items,
                        int accumulate, int finalize, int q_part, hipStream_t s) {
    using B = BlockNtt<LOGM, LOGE>;
    const int qend = tgt1 < tb.ell ? tgt1 : tb.ell;
    if (q_part && tgt0 < qend) {
      allow_lds<k_keymult_blocks<LOGM, LOGE, true>>();
      k_keymult_blocks<LOGM, LOGE, true><<<dim3(xcd_grid((qend - tgt0) << (tb.log_n - LOGM), items)), dim3(B::T),
                                           block_lds<LOGM, LOGE>(), s>>>(tb, d, ext1, evk, acc, j0, j1, nslots,
                                                                         slot_stride, tgt0, qend - tgt0, items,
                                                                         accumulate, finalize);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    const int pbeg = tgt0 > tb.ell ? tgt0 : tb.ell;
    if (pbeg < tgt1) {
      allow_lds<k_keymult_blocks<LOGM, LOGE, false>>();
      k_keymult_blocks<LOGM, LOGE, false><<<dim3(xcd_grid((tgt1 - pbeg) << (tb.log_n - LOGM), items)), dim3(B::T),
                                            block_lds<LOGM, LOGE>(), s>>>(tb, d, ext1, evk, acc, j0, j1, nslots,
                                                                          slot_stride, pbeg, tgt1 - pbeg, items,
                                                                          accumulate, finalize);
    }
    return hipGetLastError();
  }
};
template <int LOGR>
struct ModdownCols {
  static hipError_t run(const DevTables& tb, const uint64_t* accp, uint64_t* t2, int tgt0, int tgt1, int items,
                        int log_m, hipStream_t s) {
    allow_lds<k_moddown_cols<LOGR>>();
    const size_t lds = sizeof(uint64_t) * (size_t)tb.k * (1 << LOGR) * TC;
    k_moddown_cols<LOGR><<<col_grid(log_m, 2, items), dim3(CT), lds, s>>>(tb, accp, t2, tgt0, tgt1, log_m);
    return hipGetLastError();
  }
};
template <int LOGR, int NM>
struct ModdownColsMxN {
  static hipError_t run(const DevTables& tb, const uint64_t* accp, uint64_t* t2, int tgt0, int tgt1, int items,
                        int log_m, hipStream_t s) {
    const auto kernel =
        tgt0 == 0 && tgt1 == tb.ell ? k_moddown_cols_mx<LOGR, NM, true> : k_moddown_cols_mx<LOGR, NM, false>;
    allow_lds<k_moddown_cols_mx<LOGR, NM, true>>();
    allow_lds<k_moddown_cols_mx<LOGR, NM, false>>();
    dim3 g = col_grid(log_m, 2, items, mx_cols(LOGR, NM));
    const int parts = mx_parts((long)g.x * g.y * g.z, (tgt1 - tgt0 + 3) / 4, mx_cols(LOGR, NM));
    g.x *= parts;
    kernel<<<g, dim3(CT), mx_lds(LOGR, NM), s>>>(tb, accp, t2, tgt0, tgt1, log_m, parts);
    return hipGetLastError();
  }
};
template <int LOGR>
struct ModdownColsMx {
  template <typename... A>
  static hipError_t run(const DevTables& tb, A... a) {
    return by_nm<ModdownColsMxN, LOGR>(tb.dn_nm, tb, a...);
  }
};
template <int LOGR, int NM>
struct BconvMxN {
  static hipError_t run(const DevTables& tb, const uint64_t* src, int set, uint64_t* dst, int items, hipStream_t s) {
    allow_lds<k_bconv_mx<NM>>();
    dim3 g = col_grid(tb.log_n - BC_LOGR, items, 1, mx_cols(BC_LOGR, NM));
    // few workgroups: the target groups are shared out over up to 4 of them
    // (each scales the sources again), until there are two for every CU
    while (g.z < 4 && g.x * g.y * g.z < 512) g.z *= 2;
    k_bconv_mx<NM><<<g, dim3(CT), mx_lds(BC_LOGR, NM), s>>>(tb, src, dst, set);
    return hipGetLastError();
  }
};
template <int LOGM, int LOGE>
struct ModdownBlocks {
  static hipError_t run(const DevTables& tb, const uint64_t* t2, const uint64_t* acc, uint64_t* out, int tgt0,
                        int tgt1, int items, EvalIn ev, hipStream_t s) {
    using B = BlockNtt<LOGM, LOGE>;
    allow_lds<k_moddown_blocks<LOGM, LOGE>>();
    k_moddown_blocks<LOGM, LOGE><<<dim3(xcd_grid((tgt1 - tgt0) << (tb.log_n - LOGM), items * 2)), dim3(B::T),
                                   block_lds<LOGM, LOGE>(), s>>>(tb, t2, acc, out, tgt0, tgt1 - tgt0, items * 2, ev);
    return hipGetLastError();
  }
};
template <int LOGM, int LOGE>
struct EvalBlocks {
  static hipError_t run(const DevTables& tb, EvalIn ev, uint64_t* d2, uint64_t* t1, int items, hipStream_t s) {
    using B = BlockNtt<LOGM, LOGE>;
    allow_lds<k_eval_blocks<LOGM, LOGE>>();
    k_eval_blocks<LOGM, LOGE><<<dim3(xcd_grid(tb.ell << (tb.log_n - LOGM), items)), dim3(B::T),
                                block_lds<LOGM, LOGE>(), s>>>(tb, ev, d2, t1, items);
    return hipGetLastError();
  }
};
template <int LOGM, int LOGE>
size_t km_lds() {
  using B = BlockNtt<LOGM, LOGE>;
  return LOGM <= 12 ? sizeof(double) * (B::LDS_WORDS + B::M) : block_lds<LOGM, LOGE>();
}
template <int LOGM, int LOGE>
struct ModdownKmBlocks {
  static hipError_t run(const DevTables& tb, const uint64_t* d, const uint64_t* ext1, const uint64_t* evk,
                        const uint64_t* t2, uint64_t* out, int j0, int j1, int nslots, int slot_stride, int tgt0,
                        int tgt1, int items, EvalIn ev, hipStream_t s) {
    using B = BlockNtt<LOGM, LOGE>;
    allow_lds<k_moddown_km_blocks<LOGM, LOGE>>();
    k_moddown_km_blocks<LOGM, LOGE><<<dim3(xcd_grid((tgt1 - tgt0) << (tb.log_n - LOGM), items)), dim3(B::T),
                                      km_lds<LOGM, LOGE>(), s>>>(tb, d, ext1, evk, t2, out, j0, j1, nslots,
                                                                    slot_stride, tgt0, tgt1 - tgt0, items, ev);
    return hipGetLastError();
  }
};
template <int LOGM, int LOGE>
struct KeymultPre {
  static hipError_t run(const DevTables& tb, const uint64_t* ext1, const uint64_t* evk, uint64_t* acc, int items,
                        hipStream_t s) {
    using B = BlockNtt<LOGM, LOGE>;
    allow_lds<k_keymult_pre<LOGM, LOGE>>();
    k_keymult_pre<LOGM, LOGE><<<dim3(xcd_grid(tb.k << (tb.log_n - LOGM), 2 * items)), dim3(B::T),
                                block_lds<LOGM, LOGE>(), s>>>(tb, ext1, evk, acc, 2 * items);
    return hipGetLastError();
  }
};
template <int LOGM, int LOGE>
struct ModdownPre {
  static hipError_t run(const DevTables& tb, const uint64_t* d, const uint64_t* ext1, const uint64_t* evk,
                        const uint64_t* t2, uint64_t* out, int items, EvalIn ev, hipStream_t s) {
    using B = BlockNtt<LOGM, LOGE>;
    allow_lds<k_moddown_pre<LOGM, LOGE>>();
    k_moddown_pre<LOGM, LOGE><<<dim3(xcd_grid(tb.ell << (tb.log_n - LOGM), 2 * items)), dim3(B::T),
                                block_lds<LOGM, LOGE>(), s>>>(tb, d, ext1, evk, t2, out, 2 * items, ev);
    return hipGetLastError();
  }
};
template <int LOGM, int LOGE>
struct ExtBlocks {
  static hipError_t run(const DevTables& tb, uint64_t* ext, int items, hipStream_t s) {
    using B = BlockNtt<LOGM, LOGE>;
    allow_lds<k_ext_blocks<LOGM, LOGE>>();
    k_ext_blocks<LOGM, LOGE><<<dim3(1u << (tb.log_n - LOGM), tb.nl, items * tb.ndig), dim3(B::T),
                               block_lds<LOGM, LOGE>(), s>>>(tb, ext);
    return hipGetLastError();
  }
};
template <int LOGM, int LOGE>
struct PBlocksInv {
  static hipError_t run(const DevTables& tb, const uint64_t* acc, uint64_t* accp, int items, hipStream_t s) {
    using B = BlockNtt<LOGM, LOGE>;
    allow_lds<k_pblocks_inv<LOGM, LOGE>>();
    k_pblocks_inv<LOGM, LOGE><<<dim3(1u << (tb.log_n - LOGM), tb.k, items * 2), dim3(B::T),
                                block_lds<LOGM, LOGE>(), s>>>(tb, acc, accp);
    return hipGetLastError();
  }
};

}  // namespace

// ------------------------------------------------------------ launchers

// The column kernels stage count * 2^log_r values per column in LDS (64
// columns per workgroup, 8 bytes each, at most 160 KB).
int stage_cap(int count, int log_r) { return (size_t)count * ((size_t)1 << log_r) * 64 * 8 <= 160 * 1024 ? 1 : 0; }

// What KS_PLAN_MFMA_BCONV accepts: at most 16 sources, and the digits of 64
// columns within 160 KB of LDS.
int mx_ok(const DevTables& tb, int log_r) {
  auto fits = [log_r](int nm) { return nm <= 4 && (nm << log_r) * 64 * 32 <= 160 * 1024; };
  return log_r <= 5 && fits(tb.up_nm) && fits(tb.dn_nm);
}

// Whether a column pass whose BConv has `count` sources (nm steps of four) runs it
// on the matrix cores without being asked to: wherever the kernel exists, from
// 4 sources on. The scalar products grow with the sources, the matrix form's
// folds do not: whole KeySwitch, scalar / matrix, at batch 4 and the best split,
// (8, 2^16, 16), 2 sources, 340 / 370 us; (8, 2^16, 24), 3: 476 / 482;
// (8, 2^16, 32), 4: 643 / 591; (2, 2^17, 50), one ciphertext, 25: 852 / 567.
inline bool mx_auto(int count, int nm, int log_r) {
  return count >= 4 && nm <= mx_max_nm(log_r) && mx_lds(log_r, nm) <= 160 * 1024;
}

// ks_bconv calls that stay on the scalar kernel though mx_auto holds. The matrix kernel's
// chain (scale, pack, a barrier, the constants, the folds) takes 6.1 us (4.0 from P,
// which has no P targets to fold) at the smallest sizes; the scalar one's grows with the sources and, from about 2^20
// products on, with the products. us, scalar / matrix, 4 sources: 0.5 M products 3.8 /
// 6.5, 2.1 M 6.8 / 7.1, 4.2 M 11.1 / 8.9; 8 sources: 0.5 M 5.7 / 7.1, 2.1 M 7.0 / 7.4,
// 4.2 M 10.3 / 7.8; 12 sources, up to 1.2 M, 3% apart, and 16, 10% slower; from P, 4 sources: 0.5 M
// 3.8 / 4.5, 1.05 M 4.7 / 4.7, 2.1 M 6.8 / 5.1; 6 sources, up to 0.9 M, equal; 8: 5.6 / 4.8.
// Below N = 2^8 the matrix form's columns are mostly empty: N = 2^6, 16 sources, 7.5 /
// 9.2, from P, 8 sources, 4.8 / 5.2 (and 24 sources, 12 from P, faster there too).
inline bool bconv_small(bool from_p, int ns, int log_n, long products) {
  if (from_p) return ns <= (log_n < 8 ? 8 : 6) && products <= (1L << 20);
  return ns <= (log_n < 8 ? 16 : 12) && products <= (5L << 19);
}

hipError_t launch_ntt(const DevTables& tb, int log_r, uint64_t* x, int first, int nlimbs, int items, hipStream_t s) {
  const int log_m = tb.log_n - log_r;
  hipError_t e = hipSuccess;
  if (log_r > 0) e = by_logr<ColsFwd>(log_r, tb, x, first, nlimbs, items, log_m, s);
  if (e != hipSuccess) return e;
  return by_logm<BlocksFwd>(log_m, (long)(nlimbs << log_r) * items, tb, (const uint64_t*)x, x, first, nlimbs, items,
                            log_r == 0 ? 1 : 0, s);
}

hipError_t launch_intt(const DevTables& tb, int log_r, uint64_t* x, int first, int nlimbs, int items, hipStream_t s) {
  const int log_m = tb.log_n - log_r;
  hipError_t e = by_logm<BlocksInv, true>(log_m, (long)(nlimbs << log_r) * items, tb, (const uint64_t*)x, x, first, nlimbs,
                                    items, log_r == 0 ? 1 : 0, s);
  if (e != hipSuccess || log_r == 0) return e;
  return by_logr<ColsInv>(log_r, tb, x, first, nlimbs, items, log_m, s);
}

hipError_t launch_intt_blocks(const DevTables& tb, int log_r, const uint64_t* src, uint64_t* dst, int nlimbs,
                              int items, hipStream_t s) {
  return by_logm<BlocksInv, true>(tb.log_n - log_r, (long)(nlimbs << log_r) * items, tb, src, dst, 0, nlimbs, items, 0, s);
}

hipError_t launch_eval_blocks(const DevTables& tb, int log_r, EvalIn ev, uint64_t* d2, uint64_t* t1, int items,
                              hipStream_t s) {
  return by_logm<EvalBlocks>(tb.log_n - log_r, (long)(tb.ell << log_r) * items, tb, ev, d2, t1, items, s);
}

hipError_t launch_modup_cols(const DevTables& tb, int log_r, const uint64_t* t1, uint64_t* ext1, int j0, int nj,
                             int nslots, int slot_stride, int tgt0, int tgt1, int items, int mfma, hipStream_t s) {
  if (mfma || mx_auto(tb.alpha < tb.ell ? tb.alpha : tb.ell, tb.up_nm, log_r))
    return by_logr<ModupColsMx>(log_r, tb, t1, ext1, j0, nj, nslots, slot_stride, tgt0, tgt1, items,
                                tb.log_n - log_r, s);
  return by_logr<ModupCols>(log_r, tb, t1, ext1, j0, nj, nslots, slot_stride, tgt0, tgt1, items, tb.log_n - log_r, s);
}

hipError_t launch_keymult_blocks(const DevTables& tb, int log_r, const uint64_t* d, const uint64_t* ext1,
                                 const uint64_t* evk, uint64_t* acc, int j0, int j1, int nslots, int slot_stride,
                                 int tgt0, int tgt1, int items, int accumulate, int finalize, int q_part,
                                 hipStream_t s) {
  // Without q_part only the P limbs are launched, and the latency variant pays only
  // where they leave CUs without a workgroup (128 of them, one ciphertext of
  // (4, 2^16, 32): 162 -> 157 us the call; with 384, level 13 of it, batch 3, 158 -> 163).
  const long wgs = q_part ? (long)((tgt1 - tgt0) << log_r) * items
                          : 2 * ((long)((tgt1 - (tgt0 > tb.ell ? tgt0 : tb.ell)) << log_r) * items);
  return by_logm_k3<KeymultBlocks>(tb.log_n - log_r, wgs, tb, d, ext1, evk, acc,
                                   j0, j1, nslots, slot_stride, tgt0, tgt1, items, accumulate, finalize, q_part, s);
}

hipError_t launch_moddown_km_blocks(const DevTables& tb, int log_r, const uint64_t* d, const uint64_t* ext1,
                                    const uint64_t* evk, const uint64_t* t2, uint64_t* out, int j0, int j1,
                                    int nslots, int slot_stride, int tgt0, int tgt1, int items, EvalIn ev,
                                    hipStream_t s) {
  return by_logm_k3<ModdownKmBlocks, true>(tb.log_n - log_r, (long)((tgt1 - tgt0) << log_r) * items, tb, d, ext1, evk,
                                           t2, out, j0, j1, nslots, slot_stride, tgt0, tgt1, items, ev, s);
}

hipError_t launch_moddown_cols(const DevTables& tb, int log_r, const uint64_t* accp, uint64_t* t2, int tgt0,
                               int tgt1, int items, int mfma, hipStream_t s) {
  if (mfma || mx_auto(tb.k, tb.dn_nm, log_r))
    return by_logr<ModdownColsMx>(log_r, tb, accp, t2, tgt0, tgt1, items, tb.log_n - log_r, s);
  return by_logr<ModdownCols>(log_r, tb, accp, t2, tgt0, tgt1, items, tb.log_n - log_r, s);
}

hipError_t launch_moddown_blocks(const DevTables& tb, int log_r, const uint64_t* t2, const uint64_t* acc,
                                 uint64_t* out, int tgt0, int tgt1, int items, EvalIn ev, hipStream_t s) {
  return by_logm<ModdownBlocks>(tb.log_n - log_r, (long)((tgt1 - tgt0) << log_r) * items * 2, tb, t2, acc, out, tgt0,
                                tgt1, items, ev, s);
}

hipError_t launch_ext_blocks(const DevTables& tb, int log_r, uint64_t* ext, int items, hipStream_t s) {
  return by_logm<ExtBlocks>(tb.log_n - log_r, (long)(tb.nl << log_r) * items * tb.ndig, tb, ext, items, s);
}

hipError_t launch_keymult_pre(const DevTables& tb, int log_r, const uint64_t* ext1, const uint64_t* evk,
                              uint64_t* acc, int items, hipStream_t s) {
  return by_logm<KeymultPre, true>(tb.log_n - log_r, (long)(tb.k << log_r) * items * 2, tb, ext1, evk, acc, items, s);
}

hipError_t launch_moddown_pre(const DevTables& tb, int log_r, const uint64_t* d, const uint64_t* ext1,
                              const uint64_t* evk, const uint64_t* t2, uint64_t* out, int items, EvalIn ev,
                              hipStream_t s) {
  return by_logm<ModdownPre, true>(tb.log_n - log_r, (long)(tb.ell << log_r) * items * 2, tb, d, ext1, evk, t2, out, items,
                             ev, s);
}

hipError_t launch_pblocks_inv(const DevTables& tb, int log_r, const uint64_t* acc, uint64_t* accp, int items,
                              hipStream_t s) {
  return by_logm<PBlocksInv, true>(tb.log_n - log_r, (long)(tb.k << log_r) * items * 2, tb, acc, accp, items, s);
}

hipError_t launch_copy_digits(const DevTables& tb, const uint64_t* d, uint64_t* ext, int items, hipStream_t s) {
  const unsigned n = 1u << tb.log_n;
  k_copy_digits<<<dim3((n + 255) / 256, tb.ell, items), dim3(256), 0, s>>>(tb, d, ext);
  return hipGetLastError();
}

hipError_t launch_bconv(const DevTables& tb, const uint64_t* src, int set, uint64_t* dst, int items, hipStream_t s) {
  const unsigned n = 1u << tb.log_n;
  int nd;
  if (set < 0) {
    nd = tb.ell;
  } else {
    const int lo = set * tb.alpha;
    const int hi = lo + tb.alpha < tb.ell ? lo + tb.alpha : tb.ell;
    nd = tb.nl - (hi - lo);
  }
  const int ns = tb.nl - (set < 0 ? tb.ell : nd);
  const int nm = set < 0 ? tb.dn_nm : tb.up_nm;
  const long products = (long)ns * nd * items << tb.log_n;
  if (mx_auto(ns, nm, BC_LOGR) && !bconv_small(set < 0, ns, tb.log_n, products))
    return by_nm<BconvMxN, BC_LOGR>(nm, tb, src, set, dst, items, s);
  k_bconv<<<dim3((n + 255) / 256, nd, items), dim3(256), 0, s>>>(tb, src, dst, set);
  return hipGetLastError();
}

hipError_t launch_tensor(const DevTables& tb, const uint64_t* a, const uint64_t* b, uint64_t* t01, uint64_t* d2,
                         int items, hipStream_t s) {
  const unsigned n = 1u << tb.log_n;
  k_tensor<<<dim3((n + 255) / 256, tb.ell, items), dim3(256), 0, s>>>(tb, a, b, t01, d2);
  return hipGetLastError();
}

hipError_t launch_automorph(const DevTables& tb, const uint64_t* src, uint64_t* dst, int rows, size_t src_item_stride,
                            size_t dst_item_stride, uint32_t g, int items, hipStream_t s) {
  const unsigned n = 1u << tb.log_n;
  k_automorph<<<dim3((n + 255) / 256, rows, items), dim3(256), 0, s>>>(tb.log_n, src, dst, g, src_item_stride,
                                                                       dst_item_stride);
  return hipGetLastError();
}

hipError_t launch_add_q(const DevTables& tb, uint64_t* out, const uint64_t* add, int ncomp, int items,
                        hipStream_t s) {
  const unsigned n = 1u << tb.log_n;
  k_add_q<<<dim3((n + 255) / 256, ncomp * tb.ell, items), dim3(256), 0, s>>>(tb, out, add);
  return hipGetLastError();
}

// Throughput probe of the three modular products the kernels are built
// from. Every thread runs MM_CHAINS independent chains of `iters` dependent
// products by a fixed operand (enough chains to hide the latency of one
// product), then writes the canonical sum of its chains to sink[thread]. kind 0: FP64
// product of the Q primes (f_mul); 1: product by a constant of the P primes
// (mul_shoup_lazy); 2: product of two variables of the P primes, with the fold of one of
// them that KeyMult does (p_red, p_mul).
constexpr int MM_CHAINS = MODMUL_CHAINS;

template <int KIND>
__global__ __launch_bounds__(256) void k_modmul_rate(int iters, uint64_t q, uint64_t w, uint64_t ws, uint32_t delta,
                                                     double qd, double qinv, double wd, uint64_t* sink) {
  const uint32_t tid = blockIdx.x * 256u + threadIdx.x;
  if (KIND == 0) {
    double a[MM_CHAINS];
#pragma unroll
    for (int c = 0; c < MM_CHAINS; ++c) a[c] = (double)(tid * MM_CHAINS + c + 1);
    for (int i = 0; i < iters; ++i) {
#pragma unroll
      for (int c = 0; c < MM_CHAINS; ++c) a[c] = f_mul(a[c], wd, qd, qinv);
    }
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < MM_CHAINS; ++c) acc = f_red(acc + a[c], qd, qinv);
    sink[tid] = f_canon(acc, qd, qinv);
  } else {
    uint64_t a[MM_CHAINS];
#pragma unroll
    for (int c = 0; c < MM_CHAINS; ++c) a[c] = (uint64_t)(tid * MM_CHAINS + c + 1);
    for (int i = 0; i < iters; ++i) {
#pragma unroll
      for (int c = 0; c < MM_CHAINS; ++c)
        a[c] = KIND == 1 ? mul_shoup_lazy(a[c], w, ws, ~q + 1) : p_mul(p_red(a[c], delta), w, delta);
    }
    uint64_t acc = 0;
#pragma unroll
    for (int c = 0; c < MM_CHAINS; ++c) acc = p_red(acc + p_red(a[c], delta), delta);
    sink[tid] = p_canon(acc, q, delta);
  }
}

hipError_t launch_modmul_rate(int kind, int blocks, int iters, uint64_t q, uint64_t w, uint64_t ws, uint64_t* sink,
                              hipStream_t s) {
  const double qd = (double)q, qinv = 1.0 / qd;
  // the fixed operand in balanced form for the FP64 product
  const double wd = w > q / 2 ? (double)w - qd : (double)w;
  const uint32_t delta = (uint32_t)(((uint64_t)1 << 60) - q);  // P primes
  switch (kind) {
    case 0: k_modmul_rate<0><<<dim3(blocks), dim3(256), 0, s>>>(iters, q, w, ws, delta, qd, qinv, wd, sink); break;
    case 1: k_modmul_rate<1><<<dim3(blocks), dim3(256), 0, s>>>(iters, q, w, ws, delta, qd, qinv, wd, sink); break;
    case 2: k_modmul_rate<2><<<dim3(blocks), dim3(256), 0, s>>>(iters, q, w, ws, delta, qd, qinv, wd, sink); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Input check of the debug build: flag[0] = 1 if some word of x is not a
// canonical residue of its row's prime. x holds `items` blocks of item_words
// words; row r of an item (N words at offset r * N) belongs to limb
// row_limb[r] of the extended basis (negative: a row the call does not read).
// Grid: (ceil(N / 256), rows, items).
__global__ __launch_bounds__(256) void k_check_rows(DevTables tb, const uint64_t* x, const int* row_limb,
                                                    size_t item_words, int* flag) {
  const size_t N = (size_t)1 << tb.log_n;
  const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int limb = row_limb[blockIdx.y];
  if (c >= N || limb < 0) return;
  if (x[(size_t)blockIdx.z * item_words + (size_t)blockIdx.y * N + c] >= tb.limb[limb].q) *flag = 1;
}

hipError_t launch_check_rows(const DevTables& tb, const uint64_t* x, const int* row_limb, int rows, int items,
                             size_t item_words, int* flag, hipStream_t s) {
  const unsigned n = 1u << tb.log_n;
  k_check_rows<<<dim3((n + 255) / 256, rows, items), dim3(256), 0, s>>>(tb, x, row_limb, item_words, flag);
  return hipGetLastError();
}

// HBM copy probe: dst[i] = src[i] for `words` 64-bit words, each thread
// moving 8 (kind 0) or 16 bytes (kind 1) per access with a grid-stride loop,
// stores cached or non-temporal (nt). The practical streaming ceiling of the
// access widths the kernels use.
template <int WIDE, bool NT>
__global__ __launch_bounds__(256) void k_copy_rate(const uint64_t* __restrict__ src, uint64_t* __restrict__ dst,
                                                   size_t words) {
  const size_t stride = (size_t)gridDim.x * 256;
  if (WIDE) {
    const ulonglong2* s2 = reinterpret_cast<const ulonglong2*>(src);
    ulonglong2* d2 = reinterpret_cast<ulonglong2*>(dst);
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words / 2; i += stride) {
      const ulonglong2 v = s2[i];
      if (NT) {
        __builtin_nontemporal_store(v.x, &d2[i].x);
        __builtin_nontemporal_store(v.y, &d2[i].y);
      } else {
        d2[i] = v;
      }
    }
  } else {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words; i += stride) {
      if (NT)
        __builtin_nontemporal_store(src[i], dst + i);
      else
        dst[i] = src[i];
    }
  }
}

hipError_t launch_copy_rate(int kind, int nt, int blocks, const uint64_t* src, uint64_t* dst, size_t words,
                            hipStream_t s) {
  const dim3 g(blocks), t(256);
  if (kind == 0 && !nt) k_copy_rate<0, false><<<g, t, 0, s>>>(src, dst, words);
  else if (kind == 0) k_copy_rate<0, true><<<g, t, 0, s>>>(src, dst, words);
  else if (kind == 1 && !nt) k_copy_rate<1, false><<<g, t, 0, s>>>(src, dst, words);
  else if (kind == 1) k_copy_rate<1, true><<<g, t, 0, s>>>(src, dst, words);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_keymult(const DevTables& tb, const uint64_t* ext, const uint64_t* evk, uint64_t* acc, int items,
                          hipStream_t s) {
  auto launch = [&](auto it, auto e) {
    constexpr int IT = decltype(it)::value, E = decltype(e)::value;
    const unsigned n = 1u << tb.log_n;
    k_keymult<IT, E><<<dim3((n + 256 * E - 1) / (256 * E), tb.nl, (items + IT - 1) / IT), dim3(256), 0, s>>>(
        tb, ext, evk, acc, items);
  };
  using One = std::integral_constant<int, 1>;
  using Two = std::integral_constant<int, 2>;
  // Below 3 * 2^18 coefficients of acc (at most 3 wavefronts for each SIMD with one a thread)
  // every thread counts more than a key word read twice, as long as ext (2^22 words) fits
  // the L2s. us, one coefficient / two / two for two items: (2, 2^10, 10), batch 4 (61 K),
  // 2.7 / 3.4 / 4.2; (4, 2^13, 16), batch 2 (328 K), 5.1 / 6.3 / 7.3; (2, 2^12, 10), batch 16
  // (983 K), 7.8 / 8.5 / 8.3; with 8 digits, (8, 2^13, 24), batch 3 (664 K, ext 5.3 M),
  // 19.9 / 17.6 / 17.8, and (8, 2^14, 24), batch 2 (885 K, 7.1 M), 28 / 27 / 23.
  const size_t words = (size_t)items * tb.nl << tb.log_n;
  if (words < ((size_t)3 << 18) && words * tb.ndig < ((size_t)1 << 22))
    launch(One{}, One{});
  else if (items == 1)
    launch(One{}, Two{});
  else
    launch(Two{}, Two{});
  return hipGetLastError();
}

}  // namespace ks
