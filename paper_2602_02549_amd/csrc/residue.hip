// INT8 operand slices for the matrix-core products, written K-major
// (k contiguous per row of A, per column of B) and zero-padded to
// [rows_pad][k_pad]:
//   mode 0: Abar = ceil(diag(2^mu') |A|)            (Algorithm 2)
//   mode 1: A'_l = mod(trunc(diag(2^mu) A), p_l)     (Algorithms 2-3)
//
// A block stages a 32-row x 128-k tile of the FP64/FP32 source through LDS:
// the column-major A (rows contiguous) and the column-major B (k contiguous)
// are both read coalesced, then each thread owns 16 consecutive k of one row
// and writes 16 bytes per slice, 8 threads covering one full 128-byte line.
// The LDS rows are 132 doubles apart and the low bits of each column index
// XOR-swizzled, so that the staging stores and the in-order reads
// of a wave spread evenly over 64 four-byte banks, and no thread indexes its
// registers with a per-lane value.
// Each workgroup walks tiles in a grid-stride loop and issues the loads of
// its next tile before computing the current one.
//
// Residues of the scaled integer v = trunc(2^mu a) (|v| < 2^B, B = 6 + floor P')
// are exact in FP64.  v is split once per element into limbs, and per modulus
// r = sum_t v_t c_t with c_0 = 1, c_t = mod(2^(s t), p), |c_t| <= 127, is
// exact and below 2^50; one step r <- r - p * round(r / p) then lands in
// [-(p-1)/2, (p-1)/2] for odd p.
//   two limbs (B <= 90, N = 12..22): v = v_1 2^48 + v_0, |v_0| <= 2^47,
//     |v_1| <= 2^42, so |r| <= 2^47 + 127 * 2^42 < 2^49.4;
//   three limbs (B <= 122, N = 23..31): v = v_2 2^80 + v_1 2^40 + v_0,
//     |v_0|, |v_1| <= 2^39, |v_2| <= 2^42, so |r| <= 128 * 2^39 + 127 * 2^42
//     < 2^49.2.
// Other N take nsteps such steps from v itself (each exact, shrinking |r| by
// ~2^-52 relative; the last starts from |r| < 2^50).  For p = 256 the result
// lies in [-128, 128] and the byte store wraps 128 to -128; 2^48, 2^40 and
// 2^80 are 0 mod 256.
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <type_traits>

#include "ozaki2_internal.h"
#include "small_mod.h"

namespace oz2 {
namespace {

constexpr int kTR = 32;           // slice tile: rows
constexpr int kTK = 128;          // slice tile: k
constexpr int kRS = kTK + 4;      // LDS row stride (doubles)
constexpr int kPlanTile = 64;     // planner operand tile

__device__ __forceinline__ double round_prod(double x, double y) {
  return fma(x, y, kRound) - kRound;
}

// The low 32 bits, in two's complement, of an integer-valued |x| < 2^51.
__device__ __forceinline__ uint32_t low32(double x) {
  return (uint32_t)__double2loint(x + kRound);
}

// Low bytes of a, b, c, d as one word (byte 0 = a), three byte permutes:
// v_perm_b32 picks bytes 0-3 of its second source with selectors 0-3, of its
// first with 4-7, and zero with 0x0c.
__device__ __forceinline__ uint32_t pack4(int a, int b, int c, int d) {
  const uint32_t ab = __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0c0c0400u);
  const uint32_t cd = __builtin_amdgcn_perm((uint32_t)d, (uint32_t)c, 0x0c0c0400u);
  return __builtin_amdgcn_perm(cd, ab, 0x05040100u);
}

// Residue paths of mode 1: limbs (2 or 3) or exact reduction steps (1, 3 or
// 4; the limbs cover every N that would take two steps, and an extra step is
// exact anyway); kAnyPath chooses at run time from the constants (grouped
// launches, whose problems differ in N).
enum ResiduePath { kLimbs2, kLimbs3, kSteps1, kSteps3, kSteps4, kAnyPath };

// The constants of one modulus; 2^-40 (three limbs) or 2^-48 as a scalar that
// the compiler takes for another value for each modulus, so that the mid limbs
// computed from it are not kept in registers across the moduli.
struct Modulus : ModConst {
  double minv = 0.0;
  __device__ __forceinline__ explicit Modulus(const ModConst& m) : ModConst(m) {}
  __device__ __forceinline__ void forget(double mid_inv) {
    minv = mid_inv;
    __asm__ volatile("" : "+s"(minv));
  }
};

// Calls f(l, modulus l) for this workgroup's moduli; the next modulus'
// constants are loaded while f works on this one's.  The workgroups of grid
// row y of Y take moduli [y N / Y, (y + 1) N / Y): when a launch has too few
// tiles to occupy the GPU, several workgroups share a tile.
template <typename F>
__device__ __forceinline__ void for_moduli(const CrtConsts& cc, F&& f) {
  const int y = (int)blockIdx.y, parts = (int)gridDim.y;
  const int l0 = y * cc.N / parts, l1 = (y + 1) * cc.N / parts;
  ModConst next = cc.mod[l0];
  for (int l = l0; l < l1; ++l) {
    const Modulus md(next);
    next = cc.mod[min(l + 1, kMaxModuli - 1)];
    f(l, md);
  }
}

// M scaled integers v, |v| < 2^B, prepared for their residues on one path.
// Only the rounded quotient needs FP64: q = round(r / p) of the limb sum
// r = hi c2 + mid c1 + lo, |r| < 2^50 (exact), comes out of one fma with
// kRound (its low bits are q; the rounded product is the nearest integer to
// r / p itself, because |r| |pinv - 1/p| <= 2^-3 / p is below the distance
// 1 / (2p) from r / p to a half-integer for odd p, and pinv is exact for
// p = 256).  The residue r - q p, which lies in [-(p-1)/2, (p-1)/2] for odd p
// and in [-128, 128] for p = 256, is then formed mod 2^16 from the low 16
// bits of the limbs and of q, two elements per packed instruction.
// KEEP: the limbs stay in registers, and an element and modulus cost 2 FP64
// instructions (3 for three limbs, 1 for one step).  Otherwise (the complex
// forms, with twice the elements) the mid limbs are formed again for each
// modulus, through mid c1 + lo = w + mid (c1 - 2^48), w = mid 2^48 + lo: 4
// FP64 (5).  Either way 1 packed
// (1.5, 0.5) and 0.75 permute instructions follow.  Forming r - q p in FP64
// and reading its low word took 5 (6, 4) FP64 with the limbs kept and 8 (12)
// without.  At 2048^3 (N = 14) a side's residues went from 23.7 to 20.0 us, at
// 4096^3 (N = 18) from 103 to 91 us, at 8192^3 (N = 14), where the pass runs
// at the copy rate, from 301 to 289 us.
template <int PATH, int M, bool KEEP>
struct Scaled {
  static constexpr bool kLimbs = PATH == kLimbs2 || PATH == kLimbs3;
  static constexpr bool k3 = PATH == kLimbs3;
  static constexpr bool kOne = kLimbs || PATH == kSteps1;   // r needs no earlier step
  static constexpr double kS = k3 ? 0x1p40 : 0x1p48, kSinv = k3 ? 0x1p-40 : 0x1p-48;
  // KEEP: lo; otherwise mid kS + lo
  double lo[M], mid[kLimbs && KEEP ? M : 1], hi[k3 ? M : 1];
  uint32_t lo16[kOne ? M / 2 : 1], mid16[kLimbs ? M / 2 : 1], hi16[k3 ? M / 2 : 1];

  __device__ __forceinline__ explicit Scaled(const double (&v)[M]) {
#pragma unroll
    for (int e = 0; e < M; e += 2) {
      uint32_t lw[2], mw[2], hw[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        double rem = v[e + u];
        if constexpr (k3) {
          const double t = fma(rem, 0x1p-80, kRound);   // |v| < 2^122: |hi| <= 2^42
          hw[u] = (uint32_t)__double2loint(t);
          hi[e + u] = t - kRound;
          rem = fma(-hi[e + u], 0x1p80, rem);           // exact, |rem| <= 2^79
        }
        if constexpr (kLimbs) {
          lo[e + u] = rem;
          const double t = fma(rem, kSinv, kRound);
          mw[u] = (uint32_t)__double2loint(t);
          if constexpr (KEEP) mid[e + u] = t - kRound;
          rem = fma(-(t - kRound), kS, rem);            // exact, <= 2^47 (2), 2^39 (3)
        }
        if constexpr (KEEP || !kLimbs) lo[e + u] = rem;
        if constexpr (kOne) lw[u] = low32(rem);
      }
      if constexpr (kOne) lo16[e / 2] = pair16(lw[0], lw[1]);
      if constexpr (kLimbs) mid16[e / 2] = pair16(mw[0], mw[1]);
      if constexpr (k3) hi16[e / 2] = pair16(hw[0], hw[1]);
    }
  }

  // Residues of elements 2e and 2e + 1 as signed 16-bit halves.
  __device__ __forceinline__ uint32_t pair(int e, const Modulus& md) const {
    if constexpr (kOne) {
      double q[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        double r = lo[2 * e + u];
        if constexpr (KEEP) {
          if constexpr (kLimbs) r = fma(mid[2 * e + u], md.c1, r);
          if constexpr (k3) r = fma(hi[2 * e + u], md.c2, r);
        } else {
          if constexpr (kLimbs) r = fma(round_prod(r, md.minv), md.c1 - kS, r);
          if constexpr (k3) r = fma(hi[2 * e + u], md.c2, r);
        }
        q[u] = fma(r, md.pinv, kRound);
      }
      uint32_t x = lo16[e];
      if constexpr (kLimbs) x = pk_mad(mid16[e], md.c1p, x);
      if constexpr (k3) x = pk_mad(hi16[e], md.c2p, x);
      return pk_mad(pair16(__double2loint(q[0]), __double2loint(q[1])), md.negp, x);
    } else {
      // Two (three) earlier steps only shrink |r| exactly, for which rint of
      // the rounded product suffices; the last starts from |r| < 2^50.
      uint32_t q[2], w[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        double r = lo[2 * e + u];
#pragma unroll
        for (int s = 0; s < (PATH == kSteps3 ? 2 : 3); ++s) r = fma(-rint(r * md.pinv), (double)md.p, r);
        q[u] = (uint32_t)__double2loint(fma(r, md.pinv, kRound));
        w[u] = low32(r);
      }
      return pk_mad(pair16(q[0], q[1]), md.negp, pair16(w[0], w[1]));
    }
  }

  // The residue bytes of elements 4q .. 4q + 3.
  __device__ __forceinline__ uint32_t word(int q, const Modulus& md) const {
    return bytes_of_pairs(pair(2 * q, md), pair(2 * q + 1, md));
  }
  __device__ __forceinline__ uint4 words(const Modulus& md) const {
    static_assert(M == 16, "16 bytes");
    return make_uint4(word(0, md), word(1, md), word(2, md), word(3, md));
  }
};

// The N residue bytes of 16 consecutive k of one row, one 16-byte store per
// modulus.  (8 k of two rows per thread, with 116 registers and 4 workgroups
// per CU against 164 and 3, walks the moduli twice: 22 us against 20 us a
// side at 2048^3, 299 against 287 us at 8192^3.)
template <int PATH>
__device__ __forceinline__ void store_residues(const double (&v)[16], const CrtConsts& cc,
                                               int8_t* __restrict__ dst, size_t slice) {
  const Scaled<PATH, 16, true> x(v);
  for_moduli(cc, [&](int l, const Modulus& md) {
    *reinterpret_cast<uint4*>(dst + (size_t)l * slice) = x.words(md);
  });
}

// Workgroup barrier for the LDS tile only: it waits for this wave's LDS
// (and scalar) traffic, not for its global loads, so the next tile's loads
// stay in flight across it.  The memory clobber keeps the compiler from
// moving memory accesses across it.
__device__ __forceinline__ void lds_barrier() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The 16 source elements of one thread for the tile at rows r0.., k h0..;
// all 16 loads go out before any is used.  Addresses are clamped into the
// matrix (rows, k >= 1); out-of-range elements are zeroed when staged.
template <typename T, bool TRANS>
__device__ __forceinline__ void tile_loads(const T* __restrict__ src, int ld, int rows, int k,
                                           int r0, int h0, T (&x)[16]) {
  const int t = threadIdx.x;
  if (TRANS) {  // src[r + h*ld]: 32 consecutive rows per half-wave, two columns per wave
    const T* a = src + min(r0 + (t & 31), rows - 1);
    const int hb = h0 + (t >> 5);
#pragma unroll
    for (int q = 0; q < 16; ++q) x[q] = a[(size_t)min(hb + 8 * q, k - 1) * ld];
  } else {      // src[h + r*ld]: 128 consecutive k per half-block
    const T* a = src + min(h0 + (t & 127), k - 1);
    const int rb = r0 + (t >> 7);
#pragma unroll
    for (int q = 0; q < 16; ++q) x[q] = a[(size_t)min(rb + 2 * q, rows - 1) * ld];
  }
}

// One operand of a slice launch.
struct SliceSide {
  const void* src;
  const uint64_t* bits;   // abs-max bit patterns of the rows
  const int* mx;          // mode 1: maxima of Cbar over the rows
  int* shift;             // mode 1: where the rows' shifts (mu, nu) go
  int8_t* out;
  size_t slice;           // bytes from one slice to the next
  int ld, rows, gy;       // gy: row tiles
  int tiles, blocks;      // tiles, and the workgroups that walk them
};
struct SliceArgs {
  SliceSide a, b;         // A (column-major) and B (k contiguous)
  int k, k_pad;           // k_pad: padded k (the embedding: of one k half)
  int half;               // the embedding: rows of one row half on the A side
  int bias;               // added to mu' and nu' of nonzero rows (mode 1)
  int* flag;              // set by a non-finite row (mode 1)
};

// The shift of a row, stored once for the CRT, and the non-finite flag.
struct RowResult {
  int sh;
  bool bad;
  __device__ __forceinline__ void store(int* __restrict__ shift, int rg,
                                        int* __restrict__ flag) const {
    shift[rg] = sh;
    if (bad) *flag = 1;
  }
};

// Shift of the thread's output row rg (clamped): mu' from the abs-max bit
// pattern (mode 0; mode 2: mu' - 1), or mu / nu from the pattern and the
// maximum of Cbar (mode 1: Algorithm 2's shift, from the table of its steps).
// The inputs are loaded early (load) and used later (get).
template <int MODE>
struct RowShift {
  uint64_t bits;
  int mx;
  __device__ __forceinline__ void load(const uint64_t* __restrict__ b, const int* __restrict__ m,
                                       int rows, int rg) {
    rg = min(rg, rows - 1);
    bits = b[rg];
    mx = MODE == 1 ? m[rg] : 0;
  }
  __device__ __forceinline__ RowResult get(const CrtConsts& cc, int bias) const {
    if (MODE == 1) return {shift_of(bits, mx, cc, bias), nonfinite_bits(bits)};
    return {shift_prime_bits(bits) - (MODE == 2 ? 1 : 0), false};
  }
};

// LDS position of element (r, h) of a tile:
//   r * kRS + (h ^ (((h / 32) ^ (r / 8)) & 3)),
// rows kRS doubles apart and the low two bits of h XORed with bits of h / 32
// and r / 8.  Counted over 64 four-byte banks, both staging patterns and the
// in-order reads of tile_finish put exactly two of a wave's 8-byte accesses
// on each bank.  tile_stage and tile_finish address it as four base
// addresses plus constant offsets (the XOR term is constant within each
// group of four steps).

// Writes the thread's 16 elements into the LDS tile (zero outside the matrix).
// Within each group of four steps q the XOR term of the position map is constant
// (h / 32 and r / 8 depend on q / 4 only), so the positions are four bases
// plus constant offsets.
template <typename T, bool TRANS>
__device__ __forceinline__ void tile_stage(const T (&x)[16], int rows, int k, int r0, int h0,
                                           double* tile) {
  const int t = threadIdx.x;
  if (TRANS) {  // element (r, h = hb + 8q): position r*kRS + 8q + (hb ^ ((q/4 ^ r/8) & 3))
    const int r = t & 31, rg = r0 + r, hb = t >> 5;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      double* base = tile + r * kRS + (hb ^ ((j ^ (r >> 3)) & 3));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q = 4 * j + i, h = hb + 8 * q;
        base[8 * q] = (rg < rows && h0 + h < k) ? (double)x[q] : 0.0;
      }
    }
  } else {      // element (r = 2q + t/128, h): position r*kRS + (h ^ ((h/32 ^ q/4) & 3))
    const int h = t & 127, hg = h0 + h, rb = t >> 7;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      double* base = tile + rb * kRS + (h ^ (((h >> 5) ^ j) & 3));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q = 4 * j + i, rg = r0 + 2 * q + rb;
        base[2 * q * kRS] = (rg < rows && hg < k) ? (double)x[q] : 0.0;
      }
    }
  }
}

int residue_path(const CrtConsts& cc) {
  if (cc.nlimbs == 2) return kLimbs2;
  if (cc.nlimbs == 3) return kLimbs3;
  return cc.nsteps <= 1 ? kSteps1 : cc.nsteps <= 3 ? kSteps3 : kSteps4;
}

template <int PATH>
__device__ __forceinline__ void store_residues_path(const double (&v)[16], const CrtConsts& cc,
                                                    int8_t* __restrict__ dst, size_t slice) {
  if constexpr (PATH != kAnyPath) {
    store_residues<PATH>(v, cc, dst, slice);
  } else if (cc.nlimbs == 2) {          // uniform branches
    store_residues<kLimbs2>(v, cc, dst, slice);
  } else if (cc.nlimbs == 3) {
    store_residues<kLimbs3>(v, cc, dst, slice);
  } else if (cc.nsteps <= 1) {
    store_residues<kSteps1>(v, cc, dst, slice);
  } else if (cc.nsteps <= 3) {
    store_residues<kSteps3>(v, cc, dst, slice);
  } else {
    store_residues<kSteps4>(v, cc, dst, slice);
  }
}

// Each thread reads 16 consecutive k of one row from the staged tile and
// writes 16 bytes per slice (mode 0: Abar; mode 1: the N residues).
template <int MODE, int PATH>
__device__ __forceinline__ void tile_finish(const double* tile, RowResult row,
                                            int* __restrict__ shift_out, int* __restrict__ flag,
                                            int rows, int k_pad, size_t slice, const CrtConsts& cc,
                                            int8_t* __restrict__ out, int r0, int h0) {
  const int sh = row.sh;
  const int t = threadIdx.x;
  const int r = t >> 3, c = t & 7, rg = r0 + r;
  // element (r, 16c + e): position r*kRS + 16c + 4(e/4) + ((e%4) ^ g)
  const int g = ((c >> 1) ^ (r >> 3)) & 3;
  double v[16];
#pragma unroll
  for (int el = 0; el < 4; ++el) {
    const double* base = tile + r * kRS + 16 * c + (el ^ g);
#pragma unroll
    for (int eh = 0; eh < 4; ++eh) v[4 * eh + el] = base[4 * eh];
  }
  int8_t* dst = out + (size_t)rg * k_pad + h0 + 16 * c;

  if (MODE != 1) {
    int b[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      double x = fabs(v[e]);
      double cl = ceil(ldexp(x, sh));
      b[e] = x == 0.0 ? 0 : (cl < 1.0 ? 1 : (int)cl);
    }
    uint4 w;
    w.x = pack4(b[0], b[1], b[2], b[3]);
    w.y = pack4(b[4], b[5], b[6], b[7]);
    w.z = pack4(b[8], b[9], b[10], b[11]);
    w.w = pack4(b[12], b[13], b[14], b[15]);
    *reinterpret_cast<uint4*>(dst) = w;
  } else if (rg < rows) {
    if (h0 == 0 && c == 0 && blockIdx.y == 0) row.store(shift_out, rg, flag);
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = trunc(ldexp(v[e], sh));
    store_residues_path<PATH>(v, cc, dst, slice);
  }
}

// Tile b of an operand with gy row tiles of 32: for the column-major A side
// (TRANS) row tiles vary fastest, so workgroups running together read
// neighbouring 256-byte pieces of the same columns (DRAM pages); for B, whose
// rows are contiguous in k, k tiles vary fastest.
template <bool TRANS>
__device__ inline void slice_tile(int b, int k_pad, int gy, int* kx, int* ry) {
  if (TRANS) {
    *kx = b / gy;
    *ry = b % gy;
  } else {
    const int gx = k_pad / kTK;
    *kx = b % gx;
    *ry = b / gx;
  }
}

// Workgroup `w` of the s.blocks that walk one operand's tiles in a stride
// (mode 1 leaves out the tiles of padding rows, whose residues no product of
// real rows reads; Abar and Bbar padding must stay zero, since the scaling
// product's maxima cover whole rows and columns).  Each workgroup stages tile
// i in LDS, issues the loads of its next tile, and only then computes and
// stores tile i, so that HBM reads overlap the residue arithmetic.
template <typename T, bool TRANS, int MODE, int PATH>
__device__ __forceinline__ void walk_real(const SliceArgs& a, const SliceSide& s, int w,
                                          const CrtConsts& cc, double* tile) {
  int i = w;
  if (i >= s.tiles) return;
  const T* src = static_cast<const T*>(s.src);
  const int row = (int)(threadIdx.x >> 3);
  int kx, ry;
  slice_tile<TRANS>(i, a.k_pad, s.gy, &kx, &ry);
  T x[16];
  tile_loads<T, TRANS>(src, s.ld, s.rows, a.k, ry * kTR, kx * kTK, x);
  RowShift<MODE> rs;
  rs.load(s.bits, s.mx, s.rows, ry * kTR + row);
  for (;;) {
    const int r0 = ry * kTR, h0 = kx * kTK;
    lds_barrier();                 // every wave is done with the previous tile
    tile_stage<T, TRANS>(x, s.rows, a.k, r0, h0, tile);
    __asm__ volatile("" ::: "memory");  // x is free: the next loads reuse its registers
    const RowResult rr = rs.get(cc, a.bias);
    const int ni = i + s.blocks;
    if (ni < s.tiles) {
      slice_tile<TRANS>(ni, a.k_pad, s.gy, &kx, &ry);
      tile_loads<T, TRANS>(src, s.ld, s.rows, a.k, ry * kTR, kx * kTK, x);
      rs.load(s.bits, s.mx, s.rows, ry * kTR + row);
    }
    lds_barrier();                 // the tile is staged
    tile_finish<MODE, PATH>(tile, rr, s.shift, a.flag, s.rows, a.k_pad, s.slice, cc, s.out, r0, h0);
    if (ni >= s.tiles) break;
    i = ni;
  }
}

// ---- complex operands of the 3-product form (ozaki2_zgemm3m) -------------
// The source holds interleaved (re, im) pairs, column-major, ld in complex
// elements.  Both parts of a tile are loaded together (the complex matrix is
// read once per pass) and staged one after the other through the one LDS
// tile of k_slices, each thread taking its 16 values of each part into
// registers:
//   mode 2: Abar of the complex rows, ceil(2^(mu'-1) |re|) + ceil(2^(mu'-1) |im|)
//     (each at most 32), one slice at out;
//   mode 1: the residues of A'r, A'i and A'r + A'i, N slices each, at out,
//     out + N slice and out + 2 N slice.  Per modulus the residues of the two
//     parts come from the residue path's arithmetic, and the third is their
//     sum brought back into the symmetric range by one correction.

// The residues of the sums of two pairs of residues: each in [-(p-1)/2,
// (p-1)/2] (odd p) or [-128, 128] (p = 256, bytes mod 256), so with lo =
// -(p-1)/2 (-128) the sum less lo, u, lies in (-p, 2p), and the smallest of
// u, u + p and u - p as unsigned 16-bit values is the one in [0, p).
__device__ __forceinline__ uint32_t pair_sum(uint32_t a, uint32_t b, int p) {
  const int lo = (p - 1) / 2 + 1 - p;
  const uint32_t u = pk_add(pk_add(a, b), both16(-lo));
  const uint32_t w = pk_min(pk_min(u, pk_add(u, both16(p))), pk_add(u, both16(-p)));
  return pk_add(w, both16(lo));
}

// The thread's 16 staged elements of its row (the order of tile_finish).
__device__ __forceinline__ void tile_row16(const double* tile, double (&v)[16]) {
  const int t = threadIdx.x;
  const int r = t >> 3, c = t & 7;
  const int g = ((c >> 1) ^ (r >> 3)) & 3;
#pragma unroll
  for (int el = 0; el < 4; ++el) {
    const double* base = tile + r * kRS + 16 * c + (el ^ g);
#pragma unroll
    for (int eh = 0; eh < 4; ++eh) v[4 * eh + el] = base[4 * eh];
  }
}

template <int MODE, int PATH>
__device__ __forceinline__ void tile_finish_cx(double (&vr)[16], double (&vi)[16], RowResult row,
                                               int* __restrict__ shift_out, int* __restrict__ flag,
                                               int rows, int k_pad, size_t slice,
                                               const CrtConsts& cc, int8_t* __restrict__ out,
                                               int r0, int h0) {
  const int sh = row.sh;
  const int t = threadIdx.x;
  const int rg = r0 + (t >> 3);
  int8_t* dst = out + (size_t)rg * k_pad + h0 + 16 * (t & 7);
  if constexpr (MODE == 2) {
    auto bar = [&](double v) {
      const double x = fabs(v);
      const double cl = ceil(ldexp(x, sh));
      return x == 0.0 ? 0 : (cl < 1.0 ? 1 : (int)cl);
    };
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      w[q] = pack4(bar(vr[4 * q]) + bar(vi[4 * q]), bar(vr[4 * q + 1]) + bar(vi[4 * q + 1]),
                   bar(vr[4 * q + 2]) + bar(vi[4 * q + 2]), bar(vr[4 * q + 3]) + bar(vi[4 * q + 3]));
    *reinterpret_cast<uint4*>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
  } else {
    if (rg >= rows) return;
    if (h0 == 0 && (t & 7) == 0 && blockIdx.y == 0) row.store(shift_out, rg, flag);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      vr[e] = trunc(ldexp(vr[e], sh));
      vi[e] = trunc(ldexp(vi[e], sh));
    }
    const size_t set = (size_t)cc.N * slice;
    const Scaled<PATH, 16, false> xr(vr), xi(vi);
    for_moduli(cc, [&](int l, Modulus md) {
      md.forget(decltype(xr)::kSinv);
      const int p = md.p;
      uint32_t wr[4], wi[4], ws[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t r0p = xr.pair(2 * q, md), r1p = xr.pair(2 * q + 1, md);
        const uint32_t i0p = xi.pair(2 * q, md), i1p = xi.pair(2 * q + 1, md);
        wr[q] = bytes_of_pairs(r0p, r1p);
        wi[q] = bytes_of_pairs(i0p, i1p);
        ws[q] = bytes_of_pairs(pair_sum(r0p, i0p, p), pair_sum(r1p, i1p, p));
      }
      int8_t* d = dst + (size_t)l * slice;
      *reinterpret_cast<uint4*>(d) = make_uint4(wr[0], wr[1], wr[2], wr[3]);
      *reinterpret_cast<uint4*>(d + set) = make_uint4(wi[0], wi[1], wi[2], wi[3]);
      *reinterpret_cast<uint4*>(d + 2 * set) = make_uint4(ws[0], ws[1], ws[2], ws[3]);
    });
  }
}

template <typename T, bool TRANS>
__device__ __forceinline__ void tile_loads_cx(const T* __restrict__ src, int ld, int rows, int k,
                                              int r0, int h0, T (&x)[16], T (&y)[16]) {
  const int t = threadIdx.x;
  if (TRANS) {  // element (r, h) at src[2 (r + h ld)]: as tile_loads, pairs
    const T* a = src + 2 * (size_t)min(r0 + (t & 31), rows - 1);
    const int hb = h0 + (t >> 5);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const T* e = a + 2 * ((size_t)min(hb + 8 * q, k - 1) * ld);
      x[q] = e[0];
      y[q] = e[1];
    }
  } else {      // element (h, r) at src[2 (h + r ld)]
    const T* a = src + 2 * (size_t)min(h0 + (t & 127), k - 1);
    const int rb = r0 + (t >> 7);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const T* e = a + 2 * ((size_t)min(rb + 2 * q, rows - 1) * ld);
      x[q] = e[0];
      y[q] = e[1];
    }
  }
}

// The walk over complex tiles: the real parts are staged and read back, then
// the imaginary parts, then the next tile's loads go out before the
// arithmetic of this one.
template <typename T, bool TRANS, int MODE, int PATH>
__device__ __forceinline__ void walk_cx(const SliceArgs& a, const SliceSide& s, int w,
                                        const CrtConsts& cc, double* tile) {
  int i = w;
  if (i >= s.tiles) return;
  const T* src = static_cast<const T*>(s.src);
  const int row = (int)(threadIdx.x >> 3);
  int kx, ry;
  slice_tile<TRANS>(i, a.k_pad, s.gy, &kx, &ry);
  // The next tile's loads go out early only for the residues, and not for the
  // three-limb ones, which hold too many registers for it (two workgroups a CU
  // instead of one); the bars run four workgroups a CU without.
  constexpr bool kPrefetch = MODE == 1 && PATH != kLimbs3;
  T x[16], y[16];
  if (kPrefetch) tile_loads_cx<T, TRANS>(src, s.ld, s.rows, a.k, ry * kTR, kx * kTK, x, y);
  RowShift<MODE> rs;
  rs.load(s.bits, s.mx, s.rows, ry * kTR + row);
  for (;;) {
    const int r0 = ry * kTR, h0 = kx * kTK;
    double vr[16], vi[16];
    if (!kPrefetch) tile_loads_cx<T, TRANS>(src, s.ld, s.rows, a.k, r0, h0, x, y);
    lds_barrier();                 // every wave is done with the previous tile
    tile_stage<T, TRANS>(x, s.rows, a.k, r0, h0, tile);
    lds_barrier();
    tile_row16(tile, vr);
    lds_barrier();
    tile_stage<T, TRANS>(y, s.rows, a.k, r0, h0, tile);
    __asm__ volatile("" ::: "memory");  // x, y are free: the next loads reuse their registers
    const RowResult rr = rs.get(cc, a.bias);
    const int ni = i + s.blocks;
    if (ni < s.tiles) {
      slice_tile<TRANS>(ni, a.k_pad, s.gy, &kx, &ry);
      if (kPrefetch) tile_loads_cx<T, TRANS>(src, s.ld, s.rows, a.k, ry * kTR, kx * kTK, x, y);
      rs.load(s.bits, s.mx, s.rows, ry * kTR + row);
    }
    lds_barrier();
    tile_row16(tile, vi);
    tile_finish_cx<MODE, PATH>(vr, vi, rr, s.shift, a.flag, s.rows, a.k_pad, s.slice, cc, s.out, r0,
                               h0);
    if (ni >= s.tiles) break;
    i = ni;
  }
}

// ---- the real embedding of a complex product (ozaki2_zgemm) --------------
// Ahat = [[Ar, -Ai], [Ai, Ar]] and Bhat = [[Br], [Bi]] written as slices
// straight from the interleaved complex source: k-half kh (slice rows 2 kh
// long), and on the A side row half `half`.  A complex element (i, h) of A
// lands in Ahat at (i, h) as re, (i, kh + h) as -im, (half + i, h) as im and
// (half + i, kh + h) as re; of B at row j of Bhat^T: (j, h) re, (j, kh + h) im.
//   mode 0: the bars; rows i and half + i share mu'_i (the same maximum).
//   mode 1: the residues; row i is scaled by shift[i], row half + i by
//     shift[half + i] (their Cbar maxima differ).
template <int MODE, int PATH, bool ASIDE>
__device__ __forceinline__ void tile_finish_emb(const double (&vr)[16], const double (&vi)[16],
                                                const SliceArgs& a, const SliceSide& s,
                                                const CrtConsts& cc, int r0, int h0) {
  const int t = threadIdx.x;
  const int rg = r0 + (t >> 3);
  const int rows = s.rows, kh = a.k_pad, ldo = 2 * kh, half = a.half;
  const size_t slice = s.slice;
  int8_t* __restrict__ out = s.out;
  int8_t* d0 = out + (size_t)rg * ldo + h0 + 16 * (t & 7);    // (rg, h)
  int8_t* d1 = d0 + kh;                                         // (rg, kh + h)
  const size_t dh = (size_t)half * ldo;                         // to row half + rg
  if constexpr (MODE == 0) {
    const int sh = shift_prime_bits(s.bits[min(rg, rows - 1)]);
    auto bar = [&](double v) {
      const double x = fabs(v);
      const double cl = ceil(ldexp(x, sh));
      return x == 0.0 ? 0 : (cl < 1.0 ? 1 : (int)cl);
    };
    uint32_t wr[4], wi[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      wr[q] = pack4(bar(vr[4 * q]), bar(vr[4 * q + 1]), bar(vr[4 * q + 2]), bar(vr[4 * q + 3]));
      wi[q] = pack4(bar(vi[4 * q]), bar(vi[4 * q + 1]), bar(vi[4 * q + 2]), bar(vi[4 * q + 3]));
    }
    const uint4 ur = make_uint4(wr[0], wr[1], wr[2], wr[3]), ui = make_uint4(wi[0], wi[1], wi[2], wi[3]);
    *reinterpret_cast<uint4*>(d0) = ur;
    *reinterpret_cast<uint4*>(d1) = ui;
    if (ASIDE) {
      *reinterpret_cast<uint4*>(d0 + dh) = ui;
      *reinterpret_cast<uint4*>(d1 + dh) = ur;
    }
  } else {
    if (rg >= rows) return;
    // block 0: rows rg (A side) or the only row (B side); block 1: row half + rg
    for (int blk = 0; blk < (ASIDE ? 2 : 1); ++blk) {
      const int ro = rg + blk * half;
      const int e2 = shift_of(s.bits[ro], s.mx[ro], cc, a.bias);
      if (h0 == 0 && (t & 7) == 0 && blockIdx.y == 0)
        RowResult{e2, nonfinite_bits(s.bits[ro])}.store(s.shift, ro, a.flag);
      double xr[16], xi[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        xr[e] = trunc(ldexp(vr[e], e2));
        xi[e] = trunc(ldexp(vi[e], e2));
      }
      // A side: row rg holds [re, -im], row half + rg [im, re]; B side [re, im]
      int8_t* br = (ASIDE && blk == 1 ? d1 : d0) + blk * dh;
      int8_t* bi = (ASIDE && blk == 1 ? d0 : d1) + blk * dh;
      if (ASIDE && blk == 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) xi[e] = -xi[e];
      }
      const Scaled<PATH, 16, PATH != kLimbs3> sr(xr), si(xi);
      for_moduli(cc, [&](int l, Modulus md) {
        md.forget(decltype(sr)::kSinv);
        *reinterpret_cast<uint4*>(br + (size_t)l * slice) = sr.words(md);
        *reinterpret_cast<uint4*>(bi + (size_t)l * slice) = si.words(md);
      });
    }
  }
}

// The walk of walk_cx over the complex source's tiles (kh / 128 k tiles by gy
// row tiles), without early loads: the residues hold both parts' limbs (on the
// A side for two row blocks), and only without them do two workgroups share a
// CU.
template <typename T, bool TRANS, int MODE, int PATH>
__device__ __forceinline__ void walk_emb(const SliceArgs& a, const SliceSide& s, int w,
                                         const CrtConsts& cc, double* tile) {
  int i = w;
  if (i >= s.tiles) return;
  const T* src = static_cast<const T*>(s.src);
  int kx, ry;
  slice_tile<TRANS>(i, a.k_pad, s.gy, &kx, &ry);
  T x[16], y[16];
  for (;;) {
    const int r0 = ry * kTR, h0 = kx * kTK;
    double vr[16], vi[16];
    tile_loads_cx<T, TRANS>(src, s.ld, s.rows, a.k, r0, h0, x, y);
    lds_barrier();                 // every wave is done with the previous tile
    tile_stage<T, TRANS>(x, s.rows, a.k, r0, h0, tile);
    lds_barrier();
    tile_row16(tile, vr);
    lds_barrier();
    tile_stage<T, TRANS>(y, s.rows, a.k, r0, h0, tile);
    const int ni = i + s.blocks;
    if (ni < s.tiles) slice_tile<TRANS>(ni, a.k_pad, s.gy, &kx, &ry);
    lds_barrier();
    tile_row16(tile, vi);
    tile_finish_emb<MODE, PATH, TRANS>(vr, vi, a, s, cc, r0, h0);
    if (ni >= s.tiles) break;
    i = ni;
  }
}

// The slices of A and of B in one launch: the first a.a.blocks workgroups walk
// A's tiles, the others B's.  One launch of both sides saves a launch (about
// 5 us) and a partly empty last round of workgroups per pass.
// The bounds hold two workgroups on a CU for the two complex forms' residues
// (three for their slices of the scaling product).  Both walks in one kernel need
// more registers than one, and some forms keep a few in scratch for it: the
// embedding 3 with two limbs and 22 with three (92 bytes a thread), the complex
// form's three steps in FP64 28.  A launch a side without scratch (A's and B's
// added) and this one, kernel times at 2000^3: embedding FP64 N = 14 136 and
// 110 us, N = 24 288 and 267, N = 31 353 and 290, FP32 N = 7 59 and 46; complex
// N = 24 254 and 210, N = 36 376 and 328.  The real FP64 form in one step takes
// 130 registers for 116, three workgroups a CU for four: 2500^3 N = 8 43 and 37 us,
// 8192^3 N = 10 488 and 485.
enum SliceForm { kReal, kCx, kEmb };
template <typename T, int FORM, int MODE, int PATH>
__global__ __launch_bounds__(256, FORM == kReal ? 1 : MODE == 1 ? 2 : 3) void k_slices(
    SliceArgs a, CrtConsts cc) {
  __shared__ double tile[kTR * kRS];
  const int w = (int)blockIdx.x;
  if (w < a.a.blocks) {
    if constexpr (FORM == kReal) walk_real<T, true, MODE, PATH>(a, a.a, w, cc, tile);
    if constexpr (FORM == kCx) walk_cx<T, true, MODE, PATH>(a, a.a, w, cc, tile);
    if constexpr (FORM == kEmb) walk_emb<T, true, MODE, PATH>(a, a.a, w, cc, tile);
  } else {
    if constexpr (FORM == kReal) walk_real<T, false, MODE, PATH>(a, a.b, w - a.a.blocks, cc, tile);
    if constexpr (FORM == kCx) walk_cx<T, false, MODE, PATH>(a, a.b, w - a.a.blocks, cc, tile);
    if constexpr (FORM == kEmb) walk_emb<T, false, MODE, PATH>(a, a.b, w - a.a.blocks, cc, tile);
  }
}

// One tile of the grouped launch: which problem side and where.
struct TileJob {
  const void* src;
  const uint64_t* bits;
  const int* mx;
  int* shift;
  int* flag;
  int8_t* out;
  size_t slice;
  int ld, rows, k, k_pad, r0, h0, N;
};

// Map entry i of the grouped launch; false for a mode-1 tile of padding rows.
template <bool ASIDE, int MODE>
__device__ __forceinline__ bool tile_job(const ProbDesc* __restrict__ P,
                                         const BlockRef* __restrict__ map, int i, TileJob* j) {
  const BlockRef e = map[i];
  const ProbDesc& d = P[e.x];
  const int rows = ASIDE ? d.m : d.n, rows_pad = ASIDE ? d.mp : d.np;
  int kx, ry;
  slice_tile<ASIDE>(e.y, d.kp, rows_pad / kTR, &kx, &ry);
  j->r0 = ry * kTR;
  j->h0 = kx * kTK;
  if (MODE == 1 && j->r0 >= rows) return false;
  j->src = ASIDE ? d.A : d.B;
  j->bits = ASIDE ? d.rowbits : d.colbits;
  j->mx = ASIDE ? d.rmax : d.cmax;
  j->shift = ASIDE ? d.mu : d.nu;
  j->flag = d.flag;
  j->out = ASIDE ? d.As : d.Bs;
  j->slice = (size_t)rows_pad * d.kp;
  j->ld = ASIDE ? d.lda : d.ldb;
  j->rows = rows;
  j->k = d.k;
  j->k_pad = d.kp;
  j->N = d.N;
  return true;
}

// Workgroup w of G that walk the `tiles` entries of one side's block map (A
// rows = m, B rows = n) of every problem, as walk_real.
template <typename T, bool ASIDE, int MODE, int PATH>
__device__ __forceinline__ void walk_group(const ProbDesc* __restrict__ P,
                                           const BlockRef* __restrict__ map, int tiles, int w, int G,
                                           const CrtConsts* __restrict__ ctab, double* tile) {
  const int row = (int)(threadIdx.x >> 3);
  int i = w;
  TileJob cur;
  while (i < tiles && !tile_job<ASIDE, MODE>(P, map, i, &cur)) i += G;
  if (i >= tiles) return;
  T x[16];
  tile_loads<T, ASIDE>(static_cast<const T*>(cur.src), cur.ld, cur.rows, cur.k, cur.r0, cur.h0, x);
  RowShift<MODE> rs;
  rs.load(cur.bits, cur.mx, cur.rows, cur.r0 + row);
  for (;;) {
    lds_barrier();
    tile_stage<T, ASIDE>(x, cur.rows, cur.k, cur.r0, cur.h0, tile);
    __asm__ volatile("" ::: "memory");
    const RowResult rr = rs.get(ctab[cur.N], 0);
    TileJob nxt;
    int ni = i + G;
    while (ni < tiles && !tile_job<ASIDE, MODE>(P, map, ni, &nxt)) ni += G;
    if (ni < tiles) {
      tile_loads<T, ASIDE>(static_cast<const T*>(nxt.src), nxt.ld, nxt.rows, nxt.k, nxt.r0,
                           nxt.h0, x);
      rs.load(nxt.bits, nxt.mx, nxt.rows, nxt.r0 + row);
    }
    lds_barrier();
    tile_finish<MODE, PATH>(tile, rr, cur.shift, cur.flag, cur.rows, cur.k_pad, cur.slice,
                            ctab[cur.N], cur.out, cur.r0, cur.h0);
    if (ni >= tiles) break;
    i = ni;
    cur = nxt;
  }
}

// Grouped: both sides of every problem in one launch (the first `ablocks`
// workgroups walk the A side's map).
template <typename T, int MODE, int PATH>
__global__ __launch_bounds__(256) void kg_slices(const ProbDesc* __restrict__ P,
                                                 const BlockRef* __restrict__ amap, int atiles,
                                                 int ablocks, const BlockRef* __restrict__ bmap,
                                                 int btiles, const CrtConsts* __restrict__ ctab) {
  __shared__ double tile[kTR * kRS];
  const int w = (int)blockIdx.x;
  if (w < ablocks)
    walk_group<T, true, MODE, PATH>(P, amap, atiles, w, ablocks, ctab, tile);
  else
    walk_group<T, false, MODE, PATH>(P, bmap, btiles, w - ablocks, (int)gridDim.x - ablocks, ctab,
                                     tile);
}

// Planner operands: x = |a| 2^-alpha (alpha = floor(log2 max_h |a_ih|), so
// x < 2) truncated toward zero to BF16 -- every stored value is a lower bound
// of the exact one -- and, per 64-k tile, the FP64 sum of the exact x of each
// row (partial[tile][row], reduced in a fixed order).  Workgroups walk the
// 64 x 64 tiles in a grid-stride loop and load the next tile into registers
// before they convert the current one.
template <typename T, bool TRANS>
__global__ __launch_bounds__(256) void k_plan_slices(const T* __restrict__ src, int ld, int rows,
                                                     int k, int k_pad, int rows_pad,
                                                     const uint64_t* __restrict__ bits,
                                                     uint16_t* __restrict__ out,
                                                     double* __restrict__ partial,
                                                     int* __restrict__ flag) {
  __shared__ double tile[kPlanTile][kPlanTile + 1];
  const int t = threadIdx.x;
  const int tk = k_pad / kPlanTile;
  const int ntiles = tk * (rows_pad / kPlanTile);
  int id = blockIdx.x;
  if (id >= ntiles) return;   // whole workgroup, before any barrier
  // thread t stages element (r, h) = (t & 63, (t >> 6) + 4q) of the tile
  // (TRANS: rows contiguous in memory) or (r, h) = ((t >> 6) + 4q, t & 63)
  auto load = [&](int tid, T (&x)[16]) {
    const int r0 = (tid / tk) * kPlanTile, h0 = (tid % tk) * kPlanTile;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int a = t & 63, b = (t >> 6) + 4 * q;
      const int rg = r0 + (TRANS ? a : b), hg = h0 + (TRANS ? b : a);
      x[q] = (rg < rows && hg < k) ? (TRANS ? src[rg + (size_t)hg * ld] : src[hg + (size_t)rg * ld])
                                   : (T)0;
    }
  };
  T x[16];
  load(id, x);
  for (;;) {
    __syncthreads();   // the previous tile has been read
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int a = t & 63, b = (t >> 6) + 4 * q;
      if (TRANS)
        tile[a][b] = (double)x[q];
      else
        tile[b][a] = (double)x[q];
    }
    __syncthreads();
    const int cur = id;
    id += (int)gridDim.x;
    if (id < ntiles) load(id, x);
    const int r0 = (cur / tk) * kPlanTile, h0 = (cur % tk) * kPlanTile;
    const int r = t >> 2, hc = (t & 3) * 16, rg = r0 + r;
    const int sh = rg < rows ? shift_prime_bits(bits[rg]) - 5 : 0;   // -alpha
    uint32_t packed[8];
    double sum = 0.0;
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
      const double x0 = ldexp(fabs(tile[r][hc + e]), sh), x1 = ldexp(fabs(tile[r][hc + e + 1]), sh);
      sum += x0;
      sum += x1;
      const uint32_t b0 = __float_as_uint(__double2float_rz(x0)) >> 16;
      const uint32_t b1 = __float_as_uint(__double2float_rz(x1)) >> 16;
      packed[e >> 1] = b0 | (b1 << 16);
    }
    uint4* dst = reinterpret_cast<uint4*>(out + (size_t)rg * k_pad + h0 + hc);
    dst[0] = make_uint4(packed[0], packed[1], packed[2], packed[3]);
    dst[1] = make_uint4(packed[4], packed[5], packed[6], packed[7]);
    sum += __shfl_xor(sum, 1);
    sum += __shfl_xor(sum, 2);
    if ((t & 3) == 0) {
      partial[(size_t)(cur % tk) * rows_pad + rg] = sum;
      if (h0 == 0 && rg < rows && nonfinite_bits(bits[rg])) *flag = 1;
    }
    if (id >= ntiles) break;
  }
}

// Resident workgroups per compute unit of each slice kernel and compute
// units per device, filled once per device by init_slice_launch (outside
// any stream capture); a launch uses at most that many workgroups.  Index:
// [float][kReal, kCx, kEmb, grouped][variant], variant 0 = the bars, 1 + path =
// the residues on that path (kAnyPath, chosen per tile: grouped only).
constexpr int kMaxDevices = 64;
constexpr int kVariants = 2 + kAnyPath;
constexpr int kGroupForm = 3;
constexpr int kPartSlots = 512;   // workgroups that shared tiles may fill (two per CU)
std::atomic<int> g_cus[kMaxDevices];
std::atomic<int> g_occ[2][4][kVariants];

template <typename K>
int resident_per_cu(K* kern) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(kern), 256, 0) !=
          hipSuccess ||
      n < 1)
    n = 1;
  return n;
}

template <typename T, int FORM>
void fill_occ_form() {
  constexpr int kBar = FORM == kCx ? 2 : 0;
  std::atomic<int>* o = g_occ[std::is_same<T, float>::value ? 1 : 0][FORM];
  o[0] = resident_per_cu(k_slices<T, FORM, kBar, kAnyPath>);
  o[1 + kLimbs2] = resident_per_cu(k_slices<T, FORM, 1, kLimbs2>);
  o[1 + kLimbs3] = resident_per_cu(k_slices<T, FORM, 1, kLimbs3>);
  o[1 + kSteps1] = resident_per_cu(k_slices<T, FORM, 1, kSteps1>);
  o[1 + kSteps3] = resident_per_cu(k_slices<T, FORM, 1, kSteps3>);
  o[1 + kSteps4] = resident_per_cu(k_slices<T, FORM, 1, kSteps4>);
}

template <typename T>
void fill_occ() {
  fill_occ_form<T, kReal>();
  fill_occ_form<T, kCx>();
  fill_occ_form<T, kEmb>();
  std::atomic<int>* o = g_occ[std::is_same<T, float>::value ? 1 : 0][kGroupForm];
  o[0] = resident_per_cu(kg_slices<T, 0, kAnyPath>);
  o[1 + kLimbs2] = resident_per_cu(kg_slices<T, 1, kLimbs2>);
  o[1 + kLimbs3] = resident_per_cu(kg_slices<T, 1, kLimbs3>);
  o[1 + kSteps1] = resident_per_cu(kg_slices<T, 1, kSteps1>);
  o[1 + kSteps3] = resident_per_cu(kg_slices<T, 1, kSteps3>);
  o[1 + kSteps4] = resident_per_cu(kg_slices<T, 1, kSteps4>);
  o[1 + kAnyPath] = resident_per_cu(kg_slices<T, 1, kAnyPath>);
}

// Workgroups *ba and *bb for ta and tb tiles of the two sides, whose tiles cost
// wa and wb: one per tile while they all fit the resident slots of
// the device (or the device's figures are unknown), else the slots in
// proportion to the work.  A positive g_slice_cap (a test knob set through
// ozaki2_debug_tuning) caps each side's count, so that each workgroup walks
// many tiles.
void slice_blocks(bool f32, int form, int variant, int ta, int tb, int wa, int wb, int* ba,
                  int* bb) {
  *ba = ta;
  *bb = tb;
  int dev = 0;
  if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices) {
    const int64_t slots = (int64_t)g_cus[dev].load(std::memory_order_relaxed) *
                          g_occ[f32 ? 1 : 0][form][variant].load(std::memory_order_relaxed);
    if (slots > 1 && (int64_t)ta + tb > slots) {
      const double share = (double)wa * ta / ((double)wa * ta + (double)wb * tb);
      int64_t a = (int64_t)(share * (double)slots + 0.5);
      if (ta > 0) a = std::max<int64_t>(a, 1);
      if (tb > 0) a = std::min<int64_t>(a, slots - 1);
      *ba = (int)std::min<int64_t>(ta, a);
      *bb = (int)std::min<int64_t>(tb, slots - a);
    }
  }
  const int cap = g_slice_cap.load(std::memory_order_relaxed);
  if (cap > 0) {
    *ba = std::min(*ba, cap);
    *bb = std::min(*bb, cap);
  }
}

template <typename T, int FORM, int MODE, int PATH>
void launch_one(hipStream_t s, SliceArgs& a, const CrtConsts& cc) {
  const int variant = MODE != 1 ? 0 : 1 + PATH;
  const int tiles = a.a.tiles + a.b.tiles;
  if (tiles <= 0) return;
  // The embedding's residues: a tile of A is read once, as one of B, and each of its
  // moduli written twice.  Apart, a tile of A took 1.4 times one of B's time at N = 2,
  // 1.8 times at N = 7 and 15.  8192 x 2000 x 33000 in FP64, N = 2: 1966 us at two to
  // one, 1729 so.
  const bool two_rows = FORM == kEmb && MODE == 1;
  slice_blocks(std::is_same<T, float>::value, FORM, variant, a.a.tiles, a.b.tiles,
               two_rows ? 3 + 2 * cc.N : 1, two_rows ? 3 + cc.N : 1, &a.a.blocks, &a.b.blocks);
  // While the tiles leave slots free, the moduli of a tile are dealt to several
  // workgroups (for_moduli), at least two each; the tile is then read again by
  // each of them, from L2.  At 256^3 (16 tiles a side, N = 14) this took the
  // residues of a side from 9.8 to 6.7 us.
  const bool one_each = a.a.blocks == a.a.tiles && a.b.blocks == a.b.tiles;
  const int parts = MODE == 1 && one_each ? std::min(cc.N / 2, kPartSlots / tiles) : 1;
  const dim3 grid((unsigned)(a.a.blocks + a.b.blocks), (unsigned)std::max(parts, 1));
  hipLaunchKernelGGL((k_slices<T, FORM, MODE, PATH>), grid, dim3(256), 0, s, a, cc);
}

template <typename T, int FORM>
void launch_residues_t(hipStream_t s, SliceArgs& a, const CrtConsts& cc) {
  switch (residue_path(cc)) {
    case kLimbs2: launch_one<T, FORM, 1, kLimbs2>(s, a, cc); break;
    case kLimbs3: launch_one<T, FORM, 1, kLimbs3>(s, a, cc); break;
    case kSteps1: launch_one<T, FORM, 1, kSteps1>(s, a, cc); break;
    case kSteps3: launch_one<T, FORM, 1, kSteps3>(s, a, cc); break;
    default: launch_one<T, FORM, 1, kSteps4>(s, a, cc); break;
  }
}

template <typename T>
void launch_form(hipStream_t s, SliceSet set, bool bars, SliceArgs& a, const CrtConsts& cc) {
  if (set == SliceSet::Real)
    bars ? launch_one<T, kReal, 0, kAnyPath>(s, a, cc) : launch_residues_t<T, kReal>(s, a, cc);
  else if (set == SliceSet::Complex3)
    bars ? launch_one<T, kCx, 2, kAnyPath>(s, a, cc) : launch_residues_t<T, kCx>(s, a, cc);
  else
    bars ? launch_one<T, kEmb, 0, kAnyPath>(s, a, cc) : launch_residues_t<T, kEmb>(s, a, cc);
}

template <typename T, int MODE, int PATH>
void launch_group_one(hipStream_t s, const ProbDesc* P, const BlockRef* amap, int atiles,
                      const BlockRef* bmap, int btiles, const CrtConsts* ctab) {
  int ba, bb;
  slice_blocks(std::is_same<T, float>::value, kGroupForm, MODE == 0 ? 0 : 1 + PATH, atiles, btiles,
               1, 1, &ba, &bb);
  hipLaunchKernelGGL((kg_slices<T, MODE, PATH>), dim3((unsigned)(ba + bb)), dim3(256), 0, s, P,
                     amap, atiles, ba, bmap, btiles, ctab);
}

template <typename T>
void group_slices_t(hipStream_t s, bool bars, int path, const ProbDesc* P, const BlockRef* amap,
                    int atiles, const BlockRef* bmap, int btiles, const CrtConsts* ctab) {
  if (bars) {
    launch_group_one<T, 0, kAnyPath>(s, P, amap, atiles, bmap, btiles, ctab);
    return;
  }
  switch (path) {
    case kLimbs2: launch_group_one<T, 1, kLimbs2>(s, P, amap, atiles, bmap, btiles, ctab); break;
    case kLimbs3: launch_group_one<T, 1, kLimbs3>(s, P, amap, atiles, bmap, btiles, ctab); break;
    case kSteps1: launch_group_one<T, 1, kSteps1>(s, P, amap, atiles, bmap, btiles, ctab); break;
    case kSteps3: launch_group_one<T, 1, kSteps3>(s, P, amap, atiles, bmap, btiles, ctab); break;
    case kSteps4: launch_group_one<T, 1, kSteps4>(s, P, amap, atiles, bmap, btiles, ctab); break;
    default: launch_group_one<T, 1, kAnyPath>(s, P, amap, atiles, bmap, btiles, ctab); break;
  }
}

}  // namespace

std::atomic<int> g_slice_cap{0};

void init_slice_launch(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
  fill_occ<double>();
  fill_occ<float>();
  g_cus[dev].store(cus, std::memory_order_relaxed);
}

int group_residue_path(const CrtConsts* const* cc, int count) {
  int path = -1;
  for (int q = 0; q < count; ++q) {
    const int r = residue_path(*cc[q]);
    if (path >= 0 && r != path) return kAnyPath;
    path = r;
  }
  return path < 0 ? kAnyPath : path;
}

void launch_group_slices(hipStream_t s, Prec pr, bool bars, int path, const ProbDesc* P,
                         const BlockRef* amap, int atiles, const BlockRef* bmap, int btiles,
                         const CrtConsts* ctab) {
  if (atiles + btiles <= 0) return;
  if (path < 0 || path > kAnyPath) path = kAnyPath;
  if (pr == Prec::F64)
    group_slices_t<double>(s, bars, path, P, amap, atiles, bmap, btiles, ctab);
  else
    group_slices_t<float>(s, bars, path, P, amap, atiles, bmap, btiles, ctab);
}

void launch_plan_slices(hipStream_t s, Prec pr, bool trans, const void* src, int ld, int rows,
                        int k, int rows_pad, int k_pad, const uint64_t* bits, uint16_t* out,
                        double* partial, int* flag) {
  // Four workgroups per CU (33 KB of LDS each) walk the tiles.
  const int64_t tiles = (int64_t)(k_pad / kPlanTile) * (rows_pad / kPlanTile);
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices)
    cus = g_cus[dev].load(std::memory_order_relaxed);
  if (tiles <= 0) return;
  const int64_t cap = 4 * (int64_t)(cus > 0 ? cus : 256);
  const dim3 grid((unsigned)(tiles < cap ? tiles : cap));
  if (pr == Prec::F64) {
    if (trans)
      hipLaunchKernelGGL((k_plan_slices<double, true>), grid, dim3(256), 0, s, (const double*)src,
                         ld, rows, k, k_pad, rows_pad, bits, out, partial, flag);
    else
      hipLaunchKernelGGL((k_plan_slices<double, false>), grid, dim3(256), 0, s, (const double*)src,
                         ld, rows, k, k_pad, rows_pad, bits, out, partial, flag);
  } else {
    if (trans)
      hipLaunchKernelGGL((k_plan_slices<float, true>), grid, dim3(256), 0, s, (const float*)src, ld,
                         rows, k, k_pad, rows_pad, bits, out, partial, flag);
    else
      hipLaunchKernelGGL((k_plan_slices<float, false>), grid, dim3(256), 0, s, (const float*)src, ld,
                         rows, k, k_pad, rows_pad, bits, out, partial, flag);
  }
}

void launch_slices(hipStream_t s, Prec pr, SliceSet set, bool bars, const SliceOperand* A,
                   const SliceOperand* B, int k, int k_pad, const CrtConsts& cc, int* flag,
                   int bias) {
  SliceArgs a{};
  a.flag = flag;
  a.k = k;
  a.k_pad = k_pad;
  a.bias = bias;
  const bool emb = set == SliceSet::Embedding;
  auto fill = [&](SliceSide* d, const SliceOperand* o, bool aside) {
    if (!o) return;
    // the embedding's A side: tiles cover its first row half
    const int span = emb && aside ? o->rows_pad / 2 : o->rows_pad;
    d->src = o->src;
    d->bits = o->bits;
    d->mx = o->mx;
    d->shift = o->shift;
    d->out = o->out;
    d->slice = (size_t)o->rows_pad * k_pad * (emb ? 2 : 1);
    d->ld = o->ld;
    d->rows = o->rows;
    d->gy = bars ? span / kTR : cdiv_i(o->rows, kTR);   // bars cover the padding rows
    d->tiles = (k_pad / kTK) * d->gy;
    if (emb && aside) a.half = span;
  };
  fill(&a.a, A, true);
  fill(&a.b, B, false);
  if (pr == Prec::F64)
    launch_form<double>(s, set, bars, a, cc);
  else
    launch_form<float>(s, set, bars, a, cc);
}

}  // namespace oz2
