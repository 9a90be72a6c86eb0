// CRT accumulation, final reduction and inverse scaling (Algorithm 3 from the
// weighted sums on, and the last step of Algorithm 1), fused in one pass over
// the N INT8 slices W_l:
//   C'(1) = fl(sum_l s_l1 W_l)      (exact for b = 64, Lemma 2)
//   C'(2) = fl(sum_l s_l2 W_l)      (fma chain in l order; b = 64 only)
//   Q     = round(fl(P_inv C'(1)))  (equals round(C'/P), Lemma 3)
//   C''   = fl(fma(-Q, P2, fma(-Q, P1, C'(1)) + C'(2)))   (b = 64)
//   C''   = single(fma(-Q, P1, C'(1)))                      (b = 32)
//   C     = C'' * 2^(-mu_i - nu_j), one rounding.
// Every operation is an explicit fma / single rounding (built with
// -ffp-contract=off), so the result is deterministic.
//
// Bound by memory: N bytes read and one entry written per entry of C.  So the
// loads of the next moduli go out before a group is used, C leaves in whole
// lines (through LDS where a lane's entries are more than one store), and both
// are marked as streaming, since nothing here reads a line twice.  FP64, N = 14,
// 8192^2 (1.48 GB): 307 us before, 275 with the first two, 250 with all three
// (5.9 TB/s); FP32, N = 7: 167 and 127 us; 4093 x 4095 with unaligned columns
// 98 and 72 us.
#include <cstdint>
#include <type_traits>

#include "ozaki2_internal.h"
#include "small_mod.h"

namespace oz2 {
namespace {

template <typename V>
__device__ __forceinline__ V load_stream(const V* p) {
  return __builtin_nontemporal_load(p);
}

template <typename T, int E>
__device__ __forceinline__ void store_entry(T* __restrict__ p, const T* v) {
  typedef T V __attribute__((ext_vector_type(E)));
  if (E == 1 || ((uintptr_t)p & (E * sizeof(T) - 1)) == 0) {
    __builtin_nontemporal_store(*reinterpret_cast<const V*>(v), reinterpret_cast<V*>(p));
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) p[e] = v[e];
  }
}

// Place of a thread: row chunk `i0 / R` of column j, and whether it has one (a
// thread past the last takes the last column again and stores nothing).  The
// block's first place is divided once, the threads' with 32 bits.
struct CrtPlace {
  int j, i0;
  bool in;
};
__device__ __forceinline__ CrtPlace crt_place(int64_t block, int m, int n, int R) {
  const unsigned chunks = (unsigned)cdiv_i(m, R);
  const uint64_t g0 = (uint64_t)block * 256;
  unsigned j0, r0;
  if (g0 >> 32) {
    j0 = (unsigned)(g0 / chunks);
    r0 = (unsigned)(g0 - (uint64_t)j0 * chunks);
  } else {
    j0 = (unsigned)g0 / chunks;
    r0 = (unsigned)g0 - j0 * chunks;
  }
  const unsigned t = r0 + threadIdx.x, dj = t / chunks;
  const int j = (int)(j0 + dj);
  return {j < n ? j : n - 1, (int)(t - dj * chunks) * R, j < n};
}

// The R entries of E values that each lane of a wave holds (rows i0.. of column
// j), through LDS so that consecutive lanes store consecutive entries: whole
// lines per store at any alignment of C.
template <typename T, int R, int E>
struct CrtStage {
  T v[4][64 * R * E];
};
template <typename T, int R, int E>
__device__ __forceinline__ void store_rows(CrtStage<T, R, E>& lds, T* __restrict__ C, int ldc, int m,
                                           const CrtPlace& pl, const T (&out)[R * E]) {
  const int lane = threadIdx.x & 63;
  const int64_t off = (int64_t)pl.j * ldc + pl.i0;
  const int have = pl.in ? min(m - pl.i0, R) : 0;
  if constexpr (sizeof(T) * R * E == 16) {               // a lane's entries are one store
    typedef T V __attribute__((ext_vector_type(R * E)));
    if (__all(have == R && ((uintptr_t)(C + off * E) & 15) == 0)) {
      V v;
#pragma unroll
      for (int e = 0; e < R * E; ++e) v[e] = out[e];
      __builtin_nontemporal_store(v, reinterpret_cast<V*>(C + off * E));
      return;
    }
  }
  T* st = lds.v[threadIdx.x >> 6];
#pragma unroll
  for (int e = 0; e < R * E; ++e) st[lane * R * E + e] = out[e];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int64_t off0 = ((int64_t)__builtin_amdgcn_readfirstlane((int)(off >> 32)) << 32) |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)off);
  // a wave inside one column, all rows real: consecutive entries of C
  const bool whole = __all(have == R && off == off0 + lane * R);
#pragma unroll
  for (int s = 0; s < R; ++s) {
    const int q = 64 * s + lane;                         // entry of the wave
    int64_t o = off0 + q;
    bool in = true;
    if (!whole) {
      const int src = q / R, e = q % R;
      const int64_t lo = (uint32_t)__shfl((int)off, src), hi = __shfl((int)(off >> 32), src);
      o = (hi << 32 | lo) + e;
      in = e < __shfl(have, src);
    }
    if (in) store_entry<T, E>(C + o * E, st + q * E);
  }
}

// One thread handles R = kCrtRows consecutive rows i of one column j: one
// R-byte load per modulus (64 R contiguous bytes per wave).
// Thread g (g = 0 .. ceil(m/R) n - 1) takes row chunk g % ceil(m/R) of column
// g / ceil(m/R): consecutive threads walk down a column and continue in the
// next, so small-m problems keep every lane busy.
// With DBG, C'(1), C'(2), Q and C'' of every entry are also stored, as FP64
// column-major m x n arrays at dbg + s * m * n for s = 0..3 (stage dumps).

// C'(1) and C'(2) of R consecutive rows (wp: row i0 of column j of slice 0, a
// multiple of R bytes, so that each slice's R bytes are one load).
template <typename T, int R>
__device__ __forceinline__ void crt_sums(const int8_t* __restrict__ wp, size_t sw,
                                         const CrtConsts& cc, double (&c1)[R], double (&c2)[R]) {
  typedef typename std::conditional<R == 2, uint16_t,
                                    typename std::conditional<R == 4, uint32_t, uint64_t>::type>::type
      WordT;
#pragma unroll
  for (int e = 0; e < R; ++e) c1[e] = c2[e] = 0.0;
  // Moduli in groups of 4; the next group's loads (clamped to the last slice) go
  // out before a group is used, so that four to eight are under way.
  // An INT8 value w with stored byte b becomes a double without the convert
  // instruction: the bit pattern 0x43300000:(b ^ 0x80) is 2^52 + w + 128, and
  // subtracting 2^52 + 128 is exact.
  auto load = [&](int l0, WordT (&v)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int8_t* src = wp + (size_t)min(l0 + u, cc.N - 1) * sw;
      v[u] = load_stream(reinterpret_cast<const WordT*>(src));
    }
  };
  auto use = [&](WordT v, double s1, double s2) {
    const uint64_t biased = (uint64_t)v ^ 0x8080808080808080ull;
#pragma unroll
    for (int e = 0; e < R; ++e) {
      const int byte = (int)((biased >> (8 * e)) & 0xFF);
      const double w = __hiloint2double(0x43300000, byte) - 4503599627370624.0;  // 2^52 + 128
      c1[e] = fma(s1, w, c1[e]);
      if (sizeof(T) == 8) c2[e] = fma(s2, w, c2[e]);
    }
  };
  WordT cur[4], next[4];
  load(0, cur);
  int l0 = 0;
  for (; l0 + 4 <= cc.N; l0 += 4) {
    if (l0 + 4 < cc.N) load(l0 + 4, next);
#pragma unroll
    for (int u = 0; u < 4; ++u) use(cur[u], cc.s1[l0 + u], cc.s2[l0 + u]);
#pragma unroll
    for (int u = 0; u < 4; ++u) cur[u] = next[u];
  }
  // up to three more; a modulus past N gets weight 0, and fma(0, w, c) = c
  if (l0 < cc.N) {
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int l = min(l0 + u, cc.N - 1);
      use(cur[u], l0 + u < cc.N ? cc.s1[l] : 0.0, l0 + u < cc.N ? cc.s2[l] : 0.0);
    }
  }
}

// One thread of a launch folds the call's non-finite flag into the sticky word.
__device__ __forceinline__ void fold_status(const int* __restrict__ flag,
                                            int* __restrict__ status) {
  if (threadIdx.x == 0 && *flag) atomicOr(status, 1);
}

// Q, C'' and the output 2^ex C'' (NaN when the non-finite flag is set) of
// one entry from its C'(1), C'(2).
template <typename T>
__device__ __forceinline__ T crt_value(double c1, double c2, const CrtConsts& cc, int ex, bool bad,
                                       double* q_out, double* cpp_out) {
  const double q = rint(c1 * cc.Pinv);
  const double t = fma(-q, cc.P1, c1);
  double cppd;
  T out;
  if (sizeof(T) == 8) {
    const double cpp = fma(-q, cc.P2, t + c2);
    out = bad ? (T)NAN : (T)ldexp(cpp, ex);
    cppd = cpp;
  } else {
    const float cpp = (float)t;
    out = bad ? (T)NAN : (T)ldexp((double)cpp, ex);
    cppd = (double)cpp;
  }
  *q_out = q;
  *cpp_out = cppd;
  return out;
}

template <typename T, int R, bool DBG = false>
__device__ __forceinline__ void crt_body(const int8_t* __restrict__ W, size_t sw, int ldw,
                                         const int* __restrict__ mu, const int* __restrict__ nu,
                                         int m, int n, const CrtConsts& cc,
                                         const int* __restrict__ flag, T* __restrict__ C, int ldc,
                                         int64_t block, double* __restrict__ dbg = nullptr) {
  __shared__ __attribute__((aligned(16))) CrtStage<T, R, 1> lds;
  const CrtPlace pl = crt_place(block, m, n, R);
  const bool bad = *flag != 0;
  const int nuj = nu[pl.j];
  int ex[R];
#pragma unroll
  for (int e = 0; e < R; ++e) ex[e] = -mu[min(pl.i0 + e, m - 1)] - nuj;
  double c1[R], c2[R];
  crt_sums<T, R>(W + (size_t)pl.j * ldw + pl.i0, sw, cc, c1, c2);
  T out[R];
#pragma unroll
  for (int e = 0; e < R; ++e) {
    double q, cppd;
    out[e] = crt_value<T>(c1[e], c2[e], cc, ex[e], bad, &q, &cppd);
    if constexpr (DBG) {
      if (pl.in && pl.i0 + e < m) {
        const size_t mn = (size_t)m * n, o = (size_t)pl.j * m + pl.i0 + e;
        dbg[o] = c1[e];
        dbg[mn + o] = c2[e];
        dbg[2 * mn + o] = q;
        dbg[3 * mn + o] = cppd;
      }
    }
  }
  store_rows<T, R, 1>(lds, C, ldc, m, pl, out);
}

// Complex output: the real parts from (Wr, mur) and the imaginary parts from
// (Wi, mui), both with the column shifts nu, written as interleaved (re, im)
// pairs into the column-major complex C (ldc in complex elements).  The
// imaginary rows start at half of the padded rows, a multiple of 64, and the
// loads of a partial last chunk stay inside each half.
template <typename T, int R>
__device__ __forceinline__ void crt_complex_body(const int8_t* __restrict__ Wr,
                                                 const int8_t* __restrict__ Wi, size_t sw, int ldw,
                                                 const int* __restrict__ mur,
                                                 const int* __restrict__ mui,
                                                 const int* __restrict__ nu, int m, int n,
                                                 const CrtConsts& cc, const int* __restrict__ flag,
                                                 T* __restrict__ C, int ldc, int64_t block) {
  __shared__ __attribute__((aligned(16))) CrtStage<T, R, 2> lds;
  const CrtPlace pl = crt_place(block, m, n, R);
  const size_t o = (size_t)pl.j * ldw + pl.i0;
  const bool bad = *flag != 0;
  const int nuj = nu[pl.j];
  double c1[R], c2[R], q, cppd;
  T out[2 * R];
  crt_sums<T, R>(Wr + o, sw, cc, c1, c2);
#pragma unroll
  for (int e = 0; e < R; ++e)
    out[2 * e] = crt_value<T>(c1[e], c2[e], cc, -mur[min(pl.i0 + e, m - 1)] - nuj, bad, &q, &cppd);
  crt_sums<T, R>(Wi + o, sw, cc, c1, c2);
#pragma unroll
  for (int e = 0; e < R; ++e)
    out[2 * e + 1] =
        crt_value<T>(c1[e], c2[e], cc, -mui[min(pl.i0 + e, m - 1)] - nuj, bad, &q, &cppd);
  store_rows<T, R, 2>(lds, C, ldc, m, pl, out);
}

// The 3-product form (reading R25 of the complex GEMM): per modulus l the
// real and imaginary residues are mod(W1 - W2, p_l) and mod(W3 - W1 - W2,
// p_l) of the three products' bytes, formed here and summed into C'(1),
// C'(2) of both parts with the l-ordered fma chains of crt_sums.  The bytes
// lie in [lo, hi] = [(1-p)/2, (p-1)/2] (odd p) or [-128, 127] (p = 256), so
// a difference or sum of two lies in [-(p-1), p-1] and one correction by p
// brings it back into [lo, hi]: W1 - W2 directly, W3 - W1 - W2 as W3 minus
// the corrected W1 + W2, two values per packed 16-bit instruction (12.5 integer
// operations per modulus and entry against 26 one value at a time, which took
// longer than the loads).  Moduli as in crt_sums.  W1, W2, W3 are whole planes
// (tile-aligned), so each R-byte load is aligned.
template <typename T, int R>
__device__ __forceinline__ void crt_sums_3m(const int8_t* __restrict__ w1,
                                            const int8_t* __restrict__ w2,
                                            const int8_t* __restrict__ w3, size_t sw,
                                            const CrtConsts& cc, double (&c1r)[R], double (&c2r)[R],
                                            double (&c1i)[R], double (&c2i)[R]) {
#pragma unroll
  for (int e = 0; e < R; ++e) c1r[e] = c2r[e] = c1i[e] = c2i[e] = 0.0;
  static_assert(R == 4, "two pairs");
  struct Three {
    uint32_t a[4], b[4], c[4];
  } cur, next;
  auto load = [&](int l0, Three& v) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t off = (size_t)min(l0 + u, cc.N - 1) * sw;
      v.a[u] = load_stream(reinterpret_cast<const uint32_t*>(w1 + off));
      v.b[u] = load_stream(reinterpret_cast<const uint32_t*>(w2 + off));
      v.c[u] = load_stream(reinterpret_cast<const uint32_t*>(w3 + off));
    }
  };
  auto use = [&](uint32_t wa, uint32_t wb, uint32_t wc, int p, double s1, double s2) {
    const int lo = (p - 1) / 2 + 1 - p;
    // x - lo for the representative x of a value in [lo, lo + p): of d, d + p
    // and d - p the smallest as an unsigned 16-bit number
    auto fix = [&](uint32_t d, int bias) {
      return pk_min(pk_min(pk_add(d, both16(bias - lo)), pk_add(d, both16(bias - lo + p))),
                    pk_add(d, both16(bias - lo - p)));
    };
    const uint32_t a = wa ^ 0x80808080u, b = wb ^ 0x80808080u, c = wc ^ 0x80808080u;
    // 2^52 + (x - lo) less 2^52 - lo is x exactly
    const double base = 4503599627370496.0 - (double)lo;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t sel = h ? 0x0c030c02u : 0x0c010c00u;
      const uint32_t a2 = __builtin_amdgcn_perm(0, a, sel), b2 = __builtin_amdgcn_perm(0, b, sel),
                     c2 = __builtin_amdgcn_perm(0, c, sel);
      const uint32_t xr = fix(pk_sub(a2, b2), 0);
      const uint32_t xs = fix(pk_add(a2, b2), -256);     // t1 + t2, less lo
      const uint32_t xi = fix(pk_sub(c2, xs), -128 - lo);  // t3 - (t1 + t2)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int e = 2 * h + q;
        const double wr = __hiloint2double(0x43300000, q ? xr >> 16 : xr & 0xFFFF) - base;
        const double wi = __hiloint2double(0x43300000, q ? xi >> 16 : xi & 0xFFFF) - base;
        c1r[e] = fma(s1, wr, c1r[e]);
        c1i[e] = fma(s1, wi, c1i[e]);
        if (sizeof(T) == 8) {
          c2r[e] = fma(s2, wr, c2r[e]);
          c2i[e] = fma(s2, wi, c2i[e]);
        }
      }
    }
  };
  load(0, cur);
  int l0 = 0;
  for (; l0 + 4 <= cc.N; l0 += 4) {
    if (l0 + 4 < cc.N) load(l0 + 4, next);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      use(cur.a[u], cur.b[u], cur.c[u], cc.mod[l0 + u].p, cc.s1[l0 + u], cc.s2[l0 + u]);
    cur = next;
  }
  if (l0 < cc.N) {                                       // as in crt_sums
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int l = min(l0 + u, cc.N - 1);
      use(cur.a[u], cur.b[u], cur.c[u], cc.mod[l].p, l0 + u < cc.N ? cc.s1[l] : 0.0,
          l0 + u < cc.N ? cc.s2[l] : 0.0);
    }
  }
}

template <typename T, int R>
__device__ __forceinline__ void crt_3m_body(const int8_t* __restrict__ W1,
                                            const int8_t* __restrict__ W2,
                                            const int8_t* __restrict__ W3, size_t sw, int ldw,
                                            const int* __restrict__ mu, const int* __restrict__ nu,
                                            int m, int n, const CrtConsts& cc,
                                            const int* __restrict__ flag, T* __restrict__ C,
                                            int ldc, int64_t block) {
  __shared__ __attribute__((aligned(16))) CrtStage<T, R, 2> lds;
  const CrtPlace pl = crt_place(block, m, n, R);
  const bool bad = *flag != 0;
  const int nuj = nu[pl.j];
  const size_t o = (size_t)pl.j * ldw + pl.i0;
  double c1r[R], c2r[R], c1i[R], c2i[R], q, cppd;
  crt_sums_3m<T, R>(W1 + o, W2 + o, W3 + o, sw, cc, c1r, c2r, c1i, c2i);
  T out[2 * R];
#pragma unroll
  for (int e = 0; e < R; ++e) {
    const int ex = -mu[min(pl.i0 + e, m - 1)] - nuj;
    out[2 * e] = crt_value<T>(c1r[e], c2r[e], cc, ex, bad, &q, &cppd);
    out[2 * e + 1] = crt_value<T>(c1i[e], c2i[e], cc, ex, bad, &q, &cppd);
  }
  store_rows<T, R, 2>(lds, C, ldc, m, pl, out);
}

// The constants come last, so that the arguments before them share a line or two.
template <typename T, int R>
__global__ __launch_bounds__(256) void k_crt_3m(const int8_t* __restrict__ W1,
                                                const int8_t* __restrict__ W2,
                                                const int8_t* __restrict__ W3, size_t sw, int ldw,
                                                const int* __restrict__ mu,
                                                const int* __restrict__ nu, int m, int n,
                                                const int* __restrict__ flag,
                                                int* __restrict__ status, T* __restrict__ C,
                                                int ldc, CrtConsts cc) {
  crt_3m_body<T, R>(W1, W2, W3, sw, ldw, mu, nu, m, n, cc, flag, C, ldc, blockIdx.x);
  if (blockIdx.x == 0) fold_status(flag, status);
}

template <typename T, int R>
__global__ __launch_bounds__(256) void k_crt_complex(
    const int8_t* __restrict__ Wr, const int8_t* __restrict__ Wi, size_t sw, int ldw,
    const int* __restrict__ mur, const int* __restrict__ mui, const int* __restrict__ nu, int m,
    int n, const int* __restrict__ flag, int* __restrict__ status, T* __restrict__ C, int ldc,
    CrtConsts cc) {
  crt_complex_body<T, R>(Wr, Wi, sw, ldw, mur, mui, nu, m, n, cc, flag, C, ldc, blockIdx.x);
  if (blockIdx.x == 0) fold_status(flag, status);
}

template <typename T, int R>
__global__ __launch_bounds__(256) void k_crt(const int8_t* __restrict__ W, size_t sw, int ldw,
                                             const int* __restrict__ mu, const int* __restrict__ nu,
                                             int m, int n, const int* __restrict__ flag,
                                             int* __restrict__ status, T* __restrict__ C, int ldc,
                                             CrtConsts cc) {
  crt_body<T, R>(W, sw, ldw, mu, nu, m, n, cc, flag, C, ldc, blockIdx.x);
  if (blockIdx.x == 0) fold_status(flag, status);
}

template <typename T>
__global__ __launch_bounds__(256) void k_crt_debug(const int8_t* __restrict__ W, size_t sw, int ldw,
                                                   const int* __restrict__ mu,
                                                   const int* __restrict__ nu, int m, int n,
                                                   CrtConsts cc, const int* __restrict__ flag,
                                                   T* __restrict__ C, int ldc,
                                                   double* __restrict__ dbg) {
  crt_body<T, kCrtRows, true>(W, sw, ldw, mu, nu, m, n, cc, flag, C, ldc, blockIdx.x, dbg);
}

template <typename T>
__global__ __launch_bounds__(256) void kg_crt(const ProbDesc* __restrict__ P,
                                              const BlockRef* __restrict__ map,
                                              const CrtConsts* __restrict__ ctab,
                                              int* __restrict__ status) {
  const BlockRef e = map[blockIdx.x];
  const ProbDesc& d = P[e.x];
  crt_body<T, kCrtRows>(d.W, (size_t)d.np * d.mp, d.mp, d.mu, d.nu, d.m, d.n, ctab[d.N], d.flag,
                        (T*)d.C, d.ldc, e.y);
  if (e.y == 0) fold_status(d.flag, status);
}

template <typename T>
__global__ __launch_bounds__(256) void k_fill_zero(T* __restrict__ C, int ldc, int m,
                                                   int iblocks) {
  const int j = blockIdx.x / iblocks;
  const int i = (blockIdx.x % iblocks) * 256 + threadIdx.x;
  if (i < m) C[i + (size_t)j * ldc] = (T)0;
}

}  // namespace

void launch_group_crt(hipStream_t s, Prec pr, const ProbDesc* P, const BlockRef* map, int blocks,
                      const CrtConsts* ctab, int* status) {
  if (blocks <= 0) return;
  const dim3 g((unsigned)blocks), b(256);
  if (pr == Prec::F64)
    hipLaunchKernelGGL(kg_crt<double>, g, b, 0, s, P, map, ctab, status);
  else
    hipLaunchKernelGGL(kg_crt<float>, g, b, 0, s, P, map, ctab, status);
}

namespace {

template <typename T>
void launch_crt_t(hipStream_t s, const int8_t* W, size_t sw, int ldw, const int* mu, const int* nu,
                  int m, int n, const CrtConsts& cc, const int* flag, int* status,
                  void* C, int ldc) {
  hipLaunchKernelGGL((k_crt<T, kCrtRows>), dim3((unsigned)crt_blocks(m, n)), dim3(256), 0, s, W, sw,
                     ldw, mu, nu, m, n, flag, status, (T*)C, ldc, cc);
}

}  // namespace

void launch_crt(hipStream_t s, Prec pr, const int8_t* W, size_t sw, int ldw, const int* mu,
                const int* nu, int m, int n, const CrtConsts& cc, const int* flag, int* status,
                void* C, int ldc) {
  if (pr == Prec::F64)
    launch_crt_t<double>(s, W, sw, ldw, mu, nu, m, n, cc, flag, status, C, ldc);
  else
    launch_crt_t<float>(s, W, sw, ldw, mu, nu, m, n, cc, flag, status, C, ldc);
}

void launch_crt_3m(hipStream_t s, Prec pr, const int8_t* W1, const int8_t* W2, const int8_t* W3,
                   size_t sw, int ldw, const int* mu, const int* nu, int m, int n,
                   const CrtConsts& cc, const int* flag, int* status, void* C, int ldc) {
  const dim3 grid((unsigned)crt_blocks(m, n)), block(256);
  if (pr == Prec::F64)
    hipLaunchKernelGGL((k_crt_3m<double, kCrtRows>), grid, block, 0, s, W1, W2, W3, sw, ldw, mu, nu,
                       m, n, flag, status, (double*)C, ldc, cc);
  else
    hipLaunchKernelGGL((k_crt_3m<float, kCrtRows>), grid, block, 0, s, W1, W2, W3, sw, ldw, mu, nu,
                       m, n, flag, status, (float*)C, ldc, cc);
}

void launch_crt_complex(hipStream_t s, Prec pr, const int8_t* Wr, const int8_t* Wi, size_t sw,
                        int ldw, const int* mur, const int* mui, const int* nu, int m, int n,
                        const CrtConsts& cc, const int* flag, int* status, void* C, int ldc) {
  const dim3 grid((unsigned)crt_blocks(m, n)), block(256);
  if (pr == Prec::F64)
    hipLaunchKernelGGL((k_crt_complex<double, kCrtRows>), grid, block, 0, s, Wr, Wi, sw, ldw, mur,
                       mui, nu, m, n, flag, status, (double*)C, ldc, cc);
  else
    hipLaunchKernelGGL((k_crt_complex<float, kCrtRows>), grid, block, 0, s, Wr, Wi, sw, ldw, mur,
                       mui, nu, m, n, flag, status, (float*)C, ldc, cc);
}

void launch_crt_debug(hipStream_t s, Prec pr, const int8_t* W, size_t sw, int ldw, const int* mu,
                      const int* nu, int m, int n, const CrtConsts& cc, const int* flag, void* C,
                      int ldc, double* dbg) {
  const dim3 grid((unsigned)crt_blocks(m, n)), block(256);
  if (pr == Prec::F64)
    hipLaunchKernelGGL(k_crt_debug<double>, grid, block, 0, s, W, sw, ldw, mu, nu, m, n, cc, flag,
                       (double*)C, ldc, dbg);
  else
    hipLaunchKernelGGL(k_crt_debug<float>, grid, block, 0, s, W, sw, ldw, mu, nu, m, n, cc, flag,
                       (float*)C, ldc, dbg);
}

void launch_fill_zero(hipStream_t s, Prec pr, void* C, int ldc, int m, int n) {
  const int iblocks = (m + 255) / 256;
  dim3 grid((unsigned)iblocks * (unsigned)n);
  if (pr == Prec::F64)
    hipLaunchKernelGGL(k_fill_zero<double>, grid, dim3(256), 0, s, (double*)C, ldc, m, iblocks);
  else
    hipLaunchKernelGGL(k_fill_zero<float>, grid, dim3(256), 0, s, (float*)C, ldc, m, iblocks);
}

}  // namespace oz2
