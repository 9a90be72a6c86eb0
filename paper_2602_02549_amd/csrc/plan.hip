// Required number of moduli from the Theorem 1 bound (eq. thm:err-2).
//
// With alpha_i = floor(log2 max_h |a_ih|), beta_j likewise, and the row and
// column powers of two factored out of every quantity, the N-dependent part of
// the bound relative to S_ij = (|A||B|)_ij 2^-(alpha_i + beta_j) is
//   T_ij(N) = t(N) (rs_i sc_j + sr_i cs_j) + (k t(N)^2 + extra(N)) sr_i sc_j,
// where rs_i = sum_h |a_ih| 2^-alpha_i, cs_j likewise for B, sr_i =
// sqrt(max_h Cbar_ih) (2^(e'_i/2)), sc_j likewise, t(N) = 1/sqrt(2^5 (P-1)) and
// extra(N) t^-2 is r_b(N) minus its N-independent output-rounding part.
// rs, cs, sr, sc are rounded up and S_ij is replaced by a lower bound, so every
// decision errs towards a larger N.  Entries with S_ij = 0 are exact zeros and
// are skipped, unless the byte nz_ij (Cbar_ij != 0, which holds exactly when
// (|A||B|)_ij > 0) says the lower bound merely underflowed: such an entry
// accepts no N (and certifies no eps).
#include <cstdint>

#include "ozaki2_internal.h"

namespace oz2 {
namespace {

// Upward factors: FP64 sums of fewer than 2^19 nonnegative terms are within
// 2^-34 (relative) of the exact sum; one correctly rounded sqrt within 2^-53.
constexpr double kSumUp = 1.0 + 0x1p-30;
constexpr double kSqrtUp = 1.0 + 0x1p-50;
constexpr double kTUp = 1.0 + 0x1p-40;   // a few roundings in T itself

// One workgroup per 64 entries (rows of A first, then columns of B); its four
// waves sum every fourth tile of the partial sums, coalesced across the 64
// entries, and the four partial sums are added in a fixed order.
__global__ __launch_bounds__(256) void k_plan_vectors(const double* __restrict__ pr, int m_pad,
                                                      const double* __restrict__ pc, int n_pad,
                                                      int tiles, const int* __restrict__ rmax,
                                                      const int* __restrict__ cmax, int m, int n,
                                                      double* __restrict__ rs, double* __restrict__ cs,
                                                      double* __restrict__ sr,
                                                      double* __restrict__ sc) {
  __shared__ double part[4][64];
  const int e = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int t = blockIdx.x * 64 + e;
  const bool valid = t < m + n;
  const bool row = t < m;
  const int idx = row ? t : t - m;
  double s = 0.0;
  if (valid) {
    const double* p = row ? pr + idx : pc + idx;
    const int stride = row ? m_pad : n_pad;
    for (int q = g; q < tiles; q += 4) s += p[(size_t)q * stride];
  }
  part[g][e] = s;
  __syncthreads();
  if (g != 0 || !valid) return;
  s = (part[0][e] + part[1][e]) + (part[2][e] + part[3][e]);
  const double M = (double)(row ? rmax[idx] : cmax[idx]);
  if (row) {
    rs[idx] = s * kSumUp;
    sr[idx] = sqrt(M) * kSqrtUp;
  } else {
    cs[idx] = s * kSumUp;
    sc[idx] = sqrt(M) * kSqrtUp;
  }
}

__device__ inline bool plan_ok(const PlanTable& pt, int N, double A1, double P2, double target) {
  const double T = (pt.t[N] * A1 + (pt.k * pt.tt[N] + pt.extra[N]) * P2) * kTUp;
  return T <= target;
}

// The per-entry kernels below walk the m x n entries by waves in a grid-stride
// loop over tasks of 256 consecutive i of one column j, four rows per lane, and
// combine their results with one atomic per workgroup: one per 256 entries would
// serialise on the single result word (about 11 ns each).  With one row per lane
// and a division, a reduction or both per 256 entries they were bound by
// instructions: 64 us (plan_entries), 38 (plan_verify) and 74 (certify) at
// 4096^2 against 52, 25 and 58 so; the bytes take 13, 13 and 40.
constexpr int kEntryWorkgroups = 2048;

template <typename F>
__device__ __forceinline__ void for_quads(int m, int n, F&& f) {
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int blocks = cdiv_i(m, 256), stride = (int)gridDim.x * 4;
  const int first = (int)blockIdx.x * 4 + wave;
  const int dj = stride / blocks, db = stride - dj * blocks;
  int64_t j = first / blocks;
  int b = first % blocks;
  while (j < n) {
    f(b * 256 + 4 * lane, (int)j);
    j += dj;
    b += db;
    if (b >= blocks) {
      b -= blocks;
      ++j;
    }
  }
}

// v[i0 .. i0 + 3], past the last row m - 1 that one again.
template <typename T>
__device__ __forceinline__ void load_rows(const T* __restrict__ v, int i0, int m, T (&x)[4]) {
  if (i0 + 4 <= m) {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = v[i0 + e];
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = v[min(i0 + e, m - 1)];
  }
}

// Four entries of a column of S (columns lds_ apart, a multiple of 128) with
// their lower bounds: `pos` marks those with a positive one, `null` those that
// are nonzero without.
struct Quad {
  double Sl[4];
  bool pos[4], null[4];
  __device__ __forceinline__ Quad(const float* __restrict__ S, const uint8_t* __restrict__ nz,
                                  int lds_, int m, int i0, int j, double scale) {
    const size_t o = (size_t)j * lds_ + i0;
    const float4 v = *reinterpret_cast<const float4*>(S + o);
    const float w[4] = {v.x, v.y, v.z, v.w};
    bool some = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      Sl[e] = (double)w[e] * scale;
      pos[e] = i0 + e < m && Sl[e] > 0.0;
      null[e] = i0 + e < m && !(Sl[e] > 0.0);
      some |= null[e];
    }
    if (some) {
      const uint32_t b = *reinterpret_cast<const uint32_t*>(nz + o);
#pragma unroll
      for (int e = 0; e < 4; ++e) null[e] = null[e] && (b >> (8 * e) & 0xFF) != 0;
    }
  }
};

// Maximum of v over the workgroup (256 threads), valid in thread 0.
template <typename T>
__device__ __forceinline__ T block_max(T v) {
  for (int off = 32; off >= 1; off >>= 1) v = max(v, __shfl_xor(v, off));
  __shared__ T red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return max(max(red[0], red[1]), max(red[2], red[3]));
}

// Pass 1: a lower bound of the smallest N in [nlo, nhi] that satisfies
// T(N) <= eps S on every entry with S > 0 (nhi + 1 if an entry has none); the
// maximum over the workgroups goes to *out.  Each wave keeps a running bound
// `need` and, for its next 256 entries, looks for the first N >= need that
// each entry satisfies.  Any N that satisfies every entry is >= every such
// first N (by induction over the entries: it is >= each earlier bound, so it
// is one of the candidates searched), so the maximum stays a lower bound;
// pass 2 then searches upward from it.  Most entries pass at the running
// bound in one step.  N advances in step across the wave, so the per-N
// coefficients are wave-uniform (scalar) loads.
__global__ __launch_bounds__(256) void k_plan_entries(const float* __restrict__ S,
                                                      const uint8_t* __restrict__ nz, int lds_,
                                                      int m, int n, const double* __restrict__ rs,
                                                      const double* __restrict__ cs,
                                                      const double* __restrict__ sr,
                                                      const double* __restrict__ sc, PlanTable pt,
                                                      int* __restrict__ out) {
  int need = 0;   // wave-uniform running bound
  for_quads(m, n, [&](int i0, int j) {
    bool live[4] = {false, false, false, false};
    double A1[4], P2[4], target[4];
    if (i0 < m) {
      const Quad q(S, nz, lds_, m, i0, j, pt.acc_scale);
      double r[4], g[4];
      load_rows(rs, i0, m, r);
      load_rows(sr, i0, m, g);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        A1[e] = r[e] * sc[j] + g[e] * cs[j];
        P2[e] = g[e] * sc[j];
        // nonzero (|A||B|)_ij with no positive lower bound: T >= 0 never meets
        // -1, so no N is accepted
        target[e] = q.pos[e] ? pt.eps * q.Sl[e] : -1.0;
        live[e] = q.pos[e] || q.null[e];
      }
    }
    int found = 0;
    for (int N = max(pt.nlo, need); N <= pt.nhi; ++N) {
      if (!__any(live[0] || live[1] || live[2] || live[3])) break;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (live[e] && plan_ok(pt, N, A1[e], P2[e], target[e])) {
          found = N;
          live[e] = false;
        }
    }
    if (live[0] || live[1] || live[2] || live[3]) found = pt.nhi + 1;
    if (__any(found > need)) {
      for (int off = 32; off >= 1; off >>= 1) found = max(found, __shfl_xor(found, off));
      need = __builtin_amdgcn_readfirstlane(max(need, found));
    }
  });
  need = block_max(need);
  if (threadIdx.x == 0 && need > 0) atomicMax(out, need);
}

// Pass 2: does N satisfy every entry?  Any failure sets *bad.  With Nsrc,
// N is read from there (pass 1's result, at least nlo), and nothing is
// checked if it exceeds nhi.
__global__ __launch_bounds__(256) void k_plan_verify(const float* __restrict__ S,
                                                     const uint8_t* __restrict__ nz, int lds_, int m,
                                                     int n, const double* __restrict__ rs,
                                                     const double* __restrict__ cs,
                                                     const double* __restrict__ sr,
                                                     const double* __restrict__ sc, PlanTable pt,
                                                     int N, const int* __restrict__ Nsrc,
                                                     int* __restrict__ bad) {
  if (Nsrc) N = max(__builtin_amdgcn_readfirstlane(*Nsrc), pt.nlo);
  if (N > pt.nhi) return;   // uniform: before any barrier
  int fail = 0;
  for_quads(m, n, [&](int i0, int j) {
    if (i0 >= m) return;
    const Quad q(S, nz, lds_, m, i0, j, pt.acc_scale);
    double r[4], g[4];
    load_rows(rs, i0, m, r);
    load_rows(sr, i0, m, g);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double A1 = r[e] * sc[j] + g[e] * cs[j];
      const double P2 = g[e] * sc[j];
      if (q.null[e] || (q.pos[e] && !plan_ok(pt, N, A1, P2, pt.eps * q.Sl[e]))) fail = 1;
    }
  });
  fail = block_max(fail);
  if (threadIdx.x == 0 && fail) atomicOr(bad, 1);
}

// A-posteriori est1 of Theorem 1 (eq. thm:err-1) relative to the lower bound
// of S, per entry.  |A'B'| is bounded through Lemma 4 by the computed C'':
// |A'B'| <= (|C''| + R_const) / (1 - R_rel).  C'' is recovered from the output
// and the shifts: C = C'' 2^-(mu_i + nu_j) rounded once, exactly unless C is
// subnormal, so |C''| <= (|C| + tiny) 2^(mu_i + nu_j) in every case (for b = 32
// this is the FP32 C'' of Algorithm 3, to which Lemma 4 refers).  In factored
// form (row and column powers of two removed, as in the planner):
//   est1 = t A1 + (k t^2 + R_const t^2 + rel (|C''| + R_const)) P2,
// every rounding pushed upward.  The maximum of est1 / S over entries with
// S > 0 goes to *out as the bit pattern of a nonnegative double (whose order
// is that of the unsigned integers).
template <typename T>
__global__ __launch_bounds__(256) void k_certify(const T* __restrict__ C, int ldc,
                                                 const int* __restrict__ mu,
                                                 const int* __restrict__ nu,
                                                 const float* __restrict__ S,
                                                 const uint8_t* __restrict__ nz, int lds_, int m,
                                                 int n, const double* __restrict__ rs,
                                                 const double* __restrict__ cs,
                                                 const double* __restrict__ sr,
                                                 const double* __restrict__ sc, CertTable ct,
                                                 unsigned long long* __restrict__ out) {
  double ratio = 0.0;
  for_quads(m, n, [&](int i0, int j) {
    if (i0 >= m) return;
    const Quad q(S, nz, lds_, m, i0, j, ct.acc_scale);
    double r[4], g[4];
    int u[4];
    T c[4];
    load_rows(rs, i0, m, r);
    load_rows(sr, i0, m, g);
    load_rows(mu, i0, m, u);
    load_rows(C + (size_t)j * ldc, i0, m, c);
    const int nuj = nu[j];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (q.null[e]) ratio = INFINITY;   // nonzero (|A||B|)_ij with no positive lower bound
      if (!q.pos[e]) continue;
      const double cpp = ldexp(fabs((double)c[e]) + ct.tiny, u[e] + nuj);
      const double A1 = r[e] * sc[j] + g[e] * cs[j];
      const double P2 = g[e] * sc[j];
      const double est =
          (ct.t * A1 + (ct.k * ct.tt + ct.extra + ct.rel * (cpp + ct.rconst) * kTUp) * P2) * kTUp;
      // the quotient only where it can be the maximum
      if (!(est <= ratio * q.Sl[e] * (1.0 - 0x1p-20))) ratio = fmax(ratio, est / q.Sl[e] * kTUp);
    }
  });
  ratio = block_max(ratio);
  if (threadIdx.x == 0 && ratio > 0.0)
    atomicMax(out, (unsigned long long)__double_as_longlong(ratio));
}

unsigned entry_grid(int m, int n) {
  const int64_t groups = ((int64_t)cdiv_i(m, 256) * n + 3) / 4;
  return (unsigned)(groups < kEntryWorkgroups ? groups : kEntryWorkgroups);
}

}  // namespace

void launch_certify(hipStream_t s, Prec pr, const void* C, int ldc, const int* mu, const int* nu,
                    const float* S, const uint8_t* nz, int lds_, int m, int n, const double* rs,
                    const double* cs, const double* sr, const double* sc, const CertTable& ct,
                    unsigned long long* out) {
  const dim3 grid(entry_grid(m, n)), block(256);
  if (pr == Prec::F64)
    hipLaunchKernelGGL(k_certify<double>, grid, block, 0, s, (const double*)C, ldc, mu, nu, S, nz,
                       lds_, m, n, rs, cs, sr, sc, ct, out);
  else
    hipLaunchKernelGGL(k_certify<float>, grid, block, 0, s, (const float*)C, ldc, mu, nu, S, nz,
                       lds_, m, n, rs, cs, sr, sc, ct, out);
}

void launch_plan_vectors(hipStream_t s, const double* pr, int m_pad, const double* pc, int n_pad,
                         int tiles, const int* rmax, const int* cmax, int m, int n, double* rs,
                         double* cs, double* sr, double* sc) {
  hipLaunchKernelGGL(k_plan_vectors, dim3((m + n + 63) / 64), dim3(256), 0, s, pr, m_pad, pc,
                     n_pad, tiles, rmax, cmax, m, n, rs, cs, sr, sc);
}

void launch_plan_entries(hipStream_t s, const float* S, const uint8_t* nz, int lds_, int m, int n,
                         const double* rs, const double* cs, const double* sr, const double* sc,
                         const PlanTable& pt, int* out) {
  hipLaunchKernelGGL(k_plan_entries, dim3(entry_grid(m, n)), dim3(256), 0, s, S, nz,
                     lds_, m, n, rs, cs, sr, sc, pt, out);
}

void launch_plan_verify(hipStream_t s, const float* S, const uint8_t* nz, int lds_, int m, int n,
                        const double* rs, const double* cs, const double* sr, const double* sc,
                        const PlanTable& pt, int N, const int* Nsrc, int* bad) {
  hipLaunchKernelGGL(k_plan_verify, dim3(entry_grid(m, n)), dim3(256), 0, s, S, nz,
                     lds_, m, n, rs, cs, sr, sc, pt, N, Nsrc, bad);
}

}  // namespace oz2
