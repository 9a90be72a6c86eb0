// Scaling-vector kernels of Algorithm 2 (Section 3.2):
//   - per-row / per-column maximum of |a| (kept as the IEEE bit pattern of
//     the FP64 value, whose unsigned order equals the numeric order), from
//     which mu' = 5 - floor(log2 max|a|) follows exactly, and the bars that mu'
//     scales;
//   - log2f, correctly rounded to FP32 (double-double series evaluation), for
//     the stage dumps and the exhaustive check; the final shifts mu = mu' +
//     floor(fma_down(c, e, P')), e = log2f(single_up(max_j Cbar_ij)), come from
//     their table of steps where they are used (shift_of).
#include <cstdint>

#include "ozaki2_internal.h"

namespace oz2 {
namespace {

// ---------------------------------------------------------------------------
// The scan: abs-max bit patterns and bars of both operands of Algorithm 2,
//   bits_i = max_h |a_ih|,  Abar = ceil(2^mu' |A|)  (and of B's columns),
// with the maxima of Cbar and the non-finite flag cleared for the kernels that
// follow, in one launch.  HBM bound; what it saves is the second read of A
// (from HBM to the workgroup's registers, to L2 or to the MALL) and launches.
//   A (column-major): a workgroup takes a strip of rows over all of k, 16
//     consecutive k of one row per thread: 128 bytes of each column for k >= 512,
//     more rows for a shorter k, so that every thread has work.  It reduces the
//     rows' maxima, keeps its first chunks of k in registers and reads the
//     others again, latest first, for the bars, whose 16 bytes per thread go
//     through LDS so that rows are written in whole lines.
//   B (k contiguous): 4 to 64 lanes (up to kColWaveK) or a workgroup take a
//     column, 4 consecutive k per thread, up to 32 elements per thread kept in
//     registers and the others read again.
// The launch rate of waves, about one a nanosecond, bounds batches of small
// problems: a wave per column and 16-row strips took 406 us on 2048 problems
// of 128^3.
// A strip reads all of k by itself, so few strips over a long k would leave the
// GPU idle: see strips_fit.  There A's maxima run over chunks of columns, those
// of few columns of B over chunks of rows (cols_chunked), with one atomic per
// chunk and row (one per wave or thread took 110 us at 64x64x262144, these 58:
// the atomics of a row go one at a time), and the bars in the slice kernel.
constexpr int kScanThreads = 512;
constexpr int kColWaveK = 2048;

// Rows of a strip for k_pad as a power of two: 16 k per thread over 512 threads,
// at least 128 bytes of a column, at most a wave of rows.  `fine` (a launch of
// few workgroups, which waits for latency and not for the launch rate): the
// fewest rows, and a wave per column below.
template <typename T>
constexpr int kMinStripLog2 = sizeof(T) == 8 ? 4 : 5;
template <typename T>
__host__ __device__ inline int strip_rows_log2(int k_pad, bool fine) {
  int lr = fine ? kMinStripLog2<T> : 6;
  while (lr > kMinStripLog2<T> && (kScanThreads >> lr) * 16 < k_pad) --lr;
  return lr;
}
// Threads per column for k_pad: the fewest that keep it in registers (keep
// elements a thread), a wave up to wave_k, else a workgroup.
__host__ __device__ inline int col_threads(int k_pad, int keep, bool fine,
                                           int wave_k = kColWaveK) {
  if (k_pad > wave_k) return kScanThreads;
  int tpc = fine ? 64 : 4;
  while (tpc < 64 && tpc * keep < k_pad) tpc *= 2;
  return tpc;
}
// In a batch of many workgroups, which the launch rate of waves bounds, a wave takes
// columns of up to 32 KB.  Whole batches with a workgroup and with a wave a column:
// FP32, 200 of 64 x 64 x 2500 791 and 688 us (778 before the merged scan), 40 of 500 x
// 700 x 2100 903 and 781, 20 of 100 x 1000 x 6000 889 and 812; FP64, 200 of 64 x 64 x
// 2500 1192 and 1107, but 20 of 300 x 300 x 8000 1276 and 1303.
__host__ __device__ inline int group_wave_k(bool fine, size_t size) {
  return fine ? kColWaveK : (int)(32768 / size);
}
// Whether `units` workgroups of the finest split are few.
__host__ __device__ inline bool scan_fine(int64_t units) { return units <= 512; }
template <SliceSet F>
constexpr int kColKeep = F == SliceSet::Real ? 32 : 16;   // elements (pairs) a thread

// One operand of the scan (real, or interleaved pairs for the complex forms).
struct ScanSide {
  const void* src;
  uint64_t* bits;
  int* mx;
  int8_t* out;
  int ld, rows, rows_pad;
  int units;       // workgroups
};
struct ScanArgs {
  ScanSide a, b;
  int* flag;
  int k, k_pad;    // k_pad: padded k (the embedding: of one k half)
  int half;        // the embedding: rows of one row half of A
  int lr;          // log2 of the rows of a strip
  int tpc;         // threads per column
  int chunked;     // A's units are chunks, for the abs-max only
  int tr;          // rows of such a chunk
  int cols_chunked;   // so are B's: kColChunk elements of a column each
};

template <typename T>
__device__ __forceinline__ uint64_t abs_bits(T x) {
  return (uint64_t)__double_as_longlong(fabs((double)x));
}
__device__ __forceinline__ uint64_t max64(uint64_t a, uint64_t b) { return a > b ? a : b; }

// Bar byte of Algorithm 2: ceil(2^sh |x|), 1 for a tiny nonzero x, 0 for 0.
__device__ __forceinline__ int bar_of(double x, int sh) {
  const double a = fabs(x), cl = ceil(ldexp(a, sh));
  return a == 0.0 ? 0 : (cl < 1.0 ? 1 : (int)cl);
}

// The bars of one element in the form's slices: real b0; the 3-product form
// b0 = bar(re) + bar(im); the embedding b0 = bar(re), b1 = bar(im).
template <typename T, SliceSet F>
__device__ __forceinline__ void bars_of(T re, T im, int sh, int* b0, int* b1) {
  *b0 = bar_of((double)re, sh);
  if constexpr (F != SliceSet::Real) {
    const int i = bar_of((double)im, sh);
    if constexpr (F == SliceSet::Complex3) *b0 += i;
    *b1 = i;
  }
}

// By thread t of `stride` (at most 2^31, so that no index wraps).
__device__ __forceinline__ void scan_clear(int* mx_a, int na, int* mx_b, int nb, int* flag,
                                           unsigned t, unsigned stride) {
  for (unsigned i = t; i < (unsigned)na; i += stride) mx_a[i] = 0;
  for (unsigned j = t; j < (unsigned)nb; j += stride) mx_b[j] = 0;
  if (t == 0) *flag = 0;
}

// Workgroups of a scan in two grid dimensions: a launch takes fewer than 2^32
// threads along x, which 2^23 columns of more than kColWaveK rows, a workgroup
// each (69 GB of FP32), would exceed.
constexpr int kScanGridX = 1 << 22;
inline dim3 scan_grid(int units) {
  return dim3((unsigned)(units < kScanGridX ? units : kScanGridX),
              (unsigned)((units - 1) / kScanGridX + 1));
}
__device__ __forceinline__ int scan_unit() {
  return (int)(blockIdx.y * gridDim.x + blockIdx.x);
}

// LDS of a strip: maxima per wave and row, and the bars of one chunk (two for
// the embedding), 16 bytes of padding per row.
template <SliceSet F>
struct StripLds {
  unsigned long long red[kScanThreads / 64][64];
  int8_t bars[F == SliceSet::Embedding ? 2 : 1][16 * kScanThreads + 16 * 64];
};

// Strip `u` of A, 2^lr rows.
template <typename T, SliceSet F>
__device__ __forceinline__ void scan_strip(const T* __restrict__ src, int ld, int rows, int k,
                                           int k_pad, int half, uint64_t* __restrict__ bits,
                                           int8_t* __restrict__ out, int u, int lr,
                                           StripLds<F>& lds) {
  constexpr int E = F == SliceSet::Real ? 1 : 2;
  constexpr bool kEmb = F == SliceSet::Embedding;
  constexpr int KEEP = E == 1 ? 2 : 1;                   // chunks kept in registers
  const int R = 1 << lr, lg = 9 - lr, KG = 1 << lg;      // rows, threads per row
  const int CH = 16 << lg, row_bytes = CH + 16;          // k per pass
  static_assert(kScanThreads == 1 << 9, "threads");
  const int t = threadIdx.x, row = t & (R - 1), kg = t >> lr;
  const int r0 = u * R, rg = r0 + row;
  const bool in = rg < rows;
  const int ldo = kEmb ? 2 * k_pad : k_pad;
  const uint32_t rc = (uint32_t)(min(rg, rows - 1) - r0);
  const int nch = (k_pad + CH - 1) / CH;
  // 16 loads before any use; clamped to the matrix (a repeated element of the
  // row does not change its maximum)
  auto load = [&](int c, T (&x)[16], T (&y)[16]) {
    // uniform, with offsets below 2^32 (strips_fit)
    const char* base =
        reinterpret_cast<const char*>(src + (size_t)E * (r0 + (size_t)(c * CH) * ld));
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const uint32_t h = (uint32_t)min(16 * kg + e, k - 1 - c * CH);
      const T* p =
          reinterpret_cast<const T*>(base + (h * (uint32_t)ld + rc) * (uint32_t)(E * sizeof(T)));
      x[e] = p[0];
      y[e] = E == 2 ? p[E - 1] : (T)0;
    }
  };
  uint64_t mx = 0;
  auto take = [&](const T (&x)[16], const T (&y)[16]) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      mx = max64(mx, abs_bits(x[e]));
      if (E == 2) mx = max64(mx, abs_bits(y[e]));
    }
  };
  T kx[KEEP][16], ky[KEEP][16];
  const bool some = r0 < rows;                           // uniform: any real row
  if (some) {
#pragma unroll
    for (int c = 0; c < KEEP; ++c)
      if (c < nch) load(c, kx[c], ky[c]);
#pragma unroll
    for (int c = 0; c < KEEP; ++c)
      if (c < nch) take(kx[c], ky[c]);
    for (int c = KEEP; c < nch; ++c) {
      T x[16], y[16];
      load(c, x, y);
      take(x, y);
    }
  }
  for (int off = R; off < 64; off <<= 1) mx = max64(mx, __shfl_xor((unsigned long long)mx, off));
  if ((t & 63) < R) lds.red[t >> 6][row] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) mx = max64(mx, lds.red[w][row]);
  if (in && kg == 0) {
    bits[rg] = mx;
    if (kEmb) bits[half + rg] = mx;                      // both row blocks of the embedding
  }
  const int sh = shift_prime_bits(mx) - (F == SliceSet::Complex3 ? 1 : 0);
  auto put = [&](int c, const T (&x)[16], const T (&y)[16]) {
    const int h = c * CH + 16 * kg;
    uint32_t w0[4] = {0, 0, 0, 0}, w1[4] = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      int b0 = 0, b1 = 0;
      bars_of<T, F>(x[e], y[e], sh, &b0, &b1);
      const bool ok = in && h + e < k;
      w0[e >> 2] |= (ok ? (uint32_t)b0 & 0xFF : 0u) << (8 * (e & 3));
      if (kEmb) w1[e >> 2] |= (ok ? (uint32_t)b1 & 0xFF : 0u) << (8 * (e & 3));
    }
    int8_t* const q = &lds.bars[0][row * row_bytes + 16 * kg];
    *reinterpret_cast<uint4*>(q) = make_uint4(w0[0], w0[1], w0[2], w0[3]);
    if (kEmb)
      *reinterpret_cast<uint4*>(q + sizeof(lds.bars[0])) = make_uint4(w1[0], w1[1], w1[2], w1[3]);
    __syncthreads();
    // 16 bytes of row r, rows in whole lines
    const int r = t >> lg, ho = c * CH + 16 * (t & (KG - 1));
    if (ho < k_pad) {
      const int8_t* p = &lds.bars[0][r * row_bytes + 16 * (t & (KG - 1))];
      const uint4 v = *reinterpret_cast<const uint4*>(p);
      int8_t* d = out + (size_t)(r0 + r) * ldo + ho;
      *reinterpret_cast<uint4*>(d) = v;
      if (kEmb) {
        const uint4 v1 = *reinterpret_cast<const uint4*>(p + sizeof(lds.bars[0]));
        int8_t* d2 = d + (size_t)half * ldo;             // the row of the lower block
        *reinterpret_cast<uint4*>(d + k_pad) = v1;
        *reinterpret_cast<uint4*>(d2) = v1;
        *reinterpret_cast<uint4*>(d2 + k_pad) = v;
      }
    }
    __syncthreads();
  };
  for (int c = nch - 1; c >= KEEP; --c) {
    T x[16], y[16];
    if (some) load(c, x, y);
    put(c, x, y);
  }
#pragma unroll
  for (int c = KEEP - 1; c >= 0; --c)
    if (c < nch) put(c, kx[c], ky[c]);
}

// Workgroup `u` of B's columns.
template <typename T, SliceSet F>
__device__ __forceinline__ void scan_cols(const T* __restrict__ src, int ld, int n, int n_pad,
                                          int k, int k_pad, uint64_t* __restrict__ bits,
                                          int8_t* __restrict__ out, int u, int tpc,
                                          unsigned long long* __restrict__ red) {
  constexpr int E = F == SliceSet::Real ? 1 : 2;
  constexpr bool kEmb = F == SliceSet::Embedding;
  constexpr int KEEP = kColKeep<F> / 4;                  // quads kept in registers
  const int t = (int)threadIdx.x & (tpc - 1);
  const int j = u * (kScanThreads / tpc) + (int)threadIdx.x / tpc;
  const bool in = j < n;                                 // j < n_pad: whole units
  const T* col = src + (size_t)E * ((size_t)min(j, n - 1) * ld);
  const int ldo = kEmb ? 2 * k_pad : k_pad;
  const int span = 4 * tpc, nq = (k_pad + span - 1) / span;
  auto load = [&](int q, T (&x)[4], T (&y)[4]) {
    const int h = 4 * t + span * q;
    const T* p = col + (size_t)E * h;
    if (span * (q + 1) <= k) {                           // uniform: the whole pass is inside
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[e] = p[E * e];
        y[e] = E == 2 ? p[E * e + E - 1] : (T)0;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const T* c = col + (size_t)E * min(h + e, k - 1);
        x[e] = c[0];
        y[e] = E == 2 ? c[E - 1] : (T)0;
      }
    }
  };
  uint64_t mx = 0;
  auto take = [&](const T (&x)[4], const T (&y)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      mx = max64(mx, abs_bits(x[e]));
      if (E == 2) mx = max64(mx, abs_bits(y[e]));
    }
  };
  T kx[KEEP][4], ky[KEEP][4];
  if (in) {
#pragma unroll
    for (int q = 0; q < KEEP; ++q)
      if (q < nq) load(q, kx[q], ky[q]);
#pragma unroll
    for (int q = 0; q < KEEP; ++q)
      if (q < nq) take(kx[q], ky[q]);
    for (int q = KEEP; q < nq; q += 4) {
      T x[4][4], y[4][4];
#pragma unroll
      for (int v = 0; v < 4; ++v) load(min(q + v, nq - 1), x[v], y[v]);
#pragma unroll
      for (int v = 0; v < 4; ++v) take(x[v], y[v]);
    }
  }
  for (int off = 1; off < min(tpc, 64); off <<= 1)
    mx = max64(mx, __shfl_xor((unsigned long long)mx, off));
  if (tpc > 64) {                                        // uniform
    if ((t & 63) == 0) red[t >> 6] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) mx = max64(mx, red[w]);
  }
  if (in && t == 0) bits[j] = mx;
  const int sh = shift_prime_bits(mx) - (F == SliceSet::Complex3 ? 1 : 0);
  int8_t* dst = out + (size_t)j * ldo;
  auto put = [&](int q, const T (&x)[4], const T (&y)[4]) {
    const int h = 4 * t + span * q;
    if (h >= k_pad) return;
    uint32_t w0 = 0, w1 = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      int b0 = 0, b1 = 0;
      bars_of<T, F>(x[e], y[e], sh, &b0, &b1);
      const bool ok = in && h + e < k;
      w0 |= (ok ? (uint32_t)b0 & 0xFF : 0u) << (8 * e);
      if (kEmb) w1 |= (ok ? (uint32_t)b1 & 0xFF : 0u) << (8 * e);
    }
    *reinterpret_cast<uint32_t*>(dst + h) = w0;
    if (kEmb) *reinterpret_cast<uint32_t*>(dst + k_pad + h) = w1;
  };
  for (int q = nq - 1; q >= KEEP; q -= 4) {
    T x[4][4], y[4][4];
    if (in) {
#pragma unroll
      for (int v = 0; v < 4; ++v) load(max(q - v, KEEP), x[v], y[v]);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (q - v >= KEEP) put(q - v, x[v], y[v]);
  }
#pragma unroll
  for (int q = KEEP - 1; q >= 0; --q)
    if (q < nq) put(q, kx[q], ky[q]);
}

// Abs-max of row i over the 64 columns from h0 of the column-major A, 16 loads
// at a time from clamped addresses (0 past the last column).
template <typename T, SliceSet F>
__device__ __forceinline__ uint64_t absmax_row_part(const T* __restrict__ A, int lda, int m, int k,
                                                    int i, int h0) {
  constexpr int E = F == SliceSet::Real ? 1 : 2;
  const T* a = A + (size_t)E * min(i, m - 1);
  uint64_t mx = 0;
  if (h0 >= k) return mx;
#pragma unroll
  for (int q0 = 0; q0 < 64; q0 += 16) {
    T x[16], y[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const T* e = a + (size_t)E * ((size_t)min(h0 + q0 + u, k - 1) * lda);
      x[u] = e[0];
      y[u] = E == 2 ? e[E - 1] : (T)0;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      mx = max64(mx, abs_bits(x[u]));
      if (E == 2) mx = max64(mx, abs_bits(y[u]));
    }
  }
  return mx;
}

// Abs-max of chunk p of A by a workgroup (atomicMax on bits that a launch before
// has cleared): tr rows by kScanThreads / tr times 64 columns, combined in LDS
// first, since the atomics of a row go one at a time.
__host__ __device__ inline int chunk_rows(int m) { return m > 128 ? 256 : m > 64 ? 128 : 64; }
__host__ __device__ inline int row_chunks(int m, int k, int tr) {
  return cdiv_i(m, tr) * cdiv_i(k, 64 * (kScanThreads / tr));
}
template <typename T, SliceSet F>
__device__ __forceinline__ void absmax_row_chunk(const T* __restrict__ A, int lda, int m, int k,
                                                 int half, uint64_t* __restrict__ bits, int p,
                                                 int tr, unsigned long long* __restrict__ red) {
  const int t = (int)threadIdx.x, gx = cdiv_i(m, tr), groups = kScanThreads / tr;
  const int i = p % gx * tr + (t & (tr - 1));
  uint64_t mx = absmax_row_part<T, F>(A, lda, m, k, i, (p / gx * groups + t / tr) * 64);
  red[t] = mx;
  __syncthreads();
  if (t >= tr || i >= m) return;
  for (int g = 1; g < groups; ++g) mx = max64(mx, red[g * tr + t]);
  if (!mx) return;
  atomicMax((unsigned long long*)&bits[i], (unsigned long long)mx);
  if (F == SliceSet::Embedding)
    atomicMax((unsigned long long*)&bits[i + half], (unsigned long long)mx);
}

// Abs-max of chunk u of B: kColChunk elements of one column, 16 per thread in
// quads (the first column index fastest, so that chunks of a column do not
// meet at its maximum).
constexpr int kColChunk = 16 * kScanThreads;
template <typename T, SliceSet F>
__device__ __forceinline__ void absmax_col_chunk(const T* __restrict__ B, int ldb, int n, int k,
                                                 uint64_t* __restrict__ bits, int u,
                                                 unsigned long long* __restrict__ red) {
  constexpr int E = F == SliceSet::Real ? 1 : 2;
  const int j = u % n, c0 = u / n * kColChunk, h0 = c0 + (int)threadIdx.x * 4;
  const T* b = B + (size_t)E * ((size_t)j * ldb);
  uint64_t mx = 0;
  if (c0 + kColChunk <= k) {                             // uniform: the whole chunk is inside
    const T* p = b + (size_t)E * h0;
    T x[16 * E];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4 * E; ++e) x[4 * E * q + e] = p[E * (4 * kScanThreads * q) + e];
#pragma unroll
    for (int q = 0; q < 16 * E; ++q) mx = max64(mx, abs_bits(x[q]));
  } else {
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const T* p = b + (size_t)E * min(h0 + 4 * kScanThreads * q + e, k - 1);
        mx = max64(mx, abs_bits(p[0]));
        if (E == 2) mx = max64(mx, abs_bits(p[E - 1]));
      }
  }
  for (int off = 1; off < 64; off <<= 1) mx = max64(mx, __shfl_xor((unsigned long long)mx, off));
  red[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x) return;
  for (int w = 1; w < kScanThreads / 64; ++w) mx = max64(mx, red[w]);
  if (mx) atomicMax((unsigned long long*)&bits[j], (unsigned long long)mx);
}

template <typename T, SliceSet F>
__global__ __launch_bounds__(kScanThreads, F == SliceSet::Real ? 4 : 2) void k_scan(ScanArgs s) {
  __shared__ StripLds<F> lds;
  const int u = scan_unit();
  if (u >= s.a.units + s.b.units) return;                // whole workgroup
  if (blockIdx.y == 0)                                   // at most 2^31 threads
    scan_clear(s.a.mx, s.a.rows_pad, s.b.mx, s.b.rows_pad, s.flag,
               blockIdx.x * kScanThreads + threadIdx.x, gridDim.x * kScanThreads);
  if (u >= s.a.units)
    scan_cols<T, F>(static_cast<const T*>(s.b.src), s.b.ld, s.b.rows, s.b.rows_pad, s.k, s.k_pad,
                    s.b.bits, s.b.out, u - s.a.units, s.tpc, &lds.red[0][0]);
  else
    scan_strip<T, F>(static_cast<const T*>(s.a.src), s.a.ld, s.a.rows, s.k, s.k_pad, s.half,
                     s.a.bits, s.a.out, u, s.lr, lds);
}

// The chunked scan, in a kernel of its own for the registers of k_scan.
template <typename T, SliceSet F>
__global__ __launch_bounds__(kScanThreads, F == SliceSet::Real ? 4 : 2) void k_scan_chunks(
    ScanArgs s) {
  __shared__ unsigned long long red[kScanThreads];
  const int u = scan_unit();
  if (u >= s.a.units + s.b.units) return;                // whole workgroup
  if (u < s.a.units)
    absmax_row_chunk<T, F>(static_cast<const T*>(s.a.src), s.a.ld, s.a.rows, s.k, s.half, s.a.bits,
                           u, s.tr, red);
  else if (s.cols_chunked)
    absmax_col_chunk<T, F>(static_cast<const T*>(s.b.src), s.b.ld, s.b.rows, s.k, s.b.bits,
                           u - s.a.units, red);
  else
    scan_cols<T, F>(static_cast<const T*>(s.b.src), s.b.ld, s.b.rows, s.b.rows_pad, s.k, s.k_pad,
                    s.b.bits, s.b.out, u - s.a.units, s.tpc, red);
}

// What the atomics of a chunked scan need cleared, with the maxima and the flag.
__global__ __launch_bounds__(256) void k_clear(uint64_t* bits, int* mx_a, int na, uint64_t* bits_b,
                                               int* mx_b, int nb, int* flag) {
  const unsigned t = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
  for (unsigned i = t; i < (unsigned)na; i += stride) bits[i] = 0;
  if (bits_b)
    for (unsigned j = t; j < (unsigned)nb; j += stride) bits_b[j] = 0;
  scan_clear(mx_a, na, mx_b, nb, flag, t, stride);
}

// Strips over all of k: each strip streams its columns by itself in passes of 512 k
// (FP64; 256 for FP32, whose strips have twice the rows), waiting for one after the
// other, and all but the first twice.  A chunked scan moves the same bytes at the rate
// of memory, for two or three launches more (about 10 us).  A round of 256 strips
// takes 7 us a pass, as chunks of as much do, a partial one 4 to 5 however few strips
// it has.  So strips are taken for few passes, the more the fuller their rounds, and
// for whole rounds up to 24576 of k (longer ones fall behind).  Scans of FP64 with
// strips and in chunks: 96 strips of 9 passes 32 and 32 us, of 16 52 and 45, of 32 131
// and 80; 192 of 16 72 and 77, of 32 193 and 178; 384 of 16 172 and 172, of 32 376 and
// 343; 256 of 32 222 and 236, of 137 1052 and 985; 512 of 16 203 and 234, of 137 2085
// and 1995.  (Strips of every k from 96 on, the rule before, lost up to 40% to the
// separate passes that the scan replaced.)  FP32 calls: cgemm 130 x 1000 x 4096 161
// and 124 us, sgemm of 16 x 16 x 3000 53 and 41, of 2000 x 3000 x 2100 163 and 169.
// More passes also fit, up to 4096 of k, while the n columns of B, which start a
// workgroup every 8 ns, and chunks of as many rows take as long as the strips (sgemm
// of 2304^3 149 and 153), and beside the other problems of a batch of many
// workgroups (`many`).
// A pass of a strip addresses its columns with 32 bits (pitch: bytes from one to
// the next), which saves the registers that 64-bit addresses spilled: 16.5 and
// 13.5 us at 1000x700x1300.
__host__ __device__ inline bool strips_fit(int rows_pad, int lr, int k, int n, bool many,
                                           size_t pitch) {
  const int pass = 16 << (9 - lr), passes = (k + pass - 1) >> (13 - lr);
  const int64_t strips = rows_pad >> lr, rounds = (strips + 255) >> 8;
  const bool brief =
      passes <= 8 || (k <= 4096 && (many || 450 * passes <= n + 16 * strips + 1250));
  const bool full = 16 * strips >= 15 * 256 * rounds;
  return (brief || (full ? k <= 24576 : 16 * (passes - 4) * rounds <= strips)) &&
         (size_t)((pass < k ? pass : k) + 1) * pitch < (size_t)1 << 32;
}

// B's columns in chunks too, with bars in the slice kernel.  By columns, a
// workgroup streams each twice, which is as much traffic in less work but leaves
// most compute units idle when there are few.  Whole calls by columns and in
// chunks: 60 columns of 100000 493 and 474 us, 64 of 262144 533 and 445; 128 of
// 16384 69 and 71, 200 of 100000 479 and 493.  Pairs of FP32 always go in chunks: a
// workgroup streams them no faster than pairs of FP64, for half the bytes (N = 2, 64
// x 2000 x 100000, both forms: by columns 2230 and 2320 us, in chunks 1540 and 1600;
// in FP64 2370 and 2440, in chunks 2510 and 2610).
template <typename T, SliceSet F>
bool cols_chunked(int n) {
  return n <= 100 || (F != SliceSet::Real && sizeof(T) == 4);
}

// ---------------------------------------------------------------------------
// double-double helpers (Dekker / Knuth error-free transformations)
// ---------------------------------------------------------------------------
struct dd {
  double h, l;
};
__device__ inline dd two_sum(double a, double b) {
  double s = a + b;
  double bb = s - a;
  return {s, (a - (s - bb)) + (b - bb)};
}
__device__ inline dd fast_two_sum(double a, double b) {  // |a| >= |b|
  double s = a + b;
  return {s, b - (s - a)};
}
__device__ inline dd dd_add(dd a, dd b) {
  dd s = two_sum(a.h, b.h);
  double e = s.l + (a.l + b.l);
  return fast_two_sum(s.h, e);
}
__device__ inline dd dd_mul(dd a, dd b) {
  double p = a.h * b.h;
  double e = fma(a.h, b.h, -p);
  e = fma(a.h, b.l, e);
  e = fma(a.l, b.h, e);
  return fast_two_sum(p, e);
}
__device__ inline dd dd_recip_int(int q) {  // 1/q as a double-double
  double h = 1.0 / (double)q;
  double r = fma(-h, (double)q, 1.0);      // exact remainder
  return {h, r / (double)q};
}

// log2 of an integer-valued d in [1, 2^30), rounded to nearest FP32.
// d = 2^E m with m in (1/sqrt2, sqrt2]; ln m = 2 atanh(z), z = (m-1)/(m+1),
// |z| <= 0.1716, summed to 23 terms in double-double (error < 2^-100), then
// multiplied by 1/ln2 (double-double constant).  The FP32 rounding of a
// double-double h + l is RN(h) unless h is exactly an FP32 midpoint, in which
// case the sign of l decides.
__device__ float log2f_rn(float dval) {
  double d = (double)dval;
  int E = ilogb(d);
  double mnt = ldexp(d, -E);
  if (mnt > 1.4142135623730951) {
    mnt *= 0.5;
    E += 1;
  }
  double num = mnt - 1.0;   // exact: mnt has at most 31 significant bits
  double den = mnt + 1.0;   // exact
  double zh = num / den;
  double zl = fma(-zh, den, num) / den;
  dd z = {zh, zl};
  dd z2 = dd_mul(z, z);
  dd T = dd_recip_int(2 * 22 + 1);
  for (int j = 21; j >= 0; --j) T = dd_add(dd_recip_int(2 * j + 1), dd_mul(z2, T));
  dd ln = dd_mul(z, T);
  ln.h *= 2.0;
  ln.l *= 2.0;
  const dd log2e = {0x1.71547652b82fep+0, 0x1.777d0ffda0d24p-56};
  dd r = dd_add(dd_mul(ln, log2e), dd{(double)E, 0.0});
  float y = (float)r.h;
  float yu = nextafterf(y, INFINITY), yd = nextafterf(y, -INFINITY);
  double mid_up = 0.5 * ((double)y + (double)yu), mid_dn = 0.5 * ((double)y + (double)yd);
  if (r.h == mid_up && r.l > 0) return yu;
  if (r.h == mid_dn && r.l < 0) return yd;
  return y;
}

// single_up of a nonnegative integer M <= 2^29 (exact below 2^24).
__device__ inline float single_up_int(int M) {
  unsigned u = (unsigned)M;
  int bl = 32 - __clz(u);
  if (bl > 24) {
    int s = bl - 24;
    u = ((u + (1u << s) - 1u) >> s) << s;
  }
  return (float)u;
}

// Stage dumps only: mu', nu' and the log2f values (the residue kernels form
// the shifts from the table of steps, shift_of).
__global__ __launch_bounds__(256) void k_debug_shifts(const uint64_t* __restrict__ rowbits,
                                                      const int* __restrict__ rmax, int m,
                                                      const uint64_t* __restrict__ colbits,
                                                      const int* __restrict__ cmax, int n,
                                                      int* __restrict__ mu_p, int* __restrict__ nu_p,
                                                      float* __restrict__ ef) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= m + n) return;
  const bool row = t < m;
  const int idx = row ? t : t - m;
  const int M = row ? rmax[idx] : cmax[idx];
  (row ? mu_p : nu_p)[idx] = shift_prime_bits(row ? rowbits[idx] : colbits[idx]);
  ef[t] = log2f_rn(single_up_int(M > 1 ? M : 1));       // R7: a zero maximum is treated as 1
}

// ---- grouped versions ------------------------------------------------------
__global__ __launch_bounds__(256) void kg_clear(const ProbDesc* __restrict__ P,
                                                const BlockRef* __restrict__ map) {
  const BlockRef e = map[blockIdx.x];
  const ProbDesc& d = P[e.x];
  const unsigned t = (unsigned)e.y * 256 + threadIdx.x;
  const unsigned stride = (unsigned)group_clear_blocks(d.mp, d.np) * 256;
  for (unsigned i = t; i < (unsigned)d.mp; i += stride) d.rowbits[i] = 0;
  scan_clear(d.rmax, d.mp, d.cmax, d.np, d.flag, t, stride);
}

// One atomic per row and 64 columns, not one per chunk as in absmax_row_chunk: in a
// batch the atomics of one row meet only those of its own problem, and the passes of
// other problems run beside them.
template <typename T>
__global__ __launch_bounds__(256) void kg_absmax_rows(const ProbDesc* __restrict__ P,
                                                      const BlockRef* __restrict__ map) {
  const BlockRef e = map[blockIdx.x];
  const ProbDesc& d = P[e.x];
  const int gx = cdiv_i(d.m, 256), i = e.y % gx * 256 + (int)threadIdx.x;
  const uint64_t mx =
      absmax_row_part<T, SliceSet::Real>((const T*)d.A, d.lda, d.m, d.k, i, e.y / gx * 64);
  if (i < d.m && mx) atomicMax((unsigned long long*)&d.rowbits[i], (unsigned long long)mx);
}

// A problem's strips (none where its scan is chunked), then its columns.
template <typename T>
__global__ __launch_bounds__(kScanThreads, 4) void kg_scan(const ProbDesc* __restrict__ P,
                                                        const BlockRef* __restrict__ map,
                                                        int units, int fine) {
  __shared__ StripLds<SliceSet::Real> lds;
  if (scan_unit() >= units) return;                      // whole workgroup
  const BlockRef e = map[scan_unit()];
  const ProbDesc& d = P[e.x];
  const int lr = strip_rows_log2<T>(d.kp, fine);
  const bool chunked = !strips_fit(d.mp, lr, d.k, d.n, !fine, d.lda * sizeof(T));
  const int strips = chunked ? 0 : d.mp >> lr;
  if (!chunked && e.y == 0)
    scan_clear(d.rmax, d.mp, d.cmax, d.np, d.flag, threadIdx.x, kScanThreads);
  if (e.y < strips)
    scan_strip<T, SliceSet::Real>((const T*)d.A, d.lda, d.m, d.k, d.kp, 0, d.rowbits, d.As, e.y, lr,
                                  lds);
  else
    scan_cols<T, SliceSet::Real>((const T*)d.B, d.ldb, d.n, d.np, d.k, d.kp, d.colbits, d.Bs,
                                 e.y - strips,
                                 col_threads(d.kp, kColKeep<SliceSet::Real>, fine,
                                             group_wave_k(fine, sizeof(T))),
                                 &lds.red[0][0]);
}

__global__ __launch_bounds__(256) void k_log2f(const float* __restrict__ d, float* __restrict__ out,
                                               int count) {
  int t = blockIdx.x * 256 + threadIdx.x;
  if (t < count) out[t] = log2f_rn(d[t]);
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

}  // namespace

namespace {

int col_units(int n_pad, int tpc) { return n_pad / (kScanThreads / tpc); }   // 128 divides n_pad
int clear_blocks(int na, int nb) {
  const int blocks = cdiv(na > nb ? na : nb, 256);
  return blocks > 1024 ? 1024 : blocks;
}

template <typename T, SliceSet F>
void scan_t(hipStream_t s, ScanArgs& a) {
  constexpr bool kEmb = F == SliceSet::Embedding;
  const int span = kEmb ? a.half : a.a.rows_pad;        // rows that strips cover
  const bool fine = scan_fine((int64_t)(span >> kMinStripLog2<T>) + a.b.rows_pad / 8);
  a.lr = strip_rows_log2<T>(a.k_pad, fine);
  a.tpc = col_threads(a.k_pad, kColKeep<F>, fine);
  a.chunked = !strips_fit(span, a.lr, a.k, a.b.rows, false,
                          a.a.ld * sizeof(T) * (F == SliceSet::Real ? 1 : 2));
  a.cols_chunked = a.chunked && cols_chunked<T, F>(a.b.rows);
  a.tr = chunk_rows(a.a.rows);
  if (a.chunked)
    hipLaunchKernelGGL(k_clear, dim3(clear_blocks(a.a.rows_pad, a.b.rows_pad)), dim3(256), 0, s,
                       a.a.bits, a.a.mx, a.a.rows_pad, a.cols_chunked ? a.b.bits : nullptr, a.b.mx,
                       a.b.rows_pad, a.flag);
  a.a.units = a.chunked ? row_chunks(a.a.rows, a.k, a.tr) : span >> a.lr;
  a.b.units = a.cols_chunked ? a.b.rows * cdiv(a.k, kColChunk) : col_units(a.b.rows_pad, a.tpc);
  const dim3 grid = scan_grid(a.a.units + a.b.units), block(kScanThreads);
  if (a.chunked)
    hipLaunchKernelGGL((k_scan_chunks<T, F>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((k_scan<T, F>), grid, block, 0, s, a);
}

template <typename T>
void scan_set(hipStream_t s, SliceSet set, ScanArgs& a) {
  if (set == SliceSet::Real)
    scan_t<T, SliceSet::Real>(s, a);
  else if (set == SliceSet::Complex3)
    scan_t<T, SliceSet::Complex3>(s, a);
  else
    scan_t<T, SliceSet::Embedding>(s, a);
}

}  // namespace

void launch_scan(hipStream_t s, Prec pr, SliceSet set, const SliceOperand& A, const SliceOperand& B,
                 int k, int k_pad, int* flag) {
  ScanArgs a{};
  auto side = [](const SliceOperand& o) {
    return ScanSide{o.src, o.bits, o.mx, o.out, o.ld, o.rows, o.rows_pad, 0};
  };
  a.a = side(A);
  a.b = side(B);
  a.flag = flag;
  a.k = k;
  a.k_pad = k_pad;
  a.half = A.rows_pad / 2;
  if (pr == Prec::F64)
    scan_set<double>(s, set, a);
  else
    scan_set<float>(s, set, a);
  if (a.chunked) {   // A's bars, and B's: the constants are not used
    CrtConsts cc{};
    launch_slices(s, pr, set, true, &A, a.cols_chunked ? &B : nullptr, k, k_pad, cc, nullptr);
  }
}

namespace {
size_t elem_size(Prec pr) { return pr == Prec::F64 ? sizeof(double) : sizeof(float); }
int group_strip_log2(Prec pr, int k_pad, bool fine) {
  return pr == Prec::F64 ? strip_rows_log2<double>(k_pad, fine)
                         : strip_rows_log2<float>(k_pad, fine);
}
}  // namespace

bool scan_group_fine(int64_t units) { return scan_fine(units); }
bool scan_group_chunked(Prec pr, const ProbDesc& d, bool fine) {
  return !strips_fit(d.mp, group_strip_log2(pr, d.kp, fine), d.k, d.n, !fine,
                     d.lda * elem_size(pr));
}
int scan_group_blocks(Prec pr, const ProbDesc& d, bool fine) {
  const int strips =
      scan_group_chunked(pr, d, fine) ? 0 : d.mp >> group_strip_log2(pr, d.kp, fine);
  return strips + col_units(d.np, col_threads(d.kp, kColKeep<SliceSet::Real>, fine,
                                              group_wave_k(fine, elem_size(pr))));
}

void launch_debug_shifts(hipStream_t s, const uint64_t* rowbits, const int* rmax, int m,
                         const uint64_t* colbits, const int* cmax, int n, int* mu_p, int* nu_p,
                         float* ef) {
  hipLaunchKernelGGL(k_debug_shifts, dim3(cdiv(m + n, 256)), dim3(256), 0, s, rowbits, rmax, m,
                     colbits, cmax, n, mu_p, nu_p, ef);
}

void launch_log2f(hipStream_t s, const float* d, float* out, int count) {
  hipLaunchKernelGGL(k_log2f, dim3(cdiv(count, 256)), dim3(256), 0, s, d, out, count);
}

void launch_group_scan(hipStream_t s, Prec pr, const ProbDesc* P, const BlockRef* clear_map,
                       int clear_blocks, const BlockRef* abs_map, int abs_blocks,
                       const BlockRef* scan_map, int scan_blocks, bool fine) {
  if (clear_blocks > 0)
    hipLaunchKernelGGL(kg_clear, dim3((unsigned)clear_blocks), dim3(256), 0, s, P, clear_map);
  if (abs_blocks > 0) {
    if (pr == Prec::F64)
      hipLaunchKernelGGL(kg_absmax_rows<double>, dim3((unsigned)abs_blocks), dim3(256), 0, s, P,
                         abs_map);
    else
      hipLaunchKernelGGL(kg_absmax_rows<float>, dim3((unsigned)abs_blocks), dim3(256), 0, s, P,
                         abs_map);
  }
  if (scan_blocks > 0) {
    if (pr == Prec::F64)
      hipLaunchKernelGGL(kg_scan<double>, scan_grid(scan_blocks), dim3(kScanThreads), 0, s, P,
                         scan_map, scan_blocks, fine ? 1 : 0);
    else
      hipLaunchKernelGGL(kg_scan<float>, scan_grid(scan_blocks), dim3(kScanThreads), 0, s, P,
                         scan_map, scan_blocks, fine ? 1 : 0);
  }
}

}  // namespace oz2
