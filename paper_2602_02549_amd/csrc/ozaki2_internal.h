// Internal declarations shared by the library's translation units.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstddef>
#include <cstdint>

namespace oz2 {

constexpr int kMaxModuli = 49;   // Section 3.1: p_l <= 256 pairwise coprime => N <= 49
// k < 2^19: Section 3 assumes k <= 2^17; beyond it Cbar <= 2^12 k stays below
// 2^31 and the residue products are reduced mod p_l every 2^17 of k.
constexpr int kMaxK = (1 << 19) - 1;
constexpr int kRowPad = 256;     // m and n are padded to this multiple in the workspace
constexpr int kMaxDim = 0x7FFFFF00; // largest m, n whose padding to kRowPad fits in int
constexpr int kKPad = 128;       // k is padded to this multiple (bytes of INT8 per row)
constexpr int kShiftSteps = 17;  // c log2f(M) + P' spans less than 16 for M < 2^31
constexpr int kCrtRows = 4;      // CRT: consecutive rows per thread (256 threads per block)

// Per-(N, b) constants of Section 3.1 and Algorithms 2-3, passed to kernels
// by value (they land in the kernel-argument segment and are read with
// scalar loads).
struct ModConst {   // one modulus, as the kernels use it (uniform, scalar loads)
  double pinv;             // double(1/p)
  // Limb weights of the residue paths, symmetric mod p (0 for p = 256): two
  // limbs: c1 = mod(2^48, p); three: c1 = mod(2^40, p), c2 = mod(2^80, p).
  double c1, c2;
  uint32_t c1p, c2p, negp; // c1, c2 and -p in both 16-bit halves
  int p;
};

struct CrtConsts {
  int N;
  int b;            // 64 or 32
  int table;        // moduli: kTablePaper or kTableOptimal
  int nsteps;       // exact-reduction steps for |A'| < 2^(6 + floor(P'))
  int nlimbs;       // 2 or 3: residues from limbs of A' (0: use nsteps)
  float Pprime;     // P' = single_down(log2(P-1)/2 - 0.5)
  float c;          // single_down(-0.5 / (1 - 4 u_32))
  // Algorithm 2's shift as a step function of the maximum M of Cbar:
  // floor(c log2f(single_up(max(M, 1))) + P') = shift0 - #{j : M >= step[j]}.
  int shift0;
  int step[kShiftSteps];
  double P1, P2;    // double-double P (P2 = 0 for b = 32)
  double Pinv;      // double(1/P)
  ModConst mod[kMaxModuli]; // p_l
  double s1[kMaxModuli];    // s_l1
  double s2[kMaxModuli];    // s_l2 (0 for b = 32)
};

// Moduli tables (Section 3.1): the first N of the paper's fixed list, or the
// N pairwise coprime integers <= 256 of largest product (descending).
constexpr int kTablePaper = 0;
constexpr int kTableOptimal = 1;
bool moduli_of(int table, int N, int* p);

// Host-side tables (tables.cpp).  Returns false if a constant could not be
// established (e.g. P' too close to the FP32 grid for the host's precision).
bool build_consts(int N, int b, int table, CrtConsts* out);
// N-dependent coefficients of the planner bound for every N in [2, 49]:
//   t(N) = 1/sqrt(32 (P-1)), tt(N) = t^2, extra(N) = (r_b(N) - r_rnd) t^2,
//   rnd(N) = r_rnd t^2 (the N-independent output rounding part).
struct PlanCoef {
  double t[kMaxModuli + 1];
  double tt[kMaxModuli + 1];
  double extra[kMaxModuli + 1];
  double rnd[kMaxModuli + 1];
  double rconst[kMaxModuli + 1];  // R_const of Lemma 4
  double rel[kMaxModuli + 1];     // R_rel t^2 / (1 - R_rel)
};
bool build_plan_coef(int b, int table, PlanCoef* out);

// The a-posteriori est1 of Theorem 1 at one N, in the planner's factored form
// (passed by value to the certification kernel).
struct CertTable {
  double t, tt, extra;  // t(N), t(N)^2, R_const t(N)^2
  double rconst, rel;   // R_const; R_rel t(N)^2 / (1 - R_rel)
  double k;             // inner dimension
  double acc_scale;     // lower-bound factor of the BF16 product S
  double tiny;          // smallest positive subnormal of the output type
};

// Everything the per-entry planner kernels need (passed by value).
struct PlanTable {
  int nlo, nhi;        // search range of N
  double k;            // inner dimension
  double eps;          // target
  double acc_scale;    // lower-bound factor for the FP32-accumulated BF16 product
  double t[kMaxModuli + 1], tt[kMaxModuli + 1], extra[kMaxModuli + 1];
};

// mu' = 5 - floor(log2 x) (Algorithm 2, eq. mu'nu') from the IEEE bit pattern
// of x = max_h |a_ih| as an FP64 number; a zero row gets 0 (its outputs are
// exact zeros).  Exact for subnormals.
__device__ inline int shift_prime_bits(uint64_t bits) {
  if (bits == 0) return 0;
  int ex = (int)(bits >> 52);
  if (ex == 0x7FF) return 0;  // non-finite input: every output is forced to NaN
  int fl;
  if (ex == 0) {
    uint64_t mant = bits & 0x000FFFFFFFFFFFFFull;
    fl = (63 - __clzll((long long)mant)) - 1074;
  } else {
    fl = ex - 1023;
  }
  return 5 - fl;
}

// The bit pattern of an infinity or a NaN.
__device__ __forceinline__ bool nonfinite_bits(uint64_t bits) {
  return (bits >> 52 & 0x7FF) == 0x7FF;
}

// mu (nu) of Algorithm 2 from a row's abs-max bit pattern and its maximum M of
// Cbar; bias is added to mu' of nonzero rows.  A zero maximum counts as 1 (R7).
// The table of steps stands for the log2f and the floor (24 integer
// instructions a row against about 1500 for the double-double log2f), so that
// the residue kernels form the shifts they need themselves.
__device__ __forceinline__ int shift_of(uint64_t bits, int M, const CrtConsts& cc, int bias) {
  int s = shift_prime_bits(bits) + (bits ? bias : 0) + cc.shift0;
#pragma unroll
  for (int j = 0; j < kShiftSteps; ++j) s -= M >= cc.step[j] ? 1 : 0;
  return s;
}

// ---------------------------------------------------------------------------
// Grouped (batched) execution: one launch per phase covers every problem of a
// batch.  Each problem has a descriptor; per phase, a block map gives every
// workgroup its problem and its index among that problem's workgroups (one
// uniform load, no search).
struct ProbDesc {
  int m, n, k, N;
  int mp, np, kp;           // padded sizes (workspace layout)
  int lda, ldb, ldc;
  const void* A;
  const void* B;
  void* C;
  uint64_t* rowbits;
  uint64_t* colbits;
  int* rmax;
  int* cmax;
  int* mu;
  int* nu;
  int* flag;
  int8_t* As;               // [N][mp][kp]
  int8_t* Bs;               // [N][np][kp]
  int8_t* W;                // [N][np][mp]
};

// Block map entry: x = problem index, y = local workgroup index.
typedef int2 BlockRef;

__host__ __device__ inline int cdiv_i(int a, int b) { return (a + b - 1) / b; }

// Workgroups of one problem in the grouped clearing (a grid-stride loop over
// max(mp, np) entries) and in a grouped product with `tile` x `tile` output
// tiles and nz slices (padded to a multiple of 8 so that every problem starts
// on XCD 0).
__host__ __device__ inline int group_clear_blocks(int mp, int np) {
  return cdiv_i(mp > np ? mp : np, 256);
}
__host__ __device__ inline int group_gemm_blocks(int mp, int np, int tile, int nz) {
  return ((mp / tile) * (np / tile) * nz + 7) / 8 * 8;
}
// Workgroups of the CRT (one thread per kCrtRows rows of one column).
__host__ __device__ inline int64_t crt_blocks(int m, int n) {
  return ((int64_t)cdiv_i(m, kCrtRows) * n + 255) / 256;
}

// ---------------------------------------------------------------------------
// Kernel launchers (each defined next to its kernel)
// ---------------------------------------------------------------------------
enum class Prec { F64, F32 };

// scale.hip
// mu', nu' and the log2f values e (rows) then f (columns) for the stage dumps.
void launch_debug_shifts(hipStream_t s, const uint64_t* rowbits, const int* rmax, int m,
                         const uint64_t* colbits, const int* cmax, int n, int* mu_p, int* nu_p,
                         float* ef);
void launch_log2f(hipStream_t s, const float* d, float* out, int count);

// Tuning and test knobs (ozaki2_debug_tuning): a cap on the workgroups of a
// slice launch (0: none; residue.hip) and the forced tile of the single-problem
// products (0: automatic, 1: 256x256, 2: 128x128; gemm_i8.hip).
extern std::atomic<int> g_slice_cap;
extern std::atomic<int> g_gemm_tile;
// Split-k of the single-problem products: 0 automatic (default), 1 off.
extern std::atomic<int> g_split_k;

// residue.hip: per-device launch figures of the slice kernels (resident workgroups);
// called once per device before its first launch, outside stream capture.
void init_slice_launch(int dev);

// residue.hip: INT8 slices in K-major layout [S][rows_pad][k_pad] of A
// (column-major m x k: element (r, h) at src[r + h ld]) and of B (k x n: element
// (h, r) at src[h + r ld]), either or both in one launch (null: not this one).
//   bars:     S = 1, byte = ceil(2^shift |x|) (>= 1 if x != 0), shift = mu'
//             from `bits`; zero in the padding rows.
//   residues: S = N, byte_l = mod(trunc(2^shift x), p_l), shift = mu / nu of
//             Algorithm 2 from `bits` (with bias added to mu' and nu' of nonzero
//             rows) and the maxima of Cbar `mx`, also written to `shift`.
//   Real:      as above.
//   Complex3:  the 3-product form, from interleaved (re, im) pairs (ld in
//              complex elements): bars ceil(2^(mu'-1) |re|) + ceil(2^(mu'-1) |im|);
//              residues 3 N slices: of the real parts, of the imaginary parts
//              and of their sums (mod p_l of the two bytes).
//   Embedding: the slices of the real embedding Ahat = [[Ar, -Ai], [Ai, Ar]],
//              Bhat = [[Br], [Bi]] of a complex product, from the pairs in place,
//              laid out with the halves at aligned offsets, zeros between: k
//              half k_pad (slice rows are 2 k_pad long) and, on the A side, row
//              half rows_pad / 2 (rows i and rows_pad / 2 + i of the embedding
//              come from complex row i).  Zero rows and columns change none of
//              the embedding's products, maxima or shifts.  bits, mx and shift
//              are indexed by the embedding's rows.
enum class SliceSet { Real, Complex3, Embedding };
struct SliceOperand {
  const void* src;
  int ld, rows, rows_pad;
  uint64_t* bits;
  int* mx;
  int* shift;
  int8_t* out;
};
// A non-finite entry (its row's bit pattern) sets *flag in the residue launch.
void launch_slices(hipStream_t s, Prec pr, SliceSet set, bool bars, const SliceOperand* A,
                   const SliceOperand* B, int k, int k_pad, const CrtConsts& cc, int* flag,
                   int bias = 0);

// scale.hip: the abs-max bit patterns `bits` of the rows of A and the columns of
// B (over both parts of pairs) and their bars (`out`, as above), with the
// maxima of Cbar (both `mx`) and *flag cleared.
void launch_scan(hipStream_t s, Prec pr, SliceSet set, const SliceOperand& A, const SliceOperand& B,
                 int k, int k_pad, int* flag);
// A batch's scan: cleared rows and abs-max of A (kg_clear, kg_absmax_rows) for
// the problems whose scan is chunked (their bars of A are then a slice launch),
// and the scan itself.
// fine: the whole batch's finest split has few workgroups (scan_group_fine).
bool scan_group_fine(int64_t units);
bool scan_group_chunked(Prec pr, const ProbDesc& d, bool fine);
int scan_group_blocks(Prec pr, const ProbDesc& d, bool fine);
void launch_group_scan(hipStream_t s, Prec pr, const ProbDesc* P, const BlockRef* clear_map,
                       int clear_blocks, const BlockRef* abs_map, int abs_blocks,
                       const BlockRef* scan_map, int scan_blocks, bool fine);

// Planner operands (BF16, K-major [rows_pad][k_pad]) and per-64-k-tile row
// sums partial[k_pad/64][rows_pad] of |x| 2^-alpha; a non-finite row sets *flag.
void launch_plan_slices(hipStream_t s, Prec pr, bool trans, const void* src, int ld, int rows,
                        int k, int rows_pad, int k_pad, const uint64_t* bits, uint16_t* out,
                        double* partial, int* flag);

// gemm_i8.hip
//   D[x][y] = sum_h X[x][h] * Y[y][h] over k_pad, for slices z = 0..nz-1 with
//   X_z = X + z*sx, Y_z = Y + z*sy (X: A side, x = i; Y: B side, y = j).
//   epi 0: W_z[y][x] = mod(D, p_z) as int8 into W + z*sw, row length ldw.
//   epi 1: xmax[x] = max_y D, ymax[y] = max_x D (atomicMax; D >= 0).
//   epi 3: epi 1, and W[y][x] = (D != 0) as one byte (row length ldw).
//   epi 4: D_z[y][x] as INT32 into (int*)W + z*sw, row length ldw (elements).
//   part, part_bytes: scratch for split-k (epi 0 and 1, when few output
//   tiles leave the CUs idle): the partial products of the k ranges go there
//   and a reduction kernel combines them into the same result (epi 0: the
//   sum of the partial mod-p bytes, mod p; epi 1: the INT32 sum, then its
//   maxima).  With too little scratch (or none) the product is not split.
//   vx, vy: real rows of X and Y (0: all); a split product reads no others.
void launch_gemm_i8(hipStream_t s, int epi, const int8_t* X, size_t sx, const int8_t* Y, size_t sy,
                    int nx_pad, int ny_pad, int k_pad, int nz, const CrtConsts& cc, int8_t* W,
                    size_t sw, int ldw, int* xmax, int* ymax, int8_t* part = nullptr,
                    size_t part_bytes = 0, int vx = 0, int vy = 0);
// Scratch bytes that lets launch_gemm_i8 split both the scaling product (epi
// 1) and the nz residue products (epi 0) of this shape; 0 if neither splits.
size_t split_scratch_bytes(int nx_pad, int ny_pad, int k_pad, int nz);

// S[y][x] = sum_h X[x][h] Y[y][h] over BF16 slices (FP32 accumulation on
// the matrix cores), stored column-major with row length lds_.
void launch_gemm_bf16_store(hipStream_t s, const uint16_t* X, const uint16_t* Y, int nx_pad,
                            int ny_pad, int k_pad, float* S, int lds_);

// plan.hip
void launch_plan_vectors(hipStream_t s, const double* pr, int m_pad, const double* pc, int n_pad,
                         int tiles, const int* rmax, const int* cmax, int m, int n, double* rs,
                         double* cs, double* sr, double* sc);
// S: lower bound of (|A||B|)_ij (scaled), nz: one byte per entry, nonzero
// exactly when (|A||B|)_ij > 0; both column-major with row length lds_.
void launch_plan_entries(hipStream_t s, const float* S, const uint8_t* nz, int lds_, int m, int n,
                         const double* rs, const double* cs, const double* sr, const double* sc,
                         const PlanTable& pt, int* out);
// N from Nsrc (device) when it is not null; see k_plan_verify.
void launch_plan_verify(hipStream_t s, const float* S, const uint8_t* nz, int lds_, int m, int n,
                        const double* rs, const double* cs, const double* sr, const double* sc,
                        const PlanTable& pt, int N, const int* Nsrc, int* bad);
// Maximum over entries of the a-posteriori est1 / S (bit pattern into *out,
// which the caller zeroes); C is the output of the run whose shifts are mu, nu.
void launch_certify(hipStream_t s, Prec pr, const void* C, int ldc, const int* mu, const int* nu,
                    const float* S, const uint8_t* nz, int lds_, int m, int n, const double* rs,
                    const double* cs, const double* sr, const double* sc, const CertTable& ct,
                    unsigned long long* out);

// Grouped launches (one per phase for a whole batch of `count` problems);
// `map` holds `blocks` entries, one per workgroup.
// The residue path every problem of a batch shares (a code for
// launch_group_slices), or the per-tile choice when they differ.
int group_residue_path(const CrtConsts* const* cc, int count);
void launch_group_slices(hipStream_t s, Prec pr, bool bars, int path, const ProbDesc* P,
                         const BlockRef* amap, int atiles, const BlockRef* bmap, int btiles,
                         const CrtConsts* ctab);
void launch_group_gemm(hipStream_t s, int epi, int tile, const ProbDesc* P, const BlockRef* map,
                       int blocks, const CrtConsts* ctab);
// Persistent grouped residue products: `grid` resident workgroups (a multiple
// of 8, from persist_grid, queried outside any capture) walk the `items`
// entries of the block map.
int persist_grid(int tile);
// `fold`: some problem has k_pad > 2^17 (the build with reductions mod p).
void launch_group_gemm_persist(hipStream_t s, int tile, bool fold, int grid, const ProbDesc* P,
                               const BlockRef* map, int items, const CrtConsts* ctab);
void launch_group_crt(hipStream_t s, Prec pr, const ProbDesc* P, const BlockRef* map, int blocks,
                      const CrtConsts* ctab, int* status);

// crt.hip: C(i, j) from W_l[j][i] (slices of row length ldw), mu, nu.  A set
// non-finite flag makes every entry NaN and also sets *status, the sticky word.
void launch_crt(hipStream_t s, Prec pr, const int8_t* W, size_t sw, int ldw, const int* mu,
                const int* nu, int m, int n, const CrtConsts& cc, const int* flag, int* status,
                void* C, int ldc);
// The CRT of a complex result: real parts from (Wr, mur), imaginary parts
// from (Wi, mui), column shifts nu, written as interleaved (re, im) pairs into
// the column-major complex C (ldc in complex elements).
void launch_crt_complex(hipStream_t s, Prec pr, const int8_t* Wr, const int8_t* Wi, size_t sw,
                        int ldw, const int* mur, const int* mui, const int* nu, int m, int n,
                        const CrtConsts& cc, const int* flag, int* status, void* C, int ldc);
// The CRT of the 3-product form: the real and imaginary residues of modulus l
// are mod(W1 - W2, p_l) and mod(W3 - W1 - W2, p_l), formed per byte from the
// three products' W; shifts mu (rows) and nu (columns) for both parts;
// interleaved complex output as launch_crt_complex.
void launch_crt_3m(hipStream_t s, Prec pr, const int8_t* W1, const int8_t* W2, const int8_t* W3,
                   size_t sw, int ldw, const int* mu, const int* nu, int m, int n,
                   const CrtConsts& cc, const int* flag, int* status, void* C, int ldc);
// launch_crt plus C'(1), C'(2), Q, C'' as FP64 [4][n][m] into dbg (stage dumps).
void launch_crt_debug(hipStream_t s, Prec pr, const int8_t* W, size_t sw, int ldw, const int* mu,
                      const int* nu, int m, int n, const CrtConsts& cc, const int* flag, void* C,
                      int ldc, double* dbg);
void launch_fill_zero(hipStream_t s, Prec pr, void* C, int ldc, int m, int n);

// complex.hip: the real embedding of a complex product (interleaved (re, im)
// column-major inputs; leading dimensions in complex elements) into
// Ahat = [[Ar, -Ai], [Ai, Ar]] (2m x 2k, ld 2m) and Bhat = [[Br], [Bi]]
// (2k x n, ld 2k).
void launch_embed_complex(hipStream_t s, Prec pr, const void* A, int lda, const void* B, int ldb,
                          int m, int n, int k, void* Ah, void* Bh);

// api.cpp: Algorithm 1 for one problem on a workspace of `cap` bytes that
// `get` supplies, with its sticky status word; checks the arguments and the
// size (OZAKI2_ERR_WORKSPACE if the layout needs more than cap) before any
// HIP call and allocates nothing.
typedef int (*BufferSource)(char** ws, int** status);
int gemm_on_buffer(Prec pr, int m, int n, int k, const void* A, int lda, const void* B, int ldb,
                   void* C, int ldc, int N, size_t cap, BufferSource get);
// noalloc.hip: the status word of the allocation-free entry point on device
// `dev`, or nullptr while that entry point has not been set up there.
int* noalloc_status(int dev);

// probe.hip: the MFMA-rate probe (ozaki2_debug_mfma_probe): `blocks`
// workgroups of 8 waves, `iters` steps of 16 MFMAs each, operands changing
// every step or fixed; returns its duration (ms, HIP events on s,
// synchronised) and its INT8 operation count.
int probe_mfma(hipStream_t s, int blocks, int iters, bool change, float* ms, double* ops);

}  // namespace oz2
