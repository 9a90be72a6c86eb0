// INT8 x INT8 -> INT32 matrix-core products (CDNA4 v_mfma_i32_16x16x64_i8):
//   epi 0: the N residue products C'_l = A'_l B'_l of Algorithm 3 with the
//          reduction W_l = mod(C'_l, p_l) fused into the epilogue;
//   epi 1: the scaling product Cbar = Abar Bbar of Algorithm 2, of which only
//          the row and column maxima are kept (atomicMax, order-free);
//   epi 3: epi 1 plus one byte per entry, Cbar_ij != 0 (the planner's
//          indicator of (|A||B|)_ij > 0);
//   epi 4: the raw INT32 accumulators C'_l (stage dumps only).
//
// Operands are K-major INT8 slices (k contiguous), zero padded, so the kernel
// needs no bounds checks:  D[x][y] = sum_h X[x][h] Y[y][h], with X the A side
// (x = output row i) and Y the B side (y = output column j).  In the MFMA
// accumulator layout a lane holds 4 consecutive x for one y, so the W_l bytes
// of 4 consecutive rows i are packed into one word, and four such words into
// one 16-byte store of the column-major W_l[j][i].
//
// Instruction: large products run at a clock that the power limit lowers, so an
// instruction with less energy per product is faster.  16x16x64 adds 64 products
// for each accumulator it reads and writes, 32x32x32 half as many.  Alone, from
// registers (the probe), the first runs at 3.8 to 4.0 PO/s on fixed random bytes
// and 3.0 to 3.3 on bytes that change every step, the second at 3.3 to 3.4 and
// 2.95 to 3.1; on zeros both at 4.9.  Here: 14 products of 8192^3 6410 (32x32x32)
// and 5800 us (2.43 and 2.65 PO/s), 18 of 4096^3 1060 and 970, 7 of 16384^3 27.2
// and 24.3 ms.  Power and the loop's own waits both cap it: on zeros, at 2.34 GHz,
// the loop keeps the pipes 67% busy (3.1 to 3.3 PO/s); on random residues the clock
// falls to 1.68 GHz and, memory being nearer by as much, they are 77% busy (2.85).
// The BF16 product (the planner's lower bound of |A||B|) stays with 32x32x16, whose
// order of FP32 additions its results depend on.
//
// Tiling: a workgroup of NWX x NWY waves computes a BX x BY tile; each wave
// owns (BX/NWX) x (BY/NWY).  A 256 x 256 tile runs 8 waves (4 x 2, each 64 x
// 128: two waves per SIMD, so one wave's MFMAs overlap the other's LDS reads
// and barrier waits; four waves of 128 x 128 read a third less from LDS but
// took 37% longer), a 128 x 128 tile 4 waves (2 x 2) with two workgroups per
// CU.  K advances in groups of 128 bytes through a ring of two LDS group
// buffers (four where a CU holds one workgroup of 128 x 128): direct
// global->LDS copies fill the buffers ahead (every 128-byte line of an operand
// row requested as one unit) while the MFMAs consume one.  BF16 operands run
// through the same loop, counting k in bytes.
//
// Workgroup order: the hardware deals workgroups round-robin to the 8 XCDs;
// the linear id is remapped so each XCD works on a contiguous range of
// tiles, and tiles are walked in groups of GROUP rows of tiles so that the
// workgroups resident on one XCD share A- and B-panels in its L2.
//
// Accumulator layout of the 16x16x64 MFMA (lane l, register r):
//   row (X side) = 4*(l/16) + r,   column (Y side) = l%16;
// of the 32x32x16 one:
//   row (X side) = 8*(r/4) + 4*(l/32) + r%4,   column (Y side) = l%32.
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <type_traits>

#include "ozaki2_internal.h"
#include "small_mod.h"
#include "tile_walk.h"

namespace oz2 {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf16 __attribute__((ext_vector_type(8)));

constexpr size_t kRoundBytes = (size_t)96 << 20;   // operands of a slice: see walk_in_rounds
constexpr int kFoldGroups = (1 << 17) / 128;   // 128-k groups per 2^17 of k

// mod(x, p) of an INT32 product as an INT8 value (Section 1.2), odd p: the
// FP64 quotient x * (1/p) is within 2^-25 of x/p, which is never within
// 1/(2p) of a half-integer, so rint gives round(x/p) exactly and one fma
// gives x - round(x/p) p exactly.  (p = 256 takes the low byte, the
// two's-complement wrap of Section 3.1, in the caller.)
__device__ inline int mod_odd(int x, double p, double pinv) {
  const double xd = (double)x;
  return (int)fma(-rint(xd * pinv), p, xd);
}

// The bytes mod(x, p) of four products (odd p, or p = 256: the low bytes): q =
// round(x/p) is in the low bits of one fma with kRound, as exact as rint in
// mod_odd, and x - q p is formed mod 2^16, two values per packed instruction:
// per value a conversion, an fma and 1.75 integer instructions instead of five
// FP64 ones and 1.5 to pack.  The epilogue is a tenth of the products at k =
// 4096: 18 of 4096^3 took 1084 us with FP64 remainders, 1057 with these.
__device__ __forceinline__ uint32_t mod_word(int a, int b, int c, int d, double pinv,
                                             uint32_t negp) {
  const uint32_t qa = (uint32_t)__double2loint(fma((double)a, pinv, kRound));
  const uint32_t qb = (uint32_t)__double2loint(fma((double)b, pinv, kRound));
  const uint32_t qc = (uint32_t)__double2loint(fma((double)c, pinv, kRound));
  const uint32_t qd = (uint32_t)__double2loint(fma((double)d, pinv, kRound));
  const uint32_t x = pk_mad(pair16(qa, qb), negp, pair16((uint32_t)a, (uint32_t)b));
  const uint32_t y = pk_mad(pair16(qc, qd), negp, pair16((uint32_t)c, (uint32_t)d));
  return bytes_of_pairs(x, y);
}

__device__ inline uint32_t pack_bytes(int a, int b, int c, int d) {
  return (uint32_t)(a & 0xFF) | ((uint32_t)(b & 0xFF) << 8) | ((uint32_t)(c & 0xFF) << 16) |
         ((uint32_t)(d & 0xFF) << 24);
}

typedef __attribute__((address_space(3))) int8_t lds_i8_t;

// One wave-wide direct global->LDS copy (CDNA4 global_load_lds_dwordx4):
// lane l copies 16 bytes from its address g to LDS byte M0 + 16 l.  Issued as
// inline asm so the compiler's wait-count insertion does not treat every LDS
// read as depending on every copy in flight; the kernel waits explicitly.
// M0 is saved in a scratch SGPR and restored, so no value the compiler keeps
// in M0 is disturbed.
__device__ inline void dma16(const void* g, uint32_t lds_addr) {
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(g), "s"(lds_addr)
      : "memory");
}

__device__ inline uint32_t lds_addr(const int8_t* p) {
  return (uint32_t)(uintptr_t)(lds_i8_t*)p;
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding).
template <int V>
__device__ inline void wait_vmcnt() {
  static_assert(V >= 0 && V < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((V & 0xF) | (((V >> 4) & 3) << 14) | (0x7 << 4) | (0xF << 8));
}

// Chunk swizzle of an LDS row (128 bytes of k, 32 banks apart): chunk c of
// row r is stored at position c ^ swz(r), so that the 16-byte fragment reads
// of rows r..r+15 land in distinct bank groups (64 banks).
__device__ inline int swz(int r) { return (r >> 1) & 7; }

// Interleaving of a sub-step for the scheduler: READS fragment reads (of the
// next sub-step) alternate one for one with MFMAS matrix instructions, the rest
// of either follow.
template <int READS, int MFMAS>
__device__ __forceinline__ void interleave() {
  constexpr int BOTH = READS < MFMAS ? READS : MFMAS;
#pragma unroll
  for (int q = 0; q < BOTH; ++q) {
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
  }
  if constexpr (READS > BOTH) __builtin_amdgcn_sched_group_barrier(0x100, READS - BOTH, 0);
  if constexpr (MFMAS > BOTH) __builtin_amdgcn_sched_group_barrier(0x008, MFMAS - BOTH, 0);
}

// A wave's share of a BX x BY tile of bytes, WX x WY as 16 x 16 blocks: its
// accumulators and the products of one 128-k group in LDS (rows of 128 bytes,
// X then Y).  Four sub-steps: 64 of k times half of the Y blocks.
template <int BX, int BY, int NWX, int NWY>
struct WaveTile {
  static constexpr int WX = BX / NWX, WY = BY / NWY;
  static constexpr int TX = WX / 16, TY = WY / 16, TH = TY / 2;
  static_assert(TX == 4 && TY % 2 == 0, "wave shape");
  v4i acc[TX][TY];
  int lane, xrow, yrow;     // first rows of the share in LDS
  int fo[2];                // lane: row lane % 16 of a block, 16-byte chunk lane / 16 of 64 k

  __device__ __forceinline__ WaveTile() {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    lane = threadIdx.x & 63;
    xrow = wave / NWY * WX;
    yrow = wave % NWY * WY;
    const int r = lane & 15;
#pragma unroll
    for (int h = 0; h < 2; ++h) fo[h] = r * 128 + (((4 * h + (lane >> 4)) ^ swz(r)) * 16);
  }
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int a = 0; a < TX; ++a)
#pragma unroll
      for (int b = 0; b < TY; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[a][b][r] = 0;
  }
  __device__ __forceinline__ void load_x(const int8_t* buf, int h, v4i (&a)[TX]) const {
#pragma unroll
    for (int t = 0; t < TX; ++t)
      a[t] = *reinterpret_cast<const v4i*>(buf + (xrow + t * 16) * 128 + fo[h]);
  }
  __device__ __forceinline__ void load_y(const int8_t* buf, int h, int half, v4i (&b)[TH]) const {
#pragma unroll
    for (int t = 0; t < TH; ++t)
      b[t] = *reinterpret_cast<const v4i*>(buf + (BX + yrow + (half * TH + t) * 16) * 128 + fo[h]);
  }
  // back and forth over X: each instruction shares an operand with the one before
  __device__ __forceinline__ void mfmas(const v4i (&a)[TX], const v4i (&b)[TH], int half) {
#pragma unroll
    for (int t = 0; t < TH; ++t)
#pragma unroll
      for (int q = 0; q < TX; ++q) {
        const int x = t & 1 ? TX - 1 - q : q, y = half * TH + t;
        acc[x][y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[x], b[t], acc[x][y], 0, 0, 0);
      }
  }
  // The first fragment reads go out before the next group's copies, so their
  // LDS latency overlaps the copy issue; the X-row copies follow them and the
  // Y-row copies come one sub-step later, spreading the copies over the group.
  template <class CopyX, class CopyY>
  __device__ __forceinline__ void group(const int8_t* buf, CopyX copy_x, CopyY copy_y) {
    v4i a0[TX], a1[TX], b0[TH], b1[TH];
    load_x(buf, 0, a0);
    load_y(buf, 0, 0, b0);
    copy_x();
    __builtin_amdgcn_sched_barrier(0);
    load_y(buf, 0, 1, b1);
    mfmas(a0, b0, 0);
    interleave<TH, TX * TH>();
    __builtin_amdgcn_sched_barrier(0);
    copy_y();
    __builtin_amdgcn_sched_barrier(0);
    load_x(buf, 1, a1);
    load_y(buf, 1, 0, b0);
    mfmas(a0, b1, 1);
    interleave<TX + TH, TX * TH>();
    __builtin_amdgcn_sched_barrier(0);
    load_y(buf, 1, 1, b1);
    mfmas(a1, b0, 0);
    interleave<TH, TX * TH>();
    __builtin_amdgcn_sched_barrier(0);
    mfmas(a1, b1, 1);
  }
  // The same with one wave per SIMD, where nothing else covers the latency of a
  // fragment read: all of them go out at once, and the MFMAs follow as they come
  // (scaling product of 2048^3, 16 groups, with its events: 15.6 us, interleaved
  // 16.7).
  template <class CopyX, class CopyY>
  __device__ __forceinline__ void group_alone(const int8_t* buf, CopyX copy_x, CopyY copy_y) {
    v4i a0[TX], a1[TX], b00[TH], b01[TH], b10[TH], b11[TH];
    load_x(buf, 0, a0);
    load_y(buf, 0, 0, b00);
    load_y(buf, 0, 1, b01);
    load_x(buf, 1, a1);
    load_y(buf, 1, 0, b10);
    load_y(buf, 1, 1, b11);
    __builtin_amdgcn_sched_barrier(0);
    copy_x();
    copy_y();
    __builtin_amdgcn_sched_barrier(0);
    mfmas(a0, b00, 0);
    mfmas(a0, b01, 1);
    mfmas(a1, b10, 0);
    mfmas(a1, b11, 1);
  }
  // acc = mod(acc, p), odd p
  __device__ __forceinline__ void reduce(double p, double pinv) {
#pragma unroll
    for (int a = 0; a < TX; ++a)
#pragma unroll
      for (int b = 0; b < TY; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[a][b][r] = mod_odd(acc[a][b][r], p, pinv);
  }
  // One byte per entry, word(v4i) of each block, into the column-major byte
  // matrix at W (the share's first entry; columns ldw apart).  A lane holds rows
  // 4 (l/16) .. + 3 of column l%16 of the blocks 0..3; exchanging words between
  // its rows of 16 lanes leaves it rows 0..15 of block l/16, one 16-byte store.
  template <class Word>
  __device__ __forceinline__ void store_bytes(int8_t* __restrict__ W, int ldw, Word word) const {
#pragma unroll
    for (int t = 0; t < TY; ++t) {
      const uint32_t w0 = word(acc[0][t]), w1 = word(acc[1][t]), w2 = word(acc[2][t]),
                     w3 = word(acc[3][t]);
      const auto a = __builtin_amdgcn_permlane32_swap(w0, w2, false, false);
      const auto b = __builtin_amdgcn_permlane32_swap(w1, w3, false, false);
      const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
      const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
      *reinterpret_cast<uint4*>(W + (size_t)(t * 16 + (lane & 15)) * ldw + 16 * (lane >> 4)) =
          make_uint4(c[0], c[1], d[0], d[1]);
    }
  }
  // Row and column maxima of the accumulators (>= 0) into xmax and ymax (the
  // share's first row and column), atomicMax, order-free.
  __device__ __forceinline__ void maxima(int* __restrict__ xmax, int* __restrict__ ymax) const {
#pragma unroll
    for (int t = 0; t < TY; ++t) {
      int mv = 0;
#pragma unroll
      for (int x = 0; x < TX; ++x)
#pragma unroll
        for (int r = 0; r < 4; ++r) mv = max(mv, acc[x][t][r]);
      mv = max(mv, __shfl_xor(mv, 16));
      mv = max(mv, __shfl_xor(mv, 32));
      if (lane < 16) atomicMax(&ymax[t * 16 + lane], mv);
    }
    // The 16 rows of a lane against the 16 lanes of its row of lanes (columns):
    // in each step a lane passes on half of its rows and keeps the other, 15
    // exchanges instead of four for every row; lane % 16 then names the row that
    // a lane holds.
    int v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      v[r] = 0;
#pragma unroll
      for (int t = 0; t < TY; ++t) v[r] = max(v[r], acc[r >> 2][t][r & 3]);
    }
#pragma unroll
    for (int half = 8; half >= 1; half >>= 1) {
      const int up = (lane & half) != 0 ? -1 : 0;        // as a mask: v stays in registers
#pragma unroll
      for (int r = 0; r < half; ++r) {
        const int send = (v[r] & up) | (v[r + half] & ~up);
        const int keep = (v[r + half] & up) | (v[r] & ~up);
        v[r] = max(keep, __shfl_xor(send, half));
      }
    }
    const int r = lane & 15;
    atomicMax(&xmax[16 * (r >> 2) + 4 * (lane >> 4) + (r & 3)], v[0]);
  }
  // The INT32 accumulators, column-major (the share's first entry, columns ld apart).
  __device__ __forceinline__ void store_words(int* __restrict__ D, int ld) const {
#pragma unroll
    for (int t = 0; t < TY; ++t)
#pragma unroll
      for (int x = 0; x < TX; ++x)
        *reinterpret_cast<v4i*>(D + (size_t)(t * 16 + (lane & 15)) * ld + 16 * x +
                                4 * (lane >> 4)) = acc[x][t];
  }
};

// The same for BF16 rows (128 bytes are 64 of k) as 32 x 32 blocks with FP32
// accumulators, k in steps of 16.
template <int BX, int BY, int NWX, int NWY>
struct WaveTileBf16 {
  static constexpr int WX = BX / NWX, WY = BY / NWY, TX = WX / 32, TY = WY / 32;
  v16f acc[TX][TY];
  int lane, xrow, yrow;
  int fo[4];                // lane: row lane % 32 of a block, chunk lane / 32 of 32 bytes

  __device__ __forceinline__ WaveTileBf16() {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    lane = threadIdx.x & 63;
    xrow = wave / NWY * WX;
    yrow = wave % NWY * WY;
    const int r = lane & 31;
#pragma unroll
    for (int j = 0; j < 4; ++j) fo[j] = r * 128 + (((2 * j + (lane >> 5)) ^ swz(r)) * 16);
  }
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int a = 0; a < TX; ++a)
#pragma unroll
      for (int b = 0; b < TY; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][b][r] = 0;
  }
  __device__ __forceinline__ void load(const int8_t* buf, int j, v4i (&a)[TX], v4i (&b)[TY]) const {
#pragma unroll
    for (int t = 0; t < TX; ++t)
      a[t] = *reinterpret_cast<const v4i*>(buf + (xrow + t * 32) * 128 + fo[j]);
#pragma unroll
    for (int t = 0; t < TY; ++t)
      b[t] = *reinterpret_cast<const v4i*>(buf + (BX + yrow + t * 32) * 128 + fo[j]);
  }
  __device__ __forceinline__ void mfmas(const v4i (&a)[TX], const v4i (&b)[TY]) {
#pragma unroll
    for (int x = 0; x < TX; ++x)
#pragma unroll
      for (int y = 0; y < TY; ++y)
        acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf16, a[x]),
                                                            __builtin_bit_cast(v8bf16, b[y]),
                                                            acc[x][y], 0, 0, 0);
  }
  template <class CopyX, class CopyY>
  __device__ __forceinline__ void group(const int8_t* buf, CopyX copy_x, CopyY copy_y) {
    v4i a0[TX], b0[TY], a1[TX], b1[TY];
    load(buf, 0, a0, b0);
    copy_x();
    __builtin_amdgcn_sched_barrier(0);
    load(buf, 1, a1, b1);
    mfmas(a0, b0);
    interleave<TX + TY, TX * TY>();
    __builtin_amdgcn_sched_barrier(0);
    copy_y();
    __builtin_amdgcn_sched_barrier(0);
    load(buf, 2, a0, b0);
    mfmas(a1, b1);
    interleave<TX + TY, TX * TY>();
    __builtin_amdgcn_sched_barrier(0);
    load(buf, 3, a1, b1);
    mfmas(a0, b0);
    interleave<TX + TY, TX * TY>();
    __builtin_amdgcn_sched_barrier(0);
    mfmas(a1, b1);
  }
  // FP32 accumulators, column-major: 4 consecutive rows per lane and store
  __device__ __forceinline__ void store(float* __restrict__ S, int ld) const {
#pragma unroll
    for (int x = 0; x < TX; ++x)
#pragma unroll
      for (int y = 0; y < TY; ++y)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *reinterpret_cast<float4*>(S + (size_t)(y * 32 + (lane & 31)) * ld + x * 32 + 8 * r4 +
                                     4 * (lane >> 5)) =
              make_float4(acc[x][y][4 * r4 + 0], acc[x][y][4 * r4 + 1], acc[x][y][4 * r4 + 2],
                          acc[x][y][4 * r4 + 3]);
  }
};

// One BX x BY tile at (x0, y0) of slice z.  k advances in groups of 128 bytes;
// a group buffer in LDS holds the X tile then the Y tile as rows of 128 bytes,
// and NS of them are a ring.  The copies of group g + NS - 1 (direct
// global->LDS, every 128-byte line requested as one unit) run while the MFMAs
// consume group g.  NS = 2 where the workgroups of a CU fill its LDS (128 KB
// for a 256x256 tile); NS = 4 for launches of 128x128 tiles with at most one
// workgroup per CU, whose groups otherwise wait for a copy each (0.65 us a
// group, 0.3 us with three copies under way).  Scaling product in the kernel
// trace, NS = 2 on 32x32x32 and as it is: 256^3 8.8 and 4.2 us, 1000x700x1300
// 15.1 and 9.3, 2048^3 20.2 and 13.3 (with its events 14.5 when the deep ring ran
// 32x32x32, 15.3 since).
// Split-k: with nsplit > 1, split sidx takes the k-groups [sidx G / nsplit,
// (sidx + 1) G / nsplit) of the G = k_pad / 128 (nsplit <= G), and its
// epilogue writes slice sidx * nz + z of W (EPI 0: mod p_z of its partial
// sum; EPI 4: the INT32 partial sum); the caller reduces the partials.
// SPLIT selects that build; without it nsplit is 1 and the k loop is the
// plain one from group 0 (a dynamic start cost 2% at 8192^3).
template <int BX, int BY, int NWX, int NWY, int EPI, bool BF16, bool FOLD, bool SPLIT, int NS>
__device__ __forceinline__ void gemm_body(int8_t* __restrict__ lds, const int8_t* __restrict__ X,
                                          size_t sx, const int8_t* __restrict__ Y, size_t sy, int x0,
                                          int y0, int z, int nz, int k_pad, const CrtConsts& cc,
                                          int8_t* __restrict__ W, size_t sw, int ldw,
                                          int* __restrict__ xmax, int* __restrict__ ymax, int sidx,
                                          int nsplit, int vx, int vy) {
  constexpr int BK = 128;                        // bytes of k per LDS row (one group)
  constexpr int NW = NWX * NWY;                  // waves
  constexpr int CPR = BK / 16;                   // 16-byte chunks per LDS row
  constexpr int RPI = 1024 / BK;                 // rows per copy instruction
  constexpr int IX = BX / RPI / NW, IY = BY / RPI / NW;
  // Each wave copies IX (IY) instructions of RPI rows; the chunk swizzle
  // repeats every 16 rows and the even/odd instruction offsets below assume
  // that every wave's share starts at a multiple of 16 rows.
  static_assert(IX % 2 == 0 && IY % 2 == 0, "tile / wave shape");
  constexpr int GROUP_BYTES = (BX + BY) * BK;    // one 128-k group
  static_assert((NS & (NS - 1)) == 0 && (NS - 2) * (IX + IY) < 64, "ring");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // Copy instruction q of this wave covers rows RPI*q .. RPI*q + RPI - 1 of
  // its share; lane l takes row RPI*q + l/CPR and stores LDS chunk l%CPR,
  // which holds k-chunk (l%CPR) ^ swz(row).
  const int lr = lane / CPR, slot = lane % CPR;
  const int ch_e = (slot ^ swz(lr)) * 16, ch_o = (slot ^ swz(RPI + lr)) * 16;
  const int8_t* xsrc = X + (size_t)(x0 + wave * IX * RPI + lr) * k_pad;
  const int8_t* ysrc = Y + (size_t)(y0 + wave * IY * RPI + lr) * k_pad;
  const size_t rowstep = (size_t)RPI * k_pad;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);

  // The copies of one group: the X rows (issue_x) and the Y rows (issue_y).
  // SPLIT (a small output over a long k, bound by reading the operands): rows
  // past the vx (vy) real ones copy the last real row again, from L2.  Nothing
  // reads their products, and a repeated row changes no maximum of Cbar.
  // Residue products, all rows read and this: 200x200x100000 191 and 159 us,
  // 64x64x262144 245 and 142 us.
  auto row_of = [&](const int8_t* src, int q, int first, int valid) {
    if constexpr (SPLIT) {
      const int over = first + q * RPI + lr - (valid - 1);
      return src + q * rowstep - (over > 0 ? (size_t)over * k_pad : 0);
    } else {
      return src + q * rowstep;
    }
  };
  auto issue_x = [&](int8_t* buf, int z, int k0) {
    const uint32_t b = lds_addr(buf);
    const int8_t* xs = xsrc + (size_t)z * sx + k0;
#pragma unroll
    for (int q = 0; q < IX; ++q)
      dma16(row_of(xs, q, x0 + wave * IX * RPI, vx) + ((q & 1) ? ch_o : ch_e),
            b + (uint32_t)((wave_u * IX + q) * 1024));
  };
  auto issue_y = [&](int8_t* buf, int z, int k0) {
    const uint32_t b = lds_addr(buf);
    const int8_t* ys = ysrc + (size_t)z * sy + k0;
#pragma unroll
    for (int q = 0; q < IY; ++q)
      dma16(row_of(ys, q, y0 + wave * IY * RPI, vy) + ((q & 1) ? ch_o : ch_e),
            b + (uint32_t)(BX * BK + (wave_u * IY + q) * 1024));
  };

  using Tile = typename std::conditional<BF16, WaveTileBf16<BX, BY, NWX, NWY>,
                                         WaveTile<BX, BY, NWX, NWY>>::type;
  Tile tile;
  tile.clear();

  const double pinv = EPI == 0 ? cc.mod[z].pinv : 0.0;
  const uint32_t negp = EPI == 0 ? cc.mod[z].negp : 0;
  // Epilogue (EPI 0: mod p_z into W_z; EPI 1: maxima; EPI 2: FP32 store;
  // EPI 3: maxima and nonzero bytes; EPI 4: INT32 store).
  auto finish = [&]() {
    const int xb = x0 + tile.xrow, yb = y0 + tile.yrow;
    const size_t first = (size_t)yb * ldw + xb;
    if constexpr (EPI == 0) {
      tile.store_bytes(W + (size_t)(sidx * nz + z) * sw + first, ldw, [&](const v4i& v) {
        return mod_word(v[0], v[1], v[2], v[3], pinv, negp);
      });
    } else if constexpr (EPI == 2) {
      tile.store(reinterpret_cast<float*>(W) + first, ldw);
    } else if constexpr (EPI == 4) {
      tile.store_words(reinterpret_cast<int*>(W) + (size_t)(sidx * nz + z) * sw + first, ldw);
    } else {
      if constexpr (EPI == 3)
        tile.store_bytes(W + first, ldw, [](const v4i& v) {
          return pack_bytes(v[0] != 0, v[1] != 0, v[2] != 0, v[3] != 0);
        });
      tile.maxima(xmax + xb, ymax + yb);
    }
  };

  // k_pad is a multiple of 128.  Group gi lives in buffer gi % NS of the ring;
  // it is issued while group gi - NS + 1 is consumed and waited for (its copies
  // done + barrier) before use, which also certifies that every wave has
  // finished reading group gi - 1.  No branch encloses an MFMA, so the
  // accumulators stay in place across iterations.
  const int NGall = k_pad / 128;
  const int g_lo = SPLIT ? (int)((int64_t)sidx * NGall / nsplit) : 0;
  // end of this workgroup's groups
  const int NG = SPLIT ? (int)((int64_t)(sidx + 1) * NGall / nsplit) : NGall;
  // Beyond 2^17 of k (residue products, EPI 0 and its INT32 dump EPI 4) the
  // accumulators are reduced mod p_z (odd p) after every 2^17 of k: a chunk
  // adds at most 127^2 2^17 < 2^31 - 127 in magnitude to a reduced value, so
  // every partial sum stays exact in INT32 and the result is congruent to
  // C'_l mod p_z.  For p = 256 the two's-complement wrap is already exact
  // mod 256.  The inner loop is the same for every chunk.  FOLD selects the
  // build of the kernel for k_pad > 2^17, so that the usual one keeps the
  // plain loop and its register budget.
  constexpr bool kFold = FOLD && (EPI == 0 || EPI == 4);
  const int chunk = kFold ? kFoldGroups : NG - g_lo;
  auto fold = [&]() {
    const int p = cc.mod[z].p;
    if (p == 256) return;
    if constexpr (!BF16) tile.reduce((double)p, cc.mod[z].pinv);
  };
  auto ring = [&](int gi) { return lds + (gi & (NS - 1)) * GROUP_BYTES; };
#pragma unroll
  for (int g = 0; g < NS - 1; ++g)
    if (g == 0 || g_lo + g < NG) {
      issue_x(SPLIT || NS > 2 ? ring(g_lo + g) : lds, z, (g_lo + g) * 128);
      issue_y(SPLIT || NS > 2 ? ring(g_lo + g) : lds, z, (g_lo + g) * 128);
    }
  // The epilogue's constants are loaded here, while the first copies are under
  // way, and not by every tile's epilogue, and the loop starts on a line of its
  // own: 14 products of 8192^3 5815 us before, 5560 with the first, 5545 with
  // both; of 2048^3 104, 104 and 102 us.
  if constexpr (EPI == 0) asm volatile("" ::"s"(pinv), "s"(negp));
  asm volatile(".p2align 7");
  for (int g0 = g_lo; g0 < NG; g0 += chunk) {
  const int g1 = min(NG, g0 + chunk);
  for (int gi = g0; gi < g1; ++gi) {
    int8_t* const buf = ring(gi);
    int8_t* const next = ring(gi + NS - 1);
    // the copies of the groups after gi may still be under way
    if constexpr (NS == 4) {
      if (gi + 2 < NG)
        wait_vmcnt<2 * (IX + IY)>();
      else if (gi + 1 < NG)
        wait_vmcnt<IX + IY>();
      else
        wait_vmcnt<0>();
    } else {
      static_assert(NS == 2, "ring");
      wait_vmcnt<0>();
    }
    __builtin_amdgcn_s_barrier();
    auto copy_x = [&] {
      if (gi + NS - 1 < NG) issue_x(next, z, (gi + NS - 1) * 128);
    };
    auto copy_y = [&] {
      if (gi + NS - 1 < NG) issue_y(next, z, (gi + NS - 1) * 128);
    };
    if constexpr (NS == 4)
      tile.group_alone(buf, copy_x, copy_y);
    else
      tile.group(buf, copy_x, copy_y);
  }
  if constexpr (kFold) {
    if (g1 < NG) fold();
  }
  }
  finish();
}

// Persistent form of the residue products (EPI 0) for batches: a grid of
// resident workgroups walks the block map in a fixed stride (workgroup g
// takes entries g, g + G, g + 2G, ...; G a multiple of 8, so every entry
// runs on the XCD its local index maps to, as in the one-workgroup-per-entry
// launch).  While a workgroup consumes the last k-group of one tile it
// already copies the first k-group of its next tile into the other LDS
// buffer, so that copy overlaps the last MFMAs and the epilogue instead of
// starting the next tile cold; short-k problems spend most of their time in
// that first copy.  The arithmetic of every tile is the one of gemm_body
// (the same fragment order, MFMAs and epilogue), so the results are the same
// bits.
template <int BX, int BY, int NWX, int NWY, bool FOLD>
__device__ __forceinline__ void gemm_persist(const ProbDesc* __restrict__ P,
                                             const BlockRef* __restrict__ map, int items,
                                             const CrtConsts* __restrict__ ctab) {
  constexpr int BK = 128;
  constexpr int NW = NWX * NWY;
  constexpr int CPR = BK / 16;
  constexpr int RPI = 1024 / BK;
  constexpr int IX = BX / RPI / NW, IY = BY / RPI / NW;
  static_assert(IX % 2 == 0 && IY % 2 == 0, "tile / wave shape");
  static_assert(BX == BY, "square tiles");
  constexpr int GROUP_BYTES = (BX + BY) * BK;
  __shared__ __attribute__((aligned(1024))) int8_t lds[2 * GROUP_BYTES];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int lr = lane / CPR, slot = lane % CPR;
  const int ch_e = (slot ^ swz(lr)) * 16, ch_o = (slot ^ swz(RPI + lr)) * 16;

  // One tile of one residue product.
  struct Job {
    const int8_t* xs;   // this lane's first copy source row of X (slice z, k = 0)
    const int8_t* ys;
    int8_t* Wz;
    int k_pad, ldw, x0, y0, z, p;
    uint32_t negp;
    double pinv;
  };
  // Entry i of the map as a job; false for the padding entries.
  auto decode = [&](int i, Job& j) -> bool {
    const BlockRef e = map[i];
    const ProbDesc& d = P[e.x];
    const int tiles_x = d.mp / BX, tiles_y = d.np / BY, nz = d.N;
    const int launched = group_gemm_blocks(d.mp, d.np, BX, nz);
    const int total = tiles_x * tiles_y * nz;
    const int place = xcd_place(e.y, launched);
    if (place >= total) return false;
    const TilePos pos = tile_at(place, tiles_x, tiles_y);
    const int z = pos.z;
    j.x0 = pos.tx * BX;
    j.y0 = pos.ty * BY;
    j.z = z;
    j.k_pad = d.kp;
    j.ldw = d.mp;
    j.xs = d.As + (size_t)z * d.mp * d.kp + (size_t)(j.x0 + wave * IX * RPI + lr) * d.kp;
    j.ys = d.Bs + (size_t)z * d.np * d.kp + (size_t)(j.y0 + wave * IY * RPI + lr) * d.kp;
    j.Wz = d.W + (size_t)z * d.np * d.mp;
    j.p = ctab[d.N].mod[z].p;
    j.pinv = ctab[d.N].mod[z].pinv;
    j.negp = ctab[d.N].mod[z].negp;
    return true;
  };
  auto issue_x = [&](int8_t* buf, const Job& j, int k0) {
    const uint32_t b = lds_addr(buf);
    const size_t rowstep = (size_t)RPI * j.k_pad;
#pragma unroll
    for (int q = 0; q < IX; ++q)
      dma16(j.xs + k0 + q * rowstep + ((q & 1) ? ch_o : ch_e),
            b + (uint32_t)((wave_u * IX + q) * 1024));
  };
  auto issue_y = [&](int8_t* buf, const Job& j, int k0) {
    const uint32_t b = lds_addr(buf);
    const size_t rowstep = (size_t)RPI * j.k_pad;
#pragma unroll
    for (int q = 0; q < IY; ++q)
      dma16(j.ys + k0 + q * rowstep + ((q & 1) ? ch_o : ch_e),
            b + (uint32_t)(BX * BK + (wave_u * IY + q) * 1024));
  };
  auto next_job = [&](int i, Job& j) -> int {   // first valid entry at or after i (stride G)
    for (; i < items; i += (int)gridDim.x)
      if (decode(i, j)) return i;
    return items;
  };

  WaveTile<BX, BY, NWX, NWY> tile;
  Job cur, nxt;
  int i = next_job((int)blockIdx.x, cur);
  if (i >= items) return;   // whole workgroup, before any barrier
  issue_x(lds, cur, 0);
  issue_y(lds, cur, 0);
  int ph = 0;               // LDS buffer of the current job's group 0
  for (;;) {
    const int inext = next_job(i + (int)gridDim.x, nxt);
    const bool more = inext < items;
    tile.clear();
    const int NG = cur.k_pad / 128;
    for (int g0 = 0; g0 < NG; g0 += FOLD ? kFoldGroups : NG) {
      const int g1 = FOLD ? min(NG, g0 + kFoldGroups) : NG;
      for (int gi = g0; gi < g1; ++gi) {
        int8_t* const buf = lds + ((ph + gi) & 1) * GROUP_BYTES;
        int8_t* const next = lds + ((ph + gi + 1) & 1) * GROUP_BYTES;
        wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        tile.group(
            buf,
            [&] {
              if (gi + 1 < NG)
                issue_x(next, cur, (gi + 1) * 128);
              else if (more)
                issue_x(next, nxt, 0);
            },
            [&] {
              if (gi + 1 < NG)
                issue_y(next, cur, (gi + 1) * 128);
              else if (more)
                issue_y(next, nxt, 0);
            });
      }
      // reduction every 2^17 of k (see gemm_body)
      if (FOLD && g1 < NG && cur.p != 256) tile.reduce((double)cur.p, cur.pinv);
    }
    ph = (ph + NG) & 1;
    // epilogue: W_z = mod(C'_z, p_z), as in gemm_body
    tile.store_bytes(
        cur.Wz + (size_t)(cur.y0 + tile.yrow) * cur.ldw + cur.x0 + tile.xrow, cur.ldw,
        [&](const v4i& v) { return mod_word(v[0], v[1], v[2], v[3], cur.pinv, cur.negp); });
    if (!more) break;
    cur = nxt;
    i = inext;
  }
}

// Wave grid and residency of the two tile sizes.
template <int B>
struct TileShape;
template <>
struct TileShape<256> {
  static constexpr int NWX = 4, NWY = 2, OCC = 1;
};
template <>
struct TileShape<128> {
  static constexpr int NWX = 2, NWY = 2, OCC = 2;
};
template <int B>
constexpr int tile_threads() {
  return 64 * TileShape<B>::NWX * TileShape<B>::NWY;
}

// One product (nz slices): `full` workgroups of whole tiles, and with TAIL = 2
// (4) the tiles from place `full` on as that many 256x128 (128x128) parts each,
// one workgroup per part.  The constants come last, so that the arguments before
// them share two lines.  A last round of few tiles leaves most CUs idle for
// the time of a whole tile; cut up, it occupies them for half or a quarter.
template <int B, int EPI, bool BF16 = false, bool FOLD = false, bool SPLIT = false, int NS = 2,
          int TAIL = 0>
__global__ __launch_bounds__(tile_threads<B>(), TileShape<B>::OCC) void k_gemm_i8(
    const int8_t* __restrict__ X, size_t sx, const int8_t* __restrict__ Y, size_t sy, int tiles_x,
    int tiles_y, int nz, int k_pad, int8_t* __restrict__ W, size_t sw, int ldw,
    int* __restrict__ xmax, int* __restrict__ ymax, int nsplit, int full, int vx, int vy,
    int rounds, CrtConsts cc) {
  __shared__ __attribute__((aligned(1024))) int8_t lds[NS * 2 * B * 128];
  constexpr int NWX = TileShape<B>::NWX, NWY = TileShape<B>::NWY;
  const int bid = (int)blockIdx.x;
  const int group = B == 256 && rounds ? 16 : 8;
  if constexpr (TAIL > 0) {
    if (bid >= full) {
      const int place = xcd_place(bid - full, (int)gridDim.x - full);
      const TilePos t = tile_at(full + place / TAIL, tiles_x, tiles_y, group);
      const int part = place % TAIL;
      constexpr int SX = TAIL == 4 ? B / 2 : B, SY = B / 2;
      // a wave's share is 64 rows of X in every build
      constexpr int PX = SX / 64, PY = NWX * NWY / PX;
      gemm_body<SX, SY, PX, PY, EPI, BF16, FOLD, false, NS>(
          lds, X, sx, Y, sy, t.tx * B + (TAIL == 4 ? (part & 1) * SX : 0),
          t.ty * B + (TAIL == 4 ? part >> 1 : part) * SY, t.z, nz, k_pad, cc, W, sw, ldw, xmax, ymax,
          0, 1, 0, 0);
      return;
    }
  }
  const int whole = TAIL > 0 ? full : (int)gridDim.x;
  int place = B == 256 && rounds ? round_place(bid, whole) : xcd_place(bid, whole);
  const int per_split = tiles_x * tiles_y * nz;
  const int sidx = SPLIT ? place / per_split : 0;
  place -= sidx * per_split;
  const TilePos t = tile_at(place, tiles_x, tiles_y, group);
  gemm_body<B, B, NWX, NWY, EPI, BF16, FOLD, SPLIT, NS>(lds, X, sx, Y, sy, t.tx * B, t.ty * B, t.z,
                                                        nz, k_pad, cc, W, sw, ldw, xmax, ymax, sidx,
                                                        SPLIT ? nsplit : 1, vx, vy);
}

// ---- split-k reductions ------------------------------------------------------
// W (EPI 0): slice z = mod(sum over s of partial slice s * nz + z, p_z); each
// partial is in [-128, 127], so for nsplit <= 64 the sum stays below 2^13 in
// magnitude.  Workgroup row blockIdx.y is slice z; 16 bytes a thread.
__global__ __launch_bounds__(256) void k_reduce_w(const int8_t* __restrict__ part, int nsplit,
                                                  int nz, int64_t sw16, CrtConsts cc,
                                                  int8_t* __restrict__ W) {
  const int z = blockIdx.y;
  const SmallMod md(cc, z);
  const uint4* src = reinterpret_cast<const uint4*>(part);
  uint4* dst = reinterpret_cast<uint4*>(W) + z * sw16;
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < sw16;
       t += (int64_t)gridDim.x * 256) {
    int acc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0;
    // eight loads before any use; past the last split the last one again, not added
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
      uint4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        v[u] = src[((int64_t)min(s0 + u, nsplit - 1) * nz + z) * sw16 + t];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (s0 + u >= nsplit) break;
        const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] += sbyte(w[e >> 2], e & 3);
      }
    }
    uint32_t o[4] = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 16; ++e) o[e >> 2] |= md.byte(acc[e], e & 3);
    dst[t] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// Cbar (EPI 1) from nsplit INT32 partial sums (column-major, ld nx): one
// entry (x, y) per thread, workgroups of 64 x by 4 y.  Each wave (64
// consecutive x of one y) sends its maximum to ymax[y]; the four rows of a
// workgroup are combined in LDS and sent to xmax[x] (atomicMax, order-free;
// Cbar >= 0).  nx is a multiple of 128.
__global__ __launch_bounds__(256) void k_reduce_cbar(const int* __restrict__ part, int nsplit,
                                                     int nx, int ny, int* __restrict__ xmax,
                                                     int* __restrict__ ymax) {
  __shared__ int rows[4][64];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int x = blockIdx.x * 64 + tx, y = blockIdx.y * 4 + ty;
  const size_t per = (size_t)nx * ny;
  int v = 0;
  if (y < ny) {
    const int* src = part + (size_t)y * nx + x;
    for (int s0 = 0; s0 < nsplit; s0 += 8) {   // eight loads before any use
      int w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) w[u] = src[min(s0 + u, nsplit - 1) * per];
#pragma unroll
      for (int u = 0; u < 8; ++u) v += s0 + u < nsplit ? w[u] : 0;
    }
    int cm = v;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) cm = max(cm, __shfl_xor(cm, off));
    if (tx == 0) atomicMax(&ymax[y], cm);
  }
  rows[ty][tx] = v;
  __syncthreads();
  if (ty == 0)
    atomicMax(&xmax[x], max(max(rows[0][tx], rows[1][tx]), max(rows[2][tx], rows[3][tx])));
}

// Grouped: the scaling product (EPI 1) or the N residue products (EPI 0) of
// every problem of a batch.
template <int B, int EPI, bool FOLD>
__global__ __launch_bounds__(tile_threads<B>(), TileShape<B>::OCC) void kg_gemm(
    const ProbDesc* __restrict__ P, const BlockRef* __restrict__ map,
    const CrtConsts* __restrict__ ctab) {
  const BlockRef e = map[blockIdx.x];
  const ProbDesc& d = P[e.x];
  const int nz = EPI == 0 ? d.N : 1;
  __shared__ __attribute__((aligned(1024))) int8_t lds[2 * 2 * B * 128];
  const int tiles_x = d.mp / B, tiles_y = d.np / B;
  const int place = xcd_place(e.y, group_gemm_blocks(d.mp, d.np, B, nz));
  if (place >= tiles_x * tiles_y * nz) return;   // whole workgroup, before any barrier
  const TilePos t = tile_at(place, tiles_x, tiles_y);
  gemm_body<B, B, TileShape<B>::NWX, TileShape<B>::NWY, EPI, false, FOLD, false, 2>(
      lds, d.As, EPI == 0 ? (size_t)d.mp * d.kp : 0, d.Bs, EPI == 0 ? (size_t)d.np * d.kp : 0,
      t.tx * B, t.ty * B, t.z, nz, d.kp, ctab[d.N], d.W, (size_t)d.np * d.mp, d.mp, d.rmax, d.cmax, 0,
      1, 0, 0);
}

// Persistent grouped residue products (see gemm_persist).
template <int B, bool FOLD>
__global__ __launch_bounds__(tile_threads<B>(), TileShape<B>::OCC) void kp_gemm(
    const ProbDesc* __restrict__ P, const BlockRef* __restrict__ map, int items,
    const CrtConsts* __restrict__ ctab) {
  gemm_persist<B, B, TileShape<B>::NWX, TileShape<B>::NWY, FOLD>(P, map, items, ctab);
}

// Whether a launch walks its tiles in rounds over all XCDs (round_place) or
// gives each XCD a range of its own.  In ranges, the XCDs work on up to eight
// slices at once, whose operands the MALL (256 MB) holds when they are small; in
// rounds all read the same panels.  Residue products in ranges and in rounds:
// 7 of 16384^3 (537 MB a slice) 23.8 and 21.4 ms, 14 of 8192^3 (134 MB) 5550 and
// 5390 us, of 3000x3000x20000 (122 MB) 2160 and 2045; but of 4096x4096x8192 (67
// MB) 1383 and 1445, 18 of 4096^3 (34 MB) 936 and 987.  The bytes are not all of it:
// below the line 5000^3 (52 MB) and 6000^3 (75 MB) would gain 3 to 4%, where their
// neighbours at powers of two lose as much.  Outputs of fewer than 8 tiles one way
// and no more than a round of them have no 16 x 16 places to share panels in and gain
// only from a longer k: 7 products of 24576x256x8192 429 and 486 us, x 66000 3810 and
// 3595; of 16384x1000x8192 663 and 743, x 66000 7019 and 6586 (but the whole call of
// 60000x500x8192, 470 tiles, 3766 and 3634).  A launch of less than one round stays
// in ranges (scaling product of 3000x3000x66000, 144 tiles: 909 and 1027 us).
bool walk_in_rounds(int nx_pad, int ny_pad, int k_pad, int wgs) {
  const int tx = nx_pad / 256, ty = ny_pad / 256;
  const bool thin = std::min(tx, ty) < 8 && (int64_t)tx * ty <= kCus;
  return (size_t)(nx_pad + ny_pad) * k_pad > kRoundBytes && wgs >= kCus &&
         (!thin || k_pad >= 1 << 15);
}

template <int B>
void launch_cfg(hipStream_t s, int epi, const int8_t* X, size_t sx, const int8_t* Y, size_t sy,
                int nx_pad, int ny_pad, int k_pad, int nz, const CrtConsts& cc, int8_t* W,
                size_t sw, int ldw, int* xmax, int* ymax, int nsplit, bool fold, int vx, int vy) {
  const int tiles_x = nx_pad / B, tiles_y = ny_pad / B;
  const int wgs = tiles_x * tiles_y * nz * nsplit;
  int full = wgs;
  const int rounds = B == 256 && nsplit == 1 && walk_in_rounds(nx_pad, ny_pad, k_pad, wgs);
  dim3 grid((unsigned)wgs);
  const dim3 block(tile_threads<B>());
  const bool deep = B == 128 && wgs <= kCus;   // one workgroup per CU: the deep ring
#define OZ2_GEMM_NS(E, F, S, NS, T)                                                             \
  hipLaunchKernelGGL((k_gemm_i8<B, E, false, F, S, NS, T>), grid, block, 0, s, X, sx, Y, sy,     \
                     tiles_x, tiles_y, nz, k_pad, W, sw, ldw, xmax, ymax, nsplit, full, vx, \
                     vy, rounds, cc)
#define OZ2_GEMM(E, F, S)                                                                       \
  do {                                                                                          \
    if constexpr (B == 128) {                                                                   \
      if (deep)                                                                                 \
        OZ2_GEMM_NS(E, F, S, 4, 0);                                                             \
      else                                                                                      \
        OZ2_GEMM_NS(E, F, S, 2, 0);                                                             \
    } else {                                                                                    \
      OZ2_GEMM_NS(E, F, S, 2, 0);                                                               \
    }                                                                                           \
  } while (0)
  const bool split = nsplit > 1;
  switch (epi) {
    case 0:
      if (split) {
        if (fold)
          OZ2_GEMM(0, true, true);
        else
          OZ2_GEMM(0, false, true);
      } else {
        if constexpr (B == 256) {
          const int parts = fold ? 0 : tail_parts(wgs);
          if (parts) {
            full = wgs / kCus * kCus;
            grid = dim3((unsigned)(full + (wgs - full) * parts));
            if (parts == 2)
              OZ2_GEMM_NS(0, false, false, 2, 2);
            else
              OZ2_GEMM_NS(0, false, false, 2, 4);
            break;
          }
        }
        if (fold)
          OZ2_GEMM(0, true, false);
        else
          OZ2_GEMM(0, false, false);
      }
      break;
    case 1:
      OZ2_GEMM(1, false, false);
      break;
    case 3:
      OZ2_GEMM(3, false, false);
      break;
    default:
      if (split)
        OZ2_GEMM(4, false, true);   // the split scaling product (never folded)
      else if (fold)
        OZ2_GEMM(4, true, false);
      else
        OZ2_GEMM(4, false, false);
      break;
  }
#undef OZ2_GEMM
#undef OZ2_GEMM_NS
}

// Tile configuration: 0 = automatic; 1 = 256x256, 2 = 128x128 (g_gemm_tile,
// a tuning knob set through ozaki2_debug_tuning).
int forced_cfg() { return g_gemm_tile.load(std::memory_order_relaxed); }

// 256x256 tiles (one workgroup per CU, 128 KB of LDS) when there are more
// than 128 of them, that is when the 128x128 tiles (two workgroups per CU,
// 64 KB of LDS each) would need more than one round of the 512 workgroup
// slots; otherwise 128x128.  Measured on square products from 1024^3 to
// 4096^3 (16 to 896 tiles of 256x256): 144 or more tiles ran 7-25% faster
// as 256x256, 64 or fewer 30-40% faster as 128x128.
bool use_256(int nx_pad, int ny_pad, int nz) {
  const bool fits256 = nx_pad % 256 == 0 && ny_pad % 256 == 0;
  const int cfg = forced_cfg();
  if (cfg == 1 || cfg == 2) return cfg == 1 && fits256;
  const long t256 = (long)(nx_pad / 256) * (ny_pad / 256) * nz;
  return fits256 && t256 > 128;
}

// Split-k of a product with few output workgroups.  The residue products (EPI
// 0), W0 = tiles * nz workgroups of G = k_pad / 128 groups of k: nsplit = the
// number of copies of W0 that fill the workgroup slots once (CUs x occupancy:
// 256 for 256x256 tiles, 512 for 128x128), at most G / 4 (512 k or more per
// split) and 64; 1 when W0 already fills a quarter of the slots.  Measured
// (FP64, N = 14): 512^2 x 32768 (224 workgroups) ran 3% slower with two splits
// than with none; at 256^2 x 131072 the split products ran 2.4x faster.  A
// fixed count of 256 CUs keeps the choice, and with it the workspace size, a
// function of the shape alone.
int choose_split(int nx_pad, int ny_pad, int k_pad, int nz) {
  if (g_split_k.load(std::memory_order_relaxed) == 1) return 1;
  const int B = use_256(nx_pad, ny_pad, nz) ? 256 : 128;
  const long w0 = (long)(nx_pad / B) * (ny_pad / B) * nz;
  const long slots = B == 256 ? kCus : 2 * kCus;
  if (w0 <= 0 || 4 * w0 > slots) return 1;
  long sp = slots / w0;
  sp = std::min<long>(sp, (k_pad / 128) / 4);
  sp = std::min<long>(sp, 64);
  return sp >= 2 ? (int)sp : 1;
}

// Splits of the scaling product (EPI 1), whose partials are INT32, at most what
// `bytes` of scratch hold: the count with the least modelled time.  With one
// workgroup per CU a group of k takes about 0.3 us; splitting costs another
// launch and the partials' way through memory (about 3 TB/s both ways).
// Measured, with the fixed count of 4096 of k a split that this replaces and
// with this one (the scratch is the same): 128x128x8192 (64 groups) 27.5 and
// 12.2 us, 200x200x100000 (782) 54 and 26, 64x64x262144 (2048) 122 and 28.  At
// 1024^2 x 1024 and x 4096 two and more splits were slower than one.
// With more than 32 tiles over 256 groups or more the L2 bounds it, not the latency
// of a group: one workgroup per CU reads 10 to 12 TB/s, two read 13 to 15, if they
// fill the slots (at least 16 of 9 splits).  One and two per CU, scratch permitting:
// 36 tiles of 1024 groups 108 and 100 us, 54 of 256 59 and 54, of 2048 332 and 265,
// 100 of 256 97 and 78, of 2048 614 and 432; but 32 of 1024 97 and 102, and two of
// the 15 shapes from 512 groups on lose 2 and 4% (64 and 48 tiles of 512).
int choose_split_cbar(int nx_pad, int ny_pad, int k_pad, size_t bytes) {
  if (g_split_k.load(std::memory_order_relaxed) == 1) return 1;
  const int B = use_256(nx_pad, ny_pad, 1) ? 256 : 128;
  const long w0 = (long)(nx_pad / B) * (ny_pad / B), G = k_pad / 128;
  const double plane = 4.0 * nx_pad * ny_pad;
  if (B == 256 || w0 <= 0) return 1;
  auto fit = [&](long slots) {
    return std::min<long>({slots / w0, G / 4, (long)((double)bytes / plane), 64});
  };
  const long most = fit(kCus), two = fit(2 * kCus);
  if (w0 > 32 && G >= 256 && two >= 2 && 9 * two >= 16 * most) return (int)two;
  int best = 1;
  double t_best = 0.3 * (double)G;
  for (long sp = 2; sp <= most; ++sp) {
    const double t = 0.3 * (double)((G + sp - 1) / sp) + 5.0 + 2.0 * (double)sp * plane / 3e6;
    if (t < t_best) {
      t_best = t;
      best = (int)sp;
    }
  }
  return best;
}

}  // namespace

std::atomic<int> g_split_k{0};

size_t split_scratch_bytes(int nx_pad, int ny_pad, int k_pad, int nz) {
  const size_t plane = (size_t)nx_pad * ny_pad;
  const int s0 = choose_split(nx_pad, ny_pad, k_pad, nz);
  const size_t b0 = s0 > 1 ? (size_t)s0 * nz * plane : 0;
  // INT32 partials of the scaling product: a slot for each time that its tiles
  // fit the 512 slots (few tiles), 4096 of k or more and at most 16
  size_t b1 = 0;
  if (g_split_k.load(std::memory_order_relaxed) != 1) {
    const int B = use_256(nx_pad, ny_pad, 1) ? 256 : 128;
    const long w0 = (long)(nx_pad / B) * (ny_pad / B), slots = B == 256 ? kCus : 2 * kCus;
    if (w0 > 0 && 4 * w0 <= slots) {
      const long s1 = std::min<long>({slots / w0, k_pad / 128 / 32, 16});
      if (s1 >= 2) b1 = (size_t)s1 * plane * 4;
    }
  }
  return b0 > b1 ? b0 : b1;
}

std::atomic<int> g_gemm_tile{0};

int persist_grid(int tile) {
  int dev = 0, cus = 0, occ = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus < 1)
    cus = 256;
  const void* k = tile == 256 ? reinterpret_cast<const void*>(kp_gemm<256, true>)
                              : reinterpret_cast<const void*>(kp_gemm<128, true>);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, tile == 256 ? tile_threads<256>()
                                                                        : tile_threads<128>(),
                                                   0) != hipSuccess ||
      occ < 1)
    occ = 1;
  return (cus * occ + 7) / 8 * 8;   // a multiple of 8: entries keep their XCD
}

void launch_group_gemm_persist(hipStream_t s, int tile, bool fold, int grid, const ProbDesc* P,
                               const BlockRef* map, int items, const CrtConsts* ctab) {
  if (items <= 0) return;
  const dim3 g((unsigned)(grid < items ? grid : (items + 7) / 8 * 8));
  if (tile == 256) {
    const dim3 b(tile_threads<256>());
    if (fold)
      hipLaunchKernelGGL((kp_gemm<256, true>), g, b, 0, s, P, map, items, ctab);
    else
      hipLaunchKernelGGL((kp_gemm<256, false>), g, b, 0, s, P, map, items, ctab);
  } else {
    const dim3 b(tile_threads<128>());
    if (fold)
      hipLaunchKernelGGL((kp_gemm<128, true>), g, b, 0, s, P, map, items, ctab);
    else
      hipLaunchKernelGGL((kp_gemm<128, false>), g, b, 0, s, P, map, items, ctab);
  }
}

void launch_group_gemm(hipStream_t s, int epi, int tile, const ProbDesc* P, const BlockRef* map,
                       int blocks, const CrtConsts* ctab) {
  if (blocks <= 0) return;
  const dim3 g((unsigned)blocks);
  if (tile == 256) {
    const dim3 b(tile_threads<256>());
    if (epi == 0)
      hipLaunchKernelGGL((kg_gemm<256, 0, true>), g, b, 0, s, P, map, ctab);
    else
      hipLaunchKernelGGL((kg_gemm<256, 1, false>), g, b, 0, s, P, map, ctab);
  } else {
    const dim3 b(tile_threads<128>());
    if (epi == 0)
      hipLaunchKernelGGL((kg_gemm<128, 0, true>), g, b, 0, s, P, map, ctab);
    else
      hipLaunchKernelGGL((kg_gemm<128, 1, false>), g, b, 0, s, P, map, ctab);
  }
}

void launch_gemm_bf16_store(hipStream_t s, const uint16_t* X, const uint16_t* Y, int nx_pad,
                            int ny_pad, int k_pad, float* S, int lds_) {
  // BF16 rows are 2*k_pad bytes; the kernel works in bytes of k.
  const int kb = 2 * k_pad;
  CrtConsts cc{};
  if (use_256(nx_pad, ny_pad, 1)) {
    const int tiles_x = nx_pad / 256, tiles_y = ny_pad / 256;
    hipLaunchKernelGGL((k_gemm_i8<256, 2, true>), dim3((unsigned)(tiles_x * tiles_y)),
                       dim3(tile_threads<256>()), 0, s, (const int8_t*)X, 0, (const int8_t*)Y, 0,
                       tiles_x, tiles_y, 1, kb, (int8_t*)S, 0, lds_, nullptr, nullptr, 1,
                       tiles_x * tiles_y, nx_pad, ny_pad, 0, cc);
  } else {
    const int tiles_x = nx_pad / 128, tiles_y = ny_pad / 128;
    hipLaunchKernelGGL((k_gemm_i8<128, 2, true>), dim3((unsigned)(tiles_x * tiles_y)),
                       dim3(tile_threads<128>()), 0, s, (const int8_t*)X, 0, (const int8_t*)Y, 0,
                       tiles_x, tiles_y, 1, kb, (int8_t*)S, 0, lds_, nullptr, nullptr, 1,
                       tiles_x * tiles_y, nx_pad, ny_pad, 0, cc);
  }
}

void launch_gemm_i8(hipStream_t s, int epi, const int8_t* X, size_t sx, const int8_t* Y, size_t sy,
                    int nx_pad, int ny_pad, int k_pad, int nz, const CrtConsts& cc, int8_t* W,
                    size_t sw, int ldw, int* xmax, int* ymax, int8_t* part, size_t part_bytes,
                    int vx, int vy) {
  const bool b256 = use_256(nx_pad, ny_pad, nz);
  if (vx <= 0) vx = nx_pad;
  if (vy <= 0) vy = ny_pad;
  const int G = k_pad / 128;
  int sp = 1;
  if (epi == 0 || epi == 1) {
    sp = epi == 0 ? choose_split(nx_pad, ny_pad, k_pad, nz)
                  : choose_split_cbar(nx_pad, ny_pad, k_pad, part ? part_bytes : 0);
    const size_t plane = (size_t)nx_pad * ny_pad;
    const size_t need = epi == 0 ? (size_t)sp * nz * plane : (size_t)sp * plane * 4;
    // Fewer splits, one workgroup per CU with the deep ring, where these fill 15 of
    // 16 CUs.  Residue products with two workgroups per CU and with one: 128x128 x
    // 16384 27.8 and 22.8 us, 100x100x50000 42.3 and 35.3, 64x64x262144 143 and
    // 135; where 224 of 256 CUs would have one, 200x200x100000, 158 and 164.  With
    // more than 4 tiles a slice, whose workgroups share panels in L2, two are faster
    // (16 tiles, N = 8: 16384 of k 41 and 47; 60 tiles, N = 2: 36 and 45, 50000 107
    // and 125), up to 16 tiles below 2^17 of k (there 363 and 346; 25 tiles, N = 5,
    // 309 and 327).
    if (epi == 0 && !b256 && sp > 1) {
      const long tiles = (long)(nx_pad / 128) * (ny_pad / 128), w0 = tiles * nz;
      const long sp1 = kCus / w0;
      if (sp1 >= 2 && 16 * sp1 * w0 >= 15 * kCus && (tiles <= 4 || (tiles <= 16 && G >= 1024)))
        sp = (int)std::min<long>(sp, sp1);
    }
    // the partials use the plane layout (stride nx_pad * ny_pad, rows of
    // nx_pad): W must have it too
    const bool plane_w = epi == 1 || (sw == plane && ldw == nx_pad);
    if (sp > 1 && (!part || part_bytes < need || !plane_w)) sp = 1;
  }
  // every split keeps at least one group; fold when a split spans more than 2^17 of k
  const bool fold = (G + sp - 1) / sp > kFoldGroups;
  auto launch = [&](int e, int8_t* out, size_t so, int ld, int* xm, int* ym, int z, bool f) {
    if (b256)
      launch_cfg<256>(s, e, X, sx, Y, sy, nx_pad, ny_pad, k_pad, z, cc, out, so, ld, xm, ym, sp, f, vx,
                      vy);
    else
      launch_cfg<128>(s, e, X, sx, Y, sy, nx_pad, ny_pad, k_pad, z, cc, out, so, ld, xm, ym, sp, f, vx,
                      vy);
  };
  if (sp == 1) {
    launch(epi, W, sw, ldw, xmax, ymax, nz, fold && (epi == 0 || epi == 4));
    return;
  }
  const size_t plane = (size_t)nx_pad * ny_pad;
  if (epi == 0) {
    // partial W of every split (mod p of its partial sum), then their sum mod p
    launch(0, part, plane, nx_pad, nullptr, nullptr, nz, fold);
    const int64_t sw16 = (int64_t)(plane / 16);
    const int64_t b = (sw16 + 255) / 256;
    hipLaunchKernelGGL(k_reduce_w, dim3((unsigned)(b < 1024 ? b : 1024), (unsigned)nz), dim3(256),
                       0, s, part, sp, nz, sw16, cc, W);
  } else {
    // INT32 partial sums of Cbar (never reduced mod p: Cbar < 2^31), then
    // their sum and its row and column maxima
    launch(4, part, plane, nx_pad, nullptr, nullptr, 1, false);
    const dim3 g((unsigned)(nx_pad / 64), (unsigned)((ny_pad + 3) / 4));
    hipLaunchKernelGGL(k_reduce_cbar, g, dim3(256), 0, s, (const int*)part, sp, nx_pad, ny_pad,
                       xmax, ymax);
  }
}

}  // namespace oz2
