// bf16 GEMM on gfx950 matrix cores (v_mfma_f32_32x32x16_bf16), fp32 accumulation.
//
//   C[m, n] = alpha * sum_k A(m, k) B(n, k) + beta * C[m, n]
//
// Either operand may be K-contiguous ("k-major": rows of a weight or of activations) or
// M/N-contiguous (the transposed operand of the weight-gradient and data-gradient
// products).  A workgroup owns a BM x BN output tile and walks K in BK = 64 slices staged
// in LDS in the operand's natural layout: k-major tiles as [row][k] (16-byte operand reads,
// 8 consecutive k per lane) and m-major tiles as [k][row], whose operands come from
// gfx950's transposing LDS read.  Both give the same k order inside an MFMA step, so the
// two kinds mix freely.  LDS is double buffered: full K slices are copied straight from
// HBM into LDS (global_load_lds) while the current slice feeds the matrix cores; a ragged
// last slice goes through registers with zero fill.  Operand fragments are double buffered
// in registers as well: the LDS reads of the next 16-wide k step are in flight while the
// matrix cores work on the current one, and the first step of the next slice is read
// right after the barrier that publishes it.  The epilogue stages each 32-row strip of a
// wavefront's tile in LDS and writes it back with 16-byte (fp32) or 8-byte (bf16) stores.
// Plain products run persistent: one workgroup per CU slot walks the tiles, and the next
// tile's first slice is copied while the current one finishes and writes its epilogue.
// The operand reads of a wavefront hit distinct banks: k-major rows are XOR-swizzled in
// 16-byte chunks, m-major row strides are padded.  Large problems use 256 x 256 tiles on
// 8 wavefronts (128 x 64 each), which halves the LDS bytes per MFMA compared with
// 128 x 128 tiles on 4 wavefronts (64 x 64 each), used for middling problems.  Workgroup
// ids are remapped so that neighbouring tiles (sharing A row panels or B column panels)
// run on one XCD and hit its L2.  Weight gradients reduce over all tokens (K up to 1e5)
// and have few output tiles: they are split along K into fp32 partials that a second
// kernel sums in a fixed order (deterministic).  Products too small to fill the chip take
// 64 x 64 tiles with four slices in flight, and split along K in any layout.  Large NT
// products run on a four-wavefront kernel whose k steps are scheduled by hand (below,
// gemm_nt4).  A tile that the matrix edge would cut is moved back to end at the edge, so
// that its copies stay whole, and stores only its own rows and columns.  Several products
// of one layout can share a launch (gemm_mfma_group).  Which tiles, split and grouping a
// product gets is the cheapest by a fitted time model (plan_of).
#include <atomic>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "mfma.h"

#include <algorithm>

namespace mla {

namespace {

constexpr int BK = 64;  // K granule of split-K chunks (and the slice of the small tiles)
// slice depth, LDS ring depth and wavefront grid of the 256 x 256 tiles (measured on the
// step's shapes: deeper rings of 32-deep slices and 4-wavefront grids of 128 x 128 were
// slower)
constexpr int GBK = 64, GNST = 2, GWM = 2, GWN = 4;

struct GemmDev {
  int M, N;
  const bf16_t* A; int64_t lda;
  const bf16_t* B; int64_t ldb;
  void* C; int64_t ldc;
  float* part;        // split-K partials [splits][M][N], or null
  // masked-loss epilogue (with lscale set): C = lscale[0] mask[m] acc (not stored when C is
  // NULL) and, with lpart set, lpart[tile] = the sum over the tile of mask[m] acc^2, or of mask[m] acc
  // lref[m, n] when lref is set
  const float* lscale; const uint8_t* lmask; double* lpart;
  const bf16_t* lref; int64_t ldref;
  float alpha, beta;
  int kchunk;         // K elements per split (multiple of BK)
  int nsplit;         // split-K chunks (persistent launch)
  int aligned;        // rows of A and B 16-byte aligned (gemm_tile)
  int ktotal;
  int mstore;         // rows of C written (M is the row count operand A may be read at)
  // batched causal mode (causal != 0): workgroup z of nbatch works on A + z sA,
  // B + (z / zdiv) sB1 + ((z % zdiv) / bdiv) sB2, C + (z / zdiv) sC1 + (z % zdiv) sC2; the
  // K range of an M tile ends at its last row (entries with k > m are zero) or, with rev,
  // starts at its first row (entries with k < m are zero); it is walked kgroups times, the
  // j-th time on A + j sAk and B + j sBk (a sum over stacked operands)
  int causal, rev, nbatch, zdiv, bdiv, kgroups;
  int64_t sA, sB1, sB2, sC1, sC2, sAk, sBk;
  // split output of the persistent causal k-major product (dK), when split_n > 0: columns
  // n < split_n in bf16 at c_lo + z1 sC1_lo + z2 sC2_lo + m ldc_lo + n, the rest (fp32) at C
  // with the strides above, column n - split_n
  int split_n;
  bf16_t* c_lo; int64_t ldc_lo, sC1_lo, sC2_lo;
};

// row stride (elements) of an m-major [k][ROWS] tile, read only through the transposing
// read (32 lanes cover 4 consecutive rows x 64 bytes): a stride of 16 or 48 banks modulo
// 64 puts the 4 rows on disjoint banks
constexpr int mm_ld(int rows) {
  for (int p = 8; p <= 64; p += 8) {
    const int r = ((rows + p) / 2) % 64;
    if (r == 16 || r == 48) return rows + p;
  }
  return rows + 32;
}
// A operand of the batched causal products: dS^T stored in 32 x 32 tiles, element (key r,
// query c) at ((r / 32) tq + c / 32) 1024 + (r % 32) 32 + c % 32 (tq: tiles per row of
// tiles), so that each wavefront of the producer writes its 32 x 32 block as 2 KB of
// whole lines and a slice of 32 keys x 256 queries is 16 KB of consecutive tiles
__device__ __forceinline__ int64_t tile32_off(int64_t r, int64_t c, int64_t tq) {
  return ((r >> 5) * tq + (c >> 5)) * 1024 + (r & 31) * 32 + (c & 31);
}

// ---- global -> register staging -------------------------------------------------------
// (rows of the caller's arrays need no more than their elements' alignment here)
typedef u32x4 u32x4_any __attribute__((aligned(2)));
template <bool KMAJOR, int ROWS, int NTHR, int BK, bool TILED = false>
struct Loader;

// k-major tile: ROWS x BK, chunk c -> row c / (BK/8), k-chunk c % (BK/8).  Rows are not
// padded: the 16-byte chunk holding k-chunk c of row r sits at position c ^ swz(r) of its
// row, so that the 16 rows one operand read covers per LDS cycle (one k-chunk each) fall on
// 16 distinct 16-byte bank groups (a 256-byte bank window holds 128 / BK rows)
template <int ROWS, int NTHR, int BK>
struct Loader<true, ROWS, NTHR, BK, false> {
  static constexpr int KM_LD = BK;
  static constexpr int NCH = BK / 8;    // 16-byte chunks per row
  static constexpr int RPW = 128 / BK;  // rows per 256-byte bank window
  static_assert(BK == 32 || BK == 64, "k-major slice depth");
  static __device__ __forceinline__ int swz(int row) { return (row / RPW) % NCH; }
  static constexpr int CHUNKS = ROWS * NCH;
  static constexpr int PER = (CHUNKS + NTHR - 1) / NTHR;
  using Dma = DmaTile<ROWS, BK, KM_LD, NTHR / 64, true>;
  static constexpr int ELEMS = Dma::ALLOC;  // whole 1 KB blocks, a multiple per wavefront
  // the copy that fills LDS position (row, p) fetches k-chunk p ^ swz(row)
  static __device__ __forceinline__ void swizzle(Dma& t) {
#pragma unroll
    for (int p = 0; p < Dma::PER; ++p)
      t.col[p] = (short)(8 * ((t.col[p] / 8) ^ swz(t.row[p])));
  }
  u32x4 r[PER];
  __device__ __forceinline__ void load(const bf16_t* __restrict__ p, int64_t ld, int row0,
                                       int rows_valid, int k0, int kend) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = threadIdx.x + i * NTHR;
      const int row = c / NCH, kc = (c % NCH) * 8;
      u32x4 v = {0u, 0u, 0u, 0u};
      if ((CHUNKS % NTHR == 0 || c < CHUNKS) && row < rows_valid && k0 + kc < kend)
        v = *(const u32x4_any*)(p + (int64_t)(row0 + row) * ld + k0 + kc);
      r[i] = v;
    }
  }
  __device__ __forceinline__ void store(bf16_t* lds) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = threadIdx.x + i * NTHR;
      const int row = c / NCH;
      if (CHUNKS % NTHR == 0 || c < CHUNKS)
        *(u32x4*)(lds + row * KM_LD + 8 * ((c % NCH) ^ swz(row))) = r[i];
    }
  }
  // full k-slice of a full tile straight from HBM into LDS (uniform base + lane offset)
  __device__ __forceinline__ void dma(const Dma& t, const bf16_t* __restrict__ p, int64_t ld,
                                      int row0, int rows_valid, int k0, bf16_t* lds) const {
    t.issue_s(lds, p + (int64_t)row0 * ld + k0, [&](int r, int c) { return r * (int)ld + c; });
  }
  // the same for a tile cut by the matrix edge: rows past it repeat the last valid one
  // (they feed only output rows that are not stored)
  __device__ __forceinline__ void dma_edge(const Dma& t, const bf16_t* __restrict__ p, int64_t ld,
                                           int row0, int rows_valid, int k0, bf16_t* lds) const {
    t.issue_s(lds, p + (int64_t)row0 * ld + k0,
              [&](int r, int c) { return min(r, rows_valid - 1) * (int)ld + c; });
  }
  // operand fragment: rows row0 + lane%32, k = 16 kk + 8 half + 0..7 (row0 is a multiple of
  // 32, so the swizzle depends on the lane only)
  static __device__ __forceinline__ bf16x8 frag(const bf16_t* lds, int row0, int kk) {
    const int lane = threadIdx.x & 63, l = lane & 31;
    const int c = 2 * kk + (lane >> 5);
    return *(const bf16x8*)(lds + (row0 + l) * KM_LD + 8 * (c ^ swz(l)));
  }
};

// m-major tile (global [k][row]): BK x ROWS, chunk c -> k-row c / (ROWS/8), row-chunk c % (ROWS/8).
// Rows of a multiple of 64 elements are unpadded and XOR-swizzled in aligned groups of four
// 16-byte chunks (64 bytes, 16 banks), so that the 4 k-rows x 64 bytes one transposing read
// covers per half-wavefront fall on 4 distinct 16-bank groups: with rows a multiple of
// 256 bytes long every row starts on the same bank, and group G of k-row k sits at
// G ^ (k mod 4); with rows an odd multiple of 128 bytes, odd rows start half a bank
// window (two groups) later, and group G sits at G ^ ((k / 2) mod 2).  Other widths keep padded rows.
template <int ROWS, int NTHR, int BK>
struct Loader<false, ROWS, NTHR, BK, false> {
  static constexpr bool SWZ = ROWS % 64 == 0;
  static constexpr bool SWZ4 = ROWS % 128 == 0;  // else rows are an odd multiple of 128 B
  static constexpr int LD = SWZ ? ROWS : mm_ld(ROWS);
  static constexpr int CPR = ROWS / 8;
  static constexpr int CHUNKS = BK * CPR;
  static constexpr int PER = (CHUNKS + NTHR - 1) / NTHR;
  using Dma = DmaTile<BK, ROWS, LD, NTHR / 64, true>;
  static constexpr int ELEMS = Dma::ALLOC;  // whole 1 KB blocks, a multiple per wavefront
  static __device__ __forceinline__ int pos(int k, int c) {
    return !SWZ ? c : SWZ4 ? c ^ (4 * (k & 3)) : c ^ (4 * ((k >> 1) & 1));
  }
  // the copy that fills LDS position (k, p) fetches chunk pos(k, p) (an involution)
  static __device__ __forceinline__ void swizzle(Dma& t) {
    if constexpr (SWZ) {
#pragma unroll
      for (int p = 0; p < Dma::PER; ++p) t.col[p] = (short)(8 * pos(t.row[p], t.col[p] / 8));
    }
  }
  u32x4 r[PER];
  __device__ __forceinline__ void load(const bf16_t* __restrict__ p, int64_t ld, int row0,
                                       int rows_valid, int k0, int kend) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = threadIdx.x + i * NTHR;
      const int kr = c / CPR, rc = (c % CPR) * 8;
      u32x4 v = {0u, 0u, 0u, 0u};
      if ((CHUNKS % NTHR == 0 || c < CHUNKS) && rc < rows_valid && k0 + kr < kend)
        v = *(const u32x4_any*)(p + (int64_t)(k0 + kr) * ld + row0 + rc);
      r[i] = v;
    }
  }
  __device__ __forceinline__ void store(bf16_t* lds) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = threadIdx.x + i * NTHR;
      const int kr = c / CPR;
      if (CHUNKS % NTHR == 0 || c < CHUNKS)
        *(u32x4*)(lds + kr * LD + pos(kr, c % CPR) * 8) = r[i];
    }
  }
  __device__ __forceinline__ void dma(const Dma& t, const bf16_t* __restrict__ p, int64_t ld,
                                      int row0, int rows_valid, int k0, bf16_t* lds) const {
    t.issue_s(lds, p + (int64_t)k0 * ld + row0, [&](int r, int c) { return r * (int)ld + c; });
  }
  // (chunks past the edge repeat the last valid one)
  __device__ __forceinline__ void dma_edge(const Dma& t, const bf16_t* __restrict__ p, int64_t ld,
                                           int row0, int rows_valid, int k0, bf16_t* lds) const {
    const int last = (rows_valid - 1) & ~7;
    t.issue_s(lds, p + (int64_t)k0 * ld + row0,
              [&](int r, int c) { return r * (int)ld + min(c, last); });
  }

  // operand fragment through the transposing read (lds_operand_tr's lane pattern: k-rows
  // klo + lane%16/4 and klo + 4 + lane%16/4, columns row0 + 16 ((lane/16) % 2) + 4 (lane % 4));
  // klo is a multiple of 4, so the swizzle's k mod 4 is the lane's lane%16/4
  static __device__ __forceinline__ bf16x8 frag(const bf16_t* lds, int row0, int kk) {
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
    const int klo = 16 * kk + 8 * (lane >> 5), kq = r >> 2;
    const int m = row0 + 16 * (g & 1) + 4 * (r & 3);
    const int mc = SWZ ? pos(kq, m >> 3) * 8 + (m & 7) : m;
    const u32x2 lo = lds_read_tr4(lds + (klo + kq) * LD + mc);
    const u32x2 hi = lds_read_tr4(lds + (klo + 4 + kq) * LD + mc);
    const u32x4 w = {lo[0], lo[1], hi[0], hi[1]};
    return __builtin_bit_cast(bf16x8, w);
  }
};

// A of the batched causal products: dS^T in 32 x 32 tiles (tile32_off), ld = the plane's
// row length (a multiple of 32).  The LDS copy of a slice holds the slice's tiles whole and
// in order, so that each 1 KB copy instruction moves 1 KB of consecutive global memory.
//
// Rows = keys, k = queries (the dK product): the slice's tiles (key tile i, query tile j)
// at (i NQT + j) 1024 elements; inside a tile, key row r (64 bytes) holds its 16-byte chunk
// q at position q ^ ((r / 4) % 4), so that the 16 rows one operand read covers per LDS
// cycle fall on 16 distinct 16-byte bank groups.
template <int ROWS, int NTHR, int BK>
struct Loader<true, ROWS, NTHR, BK, true> {
  static_assert(ROWS % 32 == 0 && BK % 32 == 0, "whole tiles");
  static constexpr int NQT = BK / 32;   // query tiles per slice
  static constexpr int NCH = BK / 8;    // 16-byte chunks per row
  static constexpr int CHUNKS = ROWS * NCH;
  static constexpr int PER = (CHUNKS + NTHR - 1) / NTHR;
  using Dma = DmaTile<ROWS * BK / 64, 64, 64, NTHR / 64, true>;  // the slice as flat 1 KB blocks
  static constexpr int ELEMS = Dma::ALLOC;
  static __device__ __forceinline__ int sw(int r) { return (r >> 2) & 3; }
  // LDS element of (row, k) of the slice (k a multiple of 8)
  static __device__ __forceinline__ int lds_off(int row, int k) {
    return ((row >> 5) * NQT + (k >> 5)) * 1024 + (row & 31) * 32 + 8 * (((k & 31) >> 3) ^ sw(row & 31));
  }
  static __device__ __forceinline__ void swizzle(Dma&) {}
  u32x4 r[PER];
  __device__ __forceinline__ void load(const bf16_t* __restrict__ p, int64_t ld, int row0,
                                       int rows_valid, int k0, int kend) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = threadIdx.x + i * NTHR;
      const int row = c / NCH, kc = (c % NCH) * 8;
      u32x4 v = {0u, 0u, 0u, 0u};
      if ((CHUNKS % NTHR == 0 || c < CHUNKS) && row < rows_valid && k0 + kc < kend)
        v = *(const u32x4*)(p + tile32_off(row0 + row, k0 + kc, ld >> 5));
      r[i] = v;
    }
  }
  __device__ __forceinline__ void store(bf16_t* lds) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = threadIdx.x + i * NTHR;
      if (CHUNKS % NTHR == 0 || c < CHUNKS) *(u32x4*)(lds + lds_off(c / NCH, (c % NCH) * 8)) = r[i];
    }
  }
  // LDS element e = 64 r + c of the flat block layout holds tile e / 1024 (key tile i,
  // query tile j), row (e % 1024) / 32, chunk position (e % 32) / 8; it is copied from the
  // same row of global tile (i, j), chunk position ^ sw(row)
  __device__ __forceinline__ void dma(const Dma& t, const bf16_t* __restrict__ p, int64_t ld,
                                      int row0, int rows_valid, int k0, bf16_t* lds) const {
    const int tq = (int)(ld >> 5);
    // dS^T is streamed once per product: non-temporal, so that it displaces less of the
    // B operand (Q) the caches keep between the row tiles of a batch entry
    t.template issue_s<true>(lds, p + tile32_off(row0, k0, tq), [&](int r, int c) {
      const int e = 64 * r + c, tile = e >> 10, w = e & 1023, rr = w >> 5;
      return ((tile / NQT) * tq + tile % NQT) * 1024 + rr * 32 + 8 * (((w & 31) >> 3) ^ sw(rr));
    });
  }
  // operand fragment: rows row0 + lane%32 (row0 a multiple of 32: one key tile), k = 16 kk +
  // 8 half + 0..7
  static __device__ __forceinline__ bf16x8 frag(const bf16_t* lds, int row0, int kk) {
    const int lane = threadIdx.x & 63, l = lane & 31;
    const int c = 2 * kk + (lane >> 5);
    return *(const bf16x8*)(lds + ((row0 >> 5) * NQT + (c >> 2)) * 1024 + l * 32 + 8 * ((c & 3) ^ sw(l)));
  }
};

// k = keys, rows = queries (the dQ product, 32-deep slices: one key tile per slice): the
// slice's query tiles in order, each a copy of its global tile ([32 keys][32 queries]); the
// transposing read of 4 key rows x 32 queries is then 256 consecutive bytes
template <int ROWS, int NTHR, int BK>
struct Loader<false, ROWS, NTHR, BK, true> {
  static_assert(BK == 32 && ROWS % 32 == 0, "one key tile per slice");
  static constexpr int CPR = ROWS / 8;
  static constexpr int CHUNKS = BK * CPR;
  static constexpr int PER = (CHUNKS + NTHR - 1) / NTHR;
  using Dma = DmaTile<BK, ROWS, ROWS, NTHR / 64, true>;
  static constexpr int ELEMS = Dma::ALLOC;
  static __device__ __forceinline__ int lds_off(int k, int m) { return (m >> 5) * 1024 + k * 32 + (m & 31); }
  static __device__ __forceinline__ void swizzle(Dma&) {}
  u32x4 r[PER];
  __device__ __forceinline__ void load(const bf16_t* __restrict__ p, int64_t ld, int row0,
                                       int rows_valid, int k0, int kend) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = threadIdx.x + i * NTHR;
      const int kr = c / CPR, rc = (c % CPR) * 8;
      u32x4 v = {0u, 0u, 0u, 0u};
      if ((CHUNKS % NTHR == 0 || c < CHUNKS) && rc < rows_valid && k0 + kr < kend)
        v = *(const u32x4*)(p + tile32_off(k0 + kr, row0 + rc, ld >> 5));
      r[i] = v;
    }
  }
  __device__ __forceinline__ void store(bf16_t* lds) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = threadIdx.x + i * NTHR;
      if (CHUNKS % NTHR == 0 || c < CHUNKS) *(u32x4*)(lds + lds_off(c / CPR, (c % CPR) * 8)) = r[i];
    }
  }
  // LDS element e = ROWS r + c of the flat block layout is element e of the slice's tiles
  // in global memory (they are consecutive)
  __device__ __forceinline__ void dma(const Dma& t, const bf16_t* __restrict__ p, int64_t ld,
                                      int row0, int rows_valid, int k0, bf16_t* lds) const {
    // dS^T streamed once: non-temporal (the keys stay cached between row tiles)
    t.template issue_s<true>(lds, p + tile32_off(k0, row0, ld >> 5),
                             [&](int r, int c) { return ROWS * r + c; });
  }
  static __device__ __forceinline__ bf16x8 frag(const bf16_t* lds, int row0, int kk) {
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
    const int klo = 16 * kk + 8 * (lane >> 5), kq = r >> 2;
    const int m = row0 + 16 * (g & 1) + 4 * (r & 3);
    const u32x2 lo = lds_read_tr4(lds + lds_off(klo + kq, m));
    const u32x2 hi = lds_read_tr4(lds + lds_off(klo + 4 + kq, m));
    const u32x4 w = {lo[0], lo[1], hi[0], hi[1]};
    return __builtin_bit_cast(bf16x8, w);
  }
};

template <typename TC>
__device__ __forceinline__ void store_out(TC* p, float v);
template <>
__device__ __forceinline__ void store_out<float>(float* p, float v) { *p = v; }
template <>
__device__ __forceinline__ void store_out<bf16_t>(bf16_t* p, float v) { *p = f2bf(v); }

// four consecutive outputs: alpha * v + beta * C
template <typename TC>
__device__ __forceinline__ void store4(TC* p, f32x4 v, float alpha, float beta);
template <>
__device__ __forceinline__ void store4<float>(float* p, f32x4 v, float alpha, float beta) {
  f32x4 o = v * alpha;
  if (beta != 0.f) o += beta * *(const f32x4*)p;
  *(f32x4*)p = o;
}
template <>
__device__ __forceinline__ void store4<bf16_t>(bf16_t* p, f32x4 v, float alpha, float beta) {
  f32x4 o = v * alpha;
  if (beta != 0.f) {
    const u32x2 c = *(const u32x2*)p;
    o[0] += beta * bf2f((bf16_t)(c[0] & 0xffff)); o[1] += beta * bf2f((bf16_t)(c[0] >> 16));
    o[2] += beta * bf2f((bf16_t)(c[1] & 0xffff)); o[3] += beta * bf2f((bf16_t)(c[1] >> 16));
  }
  *(u32x2*)p = u32x2{pack2bf(o[0], o[1]), pack2bf(o[2], o[3])};
}

// ---- edge tiles --------------------------------------------------------------------------
// A last row or column tile that the matrix edge cuts is moved back so that it is whole (and
// is copied straight to LDS like every other tile); it stores only the rows and columns that
// no other tile owns.  Through registers, with zero fill, each of its slices had cost a whole
// memory latency (about 1.7 us).  Not where the matrix is smaller than a tile, nor where the
// shift would break the 16-byte chunks of an M- or N-contiguous operand or the 4-column
// stores.  dS^T (ATILE) holds whole 32-row tiles past M.
template <bool ATILE>
__device__ __forceinline__ int edge_rows(const GemmDev& g) { return ATILE ? (g.M + 31) & ~31 : g.M; }
template <int BM, int BN, bool AK, bool BKM, bool ATILE>
__device__ __forceinline__ void shift_edge(const GemmDev& g, int& m0, int& n0) {
  const int mtop = edge_rows<ATILE>(g);
  if (mtop >= BM && (AK || mtop % 8 == 0)) m0 = min(m0, mtop - BM);
  if (g.N >= BN && g.N % (BKM ? 4 : 8) == 0) n0 = min(n0, g.N - BN);
}

// ---- the kernel --------------------------------------------------------------------------
// (SHIFT: the launch has tiles that the matrix edge cuts.  Whole-tile launches of the
// matrix-core-bound products go without: the compare in their epilogues and the moved tile
// origin cost the dS^T products and the NT kernel 1.5-2.5% at 16384 tokens.)
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, typename TC, int BK, int NST,
          bool ATILE = false, bool SHIFT = true>
__device__ __forceinline__ void gemm_tile(const GemmDev& g, int wg, int split) {
  constexpr int NTHR = 64 * WM * WN;
  constexpr int TM = BM / WM / 32;  // 32x32 MFMA tiles per wave along M
  constexpr int TN = BN / WN / 32;
  constexpr int KK = BK / 16;       // MFMA k-steps per slice
  using LA = Loader<AK, BM, NTHR, BK, ATILE>;
  using LB = Loader<BKM, BN, NTHR, BK>;
  constexpr int STAGE = LA::ELEMS + LB::ELEMS;
  constexpr int D = LA::Dma::PER + LB::Dma::PER;  // copies per wavefront per slice
  static_assert(NST >= 2 && NST <= 4 && (NST - 2) * D < 64, "stages / counter range");
  __shared__ __attribute__((aligned(1024))) bf16_t lds[NST * STAGE];

  const int ntm = (g.M + BM - 1) / BM, ntn = (g.N + BN - 1) / BN;
  const int ntiles = ntm * ntn;
  int tm, tn;
  const bf16_t* gA = g.A;
  const bf16_t* gB = g.B;
  TC* C = (TC*)g.C;
  if (g.causal) {
    // the longest K ranges first (row tile by row tile); inside one row tile, batch entries
    // that share their B panel (bdiv consecutive entries) are dispatched to one XCD
    // (workgroup ids go round-robin over the 8 XCDs) so that they stream it through one L2
    const int pid = wg;
    const int per = g.nbatch * ntn;
    tm = g.rev ? pid / per : ntm - 1 - pid / per;
    const int r = pid % per;
    tn = r / g.nbatch;
    int z = r % g.nbatch;
    if (g.bdiv > 1 && g.nbatch % (8 * g.bdiv) == 0) {
      const int x = z % 8, j = z / 8;
      z = (x + 8 * (j / g.bdiv)) * g.bdiv + j % g.bdiv;
    }
    const int z1 = z / g.zdiv, z2 = z % g.zdiv;
    gA += z * g.sA;
    gB += z1 * g.sB1 + (z2 / g.bdiv) * g.sB2;
    C += z1 * g.sC1 + z2 * g.sC2;
  } else {
    // XCD-aware remap, then group 8 row panels together for L2 reuse
    const int pid = xcd_remap(wg, ntiles);
    const int GROUP = 8;
    const int group = pid / (GROUP * ntn);
    const int first = group * GROUP;
    const int gsz = min(ntm - first, GROUP);
    tm = first + (pid % (GROUP * ntn)) % gsz;
    tn = (pid % (GROUP * ntn)) / gsz;
  }
  const int mlo = tm * BM, nlo = tn * BN;  // first row and column this tile stores
  int m0 = mlo, n0 = nlo;
  if constexpr (SHIFT) shift_edge<BM, BN, AK, BKM, ATILE>(g, m0, n0);
  int kbeg, kend;
  if (g.causal) {
    kbeg = g.rev ? mlo : 0;
    kend = g.rev ? g.ktotal : min(g.ktotal, mlo + BM);
  } else {
    kbeg = split * g.kchunk;
    kend = min(g.ktotal, kbeg + g.kchunk);
  }

  const int lane = threadIdx.x & 63, wave = wave_id();
  const int wm = wave / WN, wn = wave % WN;
  const int wrow0 = wm * (BM / WM), wcol0 = wn * (BN / WN);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  LA la;
  LB lb;
  typename LA::Dma da;
  typename LB::Dma db;
  da.init();
  db.init();
  LA::swizzle(da);
  LB::swizzle(db);
  const int nkg = (kend - kbeg + BK - 1) / BK;  // slices per operand group
  const int nk = nkg * (g.causal ? g.kgroups : 1);
  // slices copied straight to LDS (small tiles: also in a matrix smaller than the tile, with
  // clamped rows); a ragged last slice, and every slice of a tile whose operand rows are too far
  // apart for 32-bit offsets, goes through registers with zero fill.  So does every slice of
  // operands that are not 16-byte aligned, which the copies are not known to take: a product
  // of few tokens must not depend on how its caller's arrays lie.
  const int mvalid = edge_rows<ATILE>(g) - m0, nvalid = g.N - n0;
  constexpr bool EDGE = BM <= 128 && !ATILE;  // (larger tiles are not used below their size)
  const bool edge = mvalid < BM || nvalid < BN;  // uniform
  const bool dma_ok = (ATILE || g.aligned) && (EDGE || !edge) && (AK ? (int64_t)BM * g.lda : (int64_t)BK * g.lda) < (1ll << 30) &&
                      (BKM ? (int64_t)BN * g.ldb : (int64_t)BK * g.ldb) < (1ll << 30);
  const int nfull = dma_ok ? (kend - kbeg) / BK : 0;
  // rev: slices are walked from the top of the K range down, so that all row tiles of a
  // batch entry (whose ranges share their top) stream the same B rows at the same time
  auto stage = [&](int kt, bf16_t* dst) {
    const int grp = g.causal && g.kgroups > 1 ? kt / nkg : 0, ks0 = kt - grp * nkg;
    const int ks = g.causal && g.rev ? nkg - 1 - ks0 : ks0;
    const int k0 = kbeg + ks * BK;
    const bf16_t* pa = gA + grp * g.sAk;
    const bf16_t* pb = gB + grp * g.sBk;
    if (ks < nfull && !(EDGE && edge)) {
      la.dma(da, pa, g.lda, m0, mvalid, k0, dst);
      lb.dma(db, pb, g.ldb, n0, nvalid, k0, dst + LA::ELEMS);
    } else if (EDGE && ks < nfull) {
      if constexpr (EDGE) {
        la.dma_edge(da, pa, g.lda, m0, mvalid, k0, dst);
        lb.dma_edge(db, pb, g.ldb, n0, nvalid, k0, dst + LA::ELEMS);
      }
    } else {
      la.load(pa, g.lda, m0, mvalid, k0, kend);
      lb.load(pb, g.ldb, n0, nvalid, k0, kend);
      la.store(dst);
      lb.store(dst + LA::ELEMS);
    }
  };
  // slice s waits for its own copies while up to n later slices may still be in flight
  auto wait_slice = [&](int n) {
    if constexpr (NST >= 4) {
      if (n >= 2) { wait_vm<2 * D>(); return; }
    }
    if constexpr (NST >= 3) {
      if (n >= 1) { wait_vm<D>(); return; }
    }
    wait_vm<0>();
  };
  // fragments of one 16-wide k step, double buffered in registers: the reads of step
  // kk + 1 are issued before the matrix ops of step kk
  bf16x8 af[2][TM], bfr[2][TN];
  auto load_frags = [&](const bf16_t* As, int kk, bf16x8* a, bf16x8* b) {
    const bf16_t* Bs = As + LA::ELEMS;
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = LA::frag(As, wrow0 + i * 32, kk);
#pragma unroll
    for (int j = 0; j < TN; ++j) b[j] = LB::frag(Bs, wcol0 + j * 32, kk);
  };
  auto mma = [&](const bf16x8* a, const bf16x8* b) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  };
  // ring of NST slices: slices kt + 1 .. kt + NST - 1 are in flight while slice kt feeds the
  // matrix cores
#pragma unroll
  for (int s0 = 0; s0 < NST - 1; ++s0)
    if (s0 < nk) stage(s0, lds + s0 * STAGE);
  wait_slice(min(NST - 2, nk - 1));
  lds_barrier();
  if (nk > 0) load_frags(lds, 0, af[0], bfr[0]);
  for (int kt = 0; kt < nk; ++kt) {
    const bf16_t* As = lds + (kt % NST) * STAGE;
    // the stage of slice kt - 1 is free: every wave passed the barrier after its last read
    if (kt + NST - 1 < nk) stage(kt + NST - 1, lds + ((kt + NST - 1) % NST) * STAGE);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk + 1 < KK) {
        load_frags(As, kk + 1, af[(kk + 1) & 1], bfr[(kk + 1) & 1]);
      } else {
        // next slice: its copies must have landed (later ones may still fly) and every
        // wave must be done reading this one
        wait_slice(min(NST - 2, nk - 2 - kt));
        lds_barrier();
        if (kt + 1 < nk) load_frags(lds + ((kt + 1) % NST) * STAGE, 0, af[0], bfr[0]);
      }
      __builtin_amdgcn_sched_barrier(0);
      mma(af[kk & 1], bfr[kk & 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // epilogue: each wavefront stages one 32-row strip of its tile at a time in a private
  // LDS region (the main loop's last barrier has retired every operand read) and writes
  // it back row by row, 4 consecutive columns per lane.  In the MFMA result a lane holds
  // column lane % 32 and rows 8 (e / 4) + 4 (lane / 32) + e % 4 of each 32 x 32 block.
  constexpr int WTN = BN / WN;              // columns of the wave tile
  constexpr int SLD = WTN + 8;              // strip row stride (floats)
  static_assert(NTHR / 64 * 32 * SLD * 4 <= (int)sizeof(lds), "epilogue strip too large");
  float* strip = (float*)lds + wave * 32 * SLD;
  const bool vec = (g.ldc % 4) == 0;
  const bool lmode = g.lscale != nullptr;  // uniform
  const float lsc = lmode ? *g.lscale : 0.f;
  float sse = 0.f;
  // two copies, as in the persistent epilogue: with beta = 0 no C is read
  auto epilogue = [&](auto with_beta) {
    constexpr bool WB = decltype(with_beta)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          strip[((e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)) * SLD + j * 32 + (lane & 31)] =
              acc[i][j][e];
      constexpr int CPR = WTN / 4;            // float4 chunks per strip row
      constexpr int NIT = 32 * CPR / 64;
      // the strip's reads first (all inside the strip), then the stores
      f32x4 vv[NIT];
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int c = it * 64 + lane;
        vv[it] = *(const f32x4*)(strip + (c / CPR) * SLD + (c % CPR) * 4);
      }
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int c = it * 64 + lane;
        const int r = c / CPR, col = (c % CPR) * 4;
        const int m = m0 + wrow0 + i * 32 + r, n = n0 + wcol0 + col;
        if (m >= g.mstore || n >= g.N || (SHIFT && (m < mlo || n < nlo))) continue;
        f32x4 v = vv[it];
        if (lmode) {
          if (n + 4 > g.N) v = f32x4{v[0], n + 1 < g.N ? v[1] : 0.f, n + 2 < g.N ? v[2] : 0.f, 0.f};
          if (g.lmask && !g.lmask[m]) v = f32x4{0.f, 0.f, 0.f, 0.f};
          f32x4 r = v;
          if (g.lref) {
            const bf16_t* rp = g.lref + (int64_t)m * g.ldref + n;
            if (n + 4 <= g.N && (g.ldref & 3) == 0) {
              const u32x2 w = *(const u32x2*)rp;
              r = f32x4{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u),
                        __uint_as_float(w[1] << 16), __uint_as_float(w[1] & 0xffff0000u)};
            } else {
              r = f32x4{bf2f(rp[0]), n + 1 < g.N ? bf2f(rp[1]) : 0.f,
                        n + 2 < g.N ? bf2f(rp[2]) : 0.f, n + 3 < g.N ? bf2f(rp[3]) : 0.f};
            }
          }
          sse += v[0] * r[0] + v[1] * r[1] + v[2] * r[2] + v[3] * r[3];
          if (C == nullptr) continue;  // tile sums only
          v *= lsc;
        }
        if (g.part) {
          float* p = g.part + ((int64_t)split * g.M + m) * g.N + n;
          if (n + 4 <= g.N && (g.N % 4) == 0) {
            *(f32x4*)p = v;
          } else {
            for (int q = 0; q < 4 && n + q < g.N; ++q) p[q] = v[q];
          }
          continue;
        }
        TC* p = C + (int64_t)m * g.ldc + n;
        if (vec && n + 4 <= g.N) {
          store4<TC>(p, v, g.alpha, WB ? g.beta : 0.f);
        } else {
          for (int q = 0; q < 4 && n + q < g.N; ++q) {
            float x = g.alpha * v[q];
            if (WB && g.beta != 0.f) x += g.beta * ld(p + q);
            store_out<TC>(p + q, x);
          }
        }
      }
    }
  };
  // (the dS^T products never accumulate into C: beta = 0 is checked at their launch)
  if constexpr (ATILE) epilogue(std::false_type{});
  else if (g.beta != 0.f) epilogue(std::true_type{}); else epilogue(std::false_type{});
  if (g.lpart != nullptr) {  // uniform
    // the tile's sum in a fixed order: lanes (fixed tree), then wavefronts in order
    // (the last bytes of the operand LDS, past every wavefront's strip)
    static_assert(NTHR / 64 * 32 * SLD * 4 + 8 * (NTHR / 64) <= (int)sizeof(lds), "LDS");
    double* lred = (double*)((char*)lds + sizeof(lds)) - NTHR / 64;
    const double ws = warp_sum_d((double)sse);
    if (lane == 0) lred[wave] = ws;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int w = 0; w < NTHR / 64; ++w) t += lred[w];
      g.lpart[wg] = t;
    }
  }
}


// Persistent variant (no loss epilogue): a grid of one workgroup per CU slot walks the
// output tiles (x split-K chunks, or x batch entries of the causal products) in steps of the
// grid size, in the same tile order as the one-tile-per-workgroup launch.  The ring of two
// LDS stages runs on across tiles: the next tile's first slice is copied into the free
// stage while the last slice of this tile feeds the matrix cores, and while the epilogue
// stages its 16-row half strips in the stage the last slice occupied.  The causal tiles come
// longest K range first, and a workgroup takes them in snake order (forward in even rounds,
// backward in odd ones), so that long and short ranges pair up on every CU.
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, typename TC, int BK, int NST,
          bool CAUSAL, bool SHIFT = true>
__device__ __forceinline__ void gemm_persist(const GemmDev& g) {
  // the causal products read a 32 x 32-tiled A (tile32_off)
  constexpr bool ATILE = CAUSAL;
  static_assert(NST == 2, "the cross-tile copy assumes a two-stage ring");
  constexpr int NTHR = 64 * WM * WN;
  constexpr int TM = BM / WM / 32;
  constexpr int TN = BN / WN / 32;
  constexpr int KK = BK / 16;
  using LA = Loader<AK, BM, NTHR, BK, ATILE>;
  using LB = Loader<BKM, BN, NTHR, BK>;
  constexpr int STAGE = LA::ELEMS + LB::ELEMS;
  __shared__ __attribute__((aligned(1024))) bf16_t lds[NST * STAGE];

  const int ntm = (g.M + BM - 1) / BM, ntn = (g.N + BN - 1) / BN;
  const int ntiles = ntm * ntn;
  const int nitems = ntiles * (CAUSAL ? g.nbatch : g.nsplit);
  const int G = (int)gridDim.x;
  int round = 0;
  int w = blockIdx.x;
  if (w >= nitems) return;

  const int lane = threadIdx.x & 63, wave = wave_id();
  const int wm = wave / WN, wn = wave % WN;
  const int wrow0 = wm * (BM / WM), wcol0 = wn * (BN / WN);

  LA la;
  LB lb;
  typename LA::Dma da;
  typename LB::Dma db;
  da.init();
  db.init();
  LA::swizzle(da);
  LB::swizzle(db);

  // nkg: slices of one operand group (the causal products walk kgroups stacked operands)
  struct Item { int m0, n0, mlo, nlo, split, kbeg, kend, nk, nkg, nfull; int64_t aoff, boff, coff, coff_lo; };
  auto item = [&](int it) {
    Item t;
    int tm, tn;
    t.aoff = t.boff = t.coff = t.coff_lo = 0;
    if constexpr (CAUSAL) {
      // the one-tile launch's order: row tiles by K range, longest first; inside one, batch
      // entries that share their B panel on one XCD
      const int per = g.nbatch * ntn;
      tm = g.rev ? it / per : ntm - 1 - it / per;
      const int r = it % per;
      tn = r / g.nbatch;
      int z = r % g.nbatch;
      if (g.bdiv > 1 && g.nbatch % (8 * g.bdiv) == 0) {
        const int x = z % 8, j = z / 8;
        z = (x + 8 * (j / g.bdiv)) * g.bdiv + j % g.bdiv;
      }
      const int z1 = z / g.zdiv, z2 = z % g.zdiv;
      t.aoff = z * g.sA;
      t.boff = z1 * g.sB1 + (z2 / g.bdiv) * g.sB2;
      t.coff = z1 * g.sC1 + z2 * g.sC2;
      if constexpr (AK) t.coff_lo = z1 * g.sC1_lo + z2 * g.sC2_lo;
      t.split = 0;
    } else {
      const int x = it % ntiles;
      t.split = it / ntiles;
      const int pid = xcd_remap(x, ntiles);
      const int GROUP = 8;
      const int group = pid / (GROUP * ntn);
      const int first = group * GROUP;
      const int gsz = min(ntm - first, GROUP);
      tm = first + (pid % (GROUP * ntn)) % gsz;
      tn = (pid % (GROUP * ntn)) / gsz;
    }
    t.m0 = tm * BM;
    t.n0 = tn * BN;
    if constexpr (CAUSAL) {
      t.kbeg = g.rev ? t.m0 : 0;
      t.kend = g.rev ? g.ktotal : min(g.ktotal, t.m0 + BM);
      t.nkg = (t.kend - t.kbeg + BK - 1) / BK;
      t.nk = t.nkg * g.kgroups;
    } else {
      t.kbeg = t.split * g.kchunk;
      t.kend = min(g.ktotal, t.kbeg + g.kchunk);
      t.nk = t.nkg = (t.kend - t.kbeg + BK - 1) / BK;
    }
    // a last tile cut by the edge starts early enough to be whole, and stores only its own
    // rows and columns (the K range of a causal row tile is that of its own rows, set above)
    t.mlo = t.m0;
    t.nlo = t.n0;
    if constexpr (SHIFT) shift_edge<BM, BN, AK, BKM, ATILE>(g, t.m0, t.n0);
    const bool dma_ok = edge_rows<ATILE>(g) - t.m0 >= BM && g.N - t.n0 >= BN &&
                        (AK ? (int64_t)BM * g.lda : (int64_t)BK * g.lda) < (1ll << 30) &&
                        (BKM ? (int64_t)BN * g.ldb : (int64_t)BK * g.ldb) < (1ll << 30);
    t.nfull = dma_ok ? (t.kend - t.kbeg) / BK : 0;
    // uniform by construction: keep every field in scalar registers
    t.m0 = __builtin_amdgcn_readfirstlane(t.m0);
    t.n0 = __builtin_amdgcn_readfirstlane(t.n0);
    t.split = __builtin_amdgcn_readfirstlane(t.split);
    t.kbeg = __builtin_amdgcn_readfirstlane(t.kbeg);
    t.kend = __builtin_amdgcn_readfirstlane(t.kend);
    t.nk = __builtin_amdgcn_readfirstlane(t.nk);
    t.nkg = __builtin_amdgcn_readfirstlane(t.nkg);
    t.nfull = __builtin_amdgcn_readfirstlane(t.nfull);
    t.mlo = __builtin_amdgcn_readfirstlane(t.mlo);
    t.nlo = __builtin_amdgcn_readfirstlane(t.nlo);
    return t;
  };
  // slice kt of a tile: operand group kt / nkg, walked from the top of its K range down
  // with rev (so that all row tiles of a batch entry stream the same B rows together)
  auto stage = [&](const Item& t, int kt, bf16_t* dst) {
    const bf16_t* pa = g.A + t.aoff;
    const bf16_t* pb = g.B + t.boff;
    int ks = kt;
    if constexpr (CAUSAL) {
      const int grp = g.kgroups > 1 ? kt / t.nkg : 0, ks0 = kt - grp * t.nkg;
      ks = g.rev ? t.nkg - 1 - ks0 : ks0;
      pa += grp * g.sAk;
      pb += grp * g.sBk;
    }
    const int k0 = t.kbeg + ks * BK;
    if (ks < t.nfull) {
      la.dma(da, pa, g.lda, t.m0, g.M - t.m0, k0, dst);
      lb.dma(db, pb, g.ldb, t.n0, g.N - t.n0, k0, dst + LA::ELEMS);
    } else {
      la.load(pa, g.lda, t.m0, g.M - t.m0, k0, t.kend);
      lb.load(pb, g.ldb, t.n0, g.N - t.n0, k0, t.kend);
      la.store(dst);
      lb.store(dst + LA::ELEMS);
    }
  };
  bf16x8 af[2][TM], bfr[2][TN];
  auto load_frags = [&](const bf16_t* As, int kk, bf16x8* a, bf16x8* b) {
    const bf16_t* Bs = As + LA::ELEMS;
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = LA::frag(As, wrow0 + i * 32, kk);
#pragma unroll
    for (int j = 0; j < TN; ++j) b[j] = LB::frag(Bs, wcol0 + j * 32, kk);
  };
  f32x16 acc[TM][TN];
  auto mma = [&](const bf16x8* a, const bf16x8* b) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  };

  constexpr int WTN = BN / WN;
  constexpr int SLD = WTN + 8;
  static_assert(NTHR / 64 * 16 * SLD * 4 <= STAGE * 2, "epilogue half strip too large");
  const bool vec = (g.ldc % 4) == 0;
  TC* C = (TC*)g.C;

  Item cur = item(w);
  int rb = 0;          // stage of the current tile's first slice
  bool issued = false; // the current tile's first slice is already in flight
  for (;;) {
    const int wnext = CAUSAL ? (round + 1) * G + ((round & 1) ? (int)blockIdx.x : G - 1 - (int)blockIdx.x)
                             : w + G;
    const bool has_next = wnext < nitems;
    Item nxt{};
    if (has_next) nxt = item(wnext);
    if (!issued) {
      lds_barrier();  // every wavefront is past its previous epilogue
      if (cur.nk > 0) stage(cur, 0, lds + rb * STAGE);
    }
    bool pre = false;  // the next tile's first slice was issued during this tile
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // the first slice (and the previous epilogue's stores) complete; every wavefront is done
    // with the previous epilogue's strips before the other stage is refilled
    wait_vm<0>();
    lds_barrier();
    if (cur.nk > 0) load_frags(lds + rb * STAGE, 0, af[0], bfr[0]);
    for (int kt = 0; kt < cur.nk; ++kt) {
      const bf16_t* As = lds + ((rb + kt) & 1) * STAGE;
      bf16_t* other = lds + ((rb + kt + 1) & 1) * STAGE;
      const bool last = kt + 1 == cur.nk;
      // the other stage is free: every wave passed the barrier after its last read
      if (!last) {
        stage(cur, kt + 1, other);
      } else if (has_next && nxt.nk > 0) {
        stage(nxt, 0, other);
        pre = true;
      }
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        if (kk + 1 < KK) {
          load_frags(As, kk + 1, af[(kk + 1) & 1], bfr[(kk + 1) & 1]);
        } else if (!last) {
          wait_vm<0>();
          lds_barrier();
          load_frags(other, 0, af[0], bfr[0]);
        } else {
          // every wave is done reading this stage (the epilogue reuses it); the next
          // tile's copies stay in flight
          lds_barrier();
        }
        __builtin_amdgcn_sched_barrier(0);
        mma(af[kk & 1], bfr[kk & 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }

    // epilogue in the stage of the last slice, 16 rows of a wavefront's strip at a time
    const int es = cur.nk > 0 ? (rb + cur.nk - 1) & 1 : rb;
    // the lane index made opaque here, so that the epilogue's per-lane addresses are formed
    // per tile instead of being hoisted out of the tile loop (and held through the main loop)
    int el = lane;
    asm volatile("" : "+v"(el));
    float* strip = (float*)(lds + es * STAGE) + wave * 16 * SLD;
    // two copies: with beta = 0 the epilogue reads no C, so the compiler has no loads to
    // wait for before each store (a wait that would also cover the next tile's copy and
    // every earlier store)
    auto epilogue = [&](auto with_beta) {
      constexpr bool WB = decltype(with_beta)::value;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 8 * h; e < 8 * h + 8; ++e)
              strip[(((e >> 2) & 1) * 8 + (el >> 5) * 4 + (e & 3)) * SLD + j * 32 + (el & 31)] =
                  acc[i][j][e];
          constexpr int CPR = WTN / 4;
          constexpr int NIT = 16 * CPR / 64;
          // the strip's reads first (all inside the strip), then the stores: the reads go
          // out together instead of one wait per store (not for the causal products, where
          // reading as it stores measured faster)
          constexpr bool BATCH = !CAUSAL;
          f32x4 vv[BATCH ? NIT : 1];
          if constexpr (BATCH) {
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
              const int c = it * 64 + el;
              vv[it] = *(const f32x4*)(strip + (c / CPR) * SLD + (c % CPR) * 4);
            }
          }
#pragma unroll
          for (int it = 0; it < NIT; ++it) {
            const int c = it * 64 + el;
            const int r = c / CPR, col = (c % CPR) * 4;
            const int m = cur.m0 + wrow0 + i * 32 + 16 * h + r, n = cur.n0 + wcol0 + col;
            if (m >= g.mstore || n >= g.N || (SHIFT && (m < cur.mlo || n < cur.nlo))) continue;
            f32x4 v;
            if constexpr (BATCH) v = vv[it];
            else v = *(const f32x4*)(strip + r * SLD + col);
            if (g.part) {
              float* p = g.part + ((int64_t)cur.split * g.M + m) * g.N + n;
              if (n + 4 <= g.N && (g.N % 4) == 0) {
                *(f32x4*)p = v;
              } else {
                for (int q = 0; q < 4 && n + q < g.N; ++q) p[q] = v[q];
              }
              continue;
            }
            if constexpr (CAUSAL && AK) {
              if (g.split_n > 0) {  // uniform; whole 4-column groups (split_n % 4 == 0)
                if (n < g.split_n) {
                  const f32x4 o = v * g.alpha;
                  *(u32x2*)(g.c_lo + cur.coff_lo + (int64_t)m * g.ldc_lo + n) =
                      u32x2{pack2bf(o[0], o[1]), pack2bf(o[2], o[3])};
                } else {
                  *(f32x4*)((float*)g.C + cur.coff + (int64_t)m * g.ldc + (n - g.split_n)) = v * g.alpha;
                }
                continue;
              }
            }
            TC* p = C + cur.coff + (int64_t)m * g.ldc + n;
            if (vec && n + 4 <= g.N) {
              store4<TC>(p, v, g.alpha, WB ? g.beta : 0.f);
            } else {
              for (int q = 0; q < 4 && n + q < g.N; ++q) {
                float x = g.alpha * v[q];
                if (WB && g.beta != 0.f) x += g.beta * ld(p + q);
                store_out<TC>(p + q, x);
              }
            }
          }
        }
      }
    };
    // (the causal products never accumulate into C: beta = 0 is checked at their launch)
    if constexpr (CAUSAL) epilogue(std::false_type{});
    else if (g.beta != 0.f) epilogue(std::true_type{}); else epilogue(std::false_type{});
    if (!has_next) break;
    rb = (rb + cur.nk) & 1;
    issued = pre;
    cur = nxt;
    w = wnext;
    ++round;
  }
}

template <int BM, int BN, int WM, int WN, bool AK, bool BKM, typename TC, int BK, int NST>
__global__ __launch_bounds__(64 * WM * WN) void gemm_mfma_persist_kernel(GemmDev g) {
  gemm_persist<BM, BN, WM, WN, AK, BKM, TC, BK, NST, false>(g);
}
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, typename TC, int BK, int NST, bool SHIFT>
__global__ __launch_bounds__(64 * WM * WN) void attn_ds_gemm_persist_kernel(GemmDev g) {
  gemm_persist<BM, BN, WM, WN, AK, BKM, TC, BK, NST, true, SHIFT>(g);
}
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, typename TC, int BK, int NST>
__global__ __launch_bounds__(64 * WM * WN) void gemm_mfma_kernel(GemmDev g) {
  gemm_tile<BM, BN, WM, WN, AK, BKM, TC, BK, NST>(g, blockIdx.x, blockIdx.y);
}
// Several products of one layout in one launch: workgroup ids run over the (split, tile) pairs
// of the first product, then of the second, ..
constexpr int GROUP_MAX = 5;
struct GroupDev {
  int n;
  int end[GROUP_MAX];    // workgroups of products 0 .. i
  int tiles[GROUP_MAX];  // tiles of product i
  GemmDev p[GROUP_MAX];
};
template <int BM, int BN, int NST, bool AK, bool BKM, typename TC>
__global__ __launch_bounds__(256) void gemm_group_kernel(GroupDev gr) {
  const int w = blockIdx.x;
  int i = 0, beg = 0;
#pragma unroll
  for (int j = 0; j < GROUP_MAX - 1; ++j)
    if (j + 1 < gr.n && w >= gr.end[j]) {
      i = j + 1;
      beg = gr.end[j];
    }
  const int tiles = gr.tiles[i];
  gemm_tile<BM, BN, 2, 2, AK, BKM, TC, 64, NST>(gr.p[i], (w - beg) % tiles, (w - beg) / tiles);
}
// the same tile program for the dS products of attention's backward, on the 32 x 32-tiled
// dS^T (own name, so that profiles tell them apart)
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, typename TC, int BK, int NST, bool SHIFT>
__global__ __launch_bounds__(64 * WM * WN) void attn_ds_gemm_kernel(GemmDev g) {
  gemm_tile<BM, BN, WM, WN, AK, BKM, TC, BK, NST, true, SHIFT>(g, blockIdx.x, blockIdx.y);
}

// ---- NT products on four wavefronts, k-steps scheduled by hand ------------------------
//
// Both operands K-contiguous, M >= 256, N at least the tile width (256 or 192), K a
// multiple of 128.  A workgroup of four wavefronts (one per SIMD) owns a 256 x 256 tile,
// 128 x 128 per wavefront (16 accumulators of 32 x 32 in AGPRs; 256 x 192 tiles: 128 x 96,
// 12 accumulators); per 16-wide k step each wavefront reads 8 KB of operands from LDS,
// a third fewer LDS bytes per MFMA than the 8-wavefront tiles.  With one wavefront per SIMD no other wavefront hides its waits, so
// each k step is one block of inline assembly in a fixed order: the 16 MFMAs of the step,
// one operand read for the step after next between every other pair of them (operands
// are read two k steps ahead into four register buffers), and on the two steps after
// each slice barrier the 8 LDS DMA copies of the next-but-one slice between the others.
// The compiler does not see the assembly's LDS and memory operations: every block starts
// with the wait for the reads of the step before last (at most 8 reads are younger), and
// each slice barrier waits for all copies.  A persistent grid walks the tiles; the next
// tile's first two slices are copied, and its first two k steps read, while the current
// tile finishes, and the epilogue stages 8-row strips in a 17 KB LDS region of its own.
// Measured on the 16384 x 4096 x 4096 product: 475 us against 532 us for the 8-wavefront
// tile, the matrix cores 81% busy instead of 62%.  (The other operand layouts read one
// operand with the transposing LDS read, 8 bytes of a fragment per instruction; inline
// assembly cannot name the halves of a 128-bit operand, so they stay compiler-scheduled.)
#define NT4_MF(c, a, b) "v_mfma_f32_32x32x16_bf16 %[" #c "], %[" #a "], %[" #b "], %[" #c "]\n"
#define NT4_RD(d, base, off) "ds_read_b128 %[" #d "], %[" #base "] offset:" #off "\n"
#define NT4_CP(o, src, m, off) \
  "s_add_u32 m0, %[" #m "], " #off "\ns_nop 0\nglobal_load_lds_dwordx4 %[" #o "], %[" #src "]\n"
// the 16 MFMAs of one k step with the 8 operand reads of the step after next after
// MFMAs 0, 2, .., 14 (read order = first use: A0, B0..B3, A1..A3)
#define NT4_STEP_BODY(X0, X1, X2, X3, X4, X5, X6, X7)                                       \
  "s_waitcnt lgkmcnt(8)\n"                                                                \
  NT4_MF(c00, a0, b0) NT4_RD(nA0, ra, 0) NT4_MF(c01, a0, b1) X0                             \
  NT4_MF(c02, a0, b2) NT4_RD(nB0, rb, 0) NT4_MF(c03, a0, b3) X1                             \
  NT4_MF(c10, a1, b0) NT4_RD(nB1, rb, 4096) NT4_MF(c11, a1, b1) X2                          \
  NT4_MF(c12, a1, b2) NT4_RD(nB2, rb, 8192) NT4_MF(c13, a1, b3) X3                          \
  NT4_MF(c20, a2, b0) NT4_RD(nB3, rb, 12288) NT4_MF(c21, a2, b1) X4                         \
  NT4_MF(c22, a2, b2) NT4_RD(nA1, ra, 4096) NT4_MF(c23, a2, b3) X5                          \
  NT4_MF(c30, a3, b0) NT4_RD(nA2, ra, 8192) NT4_MF(c31, a3, b1) X6                          \
  NT4_MF(c32, a3, b2) NT4_RD(nA3, ra, 12288) NT4_MF(c33, a3, b3) X7
#define NT4_OUTS                                                                            \
  [c00] "+a"(acc[0][0]), [c01] "+a"(acc[0][1]), [c02] "+a"(acc[0][2]), [c03] "+a"(acc[0][3]), \
  [c10] "+a"(acc[1][0]), [c11] "+a"(acc[1][1]), [c12] "+a"(acc[1][2]), [c13] "+a"(acc[1][3]), \
  [c20] "+a"(acc[2][0]), [c21] "+a"(acc[2][1]), [c22] "+a"(acc[2][2]), [c23] "+a"(acc[2][3]), \
  [c30] "+a"(acc[3][0]), [c31] "+a"(acc[3][1]), [c32] "+a"(acc[3][2]), [c33] "+a"(acc[3][3]), \
  [nA0] "=&v"(nx[0]), [nA1] "=&v"(nx[1]), [nA2] "=&v"(nx[2]), [nA3] "=&v"(nx[3]),          \
  [nB0] "=&v"(nx[4]), [nB1] "=&v"(nx[5]), [nB2] "=&v"(nx[6]), [nB3] "=&v"(nx[7])
#define NT4_INS                                                                             \
  [a0] "v"(cu[0]), [a1] "v"(cu[1]), [a2] "v"(cu[2]), [a3] "v"(cu[3]), [b0] "v"(cu[4]),      \
  [b1] "v"(cu[5]), [b2] "v"(cu[6]), [b3] "v"(cu[7]), [ra] "v"(ra), [rb] "v"(rb)
// the same for 256 x 192 tiles (128 x 96 per wavefront): 12 MFMAs, 7 reads (A0, B0..B2,
// A1..A3), up to 7 copies
#define NT4_STEP_BODY3(X0, X1, X2, X3, X4, X5, X6)                                          \
  "s_waitcnt lgkmcnt(7)\n"                                                                \
  NT4_MF(c00, a0, b0) NT4_RD(nA0, ra, 0) NT4_MF(c01, a0, b1) X0                             \
  NT4_MF(c02, a0, b2) NT4_RD(nB0, rb, 0) NT4_MF(c10, a1, b0) X1                             \
  NT4_MF(c11, a1, b1) NT4_RD(nB1, rb, 4096) NT4_MF(c12, a1, b2) X2                          \
  NT4_MF(c20, a2, b0) NT4_RD(nB2, rb, 8192) NT4_MF(c21, a2, b1) X3                          \
  NT4_MF(c22, a2, b2) NT4_RD(nA1, ra, 4096) NT4_MF(c30, a3, b0) X4                          \
  NT4_MF(c31, a3, b1) NT4_RD(nA2, ra, 8192) NT4_MF(c32, a3, b2) X5                          \
  NT4_RD(nA3, ra, 12288) X6
#define NT4_OUTS3                                                                           \
  [c00] "+a"(acc[0][0]), [c01] "+a"(acc[0][1]), [c02] "+a"(acc[0][2]), [c10] "+a"(acc[1][0]), \
  [c11] "+a"(acc[1][1]), [c12] "+a"(acc[1][2]), [c20] "+a"(acc[2][0]), [c21] "+a"(acc[2][1]), \
  [c22] "+a"(acc[2][2]), [c30] "+a"(acc[3][0]), [c31] "+a"(acc[3][1]), [c32] "+a"(acc[3][2]), \
  [nA0] "=&v"(nx[0]), [nA1] "=&v"(nx[1]), [nA2] "=&v"(nx[2]), [nA3] "=&v"(nx[3]),          \
  [nB0] "=&v"(nx[4]), [nB1] "=&v"(nx[5]), [nB2] "=&v"(nx[6])
#define NT4_INS3                                                                            \
  [a0] "v"(cu[0]), [a1] "v"(cu[1]), [a2] "v"(cu[2]), [a3] "v"(cu[3]), [b0] "v"(cu[4]),      \
  [b1] "v"(cu[5]), [b2] "v"(cu[6]), [ra] "v"(ra), [rb] "v"(rb)

// Several products of one A (the same rows, K and row strides): column tiles run over the
// outputs of the first product, then of the second, .. (g.N, g.B, g.C, g.ldc are not used)
struct Nt4Group {
  int n;
  int end[GROUP_MAX];  // column tiles of products 0 .. i
  int N[GROUP_MAX];
  const bf16_t* B[GROUP_MAX];
  void* C[GROUP_MAX];
  int64_t ldc[GROUP_MAX];
};

template <int BN, typename TC, bool SHIFT, bool GROUP>
__device__ __forceinline__ void gemm_nt4(const GemmDev& g, const Nt4Group& gr) {
  constexpr int BM = 256, BKK = 64, TM = 4, TN = BN / 64;  // 4 or 3 fragments of B
  constexpr int WTN = BN / 2;                              // columns per wavefront
  using LA = Loader<true, BM, 256, BKK>;  // operand tile layouts (swizzled rows)
  using LB = Loader<true, BN, 256, BKK>;
  constexpr int STAGE = LA::ELEMS + LB::ELEMS;  // elements: A [256][64], then B [BN][64]
  constexpr int SLD = WTN + 4;                  // epilogue strip row (floats)
  constexpr int EPI = 4 * 8 * SLD;              // floats: four wavefronts x 8 rows
  constexpr int PB = LB::Dma::PER;              // B copies per lane per slice: 8 or 6
  static_assert(BN == 256 || BN == 192, "tile widths");
  static_assert(LA::Dma::PER == 8 && PB == TN * 2, "copies per lane per operand slice");
  __shared__ __attribute__((aligned(1024))) bf16_t lds[2 * STAGE + 2 * EPI];
  const int ntm = (g.M + BM - 1) / BM, ntn = GROUP ? gr.end[gr.n - 1] : (g.N + BN - 1) / BN, ntiles = ntm * ntn;
  const int G = (int)gridDim.x;
  int w = blockIdx.x;
  if (w >= ntiles) return;
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int wrow0 = (wave >> 1) * 128, wcol0 = (wave & 1) * WTN;
  // the tile order of the one-tile launch: XCD-aware remap, 8 row panels per group
  // (a tile that the edge cuts starts at M - BM or N - BN instead and stores only the rows
  // and columns of its own)
  auto tile_of = [&](int x, int& m0, int& n0, int& mlo, int& nlo, int& pi) {
    const int pid = xcd_remap(x, ntiles);
    const int group = pid / (8 * ntn), first = group * 8, gsz = min(ntm - first, 8);
    mlo = __builtin_amdgcn_readfirstlane((first + (pid % (8 * ntn)) % gsz) * BM);
    int tn = __builtin_amdgcn_readfirstlane((pid % (8 * ntn)) / gsz);
    pi = 0;
    if constexpr (GROUP) {
      int beg = 0;
#pragma unroll
      for (int j = 0; j < GROUP_MAX - 1; ++j)
        if (j + 1 < gr.n && tn >= gr.end[j]) {
          pi = j + 1;
          beg = gr.end[j];
        }
      tn -= beg;
    }
    nlo = tn * BN;
    m0 = SHIFT ? min(mlo, g.M - BM) : mlo;
    n0 = SHIFT ? min(nlo, (GROUP ? gr.N[pi] : g.N) - BN) : nlo;
  };
  auto b_of = [&](int pi) { return GROUP ? gr.B[pi] : g.B; };
  typename LA::Dma da;
  typename LB::Dma db;
  da.init();
  db.init();
  LA::swizzle(da);
  LB::swizzle(db);
  // copy p of a slice: this lane's byte offset from the slice's first element (A, B) and
  // LDS block wave + 4 p of the operand tile
  uint32_t oA[8], oB[8];
#pragma unroll
  for (int p = 0; p < 8; ++p) oA[p] = 2u * (uint32_t)(da.row[p] * (int)g.lda + da.col[p]);
#pragma unroll
  for (int p = 0; p < PB; ++p) oB[p] = 2u * (uint32_t)(db.row[p] * (int)g.ldb + db.col[p]);
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;  // LDS byte address
  // operand read addresses of stage st, k step kk (fragment i / j at + 4096 i bytes)
  const int l = lane & 31, h = lane >> 5;
  uint32_t adA[2][4], adB[2][4];
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const uint32_t sw = 16u * (uint32_t)((2 * kk + h) ^ LA::swz(l));
      adA[st][kk] = lds0 + st * STAGE * 2 + (wrow0 + l) * BKK * 2 + sw;
      adB[st][kk] = lds0 + st * STAGE * 2 + LA::ELEMS * 2 + (wcol0 + l) * BKK * 2 +
                    16u * (uint32_t)((2 * kk + h) ^ LB::swz(l));
    }
  const int nk = g.ktotal / BKK;  // even
  int m0, n0, mlo, nlo, pi, nm0 = 0, nn0 = 0, nmlo = 0, nnlo = 0, npi = 0;
  tile_of(w, m0, n0, mlo, nlo, pi);
  const bf16_t* baseA = g.A + (int64_t)m0 * g.lda;
  const bf16_t* baseB = b_of(pi) + (int64_t)n0 * g.ldb;
  int wnext = w + G;
  bool has_next = wnext < ntiles;
  const bf16_t* nbaseA = baseA;
  const bf16_t* nbaseB = baseB;
  if (has_next) {
    tile_of(wnext, nm0, nn0, nmlo, nnlo, npi);
    nbaseA = g.A + (int64_t)nm0 * g.lda;
    nbaseB = b_of(npi) + (int64_t)nn0 * g.ldb;
  }
  f32x16 acc[TM][TN];
  bf16x8 F[4][8];  // operand buffers of four k steps: A 0..3, B 4..7
  // k step on buffer cur, reading step kk of stage st into buffer nxt
  auto step = [&](int cur, int nxt, int st, int kk) {
    const bf16x8* cu = F[cur];
    bf16x8* nx = F[nxt];
    const uint32_t ra = adA[st][kk], rb = adB[st][kk];
    if constexpr (TN == 4)
      asm volatile(NT4_STEP_BODY("", "", "", "", "", "", "", "") : NT4_OUTS : NT4_INS : "memory");
    else
      asm volatile(NT4_STEP_BODY3("", "", "", "", "", "", "") : NT4_OUTS3 : NT4_INS3 : "memory");
  };
  // the same with copies q (0: 0..3, 1: 4..7) of slice ks of this tile into stage ks % 2,
  // or of slice ks - nk of the next one (after the last tile: a repeat of this tile's last
  // slice into the stage nobody reads any more)
  auto step_copy = [&](int cur, int nxt, int st, int kk, int ks, int q) {
    const bf16x8* cu = F[cur];
    bf16x8* nx = F[nxt];
    const uint32_t ra = adA[st][kk], rb = adB[st][kk];
    const bool in_next = ks >= nk;
    const int kq = in_next ? (has_next ? ks - nk : nk - 1) : ks;
    const bf16_t* pa = (in_next && has_next ? nbaseA : baseA) + kq * BKK;
    const bf16_t* pb = (in_next && has_next ? nbaseB : baseB) + kq * BKK;
    // copies q of A: blocks wave + 4 p, p = 4 q .. 4 q + 3; of B: p = (PB / 2) q + u
    const uint32_t stg = lds0 + (ks & 1) * STAGE * 2 + wave * 1024;
    const uint32_t ma = (uint32_t)__builtin_amdgcn_readfirstlane((int)(stg + 16384 * q));
    const uint32_t mb = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(stg + LA::ELEMS * 2 + 4096 * (PB / 2) * q));
    const uint64_t sa = uniform_ptr(pa), sb = uniform_ptr(pb);
    const uint32_t oa0 = oA[4 * q], oa1 = oA[4 * q + 1], oa2 = oA[4 * q + 2], oa3 = oA[4 * q + 3];
    const int qb = (PB / 2) * q;
    const uint32_t ob0 = oB[qb], ob1 = oB[qb + 1], ob2 = oB[qb + 2], ob3 = oB[PB == 8 ? qb + 3 : qb];
    uint32_t m0v;  // m0 (the copies' LDS destination) is written early by the block
    if constexpr (TN == 4)
      asm volatile(NT4_STEP_BODY(NT4_CP(oa0, sa, ma, 0), NT4_CP(oa1, sa, ma, 4096),
                                 NT4_CP(oa2, sa, ma, 8192), NT4_CP(oa3, sa, ma, 12288),
                                 NT4_CP(ob0, sb, mb, 0), NT4_CP(ob1, sb, mb, 4096),
                                 NT4_CP(ob2, sb, mb, 8192), NT4_CP(ob3, sb, mb, 12288))
                   : NT4_OUTS, [m0v] "=&{m0}"(m0v)
                   : NT4_INS, [oa0] "v"(oa0), [oa1] "v"(oa1), [oa2] "v"(oa2), [oa3] "v"(oa3),
                     [ob0] "v"(ob0), [ob1] "v"(ob1), [ob2] "v"(ob2), [ob3] "v"(ob3), [sa] "s"(sa),
                     [sb] "s"(sb), [ma] "s"(ma), [mb] "s"(mb)
                   : "memory");
    else
      asm volatile(NT4_STEP_BODY3(NT4_CP(oa0, sa, ma, 0), NT4_CP(oa1, sa, ma, 4096),
                                  NT4_CP(oa2, sa, ma, 8192), NT4_CP(oa3, sa, ma, 12288),
                                  NT4_CP(ob0, sb, mb, 0), NT4_CP(ob1, sb, mb, 4096),
                                  NT4_CP(ob2, sb, mb, 8192))
                   : NT4_OUTS3, [m0v] "=&{m0}"(m0v)
                   : NT4_INS3, [oa0] "v"(oa0), [oa1] "v"(oa1), [oa2] "v"(oa2), [oa3] "v"(oa3),
                     [ob0] "v"(ob0), [ob1] "v"(ob1), [ob2] "v"(ob2), [sa] "s"(sa), [sb] "s"(sb),
                     [ma] "s"(ma), [mb] "s"(mb)
                   : "memory");
  };
  // prologue: slices 0 and 1 of the first tile, steps 0 and 1 read
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    bf16_t* dst = lds + kt * STAGE;
#pragma unroll
    for (int p = 0; p < 8; ++p) dma16_s(baseA + kt * BKK, oA[p], dst + (wave + p * 4) * 512);
#pragma unroll
    for (int p = 0; p < PB; ++p) dma16_s(baseB + kt * BKK, oB[p], dst + LA::ELEMS + (wave + p * 4) * 512);
  }
  wait_vm<8 + PB>();
  lds_barrier();
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
    for (int i = 0; i < 4; ++i) F[kk][i] = LA::frag(lds, wrow0 + i * 32, kk);
#pragma unroll
    for (int j = 0; j < TN; ++j) F[kk][4 + j] = LB::frag(lds + LA::ELEMS, wcol0 + j * 32, kk);
  }
  // every read of the compiler's own has landed: its counter bookkeeping starts empty
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  // row-masked scale of the result, through a scalar load: a vector load would leave the
  // compiler counting it as outstanding in the tile loop, where its waits would also wait
  // for the copies in flight
  float lsc = 0.f;
  if (g.lscale) {  // uniform
    const uint64_t pl = uniform_ptr(g.lscale);
    uint32_t u;
    asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(u) : "s"(pl) : "memory");
    lsc = __uint_as_float(u);
  }
  float* strip = (float*)(lds + 2 * STAGE) + wave * 8 * SLD;
  for (;;) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // two slices per pass: slice kt in stage 0, slice kt + 1 in stage 1
    for (int kt = 0; kt < nk; kt += 2) {
      step(0, 2, 0, 2);
      step(1, 3, 0, 3);
      wait_vm<0>();
      lds_barrier();  // slice kt + 1 has landed; nobody reads stage 0 any more
      step_copy(2, 0, 1, 0, kt + 2, 0);
      step_copy(3, 1, 1, 1, kt + 2, 1);
      step(0, 2, 1, 2);
      step(1, 3, 1, 3);
      wait_vm<0>();
      lds_barrier();  // slice kt + 2 (or the next tile's slice 0) has landed
      step_copy(2, 0, 0, 0, kt + 3, 0);
      step_copy(3, 1, 0, 1, kt + 3, 1);
    }
    // epilogue: rows 8 gq .. 8 gq + 7 of each 32-row block, staged in this wavefront's
    // region (a lane holds column l of rows 4 h .. 4 h + 3 of the group) and written back
    // 4 columns per lane.  Two copies: with beta = 0 (every product of the step) the
    // epilogue reads no C, so the compiler has no loads to wait for before each store (it
    // would otherwise wait for every memory operation in flight, the next tile's copies
    // included)
    TC* C = (TC*)(GROUP ? gr.C[pi] : g.C);
    const int64_t ldc = GROUP ? gr.ldc[pi] : g.ldc;
    // (beta and the masked scale are compile-time in each copy: with no branch inside, the
    // four strip reads of a row group are issued together, then converted and stored)
    auto epilogue = [&](auto with_beta, auto with_scale) {
      constexpr bool WB = decltype(with_beta)::value;
      constexpr bool LS = decltype(with_scale)::value;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        // the row mask of this 32-row block through scalar loads of whole dwords (the launcher
        // checks the mask's 4-byte alignment): a vector load here would wait, in order, for the
        // next tile's copies already in flight. The last row tile, moved back, starts at any
        // byte: the block's nine dwords are shifted down to it (each holds a byte of the block).
        // (dO of 6002 tokens, 4096 x 4096: 189 us; on 256-wide tiles of the kernel that lets
        // the compiler place the copies, 250 us)
        constexpr uint32_t ALL = 0x01010101u;  // (a byte per row; no mask: every row kept)
        u32x8 mk = {ALL, ALL, ALL, ALL, ALL, ALL, ALL, ALL};
        if (LS && g.lmask) {  // uniform
          const int r0 = m0 + wrow0 + i * 32, sh = SHIFT ? r0 & 3 : 0;
          const uint64_t pa = uniform_ptr(g.lmask + r0 - sh);
          asm volatile("s_load_dwordx8 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(mk) : "s"(pa) : "memory");
          if (SHIFT && __builtin_amdgcn_readfirstlane(sh) != 0) {
            uint32_t top;
            asm volatile("s_load_dword %0, %1, 0x20\n\ts_waitcnt lgkmcnt(0)" : "=s"(top) : "s"(pa) : "memory");
#pragma unroll
            for (int q = 0; q < 8; ++q)
              mk[q] = (uint32_t)(((uint64_t)(q < 7 ? mk[q + 1] : top) << 32 | mk[q]) >> (8 * sh));
          }
        }
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) strip[(4 * h + q) * SLD + j * 32 + l] = acc[i][j][4 * gq + q];
          f32x4 v[TN];
#pragma unroll
          for (int it = 0; it < TN; ++it) {
            const int c = it * 64 + lane;
            v[it] = *(const f32x4*)(strip + (c / (WTN / 4)) * SLD + (c % (WTN / 4)) * 4);
          }
#pragma unroll
          for (int it = 0; it < TN; ++it) {
            const int c = it * 64 + lane;
            const int r = c / (WTN / 4), col = (c % (WTN / 4)) * 4;
            const int m = m0 + wrow0 + i * 32 + 8 * gq + r, n = n0 + wcol0 + col;
            f32x4 o = v[it];
            if constexpr (LS) {  // row r of the block's 8-row group gq: byte 8 gq + r of mk
              const uint32_t dw = r >= 4 ? mk[2 * gq + 1] : mk[2 * gq];
              const bool keep = ((dw >> (8 * (r & 3))) & 0xffu) != 0u;
              const f32x4 so = o * lsc;  // masked rows exactly 0 (also where o is not finite)
              o = f32x4{keep ? so[0] : 0.f, keep ? so[1] : 0.f, keep ? so[2] : 0.f, keep ? so[3] : 0.f};
            }
            if (!SHIFT || (m >= mlo && n >= nlo)) store4<TC>(C + (int64_t)m * ldc + n, o, g.alpha, WB ? g.beta : 0.f);
          }
        }
      }
    };
    if constexpr (GROUP) {
      epilogue(std::false_type{}, std::false_type{});
    } else if (g.lscale) {  // the masked dO product (beta = 0)
      if (g.beta != 0.f) epilogue(std::true_type{}, std::true_type{});
      else epilogue(std::false_type{}, std::true_type{});
    } else {
      if (g.beta != 0.f) epilogue(std::true_type{}, std::false_type{});
      else epilogue(std::false_type{}, std::false_type{});
    }
    if (!has_next) break;
    w = wnext;
    m0 = nm0;
    n0 = nn0;
    mlo = nmlo;
    nlo = nnlo;
    pi = npi;
    baseA = nbaseA;
    baseB = nbaseB;
    wnext = w + G;
    has_next = wnext < ntiles;
    if (has_next) {
      tile_of(wnext, nm0, nn0, nmlo, nnlo, npi);
      nbaseA = g.A + (int64_t)nm0 * g.lda;
      nbaseB = b_of(npi) + (int64_t)nn0 * g.ldb;
    }
  }
}

template <int BN, typename TC, bool SHIFT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gemm_nt4_persist_kernel(GemmDev g) {
  gemm_nt4<BN, TC, SHIFT, false>(g, Nt4Group{});
}
template <int BN, typename TC, bool SHIFT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gemm_nt4_group_kernel(GemmDev g, Nt4Group gr) {
  gemm_nt4<BN, TC, SHIFT, true>(g, gr);
}

// C = alpha * sum_s part[s] + beta * C, summed in split order (split s of the M x N block at
// part + s * sstride)
template <typename TC>
__global__ void splitk_reduce_kernel(const float* __restrict__ part, int splits, int64_t sstride,
                                     int M, int N, TC* __restrict__ C, int64_t ldc, float alpha,
                                     float beta) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t total = (int64_t)M * N;
  if (idx >= total) return;
  int m = (int)(idx / N), n = (int)(idx % N);
  float s = 0.f;
  for (int z = 0; z < splits; ++z) s += part[(int64_t)z * sstride + idx];
  TC* c = C + (int64_t)m * ldc + n;
  float v = alpha * s;
  if (beta != 0.f) v += beta * ld(c);
  store_out<TC>(c, v);
}

// the same, four consecutive outputs per thread (N and ldc multiples of 4), for several sums
// in one launch
struct SumDev {
  const float* part;
  int64_t sstride, ldc, end;  // end: quadruples of sums 0 .. i
  void* C;
  int splits, N;
  float alpha, beta;
};
constexpr int SUM_MAX = GROUP_MAX + 1;
struct SumGroup {
  int n;
  SumDev s[SUM_MAX];
};
template <typename TC>
__global__ __launch_bounds__(256) void splitk_reduce4_kernel(SumGroup gr) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= gr.s[gr.n - 1].end) return;
  int i = 0;
  while (q >= gr.s[i].end) ++i;
  const SumDev& d = gr.s[i];
  const int64_t idx = 4 * (i ? q - gr.s[i - 1].end : q);
  const int64_t m = idx / d.N;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int z = 0; z < d.splits; ++z) acc += *(const f32x4*)(d.part + z * d.sstride + idx);
  store4<TC>((TC*)d.C + m * d.ldc + (idx - m * d.N), acc, d.alpha, d.beta);
}

// Tile shape and split-K factor.
enum TileKind {
  T256 = 0,     // 256 x 256, 8 wavefronts, persistent
  T256x192 = 1, // 256 x 192, 8 wavefronts, persistent
  T128 = 2,     // 128 x 128, 4 wavefronts, persistent, two per CU
  T192x256 = 3, // 192 x 256, 8 wavefronts, persistent (weight gradients)
  T64 = 4,      // 64 x 64, 4 wavefronts, one tile per workgroup, two per CU
  TNT256 = 5,   // gemm_nt4_persist_kernel<256>
  TNT192 = 6,   // gemm_nt4_persist_kernel<192>
  T_KINDS = 7
};
struct Plan {
  int kind;
  int bm, bn, splits, kchunk;
  double t = 0.0;  // modelled us
};

constexpr int NUM_CU = 256;

// Launch time model, in us: a round of workgroups on the chip's slots costs
// tile + slices * max(lat, bw * (workgroups in the round / 256 + 1/4, at most per_cu)), a
// launch `fixed` more.  lat is the time of a 64-deep slice that waits for its copies (few
// workgroups), bw the same per workgroup on a CU where the matrix cores, the caches and the
// power limit are shared by all (a half-full round runs at three quarters of that, not at a
// half: the clock does not rise so fast).  Fitted per layout and tile to 387 shapes of the
// step (64 to 16384 tokens, splits 1 to 32), each timed right behind some milliseconds of
// matrix work, as in a step: 6-9% rms.  The small tile keeps four slices in flight and
// costs 0.4 us per slice where the 256-wide tiles cost 1.2-1.5: it takes every product that
// would leave most CUs idle (666 x 2048 x 2048 NT: 21 us against 40 us on 256 x 192, 57 us
// before edge tiles were whole).  Over the shapes the choice is on average 1% above the best
// measured one.
struct TileCost {
  int bm, bn, per_cu;
  float fixed, tile, lat, bw;
};
constexpr TileCost TILE_COST[3][T_KINDS] = {
    // NT
    {{256, 256, 1, 3.3f, 9.0f, 1.50f, 1.81f}, {256, 192, 1, 3.8f, 6.0f, 1.24f, 1.46f},
     {128, 128, 2, 4.2f, 3.1f, 0.82f, 0.577f}, {0, 0, 0, 0, 0, 0, 0},
     {64, 64, 2, 3.2f, 1.6f, 0.38f, 0.316f}, {256, 256, 1, 5.3f, 6.8f, 1.20f, 1.63f},
     {256, 192, 1, 4.7f, 5.1f, 1.07f, 1.32f}},
    // NN
    {{256, 256, 1, 7.1f, 7.2f, 1.47f, 1.82f}, {256, 192, 1, 3.9f, 6.1f, 1.25f, 1.44f},
     {128, 128, 2, 6.5f, 1.4f, 0.92f, 0.610f}, {0, 0, 0, 0, 0, 0, 0},
     {64, 64, 2, 2.9f, 1.7f, 0.39f, 0.322f}, {0, 0, 0, 0, 0, 0, 0}, {0, 0, 0, 0, 0, 0, 0}},
    // TN
    {{256, 256, 1, 6.6f, 4.9f, 1.51f, 1.97f}, {256, 192, 1, 1.8f, 7.9f, 1.26f, 1.51f},
     {128, 128, 2, 0.9f, 6.7f, 0.94f, 0.605f}, {192, 256, 1, 2.4f, 7.1f, 1.27f, 1.56f},
     {64, 64, 2, 1.5f, 2.8f, 0.45f, 0.303f}, {0, 0, 0, 0, 0, 0, 0}, {0, 0, 0, 0, 0, 0, 0}}};
constexpr int MAX_SPLITS = 32;

// The four-wavefront NT kernel: both operands K-contiguous with 16-byte aligned rows, K a
// multiple of 128, at least one whole tile, rows within 32-bit offsets, 4-column stores.
bool nt4_ok(const Gemm& g, int bn) {
  return g.a_kmajor && g.b_kmajor && g.M >= 256 && g.N >= bn && g.N % 4 == 0 && g.K % 128 == 0 &&
         g.K >= 128 && g.lda % 8 == 0 && g.ldb % 8 == 0 && g.ldc % 4 == 0 &&
         (uintptr_t)g.A % 16 == 0 && (uintptr_t)g.B % 16 == 0 && (uintptr_t)g.C % 16 == 0 &&
         (int64_t)256 * g.lda * 2 < (1ll << 31) && (int64_t)256 * g.ldb * 2 < (1ll << 31);
}

// The cheapest tile kind of `kinds` (bit mask) and split factor; the partials of a split
// product (or of a two-output one, which always goes through them) fit scratch_elems.
Plan plan_of(const Gemm& g, size_t scratch_elems, unsigned kinds) {
  const int layout = g.a_kmajor ? (g.b_kmajor ? 0 : 1) : 2;
  const int kslices = std::max(1, (g.K + BK - 1) / BK);
  const double mn = (double)g.M * g.N;
  const bool two = g.C2 != nullptr;
  Plan best{T64, 64, 64, 1, kslices * BK, 1e300};
  double best_t = 1e300;
  for (int k = 0; k < T_KINDS; ++k) {
    const TileCost& c = TILE_COST[layout][k];
    if (!(kinds >> k & 1) || c.bm == 0) continue;
    // (tiles larger than the matrix would go through registers)
    if (k != T64 && (g.M < c.bm || g.N < c.bn)) continue;
    const bool nt4 = k == TNT256 || k == TNT192;
    if (nt4 && (two || !nt4_ok(g, c.bn))) continue;
    const int64_t tiles = (int64_t)((g.M + c.bm - 1) / c.bm) * ((g.N + c.bn - 1) / c.bn);
    const int64_t slots = (int64_t)NUM_CU * c.per_cu;
    for (int sp = 1; sp <= (nt4 ? 1 : std::min(MAX_SPLITS, std::max(1, kslices / 2))); ++sp) {
      const int kc = (kslices + sp - 1) / sp;  // K slices per split
      if ((kslices + kc - 1) / kc != sp) continue;
      if ((sp > 1 || two) && (double)sp * mn > (double)scratch_elems) break;
      const int64_t wgs = tiles * sp, full = wgs / slots, rem = wgs % slots;
      double t = c.fixed + full * (c.tile + kc * std::max(c.lat, c.bw * c.per_cu));
      if (rem) t += c.tile + kc * std::max((double)c.lat, c.bw * std::min<double>(c.per_cu, rem / 256.0 + 0.25));
      // the sum of the partials: a launch, its serial reads, its traffic
      if (sp > 1 || two) t += 2.5 + 0.24 * sp + 0.16 * (sp + 1) * mn * 4e-6;
      if (t < best_t) {
        best_t = t;
        best = Plan{k, c.bm, c.bn, sp, kc * BK, t};
      }
    }
  }
  return best;
}
constexpr unsigned ALL_KINDS = (1u << T_KINDS) - 1;

// Split-K factor that the workspace reserves partials for.  Callers keep workspaces sized by
// it, so it stays as it is; plan_of takes what fits.  (Rounds of workgroups x their work, plus
// the partials' traffic.)
int reserved_splits(const Gemm& g) {
  struct Cand { int bm, bn, per_cu; double rate; };
  const Cand cands[] = {{256, 256, 1, 1.0}, {256, 192, 1, g.a_kmajor ? 0.93 : 0.7},
                        {128, 128, 2, 0.62}, {192, 256, 1, 0.8}};
  const int kslices = (g.K + BK - 1) / BK;
  const int max_s = g.K >= 8 * BK * 8 ? std::min(64, std::max(1, kslices / 8)) : 1;
  int best = 1;
  double best_t = 1e300;
  for (const Cand& c : cands) {
    if (c.bm == 192 && (g.a_kmajor || g.b_kmajor || g.M % 192)) continue;
    const int64_t tiles = (int64_t)((g.M + c.bm - 1) / c.bm) * ((g.N + c.bn - 1) / c.bn);
    for (int sp = 1; sp <= max_s; ++sp) {
      const int kc = (kslices + sp - 1) / sp;
      if ((kslices + kc - 1) / kc != sp) continue;
      const int64_t slots = (int64_t)NUM_CU * c.per_cu, rounds = (tiles * sp + slots - 1) / slots;
      double t = (double)rounds * kc * ((double)c.bm * c.bn / 65536.0) * c.per_cu / c.rate;
      if (sp > 1) t += (double)(sp + 1) * g.M * g.N * 4 / 3.0e6;
      if (t < best_t * 0.999) {
        best_t = t;
        best = sp;
      }
    }
  }
  return best;
}

template <bool AK, bool BKM, typename TC>
const char* launch(const GemmDev& d, const Plan& p, hipStream_t s) {
  const int tiles = ((d.M + p.bm - 1) / p.bm) * ((d.N + p.bn - 1) / p.bn);
  if constexpr (AK && BKM) {
    const bool whole = d.M % 256 == 0 && d.N % p.bn == 0;
    const int nt_grid = std::min(tiles, NUM_CU);
    if (p.kind == TNT256) {
      if (whole) gemm_nt4_persist_kernel<256, TC, false><<<nt_grid, 256, 0, s>>>(d);
      else gemm_nt4_persist_kernel<256, TC, true><<<nt_grid, 256, 0, s>>>(d);
      return KLABEL("gemm_nt4_persist_kernel<256,256,NT,%s>", sizeof(TC) == 4 ? "fp32" : "bf16");
    }
    if (p.kind == TNT192) {
      if (whole) gemm_nt4_persist_kernel<192, TC, false><<<nt_grid, 256, 0, s>>>(d);
      else gemm_nt4_persist_kernel<192, TC, true><<<nt_grid, 256, 0, s>>>(d);
      return KLABEL("gemm_nt4_persist_kernel<256,192,NT,%s>", sizeof(TC) == 4 ? "fp32" : "bf16");
    }
  }
  const bool persist = d.lscale == nullptr && p.kind != T64;
#define GL_(name, bm, bn) KLABEL(name "<%d,%d,%s,%s>", bm, bn, AK ? (BKM ? "NT" : "NN") : "TN", \
                                 sizeof(TC) == 4 ? "fp32" : "bf16")
  if (persist) {
    GemmDev e = d;
    e.nsplit = p.splits;
    const int per_cu = p.kind == T128 ? 2 : 1;
    const int grid = std::min(tiles * p.splits, NUM_CU * per_cu);
    if (p.kind == T256) {
      gemm_mfma_persist_kernel<256, 256, GWM, GWN, AK, BKM, TC, GBK, GNST><<<grid, 64 * GWM * GWN, 0, s>>>(e);
      return GL_("gemm_mfma_persist_kernel", 256, 256);
    } else if (p.kind == T256x192) {
      gemm_mfma_persist_kernel<256, 192, 4, 2, AK, BKM, TC, GBK, GNST><<<grid, 512, 0, s>>>(e);
      return GL_("gemm_mfma_persist_kernel", 256, 192);
    } else if (p.kind == T192x256) {
      if constexpr (!AK && !BKM) {
        gemm_mfma_persist_kernel<192, 256, 2, 4, AK, BKM, TC, GBK, GNST><<<grid, 512, 0, s>>>(e);
        return GL_("gemm_mfma_persist_kernel", 192, 256);
      }
    }
    gemm_mfma_persist_kernel<128, 128, 2, 2, AK, BKM, TC, 64, 2><<<grid, 256, 0, s>>>(e);
    return GL_("gemm_mfma_persist_kernel", 128, 128);
  }
  // the small tiles, and the masked-loss epilogue (NT only)
  const dim3 grid(tiles, p.splits);
  if (p.kind == T64) {
    gemm_mfma_kernel<64, 64, 2, 2, AK, BKM, TC, 64, 4><<<grid, 256, 0, s>>>(d);
    return GL_("gemm_mfma_kernel", 64, 64);
  }
  if constexpr (AK && BKM) {
    if (p.kind == T256) {
      gemm_mfma_kernel<256, 256, GWM, GWN, AK, BKM, TC, GBK, GNST><<<grid, 64 * GWM * GWN, 0, s>>>(d);
      return GL_("gemm_mfma_kernel(masked loss)", 256, 256);
    } else if (p.kind == T256x192) {
      gemm_mfma_kernel<256, 192, 4, 2, AK, BKM, TC, GBK, GNST><<<grid, 512, 0, s>>>(d);
      return GL_("gemm_mfma_kernel(masked loss)", 256, 192);
    }
    gemm_mfma_kernel<128, 128, 2, 2, AK, BKM, TC, 64, 2><<<grid, 256, 0, s>>>(d);
    return GL_("gemm_mfma_kernel(masked loss)", 128, 128);
  }
  return nullptr;
#undef GL_
}


}  // namespace

size_t gemm_mfma_scratch_elems(const Gemm& g) {
  const int splits = reserved_splits(g);
  return splits > 1 || g.C2 ? (size_t)splits * g.M * g.N : 0;
}

// the device arguments of a plain product
static GemmDev dev_of(const Gemm& g) {
  GemmDev d;
  d.M = g.M; d.N = g.N; d.ktotal = g.K; d.nsplit = 1;
  d.A = (const bf16_t*)g.A; d.lda = g.lda;
  d.B = (const bf16_t*)g.B; d.ldb = g.ldb;
  d.aligned = ((uintptr_t)g.A | (uintptr_t)g.B) % 16 == 0 && g.lda % 8 == 0 && g.ldb % 8 == 0;
  d.C = g.C; d.ldc = g.ldc; d.alpha = g.alpha; d.beta = g.beta;
  d.mstore = g.M; d.part = nullptr; d.kchunk = 0;
  d.lscale = nullptr; d.lmask = nullptr; d.lpart = nullptr; d.lref = nullptr; d.ldref = 0;
  d.causal = 0; d.rev = 0; d.nbatch = 1; d.zdiv = 1; d.bdiv = 1; d.kgroups = 1;
  d.sA = d.sB1 = d.sB2 = d.sC1 = d.sC2 = d.sAk = d.sBk = 0;
  d.split_n = 0; d.c_lo = nullptr; d.ldc_lo = d.sC1_lo = d.sC2_lo = 0;
  return d;
}

// whether the four-column sum takes this output
static bool sum4_ok(const Gemm& g) {
  return g.N % 4 == 0 && g.ldc % 4 == 0 && (uintptr_t)g.C % (g.c_t == DT_F32 ? 16 : 8) == 0;
}
static bool two_ok(const Gemm& g) {
  return g.beta == 0.f && g.m2 > 0 && g.m2 < g.M && g.N % 4 == 0 && g.ldc % 4 == 0 &&
         (uintptr_t)g.C % 16 == 0 && (uintptr_t)g.C2 % 16 == 0 && g.c_t == DT_F32;
}
// the sums of one product's partials (two of them for a two-output product) added to gr
static void add_sum(SumGroup& gr, const Gemm& g, const float* part, int splits) {
  const int64_t total = (int64_t)g.M * g.N;
  auto add = [&](const float* p, int64_t n, void* C, float beta) {
    SumDev& d = gr.s[gr.n];
    d.part = p; d.sstride = total; d.ldc = g.ldc; d.C = C; d.splits = splits; d.N = g.N;
    d.alpha = g.alpha; d.beta = beta;
    d.end = (gr.n ? gr.s[gr.n - 1].end : 0) + n / 4;
    ++gr.n;
  };
  if (g.C2) {  // rows [0, m2) into C, [m2, M) into C2
    const int64_t t1 = (int64_t)g.m2 * g.N;
    add(part, t1, g.C, 0.f);
    add(part + t1, total - t1, g.C2, 0.f);
  } else {
    add(part, total, g.C, g.beta);
  }
}
static hipError_t run_sums(const SumGroup& gr, bool f32, double bytes, hipStream_t s) {
  const unsigned grid = (unsigned)((gr.s[gr.n - 1].end + 255) / 256);
  prof_begin(KC_ELEM, s);
  if (f32) splitk_reduce4_kernel<float><<<grid, 256, 0, s>>>(gr);
  else splitk_reduce4_kernel<bf16_t><<<grid, 256, 0, s>>>(gr);
  prof_end(KC_ELEM, s, 0.0, bytes, KLABEL("splitk_reduce4_kernel"));
  return hipGetLastError();
}
static double sum_bytes(const Gemm& g, int splits) {
  return (double)g.M * g.N * (4.0 * splits + (g.c_t == DT_F32 ? 4.0 : 2.0) * (g.beta != 0.f ? 2.0 : 1.0));
}

hipError_t gemm_mfma(const Gemm& g, float* scratch, size_t scratch_elems, hipStream_t s, int kc,
                     double flops, double bytes) {
  GemmDev d = dev_of(g);
  // two outputs: always through the partials (also unsplit), summed into C and C2
  const bool two = g.C2 != nullptr;
  if (!g.a_kmajor && g.b_kmajor) return hipErrorInvalidValue;  // (no such product)
  if (two && (!two_ok(g) || !scratch || scratch_elems < (size_t)g.M * g.N)) return hipErrorInvalidValue;
  const Plan p = plan_of(g, scratch ? scratch_elems : 0, ALL_KINDS);
  d.kchunk = p.kchunk;
  d.part = p.splits > 1 || two ? scratch : nullptr;
  const bool f32 = g.c_t == DT_F32;
  const char* kname = nullptr;
  prof_begin(kc, s);
#define L_(AK, BK_)                                                                     \
  if (g.a_kmajor == AK && g.b_kmajor == BK_) {                                          \
    if (f32) kname = launch<AK, BK_, float>(d, p, s);                                   \
    else kname = launch<AK, BK_, bf16_t>(d, p, s);                                      \
  }
  L_(true, true) else L_(true, false) else L_(false, false)
#undef L_
  prof_end(kc, s, flops, bytes, kname);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || (p.splits == 1 && !two)) return e;
  // the split-K partials summed in a fixed order (an elementwise launch of its own)
  if (two || sum4_ok(g)) {
    SumGroup gr;
    gr.n = 0;
    add_sum(gr, g, scratch, p.splits);
    return run_sums(gr, f32, sum_bytes(g, p.splits), s);
  }
  const int64_t total = (int64_t)g.M * g.N;
  const unsigned grid = (unsigned)((total + 255) / 256);
  prof_begin(KC_ELEM, s);
  if (f32)
    splitk_reduce_kernel<float><<<grid, 256, 0, s>>>(scratch, p.splits, total, g.M, g.N,
                                                     (float*)g.C, g.ldc, g.alpha, g.beta);
  else
    splitk_reduce_kernel<bf16_t><<<grid, 256, 0, s>>>(scratch, p.splits, total, g.M, g.N,
                                                      (bf16_t*)g.C, g.ldc, g.alpha, g.beta);
  prof_end(KC_ELEM, s, 0.0, sum_bytes(g, p.splits), KLABEL("splitk_reduce_kernel"));
  return hipGetLastError();
}

// 128 x 64 tiles, three slices in flight, two workgroups per CU (group launches only; fitted as
// TILE_COST)
constexpr TileCost COST_128x64[3] = {{128, 64, 2, 5.5f, 0.f, 0.54f, 0.45f},
                                     {128, 64, 2, 5.6f, 0.f, 0.56f, 0.452f},
                                     {128, 64, 2, 2.2f, 3.5f, 0.69f, 0.494f}};

// One launch for all n products (plus one for the sums of their partials) where the time model
// finds that quicker than a launch each: few tokens, where a launch costs more than its work
// (about 4.6 us behind another one) and each product alone leaves CUs idle.  All on one of
// three tiles: the launch takes as long as its longest walk (`lat` per slice) or the CUs' share
// of all slices (`bw`, per output least for the largest tile), so the products are split to
// walks of at most kc slices, tile and kc chosen.
// Returns hipErrorNotSupported (nothing launched) where separate launches are better.
hipError_t gemm_mfma_group(const Gemm* g, int n, float* scratch, size_t scratch_elems, hipStream_t s,
                           int kclass, double flops, double bytes) {
  if (n < 2 || n > GROUP_MAX) return hipErrorNotSupported;
  const int layout = g[0].a_kmajor ? (g[0].b_kmajor ? 0 : 1) : 2;
  const size_t room = scratch ? scratch_elems : 0;
  double sep = 0.0;
  int kmax = 1;
  for (int i = 0; i < n; ++i) {
    if (g[i].a_kmajor != g[0].a_kmajor || g[i].b_kmajor != g[0].b_kmajor || g[i].c_t != g[0].c_t ||
        (!g[i].a_kmajor && g[i].b_kmajor) || g[i].M <= 0 || g[i].N <= 0)
      return hipErrorNotSupported;
    if (g[i].C2 ? !two_ok(g[i]) : !sum4_ok(g[i])) return hipErrorNotSupported;
    // (a product that adds to the one before it: both go as partials of one sum)
    if (g[i].beta != 0.f && !(i > 0 && g[i].beta == 1.f && g[i].C == g[i - 1].C && g[i].M == g[i - 1].M &&
                              g[i].N == g[i - 1].N && g[i].ldc == g[i - 1].ldc && !g[i].C2 && !g[i - 1].C2 &&
                              g[i - 1].beta == 0.f && g[i].alpha == g[i - 1].alpha))
      return hipErrorNotSupported;
    sep += plan_of(g[i], room, ALL_KINDS).t;
    kmax = std::max(kmax, (g[i].K + BK - 1) / BK);
  }
  // (the mixes of output types that the step has: bf16, and fp32 for the weight gradients)
  if ((g[0].c_t == DT_F32) != (layout == 2)) return hipErrorNotSupported;
  auto joined = [&](int i) { return g[i].beta != 0.f || (i + 1 < n && g[i + 1].beta != 0.f); };
  auto splits_of = [&](int i, int kc) {
    const int ks = std::max(1, (g[i].K + BK - 1) / BK), sp = (ks + kc - 1) / kc;
    const int per = (ks + sp - 1) / sp;
    return (ks + per - 1) / per;
  };
  int best_kc = 0, best_tile = 0;
  double best_t = sep;
  for (int tile = 0; tile < 3; ++tile) {
    const TileCost& c = tile == 0   ? TILE_COST[layout][T64]
                        : tile == 1 ? COST_128x64[layout]
                                    : TILE_COST[layout][T128];
    const int64_t slots = (int64_t)NUM_CU * c.per_cu;
    for (int kc = kmax; kc >= std::min(2, kmax); kc = std::min(kc - 1, kc * 3 / 4)) {
      double slices = 0.0, elems = 0.0;
      int64_t wgs = 0;
      int walk = 0, msp = 0;
      for (int i = 0; i < n; ++i) {
        const int64_t tiles = (int64_t)((g[i].M + c.bm - 1) / c.bm) * ((g[i].N + c.bn - 1) / c.bn);
        const int ks = std::max(1, (g[i].K + BK - 1) / BK), sp = splits_of(i, kc);
        wgs += tiles * sp;
        slices += (double)tiles * ks;
        walk = std::max(walk, (ks + sp - 1) / sp);
        if (sp > 1 || g[i].C2 || joined(i)) {
          elems += (double)sp * g[i].M * g[i].N;
          msp = std::max(msp, sp);
        }
      }
      if (elems > (double)room) break;  // (shorter walks need more partials)
      // one round: as in plan_of; more: the CUs' share of all slices, then the last walks alone
      double t = c.fixed + c.tile * ((wgs + slots - 1) / slots);
      if (wgs <= slots) t += walk * std::max<double>(c.lat, c.bw * std::min<double>(c.per_cu, wgs / 256.0 + 0.25));
      else t += slices / 256.0 * c.bw + 0.7 * walk * c.lat;
      if (msp) t += 2.5 + 0.24 * msp + 0.16 * elems * 4e-6;
      if (t < best_t) {
        best_t = t;
        best_kc = kc;
        best_tile = tile;
      }
    }
  }
  // Large products of one A on the four-wavefront kernel: one grid of tiles instead of a partly
  // filled last round of each. Measured against the launches it replaces: Q/K/V of 8192 tokens
  // of the 8B layer 339 us, apart 232 + 85 + 85; the five products of h and the two of c^KV of
  // 6002 tokens of the 4096-wide layer with 32 full heads: the whole step 3050 us, before 3125.
  // The rule is the fitted time: where each product fills its rounds by itself, or is too small
  // for 256-row tiles, the launches apart or the smaller tiles come out cheaper.
  int best_bn = 0;
  bool same_a = layout == 0 && g[0].c_t == DT_BF16;
  for (int i = 0; i < n; ++i)
    same_a = same_a && g[i].A == g[0].A && g[i].lda == g[0].lda && g[i].M == g[0].M && g[i].K == g[0].K &&
             g[i].ldb == g[0].ldb && g[i].alpha == g[0].alpha && g[i].beta == 0.f && !g[i].C2;
  for (int bn = 256; same_a && bn >= 192; bn -= 64) {
    const TileCost& c = TILE_COST[0][bn == 256 ? TNT256 : TNT192];
    bool ok = true;
    int64_t tn = 0;
    for (int i = 0; i < n; ++i) {
      ok = ok && nt4_ok(g[i], bn);
      tn += (g[i].N + bn - 1) / bn;
    }
    const int64_t tiles = tn * ((g[0].M + 255) / 256), full = tiles / NUM_CU, rem = tiles % NUM_CU;
    const int ks = (g[0].K + BK - 1) / BK;
    double t = c.fixed + full * (c.tile + ks * c.bw);
    if (rem) t += c.tile + ks * std::max<double>(c.lat, c.bw * std::min(1.0, rem / 256.0 + 0.25));
    if (ok && t < best_t) {
      best_t = t;
      best_bn = bn;
    }
  }
  if (best_bn) {
    Nt4Group gr;
    gr.n = n;
    int tn = 0;
    bool whole = g[0].M % 256 == 0;
    for (int i = 0; i < n; ++i) {
      tn += (g[i].N + best_bn - 1) / best_bn;
      whole = whole && g[i].N % best_bn == 0;
      gr.end[i] = tn;
      gr.N[i] = g[i].N;
      gr.B[i] = (const bf16_t*)g[i].B;
      gr.C[i] = g[i].C;
      gr.ldc[i] = g[i].ldc;
    }
    const GemmDev d = dev_of(g[0]);
    const int grid = std::min(tn * ((g[0].M + 255) / 256), NUM_CU);
    prof_begin(kclass, s);
    if (best_bn == 256) {
      if (whole) gemm_nt4_group_kernel<256, bf16_t, false><<<grid, 256, 0, s>>>(d, gr);
      else gemm_nt4_group_kernel<256, bf16_t, true><<<grid, 256, 0, s>>>(d, gr);
    } else {
      if (whole) gemm_nt4_group_kernel<192, bf16_t, false><<<grid, 256, 0, s>>>(d, gr);
      else gemm_nt4_group_kernel<192, bf16_t, true><<<grid, 256, 0, s>>>(d, gr);
    }
    prof_end(kclass, s, flops, bytes, best_bn == 256 ? KLABEL("gemm_nt4_group_kernel<256,256,NT,bf16>")
                                                     : KLABEL("gemm_nt4_group_kernel<256,192,NT,bf16>"));
    return hipGetLastError();
  }
  if (best_kc == 0) return hipErrorNotSupported;
  const int bm = best_tile == 0 ? 64 : 128, bn = best_tile == 2 ? 128 : 64;
  GroupDev gr;
  SumGroup sums;
  gr.n = n;
  sums.n = 0;
  size_t off = 0;
  int wgs = 0;
  double sbytes = 0.0;
  for (int i = 0; i < n; ++i) {
    GemmDev d = dev_of(g[i]);
    const int ks = std::max(1, (g[i].K + BK - 1) / BK), sp = splits_of(i, best_kc);
    d.kchunk = (ks + sp - 1) / sp * BK;
    if (sp > 1 || g[i].C2 || joined(i)) {
      d.part = scratch + off;
      const bool adds = g[i].beta != 0.f;
      int all = sp;
      if (adds) {  // its partials follow those of the product before it, one sum for both
        all = sp + sums.s[sums.n - 1].splits;
        sums.s[sums.n - 1].splits = all;
      } else {
        add_sum(sums, g[i], d.part, sp);
      }
      d.beta = 0.f;
      sbytes += sum_bytes(g[i], sp);
      off += (size_t)sp * g[i].M * g[i].N;
    }
    gr.tiles[i] = ((g[i].M + bm - 1) / bm) * ((g[i].N + bn - 1) / bn);
    wgs += gr.tiles[i] * sp;
    gr.end[i] = wgs;
    gr.p[i] = d;
  }
  const bool f32 = g[0].c_t == DT_F32;
  const char* kname = nullptr;
  prof_begin(kclass, s);
#define T_(bm_, bn_, nst, AK, BK_, TC)                                                            \
  {                                                                                               \
    gemm_group_kernel<bm_, bn_, nst, AK, BK_, TC><<<wgs, 256, 0, s>>>(gr);                        \
    kname = KLABEL("gemm_group_kernel<%d,%d,%s,%s>", bm_, bn_, AK ? (BK_ ? "NT" : "NN") : "TN",   \
                   sizeof(TC) == 4 ? "fp32" : "bf16");                                            \
  }
#define L_(AK, BK_, TC)                                                                           \
  {                                                                                               \
    if (best_tile == 0) T_(64, 64, 4, AK, BK_, TC)                                                \
    else if (best_tile == 1) T_(128, 64, 3, AK, BK_, TC)                                          \
    else T_(128, 128, 2, AK, BK_, TC)                                                             \
  }
  if (layout == 0) L_(true, true, bf16_t) else if (layout == 1) L_(true, false, bf16_t) else L_(false, false, float)
#undef L_
#undef T_
  prof_end(kclass, s, flops, bytes, kname);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || sums.n == 0) return e;
  return run_sums(sums, f32, sbytes, s);
}

size_t gemm_mfma_masked_sse_parts(const Gemm& g) {
  return (size_t)((g.M + 127) / 128) * ((g.N + 127) / 128);
}

hipError_t gemm_mfma_masked_scale(const Gemm& g, const float* scale, const uint8_t* mask,
                                  hipStream_t s, const char** kernel) {
  if (g.beta != 0.f || g.alpha != 1.f || g.in_t != DT_BF16 || !scale || !g.C ||
      !g.a_kmajor || !g.b_kmajor)
    return hipErrorInvalidValue;
  GemmDev d = dev_of(g);
  d.lscale = scale; d.lmask = mask; d.lpart = nullptr; d.lref = nullptr; d.ldref = 0;
  // (the four-wavefront kernel reads the row mask with scalar loads of aligned dwords)
  const bool nt4_mask = (uintptr_t)mask % 4 == 0;
  const Plan p = plan_of(g, 0, nt4_mask ? ALL_KINDS : ALL_KINDS & ~(1u << TNT256 | 1u << TNT192));
  d.kchunk = p.kchunk;
  d.part = nullptr;
  *kernel = g.c_t == DT_F32 ? launch<true, true, float>(d, p, s) : launch<true, true, bf16_t>(d, p, s);
  return hipGetLastError();
}

hipError_t gemm_mfma_masked_sse(const Gemm& g, const float* scale, const uint8_t* mask,
                                const void* ref, int64_t ldref, double* part, int* nparts,
                                hipStream_t s, const char** kernel) {
  if (g.beta != 0.f || g.alpha != 1.f || g.in_t != DT_BF16) return hipErrorInvalidValue;
  GemmDev d = dev_of(g);
  d.lscale = scale; d.lmask = mask; d.lpart = part;
  d.lref = (const bf16_t*)ref; d.ldref = ldref;
  // (tiles of at least 128 x 128: gemm_mfma_masked_sse_parts bounds their number; smaller
  // matrices go through one such tile)
  Plan p = plan_of(g, 0, 1u << T256 | 1u << T256x192 | 1u << T128);
  if (p.kind == T64) p = Plan{T128, 128, 128, 1, p.kchunk, p.t};
  d.kchunk = p.kchunk;
  d.part = nullptr;
  *nparts = ((g.M + p.bm - 1) / p.bm) * ((g.N + p.bn - 1) / p.bn);
  const bool f32 = g.c_t == DT_F32;
  if (!g.a_kmajor || !g.b_kmajor) return hipErrorInvalidValue;
  *kernel = f32 ? launch<true, true, float>(d, p, s) : launch<true, true, bf16_t>(d, p, s);
  return hipGetLastError();
}

// Batched causal products of attention's backward: dQ = dS K (A = dS^T stored [key][query],
// M/N-contiguous, bf16 result) and dK = dS^T Q summed over a group's heads (A k-major, fp32
// result).  BN is the output width rounded up to the supported tile widths.
template <int BM, int BN, int WM, int WN, bool AK, typename TC, bool SHIFT>
static void launch_causal(const GemmDev& d, int nbatch, hipStream_t s) {
  static_assert(CAUSAL_BM % BM == 0, "row tiles that the producer of A counts on");
  const int ntm = (d.M + BM - 1) / BM, ntn = (d.N + BN - 1) / BN;
  const int items = ntm * ntn * nbatch;
  if constexpr (!AK) {
    // dQ (M-contiguous A; K ranges end at the diagonal): one tile per workgroup, dispatched
    // longest range first, in 32-deep slices through a ring of four LDS stages.  The
    // product waits on its copies (the dS^T stream): three slices in flight (84 KB per CU)
    // instead of one 64-deep slice (56 KB) measured 3-6% faster (five stages, and a
    // persistent grid of the two-stage ring, were slower)
    attn_ds_gemm_kernel<BM, BN, WM, WN, AK, false, TC, 32, 4, SHIFT>
        <<<dim3(items, 1), 64 * WM * WN, 0, s>>>(d);
  } else {
    // dK (K ranges start at the diagonal): persistent, 2.6% faster; as many workgroups as
    // fit on the CUs at once (the narrow tiles leave room for two per CU)
    // resident workgroups per CU, queried once per device
    constexpr int MAXDEV = 64;
    static std::atomic<int> occ[MAXDEV];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAXDEV) dev = 0;
    int per_cu = occ[dev].load(std::memory_order_relaxed);
    if (per_cu == 0) {
      int n = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
              &n, attn_ds_gemm_persist_kernel<BM, BN, WM, WN, AK, false, TC, 64, 2, SHIFT>,
              64 * WM * WN, 0) != hipSuccess || n < 1)
        n = 1;
      per_cu = n;
      occ[dev].store(n, std::memory_order_relaxed);
    }
    attn_ds_gemm_persist_kernel<BM, BN, WM, WN, AK, false, TC, 64, 2, SHIFT>
        <<<dim3(std::min(items, NUM_CU * per_cu), 1), 64 * WM * WN, 0, s>>>(d);
  }
}

template <bool AK, typename TC, bool SHIFT>
static hipError_t dispatch_causal(const GemmDev& d, int nbatch, hipStream_t s) {
  if (d.N <= 64) launch_causal<256, 64, 4, 2, AK, TC, SHIFT>(d, nbatch, s);
  // 96 columns: 128-row tiles, two workgroups of four wavefronts per CU (a 256-row tile left
  // one, a wavefront per SIMD that waits alone): 8 x 2048 tokens, 14 heads, dK 168 -> 131 us,
  // dQ 139 -> 131 us
  else if (d.N <= 96) launch_causal<128, 96, 4, 1, AK, TC, SHIFT>(d, nbatch, s);
  else if (d.N <= 128) launch_causal<256, 128, 4, 2, AK, TC, SHIFT>(d, nbatch, s);
  else if (d.N <= 192) launch_causal<256, 192, 4, 2, AK, TC, SHIFT>(d, nbatch, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t gemm_mfma_causal(const Gemm& g, const GemmBatch& bt, hipStream_t s) {
  // (an M-contiguous A is read in 8-row chunks)
  const bool ok = !g.b_kmajor && g.in_t == DT_BF16 && g.beta == 0.f &&
                  (g.a_kmajor || g.M % 8 == 0) &&
                  g.N % 32 == 0 && g.lda % 8 == 0 && g.ldb % 8 == 0 && bt.mstore <= g.M &&
                  bt.kgroups >= 1 && (g.a_kmajor ? (bt.rev && g.c_t == DT_F32)
                                                 : (!bt.rev && g.c_t == DT_BF16)) &&
                  (bt.split_n == 0 || (g.a_kmajor && bt.split_n % 4 == 0 && bt.split_n <= g.N &&
                                       bt.c_lo && bt.ldc_lo % 4 == 0 && bt.sC1_lo % 4 == 0 &&
                                       bt.sC2_lo % 4 == 0 && (uintptr_t)bt.c_lo % 8 == 0 &&
                                       g.ldc % 4 == 0 && bt.sC1 % 4 == 0 && bt.sC2 % 4 == 0 &&
                                       (uintptr_t)g.C % 16 == 0));
  if (!ok) return hipErrorInvalidValue;
  GemmDev d;
  d.M = g.M; d.N = g.N; d.ktotal = g.K; d.nsplit = 1;
  d.A = (const bf16_t*)g.A; d.lda = g.lda;
  d.B = (const bf16_t*)g.B; d.ldb = g.ldb;
  d.aligned = 1;  // (checked above)
  d.C = g.C; d.ldc = g.ldc; d.alpha = g.alpha; d.beta = 0.f;
  d.part = nullptr;
  d.lscale = nullptr; d.lmask = nullptr; d.lpart = nullptr; d.lref = nullptr; d.ldref = 0;
  d.kchunk = (g.K + BK - 1) / BK * BK;
  d.mstore = bt.mstore;
  d.causal = 1; d.rev = bt.rev; d.nbatch = bt.nbatch; d.zdiv = bt.zdiv; d.bdiv = bt.bdiv;
  d.kgroups = bt.kgroups;
  d.sA = bt.sA; d.sB1 = bt.sB1; d.sB2 = bt.sB2; d.sC1 = bt.sC1; d.sC2 = bt.sC2;
  d.sAk = bt.sAk; d.sBk = bt.sBk;
  d.split_n = bt.split_n; d.c_lo = (bf16_t*)bt.c_lo;
  d.ldc_lo = bt.ldc_lo; d.sC1_lo = bt.sC1_lo; d.sC2_lo = bt.sC2_lo;
  if (g.M % CAUSAL_BM == 0)  // whole row tiles of any height
    return g.a_kmajor ? dispatch_causal<true, float, false>(d, bt.nbatch, s)
                      : dispatch_causal<false, bf16_t, false>(d, bt.nbatch, s);
  return g.a_kmajor ? dispatch_causal<true, float, true>(d, bt.nbatch, s)
                    : dispatch_causal<false, bf16_t, true>(d, bt.nbatch, s);
}

}  // namespace mla
