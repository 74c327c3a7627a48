// Batched bf16 matrix-core GEMM for the three products of a Newton-Schulz iteration
// (paper Sec. 2 "Muon": Gram matrix X X^T, polynomial b A + c A^2, product with X).
//
// One workgroup = 256 threads = 4 wavefronts in a 2 x 2 arrangement; each wavefront owns a
// (BM/2) x (BN/2) block of the output tile as TI x TJ accumulators of v_mfma_f32_16x16x32_bf16.
// The 16x16x32 shape moves half the accumulator traffic per FLOP of the 32x32x16 one, and this
// part is power-limited under matrix-core load: register-only loops on normally distributed
// operands run at 1.84 PFLOP/s with it and 1.75 with the other (microbench.hip).
//
// Operand tiles travel HBM -> LDS directly (buffer_load ... lds): no staging registers, no LDS
// store instructions.  One LDS buffer holds one operand of one 64-deep K tile, so that a
// K-contiguous row is a whole 128-byte line, and the buffers form a ring A0 B0 A1 B1 ... of NB
// (five for the 256 x 256 tile: all 160 KiB of a CU).  A K tile is two 32-deep slices: while
// the matrix cores work on one slice out of registers the next slice's fragments are read from
// LDS, and the transfers of the K tile D = (NB - 1) / 2 ahead are issued, both a few at a time
// between MFMAs: a burst fills the vector-memory queue, and a wavefront issues in order.  One
// barrier per K tile, in its middle, publishes the next K tile and frees both of its own
// buffers.  The ring does not drain between output tiles.  The compiler does not model these
// transfers, so their completion is awaited explicitly (s_waitcnt vmcnt(n): completion of a
// wavefront's vector-memory operations, loads and stores alike, is reported in the order in which they
// were issued, as the public gfx9 memory model has it and as the compiler's own waits assume).  The n
// of a wait is the number of operations certain to have been issued after what is awaited, stores
// included, so that no wait is one for stores that are still on their way.
//
// An operand whose K index is the slow one in memory ("K-strided": X in B'X) is never
// transposed in HBM.  Its tile is stored in LDS as it is in memory ([k][row]) and read with the
// transposing LDS read (ds_read_b64_tr_b16), which hands a lane 4 consecutive k of its row.
//
// A lane of the MFMA may own any row as long as the epilogue knows which.  Accumulator tile i of
// a wavefront's block holds rows TI * idx + i (idx = 0..15), so that a lane (idx = lane % 16)
// owns TI adjacent rows; tile j holds columns 32 (j / 2) + 8 (idx / 4) + 4 (j % 2) + idx % 4, and
// operand order is swapped (the N operand is the MFMA's first), so that a lane owns 8 adjacent
// columns in two tiles.  Both the tile and its transposed copy then leave as 16-byte stores.
//
// Between two output tiles the matrix cores stand still only while the accumulators are rounded and
// half of the tile is stored; the other half waits in registers and leaves during the next tile's
// first K tiles.  256 x 256 tile, cycles at K = 2048: 32 K tiles of 2470 (2048 are MFMAs), 3460 of
// epilogue, about 3000 that the stores behind it cost the first K tiles.  Before this (one epilogue
// of 7 us that also waited for all its stores, staged through the LDS) the same work took 1.04 (2048
// wide) to 1.06 (768 wide) times as long.  Cycles are not time here: the part runs at its power limit,
// 1.7 GHz in these launches, and 16 % fewer cycles at 768 gave 5 %.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "common.h"
#include "tile_deal.h"

namespace mlc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

template <int V> using I = std::integral_constant<int, V>;

namespace {

constexpr int BK = 64;           // K depth of one LDS buffer
constexpr int NTHREADS = 256;
constexpr int NUM_XCD = 8;
constexpr int GROUP_M = 8;        // most tile rows per group of the tile order
constexpr size_t CU_LDS = 160 * 1024;
constexpr int SC1 = 16;           // of a buffer store: write through

struct GemmArgs {
  const bf16_t* A; long lda, strideA;
  const bf16_t* B; long ldb, strideB;
  bf16_t* D; long ldd, strideD;
  const bf16_t* C; long ldc, strideC;
  int K, batch;
  int tiles_m, tiles_n, tiles_per_mat, total_tiles, tiles_per_xcd;
  int last_m, last_n;             // first row and column of the last tile row and column
  int group_m;                    // tile rows per group of the tile order
  int symmetric, transposed;
  float alpha, beta, gamma;
  const float* bscale; int bscale_pow;
};

// Raw buffer resource (base, no stride, unbounded, dword data format) for a matrix.
__device__ __forceinline__ i32x4 make_rsrc(const void* p) {
  const unsigned long a = (unsigned long)p;
  i32x4 r;
  r.x = __builtin_amdgcn_readfirstlane((int)(a & 0xffffffffu));
  r.y = __builtin_amdgcn_readfirstlane((int)((a >> 32) & 0xffffu));
  r.z = -1;
  r.w = 0x00020000;
  return r;
}

// 16 bytes per lane from rsrc[voff + soff] straight into LDS at lds_base + OFF + 16 * lane
// (wavefront-uniform and relative to the workgroup's LDS allocation).
// The statement writes m0; it is on the clobber list so that the compiler keeps nothing live
// in it across a transfer (clang notes that m0 is a reserved register: that note is expected).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int OFF>
__device__ __forceinline__ void dma16(const i32x4& rsrc, unsigned voff, unsigned soff, unsigned lds_base) {
  asm volatile("s_add_u32 m0, %0, %4\n\t"
               "s_nop 0\n\t"
               "buffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds_base), "v"(voff), "s"(rsrc), "s"(soff), "n"(OFF) : "memory", "m0", "scc");
}
// One MFMA of the 256 x 256 tile: acc = b a (+ acc).  Written out so that the accumulator stays where it
// is: left to choose, the compiler moves accumulators about where code paths meet.
template <bool ZERO>
__device__ __forceinline__ void mfma(f32x4& acc, const u32x4& b, const u32x4& a) {
  if constexpr (ZERO) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc) : "v"(b), "v"(a));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}
// The same with a transfer (see dma16): the MFMA stands between the write of m0 and its use.
template <bool ZERO, int OFF>
__device__ __forceinline__ void mfma_dma(f32x4& acc, const u32x4& b, const u32x4& a, const i32x4& rsrc,
                                         unsigned voff, unsigned soff, unsigned lds_base) {
  if constexpr (ZERO)
    asm volatile("s_add_u32 m0, %3, %7\n\t"
                 "v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0\n\t"
                 "buffer_load_dwordx4 %4, %5, %6 offen lds"
                 : "=&a"(acc) : "v"(b), "v"(a), "s"(lds_base), "v"(voff), "s"(rsrc), "s"(soff), "n"(OFF)
                 : "memory", "m0", "scc");
  else
    asm volatile("s_add_u32 m0, %3, %7\n\t"
                 "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\t"
                 "buffer_load_dwordx4 %4, %5, %6 offen lds"
                 : "+a"(acc) : "v"(b), "v"(a), "s"(lds_base), "v"(voff), "s"(rsrc), "s"(soff), "n"(OFF)
                 : "memory", "m0", "scc");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
// Workgroup barrier that waits for this wavefront's LDS reads only (a fence would also wait for
// every store of the previous tile's epilogue that is still on its way).
__device__ __forceinline__ void block_sync() {
  __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0), other counters unconstrained
  asm volatile("s_barrier" ::: "memory");
}

__device__ __forceinline__ unsigned int pair_lo(unsigned int x, unsigned int y) {   // low halves, x first
  return __builtin_amdgcn_perm(y, x, 0x05040100u);
}
__device__ __forceinline__ unsigned int pair_hi(unsigned int x, unsigned int y) {
  return __builtin_amdgcn_perm(y, x, 0x07060302u);
}

// Four accumulator elements, moved to ordinary registers here: the statement keeps the accumulators
// in their accumulation registers until then (left to itself the compiler copies all of them first,
// and from there to scratch memory).
__device__ __forceinline__ f32x4 acc_read(f32x4 a) {
  asm volatile("" : "+v"(a));
  return a;
}
// The wait states between the last MFMA written out above and the first acc_read of its result, which the
// compiler does not know of.  Every accumulator passes through a statement behind the wait, so that
// nothing can read one's value from before it.
template <int TI, int TJ>
__device__ __forceinline__ void acc_settle(f32x4 (&acc)[TI][TJ]) {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 7" ::: "memory");
#pragma unroll
  for (int n = 0; n < TI * TJ; ++n) asm volatile("" : "+a"(acc[n / TJ][n % TJ]));
  __builtin_amdgcn_sched_barrier(0);
}

// In the accumulator layout the 16 lanes of a store meet 16 rows, 64 bytes of each: half a line.  Lanes
// whose rows are neighbours therefore swap: x and y are 16 bytes each of a lane's row, 32 columns
// apart; a becomes 16 bytes of the even lane's row, b of the odd lane's, and a store covers 8 rows of
// 128 bytes (a store costs the address path about five cycles a line).
__device__ __forceinline__ void pair_rows(const u32x4& x, const u32x4& y, bool odd, u32x4& a, u32x4& b) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const unsigned int xs = (unsigned int)__builtin_amdgcn_mov_dpp((int)x[w], 0xb1, 0xf, 0xf, true);   // from the neighbour
    const unsigned int ys = (unsigned int)__builtin_amdgcn_mov_dpp((int)y[w], 0xb1, 0xf, 0xf, true);
    a[w] = odd ? ys : x[w];
    b[w] = odd ? y[w] : xs;
  }
}

// End of the buffers that a tile is stored through: no matrix reaches it (with its row padding one has at most 2^32 bytes), and
// a store at this offset is dropped, whatever its scalar offset.
constexpr unsigned int BUFFER_END = 0xfffffff0u;

// Position of an output tile.
struct TileCoord { int b, m0, n0, mirror, diag, edge; };

// TI adjacent bf16 values of a row <-> TI / 2 words.
template <int TI, int AUX>
__device__ __forceinline__ void store_words(const unsigned int (&w)[TI / 2], __amdgpu_buffer_rsrc_t r,
                                            unsigned int voff, unsigned int soff) {
  if constexpr (TI == 8) {
    u32x4 v;
    v.x = w[0]; v.y = w[1]; v.z = w[2]; v.w = w[3];
    __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, soff, AUX);
  } else if constexpr (TI == 2) {
    __builtin_amdgcn_raw_buffer_store_b32(w[0], r, voff, soff, AUX);
  } else {
    u32x2 v;
    v.x = w[0]; v.y = w[1];
    __builtin_amdgcn_raw_buffer_store_b64(v, r, voff, soff, AUX);
  }
}

// Epilogue of one tile: D = alpha_b * acc + beta * C + gamma * I, stored as bf16.  MIRROR: the
// transposed tile is stored as well (symmetric outputs compute only the lower triangle of
// tiles).  TOUT: only the transposed tile is stored, and C is read transposed.  DIAG: the
// diagonal may cross the tile.  UNIT: alpha_b is 1.
//
// Of the 256 x 256 tile only the first 64 of a wavefront's 128 columns leave here; the others are
// left packed in `pend`, and run_tiles stores them between the MFMAs of the next tile's first K
// tiles.  (All 128 columns at once would not fit beside the next tile's fragments.)  What bounds this
// is the stores: a CU sends about one line in five cycles, so a row is rounded while the one before it
// is on its way (one row after the other 3460 cycles, all rows before the first store 4500; with rows
// gathered to whole lines through the LDS instead of pair_rows 4600, and as half lines 6400).
constexpr int epilogue_stores(int ti, bool mirror) {      // what store_tile leaves in flight, at least
  const int plain = ti == 8 ? 16 : ti == 4 ? 8 : 2, transposed = ti == 2 ? 8 : 16;
  return mirror ? plain + transposed : plain;
}
template <int TI, int TJ, int AUX, bool HAS_C, bool MIRROR, bool TOUT, bool DIAG, bool UNIT>
__device__ __forceinline__ void store_tile(const GemmArgs& g, const f32x4 (&acc)[TI][TJ],
                                           const TileCoord& tc, float alpha, int wbase_m, int wbase_n,
                                           int lane, bool drop, u32x4 (&pend)[TI == 8 ? 16 : 1]) {
  // what follows from the lane is computed here, not kept in registers through the K loop
  asm volatile("" : "+v"(lane));
  // lane's first row and column; its element (i, J, e) is row row0 + i, column col0 + 32 J + e.
  // All accesses go through buffer resources on the batch's matrix: one lane offset in a VGPR,
  // the row offset in a scalar register.
  const int idx = lane & 15, lg = lane >> 4;
  const int row0 = tc.m0 + wbase_m + TI * idx;
  const int col0 = tc.n0 + wbase_n + 8 * lg;
  constexpr int NJ = TJ / 2;
  constexpr int NH = NJ > 1 ? 2 : 1;      // 32-column blocks handled together
  constexpr int NP = NJ / NH;             // the second of two such groups is the one left in `pend`
  static_assert(NP == (TI == 8 ? 2 : 1), "which columns are stored when");
  const __amdgpu_buffer_rsrc_t rd =
      __builtin_amdgcn_make_buffer_rsrc(g.D + (long)tc.b * g.strideD, 0, BUFFER_END, 0x00020000);
  __amdgpu_buffer_rsrc_t rc = rd;
  if constexpr (HAS_C)
    rc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(g.C) + (long)tc.b * g.strideC, 0,
                                           BUFFER_END, 0x00020000);
  const unsigned int ldd2 = (unsigned int)(g.ldd * 2), ldc2 = (unsigned int)(g.ldc * 2);
  const unsigned int voff_m = drop ? BUFFER_END : (unsigned int)(((long)col0 * g.ldd + row0) * 2);   // transposed
  const unsigned int voff_c =
      HAS_C ? (unsigned int)(((TOUT ? (long)col0 * g.ldc + row0 : (long)row0 * g.ldc + col0)) * 2) : 0u;
  auto value = [&](float v) { return UNIT ? v : alpha * v; };
  // All of C is requested before the first store: vector-memory operations count down in order, so
  // a wait for a later load would be one for the stores before it.
  if constexpr (TOUT) {
    constexpr int NX = 8 * NH;            // columns of a group
    u32x4 c[NP][NX];
    if constexpr (HAS_C)
#pragma unroll
      for (int x = 0; x < NP * NX; ++x) {
        const unsigned int soff = (unsigned int)(32 * (x / 8) + x % 8) * ldc2;
        u32x4& d = c[x / NX][x % NX];
        if constexpr (TI == 8) d = __builtin_amdgcn_raw_buffer_load_b128(rc, voff_c, soff, 0);
        else if constexpr (TI == 2) d.x = __builtin_amdgcn_raw_buffer_load_b32(rc, voff_c, soff, 0);
        else {
          const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rc, voff_c, soff, 0);
          d.x = v.x;
          d.y = v.y;
        }
      }
#pragma unroll
    for (int x4 = 0; x4 < NX; x4 += 4)
#pragma unroll
      for (int P = 0; P < NP; ++P) {
        // keep the scheduler from pulling later accumulator reads up here: all accumulators in
        // VGPRs at once do not fit
        __builtin_amdgcn_sched_barrier(0);
        unsigned int w[4][TI / 2];
#pragma unroll
        for (int i = 0; i < TI; i += 2) {
          const f32x4 lo = acc_read(acc[i][2 * NH * P + x4 / 4]), hi = acc_read(acc[i + 1][2 * NH * P + x4 / 4]);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float v0 = value(lo[e]), v1 = value(hi[e]);
            if constexpr (HAS_C) {
              v0 += g.beta * bf16lo(c[P][x4 + e][i / 2]);
              v1 += g.beta * bf16hi(c[P][x4 + e][i / 2]);
            }
            w[e][i / 2] = pack_bf16x2(v0, v1);
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int x = x4 + e;
          if constexpr (TI == 8) {
            if (P > 0) { pend[x] = u32x4{w[e][0], w[e][1], w[e][2], w[e][3]}; continue; }
          }
          store_words<TI, AUX>(w[e], rd, voff_m, (unsigned int)(32 * (x / 8) + x % 8) * ldd2);
        }
      }
  } else {
    u32x4 c[NP][NH][TI];
    if constexpr (HAS_C)
#pragma unroll
      for (int x = 0; x < NJ * TI; ++x)
        c[x / TI / NH][x / TI % NH][x % TI] =
            __builtin_amdgcn_raw_buffer_load_b128(rc, voff_c + 64u * (x / TI), (unsigned int)(x % TI) * ldc2, 0);
    const bool odd = idx & 1;
    const unsigned int voff_n = drop ? BUFFER_END :
        (unsigned int)(((long)(row0 - (NH == 2 && odd ? TI : 0)) * g.ldd + col0 + (NH == 2 && odd ? 32 : 0)) * 2);
    const int diag = col0 - row0;         // i - (32 J + e) of the lane's elements on the diagonal
    u32x4 first[TI][NH];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int P = 0; P < NP; ++P) {
        __builtin_amdgcn_sched_barrier(0);
        u32x4 packed[NH];
#pragma unroll
        for (int h = 0; h < NH; ++h) {
          const int J = NH * P + h;
          const f32x4 lo = acc_read(acc[i][2 * J]), hi = acc_read(acc[i][2 * J + 1]);
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            float v0 = value(e < 4 ? lo[e % 4] : hi[e % 4]), v1 = value(e < 4 ? lo[e % 4 + 1] : hi[e % 4 + 1]);
            if constexpr (HAS_C) {
              v0 += g.beta * bf16lo(c[P][h][i][e / 2]);
              v1 += g.beta * bf16hi(c[P][h][i][e / 2]);
            }
            if constexpr (DIAG) {
              if (i - (32 * J + e) == diag) v0 += g.gamma;
              if (i - (32 * J + e + 1) == diag) v1 += g.gamma;
            }
            packed[h][e / 2] = pack_bf16x2(v0, v1);
          }
        }
        if constexpr (TI == 8) {
          if (P > 0) { pend[2 * i] = packed[0]; pend[2 * i + 1] = packed[1]; continue; }
        }
        if constexpr (NH == 1) {          // a wavefront's rows are 64 bytes: nothing to gather
          __builtin_amdgcn_raw_buffer_store_b128(packed[0], rd, voff_n, (unsigned int)i * ldd2, AUX);
        } else {
          u32x4 x, y;
          pair_rows(packed[0], packed[1], odd, x, y);
          __builtin_amdgcn_raw_buffer_store_b128(x, rd, voff_n, (unsigned int)i * ldd2, AUX);
          __builtin_amdgcn_raw_buffer_store_b128(y, rd, voff_n, (unsigned int)(TI + i) * ldd2, AUX);
        }
#pragma unroll
        for (int h = 0; h < NH; ++h) first[i][h] = packed[h];
      }
    if constexpr (MIRROR) {
      // column col0 + 32 J + e of this tile becomes a row of the mirrored tile
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          unsigned int w[TI / 2];
#pragma unroll
          for (int i = 0; i < TI; i += 2)
            w[i / 2] = (e & 1) ? pair_hi(first[i][h][e / 2], first[i + 1][h][e / 2])
                               : pair_lo(first[i][h][e / 2], first[i + 1][h][e / 2]);
          store_words<TI, AUX>(w, rd, voff_m, (unsigned int)(32 * h + e) * ldd2);
        }
    }
  }
}

// Epilogue of a tile on the diagonal of a symmetric product, in which a lane holds rows 32 (i / 2) + 8 (idx / 4) + 4 (i % 2)
// + idx % 4 in accumulator tile i, and columns as everywhere.  DG: a quarter on the diagonal, of which the
// blocks (I, J) of 32 x 32 with J <= I have been computed; its diagonal is the matrix's.  Otherwise 128 x 64 of the
// lower left quarter.  Every block off the diagonal is stored a second time, transposed: four lanes hold a column's
// 8 adjacent rows between them, and turn them over.  Stores cover whole lines except where a row of blocks
// ends in the middle of one.
constexpr int TRIANGLE_STORES = 32;
// Deepest product whose triangles leave operand A's transfers out.  A triangle then takes 0.7 to 0.8 of a whole
// tile's time (0.9 with the transfers), and the workgroups behind one L2 no longer read the same K tiles at the same time:
// deeper operands do not fit there, and come from memory again.  Without the transfers against with them, newton_schulz over
// 3e8 elements, 512 to 5120 wide: 0.97 to 1.00 up to K = 1536, 0.99 to 1.01 at 2048 and 2560, 0.99 to 1.02 at 2304, 0.99 to 1.03 from
// 2816 to 3584, 0.97 to 1.01 beyond.  Gram and polynomial products of 150M-scale, eight
// replicas (K = 768 and 3072): 590 and 414 us with whole tiles, 556 and 387 with the transfers, 530 and 357 by this rule; the
// Gram products of 1.76B-scale (K = 2048 and 8192) 1940, 1860, and without the transfers at any depth 2280.
constexpr int TRIANGLE_ONE_OPERAND = 2560;
template <bool DG>
__device__ __forceinline__ void triangle_settle(f32x4 (&acc)[8][8]) {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 7" ::: "memory");
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < (DG ? 8 : 4); ++j)
      if (!DG || j / 2 <= i / 2) asm volatile("" : "+a"(acc[i][j]));
  __builtin_amdgcn_sched_barrier(0);
}
template <bool DG>
__device__ __forceinline__ void store_triangle(const GemmArgs& g, const f32x4 (&acc)[8][8], int b, int row0, int col0,
                                               float alpha, bool drop, int lane) {
  asm volatile("" : "+v"(lane));
  const int idx = lane & 15, lg = lane >> 4, q = idx >> 2, p = idx & 3, odd = idx & 1;
  const __amdgpu_buffer_rsrc_t rd =
      __builtin_amdgcn_make_buffer_rsrc(g.D + (long)b * g.strideD, 0, BUFFER_END, 0x00020000);
  // (opaque: its multiples would otherwise be kept in scalar registers all through the K loop)
  unsigned int ldd2 = (unsigned int)(g.ldd * 2);
  asm volatile("" : "+s"(ldd2));
  const int row = row0 + 8 * q + p, col = col0 + 8 * lg;
  constexpr int NJ = DG ? 4 : 2;
  auto has = [](int i, int J) { return !DG || J <= i / 2; };
  auto up = [](int i) { return (unsigned int)(32 * (i / 2) + 4 * (i & 1)); };       // rows of tile i above `row`
  // C of the upper half is awaited before the first store, and that of the lower half requested before it (see
  // store_tile: a wait for a load is one for the stores before it)
  u32x4 c[8][NJ];
  auto load_c = [&](int half) {
    if (!g.C) {
      if constexpr (!DG)
#pragma unroll
        for (int i = 4 * half; i < 4 * half + 4; ++i)
#pragma unroll
          for (int J = 0; J < NJ; ++J) c[i][J] = u32x4{0u, 0u, 0u, 0u};
      return;
    }
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(g.C) + (long)b * g.strideC, 0, BUFFER_END, 0x00020000);
    unsigned int ldc2 = (unsigned int)(g.ldc * 2);
    asm volatile("" : "+s"(ldc2));
    const unsigned int voff_c = (unsigned int)(((long)row * g.ldc + col) * 2);
#pragma unroll
    for (int i = 4 * half; i < 4 * half + 4; ++i)
#pragma unroll
      for (int J = 0; J < NJ; ++J)
        if (has(i, J)) c[i][J] = __builtin_amdgcn_raw_buffer_load_b128(rc, voff_c + 64u * J, up(i) * ldc2, 0);
  };
  const int diag = col - row;              // 32 (i / 2) + 4 (i % 2) - (32 J + e) on the diagonal
  u32x4 v[8][NJ];
  auto round_half = [&](int half, auto c_tag, auto unit_tag) {
    constexpr bool HAS_C = decltype(c_tag)::value, UNIT = decltype(unit_tag)::value;
#pragma unroll
    for (int i = 4 * half; i < 4 * half + 4; ++i)
#pragma unroll
      for (int J = 0; J < NJ; ++J) {
        if (!has(i, J)) continue;
        __builtin_amdgcn_sched_barrier(0);
        const f32x4 lo = acc_read(acc[i][2 * J]), hi = acc_read(acc[i][2 * J + 1]);
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          float v0 = e < 4 ? lo[e % 4] : hi[e % 4], v1 = e < 4 ? lo[e % 4 + 1] : hi[e % 4 + 1];
          if constexpr (!UNIT) { v0 *= alpha; v1 *= alpha; }
          if constexpr (HAS_C) {
            v0 += g.beta * bf16lo(c[i][J][e / 2]);
            v1 += g.beta * bf16hi(c[i][J][e / 2]);
          }
          if (DG && J == i / 2) {
            if (4 * (i & 1) - e == diag) v0 += g.gamma;
            if (4 * (i & 1) - (e + 1) == diag) v1 += g.gamma;
          }
          v[i][J][e / 2] = pack_bf16x2(v0, v1);
        }
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  const unsigned int at = drop ? BUFFER_END : (unsigned int)(((long)row * g.ldd + col) * 2);
  const unsigned int at2 = drop ? BUFFER_END : (unsigned int)(((long)(row - odd) * g.ldd + col + 32 * odd) * 2);     // two blocks' lines
  auto store_row = [&](int i) {
#pragma unroll
    for (int J = 0; J < NJ; J += 2) {
      if (!has(i, J)) continue;
      const unsigned int soff = up(i) * ldd2;
      if (has(i, J + 1)) {
        u32x4 x, y;
        pair_rows(v[i][J], v[i][J + 1], odd, x, y);
        __builtin_amdgcn_raw_buffer_store_b128(x, rd, at2, soff + 64u * J, 0);
        __builtin_amdgcn_raw_buffer_store_b128(y, rd, at2, soff + ldd2 + 64u * J, 0);
      } else {
        __builtin_amdgcn_raw_buffer_store_b128(v[i][J], rd, at, soff + 64u * J, 0);
      }
    }
  };
  // columns 32 J + 8 lg + 2 p and + 1 of block (I, J), rows 8 q .. + 7
  auto turn = [&](int I, int J, u32x4& even, u32x4& next) {
    const u32x4 r0 = transpose_quad(v[2 * I][J], p), r1 = transpose_quad(v[2 * I + 1][J], p);
    even = u32x4{pair_lo(r0[0], r0[1]), pair_lo(r0[2], r0[3]), pair_lo(r1[0], r1[1]), pair_lo(r1[2], r1[3])};
    next = u32x4{pair_hi(r0[0], r0[1]), pair_hi(r0[2], r0[3]), pair_hi(r1[0], r1[1]), pair_hi(r1[2], r1[3])};
  };
  const int trow = col0 + 8 * lg + 2 * p, tcol = row0 + 8 * q;
  const unsigned int mt = drop ? BUFFER_END : (unsigned int)(((long)trow * g.ldd + tcol) * 2);
  const unsigned int mt2 = drop ? BUFFER_END : (unsigned int)(((long)(trow - 2 * odd) * g.ldd + tcol + 32 * odd) * 2);
  auto store_turned = [&](int I, int J) {            // one block
    u32x4 x, y;
    turn(I, J, x, y);
    const unsigned int soff = 32u * J * ldd2;
    __builtin_amdgcn_raw_buffer_store_b128(x, rd, mt, soff + 64u * I, 0);
    __builtin_amdgcn_raw_buffer_store_b128(y, rd, mt, soff + ldd2 + 64u * I, 0);
  };
  auto store_turned2 = [&](int I, int J) {           // blocks (I, J) and (I + 1, J)
    u32x4 x[2], y[2];
    turn(I, J, x[0], y[0]);
    turn(I + 1, J, x[1], y[1]);
    const unsigned int soff = 32u * J * ldd2;
    u32x4 s, t;
    pair_rows(x[0], x[1], odd, s, t);
    __builtin_amdgcn_raw_buffer_store_b128(s, rd, mt2, soff + 64u * I, 0);
    __builtin_amdgcn_raw_buffer_store_b128(t, rd, mt2, soff + 2 * ldd2 + 64u * I, 0);
    pair_rows(y[0], y[1], odd, s, t);
    __builtin_amdgcn_raw_buffer_store_b128(s, rd, mt2, soff + ldd2 + 64u * I, 0);
    __builtin_amdgcn_raw_buffer_store_b128(t, rd, mt2, soff + 3 * ldd2 + 64u * I, 0);
  };
  using T = std::true_type;
  using F = std::false_type;
  const bool unit = alpha == 1.f;
  load_c(0);
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int I = 2 * half;
    if constexpr (!DG) round_half(half, T{}, F{});           // (C is zero where there is none)
    else if (g.C && unit) round_half(half, T{}, T{});
    else if (g.C) round_half(half, T{}, F{});
    else if (unit) round_half(half, F{}, T{});
    else round_half(half, F{}, F{});
    if (half == 0) load_c(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 2 * I; i < 2 * I + 4; ++i) {
      store_row(i);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (DG) {
      store_turned(I + 1, I);
      if (half) { store_turned2(2, 0); store_turned2(2, 1); }
    } else {
      store_turned2(I, 0);
      store_turned2(I, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Persistent kernel: one workgroup per CU slot walks over its share of the output tiles.
// Workgroups are dealt round-robin to the 8 XCDs, so XCD x owns the contiguous range of
// tiles [x * tiles_per_xcd, (x + 1) * tiles_per_xcd) and its workgroups take them in
// order: tiles that share operand panels run at the same time behind the same L2.
// BKS: operand B is K-strided.  NB: buffers of the ring; K >= 64 * (NB - 1) / 2.  WT: results are written through.
template <int BM, int BN, bool BKS, int NB, bool WT>
__device__ __forceinline__ void run_tiles(const GemmArgs& g, Deal deal) {
  static_assert(BM == BN && NB % 2 == 1, "one buffer size, an odd ring");
  constexpr int TI = BM / 32, TJ = BN / 32;          // accumulator tiles per wavefront
  constexpr int NM = TI * TJ;                        // MFMAs per slice
  constexpr unsigned int BUF = BM * BK * 2;          // bytes of a buffer
  constexpr unsigned int RING = NB * BUF;
  constexpr int NCH = BM / 32;                       // transfers per thread and buffer
  constexpr int D = (NB - 1) / 2;                    // K tiles requested ahead
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  const unsigned int lds0 = (unsigned int)(unsigned long)(lds_byte*)smem;
  auto second = [&] { deal.at = deal.at2; deal.end = deal.end2; deal.step = deal.step2; deal.at2 = deal.end2; };
  if (deal.at >= deal.end) second();
  if (deal.at >= deal.end) return;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // A tile on the diagonal of a symmetric product is symmetric itself, and only its lower triangle of 32 x 32 blocks is
  // computed (store_triangle).
  constexpr bool TRI = BM == 256 && !BKS;
  auto decode = [&](int t) {
    TileCoord tc;
    tc.b = t / g.tiles_per_mat;
    const int rem = t - tc.b * g.tiles_per_mat;
    int tm, tn;
    if (g.symmetric) {          // lower triangle, row-major: rem = tm (tm + 1) / 2 + tn
      tm = (int)((sqrtf(8.f * (float)rem + 1.f) - 1.f) * 0.5f);
      while ((tm + 1) * (tm + 2) / 2 <= rem) ++tm;
      while (tm * (tm + 1) / 2 > rem) --tm;
      tn = rem - tm * (tm + 1) / 2;
    } else {
      // Groups of group_m tile rows, column by column inside a group: the tiles an XCD works
      // on at one time (consecutive indices) then form a block about as tall as it is wide
      // and share few operand panels, which its L2 can hold.
      const int per_group = g.group_m * g.tiles_n;
      const int grp = rem / per_group, r = rem - grp * per_group;
      const int first_m = grp * g.group_m;
      const int rows = min(g.tiles_m - first_m, g.group_m);
      tn = r / rows;
      tm = first_m + (r - tn * rows);
    }
    // the last tile row (column) of a matrix that is no multiple of the tile begins half a tile early
    tc.m0 = __builtin_amdgcn_readfirstlane(min(tm * BM, g.last_m));
    tc.n0 = __builtin_amdgcn_readfirstlane(min(tn * BN, g.last_n));
    tc.edge = BM == 256 ? (tc.m0 % BM ? 1 : 0) + (tc.n0 % BN ? 2 : 0) : 0;
    tc.b = __builtin_amdgcn_readfirstlane(tc.b);
    tc.mirror = g.symmetric && tm != tn ? 1 : 0;
    tc.diag = TRI && tm == tn ? 1 : 0;
    return tc;
  };

  const int idx = lane & 15, lg = lane >> 4;
  const int wbase_m = (wave >> 1) * (BM / 2), wbase_n = (wave & 1) * (BN / 2);

  // ---- transfers: LDS chunk c = it * 256 + tid (16 bytes) of a buffer; which global chunk a
  // lane fetches follows from the buffer's layout.
  // K-contiguous buffer: [slot][8 chunks of 16 B], slot (B/2) * half + 16 * tile + idx, chunk x of a
  // slot's row at position x ^ ((slot / 2) % 8): the LDS serves a 128-bit read 16 lanes at a
  // time over 64 banks, and the 16 lanes of one k chunk then meet 16 different 16-byte columns.
  // K-strided buffer: [k][BN], chunk x of row k at position x ^ 4 (k % 4), for the same reason
  // (a transposing read takes 4 chunks of each of 4 consecutive k); with BN = 64 two rows share
  // the 256 bytes of a bank line and the position is x ^ 4 (k / 2 % 2).
  auto ks_swizzle = [](int k) { return BN == 64 ? 4 * ((k >> 1) & 1) : 4 * (k & 3); };
  const int slot = tid >> 3;
  const unsigned int kc_chunk = (unsigned int)(((tid & 7) ^ ((tid >> 4) & 7)) * 16);
  const unsigned int lda2 = (unsigned int)(g.lda * 2), ldb2 = (unsigned int)(g.ldb * 2);
  const unsigned int voffA = (unsigned int)(TI * (slot & 15) + (slot >> 4)) * lda2 + kc_chunk;
  unsigned int voffB;
  if constexpr (BKS) {
    constexpr int CPR = BN / 8;
    voffB = (unsigned int)(tid / CPR) * ldb2 + (unsigned int)(((tid % CPR) ^ ks_swizzle(tid / CPR)) * 16);
  } else {
    voffB = (unsigned int)(8 * ((slot & 15) >> 2) + 4 * (slot >> 4) + (slot & 3)) * ldb2 + kc_chunk;
  }
  const unsigned int stepA = 2 * lda2;                               // rows two apart ...
  const unsigned int jumpA = (unsigned int)(BM / 2 - (TI - 2)) * lda2;   // ... then the other half
  const unsigned int stepB = BKS ? (unsigned int)(NTHREADS / (BN / 8)) * ldb2 : 32u * ldb2;
  const unsigned int advA = BK * 2, advB = BKS ? (unsigned int)BK * ldb2 : BK * 2;
  const unsigned int lds_wave = lds0 + (unsigned int)__builtin_amdgcn_readfirstlane(wave * 1024);

  // ---- fragments: offsets inside a buffer
  const unsigned int swz = (unsigned int)((idx >> 1) & 7);
  const unsigned int fragA = (unsigned int)(wbase_m + idx) * 128 + (((unsigned int)lg ^ swz) * 16);
  unsigned int fragB[BKS ? TJ / 2 : 1];
  if constexpr (BKS) {
    const int k4 = idx >> 2, q = idx & 3;
#pragma unroll
    for (int J = 0; J < TJ / 2; ++J)
      fragB[J] = (unsigned int)(8 * lg + k4) * (BN * 2) + (unsigned int)(((wbase_n / 8 + 4 * J + q) ^ ks_swizzle(k4)) * 16);
  } else {
    fragB[0] = (unsigned int)(wbase_n + idx) * 128 + (((unsigned int)lg ^ swz) * 16);
  }

  u32x4 fa[2][TI], fb[2][TJ];
  f32x4 acc[TI][TJ];
  constexpr int NR = TI + (BKS ? 2 * TJ : TJ);       // LDS reads per slice
  constexpr int RSTEP = NM / 2 / NR > 0 ? NM / 2 / NR : 1;      // MFMAs between reads ...
  constexpr int RPER = (NR + NM - 1) / NM;                      // ... and reads at a time
  constexpr int DSTEP = NM / NCH;                    // MFMAs between transfers

  // LDS read r of a slice: A0, all of B, the rest of A.
  unsigned int ra = 0, rb[BKS ? TJ / 2 : 1];         // LDS addresses of this lane's fragments
  auto point_at = [&](unsigned int bufA, unsigned int bufB, int kk) {
    // the second slice: chunk + 4 (K-contiguous; an xor of bit 2), 32 rows further (K-strided)
    ra = (fragA ^ (kk ? 64u : 0u)) + bufA;
    if constexpr (BKS) {
#pragma unroll
      for (int J = 0; J < TJ / 2; ++J) rb[J] = fragB[J] + bufB + (kk ? 32u * BN * 2 : 0u);
    } else {
      rb[0] = (fragB[0] ^ (kk ? 64u : 0u)) + bufB;
    }
  };
  auto read_one = [&](int set, int r) {
    constexpr int NRB = BKS ? 2 * TJ : TJ;
    if (r == 0 || r > NRB) {
      const int i = r == 0 ? 0 : r - NRB;
      fa[set][i] = *reinterpret_cast<const u32x4*>(smem + ra + i * 2048);
    } else if constexpr (BKS) {
      const int j = (r - 1) >> 1, h = (r - 1) & 1;
      typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
      const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_s16x4)((lds_byte*)smem + rb[j >> 1] + (j & 1) * 8 + h * 4 * (BN * 2)));
      const u32x2 w = __builtin_bit_cast(u32x2, v);
      fb[set][j][2 * h] = w.x;
      fb[set][j][2 * h + 1] = w.y;
    } else {
      fb[set][r - 1] = *reinterpret_cast<const u32x4*>(smem + rb[0] + (r - 1) * 2048);
    }
  };

  // ---- where the transfers stand: K tile `ck` of a tile (this workgroup's current or next one)
  i32x4 rsA, rsB;
  unsigned int soA, soB;              // scalar byte offsets of the tile's rows and the K tile
  int left;                           // K tiles of that output tile still to be requested
  const int KT = g.K / BK;
  auto aim = [&](const TileCoord& tc) {
    rsA = make_rsrc(g.A + (long)tc.b * g.strideA);
    rsB = make_rsrc(g.B + (long)tc.b * g.strideB);
    soA = (unsigned int)tc.m0 * lda2;
    soB = BKS ? (unsigned int)tc.n0 * 2 : (unsigned int)tc.n0 * ldb2;
    left = KT;
  };
  unsigned int runA = 0, runB = 0;    // offsets of the next transfer
  // what transfer `it` of an operand's buffer is followed by
  auto next_a = [&](int it) { runA += it == TI / 2 - 1 ? jumpA : stepA; };
  auto next_b = [&](int) { runB += stepB; };
  auto dma_a = [&](auto it_tag, unsigned int dst) {
    constexpr int it = decltype(it_tag)::value;
    dma16<it * 4096>(rsA, voffA, runA, dst);
    next_a(it);
  };
  auto dma_b = [&](auto it_tag, unsigned int dst) {
    constexpr int it = decltype(it_tag)::value;
    dma16<it * 4096>(rsB, voffB, runB, dst);
    next_b(it);
  };
  auto dma_n = [&](int n, auto&& f) {        // f(I<n>): n is a constant after unrolling
    switch (n) {
      case 0: f(I<0>{}); break;
      case 1: f(I<1>{}); break;
      case 2: if constexpr (NCH > 2) f(I<2 % NCH>{}); break;
      case 3: if constexpr (NCH > 2) f(I<3 % NCH>{}); break;
      case 4: if constexpr (NCH > 4) f(I<4 % NCH>{}); break;
      case 5: if constexpr (NCH > 4) f(I<5 % NCH>{}); break;
      case 6: if constexpr (NCH > 4) f(I<6 % NCH>{}); break;
      default: if constexpr (NCH > 4) f(I<7 % NCH>{}); break;
    }
  };

  // One slice: NM MFMAs on fragment set `set`, with the reads of the next slice into the other
  // set and the NCH transfers `issue` between them.
  // The second half of the last output tile (64 of each wavefront's 128 columns) waits in `pend` and
  // leaves during the first eight K tiles, two stores (four with a transposed copy) each in its first
  // slice: they then have a K tile's time before a wait can reach them.  (In the second slice they had
  // half of that: 2600 cycles more a K tile.)
  constexpr bool DEFER = TI == 8;
  u32x4 pend[DEFER ? 16 : 1];
  // this workgroup's last tile: has it left half of it in `pend`, has that a transposed copy, was it a triangle
  bool stored = false, mirrored = false, triangle = false;
  __amdgpu_buffer_rsrc_t pend_rd;
  unsigned int pend_n = 0, pend_m = 0, pend_ld = 0;      // lane offsets, plain and transposed; row pitch
  auto drain = [&](int i) {          // row i of a lane's eight (transposed: columns 2 i and 2 i + 1 of its 16)
    u32x4 x = pend[2 * i], y = pend[2 * i + 1];
    unsigned int at = (unsigned int)i * pend_ld, step = TI * pend_ld;
    if (BKS && g.transposed) {
      at = (unsigned int)(32 * (i / 4) + 2 * (i % 4)) * pend_ld;
      step = pend_ld;
    } else {
      pair_rows(pend[2 * i], pend[2 * i + 1], lane & 1, x, y);
    }
    __builtin_amdgcn_raw_buffer_store_b128(x, pend_rd, pend_n, at, 0);
    __builtin_amdgcn_raw_buffer_store_b128(y, pend_rd, pend_n, at + step, 0);
  };
  auto drain_mirror = [&](int q) {   // column q of a lane's 16
    const int h = q / 8, e = q % 8;
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 8; i += 2)
      w[i / 2] = (e & 1) ? pair_hi(pend[2 * i + h][e / 2], pend[2 * i + 2 + h][e / 2])
                         : pair_lo(pend[2 * i + h][e / 2], pend[2 * i + 2 + h][e / 2]);
    __builtin_amdgcn_raw_buffer_store_b128(w, pend_rd, pend_m, (unsigned int)(32 * h + e) * pend_ld, 0);
  };
  auto slice = [&](auto set_tag, auto zero_tag, auto drain_tag, auto b_tag, unsigned int dst) {
    constexpr int DR = decltype(drain_tag)::value;
    constexpr bool OPB = decltype(b_tag)::value;       // operand of the transfers
    constexpr int S = decltype(set_tag)::value;
    constexpr bool ZERO = decltype(zero_tag)::value;
#pragma unroll
    for (int n = 0; n < NM; ++n) {
      const int i = n / TJ, j = (i & 1) ? TJ - 1 - n % TJ : n % TJ;   // back and forth: one operand changes at a time
      if constexpr (!DEFER) {
        f32x4 c = acc[i][j];
        if constexpr (ZERO) c = f32x4{0.f, 0.f, 0.f, 0.f};
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, fb[S][j]), __builtin_bit_cast(bf16x8, fa[S][i]), c, 0, 0, 0);
        if (n % DSTEP == 1)
          dma_n(n / DSTEP, [&](auto it) { if constexpr (OPB) dma_b(it, dst); else dma_a(it, dst); });
      } else if (n % DSTEP == 1) {
        dma_n(n / DSTEP, [&](auto it) {
          mfma_dma<ZERO, decltype(it)::value * 4096>(acc[i][j], fb[S][j], fa[S][i], OPB ? rsB : rsA, OPB ? voffB : voffA,
                                                     OPB ? runB : runA, dst);
        });
      } else {
        mfma<ZERO>(acc[i][j], fb[S][j], fa[S][i]);
        if (n % DSTEP == 2) { if constexpr (OPB) next_b(n / DSTEP); else next_a(n / DSTEP); }
      }
#pragma unroll
      for (int r = 0; r < RPER; ++r)
        if (n % RSTEP == 0 && n / RSTEP * RPER + r < NR) read_one(1 - S, n / RSTEP * RPER + r);
      if constexpr (DR >= 0) {
        if (n == 12 && stored) drain(DR);
        if constexpr (!BKS)
          if (n % 32 == 28 && mirrored) drain_mirror(2 * DR + n / 32);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto wrap = [](unsigned int p) { return p >= RING ? p - RING : p; };

  TileCoord tc = decode(deal.at);
  aim(tc);
#pragma unroll
  for (int t = 0; t < D; ++t) {
    runA = soA;
    runB = soB;
#pragma unroll
    for (int it = 0; it < NCH; ++it) {
      dma_n(it, [&](auto n) { dma_a(n, lds_wave + (2 * t) * BUF); });
      dma_n(it, [&](auto n) { dma_b(n, lds_wave + (2 * t + 1) * BUF); });
    }
    soA += advA;
    soB += advB;
  }
  left -= D;
  // The first K tile alone has to be there now; the first step waits for the second.  (Waiting for
  // all D here cost products that are a few K tiles deep up to 5 %: one 1024 x 1024 matrix 137.4 us
  // instead of 134.8, six of 3001 x 1000 513 instead of 501.)
  wait_vmcnt<(D - 1) * 2 * NCH>();
  block_sync();
  unsigned int p = 0;                 // buffer of operand A of the current K tile

  using T = std::true_type;
  using F = std::false_type;
  // Transfers that may be in flight at a K tile's barrier, which publishes the next K tile: all
  // requested after it.
  constexpr int STEADY = (NB - 4) * NCH;
  // ---- a tile on the diagonal.  Rows and columns are the same, so operand B's buffer serves for both, and tile i of
  // rows holds what tile j = i of columns does.  Wavefronts 0 and 3 take the quarters on the diagonal (DG: ten of
  // their sixteen 32 x 32 blocks, from one set of fragments), 1 and 2 half of the lower left quarter each (128
  // rows, 64 columns): 40 and 32 MFMAs a slice instead of 64.  Leaving out the upper right quarter alone, with its
  // wavefront idle, gave 0.5 % of an inner step, this 1 to 4 %.
  // B's transfers go first: its buffer of two K tiles ahead is the one that A's of this K tile would fill.  A's, where
  // they go out (always towards a whole tile that follows), come in the second slice.  Either way a wait leaves
  // as many transfers in flight as in a whole tile, all of them behind what it awaits.
  // The last tile's left-over stores leave in four K tiles, and the K loop is unrolled by two: the
  // whole kernel stays within the reach of a branch.
  auto run_triangle = [&](auto tri_tag, const TileCoord& tn) {
    constexpr bool DG = decltype(tri_tag)::value;
    constexpr int MF = DG ? 40 : 32, NF = DG ? 8 : 12;        // MFMAs and fragments of a slice
    u32x4 ta[2][8], tb[2][8];
    bool rows_a = g.K > TRIANGLE_ONE_OPERAND;       // do operand A's transfers go out
    const unsigned int base = fragB[0] - (unsigned int)wbase_n * 128;
    auto point = [&](unsigned int bufB, int kk) {
      const unsigned int at = (base ^ (kk ? 64u : 0u)) + bufB;
      rb[0] = at + (DG ? (unsigned int)wbase_n * 128 : wave == 1 ? 4u * 2048 : 0u);
      ra = at + 128u * 128;
    };
    // in the order of their use
    auto read = [&](int set, int r) {
      if constexpr (DG) tb[set][r] = *reinterpret_cast<const u32x4*>(smem + rb[0] + r * 2048);
      else if (r == 0 || r > 4) ta[set][r == 0 ? 0 : r - 4] = *reinterpret_cast<const u32x4*>(smem + ra + (r == 0 ? 0 : r - 4) * 2048);
      else tb[set][r - 1] = *reinterpret_cast<const u32x4*>(smem + rb[0] + (r - 1) * 2048);
    };
    auto tri_slice = [&](auto set_tag, auto zero_tag, auto drain_tag, auto rows_tag, auto b_tag, unsigned int dst) {
      constexpr int DR = decltype(drain_tag)::value, ROWS = decltype(rows_tag)::value;       // rows that leave
      constexpr bool OPB = decltype(b_tag)::value;
      constexpr int S = decltype(set_tag)::value;
      constexpr bool ZERO = decltype(zero_tag)::value;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int m = i / 2, cols = DG ? 2 * m + 2 : 4;
        const int n0 = DG ? 2 * m * (m + 1) + (i & 1) * (2 * m + 2) : 4 * i;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          if (x >= cols) break;
          const int n = n0 + x, j = (i & 1) ? cols - 1 - x : x;
          const u32x4& a = DG ? tb[S][i] : ta[S][i];
          if (OPB && n % (MF / NCH) == 1) {
            dma_n(n / (MF / NCH), [&](auto it) {
              mfma_dma<ZERO, decltype(it)::value * 4096>(acc[i][j], tb[S][j], a, rsB, voffB, runB, dst);
            });
          } else {
            mfma<ZERO>(acc[i][j], tb[S][j], a);
            if (OPB && n % (MF / NCH) == 2) next_b(n / (MF / NCH));
            if (!OPB && n == 8 && rows_a)
#pragma unroll 1
              for (int it = 0; it < NCH; ++it) {
                dma16<0>(rsA, voffA, runA, dst + (unsigned int)it * 4096);
                next_a(it);
              }
          }
          if (n % 2 == 0 && n / 2 < NF) read(1 - S, n / 2);
          if constexpr (ROWS > 0) {
            if (n == 8 && stored) drain(DR);
            if (n == 18 && mirrored) drain_mirror(2 * DR);
            if (n == 21 && mirrored) drain_mirror(2 * DR + 1);
          }
          if constexpr (ROWS > 1) {
            if (n == 14 && stored) drain(DR + 1);
            if (n == 24 && mirrored) drain_mirror(2 * DR + 2);
            if (n == 27 && mirrored) drain_mirror(2 * DR + 3);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    point(wrap(p + BUF), 0);
#pragma unroll
    for (int r = 0; r < NF; ++r) read(0, r);
    auto tri_step = [&](auto first_tag, auto drain_tag, auto rows_tag) {
      if (left == 0) {
        aim(tn);
        rows_a = !tn.diag;
      }
      runA = soA;
      runB = soB;
      const unsigned int pb = wrap(p + BUF), pa1 = wrap(p + 2 * BUF), pb1 = wrap(p + 3 * BUF);
      const unsigned int free0 = lds_wave + (p == 0 ? RING - BUF : p - BUF), free1 = lds_wave + p;
      point(pb, 1);
      tri_slice(I<0>{}, first_tag, drain_tag, rows_tag, T{}, free1);
      constexpr int DR = 2 * decltype(rows_tag)::value;
      constexpr bool FIRST = decltype(first_tag)::value;
      if (FIRST && triangle) wait_vmcnt<STEADY + TRIANGLE_STORES>();
      else if (DR + FIRST == 0 || !stored) wait_vmcnt<STEADY>();
      else if (mirrored) wait_vmcnt<STEADY + 2 * DR + (FIRST ? epilogue_stores(TI, true) : 0)>();
      else wait_vmcnt<STEADY + DR + (FIRST ? epilogue_stores(TI, false) : 0)>();
      block_sync();
      point(pb1, 0);
      tri_slice(I<1>{}, F{}, I<0>{}, I<0>{}, F{}, free0);
      soA += advA;
      soB += advB;
      --left;
      p = pa1;
    };
    // (two rows a K tile; the number of K tiles is even)
    tri_step(T{}, I<0>{}, I<2>{});
    tri_step(F{}, I<2>{}, I<2>{});
    tri_step(F{}, I<4>{}, I<2>{});
    tri_step(F{}, I<6>{}, I<2>{});
    int t = 4;
    if (DG && KT > 4) {
      tri_step(F{}, I<0>{}, I<0>{});
      tri_step(F{}, I<0>{}, I<0>{});
      t = 6;
    }
#pragma unroll 1
    for (; t < KT; t += 2) {
      tri_step(F{}, I<0>{}, I<0>{});
      tri_step(F{}, I<0>{}, I<0>{});
    }
    triangle_settle<DG>(acc);
    float alpha = g.alpha;
    if (g.bscale) {
      const float sc = g.bscale[tc.b];
      alpha *= (g.bscale_pow == 2) ? sc * sc : sc;
    }
    const int row0 = tc.m0 + (DG ? wbase_n : 128), col0 = tc.n0 + (DG ? wbase_n : wave == 1 ? 64 : 0);
    store_triangle<DG>(g, acc, tc.b, row0, col0, alpha, tc.edge && wave != 3, lane);
  };

  while (true) {
    // The next output tile of this workgroup; after the last one the same requests go to this
    // tile's own first K tiles again (in bounds, never read).
    bool more;
    TileCoord tn;
    auto advance = [&] {
      deal.at += deal.step;
      if (deal.at >= deal.end) second();
      more = deal.at < deal.end;
      tn = more ? decode(deal.at) : tc;
    };
    if constexpr (TRI) {
      if (tc.diag) {
        advance();
        if (wave == 1 || wave == 2) run_triangle(F{}, tn);
        else run_triangle(T{}, tn);
        stored = mirrored = false;
        triangle = true;
        if (!more) break;
        tc = tn;
        continue;
      }
    }
    point_at(p, wrap(p + BUF), 0);
#pragma unroll
    for (int r = 0; r < NR; ++r) read_one(0, r);
    advance();
    auto step = [&](auto first_tag, auto drain_tag) {
      if (left == 0) aim(tn);
      runA = soA;
      runB = soB;
      const unsigned int pb = wrap(p + BUF), pa1 = wrap(p + 2 * BUF), pb1 = wrap(p + 3 * BUF);
      const unsigned int free0 = lds_wave + (p == 0 ? RING - BUF : p - BUF), free1 = lds_wave + p;
      point_at(p, pb, 1);
      slice(I<0>{}, first_tag, drain_tag, F{}, free0);
      // in flight behind what has to be there now: this slice's transfers and stores and, on the first
      // K tile, the last epilogue's stores
      constexpr int DR = decltype(drain_tag)::value >= 0 ? 2 : 0;
      constexpr bool FIRST = decltype(first_tag)::value;
      if (TRI && FIRST && triangle) wait_vmcnt<STEADY + TRIANGLE_STORES>();
      else if (DR + FIRST == 0 || !stored) wait_vmcnt<STEADY>();
      else if (!BKS && mirrored) wait_vmcnt<STEADY + 2 * DR + (FIRST ? epilogue_stores(TI, true) : 0)>();
      else wait_vmcnt<STEADY + DR + (FIRST ? epilogue_stores(TI, false) : 0)>();
      block_sync();
      point_at(pa1, pb1, 0);
      slice(I<1>{}, F{}, I<-1>{}, T{}, free1);
      soA += advA;
      soB += advB;
      --left;
      p = pa1;
    };
    if constexpr (DEFER) {
      step(T{}, I<0>{});
      step(F{}, I<1>{});
      step(F{}, I<2>{});
      step(F{}, I<3>{});
      if (KT >= 8) {
        step(F{}, I<4>{});
        step(F{}, I<5>{});
        step(F{}, I<6>{});
        step(F{}, I<7>{});
      } else if (stored) {
#pragma unroll
        for (int i = 4; i < 8; ++i) drain(i);
        if (!BKS && mirrored)
#pragma unroll
          for (int q = 8; q < 16; ++q) drain_mirror(q);
      }
#pragma unroll 1
      for (int t = KT >= 8 ? 8 : 4; t < KT; ++t) step(F{}, I<-1>{});
    } else {
      step(T{}, I<-1>{});
#pragma unroll 1
      for (int t = 1; t < KT; ++t) step(F{}, I<-1>{});
    }

    if constexpr (DEFER) acc_settle(acc);
    // what a neighbouring tile computes too is left to it: beyond the reach of a buffer stores are dropped
    const bool drop = ((tc.edge & 1) && wbase_m == 0) || ((tc.edge & 2) && wbase_n == 0);
    float alpha = g.alpha;
    if (g.bscale) {
      const float sc = g.bscale[tc.b];
      alpha *= (g.bscale_pow == 2) ? sc * sc : sc;
    }
#define MLC_STORE(C, M, T, DG, U) \
  store_tile<TI, TJ, WT ? SC1 : 0, C, M, T, DG, U>(g, acc, tc, alpha, wbase_m, wbase_n, lane, drop, pend)
    // Symmetric products (Gram, polynomial) are those with a K-contiguous B, the apply products
    // those with a K-strided one: each kernel holds only the forms its products have.
    if constexpr (!BKS) {
      if (!TRI && !tc.mirror) {
        if (g.C) MLC_STORE(true, false, false, true, false);
        else MLC_STORE(false, false, false, true, false);
      } else if (g.C) {
        MLC_STORE(true, true, false, false, false);
      } else if (alpha == 1.f) {
        MLC_STORE(false, true, false, false, true);
      } else {
        MLC_STORE(false, true, false, false, false);
      }
    } else if (g.transposed) {
      if (g.C) MLC_STORE(true, false, true, false, false);
      else MLC_STORE(false, false, true, false, false);
    } else if (g.C) {
      MLC_STORE(true, false, false, false, false);
    } else if (alpha == 1.f) {
      MLC_STORE(false, false, false, false, true);
    } else {
      MLC_STORE(false, false, false, false, false);
    }
#undef MLC_STORE
    stored = true;
    triangle = false;
    mirrored = tc.mirror;
    if constexpr (DEFER) {
      pend_rd = __builtin_amdgcn_make_buffer_rsrc(g.D + (long)tc.b * g.strideD, 0, BUFFER_END, 0x00020000);
      int l = lane;
      asm volatile("" : "+v"(l));
      const int row0 = tc.m0 + wbase_m + TI * (l & 15), col0 = tc.n0 + wbase_n + 8 * (l >> 4);
      pend_ld = (unsigned int)(g.ldd * 2);
      pend_m = (unsigned int)(((long)(col0 + 64) * g.ldd + row0) * 2);
      const int o = l & 1;
      if (drop) pend_m = BUFFER_END;
      pend_n = drop || (BKS && g.transposed) ? pend_m : (unsigned int)(((long)(row0 - TI * o) * g.ldd + col0 + 64 + 32 * o) * 2);
    }
    if (!more) break;
    tc = tn;
  }
  if constexpr (DEFER) {
    if (stored)
#pragma unroll
      for (int i = 0; i < 8; ++i) drain(i);
    if (!BKS && mirrored)
#pragma unroll
      for (int q = 0; q < 16; ++q) drain_mirror(q);
  }
  // nothing may land in the ring after this workgroup has left it
  __builtin_amdgcn_s_waitcnt(0x0f70);
  block_sync();
}

// Up to MAX_MULTI products in one launch (the same product of a Newton-Schulz iteration for several
// shape groups), the deepest first.  A launch whose tile count is not a multiple of the number of
// compute units pays for a partly empty last round; sharing a launch leaves one such round instead
// of one per group.  XCD x still owns a contiguous range of every product's tile order; inside it
// each product of one depth starts with the workgroup after the one that took the previous product's last
// tile, and so do small tiles of any depth; deal_tiles evens out the time of large tiles of different depths.  (Gram products of 16 x 1024 x 2816, 0.6
// rounds, and 32 x 1024 x 1024, 1.25: 135 us in two launches, 100 in one; of a 15B-scale layer 1350
// and 1240.  Launches apart cost about 7 us each beside what their rounds cost.)
constexpr int MAX_MULTI = 3;
struct MultiArgs { GemmArgs seg[MAX_MULTI]; int nseg, mixed; };

template <int BM, int BN, bool BKS, int NB, bool WT>
__global__ __launch_bounds__(NTHREADS, 1) void ns_gemm_bf16_kernel(MultiArgs m) {
  const int xcd = blockIdx.x % NUM_XCD, slot = blockIdx.x / NUM_XCD;
  const int W = (int)(gridDim.x / NUM_XCD);
  int first = 0;                       // of equal depth: the workgroup whose turn it is
  // Of different depth.  Small tiles are dealt as if of equal depth: the arithmetic alone, whether used or not, makes each of their
  // launches 0.8 us longer (of about 4 to 8).
  Dealer dealer{W, slot, 0, 0};
#pragma unroll 1
  for (int j = 0; j < m.nseg; ++j) {
    const GemmArgs g = m.seg[j];
    const int lo = min(xcd * g.tiles_per_xcd, g.total_tiles);
    const int hi = min((xcd + 1) * g.tiles_per_xcd, g.total_tiles);
    const bool more = j + 1 < m.nseg;
    Deal deal;
    if (BM == 256 && m.mixed) {
      deal = deal_tiles(dealer, lo, hi - lo, g.K / BK + 3, more);
    } else {
      const int pos = slot - first;
      deal = Deal{lo + (pos < 0 ? pos + W : pos), hi, W, hi, hi, W};
      if (more) first = (int)((unsigned)(first + hi - lo) % (unsigned)W);
    }
    run_tiles<BM, BN, BKS, NB, WT>(g, deal);
    // the next product's first transfers overwrite the ring: every wavefront must have left it
    __syncthreads();
  }
}

// Compute units behind one L2 (one XCD) of the current device.
int cus_per_xcd(int slot) {
  static std::atomic<int> cached[MAX_DEVICES];
  if (slot >= 0) {
    const int c = cached[slot].load(std::memory_order_relaxed);
    if (c > 0) return c;
  }
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < NUM_XCD)
    cus = 256;
  if (slot >= 0) cached[slot].store(cus / NUM_XCD, std::memory_order_relaxed);
  return cus / NUM_XCD;
}

// Kernel arguments of one product with BM x BN tiles.  Tiles cover M x N; the last row and column of 256 x 256 tiles may
// begin half a tile before the end of those before them.
template <int BM, int BN>
int make_args(const GemmDesc& d, GemmArgs& g) {
  g.A = d.A; g.lda = d.lda; g.strideA = d.strideA;
  g.B = d.B; g.ldb = d.ldb; g.strideB = d.strideB;
  g.D = d.D; g.ldd = d.ldd; g.strideD = d.strideD;
  g.C = d.C; g.ldc = d.ldc; g.strideC = d.strideC;
  g.K = d.K; g.batch = d.batch;
  g.tiles_m = (d.M + BM - 1) / BM; g.tiles_n = (d.N + BN - 1) / BN;
  g.last_m = d.M - BM; g.last_n = d.N - BN;
  if (g.last_m < 0 || g.last_n < 0) return MLC_ERR_SHAPE;
  g.symmetric = d.symmetric ? 1 : 0;
  g.transposed = d.transposed ? 1 : 0;
  {   // equal groups of at most GROUP_M tile rows (10 rows -> 5 + 5, not 8 + 2)
    const int ngroups = (g.tiles_m + GROUP_M - 1) / GROUP_M;
    g.group_m = (g.tiles_m + ngroups - 1) / ngroups;
  }
  if (g.symmetric && (BM != BN || d.M != d.N || g.transposed)) return MLC_ERR_SHAPE;
  // the forms the kernels hold: symmetric results from K-contiguous operands, others from a
  // K-strided B, the identity only on symmetric ones
  if ((g.symmetric != 0) == (d.b_kstrided != 0) || (!g.symmetric && d.gamma != 0.f)) return MLC_ERR_UNSUPPORTED;
  g.tiles_per_mat = g.symmetric ? g.tiles_m * (g.tiles_m + 1) / 2 : g.tiles_m * g.tiles_n;
  const long total = (long)g.tiles_per_mat * d.batch;
  if (total <= 0 || total > (1L << 30)) return MLC_ERR_SHAPE;
  g.total_tiles = (int)total;
  g.tiles_per_xcd = (int)((total + NUM_XCD - 1) / NUM_XCD);
  g.alpha = d.alpha; g.beta = d.beta; g.gamma = d.gamma;
  g.bscale = d.bscale; g.bscale_pow = d.bscale_pow;
  return MLC_OK;
}

// The LDS limit of a kernel is raised once per instantiation and device (the call is
// idempotent, so a race between two host threads only repeats it).
template <typename Kern>
int raise_lds_limit(Kern kern, std::atomic<bool>* done, int slot, size_t lds) {
  if (slot < 0 || !done[slot].load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return MLC_ERR_LAUNCH;
    if (slot >= 0) done[slot].store(true, std::memory_order_release);
  }
  return MLC_OK;
}

bool valid_desc(const GemmDesc& d) {
  if (d.M % 128 || d.N % 128 || d.K % 128 || d.M <= 0 || d.N <= 0 || d.K <= 0 || d.batch <= 0) return false;
  if ((d.lda | d.ldb | d.ldd | d.strideA | d.strideB | d.strideD) % 8) return false;
  if (d.C && ((d.ldc | d.strideC) % 8)) return false;
  return true;
}

// n (1 .. MAX_MULTI) products of one layout in one launch, in descending order of depth.
template <int BM, int BN, bool BKS, int NB, bool WT>
int launch_cfg(const GemmDesc* const* d, int n, hipStream_t stream) {
  MultiArgs m;
  m.nseg = n;
  m.mixed = d[0]->K != d[n - 1]->K;
  // Every launch asks for the whole LDS of a CU, however small its ring, so that its workgroups
  // share a CU with no other workgroup that holds LDS, neither of this kernel nor of one that runs on
  // another stream: an earlier 128 x 128 kernel gave wrong tiles when two of its workgroups were on
  // one CU, and why is not known.  (Not the LDS address of the transfers: `buffer_load ... lds`
  // lands where it should in allocations of 20, 40 and 80 KiB that do not start at 0, measured on
  // 5600 such workgroups.)  The schedule wants one workgroup per CU anyway.
  const int slot = device_slot();
  int W = cus_per_xcd(slot);
  double flops = 0.0;
  int most = 0;
  for (int j = 0; j < MAX_MULTI; ++j) {
    const GemmDesc& dj = *d[j < n ? j : 0];
    const int rc = make_args<BM, BN>(dj, m.seg[j]);
    if (rc != MLC_OK) return rc;
    if (j >= n) continue;
    // executed, not nominal: whole output tiles, and 144 of 256 MFMAs of a 256 x 256 tile on the diagonal
    const double diagonal = BM == 256 && !BKS ? (double)m.seg[j].tiles_m * m.seg[j].batch : 0.0;
    flops += 2.0 * BM * BN * (double)dj.K * ((double)m.seg[j].total_tiles - diagonal * 112 / 256);
    most += m.seg[j].tiles_per_xcd;
  }
  if (most < W) W = most;    // fewer tiles than compute units
  static_assert((size_t)NB * BM * BK * 2 <= CU_LDS, "the ring fits a CU");
  auto kern = ns_gemm_bf16_kernel<BM, BN, BKS, NB, WT>;
  static std::atomic<bool> attr_set[MAX_DEVICES];
  const int rc = raise_lds_limit(kern, attr_set, slot, CU_LDS);
  if (rc != MLC_OK) return rc;
  LaunchScope scope(MLC_KERNEL_NS_GEMM, stream, flops, 0.0);
  hipLaunchKernelGGL(kern, dim3(W * NUM_XCD), dim3(NTHREADS), CU_LDS, stream, m);
  return hipGetLastError() == hipSuccess ? MLC_OK : MLC_ERR_LAUNCH;
}

// Can the 256 x 256 tile serve this product?  A side that it does not divide ends with half a tile that two tile rows
// (columns) compute; below 896 that is more than a seventh of the work.  All products in that tile against all in the smaller
// ones, newton_schulz: 192 of 896 x 896 4440 -> 3606 us, 63 of 1664 x 1664 7353 -> 5721, 18 of 3200 x 3200 13650 -> 9900;
// but 63 of 640 x 640 520 -> 700, 70 of 384 x 1536 440 -> 565, 341 of 640 x 640 3266 -> 2955.
bool large_fits(const GemmDesc& d) {
  return d.M >= 256 && d.N >= 256 && (d.M % 256 == 0 || d.M >= 896) && (d.N % 256 == 0 || d.N >= 896);
}

long tiles_of(const GemmDesc& d, int tile) {
  const long tm = (d.M + tile - 1) / tile, tn = (d.N + tile - 1) / tile;
  return (d.symmetric ? tm * (tm + 1) / 2 : tm * tn) * d.batch;
}

// Microseconds that a launch of `tiles` output tiles of kt K tiles takes: a first round of one tile per
// compute unit, and further ones that overlap its ends.  The 256 x 256 tile runs faster in a round that
// leaves compute units idle (the chip is power-limited).  Symmetric results pay for the transposed
// copy, the polynomial for its C operand too.  Fitted to kernel traces of earlier forms of all three tiles, with longer
// epilogues, no triangles on the diagonal, no half tiles at the edge and no results written through: over 194 batches (1 to
// 200 matrices of 128 to 2048, K to 4096) in each tile that fits, nine in ten launches now take 0.82 to 1.01 of this with 256 x 256
// tiles, 0.83 to 1.17 with 128 x 128 and 0.82 to 1.19 with 64 x 64, the medians 0.94, 0.92 and 0.95.
enum { FORM_GRAM, FORM_POLY, FORM_APPLY };
int form_of(const GemmDesc& d) { return !d.symmetric ? FORM_APPLY : d.C ? FORM_POLY : FORM_GRAM; }
double estimate_us(int tile, int form, long tiles, int kt, int cus) {
  const long full = tiles / cus, rest = tiles - full * cus;
  if (tile == 256) {
    constexpr double E[3] = {8.7, 14.8, 6.9}, R[3] = {4.8, 8.9, 4.4}, F[3] = {3.3, 7.3, 3.2};
    const double f = (double)rest / cus;
    return 3.5 + full * (kt * 1.40 + E[form]) + (rest ? kt * (1.02 + 0.38 * f) + R[form] + F[form] * f : 0.0);
  }
  struct Fit { double base, first, more, epi; };
  constexpr Fit F128[3] = {{5.8, 0.38, 0.47, 3.1}, {5.1, 0.50, 0.39, 4.1}, {5.1, 0.45, 0.44, 2.5}};
  constexpr Fit F64[3] = {{5.0, 0.18, 0.19, 1.2}, {4.8, 0.21, 0.18, 1.3}, {4.8, 0.22, 0.16, 1.3}};
  const Fit& x = tile == 128 ? F128[form] : F64[form];
  return x.base + x.first * kt + (double)(full + (rest ? 1 : 0) - 1) * (x.more * kt + x.epi);
}

// The tile for a launch of these products.  One large tile moves half the operand bytes per FLOP
// of a 128 x 128 one (20 of 2048 x 2048: 1.2 to 1.3 against 0.84 to 0.89 PFLOP/s), but products with few
// tiles leave most of the chip idle: one 1024 x 1024 matrix takes 26 us a product in 16 tiles of
// 256, 12 in 64 of 128, 8 in 256 of 64; 200 of 256 x 256 take 15 / 18 / 18 in tiles of 256 and
// 14 / 16 / 17 in tiles of 128.  A smaller tile has to be ahead by 5 %, and by 15 % over operands of
// more than 64 MB, of which X, its next iterate, A and B' fill the 256 MB memory-side cache: the operand
// bytes then decide (Gram products of 32 x 1024 x 1024, alone 56 us in tiles of 256 and 52 in tiles of
// 128, took 62 and 68 beside 16 of 1024 x 2816, with earlier epilogues).  Over those 194 batches the choice takes
// 1.007 of the time of the best tile for each; one launch in thirteen is over 1.03, the worst (polynomial of 148 x 1152 x
// 1152, whose half tiles the 256 x 256 tile would do faster) 1.25.  The tile is chosen before it is known whether sets of different depth will share a launch.  The 64 x 64
// tile's ring needs four K tiles.
int pick_tile(const GemmDesc* const* d, int n, int cus) {
  long tiles[3] = {0, 0, 0};
  bool large = true;
  double bytes = 0.0;
  for (int j = 0; j < n; ++j) {
    bytes += 2.0 * d[j]->batch * d[j]->K * (d[j]->M + (d[j]->symmetric ? 0.0 : (double)d[j]->N));
    large = large && large_fits(*d[j]);
    for (int t = 0; t < 3; ++t) tiles[t] += tiles_of(*d[j], 256 >> t);
  }
  const int kt = d[0]->K / BK;
  const int form = form_of(*d[0]);
  int small = 128;
  double us = estimate_us(128, form, tiles[1], kt, cus);
  const double e64 = estimate_us(64, form, tiles[2], kt, cus);
  if (kt >= 4 && e64 < 0.95 * us) { small = 64; us = e64; }
  if (!large || kt < 4) return small;        // the large tile leaves stores for its first four K tiles
  return us < (bytes > 64e6 ? 0.85 : 0.95) * estimate_us(256, form, tiles[0], kt, cus) ? small : 256;
}

// Products of one layout, at first of one depth, and the kernel that they run in.
struct GemmSet { const GemmDesc* d[MAX_MULTI]; int n, tile, ring; };

long tiles_in(const GemmSet& s, int tile) {
  long tiles = 0;
  for (int j = 0; j < s.n; ++j) tiles += tiles_of(*s.d[j], tile);
  return tiles;
}
double set_us(const GemmSet& s, int cus) {
  return estimate_us(s.tile, form_of(*s.d[0]), tiles_in(s, s.tile), s.d[0]->K / BK, cus);
}

// Do set t's products go out with those of set s, which are as deep or deeper?  If so s is left with the kernel for both.  Large
// tiles always do (a tile that is small because there are few of them stays apart from them: its launch is shorter than a large
// tile).  Small ones do where their results are of one size (a layer's square and rectangular matrices: Gram products) or the
// depth is the same, and where the two leave much of the chip idle: together less than 1.75 rounds (1.5 of 64 x 64 tiles), or one
// of them at most three quarters (half) of one; others keep launches of their own.  Sets that run different small tiles take one
// if that makes one round of all and the estimate is lower.  A launch costs 2.7 us however little it does, its first transfers and
// last stores as much again, and a partly empty round more: inner steps of three groups, 4 c of d x d, c of d x f and f x d, with sets
// of different depth and divisors apart and together (6 to 10 us of it are launches of elementwise kernels): 4, 256 / 1000: 151 -> 119 us;
// 2, 303 / 640: 179 -> 146; 1, 512 / 1536: 167 -> 133; 4, 768 / 2449: 645 -> 577; 3, 896 / 2944: 725 -> 645; 10, 512 / 640: 481 -> 465.
// The bounds on rounds are not sharp: over 110 steps of two and three groups, 256 to 1280 wide, sets of one tile take 0.93 of their time
// apart (0.83 to 1.00), and with every such pair together 0.98 to 1.01 of that.  Which launches they give is in the tests' sizes.
bool join_sets(GemmSet& s, const GemmSet& t, int cus) {
  if (s.n + t.n > MAX_MULTI || (t.d[0]->b_kstrided != 0) != (s.d[0]->b_kstrided != 0)) return false;
  if (s.tile == 256 || t.tile == 256) return s.tile == t.tile;
  int tile = s.tile;
  const int64_t deep = s.d[0]->K, shallow = t.d[0]->K;
  if (s.tile == t.tile) {
    const long a = tiles_in(s, tile), b = tiles_in(t, tile);
    const int quarters = tile == 64 ? 2 : 3;
    if (deep != shallow && s.d[0]->M != t.d[0]->M && (a + b) * 4 > (quarters + 4L) * cus && std::min(a, b) * 4 > quarters * cus)
      return false;
  } else {
    double us = set_us(s, cus) + set_us(t, cus);
    tile = 0;
    for (int x = 128; x >= 64; x /= 2) {
      const long tiles = tiles_in(s, x) + tiles_in(t, x);
      if (tiles > cus || (x == 64 && shallow < 4 * BK)) continue;
      const double e = estimate_us(x, form_of(*s.d[0]), tiles, (int)(deep / BK), cus);
      if (e < us) { us = e; tile = x; }
    }
    if (!tile) return false;
  }
  const bool nine = tile == 64 || deep > 640 || (s.tile == 128 && s.ring == 9) || (t.tile == 128 && t.ring == 9);
  if (nine && shallow < 4 * BK) return false;       // the long ring needs four K tiles
  s.tile = tile;
  s.ring = nine ? 9 : 5;
  return true;
}

void choose_kernel(GemmSet& s) {
  const int cus = cus_per_xcd(device_slot()) * NUM_XCD;
  s.tile = pick_tile(s.d, s.n, cus);
  s.ring = s.tile == 64 ? 9 : 5;
  if (s.tile != 128) return;
  // The small tiles leave room for a ring of nine buffers, four K tiles ahead.  Up to ten K tiles
  // two are better while a launch is short: a wavefront has requested all that its ring holds ahead
  // before its first MFMA, and a CU takes 64 bytes a cycle (15 products of 32 / 64 matrices of
  // 256 x 256: 113 / 126 us instead of 120 / 135, of 8 / 16 of 640 x 640 152 / 208 instead of 157 / 211).
  // Where workgroups take more than two tiles the longer ring is ahead again from six K tiles on
  // (400 matrices of 384 x 384: 1273 us, with the short one 1320; 96 of 640 x 640 977, 1022), and with
  // four from about eight tiles on (400 of 256 x 256 491, short 481; 101 of 2088 x 178 623, short 638).
  long tiles = 0;
  for (int j = 0; j < s.n; ++j) tiles += tiles_of(*s.d[j], 128);
  const int64_t K = s.d[0]->K;
  if (!(K < 256 || tiles <= (K == 256 ? 8 : K <= 640 ? 2 : 0) * cus)) s.ring = 9;
}

// The small tiles' results are written through to memory.  Their launches are short, and one ends only when the L2s
// have written back what it left in them: inner steps of 12 x 401 x 401 and two groups of 3 beside it 190 -> 178 us, of
// 24 x 512 x 512 and 6 346 -> 333, newton_schulz of 6 of 3001 x 1000 434 -> 421.  Of a few 64 x 64 tiles nothing is left to wait for
// (a 256 x 256 matrix, ten and sixteen tiles: 73 to 76 us, written through 77 to 78; a 512 x 512 one, 36 and 64, alike).  In long
// launches of large tiles it is worth nothing, in short ones it costs 1 %.
constexpr long THROUGH_TILES = 64;
template <bool BKS>
int launch_set(const GemmSet& s, hipStream_t stream) {
  if (s.tile == 256) return launch_cfg<256, 256, BKS, 5, false>(s.d, s.n, stream);
  if (s.tile == 64) {
    if (tiles_in(s, 64) < THROUGH_TILES) return launch_cfg<64, 64, BKS, 9, false>(s.d, s.n, stream);
    return launch_cfg<64, 64, BKS, 9, true>(s.d, s.n, stream);
  }
  if (s.ring == 5) return launch_cfg<128, 128, BKS, 5, true>(s.d, s.n, stream);
  return launch_cfg<128, 128, BKS, 9, true>(s.d, s.n, stream);
}

}  // namespace

int launch_ns_gemm_set(const GemmDesc* d, int n, hipStream_t stream) {
  if (n < 0 || n > 64) return MLC_ERR_ARG;
  bool done[64] = {};
  for (int i = 0; i < n; ++i)
    if (!valid_desc(d[i])) return MLC_ERR_SHAPE;
  const int cus = cus_per_xcd(device_slot()) * NUM_XCD;
  GemmSet sets[64];
  int n_sets = 0;
  for (int i = 0; i < n; ++i) {
    if (done[i]) continue;
    // products that share a launch with product i whatever their tile: same depth (a whole tile then takes the
    // same time in each, so dealing tiles out evenly balances the time but for triangles, which take 0.7 to 0.9 of
    // it), both fit for the large tile or neither, same layout
    GemmSet& s = sets[n_sets++];
    s.n = 0;
    for (int j = i; j < n && s.n < MAX_MULTI; ++j) {
      if (done[j] || d[j].K != d[i].K || large_fits(d[j]) != large_fits(d[i]) ||
          (d[j].b_kstrided != 0) != (d[i].b_kstrided != 0))
        continue;
      s.d[s.n++] = &d[j];
      done[j] = true;
    }
    choose_kernel(s);
  }
  // Sets share launches as well, the deeper ones first
  std::stable_sort(sets, sets + n_sets, [](const GemmSet& a, const GemmSet& b) { return a.d[0]->K > b.d[0]->K; });
  for (int i = 0; i < n_sets; ++i) {
    GemmSet& s = sets[i];
    if (s.n == 0) continue;            // went out with an earlier one
    for (int j = i + 1; j < n_sets; ++j) {
      GemmSet& t = sets[j];
      if (t.n == 0 || !join_sets(s, t, cus)) continue;
      for (int k = 0; k < t.n; ++k) s.d[s.n++] = t.d[k];
      t.n = 0;
    }
    const int rc = s.d[0]->b_kstrided ? launch_set<true>(s, stream) : launch_set<false>(s, stream);
    if (rc != MLC_OK) return rc;
  }
  return MLC_OK;
}

}  // namespace mlc
