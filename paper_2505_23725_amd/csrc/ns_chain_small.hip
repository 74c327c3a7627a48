// Whole Newton-Schulz chain of a small matrix inside one workgroup (paper Sec. 2 "Muon":
// the quintic iteration X <- a X + b (X X^T) X + c (X X^T)^2 X, run `iters` times).
//
// For matrices whose short side pads to 128 and whose long side pads to at most 512 the
// fifteen products of the five iterations are far too small to fill the chip one launch at
// a time: their cost is launch latency and the round trips of X, A and B' through memory.
// Here one workgroup (256 threads, 4 wavefronts) owns one matrix of the batch and keeps
// X (128 x L, bf16) and the 128 x 128 matrix A = X X^T, later B' = a I + b A + c A^2, in LDS
// from the first iteration to the last; HBM is touched once to read X and once to write it.
// The arithmetic and its rounding points are those of the batched path: A, B' and X are
// rounded to bf16 where that path stores them, products accumulate in fp32 on
// v_mfma_f32_16x16x32_bf16, the normalisation s = 1/(|U| + eps) enters as a factor s^2 of the
// first Gram matrix and s of the first product with X.  The kernel forms s itself from the
// partial sums of squares that the pass which wrote U left per matrix.
//
// A tall matrix (more rows than columns) is held transposed, so that the resident X is
// always 128 x L with L >= 128: the iteration commutes with transposition.
//
// LDS layout: X is [128][LP] bf16 (LP = 128, 256 or 512), A is [128][128] bf16 behind it;
// with LP = 512 that is all 160 KiB of a CU.  The 16-byte chunks of a row are swizzled within
// aligned groups of 16 (row_swizzle).
#include <atomic>
#include <type_traits>

#include "common.h"

namespace mlc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
namespace {

constexpr int S = 128;                 // padded short side
constexpr int A_PITCH = S * 2;         // bytes per row of A

constexpr int64_t CHAIN_SHARE_MAX = 256;     // compute units of the chip
struct ChainArgs {
  const bf16_t* in;        // [batch] matrices, row pitch ld, batch stride `stride` (elements)
  bf16_t* out;             // row pitch ldo, batch stride strideo
  long ld, stride, ldo, strideo;
  int tall;                // 0: matrix is 128 x L in memory ; 1: L x 128
  int L;                   // padded long side, a multiple of 128, <= LP
  const float* partials;   // per matrix nblk partial sums of squares of the input
  int nblk;
  float eps;               // scale = 1 / (sqrt(sum) + eps)
  int iters;               // >= 1
  float a, b, c;
};

// the low (high) 16-bit halves of x and y, x in the low half
__device__ __forceinline__ unsigned int halves_lo(unsigned int x, unsigned int y) {
  return __builtin_amdgcn_perm(y, x, 0x05040100u);
}
__device__ __forceinline__ unsigned int halves_hi(unsigned int x, unsigned int y) {
  return __builtin_amdgcn_perm(y, x, 0x07060302u);
}

// Byte offset of 16-byte chunk `chunk` of row r in a matrix of `pitch` bytes (a multiple of 256) per
// row.  The LDS serves a 128-bit read 16 lanes at a time over 256 bytes, so the 16 rows of a
// fragment's k chunk must meet 16 different positions: rows 16 i + idx, and rows 32 J + 8 (idx / 4) + 4 p
// + idx % 4.  A transposing read takes 4 chunks of each of 4 consecutive rows: the row's lowest two
// bits therefore choose among groups of four chunks.  The function is linear in the bits of r, so a
// lane's part of an address is computed once and the rest is an exclusive or with a constant.
__device__ __forceinline__ int row_swizzle(int r) {
  return ((r & 3) << 2) ^ ((((r >> 2) ^ (r >> 4)) & 1) << 1) ^ (3 * ((r >> 3) & 1));
}
__device__ __forceinline__ int chunk_pos(int r, int chunk, int pitch) { return r * pitch + ((chunk ^ row_swizzle(r)) << 4); }
constexpr int SWZ_ROW4 = 32;      // what bit 2 (or 4) of the row does to a position

// acc = b a (+ acc).  Inline assembly keeps the accumulators where they are (left to choose, the
// compiler copies them between slices, with wait states around every copy); it then does not know of
// the MFMAs' latency, so `settle` stands between the last of them and the first acc_read.
template <bool ZERO>
__device__ __forceinline__ void mfma(f32x4& acc, const u32x4& b, const u32x4& a) {
  if constexpr (ZERO) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc) : "v"(b), "v"(a));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}
template <int M, int N>
__device__ __forceinline__ void settle(f32x4 (&acc)[M][N]) {
  asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
  // nothing may read an accumulator's value from before the wait
#pragma unroll
  for (int n = 0; n < M * N; ++n) asm volatile("" : "+a"(acc[n / N][n % N]));
}
// of a part of a symmetric product (DG: on the diagonal)
template <bool DG>
__device__ __forceinline__ void settle_part(f32x4 (&acc)[4][4]) {
  asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < (DG ? 2 * (i / 2) + 2 : 2); ++j) asm volatile("" : "+a"(acc[i][j]));
}
__device__ __forceinline__ f32x4 acc_read(f32x4 a) {
  asm volatile("" : "+v"(a));
  return a;
}

// Fragments and results.  Operand order is swapped, so a lane (idx = lane % 16, lg = lane / 16) holds, in
// accumulator tiles 2 J and 2 J + 1 of a row, columns 32 J + 8 lg .. + 7 (tile j's fragment has column
// 32 (j / 2) + 8 (idx / 4) + 4 (j % 2) + idx % 4 in lane idx): results leave as 16-byte LDS writes.  Rows
// go the same way in the products of a matrix with its own transpose, so that a wavefront on the
// diagonal reads its fragments once for both operands; B' X has row 16 i + idx in tile i.
// Lane parts of the addresses: `row` + (chunk byte ^ `x`) is the position of k chunk lg of row idx (or
// of tile 0's column); tile i is 16 i rows further, and the chunk byte of k chunk 4 c is 64 c.
struct LanePos { int row, x; };
__device__ __forceinline__ LanePos lane_rows(int pitch, int row0, int idx, int lg) {
  return LanePos{(row0 + idx) * pitch, (row_swizzle(idx) ^ lg) << 4};
}
__device__ __forceinline__ LanePos lane_cols(int pitch, int row0, int idx, int lg) {
  const int r = 8 * (idx >> 2) + (idx & 3);
  return LanePos{(row0 + r) * pitch, (row_swizzle(r) ^ lg) << 4};
}
__device__ __forceinline__ u32x4 frag_row(const unsigned char* m, int pitch, const LanePos& p, int i, int at) {
  return *reinterpret_cast<const u32x4*>(m + p.row + (p.x ^ at ^ ((i & 1) * SWZ_ROW4)) + 16 * i * pitch);
}
__device__ __forceinline__ u32x4 frag_col(const unsigned char* m, int pitch, const LanePos& p, int j, int at) {
  return *reinterpret_cast<const u32x4*>(m + p.row + (p.x ^ at ^ ((j & 1) * SWZ_ROW4)) + (32 * (j >> 1) + 4 * (j & 1)) * pitch);
}
// K-strided fragment of rows 32 sl + 8 lg .. + 7, two transposing reads of 4; `at`: byte of column block 0
__device__ __forceinline__ LanePos lane_strided(int pitch, int idx, int lg, int at) {
  const int k = 8 * lg + (idx >> 2);
  return LanePos{k * pitch, ((row_swizzle(k) ^ (idx & 3)) << 4) ^ at};
}
__device__ __forceinline__ u32x4 frag_tr(const unsigned char* m, int pitch, const LanePos& p, int j, int sl) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  u32x4 v;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int pos = p.row + (p.x ^ (64 * (j >> 1)) ^ (h * SWZ_ROW4)) + (32 * sl + 4 * h) * pitch + 8 * (j & 1);
    const u32x2 w = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)((lds_byte*)m + pos)));
    v[2 * h] = w.x;
    v[2 * h + 1] = w.y;
  }
  return v;
}
__device__ __forceinline__ u32x4 pack8(const f32x4& x, const f32x4& y) {
  u32x4 w;
  w.x = pack_bf16x2(x[0], x[1]); w.y = pack_bf16x2(x[2], x[3]);
  w.z = pack_bf16x2(y[0], y[1]); w.w = pack_bf16x2(y[2], y[3]);
  return w;
}

// The whole chain of matrix `mat` of a batch, by one workgroup.
//
// Bound by what cannot overlap in one wavefront per SIMD: a phase's conversions and its barriers.  The Gram matrix and the square are
// symmetric, and only blocks on and below their diagonals are computed, 12 or 8 MFMAs a slice instead of 16, with 20 KB of fragments instead
// of 24.  (Cycles of an iteration on 128 x 512 before that: Gram 5200, its result 900, square 1750, polynomial 2400, product with
// X 4900, its result 3000; MFMAs 4100, 1000 and 4100.)  An iteration took 7.5 us and takes 7.1 (128 x 256: 5.2 and 4.9; 128 x 128:
// 3.96 and 3.88, and with more matrices than compute units 5.6 and 5.3), the launch around five of them 7.1 us (128 x 128: 4.6): fragments are
// read ahead of their use, K-strided ones with the transposing read, and all loads of X are in flight at once.
template <int TT>
__device__ __forceinline__ void ns_chain_body(const ChainArgs& g, long mat) {
  constexpr int LP = 128 * TT;
  constexpr int X_PITCH = LP * 2;
  constexpr int X_BYTES = S * X_PITCH;
  constexpr int CPR = LP / 8;              // 16-byte chunks per row of X
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* xs = smem;
  unsigned char* as = smem + X_BYTES;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int idx = lane & 15, lg = lane >> 4;
  const bf16_t* in = g.in + mat * g.stride;
  bf16_t* out = g.out + mat * g.strideo;
  const int L = g.L;

  // 1 / (|U| + eps) from the partial sums the pass that wrote U left behind (every wavefront
  // adds them up for itself, in the same order)
  const float* partials = g.partials + mat * g.nblk;
  float tot = lane < g.nblk ? partials[lane] : 0.f;

  // ---- X from memory into LDS (columns L .. LP-1 are zero).  All of a thread's loads go out before the
  // first is awaited: one workgroup has a round trip to memory to itself.
  if (!g.tall) {
    u32x4 v[8 * TT];
#pragma unroll
    for (int t = 0; t < 8 * TT; ++t) {
      const int r = (t * 256 + tid) / CPR, ch = (t * 256 + tid) % CPR;
      v[t] = *reinterpret_cast<const u32x4*>(in + (long)r * g.ld + (ch * 8 < L ? ch * 8 : 0));
    }
#pragma unroll
    for (int t = 0; t < 8 * TT; ++t) {
      const int r = (t * 256 + tid) / CPR, ch = (t * 256 + tid) % CPR;
      if (ch * 8 >= L) v[t] = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(xs + chunk_pos(r, ch, X_PITCH)) = v[t];
    }
  } else {
    // a thread turns 8 columns of 4 rows of memory over
    const int cg = tid & 15;
    u32x4 v[2 * TT][4];
#pragma unroll
    for (int t = 0; t < 2 * TT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int rg = (t * 16 + (tid >> 4)) * 4 + e;
        v[t][e] = *reinterpret_cast<const u32x4*>(in + (long)(rg < L ? rg : 0) * g.ld + cg * 8);
      }
#pragma unroll
    for (int t = 0; t < 2 * TT; ++t) {
      const int rg = (t * 16 + (tid >> 4)) * 4;
      if (rg >= L)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[t][e] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        u32x2 w;
        w.x = (e & 1) ? halves_hi(v[t][0][e / 2], v[t][1][e / 2]) : halves_lo(v[t][0][e / 2], v[t][1][e / 2]);
        w.y = (e & 1) ? halves_hi(v[t][2][e / 2], v[t][3][e / 2]) : halves_lo(v[t][2][e / 2], v[t][3][e / 2]);
        *reinterpret_cast<u32x2*>(xs + chunk_pos(cg * 8 + e, rg >> 3, X_PITCH) + (rg & 4) * 2) = w;
      }
    }
  }
  for (int i = lane + 64; i < g.nblk; i += 64) tot += partials[i];
  const float sumsq = wave_sum(tot);
  const float s = sumsq > 0.f ? 1.0f / (sqrtf(sumsq) + g.eps) : 0.f;   // all-zero matrix: 0, also when eps = 0
  __syncthreads();

  // The products of a matrix with its own transpose: wavefronts 0 and 3 take the 64 x 64 blocks on the diagonal, of their four
  // 32 x 32 blocks the three on and below it, 1 and 2 half of the lower left block each.
  const bool dg = wave == 0 || wave == 3;
  const int rm = wave ? 64 : 0, rn = wave == 3 ? 64 : wave == 2 ? 32 : 0;     // first row and column
  constexpr int NT = 2 * TT;                                 // column tiles of the wavefront's block of X
  const int cb = wave * 32 * TT;                             // and its first column

  // What follows from the lane is computed at the start of each phase: kept across the phases the
  // addresses would take the registers that the accumulators need.
  int ix = idx, gx = lg;
  auto fresh = [&] { asm volatile("" : "+v"(ix), "+v"(gx)); };

  // This wavefront's part of m m^T over `bytes` of a row, 32-deep slices: 12 MFMAs a slice on the diagonal (DG, from one set of
  // fragments, since rows and columns are the same), 8 elsewhere.  They take about as long as an LDS read, so fragments are
  // read two slices ahead, into the set of four that the last slice but one has left.
  u32x4 fa[4][4], fb[4][4];
  f32x4 sq[4][4];
  LanePos pr, pc;
  auto read_sq = [&](auto diag, const unsigned char* m, int pitch, int set, int r, int at) {
    constexpr int NB = decltype(diag)::value ? 4 : 2;
    if (r < NB) fb[set][r] = frag_col(m, pitch, pc, r, at);
    else fa[set][r - NB] = frag_col(m, pitch, pr, r - NB, at);
  };
  auto group_sq = [&](auto diag, auto first, const unsigned char* m, int pitch, int c, int last) {
    constexpr bool DG = decltype(diag)::value;
    constexpr int NR = DG ? 4 : 6;
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) {
      const int next = sl < 2 ? c + 64 * (sl + 2) : last + 64 * (sl - 2);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < (DG ? 2 * (i / 2) + 2 : 2); ++j) {
          const int n = DG ? (i < 2 ? 2 * i : 4 * (i - 1)) + j : 2 * i + j;
          const u32x4& a = DG ? fb[sl][i] : fa[sl][i];
          if (decltype(first)::value && sl == 0) mfma<true>(sq[i][j], fb[sl][j], a);
          else mfma<false>(sq[i][j], fb[sl][j], a);
          if (DG ? n % 2 == 0 && n / 2 < NR : n < NR) read_sq(diag, m, pitch, (sl + 2) & 3, DG ? n / 2 : n, next);
          __builtin_amdgcn_sched_barrier(0);
        }
    }
  };
  auto product_sq = [&](auto diag, const unsigned char* m, int pitch, int bytes) {
    constexpr bool DG = decltype(diag)::value;
    constexpr int NR = DG ? 4 : 6;
#pragma unroll
    for (int r = 0; r < 2 * NR; ++r) read_sq(diag, m, pitch, r / NR, r % NR, 64 * (r / NR));
    // (after the last group the reads ahead are of the first slices again, and not used)
    group_sq(diag, std::true_type{}, m, pitch, 0, bytes > 256 ? 256 : 0);
#pragma unroll 1
    for (int c = 256; c < bytes; c += 256) group_sq(diag, std::false_type{}, m, pitch, c, c + 256 < bytes ? c + 256 : 0);
    settle_part<DG>(sq);
  };
  // this lane's 16 bytes of the wavefront's part of A: tile row i, columns 32 J + 8 lg .. + 7
  auto a_at = [&](int i, int J) -> u32x4* {
    const LanePos p = lane_cols(A_PITCH, rm, ix, gx);
    return reinterpret_cast<u32x4*>(as + p.row + (p.x ^ (2 * rn) ^ (64 * J) ^ ((i & 1) * SWZ_ROW4)) +
                                    (32 * (i >> 1) + 4 * (i & 1)) * A_PITCH);
  };

  // A block of 32 x 32 of the part, rows from 32 I, columns from 32 J, turned over to the other side of the diagonal: four lanes hold a
  // column's 8 adjacent rows between them.
  auto put_turned = [&](int I, int J, const u32x4& v0, const u32x4& v1) {
    const int p = ix & 3;
    const u32x4 r0 = transpose_quad(v0, p), r1 = transpose_quad(v1, p);
    const int row = rn + 32 * J + 8 * gx + 2 * p, chunk = (rm + 32 * I) / 8 + (ix >> 2);
    *reinterpret_cast<u32x4*>(as + chunk_pos(row, chunk, A_PITCH)) =
        u32x4{halves_lo(r0[0], r0[1]), halves_lo(r0[2], r0[3]), halves_lo(r1[0], r1[1]), halves_lo(r1[2], r1[3])};
    *reinterpret_cast<u32x4*>(as + chunk_pos(row + 1, chunk, A_PITCH)) =
        u32x4{halves_hi(r0[0], r0[1]), halves_hi(r0[2], r0[3]), halves_hi(r1[0], r1[1]), halves_hi(r1[2], r1[3])};
  };
  // This wavefront's part of m m^T: in v its values, value(i, J) as they are stored.  Nothing that is called from here may wait for
  // the other wavefronts, half of which take the other form of the code.
  u32x4 v[4][2];
  auto square_part = [&](auto diag, const unsigned char* m, int pitch, int bytes, auto&& value) {
    constexpr bool DG = decltype(diag)::value;
    fresh();
    pr = lane_cols(pitch, rm, ix, gx);
    pc = lane_cols(pitch, rn, ix, gx);
    product_sq(diag, m, pitch, bytes);
    fresh();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int J = 0; J < (DG ? i / 2 + 1 : 1); ++J) v[i][J] = value(i, J);
  };
  // They go to both sides of the diagonal of A.
  auto put_part = [&](auto diag) {
    constexpr bool DG = decltype(diag)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int J = 0; J < (DG ? i / 2 + 1 : 1); ++J) *a_at(i, J) = v[i][J];
    if (!DG) put_turned(0, 0, v[0][0], v[1][0]);
    put_turned(1, 0, v[2][0], v[3][0]);
  };
  auto either = [&](auto&& f) {
    if (dg) f(std::true_type{});
    else f(std::false_type{});
  };

  for (int it = 0; it < g.iters; ++it) {
    const float alpha_a = it == 0 ? s * s : 1.f;

    // ---- A = alpha_a X X^T ---------------------------------------------------------------
    {
      auto value = [&](int i, int J) { return pack8(alpha_a * acc_read(sq[i][2 * J]), alpha_a * acc_read(sq[i][2 * J + 1])); };
      either([&](auto diag) {
        square_part(diag, xs, X_PITCH, 2 * L, value);          // L is a multiple of 128
        put_part(diag);
      });
    }
    __syncthreads();

    // ---- B' = c A A + b A + a I, in place over A (a column of A is its row) -------------
    {
      auto value = [&](int i, int J) {
        const u32x4 av = *a_at(i, J);
        f32x4 b[2] = {acc_read(sq[i][2 * J]), acc_read(sq[i][2 * J + 1])};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float ae = (e & 1) ? bf16hi(av[e / 2]) : bf16lo(av[e / 2]);
          b[e / 4][e % 4] = g.c * b[e / 4][e % 4] + g.b * ae;
        }
        if (J == i / 2 && dg) {                                // the diagonal crosses this tile
          const int d = 8 * (ix >> 2) + 4 * (i & 1) + (ix & 3) - 8 * gx;
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (e == d) b[e / 4][e % 4] += g.a;
        }
        return pack8(b[0], b[1]);
      };
      either([&](auto diag) { square_part(diag, as, A_PITCH, A_PITCH, value); });
      __syncthreads();            // every wavefront is done reading A
      either(put_part);
    }
    __syncthreads();

    // ---- X <- B' X (s B' X at first), in place: each wavefront all 128 rows of 32 TT columns --------
    {
      fresh();
      f32x4 acc[8][NT];
      // fragments of the next slice in the other set, or, where slices are short, of the next but one
      constexpr int SETS = TT == 4 ? 2 : 4, AHEAD = SETS / 2;
      u32x4 ga[SETS][8], gb[SETS][NT];
      pr = lane_rows(A_PITCH, 0, ix, gx);
      pc = lane_strided(X_PITCH, ix, gx, 2 * cb);
      auto read = [&](int r, int sl) {
        if (r == 0 || r > NT) ga[sl % SETS][r == 0 ? 0 : r - NT] = frag_row(as, A_PITCH, pr, r == 0 ? 0 : r - NT, 64 * sl);
        else gb[sl % SETS][r - 1] = frag_tr(xs, X_PITCH, pc, r - 1, sl);
      };
#pragma unroll
      for (int r = 0; r < AHEAD * (8 + NT); ++r) read(r % (8 + NT), r / (8 + NT));
      constexpr int NM = 8 * NT;                              // MFMAs of a slice
      constexpr int STEP = NM / (8 + NT) > 2 ? 2 : 1;         // MFMAs per read
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) {
#pragma unroll
        for (int n = 0; n < NM; ++n) {
          const int i = n / NT, j = n % NT;
          if (sl == 0) mfma<true>(acc[i][j], gb[sl % SETS][j], ga[sl % SETS][i]);
          else mfma<false>(acc[i][j], gb[sl % SETS][j], ga[sl % SETS][i]);
          if (sl + AHEAD < 4 && n % STEP == 0 && n / STEP < 8 + NT) read(n / STEP, sl + AHEAD);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      settle(acc);
      __syncthreads();            // every wavefront is done reading X and B'
      fresh();
      auto put = [&](auto&& value) {
        const LanePos p = lane_rows(X_PITCH, 0, ix, gx);
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int J = 0; J < TT; ++J) {
            // keep the scheduler from pulling all accumulator reads up here
            __builtin_amdgcn_sched_barrier(0);
            *reinterpret_cast<u32x4*>(xs + p.row + (p.x ^ (2 * cb) ^ (64 * J) ^ ((i & 1) * SWZ_ROW4)) + 16 * i * X_PITCH) =
                pack8(value(acc_read(acc[i][2 * J])), value(acc_read(acc[i][2 * J + 1])));
          }
      };
      if (it == 0) put([&](const f32x4& v) { return s * v; });
      else put([](const f32x4& v) { return v; });
    }
    __syncthreads();
  }

  // ---- X back to memory (the padded columns L .. LP-1 are not stored) --------------------
  if (!g.tall) {
#pragma unroll 4
    for (int q = tid; q < S * CPR; q += 256) {
      const int r = q / CPR, ch = q % CPR;
      if (ch * 8 < L)
        *reinterpret_cast<u32x4*>(out + (long)r * g.ldo + ch * 8) =
            *reinterpret_cast<const u32x4*>(xs + chunk_pos(r, ch, X_PITCH));
    }
  } else {
    // a K-strided fragment is 8 adjacent values of a row of memory
    pc = lane_strided(X_PITCH, idx, lg, 2 * cb);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int rg = cb + 32 * (j >> 1) + 8 * (idx >> 2) + 4 * (j & 1) + (idx & 3);
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) {
        const u32x4 v = frag_tr(xs, X_PITCH, pc, j, sl);
        if (cb + 32 * (j >> 1) < L) *reinterpret_cast<u32x4*>(out + (long)rg * g.ldo + (4 * sl + lg) * 8) = v;
      }
    }
  }
}

template <int TT>
__global__ __launch_bounds__(256) void ns_chain_small_kernel(ChainArgs g) {
  ns_chain_body<TT>(g, (long)blockIdx.x);
}

// Batches of several shapes in one launch.  A chain is a serial walk of one workgroup (24 us for
// 128 x 128, 43 for 128 x 512, 45 for 512 x 128) that leaves the other compute units idle, so batches
// that fit the chip together go side by side: 8 / 2 / 2 matrices of these shapes take 45 us instead of
// 115 one after the other.
struct ChainTable { ChainArgs s[MAX_CHAINS]; unsigned int blk0[MAX_CHAINS]; int n; };
__global__ __launch_bounds__(256) void ns_chain_multi_kernel(ChainTable tab) {
  int si = 0;
  for (int i = 1; i < tab.n; ++i)
    if (blockIdx.x >= tab.blk0[i]) si = i;
  const ChainArgs g = tab.s[si];
  const long mat = (long)(blockIdx.x - tab.blk0[si]);
  if (g.L <= 128) ns_chain_body<1>(g, mat);
  else if (g.L <= 256) ns_chain_body<2>(g, mat);
  else ns_chain_body<4>(g, mat);
}

constexpr size_t chain_lds(int tt) { return (size_t)S * 128 * tt * 2 + (size_t)S * A_PITCH; }
int chain_tt(const ChainArgs& g) { return g.L <= 128 ? 1 : g.L <= 256 ? 2 : 4; }
// executed: 40 of 64 MFMAs of the Gram matrix and the square, all LP columns of X
double chain_flops(const ChainArgs& g) {
  return ((2.0 * S * S * (double)g.L + 2.0 * S * S * S) * 40 / 64 + 2.0 * S * S * (128.0 * chain_tt(g))) * g.iters;
}
// raised once per kernel and device; the call is idempotent
int raise_lds_limit(const void* kern, std::atomic<bool>* done, size_t lds) {
  const int slot = device_slot();
  if (slot < 0 || !done[slot].load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return MLC_ERR_LAUNCH;
    if (slot >= 0) done[slot].store(true, std::memory_order_release);
  }
  return MLC_OK;
}

template <int TT>
int launch_tt(const ChainArgs& g, int64_t count, hipStream_t stream) {
  auto kern = ns_chain_small_kernel<TT>;
  static std::atomic<bool> attr_set[MAX_DEVICES];
  const int rc = raise_lds_limit(reinterpret_cast<const void*>(kern), attr_set, chain_lds(TT));
  if (rc != MLC_OK) return rc;
  LaunchScope scope(MLC_KERNEL_NS_GEMM, stream, chain_flops(g) * (double)count, 0.0);
  hipLaunchKernelGGL(kern, dim3((unsigned int)count), dim3(256), chain_lds(TT), stream, g);
  return hipGetLastError() == hipSuccess ? MLC_OK : MLC_ERR_LAUNCH;
}

int launch_one(const ChainArgs& g, int64_t count, hipStream_t stream) {
  const int tt = chain_tt(g);
  if (tt == 1) return launch_tt<1>(g, count, stream);
  if (tt == 2) return launch_tt<2>(g, count, stream);
  return launch_tt<4>(g, count, stream);
}

}  // namespace

bool ns_chain_small_fits(int64_t mp, int64_t np) {
  const int64_t sp = mp < np ? mp : np, lp = mp < np ? np : mp;
  return sp == S && lp <= 512;
}

int launch_ns_chain_small(const ChainDesc* d, int n, float eps, int iters, float a, float b, float c,
                          hipStream_t stream) {
  if (n < 1 || n > MAX_CHAINS || iters < 1) return MLC_ERR_ARG;
  ChainTable tab;
  tab.n = n;
  int64_t total = 0;
  int tt = 1;
  double flops = 0.0;
  for (int i = 0; i < MAX_CHAINS; ++i) {
    const ChainDesc& c_ = d[i < n ? i : 0];
    if (!ns_chain_small_fits(c_.mp, c_.np) || c_.mp % 128 || c_.np % 128) return MLC_ERR_SHAPE;
    if (!c_.in || !c_.out || !c_.partials) return MLC_ERR_NULL;
    if (c_.count < 1 || c_.count > 0x7fffffff || c_.nblk < 1) return MLC_ERR_ARG;
    // every 16-byte access stays inside a row of the padded matrix
    if (c_.ld % 8 || c_.stride % 8 || c_.ld < c_.np || c_.stride < c_.mp * c_.ld) return MLC_ERR_SHAPE;
    if (c_.ldo % 8 || c_.strideo % 8 || c_.ldo < c_.np || c_.strideo < c_.mp * c_.ldo) return MLC_ERR_SHAPE;
    const bool tall = c_.mp > c_.np;
    ChainArgs& g = tab.s[i];
    g.in = c_.in; g.out = c_.out; g.ld = c_.ld; g.stride = c_.stride;
    g.ldo = c_.ldo; g.strideo = c_.strideo;
    g.tall = tall ? 1 : 0;
    g.L = (int)(tall ? c_.mp : c_.np);
    g.partials = c_.partials; g.nblk = c_.nblk; g.eps = eps;
    g.iters = iters; g.a = a; g.b = b; g.c = c;
    tab.blk0[i] = i < n ? (unsigned int)total : 0xffffffffu;
    if (i >= n) continue;
    total += c_.count;
    if (chain_tt(g) > tt) tt = chain_tt(g);
    flops += chain_flops(g) * (double)c_.count;
  }
  // Side by side as long as every matrix finds a compute unit of its own.  Beyond that a launch of
  // its own is better for each batch: it asks for no more LDS than its shape needs, and two
  // workgroups of the narrow shapes fit a compute unit.
  if (n == 1 || total > CHAIN_SHARE_MAX) {
    for (int i = 0; i < n; ++i) {
      const int rc = launch_one(tab.s[i], d[i].count, stream);
      if (rc != MLC_OK) return rc;
    }
    return MLC_OK;
  }
  static std::atomic<bool> attr_set[MAX_DEVICES];
  const int rc = raise_lds_limit(reinterpret_cast<const void*>(ns_chain_multi_kernel), attr_set, chain_lds(4));
  if (rc != MLC_OK) return rc;
  LaunchScope scope(MLC_KERNEL_NS_GEMM, stream, flops, 0.0);
  hipLaunchKernelGGL(ns_chain_multi_kernel, dim3((unsigned int)total), dim3(256), chain_lds(tt), stream, tab);
  return hipGetLastError() == hipSuccess ? MLC_OK : MLC_ERR_LAUNCH;
}

}  // namespace mlc
