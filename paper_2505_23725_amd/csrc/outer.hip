// HBM-bound kernels of the DiLoCo outer step (paper Sec. 4.1 eqs. 2-3, Algorithm 1 lines
// after the inner loop, Algorithm 2 "compress parameter delta"):
//   * fused pseudogradient / K-way average / outer Nesterov / write-back,
//   * 2/4/8-bit linear quantiser of theta_g - theta_k (IEEE fp32, ties to even), range per row
//     or per matrix, with or without an offset, optionally with error feedback (Algorithm 2,
//     EF branch) and a second quantisation of the mean,
//   * dequantise + K-way average + outer update + write-back.
// The K worker replicas live on this GPU, so the average is a loop over K pointers
// in a fixed order: ((d_1 + d_2) + ...) * (1/K).
#include "common.h"
#include "quant_rule.h"

namespace mlc {
namespace {

constexpr int OT_THREADS = 256;

// eq. 3; theta comes back as the value the global buffer will hold after the store, so the
// write-back hands every worker exactly the new theta_g.
template <typename GT>
__device__ __forceinline__ void outer_update(float& theta, float& u, float psi, float eta, float mu,
                                             int nesterov) {
  const float step = eta * psi;
  u = mu * u + step;
  theta = Vec8<GT>::round(nesterov ? theta - mu * u - step : theta - u);
}

// 8 elements, `left` of them before the end of the row or matrix (RAG: perhaps fewer than 8, and at
// any alignment).
template <typename T, bool RAG>
__device__ __forceinline__ void load8(const T* p, int left, float (&v)[8]) {
  if constexpr (RAG) Vec8<T>::unpack(Vec8U<T>::load_raw(p, left), v);
  else Vec8<T>::load(p, v);
}
template <typename T, bool RAG>
__device__ __forceinline__ void store8(T* p, const float (&v)[8], int left) {
  if constexpr (RAG) Vec8U<T>::store(p, v, left);
  else Vec8<T>::store(p, v);
}

// ---- unquantised fused outer step ---------------------------------------------------
// Workgroup blk of nblk walks over its share of the n_elems elements.
template <typename WT, typename GT, typename PW>
__device__ __forceinline__ void outer_fused_body(
    const PW& w, GT* __restrict__ theta_g, float* __restrict__ u, long n_elems, int K, float eta,
    float mu, float inv_k, int nesterov, int write_back, long blk, long nblk) {
  const long n_vec = n_elems / 8;
  for (long i = blk * OT_THREADS + threadIdx.x; i < n_vec; i += nblk * OT_THREADS) {
    const long off = i * 8;
    float tg[8], uv[8], acc[8];
    Vec8<GT>::load(theta_g + off, tg);
    Vec8<float>::load(u + off, uv);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    for (int k = 0; k < K; ++k) {
      float tk[8];
      Vec8<WT>::load(reinterpret_cast<const WT*>(w.p[k]) + off, tk);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += tg[j] - tk[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) outer_update<GT>(tg[j], uv[j], acc[j] * inv_k, eta, mu, nesterov);
    Vec8<GT>::store(theta_g + off, tg);
    Vec8<float>::store(u + off, uv);
    if (write_back)
      for (int k = 0; k < K; ++k) Vec8<WT>::store(reinterpret_cast<WT*>(w.p[k]) + off, tg);
  }
  // ragged tail (fewer than 8 elements), one thread each
  const long tail0 = n_vec * 8;
  const long t = tail0 + blk * OT_THREADS + threadIdx.x;
  if (t < n_elems) {
    float tg = Vec8<GT>::load1(theta_g + t), uv = u[t], acc = 0.f;
    for (int k = 0; k < K; ++k) acc += tg - Vec8<WT>::load1(reinterpret_cast<const WT*>(w.p[k]) + t);
    outer_update<GT>(tg, uv, acc * inv_k, eta, mu, nesterov);
    Vec8<GT>::store1(theta_g + t, tg);
    u[t] = uv;
    if (write_back)
      for (int k = 0; k < K; ++k) Vec8<WT>::store1(reinterpret_cast<WT*>(w.p[k]) + t, tg);
  }
}

template <typename WT, typename GT>
__global__ __launch_bounds__(OT_THREADS) void outer_fused_kernel(
    WorkerPtrs w, GT* __restrict__ theta_g, float* __restrict__ u, long n_elems, int K, float eta,
    float mu, float inv_k, int nesterov, int write_back) {
  outer_fused_body<WT, GT>(w, theta_g, u, n_elems, K, eta, mu, inv_k, nesterov, write_back,
                           (long)blockIdx.x, (long)gridDim.x);
}

// ---- linear quantiser (Sec. 2 "Compressed Communication"; Algorithm 2) -----------------
// bits = 2, 4 or 8.  Without offset: levels -L..L, L = 2^(bits-1) - 1, over [-amax, amax],
// stored code = level + 2^(bits-1).  With offset: levels 0..L, L = 2^bits - 1, over
// [min, max], stored as they are, dequantised value = level * scale + min.  8 / bits codes
// per byte, the lowest column in the lowest bits.  The range is taken per row, or per matrix
// (then it has been computed beforehand and is read from the scale / offset arrays).  With
// error feedback the value quantised is e = fl32(fl32(beta * E) + delta) and the residual
// becomes E <- fl32(e - dequantised value).  Every operation is a single fp32 operation
// (no fused multiply-add) so that codes and residuals are reproducible bit for bit.
struct Range { float scale, lo; };

__device__ __forceinline__ Range make_range(float mn, float mx, const QuantForm& f) {
  Range r;
  if (f.offset) { r.lo = mn; r.scale = __fsub_rn(mx, mn) / f.levels; }
  else { r.lo = 0.f; r.scale = fmaxf(mx, -mn) / f.levels; }
  return r;
}

__device__ __forceinline__ int quant_level(float v, const Range& r, const QuantForm& f) {
  if (!(r.scale > 0.f)) return 0;
  const float x = f.offset ? __fsub_rn(v, r.lo) : v;
  float q = rintf(x / r.scale);             // IEEE division, round half to even
  q = fminf(fmaxf(q, f.offset ? 0.f : -f.levels), f.levels);
  return (int)q;
}

__device__ __forceinline__ float dequant_level(int q, const Range& r, const QuantForm& f) {
  const float s = __fmul_rn((float)q, r.scale);
  return f.offset ? __fadd_rn(s, r.lo) : s;
}

__device__ __forceinline__ float ef_input(float delta, float residual, float beta) {
  return __fadd_rn(__fmul_rn(beta, residual), delta);
}

// The level of a value without a division, where that is certain.  With i = 1 / scale to within 2^-24, fl(x i) is within
// 3 * 2^-24 of fl(x / scale), relative to it; both round to the same integer unless that distance reaches from fl(x i) to a
// half-integer, so unless |fl(x i) - rint(fl(x i))| >= 0.5 - (levels + 1) 2^-22.  Values closer to a tie (4 in 10^6 of 4-bit levels, 1 in 10^4
// of 8-bit offset ones, more where data sit on a grid), and scales for which 1 / scale is no ordinary number, are divided.
// Levels stay in floating point from there to the codes and to what is sent.  (Without an offset lo is 0, and to subtract
// and add it changes nothing but the sign of a level -0, which counts as 0.)
//
// The one-pass kernels are bound by the memory stream and, from about three workers on, by vector instructions, of which each
// value took 34 a worker, ten of them the division: with eight workers the SIMDs issued them for 0.7 of the time.  Now about 20.  4-bit
// steps, us before and after: rows of 736 and 2432, eight workers, 182 -> 153; 528 and 1664, four, 267 -> 238, one, 293 -> 280; 1024 and
// 4096, eight, 151 -> 134, one, 423 -> 420.
struct Divider { float scale, lo, inv, limit, low, high; };
// SCALAR: in scalar registers, for a range that a wavefront's lanes share.  (It frees vector registers where rows are alone in a
// launch, rows of 2560 and 10240 with four workers 560 -> 552 us, or have four vectors a thread, which go to memory by the dozen
// otherwise: 8 of 1280 x 1280 and 2 of 1280 x 4416, eight workers of float32 with error feedback, 628 -> 587, 24 of 1024 x 1536 and 6 of
// 1536 x 1024, two of bf16, 206 -> 199.  Fewer vectors beside others it only costs moves: 736 and 2432 with eight 153 -> 160.)
template <bool SCALAR>
__device__ __forceinline__ Divider make_divider(const Range& r, const QuantForm& f) {
  auto uniform = [](float v) { return SCALAR ? __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))) : v; };
  Divider d;
  d.scale = uniform(r.scale);
  d.lo = uniform(r.lo);
  const float i = __builtin_amdgcn_rcpf(d.scale);
  d.inv = uniform(fmaf(i, fmaf(-d.scale, i, 1.f), i));
  const bool ordinary = d.scale >= 0x1p-100f && d.scale <= 0x1p100f;
  d.limit = uniform(ordinary ? 0.5f - (f.levels + 1.f) * 0x1p-22f : -1.f);
  d.low = f.offset ? 0.f : -f.levels;
  d.high = f.levels;
  return d;
}
__device__ __forceinline__ void quant_levels4(const float* v, const Divider& d, float (&q)[4]) {
  float worst = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float t = __fmul_rn(__fsub_rn(v[j], d.lo), d.inv);
    q[j] = rintf(t);
    worst = fmaxf(worst, fabsf(__fsub_rn(t, q[j])));
  }
  if (worst >= d.limit) {
    if (d.scale > 0.f) {
#pragma unroll
      for (int j = 0; j < 4; ++j) q[j] = rintf(__fsub_rn(v[j], d.lo) / d.scale);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) q[j] = 0.f;
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) q[j] = __builtin_amdgcn_fmed3f(q[j], d.low, d.high);     // (a NaN becomes the lowest level)
}
__device__ __forceinline__ float dequant_level(float q, const Divider& d) {
  return __fadd_rn(__fmul_rn(q, d.scale), d.lo);
}
// The codes of 4 levels, first one lowest: levels that take up to 16 bits are added up exactly in fp32, their bias with them.
__device__ __forceinline__ unsigned int pack_levels4(const float (&q)[4], int bits, int bias) {
  const float b = (float)bias;
  if (bits == 4) return (unsigned int)fmaf(fmaf(fmaf(q[3] + b * (4369.f / 4096.f), 16.f, q[2]), 16.f, q[1]), 16.f, q[0]);
  if (bits == 2) return (unsigned int)fmaf(fmaf(fmaf(q[3] + b * (85.f / 64.f), 4.f, q[2]), 4.f, q[1]), 4.f, q[0]);
  const float c = b * (257.f / 256.f);
  return (unsigned int)fmaf(q[1] + c, 256.f, q[0]) | (unsigned int)fmaf(q[3] + c, 256.f, q[2]) << 16;
}
__device__ __forceinline__ void store_packed8(uint8_t* crow, int c, const u32x2& p, int bits) {
  if (bits == 4) *reinterpret_cast<unsigned int*>(crow + c / 2) = p.x;
  else if (bits == 8) *reinterpret_cast<u32x2*>(crow + c) = p;
  else *reinterpret_cast<unsigned short*>(crow + c / 4) = (unsigned short)p.x;
}
// The first cnt of 8 levels at an address aligned to a byte only (cnt * bits is a multiple of 8).
__device__ __forceinline__ void store_packed8_part(uint8_t* crow, int c, const u32x2& p, int bits, int cnt) {
  typedef unsigned short u16_u __attribute__((aligned(1)));
  typedef unsigned int u32_u __attribute__((aligned(1)));
  uint8_t* const at = crow + c * bits / 8;
  if (cnt >= 8) {
    if (bits == 2) *reinterpret_cast<u16_u*>(at) = (unsigned short)p.x;
    else *reinterpret_cast<u32_u*>(at) = p.x;
    if (bits == 8) *reinterpret_cast<u32_u*>(at + 4) = p.y;
  } else {
    const unsigned long w = p.x | (unsigned long)p.y << 32;
    for (int j = 0; j < cnt * bits / 8; ++j) at[j] = (uint8_t)(w >> (8 * j));
  }
}
// Largest value of a wavefront, in all its lanes, through lanes' neighbours in registers (six round trips through the LDS
// otherwise, which every worker's row waits for).
__device__ __forceinline__ float wave_max_dpp(float v) {
#define MLC_DPP_MAX(CTRL) \
  v = fmaxf(v, __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(v), __float_as_uint(v), CTRL, 0xf, 0xf, false)))
  MLC_DPP_MAX(0xb1);        // the neighbour of a pair, the other pair of four, the mirrored half of 8, of 16
  MLC_DPP_MAX(0x4e);
  MLC_DPP_MAX(0x141);
  MLC_DPP_MAX(0x140);
  MLC_DPP_MAX(0x142);       // lane 15 of the row before, lane 31 of the half before
  MLC_DPP_MAX(0x143);
#undef MLC_DPP_MAX
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), 63));
}

// 8 adjacent levels of a row, first column c (a multiple of 8) <-> bits bytes of its codes
__device__ __forceinline__ void store_codes8(uint8_t* crow, int c, const int (&q)[8], int bits, int bias) {
  if (bits == 4) {
    unsigned int p = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) p |= (unsigned int)(q[j] + bias) << (4 * j);
    *reinterpret_cast<unsigned int*>(crow + c / 2) = p;
  } else if (bits == 8) {
    u32x2 p = {0u, 0u};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      p.x |= (unsigned int)(q[j] + bias) << (8 * j);
      p.y |= (unsigned int)(q[j + 4] + bias) << (8 * j);
    }
    *reinterpret_cast<u32x2*>(crow + c) = p;
  } else {
    unsigned int p = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) p |= (unsigned int)(q[j] + bias) << (2 * j);
    *reinterpret_cast<unsigned short*>(crow + c / 4) = (unsigned short)p;
  }
}

__device__ __forceinline__ void load_levels8(const uint8_t* crow, int c, int (&q)[8], int bits, int bias) {
  if (bits == 4) {
    const unsigned int p = *reinterpret_cast<const unsigned int*>(crow + c / 2);
#pragma unroll
    for (int j = 0; j < 8; ++j) q[j] = (int)((p >> (4 * j)) & 0xfu) - bias;
  } else if (bits == 8) {
    const u32x2 p = *reinterpret_cast<const u32x2*>(crow + c);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      q[j] = (int)((p.x >> (8 * j)) & 0xffu) - bias;
      q[j + 4] = (int)((p.y >> (8 * j)) & 0xffu) - bias;
    }
  } else {
    const unsigned int p = *reinterpret_cast<const unsigned short*>(crow + c / 4);
#pragma unroll
    for (int j = 0; j < 8; ++j) q[j] = (int)((p >> (2 * j)) & 0x3u) - bias;
  }
}

// Range of worker k's row (or of the matrix the row belongs to) as stored by an earlier pass.
template <typename PS, typename PO>
__device__ __forceinline__ Range stored_range(const PS& scales, const PO& offsets, int k,
                                              long grp, const QuantForm& f) {
  Range r;
  r.scale = scales.p[k][grp];
  r.lo = f.offset ? offsets.p[k][grp] : 0.f;
  return r;
}

// ---- ranges per matrix (the "global" scope): init, reduce with atomics, finalise --------
// Floats are ordered through an order-preserving map to unsigned keys, so that the
// reduction is exact and independent of the order in which workgroups arrive.
__device__ __forceinline__ unsigned int float_key(float v) {
  const unsigned int b = __float_as_uint(v);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_float(unsigned int k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Up to OUTER_MAX_SEG groups of OUTER_MAX_SEG_K workers a launch, or as many such parts of a group's workers, each in a layer of the
// grid (12 workers, 4 bits, error feedback, two groups of 4 x 1053 x 128 and 18 x 96 x 1024: 145 us with three launches for each
// part, 126 like this).
template <typename T> struct SegPtrs { T p[OUTER_MAX_SEG_K]; };
static_assert(OUTER_MAX_SEG * OUTER_MAX_SEG_K >= MLC_MAX_WORKERS, "any group's workers go into one launch");
struct RangeSeg {
  SegPtrs<void*> w;
  SegPtrs<float*> ef, scales, offsets;
  const void* theta_g;
  long elems;
  unsigned int count, nblk;            // matrices; workgroups a matrix
  int workers;
};
struct RangeTable { RangeSeg s[OUTER_MAX_SEG]; };

__global__ void matrix_range_init_kernel(RangeTable tab, int offset) {
  const RangeSeg& sg = tab.s[blockIdx.z];
  const long b = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int k = blockIdx.y;
  if (b >= sg.count || k >= sg.workers) return;
  reinterpret_cast<unsigned int*>(sg.scales.p[k])[b] = 0u;                      // below every key
  if (offset) reinterpret_cast<unsigned int*>(sg.offsets.p[k])[b] = 0xffffffffu;   // above every key
}

// The ranges of all workers of a piece, so that theta_g is read once and not once a worker (KM: their number, or the next power of two
// above it; without residuals all their loads are under way together, with them a worker's at a time).  Whole steps with error feedback, eight workers, a grid
// dimension for the workers and now, us: 2 x 3560 x 5504 and its square 3611 and 3200; without feedback 12 x 512 x 1024 with bf16 workers
// 782 and 470.
template <typename WT, typename GT, bool VEC, int KM>
__global__ __launch_bounds__(OT_THREADS) void matrix_range_kernel(RangeTable tab, QuantForm form) {
  __shared__ float red[2][KM][OT_THREADS / 64];
  const RangeSeg& sg = tab.s[blockIdx.z];
  const int K = sg.workers;
  const unsigned int blk = blockIdx.x % sg.nblk;
  const long b = blockIdx.x / sg.nblk, elems = sg.elems;
  if (b >= sg.count) return;
  const GT* tg = reinterpret_cast<const GT*>(sg.theta_g) + b * elems;
  const bool fb = sg.ef.p[0] != nullptr;                  // all workers have residuals, or none
  float mn[KM], mx[KM];
#pragma unroll
  for (int k = 0; k < KM; ++k) { mn[k] = INFINITY; mx[k] = -INFINITY; }
  for (long i = ((long)blk * OT_THREADS + threadIdx.x) * 8; i < elems; i += (long)sg.nblk * OT_THREADS * 8) {
    float a[8];
    const int left = (int)min(elems - i, 8L);
    load8<GT, !VEC>(tg + i, left, a);
#pragma unroll
    for (int k = 0; k < KM; ++k) {
      if (k >= K) break;
      float c[8], e[8];
      load8<WT, !VEC>(reinterpret_cast<const WT*>(sg.w.p[k]) + b * elems + i, left, c);
      if (fb) load8<float, !VEC>(sg.ef.p[k] + b * elems + i, left, e);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float d = a[j] - c[j];
        const float v = fb ? ef_input(d, e[j], form.ef_beta) : d;
        if (VEC || j < left) { mn[k] = fminf(mn[k], v); mx[k] = fmaxf(mx[k], v); }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < KM; ++k) {
    const float lo = -wave_max_dpp(-mn[k]), hi = wave_max_dpp(mx[k]);
    if ((threadIdx.x & 63) == 0) { red[0][k][threadIdx.x >> 6] = lo; red[1][k][threadIdx.x >> 6] = hi; }
  }
  __syncthreads();
  const int k = threadIdx.x;
  if (k >= K) return;
  const float lo = fminf(fminf(red[0][k][0], red[0][k][1]), fminf(red[0][k][2], red[0][k][3]));
  const float hi = fmaxf(fmaxf(red[1][k][0], red[1][k][1]), fmaxf(red[1][k][2], red[1][k][3]));
  if (!(lo <= hi)) return;   // not a single element was a number
  if (form.offset) {
    atomicMax(reinterpret_cast<unsigned int*>(sg.scales.p[k]) + b, float_key(hi));
    atomicMin(reinterpret_cast<unsigned int*>(sg.offsets.p[k]) + b, float_key(lo));
  } else {                   // amax >= 0: its bit pattern is ordered like an unsigned
    atomicMax(reinterpret_cast<unsigned int*>(sg.scales.p[k]) + b, __float_as_uint(fmaxf(hi, -lo)));
  }
}

__global__ void matrix_range_finish_kernel(RangeTable tab, QuantForm form) {
  const RangeSeg& sg = tab.s[blockIdx.z];
  const long b = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int k = blockIdx.y;
  if (b >= sg.count || k >= sg.workers) return;
  float* scale = sg.scales.p[k] + b;
  if (form.offset) {
    float* lo = sg.offsets.p[k] + b;
    const Range r = make_range(key_float(__float_as_uint(*lo)), key_float(__float_as_uint(*scale)), form);
    *scale = r.scale;
    *lo = r.lo;
  } else {
    *scale = *scale / form.levels;     // the array holds amax
  }
}

// Two passes over the row (range, then codes), one wavefront per row, all K workers; the
// second pass re-reads data the first pass just pulled through L2.  Rows whose length is
// not a multiple of 8 go one code byte (8 / bits columns) per lane and step.
template <typename WT, typename GT, bool VEC>
__global__ __launch_bounds__(OT_THREADS) void quantize_rows_kernel(
    WorkerPtrs w, const GT* __restrict__ theta_g, CodePtrs codes, ScalePtrs scales, OffsetPtrs offsets,
    ResidualPtrs ef, long rows, int n, int K, QuantForm form) {
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * (OT_THREADS / 64) + (threadIdx.x >> 6);
  if (row >= rows) return;
  const GT* tg = theta_g + row * n;
  const int bits = form.bits;
  const int W = VEC ? 8 : 8 / bits;         // elements per lane per step
  const long row_bytes = (long)n * bits / 8;
  for (int k = 0; k < K; ++k) {
    const WT* tk = reinterpret_cast<const WT*>(w.p[k]) + row * n;
    float* res = ef.p[k] ? ef.p[k] + row * n : nullptr;
    Range rg;
    if (form.rows_per_range) {
      rg = stored_range(scales, offsets, k, row / form.rows_per_range, form);
    } else {
      float mn = INFINITY, mx = -INFINITY;
      for (int c = lane * W; c < n; c += 64 * W) {
        float a[8], b[8], e[8];
        if (VEC) {
          Vec8<GT>::load(tg + c, a); Vec8<WT>::load(tk + c, b);
          if (res) Vec8<float>::load(res + c, e);
        } else {
          for (int j = 0; j < W; ++j) {
            a[j] = Vec8<GT>::load1(tg + c + j); b[j] = Vec8<WT>::load1(tk + c + j);
            if (res) e[j] = res[c + j];
          }
        }
        for (int j = 0; j < W; ++j) {
          const float d = a[j] - b[j];
          const float v = res ? ef_input(d, e[j], form.ef_beta) : d;
          mn = fminf(mn, v); mx = fmaxf(mx, v);
        }
      }
      rg = make_range(wave_min(mn), wave_max(mx), form);
      if (lane == 0) {
        scales.p[k][row] = rg.scale;
        if (form.offset) offsets.p[k][row] = rg.lo;
      }
    }
    uint8_t* crow = codes.p[k] + row * row_bytes;
    for (int c = lane * W; c < n; c += 64 * W) {
      float a[8], b[8], e[8];
      if (VEC) {
        Vec8<GT>::load(tg + c, a); Vec8<WT>::load(tk + c, b);
        if (res) Vec8<float>::load(res + c, e);
      } else {
        for (int j = 0; j < W; ++j) {
          a[j] = Vec8<GT>::load1(tg + c + j); b[j] = Vec8<WT>::load1(tk + c + j);
          if (res) e[j] = res[c + j];
        }
      }
      int q[8];
      for (int j = 0; j < W; ++j) {
        const float d = a[j] - b[j];
        const float v = res ? ef_input(d, e[j], form.ef_beta) : d;
        q[j] = quant_level(v, rg, form);
        e[j] = __fsub_rn(v, dequant_level(q[j], rg, form));
      }
      if (VEC) {
        store_codes8(crow, c, q, bits, form.code_bias);
        if (res) Vec8<float>::store(res + c, e);
      } else {
        unsigned int p = 0;
        for (int j = 0; j < W; ++j) p |= (unsigned int)(q[j] + form.code_bias) << (bits * j);
        crow[c / W] = (uint8_t)p;
        if (res)
          for (int j = 0; j < W; ++j) res[c + j] = e[j];
      }
    }
  }
}

// Single-pass variant: a group of G threads (a wavefront or the whole workgroup) owns a row
// and keeps it in registers (NV vectors of 8 elements per thread), so theta_g is read once
// for all K workers and every theta_k exactly once.  Same arithmetic as above.  With
// OUTER the dequantised values go straight into the mean and eq. 3 without re-reading
// theta_g or the codes; codes, scales and offsets are written either way.
// G0 = 0: the workgroup is as large as one row needs (quant_whole_row), G0 > 0: the group's threads.
// `blk` is the index of the workgroup among those that share these arguments; the pointer sets
// may be the 32-wide ones of a single-group launch or the narrow ones of a launch that covers
// several groups.
// KC: the number of workers where it is known (1: nothing is requested ahead, which takes a third of the registers).
// RAG: rows of any length, so neither the rows nor their codes are aligned and the last vector of
// a row may be a part of one (24 / 6 / 6 matrices of 1001 x 1001, 1001 x 2730 and 2730 x 1001, two
// workers, 8 bits with error feedback: 1500 us element by element in two passes, 516 like this).
template <typename WT, typename GT, int NV, int G0, bool OUTER, bool RAG, int KC, bool SCALAR, typename PW, typename PC, typename PS,
          typename PO, typename PE>
__device__ __forceinline__ void quantize_rows_reg_body(
    const PW& w, GT* __restrict__ theta_g, float* __restrict__ u, const PC& codes, const PS& scales,
    const PO& offsets, const PE& ef, long rows, int n, int workers, const QuantForm& form, float eta, float mu,
    float inv_k, int nesterov, int write_back, int requant, uint8_t* mean_codes, float* mean_scales,
    float* mean_offsets, long blk) {
  const int K = KC ? KC : workers;
  constexpr bool WHOLE = G0 == 0;
  const int G = WHOLE ? (int)blockDim.x : G0;
  constexpr int NW = WHOLE ? 16 : OT_THREADS / 64;
  const int waves = WHOLE ? (int)blockDim.x / 64 : NW;
  __shared__ float red[2][2][NW];          // [parity of k][min, max][wavefront]
  __shared__ float red2[2][NW];
  const int t = WHOLE ? threadIdx.x : threadIdx.x % G;
  const long row = WHOLE ? blk : blk * (OT_THREADS / G) + threadIdx.x / G;
  auto across = [&](const float (&r)[2][NW], float& mn, float& mx) {
    mn = r[0][0];
    mx = r[1][0];
#pragma unroll
    for (int wv = 1; wv < NW; ++wv)
      if (wv < waves) { mn = fminf(mn, r[0][wv]); mx = fmaxf(mx, r[1][wv]); }
  };
  const bool live = row < rows;            // whole groups are live or not; no early return
  const long rbase = live ? row * n : 0;   // (the workgroup-wide barrier below needs everyone)
  const int bits = form.bits;
  const long row_bytes = (long)n * bits / 8;
  const long grp = form.rows_per_range ? (live ? row / form.rows_per_range : 0) : (live ? row : 0);
  float tg[NV][8], acc[OUTER ? NV : 1][8];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = (t + i * G) * 8;
    if (live && c < n) load8<GT, RAG>(theta_g + rbase + c, n - c, tg[i]);
    else
#pragma unroll
      for (int j = 0; j < 8; ++j) tg[i][j] = 0.f;
    if constexpr (OUTER)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[i][j] = 0.f;
  }
  // The next worker's row is requested before this worker's row is reduced and quantised, so
  // that with several workers only the first request waits for memory with nothing to do.
  typedef typename Vec8<WT>::raw_t RawT;
  RawT ahead[NV];
  auto request = [&](int k) {
    const WT* tk = reinterpret_cast<const WT*>(w.p[k]) + rbase;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = (t + i * G) * 8;
      if (live && c < n) {
        if constexpr (RAG) ahead[i] = Vec8U<WT>::load_raw(tk + c, n - c);
        else ahead[i] = Vec8<WT>::load_raw(tk + c);
      }
    }
  };
  request(0);
  for (int k = 0; k < K; ++k) {
    float* res = ef.p[k] ? ef.p[k] + rbase : nullptr;
    float d[NV][8];
    float mn = INFINITY, mx = -INFINITY;
    RawT cur[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) cur[i] = ahead[i];
    if (k + 1 < K) request(k + 1);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = (t + i * G) * 8;
      if (live && c < n) {
        float b[8];
        Vec8<WT>::unpack(cur[i], b);
#pragma unroll
        for (int j = 0; j < 8; ++j) d[i][j] = tg[i][j] - b[j];
        if (res) {
          float e[8];
          load8<float, RAG>(res + c, n - c, e);
#pragma unroll
          for (int j = 0; j < 8; ++j) d[i][j] = ef_input(d[i][j], e[j], form.ef_beta);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (!RAG || c + j < n) { mn = fminf(mn, d[i][j]); mx = fmaxf(mx, d[i][j]); }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) d[i][j] = 0.f;
      }
    }
    Range rg;
    if (form.rows_per_range) {
      rg = stored_range(scales, offsets, k, grp, form);
    } else {
      mn = -wave_max_dpp(-mn); mx = wave_max_dpp(mx);
      if constexpr (WHOLE || G0 > 64) {
        if ((threadIdx.x & 63) == 0) { red[k & 1][0][threadIdx.x >> 6] = mn; red[k & 1][1][threadIdx.x >> 6] = mx; }
        __syncthreads();
        across(red[k & 1], mn, mx);
      }
      rg = make_range(mn, mx, form);
      if (live && t == 0) {
        scales.p[k][row] = rg.scale;
        if (form.offset) offsets.p[k][row] = rg.lo;
      }
    }
    const Divider dv = make_divider<SCALAR>(rg, form);
    uint8_t* crow = codes.p[k] + row * row_bytes;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = (t + i * G) * 8;
      if (live && c < n) {
        unsigned int h4[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {          // (four at a time: registers)
          float q[4];
          quant_levels4(&d[i][4 * h], dv, q);
          h4[h] = pack_levels4(q, bits, form.code_bias);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float sent = dequant_level(q[j], dv);
            if constexpr (OUTER) acc[i][4 * h + j] += sent;
            d[i][4 * h + j] = __fsub_rn(d[i][4 * h + j], sent);
          }
        }
        const u32x2 packed = {bits == 8 ? h4[0] : h4[0] | h4[1] << (4 * bits), h4[1]};
        if constexpr (RAG) store_packed8_part(crow, c, packed, bits, n - c);
        else store_packed8(crow, c, packed, bits);
        if (res) store8<float, RAG>(res + c, d[i], n - c);
      }
    }
  }
  if constexpr (OUTER) {
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[i][j] = __fmul_rn(acc[i][j], inv_k);     // Psi
    if (!RAG && requant) {
      // Second quantisation (the dequantise-reduce-quantise step between the two modelled
      // collectives): Psi is quantised row-wise again and its dequantised value is used.
      float mn = INFINITY, mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = (t + i * G) * 8;
        if (live && c < n)
#pragma unroll
          for (int j = 0; j < 8; ++j) { mn = fminf(mn, acc[i][j]); mx = fmaxf(mx, acc[i][j]); }
      }
      mn = wave_min(mn); mx = wave_max(mx);
      if constexpr (WHOLE || G0 > 64) {
        if ((threadIdx.x & 63) == 0) { red2[0][threadIdx.x >> 6] = mn; red2[1][threadIdx.x >> 6] = mx; }
        __syncthreads();
        across(red2, mn, mx);
      }
      const Range rg = make_range(mn, mx, form);
      if (live && t == 0) {
        if (mean_scales) mean_scales[row] = rg.scale;
        if (mean_offsets && form.offset) mean_offsets[row] = rg.lo;
      }
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = (t + i * G) * 8;
        if (live && c < n) {
          int q[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            q[j] = quant_level(acc[i][j], rg, form);
            acc[i][j] = dequant_level(q[j], rg, form);
          }
          if (mean_codes) store_codes8(mean_codes + row * row_bytes, c, q, bits, form.code_bias);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = (t + i * G) * 8;
      if (live && c < n) {
        float uv[8];
        load8<float, RAG>(u + rbase + c, n - c, uv);
#pragma unroll
        for (int j = 0; j < 8; ++j) outer_update<GT>(tg[i][j], uv[j], acc[i][j], eta, mu, nesterov);
        store8<GT, RAG>(theta_g + rbase + c, tg[i], n - c);
        store8<float, RAG>(u + rbase + c, uv, n - c);
        if (write_back)
          for (int k = 0; k < K; ++k) store8<WT, RAG>(reinterpret_cast<WT*>(w.p[k]) + rbase + c, tg[i], n - c);
      }
    }
  }
}

// Wavefronts per SIMD the register allocation is held to: one more than the compiler reaches on
// its own where that is a few registers away (these kernels wait on memory with little else to
// do, so a resident wavefront more is worth more than the registers).  Not so the update of ragged rows with four vectors, whose loop
// over the workers spilt up to 57 of them (2 x 1402 x 4096 and its squares, eight workers of float32, 799 us, now 531), unless
// three make do with one round of workgroups where two need another (quant_three_waves).
constexpr int quant_min_waves(int nv, bool outer, bool ragged) {
  return outer ? (nv <= 1 ? 6 : nv <= 2 ? 4 : nv <= 4 ? (ragged ? 2 : 3) : 1) : (nv <= 1 ? 7 : nv <= 2 ? 5 : nv <= 4 ? 3 : 1);
}

template <typename WT, typename GT, int NV, int G, bool OUTER, bool RAG, int MW = quant_min_waves(NV, OUTER, RAG)>
__global__ __launch_bounds__(G ? OT_THREADS : 1024, MW) void quantize_rows_reg_kernel(
    WorkerPtrs w, GT* __restrict__ theta_g, float* __restrict__ u, CodePtrs codes, ScalePtrs scales,
    OffsetPtrs offsets, ResidualPtrs ef, long rows, int n, int K, QuantForm form, float eta, float mu,
    float inv_k, int nesterov, int write_back, int requant, uint8_t* mean_codes, float* mean_scales,
    float* mean_offsets) {
  quantize_rows_reg_body<WT, GT, NV, G, OUTER, RAG, 0, true>(w, theta_g, u, codes, scales, offsets, ef, rows, n, K, form,
                                               eta, mu, inv_k, nesterov, write_back, requant, mean_codes,
                                               mean_scales, mean_offsets, (long)blockIdx.x);
}

// ---- one launch over several groups ----------------------------------------------------
// A streaming fragment (one transformer layer: three shape groups) is small enough that
// three launches of 70-80 us each spend a good part of their time filling and draining the
// chip; here the workgroups of one launch are dealt to the groups of a table that travels in
// the kernel arguments (up to OUTER_MAX_SEG groups, OUTER_MAX_SEG_K workers).
struct QuantSeg {
  SegPtrs<void*> w;
  SegPtrs<uint8_t*> codes;
  SegPtrs<float*> scales, offsets, ef;
  void* theta_g;
  float* u;
  long rows;
  int n;
  int rows_per_range;       // as in QuantForm
  int cfg;                  // index into the (vectors per thread, threads per row) table below
  unsigned int blk0;        // first workgroup of this group
};
struct QuantSegTable { QuantSeg s[OUTER_MAX_SEG]; int nseg; };

// Vectors per thread and threads per row in a launch that several groups share (its workgroups have 256 threads, so
// none is of its row's size)
struct RegCfg { int nv, g; };
__host__ __device__ constexpr RegCfg reg_cfg(int idx) {
  return idx == 0 ? RegCfg{1, 64} : idx == 1 ? RegCfg{2, 64} : idx == 2 ? RegCfg{4, 64}
       : idx == 3 ? RegCfg{2, 256} : RegCfg{4, 256};
}

// TOP: which entries of the table above the groups use: the first, the first two, those of four vectors (4) or any (5).
template <typename WT, typename GT, bool RAG, int KC, int TOP>
__device__ __forceinline__ void quantize_outer_multi_body(const QuantSegTable& tab, int K, QuantForm form, float eta, float mu,
                                                          float inv_k, int nesterov, int write_back) {
  int si = 0;
#pragma unroll
  for (int i = 1; i < OUTER_MAX_SEG; ++i)
    if (i < tab.nseg && blockIdx.x >= tab.s[i].blk0) si = i;
  const QuantSeg& sg = tab.s[si];
  form.rows_per_range = sg.rows_per_range;
  const long blk = (long)(blockIdx.x - sg.blk0);
#define MLC_SEG_BODY(IDX)                                                                              \
  quantize_rows_reg_body<WT, GT, reg_cfg(IDX).nv, reg_cfg(IDX).g, true, RAG, KC, (reg_cfg(IDX).nv == 4)>(                             \
      sg.w, (GT*)sg.theta_g, sg.u, sg.codes, sg.scales, sg.offsets, sg.ef, sg.rows, sg.n, K, form, eta, \
      mu, inv_k, nesterov, write_back, 0, nullptr, nullptr, nullptr, blk)
  // uniform over the workgroup
  if constexpr (TOP == 0) {
    MLC_SEG_BODY(0);
  } else if constexpr (TOP == 1) {
    if (sg.cfg == 0) MLC_SEG_BODY(0);
    else MLC_SEG_BODY(1);
  } else if constexpr (TOP == 4) {
    if (sg.cfg == 2) MLC_SEG_BODY(2);
    else MLC_SEG_BODY(4);
  } else {
    switch (sg.cfg) {
      case 0: MLC_SEG_BODY(0); break;
      case 1: MLC_SEG_BODY(1); break;
      case 2: MLC_SEG_BODY(2); break;
      case 3: MLC_SEG_BODY(3); break;
      default: MLC_SEG_BODY(4); break;
    }
  }
#undef MLC_SEG_BODY
}

// (Three wavefronts a SIMD: more of them, which one worker's registers would allow, make its long rows 1 to 2 % slower.)
template <typename WT, typename GT, bool RAG, int KC>
__global__ __launch_bounds__(OT_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3))) void quantize_outer_multi_kernel(
    QuantSegTable tab, int K, QuantForm form, float eta, float mu, float inv_k, int nesterov, int write_back) {
  quantize_outer_multi_body<WT, GT, RAG, KC, 5>(tab, K, form, eta, mu, inv_k, nesterov, write_back);
}

// Rows of up to 512 (TOP 0) or 1024 columns: as many wavefronts a SIMD as their registers allow, where the kernel of
// all lengths has three.  160 / 40 / 40 matrices of 128 x 128, 128 x 256 and 256 x 128, 4 bits, us: one worker 37 to 31, two 53 to 39, eight
// 138 to 96, with error feedback 273 to 173; 24 / 6 / 6 of 512 x 512 and 512 x 1024, eight workers 174 to 153, with error feedback 296
// to 299 (where the memory stream bounds both); 800 / 200 / 200 of 303 x 303 and 303 x 831, 8 bits, one worker 1097 to 988, which ranges per
// matrix in launches of a group each, with registers for their own rows alone, would do in 899.
// Or, TOP 4, ragged rows of four vectors a thread alone: two wavefronts a SIMD, since for three 60 and more registers of the loop over the
// workers go to memory (8 / 2 / 2 of 1402 x 1402 and 1402 x 4098, eight workers of float32, 846 to 574; two of bf16 with error
// feedback 442 to 383; next to rows of two vectors, 606 and 1818 columns, it would be 341 to 378).
template <typename WT, typename GT, bool RAG, int TOP, int MW = quant_min_waves(reg_cfg(TOP).nv, true, RAG)>
__global__ __launch_bounds__(OT_THREADS, MW) void quantize_outer_narrow_kernel(
    QuantSegTable tab, int K, QuantForm form, float eta, float mu, float inv_k, int nesterov, int write_back) {
  quantize_outer_multi_body<WT, GT, RAG, 0, TOP>(tab, K, form, eta, mu, inv_k, nesterov, write_back);
}

struct OuterSeg {
  SegPtrs<void*> w;
  void* theta_g;
  float* u;
  long n_elems;
  unsigned int blk0, nblk;
};
struct OuterSegTable { OuterSeg s[OUTER_MAX_SEG]; int nseg; };

template <typename WT, typename GT>
__global__ __launch_bounds__(OT_THREADS) void outer_fused_multi_kernel(
    OuterSegTable tab, int K, float eta, float mu, float inv_k, int nesterov, int write_back) {
  int si = 0;
#pragma unroll
  for (int i = 1; i < OUTER_MAX_SEG; ++i)
    if (i < tab.nseg && blockIdx.x >= tab.s[i].blk0) si = i;
  const OuterSeg& sg = tab.s[si];
  outer_fused_body<WT, GT>(sg.w, (GT*)sg.theta_g, sg.u, sg.n_elems, K, eta, mu, inv_k, nesterov, write_back,
                           (long)(blockIdx.x - sg.blk0), (long)sg.nblk);
}

// ---- dequantise + average + outer update --------------------------------------------
template <typename WT, typename GT, bool VEC>
__global__ __launch_bounds__(OT_THREADS) void dequant_outer_kernel(
    WorkerPtrs w, GT* __restrict__ theta_g, float* __restrict__ u, CodePtrs codes, ScalePtrs scales,
    OffsetPtrs offsets, long rows, int n, int K, QuantForm form, float eta, float mu, float inv_k,
    int nesterov, int write_back) {
  const int bits = form.bits;
  const int W = VEC ? 8 : 8 / bits;
  const int per_row = n / W;
  const long items = rows * per_row;
  const long row_bytes = (long)n * bits / 8;
  for (long i = (long)blockIdx.x * OT_THREADS + threadIdx.x; i < items;
       i += (long)gridDim.x * OT_THREADS) {
    const long row = i / per_row;
    const int c = (int)(i - row * per_row) * W;
    const long off = row * n + c;
    const long grp = form.rows_per_range ? row / form.rows_per_range : row;
    float tg[8], uv[8], acc[8];
    if (VEC) { Vec8<GT>::load(theta_g + off, tg); Vec8<float>::load(u + off, uv); }
    else
      for (int j = 0; j < W; ++j) { tg[j] = Vec8<GT>::load1(theta_g + off + j); uv[j] = u[off + j]; }
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    for (int k = 0; k < K; ++k) {
      const Range rg = stored_range(scales, offsets, k, grp, form);
      const uint8_t* crow = codes.p[k] + row * row_bytes;
      int q[8];
      if (VEC) {
        load_levels8(crow, c, q, bits, form.code_bias);
      } else {
        const unsigned int p = crow[c / W];
        for (int j = 0; j < W; ++j) q[j] = (int)((p >> (bits * j)) & ((1u << bits) - 1u)) - form.code_bias;
      }
      for (int j = 0; j < W; ++j) acc[j] += dequant_level(q[j], rg, form);
    }
    for (int j = 0; j < W; ++j) outer_update<GT>(tg[j], uv[j], __fmul_rn(acc[j], inv_k), eta, mu, nesterov);
    if (VEC) {
      Vec8<GT>::store(theta_g + off, tg);
      Vec8<float>::store(u + off, uv);
      if (write_back)
        for (int k = 0; k < K; ++k) Vec8<WT>::store(reinterpret_cast<WT*>(w.p[k]) + off, tg);
    } else {
      for (int j = 0; j < W; ++j) {
        Vec8<GT>::store1(theta_g + off + j, tg[j]);
        u[off + j] = uv[j];
        if (write_back)
          for (int k = 0; k < K; ++k) Vec8<WT>::store1(reinterpret_cast<WT*>(w.p[k]) + off + j, tg[j]);
      }
    }
  }
}

// ---- top-k sparsification (Sec. 2 "Compressed Communication") --------------------------
// Of each matrix of each worker the k entries of largest magnitude are kept (all entries
// that tie with the k-th one, tau, included).  Magnitudes are compared as the bit patterns of |v|
// (ordered like unsigned numbers; bit 31 is always clear).  The state of a (worker, matrix) pair is
// an interval of 2^width such keys from `lo` on that holds tau's, and tau's rank in it; a pass over
// the values counts those of the interval in up to 2048 bins, and the workgroup that ends last, or a launch of its own,
// narrows the interval to the bin that holds tau.  Three passes lead from all 2^31 keys to one.
//
// Large matrices and groups (topk_window) start from an interval that a sample of 16384 values suggests, which the pass that
// computes v counts in bins of its own.  Where the bin that holds tau has at most TOPK_LIST values for every
// worker, the update of the matrix follows at once: values above the interval are sent, those
// below are not, and the few inside are listed and left as they are, for topk_threshold to select
// tau among them exactly and topk_settle to update their elements.  The values are then read twice in all.
//
// What this leaves open goes through up to three further passes, one where the bin was merely too full: equal
// magnitudes (bf16 replicas of a bf16 global copy), and matrices too large for bins that a fixed sample spreads.  Normally
// distributed values settle up to 67 M at 2 % and less, 50 M at 5 %, 33 M at 10 % and 25 M at 20 %; of 110 M (5120 x
// 20480) at 5 % and of 67 M (4096 x 16384) at 20 % none do.  A sample misleads seldom: in none of 2900 draws of matrices with normal, heavy-tailed
// or row- or column-scaled values, in 2 of 100 where each 8 adjacent magnitudes are alike.
//
// All of this is bound by memory, per element with error feedback (bf16 replicas, fp32 global copy): 14 bytes in the
// window's pass and 26 in the update, and 4 a further pass; by passes from the start 48.  Against those: six layers of
// 2048 / 8192, one worker, 5 %, 2873 -> 2520 us; 4096 x 16384 at 20 % and left open 745 -> 588; 24 matrices of 2048 x 2048
// 921 -> 808, whose magnitudes all tie 906 -> 790, and 925 -> 1046 if all are misled about.
constexpr int TOPK_LIST = (TOPK_BINS - 2) / 2;     // primaries of two words and the two counts fit the histogram
constexpr int TOPK_WINDOW = TOPK_BINS - 1;         // bins of the first pass; the last word counts what is above
constexpr unsigned int TOPK_EARLY = 1u << 31;      // in ctl: the pass over the window left few enough values;
constexpr unsigned int TOPK_OPEN = 1u << 30;       // in the group's first ctl: for some state it did not
constexpr unsigned int TOPK_TICKETS = 0xffffu;     // in ctl: workgroups that have ended a pass over the state
constexpr int TOPK_WINDOW_THREADS = 1024;
constexpr int TOPK_SAMPLE_THREADS = 1024;
constexpr int TOPK_SAMPLE_PER = 2;                 // runs of 8 values that a thread of the sample reads

__device__ __forceinline__ unsigned int magnitude_key(float v) { return __float_as_uint(fabsf(v)); }

// Pointers of the G groups of a launch, one or two of equally large matrices, which are numbered through: those of the second
// group are the addresses that matrix 0 would have, so that matrix b's are found alike in both.
//
// A group alone has kernels without the choice: its pointers are then requested with the other arguments, not in a second trip to
// them, which every workgroup waits for (us with the choice and without, one worker and 48 of 32 x 32 and 12 of 32 x 34 45.4 and 43.8;
// four and 4 of 128 x 128 and one of 128 x 232 51.1 and 46.8; four and 800 of 112 x 112 253 and 244).
struct TopkPtrs { WorkerPtrs w; ResidualPtrs ef; ScalePtrs thresholds; void* theta_g; float* u; };
template <int G>
struct TopkArgs {
  TopkPtrs g[G];
  int split;                         // first matrix of the second group
  __device__ __forceinline__ const TopkPtrs& of(long b) const { return g[G > 1 && b >= split ? 1 : 0]; }
};

__global__ void topk_init_kernel(TopkState* st, unsigned int kcount) {
  TopkState& s = st[blockIdx.x];
  for (int i = threadIdx.x; i < TOPK_BINS; i += blockDim.x) s.hist[i] = 0u;
  if (threadIdx.x == 0) { s.lo = 0u; s.width = 31u; s.rank = kcount; s.ctl = 0u; }
}

// The 8 values v of worker k from element i on (`left` of them before the end of the matrix).
template <typename WT, typename GT, bool VEC>
__device__ __forceinline__ void topk_values(const GT* tg, const WT* tk, const float* res, long i, int left,
                                            float ef_beta, float (&vals)[8]) {
  float a[8], c[8];
  load8<GT, !VEC>(tg + i, left, a); load8<WT, !VEC>(tk + i, left, c);
#pragma unroll
  for (int j = 0; j < 8; ++j) vals[j] = a[j] - c[j];
  if (res) {
    float e[8];
    load8<float, !VEC>(res + i, left, e);
#pragma unroll
    for (int j = 0; j < 8; ++j) vals[j] = ef_input(vals[j], e[j], ef_beta);
  }
}

// Bin of a sampled key: 32 to an octave over the 64 octaves below 2^5; what is smaller or larger
// falls into the first or the last bin.
constexpr unsigned int TOPK_SAMPLE_BASE = (127u - 59u) << 23;
__device__ __forceinline__ unsigned int sample_bin(unsigned int key) {
  return key < TOPK_SAMPLE_BASE ? 0u : min((key - TOPK_SAMPLE_BASE) >> 18, (unsigned int)TOPK_BINS - 1u);
}

// First interval of each state, one workgroup each, from a histogram of 2048 runs of 8 values, one from each
// of 2048 equal stretches of the matrix at a place that a hash picks (a fixed stride would meet the same
// columns again and again): the keys from five standard deviations of a sample's rank below
// the rank sought to as many above, at the resolution of the bins.  Where so many magnitudes tie that they fill all of
// that (replicas that did not move), the interval is one key and the pass over the window settles it.
template <typename WT, typename GT, bool VEC, int G>
__global__ __launch_bounds__(TOPK_SAMPLE_THREADS) void topk_sample_kernel(
    TopkArgs<G> args, TopkState* st, long elems, int count, unsigned int kcount, float ef_beta) {
  constexpr int WAVES = TOPK_SAMPLE_THREADS / 64, RUNS = TOPK_SAMPLE_THREADS * TOPK_SAMPLE_PER;
  static_assert(TOPK_BINS == 2 * TOPK_SAMPLE_THREADS, "a thread owns two bins");
  __shared__ unsigned int hist[TOPK_BINS];
  __shared__ unsigned int part[WAVES], first, last, least, most;
  const long b = blockIdx.x;
  const int k = blockIdx.y, t = threadIdx.x;
  TopkState& s = st[(long)k * count + b];
  const TopkPtrs& g = args.of(b);
  const GT* tg = reinterpret_cast<const GT*>(g.theta_g) + b * elems;
  const WT* tk = reinterpret_cast<const WT*>(g.w.p[k]) + b * elems;
  const float* res = g.ef.p[k] ? g.ef.p[k] + b * elems : nullptr;
  const unsigned int stretch = (unsigned int)(elems / 8 / RUNS);           // >= 1, below 2^18
  hist[t] = 0u; hist[t + TOPK_SAMPLE_THREADS] = 0u;
  s.hist[t] = 0u; s.hist[t + TOPK_SAMPLE_THREADS] = 0u;
  if (t == 0) { first = 0u; last = TOPK_BINS - 1; least = ~0u; most = 0u; }
  float v[TOPK_SAMPLE_PER][8];
#pragma unroll
  for (int c = 0; c < TOPK_SAMPLE_PER; ++c) {
    const unsigned int r = (unsigned int)(c * TOPK_SAMPLE_THREADS + t);
    unsigned int h = r * 2654435761u;
    h = (h ^ (h >> 15)) * 2246822519u;
    const long at = (long)r * stretch + __umulhi(h, stretch);
    topk_values<WT, GT, VEC>(tg, tk, res, at * 8, 8, ef_beta, v[c]);
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < TOPK_SAMPLE_PER; ++c)
#pragma unroll
    for (int j = 0; j < 8; ++j) atomicAdd(&hist[sample_bin(magnitude_key(v[c][j]))], 1u);
  __syncthreads();
  const unsigned int h0 = hist[2 * t], h1 = hist[2 * t + 1];
  unsigned int from = h0 + h1;                   // entries of this lane and the lanes above it
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned int add = __shfl_down(from, off, 64);
    if ((t & 63) + off < 64) from += add;
  }
  if ((t & 63) == 0) part[t >> 6] = from;
  __syncthreads();
  for (int wv = (t >> 6) + 1; wv < WAVES; ++wv) from += part[wv];
  const float share = (float)kcount / (float)elems;
  const float mean = share * (RUNS * 8);
  const float margin = 5.f * sqrtf(mean * (1.f - share)) + 12.f;
  const unsigned int few = (unsigned int)fmaxf(mean - margin, 0.f), many = (unsigned int)(mean + margin);
  // the lowest bin that `many` entries reach, and the highest that more than `few` do
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const unsigned int upto = i ? h1 + from - h0 - h1 : from, beyond = i ? from - h0 - h1 : from - h0;
    if (beyond < many && upto >= many) first = (unsigned int)(2 * t + i);
    if (beyond <= few && upto > few) last = (unsigned int)(2 * t + i);
  }
  __syncthreads();
  // the lowest key sampled in the first of these bins and the highest in the last: one key, where many tie
  const unsigned int low = first, high = last;
  unsigned int min_key = ~0u, max_key = 0u;
#pragma unroll
  for (int c = 0; c < TOPK_SAMPLE_PER; ++c)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const unsigned int key = magnitude_key(v[c][j]), at = sample_bin(key);
      if (at == low) min_key = min(min_key, key);
      if (at == high) max_key = max(max_key, key);
    }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    min_key = min(min_key, (unsigned int)__shfl_xor((int)min_key, off, 64));
    max_key = max(max_key, (unsigned int)__shfl_xor((int)max_key, off, 64));
  }
  if ((t & 63) == 0) { atomicMin(&least, min_key); atomicMax(&most, max_key); }
  __syncthreads();
  if (t == 0) {
    // a rank outside the sample: from 0 on, or to four times the largest
    const unsigned int lo = many > RUNS * 8 ? 0u : least;
    const unsigned int keys = most + (few ? 1u : 1u << 24) - lo;
    unsigned int shift = 0u;
    while (shift < 20u && (keys + (1u << shift) - 1u) >> shift > (unsigned int)TOPK_WINDOW) ++shift;
    s.lo = lo; s.width = shift; s.rank = kcount; s.ctl = 0u;
  }
}

// True in every thread of the workgroup of `n` that comes last to this state.  What the
// workgroups hand over are atomic sums at device scope: each thread's have been performed when its wait returns,
// so they precede the workgroup's ticket.  (A release fence would also write back
// the L2 cache, which holds the values that the pass has just stored.)
__device__ __forceinline__ bool last_of_state(TopkState& s, unsigned int n) {
  __shared__ unsigned int ticket;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) ticket = __hip_atomic_fetch_add(&s.ctl, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  return (ticket & TOPK_TICKETS) == n - 1;
}

// The interval is narrowed: `nbins` bins of 2^shift keys from s.lo on have been counted; the one that
// holds the rank-th largest entry is the new interval.  Thread t owns 8 adjacent bins, or 4 of 1024.
// By the workgroup that ends the pass over the window (the last word holds the number of entries above all bins; where tau
// is not in any bin, the interval becomes all keys; st: the group's states) or another pass last, or in a
// launch of its own, which needs no atomics.
enum Narrow { WINDOW_LAST, PASS_LAST, OWN_LAUNCH };
template <Narrow BY>
__device__ __forceinline__ void topk_narrow(TopkState& s, int nbins, int shift, TopkState* st) {
  constexpr bool WINDOW = BY == WINDOW_LAST;
  __shared__ unsigned int part[OT_THREADS / 64];  // entries in the bins of a wavefront
  constexpr int PER = TOPK_BINS / OT_THREADS;
  const int t = threadIdx.x, per = WINDOW || nbins > TOPK_BINS / 2 ? PER : PER / 2;
  const bool owns = t < OT_THREADS;
  unsigned int h[PER] = {};
  unsigned int mine = 0u, beyond = 0u;
  if (owns) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (i >= per) break;
      h[i] = BY == OWN_LAUNCH ? s.hist[t * per + i]
                              : __hip_atomic_load(&s.hist[t * per + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (WINDOW && i == PER - 1 && t == OT_THREADS - 1) h[i] = 0u;
      mine += h[i];
    }
  }
  if (WINDOW) beyond = __hip_atomic_load(&s.hist[TOPK_WINDOW], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned int rank = s.rank, lo = s.lo;
  unsigned int upto = mine;                                   // entries in the bins of this lane and those above it
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned int add = __shfl_down(upto, off, 64);
    if ((t & 63) + off < 64) upto += add;
  }
  if (owns && (t & 63) == 0) part[t >> 6] = upto;
  __syncthreads();                                            // and everyone has read the state
  unsigned int total = 0u, above = beyond + upto - mine;      // entries above the bins of thread t
#pragma unroll
  for (int wv = 0; wv < OT_THREADS / 64; ++wv) {
    total += part[wv];
    if (wv > t >> 6) above += part[wv];
  }
  if (!owns) return;
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (i < per) s.hist[t * per + i] = 0u;                    // for the next pass, or the counts of the list
  if (BY == PASS_LAST && t == 0)
    __hip_atomic_fetch_and(&s.ctl, ~TOPK_TICKETS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  auto set_early = [&](bool early) {
    if (&s != st) {
      s.ctl = early ? TOPK_EARLY : 0u;
    } else {                       // other states' workgroups may be setting TOPK_OPEN in this word
      __hip_atomic_fetch_and(&s.ctl, ~TOPK_TICKETS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (early) __hip_atomic_fetch_or(&s.ctl, TOPK_EARLY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!early) __hip_atomic_fetch_or(&st->ctl, TOPK_OPEN, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if (WINDOW && (beyond >= rank || beyond + total < rank)) {
    if (t == 0) { s.lo = 0u; s.width = 31u; set_early(false); }
  } else if (above < rank && above + mine >= rank) {
    unsigned int ab = above, held = h[0];
    int pick = 0;
    bool found = false;
#pragma unroll
    for (int i = PER - 1; i >= 0; --i) {
      if (!found) {
        if (ab + h[i] >= rank) { pick = i; held = h[i]; found = true; }
        else ab += h[i];
      }
    }
    s.lo = lo + ((unsigned int)(t * per + pick) << shift);
    s.width = (unsigned int)shift;
    s.rank = rank - ab;
    if (WINDOW) set_early(held <= (unsigned int)TOPK_LIST || shift == 0);
  }
}

// The pass that computes v = beta E + (theta_g - theta_k) of every matrix and counts it in the window.
// With error feedback it leaves v in E, where it ends up anyway unless it is sent: the update then reads
// 4 bytes an element instead of 6 and needs no worker parameters.  A few per cent of the values fall
// into the window, so one histogram a workgroup takes them; 16 wavefronts share it, since its
// bins leave as one atomic each at the end (4 wavefronts: 0 to 3 % slower).  14 bytes an element at 4.8 TB/s.
// TURN: the grid's first dimension is the workers, otherwise the pieces of a matrix (topk_turn).
template <typename WT, typename GT, bool VEC, bool TURN, int G>
__global__ __launch_bounds__(TOPK_WINDOW_THREADS) void topk_window_kernel(
    TopkArgs<G> args, TopkState* st, long elems, int count, float ef_beta) {
  __shared__ unsigned int lh[TOPK_BINS];
  const long b = TURN ? blockIdx.z : blockIdx.y;
  const int k = TURN ? blockIdx.x : blockIdx.z, blk = TURN ? blockIdx.y : blockIdx.x, nblk = TURN ? gridDim.y : gridDim.x;
  TopkState& s = st[(long)k * count + b];
  const unsigned int lo = s.lo, shift = s.width;
  for (int i = threadIdx.x; i < TOPK_BINS; i += TOPK_WINDOW_THREADS) lh[i] = 0u;
  __syncthreads();
  const TopkPtrs& g = args.of(b);
  const GT* tg = reinterpret_cast<const GT*>(g.theta_g) + b * elems;
  const WT* tk = reinterpret_cast<const WT*>(g.w.p[k]) + b * elems;
  float* res = g.ef.p[k] ? g.ef.p[k] + b * elems : nullptr;
  unsigned int above = 0u;
  for (long i = ((long)blk * TOPK_WINDOW_THREADS + threadIdx.x) * 8; i < elems;
       i += (long)nblk * TOPK_WINDOW_THREADS * 8) {
    float vals[8];
    const int left = (int)min(elems - i, 8L);
    topk_values<WT, GT, VEC>(tg, tk, res, i, left, ef_beta, vals);
    if (res) store8<float, !VEC>(res + i, vals, left);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (!VEC && j >= left) break;
      const unsigned int key = magnitude_key(vals[j]);
      const unsigned int at = (key - lo) >> shift;        // a key below lo wraps round to 2^31 and more
      const bool in = at < (unsigned int)TOPK_WINDOW;
      above += !in && key >= lo ? 1u : 0u;
      const unsigned long lanes = __ballot(in);
      if (__popcll(lanes) < 16) {
        if (in) atomicAdd(&lh[at], 1u);
      } else {                                            // many equal magnitudes: those of one bin at once
        const int head = __builtin_ctzl(lanes);
        const unsigned int bin = (unsigned int)__builtin_amdgcn_readlane((int)at, head);
        const unsigned long same = __ballot(in && at == bin);
        if ((int)(threadIdx.x & 63) == head) atomicAdd(&lh[bin], (unsigned int)__popcll(same));
        if (in && at != bin) atomicAdd(&lh[at], 1u);
      }
    }
  }
  if (above) atomicAdd(&lh[TOPK_WINDOW], above);
  __syncthreads();
  for (int i = threadIdx.x; i < TOPK_BINS; i += TOPK_WINDOW_THREADS)
    if (lh[i]) __hip_atomic_fetch_add(&s.hist[i], lh[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (last_of_state(s, nblk)) topk_narrow<WINDOW_LAST>(s, TOPK_BINS, (int)shift, st);
}

// The first digits (bits from `shift` up) of a lane's first cnt of 8 values.  They mostly change
// from element to element, so each is counted by itself (counting runs took 335 us a pass instead
// of 290); zeros, of which a step that moved little has many, are left to the lane's `zeros`.  Where
// a quarter of the wavefront starts with one digit (replicas that all moved by about the same amount),
// that digit and the next one met are counted for the wavefront by one lane: the LDS takes atomics
// on one counter one after the other (24 matrices of 2048 x 2048, all magnitudes equal: 875 us a
// call without this, 683 with it; normal values: 700 either way).
__device__ __forceinline__ void count_first_digit(unsigned int* hist, const float (&vals)[8], int cnt, int shift,
                                                  unsigned int& zeros) {
  unsigned int key[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) key[j] = magnitude_key(vals[j]);
  const unsigned int mine = key[0] >> shift;
  const unsigned int d0 = (unsigned int)__builtin_amdgcn_readfirstlane((int)mine);
  if (__popcll(__ballot(mine == d0)) < 16) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (j >= cnt) break;
      if (key[j] == 0u) ++zeros;
      else atomicAdd(&hist[key[j] >> shift], 1u);
    }
    return;
  }
  const unsigned long other = __ballot(mine != d0);
  const unsigned int d1 =
      other ? (unsigned int)__builtin_amdgcn_readlane((int)mine, __builtin_ctzl(other)) : 0xffffffffu;
  unsigned int n0 = 0u, n1 = 0u;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const unsigned int d = key[j] >> shift;
    const bool in = j < cnt;
    n0 += (unsigned int)__popcll(__ballot(in && d == d0));
    n1 += (unsigned int)__popcll(__ballot(in && d == d1));
    if (in && d != d0 && d != d1) atomicAdd(&hist[d], 1u);
  }
  if ((int)(threadIdx.x & 63) == __builtin_ctzl(__ballot(true))) {
    atomicAdd(&hist[d0], n0);
    if (n1) atomicAdd(&hist[d1], n1);
  }
}

// Did the pass over the window leave few enough values of this matrix for this worker?  (Later passes do not touch the
// bit.)
__device__ __forceinline__ bool state_early(const TopkState& s) {
  return (__hip_atomic_load(&s.ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & TOPK_EARLY) != 0u;
}

// And of matrix b for every worker?  A whole workgroup asks, and the workers' bits are read at the same time.
__device__ __forceinline__ bool topk_early(const TopkState* st, long b, int count, int K) {
  return __syncthreads_and((int)threadIdx.x >= K || state_early(st[(long)threadIdx.x * count + b])) != 0;
}

// And of all matrices of the group?  (One word: with the bits of all states read by every workgroup, 1000 matrices of
// 256 x 256, eight workers, took 2510 us instead of 2410.)
__device__ __forceinline__ bool topk_all_early(const TopkState* st) {
  return (__hip_atomic_load(&st->ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & TOPK_OPEN) == 0u;
}

// The launches behind a window have one grid for the whole group, whose workgroups share what is left between them:
// mostly nothing, one matrix of many, or all of them.  The matrices that the window left open are listed
// 256 at a time, the same in every workgroup, and each of their `parts` is split over as many workgroups as there
// are for it, `most` at the most.  work(matrix, part, workgroup, workgroups) is called by whole workgroups.
// (With an equal share of 1024 workgroups for every state, open or not: 6 matrices of 2048 x 2048, eight bf16 workers and
// a bf16 global copy, whose ties the window does not settle, 1125 us, now 579; 4096 x 16384, eight workers, 20 % without
// error feedback, 2627, now 1435; one open matrix of 64 of 768 x 768, eight workers, 2688, now 1717.)
constexpr int TOPK_LATE_GRID = 1024, TOPK_FINISH_GRID = 2048;
// Workgroups for the elements that wait, at least one a matrix.  (Those that find none are not free: 24 matrices of 2048 x
// 2048, eight workers, 18 us with four a matrix, 27 with 16, 63 with 64.)
constexpr int TOPK_SETTLE_GRID = 128, TOPK_SETTLE_MOST = 64;
template <typename Work>
__device__ __forceinline__ void topk_each_open(const TopkState* st, int count, int K, int parts, int most,
                                               Work&& work) {
  __shared__ unsigned int open[OT_THREADS], waves[OT_THREADS / 64];
  const int t = threadIdx.x;
  unsigned int dealt = 0u;                  // items of the matrices listed before
  for (int b0 = 0; b0 < count; b0 += OT_THREADS) {
    const int nb = min(count - b0, OT_THREADS);
    open[t] = 0u;
    __syncthreads();
    for (int i = t; i < nb * K; i += OT_THREADS) {
      const int k = i / nb, b = i - k * nb;
      if (!state_early(st[(long)k * count + b0 + b])) open[b] = 1u;
    }
    __syncthreads();
    const bool is_open = open[t] != 0u;
    const unsigned long lanes = __ballot(is_open);
    if ((t & 63) == 0) waves[t >> 6] = (unsigned int)__popcll(lanes);
    __syncthreads();
    int at = __popcll(lanes & ((1ul << (t & 63)) - 1ul)), n = 0;
#pragma unroll
    for (int wv = 0; wv < OT_THREADS / 64; ++wv) {
      if (wv < t >> 6) at += (int)waves[wv];
      n += (int)waves[wv];
    }
    if (is_open) open[at] = (unsigned int)(b0 + t);
    __syncthreads();
    const unsigned int states = (unsigned int)(n * parts), grid = gridDim.x;
    const unsigned int share = states ? min(max(grid / states, 1u), (unsigned int)most) : 1u;
    // item i of the group goes to workgroup i % grid
    const unsigned int behind = dealt % grid;
    for (unsigned int i = blockIdx.x >= behind ? blockIdx.x - behind : blockIdx.x + grid - behind; i < states * share;
         i += grid) {
      const unsigned int state = i / share, m = state / (unsigned int)parts;
      work((long)open[m], (int)(state - m * parts), (int)(i - state * share), (int)share);
      __syncthreads();                      // its shared memory may be written again
    }
    dealt += states * share;
    __syncthreads();
  }
}

// Digits of 11, 10 and 10 bits, by the width of the interval.
__device__ __forceinline__ int topk_shift(unsigned int width) { return width > 20u ? 20 : width > 10u ? 10 : 0; }

// One pass of the radix select over a state's interval, by workgroup blk of nblk.  FIRST: the pass over all keys that
// computes v, where no window was tried (with error feedback it leaves v in E).  `pick`: the workgroup that ends last narrows
// the interval; otherwise topk_pick_kernel does.
template <typename WT, typename GT, bool VEC, bool FIRST>
__device__ __forceinline__ void topk_count(const WorkerPtrs& w, const GT* __restrict__ theta_g, const ResidualPtrs& ef,
                                           TopkState& s, unsigned int (&lh)[OT_THREADS / 64][TOPK_BINS], long elems,
                                           long b, int k, float ef_beta, int blk, int nblk, bool pick) {
  const unsigned int lo = FIRST ? 0u : s.lo, width = FIRST ? 31u : s.width;
  const int shift = topk_shift(width);
  const int nbins = 1 << (width - shift);
  for (int wv = 0; wv < OT_THREADS / 64; ++wv)
    for (int i = threadIdx.x; i < nbins; i += OT_THREADS) lh[wv][i] = 0u;
  __syncthreads();
  unsigned int* mine = lh[threadIdx.x >> 6];
  const GT* tg = theta_g + b * elems;
  const WT* tk = reinterpret_cast<const WT*>(w.p[k]) + b * elems;
  float* res = ef.p[k] ? ef.p[k] + b * elems : nullptr;
  unsigned int cur = FIRST ? 0u : 0xffffffffu, run = 0u;       // run-length of the current digit
  for (long i = ((long)blk * OT_THREADS + threadIdx.x) * 8; i < elems;
       i += (long)nblk * OT_THREADS * 8) {
    float vals[8];
    const int left = (int)min(elems - i, 8L);
    if (!FIRST && res) {
      load8<float, !VEC>(res + i, left, vals);
    } else {
      topk_values<WT, GT, VEC>(tg, tk, res, i, left, ef_beta, vals);
      if (res) store8<float, !VEC>(res + i, vals, left);
    }
    if constexpr (FIRST) {
      count_first_digit(mine, vals, VEC ? 8 : left, shift, run);
      continue;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (!VEC && j >= left) break;
      const unsigned int at = magnitude_key(vals[j]) - lo;
      if (at >> width == 0u) {
        const unsigned int bin = at >> shift;
        if (bin == cur) {
          ++run;
        } else {
          if (run) atomicAdd(&mine[cur], run);
          cur = bin; run = 1u;
        }
      }
    }
  }
  if (run) atomicAdd(&mine[cur], run);
  __syncthreads();
  for (int i = threadIdx.x; i < nbins; i += OT_THREADS) {
    unsigned int tot = 0u;
#pragma unroll
    for (int wv = 0; wv < OT_THREADS / 64; ++wv) tot += lh[wv][i];
    if (tot) __hip_atomic_fetch_add(&s.hist[i], tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (pick && last_of_state(s, (unsigned int)nblk)) topk_narrow<PASS_LAST>(s, nbins, shift, nullptr);
}

template <typename WT, typename GT, bool VEC, bool FIRST, int G>
__global__ __launch_bounds__(OT_THREADS) void topk_hist_kernel(
    TopkArgs<G> args, TopkState* st, long elems, int count, float ef_beta, int pick) {
  __shared__ unsigned int lh[OT_THREADS / 64][TOPK_BINS];     // one histogram per wavefront
  const long b = blockIdx.y;
  const int k = blockIdx.z;
  const TopkPtrs& g = args.of(b);
  topk_count<WT, GT, VEC, FIRST>(g.w, (const GT*)g.theta_g, g.ef, st[(long)k * count + b], lh, elems, b, k, ef_beta, blockIdx.x,
                                 gridDim.x, pick != 0);
}

__global__ __launch_bounds__(OT_THREADS) void topk_pick_kernel(TopkState* st) {
  TopkState& s = st[blockIdx.x];
  const int shift = topk_shift(s.width);
  topk_narrow<OWN_LAUNCH>(s, 1 << (s.width - shift), shift, nullptr);
}

// Element `at` of a matrix waits for the exact threshold of this state's worker: as a primary entry with the sum
// over the workers before it, or, where an earlier worker's list has it, as one that only counts.  A settled
// state's interval holds at most TOPK_LIST values; the bounds are for residuals that share memory.
__device__ __forceinline__ void topk_wait(TopkState& s, unsigned int at, bool primary, float sum) {
  if (primary) {
    const unsigned int n = atomicAdd(&s.hist[TOPK_BINS - 2], 1u);
    if (n >= (unsigned int)TOPK_LIST) return;
    s.hist[2 * n] = at;
    s.hist[2 * n + 1] = __float_as_uint(sum);
  } else {
    const unsigned int n = atomicAdd(&s.hist[TOPK_BINS - 1], 1u);
    if (n < (unsigned int)TOPK_LIST) s.hist[TOPK_BINS - 3 - n] = at;
  }
}

// The update, of the matrices that the pass over the window settled for all workers (EARLY; values inside a worker's
// interval make their element wait), or of the others, whose intervals are single keys by now.
template <typename WT, typename GT, bool VEC, bool EARLY>
__device__ __forceinline__ void topk_update(
    const WorkerPtrs& w, GT* __restrict__ theta_g, float* __restrict__ u, const ResidualPtrs& ef,
    const ScalePtrs& thresholds, TopkState* st, long elems, int count, int K, float eta, float mu, float inv_k,
    int nesterov, int write_back, long b, int blk, int nblk) {
  __shared__ unsigned int from[MLC_MAX_WORKERS], held[MLC_MAX_WORKERS];
  if (threadIdx.x < K) {
    const TopkState& s = st[(long)threadIdx.x * count + b];
    from[threadIdx.x] = s.lo;
    held[threadIdx.x] = EARLY && s.width ? 1u << s.width : 0u;          // one key: nothing has to wait
    if (!EARLY && blk == 0 && thresholds.p[threadIdx.x])
      thresholds.p[threadIdx.x][b] = __uint_as_float(s.lo);
  }
  __syncthreads();
  GT* tg = theta_g + b * elems;
  float* ub = u + b * elems;
  for (long i = ((long)blk * OT_THREADS + threadIdx.x) * 8; i < elems;
       i += (long)nblk * OT_THREADS * 8) {
    float a[8], uv[8], acc[8];
    const int left = (int)min(elems - i, 8L);
    load8<GT, !VEC>(tg + i, left, a); load8<float, !VEC>(ub + i, left, uv);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    unsigned int wait = 0u;                // elements of which some worker's value is inside its interval
    for (int k = 0; k < K; ++k) {
      float* res = ef.p[k] ? ef.p[k] + b * elems : nullptr;
      float v[8];
      if (res) {                       // v is already there
        load8<float, !VEC>(res + i, left, v);
      } else {
        load8<WT, !VEC>(reinterpret_cast<const WT*>(w.p[k]) + b * elems + i, left, v);
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = a[j] - v[j];
      }
      const unsigned int lo = from[k], range = held[k];
      if constexpr (EARLY) {
        unsigned int inside = 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if ((VEC || j < left) && magnitude_key(v[j]) - lo < range) inside |= 1u << j;
        if (inside) {
          TopkState& s = st[(long)k * count + b];
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (inside >> j & 1u) topk_wait(s, (unsigned int)(i + j), !(wait >> j & 1u), acc[j]);
          wait |= inside;
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bool keep = magnitude_key(v[j]) >= lo + range && !(wait >> j & 1u);
        acc[j] += keep ? v[j] : 0.f;
        v[j] = keep ? 0.f : v[j];           // what was not sent
      }
      if (res) store8<float, !VEC>(res + i, v, left);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) outer_update<GT>(a[j], uv[j], __fmul_rn(acc[j], inv_k), eta, mu, nesterov);
    if (wait == 0u) {
      store8<GT, !VEC>(tg + i, a, left);
      store8<float, !VEC>(ub + i, uv, left);
      if (write_back)
        for (int k = 0; k < K; ++k) store8<WT, !VEC>(reinterpret_cast<WT*>(w.p[k]) + b * elems + i, a, left);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (j >= left || (wait >> j & 1u)) continue;
        Vec8<GT>::store1(tg + i + j, a[j]);
        ub[i + j] = uv[j];
        if (write_back)
          for (int k = 0; k < K; ++k) Vec8<WT>::store1(reinterpret_cast<WT*>(w.p[k]) + b * elems + i + j, a[j]);
      }
    }
  }
}

// The threshold of a state whose matrix topk_update<EARLY> went over, by one wavefront: the rank-th largest of the keys
// listed, built bit by bit from counts that ballots give.  The interval becomes that key.  Bound by latency: a lane
// requests four entries and their values at a time.
template <typename WT, typename GT>
__device__ __forceinline__ void topk_threshold(const TopkPtrs& g, TopkState& s, long elems, long b, int k) {
  constexpr int PER = (TOPK_LIST + 63) / 64, SIDE = 4;
  static_assert(PER % SIDE == 0, "whole batches");
  const int lane = threadIdx.x & 63;
  const unsigned int lo = s.lo, rank = s.rank;
  const int width = (int)s.width;
  const int first = width ? (int)min(s.hist[TOPK_BINS - 2], (unsigned int)TOPK_LIST) : 0;
  const int n = width ? (int)min(first + s.hist[TOPK_BINS - 1], (unsigned int)TOPK_LIST) : 0;
  const float* res = g.ef.p[k] ? g.ef.p[k] + b * elems : nullptr;
  const GT* tg = reinterpret_cast<const GT*>(g.theta_g) + b * elems;
  const WT* tk = reinterpret_cast<const WT*>(g.w.p[k]) + b * elems;
  unsigned int key[PER];                  // distance from lo, plus one: 0 is no entry
#pragma unroll
  for (int i = 0; i < PER; i += SIDE) {
#pragma unroll
    for (int j = 0; j < SIDE; ++j) key[i + j] = 0u;
    if (i * 64 < n) {
      long at[SIDE];
      float v[SIDE];
#pragma unroll
      for (int j = 0; j < SIDE; ++j) {
        const int e = min((i + j) * 64 + lane, n - 1);
        at[j] = min((long)s.hist[e < first ? 2 * e : TOPK_BINS - 3 - (e - first)], elems - 1);
      }
      if (res) {
#pragma unroll
        for (int j = 0; j < SIDE; ++j) v[j] = res[at[j]];
      } else {
#pragma unroll
        for (int j = 0; j < SIDE; ++j) v[j] = Vec8<GT>::load1(tg + at[j]) - Vec8<WT>::load1(tk + at[j]);
      }
#pragma unroll
      for (int j = 0; j < SIDE; ++j) if ((i + j) * 64 + lane < n) key[i + j] = magnitude_key(v[j]) - lo + 1u;
    }
  }
  unsigned int best = 0u;
  for (int bit = width - 1; bit >= 0; --bit) {
    const unsigned int next = best | 1u << bit;
    unsigned int reach = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (i * 64 < n) reach += (unsigned int)__popcll(__ballot(key[i] > next));
    if (reach >= rank) best = next;
  }
  if (lane == 0) {
    s.lo = lo + best;
    s.width = 0u;
    if (g.thresholds.p[k]) g.thresholds.p[k][b] = __uint_as_float(lo + best);
  }
}

// The elements of matrix b that topk_update<EARLY> left waiting, from the first worker that made them wait on, by workgroup blk of
// nblk, once the thresholds are there.  A lane requests four workers' values at a time.  (By one workgroup a matrix, thresholds
// included and value by value: 177 us for 1024 x 1024, eight workers with lists of 700; a call on 768 x 3072, sixteen bf16 workers of a
// bf16 global copy, took 445 us, 167 like this, and on 24 of 2048 x 2048, eight workers with lists of 60, 43 us of it and 17.)
template <typename WT, typename GT>
__device__ __forceinline__ void topk_settle(
    const TopkPtrs& g, const TopkState* st, long elems, int count, int K, float eta, float mu, float inv_k, int nesterov,
    int write_back, long b, int blk,
    int nblk) {
  __shared__ unsigned int tau[MLC_MAX_WORKERS], primaries[MLC_MAX_WORKERS];
  constexpr int SIDE = 4;
  if ((int)threadIdx.x < K) {
    const TopkState& s = st[(long)threadIdx.x * count + b];
    tau[threadIdx.x] = s.lo;
    primaries[threadIdx.x] = min(s.hist[TOPK_BINS - 2], (unsigned int)TOPK_LIST);
  }
  __syncthreads();
  const WorkerPtrs& w = g.w;
  const ResidualPtrs& ef = g.ef;
  GT* tg = reinterpret_cast<GT*>(g.theta_g) + b * elems;
  float* ub = g.u + b * elems;
  int k0 = 0;
  unsigned int before = 0u;                 // primary entries of the workers before k0
  for (unsigned int e = blk * OT_THREADS + threadIdx.x;; e += nblk * OT_THREADS) {
    while (k0 < K && e - before >= primaries[k0]) before += primaries[k0++];
    if (k0 == K) break;
    const TopkState& s = st[(long)k0 * count + b];
    const long at = s.hist[2 * (e - before)];
    float acc = __uint_as_float(s.hist[2 * (e - before) + 1]);
    if (at >= elems) continue;
    float a = Vec8<GT>::load1(tg + at), uv = ub[at];
    // (from the first lane's worker, which no lane precedes: a wavefront reads one worker's values at a time)
    for (int kk = __builtin_amdgcn_readfirstlane(k0); kk < K; kk += SIDE) {
      float v[SIDE];
#pragma unroll
      for (int i = 0; i < SIDE; ++i) {
        const int k = min(kk + i, K - 1);
        v[i] = ef.p[k] ? ef.p[k][b * elems + at] : a - Vec8<WT>::load1(reinterpret_cast<const WT*>(w.p[k]) + b * elems + at);
      }
#pragma unroll
      for (int i = 0; i < SIDE; ++i) {
        if (kk + i >= K) break;
        const bool keep = kk + i >= k0 && magnitude_key(v[i]) >= tau[kk + i];
        acc += keep ? v[i] : 0.f;
        if (ef.p[kk + i] && keep) ef.p[kk + i][b * elems + at] = 0.f;
      }
    }
    outer_update<GT>(a, uv, __fmul_rn(acc, inv_k), eta, mu, nesterov);
    Vec8<GT>::store1(tg + at, a);
    ub[at] = uv;
    if (write_back)
      for (int k = 0; k < K; ++k) Vec8<WT>::store1(reinterpret_cast<WT*>(w.p[k]) + b * elems + at, a);
  }
}

// What the window left: a pass over the matrices left open, except for workers whose interval is one key already, and, in the
// first of these launches, the thresholds of the others.
template <typename WT, typename GT, bool VEC, int G>
__global__ __launch_bounds__(OT_THREADS) void topk_late_kernel(
    TopkArgs<G> args, TopkState* st, long elems, int count, int K, float ef_beta, int most, int first) {
  __shared__ unsigned int lh[OT_THREADS / 64][TOPK_BINS];
  const bool none_open = topk_all_early(st);
  if (first)
    for (long i = (long)blockIdx.x * (OT_THREADS / 64) + (threadIdx.x >> 6); i < (long)count * K;
         i += (long)gridDim.x * (OT_THREADS / 64)) {
      const int k = (int)(i / count), lane = threadIdx.x & 63;
      const long b = i - (long)k * count;
      if (none_open || __all(lane >= K || state_early(st[(long)min(lane, K - 1) * count + b])))
        topk_threshold<WT, GT>(args.of(b), st[i], elems, b, k);
    }
  if (none_open) return;
  topk_each_open(st, count, K, K, most, [&](long b, int k, int blk, int nblk) {
    TopkState& s = st[(long)k * count + b];
    const TopkPtrs& g = args.of(b);
    if (s.width) topk_count<WT, GT, VEC, false>(g.w, (const GT*)g.theta_g, g.ef, s, lh, elems, b, k, ef_beta, blk, nblk, true);
  });
}

// The update behind the pass over the window.
template <typename WT, typename GT, bool VEC, int G>
__global__ __launch_bounds__(OT_THREADS) void topk_early_kernel(
    TopkArgs<G> args, TopkState* st, long elems, int count, int K, float eta, float mu, float inv_k, int nesterov, int write_back) {
  const TopkPtrs& g = args.of(blockIdx.y);
  if (topk_early(st, blockIdx.y, count, K))
    topk_update<WT, GT, VEC, true>(g.w, (GT*)g.theta_g, g.u, g.ef, g.thresholds, st, elems, count, K, eta, mu, inv_k, nesterov,
                                   write_back, blockIdx.y, blockIdx.x, gridDim.x);
}

// What is left of the matrices that the window settled, and the update of those that it left open.
template <typename WT, typename GT, bool VEC, int G>
__global__ __launch_bounds__(OT_THREADS) void topk_finish_kernel(
    TopkArgs<G> args, TopkState* st, long elems, int count, int K, float eta, float mu, float inv_k, int nesterov, int write_back,
    int most) {
  const bool none_open = topk_all_early(st);
  const int parts = max(min(TOPK_SETTLE_GRID / count, TOPK_SETTLE_MOST), 1);
  for (int i = blockIdx.x; i < count * parts; i += gridDim.x) {
    const long b = i / parts;
    if (none_open || topk_early(st, b, count, K))
      topk_settle<WT, GT>(args.of(b), st, elems, count, K, eta, mu, inv_k, nesterov, write_back, b,
                          i - (int)b * parts, parts);
    __syncthreads();                        // its shared memory may be written again
  }
  if (none_open) return;
  topk_each_open(st, count, K, 1, most, [&](long b, int, int blk, int nblk) {
    const TopkPtrs& g = args.of(b);
    topk_update<WT, GT, VEC, false>(g.w, (GT*)g.theta_g, g.u, g.ef, g.thresholds, st, elems, count, K, eta, mu, inv_k, nesterov,
                                    write_back, b, blk, nblk);
  });
}

// The update of groups that went through the three passes from the start.
template <typename WT, typename GT, bool VEC, int G>
__global__ __launch_bounds__(OT_THREADS) void topk_outer_kernel(
    TopkArgs<G> args, TopkState* st, long elems, int count, int K, float eta, float mu, float inv_k, int nesterov, int write_back) {
  const TopkPtrs& g = args.of(blockIdx.y);
  topk_update<WT, GT, VEC, false>(g.w, (GT*)g.theta_g, g.u, g.ef, g.thresholds, st, elems, count, K, eta, mu, inv_k, nesterov,
                                  write_back, blockIdx.y, blockIdx.x, gridDim.x);
}

int check_launch() { return hipGetLastError() == hipSuccess ? MLC_OK : MLC_ERR_LAUNCH; }

int cap_blocks(long blocks, long cap) {
  if (blocks > cap) blocks = cap;
  if (blocks < 1) blocks = 1;
  return (int)blocks;
}

double esize(int dtype) { return dtype == MLC_F32 ? 4.0 : 2.0; }

}  // namespace

#define MLC_DISPATCH2(WD, GD, CALL)                                  \
  do {                                                               \
    if ((WD) == MLC_F32 && (GD) == MLC_F32) { CALL(float, float); }  \
    else if ((WD) == MLC_BF16 && (GD) == MLC_F32) { CALL(bf16_t, float); } \
    else if ((WD) == MLC_BF16 && (GD) == MLC_BF16) { CALL(bf16_t, bf16_t); } \
    else { CALL(float, bf16_t); }                                    \
  } while (0)

int launch_outer_fused(const WorkerPtrs& w, int worker_dtype, void* theta_g, int global_dtype,
                       float* u, int64_t n_elems, int K, float eta_out, float mu, int nesterov,
                       int write_back, hipStream_t stream) {
  const long n_vec = n_elems / 8;
  const int blocks = cap_blocks((n_vec + OT_THREADS - 1) / OT_THREADS, 256 * 16);
  const double bytes = (double)n_elems * (K * esize(worker_dtype) * (write_back ? 2 : 1) +
                                          2 * esize(global_dtype) + 8);
  LaunchScope scope(MLC_KERNEL_OUTER, stream, 0.0, bytes);
  const float inv_k = 1.0f / (float)K;
#define MLC_CALL(WT, GT)                                                                          \
  hipLaunchKernelGGL((outer_fused_kernel<WT, GT>), dim3(blocks), dim3(OT_THREADS), 0, stream, w,  \
                     (GT*)theta_g, u, (long)n_elems, K, eta_out, mu, inv_k, nesterov, write_back)
  MLC_DISPATCH2(worker_dtype, global_dtype, MLC_CALL);
#undef MLC_CALL
  return check_launch();
}

namespace {
bool has_residuals(const ResidualPtrs& ef) { return ef.p[0] != nullptr; }
}  // namespace

QuantForm make_quant_form(int bits, int offset, int64_t rows_per_range, float ef_beta) {
  QuantForm f;
  f.bits = bits;
  f.offset = offset ? 1 : 0;
  f.rows_per_range = (int)rows_per_range;
  f.levels = offset ? (float)((1 << bits) - 1) : (float)((1 << (bits - 1)) - 1);
  f.code_bias = offset ? 0 : (1 << (bits - 1));
  f.ef_beta = ef_beta;
  return f;
}

// Workgroups a matrix.  Each ends with an atomic for every worker, and those of a worker meet in one line of memory, which takes
// one in 20 ns: one matrix of 1024 x 4096, one worker, is ready in 30 us with 256 workgroups, 31 with 512, 36 with 1024, 47 with
// 2048.  More of them are worth it where loads are slow, at element alignment from three workers without residuals on: eight of
// 4001 x 4003 260 us with 512, 234 with 1024, of 120 x 511 x 511 618, 556 and with 1536 547.  In all, several matrices: 120 of 512 x 512
// with one worker 134 us with 480 workgroups, 126 with 720 or 1440, 129 with 3000; 16 of 1024 x 1024 73, 76, 83 and 97 with 512 to 3072.
// Hundreds of matrices have many such lines, and one workgroup each for several workers is too uneven a load: 800 of 128 x 256, eight
// workers with residuals, 785 us with one, 744 and 733 with two and three; 1000 of 40 x 304 379, 364 and 360.
static long range_blocks(long count, long elems, int K, bool fb) {
  const bool many = elems % 8 && K > 2 && !fb;
  const long all = count < 4 ? (many ? 1024 : 512) : count > 512 && K > 2 ? 2400 : many ? 1536 : 768;
  return cap_blocks(((elems + 7) / 8 + OT_THREADS - 1) / OT_THREADS, all / count);
}

int launch_matrix_ranges(const OuterGroupArgs* gs, int ng, int worker_dtype, int global_dtype, int K, const QuantForm& form,
                         hipStream_t stream) {
  if (ng < 1 || ng > OUTER_MAX_SEG) return MLC_ERR_UNSUPPORTED;
  const bool fb = has_residuals(gs[0].ef);
  RangeTable tab;
  int nseg = 0;
  long most_blocks = 0, most = 0;
  bool vec = true;
  double bytes = 0.0;
  for (int i = 0; i < ng; ++i) {
    const OuterGroupArgs& g = gs[i];
    const long count = g.rows / g.m;
    if (count > 65535) return MLC_ERR_SHAPE;
    for (int k0 = 0; k0 < K; k0 += OUTER_MAX_SEG_K) {
      if (nseg == OUTER_MAX_SEG) return MLC_ERR_UNSUPPORTED;
      RangeSeg& sg = tab.s[nseg++];
      sg.workers = min(K - k0, OUTER_MAX_SEG_K);
      for (int k = 0; k < OUTER_MAX_SEG_K; ++k) {
        const bool there = k < sg.workers;
        sg.w.p[k] = there ? g.w.p[k0 + k] : nullptr;
        sg.ef.p[k] = there ? g.ef.p[k0 + k] : nullptr;
        sg.scales.p[k] = there ? g.scales.p[k0 + k] : nullptr;
        sg.offsets.p[k] = there ? g.offsets.p[k0 + k] : nullptr;
      }
      sg.theta_g = g.theta_g;
      sg.elems = g.m * g.n;
      vec = vec && sg.elems % 8 == 0;
      sg.count = (unsigned int)count;
      sg.nblk = (unsigned int)range_blocks(count, sg.elems, K, fb);
      most_blocks = max(most_blocks, (long)sg.nblk * count);
      most = max(most, count);
      bytes += (double)g.rows * g.n * (sg.workers * esize(worker_dtype) + esize(global_dtype) + (fb ? 4.0 * sg.workers : 0.0));
    }
  }
  for (int i = nseg; i < OUTER_MAX_SEG; ++i) tab.s[i] = tab.s[0];
  const int workers = min(K, OUTER_MAX_SEG_K);
  LaunchScope scope(MLC_KERNEL_QUANTIZE, stream, 0.0, bytes);
  const dim3 small((unsigned)((most + 255) / 256), (unsigned)workers, (unsigned)nseg);
  hipLaunchKernelGGL(matrix_range_init_kernel, small, dim3(256), 0, stream, tab, form.offset);
#define MLC_RANGE(WT, GT, V, KM)                                                                  \
  hipLaunchKernelGGL((matrix_range_kernel<WT, GT, V, KM>), dim3((unsigned)most_blocks, 1, (unsigned)nseg), dim3(OT_THREADS), 0, \
                     stream, tab, form)
#define MLC_RANGE_K(WT, GT, V)                                                                    \
  do {                                                                                            \
    if (workers == 1) MLC_RANGE(WT, GT, V, 1);                                                    \
    else if (workers == 2) MLC_RANGE(WT, GT, V, 2);                                               \
    else if (workers <= 4) MLC_RANGE(WT, GT, V, 4);                                               \
    else MLC_RANGE(WT, GT, V, OUTER_MAX_SEG_K);                                                   \
  } while (0)
#define MLC_CALL(WT, GT) do { if (vec) MLC_RANGE_K(WT, GT, true); else MLC_RANGE_K(WT, GT, false); } while (0)
  MLC_DISPATCH2(worker_dtype, global_dtype, MLC_CALL);
#undef MLC_CALL
#undef MLC_RANGE_K
#undef MLC_RANGE
  hipLaunchKernelGGL(matrix_range_finish_kernel, small, dim3(256), 0, stream, tab, form);
  return check_launch();
}

int launch_quantize(const WorkerPtrs& w, int worker_dtype, const void* theta_g, int global_dtype,
                    const CodePtrs& codes, const ScalePtrs& scales, const OffsetPtrs& offsets,
                    const ResidualPtrs& ef, int64_t rows, int64_t n, int K, const QuantForm& form,
                    hipStream_t stream) {
  const long blocks = (rows + OT_THREADS / 64 - 1) / (OT_THREADS / 64);
  if (blocks > 0x7fffffffL) return MLC_ERR_SHAPE;
  const int bits = form.bits;
  const double bytes = (double)rows * n * (K * esize(worker_dtype) + esize(global_dtype) + bits / 8.0 * K +
                                           (has_residuals(ef) ? 8.0 * K : 0.0)) +
                       (double)rows * 4 * K;
  LaunchScope scope(MLC_KERNEL_QUANTIZE, stream, 0.0, bytes);
  const bool vec = n % 8 == 0;
  // single-pass register kernel: a wavefront per row up to 2048 columns, a workgroup per row
  // up to 24576; otherwise the two-pass kernel
  if (n <= 24576 && !quant_two_pass(rows, n, bits) && !(worker_dtype == MLC_F32 && global_dtype == MLC_BF16)) {
    const int g = n <= 2048 ? 64 : OT_THREADS;
    const int need = (int)((n + g * 8 - 1) / (g * 8));
    const int nv = need <= 1 ? 1 : need <= 2 ? 2 : need <= 4 ? 4 : need <= 8 ? 8 : 12;
    const long rpb = OT_THREADS / g;
    const long nblk = (rows + rpb - 1) / rpb;
#define MLC_QR_R(WT, GT, NV, G, RAG)                                                              \
  hipLaunchKernelGGL((quantize_rows_reg_kernel<WT, GT, NV, G, false, RAG>), dim3((unsigned)nblk),  \
                     dim3(OT_THREADS), 0, stream, w, (GT*)const_cast<void*>(theta_g), (float*)nullptr, \
                     codes, scales, offsets, ef, (long)rows, (int)n, K, form, 0.f, 0.f, 0.f, 0, 0, 0, \
                     (uint8_t*)nullptr, (float*)nullptr, (float*)nullptr)
#define MLC_QR(WT, GT, NV, G)                                                                     \
  do { if (vec) MLC_QR_R(WT, GT, NV, G, false); else MLC_QR_R(WT, GT, NV, G, true); } while (0)
#define MLC_QR_NV(WT, GT)                                                                         \
  do {                                                                                            \
    if (g == 64) { if (nv == 1) MLC_QR(WT, GT, 1, 64); else if (nv == 2) MLC_QR(WT, GT, 2, 64);   \
                   else MLC_QR(WT, GT, 4, 64); }                                                  \
    else { if (nv <= 2) MLC_QR(WT, GT, 2, 256); else if (nv == 4) MLC_QR(WT, GT, 4, 256);         \
           else if (nv == 8) MLC_QR(WT, GT, 8, 256); else MLC_QR(WT, GT, 12, 256); }              \
  } while (0)
    if (worker_dtype == MLC_BF16 && global_dtype == MLC_F32) MLC_QR_NV(bf16_t, float);
    else if (worker_dtype == MLC_BF16) MLC_QR_NV(bf16_t, bf16_t);
    else MLC_QR_NV(float, float);
#undef MLC_QR_NV
#undef MLC_QR
#undef MLC_QR_R
    return check_launch();
  }
#define MLC_CALL(WT, GT)                                                                          \
  do {                                                                                            \
    if (vec)                                                                                      \
      hipLaunchKernelGGL((quantize_rows_kernel<WT, GT, true>), dim3((unsigned)blocks),            \
                         dim3(OT_THREADS), 0, stream, w, (const GT*)theta_g, codes, scales,       \
                         offsets, ef, (long)rows, (int)n, K, form);                               \
    else                                                                                          \
      hipLaunchKernelGGL((quantize_rows_kernel<WT, GT, false>), dim3((unsigned)blocks),           \
                         dim3(OT_THREADS), 0, stream, w, (const GT*)theta_g, codes, scales,       \
                         offsets, ef, (long)rows, (int)n, K, form);                               \
  } while (0)
  MLC_DISPATCH2(worker_dtype, global_dtype, MLC_CALL);
#undef MLC_CALL
  return check_launch();
}

int launch_dequant_outer(const WorkerPtrs& w, int worker_dtype, void* theta_g, int global_dtype,
                         float* u, const CodePtrs& codes, const ScalePtrs& scales,
                         const OffsetPtrs& offsets, int64_t rows, int64_t n, int K,
                         const QuantForm& form, float eta_out, float mu, int nesterov,
                         int write_back, hipStream_t stream) {
  const bool vec = n % 8 == 0;
  const int bits = form.bits;
  const long items = rows * (n / (vec ? 8 : 8 / bits));
  const int blocks = cap_blocks((items + OT_THREADS - 1) / OT_THREADS, 256 * 16);
  const double bytes = (double)rows * n * (bits / 8.0 * K + 2 * esize(global_dtype) + 8 +
                                           (write_back ? K * esize(worker_dtype) : 0)) +
                       (double)rows * 4 * K;
  LaunchScope scope(MLC_KERNEL_DEQUANT_OUTER, stream, 0.0, bytes);
  const float inv_k = 1.0f / (float)K;
#define MLC_CALL(WT, GT)                                                                          \
  do {                                                                                            \
    if (vec)                                                                                      \
      hipLaunchKernelGGL((dequant_outer_kernel<WT, GT, true>), dim3(blocks), dim3(OT_THREADS), 0, \
                         stream, w, (GT*)theta_g, u, codes, scales, offsets, (long)rows, (int)n,  \
                         K, form, eta_out, mu, inv_k, nesterov, write_back);                      \
    else                                                                                          \
      hipLaunchKernelGGL((dequant_outer_kernel<WT, GT, false>), dim3(blocks), dim3(OT_THREADS), 0,\
                         stream, w, (GT*)theta_g, u, codes, scales, offsets, (long)rows, (int)n,  \
                         K, form, eta_out, mu, inv_k, nesterov, write_back);                      \
  } while (0)
  MLC_DISPATCH2(worker_dtype, global_dtype, MLC_CALL);
#undef MLC_CALL
  return check_launch();
}

// Do ragged rows of four vectors of bf16 take the kernel that is held to three wavefronts a SIMD?  `blocks` workgroups of four
// wavefronts each are one round of it where two wavefronts a SIMD need a second, nearly empty one: n 1501, 8 bits, us with two
// and three, two workers with error feedback, 500 workgroups 24.1 and 26.4, 540 36.3 and 29.2, 760 39.2 and 34.3, 800 40.1 and 47.3; eight workers
// 42 and 47, 68 and 53, 70 and 55, 76 and 82.  (Of 1100 workgroups it is 0.93 to 1.05 of two, of float32 workers 1.18, of rows over
// 2048 with a bf16 global copy, which spill most, 0.98 to 1.22.)
static bool quant_three_waves(long blocks, int worker_dtype) {
  return worker_dtype == MLC_BF16 && blocks > 2 * 256 && blocks <= 3 * 256;
}

// Returns MLC_ERR_UNSUPPORTED when the one-pass kernel does not cover the request (the
// caller then runs the quantiser and the dequantising update as two launches).
int launch_quantize_outer_fused(const WorkerPtrs& w, int worker_dtype, void* theta_g, int global_dtype,
                                float* u, const CodePtrs& codes, const ScalePtrs& scales,
                                const OffsetPtrs& offsets, const ResidualPtrs& ef, int64_t rows,
                                int64_t n, int K, const QuantForm& form, float eta_out, float mu,
                                int nesterov, int write_back, int requant, uint8_t* mean_codes,
                                float* mean_scales, float* mean_offsets, hipStream_t stream) {
  if (n > 24576 || quant_two_pass(rows, n, form.bits) || (worker_dtype == MLC_F32 && global_dtype == MLC_BF16))
    return MLC_ERR_UNSUPPORTED;
  if (requant && quant_ragged(n)) return MLC_ERR_UNSUPPORTED;
  const int g = n <= 2048 ? 64 : OT_THREADS;
  const int need = (int)((n + g * 8 - 1) / (g * 8));
  // Vectors per thread.  The row, its running mean and the current worker's delta all live in
  // registers (24 floats per vector), so the steps are fine where it buys occupancy: 6 instead
  // of 8 vectors lets two workgroups share a CU (10240 columns: 3.3 -> 4.x TB/s with K = 4).
  const int nv = need <= 1 ? 1 : need <= 2 ? 2 : need <= 4 ? 4 : 6;
  const int whole = quant_whole_row(QuantRow{(long)n, K, form.bits, worker_dtype == MLC_F32,
                                             global_dtype == MLC_BF16, has_residuals(ef), requant != 0});
  const int threads = whole ? (int)((n + whole * 512 - 1) / (whole * 512)) * 64 : OT_THREADS;
  const long rpb = OT_THREADS / g;
  const long nblk = (rows + rpb - 1) / rpb;
  if (nblk > 0x7fffffffL) return MLC_ERR_SHAPE;
  const int bits = form.bits;
  const double bytes = (double)rows * n * (K * esize(worker_dtype) * (write_back ? 2 : 1) + bits / 8.0 * K +
                                           (has_residuals(ef) ? 8.0 * K : 0.0) +
                                           (mean_codes ? bits / 8.0 : 0.0) +
                                           2 * esize(global_dtype) + 8) + (double)rows * 4 * K;
  LaunchScope scope(MLC_KERNEL_DEQUANT_OUTER, stream, 0.0, bytes);
  const float inv_k = 1.0f / (float)K;
  const bool three = quant_ragged(n) && quant_three_waves(nblk, worker_dtype);
#define MLC_QO_R(WT, GT, NV, G, ...)                                                              \
  hipLaunchKernelGGL((quantize_rows_reg_kernel<WT, GT, NV, G, true, __VA_ARGS__>), dim3((unsigned)nblk), \
                     dim3(threads), 0, stream, w, (GT*)theta_g, u, codes, scales, offsets, ef,  \
                     (long)rows, (int)n, K, form, eta_out, mu, inv_k, nesterov, write_back, requant, \
                     mean_codes, mean_scales, mean_offsets)
#define MLC_QO(WT, GT, NV, G)                                                                     \
  do { if (quant_ragged(n)) MLC_QO_R(WT, GT, NV, G, true); else MLC_QO_R(WT, GT, NV, G, false); } while (0)
#define MLC_QO_4(WT, GT, G)                                                                       \
  do { if (three) MLC_QO_R(WT, GT, 4, G, true, sizeof(WT) == 2 && (G == 64 || sizeof(GT) == 4) ? 3 : 2); else MLC_QO(WT, GT, 4, G); } while (0)
#define MLC_QO_NV(WT, GT)                                                                         \
  do {                                                                                            \
    if (whole == 2) MLC_QO(WT, GT, 2, 0); else if (whole == 3) MLC_QO(WT, GT, 3, 0);              \
    else if (g == 64) { if (nv == 1) MLC_QO(WT, GT, 1, 64); else if (nv == 2) MLC_QO(WT, GT, 2, 64);   \
                   else MLC_QO_4(WT, GT, 64); }                                                   \
    else { if (nv <= 2) MLC_QO(WT, GT, 2, 256); else if (nv == 4) MLC_QO_4(WT, GT, 256);          \
           else MLC_QO(WT, GT, 6, 256); }                                                         \
  } while (0)
  if (worker_dtype == MLC_BF16 && global_dtype == MLC_F32) MLC_QO_NV(bf16_t, float);
  else if (worker_dtype == MLC_BF16) MLC_QO_NV(bf16_t, bf16_t);
  else MLC_QO_NV(float, float);
#undef MLC_QO_NV
#undef MLC_QO_4
#undef MLC_QO
#undef MLC_QO_R
  return check_launch();
}

// One launch for the fused un-quantised outer step of up to OUTER_MAX_SEG groups.
int launch_outer_fused_multi(const OuterGroupArgs* gs, int ng, int worker_dtype, int global_dtype, int K,
                             float eta_out, float mu, int nesterov, int write_back, hipStream_t stream) {
  if (ng < 1 || ng > OUTER_MAX_SEG || K > OUTER_MAX_SEG_K) return MLC_ERR_UNSUPPORTED;
  OuterSegTable tab;
  tab.nseg = ng;
  double total = 0.0;
  for (int i = 0; i < ng; ++i) total += (double)gs[i].rows * (double)gs[i].n;
  // about 16 workgroups per compute unit in all, dealt in proportion to the groups' sizes
  const double budget = 256.0 * 16.0;
  unsigned int blk = 0;
  double bytes = 0.0;
  for (int i = 0; i < OUTER_MAX_SEG; ++i) {
    OuterSeg& sg = tab.s[i];
    if (i >= ng) { sg = tab.s[0]; sg.blk0 = 0xffffffffu; sg.nblk = 0; continue; }
    const long n_elems = gs[i].rows * gs[i].n;
    for (int k = 0; k < OUTER_MAX_SEG_K; ++k) sg.w.p[k] = k < K ? gs[i].w.p[k] : nullptr;
    sg.theta_g = gs[i].theta_g;
    sg.u = gs[i].u;
    sg.n_elems = n_elems;
    const long want = (n_elems / 8 + OT_THREADS - 1) / OT_THREADS;
    long nb = (long)(budget * (double)n_elems / total + 0.5);
    if (nb > want) nb = want;
    if (nb < 1) nb = 1;
    sg.blk0 = blk;
    sg.nblk = (unsigned int)nb;
    blk += (unsigned int)nb;
    bytes += (double)n_elems * (K * esize(worker_dtype) * (write_back ? 2 : 1) + 2 * esize(global_dtype) + 8);
  }
  LaunchScope scope(MLC_KERNEL_OUTER, stream, 0.0, bytes);
  const float inv_k = 1.0f / (float)K;
#define MLC_CALL(WT, GT)                                                                              \
  hipLaunchKernelGGL((outer_fused_multi_kernel<WT, GT>), dim3(blk), dim3(OT_THREADS), 0, stream, tab, K, \
                     eta_out, mu, inv_k, nesterov, write_back)
  MLC_DISPATCH2(worker_dtype, global_dtype, MLC_CALL);
#undef MLC_CALL
  return check_launch();
}

int quant_reg_cfg(int64_t n) {
  return n <= 512 ? 0 : n <= 1024 ? 1 : n <= 2048 ? 2 : n <= 4096 ? 3 : n <= 8192 ? 4 : -1;
}

// One launch for the quantised outer step (quantise + dequantise + mean + eq. 3 + write-back)
// of up to OUTER_MAX_SEG groups; ranges per row, or per matrix and ready (launch_matrix_ranges); no second quantisation.
int launch_quantize_outer_multi(const OuterGroupArgs* gs, int ng, int worker_dtype, int global_dtype, int K,
                                const QuantForm& form, float eta_out, float mu, int nesterov, int write_back,
                                hipStream_t stream) {
  if (ng < 1 || ng > OUTER_MAX_SEG || K > OUTER_MAX_SEG_K) return MLC_ERR_UNSUPPORTED;
  if (worker_dtype == MLC_F32 && global_dtype == MLC_BF16) return MLC_ERR_UNSUPPORTED;
  QuantSegTable tab;
  tab.nseg = ng;
  unsigned long blk = 0;
  double bytes = 0.0;
  bool ef_any = false;
  int top = 0;
  bool four = true;
  for (int i = 0; i < OUTER_MAX_SEG; ++i) {
    QuantSeg& sg = tab.s[i];
    if (i >= ng) { sg = tab.s[0]; sg.blk0 = 0xffffffffu; continue; }
    const int cfg = quant_reg_cfg(gs[i].n);
    if (cfg < 0 || quant_two_pass(gs[i].rows, gs[i].n, form.bits) ||
        quant_ragged(gs[i].n) != quant_ragged(gs[0].n))
      return MLC_ERR_UNSUPPORTED;
    for (int k = 0; k < OUTER_MAX_SEG_K; ++k) {
      sg.w.p[k] = k < K ? gs[i].w.p[k] : nullptr;
      sg.codes.p[k] = k < K ? gs[i].codes.p[k] : nullptr;
      sg.scales.p[k] = k < K ? gs[i].scales.p[k] : nullptr;
      sg.offsets.p[k] = k < K ? gs[i].offsets.p[k] : nullptr;
      sg.ef.p[k] = k < K ? gs[i].ef.p[k] : nullptr;
    }
    ef_any = gs[i].ef.p[0] != nullptr;
    sg.theta_g = gs[i].theta_g;
    sg.u = gs[i].u;
    sg.rows = gs[i].rows;
    sg.n = (int)gs[i].n;
    sg.rows_per_range = form.rows_per_range ? (int)gs[i].m : 0;
    sg.cfg = cfg;
    top = max(top, cfg);
    four = four && reg_cfg(cfg).nv == 4;
    const long rpb = OT_THREADS / reg_cfg(cfg).g;
    sg.blk0 = (unsigned int)blk;
    blk += (unsigned long)((gs[i].rows + rpb - 1) / rpb);
    if (blk > 0x7fffffffUL) return MLC_ERR_SHAPE;
    bytes += (double)gs[i].rows * gs[i].n * (K * esize(worker_dtype) * (write_back ? 2 : 1) + form.bits / 8.0 * K +
                                             (ef_any ? 8.0 * K : 0.0) + 2 * esize(global_dtype) + 8) +
             (double)gs[i].rows * 4 * K;
  }
  LaunchScope scope(MLC_KERNEL_DEQUANT_OUTER, stream, 0.0, bytes);
  const float inv_k = 1.0f / (float)K;
#define MLC_QM_R(KERNEL, WT, GT, RAG, ...)                                                        \
  hipLaunchKernelGGL((KERNEL<WT, GT, RAG, __VA_ARGS__>), dim3((unsigned)blk), dim3(OT_THREADS), 0, stream, tab, K, form, eta_out, mu, \
                     inv_k, nesterov, write_back)
#define MLC_QM_K(WT, GT, RAG)                                                                     \
  do {                                                                                            \
    if (top == 0) MLC_QM_R(quantize_outer_narrow_kernel, WT, GT, RAG, 0);                         \
    else if (top == 1) MLC_QM_R(quantize_outer_narrow_kernel, WT, GT, RAG, 1);                    \
    else if (K == 1) MLC_QM_R(quantize_outer_multi_kernel, WT, GT, RAG, 1);                       \
    else if (RAG && four && quant_three_waves((long)blk, worker_dtype))                           \
      MLC_QM_R(quantize_outer_narrow_kernel, WT, GT, true, 4, sizeof(WT) == 2 ? 3 : 2);           \
    else if (RAG && four) MLC_QM_R(quantize_outer_narrow_kernel, WT, GT, true, 4);                \
    else MLC_QM_R(quantize_outer_multi_kernel, WT, GT, RAG, 0);                                   \
  } while (0)
#define MLC_QM(WT, GT)                                                                            \
  do { if (quant_ragged(gs[0].n)) MLC_QM_K(WT, GT, true); else MLC_QM_K(WT, GT, false); } while (0)
  if (worker_dtype == MLC_BF16 && global_dtype == MLC_F32) MLC_QM(bf16_t, float);
  else if (worker_dtype == MLC_BF16) MLC_QM(bf16_t, bf16_t);
  else MLC_QM(float, float);
#undef MLC_QM
#undef MLC_QM_K
#undef MLC_QM_R
  return check_launch();
}

size_t topk_workspace_bytes(int64_t count, int K) { return (size_t)count * K * sizeof(TopkState); }

// Does the window's pass take the workers of a piece in turn?  All of them read the same global parameters: worker by worker
// the second reads them from the memory-side cache, but only if what one worker touches, `bytes` a value, fits into it.  Two groups of
// 2 x 2048 x 4096, 4 workers, error feedback (470 MB a worker), call of the whole step: 1615 us worker by worker, 1508 in turn; eight
// workers 2973 and 2676.  Where it fits, in turn has more streams in flight and is up to 4 % slower: groups of
// 4 x 1024 x 4096 without feedback (201 MB), four workers, 638 and 660.
static bool topk_turn(long elems, int64_t count, double bytes) { return (double)elems * (double)count * bytes > (double)(1 << 28); }

// Does the workgroup that ends a counting pass last pick the digit?  Against a launch of its own after every pass, 0.75 of a
// call's time with up to 250 workgroups, 0.78 to 0.99 with 512, 0.83 to 0.96 with 700; with 1024 0.97 to 1.04 where a matrix has 32 of them
// and more, 1.06 to 1.15 with 2 to 20, and with 4096 1.1 to 1.7.
static bool topk_last_picks(int blocks, int n_states) { return (long)blocks * n_states <= (blocks >= 32 ? 1024 : 704); }

// Do these states start from a sample?  Microseconds that the window saves over the passes and that it costs, fitted to 1720
// groups of 3 to 70 M values (matrices of 256 x 256 to 2048 x 8192, 1 to 16 workers, calls one behind the other) that
// were timed both ways.  The workgroups of two passes, each of which adds its histogram to its state's, cost
// more than the bytes; the window, the sample of 16384 values a state, three launches that find little to do, and the lists, which
// are longer where values tie.  A single large matrix is read by 256 workgroups in every pass, and gains from 6 M values on.  By passes
// and by the window, us: 16 of 512 x 512 67 and 61, 4 of 1024 x 1024 62 and 60, 8 of them 100 and 84; without error feedback 1024 x 1024
// with four workers 46 and 49, two of 1536 x 1536 with two 63 and 68, 16 of 512 x 512 with two 73 and 59.  Over all groups the choice takes
// 1.004 of the faster way's time and 0.84 of that by passes, and in eight of them 1.02 to 1.07 of it.
static bool topk_window(long elems, int64_t count, int K, int blocks, bool feedback, bool ties) {
  const double states = (double)count * K, values = elems * states * 1e-6, workgroups = blocks * states;
  if (elems < 65536 || elems * states < (double)(1 << 22)) return false;
  if (elems >= 6 << 20) return true;
  if (feedback) return 0.37 * values + 0.0071 * workgroups > 10.5 + 0.25 * K + 0.5 * K / count + 0.13 * states;
  if (ties) return 0.1 * values + 0.0056 * workgroups > 10.0 + 0.8 * K + 0.065 * states;
  return 0.77 * values + 0.0048 * workgroups > 10.0 + 0.7 * K + 0.35 * K / count + 0.11 * states;
}

// With groups of one or two of them (G) in every launch.
template <int G>
static int launch_topk(const TopkGroup* groups, int worker_dtype, int global_dtype, long elems, int K, unsigned int kcount,
                       float ef_beta, float eta_out, float mu, int nesterov, int write_back, void* workspace, hipStream_t stream) {
  const int64_t first = groups[0].count, count = first + (G > 1 ? groups[G - 1].count : 0);
  TopkArgs<G> args;
  args.split = (int)first;
  for (int i = 0; i < G; ++i) {
    const TopkGroup& g = groups[i];
    TopkPtrs& p = args.g[i];
    const long back = i ? (long)first : 0;         // matrices before the group
    auto at = [&](const void* x, double size) { return x ? (uintptr_t)x - (uintptr_t)back * (uintptr_t)(elems * (long)size) : 0; };
    for (int k = 0; k < MLC_MAX_WORKERS; ++k) {
      p.w.p[k] = (void*)at(g.w.p[k], esize(worker_dtype));
      p.ef.p[k] = (float*)at(g.ef.p[k], 4.0);
      p.thresholds.p[k] = g.thresholds.p[k] ? (float*)((uintptr_t)g.thresholds.p[k] - (uintptr_t)back * 4) : nullptr;
    }
    p.theta_g = (void*)at(g.theta_g, esize(global_dtype));
    p.u = (float*)at(g.u, 4.0);
  }
  if (count > 65535) return MLC_ERR_SHAPE;
  TopkState* st = (TopkState*)workspace;
  const bool vec = elems % 8 == 0;
  const long full = ((elems + 7) / 8 + OT_THREADS - 1) / OT_THREADS;      // a workgroup meets each element once
  const int full_grid = cap_blocks(full, 256);
  const int window_grid = cap_blocks((full * OT_THREADS + TOPK_WINDOW_THREADS - 1) / TOPK_WINDOW_THREADS, 256);
  const int n_states = (int)(count * K);
  const bool fb = has_residuals(groups[0].ef);
  const double inputs = K * (esize(worker_dtype) + esize(global_dtype));
  // one worker: nothing to share
  const bool turn = K > 1 && topk_turn(elems, count, esize(worker_dtype) + esize(global_dtype) + (fb ? 8.0 : 0.0));
  const bool window = topk_window(elems, count, K, full_grid, fb,
                                  worker_dtype == MLC_BF16 && global_dtype == MLC_BF16);
  // the values once (or, small matrices, three times: with error feedback the inputs, then the residuals), the update
  const double passes = window ? inputs + (fb ? 8.0 * K : 0.0) : fb ? inputs + 8.0 * K + 2 * 4.0 * K : 3 * inputs;
  const double last = (fb ? 8.0 * K : K * esize(worker_dtype)) + (write_back ? K * esize(worker_dtype) : 0.0) +
                      2 * esize(global_dtype) + 8;
  LaunchScope scope(MLC_KERNEL_TOPK, stream, 0.0, (double)count * elems * (passes + last));
  const float inv_k = 1.0f / (float)K;
#define MLC_UPDATE(KERNEL, WT, GT, V, GRID, ...)                                                    \
  hipLaunchKernelGGL((KERNEL<WT, GT, V, G>), GRID, dim3(OT_THREADS), 0, stream, args, st, elems, \
                     (int)count, K, eta_out, mu, inv_k, nesterov, write_back, ##__VA_ARGS__)
  const dim3 all(full_grid, (unsigned)count);
  if (window) {
#define MLC_SAMPLE(WT, GT, V)                                                                     \
  hipLaunchKernelGGL((topk_sample_kernel<WT, GT, V, G>), dim3((unsigned)count, K), dim3(TOPK_SAMPLE_THREADS), 0, \
                     stream, args, st, elems, (int)count, kcount, ef_beta)
#define MLC_WINDOW(WT, GT, V, T, ...)                                                             \
  hipLaunchKernelGGL((topk_window_kernel<WT, GT, V, T, G>), dim3(__VA_ARGS__), dim3(TOPK_WINDOW_THREADS), 0, stream, args, \
                     st, elems, (int)count, ef_beta)
#define MLC_LATE(WT, GT, V)                                                                       \
  hipLaunchKernelGGL((topk_late_kernel<WT, GT, V, G>), dim3(TOPK_LATE_GRID), dim3(OT_THREADS), 0, stream, args,  \
                     st, elems, (int)count, K, ef_beta, late_most, (int)(pass == 0))
#define MLC_WINDOWED(WT, GT, V)                                                                   \
  do {                                                                                            \
    MLC_SAMPLE(WT, GT, V);                                                                        \
    if (turn) MLC_WINDOW(WT, GT, V, true, K, window_grid, (unsigned)count);                       \
    else MLC_WINDOW(WT, GT, V, false, window_grid, (unsigned)count, K);                           \
    MLC_UPDATE(topk_early_kernel, WT, GT, V, all);                                                \
    for (int pass = 0; pass < 3; ++pass) MLC_LATE(WT, GT, V);                                     \
    MLC_UPDATE(topk_finish_kernel, WT, GT, V, dim3(TOPK_FINISH_GRID), finish_most);               \
  } while (0)
#define MLC_CALL(WT, GT) do { if (vec) MLC_WINDOWED(WT, GT, true); else MLC_WINDOWED(WT, GT, false); } while (0)
    const int late_most = cap_blocks(full, 512), finish_most = cap_blocks(full, TOPK_FINISH_GRID);
    MLC_DISPATCH2(worker_dtype, global_dtype, MLC_CALL);
#undef MLC_CALL
#undef MLC_WINDOWED
#undef MLC_LATE
#undef MLC_WINDOW
#undef MLC_SAMPLE
  } else {
    hipLaunchKernelGGL(topk_init_kernel, dim3(n_states), dim3(256), 0, stream, st, kcount);
    const bool last_picks = topk_last_picks(full_grid, n_states);
#define MLC_HIST(WT, GT, V, F)                                                                    \
  hipLaunchKernelGGL((topk_hist_kernel<WT, GT, V, F, G>), dim3(full_grid, (unsigned)count, K),        \
                     dim3(OT_THREADS), 0, stream, args, st, elems, (int)count, ef_beta, (int)last_picks);   \
  if (!last_picks) hipLaunchKernelGGL(topk_pick_kernel, dim3(n_states), dim3(OT_THREADS), 0, stream, st)
#define MLC_PASSES(WT, GT, V)                                                                     \
  do {                                                                                            \
    MLC_HIST(WT, GT, V, true);                                                                    \
    MLC_HIST(WT, GT, V, false);                                                                   \
    MLC_HIST(WT, GT, V, false);                                                                   \
    MLC_UPDATE(topk_outer_kernel, WT, GT, V, all);                                                \
  } while (0)
#define MLC_CALL(WT, GT) do { if (vec) MLC_PASSES(WT, GT, true); else MLC_PASSES(WT, GT, false); } while (0)
    MLC_DISPATCH2(worker_dtype, global_dtype, MLC_CALL);
#undef MLC_CALL
#undef MLC_PASSES
#undef MLC_HIST
  }
#undef MLC_UPDATE
  return check_launch();
}

int launch_topk_outer(const TopkGroup* groups, int n_groups, int worker_dtype, int global_dtype, int64_t elems, int K,
                      unsigned int kcount, float ef_beta, float eta_out, float mu, int nesterov, int write_back,
                      void* workspace, hipStream_t stream) {
  return (n_groups > 1 ? launch_topk<2> : launch_topk<1>)(groups, worker_dtype, global_dtype, elems, K, kcount, ef_beta, eta_out, mu,
                                                          nesterov, write_back, workspace, stream);
}

}  // namespace mlc
