// HBM-bound kernels of the Muon inner step (paper Sec. 2 "Muon", Sec. 5 "MuLoCo"):
//   momentum + look-ahead + sum of squares in one pass, the per-matrix norm, the parameter
//   update, and the layout conversions around the stand-alone newton_schulz call.
//
// The matrix handed to the Newton-Schulz GEMMs lives in a work-space layout padded to
// multiples of 128 in both dimensions ([count][mp][np], bf16, pad = 0), so the GEMM
// kernels need no bounds checks; zero padding does not change the iteration on the real
// block.  Each thread handles 8 adjacent columns (16 bytes of bf16).  VEC = false: rows that are not
// a multiple of 8, accessed 8 elements at a time all the same, at element alignment and with a
// partial last vector (rows of 1001 and 2730: parameter update 357 -> 129 us, momentum pass
// 466 -> 211 us for 76 M elements, against one element at a time).
#include "common.h"

namespace mlc {
namespace {

constexpr int EW_THREADS = 256;

// Sum over the workgroup in a fixed order: wavefront shuffles, then an LDS tree of 4.
__device__ __forceinline__ float block_sum(float v) {
  __shared__ float part[EW_THREADS / 64];
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  float s = 0.f;
  if (threadIdx.x == 0) s = (part[0] + part[1]) + (part[2] + part[3]);
  return s;   // valid in thread 0
}

// The momentum pass of several groups in one launch (their table travels in the kernel arguments):
// a step of small matrices is a string of launches of 4 to 5 us that do next to no work (inner step
// of two layers of width 128: 78 -> 71 us).
struct MomentumSeg {
  const void* grad; float* mom; bf16_t* U; float* partials;
  int m, n, mp, np, ldx, nblk;
  int kind;                          // MOM_*
  unsigned int blk0;                 // first workgroup of this group
};
struct MomentumTable { MomentumSeg s[INNER_MAX_SEG]; };
template <typename Table>
__device__ __forceinline__ int find_seg(const Table& tab) {
  int si = 0;
#pragma unroll
  for (int i = 1; i < INNER_MAX_SEG; ++i)
    if (blockIdx.x >= tab.s[i].blk0) si = i;      // 0xffffffff beyond the last group
  return si;
}

// m <- beta m + g ; U = g + beta m (or m) -> padded bf16 ; per-workgroup sum of U^2.
// WITH_MOM = false: U = in (stand-alone Newton-Schulz entry).
template <typename GT, bool WITH_MOM, bool VEC>
__device__ __forceinline__ void momentum_rows(const MomentumSeg& sg, float beta, int nesterov) {
  const int rel = (int)(blockIdx.x - sg.blk0), b = rel / sg.nblk, bx = rel - b * sg.nblk;
  const int m = sg.m, n = sg.n, mp = sg.mp, np = sg.np, ldx = sg.ldx;
  const long mat = (long)b * m * n;
  const GT* __restrict__ g = (const GT*)sg.grad + mat;
  float* __restrict__ mo = WITH_MOM ? sg.mom + mat : nullptr;
  bf16_t* __restrict__ u = sg.U + (long)b * mp * ldx;
  const int vec_per_row = np / 8;
  const long items = (long)mp * vec_per_row;
  float ss = 0.f;
  for (long it = (long)bx * EW_THREADS + threadIdx.x; it < items;
       it += (long)sg.nblk * EW_THREADS) {
    const int row = (int)(it / vec_per_row);
    const int col = (int)(it - (long)row * vec_per_row) * 8;
    float uv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) uv[j] = 0.f;
    if (row < m && col < n) {
      const long off = (long)row * n + col;
      float gv[8], mv[8];
      if (VEC) {
        Vec8<GT>::load(g + off, gv);
        if (WITH_MOM) Vec8<float>::load(mo + off, mv);
      } else {
        Vec8<GT>::unpack(Vec8U<GT>::load_raw(g + off, n - col), gv);
        if (WITH_MOM) Vec8<float>::unpack(Vec8U<float>::load_raw(mo + off, n - col), mv);
      }
      if (WITH_MOM) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          mv[j] = beta * mv[j] + gv[j];
          uv[j] = nesterov ? gv[j] + beta * mv[j] : mv[j];
        }
        if (VEC) {
          Vec8<float>::store(mo + off, mv);
        } else {
          Vec8U<float>::store(mo + off, mv, n - col);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) uv[j] = gv[j];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) ss += uv[j] * uv[j];
    }
    Vec8<bf16_t>::store(u + (long)row * ldx + col, uv);
  }
  const float tot = block_sum(ss);
  if (threadIdx.x == 0) sg.partials[(long)b * sg.nblk + bx] = tot;
}

// The same with U stored transposed, [np][mp].  A workgroup takes 128 x 64 blocks through the LDS:
// rows are read 64 columns at a time (whole lines), and 128 adjacent values of a column leave as
// 256 bytes.  LDS chunk x (8 values of a column) of column c sits at position x ^ ((c / 8) % 8),
// which spreads a wavefront's 2-byte stores over the banks.
constexpr int TR_M = 128, TR_N = 64;
template <typename GT, bool WITH_MOM, bool VEC>
__device__ __forceinline__ void momentum_transposed(const MomentumSeg& sg, bf16_t* tile, float beta, int nesterov) {
  const int rel = (int)(blockIdx.x - sg.blk0), b = rel / sg.nblk, bx = rel - b * sg.nblk;
  const int m = sg.m, n = sg.n, mp = sg.mp, np = sg.np, ldx = sg.ldx;
  const long mat = (long)b * m * n;
  const GT* __restrict__ g = (const GT*)sg.grad + mat;
  float* __restrict__ mo = WITH_MOM ? sg.mom + mat : nullptr;
  bf16_t* __restrict__ u = sg.U + (long)b * np * ldx;
  const int blocks_n = np / TR_N;
  const int blocks = (mp / TR_M) * blocks_n;
  const int r0 = threadIdx.x >> 3, c8 = threadIdx.x & 7;      // this thread's row and 8-column chunk
  float ss = 0.f;
  for (int blk = bx; blk < blocks; blk += sg.nblk) {
    const int row0 = blk / blocks_n * TR_M, col0 = blk % blocks_n * TR_N;
    const int col = col0 + c8 * 8;
#pragma unroll
    for (int pass = 0; pass < TR_M / 32; ++pass) {
      const int lr = pass * 32 + r0, row = row0 + lr;
      float uv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) uv[j] = 0.f;
      if (row < m && col < n) {
        const long off = (long)row * n + col;
        float gv[8], mv[8];
        if (VEC) {
          Vec8<GT>::load(g + off, gv);
          if (WITH_MOM) Vec8<float>::load(mo + off, mv);
        } else {
          Vec8<GT>::unpack(Vec8U<GT>::load_raw(g + off, n - col), gv);
          if (WITH_MOM) Vec8<float>::unpack(Vec8U<float>::load_raw(mo + off, n - col), mv);
        }
        if (WITH_MOM) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            mv[j] = beta * mv[j] + gv[j];
            uv[j] = nesterov ? gv[j] + beta * mv[j] : mv[j];
          }
          if (VEC) {
            Vec8<float>::store(mo + off, mv);
          } else {
            Vec8U<float>::store(mo + off, mv, n - col);
          }
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) uv[j] = gv[j];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) ss += uv[j] * uv[j];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j)
        tile[(c8 * 8 + j) * TR_M + (((lr >> 3) ^ c8) << 3) + (lr & 7)] = f32_to_bf16(uv[j]);
    }
    __syncthreads();
#pragma unroll
    for (int pass = 0; pass < TR_N / 16; ++pass) {
      const int c = pass * 16 + (threadIdx.x >> 4), x = threadIdx.x & 15;
      const u32x4 v = *reinterpret_cast<const u32x4*>(tile + c * TR_M + ((x ^ ((c >> 3) & 7)) << 3));
      *reinterpret_cast<u32x4*>(u + (long)(col0 + c) * ldx + row0 + x * 8) = v;
    }
    __syncthreads();
  }
  const float tot = block_sum(ss);
  if (threadIdx.x == 0) sg.partials[(long)b * sg.nblk + bx] = tot;
}

// KINDS: those of the groups of a launch, a bit each.
enum { MOM_VEC = 1, MOM_TRANSPOSED = 2 };
template <typename GT, bool WITH_MOM, int KINDS>
__global__ __launch_bounds__(EW_THREADS) void muon_momentum_kernel(MomentumTable tab, float beta, int nesterov) {
  __shared__ __attribute__((aligned(16))) bf16_t tile[KINDS >> MOM_TRANSPOSED ? TR_N * TR_M : 8];
  const MomentumSeg& sg = tab.s[find_seg(tab)];
  auto is = [&](int kind) { return KINDS == 1 << kind || (KINDS >> kind & 1 && sg.kind == kind); };
  if (is(0)) momentum_rows<GT, WITH_MOM, false>(sg, beta, nesterov);
  else if (is(MOM_VEC)) momentum_rows<GT, WITH_MOM, true>(sg, beta, nesterov);
  else if (is(MOM_TRANSPOSED)) momentum_transposed<GT, WITH_MOM, false>(sg, tile, beta, nesterov);
  else if (is(MOM_TRANSPOSED | MOM_VEC)) momentum_transposed<GT, WITH_MOM, true>(sg, tile, beta, nesterov);
}

// scale[b] = 1 / (sqrt(sum_b) + eps); an all-zero matrix gets 0, also when eps = 0
struct NormSeg { const float* partials; float* scale; int nblk; unsigned int blk0; };
struct NormTable { NormSeg s[INNER_MAX_SEG]; };
__global__ __launch_bounds__(EW_THREADS) void muon_norm_kernel(NormTable tab, float eps) {
  const NormSeg& sg = tab.s[find_seg(tab)];
  const int b = (int)(blockIdx.x - sg.blk0), nblk = sg.nblk;
  float s = 0.f;
  for (int i = threadIdx.x; i < nblk; i += EW_THREADS) s += sg.partials[(long)b * nblk + i];
  const float tot = block_sum(s);
  if (threadIdx.x == 0) sg.scale[b] = tot > 0.f ? 1.0f / (sqrtf(tot) + eps) : 0.f;
}

// W <- decay_factor * W - step * oscale_b * O     (decay_factor = 1 - eta*lambda,
//                                                  step = eta * lr_scale)
// Bound by the memory stream.  Several groups share a launch: in a step of small matrices each launch
// is 2 to 5 us of next to no work (two layers of width 128, three groups: 70.8 -> 66.5 us a step).
struct UpdateSeg {
  void* W; const bf16_t* O; const float* oscale;
  int m, n, mp, ldx;
  float step;
  int nblk;                          // workgroups per matrix
  int vec;                           // rows are a multiple of 8
  unsigned int blk0;                 // first workgroup of this group
};
struct UpdateTable { UpdateSeg s[INNER_MAX_SEG]; };
template <typename WT, bool VEC>
__device__ __forceinline__ void update_rows(const UpdateSeg& sg, float decay_factor) {
  const unsigned int rel = blockIdx.x - sg.blk0, b = rel / (unsigned int)sg.nblk, bx = rel - b * (unsigned int)sg.nblk;
  const int m = sg.m, n = sg.n, ldx = sg.ldx;
  WT* w = (WT*)sg.W + (long)b * m * n;
  const bf16_t* o = sg.O + (long)b * sg.mp * ldx;
  const float st = sg.oscale ? sg.step * sg.oscale[b] : sg.step;
  const int vec_per_row = (n + 7) / 8;
  const long items = (long)m * vec_per_row;
  const long per_blk = (items + sg.nblk - 1) / sg.nblk;
  const long it_end = min(items, (long)(bx + 1) * per_blk);
#pragma unroll 2
  for (long it = (long)bx * per_blk + threadIdx.x; it < it_end; it += EW_THREADS) {
    const int row = (int)(it / vec_per_row);
    const int col = (int)(it - (long)row * vec_per_row) * 8;
    const long off = (long)row * n + col;
    float ov[8], wv[8];
    Vec8<bf16_t>::load_nt(o + (long)row * ldx + col, ov);   // padded layout: always in bounds
    if (VEC) {
      Vec8<WT>::load_nt(w + off, wv);
#pragma unroll
      for (int j = 0; j < 8; ++j) wv[j] = decay_factor * wv[j] - st * ov[j];
      Vec8<WT>::store_nt(w + off, wv);
    } else {
      Vec8<WT>::unpack(Vec8U<WT>::load_raw(w + off, n - col), wv);
#pragma unroll
      for (int j = 0; j < 8; ++j) wv[j] = decay_factor * wv[j] - st * ov[j];
      Vec8U<WT>::store(w + off, wv, n - col);
    }
  }
}

// KINDS: 1 for rows that are not a multiple of 8, 2 for others, 3 for groups of both.
template <typename WT, int KINDS>
__global__ __launch_bounds__(EW_THREADS) void muon_update_kernel(UpdateTable tab, float decay_factor) {
  const UpdateSeg& sg = tab.s[find_seg(tab)];
  if (KINDS == 2 || (KINDS == 3 && sg.vec)) update_rows<WT, true>(sg, decay_factor);
  else update_rows<WT, false>(sg, decay_factor);
}

// out = oscale_b * X (padded bf16 -> caller's layout and dtype)
template <typename OT, bool VEC>
__global__ __launch_bounds__(EW_THREADS) void ns_store_kernel(
    const bf16_t* __restrict__ X, const float* __restrict__ oscale, OT* __restrict__ out, int m,
    int n, int mp, int ldx) {
  const int b = blockIdx.y;
  OT* o = out + (long)b * m * n;
  const bf16_t* x = X + (long)b * mp * ldx;
  const float sc = oscale ? oscale[b] : 1.0f;
  const int vec_per_row = (n + 7) / 8;
  const long items = (long)m * vec_per_row;
  for (long it = (long)blockIdx.x * EW_THREADS + threadIdx.x; it < items;
       it += (long)gridDim.x * EW_THREADS) {
    const int row = (int)(it / vec_per_row);
    const int col = (int)(it - (long)row * vec_per_row) * 8;
    const long off = (long)row * n + col;
    float xv[8];
    Vec8<bf16_t>::load(x + (long)row * ldx + col, xv);
#pragma unroll
    for (int j = 0; j < 8; ++j) xv[j] *= sc;
    if (VEC) {
      Vec8<OT>::store(o + off, xv);
    } else {
      Vec8U<OT>::store(o + off, xv, n - col);
    }
  }
}

// AdamW for the parameters Muon does not cover (paper Sec. 4, "AdamW inner updates"):
//   m <- b1 m + (1 - b1) g ; v <- b2 v + (1 - b2) g^2
//   theta <- theta - lr * (m * c1) / (sqrt(v) * c2 + eps) - lr * lambda * theta
// c1 = 1 / (1 - b1^t), c2 = 1 / sqrt(1 - b2^t) with bias correction, else 1.
// (Plain loads and stores: non-temporal ones measured 6 % slower here.)
//
// Bound by the memory stream.  One launch covers up to ADAMW_MAX_SEG tensors (their table
// travels in the kernel arguments): most tensors that Muon leaves over are a few KB, and a
// launch for each of them cost more than the whole stream (a 32000 x 2048 embedding with 72
// vectors beside it: 568 us in 73 launches, 282 in two).  A workgroup takes ADAMW_CHUNK elements
// of one tensor, found by counting the first workgroups at or below its own index.
constexpr int ADAMW_CHUNK = EW_THREADS * 8 * 4;
struct AdamWSeg { void* theta; const void* grad; float* m; float* v; long n; };
template <int SEG>
struct AdamWTable { AdamWSeg s[SEG]; unsigned int blk0[SEG]; };
struct AdamWScalars { float lr, b1, b2, eps, decay, c1, c2; };

__device__ __forceinline__ void adamw_element(float& th, float g, float& m, float& v, const AdamWScalars& h) {
  m = h.b1 * m + (1.0f - h.b1) * g;
  v = h.b2 * v + (1.0f - h.b2) * g * g;
  const float step = (m * h.c1) / (sqrtf(v) * h.c2 + h.eps);
  th = th - h.lr * step - h.decay * th;
}

// SEG: entries of the table.  A call with one tensor carries a table of one: filling and sending
// the 2.8 KB of the full one made it 10.8 us apart instead of 10.4.
template <typename WT, typename GT, int SEG>
__global__ __launch_bounds__(EW_THREADS) void adamw_kernel(AdamWTable<SEG> tab, AdamWScalars h) {
  static_assert(SEG == 1 || SEG == 64, "one lane per tensor");
  const bool below = blockIdx.x >= tab.blk0[threadIdx.x & (SEG - 1)];      // 0xffffffff beyond the last tensor
  const int si = SEG == 1 ? 0 : __builtin_amdgcn_readfirstlane(__popcll(__ballot(below)) - 1);
  const AdamWSeg sg = tab.s[si];
  WT* const theta = (WT*)sg.theta;
  const GT* const grad = (const GT*)sg.grad;
  const long first = (long)(blockIdx.x - tab.blk0[si]) * ADAMW_CHUNK;
  const long end = min(sg.n, first + ADAMW_CHUNK);
#pragma unroll
  for (int u = 0; u < ADAMW_CHUNK / (EW_THREADS * 8); ++u) {
    const long off = first + (u * EW_THREADS + (int)threadIdx.x) * 8;
    if (off + 8 <= end) {
      float th[8], g[8], mv[8], vv[8];
      Vec8<WT>::load(theta + off, th); Vec8<GT>::load(grad + off, g);
      Vec8<float>::load(sg.m + off, mv); Vec8<float>::load(sg.v + off, vv);
#pragma unroll
      for (int j = 0; j < 8; ++j) adamw_element(th[j], g[j], mv[j], vv[j], h);
      Vec8<WT>::store(theta + off, th);
      Vec8<float>::store(sg.m + off, mv); Vec8<float>::store(sg.v + off, vv);
    } else {
      for (long e = off; e < end; ++e) {          // fewer than 8, the tensor's last ones
        float th = Vec8<WT>::load1(theta + e), mv = sg.m[e], vv = sg.v[e];
        adamw_element(th, Vec8<GT>::load1(grad + e), mv, vv, h);
        Vec8<WT>::store1(theta + e, th);
        sg.m[e] = mv; sg.v[e] = vv;
      }
    }
  }
}

int check_launch() { return hipGetLastError() == hipSuccess ? MLC_OK : MLC_ERR_LAUNCH; }

int grid_blocks(long items, int cap) {
  long blocks = (items + EW_THREADS - 1) / EW_THREADS;
  if (blocks > cap) blocks = cap;
  if (blocks < 1) blocks = 1;
  return (int)blocks;
}

// n (1 .. INNER_MAX_SEG) groups in one launch.
template <typename GT, bool WITH_MOM>
int launch_momentum_set(const MomentumDesc* const* d, int n, float beta, int nesterov, hipStream_t stream) {
  MomentumTable tab;
  unsigned long blk = 0;
  double bytes = 0.0;
  int kinds = 0;
  for (int i = 0; i < INNER_MAX_SEG; ++i) {
    const MomentumDesc& x = *d[i < n ? i : 0];
    const int kind = (x.n % 8 == 0 ? MOM_VEC : 0) | (x.transposed ? MOM_TRANSPOSED : 0);
    kinds |= 1 << kind;
    tab.s[i] = MomentumSeg{x.grad, x.mom, x.U, x.partials, (int)x.m, (int)x.n, (int)x.mp, (int)x.np, (int)x.ldx,
                           x.nblk, kind, i < n ? (unsigned int)blk : 0xffffffffu};
    if (i >= n) continue;
    blk += (unsigned long)x.nblk * (unsigned long)x.count;
    if (blk > 0x7fffffffUL) return MLC_ERR_SHAPE;
    bytes += (double)x.count * x.m * x.n * (sizeof(GT) + (WITH_MOM ? 8 : 0)) + (double)x.count * x.mp * x.np * 2;
  }
  const dim3 grid((unsigned)blk), block(EW_THREADS);
  LaunchScope scope(WITH_MOM ? MLC_KERNEL_MOMENTUM : MLC_KERNEL_CONVERT, stream, 0.0, bytes);
#define MLC_MOM(KINDS) \
  hipLaunchKernelGGL((muon_momentum_kernel<GT, WITH_MOM, KINDS>), grid, block, 0, stream, tab, beta, nesterov)
  switch (kinds) {
    case 1: MLC_MOM(1); break;
    case 2: MLC_MOM(2); break;
    case 4: MLC_MOM(4); break;
    case 8: MLC_MOM(8); break;
    case 10: MLC_MOM(10); break;        // rows that are a multiple of 8 throughout
    default: MLC_MOM(15);
  }
#undef MLC_MOM
  return check_launch();
}

}  // namespace

// Groups of one kind go out together, up to INNER_MAX_SEG in a launch, in the order of the first of
// each kind.
template <typename Desc, typename Kind, typename Launch>
static int launch_by_kind(const Desc* d, int n, Kind kind, Launch launch) {
  for (int i = 0; i < n; ++i) {
    bool taken = false;
    for (int j = 0; j < i && !taken; ++j) taken = kind(d[j]) == kind(d[i]);
    if (taken) continue;               // went out with an earlier group of its kind
    const Desc* pick[INNER_MAX_SEG];
    int np = 0;
    for (int j = i; j <= n; ++j) {
      if (np && (j == n || np == INNER_MAX_SEG)) {
        const int rc = launch(pick, np);
        if (rc != MLC_OK) return rc;
        np = 0;
      }
      if (j < n && kind(d[j]) == kind(d[i])) pick[np++] = &d[j];
    }
  }
  return MLC_OK;
}

int launch_momentum(const MomentumDesc* d, int n, float beta, int nesterov, hipStream_t stream) {
  auto kind = [](const MomentumDesc& x) { return x.grad_dtype; };      // groups of one dtype share launches
  return launch_by_kind(d, n, kind, [&](const MomentumDesc* const* pick, int np) {
    return pick[0]->grad_dtype == MLC_F32 ? launch_momentum_set<float, true>(pick, np, beta, nesterov, stream)
                                          : launch_momentum_set<bf16_t, true>(pick, np, beta, nesterov, stream);
  });
}

int launch_ns_load(const void* in, int dtype, bf16_t* U, float* partials, int nblk, int64_t count,
                   int64_t m, int64_t n, int64_t mp, int64_t np, int64_t ldx, bool transposed,
                   hipStream_t stream) {
  const MomentumDesc d{in, dtype, nullptr, U, partials, nblk, count, m, n, mp, np, ldx, transposed};
  const MomentumDesc* const one = &d;
  if (dtype == MLC_F32) return launch_momentum_set<float, false>(&one, 1, 0.f, 0, stream);
  return launch_momentum_set<bf16_t, false>(&one, 1, 0.f, 0, stream);
}

int launch_norm_finalize(const NormDesc* d, int n, float eps, hipStream_t stream) {
  return launch_by_kind(d, n, [](const NormDesc&) { return 0; }, [&](const NormDesc* const* pick, int np) -> int {
    NormTable tab;
    unsigned long blk = 0;
    double bytes = 0.0;
    for (int i = 0; i < INNER_MAX_SEG; ++i) {
      const NormDesc& x = *pick[i < np ? i : 0];
      tab.s[i] = NormSeg{x.partials, x.scale, x.nblk, i < np ? (unsigned int)blk : 0xffffffffu};
      if (i >= np) continue;
      blk += (unsigned long)x.count;
      bytes += (double)x.count * x.nblk * 4;
    }
    if (blk > 0x7fffffffUL) return MLC_ERR_SHAPE;
    LaunchScope scope(MLC_KERNEL_NORM, stream, 0.0, bytes);
    hipLaunchKernelGGL(muon_norm_kernel, dim3((unsigned)blk), dim3(EW_THREADS), 0, stream, tab, eps);
    return check_launch();
  });
}

// n (1 .. INNER_MAX_SEG) groups of one dtype in one launch.
static int launch_update_set(const UpdateDesc* const* d, int n, float decay_factor, hipStream_t stream) {
  UpdateTable tab;
  unsigned long blk = 0;
  double bytes = 0.0;
  const int dtype = d[0]->dtype;
  int kinds = 0;
  for (int i = 0; i < INNER_MAX_SEG; ++i) {
    const UpdateDesc& x = *d[i < n ? i : 0];
    const int nblk = grid_blocks(x.m * ((x.n + 7) / 8), 2048);
    kinds |= x.n % 8 == 0 ? 2 : 1;
    tab.s[i] = UpdateSeg{x.W, x.O, x.oscale, (int)x.m, (int)x.n, (int)x.mp, (int)x.ldx, x.step, nblk, x.n % 8 == 0,
                         i < n ? (unsigned int)blk : 0xffffffffu};
    if (i >= n) continue;
    blk += (unsigned long)nblk * (unsigned long)x.count;
    if (blk > 0x7fffffffUL) return MLC_ERR_SHAPE;
    bytes += (double)x.count * x.m * x.n * (2 + 2 * (dtype == MLC_F32 ? 4 : 2));
  }
  LaunchScope scope(MLC_KERNEL_UPDATE, stream, 0.0, bytes);
#define MLC_UPD(WT, KINDS) \
  hipLaunchKernelGGL((muon_update_kernel<WT, KINDS>), dim3((unsigned)blk), dim3(EW_THREADS), 0, stream, tab, decay_factor)
  if (dtype == MLC_F32) { if (kinds == 3) MLC_UPD(float, 3); else if (kinds == 2) MLC_UPD(float, 2); else MLC_UPD(float, 1); }
  else { if (kinds == 3) MLC_UPD(bf16_t, 3); else if (kinds == 2) MLC_UPD(bf16_t, 2); else MLC_UPD(bf16_t, 1); }
#undef MLC_UPD
  return check_launch();
}

int launch_param_update(const UpdateDesc* d, int n, float decay_factor, hipStream_t stream) {
  auto kind = [](const UpdateDesc& x) { return x.dtype; };
  return launch_by_kind(d, n, kind, [&](const UpdateDesc* const* pick, int np) {
    return launch_update_set(pick, np, decay_factor, stream);
  });
}

int launch_ns_store(const bf16_t* X, const float* oscale, void* out, int dtype, int64_t count,
                    int64_t m, int64_t n, int64_t mp, int64_t ldx, hipStream_t stream) {
  const long items = m * ((n + 7) / 8);
  const dim3 grid(grid_blocks(items, 2048), (unsigned)count), block(EW_THREADS);
  const double elems = (double)count * m * n;
  LaunchScope scope(MLC_KERNEL_CONVERT, stream, 0.0, elems * (2 + (dtype == MLC_F32 ? 4 : 2)));
  const bool vec = n % 8 == 0;
#define MLC_ST(OT, V)                                                                             \
  hipLaunchKernelGGL((ns_store_kernel<OT, V>), grid, block, 0, stream, X, oscale, (OT*)out, (int)m, \
                     (int)n, (int)mp, (int)ldx)
  if (dtype == MLC_F32) { if (vec) MLC_ST(float, true); else MLC_ST(float, false); }
  else { if (vec) MLC_ST(bf16_t, true); else MLC_ST(bf16_t, false); }
#undef MLC_ST
  return check_launch();
}

template <int SEG>
static int launch_adamw_seg(const mlc_adamw_group* gs, int n, const AdamWScalars& h, hipStream_t stream) {
  AdamWTable<SEG> tab;
  const int wd = gs[0].param_dtype, gd = gs[0].grad_dtype;
  double bytes = 0.0;
  unsigned long blk = 0;
  for (int i = 0; i < SEG; ++i) {
    if (i >= n) { tab.s[i] = tab.s[0]; tab.blk0[i] = 0xffffffffu; continue; }
    tab.s[i] = AdamWSeg{gs[i].param, gs[i].grad, gs[i].exp_avg, gs[i].exp_avg_sq, (long)gs[i].count};
    tab.blk0[i] = (unsigned int)blk;
    blk += (unsigned long)((gs[i].count + ADAMW_CHUNK - 1) / ADAMW_CHUNK);
    if (blk > 0x7fffffffUL) return MLC_ERR_SHAPE;
    bytes += (double)gs[i].count * (2 * (wd == MLC_F32 ? 4 : 2) + (gd == MLC_F32 ? 4 : 2) + 16);
  }
  LaunchScope scope(MLC_KERNEL_ADAMW, stream, 0.0, bytes);
#define MLC_AW(WT, GT) \
  hipLaunchKernelGGL((adamw_kernel<WT, GT, SEG>), dim3((unsigned)blk), dim3(EW_THREADS), 0, stream, tab, h)
  if (wd == MLC_F32 && gd == MLC_F32) MLC_AW(float, float);
  else if (wd == MLC_F32) MLC_AW(float, bf16_t);
  else if (gd == MLC_F32) MLC_AW(bf16_t, float);
  else MLC_AW(bf16_t, bf16_t);
#undef MLC_AW
  return check_launch();
}

int launch_adamw(const mlc_adamw_group* gs, int n, float lr, float b1, float b2, float eps, float decay,
                 float c1, float c2, hipStream_t stream) {
  const AdamWScalars h{lr, b1, b2, eps, decay, c1, c2};
  return n == 1 ? launch_adamw_seg<1>(gs, n, h, stream) : launch_adamw_seg<ADAMW_MAX_SEG>(gs, n, h, stream);
}

}  // namespace mlc
