// fp32 MFMA GEMM family (the fp32 model path; bf16 products are in
// gemm_bf16.hip):
//   forward projections  P = X Wx^T + b,  Z = H Wo^T + bo      (NT, bias)
//   data gradients       dH = dZ Wo,  dX = dA Wx              (NN)
//   weight gradients     [dWx | dWh] = dA^T [X | Hs],  dWo = dZ^T H   (TN)
// One 256-thread workgroup computes a tile of 128, 64 or 32 rows and columns;
// its four waves each own a quadrant as MFMA 16x16 tiles (8 x 16x16x4 fp32 per
// 32-wide k-step).  Operands are staged in LDS as [row][k] with a 16-byte pad
// per row.  A k-major operand is copied with 16-byte loads; an m/n-major one
// (the TN and NN cases) is loaded as 4(k) x 4(m) blocks that each thread
// transposes in registers, so every LDS tile is k-contiguous.  LDS is
// double-buffered, one barrier per k-tile; the loads of the next one (128),
// two (64) or four (32) k-tiles are in flight behind the MFMAs of the current.
// The small tiles serve small models, whose products are a handful of
// 128-row tiles on 256 compute units.  The products of a 2 x 64 model over 800
// frames, average us: projections 15.2 -> 4.9 (14 workgroups before, 200
// now), data gradients 35 -> 9.5 (7), weight gradients 32 -> 7.3 (6); of a 2 x
// 768 model over 16384 frames, ms a step: 1.58 -> 1.60, 1.70 -> 1.65 and, with
// more k-splits, 4.57 -> 3.3.
//
// Weight gradients reduce over all frames into a small output, so they split
// K over workgroups: each split writes an fp32 partial tile to the workspace
// and splitk_reduce adds the partials in split order (deterministic; no
// atomics).  The same pass yields the bias gradient: while loading the A tile
// (dA or dZ, m-major) each thread keeps the sums of its 4 rows over its
// k-rows, and the first column of tiles writes them.  The B operand of the TN
// product may come from two matrices side by side (X and the shifted hidden
// states), so dWx and dWh are one launch.
#include "am_device.h"
#include "am_internal.h"

namespace am {
namespace {

constexpr int NT = 256;   // threads per workgroup
constexpr int BK = 32;    // k per tile
constexpr int VEC = 4;    // floats per 16 bytes
constexpr int LDK = BK + VEC;  // padded LDS row, elements

// Per tile edge TB: k-tiles whose loads are in flight.  A 128-row tile's
// products outlast one memory latency; a small tile's take 128-1024 clocks a
// k-tile, so more of them have to be on their way.
constexpr int ahead(int TB) { return TB >= 128 ? 1 : TB >= 64 ? 2 : 4; }

// Source of one operand: rows (of the tile dimension) below `split` come
// from p0, the others from p1 at row - split.
struct Src {
  const float* p0; int64_t ld0;
  const float* p1; int64_t ld1;
  int split;
};

// Operand loader: the registers of one k-tile on its way to LDS.  A chunk
// outside the operand loads the operand's first chunk instead and becomes zero
// on the way to LDS (a load behind a branch would be waited for right there,
// so that none were in flight with another).
template <bool KMAJOR, int TB> struct Loader;

__device__ __forceinline__ uint4 keep(uint4 v, bool ok) {
  return make_uint4(ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u);
}

// k-major: rows of the operand are contiguous in k.
template <int TB> struct Loader<true, TB> {
  static constexpr int NR = TB / 32, CPR = BK / VEC;  // 16-byte chunks per row = 8
  uint4 reg[NR];
  __device__ __forceinline__ void load(const Src& s, int row0, int nrows, int k0, int kend) {
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const int c = threadIdx.x + NT * j;
      const int grow = row0 + c / CPR, gk = k0 + c % CPR * VEC;
      const bool ok = grow < nrows && gk < kend;
      reg[j] = *reinterpret_cast<const uint4*>(s.p0 + (ok ? (int64_t)grow * s.ld0 + gk : 0));
    }
  }
  template <bool SUM>
  __device__ __forceinline__ void store(float* lds, int row0, int nrows, int k0, int kend, float (&)[4]) const {
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const int c = threadIdx.x + NT * j;
      const bool ok = row0 + c / CPR < nrows && k0 + c % CPR * VEC < kend;
      *reinterpret_cast<uint4*>(lds + c / CPR * LDK + c % CPR * VEC) = keep(reg[j], ok);
    }
  }
};

// m/n-major: 4 k-rows x 4 rows-of-the-tile per thread (of the first 2 TB),
// transposed in registers on the way to LDS; SUM adds the rows up as they go.
template <int TB> struct Loader<false, TB> {
  uint4 reg[4];
  static __device__ __forceinline__ int kb() { return threadIdx.x / (TB / 4); }
  static __device__ __forceinline__ int mb() { return threadIdx.x % (TB / 4); }
  __device__ __forceinline__ void load(const Src& s, int row0, int nrows, int k0, int kend) {
    const int m = row0 + mb() * 4;
    const bool second = m >= s.split;
    const float* base = second ? s.p1 : s.p0;
    const int64_t ld = second ? s.ld1 : s.ld0;
    const int mm = second ? m - s.split : m;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = k0 + kb() * 4 + r;
      const bool ok = kb() < 8 && k < kend && m < nrows;
      reg[r] = *reinterpret_cast<const uint4*>(ok ? base + (int64_t)k * ld + mm : s.p0);
    }
  }
  template <bool SUM>
  __device__ __forceinline__ void store(float* lds, int row0, int nrows, int k0, int kend, float (&rs)[4]) const {
    if (kb() >= 8) return;
    float4 in[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      in[r] = __builtin_bit_cast(float4, keep(reg[r], k0 + kb() * 4 + r < kend && row0 + mb() * 4 < nrows));
    if (SUM) {
      rs[0] += ((in[0].x + in[1].x) + in[2].x) + in[3].x;
      rs[1] += ((in[0].y + in[1].y) + in[2].y) + in[3].y;
      rs[2] += ((in[0].z + in[1].z) + in[2].z) + in[3].z;
      rs[3] += ((in[0].w + in[1].w) + in[2].w) + in[3].w;
    }
    float* at = lds + mb() * 4 * LDK + kb() * 4;
    *reinterpret_cast<float4*>(at) = make_float4(in[0].x, in[1].x, in[2].x, in[3].x);
    *reinterpret_cast<float4*>(at + LDK) = make_float4(in[0].y, in[1].y, in[2].y, in[3].y);
    *reinterpret_cast<float4*>(at + 2 * LDK) = make_float4(in[0].z, in[1].z, in[2].z, in[3].z);
    *reinterpret_cast<float4*>(at + 3 * LDK) = make_float4(in[0].w, in[1].w, in[2].w, in[3].w);
  }
};

// Epilogue destination: columns below `split` go to c0, the others to c1.
struct Dst {
  float* c0; int64_t ld0;
  float* c1; int64_t ld1;
  int split;
  int64_t zstride;  // elements between the outputs of consecutive k-splits
};

// ROWSUM: the A operand is m-major and row sums of A over this split's
// k-range are written by the workgroups of the first column of tiles to
// rowsum[blockIdx.z * M + m].  Partial results (split-K) use c0 = the
// split's slice of the workspace with ld0 = N and split = N.
template <bool AK, bool BKM, bool BIAS, bool ROWSUM, int TB>
__global__ __launch_bounds__(NT, 2) void gemm_kernel(
    Src A, Src B, Dst C, const float* __restrict__ bias, float* __restrict__ rowsum,
    int M, int N, int K, int kps) {
  constexpr int STAGE = 2 * TB * LDK;  // A + B tiles, elements
  constexpr int MI = TB / 32;          // 16-row tiles of a wave's quadrant
  constexpr int PF = ahead(TB);
  __shared__ __align__(16) float smem[2 * STAGE];

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.y * TB, n0 = blockIdx.x * TB;
  const int kbeg = blockIdx.z * kps;
  const int kend = min(K, kbeg + kps);
  const bool do_sum = ROWSUM && blockIdx.x == 0;

  Loader<AK, TB> la[PF];  // tile j waits in set j % PF
  Loader<BKM, TB> lb[PF];
  float rs[4] = {0.f, 0.f, 0.f, 0.f}, none[4];
  f32x4_t acc[MI][MI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < MI; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int nk = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  // (tiles past the last load the first chunk over and over)
  auto load = [&](int kt, int set) {
    la[set].load(A, m0, M, kbeg + kt * BK, kend);
    lb[set].load(B, n0, N, kbeg + kt * BK, kend);
  };
  auto store = [&](int kt, int set) {
    float* to = smem + (kt & 1) * STAGE;
    const int k0 = kbeg + kt * BK;
    la[set].template store<ROWSUM>(to, m0, M, k0, kend, rs);
    lb[set].template store<false>(to + TB * LDK, n0, N, k0, kend, none);
  };
  if (nk > 0) {  // (no k: the operands may not be there at all)
#pragma unroll
    for (int p = 0; p < PF; ++p) load(p, p);
    store(0, 0);
  }
  __syncthreads();

  for (int kt0 = 0; kt0 < nk; kt0 += PF) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int kt = kt0 + u;  // (kt % PF == u)
      if (kt >= nk) break;
      load(kt + PF, u);  // (tile kt, in LDS by now, was in this set)
      // (keeps the loads ahead of the products: the compiler would sink them
      // to where their registers are stored)
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      const float* sa = smem + (kt & 1) * STAGE;
      const float* sb = sa + TB * LDK;
      const int koff = (lane >> 4) * 8;
      Frag<float> af[MI], bfr[MI];
#pragma unroll
      for (int i = 0; i < MI; ++i)
        af[i] = frag_load<float>(sa + (wm * (TB / 2) + i * 16 + (lane & 15)) * LDK + koff);
#pragma unroll
      for (int j = 0; j < MI; ++j)
        bfr[j] = frag_load<float>(sb + (wn * (TB / 2) + j * 16 + (lane & 15)) * LDK + koff);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) mma_16x16x32(acc[i][j], af[i], bfr[j]);
      if (kt + 1 < nk) store(kt + 1, (u + 1) % PF);
      __syncthreads();
    }
  }

  if (do_sum) {  // smem is free after the final barrier of the loop
    if (threadIdx.x < 2 * TB) {
#pragma unroll
      for (int q = 0; q < 4; ++q) smem[Loader<false, TB>::kb() * TB + Loader<false, TB>::mb() * 4 + q] = rs[q];
    }
    __syncthreads();
    if (threadIdx.x < TB && m0 + (int)threadIdx.x < M) {
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < 8; ++k) s += smem[k * TB + threadIdx.x];
      rowsum[(int64_t)blockIdx.z * M + m0 + threadIdx.x] = s;
    }
  }

#pragma unroll
  for (int j = 0; j < MI; ++j) {
    const int col = n0 + wn * (TB / 2) + j * 16 + mfma_col(lane);
    if (col >= N) continue;
    const float bv = BIAS ? bias[col] : 0.f;
    const bool second = col >= C.split;
    float* cbase = (second ? C.c1 : C.c0) + (int64_t)blockIdx.z * C.zstride;
    const int64_t ldc = second ? C.ld1 : C.ld0;
    const int ccol = second ? col - C.split : col;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * (TB / 2) + i * 16 + mfma_row(lane, r);
        if (row < M) cbase[(int64_t)row * ldc + ccol] = acc[i][j][r] + bv;
      }
    }
  }
}

// Sum of the split-K partials in split order, routed to the two destinations,
// and of the partial row sums.
// V4: every destination row chunk is 16-byte aligned (pointers, pitches
// and the column split multiples of 4 floats), so the sum leaves as one
// 16-byte store instead of four 4-byte ones.
template <bool V4>
__global__ __launch_bounds__(256) void splitk_reduce(const float* __restrict__ part, int S, int M,
                                                     int N, float* __restrict__ c0, int64_t ld0,
                                                     float* __restrict__ c1, int64_t ld1, int split,
                                                     const float* __restrict__ rs_part,
                                                     float* __restrict__ rowsum) {
  const int64_t MN = (int64_t)M * N;
  const int64_t nq = MN / 4;  // N % 4 == 0
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < nq) {
    const float4* p = reinterpret_cast<const float4*>(part) + i;
    float4 s = p[0];
    for (int k = 1; k < S; ++k) {
      const float4 v = p[k * nq];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    const int64_t e = i * 4;
    const int m = (int)(e / N), n = (int)(e % N);
    float* dst = n >= split ? c1 + (int64_t)m * ld1 + (n - split) : c0 + (int64_t)m * ld0 + n;
    if constexpr (V4) {
      *reinterpret_cast<float4*>(dst) = s;
    } else {
      dst[0] = s.x; dst[1] = s.y; dst[2] = s.z; dst[3] = s.w;
    }
  } else if (rowsum && i - nq < M) {
    const int64_t m = i - nq;
    float s = rs_part[m];
    for (int k = 1; k < S; ++k) s += rs_part[(int64_t)k * M + m];
    rowsum[m] = s;
  }
}

template <bool AK, bool BKM, bool BIAS, bool ROWSUM>
void launch(int tb, const GemmArgs& g, Dst dst, float* rowsum, int S, int kps, hipStream_t s) {
  const float* a = static_cast<const float*>(g.A);
  const float* b = static_cast<const float*>(g.B);
  Src A{a, g.lda, a, g.lda, 1 << 30};
  Src B{b, g.ldb, g.B2 ? static_cast<const float*>(g.B2) : b, g.B2 ? g.ldb2 : g.ldb,
        g.B2 ? g.n_split : (1 << 30)};
  const dim3 grid((g.N + tb - 1) / tb, (g.M + tb - 1) / tb, S);
  const float* bias = static_cast<const float*>(g.bias);
  if (tb == 32)
    hipLaunchKernelGGL((gemm_kernel<AK, BKM, BIAS, ROWSUM, 32>), grid, dim3(NT), 0, s, A, B, dst, bias,
                       rowsum, g.M, g.N, g.K, kps);
  else if (tb == 64)
    hipLaunchKernelGGL((gemm_kernel<AK, BKM, BIAS, ROWSUM, 64>), grid, dim3(NT), 0, s, A, B, dst, bias,
                       rowsum, g.M, g.N, g.K, kps);
  else
    hipLaunchKernelGGL((gemm_kernel<AK, BKM, BIAS, ROWSUM, 128>), grid, dim3(NT), 0, s, A, B, dst, bias,
                       rowsum, g.M, g.N, g.K, kps);
}

Dst direct_dst(const GemmArgs& g) {
  Dst d;
  d.c0 = static_cast<float*>(g.C);
  d.ld0 = g.ldc;
  d.c1 = static_cast<float*>(g.C2 ? g.C2 : g.C);
  d.ld1 = g.C2 ? g.ldc2 : g.ldc;
  d.split = g.C2 ? g.n_split : (1 << 30);
  d.zstride = 0;
  return d;
}

// Estimated clocks of a product in tiles of edge tb and S k-splits: per
// k-tile, what the compute unit with the most workgroups needs for their
// products, and at least what one workgroup's loads and LDS round trip take;
// plus the start and the end.  The clocks are measured ones (a quadrant's MFMAs
// alone are 4096, 1024 and 256): 6400 x 512 x 2048 in 200 tiles of 128 runs 170
// us against 195 in 800 of 64 and 258 in 3200 of 32; 4096 x 96 x 1000 in 32
// tiles of 128 110 us, 128 of 64 45, 384 of 32 35.
double tile_clocks(const GemmArgs& g, int tb, int S) {
  const int64_t wgs = (int64_t)((g.N + tb - 1) / tb) * ((g.M + tb - 1) / tb) * S;
  const double rounds = (double)((wgs + 255) / 256);
  const int ktiles = (g.K + BK - 1) / BK, per = (ktiles + S - 1) / S;
  const double work = tb == 128 ? 4500.0 : tb == 64 ? 1250.0 : 640.0;
  const double alone = tb == 128 ? 4500.0 : tb == 64 ? 2000.0 : 1500.0;
  return 2500.0 + per * (rounds * work > alone ? rounds * work : alone);
}

int pick_tile(const GemmArgs& g, int S) {
  int best = 128;
  for (int tb : {64, 32})
    if (tile_clocks(g, tb, S) < tile_clocks(g, best, S)) best = tb;
  return best;
}

hipError_t dispatch(const GemmArgs& g, hipStream_t s) {
  if (g.a_kmajor && g.b_kmajor) {           // NT: forward projections
    const int tb = pick_tile(g, 1);
    if (g.bias) launch<true, true, true, false>(tb, g, direct_dst(g), nullptr, 1, g.K, s);
    else launch<true, true, false, false>(tb, g, direct_dst(g), nullptr, 1, g.K, s);
    return hipGetLastError();
  }
  if (g.a_kmajor && !g.b_kmajor && !g.bias && !g.rowsum) {  // NN: data gradients
    launch<true, false, false, false>(pick_tile(g, 1), g, direct_dst(g), nullptr, 1, g.K, s);
    return hipGetLastError();
  }
  if (!g.a_kmajor && !g.b_kmajor && !g.bias) {  // TN: weight gradients
    const int ktiles = (g.K + BK - 1) / BK;
    int S = 1, tb = pick_tile(g, 1);
    if (g.ws) {
      // tile edge and splits together; a split sum costs a reduction, about a
      // launch (10,000 clocks) and its traffic
      double best = tile_clocks(g, tb, 1);
      for (int t : {128, 64, 32})
        for (int c = 2; c <= 8; ++c) {
          if (ktiles / c < 4 || (int64_t)c * g.M * g.N + (int64_t)c * g.M > g.ws_floats) break;
          const double est = tile_clocks(g, t, c) + 10000.0 + (double)c * g.M * g.N * 8.0 / 1600.0;
          if (est < best) { best = est; S = c; tb = t; }
        }
    }
    if (S == 1) {
      if (g.rowsum) launch<false, false, false, true>(tb, g, direct_dst(g), g.rowsum, 1, g.K, s);
      else launch<false, false, false, false>(tb, g, direct_dst(g), nullptr, 1, g.K, s);
      return hipGetLastError();
    }
    const int kps = ((ktiles + S - 1) / S) * BK;
    float* part = g.ws;
    float* rs_part = g.ws + (int64_t)S * g.M * g.N;
    Dst d{part, g.N, part, g.N, 1 << 30, (int64_t)g.M * g.N};  // one slice per split
    if (g.rowsum) launch<false, false, false, true>(tb, g, d, rs_part, S, kps, s);
    else launch<false, false, false, false>(tb, g, d, nullptr, S, kps, s);
    return splitk_reduce_launch(part, S, g, rs_part, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t splitk_reduce_launch(const float* part, int S, const GemmArgs& g, const float* rs_part,
                                hipStream_t s) {
  const int64_t nq = (int64_t)g.M * g.N / 4;
  const int64_t threads = nq + (g.rowsum ? g.M : 0);
  float* c0 = static_cast<float*>(g.C);
  float* c1 = static_cast<float*>(g.C2 ? g.C2 : g.C);
  const int64_t ld1 = g.C2 ? g.ldc2 : g.ldc;
  const int split = g.C2 ? g.n_split : (1 << 30);
  const bool v4 = (reinterpret_cast<uintptr_t>(c0) | reinterpret_cast<uintptr_t>(c1)) % 16 == 0 &&
                  g.ldc % 4 == 0 && ld1 % 4 == 0 && split % 4 == 0;
  if (v4)
    hipLaunchKernelGGL(splitk_reduce<true>, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s,
                       part, S, g.M, g.N, c0, g.ldc, c1, ld1, split, rs_part, g.rowsum);
  else
    hipLaunchKernelGGL(splitk_reduce<false>, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s,
                       part, S, g.M, g.N, c0, g.ldc, c1, ld1, split, rs_part, g.rowsum);
  return hipGetLastError();
}

hipError_t gemm(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  return g.bf16 ? gemm_bf16(g, s) : dispatch(g, s);
}

}  // namespace am
