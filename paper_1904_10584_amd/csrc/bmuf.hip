// BMUF-NBM global step (blockwise model update filtering with Nesterov block
// momentum, §VI-B eqs. (2)-(5)), one HBM-bound pass over the flat model:
//   Wbar  = (sum of the `count` addends) / workers       (2)
//   G     = Wbar - W_g                                   (3)
//   Delta = eta Delta + zeta G                           (4)
//   W_g   = W_g + Delta + eta_next Delta                 (5)
// and, optionally, the restart copy of the local model (fp32 and bf16).
// Each element is evaluated in fp64 from its fp32 inputs, in the order
// written, with no fused multiply-add, and each output is rounded once to
// fp32, so the result is bit-identical to the element-wise definition.
// Every thread reads all inputs of its elements before writing any output,
// so outputs may alias inputs of the same index (in-place W_g and Delta, or
// the local model written over one of the addends).
#include "am_device.h"
#include "am_internal.h"

namespace am {
namespace {

struct BmufOne {
  float w, d;
};

__device__ __forceinline__ BmufOne bmuf_one(double s, float wg, float d0, double workers,
                                            double eta, double eta_next, double zeta) {
#pragma clang fp contract(off)
  const double wbar = s / workers;
  const double g = wbar - (double)wg;
  const double d = eta * (double)d0 + zeta * g;
  const double w = ((double)wg + d) + eta_next * d;
  return BmufOne{(float)w, (float)d};
}

// Accesses of four elements at the elements' own alignment (the rows of a
// model array of odd length start anywhere), which the memory instructions
// take: 16 bytes from any multiple of 4.
typedef f32x4_t f32x4_u __attribute__((aligned(4)));
typedef uint16_t u16x4_t __attribute__((ext_vector_type(4)));
typedef u16x4_t u16x4_u __attribute__((aligned(2)));

template <bool STREAM>
__device__ __forceinline__ f32x4_t load4(const float* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const f32x4_u*>(p));
  else return *reinterpret_cast<const f32x4_u*>(p);
}
template <bool STREAM>
__device__ __forceinline__ void store4(float* p, f32x4_t v) {
  if constexpr (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<f32x4_u*>(p));
  else *reinterpret_cast<f32x4_u*>(p) = v;
}

// Four elements of K models added to s in order, the K loads requested before
// the first add.
template <int K, bool STREAM>
__device__ __forceinline__ void add_models(double* s, const float* m, int64_t stride) {
#pragma clang fp contract(off)
  f32x4_t v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = load4<STREAM>(m + k * stride);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] = s[q] + (double)v[k][q];
}

// Four elements a thread, the whole array in one grid (a loop over 8192
// workgroups ended unevenly: 258 us where one grid took 239).  What bounds it:
// HBM, or the memory-side cache.  BATCH: the models asked for eight and four at a
// time, ahead of their adds.  STREAM: every access non-temporal (see the launch
// for both).  24,145,848 elements, 8 addends, both restart copies (1.30 GB): 245 ->
// 216 us on one card, 248 -> 229 on another; 10,000,001 elements, 3 addends, whose
// rows start off the 16-byte grid (one element at a time before): 216 -> 52.
template <bool BATCH, bool STREAM>
__global__ __launch_bounds__(256) void bmuf_kernel(int64_t n, int count, double workers,
                                                   const float* models,
                                                   int64_t stride, float* wg, float* delta,
                                                   double eta, double eta_next, double zeta,
                                                   float* local, bf16_t* local_bf16) {
#pragma clang fp contract(off)
  const int64_t step = (int64_t)gridDim.x * 256 * 4;
  for (int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; e < n; e += step) {
    if (e + 3 < n) {
      double s[4] = {0.0, 0.0, 0.0, 0.0};
      const float* m = models + e;
      f32x4_t w4, d4;
      if constexpr (BATCH) {
        w4 = load4<STREAM>(wg + e);
        d4 = load4<STREAM>(delta + e);
        int i = 0;
        for (; i + 8 <= count; i += 8) add_models<8, STREAM>(s, m + (int64_t)i * stride, stride);
        if (count - i >= 4) {
          add_models<4, STREAM>(s, m + (int64_t)i * stride, stride);
          i += 4;
        }
        for (; i < count; ++i) add_models<1, STREAM>(s, m + (int64_t)i * stride, stride);
      } else {
#pragma unroll 1
        for (int i = 0; i < count; ++i, m += stride) {
          const f32x4_t v = load4<STREAM>(m);
#pragma unroll
          for (int q = 0; q < 4; ++q) s[q] = s[q] + (double)v[q];
        }
        w4 = load4<STREAM>(wg + e);
        d4 = load4<STREAM>(delta + e);
      }
      f32x4_t nw, nd;
      u16x4_t b;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const BmufOne r = bmuf_one(s[q], w4[q], d4[q], workers, eta, eta_next, zeta);
        nw[q] = r.w;
        nd[q] = r.d;
        b[q] = f32_to_bf16(r.w);
      }
      store4<STREAM>(wg + e, nw);
      store4<STREAM>(delta + e, nd);
      if (local) store4<STREAM>(local + e, nw);
      if (local_bf16) {
        if constexpr (STREAM) __builtin_nontemporal_store(b, reinterpret_cast<u16x4_u*>(local_bf16 + e));
        else *reinterpret_cast<u16x4_u*>(local_bf16 + e) = b;
      }
    } else {
      for (int64_t j = e; j < n; ++j) {
        double s = 0.0;
        for (int i = 0; i < count; ++i) s = s + (double)models[(int64_t)i * stride + j];
        const BmufOne r = bmuf_one(s, wg[j], delta[j], workers, eta, eta_next, zeta);
        wg[j] = r.w;
        delta[j] = r.d;
        if (local) local[j] = r.w;
        if (local_bf16) local_bf16[j] = f32_to_bf16(r.w);
      }
    }
  }
}

}  // namespace

hipError_t bmuf_update(int64_t n, int count, int workers, const float* models, int64_t stride,
                       float* wg, float* delta, float eta, float eta_next, float zeta,
                       float* local, uint16_t* local_bf16, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t want = ((n + 3) / 4 + 255) / 256;
  const unsigned blocks = (unsigned)(want < (1 << 20) ? want : (1 << 20));
  // Streamed where the 256 MB memory-side cache keeps nothing from one update to
  // the next: the addends alone overflow it, or everything touched does twice
  // over.  Below, what is left in it (the models were just written, and the last
  // update's results) is worth more.  Plain / streamed, us, models just written:
  // 8 M x 3 (259 MiB) 43.4 / 44.4, 10 M x 4 (362 MiB) 58.6 / 59.7, 20 M x 1 (496
  // MiB) 83.6 / 84.2, 10 M x 8 (addends 305 MiB) 97.4 / 90.5, 20 M x 2 (572 MiB)
  // 104 / 96, 24.1 M x 8 (1.2 GiB) 246 / 218; updates back to back: 40.1 / 45.5,
  // 56.1 / 62.3, 79.3 / 87.9, 94.3 / 88.4, 105.8 / 104.4 and 247 / 221.
  const int64_t addends = n * 4 * (int64_t)count;
  const int64_t bytes = addends + n * (8 + 8 + (local ? 4 : 0) + (local_bf16 ? 2 : 0));
  const bool stream = addends > ((int64_t)256 << 20) || bytes > ((int64_t)544 << 20);
  // Batches of loads where memory latency is what they hide, and for rows off the
  // 16-byte grid, whose accesses take two lines; from the cache, more waves with
  // fewer registers do as well or better.  One at a time / batches, us: 1 M x 15
  // 13.0 / 13.9, 2 M x 16 (149 MiB) 25.0 / 26.1, 6 M x 7 (286 MiB) 43.1 / 43.9, 6 M x
  // 9 (332 MiB) 54.3 / 50.5, 6 M x 11 (378 MiB) 65.5 / 63.7; 1,000,003 x 8 12.6 /
  // 10.8.
  const uintptr_t off = (reinterpret_cast<uintptr_t>(models) | reinterpret_cast<uintptr_t>(wg) |
                         reinterpret_cast<uintptr_t>(delta)) % 16;
  const bool aligned = off == 0 && (count == 1 || stride % 4 == 0);
  const bool batch = stream || !aligned || bytes > ((int64_t)288 << 20);
  auto kernel = stream ? bmuf_kernel<true, true> : batch ? bmuf_kernel<true, false> : bmuf_kernel<false, false>;
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, s, n, count,
                     (double)workers, models, stride, wg, delta, (double)eta, (double)eta_next,
                     (double)zeta, local, local_bf16);
  return hipGetLastError();
}

}  // namespace am
