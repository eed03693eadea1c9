// Teacher target generation (§V-A, §V-C): the pieces the bidirectional
// teacher adds to the student's kernels, and the k-best logits.
//
// gather_rows: copies the packed rows of a batch, optionally reversing each
// sequence in time (row (t, b) takes row (len_b - 1 - t, b)), into a column
// range of another matrix.  The teacher's backward direction runs the
// student's forward recurrence on the time-reversed input projections and
// writes its hidden states back in time order next to the forward
// direction's.  One thread per 16-byte chunk; a row's frame index comes from
// a binary search in the packed row offsets.
//
// topk_rows: the k largest logits of each row in descending order (equal
// values by ascending index, NaN after every number), one wave per row with
// the row held in registers as order-preserving integer keys.  The row's
// entries fall into 64 or 128 groups; the k-th largest of the groups' maxima
// is a bound that at least k entries reach and few more do.  Those entries are
// gathered in LDS, and each lane finds the rank of its one or two of them by
// comparing with all: the rank is the place in the output.  Where more than 128
// reach it, the equal values at the bound are cut to what is left to k, in order.
// What bounds it: the vector unit's passes over the row's registers; 16384 x 3000,
// k = 20: 93 us (k rounds for every row, loads behind branches) -> 53, rows of equal
// values 149 -> 59.  Few k of short rows (DIRECT), and rows with more than 128
// entries above the bound, take k rounds of a wave-wide maximum instead.
//
// kbest_posterior_rows: the posterior rebuilt from k stored logits with the
// missing ones at -infinity, i.e. the softmax over the k values (fp32; sums in
// the order of the entries).
#include <cmath>

#include "am_device.h"
#include "am_internal.h"

namespace am {
namespace {

// Device copies of a batch's schedule: offs[t] = sum_b min(len_b, t) for
// t = 0..T, and the lengths.
__global__ __launch_bounds__(256) void schedule_tables_kernel(SchedTables a) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t <= a.T) {
    int64_t o = 0;
    for (int b = 0; b < a.B; ++b) o += a.len[b] < t ? a.len[b] : t;
    a.offs[t] = o;
  }
  if (t < a.B) a.lens[t] = a.len[t];
}

template <typename T>
__global__ __launch_bounds__(256) void gather_rows_kernel(GatherRows a) {
  constexpr int EPC = 16 / sizeof(T);
  const int cpr = a.width / EPC;
  const int64_t total = a.N * cpr;
  const T* __restrict__ src = static_cast<const T*>(a.src);
  T* __restrict__ dst = static_cast<T*>(a.dst);
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int64_t r = e / cpr;
    const int c = (int)(e % cpr);
    int64_t sr = r;
    if (a.reverse) {
      // frame t of row r: the last t with offs[t] <= r
      int lo = 0, hi = a.T - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.offs[mid] <= r) lo = mid; else hi = mid - 1;
      }
      const int b = (int)(r - a.offs[lo]);
      sr = a.offs[a.lens[b] - 1 - lo] + b;
    }
    const uint4 v = *reinterpret_cast<const uint4*>(src + sr * a.src_ld + c * EPC);
    *reinterpret_cast<uint4*>(dst + r * a.dst_ld + a.dst_col + c * EPC) = v;
  }
}

// Order-preserving key of a logit: larger values get larger keys, -0 and +0
// the same key, NaN key 1 (below every number), and 0 marks an entry already
// taken.  A wave-wide candidate is (key << 32) | ~index, so equal keys rank
// the lower index first.
__device__ __forceinline__ uint32_t logit_key(float f) {
  if (f != f) return 1u;
  uint32_t u = __float_as_uint(f == 0.f ? 0.f : f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int CANDS = 128;  // entries that reach a row's bound, at most

// A wave's LDS accesses on either side stay there (the hardware runs them in
// order).
__device__ __forceinline__ void wave_lds_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// Wavefronts a SIMD that the registers are to leave room for: those of the common
// rows' passes, which the code for the rare ones would push down by one (16384 x
// 3000, k = 20: 61 us at three, 52 at four; the rare ones spill a few registers).
constexpr int topk_waves(int cpl, bool direct) {
  return direct ? 1 : cpl <= 16 ? 8 : cpl <= 32 ? 5 : cpl <= 48 ? 4 : cpl <= 64 ? 3 : cpl <= 96 ? 2 : 1;
}

template <int CPL, bool VEC, bool DIRECT>
__global__ __launch_bounds__(256, topk_waves(CPL, DIRECT)) void topk_rows_kernel(int64_t N, int C, int K,
                                                        const float* __restrict__ z,
                                                        int32_t* __restrict__ idx,
                                                        float* __restrict__ val) {
  static_assert(CPL % 4 == 0, "registers in fours");
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= N) return;
  const float* zr = z + row * C;
  // register q holds class cls(q): with VEC (C % 4 == 0) four consecutive
  // classes per 16-byte load, else one class per 64-lane stride
  auto cls = [&](int q) {
    return VEC ? 4 * lane + 256 * (q >> 2) + (q & 3) : lane + 64 * q;
  };
  // (a lane past the row re-reads its start and takes key 0: a load behind a
  // branch would be waited for before the next one issues)
  uint32_t key[CPL];
  {
    float f[CPL];
#pragma unroll
    for (int q = 0; q < CPL; q += VEC ? 4 : 1) {
      const int c = cls(q) < C ? cls(q) : 0;
      if (VEC) *reinterpret_cast<float4*>(f + q) = *reinterpret_cast<const float4*>(zr + c);
      else f[q] = zr[c];
    }
#pragma unroll
    for (int q = 0; q < CPL; ++q) key[q] = cls(q) < C ? logit_key(f[q]) : 0u;
  }
  // candidate of register q: (key << 32) | ~class, unique per class, larger
  // = earlier in the output; 0 for no class
  auto cand = [&](int q) -> uint64_t {
    return key[q] ? ((uint64_t)key[q] << 32) | (uint32_t)~(uint32_t)cls(q) : 0ull;
  };

  if constexpr (!DIRECT) {
    __shared__ __align__(16) uint64_t scratch[4][CANDS];
    uint64_t* mine_lds = scratch[threadIdx.x >> 6];
    // set bits of m below this lane's
    auto below = [](uint64_t m) {
      return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
    };
    // Group maxima: registers of four by four in turn, one group a lane (k <=
    // 32: about 1.4 k entries reach the k-th largest of 64 maxima) or two.
    uint32_t g0 = 0, g1 = 0;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if ((q >> 2) & 1) g1 = key[q] > g1 ? key[q] : g1;
      else g0 = key[q] > g0 ? key[q] : g0;
    }
    uint32_t bound;
    {
      // the k-th largest: the one with k - 1 before it, equal ones in the
      // order of their groups
      uint32_t* gl = reinterpret_cast<uint32_t*>(mine_lds);
      uint32_t r0 = 0, r1 = 0;
      const bool two = K > 32;  // (uniform)
      if (!two) g0 = g0 > g1 ? g0 : g1;
      gl[lane] = g0;
      gl[64 + lane] = two ? g1 : 0u;
      wave_lds_order();
      const uint4* gv = reinterpret_cast<const uint4*>(gl);
      auto count = [&](uint32_t v, int at) {
        r0 += v > g0 || (v == g0 && at < lane);
        r1 += v > g1 || (v == g1 && at < 64 + lane);
      };
      const int nv = two ? 32 : 16;
      for (int i = 0; i < nv; i += 4) {
        uint4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = gv[i + j];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          count(v[j].x, 4 * (i + j));
          count(v[j].y, 4 * (i + j) + 1);
          count(v[j].z, 4 * (i + j) + 2);
          count(v[j].w, 4 * (i + j) + 3);
        }
      }
      const uint64_t h0 = __ballot(r0 == (uint32_t)(K - 1)), h1 = two ? __ballot(r1 == (uint32_t)(K - 1)) : 0ull;
      bound = h0 ? (uint32_t)__builtin_amdgcn_readlane((int)g0, __builtin_ctzll(h0))
                 : (uint32_t)__builtin_amdgcn_readlane((int)g1, __builtin_ctzll(h1 ? h1 : 1ull));
      wave_lds_order();
    }
    // (no bound where fewer than k groups hold anything: every entry counts)
    if (bound == 0u) bound = 1u;
    int n = 0;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const uint64_t hit = __ballot(key[q] >= bound);
      if (hit) {  // (uniform)
        const int at = n + below(hit);
        if (key[q] >= bound && at < CANDS) mine_lds[at] = cand(q);
        n += __popcll(hit);
      }
    }
    if (n > CANDS) {
      // Equal values at the bound: those above it, then of the equal ones as many
      // as are left to K, by ascending class.  (More than CANDS above it: rounds.)
      int m = 0;
#pragma unroll
      for (int q = 0; q < CPL; ++q) {
        const uint64_t hit = __ballot(key[q] > bound);
        if (hit) {
          const int at = m + below(hit);
          if (key[q] > bound && at < CANDS) mine_lds[at] = cand(q);
          m += __popcll(hit);
        }
      }
      n = m;
      constexpr int E = VEC ? 4 : 1;  // classes of a lane side by side
#pragma unroll
      for (int q = 0; q < CPL; q += E)
        if (n < K) {  // (uniform)
          uint64_t tie[E];
          int at = n;
#pragma unroll
          for (int e = 0; e < E; ++e) {
            tie[e] = __ballot(key[q + e] == bound);
            at += below(tie[e]);
            n += __popcll(tie[e]);
          }
#pragma unroll
          for (int e = 0; e < E; ++e)
            if (key[q + e] == bound) {
              if (at < K) mine_lds[at] = cand(q + e);
              ++at;
            }
        }
      if (m < K) n = K;
    }
    if (n <= CANDS) {
      wave_lds_order();
      const uint64_t c0 = lane < n ? mine_lds[lane] : 0ull, c1 = 64 + lane < n ? mine_lds[64 + lane] : 0ull;
      int r0 = 0, r1 = 0;
      int i = 0;
      for (; i + 4 <= n; i += 4) {
        uint64_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = mine_lds[i + j];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          r0 += v[j] > c0;
          r1 += v[j] > c1;
        }
      }
      for (; i < n; ++i) {
        r0 += mine_lds[i] > c0;
        r1 += mine_lds[i] > c1;
      }
      if (lane < n && r0 < K) {
        const int c = (int)~(uint32_t)c0;
        idx[row * K + r0] = c;
        val[row * K + r0] = zr[c];  // (the value itself: signed zeros and NaN payloads)
      }
      if (64 + lane < n && r1 < K) {
        const int c = (int)~(uint32_t)c1;
        idx[row * K + r1] = c;
        val[row * K + r1] = zr[c];
      }
      return;
    }
  }

  // this lane's best two candidates, from one pass over its registers
  uint64_t b0 = 0ull, b1 = 0ull;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const uint64_t v = cand(q);
    const bool g0 = v > b0, g1 = v > b1;
    b1 = g0 ? b0 : (g1 ? v : b1);
    b0 = g0 ? v : b0;
  }
  bool second = true;  // b1 still holds this lane's next candidate
  int mine = -1;       // lane j keeps the class of round j
  for (int j = 0; j < K; ++j) {
    uint64_t best = b0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const uint64_t other = __shfl_xor(best, o, 64);
      best = other > best ? other : best;
    }
    if (best == 0ull) continue;  // fewer than K entries: -1 below
    if (lane == j) mine = (int)~(uint32_t)best;
    if (b0 == best) {  // the lane that held it takes its next candidate
      if (second) {
        b0 = b1;
        second = false;
      } else {  // the best of its candidates below the one taken
        uint64_t m = 0ull;
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          const uint64_t v = cand(q);
          m = (v < best && v > m) ? v : m;
        }
        b0 = m;
      }
    }
  }
  // the k results, one lane each (values reloaded from the row: exact,
  // signed zeros and NaN payloads included)
  if (lane < K) {
    idx[row * K + lane] = mine;
    val[row * K + lane] = mine >= 0 ? zr[mine] : -INFINITY;
  }
}

__global__ __launch_bounds__(256) void kbest_posterior_rows(int64_t N, int K,
                                                            const float* __restrict__ val,
                                                            float* __restrict__ prob) {
  const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (row >= N) return;
  const float* v = val + row * K;
  float m = -INFINITY;
  for (int j = 0; j < K; ++j) m = fmaxf(m, v[j]);
  float s = 0.f;
  for (int j = 0; j < K; ++j) s += expf(v[j] - m);
  for (int j = 0; j < K; ++j) prob[row * K + j] = expf(v[j] - m) / s;
}

// The same with the rows in LDS: coalesced in and out, the exponentials and
// the quotients spread over the workgroup; the maximum and the sum of a row
// stay one thread's, in the order of the entries, so the bits are those of the
// kernel above (whose threads each walk a row in memory three times: 11 us for
// 16384 rows of 20, now 5.4).
constexpr int KBP_FLOATS = 4096;
__global__ __launch_bounds__(256) void kbest_posterior_tiles(int64_t N, int K, int rows,
                                                             const float* __restrict__ val,
                                                             float* __restrict__ prob) {
  __shared__ float v[KBP_FLOATS];
  __shared__ float red[64];  // a row's maximum, then its sum
  const int64_t r0 = (int64_t)blockIdx.x * rows;
  const int nr = (int)(N - r0 < rows ? N - r0 : rows), ne = nr * K;
  for (int e = threadIdx.x; e < ne; e += 256) v[e] = val[r0 * K + e];
  __syncthreads();
  const int r = threadIdx.x;
  if (r < nr) {
    float m = -INFINITY;
    for (int j = 0; j < K; ++j) m = fmaxf(m, v[r * K + j]);
    red[r] = m;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < ne; e += 256) v[e] = expf(v[e] - red[e / K]);
  __syncthreads();
  if (r < nr) {
    float s = 0.f;
    for (int j = 0; j < K; ++j) s += v[r * K + j];
    red[r] = s;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < ne; e += 256) prob[r0 * K + e] = v[e] / red[e / K];
}

}  // namespace

hipError_t schedule_tables(const SchedTables& a, hipStream_t s) {
  const int n = (a.T + 1 > a.B ? a.T + 1 : a.B);
  hipLaunchKernelGGL(schedule_tables_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t gather_rows(const GatherRows& a, bool bf16, hipStream_t s) {
  const int epc = bf16 ? 8 : 4;
  const int64_t total = a.N * (a.width / epc);
  if (total == 0) return hipSuccess;
  const int64_t want = (total + 255) / 256;
  const unsigned grid = (unsigned)(want < 65536 ? want : 65536);
  if (bf16)
    hipLaunchKernelGGL(gather_rows_kernel<bf16_t>, dim3(grid), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(gather_rows_kernel<float>, dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

#define AM_TOPK_CASE(CPL_, DIRECT_)                                                           \
  if (cpl <= CPL_ && direct == DIRECT_) {                                                     \
    auto kernel = vec ? topk_rows_kernel<CPL_, true, DIRECT_> : topk_rows_kernel<CPL_, false, DIRECT_>; \
    hipLaunchKernelGGL(kernel, dim3((unsigned)((N + 3) / 4)), dim3(256), 0, s, N, C, K, z, idx, val); \
    return hipGetLastError();                                                                 \
  }

hipError_t topk_rows(int64_t N, int C, int K, const float* z, int32_t* idx, float* val,
                     hipStream_t s) {
  if (N == 0 || K == 0) return hipSuccess;
  const int cpl = (C + 63) / 64;
  // 16-byte row loads need every row start 16-byte aligned
  const bool vec = C % 4 == 0 && (reinterpret_cast<uintptr_t>(z) & 15) == 0;
  // k rounds at once where they are the faster ones: the bound costs about ten of
  // them on rows of up to 1024 entries, six up to 2048, and is never worth it where
  // most of a short row would reach it
  // rounds alone for few k of short rows.  Rounds / bound, us for 32768 rows: 256
  // entries, k = 4, 12 / 14, k = 5, 14 / 14; 512 entries, k = 8, 29 / 32, k = 10, 33 /
  // 31; 1024, k = 10, 45 / 48, k = 12, 52 / 48; 16384 rows of 2048, k = 6, 37 / 40, k =
  // 10, 43 / 40
  const int few = cpl <= 4 ? 5 : cpl <= 8 ? 9 : cpl <= 12 ? 10 : cpl <= 16 ? 11 : cpl <= 32 ? 8 : 0;
  // (rows of up to 256 entries fill C / 4 groups: fewer than k of them give no bound)
  const bool direct = K < few || (C > CANDS && C <= 256 && 4 * K >= C);
  AM_TOPK_CASE(4, true) AM_TOPK_CASE(8, true) AM_TOPK_CASE(12, true) AM_TOPK_CASE(16, true)
  AM_TOPK_CASE(32, true)
  AM_TOPK_CASE(4, false) AM_TOPK_CASE(8, false) AM_TOPK_CASE(12, false) AM_TOPK_CASE(16, false)
  AM_TOPK_CASE(32, false) AM_TOPK_CASE(48, false) AM_TOPK_CASE(64, false) AM_TOPK_CASE(96, false)
  AM_TOPK_CASE(128, false)
  return hipErrorInvalidValue;
}

hipError_t kbest_posteriors(int64_t N, int K, const float* val, float* prob, hipStream_t s) {
  if (N == 0 || K == 0) return hipSuccess;
  if (K <= KBP_FLOATS) {  // (longer rows do not fit the tile)
    const int rows = KBP_FLOATS / K < 64 ? KBP_FLOATS / K : 64;
    hipLaunchKernelGGL(kbest_posterior_tiles, dim3((unsigned)((N + rows - 1) / rows)), dim3(256), 0, s,
                       N, K, rows, val, prob);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(kbest_posterior_rows, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, N,
                     K, val, prob);
  return hipGetLastError();
}

}  // namespace am
