// The student's input frames and delayed targets (§II-B).
//
// lfr_features: for each utterance, raw frames (10 ms, raw_dim values each,
// utterances one after another) are stacked `stack` at a time at a `skip`
// advance from a frame offset, the causal mean of the stacked frames so far
// is subtracted, and the result is normalised by global per-dimension mean
// and standard deviation.  Output rows follow the model's packed time-major
// layout (frame (t, b) is row off_t + b), so utterances are given longest
// (in stacked frames) first.  Each value is evaluated in fp64 in the order of
// the definition (the running sum frame by frame, correctly rounded
// divisions) and rounded once to the output type, so the output is
// bit-identical to the element-wise definition.
//
// delay_targets: the targets of the packed rows shifted by `delay` frames
// within each sequence (the model's look-ahead): row (t, b) takes the target
// of row (t - delay, b); rows with t < delay get idx -1, prob 0, mask 0.
#include "am_device.h"
#include "am_internal.h"

namespace am {
namespace {

// fp64 result -> output type, rounded once to fp32 (then to bf16 for a bf16
// model, round to nearest even).
template <typename T> __device__ __forceinline__ T from_f64(double v);
template <> __device__ __forceinline__ float from_f64<float>(double v) { return (float)v; }
template <> __device__ __forceinline__ bf16_t from_f64<bf16_t>(double v) { return f32_to_bf16((float)v); }

// Sum of one value per thread over a 256-thread workgroup (all threads get
// it).  `red` is 4 LDS slots; the call contains two barriers.
__device__ __forceinline__ int64_t block_sum(int64_t v, int64_t* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();  // earlier readers of red are done
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// a / b for a divisor whose correctly rounded reciprocal r = 1 / b is known:
// the quotient of the multiply, corrected twice by its exact remainder.  The
// first correction leaves it within one ulp, and a correction of such a
// quotient with the correctly rounded reciprocal is the correctly rounded
// quotient (Markstein, "Computation of elementary functions on the IBM RISC
// System/6000 processor", 1990).  Valid where in_range holds for the result:
// zeros, infinities, NaN and anything whose remainder could underflow are
// divided instead.
__device__ __forceinline__ double quotient(double a, double b, double r) {
  double q = a * r;
  q = __builtin_fma(__builtin_fma(-q, b, a), r, q);
  return __builtin_fma(__builtin_fma(-q, b, a), r, q);
}
__device__ __forceinline__ bool in_range(double q) {
  const double m = __builtin_fabs(q);
  return m >= 0x1p-900 && m <= 0x1p900;
}

// One workgroup per utterance, one thread per stacked dimension walking the
// frames in order, the loads of the next 32 frames in flight ahead of the
// running sum.  What bounds it: the walk, with its two fp64 divisions, about 0.3
// us a frame; but a workgroup's start is paid once per utterance.
template <typename OutT>
__global__ __launch_bounds__(256) void lfr_walk_kernel(LfrArgs a) {
#pragma clang fp contract(off)
  const int b = blockIdx.x;
  const int D = a.stack * a.raw_dim;
  __shared__ uint16_t T_len[1024];
  __shared__ int64_t red[4];
  int64_t r0 = 0;  // raw frames of the utterances before this one
  for (int i = threadIdx.x; i < a.B; i += 256) {
    const int U = a.U[i];
    const int T = (U - a.offset - a.stack) / a.skip + 1;
    T_len[i] = (uint16_t)(U - a.offset - a.stack >= 0 ? T : 0);
    if (i < b) r0 += U;
  }
  r0 = block_sum(r0, red);  // its barriers also publish T_len
  const int Tb = T_len[b];
  // stacked frame t's dimension j is one raw value: stacking is contiguous
  const float* __restrict__ raw = a.raw + (r0 + a.offset) * a.raw_dim;
  const int64_t fstep = (int64_t)a.skip * a.raw_dim;
  OutT* __restrict__ x = static_cast<OutT*>(a.x);
  for (int j = threadIdx.x; j < D; j += 256) {
    const double mean = (double)a.mean[j], sd = (double)a.std[j];
    double run = 0.0;
    int64_t off = 0;  // packed offset of frame t
    int nb = a.B;     // sequences longer than t
    constexpr int AH = 32;
    float ahead[AH];
#pragma unroll
    for (int q = 0; q < AH; ++q) ahead[q] = q < Tb ? raw[q * fstep + j] : 0.f;
    for (int t0 = 0; t0 < Tb; t0 += AH) {
#pragma unroll
      for (int q = 0; q < AH; ++q) {
        const int t = t0 + q;
        if (t >= Tb) break;
        const double y = (double)ahead[q];
        const int tn = t + AH;
        ahead[q] = tn < Tb ? raw[tn * fstep + j] : 0.f;
        run = run + y;
        const double z = y - run / (double)(t + 1);
        const double v = (z - mean) / sd;
        while (nb > 0 && T_len[nb - 1] <= t) --nb;
        x[(off + b) * D + j] = from_f64<OutT>(v);
        off += nb;
      }
    }
  }
}

// One workgroup per (utterance, 32 stacked dimensions), six waves.  Only the
// running sum has to walk the frames in order, so wave 0 does nothing else: it
// adds chunk i's frames and leaves the sum at every frame in LDS.  Waves 1-4
// meanwhile put chunk i + 1 (loaded four iterations before) into LDS, load
// chunk i + 5, and evaluate and store the frames of chunk i - 1: two frames by
// 32 dimensions at a time, four times.  Wave 5 finds where later chunks'
// frames go.  What bounds it: the evaluation (two fp64 divisions a value, by
// divisors whose reciprocals are kept) and, for long utterances, the walk.  128
// utterances of 200-1500 frames x 192: 770 us by the kernel above, 63 by this one
// (78 with that search on a wave that evaluates too, for which the others waited).
constexpr int LFR_TC = 32;  // frames per chunk
constexpr int LFR_G = 32;   // dimensions per workgroup
constexpr int LFR_THREADS = 6 * 64;

template <typename OutT>
__global__ __launch_bounds__(LFR_THREADS) void lfr_features_kernel(LfrArgs a) {
#pragma clang fp contract(off)
  constexpr int TC = LFR_TC, G = LFR_G;
  constexpr int FPL = TC / 8;  // frames of a chunk per lane of waves 1-4
  constexpr int PD = 4;        // chunks whose loads are in flight
  // (the groups of an utterance side by side, so that the longest utterances'
  // groups start on compute units of their own)
  const int D = a.stack * a.raw_dim, groups = (D + G - 1) / G;
  const int b = blockIdx.x / groups;
  __shared__ uint16_t T_len[1024];
  __shared__ int64_t red[6];
  __shared__ float y[3][TC][G];     // chunks i - 1, i, i + 1
  __shared__ double run[2][TC][G];  // sums of chunks i - 1, i
  struct Frame {
    int64_t row;      // first element of its output row
    double n, rcp;    // t + 1, 1 / (t + 1)
  };
  constexpr int NF = 8;             // chunks of frames that wave 5 keeps
  __shared__ Frame fr[NF][TC];
  __shared__ int ended[1024];       // frames of the sequences from this one on
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane & (G - 1), half = lane / G;
  int64_t r0 = 0;  // raw frames of the utterances before this one
  for (int i = threadIdx.x; i < a.B; i += LFR_THREADS) {
    const int U = a.U[i];
    const int T = (U - a.offset - a.stack) / a.skip + 1;
    T_len[i] = (uint16_t)(U - a.offset - a.stack >= 0 ? T : 0);
    if (i < b) r0 += U;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) r0 += __shfl_xor(r0, o, 64);
  if (lane == 0) red[wave] = r0;
  __syncthreads();  // (T_len too)
  r0 = ((red[0] + red[1]) + (red[2] + red[3])) + (red[4] + red[5]);
  const int Tb = T_len[b];
  if (Tb == 0) return;
  if (wave == 5) {  // ended[i] = T_len[i] + ... + T_len[B - 1] (below 2^26 frames)
    const int per = (a.B + 63) / 64;
    int own = 0;
    for (int i = 0; i < per; ++i) own += lane * per + i < a.B ? T_len[lane * per + i] : 0;
    int after = own;  // frames of this lane's sequences and the later lanes'
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_down(after, o, 64);
      if (lane + o < 64) after += v;
    }
    after -= own;
    for (int i = per - 1; i >= 0; --i)
      if (lane * per + i < a.B) ended[lane * per + i] = after += T_len[lane * per + i];
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
  }
  const int j = (blockIdx.x % groups) * G + g;
  const bool in = j < D;
  // stacked frame t's dimension j is one raw value: stacking is contiguous
  const float* __restrict__ src = a.raw + (r0 + a.offset) * a.raw_dim + (in ? j : 0);
  const int64_t fstep = (int64_t)a.skip * a.raw_dim;
  OutT* __restrict__ x = static_cast<OutT*>(a.x) + j;
  const double mean = in ? (double)a.mean[j] : 0.0, sd = in ? (double)a.std[j] : 1.0;
  const double sd_rcp = 1.0 / sd;
  // frames of a chunk of this lane (waves 1-4): fw, fw + 2, ...
  const int fw = (wave - 1) * 2 * FPL + half;
  float ahead[PD][FPL];  // chunk c waits in ahead[c % PD]
  // clamped loads: frames past the last re-read it and are never used
  auto load = [&](int c, float (&v)[FPL]) {
#pragma unroll
    for (int q = 0; q < FPL; ++q) v[q] = src[(int64_t)min(c * TC + fw + 2 * q, Tb - 1) * fstep];
  };
  auto put = [&](int slot, const float (&v)[FPL]) {
#pragma unroll
    for (int q = 0; q < FPL; ++q) y[slot][fw + 2 * q][g] = v[q];
  };
  const int nch = (Tb + TC - 1) / TC;
  // where frame t of the batch starts: the sequences longer than t (T_len is
  // sorted) have t frames before it, the others all of theirs
  auto places = [&](int t0) {
    const int t = t0 + lane;
    int lo = 0, hi = a.B;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (T_len[mid] > t) lo = mid + 1; else hi = mid;
    }
    const int64_t off = (int64_t)t * lo + (lo < a.B ? ended[lo] : 0);
    fr[(t / TC) % NF][t % TC] = Frame{(off + b) * D, (double)(t + 1), 1.0 / (double)(t + 1)};
  };
  if (wave == 5) {
    places(0);
  } else if (wave > 0) {
#pragma unroll
    for (int c = 0; c < PD; ++c) load(c, ahead[c]);
    put(0, ahead[0]);
    load(PD, ahead[0]);
  } else {
    __builtin_amdgcn_s_setprio(3);  // the walk is the chain that the others wait for
  }
  __syncthreads();
  double sum = 0.0;
  for (int i0 = 0; i0 <= nch; i0 += PD)
#pragma unroll
    for (int u = 0; u < PD; ++u) {
      const int i = i0 + u;  // (i % PD == u: the register sets are picked at compile time)
      if (i > nch) break;
      if (wave == 0) {
        if (i < nch) {
          // (all reads before the first write, which the compiler would keep
          // behind each other: an LDS latency a frame)
          float yv[TC];
#pragma unroll
          for (int q = 0; q < TC; ++q) yv[q] = y[i % 3][q][g];
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int q = 0; q < TC; ++q) {
            sum = sum + (double)yv[q];  // (frames past the last: never used)
            run[i & 1][q][g] = sum;     // (both halves, the same value)
          }
        }
      } else if (wave == 5) {
        if ((i & 1) == 0) places((i + 2) * TC);
      } else {
        put((i + 1) % 3, ahead[(u + 1) % PD]);  // (past the last chunk: never read)
        load(i + 1 + PD, ahead[(u + 1) % PD]);
        if (i > 0) {
          // (frames past the last are evaluated too and not stored: no branch
          // keeps the chains apart)
          const int s = (i - 1) & 1, sy = (i - 1) % 3, sf = (i - 1) % NF, left = Tb - (i - 1) * TC;
          double v[FPL];
          bool far = false;
#pragma unroll
          for (int q = 0; q < FPL; ++q) {
            const int f = fw + 2 * q;
            const double z = (double)y[sy][f][g] - quotient(run[s][f][g], fr[sf][f].n, fr[sf][f].rcp);
            v[q] = quotient(z - mean, sd, sd_rcp);
            far |= !in_range(v[q]);
          }
          // a first quotient that is infinite or NaN leaves the second so; one
          // that is zero is exact (a sum of fp32 values is zero or far from
          // underflow), and its sign shows only in a result of zero
          if (far) {
#pragma unroll
            for (int q = 0; q < FPL; ++q) {
              const int f = fw + 2 * q;
              if (!in_range(v[q])) {
                const double z = (double)y[sy][f][g] - run[s][f][g] / fr[sf][f].n;
                v[q] = (z - mean) / sd;
              }
            }
          }
#pragma unroll
          for (int q = 0; q < FPL; ++q)
            if (in && fw + 2 * q < left) x[fr[sf][fw + 2 * q].row] = from_f64<OutT>(v[q]);
        }
      }
      __syncthreads();
    }
}

__global__ __launch_bounds__(256) void delay_targets_kernel(DelayArgs a) {
  const int t = blockIdx.x;
  __shared__ int64_t red[4];
  // packed offsets of frames t and t - delay (off_t = sum of min(len_b, t))
  // and the sequences active at t
  const int ts = t >= a.delay ? t - a.delay : 0;
  int64_t o = 0, os = 0, c = 0;
  for (int b = threadIdx.x; b < a.B; b += blockDim.x) {
    const int len = a.len[b];
    o += len < t ? len : t;
    os += len < ts ? len : ts;
    c += len > t;
  }
  const int64_t s_off = block_sum(o, red);
  const int64_t s_src = block_sum(os, red);
  const int nb = (int)block_sum(c, red);
  const bool has = t >= a.delay;
  for (int e = threadIdx.x; e < nb * a.K; e += blockDim.x) {
    const int b = e / a.K, q = e % a.K;
    const int64_t dst = (s_off + b) * a.K + q;
    if (has) {
      const int64_t src = (s_src + b) * a.K + q;
      a.idx_out[dst] = a.idx[src];
      a.prob_out[dst] = a.prob[src];
    } else {
      a.idx_out[dst] = -1;
      a.prob_out[dst] = 0.f;
    }
  }
  for (int b = threadIdx.x; b < nb; b += blockDim.x) a.mask_out[s_off + b] = has ? 1 : 0;
}

int lfr_groups(const LfrArgs& a) { return (a.stack * a.raw_dim + LFR_G - 1) / LFR_G; }

// Whether the walking kernel is the faster one: estimated microseconds of both,
// within 11 % of the faster one's in 684 measured batches (1 to 1000
// utterances, 1 to 600 frames, 3 to 4096 dimensions, uniform and ragged).  The
// walk follows the longest utterance, in passes of 256 dimensions (and each
// ended one before a frame is an LDS read there), or the memory; the chunked
// kernel pays its start for every (utterance, 32 dimensions), 1024 workgroups at
// a time.  1000 utterances of 66 frames x 240: 42 us walking, 143 in chunks;
// 512 of 21 x 120: 17 and 27; 256 of 300 x 240: 113 and 67.
bool lfr_walks(const LfrArgs& a, int longest, double frames) {
  const int D = a.stack * a.raw_dim;
  const bool ragged = frames < (double)longest * a.B;
  const int passes = (D + 255) / 256;
  double walk = 2.0 + 0.01 * a.B + 0.3 * passes * longest + (ragged ? 0.04 * a.B : 0.0);
  if (a.B > 256 && longest > 64) walk += 0.08 * passes * (longest - 64);
  const double memory = 8.0 + (passes > 1 ? 4.5e-6 : 3e-6) * frames * D;
  const double chunks = 3.5 + (double)a.B * lfr_groups(a) / 1024 * (7.0 + 0.0075 * a.B + 0.072 * frames / a.B);
  return (walk > memory ? walk : memory) < chunks;
}

}  // namespace

hipError_t lfr_features(const LfrArgs& a, int longest, int64_t frames, bool bf16, hipStream_t s) {
  if (a.B == 0) return hipSuccess;
  if (lfr_walks(a, longest, (double)frames)) {
    if (bf16) hipLaunchKernelGGL(lfr_walk_kernel<bf16_t>, dim3(a.B), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(lfr_walk_kernel<float>, dim3(a.B), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  const dim3 grid(a.B * lfr_groups(a));
  if (bf16)
    hipLaunchKernelGGL(lfr_features_kernel<bf16_t>, grid, dim3(LFR_THREADS), 0, s, a);
  else
    hipLaunchKernelGGL(lfr_features_kernel<float>, grid, dim3(LFR_THREADS), 0, s, a);
  return hipGetLastError();
}

hipError_t delay_targets(const DelayArgs& a, hipStream_t s) {
  if (a.T == 0) return hipSuccess;
  hipLaunchKernelGGL(delay_targets_kernel, dim3(a.T), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace am
