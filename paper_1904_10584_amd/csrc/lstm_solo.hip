// LSTM layer kernels for narrow layers: one workgroup runs 16 sequences
// through every time step, forward or backward, with the whole recurrent
// matrix in its registers.
//
// The recurrence is a chain of dependent steps.  Split over workgroups (the
// XCD-local kernels), a step pays for a store's completion, a barrier through
// the L2 and a copy back, about 1.5 us whatever the width; kept in one
// workgroup, h_{t-1} (dA_{t+1} backward) goes from the cell to the next
// product through LDS behind one workgroup barrier.  That holds while W_h fits
// the registers of one compute unit beside the rest: up to H = 128 in bf16 and
// 96 in fp32 (144 in bf16 spills registers).  No workgroup waits for another, so any number of sequences runs
// in one launch and nothing has to be resident at once.
//
// The products are computed transposed, weights as the MFMA's row operand and
// sequences as its columns.  Forward: rows 4 (l / 16) + r of a 16-row tile are
// gate r of unit l / 16 (weights ordered unit-major, gate-minor), so lane l
// gets all four gates of one (unit, sequence) in its four accumulators, and
// the cell follows in registers with no exchange.  Backward: the lane gets
// four consecutive units of one sequence.
//
// Waves: the compute waves (eight forward, one per 16 units backward); one
// that copies the coming steps' operands (input projections; gates, cell
// states and incoming dh) to an LDS ring with direct loads, alone with its
// memory counter, so that its partial waits count exactly its own loads; and
// one or two that write out the previous step's results from LDS in whole
// 16-byte chunks (a block's rows are contiguous in every output).
//
// What bounds a step: the compute unit's own matrix and vector rate (64 cells
// in fp32: 2048 clocks of MFMA, then the cell's exponentials; letting one wave
// of a SIMD finish its products first changed nothing) and the LDS round trip.
// 16 sequences x 50 steps, us a layer, forward / backward: 64 cells in fp32
// 225 / 154 (device-scope kernels) -> 101 / 95, a 3 x 64 model in bf16, 6
// sequences of 19 frames, whole step 256 (XCD-local kernels) -> 205.
#include <type_traits>

#include "am_device.h"
#include "am_internal.h"

namespace am {
namespace {

constexpr int SEQ = 16;  // sequences per workgroup

// The schedule as the waves walk it: the lengths in LDS (a vector load of one
// would make the copying wave wait for its direct loads).
struct Walk {
  const uint16_t* lens;
  int B, varlen;
  __device__ __forceinline__ int down(int nb, int t) const {  // sequences longer than t, from t - 1's
    if (!varlen) return B;
    while (nb > 0 && (int)lens[nb - 1] <= t) --nb;
    return nb;
  }
  __device__ __forceinline__ int up(int nb, int t) const {    // from t + 1's
    if (!varlen) return B;
    while (nb < B && (int)lens[nb] > t) ++nb;
    return nb;
  }
};
constexpr int LENS_BYTES = 2048;  // of 1024 sequences
__device__ __forceinline__ Walk make_walk(const PersistSchedule& ps, unsigned char* at, int threads) {
  uint16_t* l = reinterpret_cast<uint16_t*>(at);
  if (ps.varlen)
    for (int b = threadIdx.x; b < ps.B; b += threads) l[b] = ps.lens[b];
  return Walk{l, ps.B, ps.varlen};  // (usable behind the caller's next barrier)
}

// SEQ rows of CH 16-byte chunks copied to LDS by one wave, end to end, chunk c
// of row r in slot c ^ (r & MASK) of its row: lanes that read one column of
// sixteen rows then spread over the banks.  Rows past the active ones re-read
// the last active one; the copy is rounded up to whole instructions.
template <int CH, int MASK> struct RowCopy {
  static_assert(CH % (MASK + 1) == 0, "the swizzle stays in the row");
  static constexpr int NI = (SEQ * CH + 63) / 64;  // direct loads
  static constexpr int BYTES = NI * 1024;
  static __device__ __forceinline__ void issue(const void* src, int active, const void* lds, int lane) {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds_address(lds));
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int e = i * 64 + lane, row = e / CH, c = e % CH;
      dma16(static_cast<const char*>(src) + ((int64_t)min(row, active - 1) * CH + (c ^ (row & MASK))) * 16,
            base + i * 1024);
    }
  }
  // byte offset of byte `b` of row r
  static __device__ __forceinline__ int at(int r, int b) {
    return (r * CH + ((b >> 4) ^ (r & MASK))) * 16 + (b & 15);
  }
};

// `rows` rows of CH chunks from LDS (row stride LS bytes) to contiguous
// memory, by `waves` waves of which this is number w.
template <int CH, int LS>
__device__ __forceinline__ void write_rows(void* dst, const unsigned char* lds, int rows, int w,
                                           int waves, int lane) {
  for (int e = w * 64 + lane; e < rows * CH; e += waves * 64) {
    const int row = e / CH, c = e % CH;
    reinterpret_cast<uint4*>(dst)[e] = *reinterpret_cast<const uint4*>(lds + row * LS + c * 16);
  }
}

template <typename T> __device__ __forceinline__ T lds_get(const unsigned char* p) {
  return *reinterpret_cast<const T*>(p);
}

// ----------------------------------------------------------------- forward --

// Sizes of the forward kernel for H = 16 H16.
template <typename T, int H16> struct Fwd {
  static constexpr int H = 16 * H16, E = sizeof(T);
  static constexpr int KS = (H + 31) / 32;       // k-steps
  static constexpr int NT = H / 4;               // tiles of 4 units x 4 gates
  static constexpr int TPW = (NT + 7) / 8;       // per wave
  static constexpr int HS = KS * 32 * E + 16;    // LDS row strides: h (zero-padded to whole k-steps),
  static constexpr int CS = H * 4 + 16;          //   staged c
  static constexpr int GS = 4 * H * E + 16;      //   and gates (16 bytes spread the rows over the banks)
  using PCopy = RowCopy<4 * H * E / 16, 7>;
  static constexpr int H_AT = 0, C_AT = H_AT + 3 * SEQ * HS, G_AT = C_AT + 2 * SEQ * CS;
  static constexpr int P_AT = (G_AT + 2 * SEQ * GS + 15) / 16 * 16;
  // ring slots: as many as the LDS and the memory counter (63) allow, up to 4
  static constexpr int FIT = (160 * 1024 - LENS_BYTES - P_AT) / PCopy::BYTES;
  static constexpr int CNT = 62 / PCopy::NI + 2;
  static constexpr int D = FIT < CNT ? (FIT < 4 ? FIT : 4) : (CNT < 4 ? CNT : 4);
  static constexpr int L_AT = P_AT + D * PCopy::BYTES, LDS = L_AT + LENS_BYTES;
  static constexpr int STORERS = 2, THREADS = (8 + 1 + STORERS) * 64;
  static_assert(D >= 2, "ring");
};

template <typename T, int H16>
__global__ __launch_bounds__((Fwd<T, H16>::THREADS), 1) void lstm_fwd_solo(PersistFwd a, PersistSchedule ps) {
  using F = Fwd<T, H16>;
  constexpr int H = F::H, E = F::E, KS = F::KS, TPW = F::TPW, D = F::D;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b0 = blockIdx.x * SEQ;
  const int steps = ps.varlen ? ps.lens[b0] : ps.T;  // of the block's longest sequence
  if (steps == 0) return;
  const Walk walk = make_walk(ps, lds + F::L_AT, F::THREADS);
  const T* __restrict__ h0 = static_cast<const T*>(a.h0);
  auto hslot = [&](int t) { return lds + F::H_AT + (t % 3) * SEQ * F::HS; };  // h_{t-1} of step t

  // zero h (its k padding stays zero), then the initial state
  for (int e = threadIdx.x; e < 3 * SEQ * F::HS / 16; e += F::THREADS)
    reinterpret_cast<uint4*>(lds + F::H_AT)[e] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  if (h0)
    for (int e = threadIdx.x; e < SEQ * H; e += F::THREADS) {
      const int b = min(b0 + e / H, ps.B - 1);
      *reinterpret_cast<T*>(hslot(0) + (e / H) * F::HS + (e % H) * E) = h0[(int64_t)b * H + e % H];
    }
  __syncthreads();

  if (wave < 8) {
    const int seq = lane & 15, kq = lane >> 4;
    const T* __restrict__ Wh = static_cast<const T*>(a.Wh);
    // tile n = wave + 8 ts: its row m is gate m % 4 of unit 4 n + m / 4
    Frag<T> wf[TPW][KS];
    float c_reg[TPW];
#pragma unroll
    for (int ts = 0; ts < TPW; ++ts) {
      const int n = wave + 8 * ts;
      const int row = (lane & 3) * H + 4 * (n < F::NT ? n : 0) + (seq >> 2);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int k = s * 32 + kq * 8;
        wf[ts][s] = k < H ? frag_load<T>(Wh + (int64_t)row * H + k) : frag_zero<T>();
      }
      c_reg[ts] = a.c0[(int64_t)min(b0 + seq, ps.B - 1) * H + 4 * (n < F::NT ? n : 0) + kq];
    }
    int nb = ps.B;
    for (int t = 0; t < steps; ++t) {
      lds_barrier();  // the step's projections and h_{t-1} are in LDS
      nb = walk.down(nb, t);
      const bool ok = b0 + seq < nb;
      const unsigned char* hin = hslot(t) + seq * F::HS + kq * 8 * E;
      f32x4_t acc[TPW];
#pragma unroll
      for (int ts = 0; ts < TPW; ++ts) acc[ts] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const Frag<T> hf = frag_load<T>(reinterpret_cast<const T*>(hin + s * 32 * E));
#pragma unroll
        for (int ts = 0; ts < TPW; ++ts) mma_16x16x32(acc[ts], wf[ts][s], hf);
      }
      const unsigned char* pin = lds + F::P_AT + (t % D) * F::PCopy::BYTES;
      unsigned char* hout = hslot(t + 1) + seq * F::HS;
      unsigned char* cst = lds + F::C_AT + ((t & 1) * SEQ + seq) * F::CS;
      unsigned char* gst = lds + F::G_AT + ((t & 1) * SEQ + seq) * F::GS;
#pragma unroll
      for (int ts = 0; ts < TPW; ++ts) {
        const int n = wave + 8 * ts, unit = 4 * n + kq;
        if (n >= F::NT) break;  // (wave-uniform)
        float p[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) p[q] = to_f32<T>(lds_get<T>(pin + F::PCopy::at(seq, (q * H + unit) * E)));
        const float gi = sigm(acc[ts][0] + p[0]);
        const float gf = sigm(acc[ts][1] + p[1]);
        const float gg = tanh_f(acc[ts][2] + p[2]);
        const float go = sigm(acc[ts][3] + p[3]);
        const float c = gf * c_reg[ts] + gi * gg;
        const T h = from_f32<T>(go * tanh_f(c));
        if (ok) {  // (an ended sequence's state is not used again)
          c_reg[ts] = c;
          *reinterpret_cast<T*>(hout + unit * E) = h;
          *reinterpret_cast<float*>(cst + unit * 4) = c;
          store_gates(reinterpret_cast<T*>(gst), unit, gi, gf, gg, go);
        }
      }
    }
    lds_barrier();
  } else if (wave == 8) {
    // the projections of step t + D - 1 are requested during step t
    const char* P = static_cast<const char*>(a.P);
    int nb = ps.B, off = 0, next = 0;
    auto issue = [&]() {
      if (next >= steps) return;
      nb = walk.down(nb, next);
      F::PCopy::issue(P + (int64_t)(off + b0) * 4 * H * E, min(SEQ, nb - b0),
                      lds + F::P_AT + (next % D) * F::PCopy::BYTES, lane);
      off += nb;
      ++next;
    };
    for (int d = 0; d < D - 1; ++d) issue();
    for (int t = 0; t < steps; ++t) {
      // step t's have landed once at most the D - 2 later steps' are in flight
      if (next - t == D - 1) wait_vm_asm<(D - 2) * F::PCopy::NI>();
      else wait_vm_asm<0>();
      lds_barrier();
      issue();
    }
    lds_barrier();
  } else {
    // the results of step t - 1 leave during step t
    const int w = wave - 9;
    int nb = ps.B, off = 0, nb_done = 0, off_done = 0;
    for (int t = 0; t <= steps; ++t) {
      lds_barrier();
      if (t > 0) {
        const int rows = min(SEQ, nb_done - b0);
        const int64_t r0 = off_done + b0;
        write_rows<H * E / 16, F::HS>(static_cast<T*>(a.H) + r0 * H, hslot(t), rows, w, F::STORERS, lane);
        write_rows<H * E / 16, F::HS>(static_cast<T*>(a.Hs) + r0 * H, hslot(t - 1), rows, w, F::STORERS, lane);
        write_rows<H / 4, F::CS>(a.C + r0 * H, lds + F::C_AT + ((t - 1) & 1) * SEQ * F::CS, rows, w,
                                 F::STORERS, lane);
        write_rows<4 * H * E / 16, F::GS>(static_cast<T*>(a.G) + r0 * 4 * H,
                                          lds + F::G_AT + ((t - 1) & 1) * SEQ * F::GS, rows, w,
                                          F::STORERS, lane);
      }
      if (t < steps) {
        nb = walk.down(nb, t);
        nb_done = nb;
        off_done = off;
        off += nb;
      }
    }
  }
}

// ---------------------------------------------------------------- backward --

template <typename T, int H16> struct Bwd {
  static constexpr int H = 16 * H16, E = sizeof(T);
  static constexpr int KS = 4 * H / 32;         // k-steps of the product over 4H
  static constexpr int AS = 4 * H * E + 16;     // LDS row stride of dA
  using GCopy = RowCopy<4 * H * E / 16, 7>;
  using CCopy = RowCopy<H * 4 / 16, 3>;
  using DCopy = RowCopy<H * E / 16, E == 2 ? 1 : 3>;
  static constexpr int SLOT = GCopy::BYTES + CCopy::BYTES + DCopy::BYTES;
  static constexpr int NI = GCopy::NI + CCopy::NI + DCopy::NI;
  static constexpr int A_AT = 0, S_AT = (2 * SEQ * AS + 15) / 16 * 16;
  static constexpr int FIT = (160 * 1024 - LENS_BYTES - S_AT) / SLOT;
  static constexpr int CNT = 62 / NI + 2;
  static constexpr int D = FIT < CNT ? (FIT < 4 ? FIT : 4) : (CNT < 4 ? CNT : 4);
  static constexpr int L_AT = S_AT + D * SLOT, LDS = L_AT + LENS_BYTES;
  static constexpr int THREADS = (H16 + 2) * 64;
  static_assert(D >= 2, "ring");
};

template <typename T, int H16>
__global__ __launch_bounds__((Bwd<T, H16>::THREADS), 1) void lstm_bwd_solo(PersistBwd a, PersistSchedule ps) {
  using F = Bwd<T, H16>;
  constexpr int H = F::H, E = F::E, KS = F::KS, D = F::D;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b0 = blockIdx.x * SEQ;
  const int steps = ps.varlen ? ps.lens[b0] : ps.T;
  if (steps == 0) return;
  const Walk walk = make_walk(ps, lds + F::L_AT, F::THREADS);
  for (int e = threadIdx.x; e < 2 * SEQ * F::AS / 16; e += F::THREADS)
    reinterpret_cast<uint4*>(lds + F::A_AT)[e] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  // step i handles t = steps - 1 - i; the block's last step and its row offset
  // (offsets count every sequence's frames: sum of min(len, t_last))
  const int t_last = steps - 1;
  const int nb_last = walk.up(b0 + 1, t_last);
  int off_last = 0;
  if (ps.varlen) {
    for (int b = lane; b < ps.B; b += 64) off_last += min((int)walk.lens[b], t_last);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) off_last += __shfl_xor(off_last, o, 64);
    off_last = __builtin_amdgcn_readfirstlane(off_last);
  } else {
    off_last = t_last * ps.B;
  }
  auto aslot = [&](int i) { return lds + F::A_AT + (i & 1) * SEQ * F::AS; };  // dA of step i

  if (wave < H16) {
    const int seq = lane & 15, kq = lane >> 4, u0 = 16 * wave + 4 * kq;  // units u0 .. u0 + 3
    const T* __restrict__ Wh = static_cast<const T*>(a.Wh);
    // row m of this wave's tile is unit 16 wave + m: W_h's column, 8 gate rows at a time
    Frag<T> wf[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      T v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = Wh[(int64_t)(s * 32 + kq * 8 + e) * H + 16 * wave + seq];
      memcpy(&wf[s], v, sizeof wf[s]);
    }
    float c_cur[4], dc[4];
    {
      const float4 c = *reinterpret_cast<const float4*>(
          a.C + (int64_t)(off_last + min(b0 + seq, nb_last - 1)) * H + u0);
      c_cur[0] = c.x; c_cur[1] = c.y; c_cur[2] = c.z; c_cur[3] = c.w;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) dc[r] = 0.f;
    int nb = nb_last, nb_next = 0;
    for (int i = 0; i < steps; ++i) {
      lds_barrier();  // the step's operands and dA of the step before are in LDS
      if (i > 0) {
        nb_next = nb;
        nb = walk.up(nb, t_last - i);
      }
      f32x4_t acc[2];
      acc[0] = acc[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if (i > 0) {
        const unsigned char* ain = aslot(i - 1) + seq * F::AS + kq * 8 * E;
#pragma unroll
        for (int s = 0; s < KS; ++s)
          mma_16x16x32(acc[s & 1], wf[s], frag_load<T>(reinterpret_cast<const T*>(ain + s * 32 * E)));
      }
      const unsigned char* gin = lds + F::S_AT + (i % D) * F::SLOT;
      const unsigned char* cin = gin + F::GCopy::BYTES;
      const unsigned char* din = cin + F::CCopy::BYTES;
      const bool ok = b0 + seq < nb, cont = b0 + seq < nb_next;
      float g[4][4], dh[4];  // [unit][gate]
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        T v[4];
        load_gates(reinterpret_cast<const T*>(gin + F::GCopy::at(seq, (u0 + r) * 4 * E)), 0, v);
#pragma unroll
        for (int q = 0; q < 4; ++q) g[r][q] = to_f32<T>(v[q]);
        dh[r] = to_f32<T>(lds_get<T>(din + F::DCopy::at(seq, (u0 + r) * E)));
      }
      const float4 cp4 = lds_get<float4>(cin + F::CCopy::at(seq, u0 * 4));
      const float cp[4] = {cp4.x, cp4.y, cp4.z, cp4.w};
      T out[4][4];  // [gate][unit]
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float vi = g[r][0], vf = g[r][1], vg = g[r][2], vo = g[r][3];
        const float dhh = dh[r] + (cont ? acc[0][r] + acc[1][r] : 0.f);
        const float tc = tanh_f(c_cur[r]);
        const float d_o = dhh * tc;
        const float dcell = dhh * vo * (1.f - tc * tc) + (cont ? dc[r] : 0.f);
        const float d_i = dcell * vg, d_g = dcell * vi, d_f = dcell * cp[r];
        dc[r] = dcell * vf;
        out[0][r] = from_f32<T>(d_i * vi * (1.f - vi));
        out[1][r] = from_f32<T>(d_f * vf * (1.f - vf));
        out[2][r] = from_f32<T>(d_g * (1.f - vg * vg));
        out[3][r] = from_f32<T>(d_o * vo * (1.f - vo));
        c_cur[r] = cp[r];
      }
      if (ok) {
        unsigned char* aout = aslot(i) + seq * F::AS;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (E == 2) {
            *reinterpret_cast<uint2*>(aout + (q * H + u0) * E) =
                make_uint2((uint32_t)out[q][0] | ((uint32_t)out[q][1] << 16),
                           (uint32_t)out[q][2] | ((uint32_t)out[q][3] << 16));
          } else {
            *reinterpret_cast<float4*>(aout + (q * H + u0) * E) =
                make_float4(out[q][0], out[q][1], out[q][2], out[q][3]);
          }
        }
      }
    }
    lds_barrier();
  } else if (wave == H16) {
    // gates, incoming dh and c_{t-1} of step i + D - 1, requested during step
    // i.  c_{t-1} is copied for every row active at t - 1: it is the next
    // step's c_t too, also for the sequences that only start there
    int nb = nb_last, off = off_last, next = 0;
    auto issue = [&]() {
      if (next >= steps) return;
      const int t = t_last - next;
      const int nb_prev = t > 0 ? walk.up(nb, t - 1) : nb;
      const int off_prev = off - nb_prev;
      unsigned char* slot = lds + F::S_AT + (next % D) * F::SLOT;
      const int rows = min(SEQ, nb - b0);
      F::GCopy::issue(static_cast<const T*>(a.G) + (int64_t)(off + b0) * 4 * H, rows, slot, lane);
      F::CCopy::issue(t > 0 ? a.C + (int64_t)(off_prev + b0) * H : a.c0 + (int64_t)b0 * H,
                      min(SEQ, nb_prev - b0), slot + F::GCopy::BYTES, lane);
      F::DCopy::issue(static_cast<const T*>(a.dHa) + (int64_t)(off + b0) * H, rows,
                      slot + F::GCopy::BYTES + F::CCopy::BYTES, lane);
      nb = nb_prev;
      off = off_prev;
      ++next;
    };
    for (int d = 0; d < D - 1; ++d) issue();
    for (int i = 0; i < steps; ++i) {
      if (next - i == D - 1) wait_vm_asm<(D - 2) * F::NI>();
      else wait_vm_asm<0>();
      lds_barrier();
      issue();
    }
    lds_barrier();
  } else {
    int nb = nb_last, off = off_last;  // of step i - 1
    for (int i = 0; i <= steps; ++i) {
      lds_barrier();
      if (i == 0) continue;
      write_rows<4 * H * E / 16, F::AS>(static_cast<T*>(a.dA) + (int64_t)(off + b0) * 4 * H, aslot(i - 1),
                                        min(SEQ, nb - b0), 0, 1, lane);
      if (i < steps) {
        nb = walk.up(nb, t_last - i);
        off -= nb;
      }
    }
  }
}

// ------------------------------------------------------------------ launch --

template <typename K, typename A>
hipError_t go(K kernel, int B, int threads, int lds, A& a, PersistSchedule& ps, hipStream_t s) {
  const void* fn = reinterpret_cast<const void*>(kernel);
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3((B + SEQ - 1) / SEQ), dim3(threads), lds, s, a, ps);
  return hipGetLastError();
}

template <typename T, int H16> hipError_t fwd(PersistFwd& a, PersistSchedule& ps, hipStream_t s) {
  using F = Fwd<T, H16>;
  return go(lstm_fwd_solo<T, H16>, ps.B, F::THREADS, F::LDS, a, ps, s);
}
template <typename T, int H16> hipError_t bwd(PersistBwd& a, PersistSchedule& ps, hipStream_t s) {
  using F = Bwd<T, H16>;
  return go(lstm_bwd_solo<T, H16>, ps.B, F::THREADS, F::LDS, a, ps, s);
}

}  // namespace

bool lstm_solo_covers(int hidden, bool bf16) {
  return hidden % 16 == 0 && hidden <= (bf16 ? 128 : 96);
}

#define AM_SOLO(F, A)                                                         \
  switch (A.hidden / 16) {                                                    \
    case 1: return bf16 ? F<bf16_t, 1>(A, ps, s) : F<float, 1>(A, ps, s);     \
    case 2: return bf16 ? F<bf16_t, 2>(A, ps, s) : F<float, 2>(A, ps, s);     \
    case 3: return bf16 ? F<bf16_t, 3>(A, ps, s) : F<float, 3>(A, ps, s);     \
    case 4: return bf16 ? F<bf16_t, 4>(A, ps, s) : F<float, 4>(A, ps, s);     \
    case 5: return bf16 ? F<bf16_t, 5>(A, ps, s) : F<float, 5>(A, ps, s);     \
    case 6: return bf16 ? F<bf16_t, 6>(A, ps, s) : F<float, 6>(A, ps, s);     \
    case 7: return bf16 ? F<bf16_t, 7>(A, ps, s) : hipErrorInvalidValue;      \
    case 8: return bf16 ? F<bf16_t, 8>(A, ps, s) : hipErrorInvalidValue;      \
    default: return hipErrorInvalidValue;                                     \
  }

hipError_t lstm_fwd_solo_launch(PersistFwd a, PersistSchedule ps, bool bf16, hipStream_t s) { AM_SOLO(fwd, a) }
hipError_t lstm_bwd_solo_launch(PersistBwd a, PersistSchedule ps, bool bf16, hipStream_t s) { AM_SOLO(bwd, a) }

}  // namespace am
