// Forward pass of all layers in one launch, the layers one behind the other in
// time (a wavefront), for batches of few sequences.
//
// A layer's recurrence is a chain of dependent steps that a block of 16
// sequences runs on the workgroups of one XCD (lstm_xcd.hip).  With few blocks
// most XCDs idle while the layers take their turns: L T steps one after
// another.  Here each (layer, block) has an XCD's workgroups, or half of them,
// to itself, and layer l + 1 follows layer l a few steps behind: T + 3 (L - 1)
// steps.
//
// A layer makes its successor's input projections itself: h_{t-1} is in LDS
// for the recurrent product of step t, so behind the step's signal, in the
// time that the other members' signals take, it is multiplied by the
// successor's W_x as well (the member's own unit slice of it, resident beside
// W_h in registers, the last of its k-steps in LDS where the registers are
// short).  The result is rounded to bf16 with the bias, as the batched
// projection's, and waits in the rows of the successor's gates, which the
// successor overwrites with the gates themselves: a member's cells take 8
// bytes each in both, at the same place, and no other member reads them.
//
// Between layers the data crosses XCDs.  The projections are stored
// device-scope (written through the producer's L2) and announced, one step
// later, by a count in the member's word of a second flag line, device-scope
// too.  The consumer's XCD first touches a row's lines after every member has
// announced it (and no other layer's XCD reads them), so its ordinary loads
// fetch them fresh.  The wave that watches the lower layer's line asks a
// step ahead and looks at the answer at the next step's barrier, so the round
// trip to memory is not on the step's path unless the lower layer really is
// late.  Every wait is bounded, and a layer waits only for itself and the
// layers below.
//
// Whole forward, layer by layer -> so: 5 x 768, 12 sequences of 32 frames 460 ->
// 200 us; 3 x 512, 48 sequences of 40 frames 260 -> 178.
#include <cstdlib>

#include "xcd_sync.h"

namespace am {
namespace {

constexpr int RB = 16;  // sequences per block

// A device-scope store: write-through, so that another XCD's loads see it once
// it has completed.
__device__ __forceinline__ void store8_agent(void* dst, uint2 v) {
  __hip_atomic_store(static_cast<unsigned long long*>(dst),
                     (unsigned long long)v.x | ((unsigned long long)v.y << 32), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// H = 32 KS; the recurrent product as in lstm_fwd_xcd (TPW column tiles of 4
// units x 4 gates per wave and k-half).  The successor's projections are
// computed transposed, one tile a wave over the whole k-range (with TPW = 1 by
// waves 4-7, which have no cells): W_x the row operand in the same unit-major
// order, so a lane has the four gates of one (unit, sequence) in its four
// accumulators and stores them as 8 bytes, with no exchange between waves.  The
// last XL k-steps of these weights sit in LDS.  (Split over k-halves like the
// recurrent product, summed and staged through LDS, a step took 3.85 us at 5 x
// 768 and 2.6 at 5 x 512 instead of 3.3 and 2.2; the recurrence alone
// takes 2.0 and 1.6.)
template <int KS, int TPW, int XL>
__global__ __launch_bounds__(512, 1) void lstm_fwd_pipe(PipeFwd a, PersistSchedule ps, XcdSync y) {
  constexpr int KH = KS / 2, FIN = (TPW + 1) / 2, XR = KS - XL;
  constexpr int HS_BYTES = RB * KS * 64, RED_BYTES = 8 * TPW * 64 * 16;
  extern __shared__ __align__(16) unsigned char lds[];
  bf16_t* hl = reinterpret_cast<bf16_t*>(lds);
  f32x4_t* red = reinterpret_cast<f32x4_t*>(lds + HS_BYTES);             // [8][TPW][64]
  Frag<bf16_t>* wxl = reinterpret_cast<Frag<bf16_t>*>(lds + HS_BYTES + RED_BYTES);  // [8][XL][64]
  unsigned char* stC = lds + HS_BYTES + RED_BYTES + 8 * XL * 1024;
  __shared__ int bad_sh;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = wave & 3, kh = wave >> 2;
  const int H = KS * 32, G4 = 4 * H, U = y.units;
  const int ntiles = U / 4, members = H / U;
  const int slot = xcd_block(members), us = (blockIdx.x / NX) % members;
  if (slot >= a.layers * a.blocks) return;
  const int layer = slot / a.blocks, blk = slot % a.blocks;
  const PipeLayer& me = a.l[layer];
  const bool has_next = layer + 1 < a.layers;
  const int b0 = blk * RB, j0 = us * U;
  const int CSB = U * 4 + 16, HSB = U * 2 + 16, GSB = U * 8 + 16;  // staged row strides
  unsigned char* stH = stC + RB * CSB;
  unsigned char* stG = stH + RB * HSB;
  const bf16_t* __restrict__ Wh = static_cast<const bf16_t*>(me.Wh);
  const bf16_t* __restrict__ Wx = static_cast<const bf16_t*>(me.WxN);
  const bf16_t* __restrict__ h0 = static_cast<const bf16_t*>(me.h0);
  bf16_t* __restrict__ Hb = static_cast<bf16_t*>(me.H);
  bf16_t* __restrict__ Hs = static_cast<bf16_t*>(me.Hs);
  bf16_t* Gb = static_cast<bf16_t*>(me.G);
  bf16_t* Pn = has_next ? static_cast<bf16_t*>(a.l[layer + 1].G) : nullptr;
  const bf16_t* P = static_cast<const bf16_t*>(a.P);
  const unsigned* below = layer > 0 ? a.pflags + (slot - a.blocks) * 32 : nullptr;
  unsigned* mine = a.pflags + slot * 32 + us;

  // resident weights: column c of tile n is unit j0 + 4n + c/4, gate c%4
  const int c16 = lane & 15, kq = lane >> 4;
  auto wrow = [&](int n) { return (int64_t)((c16 & 3) * H + j0 + 4 * n + (c16 >> 2)) * H + kq * 8; };
  Frag<bf16_t> wf[TPW][KH], wx[XR];
#pragma unroll
  for (int ts = 0; ts < TPW; ++ts) {
    const int t = g + 4 * ts;
    const bf16_t* w = Wh + wrow(t < ntiles ? t : 0);
#pragma unroll
    for (int s = 0; s < KH; ++s) wf[ts][s] = frag_load<bf16_t>(w + (kh * KH + s) * 32);
  }
  const int xt = TPW == 1 ? wave - 4 : wave;  // this wave's tile of the successor's projections
  const bool projects = has_next && xt >= 0 && xt < ntiles;
  const int xu = j0 + 4 * (projects ? xt : 0) + kq;  // the lane's unit in it
  float xbias[4] = {0.f, 0.f, 0.f, 0.f};
  if (projects) {
    const bf16_t* w = Wx + wrow(xt);
#pragma unroll
    for (int s = 0; s < XR; ++s) wx[s] = frag_load<bf16_t>(w + s * 32);
#pragma unroll
    for (int s = 0; s < XL; ++s) wxl[(wave * XL + s) * 64 + lane] = frag_load<bf16_t>(w + (XR + s) * 32);
#pragma unroll
    for (int q = 0; q < 4; ++q) xbias[q] = bf16_to_f32(static_cast<const bf16_t*>(me.bN)[q * H + xu]);
  }
  const bool local = check_local(y, slot, us, members, &bad_sh);

  const int qrow = 4 * (lane >> 4) + (lane & 3);
  auto slot_ts = [&](int o) { return kh == 0 ? o : FIN + o; };
  auto slot_ok = [&](int o) { return slot_ts(o) < TPW && g + 4 * slot_ts(o) < ntiles; };
  auto unit = [&](int o) {
    const int t = g + 4 * slot_ts(o);
    return j0 + 4 * (t < ntiles ? t : 0) + ((lane & 15) >> 2);
  };
  float c_reg[FIN];
  bf16_t h_reg[FIN];
#pragma unroll
  for (int o = 0; o < FIN; ++o) {
    const int b = min(b0 + qrow, ps.B - 1), j = unit(o);
    c_reg[o] = me.c0[(int64_t)b * H + j];
    h_reg[o] = h0 ? h0[(int64_t)b * H + j] : (bf16_t)0;
  }

  // Lower layer: steps of P announced by every member, as far as this wave
  // knows, and the words asked for last.
  unsigned p_seen = 0, p_ask = 0;
  auto ask_below = [&]() {
    if (below && wave == 7)
      p_ask = lane < members ? __hip_atomic_load(below + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~0u;
  };
  auto wave_min = [](unsigned v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, (unsigned)__shfl_xor((int)v, o, 64));
    return v;
  };
  const int steps = ps.varlen ? (int)ps.lens[b0] : ps.T;  // of the block's longest sequence
  // P of steps below `want` is there (wave 7; its answer is often in already)
  auto wait_below = [&](unsigned want) {
    if (!below || wave != 7 || p_seen >= want) return;
    p_seen = wave_min(p_ask);
    for (unsigned spins = 0; p_seen < want; ++spins) {
      if (spins > SPIN_LIMIT) {
        if (lane == 0) __hip_atomic_store(y.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        p_seen = want;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
      ask_below();
      p_seen = wave_min(p_ask);
    }
    asm volatile("" ::: "memory");  // P is read only behind this
  };

  f32x4_t acc[TPW];
  // this wave's half of the product of the h rows in LDS with its resident
  // columns
  auto product = [&]() {
    constexpr int AB = KH > 4 ? 4 : KH;
    const int r = lane & 15;
#pragma unroll
    for (int s0 = 0; s0 < KH; s0 += AB) {
      Frag<bf16_t> af[AB];
#pragma unroll
      for (int s = 0; s < AB; ++s) {
        if (s0 + s >= KH) continue;
        const int c = (kh * KH + s0 + s) * 4 + (lane >> 4);
        af[s] = *reinterpret_cast<const Frag<bf16_t>*>(hl + ((c >> 3) * RB + r) * 64 + (((c & 7) ^ (r & 7)) << 3));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < AB; ++s) {
        if (s0 + s >= KH) continue;
#pragma unroll
        for (int ts = 0; ts < TPW; ++ts) mma_16x16x32(acc[ts], af[s], wf[ts][s0 + s]);
      }
    }
  };
  auto publish = [&]() {
#pragma unroll
    for (int ts = 0; ts < TPW; ++ts) red[(wave * TPW + ts) * 64 + lane] = acc[ts];
  };
  // the four gates of this lane's cell in own slot o, from both k-halves
  auto gates_of = [&](int o, float (&v)[4]) {
    const int ts = slot_ts(o) % TPW;
    const float* p0 = reinterpret_cast<const float*>(red + (g * TPW + ts) * 64 + (lane & ~3));
    const float* p1 = reinterpret_cast<const float*>(red + ((g + 4) * TPW + ts) * 64 + (lane & ~3));
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = p0[4 * q + (lane & 3)] + p1[4 * q + (lane & 3)];
  };
  // the block's rows of h (of the nbh sequences of a step, from row `at` on)
  // to LDS, by waves 1-7
  auto copy_h = [&](const bf16_t* src, int nbh) {
    constexpr int NQ = (KS / 2) * 2;
    if (wave > 0) {
      for (int q = wave - 1; q < NQ; q += 7) {
        const int line = q >> 1, rg = q & 1;
        const int r = rg * 8 + (lane >> 3);
        const int chunk = line * 8 + ((lane & 7) ^ (r & 7));
        dma16(src + (int64_t)min(b0 + r, nbh - 1) * H + chunk * 8,
              __builtin_amdgcn_readfirstlane(lds_address(hl + (line * RB + rg * 8) * 64)));
      }
      wait_vm<0>();
    }
    __syncthreads();
  };
  // the successor's projections of the step whose h rows are in LDS: its rows
  // start at `at` (nbh sequences)
  auto project = [&](int at, int nbh) {
    if (!projects) return;
    // one accumulator over the k-range in order, as the batched product's: the
    // same bits as layer after layer (two accumulators in turn were no faster:
    // 5 x 768, 12 sequences of 32 frames 201 us, one 200)
    f32x4_t p{0.f, 0.f, 0.f, 0.f};
    constexpr int AB = 4;
#pragma unroll
    for (int s0 = 0; s0 < KS; s0 += AB) {
      Frag<bf16_t> hf[AB], wl[AB];
#pragma unroll
      for (int s = 0; s < AB; ++s) {
        if (s0 + s >= KS) continue;
        const int c = (s0 + s) * 4 + kq;
        hf[s] = *reinterpret_cast<const Frag<bf16_t>*>(hl + ((c >> 3) * RB + c16) * 64 + (((c & 7) ^ (c16 & 7)) << 3));
        if (s0 + s >= XR) wl[s] = wxl[(wave * XL + (s0 + s - XR)) * 64 + lane];
      }
#pragma unroll
      for (int s = 0; s < AB; ++s) {
        if (s0 + s >= KS) continue;
        mma_16x16x32(p, s0 + s < XR ? wx[s0 + s < XR ? s0 + s : 0] : wl[s], hf[s]);
      }
    }
    if (b0 + c16 < nbh)
      store8_agent(Pn + (int64_t)(at + b0 + c16) * G4 + 4 * xu,
                   pack_gates(p[0] + xbias[0], p[1] + xbias[1], p[2] + xbias[2], p[3] + xbias[3]));
  };

  wait_vm<0>();
  if (steps > 0) {
    ask_below();
    wait_below(1);
  }
  __syncthreads();
  int nb = ps.B, off = 0, off_prev = 0, nb_prev = 0;
  for (int t = 0; t < steps; ++t) {
    nb = active_down(ps, nb, t);
    // input projections of this lane's cells (announced by the barrier
    // before); the polling waves issue theirs after their polls
    bf16_t pin[FIN][4];
    auto load_pin = [&]() {
      const int64_t row = (int64_t)(off + min(b0 + qrow, nb - 1)) * G4;
      if (layer == 0) {  // the batched projection: gate after gate
#pragma unroll
        for (int o = 0; o < FIN; ++o)
#pragma unroll
          for (int q = 0; q < 4; ++q) pin[o][q] = P[row + q * H + unit(o)];
      } else {
#pragma unroll
        for (int o = 0; o < FIN; ++o) load_gates(Gb + row, unit(o), pin[o]);
      }
    };
    if (wave != 0 && wave != 7) load_pin();
    const bf16_t* hsrc = h0;
    int nbh = ps.B;
    // the next step's projections are there before this step's barrier
    wait_below(min(t + 2, steps));
    if (t > 0) {
      xwait(y, local, slot, members, (unsigned)t);
      hsrc = Hb + (int64_t)off_prev * H;
      nbh = nb_prev;
    } else {
      __syncthreads();
    }
    if (wave == 0 || wave == 7) load_pin();
#pragma unroll
    for (int ts = 0; ts < TPW; ++ts) acc[ts] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (hsrc) {
      copy_h(hsrc, nbh);
      product();
    }
    publish();
    __syncthreads();

    const int b = b0 + qrow;
    const bool row_ok = b < nb;
#pragma unroll
    for (int o = 0; o < FIN; ++o) {
      float v[4];
      gates_of(o, v);
      const float gi = sigm(v[0] + bf16_to_f32(pin[o][0]));
      const float gf = sigm(v[1] + bf16_to_f32(pin[o][1]));
      const float gg = tanh_f(v[2] + bf16_to_f32(pin[o][2]));
      const float go = sigm(v[3] + bf16_to_f32(pin[o][3]));
      const float c = gf * c_reg[o] + gi * gg;
      const bf16_t h = f32_to_bf16(go * tanh_f(c));
      if (row_ok && slot_ok(o)) {
        const int u = unit(o) - j0;
        Hb[(int64_t)(off + b) * H + unit(o)] = h;
        *reinterpret_cast<float*>(stC + qrow * CSB + 4 * u) = c;
        *reinterpret_cast<bf16_t*>(stH + qrow * HSB + 2 * u) = h_reg[o];
        *reinterpret_cast<uint2*>(stG + qrow * GSB + 8 * u) = pack_gates(gi, gf, gg, go);
        c_reg[o] = c;
        h_reg[o] = h;
      }
    }
    // h stores complete; so are, one step late, the projections of the step
    // before the last, which this announces
    xsignal(y, local, slot, us, (unsigned)(t + 1));
    if (has_next && threadIdx.x == 0 && t > 1)
      __hip_atomic_store(mine, (unsigned)(t - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ask_below();
    // rows that only the backward pass reads, in 16-byte chunks by waves 1-7:
    // C, then Hs, then G
    if (wave > 0) {
      const int cC = U / 4, cH = U / 8, cG = U / 2;
      const int nC = RB * cC, nH = RB * cH, nG = RB * cG;
      auto divr = [](int e, int d) { return (int)(((unsigned)e * ((65536u + d - 1) / d)) >> 16); };
      for (int e = threadIdx.x - 64; e < nC + nH + nG; e += 448) {
        int r, c;
        const unsigned char* src;
        void* dst;
        if (e < nC) {
          r = divr(e, cC); c = e - r * cC;
          src = stC + r * CSB + 16 * c;
          dst = me.C + (int64_t)(off + b0 + r) * H + j0 + 4 * c;
        } else if (e < nC + nH) {
          const int f = e - nC;
          r = divr(f, cH); c = f - r * cH;
          src = stH + r * HSB + 16 * c;
          dst = Hs + (int64_t)(off + b0 + r) * H + j0 + 8 * c;
        } else {
          const int f = e - nC - nH;
          r = divr(f, cG); c = f - r * cG;
          src = stG + r * GSB + 16 * c;
          dst = Gb + (int64_t)(off + b0 + r) * G4 + 4 * j0 + 8 * c;
        }
        if (b0 + r < nb) *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
      }
    }
    // the successor's projections of step t - 1, from the h rows still in LDS
    if (has_next && t > 0) project(off_prev, nb_prev);
    off_prev = off;
    nb_prev = nb;
    off += nb;
  }
  if (has_next && steps > 0) {
    // the last step's h, then everything announced
    xwait(y, local, slot, members, (unsigned)steps);
    copy_h(Hb + (int64_t)off_prev * H, nb_prev);
    project(off_prev, nb_prev);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0)
      __hip_atomic_store(mine, (unsigned)steps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ------------------------------------------------------------------ launch --

// Slices as in the one-layer kernels: U units of H, `per` slots per XCD.
struct PipeShape {
  int per, KS, U, TPW, XL;
};

bool pipe_shape(int H, int B, int layers, PipeShape* x) {
  if (layers < 2 || layers > PipeFwd::MAX || H % 64 != 0 || H < 128 || H > 768 || B < 1) return false;
  const int slots = layers * ((B + RB - 1) / RB);
  x->KS = H / 32;
  if (slots <= NX) {  // an XCD each: 16 units, 32 beyond H = 512
    x->per = 1;
    x->U = H <= 512 ? 16 : 32;
  } else if (slots <= 2 * NX && H <= 512) {  // half an XCD each
    x->per = 2;
    x->U = H <= 256 ? 16 : 32;
  } else {
    return false;
  }
  if (H % x->U != 0 || H / x->U > 32 / x->per) return false;
  x->TPW = (x->U / 4 + 3) / 4;
  // beyond H = 512 the two take more than 32 fragments a wave: some of W_x's are
  // in LDS
  x->XL = H <= 512 ? 0 : H == 576 ? 4 : H == 640 ? 8 : 12;
  return true;
}

#define AM_PIPE_CASE(KS_, TPW_, XL_)                                               \
  if (x.KS == KS_ && x.TPW == TPW_ && x.XL == XL_) fn = reinterpret_cast<const void*>(lstm_fwd_pipe<KS_, TPW_, XL_>); \
  else

}  // namespace

bool lstm_pipe_covers(int hidden, int B, int layers) {
  PipeShape x;
  return pipe_shape(hidden, B, layers, &x);
}

hipError_t lstm_fwd_pipe_launch(PipeFwd a, PersistSchedule ps, XcdSync y, hipStream_t s, bool* used) {
  *used = false;
  PipeShape x;
  if (!pipe_shape(a.hidden, ps.B, a.layers, &x)) return hipSuccess;
  a.blocks = (ps.B + RB - 1) / RB;
  a.pflags = y.flags + 1024;
  y.units = x.U;
  const char* f = getenv("AM_XCD_FENCED");
  y.fenced = f && f[0] == '1' && f[1] == 0 ? 1 : 0;
  const void* fn = nullptr;
  AM_PIPE_CASE(4, 1, 0) AM_PIPE_CASE(6, 1, 0) AM_PIPE_CASE(8, 1, 0) AM_PIPE_CASE(10, 1, 0)
  AM_PIPE_CASE(12, 1, 0) AM_PIPE_CASE(14, 1, 0) AM_PIPE_CASE(16, 1, 0)
  AM_PIPE_CASE(10, 2, 0) AM_PIPE_CASE(12, 2, 0) AM_PIPE_CASE(14, 2, 0) AM_PIPE_CASE(16, 2, 0)
  AM_PIPE_CASE(18, 2, 4) AM_PIPE_CASE(20, 2, 8) AM_PIPE_CASE(22, 2, 12) AM_PIPE_CASE(24, 2, 12)
  return hipSuccess;
  const int blocks = NX * x.per * (a.hidden / x.U);
  const size_t lds = (size_t)RB * x.KS * 64 + 8 * x.TPW * 64 * 16 + 8 * x.XL * 1024 +
                     (size_t)RB * (14 * x.U + 48);
  int dev = 0, cus = 0, per = 0;
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
      hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, 512, lds) != hipSuccess ||
      per < 1 || blocks > per * cus) {
    (void)hipGetLastError();
    return hipSuccess;
  }
  *used = true;
  void* args[] = {&a, &ps, &y};
  return resident_launch(fn, dim3(blocks), dim3(512), args, lds, s);
}

}  // namespace am
