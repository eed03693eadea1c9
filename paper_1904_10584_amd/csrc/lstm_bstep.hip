// One backward step of a wide layer in one launch: the recurrent product
// dA_{t+1} W_h over its whole k-range (4H) and the cell backward in its
// epilogue.
//
// Split over k to fill the chip, the product (18.3 us for 512 rows x 1536
// units, k = 6144) left fp32 partials for a second launch (9.5 us) to sum.
// Tiles of 64 rows x 48 units make 256 workgroups of that shape with the whole
// k-range each, so the sums stay in the workgroup.  What bounds it is the
// compute unit's fill rate: 112 operand rows of 128 bytes per 64 k, 9 us at 64
// bytes a clock, of which it reaches 40 %; the products are a third of that.  A
// step of that shape takes 22.9 us instead of 27.8, and a training step of five
// such layers over 64 x 512 frames 26.4 ms instead of 28.5 on one card (26.5 to
// 27.5 on others).  Whole-tile waves over a third of the stages each read LDS 2.6
// times less and took 24.0 us.
//
// Fourteen waves.  Two copy: k-tiles of 128 as 28 direct loads of 1 KiB, half
// each, into a ring of five LDS stages, four of them in flight; alone with
// their memory counters, they wait for exactly the loads of the stage that is
// due.  Twelve multiply: two k-halves of a stage by 2 x 3 quadrants of 32 rows
// x 16 units.  The halves meet in LDS after the k-loop, and every compute
// thread finishes four units of one row (the operands of its cells are
// requested before the loop).  W_h is read transposed (k contiguous), both
// operands in 128-byte rows whose 16-byte chunks are XOR-swizzled by row.
// Tiles are ordered so that an XCD's workgroups share a slice of W_h's
// columns, which stays in its L2 from step to step.
#include "am_device.h"
#include "am_internal.h"

namespace am {
namespace {

constexpr int TM = 64, TU = 48;      // tile: rows, units
constexpr int KT = 128;              // k per stage
constexpr int NS = 5;                // LDS stages
constexpr int A_HALF = TM * 64 * 2, B_HALF = TU * 64 * 2;  // bytes of 64 k of each operand
constexpr int STAGE = 2 * (A_HALF + B_HALF);               // 28 KiB
constexpr int LOADS = STAGE / 1024, LPW = LOADS / 2;       // direct loads, per copying wave
constexpr int COMPUTE = 12, THREADS = (COMPUTE + 2) * 64;
constexpr int ROWF = TU + 4;         // floats per row of the partial sums in LDS
constexpr int LDS_BYTES = NS * STAGE;
static_assert(LOADS == 28 && (NS - 2) * LPW < 64, "memory counter");
static_assert(2 * TM * ROWF * 4 <= LDS_BYTES, "the partial sums reuse the stages");
static_assert(TM * TU == COMPUTE * 64 * 4, "four cells a compute thread");

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(THREADS, 1) void lstm_bwd_step_fused(LstmBwdStep a, int tm, int tu) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int H = a.hidden, K = 4 * H;
  // XCD-contiguous order, rows fastest: an XCD's workgroups share W_h columns
  const int G = tm * tu, x = blockIdx.x % 8, q = G / 8, rem = G % 8;
  const int t = x * q + min(x, rem) + (int)blockIdx.x / 8;
  const int m0 = t % tm * TM, u0 = t / tm * TU;
  const bf16_t* __restrict__ dAn = static_cast<const bf16_t*>(a.dAnext);
  const bf16_t* __restrict__ WhT = static_cast<const bf16_t*>(a.WhT);
  const int nk = m0 < a.nbn ? K / KT : 0;  // (rows without a next step: the cell alone)

  if (wave >= COMPUTE) {
    // load i of this wave is instruction q = w LPW + i of the stage: A's two
    // halves (8 instructions of 8 rows each), then B's (6 each)
    const int w = wave - COMPUTE;
    const bf16_t* src[LPW];
    const uint32_t base = lds_address(lds);
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const int n = w * LPW + i;
      const bool isa = n < 16;
      const int half = isa ? n >> 3 : (n - 16) / 6, rg = isa ? n & 7 : (n - 16) % 6;
      const int r = rg * 8 + (lane >> 3), k = half * 64 + (((lane & 7) ^ (r & 7)) << 3);
      // rows past the last re-read it; their results are not used
      src[i] = isa ? dAn + (int64_t)min(m0 + r, a.nbn - 1) * K + k : WhT + (int64_t)min(u0 + r, H - 1) * K + k;
    }
    int next = 0;
    auto issue = [&]() {
      if (next >= nk) return;
      const uint32_t at = __builtin_amdgcn_readfirstlane(base + (next % NS) * STAGE + w * LPW * 1024);
#pragma unroll
      for (int i = 0; i < LPW; ++i) {
        dma16(src[i], at + i * 1024);
        src[i] += KT;
      }
      ++next;
    };
    for (int s = 0; s < NS - 1; ++s) issue();
    for (int s = 0; s < nk; ++s) {
      // stage s has landed once at most the NS - 2 later ones are in flight
      if (next - s == NS - 1) wait_vm_asm<(NS - 2) * LPW>();
      else wait_vm_asm<0>();
      lds_barrier();
      issue();
    }
    if (nk > 0) {
      lds_barrier();  // the last stage has been read
      lds_barrier();  // the partial sums are in LDS
    }
    return;
  }

  // this thread's cells: units uu .. uu + 3 of one row (H % 4 == 0, so four
  // units are inside or outside together)
  const int e = threadIdx.x, row = m0 + e / (TU / 4), uu = u0 + e % (TU / 4) * 4;
  const bool ok = row < a.nb && uu < H, cont = ok && row < a.nbn;
  const int64_t o = (int64_t)min(row, a.nb - 1) * H + min(uu, H - 4);
  // (each read once: non-temporal, so that they do not evict W_h's columns)
  const u32x4_t ga = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(static_cast<const bf16_t*>(a.G) + 4 * o));
  const u32x4_t gb = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(static_cast<const bf16_t*>(a.G) + 4 * o + 8));
  const u32x2_t dh2 = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t*>(static_cast<const bf16_t*>(a.dHa) + o));
  const f32x4_t c4 = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(a.C + o));
  const f32x4_t cp4 = a.Cprev ? *reinterpret_cast<const f32x4_t*>(a.Cprev + o) : f32x4_t{0.f, 0.f, 0.f, 0.f};
  const f32x4_t dc4 = *reinterpret_cast<const f32x4_t*>(a.dc + o);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  float rec[4] = {0.f, 0.f, 0.f, 0.f};
  if (nk > 0) {
    const int kh = wave / 6, wq = wave % 6, wm = wq / 3 * 32, wn = wq % 3 * 16;
    f32x4_t acc[2];
    acc[0] = acc[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto at = [&](int r, int ks) { return r * 64 + (((ks * 4 + (lane >> 4)) ^ (r & 7)) << 3); };
    for (int s = 0; s < nk; ++s) {
      lds_barrier();
      const bf16_t* la = reinterpret_cast<const bf16_t*>(lds + (s % NS) * STAGE + kh * A_HALF);
      const bf16_t* lb = reinterpret_cast<const bf16_t*>(lds + (s % NS) * STAGE + 2 * A_HALF + kh * B_HALF);
      Frag<bf16_t> af[2][2], bf[2];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        bf[ks] = frag_load<bf16_t>(lb + at(wn + (lane & 15), ks));
#pragma unroll
        for (int i = 0; i < 2; ++i) af[ks][i] = frag_load<bf16_t>(la + at(wm + 16 * i + (lane & 15), ks));
      }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 2; ++i) mma_16x16x32(acc[i], af[ks][i], bf[ks]);
    }
    lds_barrier();
    float* part = reinterpret_cast<float*>(lds);  // [k-half][row][unit]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        part[(kh * TM + wm + 16 * i + mfma_row(lane, r)) * ROWF + wn + mfma_col(lane)] = acc[i][r];
    lds_barrier();
    if (cont) {
      const float4 p0 = *reinterpret_cast<const float4*>(part + (row - m0) * ROWF + uu - u0);
      const float4 p1 = *reinterpret_cast<const float4*>(part + (TM + row - m0) * ROWF + uu - u0);
      rec[0] = p0.x + p1.x; rec[1] = p0.y + p1.y; rec[2] = p0.z + p1.z; rec[3] = p0.w + p1.w;
    }
  }
  if (!ok) return;
  const uint32_t gw[8] = {ga[0], ga[1], ga[2], ga[3], gb[0], gb[1], gb[2], gb[3]};
  float dco[4];
  uint32_t out[4][2];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t w0 = gw[2 * k], w1 = gw[2 * k + 1];
    const float gi = bf16_to_f32((bf16_t)(w0 & 0xFFFFu)), gf = bf16_to_f32((bf16_t)(w0 >> 16));
    const float gg = bf16_to_f32((bf16_t)(w1 & 0xFFFFu)), go = bf16_to_f32((bf16_t)(w1 >> 16));
    const float dh = bf16_to_f32((bf16_t)((dh2[k >> 1] >> (16 * (k & 1))) & 0xFFFFu)) + rec[k];
    const float tc = tanh_f(c4[k]);
    const float d_o = dh * tc;
    const float dcell = dh * go * (1.f - tc * tc) + (cont ? dc4[k] : 0.f);
    const float d_i = dcell * gg, d_g = dcell * gi, d_f = dcell * cp4[k];
    dco[k] = dcell * gf;
    const uint32_t v[4] = {f32_to_bf16(d_i * gi * (1.f - gi)), f32_to_bf16(d_f * gf * (1.f - gf)),
                           f32_to_bf16(d_g * (1.f - gg * gg)), f32_to_bf16(d_o * go * (1.f - go))};
#pragma unroll
    for (int g = 0; g < 4; ++g) out[g][k >> 1] = (k & 1) ? out[g][k >> 1] | (v[g] << 16) : v[g];
  }
  *reinterpret_cast<float4*>(a.dc + o) = make_float4(dco[0], dco[1], dco[2], dco[3]);
  bf16_t* arow = static_cast<bf16_t*>(a.dA) + (int64_t)row * K + uu;
#pragma unroll
  for (int g = 0; g < 4; ++g) *reinterpret_cast<uint2*>(arow + g * H) = make_uint2(out[g][0], out[g][1]);
}

}  // namespace

// Which steps: a workgroup fills a compute unit, so up to 256 tiles, one round
// (backward of one layer, split product and cell / fused: 1536 cells, 9 steps of
// 512 sequences, 256 tiles, 379 / 363 us; 576 sequences, 288 tiles, 415 / 521;
// 2048 cells x 384, 258 tiles, 444 / 601), and at least 128: half of the chip
// (1536 cells x 256, 128 tiles, 301 / 286; fewer also gain 2-10 % but are not
// taken).  Beyond 2048 cells the longer k-loop reads the operands no faster than
// the split product does (2560 cells x 256, 64 steps 3247 / 3285; 3072 x 256 4295 /
// 4480).
bool lstm_bwd_step_fused_covers(int hidden, int nb) {
  const int tiles = ((nb + TM - 1) / TM) * ((hidden + TU - 1) / TU);
  return hidden % 32 == 0 && hidden <= 2048 && tiles >= 128 && tiles <= 256;
}

// Whether so many of them are worth W_h's transpose, which the split product
// does without: the transpose takes as long as 0.3 (512 cells), 2.3 (1536) to 4
// steps (2048) gain, and the last step has no product.  Split / fused at 1, 2, 3,
// 4, 6 steps, us: 768 cells x 1024 sequences 70 / 75, 101 / 100, 130 / 124, 158 /
// 148, 219 / 204; 1536 x 256 54 / 61, 88 / 94, 124 / 126, 149 / 149, 207 / 201; 2048
// x 256 64 / 76, 107 / 117, 149 / 156, 182 / 187, 256 / 256.
bool lstm_bwd_fused_pays(int hidden, int steps) {
  return (int64_t)(steps - 2) * (1 << 20) >= (int64_t)hidden * hidden;
}

hipError_t lstm_bwd_step_fused_launch(const LstmBwdStep& a, hipStream_t s) {
  static PerDevice limit;
  const hipError_t e = allow_lds(limit, reinterpret_cast<const void*>(lstm_bwd_step_fused), LDS_BYTES);
  if (e != hipSuccess) return e;
  const int tm = (a.nb + TM - 1) / TM, tu = (a.hidden + TU - 1) / TU;
  hipLaunchKernelGGL(lstm_bwd_step_fused, dim3(tm * tu), dim3(THREADS), LDS_BYTES, s, a, tm, tu);
  return hipGetLastError();
}

}  // namespace am
