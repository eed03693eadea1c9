// XCD-local persistent LSTM layer kernels.
//
// The recurrence exchanges h_{t-1} (dA_{t+1} backward) between the
// workgroups that share a block of sequences at every step.  MI355X has 8
// XCDs, each with its own L2; an exchange through device memory pays a
// write-back of the producer's L2, an invalidation of the consumer's, and
// memory latency on every step.  Here the sequences are split into blocks,
// one or two per XCD, and the workgroups of a block all run on that XCD, so
// the exchange and the step barrier stay inside one L2:
//   * with m workgroups per block, workgroup i serves block i % 8 + 8 (i / 8m)
//     and unit slice (i / 8) % m (workgroups are dispatched to XCDs
//     round-robin); at start every workgroup records its XCC id and, unless
//     every block really is on one XCD, the kernel falls back to
//     device-scope release/acquire for its whole run;
//   * backward, and forward where a block spans XCDs, the step barrier is one
//     128-byte flag line per block: every member
//     stores its count of completed steps in its own word once its stores
//     of the step have completed, and one wave polls the line; within one
//     XCD both stay in its L2 (a store that the L1 passes through, polled
//     with non-temporal loads, which the L1 does not serve from a kept
//     line), a block spanning XCDs uses device-scope accesses and fences;
//     every row exchanged that way is written once and read only after it was
//     written, so no consumer's L1 can hold a stale copy;
//   * forward, within one XCD, the data is its own flag: h goes through a ring
//     of four slots in scratch memory that stays in the L2, where a value not
//     yet written is all ones (no h is); the readers poll the rows themselves,
//     which saves the wait for the stores, the flag's way and a second read.
//     A slot is written anew every four steps, and whatever is not all ones is
//     taken for the current h, so a poll must never be served from a line that
//     this CU's L1 kept from an earlier one.  What that rests on: the ring is
//     read by non-temporal loads alone, which leave no line in the L1 (every poll
//     that has failed before it succeeds, of a flag or of the ring, shows it: the
//     same address again gives the new value).  The memory model does not promise
//     it, so the compiled polls are checked for these bits, and ring and flags
//     are compared bit for bit, also where all four slots fit the L1 (64 and 192
//     cells).
// A workgroup owns U hidden units (U % 4 == 0) of one block of RB sequences
// (RB = 16 or 32).  The forward product keeps the workgroup's 4U columns of
// W_h resident in registers in unit-major, gate-minor order, so a 16-column
// MFMA tile holds 4 units x 4 gates; reading the partial tiles back from
// LDS in 4x4-quad-transposed order then gives each lane all four gate
// pre-activations of one (sequence, unit).  The backward product keeps the
// U columns of W_h in registers too.
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "xcd_sync.h"

namespace am {
namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));

// Two numbers to bf16 (round to nearest even) by the conversion instruction,
// a at the low end.
__device__ __forceinline__ uint32_t cvt_bf16x2(float a, float b) {
  typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b16x2));
}
__device__ __forceinline__ uint2 cvt_gates(float i, float f, float g, float o) {
  return make_uint2(cvt_bf16x2(i, f), cvt_bf16x2(g, o));
}

// 4x4 transpose within each quad of lanes: out[q] of lane l is v[l % 4] of
// lane (l & ~3) + q.
__device__ __forceinline__ void quad_transpose(f32x4_t v, int lane, float* out) {
  auto swap = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  using X1 = std::integral_constant<int, 0xB1>;  // lane ^ 1
  using X2 = std::integral_constant<int, 0x4E>;  // lane ^ 2
  const bool o1 = lane & 1, o2 = lane & 2;
  // (the swaps by every lane, before the selections)
  const float s0 = swap(v[0], X1{}), s1 = swap(v[1], X1{}), s2 = swap(v[2], X1{}), s3 = swap(v[3], X1{});
  const float a0 = o1 ? s1 : v[0], a1 = o1 ? v[1] : s0, a2 = o1 ? s3 : v[2], a3 = o1 ? v[3] : s2;
  const float t0 = swap(a0, X2{}), t1 = swap(a1, X2{}), t2 = swap(a2, X2{}), t3 = swap(a3, X2{});
  out[0] = o2 ? t2 : a0;
  out[1] = o2 ? t3 : a1;
  out[2] = o2 ? a2 : t0;
  out[3] = o2 ? a3 : t1;
}

// ----------------------------------------------------------------- forward --
// Eight waves, two per SIMD (a single wave can issue independent MFMAs at
// about 87 % of the peak, but not also cover its own LDS and memory waits).
// Tile group g = wave % 4 owns the output tiles t = g + 4 ts
// (row tile t % MT, column tile t / MT; all tiles of a group share row tile
// g % MT); k-half kh = wave / 4 multiplies k-steps [kh KS/2, (kh+1) KS/2).
// The W_h fragments of a wave's tiles and k-steps stay in its registers for
// the whole launch.  Each step waves 0-3 read the block's rows of h_{t-1} from
// the ring until all are there and put them into LDS, line-major
// [H/64 lines][RB rows][128 B] with the 16-byte chunks of a row XOR-swizzled
// by row, from where they are read as MFMA fragments; waves 4-7 write the
// step before out (cell states, gates, h, h_{t-1}: staged as rows in LDS, so
// that they go as 16-byte chunks) and fetch the next step's input projections
// into LDS.  Without the ring wave 0 polls the step barrier and waves 1-7
// copy the rows with direct loads.  The two k-halves of a group exchange
// partial tiles through LDS: the k-half-0 wave finishes the first
// ceil(TPW/2) tiles, the k-half-1 wave the rest.
//
// What bounds a step is its chain, about 6600 clocks for 16 rows x 48 units of
// H = 768: sending and polling h 2300, products 1500 (1150 of MFMA issue), the
// partial tiles 500, cells 1500 (vector instructions: two waves per SIMD, four
// clocks each).  Before the ring, with each lane's projections as 2-byte loads
// (1024 clocks of line look-ups a step), partial tiles read transposed from
// LDS (bank conflicts) and bf16 rounding in integer steps it was 7900: 231 us
// for 64 steps of 256 sequences, now 187; 1500 steps of 128 sequences 4.2 ms,
// now 3.8.
template <int MT, int KS, int TPW, bool STG, bool COUNTS>
__global__ __launch_bounds__(512, 1) void lstm_fwd_xcd(PersistFwd a, PersistSchedule ps, XcdSync y) {
  constexpr int RB = 16 * MT;             // sequences per block
  constexpr int KH = KS / 2;              // k-steps per wave
  constexpr int FIN = (TPW + 1) / 2;      // tiles finished by the k-half-0 wave
  constexpr int HS_BYTES = RB * KS * 64;  // the block's h rows: RB x H bf16
  static_assert(KS % 2 == 0, "H must be a multiple of 64");
  constexpr bool RING = STG && MT == 1;   // blocks whose exchange goes through the ring
  extern __shared__ __align__(16) unsigned char lds[];
  bf16_t* hl = reinterpret_cast<bf16_t*>(lds);
  f32x4_t* red = reinterpret_cast<f32x4_t*>(lds + HS_BYTES);  // [8][FIN][64]
  // STG (U % 8 == 0): the block's cell states, h, h_{t-1} copies and gates of
  // the step, staged as rows of the unit slice (strides padded by 16 bytes,
  // which spreads a write's 16 rows over the LDS banks) and written out by
  // waves 4-7 in the next step as 16-byte row chunks: about 100 cache lines
  // per step instead of 16 per store instruction (768).
  unsigned char* stC = lds + HS_BYTES + 8 * FIN * 64 * 16;
  __shared__ int bad_sh;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = wave & 3, kh = wave >> 2;
  const int H = KS * 32, G4 = 4 * H, U = y.units;
  const int ntiles = MT * (U / 4);
  const int members = H / U;
  const int blk = xcd_block(members), us = (blockIdx.x / NX) % members;
  const int b0 = ps.first + blk * RB, j0 = us * U;
  if (b0 >= ps.B) return;  // no sequences: no weights to load (the whole block returns)
  const int mw = g % MT;
  const int CSB = U * 4 + 16, HSB = U * 2 + 16, GSB = U * 8 + 16;  // staged row strides
  unsigned char* stH = stC + RB * CSB;
  unsigned char* stG = stH + RB * HSB;
  unsigned char* stN = stG + RB * GSB;  // h_t (ring exchange)
  // STG: two steps' input projections, [gate][8 units][row] in 16-byte pieces
  bf16_t* stP = reinterpret_cast<bf16_t*>(stN + RB * HSB);
  const bf16_t* __restrict__ P = static_cast<const bf16_t*>(a.P);
  const bf16_t* __restrict__ Wh = static_cast<const bf16_t*>(a.Wh);
  const bf16_t* __restrict__ h0 = static_cast<const bf16_t*>(a.h0);
  bf16_t* __restrict__ Hb = static_cast<bf16_t*>(a.H);
  bf16_t* __restrict__ Hs = static_cast<bf16_t*>(a.Hs);
  bf16_t* __restrict__ Gb = static_cast<bf16_t*>(a.G);

  // resident weights: column c of tile n is unit j0 + 4n + c/4, gate c%4
  Frag<bf16_t> wf[TPW][KH];
#pragma unroll
  for (int ts = 0; ts < TPW; ++ts) {
    const int t = g + 4 * ts;
    const int n = (t < ntiles ? t : 0) / MT;
    const int c = lane & 15;
    const int row = (c & 3) * H + j0 + 4 * n + (c >> 2);
#pragma unroll
    for (int s = 0; s < KH; ++s)
      wf[ts][s] = frag_load<bf16_t>(Wh + (int64_t)row * H + (kh * KH + s) * 32 + (lane >> 4) * 8);
  }
  bf16_t* const hring = static_cast<bf16_t*>(a.ring);
  const int64_t slot = (int64_t)ps.B * H;  // elements of a ring slot
  // The 16-byte piece of this member's slice of a slot that this thread (of
  // the first 2U) writes and unwrites: row pr, chunk pc.
  const int u8 = STG ? U / 8 : 1;
  const int pr = threadIdx.x / u8, pc = threadIdx.x % u8;
  const bool piece_ok = RING && pr < RB && b0 + pr < ps.B;
  const uint32_t piece = (uint32_t)((b0 + pr) * H + j0 + 8 * pc);
  const u32x4_t unset = {~0u, ~0u, ~0u, ~0u};
  if (piece_ok && hring) {
#pragma unroll
    for (int q = 0; q < RING_SLOTS; ++q) *reinterpret_cast<u32x4_t*>(hring + q * slot + piece) = unset;
  }
  if (RING) {
    __builtin_amdgcn_s_waitcnt(0);  // in the L2 before the XCC id is published
    __syncthreads();
  }
  const bool local = check_local(y, blk, us, members, &bad_sh);
  const bool ring = RING && local && hring != nullptr;

  // The tiles this wave finishes ("own slots" o < FIN): tile index
  // ts = o (k-half 0) or FIN + o (k-half 1).  The lane's cells in tile t:
  // row mw*16 + 4(lane/16) + lane%4 of the block, unit j0 + 4(t/MT) + (lane%16)/4.
  const int qrow = mw * 16 + 4 * (lane >> 4) + (lane & 3);
  auto slot_ts = [&](int o) { return kh == 0 ? o : FIN + o; };
  auto slot_ok = [&](int o) { return slot_ts(o) < TPW && g + 4 * slot_ts(o) < ntiles; };
  auto unit = [&](int o) {
    const int t = g + 4 * slot_ts(o);
    return j0 + 4 * ((t < ntiles ? t : 0) / MT) + ((lane & 15) >> 2);
  };
  float c_reg[FIN];
  bf16_t h_reg[FIN];
#pragma unroll
  for (int o = 0; o < FIN; ++o) {
    const int b = min(b0 + qrow, ps.B - 1), j = unit(o);
    c_reg[o] = a.c0[(int64_t)b * H + j];
    h_reg[o] = h0 ? h0[(int64_t)b * H + j] : (bf16_t)0;
  }

  // The polling wave (wave 0) copies no h rows and issues no stores between
  // the signal and its next poll: a wave's memory counter retires in order,
  // so stores issued before the poll would hold up the poll's loads.  With
  // STG the staged rows are written out by waves 1-7; without, wave 0 stores
  // its cells' cell state, gates and h_{t-1} one step late, right after its
  // next poll, from dc / dg / dh (row drow, or -1).
  float dc[FIN];
  uint2 dg[FIN];
  bf16_t dh[FIN];
  int drow = -1;
  auto post_stores = [&](int row, const float* cv, const uint2* gv, const bf16_t* hv) {
#pragma unroll
    for (int o = 0; o < FIN; ++o) {
      if (!slot_ok(o)) continue;
      const int j = unit(o);
      const int64_t ofs = (int64_t)row * H + j;
      a.C[ofs] = cv[o];
      Hs[ofs] = hv[o];
      store_gates(Gb + (int64_t)row * G4, j, gv[o]);
    }
  };
  // Input projections of the block's cells (independent of the exchange),
  // requested one step ahead.  STG: by waves 4-7 into LDS, 16 rows x 16 bytes
  // x 4 an instruction (an eighth of the cache lines that 2-byte loads of each
  // lane's cells touch).  Else by each lane, right after the exchange, so that
  // the next exchange's loads, which come back in order behind them, find them
  // arrived; clamped, unmasked loads, so that they issue back to back.
  constexpr int PI = STG ? 2 : 1;  // instructions per wave (U <= 64)
  int pcol[PI];
#pragma unroll
  for (int i = 0; i < PI; ++i) {
    const int cg = (i * 4 + (wave & 3)) * 4 + (lane >> 4);  // gate and 8-unit group
    pcol[i] = cg / u8 * H + j0 + cg % u8 * 8;
  }
  bf16_t pnext[FIN][4];
  auto load_pin = [&](int t_, int o_, int n_) {
    if constexpr (STG) {
      if (wave < 4 || b0 >= n_) return;
      const bf16_t* base = P + (int64_t)o_ * G4;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const uint32_t row = (uint32_t)(min(b0 + 16 * m + (lane & 15), n_ - 1) * G4);
#pragma unroll
        for (int i = 0; i < PI; ++i) {
          const int n = i * 4 + (wave & 3);
          if (n >= U / 8) continue;
          dma16(base + (row + (uint32_t)pcol[i]),
                __builtin_amdgcn_readfirstlane(lds_address(stP + (((t_ & 1) * MT + m) * (U / 8) + n) * 512)));
        }
      }
    } else {
      const bf16_t* base = P + (b0 < n_ ? (int64_t)o_ * G4 : 0);
      const uint32_t row = b0 < n_ ? (uint32_t)(min(b0 + qrow, n_ - 1) * G4) : 0u;
#pragma unroll
      for (int o = 0; o < FIN; ++o)
#pragma unroll
        for (int q = 0; q < 4; ++q) pnext[o][q] = base[row + (uint32_t)(q * H + unit(o))];
    }
  };
  // STG: a finished step's staged rows, written by waves 4-7 (the other four
  // fetch h) as 16-byte chunks, an equal share each: the gates by waves 4 and
  // 5, C by wave 6, Hs and with the ring H by wave 7.  Chunk e of a section
  // with cpr chunks per row is row e / cpr (by a multiply: e is small).
  auto write_staged = [&](int off_w, int nb_w) {
    // (two sections of one shape, the second one's chunks after the first's)
    auto sections = [&](const unsigned char* st, int stride, int cpr, int first, int step, int n, char* dst,
                        char* dst2, uint32_t ld) {
      const uint32_t inv = (65536u + cpr - 1) / cpr;
      for (int e0 = lane + first; e0 < n; e0 += 4 * step) {
        uint4 v[4];
        char* d[4];
        bool ok[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int e = min(e0 + k * step, n - 1);
          const bool two = e >= RB * cpr;
          const int f = two ? e - RB * cpr : e;
          const int r = (int)((uint32_t)f * inv >> 16), c = f - r * cpr;
          v[k] = *reinterpret_cast<const uint4*>(st + (two ? stN - stH : 0) + r * stride + 16 * c);
          d[k] = (two ? dst2 : dst) + (uint32_t)(r * ld + 16 * c);
          ok[k] = e0 + k * step < n && b0 + r < nb_w;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (ok[k]) *reinterpret_cast<uint4*>(d[k]) = v[k];
      }
    };
    const int64_t row0 = off_w + b0, at = row0 * H + j0;
    if (wave < 6) {
      sections(stG, GSB, U / 2, (wave - 4) * 64, 128, RB * U / 2, reinterpret_cast<char*>(Gb + 4 * at), nullptr, 2 * G4);
    } else if (wave == 6) {
      sections(stC, CSB, U / 4, 0, 64, RB * U / 4, reinterpret_cast<char*>(a.C + at), nullptr, 4 * H);
    } else {
      sections(stH, HSB, U / 8, 0, 64, (ring ? 2 : 1) * RB * U / 8, reinterpret_cast<char*>(Hs + at),
               reinterpret_cast<char*>(Hb + at), 2 * H);
    }
  };
  int nb = active_down<COUNTS>(ps, ps.B, 0), off = 0, off_prev = 0, nb_prev = 0;
  load_pin(0, 0, nb);
  PollBudget<SPIN_LIMIT> polls;
  // every load so far (weights, state, the first projections) is complete
  // here, so the compiler keeps no waits for them inside the loop
  wait_vm<0>();
  for (int t = 0; t < ps.T; ++t) {
    if (b0 >= nb) break;  // this block of sequences has ended for good
    const int nb_next = t + 1 < ps.T ? active_down<COUNTS>(ps, nb, t + 1) : 0;

    bf16_t pin[FIN][4];
    if constexpr (STG) {
      if (wave >= 4) wait_vm_asm<0>();  // this step's projections, asked for a step ago
    } else {
#pragma unroll
      for (int o = 0; o < FIN; ++o)
#pragma unroll
        for (int q = 0; q < 4; ++q) pin[o][q] = pnext[o][q];
    }
    constexpr int RG = RB / 8, NQ = (KS / 2) * RG;  // pieces of 8 rows x 128 bytes
    const bf16_t* hsrc = h0;
    if (STG && t > 0 && wave >= 4) write_staged(off_prev, nb_prev);
    if (ring && t > 0) {
      if constexpr (RING) {
        if (wave < 4) {
          // send this member's h_{t-1}
          if (piece_ok && b0 + pr < nb_prev)
            *reinterpret_cast<u32x4_t*>(hring + ((t - 1) & (RING_SLOTS - 1)) * slot + piece) =
                *reinterpret_cast<const u32x4_t*>(stN + pr * HSB + 16 * pc);
          // waves 0-3 read the ring until every value has been written, then
          // put the rows (inactive rows read an active one) into LDS
          // (wave w: rows 8 (w % 2) .., lines w / 2, w / 2 + 2, ..; an odd
          // number of lines has its last fetched by all four)
          constexpr int PQ = (NQ + 3) / 4;
          const int r = (wave & 1) * 8 + (lane >> 3), l0 = wave >> 1;
          auto line = [&](int i) { return NQ % 4 != 0 && i == PQ - 1 ? KS / 2 - 1 - l0 : 2 * i; };  // beyond l0
          const bf16_t* hs = hring + ((t - 1) & (RING_SLOTS - 1)) * slot;
          const uint32_t at = (uint32_t)(min(b0 + r, nb - 1) * H + l0 * 64 + (lane & 7) * 8);
          u32x4_t v[PQ];
          polls.begin();
          for (;;) {
#pragma unroll
            for (int i = 0; i < PQ; ++i)
              v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(hs + (at + (uint32_t)(line(i) * 64))));
            wait_vm_asm<0>();  // (the stores issued before, too)
            u16x2_t top = 0;  // (all ones, an unwritten value, is the largest)
#pragma unroll
            for (int i = 0; i < PQ; ++i)
#pragma unroll
              for (int k = 0; k < 4; ++k)
                top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2_t, (uint32_t)v[i][k]));
            if (!__any(top[0] == 0xffffu || top[1] == 0xffffu)) break;
            if (polls.spent()) {
              if (lane == 0) __hip_atomic_store(y.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              break;
            }
          }
#pragma unroll
          for (int i = 0; i < PQ; ++i)
            *reinterpret_cast<u32x4_t*>(hl + ((l0 + line(i)) * RB + r) * 64 + (((lane & 7) ^ (r & 7)) << 3)) = v[i];
        }
      }
      load_pin(t + 1, off + nb, nb_next);
      lds_barrier();
      // All four waves have seen their part of h_{t-1}, so every member has
      // sent it and has read h_{t-2} before: unwrite this member's piece of
      // h_{t-2}.  (A wave's own poll covers some members only.)  That store
      // is complete before this wave's poll of step t + 1 ends, so before
      // h_{t+1} is sent, and a member polls the slot again only after it has
      // received h_{t+1}.
      if (t > 1 && piece_ok) *reinterpret_cast<u32x4_t*>(hring + ((t - 2) & (RING_SLOTS - 1)) * slot + piece) = unset;
    } else {
      if (t > 0) {
        xwait(y, local, blk, members, (unsigned)t);
        hsrc = Hb + (int64_t)off_prev * H;
      }
      if (wave == 0 && drow >= 0) {
        post_stores(drow, dc, dg, dh);
        drow = -1;
      }
      if (hsrc && wave > 0) {
        // the block's rows of h_{t-1} (inactive rows read an active one) to
        // LDS, by waves 1-7
        for (int q = wave - 1; q < NQ; q += 7) {
          const int line = q / RG, rg = q % RG;
          const int r = rg * 8 + (lane >> 3);
          const int chunk = line * 8 + ((lane & 7) ^ (r & 7));
          dma16(hsrc + (int64_t)min(b0 + r, nb - 1) * H + chunk * 8,
                __builtin_amdgcn_readfirstlane(lds_address(hl + (line * RB + rg * 8) * 64)));
        }
        wait_vm<0>();
      }
      load_pin(t + 1, off + nb, nb_next);
      lds_barrier();
    }
    f32x4_t acc[TPW];
#pragma unroll
    for (int ts = 0; ts < TPW; ++ts) acc[ts] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (t > 0 || hsrc) {
      // A fragments in batches of up to four, each batch read before its
      // MFMAs (the resident weights leave room for four in registers)
      constexpr int AB = TPW * KH > 32 ? 3 : KH > 4 ? 4 : KH;
      const int r = mw * 16 + (lane & 15);
#pragma unroll
      for (int s0 = 0; s0 < KH; s0 += AB) {
        Frag<bf16_t> af[AB];
#pragma unroll
        for (int s = 0; s < AB; ++s) {
          if (s0 + s >= KH) continue;  // (compile time: the last batch may be shorter)
          const int c = (kh * KH + s0 + s) * 4 + (lane >> 4);
          af[s] = *reinterpret_cast<const Frag<bf16_t>*>(
              hl + ((c >> 3) * RB + r) * 64 + (((c & 7) ^ (r & 7)) << 3));
        }
        __builtin_amdgcn_sched_barrier(0);
        // unconditional: a tile past the last holds tile 0's weights and its
        // result is never used (a guard here would branch around each MFMA)
#pragma unroll
        for (int s = 0; s < AB; ++s) {
          if (s0 + s >= KH) continue;
#pragma unroll
          for (int ts = 0; ts < TPW; ++ts) mma_16x16x32(acc[ts], af[s], wf[ts][s0 + s]);
        }
      }
    }

    // Each k-half publishes the partial tiles that the other finishes and adds
    // the other's to its own.  A 4x4 transpose over quads of lanes (DPP) then
    // gives lane l, for row 4(l/16) + l%4, the 4 gates of its unit from lanes
    // (l & ~3) + q.
    f32x4_t own[FIN];
    if (kh == 0) {
#pragma unroll
      for (int o = 0; o < FIN; ++o) {
        own[o] = acc[o];
        if (FIN + o < TPW) red[(g * FIN + o) * 64 + lane] = acc[FIN + o];
      }
    } else {
#pragma unroll
      for (int o = 0; o < FIN; ++o) {
        own[o] = FIN + o < TPW ? acc[FIN + o] : f32x4_t{0.f, 0.f, 0.f, 0.f};
        red[((g + 4) * FIN + o) * 64 + lane] = acc[o];
      }
    }
    if constexpr (STG) {
#pragma unroll
      for (int o = 0; o < FIN; ++o) {
        const int u = unit(o) - j0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          pin[o][q] = stP[((((t & 1) * MT + mw) * 4 + q) * (U / 8) + (u >> 3)) * 128 + (lane >> 4) * 32 + (lane & 3) * 8 + (u & 7)];
      }
    }
    lds_barrier();
    float gate[FIN][4];
#pragma unroll
    for (int o = 0; o < FIN; ++o) {
      // (k-half 1's slots past the last tile read unset memory; unused)
      const f32x4_t v = own[o] + red[((g + 4 * (1 - kh)) * FIN + o) * 64 + lane];
      quad_transpose(v, lane, gate[o]);
    }

    const int b = b0 + qrow;
    const bool row_ok = b < nb;
    float cnew[FIN];
    bf16_t hprev[FIN];
#pragma unroll
    for (int o = 0; o < FIN; ++o) {
      hprev[o] = h_reg[o];
      gate[o][0] = sigm(gate[o][0] + bf16_to_f32(pin[o][0]));
      gate[o][1] = sigm(gate[o][1] + bf16_to_f32(pin[o][1]));
      gate[o][2] = tanh_f(gate[o][2] + bf16_to_f32(pin[o][2]));
      gate[o][3] = sigm(gate[o][3] + bf16_to_f32(pin[o][3]));
      cnew[o] = gate[o][1] * c_reg[o] + gate[o][0] * gate[o][2];
      bf16_t h = (bf16_t)cvt_bf16x2(gate[o][3] * tanh_f(cnew[o]), 0.f);
      if ((h & 0x7fffu) > 0x7f80u) h = 0x7fc0u;  // one NaN: all ones is the ring's "not yet"
      if (row_ok && slot_ok(o)) {
        if (!ring) Hb[(int64_t)(off + b) * H + unit(o)] = h;
        c_reg[o] = cnew[o];
        h_reg[o] = h;
        if constexpr (STG) {
          const int u = unit(o) - j0;
          *reinterpret_cast<bf16_t*>(stN + qrow * HSB + 2 * u) = h;
          *reinterpret_cast<float*>(stC + qrow * CSB + 4 * u) = cnew[o];
          *reinterpret_cast<bf16_t*>(stH + qrow * HSB + 2 * u) = hprev[o];
          *reinterpret_cast<uint2*>(stG + qrow * GSB + 8 * u) =
              cvt_gates(gate[o][0], gate[o][1], gate[o][2], gate[o][3]);
        }
      }
    }
    if (ring) lds_barrier();  // the staged rows
    else xsignal(y, local, blk, us, (unsigned)(t + 1));  // h stores complete; its barrier also orders the LDS reuse
    if constexpr (!STG) {  // stores only the backward pass reads
    uint2 gp[FIN];
#pragma unroll
    for (int o = 0; o < FIN; ++o) gp[o] = cvt_gates(gate[o][0], gate[o][1], gate[o][2], gate[o][3]);
    if (wave != 0) {
      if (row_ok) post_stores(off + b, cnew, gp, hprev);
    } else if (row_ok) {
#pragma unroll
      for (int o = 0; o < FIN; ++o) {
        dc[o] = cnew[o];
        dg[o] = gp[o];
        dh[o] = hprev[o];
      }
      drow = off + b;
    }
    }
    off_prev = off;
    nb_prev = nb;
    off += nb;
    nb = nb_next;
  }
  if (wave == 0 && drow >= 0) post_stores(drow, dc, dg, dh);
  if (STG && wave >= 4 && nb_prev > 0) write_staged(off_prev, nb_prev);
}

// ---------------------------------------------------------------- backward --
// dh_rec[rows][units] = dA_{t+1}[rows][4H] W_h[4H][units]: output tiles of
// 16 units (the last one partly empty).  Eight waves split the 4H-long k
// range: wave w multiplies k-steps [w KW, (w+1) KW) and keeps the W_h^T
// fragments of those k-steps, for every unit tile, in registers.  Each wave
// fetches its k-slice of the block's dA_{t+1} rows itself, with direct loads
// into private LDS buffers in chunks of CH k-steps, so it waits only on its
// own loads: one buffer per chunk where the LDS holds them all (16-row
// blocks: three chunks, 96 KiB over the eight waves), else two used in turn.
// The eight partial products are summed in a fixed order through LDS; the
// cell backward (dc carried in registers) is spread over the first seven
// waves in items of one row per lane, an equal number per SIMD, while the
// last wave polls the step barrier.
//
// A wave's k-slice in chunks of four k-steps (256 bytes of a row), then what
// is left as two and one (hidden sizes that are odd multiples of 64).
struct BwdChunks {
  int kw;
  constexpr int full() const { return kw / 4; }
  constexpr int rem() const { return kw % 4; }
  constexpr int count() const { return full() + (rem() == 0 ? 0 : rem() == 3 ? 2 : 1); }
  constexpr int steps(int c) const { return c < full() ? 4 : rem() != 3 ? rem() : c == full() ? 2 : 1; }
  constexpr int start(int c) const { return c <= full() ? 4 * c : 4 * full() + 2; }
};
// Chunk buffers per wave, and the LDS bytes of a wave's buffers (end to end
// where every chunk has its own).
constexpr int bwd_chunk_buffers(int MT, int KW) {
  const int nch = BwdChunks{KW}.count();
  if (8 * 16 * MT * KW * 64 <= 160 * 1024) return nch;
  return nch < 2 ? nch : 2;
}
constexpr int bwd_wave_bytes(int MT, int KW) {
  const BwdChunks ch{KW};
  const int nb = bwd_chunk_buffers(MT, KW);
  return 16 * MT * 64 * (nb == ch.count() ? KW : nb * ch.steps(0));
}
template <int N, typename F, int I = 0> __device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, F, I + 1>(static_cast<F&&>(f));
  }
}
template <int MT, int NTU, int KW, bool COUNTS>
__global__ __launch_bounds__(512, 1) void lstm_bwd_xcd(PersistBwd a, PersistSchedule ps, XcdSync y) {
  constexpr int RB = 16 * MT;                 // sequences per block
  constexpr BwdChunks CK{KW};
  constexpr int NCH = CK.count();                // chunks per step
  constexpr int NB = bwd_chunk_buffers(MT, KW);  // chunk buffers per wave
  constexpr int CHB = RB * CK.steps(0) * 64;     // bytes per buffer
  constexpr int WB = bwd_wave_bytes(MT, KW);
  static_assert(NB >= 1 && NB <= NCH, "chunk buffers");
  static_assert(NB == NCH || KW % 4 == 0, "buffers used in turn: chunks of one size");
  static_assert(8 * WB <= 160 * 1024, "LDS");
  // element offset of chunk c in the wave's buffers
  auto chunk_at = [](int c) constexpr { return NB == NCH ? BwdChunks{KW}.start(c) * RB * 32 : (c % NB) * (CHB / 2); };
  static_assert(MT * NTU * 4 <= 32, "cell items: at most 8 per SIMD");
  extern __shared__ __align__(16) unsigned char lds[];
  bf16_t* buf = reinterpret_cast<bf16_t*>(lds + (threadIdx.x >> 6) * WB);
  f32x4_t* red = reinterpret_cast<f32x4_t*>(lds);  // [8][MT][NTU][64], after the products
  __shared__ int bad_sh;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int H = a.hidden, G4 = 4 * H, U = y.units;
  const int members = H / U;
  const int blk = xcd_block(members), us = (blockIdx.x / NX) % members;
  const int b0 = ps.first + blk * RB, j0 = us * U;
  if (b0 >= ps.B) return;  // no sequences: no weights to load (the whole block returns)
  const bf16_t* __restrict__ WhT = static_cast<const bf16_t*>(a.WhT);
  const bf16_t* __restrict__ dHa = static_cast<const bf16_t*>(a.dHa);
  const bf16_t* __restrict__ Gb = static_cast<const bf16_t*>(a.G);
  bf16_t* __restrict__ dA = static_cast<bf16_t*>(a.dA);

  // resident W_h^T fragments (8 consecutive k of one unit: one 16-byte load
  // of the transposed W_h): k-step wave KW + s, unit tile n, lane column
  // c -> unit j0 + 16n + min(c, vc_n - 1) (vc_n = valid columns of tile n)
  // (H = 192: 24 k-steps, four each in the first six waves)
  const int wv = __builtin_amdgcn_readfirstlane(wave);  // (scalar: wave-uniform indices and branches)
  const bool has_k = wv * KW * 32 < G4;
  Frag<bf16_t> wb[KW][NTU];
#pragma unroll
  for (int n = 0; n < NTU; ++n) {
    const int unit = j0 + 16 * n + min(lane & 15, min(16, U - 16 * n) - 1);
#pragma unroll
    for (int s = 0; s < KW; ++s)
      wb[s][n] = frag_load<bf16_t>(WhT + (int64_t)unit * G4 + (has_k ? (wave * KW + s) * 32 : 0) + (lane >> 4) * 8);
  }
  const bool local = check_local(y, blk, us, members, &bad_sh);

  // Cell work: items p = (row tile m, unit tile n, quad row r), MT NTU 4 of
  // them; item p covers, per lane, unit 16n + lane%16 and row
  // 16m + 4(lane/16) + r.  The last wave polls the barrier and takes none;
  // a wave's items run as one dependent chain (the phase is bound by its
  // latency, not by the SIMD's issue rate), so no wave takes more than
  // IPS = ceil(NI / 7): waves 0-3 (one per SIMD) IPS each, waves 4-6 the
  // rest, evenly (12 items: 2, 2, 2, 2 and 2, 1, 1).
  constexpr int NI = MT * NTU * 4, IPS = (NI + 6) / 7;
  constexpr int FIRST = NI < 4 * IPS ? NI : 4 * IPS, REST = NI - FIRST;
  int i_lo, i_hi;
  if (wv < 4) {
    i_lo = min(NI, wv * IPS);
    i_hi = min(FIRST, i_lo + IPS);
  } else if (wv < 7) {
    const int w = wv - 4;
    i_lo = FIRST + w * (REST / 3) + min(w, REST % 3);
    i_hi = i_lo + REST / 3 + (w < REST % 3 ? 1 : 0);
  } else {
    i_lo = i_hi = NI;
  }
  const int nitems = i_hi - i_lo;  // at most IPS
  auto item_m = [&](int k) { return (i_lo + k) / (NTU * 4); };
  auto item_n = [&](int k) { return ((i_lo + k) / 4) % NTU; };
  auto item_r = [&](int k) { return (i_lo + k) % 4; };
  auto item_u = [&](int k) { return 16 * item_n(k) + (lane & 15); };  // unit within the slice
  auto item_j = [&](int k) { return j0 + (item_u(k) < U ? item_u(k) : 0); };
  auto item_row = [&](int k) { return item_m(k) * 16 + mfma_row(lane, item_r(k)); };
  float dc_reg[IPS];
#pragma unroll
  for (int k = 0; k < IPS; ++k) dc_reg[k] = 0.f;

  int nb = ps.T > 0 ? active_up<COUNTS>(ps, 0, ps.T - 1) : 0;
  int off = ps.N - nb;
  int nb_next = 0, off_next = 0;
  unsigned done = 0;
  for (int t = ps.T - 1; t >= 0; --t) {
    if (t < ps.T - 1) {
      nb_next = nb;
      off_next = off;
      nb = active_up<COUNTS>(ps, nb_next, t);
      off = off_next - nb;
    }
    if (b0 >= nb) continue;
    const int nb_prev = t > 0 ? active_up<COUNTS>(ps, nb, t - 1) : 0;
    const int off_prev = off - nb_prev;

    // This wave's cell inputs (independent of the exchange), issued after
    // the first NB chunks' direct loads so that the chunk waits can leave
    // them in flight: NL loads (one instruction each), the same number in
    // every wave (clamped addresses for items past the wave's last), which
    // the wait counts below assume.  Issued before the exchange instead, they would sit ahead of
    // the chunks in the in-order memory counter and hold up the product.
    bf16_t gv[IPS][4], dhv[IPS];
    float cv[IPS], cpv[IPS];
    constexpr int NL = 4 * IPS;  // gates (8 bytes), c_t, c_{t-1}, dh_t per item
    auto load_cell = [&]() {
      const float* cprev_rows = t > 0 ? a.C + (int64_t)off_prev * H : a.c0;
#pragma unroll
      for (int k = 0; k < IPS; ++k) {
        const int b = min(b0 + item_row(k), nb - 1), j = item_j(k);
        const int64_t o = (int64_t)(off + b) * H + j;
        load_gates(Gb + (int64_t)(off + b) * G4, j, gv[k]);
        cv[k] = a.C[o];
        cpv[k] = cprev_rows[(int64_t)b * H + j];
        dhv[k] = dHa[o];
      }
    };

    f32x4_t acc[MT][NTU];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < NTU; ++n) acc[m][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (b0 < nb_next) {
      // polled from the last wave, which has no cell work and no loads in flight
      xwait(y, local, blk, members, done, 7);
      if (!has_k) {
        load_cell();
      } else {
      const bf16_t* dAn = dA + (int64_t)off_next * G4 + wave * KW * 32;
      // chunk c of this wave's k-slice into its buffer: RB rows of
      // steps(c) k-steps; instruction i covers rows i*(64/CPR) .., 16-byte
      // pieces swizzled by row
      auto issue = [&](auto cc) {
        constexpr int c = decltype(cc)::value, CPR = CK.steps(c) * 4, SW = (CPR < 8 ? CPR : 8) - 1;
#pragma unroll
        for (int i = 0; i < MT * CK.steps(c); ++i) {
          const int row = i * (64 / CPR) + lane / CPR;
          const int piece = (lane % CPR) ^ (row & SW);
          dma16(dAn + (int64_t)min(b0 + row, nb_next - 1) * G4 + CK.start(c) * 32 + piece * 8,
                __builtin_amdgcn_readfirstlane(lds_address(buf + chunk_at(c) + i * 512)));
        }
      };
      // the first NB chunks at once (every chunk where the buffers allow:
      // one memory latency per step rather than one per buffer round), then
      // the cell inputs; chunk c + NB goes into chunk c's buffer once c has
      // been read
      static_for<NB>(issue);
      load_cell();
      static_for<NCH>([&](auto cc) {
        constexpr int c = decltype(cc)::value, ST = CK.steps(c), SW = (ST < 2 ? 4 : 8) - 1;
        // in flight behind chunk c at its wait: the chunks issued after it
        // (up to c + NB - 1) and, while c is one of the first NB, the cell
        // loads
        constexpr int last = c + NB < NCH ? c + NB : NCH;  // chunks issued so far
        constexpr int end = CK.start(last - 1) + CK.steps(last - 1);
        wait_vm_n<40>((end - CK.start(c) - ST) * MT + (c < NB ? NL : 0));
        const bf16_t* bb = buf + chunk_at(c);
#pragma unroll
        for (int ks = 0; ks < ST; ++ks) {
          Frag<bf16_t> af[MT];
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            const int row = m * 16 + (lane & 15), piece = ks * 4 + (lane >> 4);
            af[m] = *reinterpret_cast<const Frag<bf16_t>*>(bb + row * ST * 32 + ((piece ^ (row & SW)) << 3));
          }
#pragma unroll
          for (int n = 0; n < NTU; ++n)
#pragma unroll
            for (int m = 0; m < MT; ++m) mma_16x16x32(acc[m][n], af[m], wb[CK.start(c) + ks][n]);
        }
        if constexpr (c + NB < NCH) {
          __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this buffer's reads are done
          issue(std::integral_constant<int, c + NB>{});
        }
      });
      }
    } else {
      load_cell();
    }
    // fixed-order sum of the eight partial products
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < NTU; ++n) red[((wave * MT + m) * NTU + n) * 64 + lane] = acc[m][n];
    __syncthreads();

#pragma unroll
    for (int k = 0; k < IPS; ++k) {
      if (k >= nitems) break;  // (wave-uniform)
      // the eight partial products of this item's cell, in wave order
      const int m = item_m(k), n = item_n(k), r = item_r(k);
      float rec = 0.f;
#pragma unroll
      for (int w = 0; w < 8; ++w) rec += reinterpret_cast<const float*>(red + ((w * MT + m) * NTU + n) * 64 + lane)[r];
      const int b = b0 + item_row(k), j = item_j(k);
      if (item_u(k) >= U || b >= nb) continue;
      const bool cont = b < nb_next;
      const float vi = bf16_to_f32(gv[k][0]), vf = bf16_to_f32(gv[k][1]);
      const float vg = bf16_to_f32(gv[k][2]), vo = bf16_to_f32(gv[k][3]);
      const float dhh = bf16_to_f32(dhv[k]) + (cont ? rec : 0.f);
      const float tc = tanh_f(cv[k]);
      const float d_o = dhh * tc;
      const float dcell = dhh * vo * (1.f - tc * tc) + (cont ? dc_reg[k] : 0.f);
      const float d_i = dcell * vg, d_g = dcell * vi, d_f = dcell * cpv[k];
      dc_reg[k] = dcell * vf;
      bf16_t* arow = dA + (int64_t)(off + b) * G4;
      arow[j] = f32_to_bf16(d_i * vi * (1.f - vi));
      arow[H + j] = f32_to_bf16(d_f * vf * (1.f - vf));
      arow[2 * H + j] = f32_to_bf16(d_g * (1.f - vg * vg));
      arow[3 * H + j] = f32_to_bf16(d_o * vo * (1.f - vo));
    }
    ++done;
    xsignal(y, local, blk, us, done);  // its barrier also orders the LDS reuse
  }
}

// ------------------------------------------------------------------ launch --

// Units per workgroup: the least multiple of `step` dividing H with at most
// `members` workgroups per block.
int xcd_units(int H, int members, int step) {
  for (int U = step; U <= H; U += step)
    if (H % U == 0 && H / U <= members) return U;
  return 0;
}

bool fits(const void* fn, int blocks, int threads, size_t lds) {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, threads, lds) != hipSuccess) return false;
  return per > 0 && blocks <= per * cus;
}

template <typename K>
hipError_t coop(K kernel, int blocks, int threads, size_t lds, void** args, hipStream_t s,
                bool* used) {
  const void* fn = reinterpret_cast<const void*>(kernel);
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
      !fits(fn, blocks, threads, lds)) {
    (void)hipGetLastError();
    *used = false;
    return hipSuccess;
  }
  *used = true;
  return resident_launch(fn, dim3(blocks), dim3(threads), args, lds, s);
}

// Shapes covered: bf16 (the resident slices are sized for it), hidden sizes
// that are multiples of 64 with the resident weight slices within the
// register budget (H <= 1024), B up to XCD_MAX_ROUNDS launches.  Blocks hold 16 sequences.  Up to 128 of
// them take one block per XCD, served by up to 32 workgroups; more take two
// per XCD of up to 16 workgroups each where their slices fit (H <= 768): per
// step each workgroup then reads the same exchanged bytes for twice as many
// units.  Beyond what one launch holds, the sequences go in rounds.
// AM_XCD_BLOCKS=1 in the environment selects blocks of 32 sequences for 128 <
// B <= 256 (MT = 2; hidden 64, 128 and 768).
struct XShape {
  int MT, BPX, KS, U, NT, TPW, NTU, KW, rounds;
  bool ok;
};

XShape xshape_of(int H, int MT, int BPX, int U) {
  XShape x{};
  x.MT = MT;
  x.BPX = BPX;
  x.KS = H / 32;
  x.U = U;
  if (U == 0) return x;
  x.NT = U / 4;
  x.TPW = (MT * x.NT + 3) / 4;
  x.NTU = (U + 15) / 16;
  x.KW = H == 192 ? 4 : 4 * H / 32 / 8;  // backward k-steps per wave (eight waves; 192: six)
  // resident weight fragments per wave (4 VGPRs each): forward TPW x KS/2,
  // backward KW x NTU
  x.ok = x.TPW * x.KS / 2 <= 36 && x.KW * x.NTU <= 36 && x.TPW <= 3 && x.NTU <= 3;
  return x;
}

XShape xshape(int H, int B) {
  XShape x{};
  if (H % 64 != 0 || B < 1) return x;
  const char* e = getenv("AM_XCD_BLOCKS");
  const bool one = e && e[0] == '1' && e[1] == 0;
  if (one && B > 128 && B <= 256 && (H == 64 || H == 128 || H == 768)) {
    x = xshape_of(H, 2, 1, xcd_units(H, 32, 4));
    x.rounds = 1;
    return x;
  }
  // whole 16-unit tiles if the width has such slices, else whole 16-byte
  // chunks of the staged rows, else whole MFMA tiles of 4 units x 4 gates
  for (int bpx = B > 128 ? 2 : 1; bpx > 0 && !x.ok; --bpx)
    for (int step : {16, 8, 4}) {
      x = xshape_of(H, 1, bpx, xcd_units(H, 32 / bpx, step));
      if (x.ok) break;
    }
  x.rounds = (B + 128 * x.BPX - 1) / (128 * x.BPX);
  if (x.rounds > XCD_MAX_ROUNDS) x.ok = false;
  return x;
}

// A ragged batch of at most 1024 steps gets the active sequences of every step in
// place of the lengths, and the kernels built for that (COUNTS): each round's
// workgroups would walk all lengths, about 150 ns for every one.  Forward and
// backward of one layer, us, walking / reading: 1000 sequences x 768, 20 steps, 4
// rounds 1352 / 623; 1000 x 256, 20 steps, 1064 / 340; 492 x 384, 8 steps, 373 /
// 172.  (A kernel of its own: with both in one, uniform batches were 2 %
// slower.)  Longer ones walk: the lengths are few beside the steps.
bool count_steps(PersistSchedule& ps) {
  constexpr int MAX = (int)(sizeof ps.lens / sizeof ps.lens[0]);
  if (ps.varlen != 1 || ps.T > MAX) return false;
  uint16_t counts[MAX] = {};
  for (int t = 0, nb = ps.B; t < ps.T; ++t) {
    while (nb > 0 && (int)ps.lens[nb - 1] <= t) --nb;
    counts[t] = (uint16_t)nb;
  }
  memcpy(ps.lens, counts, sizeof counts);
  return true;
}

// The sequences of round r, and its slot of the sync area.
void xcd_round(const XShape& x, int r, PersistSchedule& ps, XcdSync& y) {
  ps.first = r * 128 * x.BPX;
  if (r > 0) {
    y.flags += XCD_SYNC_WORDS;
    y.xcc += XCD_SYNC_WORDS;
  }
}

}  // namespace

// AM_XCD_FENCED=1 in the environment: exchange with fences (as a block that
// spans XCDs does) even when every block sits on one XCD.
bool fenced_forced() {
  const char* e = getenv("AM_XCD_FENCED");
  return e && e[0] == '1' && e[1] == 0;
}

#define AM_FWD_CASE(MT_, KS_, TPW_, STG_)                                                \
  if (x.MT == MT_ && x.KS == KS_ && x.TPW == TPW_ && (x.U % 8 == 0) == STG_)             \
    e = coop(counts ? lstm_fwd_xcd<MT_, KS_, TPW_, STG_, true> : lstm_fwd_xcd<MT_, KS_, TPW_, STG_, false>, blocks, 512, lds, args, s, used);       \
  else

hipError_t lstm_fwd_xcd_launch(PersistFwd a, PersistSchedule ps, XcdSync y, hipStream_t s, bool* used) {
  *used = false;
  const XShape x = xshape(a.hidden, ps.B);
  if (!x.ok) return hipSuccess;
  y.units = x.U;
  y.fenced = fenced_forced() ? 1 : 0;
  const bool counts = count_steps(ps);
  const int blocks = NX * x.BPX * (a.hidden / x.U);
  // h rows, partial tiles, and (U % 8 == 0) the staged rows of C, Hs, G and h
  // and two steps' projections
  const size_t lds = (size_t)16 * x.MT * x.KS * 64 + 8 * ((x.TPW + 1) / 2) * 64 * 16 +
                     (x.U % 8 == 0 ? (size_t)16 * x.MT * (32 * x.U + 64) : 0);
  for (int r = 0; r < x.rounds; ++r) {
    xcd_round(x, r, ps, y);
    void* args[] = {&a, &ps, &y};
    hipError_t e = hipSuccess;
    // one block per XCD: 16 units up to H = 512, 32 beyond
    AM_FWD_CASE(1, 2, 1, true) AM_FWD_CASE(1, 4, 1, true) AM_FWD_CASE(1, 6, 1, true)
    AM_FWD_CASE(1, 8, 1, true)
    AM_FWD_CASE(1, 10, 1, true) AM_FWD_CASE(1, 12, 1, true) AM_FWD_CASE(1, 14, 1, true)
    AM_FWD_CASE(1, 16, 1, true) AM_FWD_CASE(1, 18, 2, true) AM_FWD_CASE(1, 20, 2, true)
    AM_FWD_CASE(1, 22, 2, true) AM_FWD_CASE(1, 24, 2, true) AM_FWD_CASE(1, 26, 2, true)
    AM_FWD_CASE(1, 28, 2, true) AM_FWD_CASE(1, 30, 2, true) AM_FWD_CASE(1, 32, 2, true)
    // two: 16 units up to H = 256 (above), 32 up to 512, then 48, 40 and 44
    AM_FWD_CASE(1, 10, 2, true) AM_FWD_CASE(1, 12, 2, true) AM_FWD_CASE(1, 14, 2, true)
    AM_FWD_CASE(1, 16, 2, true) AM_FWD_CASE(1, 18, 3, true) AM_FWD_CASE(1, 20, 3, true)
    AM_FWD_CASE(1, 22, 3, false) AM_FWD_CASE(1, 24, 3, true)
    AM_FWD_CASE(2, 2, 1, false) AM_FWD_CASE(2, 4, 1, false) AM_FWD_CASE(2, 24, 3, true)
    return hipSuccess;
    if (e != hipSuccess || !*used) return e;
  }
  return hipSuccess;
}

#define AM_BWD_CASE(MT_, NTU_, KW_)                                                       \
  if (x.MT == MT_ && x.NTU == NTU_ && x.KW == KW_) {                                     \
    lds = 8 * (size_t)bwd_wave_bytes(MT_, KW_);                                          \
    if (lds < red) lds = red;                                                            \
    e = coop(counts ? lstm_bwd_xcd<MT_, NTU_, KW_, true> : lstm_bwd_xcd<MT_, NTU_, KW_, false>, blocks, 512, lds, args, s, used);             \
  } else

hipError_t lstm_bwd_xcd_launch(PersistBwd a, PersistSchedule ps, XcdSync y, hipStream_t s, bool* used) {
  *used = false;
  const XShape x = xshape(a.hidden, ps.B);
  if (!x.ok) return hipSuccess;
  y.units = x.U;
  y.fenced = fenced_forced() ? 1 : 0;
  const bool counts = count_steps(ps);
  const int blocks = NX * x.BPX * (a.hidden / x.U);
  // the waves' private chunk buffers, or the partial products if larger
  const size_t red = (size_t)8 * x.MT * x.NTU * 64 * 16;
  for (int r = 0; r < x.rounds; ++r) {
    xcd_round(x, r, ps, y);
    void* args[] = {&a, &ps, &y};
    hipError_t e = hipSuccess;
    size_t lds = 0;
    // (the same unit slices as the forward's)
    AM_BWD_CASE(1, 1, 1) AM_BWD_CASE(1, 1, 2) AM_BWD_CASE(1, 1, 4) AM_BWD_CASE(1, 1, 5)
    AM_BWD_CASE(1, 1, 6) AM_BWD_CASE(1, 1, 7) AM_BWD_CASE(1, 1, 8) AM_BWD_CASE(1, 2, 9)
    AM_BWD_CASE(1, 2, 10) AM_BWD_CASE(1, 2, 11) AM_BWD_CASE(1, 2, 12) AM_BWD_CASE(1, 2, 13)
    AM_BWD_CASE(1, 2, 14) AM_BWD_CASE(1, 2, 15) AM_BWD_CASE(1, 2, 16)
    AM_BWD_CASE(1, 2, 5) AM_BWD_CASE(1, 2, 6) AM_BWD_CASE(1, 2, 7) AM_BWD_CASE(1, 2, 8)
    AM_BWD_CASE(1, 3, 9) AM_BWD_CASE(1, 3, 10) AM_BWD_CASE(1, 3, 11) AM_BWD_CASE(1, 3, 12)
    AM_BWD_CASE(2, 1, 1) AM_BWD_CASE(2, 1, 2) AM_BWD_CASE(2, 2, 12)
    return hipSuccess;
    if (e != hipSuccess || !*used) return e;
  }
  return hipSuccess;
}

// A launch costs about as much as four steps, so a batch that needs several
// rounds has to be long enough to pay for them (2 x 1024, 400 sequences in 4
// rounds: 2 steps 483 us a training step against 297 one launch per step; 512
// sequences, 20 steps: 2047 against 2303; 2 x 512, 400 in 2 rounds: 2 steps 243
// against 220); and where one launch per step is the other choice (beyond
// H = 768 no device-scope kernel fits) a single step is left to it (4 x 1024,
// 4 sequences: 115 against 88 us forward).
bool lstm_xcd_covers(int hidden, int B, int T) {
  const XShape x = xshape(hidden, B);
  if (!x.ok || (x.rounds > 1 && T < 4 * x.rounds)) return false;
  return T > 1 || hidden <= 768;
}

}  // namespace am
