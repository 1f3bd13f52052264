// The main loop of the large bf16 GEMM tiles: C tile [BM][BN] = A [BM][K] * W [BN][K]^T, K step 64, eight wavefronts.
//
// What bounds it: a K step of a 256x256 tile is 2048 matrix-pipe cycles per SIMD, 1536 cycles of LDS reads and 512 of
// direct-to-LDS writes, so the loop is at the chip's power limit when all three run side by side and far from it
// when they take turns.  The arrangement below keeps them side by side:
//   * A wavefront owns a WTM x WTN sub-tile, cut into two halves of its rows (A0, A1) and of its columns (B0, B1).
//     A K step is the four phases A0*B0, A0*B1, A1*B1, A1*B0: a phase reuses one operand half of the phase before
//     and reads the operands of the next phase from LDS between its own matrix instructions.
//   * LDS holds two K steps.  The LDS rows of an operand half (over all wavefronts) are refilled as soon as all
//     wavefronts have read them, i.e. up to two K steps before they are needed: unit order A0, B0 | B1, A1.  The
//     loads therefore stay in flight for 1.5 K steps and are counted (s_waitcnt vmcnt(n), never 0 in the loop).
//   * Two barriers per K step, before phases 0 and 2.
// LDS reads are inline assembly, because the compiler would otherwise wait for all direct-to-LDS loads before every
// LDS read; each phase starts with a wait that names the fragments it is about to use.  The compiler takes a fragment as
// there from its read on, so between the two it must neither move nor spill it: no tile type may run out of registers
// (tests/test_gemm_code.py reads the generated code for both; a spill would also wait for every load in flight).
// Measured on 5120 x 28672 x 4096 with random operands: 1370-1390 TFLOP/s against 1200-1210 for a loop with one
// barrier and one full wait per K step (1710 with operands of zeros, which draw less power).
#pragma once

#include <type_traits>

#include "common.h"

namespace rc {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 pipe_bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float pipe_f32x4;

// Wavefronts are arranged WM x WN; FM0 + FM1 row blocks and FN0 + FN1 column blocks of 16 per wavefront (FM1 = 0: low
// tiles, whose phases 2 and 3 only read the next step's operands).
template <int WM_, int WN_, int FM0_, int FM1_, int FN0_, int FN1_>
struct PipeTile {
  static constexpr int WM = WM_, WN = WN_, FM0 = FM0_, FM1 = FM1_, FN0 = FN0_, FN1 = FN1_;
  static constexpr int FM = FM0 + FM1, FN = FN0 + FN1;
  static constexpr int WTM = 16 * FM, WTN = 16 * FN, BM = WM * WTM, BN = WN * WTN;
  static constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128;
  static constexpr int LDS_BYTES = 2 * (A_BYTES + B_BYTES);
  // 1 KB loads per wavefront of each operand half
  static constexpr int LA0 = WM * FM0 / 4, LA1 = WM * FM1 / 4, LB0 = WN * FN0 / 4, LB1 = WN * FN1 / 4;
  static_assert(WM * WN == 8, "eight wavefronts");
  static_assert(LA0 * 4 == WM * FM0 && LA1 * 4 == WM * FM1 && LB0 * 4 == WN * FN0 && LB1 * 4 == WN * FN1,
                "an operand half is a whole number of loads per wavefront");
  static_assert(FN1 > 0 && FM0 > 0 && FN0 >= FN1, "phases 0 and 1 multiply");
  static_assert(A_BYTES <= 32768 && B_BYTES <= 32768, "LDS read offsets are 16-bit");
};

// What the columns of a tile are.  kPlain: BN neighbours.  The paired modes give every wavefront both members of BN / 2 / WN pairs,
// in column blocks j and j + FN / 2.  kDual: gate (w) and up projection (w2) of an output column.  kRope: rotary partners, columns
// i and i + 64 of a head of 128; pair p is column i = p % 64 of head p / 64.
enum GemmMode : int { kPlain = 0, kDual = 1, kRope = 2 };
__device__ __host__ inline int rope_column(int pair, int second) { return (pair >> 6) * 128 + (pair & 63) + 64 * second; }

// A loads [k_begin, k_end) of rows m0.. of a (clamped to the last row) and columns (paired modes: pairs) n0.. of the weights, of
// which there are n; weight rows of the output columns below ns1 come from w, below ns2 from w2, the rest from w3
// (boundaries are multiples of 8).
// acc (i, j): rows wm * WTM + 16 i + lane % 16, columns 16 j + 4 (lane / 16) + 0..3 of the wavefront's sub-tile.
// LANE_ID: the lane number is worked out in another way, so that a kernel with two such loops shares no value between them that
// would stay in registers.
template <typename T, int MODE, bool LANE_ID = false>
__device__ __forceinline__ void gemm_pipe_loop(const bf16* __restrict__ a, const bf16* __restrict__ w,
                                               const bf16* __restrict__ w2, const bf16* __restrict__ w3, int ns1, int ns2,
                                               int m, int n, int k, int m0, int n0, int k_begin, int k_end,
                                               unsigned char* lds, pipe_f32x4 (&acc)[T::FM][T::FN]) {
  static_assert(MODE == kPlain || T::FN % 2 == 0, "blocks of pairs");
  constexpr int FM0 = T::FM0, FM1 = T::FM1, FN0 = T::FN0, FN1 = T::FN1, FMX = FM0 > FM1 ? FM0 : FM1, FNX = FN0 > FN1 ? FN0 : FN1;
  constexpr int LAX = T::LA0 > T::LA1 ? T::LA0 : T::LA1, LBX = T::LB0 > T::LB1 ? T::LB0 : T::LB1;
  const int tid = threadIdx.x;
  const int lane = LANE_ID ? __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) : tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::WN, wn = wave % T::WN;
  const int lrow = lane >> 3, lslot = lane & 7;

  // ---- loads: the i-th load of an operand half covers 8 LDS rows; chunk c of LDS row r sits at slot c ^ ((r >> 1) & 7)
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)(a + (size_t)m0 * k), 0, -1, 0x00020000);
  int va[2][LAX], la[2][LAX], vb[2][LBX], lb[2][LBX];
  const bf16* pb[2][LBX];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < (h ? T::LA1 : T::LA0); ++i) {
      const int per = 2 * (h ? FM1 : FM0), blk = wave + 8 * i;     // 8-row blocks per wavefront row
      const int r = (blk / per) * T::WTM + h * FM0 * 16 + (blk % per) * 8;
      va[h][i] = min(r + lrow, m - 1 - m0) * k * 2 + ((lslot ^ (((r + lrow) >> 1) & 7)) << 4);
      la[h][i] = r * 128;
    }
#pragma unroll
    for (int i = 0; i < (h ? T::LB1 : T::LB0); ++i) {
      const int per = 2 * (h ? FN1 : FN0), blk = wave + 8 * i;
      const int wn_i = blk / per, rr = (blk % per) * 8;
      const int r = wn_i * T::WTN + h * FN0 * 16 + rr;
      constexpr int FH = T::FN / 2;
      const int j = h * FN0 + rr / 16, second = j >= FH ? 1 : 0;
      const int unit = MODE == kPlain ? n0 + r : n0 + wn_i * FH * 16 + (j - second * FH) * 16 + rr % 16;   // column or pair
      const int u0 = min(unit, n - 1), c0 = MODE == kRope ? rope_column(min(unit, n - 8), second) : u0;
      const bf16* src;
      if (MODE == kDual) src = (second ? w2 : w) + (size_t)c0 * k;
      else src = c0 < ns1 ? w + (size_t)c0 * k : (c0 < ns2 ? w2 + (size_t)(c0 - ns1) * k : w3 + (size_t)(c0 - ns2) * k);
      pb[h][i] = src;
      vb[h][i] = (MODE == kRope ? lrow : min(unit + lrow, n - 1) - u0) * k * 2 + ((lslot ^ (((r + lrow) >> 1) & 7)) << 4);
      lb[h][i] = 2 * T::A_BYTES + r * 128;
    }
  }
  const int k_last = k_end - 64;   // past it, loads repeat the last step (their results are not used)
  auto load_a = [&](int h, int buf, int k0) {
    const int ko = min(k0, k_last) * 2;
#pragma unroll
    for (int i = 0; i < (h ? T::LA1 : T::LA0); ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)(lds + la[h][i] + buf * T::A_BYTES),
                                               16, va[h][i], ko, 0, 0);
  };
  auto load_b = [&](int h, int buf, int k0) {
    const int ko = min(k0, k_last) * 2;
#pragma unroll
    for (int i = 0; i < (h ? T::LB1 : T::LB0); ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)pb[h][i], 0, -1, 0x00020000),
                                               (__attribute__((address_space(3))) void*)(lds + lb[h][i] + buf * T::B_BYTES),
                                               16, vb[h][i], ko, 0, 0);
  };

  // ---- LDS reads: lane % 16 is the row of a block, lane / 16 the 8-k chunk; k sub-step 1 is chunk ^ 4
  const int r16 = lane & 15, kq = lane >> 4;
  const unsigned sw = (unsigned)((kq ^ ((r16 >> 1) & 7)) << 4);
  const unsigned a_rd[2] = {(unsigned)((wm * T::WTM + r16) * 128) + sw, (unsigned)((wm * T::WTM + r16) * 128) + (sw ^ 64u)};
  const unsigned b_rd[2] = {2 * T::A_BYTES + (unsigned)((wn * T::WTN + r16) * 128) + sw,
                            2 * T::A_BYTES + (unsigned)((wn * T::WTN + r16) * 128) + (sw ^ 64u)};
  pipe_bf16x8 fa[2][2][FMX], fb[2][2][FNX];   // [half of A | register slot of B][k sub-step][block]
#define RC_LDS_READ(dst, addr, off) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off))
  // reads [r0, r1) of a half, in order (sub-step, block)
  auto read_a = [&](int h, int buf, int r0, int r1) {
    const int f = h ? FM1 : FM0;
#pragma unroll
    for (int r = 0; r < 2 * FMX; ++r)
      if (r >= r0 && r < r1 && r < 2 * f) RC_LDS_READ(fa[h][r / f][r % f], a_rd[r / f], buf * T::A_BYTES + (h * FM0 + r % f) * 2048);
  };
  auto read_b = [&](int slot, int h, int buf, int r0, int r1) {
    const int f = h ? FN1 : FN0;
#pragma unroll
    for (int r = 0; r < 2 * FNX; ++r)
      if (r >= r0 && r < r1 && r < 2 * f) RC_LDS_READ(fb[slot][r / f][r % f], b_rd[r / f], buf * T::B_BYTES + (h * FN0 + r % f) * 2048);
  };
  // A wait that the named fragments depend on: their uses cannot be scheduled ahead of it.
  auto tie_a = [&](int h) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < (h ? FM1 : FM0); ++i) asm volatile("" : "+v"(fa[h][s][i]));
  };
  auto tie_b = [&](int slot, int h) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int j = 0; j < (h ? FN1 : FN0); ++j) asm volatile("" : "+v"(fb[slot][s][j]));
  };
#define RC_FENCE __builtin_amdgcn_sched_barrier(0)
  // matrix instructions [q0, q1) of a phase, in order (sub-step, row block, column block)
  auto multiply = [&](int ah, int slot, int nh, int q0, int q1) {
    const int fm = ah ? FM1 : FM0, fn = nh ? FN1 : FN0;
#pragma unroll
    for (int q = 0; q < 2 * FMX * FNX; ++q) {
      if (q < q0 || q >= q1 || q >= 2 * fm * fn) continue;
      const int s = q / (fm * fn), i = (q / fn) % fm, j = q % fn;
      pipe_f32x4& c = acc[ah * FM0 + i][nh * FN0 + j];
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[slot][s][j], fa[ah][s][i], c, 0, 0, 0);
    }
  };

#pragma unroll
  for (int i = 0; i < T::FM; ++i)
#pragma unroll
    for (int j = 0; j < T::FN; ++j) acc[i][j] = pipe_f32x4{0.f, 0.f, 0.f, 0.f};

  constexpr int L01 = T::LA0 + T::LB0, L23 = T::LB1 + T::LA1, LALL = L01 + L23;
  // Loads that may still be in flight at a barrier: those issued after the operands the next two phases read.
  load_a(0, 0, k_begin); load_b(0, 0, k_begin); load_b(1, 0, k_begin); load_a(1, 0, k_begin);
  load_a(0, 1, k_begin + 64); load_b(0, 1, k_begin + 64); load_b(1, 1, k_begin + 64); load_a(1, 1, k_begin + 64);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L23 + LALL) : "memory");
  __builtin_amdgcn_s_barrier();
  read_a(0, 0, 0, 2 * FM0);
  read_b(0, 0, 0, 0, 2 * FN0);

  // One K step on buffer P; the weights' half 0 is in register slot P.  STAGE 0: in the loop; 1: last but one step; 2: last.
  auto step = [&](auto P_, auto STAGE_, int k0) {
    constexpr int P = decltype(P_)::value, STAGE = decltype(STAGE_)::value, Q = 1 - P;
    constexpr int M00 = 2 * FM0 * FN0, M01 = 2 * FM0 * FN1, M11 = 2 * FM1 * FN1, M10 = 2 * FM1 * FN0;
    // phase 0: A0 * B0; reads B1 of this step; refills A0
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(STAGE == 2 ? 0 : LALL) : "memory");
    tie_a(0); tie_b(P, 0);
    RC_FENCE; __builtin_amdgcn_s_barrier(); RC_FENCE;
    if constexpr (STAGE == 0) load_a(0, P, k0 + 128);
#pragma unroll
    for (int r = 0; r < FN1; ++r) {
      read_b(Q, 1, P, 2 * r, 2 * r + 2);
      RC_FENCE; multiply(0, P, 0, 4 * r, r + 1 == FN1 ? M00 : 4 * r + 4); RC_FENCE;
    }
    // phase 1: A0 * B1; reads A1; refills B0
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    tie_b(Q, 1);
    RC_FENCE;
    if constexpr (STAGE == 0) load_b(0, P, k0 + 128);
    RC_FENCE;
    constexpr int RA1 = FM1 > 0 ? FM1 : 1;            // pairs of reads
#pragma unroll
    for (int r = 0; r < RA1; ++r) {
      read_a(1, P, 2 * r, 2 * r + 2);
      RC_FENCE; multiply(0, Q, 1, r * M01 / (2 * RA1), r + 1 == RA1 ? M01 : (r + 1) * M01 / (2 * RA1)); RC_FENCE;
    }
    // phase 2: A1 * B1; reads most of A0 of the next step; refills B1
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(STAGE == 2 ? 63 : STAGE == 1 ? L23 : LALL) : "memory");
    tie_a(1);
    RC_FENCE;
    if constexpr (STAGE != 2) __builtin_amdgcn_s_barrier();
    RC_FENCE;
    if constexpr (STAGE == 0) load_b(1, P, k0 + 128);
    RC_FENCE;
    constexpr int RA2 = (2 * FM0 * 3 / 4 + 1) / 2;   // pairs of reads in phase 2
#pragma unroll
    for (int r = 0; r < RA2; ++r) {
      if constexpr (STAGE != 2) read_a(0, Q, 2 * r, 2 * r + 2);
      RC_FENCE; multiply(1, Q, 1, r * M11 / (2 * RA2), r + 1 == RA2 ? M11 : (r + 1) * M11 / (2 * RA2)); RC_FENCE;
    }
    // phase 3: A1 * B0; reads the rest of A0 and B0 of the next step (into B1's registers); refills A1
    if constexpr (STAGE == 0) load_a(1, P, k0 + 128);
    RC_FENCE;
    if constexpr (STAGE != 2) read_a(0, Q, 2 * RA2, 2 * FM0);
    RC_FENCE; multiply(1, P, 0, 0, 2); RC_FENCE;
#pragma unroll
    for (int r = 0; r < FN0; ++r) {
      if constexpr (STAGE != 2) read_b(Q, 0, Q, 2 * r, 2 * r + 2);
      RC_FENCE; multiply(1, P, 0, 2 + 4 * r, r + 1 == FN0 ? M10 : 6 + 4 * r); RC_FENCE;
    }
  };
  const std::integral_constant<int, 0> i0;
  const std::integral_constant<int, 1> i1;
  const std::integral_constant<int, 2> i2;
  const int k_pair = k_begin + ((k_end - k_begin + 127) & ~127);   // an odd number of steps ends with an empty one
  int k0 = k_begin;
  for (; k0 + 128 < k_pair; k0 += 128) {
    step(i0, i0, k0);
    step(i1, i0, k0 + 64);
  }
  step(i0, i1, k0);
  if (k0 + 64 < k_end) {
    step(i1, i2, k0 + 64);
  } else {   // the loads and reads of the empty step, whose registers are not free before this
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int i = 0; i < FM0; ++i) asm volatile("" ::"v"(fa[0][s][i]));
#pragma unroll
      for (int j = 0; j < FN0; ++j) asm volatile("" ::"v"(fb[1][s][j]));
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // nothing left to wait for; says so on every path of the code
#undef RC_LDS_READ
#undef RC_FENCE
}

}  // namespace rc
