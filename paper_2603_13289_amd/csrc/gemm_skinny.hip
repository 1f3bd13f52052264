// bf16 projection GEMM for very few rows (decoding: one row per sequence, M <= 32).
//
// With so few rows the product is bound by streaming the weights once from HBM, so the kernel is laid out for
// bytes in flight rather than for tile reuse: a workgroup of 8 wavefronts owns 16 output columns (16 weight
// rows); each wavefront takes one eighth of K and walks it in 32-element steps with one 16x16x32 MFMA per
// step (operands go straight from global memory into the MFMA lane layout: lane l holds row l % 16,
// elements 8 (l / 16) .. +7 of the step); the eight partial 16x16 tiles are added through LDS in a fixed
// order and the epilogue is applied.  Rows 16..31 use a second accumulator.
//
// A wavefront keeps two register sets of U steps and refills one while the other is multiplied, so loads are always
// in flight.  Loading a group of four steps, waiting for it and multiplying it left memory idle between groups: gate/up of
// 1 x 28672 x 4096 in a decoding step 47.4 -> 42.4 us (5.5 TB/s), of 16 rows 62.5 -> 47.7 us (their activation rows come from
// the L2, which the old loop waited for as well).
#include <type_traits>

#include "common.h"

namespace rc {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8s;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4s;

static constexpr int kSkinnyWaves = 8;
// Products of at most one workgroup per CU (256) take register sets of eight steps instead of four (128 KB in flight per
// workgroup): there are too few wavefronts to hide the latency otherwise.  They need two full sets in a wavefront's
// share of K: shorter ones (K below 4096) have nothing to pipeline.  With more workgroups, two have to fit a CU:
// sets of four steps in at most 128 registers (the line at 512 workgroups and 130 registers: a decoding step of one
// sequence on the 7B shape 4.23 ms, of sixteen 7.97; as it is 4.17 and 7.88).
static constexpr int kSkinnyDeepGroups = 256;

// Rows that a workgroup normalises for itself: at most four, in at most 48 KB of LDS (with the partial tiles two workgroups fit a
// compute unit), of at most 5120 elements.  A thread keeps its share of up to two rows and of the gains in registers, 1024 elements
// of a row at a time whatever its width: at 5120 gate/up of four rows needs 121 of the 128 registers that two workgroups leave, at
// 6144 it goes through scratch memory (16 bytes a lane), at 8192 q|k|v does as well.  One or two rows would fit up to 8192 (116
// registers for 100): not built, wider models have a norm launch of their own instead (4.7 us).
static constexpr int kNormRowMax = 5120;
static constexpr size_t kNormLds = 48 * 1024;
__device__ __host__ inline int norm_pitch(int k) { return 2 * k + 16; }   // bytes; rows start in different LDS banks
bool gemm_skinny_norm_fits(int m, int k) {
  return m <= kNormRows && k <= kNormRowMax && (size_t)m * norm_pitch(k) <= kNormLds;
}

// a barrier that waits for the LDS accesses before it, not for loads in flight as __syncthreads may
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ inline float silu_s(float x) { return x / (1.0f + __expf(-x)); }

// DUAL: gate (w) and up weights (w2) of the same columns.  TWO: more than 16 rows.  U: K steps of a register set.
// NORM: the rows, at most 2 NORM of them, are RMS-normalised on the way in (NormIn), in the order of rmsnorm_kernel, so that the
// operand has the same bits.  Every workgroup does it for itself, into LDS, while its first weights are on their way: what a row of
// 4096 costs (16 KB from the L2, a reduction) hides behind them and the launch of the norm kernel goes.
// One row, K = 4096: q|k|v 12.0 + norm 4.7 + rotary 5.5 -> 14.3 us, gate/up 42.2 + 4.7 -> 43.0, LM head (32768) 43 + norm and
// gather 10.3 -> 46.3.  More than four rows keep the norm's own launch: every workgroup would read and hold them all.
// ROPE: the columns are q, k and v heads of 128 (RopeOut), below ns1 of w, below ns2 of w2, the rest of w3; a workgroup has columns 8 j .. 8 j + 7 of both halves of a head, i.e.
// eight whole rotary pairs, and its epilogue does what rope_scatter_kernel does with a row, in the same arithmetic.
// WIDE: a workgroup owns 32 columns, as two sets of 16 (takes_wide).
template <bool DUAL, bool TWO, int U, int NORM, bool ROPE, bool WIDE>
__device__ __forceinline__ void few_rows_body(const bf16* __restrict__ a, const bf16* __restrict__ w, const bf16* __restrict__ w2,
                                              const bf16* __restrict__ w3, int ns1, int ns2, void* __restrict__ c, int m, int n, int k, int ldc,
                                              int epi, const int* __restrict__ m_live, const NormIn& norm, const RopeOut& rope) {
  static_assert(!(NORM > 0 && (TWO || WIDE)) && !(DUAL && (ROPE || WIDE)), "");
  constexpr bool SETS = DUAL || WIDE;   // two sets of 16 weight rows: gate and up, or neighbouring columns
  constexpr int TILES = (SETS ? 2 : 1) * (TWO ? 2 : 1), UP = TWO ? 2 : 1;   // tiles: first set rows 0-15 (16-31), second set rows 0-15 (16-31)
  constexpr int PAIRS = WIDE ? 16 : 8;   // ROPE: rotary pairs of a workgroup
  __shared__ float part[kSkinnyWaves][TILES][64][4];   // [wave][tile][lane][e]
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_rows[];   // NORM: [m][k] bf16, rows norm_pitch(k) bytes apart
  __shared__ float norm_red[NORM > 0 ? NORM : 1][kSkinnyWaves];
  __shared__ float2 lds_cs[ROPE ? 32 : 1][PAIRS];
  __shared__ unsigned lds_dst[ROPE ? 32 : 1];
  m = live_count(m, m_live);
  if (m <= 0) return;
  int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = (int)blockIdx.x * (WIDE ? 32 : 16);
  // ROPE: columns 0-7 and 8-15 of a set are partners, half a head apart; WIDE: the second set is the next eight pairs
  const int head = n0 >> 7, pair0 = (n0 & 127) >> 1;
  int dim = pair0 + (lane & 7) + 64 * ((lane >> 3) & 1);
  int col = ROPE ? head * 128 + dim : n0 + (lane & 15);
  const int kw = k / kSkinnyWaves;
  const size_t koff = (size_t)wave * kw + 8 * (lane >> 4);
  const bf16* pw;
  const bf16* pu = nullptr;
  if constexpr (ROPE) pw = (col < ns1 ? w + (size_t)col * k : (col < ns2 ? w2 + (size_t)(col - ns1) * k : w3 + (size_t)(col - ns2) * k)) + koff;
  else pw = w + (size_t)col * k + koff;
  if constexpr (DUAL) pu = w2 + (size_t)col * k + koff;
  else if constexpr (WIDE) pu = pw + (size_t)(ROPE ? 8 : 16) * k;   // of the same matrix: its columns are whole heads
  const bf16* pa0 = a + (size_t)min(lane & 15, m - 1) * k + koff;
  const bf16* pa1 = a + (size_t)min(16 + (lane & 15), m - 1) * k + koff;
  const unsigned char* la0 = lds_rows + (size_t)min(lane & 15, m - 1) * norm_pitch(k) + 2 * koff;
  f32x4s g0 = {0.f, 0.f, 0.f, 0.f}, g1 = g0, u0 = g0, u1 = g0;
  bf16x8s fb[2][U], fu[2][SETS ? U : 1], fa0[2][NORM > 0 ? 1 : U], fa1[2][TWO ? U : 1];
  const int steps = kw / 32;
  auto load = [&](auto set, int first, auto ragged) {   // ragged: some steps of the set may lie past the last one
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (decltype(ragged)::value && first + i >= steps) continue;
      const int o = 32 * (first + i);
      fb[S][i] = *reinterpret_cast<const bf16x8s*>(pw + o);
      if constexpr (SETS) fu[S][i] = *reinterpret_cast<const bf16x8s*>(pu + o);
      if constexpr (NORM == 0) fa0[S][i] = *reinterpret_cast<const bf16x8s*>(pa0 + o);
      if constexpr (TWO) fa1[S][i] = *reinterpret_cast<const bf16x8s*>(pa1 + o);
    }
  };
  auto multiply = [&](auto set, int live, int first) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (i >= live) continue;
      bf16x8s f;
      if constexpr (NORM > 0) f = *reinterpret_cast<const bf16x8s*>(la0 + 64 * (first + i));
      else f = fa0[S][i];
      g0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, fb[S][i], g0, 0, 0, 0);
      if constexpr (TWO) g1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa1[S][i], fb[S][i], g1, 0, 0, 0);
      if constexpr (SETS) {
        u0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, fu[S][i], u0, 0, 0, 0);
        if constexpr (TWO) u1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa1[S][i], fu[S][i], u1, 0, 0, 0);
      }
    }
  };

  // NORM: wavefronts 0-3 take row 0 (and 2), 4-7 row 1 (and 3); threads and order of the sum as in rmsnorm_kernel.  No condition
  // around the loads: elements past the row repeat its last ones, rows past the last one repeat it.
  constexpr int NK = NORM > 0 ? kNormRowMax / 1024 : 1, NP = NORM > 0 ? NORM : 1;
  float4 keep[NP][NK];
  uint2 gain[NK];
  const int nt = tid & 255;
  auto norm_load = [&]() {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const float* x = norm.h + (size_t)max(norm.row[min(2 * p + (wave >> 2), m - 1)], 0) * k;
#pragma unroll
      for (int u = 0; u < NK; ++u) keep[p][u] = *reinterpret_cast<const float4*>(x + min((nt + u * 256) * 4, k - 4));
    }
#pragma unroll
    for (int u = 0; u < NK; ++u) gain[u] = *reinterpret_cast<const uint2*>(norm.gain + min((nt + u * 256) * 4, k - 4));
  };
  auto norm_rows = [&]() {
    float ss[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const bool dead = norm.row[min(2 * p + (wave >> 2), m - 1)] < 0;   // uniform
      ss[p] = 0.f;
#pragma unroll
      for (int u = 0; u < NK; ++u) {
        float4& x = keep[p][u];
        // not touched, and so not waited for, ahead of this point: the weights are asked for first
        asm volatile("" : "+v"(x.x), "+v"(x.y), "+v"(x.z), "+v"(x.w));
        if (dead || (nt + u * 256) * 4 >= k) x = make_float4(0.f, 0.f, 0.f, 0.f);
        ss[p] = add_squares(ss[p], x);
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) ss[p] += __shfl_xor(ss[p], o, 64);
      if (lane == 0) norm_red[p][wave] = ss[p];
    }
    lds_barrier();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) s += norm_red[p][(wave & 4) + i];
      const float r = 1.0f / sqrtf(s / (float)k + norm.eps);
      const int row = 2 * p + (wave >> 2);
#pragma unroll
      for (int u = 0; u < NK; ++u) {
        const int e = (nt + u * 256) * 4;
        const float4 x = keep[p][u];
        uint2 pk;
        pk.x = (uint32_t)f32_to_bf16(x.x * r * __uint_as_float(gain[u].x << 16)).v |
               ((uint32_t)f32_to_bf16(x.y * r * __uint_as_float(gain[u].x & 0xffff0000u)).v << 16);
        pk.y = (uint32_t)f32_to_bf16(x.z * r * __uint_as_float(gain[u].y << 16)).v |
               ((uint32_t)f32_to_bf16(x.w * r * __uint_as_float(gain[u].y & 0xffff0000u)).v << 16);
        if (row < m && e < k) *reinterpret_cast<uint2*>(lds_rows + (size_t)row * norm_pitch(k) + 2 * e) = pk;
      }
    }
    lds_barrier();
  };
  // ROPE: thread PAIRS r + p fetches the angle of pair p of the tile for row r, and the row's place in the cache; they wait in LDS for
  // the epilogue.  Every wavefront asks: a load that only some have in flight would make the compiler wait for all.
  int rope_pos;
  unsigned rope_dst;
  float2 rope_cs;
  auto rope_load = [&]() {
    if constexpr (ROPE) {
      const int r = min(tid / PAIRS, m - 1);
      rope_pos = rope.row_pos[r];
      rope_dst = rope.row_dst[r];
    }
  };
  auto rope_angles = [&]() {
    if constexpr (ROPE) rope_cs = rope.tab[(size_t)rope_pos * 64 + pair0 + tid % PAIRS];
  };

  const std::integral_constant<int, 0> s0;
  const std::integral_constant<int, 1> s1;
  const std::false_type whole;
  const std::true_type tail;
  constexpr bool kRopeEarly = !TWO;   // with two row tiles the registers are needed: behind the main loop
  if constexpr (kRopeEarly) rope_load();
  if constexpr (NORM > 0) norm_load();
  __builtin_amdgcn_sched_barrier(0);
  int at = 0;
  if (steps >= 2 * U) {
    load(s0, 0, whole);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NORM == 0 || !DUAL) load(s1, U, whole);   // registers: behind the norm
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kRopeEarly) rope_angles();
    if constexpr (NORM > 0) norm_rows();
    if constexpr (NORM > 0 && DUAL) load(s1, U, whole);
    __builtin_amdgcn_sched_barrier(0);
    // no condition inside: a load that may or may not be in flight would make the compiler wait for all of them
    for (; at + 4 * U <= steps; at += 2 * U) {
      multiply(s0, U, at);
      __builtin_amdgcn_sched_barrier(0);
      load(s0, at + 2 * U, whole);
      __builtin_amdgcn_sched_barrier(0);
      multiply(s1, U, at + U);
      __builtin_amdgcn_sched_barrier(0);
      load(s1, at + 3 * U, whole);
      __builtin_amdgcn_sched_barrier(0);
    }
    multiply(s0, U, at);
    if (at + 2 * U < steps) load(s0, at + 2 * U, tail);
    multiply(s1, U, at + U);
    at += 2 * U;
  } else {
    load(s0, 0, tail);
    if constexpr (kRopeEarly) rope_angles();
    if constexpr (NORM > 0) norm_rows();
  }
  if (at < steps) {
    if (at + U < steps) load(s1, at + U, tail);
    multiply(s0, steps - at, at);
    if (at + U < steps) multiply(s1, steps - at - U, at + U);
  }
  if constexpr (ROPE && TWO) {
    // worked out again, and in another way: kept over the main loop they took three registers more than the 128 there are, which
    // went through scratch memory (q|k|v of 20 rows of 4096 in a decoding step: 21.0 us with and 20.9 without, of 32 rows 24.9)
    lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    tid = 64 * wave + lane;
    dim = pair0 + (lane & 7) + 64 * ((lane >> 3) & 1);
    col = head * 128 + dim;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    part[wave][0][lane][e] = g0[e];
    if constexpr (TWO) part[wave][1][lane][e] = g1[e];
    if constexpr (SETS) part[wave][UP][lane][e] = u0[e];
    if constexpr (SETS && TWO) part[wave][UP + 1][lane][e] = u1[e];
  }
  if constexpr (ROPE) {
    if constexpr (!kRopeEarly) {
      rope_load();
      rope_angles();
    }
    if (tid < 32 * PAIRS) {
      lds_cs[tid / PAIRS][tid % PAIRS] = rope_cs;
      if (tid % PAIRS == 0) lds_dst[tid / PAIRS] = rope_dst;
    }
  }
  __syncthreads();
  // wavefront 0 finishes rows 0-15, wavefront 1 rows 16-31; WIDE: of the first set, the next ones those of the second
  if (wave >= UP * (WIDE ? 2 : 1)) return;
  const int rows16 = WIDE ? wave % UP : wave, second = WIDE ? wave / UP : 0;
  if constexpr (WIDE) {
    dim += 8 * second;
    col += (ROPE ? 8 : 16) * second;
  }
  float gs[4] = {0.f, 0.f, 0.f, 0.f}, us[4] = {0.f, 0.f, 0.f, 0.f};
  for (int p = 0; p < kSkinnyWaves; ++p) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      gs[e] += part[p][wave][lane][e];
      if constexpr (DUAL) us[e] += part[p][UP + wave][lane][e];
    }
  }
  if constexpr (ROPE) {
    const bool is_q = col < ns1, is_v = col >= ns2;   // uniform
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float other = __shfl_xor(gs[e], 8, 64);
      const int row = rows16 * 16 + 4 * (lane >> 4) + e;
      if (row >= m) continue;
      const float2 cs = lds_cs[row][8 * second + (lane & 7)];
      const unsigned dst = lds_dst[row];
      float v = gs[e];
      if (!is_v) v = dim < 64 ? fmaf(v, cs.x, -(other * cs.y)) : fmaf(v, cs.x, other * cs.y);
      if (is_q) {
        rope.q[(size_t)row * ns1 + col] = f32_to_bf16(v);
      } else if (dst != kRowNoDst) {
        const int kvh = head - (is_v ? ns2 : ns1) / 128;
        const size_t o = ((size_t)dst + (size_t)kvh * rope.block_size) * 128 + dim;
        (is_v ? rope.v_pool : rope.k_pool)[o] = f32_to_bf16(v);
        if (!is_v && rope.k_pre_pool) rope.k_pre_pool[o] = f32_to_bf16(gs[e]);
      }
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int row = rows16 * 16 + 4 * (lane >> 4) + e;
    if (row >= m) continue;
    const size_t o = (size_t)row * ldc + col;
    if (DUAL) reinterpret_cast<bf16*>(c)[o] = f32_to_bf16(silu_s(gs[e]) * us[e]);
    else if (epi == EPI_STORE_F32) reinterpret_cast<float*>(c)[o] = gs[e];
    else if (epi == EPI_ADD_F32) reinterpret_cast<float*>(c)[o] += gs[e];
    else reinterpret_cast<bf16*>(c)[o] = f32_to_bf16(gs[e]);
  }
}

template <bool DUAL, bool TWO, int U, int NORM, bool ROPE>
__global__ void __launch_bounds__(kSkinnyWaves * 64, U == 8 || (DUAL && TWO) ? 2 : 4)
gemm_skinny_kernel(const bf16* __restrict__ a, const bf16* __restrict__ w, const bf16* __restrict__ w2,
                   const bf16* __restrict__ w3, int ns1, int ns2, void* __restrict__ c, int m, int n, int k, int ldc,
                   int epi, const int* __restrict__ m_live, NormIn norm, RopeOut rope) {
  few_rows_body<DUAL, TWO, U, NORM, ROPE, false>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, epi, m_live, norm, rope);
}

template <bool TWO, bool ROPE>
__global__ void __launch_bounds__(kSkinnyWaves * 64, 2)
gemm_wide_few_rows_kernel(const bf16* __restrict__ a, const bf16* __restrict__ w, const bf16* __restrict__ w2, const bf16* __restrict__ w3,
                          int ns1, int ns2, void* __restrict__ c, int m, int n, int k, int ldc, int epi, const int* __restrict__ m_live,
                          RopeOut rope) {
  few_rows_body<false, TWO, TWO ? 4 : 8, 0, ROPE, true>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, epi, m_live, NormIn{}, rope);
}

// Products of few rows whose K is no multiple of 256: summed in the K parts of the tile kernels' partition (`parts` of `part_steps`
// steps of 32 each, the last one shorter), a part by one wavefront, added up in the same workgroup: the bits of a tile launch and
// its sum over the parts, in one launch.  3 x 512 x 1408 (eleven parts) in a decoding step: 4.1 + 6.0 -> 4.9 us.
template <bool DUAL, bool TWO>
__global__ void __launch_bounds__(kSkinnyWaves * 64, 2)
gemm_few_rows_parts_kernel(const bf16* __restrict__ a, const bf16* __restrict__ w, const bf16* __restrict__ w2, void* __restrict__ c, int m,
                           int n, int k, int ldc, int epi, int parts, int part_steps) {
  constexpr int TILES = (DUAL ? 2 : 1) * (TWO ? 2 : 1), UP = TWO ? 2 : 1, U = 4;
  extern __shared__ __attribute__((aligned(16))) f32x4s lds_parts[];   // [part][tile][lane]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = (int)blockIdx.x * 16 + (lane & 15);
  const bf16* const pw = w + (size_t)col * k + 8 * (lane >> 4);
  const bf16* const pu = DUAL ? w2 + (size_t)col * k + 8 * (lane >> 4) : nullptr;
  const bf16* const pa0 = a + (size_t)min(lane & 15, m - 1) * k + 8 * (lane >> 4);
  const bf16* const pa1 = a + (size_t)min(16 + (lane & 15), m - 1) * k + 8 * (lane >> 4);
  for (int p = wave; p < parts; p += kSkinnyWaves) {
    f32x4s acc[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) acc[t] = f32x4s{0.f, 0.f, 0.f, 0.f};
    const int first = p * part_steps, last = min(first + part_steps, k / 32);
    for (int s0 = first; s0 < last; s0 += U) {
      bf16x8s fb[U], fu[DUAL ? U : 1], fa0[U], fa1[TWO ? U : 1];
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int o = 32 * min(s0 + i, last - 1);
        fb[i] = *reinterpret_cast<const bf16x8s*>(pw + o);
        if constexpr (DUAL) fu[i] = *reinterpret_cast<const bf16x8s*>(pu + o);
        fa0[i] = *reinterpret_cast<const bf16x8s*>(pa0 + o);
        if constexpr (TWO) fa1[i] = *reinterpret_cast<const bf16x8s*>(pa1 + o);
      }
#pragma unroll
      for (int i = 0; i < U; ++i) {
        if (s0 + i >= last) continue;   // uniform
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa0[i], fb[i], acc[0], 0, 0, 0);
        if constexpr (TWO) acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa1[i], fb[i], acc[1], 0, 0, 0);
        if constexpr (DUAL) acc[UP] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa0[i], fu[i], acc[UP], 0, 0, 0);
        if constexpr (DUAL && TWO) acc[UP + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa1[i], fu[i], acc[UP + 1], 0, 0, 0);
      }
    }
#pragma unroll
    for (int t = 0; t < TILES; ++t) lds_parts[(p * TILES + t) * 64 + lane] = acc[t];
  }
  __syncthreads();
  if (wave > (TWO ? 1 : 0)) return;
  f32x4s gs = {0.f, 0.f, 0.f, 0.f}, us = gs;
  for (int p = 0; p < parts; ++p) {
    gs += lds_parts[(p * TILES + wave) * 64 + lane];
    if constexpr (DUAL) us += lds_parts[(p * TILES + UP + wave) * 64 + lane];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int row = wave * 16 + 4 * (lane >> 4) + e;
    if (row >= m) continue;
    const size_t o = (size_t)row * ldc + col;
    if (DUAL) reinterpret_cast<bf16*>(c)[o] = f32_to_bf16(silu_s(gs[e]) * us[e]);
    else if (epi == EPI_STORE_F32) reinterpret_cast<float*>(c)[o] = gs[e];
    else if (epi == EPI_ADD_F32) reinterpret_cast<float*>(c)[o] += gs[e];
    else reinterpret_cast<bf16*>(c)[o] = f32_to_bf16(gs[e]);
  }
}

hipError_t launch_gemm_few_rows_parts(const bf16* a, const bf16* w, const bf16* w2, void* c, int m, int n, int k, int ldc, GemmEpilogue epi,
                                      int parts, int part_steps, hipStream_t st) {
  auto go = [&](auto dual, auto two) {
    const size_t lds = (size_t)parts * (decltype(dual)::value ? 2 : 1) * (decltype(two)::value ? 2 : 1) * 64 * sizeof(f32x4s);
    gemm_few_rows_parts_kernel<decltype(dual)::value, decltype(two)::value><<<dim3((unsigned)(n / 16)), kSkinnyWaves * 64, lds, st>>>(
        a, w, w2, c, m, n, k, ldc, (int)epi, parts, part_steps);
  };
  auto rows = [&](auto dual) {
    if (m > 16) go(dual, std::true_type{});
    else go(dual, std::false_type{});
  };
  if (epi == EPI_SWIGLU_T) rows(std::true_type{});
  else rows(std::false_type{});
  return hipGetLastError();
}

bool gemm_skinny_applies(int m, int n, int k) { return m >= 1 && m <= 32 && n % 16 == 0 && k % (kSkinnyWaves * 32) == 0; }

// Workgroups of 32 columns.  Every workgroup reads all rows of activations, from the L2; half as many workgroups read half as much, but
// have half the wavefronts to keep weights coming.  Gain over 16 columns each, weights from HBM, K = 4096 to 14336:
//   up to 4096 columns (one round of 16-column workgroups)    0.62 to 0.84x: half the chip idle
//   4608 (144 wide workgroups)                                1.07 to 1.46x from 5 rows on; left to the old form
//   5120 to 7168 (a second, uneven round of narrow ones)      from 5 rows on 1.003 to 1.46x with K > 4096, with K = 4096 0.999 to 1.13x at 5 rows,
//                                                             1.14x and more from 12 on
//   8192 to 32768 (at least 256 wide ones, rounds of either   at 5 rows 0.75 to 1.03x; at 24 and 32 rows 1.02 to 1.40x, the least of it at 9216 to
//   form even or not)                                         12288 (1.02 to 1.11x), where the last round of both is uneven
// 5120 x 27648, 5 / 16 / 32 rows: 73.0 / 98.5 / 146 -> 64.6 / 78.2 / 99.3 us.  The line lies where no size of these lost.
static bool takes_wide(int m, int n, int k) {
  const int wgs = n / 32;
  if (n % 32 != 0 || k < kSkinnyWaves * 32 * 16 || wgs < 160) return false;
  return m >= (wgs < kSkinnyDeepGroups ? (k > 4096 ? 5 : 12) : 24);
}

hipError_t launch_gemm_skinny_bf16(const bf16* a, const bf16* w, const bf16* w2, void* c, int m, int n, int k, int ldc, GemmEpilogue epi,
                                   hipStream_t st, const int* m_live) {
  const dim3 grid((unsigned)(n / 16));
  auto go = [&](auto dual, auto two, auto u) {
    gemm_skinny_kernel<decltype(dual)::value, decltype(two)::value, decltype(u)::value, 0, false>
        <<<grid, kSkinnyWaves * 64, 0, st>>>(a, w, w2, nullptr, 0, 0, c, m, n, k, ldc, (int)epi, m_live, NormIn{}, RopeOut{});
  };
  auto rows = [&](auto dual, auto u) {
    if (m > 16) go(dual, std::true_type{}, u);
    else go(dual, std::false_type{}, u);
  };
  const std::integral_constant<int, 4> u4;
  const std::integral_constant<int, 8> u8;
  if (epi != EPI_SWIGLU_T && takes_wide(m, n, k)) {
    (m > 16 ? gemm_wide_few_rows_kernel<true, false> : gemm_wide_few_rows_kernel<false, false>)<<<dim3((unsigned)(n / 32)), kSkinnyWaves * 64, 0, st>>>(
        a, w, w2, nullptr, 0, 0, c, m, n, k, ldc, (int)epi, m_live, RopeOut{});
    return hipGetLastError();
  }
  if (epi == EPI_SWIGLU_T) rows(std::true_type{}, u4);
  else if (n <= 16 * kSkinnyDeepGroups && k >= kSkinnyWaves * 32 * 16) rows(std::false_type{}, u8);
  else rows(std::false_type{}, u4);
  return hipGetLastError();
}

hipError_t launch_gemm_skinny_normed(const NormIn& norm, const bf16* w, const bf16* w2, void* c, int m, int n, int k,
                                     GemmEpilogue epi, hipStream_t st, const int* m_live) {
  const dim3 grid((unsigned)(n / 16));
  auto go = [&](auto dual, auto passes) {
    gemm_skinny_kernel<decltype(dual)::value, false, 4, decltype(passes)::value, false>
        <<<grid, kSkinnyWaves * 64, (size_t)m * norm_pitch(k), st>>>(nullptr, w, w2, nullptr, 0, 0, c, m, n, k, n, (int)epi, m_live, norm,
                                                                    RopeOut{});
  };
  auto rows = [&](auto dual) {
    if (m > 2) go(dual, std::integral_constant<int, 2>{});
    else go(dual, std::integral_constant<int, 1>{});
  };
  if (epi == EPI_SWIGLU_T) rows(std::true_type{});
  else rows(std::false_type{});
  return hipGetLastError();
}

hipError_t launch_gemm_skinny_qkv_rope(const bf16* a, const NormIn& norm, const bf16* wq, int nq, const bf16* wk, const bf16* wv, int nkv,
                                       int m, int k, const RopeOut& rope, hipStream_t st, const int* m_live) {
  const int n = nq + 2 * nkv;
  const dim3 grid((unsigned)(n / 16));
  auto go = [&](auto two, auto passes) {
    gemm_skinny_kernel<false, decltype(two)::value, 4, decltype(passes)::value, true>
        <<<grid, kSkinnyWaves * 64, norm.h ? (size_t)m * norm_pitch(k) : 0, st>>>(a, wq, wk, wv, nq, nq + nkv, nullptr, m, n, k, n,
                                                                                 (int)EPI_STORE_T, m_live, norm, rope);
  };
  if (!norm.h && takes_wide(m, n, k)) {   // q, k and v are whole heads of 128 columns
    (m > 16 ? gemm_wide_few_rows_kernel<true, true> : gemm_wide_few_rows_kernel<false, true>)<<<dim3((unsigned)(n / 32)), kSkinnyWaves * 64, 0, st>>>(
        a, wq, wk, wv, nq, nq + nkv, nullptr, m, n, k, n, (int)EPI_STORE_T, m_live, rope);
    return hipGetLastError();
  }
  if (norm.h && m > 2) go(std::false_type{}, std::integral_constant<int, 2>{});
  else if (norm.h) go(std::false_type{}, std::integral_constant<int, 1>{});
  else if (m > 16) go(std::true_type{}, std::integral_constant<int, 0>{});
  else go(std::false_type{}, std::integral_constant<int, 0>{});
  return hipGetLastError();
}

}  // namespace rc
