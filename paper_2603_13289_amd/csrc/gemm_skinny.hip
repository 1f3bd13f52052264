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

__device__ inline float silu_s(float x) { return x / (1.0f + __expf(-x)); }

// DUAL: gate and up weights of the same columns.  TWO: more than 16 rows.  U: K steps of a register set.
template <bool DUAL, bool TWO, int U>
__global__ void __launch_bounds__(kSkinnyWaves * 64, U == 8 || (DUAL && TWO) ? 2 : 4)
gemm_skinny_kernel(const bf16* __restrict__ a, const bf16* __restrict__ w, const bf16* __restrict__ w2,
                   const bf16* __restrict__ w3, int ns1, int ns2, void* __restrict__ c, int m, int n, int k, int ldc,
                   int epi, const int* __restrict__ m_live) {
  __shared__ float part[kSkinnyWaves][4][64][4];   // [wave][tile: gate/rows 0-15, gate/16-31, up/0-15, up/16-31][lane][e]
  m = live_count(m, m_live);
  if (m <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = (int)blockIdx.x * 16;
  const int col = n0 + (lane & 15);
  const int kw = k / kSkinnyWaves;
  const size_t koff = (size_t)wave * kw + 8 * (lane >> 4);
  const bf16* pw;
  const bf16* pu = nullptr;
  if (DUAL) {
    pw = w + (size_t)col * k + koff;
    pu = w2 + (size_t)col * k + koff;
  } else {
    pw = (col < ns1 ? w + (size_t)col * k : (col < ns2 ? w2 + (size_t)(col - ns1) * k : w3 + (size_t)(col - ns2) * k)) + koff;
  }
  const bf16* pa0 = a + (size_t)min(lane & 15, m - 1) * k + koff;
  const bf16* pa1 = a + (size_t)min(16 + (lane & 15), m - 1) * k + koff;
  f32x4s g0 = {0.f, 0.f, 0.f, 0.f}, g1 = g0, u0 = g0, u1 = g0;
  bf16x8s fb[2][U], fu[2][DUAL ? U : 1], fa0[2][U], fa1[2][TWO ? U : 1];
  const int steps = kw / 32;
  auto load = [&](auto set, int first, auto ragged) {   // ragged: some steps of the set may lie past the last one
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (decltype(ragged)::value && first + i >= steps) continue;
      const int o = 32 * (first + i);
      fb[S][i] = *reinterpret_cast<const bf16x8s*>(pw + o);
      if constexpr (DUAL) fu[S][i] = *reinterpret_cast<const bf16x8s*>(pu + o);
      fa0[S][i] = *reinterpret_cast<const bf16x8s*>(pa0 + o);
      if constexpr (TWO) fa1[S][i] = *reinterpret_cast<const bf16x8s*>(pa1 + o);
    }
  };
  auto multiply = [&](auto set, int live) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (i >= live) continue;
      g0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa0[S][i], fb[S][i], g0, 0, 0, 0);
      if constexpr (TWO) g1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa1[S][i], fb[S][i], g1, 0, 0, 0);
      if constexpr (DUAL) {
        u0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa0[S][i], fu[S][i], u0, 0, 0, 0);
        if constexpr (TWO) u1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa1[S][i], fu[S][i], u1, 0, 0, 0);
      }
    }
  };
  const std::integral_constant<int, 0> s0;
  const std::integral_constant<int, 1> s1;
  const std::false_type whole;
  const std::true_type tail;
  int at = 0;
  if (steps >= 2 * U) {
    load(s0, 0, whole);
    __builtin_amdgcn_sched_barrier(0);
    load(s1, U, whole);
    __builtin_amdgcn_sched_barrier(0);
    // no condition inside: a load that may or may not be in flight would make the compiler wait for all of them
    for (; at + 4 * U <= steps; at += 2 * U) {
      multiply(s0, U);
      __builtin_amdgcn_sched_barrier(0);
      load(s0, at + 2 * U, whole);
      __builtin_amdgcn_sched_barrier(0);
      multiply(s1, U);
      __builtin_amdgcn_sched_barrier(0);
      load(s1, at + 3 * U, whole);
      __builtin_amdgcn_sched_barrier(0);
    }
    multiply(s0, U);
    if (at + 2 * U < steps) load(s0, at + 2 * U, tail);
    multiply(s1, U);
    at += 2 * U;
  } else {
    load(s0, 0, tail);
  }
  if (at < steps) {
    if (at + U < steps) load(s1, at + U, tail);
    multiply(s0, steps - at);
    if (at + U < steps) multiply(s1, steps - at - U);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    part[wave][0][lane][e] = g0[e];
    if (TWO) part[wave][1][lane][e] = g1[e];
    if (DUAL) part[wave][2][lane][e] = u0[e];
    if (DUAL && TWO) part[wave][3][lane][e] = u1[e];
  }
  __syncthreads();
  // wavefront 0 finishes rows 0-15, wavefront 1 rows 16-31
  if (wave > (TWO ? 1 : 0)) return;
  float gs[4] = {0.f, 0.f, 0.f, 0.f}, us[4] = {0.f, 0.f, 0.f, 0.f};
  for (int p = 0; p < kSkinnyWaves; ++p) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      gs[e] += part[p][wave][lane][e];
      if (DUAL) us[e] += part[p][2 + wave][lane][e];
    }
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

bool gemm_skinny_applies(int m, int n, int k, int ns1, int ns2) {
  return m >= 1 && m <= 32 && n % 16 == 0 && k % (kSkinnyWaves * 32) == 0 && ns1 % 16 == 0 && ns2 % 16 == 0;
}

hipError_t launch_gemm_skinny_bf16(const bf16* a, const bf16* w, const bf16* w2, const bf16* w3, int ns1, int ns2,
                                   void* c, int m, int n, int k, int ldc, GemmEpilogue epi, hipStream_t st,
                                   const int* m_live) {
  const dim3 grid((unsigned)(n / 16));
  auto go = [&](auto dual, auto two, auto u) {
    gemm_skinny_kernel<decltype(dual)::value, decltype(two)::value, decltype(u)::value>
        <<<grid, kSkinnyWaves * 64, 0, st>>>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, (int)epi, m_live);
  };
  auto rows = [&](auto dual, auto u) {
    if (m > 16) go(dual, std::true_type{}, u);
    else go(dual, std::false_type{}, u);
  };
  const std::integral_constant<int, 4> u4;
  const std::integral_constant<int, 8> u8;
  if (epi == EPI_SWIGLU_T) rows(std::true_type{}, u4);
  else if (n <= 16 * kSkinnyDeepGroups && k >= kSkinnyWaves * 32 * 16) rows(std::false_type{}, u8);
  else rows(std::false_type{}, u4);
  return hipGetLastError();
}

}  // namespace rc
