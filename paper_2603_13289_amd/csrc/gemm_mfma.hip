// K3: projection GEMMs of the active rows on the matrix cores (bf16 in, float accumulate).
//
//   C[M][N] (op)= A[M][K] * W[N][K]^T        A: compact activation rows, W: weights [out][in]
//
// Both operands are K-contiguous, which is exactly what the MFMA operand registers want (8
// consecutive k per lane), so tiles go global -> LDS -> registers without any transpose.
//
// Workgroup tile BM x BN, K step 64.  LDS holds one A tile [BM][64] and one B tile [BN][64] as rows of
// eight 16-byte chunks; chunk c of row r is stored at slot c ^ ((r >> 1) & 7).  With 64 LDS banks of
// 4 bytes a 128-byte row covers half the banks, so 16 lanes reading the same chunk of 16 consecutive
// rows (one MFMA operand fetch) touch 16 different (row parity, slot) pairs = all 64 banks once, and
// the row-contiguous fill is conflict free as well.  No padding is needed.
// The register-staged kernel fetches the next K step into registers while the current one is multiplied;
// the direct-to-LDS kernel keeps two K steps in flight in two LDS buffers.
// Each wavefront owns a (BM/WAVES_M) x (BN/WAVES_N) sub-tile, built from 32x32x16 MFMA blocks in the
// register-staged kernel (any K) and from 16x16x32 blocks in the direct-to-LDS kernel (K a multiple of 64).
//
// SwiGLU epilogue (DUAL): the B tile stacks BN/2 rows of W_gate on BN/2 rows of W_up for the same
// output columns, every wavefront holds matching gate/up accumulators and writes silu(gate)*up.
//
// Workgroup ids are remapped so that the workgroups resident on one XCD (ids congruent mod 8) walk
// all row tiles of the same few weight-column tiles: a weight tile is then fetched from HBM once
// per XCD-L2 instead of once per row tile.
#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"
#include "gemm_pipe.h"

namespace rc {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

static constexpr int BK = 64;
static constexpr int XCDS = 8;
static int g_xcd_remap = 1;
void set_gemm_xcd_remap(int on) { g_xcd_remap = on; }

__device__ inline float silu_mf(float x) { return x / (1.0f + __expf(-x)); }

// Accumulator element e of the 32x32 block (i, j) of a wavefront sits at row 8*(e/4) + 4*(lane/32) + e%4,
// column lane%32 of that block.
template <int FM, int FN, int WTM, int WTN, bool DUAL>
__device__ inline void store_tile(const f32x16 (&acc)[FM][FN], void* __restrict__ c, int m, int n, int ldc, int epi,
                                  int m0, int n0, int wm, int wn, int lane) {
  constexpr int FN_OUT = DUAL ? FN / 2 : FN;
  constexpr int WTN_OUT = DUAL ? WTN / 2 : WTN;
  const int khalf = lane >> 5;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
#pragma unroll
    for (int j = 0; j < FN_OUT; ++j) {
      const int col = n0 + wn * WTN_OUT + j * 32 + (lane & 31);
      if (col >= n) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = m0 + wm * WTM + i * 32 + 8 * (e / 4) + 4 * khalf + (e % 4);
        if (row >= m) continue;
        const size_t o = (size_t)row * ldc + col;
        const float v = acc[i][j][e];
        if (DUAL) {
          reinterpret_cast<bf16*>(c)[o] = f32_to_bf16(silu_mf(v) * acc[i][j + FN_OUT][e]);
        } else if (epi == EPI_STORE_F32) {
          reinterpret_cast<float*>(c)[o] = v;
        } else if (epi == EPI_ADD_F32) {
          reinterpret_cast<float*>(c)[o] += v;
        } else {
          reinterpret_cast<bf16*>(c)[o] = f32_to_bf16(v);
        }
      }
    }
  }
}

// Order in which output tiles are handed to workgroups.  The tile rows are cut into `bands` bands of (almost)
// equal height; inside a band tiles run row-first (M fastest), bands follow each other.  The 32 workgroups
// that an XCD runs at a time then cover a block of about 5 x 6 tiles instead of a whole tile column, so
// fewer distinct A and W slices have to come into that XCD's L2 per K step.
struct TileOrder { int tiles_m, tiles_n, bands; };

__device__ __host__ inline void tile_of(TileOrder o, int logical, int* tile_m, int* tile_n) {
  const int base = o.tiles_m / o.bands, rem = o.tiles_m % o.bands;
  const int cut = rem * (base + 1) * o.tiles_n;   // tiles in the taller bands
  int h, m_start, r;
  if (logical < cut) {
    h = base + 1;
    const int per = h * o.tiles_n;
    m_start = (logical / per) * h;
    r = logical % per;
  } else {
    h = base;
    const int per = h * o.tiles_n;
    const int l2 = logical - cut;
    m_start = rem * (base + 1) + (l2 / per) * h;
    r = l2 % per;
  }
  *tile_m = m_start + r % h;
  *tile_n = r / h;
}

__device__ __host__ inline TileOrder make_tile_order(int tiles_m, int tiles_n) {
  TileOrder o = {tiles_m, tiles_n, (tiles_m + 5) / 6};
  if (o.bands < 1) o.bands = 1;
  return o;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool DUAL, int OCC>
__global__ void __launch_bounds__(WAVES_M * WAVES_N * 64, OCC)
gemm_mfma_kernel(const bf16* __restrict__ a, const bf16* __restrict__ w, const bf16* __restrict__ w2,
                 const bf16* __restrict__ w3, int ns1, int ns2, void* __restrict__ c, int m, int n, int k, int ldc,
                 int epi, TileOrder order, int total_tiles, int per_xcd, const int* __restrict__ m_live) {
  constexpr int NT = WAVES_M * WAVES_N * 64;
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  constexpr int FM = WTM / 32, FN = WTN / 32;
  constexpr int A_PER = BM * 8 / NT, B_PER = BN * 8 / NT;
  constexpr int BN_OUT = DUAL ? BN / 2 : BN;
  static_assert(A_PER * NT == BM * 8 && B_PER * NT == BN * 8, "tile/threads mismatch");
  static_assert(!DUAL || (FN % 2 == 0), "dual tiles need an even number of column fragments");

  __shared__ uint4 lds_a[BM * 8];
  __shared__ uint4 lds_b[BN * 8];

  const int logical = per_xcd > 0 ? (int)(blockIdx.x % XCDS) * per_xcd + (int)(blockIdx.x / XCDS) : (int)blockIdx.x;
  if (logical >= total_tiles) return;
  int tile_m, tile_n;
  tile_of(order, logical, &tile_m, &tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN_OUT;
  m = live_count(m, m_live);
  if (m0 >= m) return;   // uniform: the grid may be sized for an upper bound of the row count

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  // per-thread global sources of the tile fill: chunk (row, ch) with row = idx / 8, ch = idx % 8
  const bf16* pa[A_PER];
  const bf16* pb[B_PER];
  const int ch = tid & 7;
#pragma unroll
  for (int i = 0; i < A_PER; ++i) {
    const int row = (tid + i * NT) >> 3;
    pa[i] = (m0 + row < m) ? a + (size_t)(m0 + row) * k + ch * 8 : nullptr;
  }
#pragma unroll
  for (int i = 0; i < B_PER; ++i) {
    const int row = (tid + i * NT) >> 3;
    if (DUAL) {
      const int half = row >= BN / 2;
      const int col = n0 + row - half * (BN / 2);
      pb[i] = (col < n) ? (half ? w2 : w) + (size_t)col * k + ch * 8 : nullptr;
    } else {
      // output columns [0, ns1) come from w, [ns1, ns2) from w2, [ns2, n) from w3 (fused q|k|v projection)
      const int col = n0 + row;
      const bf16* src = col < ns1 ? w + (size_t)col * k : (col < ns2 ? w2 + (size_t)(col - ns1) * k
                                                                     : w3 + (size_t)(col - ns2) * k);
      pb[i] = (col < n) ? src + ch * 8 : nullptr;
    }
  }

  uint4 ra[A_PER], rb[B_PER];
  auto fetch = [&](int k0) {
    const bool kin = k0 + ch * 8 < k;
#pragma unroll
    for (int i = 0; i < A_PER; ++i)
      ra[i] = (pa[i] && kin) ? *reinterpret_cast<const uint4*>(pa[i] + k0) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < B_PER; ++i)
      rb[i] = (pb[i] && kin) ? *reinterpret_cast<const uint4*>(pb[i] + k0) : make_uint4(0, 0, 0, 0);
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // LDS rows this lane reads its MFMA operands from
  int arow[FM], brow[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) arow[i] = wm * WTM + i * 32 + (lane & 31);
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    if (DUAL) brow[j] = (j < FN / 2 ? wn * (WTN / 2) + j * 32 : BN / 2 + wn * (WTN / 2) + (j - FN / 2) * 32) + (lane & 31);
    else brow[j] = wn * WTN + j * 32 + (lane & 31);
  }
  const int khalf = lane >> 5;

  fetch(0);
  for (int k0 = 0; k0 < k; k0 += BK) {
    __syncthreads();   // everyone is done reading the previous tile
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
      const int row = (tid + i * NT) >> 3;
      lds_a[row * 8 + (ch ^ ((row >> 1) & 7))] = ra[i];
    }
#pragma unroll
    for (int i = 0; i < B_PER; ++i) {
      const int row = (tid + i * NT) >> 3;
      lds_b[row * 8 + (ch ^ ((row >> 1) & 7))] = rb[i];
    }
    __syncthreads();
    if (k0 + BK < k) fetch(k0 + BK);
#pragma unroll
    for (int s = 0; s < BK / 16; ++s) {
      bf16x8 fa[FM], fb[FN];
      const int chunk = 2 * s + khalf;
#pragma unroll
      for (int i = 0; i < FM; ++i)
        fa[i] = __builtin_bit_cast(bf16x8, lds_a[arow[i] * 8 + (chunk ^ ((arow[i] >> 1) & 7))]);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        fb[j] = __builtin_bit_cast(bf16x8, lds_b[brow[j] * 8 + (chunk ^ ((brow[j] >> 1) & 7))]);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
  }

  store_tile<FM, FN, WTM, WTN, DUAL>(acc, c, m, n, ldc, epi, m0, n0, wm, wn, lane);
}

// ------------------------------------------------------------------ direct-to-LDS, double-buffered kernel
// Tiles are fetched with 16-byte global->LDS loads (no staging registers, no LDS store instructions) into two
// alternating LDS buffers, so one barrier per K step suffices: wait for my loads, barrier, start the loads
// of the step after next into the buffer just freed, multiply the current one.
//
// A direct load writes lane l's 16 bytes to (wave-uniform LDS base) + 16 l, i.e. one instruction fills
// 1 KB = 8 rows of 128 bytes.  The XOR placement (chunk c of row r at slot c ^ ((r >> 1) & 7)) is
// therefore applied on the global side: lane l of a row block fetches chunk (l & 7) ^ swz(row).
// Rows past M (or N) re-read the last valid row; their products are never stored.  K must be a
// multiple of 64.
//
// The wavefront sub-tile is built from 16x16x32 MFMA blocks (measured: with the same LDS and load traffic
// this shape sustains about 9 % more matrix throughput than 32x32x16 under the chip's power limit).  A K
// step of 64 is two sub-steps of 32; each sub-step is multiplied in two halves of the weight-column blocks,
// so a pipeline unit is FM x FN/2 MFMAs with the LDS reads of the next unit in flight.  16 lanes reading the
// same chunk of 16 consecutive rows (one operand fetch) touch all 64 LDS banks once, as in the kernel above.
//
// The weight fragment is passed as the first MFMA operand, so that accumulator (i, j) of a lane holds
//   row    i*16 + lane%16                 of the wavefront's activation rows,
//   column j*16 + 4*(lane/16) + e         of its output columns, e = 0..3:
// four consecutive output columns per lane, stored with one 16-byte (f32) or 8-byte (bf16) access.
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// Four bf16 outputs as one number.  Of a struct of two or four the compiler stores the parts one by one wherever another branch ends
// in a store of the same part, as the ragged end of a row does: the gate/up epilogue wrote nearly every group of four with three
// stores.  Gate/up products with one store instead: 1639 x 28672 x 4096 341 -> 323 us, 5120 rows 915 -> 884, 1025 rows 208 -> 198, 900 x
// 2816 x 512 9.5 -> 8.0.
__device__ __forceinline__ unsigned long long pack_bf16(float a, float b, float c, float d) {
  return (unsigned long long)f32_to_bf16(a).v | ((unsigned long long)f32_to_bf16(b).v << 16) | ((unsigned long long)f32_to_bf16(c).v << 32) |
         ((unsigned long long)f32_to_bf16(d).v << 48);
}

// four consecutive outputs at element o of C, `left` of them inside the row
__device__ __forceinline__ void store_quad(void* __restrict__ c, size_t o, const float (&v)[4], int epi, bool f32_out, bool vec, int left) {
  if (vec) {
    if (f32_out) {
      float4* dst = reinterpret_cast<float4*>(reinterpret_cast<float*>(c) + o);
      float4 t = make_float4(v[0], v[1], v[2], v[3]);
      if (epi == EPI_ADD_F32) { const float4 old = *dst; t.x += old.x; t.y += old.y; t.z += old.z; t.w += old.w; }
      *dst = t;
    } else {
      *reinterpret_cast<unsigned long long*>(reinterpret_cast<bf16*>(c) + o) = pack_bf16(v[0], v[1], v[2], v[3]);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (e >= left) continue;
      if (!f32_out) reinterpret_cast<bf16*>(c)[o + e] = f32_to_bf16(v[e]);
      else if (epi == EPI_ADD_F32) reinterpret_cast<float*>(c)[o + e] += v[e];
      else reinterpret_cast<float*>(c)[o + e] = v[e];
    }
  }
}

// Four consecutive rotary pairs of a row of q|k|v, rotated and left where they belong: the work and the arithmetic of
// rope_scatter_kernel.  lo / hi: the columns of the two halves of a head.  In the epilogue of the product it costs 2 us of 109
// (2500 rows) or nothing (60 rows, inside the sum over the K parts); the launch it replaces wrote and read the product in floats:
// 6 us at 60 rows, 12.7 at 1639, 37 at 5120.
__device__ __forceinline__ void rope_quad(const RopeOut& o, int row, int pos, unsigned dst, int pair, const f32x4& lo, const f32x4& hi, int ns1,
                                          int ns2) {
  const int col = rope_column(pair, 0), i = pair & 63;
  f32x4 a = lo, b = hi;
  if (col < ns2) {
    const float4 t01 = *reinterpret_cast<const float4*>(o.tab + (size_t)pos * 64 + i);       // (cos, sin) of pairs i, i+1
    const float4 t23 = *reinterpret_cast<const float4*>(o.tab + (size_t)pos * 64 + i + 2);   // pairs i+2, i+3
    const float c[4] = {t01.x, t01.z, t23.x, t23.z}, s[4] = {t01.y, t01.w, t23.y, t23.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      a[e] = __builtin_fmaf(lo[e], c[e], -(hi[e] * s[e]));
      b[e] = __builtin_fmaf(hi[e], c[e], lo[e] * s[e]);
    }
  }
  auto put = [](bf16* p, const f32x4& v) { *reinterpret_cast<unsigned long long*>(p) = pack_bf16(v[0], v[1], v[2], v[3]); };
  if (col < ns1) {
    bf16* q = o.q + (size_t)row * ns1 + col;
    put(q, a);
    put(q + 64, b);
    return;
  }
  if (dst == kRowNoDst) return;
  const bool is_v = col >= ns2;
  const size_t at = ((size_t)dst + (size_t)((col - (is_v ? ns2 : ns1)) >> 7) * o.block_size) * 128 + i;
  bf16* pool = is_v ? o.v_pool : o.k_pool;
  put(pool + at, a);
  put(pool + at + 64, b);
  if (!is_v && o.k_pre_pool) {
    put(o.k_pre_pool + at, lo);
    put(o.k_pre_pool + at + 64, hi);
  }
}

template <int FM, int FN, int WTM, int WTN, int MODE>
__device__ inline void store_tile16(const f32x4 (&acc)[FM][FN], void* __restrict__ c, int m, int n, int ldc, int epi,
                                    int m0, int n0, int wm, int wn, int lane, int ns1, int ns2, const RopeOut& rope) {
  constexpr bool DUAL = MODE == kDual;
  constexpr int FN_OUT = DUAL ? FN / 2 : FN;
  constexpr int WTN_OUT = DUAL ? WTN / 2 : WTN;
  if constexpr (MODE == kRope) {
    constexpr int FH = FN / 2;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int row = m0 + wm * WTM + i * 16 + (lane & 15);
      if (row >= m) continue;
      const int pos = rope.row_pos[row];
      const unsigned dst = rope.row_dst[row];
#pragma unroll
      for (int j = 0; j < FH; ++j) {
        const int pair = n0 + wn * (WTN / 2) + j * 16 + 4 * (lane >> 4);
        if (pair < n) rope_quad(rope, row, pos, dst, pair, acc[i][j], acc[i][j + FH], ns1, ns2);
      }
    }
    return;
  }
  const bool f32_out = !DUAL && (epi == EPI_STORE_F32 || epi == EPI_ADD_F32);
  const bool vec_ok = (ldc & 3) == 0 && (reinterpret_cast<size_t>(c) & (f32_out ? 15 : 7)) == 0;
  if constexpr (!DUAL) {
    // residual add with the wavefront's columns all inside C: the old values of a block row are requested together and
    // added afterwards, so the wavefront waits for memory once per block row instead of once per 16 x 16 block
    if (epi == EPI_ADD_F32 && vec_ok && n0 + wn * WTN + WTN <= n) {   // wave-uniform
      float* const cf = reinterpret_cast<float*>(c);
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int row = m0 + wm * WTM + i * 16 + (lane & 15);
        if (row >= m) continue;
        float4* const dst = reinterpret_cast<float4*>(cf + (size_t)row * ldc + n0 + wn * WTN + 4 * (lane >> 4));
        float4 old[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) old[j] = dst[j * 4];
#pragma unroll
        for (int j = 0; j < FN; ++j)
          dst[j * 4] = make_float4(old[j].x + acc[i][j][0], old[j].y + acc[i][j][1], old[j].z + acc[i][j][2],
                                   old[j].w + acc[i][j][3]);
      }
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = m0 + wm * WTM + i * 16 + (lane & 15);
    if (row >= m) continue;
#pragma unroll
    for (int j = 0; j < FN_OUT; ++j) {
      const int col = n0 + wn * WTN_OUT + j * 16 + 4 * (lane >> 4);
      if (col >= n) continue;
      const size_t o = (size_t)row * ldc + col;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = DUAL ? silu_mf(acc[i][j][e]) * acc[i][j + FN_OUT][e] : acc[i][j][e];
      store_quad(c, o, v, epi, f32_out, vec_ok && col + 3 < n, n - col);
    }
  }
}

// Where column col of row `row` of a K part's tile is kept: blocks of 16 columns (64 bytes) change places by the row, so that a store
// of 16 rows spreads over the memory channels.  With the columns in place, rows 512 to 1024 bytes apart, the products were 1 to 3 us
// slower than with register-major parts; now (weights from memory): 900 x 17920 x 1536 70.3 -> 63.4 us, 600 x 1536 x 8960 41.4 ->
// 39.3, 1025 x 4096 x 4096 45.0 -> 43.6.  Two stores of eight whole 128-byte lines instead of sixteen halves: no gain.
__device__ __forceinline__ int part_column(int col, int row, int bn) { return col ^ (16 * (row & (bn % 128 == 0 ? 7 : 3))); }

// The accumulators of a K part, as rows of BN floats (PAIRED: the first columns of all pairs, then the second) of the part's BM x BN
// block: whoever adds the parts up reads whole rows.  Rows past the product's last one are left out.
template <int FM, int FN, int BM, int BN, int WTM, int WTN, bool PAIRED>
__device__ inline void store_partial(const f32x4 (&acc)[FM][FN], float* __restrict__ partial, int part_slot, int rows, int wm, int wn,
                                     int lane) {
  constexpr int FH = FN / 2;
  float* const base = partial + (size_t)part_slot * BM * BN + 4 * (lane >> 4);
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = wm * WTM + i * 16 + (lane & 15);
    if (row >= rows) continue;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = !PAIRED ? wn * WTN + j * 16 : (j < FH ? wn * (WTN / 2) + j * 16 : BN / 2 + wn * (WTN / 2) + (j - FH) * 16);
      *reinterpret_cast<f32x4*>(base + (size_t)row * BN + part_column(col, lane, BN)) = acc[i][j];
    }
  }
}

// One output tile (or one K part of it): the work of a workgroup once it knows its tile.
template <int BM, int BN, int WAVES_M, int WAVES_N, int MODE>
__device__ __forceinline__ void gemm_tile_body(const bf16* __restrict__ a, const bf16* __restrict__ w,
                                               const bf16* __restrict__ w2, const bf16* __restrict__ w3, int ns1, int ns2,
                                               void* __restrict__ c, int m, int n, int k, int ldc, int epi, int m0, int n0,
                                               int k_begin, int k_end, int part_slot, float* __restrict__ partial, const RopeOut& rope) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  constexpr int FM = WTM / 16, FN = WTN / 16, FH = FN / 2;
  constexpr int A_BLK = BM / 8, B_BLK = BN / 8;
  constexpr int A_PER = A_BLK / NW, B_PER = B_BLK / NW;
  static_assert(A_PER * NW == A_BLK && B_PER * NW == B_BLK, "tile/waves mismatch");
  static_assert(FN % 2 == 0 && BK == 64, "two sub-steps of 32, two halves of the column blocks");
  constexpr int TILE_BYTES = (BM + BN) * 128;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];   // 2 x [A tile | B tile]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  const int lrow = lane >> 3, lslot = lane & 7;
  const bf16* pa[A_PER];
  const bf16* pb[B_PER];
#pragma unroll
  for (int i = 0; i < A_PER; ++i) {
    const int row = (wave + i * NW) * 8 + lrow;
    const int chunk = lslot ^ ((row >> 1) & 7);
    pa[i] = a + (size_t)min(m0 + row, m - 1) * k + chunk * 8;
  }
#pragma unroll
  for (int i = 0; i < B_PER; ++i) {
    const int row = (wave + i * NW) * 8 + lrow;
    const int chunk = lslot ^ ((row >> 1) & 7);
    const bf16* src;
    if (MODE == kDual) {
      const int half = row >= BN / 2;
      const int col = min(n0 + row - half * (BN / 2), n - 1);
      src = (half ? w2 : w) + (size_t)col * k;
    } else {
      const int half = MODE == kRope && row >= BN / 2 ? 1 : 0;
      const int unit = min(n0 + row - half * (BN / 2), n - 1);
      const int col = MODE == kRope ? rope_column(unit, half) : unit;
      src = col < ns1 ? w + (size_t)col * k : (col < ns2 ? w2 + (size_t)(col - ns1) * k : w3 + (size_t)(col - ns2) * k);
    }
    pb[i] = src + chunk * 8;
  }
  auto issue = [&](int k0, int buf) {
    unsigned char* base = lds + buf * TILE_BYTES;
#pragma unroll
    for (int i = 0; i < A_PER; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(pa[i] + k0),
                                       (__attribute__((address_space(3))) void*)(base + (wave + i * NW) * 1024), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < B_PER; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(pb[i] + k0),
                                       (__attribute__((address_space(3))) void*)(base + BM * 128 + (wave + i * NW) * 1024), 16, 0, 0);
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // LDS rows this lane reads its operands from: lane%16 selects the row of a 16-row block, lane/16 the 8-k chunk
  int arow[FM], brow[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) arow[i] = wm * WTM + i * 16 + (lane & 15);
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    if (MODE != kPlain) brow[j] = (j < FH ? wn * (WTN / 2) + j * 16 : BN / 2 + wn * (WTN / 2) + (j - FH) * 16) + (lane & 15);
    else brow[j] = wn * WTN + j * 16 + (lane & 15);
  }
  const int kq = lane >> 4;

  bf16x8 fa[2][FM], fb[2][FH];
  auto load_a = [&](int b, int s) {
    const uint4* la = reinterpret_cast<const uint4*>(lds + b * TILE_BYTES);
    const int chunk = 4 * s + kq;
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[s][i] = __builtin_bit_cast(bf16x8, la[arow[i] * 8 + (chunk ^ ((arow[i] >> 1) & 7))]);
  };
  auto load_b = [&](int b, int s, int h) {
    const uint4* lb = reinterpret_cast<const uint4*>(lds + b * TILE_BYTES + BM * 128);
    const int chunk = 4 * s + kq;
#pragma unroll
    for (int j = 0; j < FH; ++j) {
      const int r = brow[h * FH + j];
      fb[h][j] = __builtin_bit_cast(bf16x8, lb[r * 8 + (chunk ^ ((r >> 1) & 7))]);
    }
  };
  auto multiply = [&](int s, int h) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FH; ++j)
        acc[i][h * FH + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[h][j], fa[s][i], acc[i][h * FH + j], 0, 0, 0);
  };

  if (k_begin < k_end) {
    issue(k_begin, 0);
    if (k_begin + BK < k_end) issue(k_begin + BK, 1);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    load_a(0, 0);
    load_b(0, 0, 0);
  }
  int buf = 0;
  for (int k0 = k_begin; k0 < k_end; k0 += BK) {
    load_b(buf, 0, 1);
    __builtin_amdgcn_sched_barrier(0);   // keep the LDS reads of the next unit ahead of this unit's MFMAs
    multiply(0, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_a(buf, 1);
    load_b(buf, 1, 0);
    __builtin_amdgcn_sched_barrier(0);
    multiply(0, 1);
    __builtin_amdgcn_sched_barrier(0);
    load_b(buf, 1, 1);
    __builtin_amdgcn_sched_barrier(0);
    multiply(1, 0);
    __builtin_amdgcn_sched_barrier(0);
    // the last unit's operands are being read; once they are in registers nobody needs buffer `buf` any more
    __builtin_amdgcn_s_waitcnt(0);   // my LDS reads and my direct loads of the next step are complete
    __syncthreads();
    if (k0 + 2 * BK < k_end) issue(k0 + 2 * BK, buf);
    if (k0 + BK < k_end) { load_a(buf ^ 1, 0); load_b(buf ^ 1, 0, 0); }
    __builtin_amdgcn_sched_barrier(0);
    multiply(1, 1);
    __builtin_amdgcn_sched_barrier(0);
    buf ^= 1;
  }

  if (part_slot >= 0) {
    store_partial<FM, FN, BM, BN, WTM, WTN, MODE != kPlain>(acc, partial, part_slot, m - m0, wm, wn, lane);
    return;
  }
  store_tile16<FM, FN, WTM, WTN, MODE>(acc, c, m, n, ldc, epi, m0, n0, wm, wn, lane, ns1, ns2, rope);
}

// The same on the pipelined main loop of gemm_pipe.h; partial sums in the layout of gemm_tile_body.
template <typename T, int MODE, bool LANE_ID = false>
__device__ __forceinline__ void gemm_pipe_body(const bf16* __restrict__ a, const bf16* __restrict__ w,
                                               const bf16* __restrict__ w2, const bf16* __restrict__ w3, int ns1, int ns2,
                                               void* __restrict__ c, int m, int n, int k, int ldc, int epi, int m0, int n0,
                                               int k_begin, int k_end, int part_slot, float* __restrict__ partial, const RopeOut& rope) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  f32x4 acc[T::FM][T::FN];
  gemm_pipe_loop<T, MODE, LANE_ID>(a, w, w2, w3, ns1, ns2, m, n, k, m0, n0, k_begin, k_end, lds, acc);
  const int tid = threadIdx.x;
  const int lane = LANE_ID ? __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) : tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::WN, wn = wave % T::WN;
  if (part_slot >= 0) {
    store_partial<T::FM, T::FN, T::BM, T::BN, T::WTM, T::WTN, MODE != kPlain>(acc, partial, part_slot, m - m0, wm, wn, lane);
    return;
  }
  store_tile16<T::FM, T::FN, T::WTM, T::WTN, MODE>(acc, c, m, n, ldc, epi, m0, n0, wm, wn, lane, ns1, ns2, rope);
}

// What the launch's grid does.  Workgroups [0, n_full_wgs) each own one of the first full_tiles output tiles
// (whole K range).  The remaining tiles, too few to fill the chip, are each cut along K into `split` parts:
// workgroup n_full_wgs + j takes part j % split of the tile after the whole ones + j / split and leaves its raw
// accumulators in `partial`; gemm_fixup_kernel adds the parts in a fixed order and applies the epilogue.
//
// Thin tiles: when the last tile row has at most 64 live rows (a prompt whose live rows are a multiple of the tile
// height plus a few: the last reused token, a short suffix), its n_thin tiles are multiplied by a 64 x 256 body (the tile of
// code 13), which costs about a third of a full tile; `order` then describes the tile rows
// above it only.  The thin tiles are always whole-K tiles and are dealt out evenly over the XCDs' queues, at
// the tail of each, where they fill the last round.  (A 128-row body for up to 128 live rows was measured
// as well: no gain.)
struct GridPlan {
  TileOrder order;      // the normal tiles (all tile rows, or all but the ragged last one)
  int full_tiles;       // whole-K tiles: normal ones first, then the n_thin thin ones
  int per_xcd;          // > 0: workgroup ids are regrouped per XCD, this many queue slots each
  int n_full_wgs;       // workgroups reserved for whole-K tiles (some may stay empty)
  int split, kpp;       // K parts per remaining tile, K steps per part
  int n_thin;
};
struct BlockWork { int kind /* 0: nothing, 1: normal tile, 2: thin tile */, tile_m, tile_n, k_begin, k_end, part_slot; };

__device__ __host__ inline BlockWork block_work(const GridPlan& g, int bid, int k) {
  BlockWork bw = {0, 0, 0, 0, k, -1};
  const int n_normal_full = g.full_tiles - g.n_thin;
  int u = 0, thin_tile = -1;   // u: index among the normal tiles
  if (bid < g.n_full_wgs) {
    if (g.per_xcd > 0) {
      const int x = bid % XCDS, j = bid / XCDS;
      const int cnt = g.n_thin / XCDS + (x < g.n_thin % XCDS ? 1 : 0);                          // thin tiles of this XCD
      const int before = x * (g.n_thin / XCDS) + (x < g.n_thin % XCDS ? x : g.n_thin % XCDS);   // ... of the XCDs before it
      if (j >= g.per_xcd - cnt) thin_tile = (j - (g.per_xcd - cnt)) * XCDS + x;
      else u = x * g.per_xcd - before + j;
    } else if (bid >= n_normal_full) {
      thin_tile = bid - n_normal_full;
      if (thin_tile >= g.n_thin) return bw;
    } else {
      u = bid;
    }
    if (thin_tile < 0 && u >= n_normal_full) return bw;
  } else {
    const int j = bid - g.n_full_wgs;
    u = n_normal_full + j / g.split;
    bw.part_slot = j;
    bw.k_begin = (j % g.split) * g.kpp * BK;
    bw.k_end = bw.k_begin + g.kpp * BK < k ? bw.k_begin + g.kpp * BK : k;
  }
  if (thin_tile >= 0) {
    bw.kind = 2;
    bw.tile_m = g.order.tiles_m;   // the row below the normal ones
    bw.tile_n = thin_tile;
  } else {
    bw.kind = 1;
    tile_of(g.order, u, &bw.tile_m, &bw.tile_n);
  }
  return bw;
}

// Tile types of the direct-to-LDS kernels: the pipelined ones (eight wavefronts) and the 128x128 tile of four wavefronts.
struct Tile128 {
  static constexpr int WM = 2, WN = 2, FM = 4, FN = 4, WTM = 64, WTN = 64, BM = 128, BN = 128, NT = 256;
  static constexpr int LDS_BYTES = 2 * (BM + BN) * 128;
  static constexpr int OCC = 2, WAVES_PER_SIMD = 2;
  static constexpr bool DUAL_OK = true;
  template <int MODE, typename... Args> static __device__ __forceinline__ void body(const Args&... args) {
    gemm_tile_body<128, 128, 2, 2, MODE>(args...);
  }
};
template <int WM_, int WN_, int FM0_, int FM1_, int FN0_, int FN1_, int OCC_ = 1>
struct TilePipe : PipeTile<WM_, WN_, FM0_, FM1_, FN0_, FN1_> {
  static constexpr int NT = 512, OCC = OCC_, WAVES_PER_SIMD = 2 * OCC_;
  static constexpr bool DUAL_OK = FN0_ == FN1_;
  template <int MODE, typename... Args> static __device__ __forceinline__ void body(const Args&... args) {
    gemm_pipe_body<PipeTile<WM_, WN_, FM0_, FM1_, FN0_, FN1_>, MODE>(args...);
  }
};

template <typename T, int MODE, bool THIN>
__device__ __forceinline__ void gemm_dl_work(const bf16* __restrict__ a, const bf16* __restrict__ w, const bf16* __restrict__ w2,
                                             const bf16* __restrict__ w3, int ns1, int ns2, void* __restrict__ c, int m, int n, int k,
                                             int ldc, int epi, const GridPlan& plan, float* __restrict__ partial,
                                             const int* __restrict__ m_live, const RopeOut& rope) {
  constexpr int BM = T::BM, BN = T::BN, BN_OUT = MODE != kPlain ? BN / 2 : BN;
  BlockWork bw = {1, 0, 0, 0, k, -1};   // one call of the tile body for both cases: with two, its loop ran out of registers
  if (m_live) {
    // The row count lives on the device (rows selected by a threshold) and the host's m only sized the grid.  The
    // schedule is rebuilt here for the live count, in its plain form: every tile whole, by one workgroup, ids
    // regrouped per XCD over the live tiles (so that all XCDs share them), no K-split tail, no thin tiles.
    m = min(m, *m_live);
    if (m <= 0) return;
    const int tiles_m = (m + BM - 1) / BM, tiles_n = plan.order.tiles_n;
    const int total = tiles_m * tiles_n, per_xcd = (total + XCDS - 1) / XCDS;
    const int x = (int)blockIdx.x % XCDS, j = (int)blockIdx.x / XCDS;
    const int logical = plan.per_xcd > 0 ? x * per_xcd + j : (int)blockIdx.x;
    if ((plan.per_xcd > 0 && j >= per_xcd) || logical >= total) return;
    tile_of(make_tile_order(tiles_m, tiles_n), logical, &bw.tile_m, &bw.tile_n);
  } else {
    bw = block_work(plan, (int)blockIdx.x, k);
    if (bw.kind == 0) return;
  }
  if constexpr (THIN) {
    static_assert(BN == 256 && T::NT == 512, "the thin body covers a tile's columns");
    if (bw.kind == 2) {
      gemm_pipe_body<PipeTile<1, 8, 4, 0, 1, 1>, MODE, true>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, epi, bw.tile_m * BM,
                                                       bw.tile_n * BN_OUT, 0, k, -1, partial, rope);
      return;
    }
  }
  T::template body<MODE>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, epi, bw.tile_m * BM, bw.tile_n * BN_OUT, bw.k_begin,
                         bw.k_end, bw.part_slot, partial, rope);
}

template <typename T, bool DUAL, bool THIN>
__global__ void __launch_bounds__(T::NT, T::WAVES_PER_SIMD)
gemm_mfma_dl_kernel(const bf16* __restrict__ a, const bf16* __restrict__ w, const bf16* __restrict__ w2,
                    const bf16* __restrict__ w3, int ns1, int ns2, void* __restrict__ c, int m, int n, int k, int ldc,
                    int epi, GridPlan plan, float* __restrict__ partial, const int* __restrict__ m_live) {
  gemm_dl_work<T, DUAL ? kDual : kPlain, THIN>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, epi, plan, partial, m_live, RopeOut{});
}

// the q|k|v product with rotary and scatter; n: rotary pairs
template <typename T, bool THIN>
__global__ void __launch_bounds__(T::NT, T::WAVES_PER_SIMD)
gemm_qkv_rope_kernel(const bf16* __restrict__ a, const bf16* __restrict__ wq, const bf16* __restrict__ wk, const bf16* __restrict__ wv,
                     int ns1, int ns2, int m, int n, int k, GridPlan plan, float* __restrict__ partial, const int* __restrict__ m_live,
                     RopeOut rope) {
  gemm_dl_work<T, kRope, THIN>(a, wq, wk, wv, ns1, ns2, nullptr, m, n, k, 0, (int)EPI_STORE_T, plan, partial, m_live, rope);
}

// The parts of one product that are still to be added up: tiles [full, ...) of `order`, bm x bn, in `split` parts each.
struct PartTiles { TileOrder order; int full, split, bm, bn; const float* partial; };

// index of tile (tile_m, tile_n) in the order: the inverse of tile_of
__device__ __host__ inline int tile_index(TileOrder o, int tile_m, int tile_n) {
  const int base = o.tiles_m / o.bands, rem = o.tiles_m % o.bands;
  const int tall = rem * (base + 1);
  const bool in_tall = tile_m < tall;
  const int h = in_tall ? base + 1 : base;
  const int local = in_tall ? tile_m : tile_m - tall;
  const int m_in = local % h;
  return (tile_m - m_in) * o.tiles_n + tile_n * h + m_in;
}

// Sum of the K parts of the cut tiles (fixed order: part 0, 1, ...) followed by the epilogue.  A thread owns four columns of
// a row, consecutive threads a row's next ones.
template <int MODE>
__global__ void __launch_bounds__(256)
gemm_fixup_kernel(void* __restrict__ c, int m, int n, int ldc, int epi, PartTiles pt, int wgs_per_tile, int ns1,
                  int ns2, RopeOut rope) {
  constexpr bool PAIRED = MODE != kPlain, DUAL = MODE == kDual;
  const int bn_out = PAIRED ? pt.bn / 2 : pt.bn, quads = bn_out / 4;
  const int t = (int)blockIdx.x / wgs_per_tile;
  const int item = ((int)blockIdx.x % wgs_per_tile) * 256 + (int)threadIdx.x;
  const int r = item / quads, q = item - r * quads;
  int tile_m, tile_n;
  tile_of(pt.order, pt.full + t, &tile_m, &tile_n);
  const int row = tile_m * pt.bm + r, col = tile_n * bn_out + 4 * q;
  if (r >= pt.bm || row >= m || col >= n) return;
  const size_t part = (size_t)pt.bm * pt.bn;
  const float* src = pt.partial + (size_t)t * pt.split * part + (size_t)r * pt.bn;
  const int first = part_column(4 * q, r, pt.bn), second = PAIRED ? part_column(4 * q + bn_out, r, pt.bn) : 0;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f}, up = sum;
#pragma unroll 4
  for (int p = 0; p < pt.split; ++p) {
    sum += *reinterpret_cast<const f32x4*>(src + p * part + first);
    if (PAIRED) up += *reinterpret_cast<const f32x4*>(src + p * part + second);
  }
  if constexpr (MODE == kRope) {
    rope_quad(rope, row, rope.row_pos[row], rope.row_dst[row], col, sum, up, ns1, ns2);
    return;
  }
  const bool f32_out = !DUAL && (epi == EPI_STORE_F32 || epi == EPI_ADD_F32);
  const bool vec_ok = (ldc & 3) == 0 && (reinterpret_cast<size_t>(c) & (f32_out ? 15 : 7)) == 0;
  const size_t o = (size_t)row * ldc + col;
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = DUAL ? silu_mf(sum[e]) * up[e] : sum[e];
  store_quad(c, o, v, epi, f32_out, vec_ok && col + 3 < n, n - col);
}

// The same for the residual add (h += the product), with the RMS norm of the finished rows behind it: a workgroup per row, the
// row stays in registers.  Elements and sums are those of rmsnorm_kernel, whose thread t owns elements 4 (t + 256 u) + 0..3:
// here 256 threads take UPT u's each, so that a row's parts are asked for by up to sixteen wavefronts at once (with the four of
// rmsnorm_kernel a row of 16 parts took 21 us), and the squares are added up in its order.  Sum and norm in launches of their own
// -> here: 62 rows in 8 and 16 parts 4.8-7.8 + 4.7 -> 6.2 us, 1639 rows 22 + 9.8 -> 24.7 us (125 MB: 5 TB/s).
template <int UPT>
__global__ void __launch_bounds__(1024)
gemm_fixup_norm_kernel(float* __restrict__ h, const bf16* __restrict__ gain, bf16* __restrict__ out, int d, float eps, PartTiles pt) {
  __shared__ float squares[8][256];
  __shared__ float red[4];
  const int r = blockIdx.x, tid = threadIdx.x, t = tid & 255, u0 = (tid >> 8) * UPT;
  const int tile_m = r / pt.bm, rr = r - tile_m * pt.bm;
  float* const x = h + (size_t)r * d;
  const size_t part = (size_t)pt.bm * pt.bn;
  const float* src[UPT];
  size_t step[UPT];
  f32x4 v[UPT], sum[UPT];
  uint2 g[UPT];
  bool cut[UPT];
#pragma unroll
  for (int i = 0; i < UPT; ++i) {
    const int c = min((t + (u0 + i) * 256) * 4, d - 4);   // elements past the row repeat its last ones; no condition around a load
    v[i] = *reinterpret_cast<const f32x4*>(x + c);
    g[i] = *reinterpret_cast<const uint2*>(gain + c);
    const int tile_n = c / pt.bn;
    const int k = tile_m < pt.order.tiles_m ? tile_index(pt.order, tile_m, tile_n) - pt.full : -1;   // the thin row is never cut
    cut[i] = k >= 0;
    src[i] = pt.partial + (cut[i] ? (size_t)k * pt.split * part + (size_t)rr * pt.bn + part_column(c - tile_n * pt.bn, rr, pt.bn) : 0);
    step[i] = cut[i] ? part : 0;   // whole tiles: the same line over and over
    sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  constexpr int AHEAD = 8 / UPT;
  for (int p0 = 0; p0 < pt.split; p0 += AHEAD) {
    f32x4 q[AHEAD][UPT];
#pragma unroll
    for (int p = 0; p < AHEAD; ++p)
#pragma unroll
      for (int i = 0; i < UPT; ++i) q[p][i] = *reinterpret_cast<const f32x4*>(src[i] + min(p0 + p, pt.split - 1) * step[i]);
#pragma unroll
    for (int p = 0; p < AHEAD; ++p)
      if (p0 + p < pt.split) {   // uniform
#pragma unroll
        for (int i = 0; i < UPT; ++i) sum[i] += q[p][i];
      }
  }
#pragma unroll
  for (int i = 0; i < UPT; ++i) {
    const int c = (t + (u0 + i) * 256) * 4;
    if (cut[i]) v[i] = sum[i] + v[i];
    if (cut[i] && c < d) *reinterpret_cast<f32x4*>(x + c) = v[i];
    squares[u0 + i][t] = c < d ? add_squares(0.f, make_float4(v[i][0], v[i][1], v[i][2], v[i][3])) : 0.f;
  }
  __syncthreads();
  if (tid < 256) {
    float ss = squares[0][t];
    for (int u = 1; u * 1024 < d; ++u) ss += squares[u][t];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
  }
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) s += red[i];
  const float inv = 1.0f / sqrtf(s / (float)d + eps);
#pragma unroll
  for (int i = 0; i < UPT; ++i) {
    const int c = (t + (u0 + i) * 256) * 4;
    if (c >= d) continue;
    uint2 pk;
    pk.x = (uint32_t)f32_to_bf16(v[i][0] * inv * __uint_as_float(g[i].x << 16)).v |
           ((uint32_t)f32_to_bf16(v[i][1] * inv * __uint_as_float(g[i].x & 0xffff0000u)).v << 16);
    pk.y = (uint32_t)f32_to_bf16(v[i][2] * inv * __uint_as_float(g[i].y << 16)).v |
           ((uint32_t)f32_to_bf16(v[i][3] * inv * __uint_as_float(g[i].y & 0xffff0000u)).v << 16);
    *reinterpret_cast<uint2*>(out + (size_t)r * d + c) = pk;
  }
}

// ------------------------------------------------------------------ the K partition of a product
// Which outputs are summed over K in one go and which in parts.  This is part of the result's definition: another
// partition changes the last bit of float sums, bf16 rounding turns that into whole rounding steps and a stack of
// decoder layers carries them to about 1e-2 of the logits.  So the partition is a function of the product's sizes (rows,
// columns, K, epilogue, compute units) and of what the caller hands over (without a workspace, or with the row count on
// the device, every output is summed whole), never of the tile types below, which only decide who computes what and
// all give the same bits.  Products of at most 32 rows may go to the few-row kernel, which adds eight shares of K.
//
// The rule: 256x256, 256x192 (where they cover N exactly) or 128x128 tiles, whichever a rough time model prices lowest
// (microseconds; one K step of a full round costs kStep256, kStep192 (one workgroup per CU) or kStep128 (two per CU),
// summing one tile part in the fix-up kFixPart).  Full rounds of 256-row tiles are summed whole; the remaining tiles,
// too few to fill the chip, in parts.  128x128 tiles are always summed whole.
static constexpr float kStep256 = 1.9f, kStep192 = 1.55f, kStep128 = 1.2f, kFixPart = 0.1f, kFixLaunch = 6.f;

struct SplitPlan { int rem, split; float cost; };
// total tiles over `slots` workgroup slots: full rounds, then `rem` tiles cut into `split` K parts each
static SplitPlan plan_tail_split(int total, int slots, int ksteps, float step = kStep256) {
  SplitPlan best;
  best.rem = total % slots;
  best.split = 1;
  const int full_rounds = total / slots;
  best.cost = (full_rounds + (best.rem > 0 ? 1 : 0)) * ksteps * step;
  if (best.rem == 0) return best;
  const int gmax = std::min(std::min(slots / best.rem, 16), ksteps);
  for (int g = 2; g <= gmax; ++g) {
    if (best.rem * g > 256) break;
    const float c = full_rounds * ksteps * step + ((ksteps + g - 1) / g) * step + best.rem * g * kFixPart + kFixLaunch;
    if (c < best.cost) { best.cost = c; best.split = g; }
  }
  return best;
}

// compute units of the current device (asked once per device)
static int num_cus() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  std::atomic<int>& slot = cached[dev & 63];
  int n = slot.load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    slot.store(n, std::memory_order_relaxed);
  }
  return n;
}

static constexpr size_t kPartialFloats = (size_t)256 * 256 * 256;   // 256 parts of the largest tile
size_t gemm_partial_bytes() { return kPartialFloats * sizeof(float) + 4096; }

// Schedule of a launch of 256-row tiles: which tiles run whole, which are cut along K, and whether the ragged
// last tile row goes to the thin body.  A thin tile is priced at kThinCost of a full one.
static constexpr float kThinCost = 0.4f;
static constexpr int kThinRows = 64;
static int g_thin_tiles = 1;
void set_gemm_thin_tiles(int on) { g_thin_tiles = on; }

struct LaunchPlan {
  int n_thin;                 // tiles of the ragged last tile row handled by the thin body (0: none)
  int n_normal;               // tiles of the other rows
  int rem, split, kpp;        // the last `rem` normal tiles are cut into `split` parts of `kpp` K steps
  float cost;
};

// thin: price and schedule the launch with the ragged last tile row on the thin body; cost < 0 if that is not possible
static LaunchPlan plan_one(int m, int tiles_n, int bm, int ksteps, int slots, float step, bool may_split, bool thin) {
  const int tiles_m = (m + bm - 1) / bm;
  LaunchPlan p = {};
  p.cost = -1.f;
  if (thin) {
    const int ragged = m - (tiles_m - 1) * bm;   // live rows of the last tile row
    if (tiles_m < 2 || ragged > kThinRows) return p;
    p.n_thin = tiles_n;
  }
  p.n_normal = tiles_m * tiles_n - p.n_thin;
  const int equiv = p.n_normal + (int)(p.n_thin * kThinCost + 0.999f);
  p.split = 1;
  p.kpp = ksteps;
  float cost;
  if (may_split) {
    const SplitPlan sp = plan_tail_split(equiv, slots, ksteps, step);
    cost = sp.cost;
    if (sp.split > 1) {
      p.rem = sp.rem;
      p.kpp = (ksteps + sp.split - 1) / sp.split;
      p.split = (ksteps + p.kpp - 1) / p.kpp;
    }
  } else {
    cost = ((equiv + slots - 1) / slots) * ksteps * step;
  }
  // thin tiles only among the whole tiles of a launch that has at least one full round
  if (thin && (equiv < slots || p.rem > p.n_normal)) return p;
  p.cost = cost;
  return p;
}

static LaunchPlan plan_launch(int m, int tiles_n, int bm, int ksteps, int slots, float step, bool may_split, bool may_thin) {
  const LaunchPlan plain = plan_one(m, tiles_n, bm, ksteps, slots, step, may_split, false);
  if (may_thin && g_thin_tiles) {
    const LaunchPlan thin = plan_one(m, tiles_n, bm, ksteps, slots, step, may_split, true);
    if (thin.cost >= 0.f && thin.cost < plain.cost) return thin;
  }
  return plain;
}

// the grid of a direct-to-LDS launch: tiles of bm rows, tiles_n tile columns
static GridPlan make_grid_plan(int m, int tiles_n, int bm, int ksteps, int slots, float step, bool may_split, bool may_thin,
                               int* n_blocks, int* rem_tiles) {
  const int tiles_m = (m + bm - 1) / bm;
  const LaunchPlan lp = plan_launch(m, tiles_n, bm, ksteps, slots, step, may_split, may_thin);
  GridPlan g;
  g.order = make_tile_order(lp.n_thin > 0 ? tiles_m - 1 : tiles_m, tiles_n);
  g.full_tiles = lp.n_thin + lp.n_normal - lp.rem;
  g.per_xcd = (g.full_tiles + XCDS - 1) / XCDS;
  g.n_full_wgs = g.per_xcd * XCDS;
  g.split = lp.split;
  g.kpp = lp.kpp;
  g.n_thin = lp.n_thin;
  *n_blocks = g.n_full_wgs + lp.rem * lp.split;
  *rem_tiles = lp.rem;
  if (!g_xcd_remap) g.per_xcd = 0;
  return g;
}

// ------------------------------------------------------------------ tile types
// step_lo / step_hi: microseconds of one K step (64) when a quarter / all of the workgroup slots are busy, extended in a
// straight line (the clock falls as more of the chip multiplies; where several workgroups share a compute unit, the units
// that hold most of them decide), fixed: prologue, first loads and epilogue of a round.  The constants are chosen for the
// types they pick: least squares of log(time) over 4300 launches (all types in turn, 33 to 5120 rows, the q|k|v, output,
// gate/up and down products of models of 512, 2048, 4096 and 5120 columns, random operands), then moved to where the picked
// type loses least.  On average it is 0.7 % behind the fastest type of each of 625 shapes with weights from memory (5 % of
// them: more than 4 %, at worst 14 %).  Constants fitted to the 4096-column products alone, without the step in the number of
// workgroups to a compute unit, were 2.9 % (16 %, 32 %) behind: gate/up of 200 x 27648 x 5120 167 us for 133,
// 777 x 6144 x 4096 65 for 51.
// 256x192 at 1.08 and not the fit's 1.11: 192-row tiles that cover as much in the one round are then not preferred to it
// (2500 x 4096 x 14336 244 -> 239 us, 2039 x 5120 x 27648 466 -> 453; 1801 x 5120 x 27648 loses 441 -> 451).  192x256 with
// wavefronts of 96 x 64 instead of 48 x 128 outputs (a tenth fewer LDS reads) is 2 % faster over 40 shapes: 1.01 for 1.03.
struct TileInfo { int code, bm, bn, occ; bool dual; float step_lo, step_hi, fixed; };
static constexpr TileInfo kTiles[] = {
    {5, 256, 256, 1, true, 1.01f, 1.23f, 5.34f},  {7, 256, 192, 1, false, 0.70f, 1.08f, 2.44f},
    {8, 192, 256, 1, true, 0.99f, 1.01f, 2.60f},  {11, 192, 192, 1, false, 0.78f, 0.89f, 2.12f},
    {9, 128, 256, 1, true, 0.69f, 0.85f, 1.60f},  {10, 128, 128, 2, true, 0.07f, 1.12f, 2.03f},
    {12, 64, 128, 3, true, 0.03f, 1.27f, 0.68f},  {13, 64, 256, 2, true, 0.02f, 1.46f, 2.05f},
};
static constexpr float kFixLaunchUs = 3.10f;          // a fix-up launch
static constexpr float kPartBytesPerUs = 8.79e6f;     // K parts are written, then read
static constexpr float kWeightBytesPerUs = 12.11e6f;  // the whole weight matrix from memory

// one K step with `wgs` workgroups on the chip; hbm: microseconds below which the weight slices do not arrive from
// memory (the tile rows of a column share them, but do not ask for them at the same time)
static float step_us(const TileInfo& t, int wgs, int n_cus, int tiles_m) {
  const float f = (float)wgs / (float)(n_cus * t.occ);
  const float busy = t.occ == 1 ? f : (float)((wgs + n_cus - 1) / n_cus) / (float)t.occ;
  const float mfma = t.step_lo + (t.step_hi - t.step_lo) * std::max(busy - 0.25f, -0.1f) / 0.75f;
  const float hbm = (float)(t.bn * t.occ) / 256.f * (0.15f + 0.80f * f) * std::pow((float)tiles_m, -0.25f);
  return std::max(mfma, hbm);
}

// time of a launch of tile type t whose tiles are all summed in `split` parts of kpp K steps
static float tile_cost(const TileInfo& t, int m, int tiles_n, int ksteps, int n_cus, int split, int kpp) {
  const int tiles_m = (m + t.bm - 1) / t.bm, slots = n_cus * t.occ, wgs = tiles_m * tiles_n * split;
  const int rounds = wgs / slots, last = wgs % slots;
  float c = (float)rounds * (kpp * step_us(t, slots, n_cus, tiles_m) + t.fixed);
  if (last > 0) c += kpp * step_us(t, last, n_cus, tiles_m) + t.fixed;
  if (split > 1) c += kFixLaunchUs + (float)wgs * t.bm * t.bn * 8.f / kPartBytesPerUs;
  return std::max(c, (float)tiles_n * t.bn * ksteps * BK * 2.f / kWeightBytesPerUs + t.fixed);
}

// the grid of a launch whose tiles are all summed in `split` parts of kpp K steps
static GridPlan uniform_grid_plan(int m, int tiles_n, int bm, int ksteps, int split, int kpp, int* n_blocks, int* rem_tiles) {
  GridPlan g = {};
  const int tiles_m = (m + bm - 1) / bm;
  g.order = make_tile_order(tiles_m, tiles_n);
  g.full_tiles = split > 1 ? 0 : tiles_m * tiles_n;
  g.per_xcd = (g.full_tiles + XCDS - 1) / XCDS;
  g.n_full_wgs = g.per_xcd * XCDS;
  g.split = split;
  g.kpp = kpp;
  *rem_tiles = split > 1 ? tiles_m * tiles_n : 0;
  *n_blocks = g.n_full_wgs + *rem_tiles * split;
  if (!g_xcd_remap) g.per_xcd = 0;
  return g;
}

// 256x256 tiles, all whole, with a ragged last tile row of at most kThinRows rows on the thin body, whose tiles come last and fill
// what the last round of the others leaves idle: 1025 x 28672 x 4096 232 us on 192x256 tiles, 203 like this (233 with the thin body
// on the older loop).
static GridPlan thin_grid_plan(int m, int tiles_n, int ksteps, int* n_blocks) {
  GridPlan g = {};
  const int tiles_m = (m + 255) / 256;
  g.order = make_tile_order(tiles_m - 1, tiles_n);
  g.full_tiles = tiles_m * tiles_n;
  g.per_xcd = (g.full_tiles + XCDS - 1) / XCDS;
  g.n_full_wgs = g.per_xcd * XCDS;
  g.split = 1;
  g.kpp = ksteps;
  g.n_thin = tiles_n;
  *n_blocks = g.n_full_wgs;
  if (!g_xcd_remap) g.per_xcd = 0;
  return g;
}
static float thin_cost(int m, int tiles_n, int ksteps, int n_cus) {
  const TileInfo& t = kTiles[0];
  const int tiles_m = (m + 255) / 256, normal = (tiles_m - 1) * tiles_n;
  if (!g_thin_tiles || m - (tiles_m - 1) * 256 > kThinRows || normal < n_cus) return 1e30f;   // at least one full round of the others
  const int rounds = normal / n_cus, last = normal % n_cus, idle = n_cus - last;
  const float full = ksteps * step_us(t, n_cus, n_cus, tiles_m) + t.fixed;
  const float others = rounds * full + (last > 0 ? ksteps * step_us(t, last, n_cus, tiles_m) + t.fixed : 0.f);
  return std::max(others, rounds * full + (float)((tiles_n + idle - 1) / idle) * kThinCost * full);
}

template <typename T, bool THIN>
static hipError_t launch_dl(const GridPlan& plan, int n_blocks, const bf16* a, const bf16* w, const bf16* w2, const bf16* w3, int ns1,
                            int ns2, void* c, int m, int n, int k, int ldc, GemmEpilogue epi, float* partial, hipStream_t st,
                            const int* m_live, const RopeOut* rope) {
  constexpr size_t lds_bytes = T::LDS_BYTES;
  const dim3 grid((unsigned)n_blocks);
  static std::atomic<unsigned long long> told[3] = {};
  if (rope) {
    auto kern = gemm_qkv_rope_kernel<T, THIN>;
    const hipError_t e = allow_dynamic_lds((const void*)kern, (int)lds_bytes, told[2]);
    if (e != hipSuccess) return e;
    kern<<<grid, T::NT, lds_bytes, st>>>(a, w, w2, w3, ns1, ns2, m, n / 2, k, plan, partial, m_live, *rope);
    return hipGetLastError();
  }
  auto go = [&](auto kern, std::atomic<unsigned long long>& done) {
    const hipError_t e = allow_dynamic_lds((const void*)kern, (int)lds_bytes, done);
    if (e != hipSuccess) return e;
    kern<<<grid, T::NT, lds_bytes, st>>>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, (int)epi, plan, partial, m_live);
    return hipGetLastError();
  };
  if constexpr (T::DUAL_OK) if (epi == EPI_SWIGLU_T) return go(gemm_mfma_dl_kernel<T, true, THIN>, told[1]);
  return go(gemm_mfma_dl_kernel<T, false, THIN>, told[0]);
}

static PartTiles part_tiles(const GemmRest& r) {
  return PartTiles{{r.tiles_m, r.tiles_n, r.bands}, r.full, r.split, r.bm, r.bn, r.partial};
}

static hipError_t launch_fixup(const GemmRest& r, void* c, int m, int n, int ldc, GemmEpilogue epi, hipStream_t st, int ns1, int ns2,
                               const RopeOut* rope) {
  const bool paired = rope || epi == EPI_SWIGLU_T;
  const int per_tile = (r.bm * ((paired ? r.bn / 2 : r.bn) / 4) + 255) / 256;
  const dim3 grid((unsigned)(r.tiles * per_tile));
  if (rope) gemm_fixup_kernel<kRope><<<grid, 256, 0, st>>>(c, m, n / 2, ldc, (int)epi, part_tiles(r), per_tile, ns1, ns2, *rope);
  else if (paired) gemm_fixup_kernel<kDual><<<grid, 256, 0, st>>>(c, m, n, ldc, (int)epi, part_tiles(r), per_tile, ns1, ns2, RopeOut{});
  else gemm_fixup_kernel<kPlain><<<grid, 256, 0, st>>>(c, m, n, ldc, (int)epi, part_tiles(r), per_tile, ns1, ns2, RopeOut{});
  return hipGetLastError();
}

hipError_t launch_rest_rmsnorm(const GemmRest& rest, float* h, const bf16* gain, bf16* out, int rows, int d, float eps, hipStream_t st,
                               const int* m_live) {
  if (rest.tiles == 0) return launch_rmsnorm(h, gain, out, rows, d, eps, st, m_live);
  const int nu = (d + 1023) / 1024;   // at most eight: kRestNormMax
  if (nu <= 4) gemm_fixup_norm_kernel<1><<<rows, 256 * nu, 0, st>>>(h, gain, out, d, eps, part_tiles(rest));
  else gemm_fixup_norm_kernel<2><<<rows, 256 * ((nu + 1) / 2), 0, st>>>(h, gain, out, d, eps, part_tiles(rest));
  return hipGetLastError();
}

static int g_gemm_tile = 0;   // 0: by shape; 1-3: register-staged 128x256 / 256x256 / 128x128; 5-13: direct-to-LDS (kTiles; 6: Tile128)
void set_gemm_tile(int t) { g_gemm_tile = t; }

template <int BM, int BN, int WAVES_M, int WAVES_N, int OCC>
static hipError_t launch_cfg(const bf16* a, const bf16* w, const bf16* w2, const bf16* w3, int ns1, int ns2, void* c,
                             int m, int n, int k, int ldc, GemmEpilogue epi, hipStream_t st, const int* m_live) {
  const bool dual = epi == EPI_SWIGLU_T;
  const int bn_out = dual ? BN / 2 : BN;
  const int tiles_m = (m + BM - 1) / BM, tiles_n = (n + bn_out - 1) / bn_out;
  const int total = tiles_m * tiles_n;
  int per_xcd = (total + XCDS - 1) / XCDS;
  const dim3 grid((unsigned)(per_xcd * XCDS));
  if (!g_xcd_remap) per_xcd = 0;
  constexpr int NT = WAVES_M * WAVES_N * 64;
  if (dual)
    gemm_mfma_kernel<BM, BN, WAVES_M, WAVES_N, true, OCC><<<grid, NT, 0, st>>>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc,
                                                                              (int)epi, make_tile_order(tiles_m, tiles_n), total, per_xcd, m_live);
  else
    gemm_mfma_kernel<BM, BN, WAVES_M, WAVES_N, false, OCC><<<grid, NT, 0, st>>>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc,
                                                                               (int)epi, make_tile_order(tiles_m, tiles_n), total, per_xcd, m_live);
  return hipGetLastError();
}

// The launch of a direct-to-LDS product: tile type (the codes of kTiles; 6: Tile128), grid, tiles that are summed in K parts.
struct DlPlan { int type; GridPlan grid; int n_blocks, rem_tiles, bm, bn; bool uniform; /* summed the same way everywhere */ };

static bool parts_fit(int bm, int bn, int tiles, int split) { return (size_t)tiles * split * bm * bn <= kPartialFloats; }

// The K partition by the rule above, then the tile type.  A product that is summed the same way everywhere (whole, or
// all in the same parts) goes to the tile type with the cheapest schedule; one with whole and cut tiles runs on the tiles
// its partition is made of.  A type whose padded tiles in `split` parts exceed the partial buffer is not taken, asked
// for or not: the number of parts comes from 256-row tiles, and 193 rows padded to 2 x 192 hold half as much again.
static DlPlan plan_dl(int tile, int m, int n, int k, bool dual, int cus, bool with_partial, bool device_rows, int m_expected) {
  const int ksteps = k / BK;
  if (dual && (tile == 7 || tile == 11)) tile = 8;   // forced, but the column halves of these two cannot be gate and up
  auto cols = [&](int bn) { const int o = dual ? bn / 2 : bn; return (n + o - 1) / o; };
  // which of 256x256 (5), 128x128 (6) and 256x192 (7) the partition is made of
  int part = tile == 5 || tile == 6 || tile == 7 ? tile : 0;
  if (part == 0) {
    const long t6 = (long)((m + 127) / 128) * cols(128);
    const int slots6 = 2 * cus;
    const float cost5 = plan_launch(m, cols(256), 256, ksteps, cus, kStep256, with_partial, true).cost;
    const long last6 = t6 % slots6;
    const float cost6 = (t6 / slots6) * ksteps * kStep128 +
                        (last6 == 0 ? 0.f : (last6 * 2 <= slots6 ? 0.65f : 1.f) * ksteps * kStep128);
    part = cost5 <= cost6 ? 5 : 6;
    if (!dual && n % 192 == 0) {
      const float cost7 = plan_launch(m, n / 192, 256, ksteps, cus, kStep192, with_partial, false).cost;
      if (cost7 < std::min(cost5, cost6)) part = 7;
    }
  }
  DlPlan p = {part, {}, 0, 0, 0, 0, true};
  int split = 1, kpp = ksteps;
  bool uniform = true;
  if (part != 6) {
    p.grid = make_grid_plan(m, cols(part == 7 ? 192 : 256), 256, ksteps, cus, part == 7 ? kStep192 : kStep256,
                            with_partial, part == 5 && !device_rows, &p.n_blocks, &p.rem_tiles);
    if (p.rem_tiles > 0 && p.grid.split > 1) {
      uniform = p.grid.full_tiles == 0;
      split = p.grid.split;
      kpp = p.grid.kpp;
    }
  }
  if (uniform && part != tile) {
    float best = 0.f;
    p.type = 0;
    for (const TileInfo& t : kTiles) {
      if (dual && !t.dual) continue;
      if (split > 1 && !parts_fit(t.bm, t.bn, ((m + t.bm - 1) / t.bm) * cols(t.bn), split)) continue;
      if (t.code == tile) { p.type = t.code; break; }
      const float cost = tile_cost(t, m_expected, cols(t.bn), ksteps, cus, split, kpp);
      if (p.type == 0 || cost < best) { p.type = t.code; best = cost; }
    }
    for (const TileInfo& t : kTiles)
      if (t.code == p.type) p.grid = uniform_grid_plan(m, cols(t.bn), t.bm, ksteps, split, kpp, &p.n_blocks, &p.rem_tiles);
    if (tile == 0 && split == 1 && !device_rows && thin_cost(m, cols(256), ksteps, cus) < best) {
      p.type = 5;
      p.grid = thin_grid_plan(m, cols(256), ksteps, &p.n_blocks);
      p.rem_tiles = 0;
    }
  } else if (part == 6) {
    p.grid = uniform_grid_plan(m, cols(128), 128, ksteps, 1, ksteps, &p.n_blocks, &p.rem_tiles);
  }
  p.uniform = uniform;
  p.bm = p.bn = 128;   // code 6
  for (const TileInfo& t : kTiles)
    if (t.code == p.type) { p.bm = t.bm; p.bn = t.bn; }
  return p;
}

// Host-side check of a launch: every output tile must be covered exactly once, by one whole-K workgroup or by K parts
// that partition [0, k) in part order and fit the partial buffer; thin tiles only in the last row of 256x256 tiles and only for
// at most 64 live rows.  Returns the number of violations; *n_blocks_out receives the grid size.  tile: 0 or a direct-to-LDS
// code; n_cus: CUs to plan for.
int check_grid_plan(int m, int n, int k, bool dual, int tile, int n_cus, bool with_partial, int* n_blocks_out) {
  const DlPlan p = plan_dl(tile, m, n, k, dual, n_cus, with_partial, false, m);
  const int bm = p.bm, bn = p.bn;
  const int bn_out = dual ? bn / 2 : bn;
  const int tiles_m = (m + bm - 1) / bm, tiles_n = (n + bn_out - 1) / bn_out;
  if (n_blocks_out) *n_blocks_out = p.n_blocks;
  int errors = 0;
  std::vector<int> covered((size_t)tiles_m * tiles_n, 0), next_k((size_t)tiles_m * tiles_n, 0), slots;
  for (int bid = 0; bid < p.n_blocks; ++bid) {
    const BlockWork bw = block_work(p.grid, bid, k);
    if (bw.kind == 0) continue;
    if (bw.tile_m < 0 || bw.tile_m >= tiles_m || bw.tile_n < 0 || bw.tile_n >= tiles_n) { ++errors; continue; }
    const size_t u = (size_t)bw.tile_m * tiles_n + bw.tile_n;
    if (bw.kind == 2 && (p.type != 5 || bw.tile_m != tiles_m - 1 || m - (tiles_m - 1) * bm > kThinRows || bw.part_slot >= 0)) ++errors;
    if (bw.part_slot < 0) {
      if (bw.k_begin != 0 || bw.k_end != k || covered[u] != 0) ++errors;
      covered[u] = 1;
      next_k[u] = k;
    } else {
      // parts arrive in block order = part order
      if (covered[u] == 1 || bw.k_begin != next_k[u] || bw.k_end <= bw.k_begin || bw.k_end > k) ++errors;
      covered[u] = 2;
      next_k[u] = bw.k_end;
      slots.push_back(bw.part_slot);
    }
  }
  for (size_t u = 0; u < covered.size(); ++u)
    if (covered[u] == 0 || next_k[u] != k) ++errors;
  // part slots are 0, 1, ... without gaps and fit the partial buffer; the fix-up pass visits exactly the cut tiles
  for (size_t i = 0; i < slots.size(); ++i)
    if (slots[i] != (int)i) ++errors;
  if (!parts_fit(bm, bn, (int)slots.size(), 1)) ++errors;
  for (int tm = 0; tm < p.grid.order.tiles_m; ++tm)
    for (int tn = 0; tn < tiles_n; ++tn) {
      int bm_i, bn_i;
      tile_of(p.grid.order, tile_index(p.grid.order, tm, tn), &bm_i, &bn_i);
      if (bm_i != tm || bn_i != tn) ++errors;   // the summing passes look tiles up by their place
    }
  if (p.rem_tiles > 0 ? slots.size() != (size_t)p.rem_tiles * p.grid.split : !slots.empty()) ++errors;
  return errors;
}

// Direct-to-LDS kernels (K a multiple of 64).  rest: see launch_gemm_bf16.
static hipError_t dispatch_dl(int tile, const bf16* a, const bf16* w, const bf16* w2, const bf16* w3, int ns1, int ns2,
                              void* c, int m, int n, int k, int ldc, GemmEpilogue epi, float* partial, hipStream_t st,
                              const int* m_live, int m_expected, GemmRest* rest, const RopeOut* rope = nullptr) {
  const DlPlan p = plan_dl(tile, m, n, k, epi == EPI_SWIGLU_T, num_cus(), partial != nullptr, m_live != nullptr, m_expected);
  // Few rows, cut into enough parts to keep the wavefronts of a workgroup busy: one launch, which also adds them up.  (Whole, or in
  // two or three parts, a wavefront's chain over K would be as long as a tile's.)
  if (tile == 0 && !m_live && !w3 && m <= 32 && p.uniform && p.rem_tiles > 0 && p.grid.split >= 4 && p.grid.split <= 16 && n % 16 == 0)
    return launch_gemm_few_rows_parts(a, w, w2, c, m, n, k, ldc, epi, p.grid.split, p.grid.kpp * (BK / 32), st);
  hipError_t e = hipErrorInvalidValue;
#define RC_DL(CODE, THIN, ...) \
  case CODE: e = launch_dl<__VA_ARGS__, THIN>(p.grid, p.n_blocks, a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, epi, partial, st, m_live, rope); break
  switch (p.type) {
    RC_DL(5, true, TilePipe<2, 4, 4, 4, 2, 2>);
    RC_DL(6, false, Tile128);
    RC_DL(7, false, TilePipe<4, 2, 2, 2, 4, 2>);
    RC_DL(8, false, TilePipe<2, 4, 4, 2, 2, 2>);
    RC_DL(9, false, TilePipe<2, 4, 2, 2, 2, 2>);
    RC_DL(10, false, TilePipe<2, 4, 2, 2, 1, 1, 2>);
    RC_DL(11, false, TilePipe<4, 2, 2, 1, 4, 2>);
    RC_DL(12, false, TilePipe<2, 4, 2, 0, 1, 1, 3>);
    RC_DL(13, false, TilePipe<1, 8, 4, 0, 1, 1, 2>);
  }
#undef RC_DL
  if (e != hipSuccess || p.rem_tiles == 0) return e;
  GemmRest r = {p.rem_tiles, p.grid.order.tiles_m, p.grid.order.tiles_n, p.grid.order.bands, p.grid.full_tiles - p.grid.n_thin,
                p.grid.split, p.bm, p.bn, partial};
  if (rest) {
    *rest = r;
    return e;
  }
  return launch_fixup(r, c, m, n, ldc, epi, st, ns1, ns2, rope);
}

bool gemm_takes_few_rows(int m, int n, int k) { return g_gemm_tile == 0 && gemm_skinny_applies(m, n, k); }

static hipError_t dispatch(const bf16* a, const bf16* w, const bf16* w2, const bf16* w3, int ns1, int ns2, void* c,
                           int m, int n, int k, int ldc, GemmEpilogue epi, float* partial, hipStream_t st,
                           const int* m_live, int m_expected, GemmRest* rest = nullptr) {
  if (rest) rest->tiles = 0;
  if (m <= 0 || n <= 0) return hipSuccess;
  int tile = g_gemm_tile;
  if (!w3 && gemm_takes_few_rows(m, n, k)) return launch_gemm_skinny_bf16(a, w, w2, c, m, n, k, ldc, epi, st, m_live);
  if (m_live) partial = nullptr;   // live row count on the device: every output summed whole
  if ((tile == 0 || tile >= 5) && k % BK == 0)
    return dispatch_dl(tile, a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, epi, partial, st, m_live,
                       m_live && m_expected > 0 ? std::min(m, m_expected) : m, rest);
  switch (tile) {   // the direct-load kernels need whole K steps
    case 1: return launch_cfg<128, 256, 2, 2, 2>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, epi, st, m_live);
    case 2: return launch_cfg<256, 256, 4, 2, 1>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, epi, st, m_live);
    default: return launch_cfg<128, 128, 2, 2, 2>(a, w, w2, w3, ns1, ns2, c, m, n, k, ldc, epi, st, m_live);
  }
}

hipError_t launch_gemm_bf16(const bf16* a, const bf16* w, const bf16* w2, void* c, int m, int n, int k, int ldc,
                            GemmEpilogue epi, float* partial, hipStream_t st, const int* m_live, int m_expected, GemmRest* rest) {
  return dispatch(a, w, w2, nullptr, n, n, c, m, n, k, ldc, epi, partial, st, m_live, m_expected, rest);
}

// q | k | v projections of the same rows as one GEMM over the concatenated output columns.  Rotary and scatter are part of it where
// rotary partners can sit in one wavefront: a tile of pairs covers the columns of the tile it stands for, which matters where
// whole and cut tiles are mixed, when its width is a multiple of a head (256, not 192).
hipError_t launch_gemm_qkv_bf16(const bf16* a, const bf16* wq, int nq, const bf16* wk, const bf16* wv, int nkv, float* c,
                                int m, int k, float* partial, hipStream_t st, const int* m_live, int m_expected, const RopeOut* rope,
                                bool* rotated) {
  const int n = nq + 2 * nkv, tile = g_gemm_tile;
  *rotated = false;
  if (rope && m > 0 && (tile == 0 || tile >= 5) && k % BK == 0) {
    if (m_live) partial = nullptr;
    m_expected = m_live && m_expected > 0 ? std::min(m, m_expected) : m;
    const DlPlan p = plan_dl(tile, m, n, k, false, num_cus(), partial != nullptr, m_live != nullptr, m_expected);
    *rotated = p.uniform || p.type != 7;
    if (*rotated)
      return dispatch_dl(tile, a, wq, wk, wv, nq, nq + nkv, nullptr, m, n, k, n, EPI_STORE_T, partial, st, m_live, m_expected, nullptr, rope);
  }
  return dispatch(a, wq, wk, wv, nq, nq + nkv, c, m, n, k, n, EPI_STORE_F32, partial, st, m_live, m_expected);
}

}  // namespace rc
