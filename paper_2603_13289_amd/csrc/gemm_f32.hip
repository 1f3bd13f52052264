// Projection GEMM of the float configuration: C[M][N] = A[M][K] * W[N][K]^T on v_mfma_f32_16x16x4_f32 (exact float
// products and sums), operands straight from global memory.
//
// Both operands are K-contiguous.  A lane loads 16 bytes (4 consecutive k) of row lane % 16 at k offset 4 (lane / 16), so
// one load of each operand feeds four matrix instructions; instruction c multiplies the k's 4 (lane / 16) + c.
//
// Float models are small (hundreds of rows and columns), where a launch costs what it takes to start it, to fetch its
// operands once and to drain: the small variant gives every 16 x 16 output block to a workgroup of four wavefronts that
// share its K range, so that thousands of wavefronts have a few loads each, all in flight.  Products with enough 64 x 64
// tiles to fill the chip use the big variant (32 x 32 or 64 x 64 per wavefront, whole K).
//
// What would be launches of their own around a product is done inside it: the RMS norm of the input rows (gain applied
// to the operand, 1 / rms to the finished sums), rotary + paged scatter behind the q|k|v projection, the gather of
// each request's last row before the LM head.  Measured in a call against a 64 x 64 vector-ALU tile (24 workgroups):
// 384 x 256 x 256 22.0 -> 4.7 us, 384 x 256 x 688 53.5 -> 6.5 us; an empty launch takes about 4 us.
#include "common.h"

namespace rc {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4m;

__device__ inline float silu_f(float x) { return x / (1.0f + __expf(-x)); }

// one GEMM; `pair`: the second column block of a workgroup is not the next one but (SwiGLU) the same columns of w2 or
// (q|k|v + rotary) the rotary partners half a head further on
struct F32Gemm {
  const float *a, *w, *w2, *w3;
  int ns1, ns2;              // columns below ns1 come from w, below ns2 from w2, the rest from w3
  const float* gain;         // non-null: A is RMS-normalised with this gain
  float eps;
  const ReqTable* last_of;   // non-null: row b of A is the last live row of request b
  float* c;
  int m, n, k, ldc, epi;
  const int* m_live;
};

__device__ inline const float* f32_a_row(const F32Gemm& g, int r, int m) {
  r = min(r, m - 1);
  if (g.last_of) {
    const ReqDev& rq = g.last_of->r[r];
    return rq.n_rows > 0 ? g.a + (size_t)(rq.row_base + rq.n_rows - 1) * g.k : nullptr;
  }
  return g.a + (size_t)r * g.k;
}

__device__ inline const float* f32_w_row(const F32Gemm& g, int col) {
  col = min(col, g.n - 1);
  return col < g.ns1 ? g.w + (size_t)col * g.k : (col < g.ns2 ? g.w2 + (size_t)(col - g.ns1) * g.k : g.w3 + (size_t)(col - g.ns2) * g.k);
}

__device__ inline f32x4m load_k4(const float* row, int k0, int k) {
  return row && k0 < k ? *reinterpret_cast<const f32x4m*>(row + k0) : f32x4m{0.f, 0.f, 0.f, 0.f};
}

// The sums of a 16 x 16 block (two with `w_hi`): lane holds row lane % 16 of A, columns 4 (lane / 16) + 0..3; all four
// wavefronts return the total.  With a gain, *r is the row's 1 / rms.
constexpr int kF32Ahead = 4;
// behind_loads: runs once, with the first loads under way.
template <bool PAIR, typename F>
__device__ __forceinline__ void f32_block(const F32Gemm& g, const float* arow, const float* wrow, const float* wrow_hi,
                                          f32x4m* lo, f32x4m* hi, F&& behind_loads) {
  __shared__ f32x4m part[2][4][64];
  __shared__ float part_ss[4][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kq = lane >> 4;
  f32x4m c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
  float ss = 0.f;
  const int nt = (g.k + 15) / 16;
  for (int t0 = wave; t0 < nt; t0 += 4 * kF32Ahead) {
    f32x4m fa[kF32Ahead], fw[kF32Ahead], fh[kF32Ahead], fg[kF32Ahead];
#pragma unroll
    for (int u = 0; u < kF32Ahead; ++u) {
      const int k0 = 16 * (t0 + 4 * u) + 4 * kq;     // beyond K: zeros
      fa[u] = load_k4(arow, k0, g.k);
      fw[u] = load_k4(wrow, k0, g.k);
      if (PAIR) fh[u] = load_k4(wrow_hi, k0, g.k);
      if (g.gain) fg[u] = load_k4(g.gain, k0, g.k);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (t0 == wave) behind_loads();   // uniform
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kF32Ahead; ++u) {
      if (g.gain) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ss = fmaf(fa[u][e], fa[u][e], ss);
          fa[u][e] *= fg[u][e];
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[u][e], fa[u][e], c0, 0, 0, 0);
        if (PAIR) c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(fh[u][e], fa[u][e], c1, 0, 0, 0);
      }
    }
  }
  part[0][wave][lane] = c0;
  if (PAIR) part[1][wave][lane] = c1;
  if (g.gain) {
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    if (kq == 0) part_ss[wave][lane] = ss;
  }
  __syncthreads();
  *lo = ((part[0][0][lane] + part[0][1][lane]) + part[0][2][lane]) + part[0][3][lane];
  if (PAIR) *hi = ((part[1][0][lane] + part[1][1][lane]) + part[1][2][lane]) + part[1][3][lane];
  if (g.gain) {
    const int r = lane & 15;
    const float sq = ((part_ss[0][r] + part_ss[1][r]) + part_ss[2][r]) + part_ss[3][r];
    const float inv = 1.0f / sqrtf(sq / (float)g.k + g.eps);
    *lo *= inv;
    if (PAIR) *hi *= inv;
  }
}

__device__ inline void f32_store(const F32Gemm& g, int row, int col, f32x4m v, int m) {
  if (row >= m) return;
  float* dst = g.c + (size_t)row * g.ldc + col;
  if (col + 3 < g.n && (g.ldc & 3) == 0 && (reinterpret_cast<size_t>(g.c) & 15) == 0) {
    f32x4m* d4 = reinterpret_cast<f32x4m*>(dst);
    *d4 = g.epi == EPI_ADD_F32 ? *d4 + v : v;
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (col + e < g.n) dst[e] = g.epi == EPI_ADD_F32 ? dst[e] + v[e] : v[e];
}

template <bool DUAL>
__global__ void __launch_bounds__(256)
gemm_f32_small_kernel(F32Gemm g) {
  const int m = live_count(g.m, g.m_live), m0 = blockIdx.y * 16, n0 = blockIdx.x * 16;
  if (m0 >= m) return;   // uniform: the grid may be sized for an upper bound of the row count
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15;
  const float* wrow = DUAL ? g.w + (size_t)min(n0 + r, g.n - 1) * g.k : f32_w_row(g, n0 + r);
  f32x4m lo, hi;
  f32_block<DUAL>(g, f32_a_row(g, m0 + r, m), wrow, DUAL ? g.w2 + (size_t)min(n0 + r, g.n - 1) * g.k : nullptr, &lo, &hi, [] {});
  if (wave != 0) return;
  if (DUAL) {
#pragma unroll
    for (int e = 0; e < 4; ++e) lo[e] = silu_f(lo[e]) * hi[e];
  }
  f32_store(g, m0 + r, n0 + 4 * (lane >> 4), lo, m);
}

// q|k|v projection of 16 rows x (16 rotary pairs, or 2 x 16 value elements), rotated and written where it belongs:
// queries to q_out, keys and values to the paged cache (keys also un-rotated to k_pre_pool, if there is one)
struct F32Rope {
  const int *row_pos, *row_req;
  const ReqTable* table;
  const float2* rope_tab;
  float *q_out, *k_pool, *v_pool, *k_pre_pool;
  KvGeom geom;
  int n_q_heads;
};

// EARLY: where the row goes and its angles, a chain of three reads, are asked for ahead of the operands and behind them and not behind
// the product: 7.4 -> 6.8 us a launch of 384 x 512 x 256.  They hold twelve registers over it (108 instead of 96), which costs the fifth
// workgroup of a compute unit: takes_early.
template <bool EARLY>
__global__ void __launch_bounds__(256)
gemm_f32_rope_kernel(F32Gemm g, F32Rope p) {
  const int m = live_count(g.m, g.m_live), m0 = blockIdx.y * 16;
  if (m0 >= m) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15;
  const int dh = p.geom.head_dim, half = dh / 2, per_head = half / 16;
  const int head = (int)blockIdx.x / per_head, c0 = ((int)blockIdx.x % per_head) * 16;
  f32x4m lo, hi;
  const int row = m0 + r, i = c0 + 4 * (lane >> 4), n_kv = p.geom.n_kv_heads;
  const bool finishes = wave == 0 && row < m;
  int pos = 0, rr = 0;
  size_t off = 0;
  f32x4m cs01 = {0.f, 0.f, 0.f, 0.f}, cs23 = cs01;
  auto find_row = [&] {
    if (!finishes) return;
    pos = p.row_pos[row];
    rr = p.row_req[row];
  };
  auto find_place = [&] {
    if (!finishes) return;
    if (head < p.n_q_heads + n_kv) {
      const f32x4m* cs = reinterpret_cast<const f32x4m*>(p.rope_tab + (size_t)pos * half + i);
      cs01 = cs[0];
      cs23 = cs[1];
    }
    if (head >= p.n_q_heads)
      off = kv_row_offset(p.geom, p.table->r[rr & kRowReqMask].dst_seq, pos, head < p.n_q_heads + n_kv ? head - p.n_q_heads : head - p.n_q_heads - n_kv);
  };
  if constexpr (EARLY) find_row();
  f32_block<true>(g, f32_a_row(g, m0 + r, m), f32_w_row(g, head * dh + c0 + r), f32_w_row(g, head * dh + half + c0 + r), &lo, &hi, [&] {
    if constexpr (EARLY) find_place();
  });
  if constexpr (!EARLY) {
    find_row();
    find_place();
  }
  if (!finishes) return;
  const bool write_cache = (rr & kRowNoCacheWrite) == 0;
  if (head >= p.n_q_heads && !write_cache) return;
  if (head >= p.n_q_heads + n_kv) {
    *reinterpret_cast<f32x4m*>(p.v_pool + off + i) = lo;
    *reinterpret_cast<f32x4m*>(p.v_pool + off + half + i) = hi;
    return;
  }
  f32x4m olo, ohi;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float c = e < 2 ? cs01[2 * e] : cs23[2 * e - 4], sn = e < 2 ? cs01[2 * e + 1] : cs23[2 * e - 3];
    olo[e] = lo[e] * c - hi[e] * sn;
    ohi[e] = hi[e] * c + lo[e] * sn;
  }
  if (head < p.n_q_heads) {
    float* o = p.q_out + ((size_t)row * p.n_q_heads + head) * dh;
    *reinterpret_cast<f32x4m*>(o + i) = olo;
    *reinterpret_cast<f32x4m*>(o + half + i) = ohi;
    return;
  }
  *reinterpret_cast<f32x4m*>(p.k_pool + off + i) = olo;
  *reinterpret_cast<f32x4m*>(p.k_pool + off + half + i) = ohi;
  if (p.k_pre_pool) {
    *reinterpret_cast<f32x4m*>(p.k_pre_pool + off + i) = lo;
    *reinterpret_cast<f32x4m*>(p.k_pre_pool + off + half + i) = hi;
  }
}

// 32 F x 32 F outputs per workgroup (DUAL: half as many columns of each matrix), 16 F x 16 F per wavefront, one step of loads
// ahead.  Bound by the operands' way from the L2 and L1, so products with enough tiles take F = 4, which loads half as much
// per output: 4096 x 4096 x 4096 1880 -> 1267 us, 5120 x 4096 x 1024 590 -> 411 us against F = 2 (108 TFLOP/s; a 64 x 64
// vector-ALU tile with its operands in LDS: 1723 and 537 us).
template <bool DUAL, int F>
__global__ void __launch_bounds__(256)
gemm_f32_big_kernel(F32Gemm g) {
  constexpr int BM = 32 * F, BN = DUAL ? 16 * F : 32 * F;
  const int m = live_count(g.m, g.m_live), m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  if (m0 >= m) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, kq = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const float *arow[F], *wrow[F];   // DUAL: the first half of the column blocks is the gate, the second the up projection
#pragma unroll
  for (int i = 0; i < F; ++i) {
    arow[i] = f32_a_row(g, m0 + (wm * F + i) * 16 + r, m);
    if (DUAL) wrow[i] = (i >= F / 2 ? g.w2 : g.w) + (size_t)min(n0 + (wn * (F / 2) + i % (F / 2)) * 16 + r, g.n - 1) * g.k;
    else wrow[i] = f32_w_row(g, n0 + (wn * F + i) * 16 + r);
  }
  f32x4m acc[F][F] = {}, fa[F], fw[F], fg, na[F], nw[F], ng;
  float ss[F] = {};
  auto fetch = [&](int t) {
    const int k0 = 16 * t + 4 * kq;
#pragma unroll
    for (int i = 0; i < F; ++i) {
      na[i] = load_k4(arow[i], k0, g.k);
      nw[i] = load_k4(wrow[i], k0, g.k);
    }
    if (g.gain) ng = load_k4(g.gain, k0, g.k);
  };
  const int nt = (g.k + 15) / 16;
  fetch(0);
  for (int t = 0; t < nt; ++t) {
#pragma unroll
    for (int i = 0; i < F; ++i) { fa[i] = na[i]; fw[i] = nw[i]; }
    fg = ng;
    if (t + 1 < nt) fetch(t + 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float av[F];
#pragma unroll
      for (int i = 0; i < F; ++i) {
        av[i] = fa[i][e];
        if (g.gain) { ss[i] = fmaf(av[i], av[i], ss[i]); av[i] *= fg[e]; }
      }
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[j][e], av[i], acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < F; ++i) {
    if (g.gain) {
      float s = ss[i];
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      const float inv = 1.0f / sqrtf(s / (float)g.k + g.eps);
#pragma unroll
      for (int j = 0; j < F; ++j) acc[i][j] *= inv;
    }
    const int row = m0 + (wm * F + i) * 16 + r;
#pragma unroll
    for (int j = 0; j < (DUAL ? F / 2 : F); ++j) {
      const int col = n0 + (wn * (DUAL ? F / 2 : F) + j) * 16 + 4 * kq;
      f32x4m v = acc[i][j];
      if (DUAL) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = silu_f(acc[i][j][e]) * acc[i][j + F / 2][e];
      }
      f32_store(g, row, col, v, m);
    }
  }
}

template <int F>
static void launch_f32_big(const F32Gemm& g, hipStream_t st) {
  const bool dual = g.epi == EPI_SWIGLU_T;
  const int bn = dual ? 16 * F : 32 * F;
  const dim3 grid((unsigned)((g.n + bn - 1) / bn), (unsigned)((g.m + 32 * F - 1) / (32 * F)));
  if (dual) gemm_f32_big_kernel<true, F><<<grid, 256, 0, st>>>(g);
  else gemm_f32_big_kernel<false, F><<<grid, 256, 0, st>>>(g);
}

static hipError_t launch_f32(const F32Gemm& g, hipStream_t st) {
  if (g.m <= 0 || g.n <= 0) return hipSuccess;
  const bool dual = g.epi == EPI_SWIGLU_T;
  // output tiles of side x side (dual: of both matrices together)
  auto tiles = [&](long side) { const long bn = dual ? side / 2 : side; return ((g.m + side - 1) / side) * ((g.n + bn - 1) / bn); };
  // The large tile from two workgroups per compute unit on, with K from 1024 on from one (700 x 8192 x 688, 384 tiles: 118 us
  // against 101 with the 64 tile; 1000 x 4096 x 4096, 256 tiles: 363 against 474), if it adds at most a quarter of
  // padding to the 64 tile's (64 rows: two thirds slower).
  if (tiles(128) >= (g.k >= 1024 ? 256 : 512) && 16 * tiles(128) <= 5 * tiles(64)) {
    launch_f32_big<4>(g, st);
  } else if (tiles(64) >= 512) {   // two workgroups per compute unit
    launch_f32_big<2>(g, st);
  } else {
    const dim3 grid((unsigned)((g.n + 15) / 16), (unsigned)((g.m + 15) / 16));
    if (dual) gemm_f32_small_kernel<true><<<grid, 256, 0, st>>>(g);
    else gemm_f32_small_kernel<false><<<grid, 256, 0, st>>>(g);
  }
  return hipGetLastError();
}

hipError_t launch_gemm_f32(const float* a, const float* w, const float* w2, void* c, int m, int n, int k, int ldc,
                           GemmEpilogue epi, hipStream_t st, const int* m_live) {
  return launch_f32(F32Gemm{a, w, w2, nullptr, n, n, nullptr, 0.f, nullptr, (float*)c, m, n, k, ldc, (int)epi, m_live}, st);
}

hipError_t launch_gemm_f32_normed(const float* h, const float* gain, float eps, const ReqTable* last_of, const float* w,
                                  const float* w2, float* c, int m, int n, int k, GemmEpilogue epi, hipStream_t st, const int* m_live) {
  return launch_f32(F32Gemm{h, w, w2, nullptr, n, n, gain, eps, last_of, c, m, n, k, n, (int)epi, m_live}, st);
}

// The chain shows where the chip has room for all workgroups at once (four each to 256 compute units).  In a fuller launch other workgroups hide it
// and the fifth counts, the more the shorter the product: 512 columns of K = 256, 2048 / 4096 rows 20.6 / 35.2 us early, 19.2 / 31.0 late; 1024 of
// K = 512 54.9 / 101.6 and 54.0 / 100.2; 1536 of K = 1024 144.3 / 281.9 and 144.7 / 282.5, so long products stay with the early form.
static bool takes_early(long workgroups, int k) { return workgroups <= 1024 || k >= 1024; }

hipError_t launch_gemm_f32_qkv_rope(const float* h, const float* gain, float eps, const float* wq, const float* wk,
                                    const float* wv, int m, int k, const int* row_pos, const int* row_req,
                                    const ReqTable* table, const float2* rope_tab, float* q_out, float* k_pool, float* v_pool,
                                    float* k_pre_pool, KvGeom geom, int n_q_heads, hipStream_t st, const int* m_live) {
  if (m <= 0) return hipSuccess;
  const int nq = n_q_heads * geom.head_dim, nkv = geom.n_kv_heads * geom.head_dim, n = nq + 2 * nkv;
  const F32Gemm g = {h, wq, wk, wv, nq, nq + nkv, gain, eps, nullptr, nullptr, m, n, k, n, EPI_STORE_F32, m_live};
  const F32Rope p = {row_pos, row_req, table, rope_tab, q_out, k_pool, v_pool, k_pre_pool, geom, n_q_heads};
  const dim3 grid((unsigned)(n / 32), (unsigned)((m + 15) / 16));
  (takes_early((long)grid.x * grid.y, k) ? gemm_f32_rope_kernel<true> : gemm_f32_rope_kernel<false>)<<<grid, 256, 0, st>>>(g, p);
  return hipGetLastError();
}

}  // namespace rc
