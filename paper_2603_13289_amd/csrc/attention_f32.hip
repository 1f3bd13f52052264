// K6 for the float configuration: causal grouped-query attention of arbitrary query rows over a paged cache on
// v_mfma_f32_16x16x4_f32.
//
// A workgroup serves 16 query rows of one request and one query head; its eight (head size 128: four) wavefronts take
// every eighth (fourth) block of 16 keys, each with a running softmax of its own, and are merged through LDS at the end.
// Per key block a wavefront computes
//   S^T[key][q] = K[key][:] . Q[q][:]      lane holds query lane % 16, keys 4 (lane / 16) + 0..3
//   O^T[d][q]  += V^T[d][key] P[key][q]    P's operand is S^T's result register as it stands
// Bound by latency: float models have a few hundred keys, so the chain of one wavefront is a handful of blocks; the next block's keys
// and values are requested before the current one's softmax, and the page they are on a block before that, so that no load waits
// for a look-up.  Measured in a call, 384 rows x 4 heads of 64 x up to 384 keys: 146 us with one wavefront per (row, head) on the
// vector ALUs, 15.1 with values and their pages looked up in the block that uses them, 12.2 now (188 rows: 15.3 -> 12.8).
// GROUPED: a contiguous cache, or pages of 16, 32, 64, ... slots: the keys of a block lie one behind the other and its page is one scalar read.
// Other pages look up every key.  Two look-ups a block, one between the products and the softmax for the next keys and one ahead of the
// products for the values, are then the better chain: with both in one place 500 rows over 1000 keys on pages of 24 took 27.7 us instead
// of 25.9 (heads of 128: 53.5 instead of 41.1).  GROUPED there: 19.1 (29.0); one block of 16 keys 6.4 -> 6.0 since the kernels are two.
#include <climits>
#include <type_traits>

#include "common.h"

namespace rc {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4a;

template <int DH, bool GROUPED>
__global__ void __launch_bounds__(DH == 64 ? 512 : 256, DH == 64 ? 4 : 2)
attn_f32_kernel(const float* __restrict__ q, const int* __restrict__ row_pos, const ReqTable* __restrict__ table,
                int fixed_seq, int total_rows, const float* __restrict__ k_pool, const float* __restrict__ v_pool, KvGeom g,
                int n_q_heads, float* __restrict__ out) {
  constexpr int NB = DH / 16, NW = DH == 64 ? 8 : 4;   // wavefronts: what 32 KB of partial results allow
  __shared__ float lds_o[NW][DH][16];
  __shared__ float2 lds_ml[NW][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), qi = lane & 15, kq = lane >> 4;
  const int head = blockIdx.y, kvh = head / (n_q_heads / g.n_kv_heads);
  int r0 = blockIdx.x * 16, n_valid, seq = fixed_seq;
  if (table) {   // the tile-th group of 16 rows, counted request by request
    int tile = blockIdx.x, b = 0;
    for (; b < table->n_req; ++b) {
      const int t = (table->r[b].n_rows + 15) / 16;
      if (tile < t) break;
      tile -= t;
    }
    if (b == table->n_req) return;   // uniform: the grid is an upper bound
    r0 = table->r[b].row_base + tile * 16;
    n_valid = min(16, table->r[b].n_rows - tile * 16);
    seq = table->r[b].dst_seq;
  } else {
    n_valid = min(16, total_rows - r0);
  }
  const bool q_ok = qi < n_valid;
  const int own_pos = pos_in_cache(row_pos[r0 + min(qi, n_valid - 1)], g.last_pos);   // of every lane: under a condition it is waited for at once
  const int my_pos = q_ok ? own_pos : -1;
  int last_pos = my_pos, first_pos = q_ok ? my_pos : INT_MAX;   // the group's largest and smallest position
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    last_pos = max(last_pos, __shfl_xor(last_pos, o, 64));
    first_pos = min(first_pos, __shfl_xor(first_pos, o, 64));
  }
  const float scale = 1.4426950408889634f / sqrtf((float)DH);   // scores in log2 units
  const float* qrow = q + ((size_t)(r0 + (q_ok ? qi : 0)) * n_q_heads + head) * DH;
  f32x4a fq[NB], fk[NB], acc[NB];
  float fv[GROUPED ? 2 : 1][NB][4];   // V[key 4 kq + c][d]: the operand of instruction c, of this block and the next
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    fq[t] = q_ok ? *reinterpret_cast<const f32x4a*>(qrow + 16 * t + 4 * kq) * scale : f32x4a{0.f, 0.f, 0.f, 0.f};
    acc[t] = f32x4a{0.f, 0.f, 0.f, 0.f};
  }
  float m_run = -INFINITY, l_run = 0.f;
  last_pos = __builtin_amdgcn_readfirstlane(last_pos);
  const int n_blocks = last_pos / 16 + 1;
  // Keys past the last position repeat it.  A block's page is read a block ahead of the loads that hang on it.
  const bool contig = g.max_blocks == 1;
  const int32_t* const seq_table = g.block_table + (size_t)seq * g.max_blocks;
  auto page_of = [&](int kb) {
    return GROUPED ? seq_table[contig ? 0 : min(min(kb, n_blocks - 1) * 16 >> g.bs_shift, g.max_blocks - 1)] : 0;
  };
  auto offset_of = [&](int kb, int j, int page) -> size_t {   // of key j of the block
    if (!GROUPED) return kv_row_offset(g, seq, min(kb * 16 + j, last_pos), kvh);
    const int first = contig ? kb * 16 : kb * 16 & (g.block_size - 1);
    return (((size_t)min(max(page, 0), g.n_blocks - 1) * g.n_kv_heads + kvh) * g.block_size + first + min(j, last_pos - kb * 16)) * DH;
  };
  auto fetch_k = [&](int kb, int page) {
    const float* krow = k_pool + offset_of(kb, qi, page);
#pragma unroll
    for (int t = 0; t < NB; ++t) fk[t] = *reinterpret_cast<const f32x4a*>(krow + 16 * t + 4 * kq);
  };
  auto fetch_v = [&](auto buf, int kb, int page) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float* vrow = v_pool + offset_of(kb, 4 * kq + c, page) + qi;
#pragma unroll
      for (int t = 0; t < NB; ++t) fv[decltype(buf)::value][t][c] = vrow[16 * t];
    }
  };
  int page = 0;   // of the wavefront's next block
  const std::integral_constant<int, 0> buf0;
  const std::integral_constant<int, 1> buf1;
  if (wave < n_blocks) {
    const int first = page_of(wave);
    page = page_of(wave + NW);
    fetch_k(wave, first);
    if constexpr (GROUPED) fetch_v(buf0, wave, first);
  }
  auto block = [&](auto buf, auto other, int kb) {
    constexpr int B = decltype(buf)::value;
    const int page2 = page_of(kb + 2 * NW);
    if constexpr (!GROUPED) fetch_v(buf, kb, 0);
    f32x4a s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
    for (int t = 0; t < NB; t += 2)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(fk[t][c], fq[t][c], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(fk[t + 1][c], fq[t + 1][c], s1, 0, 0, 0);
      }
    if (kb + NW < n_blocks) {
      fetch_k(kb + NW, page);
      if constexpr (GROUPED) fetch_v(other, kb + NW, page);
    }
    page = page2;
    s0 += s1;
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (kb * 16 + 4 * kq + e > my_pos) s0[e] = -INFINITY;
      mx = fmaxf(mx, s0[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx), m_use = m_new == -INFINITY ? 0.f : m_new;
    const float corr = exp2f(m_run - m_use);
    float ps = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s0[e] = exp2f(s0[e] - m_use);
      ps += s0[e];
    }
    l_run = l_run * corr + ps;
    m_run = m_new;
    // Keys that only some rows of the group see have weight 0 for the others, and a value there that is not finite must not
    // reach them (0 x inf): such values (rare) leave the product and are added row by row to the rows that see them.
    // The test itself costs up to 2 % (2000 rows x 4 heads: 66.6 -> 67.7 us).
    bool odd = false;
    if (kb * 16 + 15 > first_pos) {
      float z = 0.f;
#pragma unroll
      for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) z = fmaf(fv[B][t][c], 0.f, z);
      odd = __any(z != z);
      if (odd) {
#pragma unroll
        for (int t = 0; t < NB; ++t)
#pragma unroll
          for (int c = 0; c < 4; ++c) fv[B][t][c] = isfinite(fv[B][t][c]) ? fv[B][t][c] : 0.f;
      }
    }
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      acc[t] *= corr;
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(fv[B][t][c], s0[c], acc[t], 0, 0, 0);
    }
    if (odd) {
#pragma unroll 1
      for (int j = 0; j < 16; ++j) {
        const int key = kb * 16 + j;
        const float mine = (j & 2) ? ((j & 1) ? s0[3] : s0[2]) : ((j & 1) ? s0[1] : s0[0]);
        const float p = __shfl(mine, qi + 16 * (j >> 2), 64);
        if (key > my_pos) continue;
        const float* vrow = v_pool + kv_row_offset(g, seq, key, kvh) + 4 * kq;
#pragma unroll
        for (int t = 0; t < NB; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (!isfinite(vrow[16 * t + e])) acc[t][e] += p * vrow[16 * t + e];
      }
    }
  };
  if constexpr (GROUPED) {
    for (int kb = wave; kb < n_blocks; kb += 2 * NW) {
      block(buf0, buf1, kb);
      if (kb + NW < n_blocks) block(buf1, buf0, kb + NW);
    }
  } else {
    for (int kb = wave; kb < n_blocks; kb += NW) block(buf0, buf0, kb);
  }
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if (kq == 0) lds_ml[wave][qi] = make_float2(m_run, l_run);
#pragma unroll
  for (int t = 0; t < NB; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) lds_o[wave][16 * t + 4 * kq + e][qi] = acc[t][e];
  __syncthreads();
  // NT / 16 threads per row, thread c of them the elements c, c + NT / 16, ...
  constexpr int NT = 64 * NW, PER = NT / 16;
  const int row = tid / PER;
  if (row >= n_valid) return;
  float m = -INFINITY, l = 0.f, f[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) m = fmaxf(m, lds_ml[w][row].x);
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    f[w] = exp2f(lds_ml[w][row].x - m);
    l += lds_ml[w][row].y * f[w];
  }
  float* orow = out + ((size_t)(r0 + row) * n_q_heads + head) * DH;
#pragma unroll
  for (int d0 = 0; d0 < DH; d0 += PER) {
    const int d = d0 + tid % PER;
    float o = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) o = fmaf(lds_o[w][d][row], f[w], o);
    orow[d] = o / l;
  }
}

template <>
hipError_t launch_attention<float>(const float* q, const int* row_pos, const int* row_req, const ReqTable* table,
                                   int fixed_seq, int total_rows, int total_tiles, const float* k_pool,
                                   const float* v_pool, KvGeom g, int n_q_heads, float* out, hipStream_t st) {
  (void)row_req;
  if (total_rows <= 0) return hipSuccess;
  // 16-row groups: at most two per query tile (32 rows) of the table
  const unsigned groups = table ? (unsigned)(2 * total_tiles) : (unsigned)((total_rows + 15) / 16);
  const dim3 grid(groups, (unsigned)n_q_heads);
  const bool grouped = g.max_blocks == 1 || g.bs_shift >= 4;   // measured both ways at the kernel
  auto* const kernel = g.head_dim == 64 ? (grouped ? attn_f32_kernel<64, true> : attn_f32_kernel<64, false>)
                                        : (grouped ? attn_f32_kernel<128, true> : attn_f32_kernel<128, false>);
  kernel<<<grid, g.head_dim == 64 ? 512 : 256, 0, st>>>(q, row_pos, table, fixed_seq, total_rows, k_pool, v_pool, g, n_q_heads, out);
  return hipGetLastError();
}

}  // namespace rc
