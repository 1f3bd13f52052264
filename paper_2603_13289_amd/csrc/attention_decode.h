// Attention of one query row per sequence (decoding): included by attention_mfma.hip, whose constants and partial-result
// layout it shares.
//
// Bound by reading K and V once.  The 32-row tile kernel computes 31 empty query rows per head and stages every tile through
// LDS behind a barrier: 125 us for 16 sequences of 1.3k-10k keys (377 MB of K/V, 8 KV heads), 27 us for one of 5k
// with its scores (each with its merge and the timing's own 1.4 us).  Here (91 us and 22 us) the query heads of a group are the
// columns of 16 x 16 x 32 MFMA blocks, and K and V go from memory straight to operand registers:
//   S^T[key][head] = K[key][:] . q[head][:]     A = K rows as they lie in memory, one 16-byte chunk per lane
//   O^T[d][head]  += V^T[d][key] P[key][head]   A: lane (c, g) loads the d chunk 8 c .. 8 c + 7 of the 8 keys whose scores it
//                                               holds (4 g .. 4 g + 3 of both 16-key blocks) and pairs keys up with byte
//                                               permutes; product j then covers d = 8 (row) + j, and P is used where it is
// The four wavefronts of a workgroup take the 32-key steps of a KV range in turn, each with a running softmax of its own, no
// barrier before the final merge; the next step's K is requested when this one's scores are done, its V after the products.
#pragma once

static constexpr int kDecWaves = 4;
static constexpr int kDecMaxG = kDecodeMaxGroup;
static constexpr int kDecPitch = DH + 4;   // floats between the heads of a wavefront's result in LDS

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4d;

template <bool SCORES>
__global__ void __launch_bounds__(64 * kDecWaves, 3)
attn_decode_kernel(const bf16* __restrict__ q, const int* __restrict__ row_pos, const ReqTable* __restrict__ table,
                   const bf16* __restrict__ k_pool, const bf16* __restrict__ v_pool, KvGeom g, int G,
                   bf16* __restrict__ out, AttnSplit sp, float* __restrict__ part_o, float2* __restrict__ part_ml,
                   float* __restrict__ scores, int scores_len, float2* __restrict__ score_ml) {
  __shared__ float lds_o[kDecWaves][kDecMaxG][kDecPitch];
  __shared__ float2 lds_ml[kDecWaves][kDecMaxG];
  const int kvh = (int)blockIdx.x % g.n_kv_heads;
  const int item = (int)blockIdx.x / g.n_kv_heads;
  if (item >= table->total_items) return;
  int b = table->n_req - 1;                 // item_base is 0 for the last request and grows towards the first
  while (b > 0 && item >= table->r[b - 1].item_base) --b;
  const ReqDev& rq = table->r[b];
  if (rq.n_rows <= 0) return;
  const int row = rq.row_base, seq = rq.dst_seq, part_base = rq.part_base;
  const bool may_split = rq.long_tile_start == 0 && sp.n_chunks > 1;
  const int chunk = item - rq.item_base;
  const int pos = row_pos[row];
  const int n_kv_tiles = pos / BKV + 1;
  const bool is_split = may_split && n_kv_tiles > sp.long_thr;
  const int t_begin = is_split ? chunk * sp.chunk_tiles : 0;
  const int t_end = is_split ? min(n_kv_tiles, t_begin + sp.chunk_tiles) : n_kv_tiles;
  if (t_begin >= t_end || (!is_split && chunk != 0)) return;   // uniform

  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, gq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_q_heads = g.n_kv_heads * G;
  const int key_end = min(t_end * BKV, pos + 1);
  constexpr int STEP = 32;

  bf16x8 qf[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (c < G) v = *reinterpret_cast<const uint4*>(q + ((size_t)row * n_q_heads + kvh * G + c) * DH + 32 * s + 8 * gq);
    qf[s] = __builtin_bit_cast(bf16x8, v);
  }

  // pages of 16 rows or more (and contiguous caches): the 16 keys of a block lie behind each other, one table look-up per
  // wavefront; other page sizes look every key up
  const bool whole_blocks = g.max_blocks == 1 || g.bs_shift >= 4;
  uint4 kr[2][4], vr[2][4];
  // first row of 16-key block `blk` of step `key0`; a block behind the last key repeats the one before (its keys are masked)
  auto block_start = [&](int key0, int blk) { return key0 + 16 * blk <= pos ? key0 + 16 * blk : key0; };
  auto load_k = [&](int key0) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      const int first = block_start(key0, blk);
      const int r = min(c, pos - first);
      const size_t o = whole_blocks ? kv_row_offset(g, seq, first, kvh) + (size_t)r * DH : kv_row_offset(g, seq, first + r, kvh);
      const bf16* p = k_pool + o + 8 * gq;
#pragma unroll
      for (int s = 0; s < 4; ++s) kr[blk][s] = *reinterpret_cast<const uint4*>(p + 32 * s);
    }
  };
  auto load_v = [&](int key0) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      const int first = block_start(key0, blk);
      const size_t base = whole_blocks ? kv_row_offset(g, seq, first, kvh) : 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = min(4 * gq + i, pos - first);
        const size_t o = whole_blocks ? base + (size_t)r * DH : kv_row_offset(g, seq, first + r, kvh);
        vr[blk][i] = *reinterpret_cast<const uint4*>(v_pool + o + 8 * c);
      }
    }
  };

  f32x4d acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = f32x4d{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const float c_scale = 1.4426950408889634f / sqrtf((float)DH);   // log2(e) / sqrt(dh)
  int key0 = t_begin * BKV + wave * STEP;
  if (key0 < key_end) {
    load_k(key0);
    load_v(key0);
  }
  for (; key0 < key_end; key0 += kDecWaves * STEP) {
    const int next = key0 + kDecWaves * STEP;
    f32x4d s[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      s[blk] = f32x4d{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 4; ++t)
        s[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[blk][t]), qf[t], s[blk], 0, 0, 0);
    }
    if (next < key_end) load_k(next);
    // element e of block blk is key key0 + 16 blk + 4 gq + e, head c
    float mx = -INFINITY;
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int key = key0 + 16 * blk + 4 * gq + e;
        if (SCORES && c < G && key <= pos)
          scores[((size_t)row * n_q_heads + kvh * G + c) * scores_len + key] = s[blk][e] * (1.0f / sqrtf((float)DH));
        if (key > pos) s[blk][e] = -INFINITY;
        mx = fmaxf(mx, s[blk][e]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx * c_scale);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;      // no visible finite score yet: every p is 0, not NaN
    const float corr = __builtin_amdgcn_exp2f(m_run - m_use);
    m_run = m_new;
    float psum = 0.f;
    f32x8 p;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      p[i] = __builtin_amdgcn_exp2f(fmaf(s[i >> 2][i & 3], c_scale, -m_use));
      psum += p[i];
    }
    l_run = l_run * corr + psum;
    const bf16x8 pf = __builtin_convertvector(p, bf16x8);
    const uint32_t* va = reinterpret_cast<const uint32_t*>(&vr[0][0]);
    const uint32_t* vb = reinterpret_cast<const uint32_t*>(&vr[1][0]);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int wi = j >> 1;
      // byte select: even j packs the low halves of two words, odd j the high halves
      const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
      uint4 f;
      f.x = __builtin_amdgcn_perm(va[4 + wi], va[wi], sel);
      f.y = __builtin_amdgcn_perm(va[12 + wi], va[8 + wi], sel);
      f.z = __builtin_amdgcn_perm(vb[4 + wi], vb[wi], sel);
      f.w = __builtin_amdgcn_perm(vb[12 + wi], vb[8 + wi], sel);
      acc[j] *= corr;
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f), pf, acc[j], 0, 0, 0);
    }
    if (next < key_end) load_v(next);
  }

  // merge of the four wavefronts; one without keys has m = -inf, l = 0, O = 0
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if (c < G) {
    if (gq == 0) lds_ml[wave][c] = make_float2(m_run, l_run);
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) lds_o[wave][c][8 * (4 * gq + e) + j] = acc[j][e];
  }
  __syncthreads();
  for (int i = tid; i < G * (DH / 2); i += 64 * kDecWaves) {
    const int h = i / (DH / 2), d = (i - h * (DH / 2)) * 2;
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) m = fmaxf(m, lds_ml[w][h].x);
    float l = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) {
      const float2 ml = lds_ml[w][h];
      const float wgt = ml.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml.x - m);
      if (ml.x == -INFINITY && ml.y == 0.f) continue;   // saw no key
      l += ml.y * wgt;
      o0 += lds_o[w][h][d] * wgt;
      o1 += lds_o[w][h][d + 1] * wgt;
    }
    const int head = kvh * G + h;
    if (is_split) {
      const size_t slot = (size_t)(part_base + chunk) * n_q_heads + head;
      if (d == 0) part_ml[slot] = make_float2(m, l);
      *reinterpret_cast<float2*>(part_o + slot * PROW + d) = make_float2(o0, o1);
    } else {
      if (SCORES && d == 0) score_ml[(size_t)row * n_q_heads + head] = make_float2(m, l);
      const float inv = 1.0f / l;
      const uint32_t pk = (uint32_t)f32_to_bf16(o0 * inv).v | ((uint32_t)f32_to_bf16(o1 * inv).v << 16);
      *reinterpret_cast<uint32_t*>(out + ((size_t)row * n_q_heads + head) * DH + d) = pk;
    }
  }
}
