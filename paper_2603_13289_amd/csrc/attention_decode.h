// Attention of phases whose requests have one live row each (decoding): included by attention_mfma.hip, whose constants, work
// items and partial-result layout it shares.
//
// Bound by reading K and V once.  The 32-row tile kernel multiplies 31 empty query rows per head, stages every tile through
// LDS behind a barrier and leaves 32 partial rows per chunk where one is live.  Here four wavefronts take a work item (KV head,
// KV chunk) and the query heads of the group are the columns of the 32x32x16 products:
//   S^T[key][head] = K[key][:] . q[head][:]     A = K rows as they lie in memory, one 16-byte chunk per lane and step; wavefront w
//                                               (0, 1) multiplies keys 32 w .. 32 w + 31 of a tile and leaves the scores in LDS
//   O^T[d][head]  += V^T[d][key] P[key][head]   wavefront 2 + w has d = 64 w .. 64 w + 63, behind a softmax of its own.  A: lane
//                                               (r, half) loads d = 64 w + 2 r and + 1 of the eight keys of a 16-key group whose
//                                               scores it holds and pairs keys up with byte permutes; product j covers
//                                               d = 64 w + 2 (row) + j
// The scores of a tile run one ahead of its softmax, so that a tile costs the longer of the two halves and not their sum.  K and V
// go from memory straight to registers, four tiles ahead (128 KB in flight per work item); one barrier per tile, which waits for
// no load.  Products, key tiles, chunks and the order of every sum are those of the tile kernel.  A row gets the bits that the tile
// kernel gives a row alone in its tile.  In company it may not: there one row whose maximum outgrows the slack moves the reference
// exponents of all rows of the tile, here those of its own head only; the weights are then rounded to bf16 at another scale.
//
// Per launch, tile kernel -> two wavefronts doing both halves in turn -> this one (32 query heads, 8 KV heads): one sequence of 5k
// keys with its scores written 18.7 -> 10.7 -> 10.5 us; sixteen of 1.3k to 10k keys 112 -> 97 -> 80 us (394 MB, 4.9 TB/s); three of 150 to 700
// keys on 2 KV heads 14.3 -> 10.2 -> 8.2.
#pragma once

static constexpr int kDecodeSets = 4;   // register sets of a tile's K or V

// SCORES: additionally write every visible score q.k / sqrt(dh) to scores[(row * n_q_heads + head) * scores_len + key] (the
// influence sums read them), and the row's reference exponent and sum, score_ml[row * n_q_heads + head], unless the KV range is
// split (then the merge has the pair).
template <bool SCORES>
__global__ void __launch_bounds__(256, 2)
attn_decode_kernel(const bf16* __restrict__ q, const int* __restrict__ row_pos, const ReqTable* __restrict__ table,
                   const bf16* __restrict__ k_pool, const bf16* __restrict__ v_pool, KvGeom g, int G,
                   bf16* __restrict__ out, AttnSplit sp, float* __restrict__ part_o, float2* __restrict__ part_ml,
                   float* __restrict__ scores, int scores_len, float2* __restrict__ score_ml) {
  __shared__ int lds_tab[kLdsTableEntries];
  __shared__ __attribute__((aligned(16))) unsigned lds_row[2][kDecodeSets][BKV];   // [second half's wavefront][set][key]
  __shared__ float4 lds_s[2][2][4][64];   // [tile parity][key block][e / 4][lane]
  const int kvh = (int)blockIdx.x % g.n_kv_heads;
  const int item = (int)blockIdx.x / g.n_kv_heads;
  if (item >= table->total_items) return;
  const ReqDev& rq = table->r[request_of_item(table, item)];
  if (rq.n_rows <= 0) return;
  const int row = rq.row_base, seq = rq.dst_seq, part_base = rq.part_base;
  const int chunk = item - rq.item_base;
  const int pos = pos_in_cache(row_pos[row], g.last_pos);
  const int n_kv_tiles = pos / BKV + 1;
  const bool is_split = sp.n_chunks > 1 && rq.long_tile_start == 0 && n_kv_tiles > sp.long_thr;
  const int t_begin = is_split ? chunk * sp.chunk_tiles : 0;
  const int t_end = is_split ? min(n_kv_tiles, t_begin + sp.chunk_tiles) : n_kv_tiles;
  if (t_begin >= t_end || (!is_split && chunk != 0)) return;   // uniform

  const int key_last = min(pos, t_end * BKV - 1);
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const int wave4 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave4 & 1;
  const int n_q_heads = g.n_kv_heads * G;
  const int head = kvh * G + min(col, G - 1);
  const bool live = col < G;

  // Pool row (of DH elements) of a key's position: a linear function in a contiguous cache; else the block ids of the range
  // are kept in LDS (pages of a power of two that fit), or looked up in memory.  A lane works out the row of one key of a
  // tile and the rows of the keys it loads come from LDS, so that nothing branches between the loads.
  const bool contig = g.max_blocks == 1;
  const unsigned crow = contig ? (unsigned)(kv_row_offset(g, seq, 0, kvh) / DH) : 0u;
  const int tab_first = contig || g.bs_shift < 0 ? 0 : (t_begin * BKV) >> g.bs_shift;
  bool tab_in_lds = false;
  if (!contig && g.bs_shift >= 0) {
    const int n_blk = min(((t_end * BKV - 1) >> g.bs_shift), g.max_blocks - 1) - tab_first + 1;
    if (n_blk <= kLdsTableEntries) {   // uniform
      for (int i = threadIdx.x; i < n_blk; i += 256) {
        const int blk = g.block_table[(size_t)seq * g.max_blocks + tab_first + i];
        lds_tab[i] = min(max(blk, 0), g.n_blocks - 1) * g.n_kv_heads + kvh;
      }
      tab_in_lds = true;
    }
  }
  __syncthreads();
  auto pool_row = [&](int p) -> unsigned {   // p <= pos
    if (contig) return crow + (unsigned)p;
    if (!tab_in_lds) return (unsigned)(kv_row_offset(g, seq, p, kvh) / DH);
    return ((unsigned)lds_tab[(p >> g.bs_shift) - tab_first] << g.bs_shift) | (unsigned)(p & (g.block_size - 1));
  };

  const std::integral_constant<int, 0> s0;
  const std::integral_constant<int, 1> s1;
  const std::integral_constant<int, 2> s2;
  const std::integral_constant<int, 3> s3;
  const std::true_type refill;
  const std::false_type last;
  // Tiles t_begin .. t_end - 1 in order, tile i on set i % 4, whose registers are asked for anew for the tile four on as soon as they
  // are free.  No condition around a load: behind one that may or may not be in flight the compiler would wait for all of
  // them.  Past the chunk every lane asks for its last key's row, which costs next to nothing.
  auto run = [&](auto load, auto tile) {
    load(s0, t_begin);
    load(s1, t_begin + 1);
    load(s2, t_begin + 2);
    load(s3, t_begin + 3);
    int t = t_begin;
    for (; t + 4 < t_end; t += 4) {
      tile(s0, t, refill);
      tile(s1, t + 1, refill);
      tile(s2, t + 2, refill);
      tile(s3, t + 3, refill);
    }
    tile(s0, t, last);
    if (t + 1 < t_end) tile(s1, t + 1, last);
    if (t + 2 < t_end) tile(s2, t + 2, last);
    if (t + 3 < t_end) tile(s3, t + 3, last);
  };
  // Behind it the scores of a tile are complete.  Their buffer is written again two tiles on, behind the other side's next barrier and
  // so behind its reads.  Not __syncthreads(): that may wait for the loads in flight as well.
  auto tile_barrier = []() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  if (wave4 < 2) {
    // Q as B operands: lane (head, half) holds q[head][16 s + 8 half .. +7].  Columns past the group repeat its last head and are
    // not written out.
    bf16x8 qf[8];
    const uint4* const qrow = reinterpret_cast<const uint4*>(q + ((size_t)row * n_q_heads + head) * DH) + half;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[s] = __builtin_bit_cast(bf16x8, qrow[2 * s]);
    uint4 kr[kDecodeSets][8];   // [set][head-dim step], key 32 wave + col of the tile
    run(
        [&](auto set, int t) {
          constexpr int S = decltype(set)::value;
          const bf16* kp = k_pool + (size_t)pool_row(min(t * BKV + 32 * wave + col, key_last)) * DH + 8 * half;
#pragma unroll
          for (int s = 0; s < 8; ++s) kr[S][s] = *reinterpret_cast<const uint4*>(kp + 16 * s);
          __builtin_amdgcn_sched_barrier(0);
        },
        [&](auto set, int t, auto again) {
          constexpr int S = decltype(set)::value;
          const int kv0 = t * BKV;
          f32x16 mine;
#pragma unroll
          for (int e = 0; e < 16; ++e) mine[e] = 0.f;
#pragma unroll
          for (int i = 0; i < 8; ++i)
            mine = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kr[S][i]), qf[i], mine, 0, 0, 0);
          if constexpr (decltype(again)::value) {
            __builtin_amdgcn_sched_barrier(0);
            const bf16* kp = k_pool + (size_t)pool_row(min((t + 4) * BKV + 32 * wave + col, key_last)) * DH + 8 * half;
#pragma unroll
            for (int s = 0; s < 8; ++s) kr[S][s] = *reinterpret_cast<const uint4*>(kp + 16 * s);
            __builtin_amdgcn_sched_barrier(0);
          }
          // element e is key kv0 + 32 wave + 8 (e/4) + 4 half + e%4
          const int key0 = kv0 + 32 * wave + 4 * half;
          if (SCORES && live) {
            float* srow = scores + ((size_t)row * n_q_heads + head) * scores_len;
            const float inv_sqrt = 1.0f / sqrtf((float)DH);
            const bool vec = (scores_len & 3) == 0 && kv0 + BKV - 1 <= pos;   // uniform
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
              const int key = key0 + 8 * e4;
              float v[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = mine[4 * e4 + e] * inv_sqrt;
              if (vec) {
                *reinterpret_cast<float4*>(srow + key) = make_float4(v[0], v[1], v[2], v[3]);
              } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (key + e <= pos) srow[key + e] = v[e];
              }
            }
          }
          if (kv0 + BKV - 1 > pos) {   // uniform: the last tile
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if (key0 + 8 * (e >> 2) + (e & 3) > pos) mine[e] = -INFINITY;
          }
          const int parity = (t - t_begin) & 1;
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4)
            lds_s[parity][wave][e4][lane] = make_float4(mine[4 * e4], mine[4 * e4 + 1], mine[4 * e4 + 2], mine[4 * e4 + 3]);
          tile_barrier();
        });
    return;
  }

  uint32_t vr[kDecodeSets][4][8];   // [set][16-key group][keys 4 half + 0..3, 8 + 4 half + 0..3]
  auto load_v = [&](auto set, int t) {
    constexpr int S = decltype(set)::value;
    lds_row[wave][S][lane] = pool_row(min(t * BKV + lane, key_last));   // this wavefront's own: its LDS accesses stay in order
    const bf16* const vcol = v_pool + 64 * wave + 2 * col;
    uint4 r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = *reinterpret_cast<const uint4*>(&lds_row[wave][S][8 * i + 4 * half]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      vr[S][i >> 1][4 * (i & 1) + 0] = *reinterpret_cast<const uint32_t*>(vcol + (size_t)r[i].x * DH);
      vr[S][i >> 1][4 * (i & 1) + 1] = *reinterpret_cast<const uint32_t*>(vcol + (size_t)r[i].y * DH);
      vr[S][i >> 1][4 * (i & 1) + 2] = *reinterpret_cast<const uint32_t*>(vcol + (size_t)r[i].z * DH);
      vr[S][i >> 1][4 * (i & 1) + 3] = *reinterpret_cast<const uint32_t*>(vcol + (size_t)r[i].w * DH);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  f32x16 acc_o[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc_o[i][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c_scale = 1.4426950408889634f / sqrtf((float)DH);   // log2(e) / sqrt(dh)
  run(load_v, [&](auto set, int t, auto again) {
    constexpr int S = decltype(set)::value;
    const int kv0 = t * BKV;
    if (kv0 + BKV - 1 > pos) {   // uniform: the last tile; rows past the last key repeat it
#pragma unroll
      for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (kv0 + 16 * tt + 8 * (i >> 2) + 4 * half + (i & 3) > pos) vr[S][tt][i] = 0;
    }
    tile_barrier();
    const int parity = (t - t_begin) & 1;
    f32x16 acc_s[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const float4 v = lds_s[parity][blk][e4][lane];
        acc_s[blk][4 * e4] = v.x; acc_s[blk][4 * e4 + 1] = v.y; acc_s[blk][4 * e4 + 2] = v.z; acc_s[blk][4 * e4 + 3] = v.w;
      }
    float mx = acc_s[0][0];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, acc_s[blk][e]);
    mx = pair_max32(mx);
    // the reference exponent follows the maximum lazily, head by head (a factor of 1 leaves the other heads' sums as they are)
    const float m_new = fmaxf(m_run, mx * c_scale);
    const bool grow = m_new > m_run + kRescaleSlack;
    if (__any(grow)) {
      const float m_to = (m_new == -INFINITY) ? 0.f : m_new;
      const float corr = grow ? __builtin_amdgcn_exp2f(m_run - m_to) : 1.f;
      l_run *= corr;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc_o[i][e] *= corr;
      if (grow) m_run = m_new;
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
    float psum = 0.f;
    bf16x8 pf[4];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        f32x8 p;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          p[j] = __builtin_amdgcn_exp2f(fmaf(acc_s[blk][8 * u + j], c_scale, -m_use));
          psum += p[j];
        }
        pf[2 * blk + u] = __builtin_convertvector(p, bf16x8);
      }
    l_run += psum;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint32_t sel = j ? 0x07060302u : 0x05040100u;   // byte select: low or high halves of two words
        uint4 f;
        f.x = __builtin_amdgcn_perm(vr[S][tt][1], vr[S][tt][0], sel);
        f.y = __builtin_amdgcn_perm(vr[S][tt][3], vr[S][tt][2], sel);
        f.z = __builtin_amdgcn_perm(vr[S][tt][5], vr[S][tt][4], sel);
        f.w = __builtin_amdgcn_perm(vr[S][tt][7], vr[S][tt][6], sel);
        acc_o[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f), pf[tt], acc_o[j], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(again)::value) load_v(set, t + 4);
  });

  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (!live) return;
  // accumulator element e of product j: d = 64 wave + 2 (8 (e/4) + 4 half + e%4) + j
  const int d0 = 64 * wave + 8 * half;
  if (is_split) {
    const size_t slot = ((size_t)(part_base + chunk) * n_q_heads + head) * BQ;
    if (half == 0 && wave == 0) part_ml[slot] = make_float2(m_run, l_tot);
    float* po = part_o + slot * PROW + d0;
#pragma unroll
    for (int e = 0; e < 16; e += 2)
      *reinterpret_cast<float4*>(po + 16 * (e >> 2) + 2 * (e & 3)) =
          make_float4(acc_o[0][e], acc_o[1][e], acc_o[0][e + 1], acc_o[1][e + 1]);
    return;
  }
  if (SCORES && half == 0 && wave == 0) score_ml[(size_t)row * n_q_heads + head] = make_float2(m_run, l_tot);
  const float inv = 1.0f / l_tot;
  bf16* orow = out + ((size_t)row * n_q_heads + head) * DH + d0;
#pragma unroll
  for (int e = 0; e < 16; e += 2) {
    uint2 pk;
    pk.x = (uint32_t)f32_to_bf16(acc_o[0][e] * inv).v | ((uint32_t)f32_to_bf16(acc_o[1][e] * inv).v << 16);
    pk.y = (uint32_t)f32_to_bf16(acc_o[0][e + 1] * inv).v | ((uint32_t)f32_to_bf16(acc_o[1][e + 1] * inv).v << 16);
    *reinterpret_cast<uint2*>(orow + 16 * (e >> 2) + 2 * (e & 3)) = pk;
  }
}
