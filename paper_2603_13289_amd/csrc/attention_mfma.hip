// K6: sparse-query causal grouped-query attention on the matrix cores (bf16, head_dim 128).
//
// Queries are the active rows of a layer: arbitrary ascending positions of one sequence.  A workgroup
// takes one tile of 32 query rows and one KV head; wavefront g of the workgroup serves query head
// kv_head * G + g, so all G heads of the group share every K/V tile that is staged in LDS.
//
// Per KV tile of 64 keys a wavefront computes, with 32x32x16 MFMA blocks,
//   S^T[key][q] = K[key][:] . Q[q][:]          (A = K rows from LDS, B = Q held in registers)
//   O^T[d][q]  += V^T[d][key] * P[key][q]      (A = V^T from LDS,    B = P straight from S^T's registers)
// Computing the transposed score tile puts a query's 64 scores into the two lanes (q, q+32), so the
// running softmax needs one cross-lane exchange per tile, and the accumulator layout of S^T is
// already the B-operand layout of the second product up to a fixed permutation of the keys inside
// each group of 16.  V is transposed while it is written to LDS, with that same permutation applied,
// so each operand is one 16-byte LDS read.
//
// LDS rows of K are padded by 16 bytes (272 apart), 16-byte pieces of V^T rows change places by the row, so that operand fetches
// and writes are free of bank conflicts (SQ_LDS_BANK_CONFLICT 0; with pieces exchanged by pairs of rows it was 14 % of the LDS cycles and
// 4096 queries over 8000 keys took 1.4 % longer).  K/V rows come from the paged cache through the block table, one tile ahead in registers
// and one tile ahead in a second pair of LDS buffers, so a tile costs one barrier.
//
// What bounds it: a tile step is a chain of S^T, softmax and O^T in which the LDS reads of the products, the LDS writes of the staging and
// the loads of the tile two on each keep a unit busy for about 500 cycles of the four wavefronts together.  Side by side with
// another's instructions they are hidden: the staging writes run under the exponentials (K's before, V's between them), the loads between the
// matrix instructions of O^T, in a main loop without conditions.  In a bunch, with the staging between the products of S^T, the loads behind
// it and a table look-up of its own in front of each load, a step took 4000 cycles alone on a compute unit and 5600 with two workgroups; now
// 2900 and 3350.  Per launch in a train of twenty, before that loop -> now, all on one card: 4096 queries over 8000 keys, 32 heads on 8: 16-token
// pages 515 -> 407 us (980 TFLOP/s), contiguous 417 -> 407, pages of 24 791 -> 463; 40 heads on 8: 810 -> 587 and 739 -> 589 contiguous.
// 32 queries over 4096 keys 135 -> 76 (pages of 24: 209 -> 105), 100 over 264 15.8 -> 11.8 (contiguous 12.3 -> 11.8).
// Ranges of a tile or two are bound by the chain to the first product and by instructions that are fetched for the first time, so what runs before it
// has few branches (look-ups by a multiplication, every lane loads a row of Q) and few links: the first block look-ups do not hang on the rows'
// positions, Q is asked for behind K and V.  61 queries over 61 keys: 16-token pages 7.68 -> 6.83, contiguous 6.84 -> 6.73 (7.11 without those).
// KV tiles entirely above the tile's last query position are skipped; the causal mask is applied
// only in tiles that reach above the tile's first query position.  Workgroups are issued longest
// first over the whole launch (KV head fastest, query tiles by decreasing KV range).
#include <type_traits>

#include "common.h"

namespace rc {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(float)))) float f32x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

static constexpr int BQ = 32;    // query rows per workgroup
static constexpr int BKV = 64;   // keys per tile
static constexpr int DH = 128;
static constexpr int KROW = DH * 2 + 16;   // bytes between K rows in LDS
static constexpr int VROW = BKV * 2;       // bytes between V^T rows in LDS
static constexpr int K_TILE_BYTES = BKV * KROW;
static constexpr int V_TILE_BYTES = DH * VROW;
static constexpr int kLdsTableEntries = 2048;   // block-table entries of the workgroup's KV range kept in LDS (attn_decode_kernel, paged caches)
static constexpr int ATTN_LDS_BYTES = 2 * (K_TILE_BYTES + V_TILE_BYTES);
static constexpr int PROW = DH + 16;         // floats between the rows of a partial result (see attention_partial_floats)
static constexpr int kFragAhead = 4;       // LDS operand fragments in flight ahead of the MFMA that uses them
static constexpr float kRescaleSlack = 8.f;   // log2 units the running maximum may lead the reference exponent

// Maximum over the lane pair (l, l ^ 32).  v_permlane32_swap exchanges the upper half of its first operand with
// the lower half of its second; fed the same value twice it returns (lower half, lower half) and (upper half,
// upper half), so the maximum of the two results is the pair's maximum in every lane, without an LDS round trip.
__device__ inline float pair_max32(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Request of a work item / of a merge row: the bases fall (rise) with the request, so the lanes compare one request each and the
// wavefront counts, instead of a chain of table loads from request to request (16 decoding requests: merge 8.8 -> 5.3 us, attention 81.5 -> 80).
static_assert(RC_MAX_REQ <= 64, "a lane per request");
__device__ __forceinline__ int request_of_item(const ReqTable* table, int item) {
  const int n = table->n_req, lane = threadIdx.x & 63;
  if (n == 1) return 0;
  const unsigned long long at = __ballot(lane < n && item >= table->r[min(lane, n - 1)].item_base);
  return __builtin_amdgcn_readfirstlane(__ffsll((long long)at) - 1);
}
__device__ __forceinline__ int request_of_merge_row(const ReqTable* table, int mr) {
  const int n = table->n_req, lane = threadIdx.x & 63;
  if (n == 1) return 0;
  const unsigned long long at = __ballot(lane < n && mr >= table->r[min(lane, n - 1)].merge_base);
  return __builtin_amdgcn_readfirstlane(__popcll(at) - 1);
}

template <int G>
__global__ void __launch_bounds__(64 * (G < 4 ? 4 : G), (G <= 4 ? 2 : 1))
attn_mfma_kernel(const bf16* __restrict__ q, const int* __restrict__ row_pos, const ReqTable* __restrict__ table,
                 int fixed_seq, int total_rows, int total_tiles, const bf16* __restrict__ k_pool,
                 const bf16* __restrict__ v_pool, KvGeom g, bf16* __restrict__ out, AttnSplit sp,
                 float* __restrict__ part_o, float2* __restrict__ part_ml) {
  // A workgroup has at least four wavefronts: with fewer, each thread would stage so much of a K/V tile that the
  // kernel runs out of registers.  In a group of one to three query heads the wavefronts beyond the group only take
  // their share of the staging; they multiply zeros for head 0 of the group and write nothing.
  constexpr int NW = G < 4 ? 4 : G;
  // K rows are 256 + 16 bytes apart.  Eight lanes (a cycle: 128 bytes) that fetch the same 16-byte chunk of consecutive rows then hit
  // every bank exactly once, and every LDS address of K is a per-thread base plus a compile-time constant.
  // Two K and two V^T buffers: tile t lives in buffer t % 2 and tile t + 1 is staged while tile t is multiplied,
  // so one barrier per tile suffices.
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_attn[];
  unsigned char* const lds_k = lds_attn;                         // [2][BKV * KROW], behind it V^T, [2][DH * VROW]

  // late tiles see the most keys: start them first.  With sp.n_chunks > 1 the KV range of a long query
  // tile is cut into chunks of sp.chunk_tiles tiles, one workgroup each, whose partial results are merged
  // by attn_merge_kernel; short tiles are done whole by their chunk-0 workgroup.
  // The KV head varies fastest: workgroups are then dispatched in order of decreasing KV range over the whole
  // grid (a longest-first schedule), and with 8 KV heads every XCD (workgroup id mod 8) keeps to one head's K/V.
  const int kvh = (int)blockIdx.x % g.n_kv_heads;
  const int item = (int)blockIdx.x / g.n_kv_heads;
  const int n_q_heads = g.n_kv_heads * G;
  int r0, n_valid, seq, chunk, split_tile, part_base = 0;   // split_tile < 0: this tile is never split
  if (table) {
    // Work items: requests last to first; inside a request first the query tiles that may be split (one item per
    // tile and KV chunk), then the whole tiles, late ones first.  The host's counts may be upper bounds
    // (rows selected on the device): the table has the live ones.
    if (item >= table->total_items) return;
    const ReqDev& rq = table->r[request_of_item(table, item)];   // item_base is 0 for the last request and grows towards the first
    const int tiles = (rq.n_rows + BQ - 1) / BQ;
    const int start = min(rq.long_tile_start, tiles);
    const int j = item - rq.item_base;
    const int n_split_items = (tiles - start) * sp.n_chunks;
    int lt;
    if (j < n_split_items) {
      // chunk-major: chunk 0 of every such tile (late tiles first), then chunk 1, ...  Tiles whose range ends before a
      // chunk have nothing to do there; in this order those empty items sit together at the end of each chunk's run
      // instead of at every n_chunks-th position of the grid (where, for even chunk counts, they kept landing on the
      // same half of the machine and left the other half with all the work)
      chunk = j / (tiles - start);
      lt = tiles - 1 - j % (tiles - start);
    } else {
      lt = start - 1 - (j - n_split_items);
      chunk = 0;
    }
    if (lt < 0) return;
    r0 = rq.row_base + lt * BQ;
    n_valid = min(BQ, rq.row_base + rq.n_rows - r0);
    seq = rq.dst_seq;
    split_tile = lt - rq.long_tile_start;
    part_base = rq.part_base;
  } else {
    chunk = item / total_tiles;
    const int tile = total_tiles - 1 - item % total_tiles;
    if (chunk >= sp.n_chunks) return;
    r0 = tile * BQ;
    n_valid = min(BQ, total_rows - r0);
    seq = fixed_seq;
    split_tile = tile;
  }
  if (n_valid <= 0) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Block of a position and slot in it; past the cache a slot of its last block.
  auto rsrc_of = [](const void* p) __attribute__((always_inline)) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, -1, 0x00020000); };
  const int32_t* const seq_table = g.block_table + (size_t)seq * g.max_blocks;
  struct Asked { int block; unsigned slot; };
  auto ask = [&](int pos) __attribute__((always_inline)) -> Asked {
    const int at = block_of(g, pos);
    return {(int)__builtin_amdgcn_raw_buffer_load_b32(rsrc_of(seq_table), 4 * min(at, g.max_blocks - 1), 0, 0), (unsigned)(pos - at * g.block_size)};
  };
  // Key kv0 + lane of the first two tiles: that does not hang on the rows' positions, which are asked for beside it.
  auto ask_tile = [&](int kv0) __attribute__((always_inline)) { return ask(kv0 + lane); };
  const int t_first = chunk * sp.chunk_tiles;   // 0 where the range is not cut
  const Asked first_tile = ask_tile(t_first * BKV), second_tile = ask_tile((t_first + 1) * BKV);
  const int ql = lane & 31, half = lane >> 5;
  const bool active = G >= 4 || wave < G;   // wave-uniform
  const int head = kvh * G + (active ? wave : 0);
  const bool q_ok = active && ql < n_valid;
  const int my_row = r0 + (q_ok ? ql : 0);
  const int my_pos = pos_in_cache(row_pos[my_row], g.last_pos);   // of every lane: under a condition it is waited for at once
  const int first_pos = pos_in_cache(row_pos[r0], g.last_pos);
  const int last_pos = pos_in_cache(row_pos[r0 + n_valid - 1], g.last_pos);

  f32x16 acc_o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc_o[i][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c_scale = 1.4426950408889634f / sqrtf((float)DH);   // log2(e) / sqrt(dh)

  // K/V tile staging, by the first NS threads: every one owns KPER 16-byte chunks of the K tile (rows krow0 + i*KSTEP, chunk
  // tid%16), the first 256 one block of the V tile each (4 consecutive keys x 8 d).  Neighbouring lanes have neighbouring chunks of a
  // row, in both: with neighbouring lanes in different rows of V a load touched 64 cache lines and the eight loads of a tile took 750 to
  // 1900 cycles to issue.  The next tile is fetched into registers while the current one is multiplied.
  constexpr int NS = G == 8 ? 512 : 256, KSTEP = NS / 16, KPER = BKV / KSTEP;
  const bool stages_k = NW * 64 == NS || wave * 64 < NS, stages_v = NW == 4 || wave < 4;   // wave-uniform
  const int krow0 = tid >> 4, kch = tid & 15;      // K: row, 16-byte chunk
  // V: quad of 4 keys, chunk of 8 d.  Eight neighbouring lanes have 128 bytes of a row; sixteen, in two quads 8 keys apart, write half a
  // row of V^T each in 128 different bytes (below).
  auto quad_of = [](int th) __attribute__((always_inline)) { return (th >> 6) * 4 + ((th >> 5) & 1) + ((th >> 2) & 2); };
  auto dch_of = [](int th) __attribute__((always_inline)) { return (th & 7) + ((th >> 1) & 8); };
  const int vquad = quad_of(tid), vdch = dch_of(tid);
  // the tile fetched during step t is staged during step t + 1 and multiplied in step t + 2
  uint4 rk[KPER], rv[4];
  // A lane looks up the pool row (of DH elements) of one key of a tile.  In blocks of 16, 32, 64, ... slots the 16 keys of a group lie
  // one behind the other, and loads go to the scalar row of their group and a constant lane offset: in the main loop lane i looks up group
  // i % 4, elsewhere key kv0 + i.  Other block sizes, and a query tile's last KV tile where it is ragged: rows handed around.  Past the last
  // position that is whatever row the cache has there: the mask sets its score, and its values are staged as zeros (sel_of).
  // A look-up comes in two halves, so that the block of a tile two on is asked for early and not waited for.
  const bool by_group = g.max_blocks == 1 || g.bs_shift >= 4;   // one block per sequence, or blocks of 16, 32, ...
  const unsigned k_lane = (unsigned)((krow0 & 15) * DH + kch * 8) * 2, v_lane = (unsigned)((vquad & 3) * 4 * DH + vdch * 8) * 2;
  auto grouped = [&](int kv0) __attribute__((always_inline)) { return by_group && kv0 + BKV - 1 <= last_pos; };   // uniform
  auto row_of = [&](Asked q) __attribute__((always_inline)) -> unsigned {
    return (unsigned)(min(max(q.block, 0), g.n_blocks - 1) * g.n_kv_heads + kvh) * (unsigned)g.block_size + q.slot;
  };
  auto group_pos = [&](int kv0) __attribute__((always_inline)) { return kv0 + 16 * (lane & 3); };
  auto group_at = [&](const bf16* pool, unsigned row, int from) __attribute__((always_inline)) {   // scalar
    return rsrc_of(pool + (size_t)(unsigned)__builtin_amdgcn_readlane((int)row, from) * DH);
  };
  auto k_chunk = [&](unsigned row, int i, int lanes) __attribute__((always_inline)) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(group_at(k_pool, row, lanes * (i * (KSTEP / 16) + (NS == 512 ? wave >> 2 : 0))), k_lane, 0, 0));
  };
  auto v_chunk_of = [&](unsigned row, int kk, int lanes) __attribute__((always_inline)) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(group_at(v_pool, row, lanes * (wave & 3)), v_lane, kk * DH * 2, 0));
  };
  auto fetch = [&](int kv0, Asked asked) __attribute__((always_inline)) {
    const unsigned row = row_of(asked);
    const unsigned char* const kp = reinterpret_cast<const unsigned char*>(k_pool);
    const unsigned char* const vp = reinterpret_cast<const unsigned char*>(v_pool);
    if (grouped(kv0)) {
      if (stages_k) {
        rk[0] = k_chunk(row, 0, 16);
        rk[1] = k_chunk(row, 1, 16);
        if constexpr (KPER == 4) {
          rk[2] = k_chunk(row, 2, 16);
          rk[3] = k_chunk(row, 3, 16);
        }
      }
      if (stages_v) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) rv[kk] = v_chunk_of(row, kk, 16);
      }
      return;
    }
    int th = tid;
    asm volatile("" : "+v"(th));   // lane numbers worked out here each time: kept over the main loop they took its registers
    if (stages_k) {
#pragma unroll
      for (int i = 0; i < KPER; ++i)
        rk[i] = *reinterpret_cast<const uint4*>(kp + (size_t)(unsigned)__shfl((int)row, (th >> 4) + i * KSTEP, 64) * (DH * 2) + (th & 15) * 16);
    }
    if (stages_v) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        rv[kk] = *reinterpret_cast<const uint4*>(vp + (size_t)(unsigned)__shfl((int)row, (quad_of(th) * 4 + kk) & 63, 64) * (DH * 2) + dch_of(th) * 16);
    }
  };
  // V transposed: key = 16 grp + 8 a + 4 h + c goes to column 16 grp + 8 h + 4 a + c; a quad shares (grp, a, h).
  // In LDS, 16-byte chunk c of V^T row d is chunk c ^ (d & 7) ^ (d/8 & 7): eight rows of an operand fetch then meet all 128 bytes of a cycle
  // once, and so do sixteen lanes that write.
  const int vgrp = vquad >> 2;
  const int v_chunk = (2 * vgrp + (vquad & 1)) ^ (vdch & 7);
  unsigned char* const k_wr = lds_k + krow0 * KROW + kch * 16;
  const unsigned v_wr = 2 * K_TILE_BYTES + vdch * 8 * VROW + 16 * v_chunk + 8 * ((vquad >> 1) & 1);   // chunk ^ e: bits 4-6 of the address
  // The selects of a thread's keys 0, 1 and 2, 3.  Values behind the last position become zeros (byte select 12): what lies there may be no
  // finite number, and is not to be multiplied by a weight of 0.
  struct Sel { uint32_t lo0, lo1, hi0, hi1; };   // byte selects: the low halves of two words (even d) or the high ones
  const Sel whole = {0x05040100u, 0x07060302u, 0x05040100u, 0x07060302u};
  auto sel_of = [&](int kv0) __attribute__((always_inline)) -> Sel {
    Sel s = whole;
    if (kv0 + BKV - 1 > last_pos) {   // uniform
      int th = tid;
      asm volatile("" : "+v"(th));
      const int n = last_pos - kv0 - quad_of(th) * 4;   // keys 0 .. n
      const uint32_t lo = n < 0 ? 0u : (n < 1 ? 0xffffu : ~0u), hi = n < 2 ? 0u : (n < 3 ? 0xffffu : ~0u);
      s = {(s.lo0 & lo) | (0x0c0c0c0cu & ~lo), (s.lo1 & lo) | (0x0c0c0c0cu & ~lo), (s.hi0 & hi) | (0x0c0c0c0cu & ~hi), (s.hi1 & hi) | (0x0c0c0c0cu & ~hi)};
    }
    return s;
  };
  auto stage_k = [&](auto buf) __attribute__((always_inline)) {
    constexpr int KOFF = decltype(buf)::value * K_TILE_BYTES;
    if (!stages_k) return;
#pragma unroll
    for (int i = 0; i < KPER; ++i) *reinterpret_cast<uint4*>(k_wr + KOFF + i * KSTEP * KROW) = rk[i];
  };
  // V^T rows e_begin .. e_end - 1 (of the 8 head-dim elements a thread's block covers)
  auto stage_v = [&](auto buf, int e_begin, int e_end, Sel sel) __attribute__((always_inline)) {
    constexpr int VOFF = decltype(buf)::value * V_TILE_BYTES;
    if (!stages_v) return;
    const uint32_t w[4][4] = {{rv[0].x, rv[0].y, rv[0].z, rv[0].w},
                              {rv[1].x, rv[1].y, rv[1].z, rv[1].w},
                              {rv[2].x, rv[2].y, rv[2].z, rv[2].w},
                              {rv[3].x, rv[3].y, rv[3].z, rv[3].w}};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (e < e_begin || e >= e_end) continue;
      const int m = e >> 1;
      uint2 pk;
      pk.x = __builtin_amdgcn_perm(w[1][m], w[0][m], (e & 1) ? sel.lo1 : sel.lo0);
      pk.y = __builtin_amdgcn_perm(w[3][m], w[2][m], (e & 1) ? sel.hi1 : sel.hi0);
      *reinterpret_cast<uint2*>(lds_attn + (v_wr ^ (16 * e)) + VOFF + e * VROW) = pk;
    }
  };
  // operand fetch addresses: K block b, dh step s -> k_rd + b*32*KROW + s*32 ; V^T block db, key step tt -> (v_rd ^ 32 (tt ^ 2 db)) + db*32*VROW
  const unsigned char* const k_rd = lds_k + ql * KROW + half * 16;
  const unsigned v_rd = 2 * K_TILE_BYTES + ql * VROW + 16 * (half ^ (ql & 7) ^ (ql >> 3));

  const int n_kv_tiles = last_pos / BKV + 1;
  const bool is_split = sp.n_chunks > 1 && split_tile >= 0 && n_kv_tiles > sp.long_thr;
  const int t_begin = is_split ? t_first : 0;
  const int t_end = is_split ? min(n_kv_tiles, t_begin + sp.chunk_tiles) : n_kv_tiles;
  if (t_begin >= t_end || (!is_split && chunk != 0)) return;   // nothing for this workgroup (uniform)
  const std::integral_constant<int, 0> buf0;
  const std::integral_constant<int, 1> buf1;
  // prologue: the first tile goes to buffer 0, the second one is on its way in registers
  fetch(t_begin * BKV, first_tile);
  // Q as B operands: lane (q, half) holds Q[q][16 s + 8 half .. +7], s = 0..7.  Lanes without a row of their own repeat the tile's first and
  // are not written out.
  bf16x8 qf[8];
  {
    const bf16* qrow = q + ((size_t)my_row * n_q_heads + head) * DH + 8 * half;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      qf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(qrow + 16 * s));
    }
  }

  stage_k(buf0);
  stage_v(buf0, 0, 8, sel_of(t_begin * BKV));
  if (t_begin + 1 < t_end) fetch((t_begin + 1) * BKV, second_tile);
  __syncthreads();
  // step i (tile t = t_begin + i) multiplies buffer i % 2; meanwhile it stages tile t + 1 into the other buffer
  // (free since the barrier that ended step i - 1) and starts the loads of tile t + 2.  how: 1 in the main loop, where there are such
  // tiles, whole ones; 2 the same for wavefronts beyond the fourth, which stage no V (and no K but in groups of eight); 0 anywhere.
  auto tile_step = [&](int t, auto buf, auto how) __attribute__((always_inline)) {
    constexpr bool steady = decltype(how)::value > 0, K_TOO = decltype(how)::value == 1 || G == 8, V_TOO = decltype(how)::value == 1;
    constexpr int KOFF = decltype(buf)::value * K_TILE_BYTES, VOFF = decltype(buf)::value * V_TILE_BYTES;
    const std::integral_constant<int, 1 - decltype(buf)::value> other;
    const int kv0 = t * BKV;
    const bool has_next = t + 1 < t_end, has_next2 = t + 2 < t_end;
    Asked asked = {};   // for the tile two on
    if constexpr (!steady) {
      if (has_next2) asked = ask_tile(kv0 + 2 * BKV);
    } else if constexpr (K_TOO) {
      asked = ask(group_pos(kv0 + 2 * BKV));
    }
    unsigned row2 = 0;
    // S^T = K Q^T : two blocks of 32 keys.  The two accumulator chains alternate and the K fragments are read
    // kFragAhead MFMAs ahead of their use, so that neither the LDS latency nor the MFMA dependency is exposed.
    f32x16 acc_s[2];
    {
      f32x16 zero;   // the first product of each chain takes a constant-zero accumulator: no registers to clear
#pragma unroll
      for (int e = 0; e < 16; ++e) zero[e] = 0.f;
      auto k_frag = [&](int i) {   // step i: key block i & 1, head-dim step i >> 1
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(k_rd + KOFF + (i & 1) * 32 * KROW + (i >> 1) * 32));
      };
      bf16x8 kf[kFragAhead];
#pragma unroll
      for (int i = 0; i < kFragAhead; ++i) kf[i] = k_frag(i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        acc_s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i % kFragAhead], qf[i >> 1], i < 2 ? zero : acc_s[i & 1], 0, 0, 0);
        if (i + kFragAhead < 16) kf[i % kFragAhead] = k_frag(i + kFragAhead);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // the first V^T fragments do not depend on the softmax: their LDS reads run under it
    auto v_frag = [&](int i) {     // step i: head-dim block i & 3, key step i >> 2
      return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(lds_attn + (v_rd ^ (32 * ((2 * (i & 1)) ^ (i >> 2)))) + VOFF + (i & 3) * 32 * VROW));
    };
    bf16x8 vf[kFragAhead];
#pragma unroll
    for (int i = 0; i < kFragAhead; ++i) vf[i] = v_frag(i);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (steady) {
      if constexpr (K_TOO) {
        stage_k(other);
        row2 = row_of(asked);
      }
      __builtin_amdgcn_sched_barrier(0);
    } else {
      if (has_next) {
        stage_k(other);
        stage_v(other, 0, 8, sel_of(kv0 + BKV));
      }
      if (has_next2) fetch(kv0 + 2 * BKV, asked);
    }
    // running softmax on raw scores; the 1/sqrt(dh) * log2(e) factor is folded into the exponent.
    // Element e of block b is key kv0 + 32 b + 8 (e/4) + 4 half + e%4.  Only tiles that reach above the
    // tile's first query position need the causal mask.
    if (kv0 + BKV - 1 > first_pos) {
      asm volatile("; causal mask tile" ::: "memory");   // keeps this a real (wave-uniform) branch
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int key = kv0 + 32 * b + 8 * (e >> 2) + 4 * half + (e & 3);
          if (key > my_pos) acc_s[b][e] = -INFINITY;
        }
    }
    float mx = acc_s[0][0];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, acc_s[b][e]);
    mx = pair_max32(mx);
    // m_run is the reference exponent of the running sums, in the scaled (log2) domain.  It follows the
    // running maximum lazily: the sums are rescaled (64 multiplies per lane) only when some row's maximum has
    // grown by more than kRescaleSlack since its last rescale, so p stays below 2^kRescaleSlack instead of 1.
    // Any reference gives the same quotient O / l; bf16 keeps p's relative precision at every magnitude.
    // A row that has not seen a visible key yet keeps m_run = -inf; m_use avoids inf - inf in that case
    // (all its p are then 0).
    const float m_new = fmaxf(m_run, mx * c_scale);
    if (__any(m_new > m_run + kRescaleSlack)) {   // wave-uniform
      const float m_to = (m_new == -INFINITY) ? 0.f : m_new;
      const float corr = __builtin_amdgcn_exp2f(m_run - m_to);
      l_run *= corr;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc_o[i][e] *= corr;
      m_run = m_new;
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
    float psum = 0.f;
    bf16x8 pf[4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        f32x8 p;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          p[j] = __builtin_amdgcn_exp2f(fmaf(acc_s[b][8 * u + j], c_scale, -m_use));
          psum += p[j];
        }
        pf[2 * b + u] = __builtin_convertvector(p, bf16x8);
        asm volatile("" : "+v"(psum));   // added up here: put off, the 32 weights stayed in registers over the second product
        if constexpr (V_TOO) {
          __builtin_amdgcn_sched_barrier(0);
          if (b == 0) stage_v(other, 4 * u, 4 * u + 4, whole);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    l_run += psum;
    // O^T += V^T P : four accumulator chains alternate, fragments read kFragAhead MFMAs ahead
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      acc_o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i % kFragAhead], pf[i >> 2], acc_o[i & 3], 0, 0, 0);
      if (i + kFragAhead < 16) vf[i % kFragAhead] = v_frag(i + kFragAhead);
      if constexpr (steady) {
        if constexpr (K_TOO)
          if (i % 2 == 0 && i < 2 * KPER) rk[i / 2] = k_chunk(row2, i / 2, 1);
        if constexpr (V_TOO)
          if (i % 2 == 0 && i >= 2 * KPER && i < 2 * KPER + 8) rv[i / 2 - KPER] = v_chunk_of(row2, i / 2 - KPER, 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();   // tile t fully consumed, tile t + 1 fully staged
  };
  int t = t_begin;
  const int t_whole = by_group ? min(t_end, (last_pos + 1) / BKV) : 0;   // tiles before it are whole ones
  auto steady_tiles = [&](auto how) __attribute__((always_inline)) {
    for (; t + 3 < t_whole; t += 2) {
      tile_step(t, buf0, how);
      tile_step(t + 1, buf1, how);
    }
  };
  if (stages_v) steady_tiles(std::integral_constant<int, 1>{});
  else steady_tiles(std::integral_constant<int, 2>{});
  const std::integral_constant<int, 0> general;
  for (; t < t_end; t += 2) {
    tile_step(t, buf0, general);
    if (t + 1 < t_end) tile_step(t + 1, buf1, general);
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (!active) return;
  if (is_split) {
    // partial result of this chunk: un-normalised O, running maximum (log2 domain) and sum
    const size_t slot = ((size_t)(part_base + split_tile * sp.n_chunks + chunk) * n_q_heads + head) * BQ + ql;
    if (half == 0) part_ml[slot] = make_float2(m_run, l_tot);
    float* po = part_o + slot * PROW;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const int d = 32 * db + 8 * e4 + 4 * half;
        *reinterpret_cast<float4*>(po + d) = make_float4(acc_o[db][4 * e4 + 0], acc_o[db][4 * e4 + 1],
                                                          acc_o[db][4 * e4 + 2], acc_o[db][4 * e4 + 3]);
      }
    return;
  }
  if (q_ok) {
    const float inv = 1.0f / l_tot;
    bf16* orow = out + ((size_t)my_row * n_q_heads + head) * DH;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const int d = 32 * db + 8 * e4 + 4 * half;
        uint2 pk;
        pk.x = (uint32_t)f32_to_bf16(acc_o[db][4 * e4 + 0] * inv).v | ((uint32_t)f32_to_bf16(acc_o[db][4 * e4 + 1] * inv).v << 16);
        pk.y = (uint32_t)f32_to_bf16(acc_o[db][4 * e4 + 2] * inv).v | ((uint32_t)f32_to_bf16(acc_o[db][4 * e4 + 3] * inv).v << 16);
        *reinterpret_cast<uint2*>(orow + d) = pk;
      }
  }
}

#include "attention_decode.h"

// Merge of the KV chunks: a wavefront takes 2 PAIRS heads of a row, 32 lanes with four head-dim elements each per head.  Only rows of
// split tiles take part; chunk c holds keys for a row iff its first key position is <= the row's position.
// The bytes are few (1476 rows x 32 heads: 75 MB); what bounds it is a chain of dependent reads (table, positions, exponents,
// outputs) per wavefront, so a wavefront has 16 rows of outputs under way behind one walk of that chain, requested before the
// exponents are reduced: four heads by four chunks where rows are many, two by eight in a decoding step, where wavefronts are few and
// chunks many.  One head per wavefront before: 1476 rows x 32 heads 31.9 -> 16.9 us, 1639 rows over 17k keys 47.9 -> 32.8, sixteen
// decoding rows 5.3 -> 4.8; four heads by four chunks for the decoding rows as well: 5.6, and the launch below 6.7 -> 7.6 instead of 6.6.
template <int PAIRS, int AHEAD>
__device__ __forceinline__ void merge_item(int item, const int* __restrict__ row_pos, const ReqTable* __restrict__ table, int total_rows,
                                           int n_q_heads, const AttnSplit& sp, int cache_last, const float* __restrict__ part_o,
                                           const float2* __restrict__ part_ml, bf16* __restrict__ out, float2* __restrict__ score_ml) {
  const int lane = threadIdx.x & 63, e = lane & 31;
  const int groups = (n_q_heads + 2 * PAIRS - 1) / (2 * PAIRS);
  item = __builtin_amdgcn_readfirstlane(item);
  int r, split_tile, ql, part_base = 0, tile_last_row;
  const int mr = item / groups;
  const int head0 = (item - mr * groups) * (2 * PAIRS) + (lane >> 5);   // and head0 + 2
  if (table) {
    // items run over the rows of the tiles that may be split only (the late tiles of every request)
    if (mr >= table->total_merge_rows) return;
    const ReqDev& rq = table->r[request_of_merge_row(table, mr)];
    const int local = min(rq.long_tile_start, 1 << 20) * BQ + (mr - rq.merge_base);     // row inside the request
    if (local >= rq.n_rows) return;
    r = rq.row_base + local;
    const int lt = local / BQ;
    split_tile = lt - rq.long_tile_start;
    ql = local % BQ;
    part_base = rq.part_base;
    tile_last_row = min(rq.row_base + (lt + 1) * BQ, rq.row_base + rq.n_rows) - 1;
  } else {
    if (mr >= total_rows) return;
    r = mr;
    split_tile = r / BQ;
    ql = r % BQ;
    tile_last_row = min((split_tile + 1) * BQ, total_rows) - 1;
  }
  const int n_kv_tiles = pos_in_cache(row_pos[tile_last_row], cache_last) / BKV + 1;
  if (split_tile < 0 || n_kv_tiles <= sp.long_thr) return;   // this row's tile was done by one workgroup
  const int nc = min(sp.n_chunks, pos_in_cache(row_pos[r], cache_last) / (sp.chunk_tiles * BKV) + 1);
  const size_t cstride = (size_t)n_q_heads * BQ;
  size_t slot0[PAIRS];
  float4 o[PAIRS][AHEAD], acc[PAIRS];
  float2 ml[PAIRS][AHEAD];
  float m[PAIRS], l[PAIRS];
#pragma unroll
  for (int p = 0; p < PAIRS; ++p) {
    slot0[p] = ((size_t)(part_base + split_tile * sp.n_chunks) * n_q_heads + min(head0 + 2 * p, n_q_heads - 1)) * BQ + ql;
    acc[p] = make_float4(0.f, 0.f, 0.f, 0.f);
    l[p] = 0.f;
  }
  auto fetch = [&](int c) {   // the chunks c .. c + AHEAD - 1, the last one again behind it
#pragma unroll
    for (int p = 0; p < PAIRS; ++p)
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        const size_t slot = slot0[p] + min(c + u, nc - 1) * cstride;
        ml[p][u] = part_ml[slot];
        o[p][u] = *reinterpret_cast<const float4*>(part_o + slot * PROW + 4 * e);
      }
  };
  // The common reference exponent (one chunk per lane, 32 at a time), then the sums in chunk order.
#pragma unroll
  for (int p = 0; p < PAIRS; ++p) m[p] = part_ml[slot0[p] + min(e, nc - 1) * cstride].x;
  fetch(0);
  for (int c = e + 32; c < nc; c += 32)
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) m[p] = fmaxf(m[p], part_ml[slot0[p] + c * cstride].x);
#pragma unroll
  for (int s = 16; s > 0; s >>= 1)
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) m[p] = fmaxf(m[p], __shfl_xor(m[p], s, 64));
  for (int c = 0;;) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      if (c + u >= nc) break;   // uniform
#pragma unroll
      for (int p = 0; p < PAIRS; ++p) {
        const float wgt = (ml[p][u].x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ml[p][u].x - m[p]);
        l[p] += ml[p][u].y * wgt;
        acc[p].x += o[p][u].x * wgt;
        acc[p].y += o[p][u].y * wgt;
        acc[p].z += o[p][u].z * wgt;
        acc[p].w += o[p][u].w * wgt;
      }
    }
    c += AHEAD;
    if (c >= nc) break;
    fetch(c);
  }
#pragma unroll
  for (int p = 0; p < PAIRS; ++p) {
    const int head = head0 + 2 * p;
    if (head >= n_q_heads) continue;
    if (score_ml && e == 0) score_ml[(size_t)r * n_q_heads + head] = make_float2(m[p], l[p]);
    const float inv = 1.0f / l[p];
    uint2 pk;
    pk.x = (uint32_t)f32_to_bf16(acc[p].x * inv).v | ((uint32_t)f32_to_bf16(acc[p].y * inv).v << 16);
    pk.y = (uint32_t)f32_to_bf16(acc[p].z * inv).v | ((uint32_t)f32_to_bf16(acc[p].w * inv).v << 16);
    *reinterpret_cast<uint2*>(out + ((size_t)r * n_q_heads + head) * DH + 4 * e) = pk;
  }
}

template <int PAIRS, int AHEAD>
__global__ void __launch_bounds__(256)
attn_merge_kernel(const int* __restrict__ row_pos, const ReqTable* __restrict__ table, int total_rows, int n_q_heads, AttnSplit sp,
                  int cache_last, const float* __restrict__ part_o, const float2* __restrict__ part_ml, bf16* __restrict__ out,
                  float2* __restrict__ score_ml) {
  merge_item<PAIRS, AHEAD>((int)blockIdx.x * 4 + (threadIdx.x >> 6), row_pos, table, total_rows, n_q_heads, sp, cache_last, part_o, part_ml, out, score_ml);
}

// A decoding step with influence sums, its KV ranges split: workgroups below `merge_wgs` merge, the others add the rows' weights to
// the influence vectors, 64 keys each (influence_add_kernel), and for that work the heads' merged exponents and sums out for
// themselves.  Both hang on the same partial results, so one launch does for two: 6.0 + 4.6 -> 6.6 us (32 heads x 5k keys).
// Four wavefronts share the heads; the weights of a key are added up head by head in ascending order.
static constexpr int kInfMaxHeads = 64;   // of a model that takes this path (LDS)
__global__ void __launch_bounds__(256)
attn_merge_influence_kernel(const int* __restrict__ row_pos, const int* __restrict__ row_req, const ReqTable* __restrict__ table,
                            int total_rows, int n_q_heads, AttnSplit sp, int cache_last, const float* __restrict__ part_o,
                            const float2* __restrict__ part_ml, bf16* __restrict__ out, const float* __restrict__ scores, int scores_len,
                            const float2* __restrict__ score_ml, InfluencePtrs inf, int merge_wgs, int wgs_per_row) {
  __shared__ float weight[kInfMaxHeads][64];
  __shared__ float2 pair[kInfMaxHeads];
  if ((int)blockIdx.x < merge_wgs) {
    merge_item<1, 8>((int)blockIdx.x * 4 + (threadIdx.x >> 6), row_pos, table, total_rows, n_q_heads, sp, cache_last, part_o, part_ml, out, nullptr);
    return;
  }
  const int row = ((int)blockIdx.x - merge_wgs) / wgs_per_row;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = (((int)blockIdx.x - merge_wgs) % wgs_per_row) * 64 + lane;
  const int pos = pos_in_cache(row_pos[row], cache_last);
  if (j - lane > pos) return;   // uniform
  const int req = row_req[row] & kRowReqMask;
  float* const dst = inf.s_inf[req];
  if (dst == nullptr) return;   // uniform
  const ReqDev& rq = table->r[req];
  const bool is_split = rq.long_tile_start == 0 && pos / BKV + 1 > sp.long_thr;
  const int nc = is_split ? min(sp.n_chunks, pos / (sp.chunk_tiles * BKV) + 1) : 0;
  const size_t slot0 = (size_t)rq.part_base * n_q_heads * BQ, cstride = (size_t)n_q_heads * BQ;
  const float old = wave == 0 && j <= pos ? dst[j] : 0.f;
  const float* s = scores + (size_t)row * n_q_heads * scores_len + min(j, pos);
  float v[kInfMaxHeads / 4];
#pragma unroll
  for (int i = 0; i < kInfMaxHeads / 4; ++i) v[i] = s[(size_t)min(wave + 4 * i, n_q_heads - 1) * scores_len];
  // Merged pair of a head: eight lanes, lane c & 7 reads chunk c, eight of its chunks at a time; the sum runs in chunk order.
  for (int h0 = 0; h0 < n_q_heads; h0 += 32) {
    const int h = h0 + (tid >> 3), cl = tid & 7;
    float m = -INFINITY, l = 0.f;
    if (is_split) {   // uniform
      const float2* ml = part_ml + slot0 + (size_t)min(h, n_q_heads - 1) * BQ;
      float2 t[8];
      auto load = [&](int c0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = ml[min(c0 + 8 * i + cl, nc - 1) * cstride];
      };
      for (int c0 = 0; c0 < nc; c0 += 64) {
        load(c0);
#pragma unroll
        for (int i = 0; i < 8; ++i) m = fmaxf(m, t[i].x);   // past the last chunk: the last one again
      }
#pragma unroll
      for (int o = 4; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
      for (int c0 = 0; c0 < nc; c0 += 64) {
        if (nc > 64) load(c0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if (c0 + 8 * i >= nc) continue;   // uniform
          const float w = t[i].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(t[i].x - m);
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const float tk = __shfl(t[i].y, (lane & 56) + k, 64), wk = __shfl(w, (lane & 56) + k, 64);
            if (c0 + 8 * i + k < nc) l = __builtin_fmaf(tk, wk, l);
          }
        }
      }
    } else if (h < n_q_heads) {   // one workgroup had the whole range and left the pair
      const float2 p = score_ml[(size_t)row * n_q_heads + h];
      m = p.x;
      l = p.y;
    }
    if (cl == 0 && h < n_q_heads) pair[h] = make_float2(m, l);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kInfMaxHeads / 4; ++i) {
    const int h = wave + 4 * i;
    if (h < n_q_heads) weight[h][lane] = __builtin_amdgcn_exp2f(v[i] * 1.4426950408889634f - pair[h].x) / pair[h].y;
  }
  __syncthreads();
  if (wave > 0 || j > pos) return;
  float acc = 0.f;
  for (int h = 0; h < n_q_heads; ++h) acc += weight[h][lane];
  dst[j] = old + acc;
}

static int g_force_chunk_tiles = 0;   // 0: by shape; > 0: this many KV tiles per chunk
void set_attention_chunk_tiles(int t) { g_force_chunk_tiles = t; }
int attention_forced_chunk_tiles() { return g_force_chunk_tiles; }

// Partial results: per (slot, head, query row) DH un-normalised output floats, stored PROW floats apart, and one
// (reference exponent, sum) pair behind all of them.  The row pitch is not a power of two on purpose: with 512-byte
// rows the slots of one KV chunk of successive query tiles lie a multiple of 1 MiB apart whenever the chunk count is
// even, and the workgroups that finish together (same chunk, neighbouring tiles) then write to the same memory
// channels (measured: even chunk counts ran the split layers up to twice as slow).
size_t attention_partial_floats(int total_slots, int n_q_heads) {
  return (size_t)total_slots * n_q_heads * BQ * (PROW + 2);
}

template <int G>
static hipError_t launch_g(const bf16* q, const int* row_pos, const ReqTable* table, int fixed_seq, int total_rows,
                           int total_tiles, const bf16* k_pool, const bf16* v_pool, KvGeom g, bf16* out,
                           AttnSplit sp, float* part, hipStream_t st) {
  // with a table, total_tiles is the phase's number of work items (ReqTable::total_items, or an upper bound of it)
  const long items = table ? (long)total_tiles : (long)total_tiles * sp.n_chunks;
  dim3 grid((unsigned)(items * g.n_kv_heads));
  float* part_o = part;
  float2* part_ml = reinterpret_cast<float2*>(part + (size_t)sp.total_slots * g.n_kv_heads * G * BQ * PROW);
  // more than the 64 KB a kernel gets without asking
  static std::atomic<unsigned long long> told{0};
  hipError_t e = allow_dynamic_lds((const void*)attn_mfma_kernel<G>, ATTN_LDS_BYTES, told);
  if (e != hipSuccess) return e;
  attn_mfma_kernel<G><<<grid, 64 * (G < 4 ? 4 : G), ATTN_LDS_BYTES, st>>>(q, row_pos, table, fixed_seq, total_rows, total_tiles, k_pool, v_pool,
                                                                          g, out, sp, part_o, part_ml);
  return hipGetLastError();
}

hipError_t launch_attention_bf16(const bf16* q, const int* row_pos, const int* row_req, const ReqTable* table,
                                 int fixed_seq, int total_rows, int total_tiles, const bf16* k_pool,
                                 const bf16* v_pool, KvGeom g, int n_q_heads, bf16* out, AttnSplit sp, float* part,
                                 hipStream_t st, float* scores, int scores_len, int merge_rows, bool one_row,
                                 const InfluencePtrs* inf, bool* inf_done) {
  if (total_rows <= 0) return hipSuccess;
  const int G = n_q_heads / g.n_kv_heads;
  if (!part || sp.total_slots <= 0) sp = attention_no_split();
  hipError_t e;
  if (table && one_row && G <= 8) {
    const unsigned grid = (unsigned)total_tiles * (unsigned)g.n_kv_heads;
    float2* part_ml = reinterpret_cast<float2*>(part + (size_t)sp.total_slots * n_q_heads * BQ * PROW);
    if (scores)
      attn_decode_kernel<true><<<grid, 256, 0, st>>>(q, row_pos, table, k_pool, v_pool, g, G, out, sp, part, part_ml, scores,
                                                     scores_len, influence_pairs(scores, total_rows, n_q_heads, scores_len));
    else
      attn_decode_kernel<false><<<grid, 256, 0, st>>>(q, row_pos, table, k_pool, v_pool, g, G, out, sp, part, part_ml, nullptr, 0, nullptr);
    e = hipGetLastError();
  } else if (scores) {   // only one live row per request has scores written, by the kernel above
    return hipErrorInvalidValue;
  } else switch (G) {
#define RC_ATTN_CASE(GG) \
    case GG: e = launch_g<GG>(q, row_pos, table, fixed_seq, total_rows, total_tiles, k_pool, v_pool, g, out, sp, part, st); break;
    RC_ATTN_CASE(1) RC_ATTN_CASE(2) RC_ATTN_CASE(3) RC_ATTN_CASE(4)
    RC_ATTN_CASE(5) RC_ATTN_CASE(6) RC_ATTN_CASE(7) RC_ATTN_CASE(8)
#undef RC_ATTN_CASE
    default:  // wider groups: one wavefront per (row, head) on the vector ALUs
      return launch_attention_simt(q, row_pos, row_req, table, fixed_seq, total_rows, k_pool, v_pool, g,
                                         n_q_heads, out, st);
  }
  if (e != hipSuccess || sp.n_chunks == 1) return e;
  const float2* part_ml = reinterpret_cast<const float2*>(part + (size_t)sp.total_slots * n_q_heads * BQ * PROW);
  // with a table, merge_rows (the rows of the tiles that may be split, or an upper bound) sizes the merge grid
  const int heads = one_row ? 2 : 4;   // per wavefront
  const int items = (table ? merge_rows : total_rows) * ((n_q_heads + heads - 1) / heads);
  if (items <= 0) return hipSuccess;
  const int merge_wgs = (items + 3) / 4;
  if (inf && scores && table && one_row && G <= 8 && n_q_heads <= kInfMaxHeads) {
    const int wgs_per_row = (scores_len + 63) / 64;
    attn_merge_influence_kernel<<<merge_wgs + total_rows * wgs_per_row, 256, 0, st>>>(
        row_pos, row_req, table, total_rows, n_q_heads, sp, g.last_pos, part, part_ml, out, scores, scores_len,
        influence_pairs(scores, total_rows, n_q_heads, scores_len), *inf, merge_wgs, wgs_per_row);
    *inf_done = true;
    return hipGetLastError();
  }
  (one_row ? attn_merge_kernel<1, 8> : attn_merge_kernel<2, 4>)<<<merge_wgs, 256, 0, st>>>(
      row_pos, table, total_rows, n_q_heads, sp, g.last_pos, part, part_ml, out,
      scores ? influence_pairs(scores, total_rows, n_q_heads, scores_len) : nullptr);
  return hipGetLastError();
}

template <>
hipError_t launch_attention<bf16>(const bf16* q, const int* row_pos, const int* row_req, const ReqTable* table,
                                  int fixed_seq, int total_rows, int total_tiles, const bf16* k_pool,
                                  const bf16* v_pool, KvGeom g, int n_q_heads, bf16* out, hipStream_t st) {
  const AttnSplit sp = attention_no_split();
  return launch_attention_bf16(q, row_pos, row_req, table, fixed_seq, total_rows, total_tiles, k_pool, v_pool, g,
                               n_q_heads, out, sp, nullptr, st);
}

}  // namespace rc
