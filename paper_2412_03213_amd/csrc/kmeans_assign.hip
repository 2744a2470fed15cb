// K-means assignment step (paper Section III-B): every key gets the label of the
// centroid with the largest cosine similarity.  Since the key's own length does
// not change the argmax, this is argmax_c <k_i, mu_hat_c> with unit-length
// centroids: a dense [tokens x d] . [d x C] contraction, run on bf16 MFMA with
// the argmax folded into the accumulator read-out, so the similarity matrix
// never exists in memory.
//
// Mapping (gfx950, v_mfma_f32_32x32x16_bf16): the CENTROIDS are the A operand
// (rows of the 32x32 result) and the KEYS the B operand (columns).  A lane then
// owns one key column and 16 centroid rows of every tile, so the running
// (max, argmax) lives in plain registers and only one exchange between lanes
// l and l+32 is needed at the very end.
//
// This file holds the form for few keys or small tables (assign_tile_tokens): 32 keys per
// wavefront in registers, so that there are many workgroups, and the centroids through LDS in
// double-buffered chunks of 64 rows.  k_assign_stream (tables of at most 512 centroids) and
// k_assign_wide (larger ones) take the rest.
#include <atomic>
#include <type_traits>

#include "chunk_sort.hpp"
#include "key_operand.hpp"

namespace ck {

constexpr int CHUNK_ROWS = 64;             // centroid rows per LDS chunk (two MFMA tiles)
constexpr int LDS_ROW = D + 8;             // bf16 elements per LDS row: 272 B, rows shift 4 banks

// One workgroup takes one chunk of the sort, 32 tokens per wavefront.
// Bound: latency.  A workgroup asks for its table rows (the first two chunks of them), bias, keys and
// previous labels in one go; the keys come in whole 64-byte pieces and change lanes in LDS
// (key_operand.hpp).  A table of more than two chunks is requested two chunks ahead.  Before, keys came
// in operand layout behind the bias, the second chunk behind the first barrier, the previous labels at
// the end, and the changed ones were counted by an atomic per workgroup.  Ten iterations, us: 8 x 2985 x 37
// 96 -> 93, 4 x 15738 x 98 155 -> 142, the same by l2 185 -> 172, by l2 until convergence 236 -> 181.
// HAS_BIAS (l2 metric): a per-centroid bias, held in LDS, is added to every similarity before the
// argmax.  ONE: a table of one chunk.  TIGHT: the keys through half of the LDS, so that a compute unit
// holds four workgroups of four wavefronts in place of three.  Where there are as many workgroups, ten
// iterations without / with it: 8 x 20000 x 128 221 / 207 us, 8 x 18000 x 160 228 / 219, 20 x 7000 x 100 217 /
// 208, 60 x 2500 x 100 300 / 293, but 8 x 20000 x 128 by l2 253 / 254, 250 x 700 x 80 598 / 604, and with eight
// wavefronts, where ragged ranges alone make more workgroups than compute units, 33 x 1900 x 100 190 / 197.
// Where there are not as many it costs: 4 x 15738 x 98 142 / 145.
template <bool HAS_BIAS, int WAVES, bool ONE, bool TIGHT, bool LOOK>
__global__ __launch_bounds__(WAVES * 64, 4) void k_assign(
    const bf16* __restrict__ K, const bf16* __restrict__ mu_hat, int32_t* __restrict__ labels,
    float* __restrict__ best_sim, const ChunkIndex chunks, int n_chunks_hp, int label_bits,
    int64_t N_cap, int64_t tok_begin, int64_t tok_count, int c_begin, int c_count,
    const KmCtl ctl, const TileMap map) {
  constexpr int THREADS = WAVES * 64, BUFS = ONE ? 1 : 2;
  constexpr int SEGS = CHUNK_ROWS * 16 / THREADS;      // 16-byte segments of a chunk per thread
  constexpr int CHUNK = WAVES * 32;                    // tokens of the workgroup = one chunk of the sort
  constexpr int W = CHUNK / WAVE, CNT = chunk_sort_cnt_ints(ONE ? CHUNK_ROWS : CK_MAX_CLUSTERS) * W;
  constexpr int STAGE = TIGHT ? KEY_STAGE_ELEMS / 2 : KEY_STAGE_ELEMS;
  constexpr int SORT_BYTES = (CHUNK + CNT + 8) * 4 + CHUNK * 2;
  constexpr int TABLE_BYTES = BUFS * CHUNK_ROWS * LDS_ROW * 2;
  __shared__ __attribute__((aligned(16))) char lds_raw[SORT_BYTES > TABLE_BYTES ? SORT_BYTES : TABLE_BYTES];
  __shared__ __attribute__((aligned(16))) bf16 key_stage[WAVES * STAGE];
  __shared__ __attribute__((aligned(16))) float lds_bias[HAS_BIAS ? (ONE ? CHUNK_ROWS : CK_MAX_CLUSTERS + 32) : 4];
  __shared__ int s_changed;
  bf16* lds = reinterpret_cast<bf16*>(lds_raw);        // [BUFS][CHUNK_ROWS][LDS_ROW]

  // one argument per 64-byte line of the argument block: fetched where it is first used, a line would
  // queue behind the key loads
  CK_FETCH_ARG(labels);
  CK_FETCH_ARG(tok_count);
  CK_FETCH_ARG(ctl.first);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, half = lane >> 5;
  int wg, hp;
  if (!map.mine<true, LOOK>(wg, hp)) return;
  const bf16* Khp = K + ((int64_t)hp * N_cap + tok_begin) * D;
  const bf16* Mhp = mu_hat + (int64_t)hp * c_count * D;

  const int n_chunks = ONE ? 1 : (c_count + CHUNK_ROWS - 1) / CHUNK_ROWS;
  const int n_tiles = (c_count + 31) / 32;
  // unconditional loads (rows beyond the table re-read its last row and are replaced by zeros when
  // they are written to LDS): under a branch each waits for the one before
  auto fetch = [&](uint4 (&stage)[SEGS], int ch) {
#pragma unroll
    for (int i = 0; i < SEGS; ++i) {
      const int seg = tid + i * THREADS;
      const int r = ch * CHUNK_ROWS + (seg >> 4);
      stage[i] = *reinterpret_cast<const uint4*>(Mhp + (int64_t)(r < c_count ? r : c_count - 1) * D + (seg & 15) * 8);
    }
  };
  auto stash = [&](const uint4 (&stage)[SEGS], int ch) {
#pragma unroll
    for (int i = 0; i < SEGS; ++i) {
      const int seg = tid + i * THREADS;
      const bool real = ch * CHUNK_ROWS + (seg >> 4) < c_count;
      uint4 v = stage[i];
      v.x = real ? v.x : 0u; v.y = real ? v.y : 0u; v.z = real ? v.z : 0u; v.w = real ? v.w : 0u;
      *reinterpret_cast<uint4*>(&lds[((ONE ? 0 : ch & 1) * CHUNK_ROWS + (seg >> 4)) * LDS_ROW + (seg & 15) * 8]) = v;
    }
  };
  // the table ahead of the keys, so that it does not queue behind them
  uint4 first[BUFS][SEGS];
#pragma unroll
  for (int i = 0; i < BUFS; ++i) fetch(first[i], i);
  float b0 = 0.f;
  if constexpr (HAS_BIAS) b0 = ctl.bias[(int64_t)hp * ctl.bias_stride + (tid < c_count ? tid : 0)];

  // ---- keys of this wavefront ----
  const int64_t wave_tok0 = ((int64_t)wg * WAVES + wave) * 32;
  KeyTile<1> keys;
  keys.load(Khp, wave_tok0, tok_count, lane);
  const int64_t my_tok = wave_tok0 + col;
  int32_t* my_label = labels + (int64_t)hp * N_cap + tok_begin + (my_tok < tok_count ? my_tok : tok_count - 1);
  int before = -1;
  if (ctl.changed) before = *my_label;                  // not looked at where there are none yet

#pragma unroll
  for (int i = 0; i < BUFS; ++i) stash(first[i], i);
  if constexpr (HAS_BIAS) {
    if (tid < n_tiles * 32) lds_bias[tid] = tid < c_count ? b0 : 0.f;
    for (int c = tid + THREADS; c < n_tiles * 32; c += THREADS)
      lds_bias[c] = c < c_count ? ctl.bias[(int64_t)hp * ctl.bias_stride + c] : 0.f;
  }
  if (tid == 0) s_changed = 0;
  if (map.stopped<LOOK>(hp)) return;                          // the word has travelled with the loads above

  // Running maximum as a "packed" float: the low 4 mantissa bits of
  // every similarity are replaced by 15 - (accumulator slot), so one v_max3 chain
  // finds value and slot together and equal values resolve to the lower centroid.
  // The truncation moves a similarity by < 2^-19 relative, far inside the 1e-4
  // cosine near-tie band in which labels may legitimately differ.  (Exception to
  // "lower id wins": when a key's best similarity is NEGATIVE and bit-equal for two
  // of the 16 rows one lane holds of a tile, the slot bits order the other way and
  // the higher of the two rows is taken -- an exact tie, so inside that band too.)
  float bestp = -INFINITY;
  int btile = 0;
  floatx16 acc;

  // similarities of tile `tile` of a chunk buffer against the keys
  auto contract = [&](const bf16* buf, int tile) {
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    const bf16* arow = buf + (tile * 32 + col) * LDS_ROW + half * 8;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(arow + kk * 16);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, keys.operand(0, kk), acc, 0, 0, 0);
    }
  };
  // folds the accumulators of tile `tile_id` into the running maximum
  auto reduce = [&](int tile_id) {
    const int row0 = tile_id * 32;
    // accumulator i of a lane is centroid row 8*(i/4) + 4*half + i%4 of the tile
    if constexpr (HAS_BIAS) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const floatx4 b = *reinterpret_cast<const floatx4*>(&lds_bias[row0 + 8 * j + 4 * half]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * j + e] += b[e];
      }
    }
    if (row0 + 32 > c_count) {                         // wave-uniform: zero-padded rows lose
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int c = row0 + 8 * (i >> 2) + 4 * half + (i & 3);
        if (c >= c_count) acc[i] = -3.0e38f;           // finite: the slot bits must not make a NaN
      }
    }
    float p[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
      p[i] = __uint_as_float((__float_as_uint(acc[i]) & 0xFFFFFFF0u) | (uint32_t)(15 - i));
    float m = bestp;
#pragma unroll
    for (int i = 0; i < 16; i += 2) m = fmaxf(fmaxf(m, p[i]), p[i + 1]);
    // a later tile takes over only with a strictly larger (truncated) value: an equal
    // one would be a higher centroid id, whatever its slot bits say
    const bool up = __uint_as_float(__float_as_uint(m) & 0xFFFFFFF0u) >
                    __uint_as_float(__float_as_uint(bestp) & 0xFFFFFFF0u);
    btile = up ? tile_id : btile;
    bestp = up ? m : bestp;
  };

  uint4 next[SEGS];
  if constexpr (!ONE)
    if (n_chunks > 2) fetch(next, 2);
  if constexpr (TIGHT) keys.to_operand_16(key_stage + wave * STAGE, lane);
  else keys.to_operand(key_stage + wave * STAGE, lane);
  __syncthreads();

  for (int ch = 0; ch < n_chunks; ++ch) {
    const bf16* buf = lds + (ONE ? 0 : ch & 1) * CHUNK_ROWS * LDS_ROW;
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      const int t = ch * 2 + tile;
      if (t < n_tiles) {                                // wave-uniform
        contract(buf, tile);
        reduce(t);
      }
    }
    if constexpr (!ONE) {
      // chunk ch + 1 is in the other buffer; ch + 2 takes this one's place
      if (ch + 1 < n_chunks) __syncthreads();
      if (ch + 2 < n_chunks) {
        stash(next, ch + 2);
        if (ch + 3 < n_chunks) fetch(next, ch + 3);
      }
    }
  }
  __syncthreads();                                      // the table's LDS is free

  // ---- lanes l and l+32 hold the two halves of each key's candidates ----
  uint32_t* tok = reinterpret_cast<uint32_t*>(lds_raw);   // pack_token words
  const bool count_only = chunks.seg && !chunks.list;   // counts by cluster in place of the words
  if (count_only) {
    static_assert((ONE ? CHUNK_ROWS : CK_MAX_CLUSTERS) * 4 <= sizeof(lds_raw), "counts");
    for (int c = tid; c < c_count; c += THREADS) tok[c] = 0;
    __syncthreads();
  }
  bool moved = false;
  const int slot = 15 - (int)(__float_as_uint(bestp) & 15u);
  float best = bestp;
  int bidx = btile * 32 + 8 * (slot >> 2) + 4 * half + (slot & 3);
  {
    const float ob = __shfl_xor(best, 32, WAVE);
    const int oi = __shfl_xor(bidx, 32, WAVE);
    // compare without the slot bits so that an exact tie goes to the lower id
    const float bt = __uint_as_float(__float_as_uint(best) & 0xFFFFFFF0u);
    const float ot = __uint_as_float(__float_as_uint(ob) & 0xFFFFFFF0u);
    if (ot > bt || (ot == bt && oi < bidx)) {
      best = ob;
      bidx = oi;
    }
    // a key with a NaN or infinite channel may have no similarity that is a number: a padded
    // row has won then, and the key goes to the last cluster
    bidx = bidx < c_count ? bidx : c_count - 1;
    if (half == 0 && my_tok < tok_count) {
      moved = ctl.first || before != c_begin + bidx;
      *my_label = c_begin + bidx;
      if (best_sim) best_sim[my_label - labels] = __uint_as_float(__float_as_uint(best) & 0xFFFFFFF0u);
      if (count_only) atomicAdd(&tok[bidx], 1u);
    }
  }
  if (ctl.changed && __ballot(moved) && lane == 0) s_changed = 1;
  if (chunks.list) {
    // 32 tokens per wavefront: the even one of a pair ranks both halves of the group
    uint32_t* raw = tok + CHUNK;
    if (half == 0) raw[wave * 32 + col] = (uint32_t)bidx;
    __syncthreads();
    if ((wave & 1) == 0)
      tok[wave * 32 + lane] = pack_token((int)raw[wave * 32 + lane],
                                         wave_tok0 + lane < tok_count, label_bits);
  }
  if (chunks.seg || ctl.changed) __syncthreads();
  if (ctl.changed && tid == 0 && s_changed) ctl.changed[hp] = 1;
  const int64_t o = (int64_t)hp * n_chunks_hp + wg;
  if (count_only) {
    for (int c = tid; c < c_count; c += THREADS) chunks.seg[o * seg_stride(c_count) + c] = tok[c] << 16;
  } else if (chunks.seg) {
    int* cnt = reinterpret_cast<int*>(tok) + CHUNK;
    chunk_sort<CHUNK / WAVE, ONE ? CHUNK_ROWS : CK_MAX_CLUSTERS, W>(
        tok, c_count, wave, wave < W, cnt, cnt + CNT, reinterpret_cast<uint16_t*>(cnt + CNT + 8),
        chunks.seg + o * seg_stride(c_count), chunks.list + o * CHUNK);
  }
}

template <int WAVES>
static hipError_t launch_assign_few(const Dims& dm, const bf16* K, int64_t tok_begin,
                                    int64_t tok_count, const bf16* mu_hat, int c_begin,
                                    int c_count, int32_t* labels, float* best_sim,
                                    const ChunkIndex& chunks, const KmCtl& ctl, int n_cu,
                                    hipStream_t st) {
  constexpr int TOK = WAVES * 32;
  const int n_chunks = (int)((tok_count + TOK - 1) / TOK);
  int label_bits = 0;
  while ((1 << label_bits) < c_count) ++label_bits;
  // more workgroups than the compute units hold of the other form
  const bool tight = (int64_t)n_chunks * dm.HP > (int64_t)n_cu * (12 / WAVES);
  const TileMap map(n_chunks, dm.HP, ctl.running);
  auto launch = [&](auto look) {
    constexpr bool L = decltype(look)::value;
    const auto kernel =
        c_count <= CHUNK_ROWS ? (ctl.bias ? k_assign<true, WAVES, true, false, L> : k_assign<false, WAVES, true, false, L>)
        : tight               ? (ctl.bias ? k_assign<true, WAVES, false, true, L> : k_assign<false, WAVES, false, true, L>)
                              : (ctl.bias ? k_assign<true, WAVES, false, false, L> : k_assign<false, WAVES, false, false, L>);
    hipLaunchKernelGGL(kernel, map.grid(), dim3(WAVES * 64), 0, st, K, mu_hat, labels,
                       best_sim, chunks, n_chunks, label_bits, dm.N_cap, tok_begin, tok_count, c_begin,
                       c_count, ctl, map);
  };
  ctl.running.first ? launch(std::true_type()) : launch(std::false_type());
  return hipGetLastError();
}

// Chunk size of the counting sort = the tokens of the workgroup (a block of its tokens in
// k_assign_stream) that leaves the label-ordered index of exactly these.
// 128 or 256 (k_assign) where that gives one workgroup per compute unit: the launch is as long as one
// workgroup, and with two on some units the others wait.  Ten iterations, 128 / 256 / 512 tokens, us
// (head-problems x tokens x clusters): 4 x 6000 x 70 112 / 117 / 147, 1 x 24000 x 400 166 / 169 / 205;
// 8 x 5000 x 102 144 / 142 / 172, 1 x 40000 x 700 247 / 222 / 265, 1 x 55000 x 500 223 / 200 / 236.
// Beyond, k_assign_stream puts 512 tokens on a unit, k_assign_wide (more than 512 clusters) as well.
// Where the contraction is nothing (64 clusters) many small workgroups stay ahead of both: 16 x 4400 x 40
// 130 / 132 / 155, 128 x 1100 x 13 151 / 155 / 212, 32 x 7800 x 40 239 / 233 / 273, 128 x 6250 x 40
// 607 / 611 / 699, 8 x 60000 x 60 432 / 427 / 468 (2 x 60000 x 50 280 / 270 / 276).  With a few more tiles
// only while the units would not be full, in the first two rounds of them: 7 x 10000 x 102 148 / 156 / 167,
// 8 x 20000 x 128 209 / 216 / 247, 8 x 8750 x 160 153 / 160 / 167.  These lines (70 and 60 per cent, 160
// clusters) are where 512 was ahead while tiles were dealt out one by one.  By eighths it is no longer: beyond
// them 8 x 15000 x 102 172 / 165 / 175, 8 x 25000 x 128 255 / 262 / 268, 8 x 32000 x 66 302 / 299 / 310,
// 8 x 11250 x 160 155 / 160 / 169, 8 x 8750 x 200 181 / 187 / 186, 4 x 32768 x 100 202 / 197 / 201.
int assign_tile_tokens(const Dims& dm, int64_t tok_count, int c_count) {
  // a constant and not the current device's: the size of a workspace follows from this
  constexpr int64_t CUS = 256, ROUND = CUS * 512;
  const int64_t tokens = tok_count * dm.HP;
  if (tokens <= CUS * 128) return 128;
  if (tokens <= CUS * 256) return 256;
  if (tok_count > 128 * CHUNK_RUNS_MAX) return 512;     // more chunks than the index holds
  if (c_count <= 64) return 128;
  const int64_t rounds = (tokens + ROUND - 1) / ROUND;
  const int fill = c_count <= 128 ? 70 : c_count <= 160 ? 60 : 0;   // per cent
  return rounds <= 2 && tokens * 100 <= rounds * ROUND * fill ? 128 : 512;
}

// Compute units of the current device, asked once per device (the query costs a few
// microseconds of host time and a clustering call launches the kernel many times).
static int compute_units() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
      n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

hipError_t launch_assign(const Dims& dm, const bf16* K, int64_t tok_begin, int64_t tok_count,
                         const bf16* mu_hat, int c_begin, int c_count, int32_t* labels,
                         float* best_sim, const ChunkIndex& chunks, const KmCtl& ctl,
                         hipStream_t st) {
  const int tokens = chunks.tokens ? chunks.tokens : assign_tile_tokens(dm, tok_count, c_count);
  if (tokens == 128)
    return launch_assign_few<4>(dm, K, tok_begin, tok_count, mu_hat, c_begin, c_count, labels, best_sim,
                                chunks, ctl, compute_units(), st);
  if (tokens == 256)
    return launch_assign_few<8>(dm, K, tok_begin, tok_count, mu_hat, c_begin, c_count, labels, best_sim,
                                chunks, ctl, compute_units(), st);
  if (assign_stream_fits(c_count))
    return launch_assign_stream(dm, K, tok_begin, tok_count, mu_hat, c_begin, c_count, labels,
                                best_sim, chunks, ctl, compute_units(), st);
  return launch_assign_wide(dm, K, tok_begin, tok_count, mu_hat, c_begin, c_count, labels, best_sim,
                            chunks, ctl, st);
}

}  // namespace ck
