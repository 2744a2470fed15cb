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
// This file holds the form for few keys (below 65536 head-problem tokens): 32 keys per
// wavefront in registers, so that there are many workgroups, and the centroids through LDS in
// double-buffered chunks of 64 rows.  k_assign_stream (tables of at most 512 centroids) and
// k_assign_wide (larger ones) take the rest.
#include <atomic>

#include "chunk_sort.hpp"

namespace ck {

constexpr int CHUNK_ROWS = 64;             // centroid rows per LDS chunk (two MFMA tiles)
constexpr int LDS_ROW = D + 8;             // bf16 elements per LDS row: 272 B, rows shift 4 banks

// HAS_BIAS (l2 metric): a per-centroid bias, held in LDS, is added to every
// similarity before the argmax; it takes 8 KB more, so three workgroups fit a CU instead of four.
constexpr int SM_WAVES = 4;
template <bool HAS_BIAS>
__global__ __launch_bounds__(SM_WAVES * 64, HAS_BIAS ? 3 : 4) void k_assign(
    const bf16* __restrict__ K, const bf16* __restrict__ mu_hat, int32_t* __restrict__ labels,
    float* __restrict__ best_sim, const ChunkIndex chunks, int n_chunks_hp, int label_bits,
    int64_t N_cap, int64_t tok_begin, int64_t tok_count, int c_begin, int c_count,
    const KmCtl ctl) {
  constexpr int WAVES = SM_WAVES, THREADS = WAVES * 64;
  constexpr int SEGS = CHUNK_ROWS * 16 / THREADS;      // 16-byte segments of a chunk per thread
  __shared__ __attribute__((aligned(16))) bf16 lds[2][CHUNK_ROWS * LDS_ROW];
  __shared__ __attribute__((aligned(16))) float lds_bias[HAS_BIAS ? CK_MAX_CLUSTERS + 32 : 4];
  __shared__ int s_changed;

  // one argument per 64-byte line of the argument block: fetched where it is first used, a line would
  // queue behind the key loads
  CK_FETCH_ARG(labels);
  CK_FETCH_ARG(tok_count);
  CK_FETCH_ARG(ctl.first);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, half = lane >> 5;
  const int hp = blockIdx.y;
  if (ctl.skip && ctl.skip[hp] == 0) return;            // converged: whole workgroup leaves
  const bf16* Khp = K + (int64_t)hp * N_cap * D;
  const bf16* Mhp = mu_hat + (int64_t)hp * c_count * D;

  const int n_chunks = (c_count + CHUNK_ROWS - 1) / CHUNK_ROWS;
  const int n_tiles = (c_count + 31) / 32;
  uint4 stage[SEGS];
  // unconditional loads (rows beyond the table re-read its last row and are replaced by zeros when
  // they are written to LDS): under a branch each waits for the one before
  auto fetch = [&](int ch) {
#pragma unroll
    for (int i = 0; i < SEGS; ++i) {
      const int seg = tid + i * THREADS;
      const int r = ch * CHUNK_ROWS + (seg >> 4);
      stage[i] = *reinterpret_cast<const uint4*>(Mhp + (int64_t)(r < c_count ? r : c_count - 1) * D + (seg & 15) * 8);
    }
  };
  auto stash = [&](int buf, int ch) {
#pragma unroll
    for (int i = 0; i < SEGS; ++i) {
      const int seg = tid + i * THREADS;
      const bool real = ch * CHUNK_ROWS + (seg >> 4) < c_count;
      uint4 v = stage[i];
      v.x = real ? v.x : 0u; v.y = real ? v.y : 0u; v.z = real ? v.z : 0u; v.w = real ? v.w : 0u;
      *reinterpret_cast<uint4*>(&lds[buf][(seg >> 4) * LDS_ROW + (seg & 15) * 8]) = v;
    }
  };
  // first centroid chunk ahead of the keys, so that it does not queue behind them
  fetch(0);
  if (tid == 0) s_changed = 0;
  if constexpr (HAS_BIAS) {
    for (int c = tid; c < n_tiles * 32; c += THREADS)
      lds_bias[c] = c < c_count ? ctl.bias[(int64_t)hp * ctl.bias_stride + c] : 0.f;
  }

  // ---- keys of this wavefront into registers, in B-operand layout ----
  const int64_t wave_tok0 = ((int64_t)blockIdx.x * WAVES + wave) * 32;
  bf16x8 bk[8];
  {
    int64_t t = wave_tok0 + col;
    if (t >= tok_count) t = tok_count - 1;              // clamp: result is discarded
    const bf16* row = Khp + (tok_begin + t) * D + half * 8;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) bk[kk] = *reinterpret_cast<const bf16x8*>(row + kk * 16);
  }

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
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bk[kk], acc, 0, 0, 0);
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

  stash(0, 0);
  __syncthreads();

  for (int ch = 0; ch < n_chunks; ++ch) {
    if (ch + 1 < n_chunks) fetch(ch + 1);
    const bf16* buf = lds[ch & 1];
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      const int t = ch * 2 + tile;
      if (t < n_tiles) {                                // wave-uniform
        contract(buf, tile);
        reduce(t);
      }
    }
    if (ch + 1 < n_chunks) stash((ch + 1) & 1, ch + 1);
    __syncthreads();
  }

  // ---- lanes l and l+32 hold the two halves of each key's candidates ----
  // (the centroid buffers are free now: the loop ended with a barrier)
  constexpr int CHUNK = WAVES * 32;                     // tokens of the workgroup = one chunk
  uint32_t* tok = reinterpret_cast<uint32_t*>(&lds[0][0]);   // pack_token words
  const bool count_only = chunks.seg && !chunks.list;   // counts by cluster in place of the words
  if (count_only) {
    static_assert(CK_MAX_CLUSTERS * 4 <= sizeof(lds), "counts");
    for (int c = tid; c < c_count; c += THREADS) tok[c] = 0;
    __syncthreads();
  }
  int diff = 0;
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
    const int64_t t = wave_tok0 + col;
    if (half == 0 && t < tok_count) {
      const int64_t o = (int64_t)hp * N_cap + tok_begin + t;
      if (ctl.changed) diff += (ctl.first || labels[o] != c_begin + bidx) ? 1 : 0;
      labels[o] = c_begin + bidx;
      if (best_sim) best_sim[o] = __uint_as_float(__float_as_uint(best) & 0xFFFFFFF0u);
      if (count_only) atomicAdd(&tok[bidx], 1u);
    }
  }
  if (ctl.changed) {
    const int wsum = __builtin_amdgcn_readlane(wave_inclusive_scan(diff), WAVE - 1);
    if (lane == 0 && wsum) atomicAdd(&s_changed, wsum);
  }
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
  if (ctl.changed && tid == 0 && s_changed) atomicAdd(&ctl.changed[hp], s_changed);
  const int64_t o = (int64_t)hp * n_chunks_hp + blockIdx.x;
  if (count_only) {
    for (int c = tid; c < c_count; c += THREADS) chunks.seg[o * seg_stride(c_count) + c] = tok[c] << 16;
  } else if (chunks.seg) {
    constexpr int W = CHUNK / WAVE, CNT = chunk_sort_cnt_ints(CK_MAX_CLUSTERS) * W;
    static_assert((CHUNK + CNT + 4) * 4 + CHUNK * 2 <= sizeof(lds), "chunk sort scratch");
    int* cnt = reinterpret_cast<int*>(tok) + CHUNK;
    chunk_sort<CHUNK / WAVE, CK_MAX_CLUSTERS, W>(
        tok, c_count, wave, wave < W, cnt, cnt + CNT, reinterpret_cast<uint16_t*>(cnt + CNT + 4),
        chunks.seg + o * seg_stride(c_count), chunks.list + o * CHUNK);
  }
}

static hipError_t launch_assign_small(const Dims& dm, const bf16* K, int64_t tok_begin,
                                      int64_t tok_count, const bf16* mu_hat, int c_begin,
                                      int c_count, int32_t* labels, float* best_sim,
                                      const ChunkIndex& chunks, const KmCtl& ctl, hipStream_t st) {
  constexpr int TOK = SM_WAVES * 32;
  const int n_chunks = (int)((tok_count + TOK - 1) / TOK);
  int label_bits = 0;
  while ((1 << label_bits) < c_count) ++label_bits;
  const auto kernel = ctl.bias ? k_assign<true> : k_assign<false>;
  hipLaunchKernelGGL(kernel, dim3(n_chunks, dm.HP), dim3(SM_WAVES * 64), 0, st, K, mu_hat, labels,
                     best_sim, chunks, n_chunks, label_bits, dm.N_cap, tok_begin, tok_count, c_begin,
                     c_count, ctl);
  return hipGetLastError();
}

// Chunk size of the counting sort = the tokens of the workgroup (a block of its tokens in
// k_assign_stream) that leaves the label-ordered index of exactly these.
int assign_tile_tokens(const Dims& dm, int64_t tok_count) {
  return tok_count * dm.HP >= 64 * 1024 ? 512 : 128;
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
  if (assign_tile_tokens(dm, tok_count) != 512)
    return launch_assign_small(dm, K, tok_begin, tok_count, mu_hat, c_begin, c_count, labels, best_sim,
                               chunks, ctl, st);
  if (assign_stream_fits(c_count))
    return launch_assign_stream(dm, K, tok_begin, tok_count, mu_hat, c_begin, c_count, labels,
                                best_sim, chunks, ctl, compute_units(), st);
  return launch_assign_wide(dm, K, tok_begin, tok_count, mu_hat, c_begin, c_count, labels, best_sim,
                            chunks, ctl, st);
}

}  // namespace ck
