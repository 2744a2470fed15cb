// K-means assignment step (paper Section III-B), streaming form: see k_assign in
// kmeans_assign.hip for the mapping onto v_mfma_f32_32x32x16_bf16 and the packed
// running maximum.  This file is compiled with the MFMA results kept in vector
// registers (the read-out works on them directly) and the operands that only the
// matrix cores touch in the accumulator half of the register file.
#include <type_traits>

#include "chunk_sort.hpp"

namespace ck {

constexpr int LDS_ROW = D + 8;             // bf16 elements per LDS row: 272 B, rows shift 4 banks

// ---------------------------------------------------------------- streaming form
// For tables of at most 512 centroids (the paper's C0 = L/80 at 32k tokens is 400): the
// WHOLE unit-centroid table of the head-problem stays in LDS for the life of the
// workgroup (one workgroup of eight wavefronts per CU, two per SIMD), so the tile loop
// has no barriers, and every wavefront walks through several blocks of 64 keys with the
// NEXT block's loads in flight while the current block is contracted against all tiles:
// the key stream (the only HBM traffic that matters) runs under the matrix work instead
// of before it.
// The loop is software-pipelined by hand inside each wavefront: the 8 MFMAs of one key
// block (a dependent chain on one accumulator: chains cost nothing) are issued with the
// read-out (packed running maximum) of the OTHER key block's accumulator cut into 8
// slices between them, about 3.5 vector instructions per MFMA, which is what issues for
// free while an MFMA executes; an A fragment is replaced by the next tile's as soon as
// its last MFMA has been issued.  Two such wavefronts per SIMD cover each other's
// remaining stalls.  Measured on a stand-alone replica of this loop (no memory traffic):
// 76 % of the 2.5 PFLOP/s peak on all-zero operands at a 2.05 GHz shader clock, 54 % on
// random operands, where the chip drops to 1.4 GHz under the load -- 93 % of what that
// clock allows.  The loop is bound by the clock the chip holds, not by its schedule.
// Eight consecutive tasks of 64 tokens are one 512-token chunk of the counting sort.
constexpr int ST_WAVES = 8;
constexpr int ST_NKB = 2;                               // 64 keys per wavefront and block
constexpr int ST_CHUNK = ST_WAVES * ST_NKB * 32;        // 512 tokens per block of a workgroup
constexpr int ST_MAX_TILES = 16;                        // 512 centroids
constexpr int ST_MAX_BLOCKS = 8;
constexpr int ST_EARLY_TILES = 4;                       // up to this size the keys are requested with the table

template <bool HAS_BIAS, bool EARLY, bool LOOK>
__global__ __launch_bounds__(ST_WAVES * 64, 2) void k_assign_stream(
    const bf16* __restrict__ K, const bf16* __restrict__ mu_hat, int32_t* __restrict__ labels,
    float* __restrict__ best_sim, const ChunkIndex chunks, int n_chunks, int label_bits,
    int64_t N_cap, int64_t tok_begin, int64_t tok_count, int c_begin, int c_count, int blocks,
    const KmCtl ctl, const TileMap map) {
  constexpr int NKB = ST_NKB, THREADS = ST_WAVES * 64;
  __shared__ __attribute__((aligned(16))) bf16 table[ST_MAX_TILES * 32 * LDS_ROW];
  __shared__ __attribute__((aligned(16))) float lds_bias[HAS_BIAS ? (ST_MAX_TILES + 1) * 32 : 4];
  __shared__ uint32_t tok[ST_MAX_BLOCKS * ST_CHUNK];     // pack_token words of this workgroup's tokens, or
                                                         // [chunk][cluster] counts (clusters <= ST_CHUNK)
  __shared__ int s_changed, s_next_task;

  // one argument per 64-byte line of the argument block: a line that is fetched where it is first
  // used queues behind the key loads
  CK_FETCH_ARG(labels);
  CK_FETCH_ARG(tok_count);
  CK_FETCH_ARG(ctl.first);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  int wg, hp;
  if (!map.mine<true, LOOK>(wg, hp)) return;
  const bf16* Khp = K + (int64_t)hp * N_cap * D;
  const bf16* Mhp = mu_hat + (int64_t)hp * c_count * D;
  int32_t* lab = labels + (int64_t)hp * N_cap + tok_begin;
  const int n_tiles = (c_count + 31) / 32;
  const int64_t wg_tok0 = (int64_t)wg * blocks * ST_CHUNK;

  // keys of task b (64 consecutive tokens of this workgroup's range), in B-operand layout
  const char* Kwg = reinterpret_cast<const char*>(Khp + (tok_begin + wg_tok0) * D);
  const int wg_count = (int)min(tok_count - wg_tok0, (int64_t)ST_MAX_BLOCKS * ST_CHUNK);
  auto load_keys = [&](int b, bf16x8 (&bk)[NKB][8]) {
    uint32_t row[NKB];
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      const int t = min(b * (NKB * 32) + kb * 32 + col, wg_count - 1);   // clamp: result is discarded
      row[kb] = (uint32_t)t * (D * 2) + half * 16;
    }
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
      for (int kk = 0; kk < 8; ++kk)
        bk[kb][kk] = *reinterpret_cast<const bf16x8*>(Kwg + row[kb] + kk * 32);
  };
  bf16x8 ka[NKB][8], kb2[NKB][8];

  // ---- the table into LDS (rows beyond c_count are zero), bias, token words ----
  {
    const int n_seg = n_tiles * 32 * 16;                // 16-byte segments
    constexpr int PER = ST_MAX_TILES * 32 * 16 / THREADS;   // 16 per thread, all in flight at once
    uint4 stage[PER];
    // every load is unconditional (rows beyond the table re-read its last row and are
    // replaced by zeros when they are written to LDS): a load under a branch makes the
    // compiler wait for it before it issues the next one
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int seg = tid + i * THREADS;
      int r = seg >> 4;
      r = r < c_count ? r : c_count - 1;
      stage[i] = *reinterpret_cast<const uint4*>(Mhp + (int64_t)r * D + (seg & 15) * 8);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int seg = tid + i * THREADS;
      const bool real = (seg >> 4) < c_count;
      uint4 v = stage[i];
      v.x = real ? v.x : 0u; v.y = real ? v.y : 0u; v.z = real ? v.z : 0u; v.w = real ? v.w : 0u;
      if (seg < n_seg)
        *reinterpret_cast<uint4*>(&table[(seg >> 4) * LDS_ROW + (seg & 15) * 8]) = v;
    }
  }
  if (map.stopped<LOOK>(hp)) return;                          // the word has travelled with the table
  // EARLY: a small table is staged before the key requests pile up.  Otherwise they come behind
  // the barrier: a compute unit has about 32 KB of loads in flight, and a wavefront whose request
  // does not fit stands still, in front of the barrier with all others (8 x 32768 x 400: barrier
  // passed after 6.0 us, now 3.1).  Ten iterations, early / behind: 64 x 8179 x 102 517 / 522 us, 128 x 4000 x 100
  // 600 / 606, 64 x 8179 x 128 532 / 537, x 160 576 / 577, 8 x 16384 x 200 198 / 195, 8 x 32768 x 400 434 / 430.
  if constexpr (EARLY) load_keys(wave, ka);
  if constexpr (HAS_BIAS) {
    for (int c = tid; c < n_tiles * 32; c += THREADS)
      lds_bias[c] = c < c_count ? ctl.bias[(int64_t)hp * ctl.bias_stride + c] : 0.f;
  }
  if (chunks.seg)
    for (int t = tid; t < blocks * ST_CHUNK; t += THREADS) tok[t] = 0;
  if (tid == 0) {
    s_changed = 0;
    s_next_task = ST_WAVES;                             // tasks 0..7 are the wavefronts' first ones
  }
  __syncthreads();
  if constexpr (!EARLY) load_keys(wave, ka);

  const int n_tasks = blocks * ST_WAVES;
  bool moved = false;
  const bf16* arow0 = table + col * LDS_ROW + half * 8; // this lane's A fragments of tile 0

  // One task, 64 keys against every centroid tile, then its labels.
  auto process = [&](int b, const bf16x8 (&bk)[NKB][8], int nxt, bf16x8 (&nk)[NKB][8]) {
    const int64_t wave_tok0 = wg_tok0 + (int64_t)b * (NKB * 32);
    if (wave_tok0 >= tok_count) return;                 // wave-uniform: nothing of this block exists
    float bestp[NKB];
    int btile[NKB];
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      bestp[kb] = -INFINITY;
      btile[kb] = 0;
    }
    floatx16 acc[NKB];
    bf16x8 a[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) a[kk] = *reinterpret_cast<const bf16x8*>(arow0 + kk * 16);

    // l2: what is added to accumulators 4 j .. 4 j + 3 of a tile, read once for both key blocks (two
    // words for every slice of a read-out, each waited for where it was added: 37.8 us a launch at
    // 8 x 32768 x 400, now 33.8, 45.6 -> 41.2 at 32 x 17623 x 220).  The registers for it come from
    // key addresses of 32 bits behind one base: with ten of them spilled it was half the gain.
    float bias[HAS_BIAS ? 16 : 1];
    auto load_bias = [&](int tile_id, int j) {
      const floatx4 v = *reinterpret_cast<const floatx4*>(&lds_bias[tile_id * 32 + 8 * j + 4 * half]);
#pragma unroll
      for (int e = 0; e < 4; ++e) bias[HAS_BIAS ? 4 * j + e : 0] = v[e];
    };
    if constexpr (HAS_BIAS) {
#pragma unroll
      for (int j = 0; j < 4; ++j) load_bias(0, j);
    }
    // Slice r (0..7) of the read-out of one accumulator: two of its 16 similarities
    // join the packed running maximum; the last slice settles tile and value.
    // accumulator i of a lane is centroid row 8*(i/4) + 4*half + i%4 of the tile
    float mrun = 0.f;
    auto readout = [&](int kb, int tile_id, int r, bool last_tile) {
      float v0 = acc[kb][2 * r], v1 = acc[kb][2 * r + 1];
      const int row = tile_id * 32 + 8 * (r >> 1) + 4 * half + 2 * (r & 1);
      if constexpr (HAS_BIAS) {
        v0 += bias[2 * r];
        v1 += bias[2 * r + 1];
        // behind the second key block of this tile: those of the next one, four accumulators at a time
        if (kb == NKB - 1 && (r & 1)) load_bias(tile_id + 1, r >> 1);
      }
      if (last_tile) {                                  // zero-padded rows lose (finite: no NaN)
        v0 = row >= c_count ? -3.0e38f : v0;
        v1 = row + 1 >= c_count ? -3.0e38f : v1;
      }
      const float p0 = __uint_as_float((__float_as_uint(v0) & 0xFFFFFFF0u) | (uint32_t)(15 - 2 * r));
      const float p1 = __uint_as_float((__float_as_uint(v1) & 0xFFFFFFF0u) | (uint32_t)(14 - 2 * r));
      if (r == 0) mrun = bestp[kb];
      mrun = fmaxf(fmaxf(mrun, p0), p1);
      if (r == 7) {
        const bool up = __uint_as_float(__float_as_uint(mrun) & 0xFFFFFFF0u) >
                        __uint_as_float(__float_as_uint(bestp[kb]) & 0xFFFFFFF0u);
        btile[kb] = up ? tile_id : btile[kb];
        bestp[kb] = up ? mrun : bestp[kb];
      }
    };
    // The 8 MFMAs of key block KB against the tile whose A fragments are in a[], with the
    // read-out of the other key block's accumulator (tile `ro_tile`) between them.  While
    // key block 1 runs, every A fragment is replaced by the next tile's.
    auto step = [&](auto KBT, auto READOUT, int ro_tile, bool ro_last, const bf16* next_arow) {
      constexpr int kb = decltype(KBT)::value;
      constexpr bool RO = decltype(READOUT)::value;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        if (kk == 0) {
          floatx16 z;
#pragma unroll
          for (int i = 0; i < 16; ++i) z[i] = 0.f;
          acc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], bk[kb][kk], z, 0, 0, 0);
        } else {
          acc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], bk[kb][kk], acc[kb], 0, 0, 0);
        }
        if (RO) readout(1 - kb, ro_tile, kk, ro_last);
        if (kb == 1 && next_arow) a[kk] = *reinterpret_cast<const bf16x8*>(next_arow + kk * 16);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    using T0 = std::integral_constant<int, 0>;
    using T1 = std::integral_constant<int, 1>;
    using Yes = std::true_type;
    using No = std::false_type;
    const int last = n_tiles - 1;
    step(T0(), No(), 0, false, nullptr);                // tile 0, key block 0: nothing to read out yet
    // label of token `lane` before, in front of the next keys: behind them it would wait for them
    int before = 0;
    if (ctl.changed) before = lab[min((uint32_t)wave_tok0 + lane, (uint32_t)tok_count - 1)];
    // not before the matrix work has begun: the wavefront stands still until its requests fit
    if (nxt < n_tasks) load_keys(nxt, nk);
    for (int tile = 0; tile < last; ++tile) {
      step(T1(), Yes(), tile, false, arow0 + (tile + 1) * 32 * LDS_ROW);   // reads out block 0 of `tile`
      step(T0(), Yes(), tile, false, nullptr);          // block 0 of tile + 1; reads out block 1 of `tile`
    }
    step(T1(), Yes(), last, true, nullptr);             // last tile, key block 1; reads out its block 0
#pragma unroll
    for (int r = 0; r < 8; ++r) readout(1, last, r, true);

    // lanes l and l+32 hold the two halves of each key's candidates
    int lane_label = 0;                                 // label of token `lane` of the 64
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      const int slot = 15 - (int)(__float_as_uint(bestp[kb]) & 15u);
      float best = bestp[kb];
      int bidx = btile[kb] * 32 + 8 * (slot >> 2) + 4 * half + (slot & 3);
      const float ob = __shfl_xor(best, 32, WAVE);
      const int oi = __shfl_xor(bidx, 32, WAVE);
      const float bt = __uint_as_float(__float_as_uint(best) & 0xFFFFFFF0u);
      const float ot = __uint_as_float(__float_as_uint(ob) & 0xFFFFFFF0u);
      if (ot > bt || (ot == bt && oi < bidx)) {
        best = ob;
        bidx = oi;
      }
      // a key with a NaN or infinite channel may have no similarity that is a number: a padded
      // row has won then, and the key goes to the last cluster
      bidx = bidx < c_count ? bidx : c_count - 1;
      if (half == kb) lane_label = bidx;
      const int64_t t = wave_tok0 + kb * 32 + col;
      if (best_sim && half == 0 && t < tok_count)
        best_sim[(int64_t)hp * N_cap + tok_begin + t] = __uint_as_float(__float_as_uint(best) & 0xFFFFFFF0u);
    }
    const uint32_t t = (uint32_t)wave_tok0 + lane;      // a range has less than 2^31 tokens
    if (t < (uint32_t)tok_count) {
      moved |= ctl.first || before != c_begin + lane_label;
      lab[t] = c_begin + lane_label;
    }
    // the ranking inside the group runs here, under the other wavefront's matrix work
    if (chunks.list)
      tok[b * (NKB * 32) + lane] = pack_token(lane_label, wave_tok0 + lane < tok_count, label_bits);
    else if (chunks.seg && wave_tok0 + lane < tok_count)   // counts only
      atomicAdd(&tok[(b / ST_WAVES) * c_count + lane_label], 1u);
  };
  static_assert(NKB == 2, "a task is one group of 64 tokens");
  static_assert(ST_MAX_TILES * 32 <= ST_CHUNK, "counts take the place of the token words");

  // A workgroup's range is cut into tasks of 64 tokens (8 per 512-token chunk).  Every
  // wavefront starts with the task of its own number and then takes the next free one
  // from a shared counter, always one task ahead so that the keys can be requested a
  // whole task early.  Two wavefronts share a SIMD and the hardware does not split it
  // evenly between them; with a fixed share the slower one would finish alone, at the
  // speed of one wavefront.
  auto grab = [&]() {
    int t = 0;
    if (lane == 0) t = atomicAdd(&s_next_task, 1);
    return __builtin_amdgcn_readfirstlane(t);
  };
  int cur = wave;
  while (cur < n_tasks) {
    int nxt = grab();
    process(cur, ka, nxt, kb2);
    cur = nxt;
    if (cur >= n_tasks) break;
    nxt = grab();
    process(cur, kb2, nxt, ka);
    cur = nxt;
  }

  if (ctl.changed && __ballot(moved) && lane == 0) s_changed = 1;
  if (chunks.seg || ctl.changed) __syncthreads();
  if (ctl.changed && tid == 0 && s_changed) ctl.changed[hp] = 1;
  if (chunks.seg && !chunks.list) {
    for (int e = tid; e < blocks * c_count; e += THREADS) {
      const int64_t ch = (int64_t)wg * blocks + e / c_count;
      if (ch < n_chunks)
        chunks.seg[((int64_t)hp * n_chunks + ch) * seg_stride(c_count) + e % c_count] = tok[e] << 16;
    }
  } else if (chunks.seg) {
    // as many wavefronts per 512-token chunk as there are; the centroid table's LDS is free by now
    auto sort = [&](auto WT) {
      constexpr int W = decltype(WT)::value, CNT = chunk_sort_cnt_ints(ST_MAX_TILES * 32) * W;
      constexpr int SCRATCH = (CNT + 8) * 4 + ST_CHUNK * 2;
      static_assert(ST_WAVES / W * SCRATCH <= sizeof(table), "chunk sort scratch");
      const int k = wave / W;
      const int64_t ch = (int64_t)wg * blocks + k, o = (int64_t)hp * n_chunks + ch;
      int* cnt = reinterpret_cast<int*>(reinterpret_cast<char*>(table) + k * SCRATCH);
      chunk_sort<ST_CHUNK / WAVE, ST_MAX_TILES * 32, W>(
          tok + k * ST_CHUNK, c_count, wave % W, k < blocks && ch < n_chunks, cnt, cnt + CNT,
          reinterpret_cast<uint16_t*>(cnt + CNT + 8), chunks.seg + o * seg_stride(c_count),
          chunks.list + o * ST_CHUNK);
    };
    if (blocks == 1) sort(std::integral_constant<int, 8>());
    else if (blocks == 2) sort(std::integral_constant<int, 4>());
    else if (blocks <= 4) sort(std::integral_constant<int, 2>());
    else sort(std::integral_constant<int, 1>());
  }
}

bool assign_stream_fits(int c_count) { return c_count <= ST_MAX_TILES * 32; }

hipError_t launch_assign_stream(const Dims& dm, const bf16* K, int64_t tok_begin,
                                int64_t tok_count, const bf16* mu_hat, int c_begin, int c_count,
                                int32_t* labels, float* best_sim, const ChunkIndex& chunks,
                                const KmCtl& ctl, int n_cu, hipStream_t st) {
  // Blocks of 512 tokens per workgroup (at most 8: the chunk index is sorted by one wavefront a block
  // at least): the number with the least rounds of workgroups (one per CU) times blocks and start-up
  // of a round, which takes about as long as a block (C = 102: 6 us and 5.2, C = 400: 8 and 9.4).
  // Filling the CUs once with floor(chunks / CUs) blocks instead, a few workgroups more than CUs are a
  // second round: 8 x 40000 x 416 764 us for ten iterations, now 545; 64 x 20000 x 250 1851, now 1632;
  // 20 x 65536 x 100 1446 / 1352, 24 x 65536 x 400 2415 / 2373.  Where the keys are more than the
  // Infinity Cache and the products few, the rounds overlap better than that: 24 x 65536 x 100 is 1.3 %
  // slower than with floor (1660 / 1681), x 129 2.3 % (1707 / 1747).
  const int64_t chunks_hp = (tok_count + ST_CHUNK - 1) / ST_CHUNK;
  int64_t blocks = 1, least = INT64_MAX;
  for (int64_t b = 1; b <= ST_MAX_BLOCKS && b <= chunks_hp; ++b) {
    const int64_t wgs = (chunks_hp + b - 1) / b * dm.HP, cost = (wgs + n_cu - 1) / n_cu * (b + 1);
    if (cost < least) {
      least = cost;
      blocks = b;
    }
  }
  const TileMap map((chunks_hp + blocks - 1) / blocks, dm.HP, ctl.running);
  int label_bits = 0;
  while ((1 << label_bits) < c_count) ++label_bits;
  auto launch = [&](auto look) {
    constexpr bool L = decltype(look)::value;
    const auto kernel = c_count <= ST_EARLY_TILES * 32
                            ? (ctl.bias ? k_assign_stream<true, true, L> : k_assign_stream<false, true, L>)
                            : (ctl.bias ? k_assign_stream<true, false, L> : k_assign_stream<false, false, L>);
    hipLaunchKernelGGL(kernel, map.grid(), dim3(ST_WAVES * 64), 0, st, K, mu_hat, labels, best_sim, chunks,
                       (int)chunks_hp, label_bits, dm.N_cap, tok_begin, tok_count, c_begin, c_count,
                       (int)blocks, ctl, map);
  };
  ctl.running.first ? launch(std::true_type()) : launch(std::false_type());
  return hipGetLastError();
}

}  // namespace ck
