// K-means assignment step (paper Section III-B) for tables that do not stay in LDS as a whole:
// see k_assign in kmeans_assign.hip for the mapping onto v_mfma_f32_32x32x16_bf16 and the packed
// running maximum.  Compiled with the MFMA results kept in vector registers.
#include <type_traits>

#include "chunk_sort.hpp"
#include "key_operand.hpp"

namespace ck {

constexpr int WD_WAVES = 4;
constexpr int WD_NKB = 4;                               // 128 keys per wavefront, in registers
constexpr int WD_CHUNK = WD_WAVES * WD_NKB * 32;        // 512 tokens per workgroup, one chunk of the sort
constexpr int WD_AHEAD = 3;                             // a tile is staged this many tiles ahead
constexpr int WD_SLOTS = 2 * WD_AHEAD;                  // centroid tiles of 32 rows in LDS
constexpr int WD_LDS_ROW = D + 8;                       // 272 B: rows shift 4 banks

// One workgroup of four wavefronts takes 512 tokens, 128 keys of each wavefront in registers, and
// walks through all centroid tiles; two workgroups share a CU, and as the hardware prefers the
// older one they drift apart, so that one's start and epilogue run under the other's matrix work.
// The tiles go through a ring of six in LDS, three tiles ahead, with a barrier every third tile.
// As in k_assign_stream the 8 MFMAs of a key block (32 keys) are issued with the read-out of the
// block before cut into slices between them; the loads and stores of the staging are such slices
// too (issued between two blocks they left the matrix pipe idle: 104 000 cycles for the loop at
// C = 2000 with one wavefront per SIMD, 89 000 in slices, 64 500 of matrix work).
// Bound: the clock.  The matrix pipe is busy 80 % of the kernel's cycles (8 x 131072 x 1600, counters),
// and the chip lowers its clock to 1.6-1.7 GHz for it (2.2 GHz on constant keys).
// It takes the place of a kernel with eight wavefronts, a barrier every second tile and the
// read-out behind the MFMAs, which ran at 2.05 GHz with the pipe 54 % busy.  Ten iterations, whole
// call: 8 x 131072 x 1600 4048 us, now 3750; 4 x 100000 x 1250 1550 / 1445; 16 x 65536 x 800
// 2390 / 2225; 8 x 60000 x 750 1170 / 1095; 8 x 9000 x 600 517 / 360 (the grid of 512 tokens per
// workgroup wastes less of the last round); with at most 512 clusters it is within 3 % of
// k_assign_stream at large tables and up to 15 % slower at small ones, where the keys count.
template <bool HAS_BIAS, bool LOOK>
__global__ __launch_bounds__(WD_WAVES * 64, 2) void k_assign_wide(
    const bf16* __restrict__ K, const bf16* __restrict__ mu_hat, int32_t* __restrict__ labels,
    float* __restrict__ best_sim, const ChunkIndex chunks, int n_chunks, int label_bits,
    int64_t N_cap, int64_t tok_begin, int64_t tok_count, int c_begin, int c_count,
    const KmCtl ctl, const TileMap map) {
  constexpr int NKB = WD_NKB, THREADS = WD_WAVES * 64, PER = 32 * 16 / THREADS;
  __shared__ __attribute__((aligned(16))) bf16 ring[WD_SLOTS * 32 * WD_LDS_ROW];
  __shared__ __attribute__((aligned(16))) float lds_bias[HAS_BIAS ? CK_MAX_CLUSTERS + 64 : 4];
  __shared__ __attribute__((aligned(16))) bf16 key_stage[WD_WAVES * KEY_STAGE_ELEMS];
  __shared__ int s_changed;

  // one argument per 64-byte line of the argument block: fetched where it is first used, a line would
  // queue behind the key loads
  CK_FETCH_ARG(labels);
  CK_FETCH_ARG(tok_count);
  CK_FETCH_ARG(ctl.first);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, half = lane >> 5;
  int wg, hp;
  if (!map.mine<true, LOOK>(wg, hp) || map.stopped<LOOK>(hp)) return;
  const bf16* Mhp = mu_hat + (int64_t)hp * c_count * D;
  const int n_tiles = (c_count + 31) / 32;

  // ---- centroid tiles, 16 lanes a row ----
  // A row beyond the table is its last row again: the read-out of the last tile leaves it out.
  const int srow = tid >> 4, sseg = tid & 15;
  auto stage_load = [&](int tile, int i) {
    const int r = min(tile * 32 + srow + i * (THREADS / 16), c_count - 1);
    return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(Mhp) +
                                           (uint32_t)(r * (D * 2) + sseg * 16));
  };
  auto stage_store = [&](int slot, int i, uint4 v) {
    *reinterpret_cast<uint4*>(&ring[(slot * 32 + srow + i * (THREADS / 16)) * WD_LDS_ROW + sseg * 8]) = v;
  };

  const int64_t wave_tok0 = ((int64_t)wg * WD_WAVES + wave) * (NKB * 32);
  {
    uint4 first[WD_AHEAD][PER];
#pragma unroll
    for (int t = 0; t < WD_AHEAD; ++t)
#pragma unroll
      for (int i = 0; i < PER; ++i) first[t][i] = stage_load(t, i);
#pragma unroll
    for (int t = 0; t < WD_AHEAD; ++t)
#pragma unroll
      for (int i = 0; i < PER; ++i) stage_store(t, i, first[t][i]);
  }
  if (tid == 0) s_changed = 0;
  if constexpr (HAS_BIAS) {
    for (int c = tid; c < n_tiles * 32; c += THREADS)
      lds_bias[c] = c < c_count ? ctl.bias[(int64_t)hp * ctl.bias_stride + c] : 0.f;
  }
  __syncthreads();
  KeyTile<NKB> keys;
  keys.load(K + ((int64_t)hp * N_cap + tok_begin) * D, wave_tok0, tok_count, lane);
  keys.to_operand(key_stage + wave * KEY_STAGE_ELEMS, lane);

  float bestp[NKB];
  int btile[NKB];
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb) {
    bestp[kb] = -INFINITY;
    btile[kb] = 0;
  }
  floatx16 acc[2];                                      // of the key block in work and the one before
  bf16x8 a[8];
  const bf16* arow = ring + col * WD_LDS_ROW + half * 8;   // this lane's fragments in slot 0
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) a[kk] = *reinterpret_cast<const bf16x8*>(arow + kk * 16);

  // l2: what is added to accumulators 4 j .. 4 j + 3 of a tile, read once for all key blocks (two words
  // for every slice of a read-out, each waited for where it was added: 147 us a launch at
  // 16 x 50000 x 600, now 121, and 392 -> 347 at 8 x 131072 x 1600; without a bias 111 and 317)
  float bias[HAS_BIAS ? 16 : 1];
  auto load_bias = [&](int tile_id, int j) {
    const floatx4 b = *reinterpret_cast<const floatx4*>(&lds_bias[tile_id * 32 + 8 * j + 4 * half]);
#pragma unroll
    for (int e = 0; e < 4; ++e) bias[HAS_BIAS ? 4 * j + e : 0] = b[e];
  };
  if constexpr (HAS_BIAS) {
#pragma unroll
    for (int j = 0; j < 4; ++j) load_bias(0, j);
  }
  // Slice r (0..7) of the read-out of key block kb: two of its 16 similarities join the packed
  // running maximum; the last slice settles tile and value.
  // accumulator i of a lane is centroid row 8*(i/4) + 4*half + i%4 of the tile
  float mrun = 0.f;
  auto readout = [&](int kb, int tile_id, int r, bool last_tile) {
    float v0 = acc[kb & 1][2 * r], v1 = acc[kb & 1][2 * r + 1];
    const int row = tile_id * 32 + 8 * (r >> 1) + 4 * half + 2 * (r & 1);
    if constexpr (HAS_BIAS) {
      v0 += bias[2 * r];
      v1 += bias[2 * r + 1];
      // behind the last key block of this tile: those of the next one, four accumulators at a time
      if (kb == NKB - 1 && (r & 1)) load_bias(tile_id + 1, r >> 1);
    }
    if (last_tile) {                                    // zero-padded rows lose (finite: no NaN)
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
      // stays where it is: the compiler would collect the read-outs of all key blocks behind the
      // next branch and keep four accumulators for it
      asm volatile("" : "+v"(bestp[kb]), "+v"(btile[kb]));
    }
  };
  // The 8 MFMAs of a key block, with the read-out of the block before and what else there is to
  // issue cut into slices between them.
  auto step = [&](auto KBT, auto READOUT, int ro_tile, bool ro_last, auto slice) {
    constexpr int kb = decltype(KBT)::value;
    constexpr bool RO = decltype(READOUT)::value;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      if (kk == 0) {
        floatx16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
        acc[kb & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], keys.operand(kb, kk), z, 0, 0, 0);
      } else {
        acc[kb & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], keys.operand(kb, kk), acc[kb & 1], 0, 0, 0);
      }
      if (RO) readout((kb + 3) & 3, ro_tile, kk, ro_last);
      slice(kk);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using T0 = std::integral_constant<int, 0>;
  using T1 = std::integral_constant<int, 1>;
  using T2 = std::integral_constant<int, 2>;
  using T3 = std::integral_constant<int, 3>;
  using Yes = std::true_type;
  using No = std::false_type;
  const int last = n_tiles - 1;
  auto none = [](int) {};
  step(T0(), No(), 0, false, none);
  int rd = 1, wr = WD_AHEAD, turn = 0;                  // slots of tile + 1 and tile + WD_AHEAD
  uint4 v[PER];                                         // of tile + WD_AHEAD, on their way for one tile
#pragma unroll
  for (int i = 0; i < PER; ++i) v[i] = stage_load(WD_AHEAD, i);
  for (int tile = 0; tile < last; ++tile) {
    step(T1(), Yes(), tile, false, none);
    step(T2(), Yes(), tile, false, [&](int kk) {
      if (kk < PER) stage_store(wr, kk, v[kk]);
      if (kk >= 4 && kk < 4 + PER) v[kk - 4] = stage_load(tile + WD_AHEAD + 1, kk - 4);
    });
    // Every WD_AHEAD tiles: what has been staged since the last barrier may be read behind this one,
    // and the slots of the tiles before may be staged over.
    if (++turn == WD_AHEAD) {
      turn = 0;
      __syncthreads();
    }
    const bf16* next = arow + rd * 32 * WD_LDS_ROW;
    step(T3(), Yes(), tile, false, [&](int kk) { a[kk] = *reinterpret_cast<const bf16x8*>(next + kk * 16); });
    step(T0(), Yes(), tile, false, none);               // of tile + 1
    rd = rd + 1 == WD_SLOTS ? 0 : rd + 1;
    wr = wr + 1 == WD_SLOTS ? 0 : wr + 1;
  }
  step(T1(), Yes(), last, true, none);
  step(T2(), Yes(), last, true, none);
  step(T3(), Yes(), last, true, none);
#pragma unroll
  for (int r = 0; r < 8; ++r) readout(3, last, r, true);
  __syncthreads();                                      // the ring is free

  // ---- lanes l and l+32 hold the two halves of each key's candidates ----
  uint32_t* tok = reinterpret_cast<uint32_t*>(ring);    // pack_token words, or the counts by cluster
  const bool count_only = chunks.seg && !chunks.list;
  if (count_only) {
    static_assert(CK_MAX_CLUSTERS * 4 <= sizeof(ring), "counts");
    for (int c = tid; c < c_count; c += THREADS) tok[c] = 0;
    __syncthreads();
  }
  int lane_label[NKB / 2];                              // labels of tokens 64 i + lane of this wavefront
  bool moved = false;
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb) {
    const int slot = 15 - (int)(__float_as_uint(bestp[kb]) & 15u);
    float best = bestp[kb];
    int bidx = btile[kb] * 32 + 8 * (slot >> 2) + 4 * half + (slot & 3);
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
    if (half == (kb & 1)) lane_label[kb / 2] = bidx;
    const int64_t t = wave_tok0 + kb * 32 + col;
    if (half == 0 && t < tok_count) {
      const int64_t o = (int64_t)hp * N_cap + tok_begin + t;
      if (ctl.changed) moved |= ctl.first || labels[o] != c_begin + bidx;
      labels[o] = c_begin + bidx;
      if (best_sim) best_sim[o] = __uint_as_float(__float_as_uint(best) & 0xFFFFFFF0u);
      if (count_only) atomicAdd(&tok[bidx], 1u);
    }
  }
  if (ctl.changed && __ballot(moved) && lane == 0) s_changed = 1;
  if (chunks.list) {
#pragma unroll
    for (int i = 0; i < NKB / 2; ++i)
      tok[(wave * (NKB / 2) + i) * WAVE + lane] =
          pack_token(lane_label[i], wave_tok0 + i * WAVE + lane < tok_count, label_bits);
  }
  if (chunks.seg || ctl.changed) __syncthreads();
  if (ctl.changed && tid == 0 && s_changed) ctl.changed[hp] = 1;
  const int64_t o = (int64_t)hp * n_chunks + wg;
  if (count_only) {
    for (int c = tid; c < c_count; c += THREADS) chunks.seg[o * seg_stride(c_count) + c] = tok[c] << 16;
  } else if (chunks.seg) {
    constexpr int CNT = chunk_sort_cnt_ints(CK_MAX_CLUSTERS) * WD_WAVES;
    static_assert((WD_CHUNK + CNT + WD_WAVES) * 4 + WD_CHUNK * 2 <= sizeof(ring), "chunk sort scratch");
    int* cnt = reinterpret_cast<int*>(ring) + WD_CHUNK;
    chunk_sort<WD_CHUNK / WAVE, CK_MAX_CLUSTERS, WD_WAVES>(
        tok, c_count, wave, true, cnt, cnt + CNT, reinterpret_cast<uint16_t*>(cnt + CNT + WD_WAVES),
        chunks.seg + o * seg_stride(c_count), chunks.list + o * WD_CHUNK);
  }
}

hipError_t launch_assign_wide(const Dims& dm, const bf16* K, int64_t tok_begin, int64_t tok_count,
                              const bf16* mu_hat, int c_begin, int c_count, int32_t* labels,
                              float* best_sim, const ChunkIndex& chunks, const KmCtl& ctl,
                              hipStream_t st) {
  const int n_chunks = (int)((tok_count + WD_CHUNK - 1) / WD_CHUNK);
  int label_bits = 0;
  while ((1 << label_bits) < c_count) ++label_bits;
  const TileMap map(n_chunks, dm.HP, ctl.running);
  auto launch = [&](auto look) {
    constexpr bool L = decltype(look)::value;
    hipLaunchKernelGGL((ctl.bias ? k_assign_wide<true, L> : k_assign_wide<false, L>), map.grid(), dim3(WD_WAVES * 64),
                       0, st, K, mu_hat, labels, best_sim, chunks, n_chunks, label_bits, dm.N_cap, tok_begin,
                       tok_count, c_begin, c_count, ctl, map);
  };
  ctl.running.first ? launch(std::true_type()) : launch(std::false_type());
  return hipGetLastError();
}

}  // namespace ck
