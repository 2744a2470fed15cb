// Whole K-means of a small token range in ONE kernel (paper Section III-B, decode
// stage: every m generated tokens are clustered among themselves into a handful of
// new clusters).  At m = 320 tokens and 4 clusters an iteration is ~0.3 MFLOP per
// head-problem, so the prefill path with its two launches per iteration would spend
// its time on them; here one workgroup per head-problem keeps the keys in registers and
// runs init, all iterations (assignment, update), the metadata and the stores itself.
// Same arithmetic rules as the large path: bf16-rounded table rows compared in fp32,
// ties to the lower id, fp32 sums in a fixed order, means of raw keys, an empty cluster
// keeps its centroid.
#include <type_traits>

#include "ck_common.hpp"

namespace ck {

// Up to here the products have sixteen columns per wavefront (of 1024 threads) instead of 32: a branch
// in the one kernel costs the large ranges registers (320 tokens 30.9 -> 31.8 us).
constexpr int KM_SMALL_FEW_TOKENS = 256;

struct SmallArgs {
  const bf16* K;
  const int32_t* init_idx;
  bf16* centroids;
  int32_t *labels, *sizes, *offsets, *sorted_idx, *iters_done;
  int64_t N_cap, tok_begin;
  int tok_count, C_cap, c_begin, c_count, max_iter, metric, converge;
};

// By how much two similarities of a key may differ from what another order of their additions gives:
// this factor, from the squared length of the key, times the length of the longest table row.  Every
// partial sum is at most |k| |row|, and 128 additions, be they rounded or cut off, are off by 2^-23
// of that each; the fixed order has a chain of twelve.  Lengths of 2^50 and more count as infinite (sums
// that overflow).  Lengths below 2^-60 count as 2^-60, and KM_SMALL_SLACK is added whatever the lengths:
// nothing is assumed of what the matrix cores make of a channel, a product or a sum below the smallest
// normal number.  Taken for zero, a channel loses 2^-126 times the other side's length, each of 128 products
// and as many sums 2^-126, in either similarity 2^-118 in all.
constexpr float KM_SMALL_SLACK = 0x1p-116f;
__device__ __forceinline__ float key_bound(float n2) {
  const float n = 1.001f * sqrtf(n2);
  return n < 0x1p50f ? 0x1.1p-15f * fmaxf(n, 0x1p-60f) : INFINITY;
}
__device__ __forceinline__ float row_bound(float n) {
  n *= 1.001f;
  return n < 0x1p49f ? fmaxf(n, 0x1p-60f) : INFINITY;
}

// MAXC: compile-time bound of the cluster count; SM_THREADS: workgroup size; MAXTOK: bound of the range.
//
// Bound: a chain of max_iter dependent iterations on one CU per head-problem, and in each the
// instructions of sixteen wavefronts on four SIMDs.
//   labels        v_mfma_f32_16x16x32_bf16, rows = the clusters (four, repeated, so that every lane has
//                 all similarities of its key and the best of them needs no lane exchange), columns =
//                 16 keys of the wavefront.  Where best and second are too close for the order of the
//                 additions not to matter, the fixed order decides (exact_label; 1 key in 5000 of a
//                 mixture), so the labels are those of the fixed order.
//   update sums   v_mfma_f32_4x4x1_16b_f32, one fp32 addition per element and step, in the order
//                 written here: block = four lanes of one key, rows = 4 clusters, A = 1 where the
//                 key's label is the row's cluster; 8 steps replace 32 multiply-adds.
// A wavefront keeps its keys in registers in both layouts for all iterations (no LDS pass over
// the keys).  The wavefront of a cluster adds up that cluster's partial sums, keeps its mean in
// registers and makes the next table row from it, so an iteration has two barriers.  A wavefront whose
// keys have all kept their labels leaves its sums of the iteration before standing.
// 128 head-problems x 320 tokens x 4 clusters, 10 iterations: 53.7 us with the dot products too as
// 4x4x1 steps (sixteen partial sums per key and cluster, added by lane swaps), 35.4 with the labels as
// above, 32.7 with the operands of a round's sums made before its first product, 30.3 with all columns'
// products issued together; same bits.  160 tokens 34.7 -> 20.1, 320 tokens x 8 clusters 90.9 -> 49.2,
// x 2 45.9 -> 27.0.
// MAXC = 2 is a form of its own: half the registers and lane exchanges of the sums.
template <int MAXC, int SM_THREADS, int MAXTOK>
__global__ __launch_bounds__(SM_THREADS) void k_kmeans_small(const SmallArgs a) {
  constexpr int WAVES = SM_THREADS / WAVE, SETS = (MAXC + 3) / 4, ROWS = 4 * SETS;
  constexpr int KEYS = WAVES * 4;                       // keys per round, four per wavefront
  constexpr int ROUNDS = (MAXTOK + KEYS - 1) / KEYS;
  constexpr int TILES = (ROUNDS + 3) / 4;               // sixteen keys of a wavefront, four rounds
  constexpr int WORDS = (ROUNDS + 7) / 8;               // of four bits per round
  constexpr int TROW = D + 32;                          // table row in LDS: 320 B, rows shift 16 banks
  static_assert((MAXC == 2 || MAXC % 4 == 0) && MAXC <= WAVES && MAXTOK <= SM_THREADS, "mapping");
  __shared__ __attribute__((aligned(16))) bf16 table[ROWS][TROW];
  __shared__ __attribute__((aligned(16))) float part[WAVES][MAXC][D];
  __shared__ int cnt[WAVES][MAXC];
  __shared__ int wave_cnt[WAVES][MAXC];
  __shared__ __attribute__((aligned(16))) float bias[ROWS];
  __shared__ float row_norm[ROWS];
  __shared__ int lab[MAXTOK];
  __shared__ int s_changed[2];

  const int hp = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, row = lane >> 4, l4 = lane & 3;
  const int n_tok = a.tok_count, C = a.c_count;
  const bf16* Khp = a.K + (int64_t)hp * a.N_cap * D;
  const uint4* R = reinterpret_cast<const uint4*>(Khp + a.tok_begin * D);

  // ---- this wavefront's keys: of round r, keys r * KEYS + 4 * wave + (0..3) ----
  // dk: the columns of the products; column n of tile T is key n % 4 of round 4 T + n / 4, and lane
  // 16 g + n holds channels 32 sl + 8 g .. + 8 of it.  uk: lanes 16 x + g hold channels 8 g .. + 8 of key x.
  uint4 dk[TILES][4], uk[ROUNDS];
  float thr[TILES];                                     // see exact_label
  {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {                  // a key beyond the range re-reads the last one
      const int tu = r * KEYS + wave * 4 + row;
      uk[r] = R[(int64_t)(tu < n_tok ? tu : n_tok - 1) * 16 + l16];
    }
#pragma unroll
    for (int T = 0; T < TILES; ++T) {
      const int td = (4 * T + (l16 >> 2)) * KEYS + wave * 4 + l4;
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) dk[T][sl] = R[(int64_t)(td < n_tok ? td : n_tok - 1) * 16 + 4 * sl + row];
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)                    // ... and adds nothing
      if (r * KEYS + wave * 4 + row >= n_tok) uk[r] = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int T = 0; T < TILES; ++T) {
      float n2 = 0.f;
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) {
        const uint32_t w[4] = {dk[T][sl].x, dk[T][sl].y, dk[T][sl].z, dk[T][sl].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) n2 = fmaf(lo_bf16(w[i]), lo_bf16(w[i]), fmaf(hi_bf16(w[i]), hi_bf16(w[i]), n2));
      }
      thr[T] = key_bound(xor32(xor16(n2, OpSum()), OpSum()));
    }
  }
  // the mean of cluster `wave`: channels 2 * lane, 2 * lane + 1
  float m0 = 0.f, m1 = 0.f;
  if (wave < C) {
    int64_t r = a.init_idx[(int64_t)hp * C + wave];
    r = r < 0 ? 0 : (r >= a.N_cap ? a.N_cap - 1 : r);
    const uint32_t w = reinterpret_cast<const uint32_t*>(Khp + r * D)[lane];
    m0 = lo_bf16(w);
    m1 = hi_bf16(w);
  }
  // rows without a cluster
  for (int e = tid; e < (ROWS - C) * (TROW / 2); e += SM_THREADS) reinterpret_cast<uint32_t*>(table[C])[e] = 0;
  if (tid >= C && tid < ROWS) bias[tid] = row_norm[tid] = 0.f;

  // The label of one token of the range in a fixed order of the additions: eight multiply-adds per
  // group of eight channels, the sixteen groups as row16_sum adds them.  The labels are those of this
  // order.  The matrix cores add the same exact products in another one; either is off by less than
  // 128 * 2^-23 |k| |row|, and where the best similarity is not ahead of the second by twice that
  // (thr, with the bound on the keys' side) the key is settled here.
  auto exact_label = [&](int t) {
    const uint4 k = R[(int64_t)t * 16 + l16];
    const uint32_t kw[4] = {k.x, k.y, k.z, k.w};
    float best = 0.f;
    int bc = 0;
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
      const uint4 x = *reinterpret_cast<const uint4*>(&table[4 * s + row][l16 * 8]);
      const uint32_t xw[4] = {x.x, x.y, x.z, x.w};
      float d = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        d = fmaf(lo_bf16(xw[i]), lo_bf16(kw[i]), d);
        d = fmaf(hi_bf16(xw[i]), hi_bf16(kw[i]), d);
      }
      float v = row16_sum(d) + bias[4 * s + row];
      // a NaN never wins over another cluster and is never beaten as cluster 0
      v = v == v && 4 * s + row < C ? v : (4 * s + row == 0 ? INFINITY : -INFINITY);
#pragma unroll
      for (int i = 0; i < 4; ++i) {                     // the lower cluster where they are equal
        const float vi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16 * i));
        if ((s == 0 && i == 0) || vi > best) {
          best = vi;
          bc = 4 * s + i;
        }
      }
    }
    return bc;
  };

  int label[TILES];                                     // of column l16, in every row of lanes
#pragma unroll
  for (int T = 0; T < TILES; ++T) label[T] = -1;

  int n_done = 0;
  for (int it = 0; it < a.max_iter; ++it) {
    // ---- table row (and l2 bias) of cluster `wave` ----
    if (wave < C) {
      uint32_t w;
      if (a.metric == CK_METRIC_COSINE) {
        // the fused product written out: the last bit of the norm must not depend on the
        // compiler's choice
        const float n2 = wave_sum(fmaf(m0, m0, m1 * m1));
        const float inv = n2 > 0.f ? 1.0f / sqrtf(n2) : 0.f;
        w = (uint32_t)float_to_bf16_bits(m0 * inv) | ((uint32_t)float_to_bf16_bits(m1 * inv) << 16);
      } else {
        w = (uint32_t)float_to_bf16_bits(m0) | ((uint32_t)float_to_bf16_bits(m1) << 16);
      }
      reinterpret_cast<uint32_t*>(table[wave])[lane] = w;
      if (a.metric != CK_METRIC_COSINE) {
        const float r0 = lo_bf16(w), r1 = hi_bf16(w);
        const float rn2 = wave_sum(fmaf(r0, r0, r1 * r1));
        if (lane == 0) {
          bias[wave] = a.metric == CK_METRIC_L2 ? -0.5f * rn2 : 0.f;
          row_norm[wave] = sqrtf(rn2);
        }
      } else if (lane == 0) {
        bias[wave] = 0.f;
      }
    }
    if (tid == 0) s_changed[it & 1] = 0;                // the other one may still be read
    __syncthreads();

    // ---- labels: rows of the products are the clusters 4 s + (0..3), four times over, so that every
    // lane ends with the similarities of key l16 to all of them ----
    bool moved = false;
    {
      bf16x8 ta[SETS][4];
      float4 bs[SETS];
#pragma unroll
      for (int s = 0; s < SETS; ++s) {
#pragma unroll
        for (int sl = 0; sl < 4; ++sl)
          ta[s][sl] = *reinterpret_cast<const bf16x8*>(&table[4 * s + l4][32 * sl + 8 * row]);
        bs[s] = *reinterpret_cast<const float4*>(&bias[4 * s]);
      }
      // length of the longest row (one, and a quarter more for means of 2^-71 to 2^-60, whose squares are
      // rounded below the smallest normal number; up to 8 for shorter ones, whose rows this does not cover:
      // a length kept per row costs 2 to 5 % of the call); rounding of the bias, and see KM_SMALL_SLACK
      float rn = 1.25f, slack = KM_SMALL_SLACK;
      if (a.metric != CK_METRIC_COSINE) {
        rn = row_norm[0];
#pragma unroll
        for (int c = 1; c < ROWS; ++c) rn = fmaxf(rn, row_norm[c]);
        rn = row_bound(rn);
        slack = fmaf(0x1p-20f * rn, rn, KM_SMALL_SLACK);
      }
      floatx4 d[TILES][SETS];
#pragma unroll
      for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int sl = 0; sl < 4; ++sl)
#pragma unroll
          for (int T = 0; T < TILES; ++T)
            d[T][s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ta[s][sl], __builtin_bit_cast(bf16x8, dk[T][sl]),
                                                              sl ? d[T][s] : floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      int bc[TILES];
      uint32_t open[TILES], any_open = 0;
#pragma unroll
      for (int T = 0; T < TILES; ++T) {
        float best = 0.f, second = -INFINITY;
        bc[T] = 0;
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
          const float b[4] = {bs[s].x, bs[s].y, bs[s].z, bs[s].w};
#pragma unroll
          for (int i = 0; i < (MAXC < 4 ? MAXC : 4); ++i) {
            const int c = 4 * s + i;
            const float v = c < C ? d[T][s][i] + b[i] : -INFINITY;
            if (c == 0) {
              best = v;
            } else {                                    // a NaN leaves no distance
              second = fmaxf(second, fminf(best, v));
              bc[T] = v > best ? c : bc[T];
              best = v > best ? v : best;
            }
          }
        }
        const int t = (4 * T + (l16 >> 2)) * KEYS + wave * 4 + l4;
        open[T] = (uint32_t)__ballot(t < n_tok && !(best - second > fmaf(thr[T], rn, slack))) & 0xFFFFu;
        any_open |= open[T];
      }
      if (any_open) {                                   // wave-uniform
#pragma unroll
        for (int T = 0; T < TILES; ++T)
          while (open[T]) {
            const int n = __builtin_ctz(open[T]);
            open[T] &= open[T] - 1;
            const int c = exact_label((4 * T + (n >> 2)) * KEYS + wave * 4 + (n & 3));
            bc[T] = l16 == n ? c : bc[T];
          }
      }
#pragma unroll
      for (int T = 0; T < TILES; ++T) {
        // a key that does not exist belongs to no cluster
        if ((4 * T + (l16 >> 2)) * KEYS + wave * 4 + l4 >= n_tok) bc[T] = 15;
        moved |= bc[T] != label[T];
        label[T] = bc[T];
      }
    }
    // ---- the sums over this wavefront's keys: where none of its labels has changed, those of the
    // iteration before stand in part and cnt ----
    const bool any_moved = __ballot(moved) != 0;
    if (any_moved && lane == 0) s_changed[it & 1] = 1;
    if (any_moved || it == 0) {
      floatx4 acc[SETS][8];                               // [channel 8 l16 + j][cluster 4 s + i], key group `row`
      uint32_t mine[SETS][WORDS];                         // bit 4 r: key `row` of round r (+ 8 per word) is in cluster 4 s + l4
#pragma unroll
      for (int s = 0; s < SETS; ++s) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[s][j] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < WORDS; ++w) mine[s][w] = 0;
        int members_n[4];
#pragma unroll
        for (int i = 0; i < (MAXC < 4 ? MAXC : 4); ++i) {
          uint32_t members[WORDS];
          int n = 0;
#pragma unroll
          for (int w = 0; w < WORDS; ++w) {
            members[w] = (uint32_t)__ballot(label[2 * w] == 4 * s + i) & 0xFFFFu;
            if (2 * w + 1 < TILES) members[w] |= (uint32_t)__ballot(label[2 * w + 1 < TILES ? 2 * w + 1 : 0] == 4 * s + i) << 16;
            n += __popc(members[w]);
            mine[s][w] = l4 == i ? members[w] : mine[s][w];
          }
          members_n[i] = n;
        }
        if (lane == 0) {
#pragma unroll
          for (int i = 0; i < (MAXC < 4 ? MAXC : 4); ++i) cnt[wave][4 * s + i] = members_n[i];
        }
#pragma unroll
        for (int w = 0; w < WORDS; ++w) mine[s][w] >>= row;
      }
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        // two clusters: wavefronts without keys in a round sit it out (with four, a round in full is the rule)
        if (r * KEYS + (MAXC == 2 ? wave * 4 : 0) < n_tok) {   // wave-uniform
          // unpacked here and not once before the iterations: there are no registers for that
          asm volatile("" : "+v"(uk[r].x), "+v"(uk[r].y), "+v"(uk[r].z), "+v"(uk[r].w));
          const uint32_t uw[4] = {uk[r].x, uk[r].y, uk[r].z, uk[r].w};
          float x[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) x[j] = j & 1 ? hi_bf16(uw[j / 2]) : lo_bf16(uw[j / 2]);
          // all eight at once: one by one each product waits for its operand
          asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]));
#pragma unroll
          for (int s = 0; s < SETS; ++s) {
            const float on = (float)((mine[s][r / 8] >> (r % 8 * 4)) & 1u);
#pragma unroll
            for (int j = 0; j < 8; ++j)
              acc[s][j] = __builtin_amdgcn_mfma_f32_4x4x1f32(on, x[j], acc[s][j], 0, 0, 0);
          }
        }
      }
      // ---- the four key groups of the wavefront; row k ends with cluster 4 s + k (of two: k & 1) ----
#pragma unroll
      for (int s = 0; s < SETS; ++s) {
        float o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[s][j][0]), __float_as_uint(acc[s][j][1]), false, false);
          const float c01 = __uint_as_float(p[0]) + __uint_as_float(p[1]);
          float c23 = c01;
          if constexpr (MAXC > 2) {
            const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[s][j][2]), __float_as_uint(acc[s][j][3]), false, false);
            c23 = __uint_as_float(q[0]) + __uint_as_float(q[1]);
          }
          const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(c01), __float_as_uint(c23), false, false);
          o[j] = __uint_as_float(w[0]) + __uint_as_float(w[1]);
        }
        if (4 * s + row < MAXC) {
          float4* dst = reinterpret_cast<float4*>(&part[wave][4 * s + row][l16 * 8]);
          dst[0] = make_float4(o[0], o[1], o[2], o[3]);
          dst[1] = make_float4(o[4], o[5], o[6], o[7]);
        }
      }
    }
    __syncthreads();
    ++n_done;
    if (it > 0 && s_changed[it & 1] == 0) {             // uniform: the previous update stands, and
      if (!a.converge) n_done = a.max_iter;             // further iterations would find it again
      break;
    }

    // ---- update: mean of the assigned keys, wavefronts in order; an empty cluster keeps its
    // centroid ----
    if (wave < C) {
      float s0 = 0.f, s1 = 0.f;
      int nn = l16 < WAVES ? cnt[l16 < WAVES ? l16 : 0][wave] : 0;
      nn += dpp_i0<DPP_XOR1>(nn);
      nn += dpp_i0<DPP_XOR2>(nn);
      nn += dpp_i0<DPP_HALF_MIRROR>(nn);
      nn += dpp_i0<DPP_MIRROR>(nn);
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const float2 v = *reinterpret_cast<const float2*>(&part[w][wave][2 * lane]);
        s0 += v.x;
        s1 += v.y;
      }
      if (nn > 0) {
        const float inv = 1.0f / (float)nn;
        m0 = s0 * inv;
        m1 = s1 * inv;
      }
    }
    // one cluster: further iterations would find the same labels, sums and mean, and the matrix
    // form does the work of four clusters for it (16 head-problems x 320 tokens x 10 iterations:
    // 39.7 us on the vector ALUs, 55 with all iterations, 10.5)
    if (C == 1 && a.max_iter > 1) {
      n_done = a.converge ? 2 : a.max_iter;
      break;
    }
  }
  if (lane < 16) {
#pragma unroll
    for (int T = 0; T < TILES; ++T) {
      const int t = (4 * T + (lane >> 2)) * KEYS + wave * 4 + (lane & 3);
      if (t < n_tok) lab[t] = label[T];
    }
  }
  __syncthreads();

  // ---- stores: centroids, labels, sizes, offsets, stable label-sorted index ----
  if (wave < C)
    reinterpret_cast<uint32_t*>(a.centroids + ((int64_t)hp * a.C_cap + a.c_begin + wave) * D)[lane] =
        (uint32_t)float_to_bf16_bits(m0) | ((uint32_t)float_to_bf16_bits(m1) << 16);
  int32_t* off_g = a.offsets + (int64_t)hp * (a.C_cap + 1);
  const int base0 = a.c_begin == 0 ? 0 : off_g[a.c_begin];
  const bool valid = tid < n_tok;
  const int l = valid ? lab[tid] : -1;
  const uint64_t lt = ((uint64_t)1 << lane) - 1;
  int rank = 0;
  for (int c = 0; c < C; ++c) {
    const uint64_t m = __ballot(l == c);
    if (l == c) rank = __popcll(m & lt);
    if (lane == 0) wave_cnt[wave][c] = __popcll(m);
  }
  __syncthreads();
  if (valid) {
    int pos = base0 + rank;
    for (int c = 0; c < l; ++c)
      for (int w = 0; w < SM_THREADS / WAVE; ++w) pos += wave_cnt[w][c];
    for (int w = 0; w < wave; ++w) pos += wave_cnt[w][l];
    if (pos >= 0 && pos < a.N_cap) a.sorted_idx[(int64_t)hp * a.N_cap + pos] = (int32_t)(a.tok_begin + tid);
    a.labels[(int64_t)hp * a.N_cap + a.tok_begin + tid] = a.c_begin + l;
  }
  if (tid == 0) {
    int run = base0;
    if (a.c_begin == 0) off_g[0] = 0;
    for (int c = 0; c < C; ++c) {
      int n = 0;
      for (int w = 0; w < SM_THREADS / WAVE; ++w) n += wave_cnt[w][c];
      a.sizes[(int64_t)hp * a.C_cap + a.c_begin + c] = n;
      run += n;
      off_g[a.c_begin + c + 1] = run;
    }
    if (a.iters_done) a.iters_done[hp] = n_done;
  }
}

bool kmeans_small_fits(int64_t tok_count, int c_count) {
  return tok_count <= KM_SMALL_MAX_TOKENS && c_count <= KM_SMALL_MAX_CLUSTERS;
}

hipError_t launch_kmeans_small(const Dims& dm, const bf16* K, int64_t tok_begin, int64_t tok_count,
                               int c_begin, int c_count, int max_iter, int metric, bool converge,
                               const int32_t* init_idx, bf16* centroids, int32_t* labels,
                               int32_t* sizes, int32_t* offsets, int32_t* sorted_idx,
                               int32_t* iters_done, hipStream_t st) {
  SmallArgs a;
  a.K = K;
  a.init_idx = init_idx;
  a.centroids = centroids;
  a.labels = labels;
  a.sizes = sizes;
  a.offsets = offsets;
  a.sorted_idx = sorted_idx;
  a.iters_done = iters_done;
  a.N_cap = dm.N_cap;
  a.tok_begin = tok_begin;
  a.tok_count = (int)tok_count;
  a.C_cap = dm.C_cap;
  a.c_begin = c_begin;
  a.c_count = c_count;
  a.max_iter = max_iter;
  a.metric = metric;
  a.converge = converge ? 1 : 0;
  auto launch = [&](auto MT) {
    constexpr int T = decltype(MT)::value;
    if (c_count <= 2)
      hipLaunchKernelGGL((k_kmeans_small<2, 1024, T>), dim3(dm.HP), dim3(1024), 0, st, a);
    else if (c_count <= 4)
      hipLaunchKernelGGL((k_kmeans_small<4, 1024, T>), dim3(dm.HP), dim3(1024), 0, st, a);
    else
      hipLaunchKernelGGL((k_kmeans_small<KM_SMALL_MAX_CLUSTERS, 512, T>), dim3(dm.HP), dim3(512), 0, st, a);
  };
  if (tok_count <= KM_SMALL_FEW_TOKENS) launch(std::integral_constant<int, KM_SMALL_FEW_TOKENS>());
  else launch(std::integral_constant<int, KM_SMALL_MAX_TOKENS>());
  return hipGetLastError();
}

}  // namespace ck
