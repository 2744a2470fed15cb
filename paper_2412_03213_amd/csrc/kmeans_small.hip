// Whole K-means of a small token range in ONE kernel (paper Section III-B, decode
// stage: every m generated tokens are clustered among themselves into a handful of
// new clusters).  At m = 320 tokens and 4 clusters an iteration is ~0.3 MFLOP per
// head-problem, so the prefill path with its two launches per iteration would spend
// its time on them; here one workgroup per head-problem keeps the keys in registers and
// runs init, all iterations (assignment, update), the metadata and the stores itself.
// Same arithmetic rules as the large path: bf16-rounded table rows compared in fp32,
// ties to the lower id, fp32 sums in a fixed order, means of raw keys, an empty cluster
// keeps its centroid.
#include "ck_common.hpp"

namespace ck {


struct SmallArgs {
  const bf16* K;
  const int32_t* init_idx;
  bf16* centroids;
  int32_t *labels, *sizes, *offsets, *sorted_idx, *iters_done;
  int64_t N_cap, tok_begin;
  int tok_count, C_cap, c_begin, c_count, max_iter, metric, converge;
};

// MAXC: compile-time bound of the cluster count; SM_THREADS: workgroup size.
//
// Bound: a chain of max_iter dependent iterations on one CU per head-problem, each of them VALU
// and cross-lane work on n_tok * C dot products.  Both halves of an iteration run on
// v_mfma_f32_4x4x1_16b_f32 (16 independent 4 x 4 outer products, one fp32 multiply-add per
// element and step, so the additions happen one by one in the order written here):
//   dot products  block = eight channels of a key (one per step), rows = 4 clusters, columns = 4
//                 keys: 8 steps replace 32 multiply-adds, and the sixteen partial sums of a
//                 (key, cluster) are added by lane swaps that halve the registers on the way;
//   update sums   block = four lanes of one key, rows = 4 clusters, A = 1 where the key's label
//                 is the row's cluster: 8 steps replace 32 multiply-adds.
// A wavefront keeps its keys in registers in both layouts for all iterations (no LDS pass over
// the keys).  The wavefront of a cluster adds up that cluster's partial sums, keeps its mean in
// registers and makes the next table row from it, so an iteration has two barriers.
// 128 head-problems x 320 tokens x 4 clusters, 10 iterations: 85.3 -> 56.6 us, same bits; 53.0 since
// a wavefront whose keys have all kept their labels leaves its sums of the iteration before standing
// (a mixture of 128 centers: labels settle after 5 to 20 iterations, 9.7 on average).
// MAXC = 2 is a form of its own: rows 2 and 3 of the products are idle there, and with the lane
// exchanges of four clusters it was slower than the vector ALUs (352 tokens x 2 clusters: 55.6 us on
// the vector ALUs, 62.8 as four clusters, 52.9 now; 100 tokens: 38.6, 33.1, 28.3).
template <int MAXC, int SM_THREADS>
__global__ __launch_bounds__(SM_THREADS) void k_kmeans_small(const SmallArgs a) {
  constexpr int WAVES = SM_THREADS / WAVE, SETS = (MAXC + 3) / 4, ROWS = 4 * SETS;
  constexpr int KEYS = WAVES * 4;                       // keys per round, four per wavefront
  constexpr int ROUNDS = (KM_SMALL_MAX_TOKENS + KEYS - 1) / KEYS;
  static_assert((MAXC == 2 || MAXC % 4 == 0) && MAXC <= WAVES && KM_SMALL_MAX_TOKENS <= SM_THREADS, "mapping");
  __shared__ __attribute__((aligned(16))) float table[ROWS][D];
  __shared__ __attribute__((aligned(16))) float part[WAVES][MAXC][D];
  __shared__ int cnt[WAVES][MAXC];
  __shared__ int wave_cnt[WAVES][MAXC];
  __shared__ float bias[ROWS];
  __shared__ int lab[KM_SMALL_MAX_TOKENS];
  __shared__ int s_changed[2];

  const int hp = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, row = lane >> 4, l4 = lane & 3;
  const int n_tok = a.tok_count, C = a.c_count;
  const bf16* Khp = a.K + (int64_t)hp * a.N_cap * D;

  // ---- this wavefront's keys: of round r, keys 4 * wave + (0..3) ----
  // dk: lane 4 b + x holds the eight channels of group bitreverse(b) of key x.  Lane bits 5, 4, 3, 2
  // are then bits 0, 1, 2, 3 of the channel group, and the partial sums are added in the order
  // of row16_sum.  uk: lanes 16 x + g hold channel group g of key x.
  const int b = lane >> 2;
  const int dgroup = ((b & 1) << 3) | ((b & 2) << 1) | ((b & 4) >> 1) | (b >> 3);
  uint4 dk[ROUNDS], uk[ROUNDS];
  {
    const uint4* R = reinterpret_cast<const uint4*>(Khp + a.tok_begin * D);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {                  // a key beyond the range re-reads the last one
      const int td = r * KEYS + wave * 4 + l4, tu = r * KEYS + wave * 4 + row;
      uk[r] = R[(int64_t)(tu < n_tok ? tu : n_tok - 1) * 16 + l16];
      dk[r] = R[(int64_t)(td < n_tok ? td : n_tok - 1) * 16 + dgroup];
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)                    // ... and adds nothing
      if (r * KEYS + wave * 4 + row >= n_tok) uk[r] = make_uint4(0, 0, 0, 0);
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
  for (int e = C * D + tid; e < ROWS * D; e += SM_THREADS) table[e / D][e % D] = 0.f;

  // After the lane swaps row r of a register holds cluster 4 s + {0, 2, 1, 3}[r], or of two
  // clusters {0, 0, 1, 1}[r]
  const int rowc = MAXC == 2 ? row >> 1 : ((row & 1) << 1) | (row >> 1);
  uint32_t labels[(ROUNDS + 7) / 8];                    // 4 bits per round: label of key `l4`
#pragma unroll
  for (int i = 0; i < (ROUNDS + 7) / 8; ++i) labels[i] = 0xFFFFFFFFu;

  int n_done = 0;
  for (int it = 0; it < a.max_iter; ++it) {
    // ---- table row (and l2 bias) of cluster `wave` ----
    if (wave < C) {
      float r0, r1;
      if (a.metric == CK_METRIC_COSINE) {
        // the fused product written out: the last bit of the norm must not depend on the
        // compiler's choice
        const float n2 = wave_sum(fmaf(m0, m0, m1 * m1));
        const float inv = n2 > 0.f ? 1.0f / sqrtf(n2) : 0.f;
        r0 = bf16_bits_to_float(float_to_bf16_bits(m0 * inv));
        r1 = bf16_bits_to_float(float_to_bf16_bits(m1 * inv));
      } else {
        r0 = bf16_bits_to_float(float_to_bf16_bits(m0));
        r1 = bf16_bits_to_float(float_to_bf16_bits(m1));
      }
      *reinterpret_cast<float2*>(&table[wave][2 * lane]) = make_float2(r0, r1);
      if (a.metric == CK_METRIC_L2) {
        const float rn2 = wave_sum(fmaf(r0, r0, r1 * r1));
        if (lane == 0) bias[wave] = -0.5f * rn2;
      } else if (lane == 0) {
        bias[wave] = 0.f;
      }
    }
    if (tid == 0) s_changed[it & 1] = 0;                // the other one may still be read
    __syncthreads();

    float ta[SETS][8], bs[SETS];
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
      const float4* t = reinterpret_cast<const float4*>(&table[4 * s + l4][dgroup * 8]);
      const float4 x = t[0], y = t[1];
      ta[s][0] = x.x; ta[s][1] = x.y; ta[s][2] = x.z; ta[s][3] = x.w;
      ta[s][4] = y.x; ta[s][5] = y.y; ta[s][6] = y.z; ta[s][7] = y.w;
      // a row without a cluster is a NaN, which never wins
      bs[s] = 4 * s + rowc < C ? bias[4 * s + rowc] : __builtin_nanf("");
    }
    uint32_t moved = 0;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      // two clusters: wavefronts without keys in a round sit it out (321 tokens 55.3 -> 51.4 us, but
      // 320 tokens 49.0 -> 50.7, and 56.0 -> 57.6 with four clusters, where a round in full is the rule)
      if (r * KEYS + (MAXC == 2 ? wave * 4 : 0) < n_tok) {   // wave-uniform
        // unpacked here and not once before the iterations: there are no registers for that
        asm volatile("" : "+v"(dk[r].x), "+v"(dk[r].y), "+v"(dk[r].z), "+v"(dk[r].w));
        const uint32_t dw[4] = {dk[r].x, dk[r].y, dk[r].z, dk[r].w};
        float best = 0.f;
        int bc = 0;
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
          floatx4 d = {0.f, 0.f, 0.f, 0.f};             // [cluster 4 s + i] of key l4, channel group of b
#pragma unroll
          for (int j = 0; j < 8; ++j)
            d = __builtin_amdgcn_mfma_f32_4x4x1f32(ta[s][j], j & 1 ? hi_bf16(dw[j / 2]) : lo_bf16(dw[j / 2]), d, 0, 0, 0);
          // sixteen channel groups: lane bits 5, 4 (two clusters share a register from there
          // on), 3, 2
          const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(d[0]), __float_as_uint(d[1]), false, false);
          const float c01 = __uint_as_float(p[0]) + __uint_as_float(p[1]);
          float c23 = c01;
          if constexpr (MAXC > 2) {
            const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(d[2]), __float_as_uint(d[3]), false, false);
            c23 = __uint_as_float(q[0]) + __uint_as_float(q[1]);
          }
          const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(c01), __float_as_uint(c23), false, false);
          float v = __uint_as_float(w[0]) + __uint_as_float(w[1]);
          v += dpp_f<DPP_ROR8>(v);
          v += dpp_f<DPP_ROR4>(v);                      // lanes x and x ^ 8 are equal by now
          v += bs[s];
          // a NaN never wins over another cluster and is never beaten as cluster 0
          v = v == v ? v : (4 * s + rowc == 0 ? INFINITY : -INFINITY);
          // best of the four, the lower cluster where they are equal: rows hold 0, 2, 1, 3
          const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
          const float x0 = __uint_as_float(x[0]), x1 = __uint_as_float(x[1]);
          if constexpr (MAXC == 2) {
            bc = x1 > x0 ? 1 : 0;
          } else {
            const float xv = x1 > x0 ? x1 : x0;
            const unsigned xc = (row & 1) * 2 + (x1 > x0 ? 1 : 0);
            const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(xv), __float_as_uint(xv), false, false);
            const auto yc = __builtin_amdgcn_permlane16_swap(xc, xc, false, false);
            const float y0 = __uint_as_float(y[0]), y1 = __uint_as_float(y[1]);
            const float yv = y1 > y0 ? y1 : y0;
            const int c = 4 * s + (int)(y1 > y0 ? yc[1] : yc[0]);
            if (s == 0 || yv > best) {
              best = yv;
              bc = c;
            }
          }
        }
        // a key that does not exist belongs to no cluster
        if (r * KEYS + wave * 4 + l4 >= n_tok) bc = 15;
        const uint32_t word = labels[r / 8], put = (word & ~(15u << (r % 8 * 4))) | ((uint32_t)bc << (r % 8 * 4));
        moved |= word ^ put;
        labels[r / 8] = put;
        __builtin_amdgcn_sched_barrier(0);              // rounds one after another: registers
      }
    }
    // ---- the sums over this wavefront's keys: where none of its labels has changed, those of the
    // iteration before stand in part and cnt ----
    const bool any_moved = __ballot(moved != 0) != 0;
    if (any_moved && lane == 0) s_changed[it & 1] = 1;
    if (any_moved || it == 0) {
      floatx4 acc[SETS][8];                               // [channel 8 l16 + j][cluster 4 s + i], key group `row`
      int n[SETS];                                        // members of cluster 4 s + l4 in key group `row`
#pragma unroll
      for (int s = 0; s < SETS; ++s) {
        n[s] = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[s][j] = {0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        if (r * KEYS + (MAXC == 2 ? wave * 4 : 0) < n_tok) {   // wave-uniform
          asm volatile("" : "+v"(uk[r].x), "+v"(uk[r].y), "+v"(uk[r].z), "+v"(uk[r].w));
          const int bc = (int)(labels[r / 8] >> (r % 8 * 4)) & 15;
          // label of key `row` into all lanes of that row: lane x of every quad has key x's
          int ub = 0;
          ub = __builtin_amdgcn_update_dpp(ub, bc, 0x00, 0x1, 0xf, false);
          ub = __builtin_amdgcn_update_dpp(ub, bc, 0x55, 0x2, 0xf, false);
          ub = __builtin_amdgcn_update_dpp(ub, bc, 0xAA, 0x4, 0xf, false);
          ub = __builtin_amdgcn_update_dpp(ub, bc, 0xFF, 0x8, 0xf, false);
          const uint32_t uw[4] = {uk[r].x, uk[r].y, uk[r].z, uk[r].w};
#pragma unroll
          for (int s = 0; s < SETS; ++s) {
            const bool mine = ub == 4 * s + l4;
            const float on = mine ? 1.f : 0.f;
            n[s] += mine ? 1 : 0;
#pragma unroll
            for (int j = 0; j < 8; ++j)
              acc[s][j] = __builtin_amdgcn_mfma_f32_4x4x1f32(on, j & 1 ? hi_bf16(uw[j / 2]) : lo_bf16(uw[j / 2]), acc[s][j], 0, 0, 0);
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
        n[s] += __shfl_xor(n[s], 16, WAVE);
        n[s] += __shfl_xor(n[s], 32, WAVE);
        if (lane < 4 && 4 * s + lane < MAXC) cnt[wave][4 * s + lane] = n[s];
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
      int nn = 0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const float2 v = *reinterpret_cast<const float2*>(&part[w][wave][2 * lane]);
        s0 += v.x;
        s1 += v.y;
        nn += cnt[w][wave];
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
  if (lane < 4) {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int t = r * KEYS + wave * 4 + lane;
      if (t < n_tok) lab[t] = (int)(labels[r / 8] >> (r % 8 * 4)) & 15;
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
  if (c_count <= 2)
    hipLaunchKernelGGL((k_kmeans_small<2, 1024>), dim3(dm.HP), dim3(1024), 0, st, a);
  else if (c_count <= 4)
    hipLaunchKernelGGL((k_kmeans_small<4, 1024>), dim3(dm.HP), dim3(1024), 0, st, a);
  else
    hipLaunchKernelGGL((k_kmeans_small<KM_SMALL_MAX_CLUSTERS, 512>), dim3(dm.HP), dim3(512), 0, st, a);
  return hipGetLastError();
}

}  // namespace ck
