// Sparse GQA decode attention over the recalled tokens (paper Section II-B:
// softmax(q K_S^T / sqrt(d)) V_S with K_S, V_S the selected rows), alone or fused
// with the centroid scoring and cluster selection of Section III-C and the index
// generation of Section IV-C: a whole decode step is then ONE kernel launch.
//
// HBM-bound: every recalled K and V row (256 B in bf16) is read exactly once per
// KV head and shared by the G query heads of the group.  A wavefront takes 16
// tokens per step, 16 lanes loading a whole row.  In bf16 both products run on the
// matrix cores (fp32 check mode keeps the all-VALU form): q K^T with the K rows, passed
// through LDS, as the A operand; P V with operands that are already in the right lanes
// (see the kernel).  One launch of the whole step takes 10.1 us at 8 head-problems, B = 1024
// (13.9 with K rows loaded in operand layout, P V on the vector ALUs and one wavefront
// selecting) and 20.3 at 64, B = 2048 (25.5), of which the row stream at 6.4 TB/s is half;
// the rest is a chain of dependent round trips.  The attended positions of a head-problem are
// split over several workgroups (split-KV) so that a batch of a few sequences still fills 256
// CUs, and never over more than are resident together (attn_plan).  Inside a workgroup every
// wavefront resolves the token rows of its own positions first, and the K/V loads of the next
// TWO steps are in flight while the current one is reduced.
//
// Merging the splits without a second launch: every workgroup publishes its partial
// (max, sum, accumulator) with agent-scope stores, takes a ticket from a counter of
// its head-problem, and the workgroup that draws the last ticket reads all partials
// back with agent-scope loads and writes the output.  Nobody waits for anybody, so
// nothing can hang; agent-scope accesses are performed past the XCD-private L2
// caches, so no cache write-back or invalidate is needed.  The merge adds the
// partials in split order, whoever runs it: results are bit-reproducible.
//
// Fused modes: every workgroup of a head-problem repeats the (cheap, LDS-only)
// selection of the recalled cluster prefix and maps its own positions through the
// cluster-contiguous index directly, from the ranked clusters in registers; the index list is
// still written out (each workgroup its own part) but never re-read.  With at most 512 clusters in bf16 the
// centroid scores are computed by every workgroup as well (the workgroups of one
// head-problem are placed on one XCD, so the table comes from HBM once and out of
// that XCD's L2 otherwise); larger or fp32 tables are scored by a launch of their own.
#include <mutex>
#include <type_traits>

#include "decode_common.hpp"

namespace ck {

constexpr int ATT_TOKENS = 16;             // tokens of a wavefront per step
constexpr int ATT_MAX_CHUNK = 2048;        // positions one workgroup may own (rows held in LDS)
constexpr int ATT_MAX_SPLITS = 1024;       // workgroups per head-problem
constexpr float NEG_BIG = -1.0e30f;        // "no token yet": finite so that differences stay finite
constexpr int ATT_XCD_CUS = 32;            // compute units of one XCD
constexpr int PART_STRIDE = D + 2;         // floats per (split, query head): max, sum, acc[128]
constexpr int N_XCD = 8;                   // workgroup i of a launch runs on XCD i % 8
constexpr unsigned long long TICKET_MAGIC = 0x434B7469636Bull;   // marks a ticket word as ours

enum { ATT_PLAIN = 0, ATT_FUSED = 1, ATT_FUSED_SCORE = 2 };

template <typename T> struct RawRow;
template <> struct RawRow<bf16> {
  uint4 w;
  __device__ __forceinline__ void load(const bf16* p) { w = *reinterpret_cast<const uint4*>(p); }
  __device__ __forceinline__ void unpack(float (&v)[8]) const {
    v[0] = lo_bf16(w.x); v[1] = hi_bf16(w.x); v[2] = lo_bf16(w.y); v[3] = hi_bf16(w.y);
    v[4] = lo_bf16(w.z); v[5] = hi_bf16(w.z); v[6] = lo_bf16(w.w); v[7] = hi_bf16(w.w);
  }
};
template <> struct RawRow<float> {
  float4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = reinterpret_cast<const float4*>(p)[0];
    b = reinterpret_cast<const float4*>(p)[1];
  }
  __device__ __forceinline__ void unpack(float (&v)[8]) const {
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
};

__device__ __forceinline__ void store_out(bf16* p, float v) {
  *reinterpret_cast<uint16_t*>(p) = float_to_bf16_bits(v);
}
__device__ __forceinline__ void store_out(float* p, float v) { *p = v; }

// ---- partials in memory: pairs of floats, moved as one 64-bit word ----
// Agent scope: the access is performed past the XCD-private L2, so a workgroup on
// another XCD sees the value without any cache maintenance.
__device__ __forceinline__ void put_pair_agent(float* p, float x, float y) {
  const unsigned long long w =
      (unsigned long long)__float_as_uint(x) | ((unsigned long long)__float_as_uint(y) << 32);
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), w, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
struct PairAgent {
  __device__ __forceinline__ float2 operator()(const float* p) const {
    const unsigned long long w =
        __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((uint32_t)w), __uint_as_float((uint32_t)(w >> 32)));
  }
};
struct PairPlain {
  __device__ __forceinline__ float2 operator()(const float* p) const {
    return *reinterpret_cast<const float2*>(p);
  }
};

// out channels (c2, c2 + 1) of one query head from its n_split partials:
//   sum_i acc_i 2^(m_i - M) / sum_i l_i 2^(m_i - M), splits added in index order,
// BATCH partials loaded together so that their latencies overlap.
// base = partial of split 0 for this head, stride = floats between splits.
template <int BATCH, typename Load>
__device__ __forceinline__ float2 merge_batches(const float* base, int64_t stride, int n_split,
                                                int c2, Load load) {
  float M = NEG_BIG, ls = 0.f, a0 = 0.f, a1 = 0.f;
  for (int i0 = 0; i0 < n_split; i0 += BATCH) {
    float2 ml[BATCH], av[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const bool ok = i0 + i < n_split;
      const float* p = base + (int64_t)(ok ? i0 + i : 0) * stride;
      ml[i] = load(p);
      av[i] = load(p + 2 + c2);
      if (!ok) {
        ml[i] = make_float2(NEG_BIG, 0.f);
        av[i] = make_float2(0.f, 0.f);
      }
    }
    float mx = M;
#pragma unroll
    for (int i = 0; i < BATCH; ++i) mx = fmaxf(mx, ml[i].x);
    const float corr = __builtin_amdgcn_exp2f(M - mx);
    ls *= corr;
    a0 *= corr;
    a1 *= corr;
    M = mx;
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const float f = __builtin_amdgcn_exp2f(ml[i].x - mx);
      ls += ml[i].y * f;
      a0 += av[i].x * f;
      a1 += av[i].y * f;
    }
  }
  const float inv = ls > 0.f ? 1.0f / ls : 0.f;
  return make_float2(a0 * inv, a1 * inv);
}
// The smallest batch that takes all splits at once (the loads go past the L2: those of a
// padded batch would cost as much as the real ones).
template <typename Load>
__device__ __forceinline__ float2 merge_splits(const float* base, int64_t stride, int n_split,
                                               int c2, Load load) {
  if (n_split <= 4) return merge_batches<4>(base, stride, n_split, c2, load);
  if (n_split <= 8) return merge_batches<8>(base, stride, n_split, c2, load);
  return merge_batches<16>(base, stride, n_split, c2, load);
}

struct AttnArgs {
  const void *q, *K, *V;
  void* out;
  float* part;                  // [HP, n_split, G, PART_STRIDE]
  unsigned long long* tickets;  // [HP]: (TICKET_MAGIC << 16) | workgroups arrived so far
  // given index list
  const int32_t* token_idx;
  const int32_t* n_tokens;
  // fused selection
  const void* centroids;        // ATT_FUSED_SCORE: the table to score
  float* scores;                // ATT_FUSED: read; ATT_FUSED_SCORE: written
  const int32_t *sizes, *offsets, *sorted_idx;
  int32_t *sel_clusters, *n_sel_clusters, *n_sel_tokens, *token_idx_out, *n_tokens_out;
  int n_clusters, budget, trim, C_cap;
  // common
  int HP, idx_stride, max_tokens, Hq, Hkv, n_sink, n_recent, chunk, n_split, two_pass, spread;
  int64_t N_cap, recent_begin;
  float scale_log2e;
  CacheArgs cache;              // CACHED: K and V above are the home copy
};

template <int G, int NW> struct PlainLds { float red[G ? NW * G * PART_STRIDE : 1]; };
template <int CMAX, int NT> struct FusedLds {
  QuickLds<NT> quick;
  SelectLds<CMAX, NT> general;
};

// Value of lane g of the 16-lane row, in every lane of the row.
template <int LANE>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + LANE, 0xf, 0xf, true));
}
// Attended position p of a head-problem -> token row:
//   [0, n_sink) sinks, then the recalled list, then [recent_begin, recent_end).
// Position i of a workgroup belongs to wavefront (i / 16) % NW.
// One-dimensional grid: workgroup i runs on XCD i % 8 (round-robin dispatch), so the
// n_split workgroups of a head-problem are given ids of one residue class and share
// that XCD's L2 (sizes, offsets, scores or the centroid table), except where launch_attn_t
// spreads them over all XCDs.  Placement only affects speed, never results.
// (Two wavefronts per SIMD is what the row stream's registers allow; the attribute keeps the
// compiler from aiming higher and spilling.)
// CACHED: the step over a home copy in host memory and the cluster cache (see cluster_cache.hip).  A
// row comes from the previous generation where its cluster is held there and from the home copy
// otherwise, and is stored into the new generation on its way into the products, so that selection,
// fetch and attention are one launch and only the host link counts: four steps at 8 head-problems,
// B = 1024 took 337 us as scoring, selection, fill and attention, 299 now (14.7 MB over the link, whose
// 55 GB/s are 267 us of it).
template <typename T, int G, int MODE, int CMAX, int NW, bool CACHED>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 2 ? 2 : 1, 2))) void k_attn(const AttnArgs a) {
  constexpr bool FUSED = MODE != ATT_PLAIN;
  constexpr int NT = NW * 64, STEP = NW * ATT_TOKENS;
  constexpr bool BF16 = std::is_same<T, bf16>::value;
  union Big {                                           // selection, later the wavefront partials (fp32)
    PlainLds<BF16 ? 0 : G, NW> plain;
    typename std::conditional<FUSED, FusedLds<CMAX, NT>, PlainLds<BF16 ? 0 : G, NW>>::type fused;
  };
  __shared__ Big big;
  __shared__ __attribute__((aligned(16))) int rows_lds[ATT_MAX_CHUNK];
  __shared__ __attribute__((aligned(16))) float sc_lds[MODE == ATT_FUSED_SCORE ? CMAX : 4];
  __shared__ __attribute__((aligned(16))) bf16 stage_lds[BF16 ? NW * STAGE_ELEMS : 8];
  __shared__ int s_last;
  static_assert(!CACHED || (FUSED && std::is_same<T, bf16>::value), "cached steps select and are bf16");
  int* held = nullptr;                                  // cluster id -> first row in the previous generation, -1
  // Partial of a wavefront: in bf16 where its rows changed lanes, which is its own, so that it need
  // not wait for the others to be through with the selection.
  constexpr int RED_STRIDE = BF16 ? STAGE_ELEMS / 2 : G * PART_STRIDE;
  static_assert(RED_STRIDE >= G * PART_STRIDE, "partial in the staging area");
  float* red = BF16 ? reinterpret_cast<float*>(stage_lds) : big.plain.red;

  // one argument per 64-byte line of the argument block: all lines are requested now
  CK_FETCH_ARG(a.q);
  CK_FETCH_ARG(a.n_tokens);
  CK_FETCH_ARG(a.sorted_idx);
  CK_FETCH_ARG(a.n_tokens_out);
  CK_FETCH_ARG(a.n_clusters);
  CK_FETCH_ARG(a.C_cap);
  CK_FETCH_ARG(a.n_sink);
  CK_FETCH_ARG(a.scale_log2e);
  if constexpr (CACHED) {
    CK_FETCH_ARG(a.cache.old_clusters);
    CK_FETCH_ARG(a.cache.cap);
  }
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, col = lane & 15, kg = lane >> 4;
  const int wg = blockIdx.x, xcd = wg % N_XCD, seq = wg / N_XCD;
  const bool spread = MODE == ATT_PLAIN && a.spread;    // see launch_attn_t
  const int hp = spread ? wg % a.HP : (seq / a.n_split) * N_XCD + xcd;
  const int split = spread ? wg / a.HP : seq % a.n_split;
  if (hp >= a.HP) return;                               // the grid is padded to whole groups of 8
  const int s = hp / a.Hkv, h = hp % a.Hkv;
  const T* q = static_cast<const T*>(a.q);
  const Stage16 stage(stage_lds + (BF16 ? wave * STAGE_ELEMS : 0), lane);

  // the query heads of the group as an MFMA operand (bf16): for the scores and for q K^T
  bf16x8 qb[4];
  if constexpr (std::is_same<T, bf16>::value)
    load_query_operand(reinterpret_cast<const bf16*>(q) + ((int64_t)s * a.Hq + h * G) * D, G, lane, qb);

  int n_idx;
  Quick sel;
  if constexpr (FUSED) {
    QuickLds<NT>& Q = big.fused.quick;
    SelectLds<CMAX, NT>& L = big.fused.general;
    constexpr int ITEMS = CMAX / NT;
    float sc[ITEMS];
    int sz[ITEMS], of[ITEMS];
    float mx = -INFINITY, mn = INFINITY;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {                   // unconditional: one round trip with the scores
      const int c = tid + i * NT, cc = c < a.n_clusters ? c : a.n_clusters - 1;
      sz[i] = a.sizes[(int64_t)hp * a.C_cap + cc];
      of[i] = a.offsets[(int64_t)hp * (a.C_cap + 1) + cc];
      if constexpr (MODE == ATT_FUSED) sc[i] = a.scores[(int64_t)hp * a.C_cap + cc];
    }
    int old_id[ITEMS], old_row[ITEMS], n_old = 0;
    if constexpr (CACHED) {
      n_old = a.cache.old_n[hp];
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const int c = tid + i * NT, cc = c < a.C_cap ? c : a.C_cap - 1;
        old_id[i] = a.cache.old_clusters[(int64_t)hp * a.C_cap + cc];
        old_row[i] = a.cache.old_starts[(int64_t)hp * (a.C_cap + 1) + cc];
      }
    }
    quick_clear(Q);
    if constexpr (MODE == ATT_FUSED_SCORE) {
      // ---- scores of all clusters of this head-problem (bf16 table, matrix cores) ----
      // Every load of the prologue is issued before the first use: the table rows of
      // this wavefront (16 rows per step, steps wave, wave + NW, ...), the query heads,
      // the sizes and offsets this thread will bring to the selection: one round trip.
      constexpr int SB = CMAX / (16 * NW);              // 16-row steps per wavefront
      const bf16* Thp = static_cast<const bf16*>(a.centroids) + (int64_t)hp * a.C_cap * D + col * 8;
      const int n_steps = (a.n_clusters + 15) >> 4;
      uint4 ar[SB][4];
#pragma unroll
      for (int u = 0; u < SB; ++u) {
        if (wave + NW * u < n_steps) {                  // wave-uniform
          const int r0 = (wave + NW * u) * 16 + 4 * kg, rl = a.n_clusters - 1;   // clamp: result is discarded
          ar[u][0] = *reinterpret_cast<const uint4*>(Thp + (int64_t)(r0 < rl ? r0 : rl) * D);
          ar[u][1] = *reinterpret_cast<const uint4*>(Thp + (int64_t)(r0 + 1 < rl ? r0 + 1 : rl) * D);
          ar[u][2] = *reinterpret_cast<const uint4*>(Thp + (int64_t)(r0 + 2 < rl ? r0 + 2 : rl) * D);
          ar[u][3] = *reinterpret_cast<const uint4*>(Thp + (int64_t)(r0 + 3 < rl ? r0 + 3 : rl) * D);
        }
      }
#pragma unroll
      for (int u = 0; u < SB; ++u) {
        if (wave + NW * u < n_steps) {
          stage.put(ar[u][0], ar[u][1], ar[u][2], ar[u][3]);
          const float v = score_rows16(stage, qb, G);
          const int r = (wave + NW * u) * 16 + lane;
          if (lane < 16 && r < a.n_clusters) {
            sc_lds[r] = v;
            if (split == 0) a.scores[(int64_t)hp * a.C_cap + r] = v;
            mx = fmaxf(mx, v);
            mn = fminf(mn, v);
          }
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {                 // a repeated last entry does not widen the range
        mx = fmaxf(mx, sc[i]);
        mn = fminf(mn, sc[i]);
      }
    }
    quick_range(Q, mx, mn);
    __syncthreads();
    if constexpr (MODE == ATT_FUSED_SCORE) {
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const int c = tid + i * NT;
        sc[i] = c < a.n_clusters ? sc_lds[c] : 0.f;
      }
    }
    sel = quick_select<NT, ITEMS>(Q, sc, sz, of, a.n_clusters, a.budget, a.trim);
    if (sel.m > WAVE) {                                 // uniform: more candidates than lanes
      select_many<CMAX, NT>(L, Q, sc, sz, of, sel.m, sel.last_bin, a.n_clusters, a.budget, a.trim);
      sel.n_sel = L.n_sel;
      sel.n_tok = L.n_tok;
    }
    n_idx = sel.n_tok;
    if constexpr (CACHED) {
      // A prefix of whole clusters fits the budget; where sizes that are no sizes make its sum wrap, no
      // row behind it is stored all the same.
      n_idx = n_idx < a.budget ? n_idx : a.budget;
      held = reinterpret_cast<int*>(L.key);             // the selection is through with it
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) held[tid + i * NT] = -1;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < ITEMS; ++i)
        if (tid + i * NT < n_old && tid + i * NT < a.C_cap && (unsigned)old_id[i] < (unsigned)CMAX)
          held[old_id[i]] = old_row[i];
      // more clusters held than this form selects from: the table was larger at the step before
      for (int j = tid + ITEMS * NT; j < n_old && j < a.C_cap; j += NT) {
        const int id = a.cache.old_clusters[(int64_t)hp * a.C_cap + j];
        if ((unsigned)id < (unsigned)CMAX) held[id] = a.cache.old_starts[(int64_t)hp * (a.C_cap + 1) + j];
      }
      __syncthreads();
    }
    if (split == 0) {
      if (sel.m <= WAVE) {
        if (tid < sel.n_sel) a.sel_clusters[(int64_t)hp * a.C_cap + tid] = sel.id;
      } else {
        for (int j = tid; j < sel.n_sel; j += NT)
          a.sel_clusters[(int64_t)hp * a.C_cap + j] = L.ord[j];
      }
      if (tid == 0) {
        a.n_sel_clusters[hp] = sel.n_sel;
        a.n_sel_tokens[hp] = n_idx;
        if constexpr (!CACHED) a.n_tokens_out[hp] = n_idx;
      }
      if constexpr (CACHED) {                           // the new generation's directory
        int miss = 0;
        if (wave == 0) {
          for (int j = lane; j < sel.n_sel; j += WAVE) {
            const bool few = sel.m <= WAVE;
            const int id = few ? sel.id : L.ord[j], end = few ? sel.cum : L.cum[j];
            const int begin = few ? sel.cum - sel.size : (j ? L.cum[j - 1] : 0);
            a.cache.new_clusters[(int64_t)hp * a.C_cap + j] = id;
            a.cache.new_starts[(int64_t)hp * (a.C_cap + 1) + j] = begin;
            if (held[id] < 0) miss += end - begin;
          }
          miss = __builtin_amdgcn_readlane(wave_inclusive_scan(miss), WAVE - 1);
          if (lane == 0) {
            a.cache.new_starts[(int64_t)hp * (a.C_cap + 1) + sel.n_sel] = n_idx;
            a.cache.new_n[hp] = sel.n_sel;
            a.cache.miss_tokens[hp] = miss;
          }
        }
      }
    }
  } else {
    n_idx = a.n_tokens ? a.n_tokens[hp] : 0;
    n_idx = n_idx < 0 ? 0 : (n_idx > a.max_tokens ? a.max_tokens : n_idx);
  }
  const int n_total = a.n_sink + n_idx + a.n_recent;
  const int p_begin = split * a.chunk;
  int p_end = p_begin + a.chunk;
  if (p_end > n_total) p_end = n_total;
  const int n_pos = p_end > p_begin ? p_end - p_begin : 0;
  const int n_steps = (n_pos + STEP - 1) / STEP;

  // ---- token rows of this wavefront's positions, entry 16 t + x: token x of step t ----
  // (a position beyond the end reads row 0 and is masked later)
  // CACHED: ~row of the previous generation, or a row of the home copy; what stands in for a
  // position beyond the end does not come over the host link
  int* rows = rows_lds + wave * (ATT_MAX_CHUNK / NW);
  int sel_held = -1;                                    // of the cluster of rank `lane`
  if constexpr (CACHED)
    if (sel.m <= WAVE && lane < sel.n_sel) sel_held = held[sel.id];
  for (int e0 = 0; e0 < n_steps * 16; e0 += WAVE) {
    const int e = e0 + lane;
    const int i = (e >> 4) * STEP + wave * 16 + (e & 15);
    const int p = p_begin + i, qpos = p - a.n_sink;
    const bool own = i < n_pos, listed = own && qpos >= 0 && qpos < n_idx;
    int64_t row = 0;
    if constexpr (FUSED) {
      int64_t src = 0;
      int from_old = -1;
      if (sel.m <= WAVE) {
        // the clusters this wavefront's positions cross, in order, out of the lanes that
        // hold them (empty clusters of the prefix cover no position)
        const int q0 = p_begin + (e0 >> 4) * STEP + wave * 16 - a.n_sink;
        const int q1 = q0 + (WAVE / 16 - 1) * STEP + 16;
        const uint64_t after = __ballot(lane < sel.m && sel.cum > q0);
        for (int j = after ? __builtin_ctzll(after) : sel.m; j < sel.n_sel; ++j) {
          const int cum = __builtin_amdgcn_readlane(sel.cum, j);
          const int size = __builtin_amdgcn_readlane(sel.size, j);
          const int off = __builtin_amdgcn_readlane(sel.off, j);
          const int prev = cum - size;
          if (prev >= q1) break;
          int take = a.budget - prev;                   // a cut cluster keeps its trailing entries
          take = take > size ? size : take;
          const int old = CACHED ? __builtin_amdgcn_readlane(sel_held, j) : -1;
          if (qpos >= prev && qpos < cum) {
            src = (int64_t)off + (size - take) + (qpos - prev);
            if (CACHED && old >= 0) from_old = old + (qpos - prev);
          }
        }
      } else if (listed) {
        SelectLds<CMAX, NT>& L = big.fused.general;
        // smallest j with cum[j] > qpos (empty clusters in the prefix are skipped)
        int lo = 0, hi = L.n_sel - 1;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (L.cum[mid] > qpos) hi = mid; else lo = mid + 1;
        }
        const int c = L.ord[lo];
        const int prev = lo ? L.cum[lo - 1] : 0;
        const int size = L.cum[lo] - prev;
        int take = a.budget - prev;
        take = take > size ? size : take;
        const int beg = L.full_rank ? L.soff[c] : L.cbeg[lo];
        src = (int64_t)beg + (size - take) + (qpos - prev);
        if constexpr (CACHED)
          if (held[c] >= 0) from_old = held[c] + (qpos - prev);
      }
      if constexpr (CACHED) {
        if (listed && from_old < 0) {
          src = src < 0 ? 0 : (src >= a.N_cap ? a.N_cap - 1 : src);
          row = a.sorted_idx[(int64_t)hp * a.N_cap + src];
          row = row < 0 ? 0 : (row >= a.N_cap ? a.N_cap - 1 : row);
        } else {
          from_old = listed ? from_old : 0;
          row = ~(int64_t)(from_old < a.cache.cap ? from_old : a.cache.cap - 1);
        }
        if (e < ATT_MAX_CHUNK / NW) rows[e] = (int)row;
        continue;
      }
      if (listed) {
        src = src < 0 ? 0 : (src >= a.N_cap ? a.N_cap - 1 : src);
        row = a.sorted_idx[(int64_t)hp * a.N_cap + src];
        a.token_idx_out[(int64_t)hp * a.idx_stride + qpos] = (int32_t)row;
      }
    } else {
      // no list: the first n_tokens rows of K/V themselves (a dense per-head-problem prefix)
      if (listed) row = a.token_idx ? a.token_idx[(int64_t)hp * a.idx_stride + qpos] : qpos;
    }
    if (own && qpos < 0) row = p;
    if (own && qpos >= n_idx) row = a.recent_begin + (qpos - n_idx);
    row = row < 0 ? 0 : (row >= a.N_cap ? a.N_cap - 1 : row);
    if (e < ATT_MAX_CHUNK / NW) rows[e] = (int)row;
  }
  wave_lds_order();

  const T* Vhp = static_cast<const T*>(a.V) + (int64_t)hp * a.N_cap * D + col * 8;

  if constexpr (std::is_same<T, bf16>::value) {
    // ---- bf16: both products on the matrix cores ----
    // q K^T: one v_mfma_f32_16x16x32_bf16 per 32-channel slab, A = the 16 token rows of the
    // step, B = the query heads as columns (columns >= G are computed and never looked at).
    // The result leaves lane (head + 16 kg) with the scores of tokens 4 kg + (0..3), so the
    // running max / sum of a head live in the four lanes of its column.
    // P V: these four probabilities are already where the A operand of a 16-token product
    // wants them (row = head = lane % 16, k = token = 4 kg + i), and lane col of group kg
    // holds channels 8 col + (0..7) of exactly these four tokens, which is the B operand of
    // the channel block {8 col + j : col = 0..15} for each j: nothing changes lanes.  The
    // accumulator of block j has the heads 4 kg + i of channel 8 col + j.  A probability
    // enters as the sum of three bf16 numbers, which hold all 24 bits of it: the first two
    // share one product (k = token and part), the third fills both places of another.
    // On the vector ALUs the same step was 32 fused multiply-adds per head, and the four
    // groups had to be added up at the end.
    float m_run = NEG_BIG, l_run = 0.f;                 // of head `col`, identical in its four lanes
    floatx4 acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = {0.f, 0.f, 0.f, 0.f};
    const bf16* Khp = static_cast<const bf16*>(a.K) + (int64_t)hp * a.N_cap * D + col * 8;
    struct Regs { uint4 k[4], v[4]; };
    auto fetch = [&](int t, Regs& r) {                  // group kg: whole rows of tokens 4 kg + (0..3)
      const int4 tr = *reinterpret_cast<const int4*>(rows + t * 16 + kg * 4);
      if constexpr (CACHED) {
        const int64_t base = (int64_t)hp * a.cache.cap * D + col * 8;
        const bf16* Ko = static_cast<const bf16*>(a.cache.K_old) + base;
        const bf16* Vo = static_cast<const bf16*>(a.cache.V_old) + base;
        const int w[4] = {tr.x, tr.y, tr.z, tr.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t at = (int64_t)(w[i] < 0 ? ~w[i] : w[i]) * D;
          r.k[i] = *reinterpret_cast<const uint4*>((w[i] < 0 ? Ko : Khp) + at);
          r.v[i] = *reinterpret_cast<const uint4*>((w[i] < 0 ? Vo : Vhp) + at);
        }
        return;
      }
      r.k[0] = *reinterpret_cast<const uint4*>(Khp + (int64_t)tr.x * D);
      r.k[1] = *reinterpret_cast<const uint4*>(Khp + (int64_t)tr.y * D);
      r.k[2] = *reinterpret_cast<const uint4*>(Khp + (int64_t)tr.z * D);
      r.k[3] = *reinterpret_cast<const uint4*>(Khp + (int64_t)tr.w * D);
      r.v[0] = *reinterpret_cast<const uint4*>(Vhp + (int64_t)tr.x * D);
      r.v[1] = *reinterpret_cast<const uint4*>(Vhp + (int64_t)tr.y * D);
      r.v[2] = *reinterpret_cast<const uint4*>(Vhp + (int64_t)tr.z * D);
      r.v[3] = *reinterpret_cast<const uint4*>(Vhp + (int64_t)tr.w * D);
    };
    auto reduce = [&](int t, const Regs& r) {
      if constexpr (CACHED) {
        const int i0 = t * STEP + wave * 16 + kg * 4;
        const int64_t at = ((int64_t)hp * a.cache.cap + p_begin + i0) * D + col * 8;
        bf16* Kn = static_cast<bf16*>(a.cache.K_new) + at;
        bf16* Vn = static_cast<bf16*>(a.cache.V_new) + at;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i0 + i < n_pos) {
            *reinterpret_cast<uint4*>(Kn + i * D) = r.k[i];
            *reinterpret_cast<uint4*>(Vn + i * D) = r.v[i];
          }
      }
      stage.put(r.k[0], r.k[1], r.k[2], r.k[3]);
      floatx4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int sl = 0; sl < 4; ++sl)
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(stage.operand(sl), qb[sl], d, 0, 0, 0);
      // d[i]: token 4 kg + i against head `col`
      float sc[4];
      const int ibase = t * STEP + wave * 16 + kg * 4;
#pragma unroll
      for (int i = 0; i < 4; ++i) sc[i] = (ibase + i < n_pos) ? d[i] * a.scale_log2e : -INFINITY;
      float mx = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
      mx = xor32(xor16(mx, OpMax()), OpMax());
      mx = fmaxf(mx, m_run);
      const float corr = __builtin_amdgcn_exp2f(m_run - mx);
      m_run = mx;
      float pw[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) pw[i] = __builtin_amdgcn_exp2f(sc[i] - mx);
      float ps = (pw[0] + pw[1]) + (pw[2] + pw[3]);
      ps = xor32(xor16(ps, OpSum()), OpSum());
      l_run = l_run * corr + ps;
      if (t > 0 && __ballot(corr != 1.f)) {             // a new maximum somewhere
        float cr[4];                                    // of heads 4 kg + i
        cr[0] = row_bcast<0>(corr);
        cr[1] = row_bcast<1>(corr);
        cr[2] = row_bcast<2>(corr);
        cr[3] = row_bcast<3>(corr);
        if constexpr (G > 4) {
          const float c4 = row_bcast<4>(corr), c5 = row_bcast<5>(corr);
          const float c6 = row_bcast<6>(corr), c7 = row_bcast<7>(corr);
          cr[0] = kg == 1 ? c4 : cr[0];
          cr[1] = kg == 1 ? c5 : cr[1];
          cr[2] = kg == 1 ? c6 : cr[2];
          cr[3] = kg == 1 ? c7 : cr[3];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[j][i] *= cr[i];
      }
      // p = hi + mid + 2 lo exactly, each with at most 8 significant bits and none of them zero
      // unless p is: zero times an infinite value would be a NaN where the sum has to be
      // infinite.  So hi and mid are what a truncation leaves of the next smaller number, and lo
      // fills both places of the second product.  Below 2^-94 the rest has bits under the
      // smallest bf16 number, 2^-133, which then stands in for it: a token is off by at most
      // 2^-131 times its value, and a probability that underflowed adds nothing.
      // (Constants 2^-126 in place of zero parts would be 0.05 us faster per step, and wrong by
      // up to 12 where a token of probability zero has a value near the largest bf16 number.)
      uint32_t hi[4], mid[4], lo[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t bits = __float_as_uint(pw[i]), least = min(bits, 0x00010000u);
        hi[i] = __builtin_elementwise_sub_sat(bits, 1u);
        const float r1 = pw[i] - __uint_as_float(hi[i] & 0xFFFF0000u);
        mid[i] = max(__builtin_elementwise_sub_sat(__float_as_uint(r1), 1u), least);
        const float r2 = r1 - __uint_as_float(mid[i] & 0xFFFF0000u);
        lo[i] = max(__float_as_int(0.5f * r2), (int)least);   // r2 < 0 where mid stood in for less
      }
      constexpr uint32_t HIGH = 0x07060302u, LOW = 0x05040100u;   // halves of (second, first) word
      const uint32_t lo01 = __builtin_amdgcn_perm(lo[1], lo[0], HIGH);
      const uint32_t lo23 = __builtin_amdgcn_perm(lo[3], lo[2], HIGH);
      const uint4 pa = make_uint4(__builtin_amdgcn_perm(hi[1], hi[0], HIGH),
                                  __builtin_amdgcn_perm(hi[3], hi[2], HIGH),
                                  __builtin_amdgcn_perm(mid[1], mid[0], HIGH),
                                  __builtin_amdgcn_perm(mid[3], mid[2], HIGH));
      const uint4 pb = make_uint4(lo01, lo23, lo01, lo23);
      uint32_t vw[4][4] = {{r.v[0].x, r.v[0].y, r.v[0].z, r.v[0].w},
                           {r.v[1].x, r.v[1].y, r.v[1].z, r.v[1].w},
                           {r.v[2].x, r.v[2].y, r.v[2].z, r.v[2].w},
                           {r.v[3].x, r.v[3].y, r.v[3].z, r.v[3].w}};
      if (t * STEP + wave * 16 + 16 > n_pos) {          // wave-uniform: the row that stands in for a
#pragma unroll                                          // position beyond the end is not looked at
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int w = 0; w < 4; ++w) vw[i][w] = ibase + i < n_pos ? vw[i][w] : 0u;
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t b01 = __builtin_amdgcn_perm(vw[1][j / 2], vw[0][j / 2], j & 1 ? HIGH : LOW);
        const uint32_t b23 = __builtin_amdgcn_perm(vw[3][j / 2], vw[2][j / 2], j & 1 ? HIGH : LOW);
        const bf16x8 vb = __builtin_bit_cast(bf16x8, make_uint4(b01, b23, b01, b23));
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pa), vb, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pb), vb, acc[j], 0, 0, 0);
      }
    };
    // NS register sets in rotation: the loads of steps t + 1 .. t + NS - 1 are in flight
    // while step t is reduced (4 and 6 sets were measured: no faster, the row stream is
    // bound by memory bandwidth, not by the depth of the prefetch)
    constexpr int NS = 3;
    Regs rs[NS];
#pragma unroll
    for (int j = 0; j < NS - 1; ++j)
      if (j < n_steps) fetch(j, rs[j]);
    for (int t = 0; t < n_steps; t += NS) {
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        if (t + j < n_steps) {
          if (t + j + NS - 1 < n_steps) fetch(t + j + NS - 1, rs[(j + NS - 1) % NS]);
          reduce(t + j, rs[j]);
        }
      }
    }
    wave_lds_order();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int g = kg * 4 + i;
      if (g < G) {
        float* r = red + wave * RED_STRIDE + g * PART_STRIDE + 2 + col * 8;
#pragma unroll
        for (int j = 0; j < 8; j += 2) *reinterpret_cast<float2*>(r + j) = make_float2(acc[j][i], acc[j + 1][i]);
      }
    }
    if (lane < G)
      *reinterpret_cast<float2*>(red + wave * RED_STRIDE + lane * PART_STRIDE) = make_float2(m_run, l_run);
  } else {
    // ---- fp32 check mode: dot products on the vector ALUs ----
    float acc[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[g][j] = 0.f;
    // this lane's 8 channels of every query head of the group, pre-scaled
    float qv[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      load_row8<T>(q + ((int64_t)s * a.Hq + h * G + g) * D + col * 8, qv[g]);
#pragma unroll
      for (int j = 0; j < 8; ++j) qv[g][j] *= a.scale_log2e;
    }

    float m[G], l[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      m[g] = NEG_BIG;
      l[g] = 0.f;
    }

    const T* Khp = static_cast<const T*>(a.K) + (int64_t)hp * a.N_cap * D + col * 8;
    RawRow<T> kc[4], vc[4], kn[4], vn[4];
    auto fetch = [&](int t, RawRow<T>(&kr)[4], RawRow<T>(&vr)[4]) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t row = rows[t * 16 + kg * 4 + u];
        kr[u].load(Khp + row * D);
        vr[u].load(Vhp + row * D);
      }
    };
    if (n_steps > 0) fetch(0, kc, vc);
    for (int t = 0; t < n_steps; ++t) {
      if (t + 1 < n_steps) fetch(t + 1, kn, vn);
      float kv[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) kc[u].unpack(kv[u]);
      float sc[G][4];
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float d = 0.f;
#pragma unroll
          for (int j = 0; j < 8; ++j) d = fmaf(qv[g][j], kv[u][j], d);
          d = row16_sum(d);
          sc[g][u] = (t * STEP + wave * 16 + kg * 4 + u < n_pos) ? d : -INFINITY;
        }
      float pw[G][4];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float mx = m[g];
#pragma unroll
        for (int u = 0; u < 4; ++u) mx = fmaxf(mx, sc[g][u]);
        const float corr = __builtin_amdgcn_exp2f(m[g] - mx);
        m[g] = mx;
        float ls = l[g] * corr;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[g][j] *= corr;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          pw[g][u] = __builtin_amdgcn_exp2f(sc[g][u] - mx);
          ls += pw[g][u];
        }
        l[g] = ls;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float vv[8];
        vc[u].unpack(vv);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int j = 0; j < 8; ++j) acc[g][j] = fmaf(pw[g][u], vv[j], acc[g][j]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        kc[u] = kn[u];
        vc[u] = vn[u];
      }
    }

    if constexpr (FUSED) __syncthreads();               // the selection's LDS is free
    // ---- combine the 4 groups of a wavefront (lanes col + 16*k) ----
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float mx = xor32(xor16(m[g], OpMax()), OpMax());
      const float w = __builtin_amdgcn_exp2f(m[g] - mx);
      const float ls = xor32(xor16(l[g] * w, OpSum()), OpSum());
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[g][j] = xor32(xor16(acc[g][j] * w, OpSum()), OpSum());
      if (lane < 16) {
        float* r = red + wave * RED_STRIDE + g * PART_STRIDE;
        r[0] = mx;
        r[1] = ls;
#pragma unroll
        for (int j = 0; j < 8; ++j) r[2 + col * 8 + j] = acc[g][j];
      }
    }
  }
  __syncthreads();
  // ---- combine the wavefronts, in order: thread = (query head g, channel pair) ----
  T* out = static_cast<T*>(a.out);
  float* part_hp = a.part + (int64_t)hp * a.n_split * G * PART_STRIDE;
  for (int e = tid; e < G * (D / 2); e += NT) {
    const int g = e / (D / 2), c2 = (e % (D / 2)) * 2;
    float2 ml[NW];
    float mx = NEG_BIG;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      ml[w] = *reinterpret_cast<const float2*>(red + w * RED_STRIDE + g * PART_STRIDE);
      mx = fmaxf(mx, ml[w].x);
    }
    float ls = 0.f, a0 = 0.f, a1 = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = __builtin_amdgcn_exp2f(ml[w].x - mx);
      const float2 av = *reinterpret_cast<const float2*>(red + w * RED_STRIDE + g * PART_STRIDE + 2 + c2);
      ls = fmaf(ml[w].y, f, ls);
      a0 = fmaf(av.x, f, a0);
      a1 = fmaf(av.y, f, a1);
    }
    if (a.n_split == 1) {
      const float inv = ls > 0.f ? 1.0f / ls : 0.f;
      T* o = out + ((int64_t)s * a.Hq + h * G + g) * D + c2;
      store_out(o, a0 * inv);
      store_out(o + 1, a1 * inv);
    } else {
      float* pr = part_hp + ((int64_t)split * G + g) * PART_STRIDE;
      if (a.two_pass) {
        if (c2 == 0) *reinterpret_cast<float2*>(pr) = make_float2(mx, ls);
        *reinterpret_cast<float2*>(pr + 2 + c2) = make_float2(a0, a1);
      } else {
        if (c2 == 0) put_pair_agent(pr, mx, ls);
        put_pair_agent(pr + 2 + c2, a0, a1);
      }
    }
  }
  if (a.n_split == 1 || a.two_pass) return;

  // ---- ticket: the last workgroup of the head-problem to get here merges ----
  // Every thread waits until its stores above have been acknowledged (they are
  // agent-scope stores: performed where every XCD looks) before it passes the barrier;
  // only then is the ticket drawn.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (tid == 0) {
    // Idle state of a ticket word: TICKET_MAGIC in the upper 48 bits, count 0.  One
    // fetch-add draws the ticket.  A word that does not carry the mark (memory this
    // library has never used: the first launch on a fresh workspace) is taken over with
    // a compare-and-swap loop instead; whoever added to it before the take-over adds
    // itself again through the same loop, so every workgroup is counted exactly once.
    unsigned long long* tk = a.tickets + hp;
    unsigned long long old =
        __hip_atomic_fetch_add(tk, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long now = old + 1;
    if ((old >> 16) != TICKET_MAGIC) {
      unsigned long long seen = now;
      do {
        now = (seen >> 16) == TICKET_MAGIC ? seen + 1 : ((TICKET_MAGIC << 16) | 1ull);
      } while (!__hip_atomic_compare_exchange_strong(tk, &seen, now, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    const int last = (int)(now & 0xFFFFull) == a.n_split;
    // back to idle: ready for the next launch (or a replay of this one from a graph)
    if (last) __hip_atomic_store(tk, TICKET_MAGIC << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = last;
  }
  __syncthreads();
  if (!s_last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  for (int e = tid; e < G * (D / 2); e += NT) {
    const int g = e / (D / 2), c2 = (e % (D / 2)) * 2;
    const float2 o2 = merge_splits(part_hp + (int64_t)g * PART_STRIDE, (int64_t)G * PART_STRIDE,
                                   a.n_split, c2, PairAgent());
    T* o = out + ((int64_t)s * a.Hq + h * G + g) * D + c2;
    store_out(o, o2.x);
    store_out(o + 1, o2.y);
  }
}

// Second pass of the two-pass form: the same merge, by a kernel of its own.
template <typename T>
__global__ __launch_bounds__(D / 2) void k_attn_merge(const float* __restrict__ part, int n_split,
                                                      int G, int Hq, int Hkv, T* __restrict__ out) {
  const int hq_lin = blockIdx.x;                        // s * Hq + hq
  const int s = hq_lin / Hq, hq = hq_lin % Hq;
  const int hp = s * Hkv + hq / G, g = hq % G, c2 = threadIdx.x * 2;
  const float* base = part + (((int64_t)hp * n_split) * G + g) * PART_STRIDE;
  const float2 o2 = merge_splits(base, (int64_t)G * PART_STRIDE, n_split, c2, PairPlain());
  store_out(out + (int64_t)hq_lin * D + c2, o2.x);
  store_out(out + (int64_t)hq_lin * D + c2 + 1, o2.y);
}

// How a call is spread over the chip.  All forms of the step take the same rule: the split
// boundaries fix the order of the fp32 sums, and they must give the same bits.
//
// All splits of a head-problem run on one XCD (those that launch_attn_t spreads are counted the same),
// ceil(HP / 8) head-problems share it, and the registers allow two wavefronts per SIMD: 32 workgroups of eight wavefronts or 64 of four are
// resident on an XCD together.  One more and it runs its whole chain -- scoring, selection, rows
// -- after the others are through, so a call takes as many splits as fit in ONE round:
//  - eight wavefronts if they do: every phase is spread over the whole CU and fewer splits
//    have to be merged;
//  - four, two workgroups per CU, where the row table (2048 positions a workgroup) asks for
//    more splits than eight allow;
//  - eight again where that is not enough either: the contexts are long and the row stream is
//    all that counts;
//  - above 256 head-problems workgroups follow each other anyway: four wavefronts, one
//    workgroup selecting while the other streams, and three splits up to 320, where whole
//    head-problems would leave half of the places empty.
// (The figures are from before the partials lost a barrier, 0.1 to 0.3 us on either side.)
// Microseconds of the fused step, eight / four wavefronts, each at its best number of splits of
// one round, and [eight wavefronts with ceil(256 / HP) splits, which is a second round for a few]:
//   HP            8           24           40           56           88           120
//   B = 1024  10.5 / 10.7  11.0 / 11.6  12.7 / 13.4  14.1 / 14.7  18.5 / 19.1  20.4 / 20.9
//                [10.5]       [11.1]       [13.3]       [18.4]       [23.1]       [29.2]
//   B = 2048  11.7 / 12.0  13.4 / 14.0  16.6 / 17.6  19.1 / 19.7  26.5 / 27.2  31.2 / 31.6
//                [11.7]       [14.3]       [19.7]       [22.0]       [32.0]       [42.1]
//   HP           160          256          320          512         1024         2048
//   B = 1024  23.7 / 24.4  30.5 / 31.9  49.4 / 43.8  62.6 / 57.4  122  / 109   231  / 205
//   B = 2048  39.0 / 37.2  55.2 / 56.3  88.4 / 81.9  115  / 110   215  / 205
//                [32.7, 49.2]     (two rounds and more of eight wavefronts from HP = 257 on)
// Four wavefronts, one / two / three splits: HP = 264: 38.3 / 40.1 / 37.3 and 71.8 / 69.2 / 61.8,
// 320: 41.5 / 42.6 / 41.7 and 77.5 / 76.0 / 73.5, 352: 43.4 / 45.9 / 46.1 and 82.3 / 82.5 / 87.5;
// full attention over 2048 tokens at HP = 264: 57.9 / 54.8 / 48.8, 352: 65.2 / 68.1 / 69.4.
// Full attention over 32864 tokens, eight / four: 8: 27.0 / 27.0, 12: 42.4 / 39.7, 24: 80.7 / 78.7;
// 32: 104.5 / 113.2 and 40: 129.9 / 134.1 are more than one round either way.
// Spread splits (HP < 8, long rows) would find 256 places for eight wavefronts, not 32 per head-problem,
// but more of them have to be merged.  Full attention, this rule / 256 / HP splits: 1 x 8192 tokens
// 9.2 / 10.8, 1 x 32864 16.8 / 20.8, 1 x 131072 37.2 / 37.6, 4 x 8192 10.8 / 14.2, 4 x 131072 56.2 /
// 55.7, 7 x 32864 27.8 / 29.2, and ahead only at 3 x 50000 27.0 / 25.4 and 7 x 131072 97.3 / 92.5.
// Two steps of eight wavefronts (129 to 256 positions) go to one workgroup, which writes the output
// itself: a second step takes 0.9 us, publishing and merging two partials takes longer.  Two splits /
// one, B = 256, 51 clusters: HP = 8 7.88 / 7.65, 32 8.0 / 7.75, 128 8.2 / 7.97; a list of 256 rows: HP = 8
// 5.64 / 5.38, 128 6.12 / 5.73.  Below six head-problems it is two workgroups all the same: the cached
// step takes the same rule, and one compute unit does not ask the host link for enough rows (four steps
// of B = 256: HP = 2 58.3 / 63.9, 4 68.9 / 70.5, 6 81.6 / 79.9, 8 94.1 / 92.0, 64 449 / 424).
// Four steps as two splits of two are slower than four of one (8.4 / 7.2).
struct AttnPlan {
  int waves;        // wavefronts per workgroup
  int max_splits;   // grows with the attended total: a workspace sized for more holds less
  int chunk;        // positions of a split, whole steps of the workgroup
  int n_split;      // splits that have positions (not monotone in the attended total)
};
static AttnPlan attn_plan(const Dims& dm, int64_t max_total) {
  const int64_t per_xcd = (dm.HP + N_XCD - 1) / N_XCD;  // head-problems of the fullest XCD
  int64_t need = (max_total + ATT_MAX_CHUNK - 1) / ATT_MAX_CHUNK;
  if (need < 1) need = 1;
  AttnPlan p;
  int64_t n;
  if (dm.dtype == CK_F32) {                             // check mode: one workgroup per CU
    p.waves = 4;
    n = (N_XCD * ATT_XCD_CUS + dm.HP - 1) / dm.HP;
    if (n > 64) n = 64;
  } else if (per_xcd * need <= ATT_XCD_CUS) {
    p.waves = 8;
    n = ATT_XCD_CUS / per_xcd;
  } else if (per_xcd > ATT_XCD_CUS) {
    p.waves = 4;
    n = per_xcd <= ATT_XCD_CUS + 8 ? 3 : 1;
  } else if (per_xcd * need <= 2 * ATT_XCD_CUS) {
    p.waves = 4;
    n = 2 * ATT_XCD_CUS / per_xcd;
  } else {
    p.waves = 8;
    n = need;
  }
  // at least one full step of tokens per workgroup, no more positions than its row table holds
  const int64_t step = p.waves * ATT_TOKENS, by_work = (max_total + step - 1) / step;
  if (n > by_work) n = by_work;
  if (p.waves == 8 && by_work == 2 && dm.HP >= 6) n = 1;
  if (n < need) n = need;
  p.max_splits = (int)n;
  // whole steps, and no split without a position: it would score and select for nothing
  int64_t chunk = ((max_total + n - 1) / n + step - 1) / step * step;
  if (chunk < step) chunk = step;
  n = (max_total + chunk - 1) / chunk;
  p.chunk = (int)chunk;
  p.n_split = n < 1 ? 1 : (int)n;
  return p;
}

// The workspace: one 64-bit ticket word per head-problem, whose place must not depend on the
// number of splits, then the split partials.
static size_t ticket_bytes(const Dims& dm) {
  return ((size_t)dm.HP * sizeof(unsigned long long) + 255) & ~(size_t)255;
}

size_t attn_workspace_bytes(const Dims& dm, int64_t max_total) {
  const size_t b =
      (size_t)dm.HP * attn_plan(dm, max_total).max_splits * dm.G * PART_STRIDE * sizeof(float);
  return ticket_bytes(dm) + ((b + 255) & ~(size_t)255);
}

template <typename T, int MODE, int CMAX, int NW, bool CACHED>
static void launch_attn_waves(int G, dim3 grid, const AttnArgs& a, hipStream_t st) {
  const dim3 block(NW * 64);
  switch (G) {
    case 1: hipLaunchKernelGGL((k_attn<T, 1, MODE, CMAX, NW, CACHED>), grid, block, 0, st, a); break;
    case 2: hipLaunchKernelGGL((k_attn<T, 2, MODE, CMAX, NW, CACHED>), grid, block, 0, st, a); break;
    case 4: hipLaunchKernelGGL((k_attn<T, 4, MODE, CMAX, NW, CACHED>), grid, block, 0, st, a); break;
    default: hipLaunchKernelGGL((k_attn<T, 8, MODE, CMAX, NW, CACHED>), grid, block, 0, st, a); break;
  }
}

template <typename T, int MODE, int CMAX, bool CACHED = false>
static hipError_t launch_attn_t(const Dims& dm, AttnArgs a, int64_t max_total, void* workspace,
                                bool two_pass, hipStream_t st) {
  const AttnPlan plan = attn_plan(dm, max_total);
  const int n_split = plan.n_split;
  if (n_split > ATT_MAX_SPLITS || plan.chunk > ATT_MAX_CHUNK) return hipErrorInvalidValue;
  if (dm.G != 1 && dm.G != 2 && dm.G != 4 && dm.G != 8) return hipErrorInvalidValue;
  a.chunk = plan.chunk;
  a.n_split = n_split;
  a.two_pass = two_pass ? 1 : 0;
  a.HP = dm.HP;
  a.tickets = reinterpret_cast<unsigned long long*>(workspace);
  a.part = reinterpret_cast<float*>(static_cast<char*>(workspace) + ticket_bytes(dm));
  const int hp_groups = (dm.HP + N_XCD - 1) / N_XCD;
  // Fewer head-problems than XCDs, no table to share and long rows: the splits of a head-problem go
  // over all XCDs, whose share of the memory's rate is the limit otherwise.  Full attention, one XCD
  // each / spread: 1 x 32864 tokens 21.6 / 16.7 us, 4 x 131072 79.2 / 55.6, 4 x 8192 14.4 / 12.8,
  // but 2 x 2048 5.2 / 5.4 (the merge reads what another XCD wrote), a list of 256 rows 5.8 / 6.1.
  a.spread = MODE == ATT_PLAIN && dm.HP < N_XCD && max_total > 2 * ATT_MAX_CHUNK;
  const dim3 grid((unsigned)(a.spread ? dm.HP : hp_groups * N_XCD) * n_split);
  if constexpr (std::is_same<T, bf16>::value) {
    if (plan.waves == 8)
      launch_attn_waves<T, MODE, CMAX, 8, CACHED>(dm.G, grid, a, st);
    else
      launch_attn_waves<T, MODE, CMAX, 4, CACHED>(dm.G, grid, a, st);
  } else {
    launch_attn_waves<T, MODE, CMAX, 4, CACHED>(dm.G, grid, a, st);
  }
  if (n_split > 1 && two_pass)
    hipLaunchKernelGGL(k_attn_merge<T>, dim3(dm.S * dm.Hq), dim3(D / 2), 0, st, a.part, n_split,
                       dm.G, dm.Hq, dm.Hkv, (T*)a.out);
  return hipGetLastError();
}

static AttnArgs common_args(const Dims& dm, const void* q, const void* K, const void* V,
                            int idx_stride, int max_tokens, int64_t n_sink, int64_t recent_begin,
                            int64_t recent_end, float softmax_scale, void* out) {
  AttnArgs a = {};
  a.q = q;
  a.K = K;
  a.V = V;
  a.out = out;
  a.idx_stride = idx_stride;
  a.max_tokens = max_tokens;
  a.Hq = dm.Hq;
  a.Hkv = dm.Hkv;
  a.C_cap = dm.C_cap;
  a.N_cap = dm.N_cap;
  a.n_sink = (int)n_sink;
  a.recent_begin = recent_begin;
  a.n_recent = (int)(recent_end > recent_begin ? recent_end - recent_begin : 0);
  a.scale_log2e = softmax_scale * 1.4426950408889634f;
  return a;
}

hipError_t launch_sparse_attn(const Dims& dm, const void* q, const void* K, const void* V,
                              const int32_t* token_idx, const int32_t* n_tokens, int idx_stride,
                              int64_t max_total, int64_t n_sink, int64_t recent_begin,
                              int64_t recent_end, float softmax_scale, void* out, void* workspace,
                              bool two_pass, hipStream_t st) {
  const int n_recent = (int)(recent_end > recent_begin ? recent_end - recent_begin : 0);
  AttnArgs a = common_args(dm, q, K, V, idx_stride, (int)(max_total - n_sink - n_recent), n_sink,
                           recent_begin, recent_end, softmax_scale, out);
  a.token_idx = token_idx;
  a.n_tokens = n_tokens;
  if (dm.dtype == CK_BF16)
    return launch_attn_t<bf16, ATT_PLAIN, SELP_SMALL>(dm, a, max_total, workspace, two_pass, st);
  return launch_attn_t<float, ATT_PLAIN, SELP_SMALL>(dm, a, max_total, workspace, two_pass, st);
}

hipError_t launch_decode_fused(const Dims& dm, const void* q, const void* K, const void* V,
                               const void* centroids, const int32_t* sizes,
                               const int32_t* offsets, const int32_t* sorted_idx, int n_clusters,
                               int budget, uint32_t flags, int64_t n_sink, int64_t recent_begin,
                               int64_t recent_end, float softmax_scale, float* scores,
                               int32_t* sel_clusters, int32_t* n_sel_clusters,
                               int32_t* n_sel_tokens, int32_t* token_idx, int idx_stride,
                               int32_t* n_tokens, void* out, void* workspace, hipStream_t st) {
  AttnArgs a = common_args(dm, q, K, V, idx_stride, budget, n_sink, recent_begin, recent_end,
                           softmax_scale, out);
  a.centroids = centroids;
  a.scores = scores;
  a.sizes = sizes;
  a.offsets = offsets;
  a.sorted_idx = sorted_idx;
  a.sel_clusters = sel_clusters;
  a.n_sel_clusters = n_sel_clusters;
  a.n_sel_tokens = n_sel_tokens;
  a.token_idx_out = token_idx;
  a.n_tokens_out = n_tokens;
  a.n_clusters = n_clusters;
  a.budget = budget;
  a.trim = (int)(flags & CK_SEL_TRIM_LAST);
  const int64_t max_total = (int64_t)budget + n_sink + a.n_recent;
  if (dm.dtype == CK_BF16 && n_clusters <= SELP_SMALL)  // one launch for the whole step
    return launch_attn_t<bf16, ATT_FUSED_SCORE, SELP_SMALL>(dm, a, max_total, workspace, false, st);
  const hipError_t e = launch_score(dm, q, centroids, n_clusters, scores, st);
  if (e != hipSuccess) return e;
  if (dm.dtype == CK_BF16)
    return launch_attn_t<bf16, ATT_FUSED, CK_MAX_CLUSTERS>(dm, a, max_total, workspace, false, st);
  if (n_clusters <= SELP_SMALL)
    return launch_attn_t<float, ATT_FUSED, SELP_SMALL>(dm, a, max_total, workspace, false, st);
  return launch_attn_t<float, ATT_FUSED, CK_MAX_CLUSTERS>(dm, a, max_total, workspace, false, st);
}

hipError_t launch_cached_step(const Dims& dm, const void* q, const void* centroids,
                              int n_clusters, int budget, float softmax_scale, float* scores,
                              int32_t* sel_clusters, int32_t* n_sel_clusters,
                              int32_t* n_sel_tokens, const CacheArgs& cache, void* out,
                              void* workspace, hipStream_t st) {
  AttnArgs a = common_args(dm, q, cache.K_home, cache.V_home, 0, budget, 0, 0, 0, softmax_scale, out);
  a.centroids = centroids;
  a.scores = scores;
  a.sizes = cache.sizes;
  a.offsets = cache.offsets;
  a.sorted_idx = cache.sorted_idx;
  a.sel_clusters = sel_clusters;
  a.n_sel_clusters = n_sel_clusters;
  a.n_sel_tokens = n_sel_tokens;
  a.n_clusters = n_clusters;
  a.budget = budget;
  a.cache = cache;
  if (n_clusters <= SELP_SMALL)
    return launch_attn_t<bf16, ATT_FUSED_SCORE, SELP_SMALL, true>(dm, a, budget, workspace, false, st);
  const hipError_t e = launch_score(dm, q, centroids, n_clusters, scores, st);
  if (e != hipSuccess) return e;
  return launch_attn_t<bf16, ATT_FUSED, CK_MAX_CLUSTERS, true>(dm, a, budget, workspace, false, st);
}

// ---- library-owned scratch for callers that cannot allocate ----
// The split partials and tickets of one attention call, in device memory that exists
// from the moment the code object is loaded: every GPU the library runs on holds its
// own copy of the array until the process ends.  Host code never passes the array's
// name anywhere; it asks the runtime once per device for the array's address on
// that device and uses that pointer from then on.
static __device__ __align__(256) unsigned char scratch[CK_STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[MAX_DEVICES];                // address of `scratch` per device

hipError_t attn_static_scratch(void** ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace ck
