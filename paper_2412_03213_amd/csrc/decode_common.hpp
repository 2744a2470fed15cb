// Device code shared by the decode-step kernels: loading rows of the storage type
// and the selection of the recalled cluster prefix (paper Section III-C and the
// size gather / prefix sum of Section IV-C, Fig. 8).
#pragma once
#include "ck_common.hpp"

namespace ck {

template <typename T>
__device__ __forceinline__ void load_row8(const T* p, float (&v)[8]);
template <>
__device__ __forceinline__ void load_row8<bf16>(const bf16* p, float (&v)[8]) {
  const uint4 w = *reinterpret_cast<const uint4*>(p);
  v[0] = lo_bf16(w.x); v[1] = hi_bf16(w.x); v[2] = lo_bf16(w.y); v[3] = hi_bf16(w.y);
  v[4] = lo_bf16(w.z); v[5] = hi_bf16(w.z); v[6] = lo_bf16(w.w); v[7] = hi_bf16(w.w);
}
template <>
__device__ __forceinline__ void load_row8<float>(const float* p, float (&v)[8]) {
  const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// ---- cluster / row scores of a bf16 table on the matrix cores ----
// s_r = sum_g <q_g, row_r> for 16 consecutive table rows per wavefront step:
// v_mfma_f32_16x16x32_bf16 with the query heads of the group as the rows of A (rows >= G
// repeat head 0, see below) and the 16 table rows as the columns of B.  Lane l < 16 then holds, for table
// row l of the step, the four heads 0..3 in its four accumulators (lanes 16..31: heads
// 4..7), so the sum over the heads is three in-lane additions (one lane exchange more for
// G = 8) and the 16 scores leave the wavefront as one 64-byte store.  Every caller that
// scores a bf16 table goes through these two functions, so that the separate scoring
// kernel and the fused decode kernel produce bit-identical scores.
// The query heads as a 16 x 32 MFMA operand per slab: lane l holds head l%16, channels
// 32*sl + 8*(l/16) .. +8.  Heads >= G do not exist: their lanes re-read head 0 (always a
// valid address) and whatever the matrix cores compute for them is never looked at --
// rows (or columns) of an MFMA result do not mix.
__device__ __forceinline__ void load_query_operand(const bf16* __restrict__ q_group, int G,
                                                   int lane, bf16x8 (&qb)[4]) {
  const int col = lane & 15, kg = lane >> 4;
  const bf16* p = q_group + (int64_t)(col < G ? col : 0) * D + kg * 8;
#pragma unroll
  for (int sl = 0; sl < 4; ++sl)
    qb[sl] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p + sl * 32));
}
// Sixteen rows of a table (or of K) as an MFMA operand.  The operand wants lane l to hold
// channels 32*sl + 8*(l/16) .. +8 of row l%16, and loading it that way makes every lane of a
// quarter wavefront touch another row: the address unit then spends about 64 cycles on a
// 1 KB instruction instead of 16 (400 rows by one workgroup: 3.0 us against 1.0 us,
// whether they come from L2 or from memory).  So 16 lanes load one whole 256-byte row --
// lane l the 16 bytes l%16 of row 4*(l/16) + i of the step, i = 0..3 -- and the rows change
// lanes through a wavefront-private piece of LDS (row stride 272 B: no bank conflicts).
constexpr int STAGE_ROW = D + 8;                          // bf16 elements per staged row
constexpr int STAGE_ELEMS = 16 * STAGE_ROW;               // of one wavefront
struct Stage16 {
  uint4* w;                                               // this lane's place in the rows it loaded
  const uint4* r;                                         // and in the row it is the operand lane of
  __device__ __forceinline__ Stage16(bf16* stage, int lane)
      : w(reinterpret_cast<uint4*>(stage + 4 * (lane >> 4) * STAGE_ROW + (lane & 15) * 8)),
        r(reinterpret_cast<const uint4*>(stage + (lane & 15) * STAGE_ROW + (lane >> 4) * 8)) {}
  // LDS serves one wavefront in order: the reads see the writes, and the next writes wait
  __device__ __forceinline__ void put(uint4 a, uint4 b, uint4 c, uint4 d) const {
    wave_lds_order();
    w[0] = a;
    w[STAGE_ROW / 8] = b;
    w[2 * (STAGE_ROW / 8)] = c;
    w[3 * (STAGE_ROW / 8)] = d;
    wave_lds_order();
  }
  __device__ __forceinline__ bf16x8 operand(int sl) const {
    return __builtin_bit_cast(bf16x8, r[4 * sl]);
  }
};
// Of the 16 staged table rows; returns in lanes 0..15 the score of row `lane`.
__device__ __forceinline__ float score_rows16(const Stage16& st, const bf16x8 (&qb)[4], int G) {
  floatx4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int sl = 0; sl < 4; ++sl)
    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qb[sl], st.operand(sl), d, 0, 0, 0);
  // accumulator i of lanes 0..15 is head i, of lanes 16..31 head 4 + i
  float v = d[0];
  if (G >= 2) v += d[1];
  if (G >= 4) v = v + (d[2] + d[3]);
  if (G == 8) v = xor16(v, OpSum());
  return v;
}

// Monotone map float -> uint32 (a < b  <=>  map(a) < map(b); -0 and +0 made equal).
__device__ __forceinline__ uint32_t ordered_bits(float f) {
  if (f == 0.f) f = 0.f;                                    // -0 -> +0
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int SELP_BINS = 256;
constexpr int SELP_MAX_CAND = 512;         // more candidates than this: rank all clusters
constexpr int SELP_SMALL = 512;            // cluster bound of the small instantiation

// LDS of select_many by NT threads, sized for at most CMAX clusters (512 or
// CK_MAX_CLUSTERS: the launcher picks the smallest that holds the table, so that a few
// hundred clusters do not reserve the LDS of two thousand and more workgroups fit a CU).
// Afterwards ord[j] and cum[j] for j < n_sel describe the recalled clusters in score order
// (cum = inclusive prefix sum of their sizes); their offsets are cbeg[j], or soff[ord[j]] if full_rank.
template <int CMAX, int NT>
struct alignas(16) SelectLds {
  static_assert(CMAX % NT == 0 && CMAX >= SELP_MAX_CAND, "cluster bound");
  uint32_t key[CMAX];              // ~ordered(score): ascending key = descending score
  int ssz[CMAX], soff[CMAX];       // size and offset; all three per candidate, or per cluster (full_rank)
  int cand[SELP_MAX_CAND];         // candidate cluster ids (compacted, any order)
  int ord[CMAX];                   // cluster id per sorted position
  int cum[CMAX];                   // inclusive prefix sum of sizes per sorted position
  int cbeg[SELP_MAX_CAND];         // offset per sorted position (not full_rank)
  int tmp[NT / WAVE + 1];
  int n_sel, n_tok, counter, full_rank;
};

// ---- the usual selection: a recalled prefix bounded by at most 64 candidates ----
// Every phase is spread over the workgroup and the three barriers are all there is: binning
// of the scores (all threads), the bin where the budget is crossed (every wavefront for
// itself), compaction of the candidates (all threads), their ranks (64 / NW candidates
// per wavefront, NW lanes each), and the prefix sum over the ranked sizes (every wavefront for
// itself, in registers, where the resolution of positions to token rows reads it).
// One wavefront doing all of it, without barriers, took 2.6 us at 400 clusters: a long chain
// of dependent instructions with nothing to issue in between.
template <int NT>
struct alignas(16) QuickLds {
  unsigned long long bin[SELP_BINS];       // sizes of the clusters of a bin | their number << 32
  unsigned long long ckey[WAVE];           // candidates: key << 32 | cluster id, any order
  int csz[WAVE], coff[WAVE];               // their sizes and offsets
  int ord[WAVE], osz[WAVE], ooff[WAVE];    // cluster id, size and offset by rank
  float mx[NT / WAVE], mn[NT / WAVE];      // score range seen by every wavefront
  int n_app;
};
// What a wavefront knows afterwards: lane j holds the cluster of rank j (j < m).
struct Quick {
  int m, last_bin;                         // candidates: the clusters of bins up to last_bin;
                                           // m > 64: nothing selected, go on with select_many
  int n_sel, n_tok;                        // recalled clusters and tokens
  int id, size, off, cum;                  // of rank `lane`; cum = inclusive prefix sum of sizes
};

// Before the score range and the first barrier.
template <int NT>
__device__ __forceinline__ void quick_clear(QuickLds<NT>& Q) {
  for (int b = threadIdx.x; b < SELP_BINS; b += NT) Q.bin[b] = 0ull;
  if (threadIdx.x < WAVE) Q.ckey[threadIdx.x] = ~0ull;   // padding that never ranks before anything
  if (threadIdx.x == 0) Q.n_app = 0;
}
// Score range of this wavefront's clusters, into Q; a workgroup barrier has to follow.
template <int NT>
__device__ __forceinline__ void quick_range(QuickLds<NT>& Q, float mx, float mn) {
  mx = wave_max(mx);
  mn = wave_min(mn);
  if ((threadIdx.x & 63) == 0) {
    Q.mx[threadIdx.x >> 6] = mx;
    Q.mn[threadIdx.x >> 6] = mn;
  }
}
// Bin of a score: monotone, a larger score never lands in a later bin.  (Any positive factor gives
// a valid binning; the clamp takes care of its rounding.)
struct ScoreBins {
  float smax, inv;
  template <int NT>
  __device__ __forceinline__ explicit ScoreBins(const QuickLds<NT>& Q) {
    smax = Q.mx[0];
    float smin = Q.mn[0];
#pragma unroll
    for (int w = 1; w < NT / WAVE; ++w) {
      smax = fmaxf(smax, Q.mx[w]);
      smin = fminf(smin, Q.mn[w]);
    }
    const float span = smax - smin;
    inv = span > 0.f ? (float)(SELP_BINS - 1) * __builtin_amdgcn_rcpf(span) : 0.f;
  }
  __device__ __forceinline__ int operator()(float score) const {
    const int b = (int)((smax - score) * inv);
    return b < 0 ? 0 : (b > SELP_BINS - 1 ? SELP_BINS - 1 : b);
  }
};
// Recalled prefix under `budget` of the clusters by descending score (ties: lower id first):
//   trim == 0: longest prefix whose sizes sum to <= budget;
//   trim == 1: shortest prefix whose sizes sum to >= budget (all if the total is smaller).
// sc, sz, of: score, size, offset of cluster tid + i * NT.  Ends without a barrier.
template <int NT, int ITEMS>
__device__ __forceinline__ Quick quick_select(QuickLds<NT>& Q, const float (&sc)[ITEMS],
                                              const int (&sz)[ITEMS], const int (&of)[ITEMS], int C,
                                              int budget, int trim) {
  constexpr int NW = NT / WAVE;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const ScoreBins bins(Q);
  int bin[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int b = bins(sc[i]);
    const bool ok = tid + i * NT < C;
    bin[i] = ok ? b : SELP_BINS;                        // never a candidate
    if (ok) atomicAdd(&Q.bin[b], (1ull << 32) | (uint32_t)sz[i]);
  }
  __syncthreads();
  // first bin at which the running size crosses the budget; everything up to and including
  // it is a candidate
  constexpr int PER = SELP_BINS / WAVE;
  int ss[PER], nn[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const unsigned long long v = Q.bin[lane * PER + i];
    ss[i] = (int)(uint32_t)v + (i ? ss[i - 1] : 0);
    nn[i] = (int)(v >> 32) + (i ? nn[i - 1] : 0);
  }
  const int sbase = wave_inclusive_scan(ss[PER - 1]) - ss[PER - 1];
  const int nbase = wave_inclusive_scan(nn[PER - 1]) - nn[PER - 1];
  int first = SELP_BINS, ncand = 0;
#pragma unroll
  for (int i = PER - 1; i >= 0; --i) {
    const int cs = sbase + ss[i];
    if (trim ? cs >= budget : cs > budget) {
      first = lane * PER + i;
      ncand = nbase + nn[i];
    }
  }
  Quick r;
  const uint64_t crossing = __ballot(first < SELP_BINS);
  r.last_bin = SELP_BINS - 1;
  r.m = C;                                              // no crossing: every cluster is recalled
  if (crossing) {
    const int src = __builtin_ctzll(crossing);          // lowest lane = lowest bin
    r.last_bin = __builtin_amdgcn_readlane(first, src);
    r.m = __builtin_amdgcn_readlane(ncand, src);
  }
  r.n_sel = r.n_tok = 0;
  r.id = r.size = r.off = r.cum = 0;
  if (r.m > WAVE) return r;                             // the same in every wavefront
  const uint64_t lt = ((uint64_t)1 << lane) - 1;
  uint64_t mask[ITEMS];
  int total = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    mask[i] = __ballot(bin[i] <= r.last_bin);
    total += __popcll(mask[i]);
  }
  if (total) {                                          // wave-uniform
    int base = 0;
    if (lane == 0) base = atomicAdd(&Q.n_app, total);
    base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      if (bin[i] <= r.last_bin) {
        const int pos = base + __popcll(mask[i] & lt);
        Q.ckey[pos] = ((unsigned long long)~ordered_bits(sc[i]) << 32) | (uint32_t)(tid + i * NT);
        Q.csz[pos] = sz[i];
        Q.coff[pos] = of[i];
      }
      base += __popcll(mask[i]);
    }
  }
  __syncthreads();
  // rank among the candidates: ascending key = descending score, ties to the lower id
  {
    constexpr int PW = WAVE / NW;                       // candidates of this wavefront, NW lanes each
    const int c = wave * PW + lane / NW, part = lane % NW;
    if (wave * PW < r.m) {                              // wave-uniform
      const unsigned long long kc = Q.ckey[c];
      const int size = Q.csz[c], off = Q.coff[c];
      int rank = 0;
#pragma unroll
      for (int i = 0; i < PW; ++i) rank += Q.ckey[part * PW + i] < kc ? 1 : 0;
      // over the NW lanes of a candidate (4 or 8, inside one row of 16)
      rank += __builtin_amdgcn_update_dpp(0, rank, DPP_XOR1, 0xf, 0xf, false);
      rank += __builtin_amdgcn_update_dpp(0, rank, DPP_XOR2, 0xf, 0xf, false);
      if (NW == 8) rank += __builtin_amdgcn_update_dpp(0, rank, DPP_HALF_MIRROR, 0xf, 0xf, false);
      if (part == 0 && c < r.m) {
        Q.ord[rank] = (int)(uint32_t)kc;
        Q.osz[rank] = size;
        Q.ooff[rank] = off;
      }
    }
  }
  __syncthreads();
  const bool in_m = lane < r.m;
  r.id = in_m ? Q.ord[lane] : 0;
  r.size = in_m ? Q.osz[lane] : 0;
  r.off = in_m ? Q.ooff[lane] : 0;
  r.cum = wave_inclusive_scan(r.size);
  const bool in = in_m && (trim ? (r.cum < budget) : (r.cum <= budget));
  r.n_sel = __popcll(__ballot(in));
  if (trim) r.n_sel = r.n_sel + 1 < r.m ? r.n_sel + 1 : r.m;
  r.n_tok = r.n_sel > 0 ? __builtin_amdgcn_readlane(r.cum, r.n_sel - 1) : 0;
  if (trim && r.n_tok > budget) r.n_tok = budget;
  return r;
}

// ---- more candidates than lanes of a wavefront (budgets of many small clusters, scores that are
// all equal, a budget beyond the total) ----
// Goes on from the histogram of quick_select: m > 64 candidates, the clusters of bins up to last_bin.
// Bound: LDS latency of the ranking loop.  With a histogram of its own, ck_select_clusters took 13.6 us
// at 8 head-problems, 1600 clusters and about 100 recalled ones, 12.4 without; the fused step 20.4, 19.0.
// (The few bins are computed anew: handing them over costs the usual path 0.06 us.)
// Up to SELP_MAX_CAND of them are compacted and ranked among themselves, more are ranked with
// every cluster.  Must be called by all NT threads; ends with a barrier.
template <int CMAX, int NT>
__device__ __forceinline__ void select_many(SelectLds<CMAX, NT>& L, QuickLds<NT>& Q,
                                            const float (&sc)[CMAX / NT],
                                            const int (&sz)[CMAX / NT],
                                            const int (&of)[CMAX / NT], int m, int last_bin,
                                            int C, int budget, int trim) {
  constexpr int SELP_ITEMS = CMAX / NT;
  const int tid = threadIdx.x;
  if (tid == 0) L.counter = 0;
  if (m <= SELP_MAX_CAND) {
    // ---- compact the candidates, then rank them among themselves ----
    const ScoreBins bins(Q);
#pragma unroll
    for (int i = 0; i < SELP_ITEMS; ++i) {
      if (tid + i * NT < C && bins(sc[i]) <= last_bin) {
        const int pos = atomicAdd(&Q.n_app, 1);  // not used by quick_select in this case
        L.cand[pos] = tid + i * NT;
        L.key[pos] = ~ordered_bits(sc[i]);
        L.ssz[pos] = sz[i];
        L.soff[pos] = of[i];
      }
    }
    const int m_pad = (m + 3) & ~3;
    if (tid < m_pad - m) {                       // padding that never ranks before anything
      L.cand[m + tid] = 0x7FFFFFFF;
      L.key[m + tid] = 0xFFFFFFFFu;
    }
    __syncthreads();
    for (int i = tid; i < m; i += NT) {
      const int c = L.cand[i];
      const uint32_t kc = L.key[i];
      const int size = L.ssz[i], off = L.soff[i];
      int rank = 0;
      for (int j = 0; j < m_pad; j += 4) {
        const uint4 k4 = *reinterpret_cast<const uint4*>(&L.key[j]);
        const int4 c4 = *reinterpret_cast<const int4*>(&L.cand[j]);
        rank += (k4.x < kc || (k4.x == kc && c4.x < c)) ? 1 : 0;
        rank += (k4.y < kc || (k4.y == kc && c4.y < c)) ? 1 : 0;
        rank += (k4.z < kc || (k4.z == kc && c4.z < c)) ? 1 : 0;
        rank += (k4.w < kc || (k4.w == kc && c4.w < c)) ? 1 : 0;
      }
      L.ord[rank] = c;
      L.cum[rank] = size;
      L.cbeg[rank] = off;
    }
  } else {
    // ---- rank every cluster ----
#pragma unroll
    for (int i = 0; i < SELP_ITEMS; ++i) {
      const int c = tid + i * NT;
      if (c < C) {
        L.key[c] = ~ordered_bits(sc[i]);
        L.ssz[c] = sz[i];
        L.soff[c] = of[i];
      }
    }
    const int n_pad = (C + 3) & ~3;
    for (int j = C + tid; j < n_pad; j += NT) L.key[j] = 0xFFFFFFFFu;
    __syncthreads();
    for (int c = tid; c < C; c += NT) {
      const uint32_t kc = L.key[c];
      int rank = 0;
      for (int j = 0; j < n_pad; j += 4) {
        const uint4 k4 = *reinterpret_cast<const uint4*>(&L.key[j]);
        rank += (k4.x < kc || (k4.x == kc && j + 0 < c)) ? 1 : 0;
        rank += (k4.y < kc || (k4.y == kc && j + 1 < c)) ? 1 : 0;
        rank += (k4.z < kc || (k4.z == kc && j + 2 < c)) ? 1 : 0;
        rank += (k4.w < kc || (k4.w == kc && j + 3 < c)) ? 1 : 0;
      }
      L.ord[rank] = c;
      L.cum[rank] = L.ssz[c];
    }
  }
  __syncthreads();
  // ---- inclusive prefix sum of the sizes in score order, and the recalled count ----
  int v[SELP_ITEMS];
#pragma unroll
  for (int i = 0; i < SELP_ITEMS; ++i) {
    const int j = tid * SELP_ITEMS + i;
    v[i] = j < m ? L.cum[j] : 0;
  }
  block_inclusive_scan<SELP_ITEMS>(v, L.tmp);
  int cnt = 0;
#pragma unroll
  for (int i = 0; i < SELP_ITEMS; ++i) {
    const int j = tid * SELP_ITEMS + i;
    if (j < m) {
      cnt += trim ? (v[i] < budget) : (v[i] <= budget);
      L.cum[j] = v[i];
    }
  }
  if (cnt) atomicAdd(&L.counter, cnt);
  __syncthreads();
  if (tid == 0) {
    int n_sel = L.counter;
    if (trim) n_sel = n_sel + 1 < m ? n_sel + 1 : m;
    int n_tok = n_sel > 0 ? L.cum[n_sel - 1] : 0;
    if (trim && n_tok > budget) n_tok = budget;
    L.n_sel = n_sel;
    L.n_tok = n_tok;
    L.full_rank = m > SELP_MAX_CAND;
  }
  __syncthreads();
}

}  // namespace ck
