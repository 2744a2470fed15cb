// K-means initialisation, clustering metadata and centroid update
// (paper Section III-B for init/update, Section IV-C / Fig. 8 for the metadata).
//
// The paper's update kernel accumulates keys into shared-memory sums with
// atomics, one thread block per head.  Here the update is a segmented
// reduction instead: the assignment leaves every chunk of tokens sorted by label, and
// one workgroup per cluster walks the chunks' runs, streams its member rows and adds
// them in a fixed order (ascending token row).  No floating-point atomics, so the
// centroids are bit-reproducible.  The cluster-contiguous index that the decode step
// needs (sizes, prefix sum, sorted indices) is emitted once, from the chunk index of the
// last assignment.  Short ranges do without the index: their update looks through the labels, and
// its last launch leaves the metadata.  The counting sort of given labels and the update from a
// sorted list serve the calls that export the steps, and ranges of more chunks than the index holds.
#include <type_traits>

#include "chunk_sort.hpp"

namespace ck {

// ------------------------------------------------------------------ init
// centroid c of head-problem hp := key row init_idx[hp][c]; also the row of the table the
// assignment reads: its unit-length copy (cosine) or the row itself (l2, inner product),
// and for l2 the bias -|row|^2 / 2.  In run-until-convergence mode n_changed rows of `changed` are
// cleared here (a launch of its own for that took 2 us).
__global__ __launch_bounds__(64) void k_init_centroids(
    const bf16* __restrict__ K, const int32_t* __restrict__ init_idx, int64_t N_cap, int C_cap,
    int c_begin, int c_count, bf16* __restrict__ centroids, bf16* __restrict__ mu_hat, int metric,
    float* __restrict__ bias, int bias_stride, int32_t* __restrict__ changed, int n_changed) {
  const int c = blockIdx.x, hp = blockIdx.y, lane = threadIdx.x;
  if (changed && c == 0)
    for (int t = lane; t < n_changed; t += WAVE) changed[(int64_t)t * gridDim.y + hp] = 0;
  int64_t row = init_idx[(int64_t)hp * c_count + c];
  row = row < 0 ? 0 : (row >= N_cap ? N_cap - 1 : row);
  const uint32_t w = reinterpret_cast<const uint32_t*>(K + ((int64_t)hp * N_cap + row) * D)[lane];
  const float a = lo_bf16(w), b = hi_bf16(w);
  const float n2 = wave_sum(a * a + b * b);
  const float inv = n2 > 0.f ? 1.0f / sqrtf(n2) : 0.f;
  reinterpret_cast<uint32_t*>(centroids + ((int64_t)hp * C_cap + c_begin + c) * D)[lane] = w;
  const uint32_t h = (uint32_t)float_to_bf16_bits(a * inv) |
                     ((uint32_t)float_to_bf16_bits(b * inv) << 16);
  reinterpret_cast<uint32_t*>(mu_hat + ((int64_t)hp * c_count + c) * D)[lane] =
      metric == CK_METRIC_COSINE ? h : w;
  if (metric == CK_METRIC_L2 && lane == 0) bias[(int64_t)hp * bias_stride + c] = -0.5f * n2;
}

__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

// iterations a head-problem ran: up to and including the first assignment that changed
// no label, or all of them; by one wavefront
__device__ __forceinline__ int iterations_run(const int32_t* __restrict__ changed, int max_iter, int HP, int hp) {
  const int lane = threadIdx.x & 63;
  for (int t0 = 1; t0 < max_iter; t0 += WAVE) {
    const int t = t0 + lane;
    const uint64_t still = __ballot(t < max_iter && changed[(int64_t)min(t, max_iter - 1) * HP + hp] == 0);
    if (still) return t0 + __builtin_ctzll(still) + 1;
  }
  return max_iter;
}

__global__ __launch_bounds__(64) void k_iters_done(const int32_t* __restrict__ changed, int max_iter,
                                                   int32_t* __restrict__ iters_done) {
  const int n = iterations_run(changed, max_iter, gridDim.x, blockIdx.x);
  if (threadIdx.x == 0) iters_done[blockIdx.x] = n;
}

hipError_t launch_iters_done(const int32_t* changed, int max_iter, int HP, int32_t* iters_done,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_iters_done, dim3(HP), dim3(64), 0, st, changed, max_iter, iters_done);
  return hipGetLastError();
}

hipError_t launch_init_centroids(const Dims& dm, const bf16* K, const int32_t* init_idx,
                                 int c_begin, int c_count, bf16* centroids, bf16* mu_hat,
                                 int metric, float* bias, int bias_stride, int32_t* changed,
                                 int n_changed, hipStream_t st) {
  hipLaunchKernelGGL(k_init_centroids, dim3(c_count, dm.HP), dim3(64), 0, st, K, init_idx,
                     dm.N_cap, dm.C_cap, c_begin, c_count, centroids, mu_hat, metric, bias,
                     bias_stride, changed, n_changed);
  return hipGetLastError();
}

// ------------------------------------------------------------------ counting sort
constexpr int SORT_THREADS = 256;                       // 4 wavefronts, one chunk each

// Pass 1 (only when the assignment kernel has not already produced it): label
// histogram of every chunk of `chunk_tokens` consecutive tokens.
__global__ __launch_bounds__(SORT_THREADS) void k_sort_hist(
    const int32_t* __restrict__ labels, int64_t N_cap, int64_t tok_begin, int64_t tok_count,
    int c_begin, int c_count, int label_bits, int n_chunks, int chunk_tokens,
    uint32_t* __restrict__ seg) {
  extern __shared__ int lds_hist[];                     // [4][c_count]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, hp = blockIdx.y;
  const int chunk = blockIdx.x * 4 + wave;
  if (chunk >= n_chunks) return;                        // whole wavefront leaves; no barriers below
  volatile int* hist = lds_hist + wave * c_count;
  for (int c = lane; c < c_count; c += WAVE) hist[c] = 0;
  __builtin_amdgcn_wave_barrier();
  const int32_t* lab = labels + (int64_t)hp * N_cap + tok_begin;
  const uint64_t lt = ((uint64_t)1 << lane) - 1;
  for (int r = 0; r < chunk_tokens / WAVE; ++r) {
    const int64_t t = (int64_t)chunk * chunk_tokens + r * WAVE + lane;
    const bool valid = t < tok_count;
    int l = valid ? lab[t] - c_begin : 0;
    l = l < 0 ? 0 : (l >= c_count ? c_count - 1 : l);   // never index outside the table
    const uint64_t peers = same_label_mask(l, valid, label_bits);
    if (valid && (peers & lt) == 0) hist[l] = hist[l] + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
  }
  uint32_t* out = seg + ((int64_t)hp * n_chunks + chunk) * seg_stride(c_count);
  for (int c = lane; c < c_count; c += WAVE) out[c] = (uint32_t)hist[c] << 16;
}

// Pass 2: per cluster, exclusive scan of the chunk counts (upper halves of seg; the
// sums replace the words) and the cluster size.  Workgroup = 64 clusters x 16 groups of chunks.
constexpr int SCAN_THREADS = 1024;
constexpr int SCAN_GROUPS = SCAN_THREADS / 64;
constexpr int SCAN_REG = 16;                            // chunk counts a thread keeps in registers
__global__ __launch_bounds__(SCAN_THREADS) void k_sort_scan(
    uint32_t* __restrict__ seg, int n_chunks, int C_cap, int c_begin, int c_count,
    int32_t* __restrict__ sizes, const int32_t* __restrict__ gate) {
  __shared__ int part[SCAN_GROUPS][64];
  const int cl = threadIdx.x & 63, grp = threadIdx.x >> 6, hp = blockIdx.y;
  if (gate && gate[hp] == 0) return;
  const int c = blockIdx.x * 64 + cl;
  const int per = (n_chunks + SCAN_GROUPS - 1) / SCAN_GROUPS;
  const int k0 = grp * per, k1 = min(k0 + per, n_chunks);
  const int stride = seg_stride(c_count);
  uint32_t* H = seg + (int64_t)hp * n_chunks * stride + c;
  int v[SCAN_REG];
  int sum = 0;
  if (c < c_count) {
    // unconditional loads, looked at when all are under way: with the shift in the condition each
    // waits for the one before (300000 tokens, 400 clusters: the scan took 17.6 us, now 12.8)
#pragma unroll
    for (int i = 0; i < SCAN_REG; ++i) v[i] = (int)H[(int64_t)min(k0 + i, n_chunks - 1) * stride];
#pragma unroll
    for (int i = 0; i < SCAN_REG; ++i) v[i] = k0 + i < k1 ? (int)((uint32_t)v[i] >> 16) : 0;
#pragma unroll
    for (int i = 0; i < SCAN_REG; ++i) sum += v[i];
    for (int k = k0 + SCAN_REG; k < k1; ++k) sum += (int)(H[(int64_t)k * stride] >> 16);
  }
  part[grp][cl] = sum;
  __syncthreads();
  int run = 0, total = 0;
#pragma unroll
  for (int g = 0; g < SCAN_GROUPS; ++g) {
    const int t = part[g][cl];
    if (g < grp) run += t;
    total += t;
  }
  if (c < c_count) {
#pragma unroll
    for (int i = 0; i < SCAN_REG; ++i)
      if (k0 + i < k1) {
        H[(int64_t)(k0 + i) * stride] = (uint32_t)run;
        run += v[i];
      }
    for (int k = k0 + SCAN_REG; k < k1; ++k) {
      const int t = (int)(H[(int64_t)k * stride] >> 16);
      H[(int64_t)k * stride] = (uint32_t)run;
      run += t;
    }
    if (grp == 0) sizes[(int64_t)hp * C_cap + c_begin + c] = total;
  }
}

// Pass 3: exclusive scan of the sizes -> offsets (every workgroup recomputes it in
// LDS, the first one of a head-problem stores it), then the stable scatter of the
// token rows of ONE chunk to their sorted positions.  The four wavefronts each rank a
// quarter of the chunk; per-wavefront label counts in LDS order the quarters.
constexpr int OFF_ITEMS = CK_MAX_CLUSTERS / SORT_THREADS;   // 8 clusters per thread
constexpr int SCAT_ROUNDS = 2;                              // chunk_tokens <= 4 * 2 * 64
__global__ __launch_bounds__(SORT_THREADS) void k_sort_scatter(
    const int32_t* __restrict__ labels, int64_t N_cap, int64_t tok_begin, int64_t tok_count,
    int C_cap, int c_begin, int c_count, int label_bits, int n_chunks, int chunk_tokens,
    const uint32_t* __restrict__ seg, const int32_t* __restrict__ sizes,
    int32_t* __restrict__ offsets, int32_t* __restrict__ sorted_idx,
    const int32_t* __restrict__ gate) {
  extern __shared__ int lds_hist[];                     // [c_count] positions + [4][c_count] counts
  __shared__ int tmp[SORT_THREADS / WAVE + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hp = blockIdx.y;
  if (gate && gate[hp] == 0) return;
  const int chunk = blockIdx.x;
  // this thread's labels are requested first, unconditionally (a token beyond the range
  // re-reads token 0), so that they travel while the offsets are being prepared
  const int per_wave = chunk_tokens / 4;
  const int32_t* lab = labels + (int64_t)hp * N_cap + tok_begin;
  int lraw[SCAT_ROUNDS];
#pragma unroll
  for (int r = 0; r < SCAT_ROUNDS; ++r) {
    const int in_wave = r * WAVE + lane;
    const int64_t t = (int64_t)chunk * chunk_tokens + wave * per_wave + in_wave;
    lraw[r] = lab[(in_wave < per_wave && t < tok_count) ? t : 0];
  }
  int* offs = lds_hist;
  int* cnt = lds_hist + c_count;
  int32_t* off_g = offsets + (int64_t)hp * (C_cap + 1);
  const int base0 = c_begin == 0 ? 0 : off_g[c_begin];
  const uint32_t* cbase = seg + ((int64_t)hp * n_chunks + chunk) * seg_stride(c_count);
  {
    const int32_t* sz = sizes + (int64_t)hp * C_cap + c_begin;
    int v[OFF_ITEMS], own[OFF_ITEMS], cb[OFF_ITEMS];
#pragma unroll
    for (int i = 0; i < OFF_ITEMS; ++i) {
      const int c = tid * OFF_ITEMS + i;
      own[i] = v[i] = c < c_count ? sz[c] : 0;
      cb[i] = c < c_count ? (int)cbase[c] : 0;
    }
    block_inclusive_scan<OFF_ITEMS>(v, tmp);
#pragma unroll
    for (int i = 0; i < OFF_ITEMS; ++i) {
      const int c = tid * OFF_ITEMS + i;
      if (c < c_count) {
        offs[c] = base0 + v[i] - own[i] + cb[i];        // first position of this chunk's tokens
        if (chunk == 0) off_g[c_begin + c + 1] = base0 + v[i];
      }
    }
    if (chunk == 0 && tid == 0 && c_begin == 0) off_g[0] = 0;
  }
  for (int i = tid; i < 4 * c_count; i += SORT_THREADS) cnt[i] = 0;
  __syncthreads();

  const uint64_t lt = ((uint64_t)1 << lane) - 1;
  volatile int* mine = cnt + wave * c_count;
  int lbl[SCAT_ROUNDS], rank[SCAT_ROUNDS];
  int64_t tok[SCAT_ROUNDS];
#pragma unroll
  for (int r = 0; r < SCAT_ROUNDS; ++r) {
    const int in_wave = r * WAVE + lane;
    const int64_t t = (int64_t)chunk * chunk_tokens + wave * per_wave + in_wave;
    const bool valid = in_wave < per_wave && t < tok_count;
    int l = valid ? lraw[r] - c_begin : 0;
    l = l < 0 ? 0 : (l >= c_count ? c_count - 1 : l);
    const uint64_t peers = same_label_mask(l, valid, label_bits);
    const int before = mine[l];
    __builtin_amdgcn_wave_barrier();
    if (valid && (peers & lt) == 0) mine[l] = before + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
    lbl[r] = l;
    rank[r] = before + __popcll(peers & lt);
    tok[r] = valid ? t : -1;
  }
  __syncthreads();
  int32_t* out = sorted_idx + (int64_t)hp * N_cap;
#pragma unroll
  for (int r = 0; r < SCAT_ROUNDS; ++r) {
    if (tok[r] >= 0) {
      int pos = offs[lbl[r]] + rank[r];
      for (int w = 0; w < wave; ++w) pos += cnt[w * c_count + lbl[r]];
      if (pos >= 0 && pos < N_cap) out[pos] = (int32_t)(tok_begin + tok[r]);
    }
  }
}

hipError_t launch_metadata(const Dims& dm, const int32_t* labels, int64_t tok_begin,
                           int64_t tok_count, int c_begin, int c_count, int32_t* sizes,
                           int32_t* offsets, int32_t* sorted_idx, const ChunkIndex& chunks,
                           bool have_seg, const int32_t* gate, hipStream_t st) {
  uint32_t* seg = chunks.seg;
  const int chunk_tokens = chunks.tokens;
  const int n_chunks = (int)((tok_count + chunk_tokens - 1) / chunk_tokens);
  int label_bits = 0;
  while ((1 << label_bits) < c_count) ++label_bits;
  const dim3 grid((n_chunks + 3) / 4, dm.HP);
  if (!have_seg)
    hipLaunchKernelGGL(k_sort_hist, grid, dim3(SORT_THREADS), (size_t)4 * c_count * sizeof(int),
                       st, labels, dm.N_cap, tok_begin, tok_count, c_begin, c_count, label_bits,
                       n_chunks, chunk_tokens, seg);
  hipLaunchKernelGGL(k_sort_scan, dim3((c_count + 63) / 64, dm.HP), dim3(SCAN_THREADS), 0, st,
                     seg, n_chunks, dm.C_cap, c_begin, c_count, sizes, gate);
  hipLaunchKernelGGL(k_sort_scatter, dim3(n_chunks, dm.HP), dim3(SORT_THREADS),
                     (size_t)5 * c_count * sizeof(int), st, labels, dm.N_cap, tok_begin, tok_count,
                     dm.C_cap, c_begin, c_count, label_bits, n_chunks, chunk_tokens, seg,
                     sizes, offsets, sorted_idx, gate);
  return hipGetLastError();
}

// ------------------------------------------------------------------ update
// One wavefront turns the member sums of channels 2*lane, 2*lane+1 into the stored mean,
// the table row of the next assignment and, for l2, its bias.
__device__ __forceinline__ void store_mean(float m0, float m1, int n, int hp, int c, int C_cap,
                                           int c_begin, int c_count, bf16* __restrict__ centroids,
                                           bf16* __restrict__ mu_hat,
                                           float* __restrict__ centroids_f32, int metric,
                                           float* __restrict__ bias, int bias_stride) {
  const int lane = threadIdx.x & 63;
  const float inv_n = 1.0f / (float)n;
  m0 *= inv_n;
  m1 *= inv_n;
  // written as one fused multiply-add: left to the compiler, its choice of the fused product
  // (and with it the last bit of the norm) would depend on the kernel this is inlined into
  const float n2 = wave_sum(fmaf(m1, m1, m0 * m0));
  const float inv = n2 > 0.f ? 1.0f / sqrtf(n2) : 0.f;
  const int64_t crow = (int64_t)hp * C_cap + c_begin + c;
  const int64_t hrow = (int64_t)hp * c_count + c;
  const uint32_t raw =
      (uint32_t)float_to_bf16_bits(m0) | ((uint32_t)float_to_bf16_bits(m1) << 16);
  reinterpret_cast<uint32_t*>(centroids + crow * D)[lane] = raw;
  // table row of the next assignment: unit length (cosine) or the stored mean itself
  reinterpret_cast<uint32_t*>(mu_hat + hrow * D)[lane] =
      metric == CK_METRIC_COSINE
          ? ((uint32_t)float_to_bf16_bits(m0 * inv) | ((uint32_t)float_to_bf16_bits(m1 * inv) << 16))
          : raw;
  if (metric == CK_METRIC_L2) {                         // wave-uniform
    const float r0 = lo_bf16(raw), r1 = hi_bf16(raw);   // the rounded row is what gets compared
    const float rn2 = wave_sum(fmaf(r1, r1, r0 * r0));
    if (lane == 0) bias[(int64_t)hp * bias_stride + c] = -0.5f * rn2;
  }
  if (centroids_f32)
    reinterpret_cast<float2*>(centroids_f32 + hrow * D)[lane] = make_float2(m0, m1);
}

// One workgroup per cluster.  A 16-lane group reads one member row per step
// (16 B per lane), 4 rows per wavefront step, UPD_UNR steps in flight.  Partial
// sums are combined in a fixed order: lane groups of a wavefront, then the
// wavefronts through LDS.
template <int UPD_WAVES, int UPD_UNR>
__global__ __launch_bounds__(UPD_WAVES * 64) void k_update(
    const bf16* __restrict__ K, int64_t N_cap, int C_cap, const int32_t* __restrict__ offsets,
    const int32_t* __restrict__ sorted_idx, int c_begin, int c_count,
    bf16* __restrict__ centroids, bf16* __restrict__ mu_hat, float* __restrict__ centroids_f32,
    int metric, float* __restrict__ bias, int bias_stride, const int32_t* __restrict__ gate) {
  constexpr int GROUPS = UPD_WAVES * 4;                 // 16-lane groups: member rows per step
  __shared__ float part[UPD_WAVES][D];
  const int c = blockIdx.x, hp = blockIdx.y, tid = threadIdx.x;
  if (gate && gate[hp] == 0) return;
  const int lane = tid & 63, wave = tid >> 6, l16 = tid & 15, grp = tid >> 4;
  const int32_t* off = offsets + (int64_t)hp * (C_cap + 1) + c_begin + c;
  const int beg = off[0], n = off[1] - beg;
  if (n <= 0) return;                                   // empty cluster keeps its centroid
  const int32_t* idx = sorted_idx + (int64_t)hp * N_cap + beg;
  const bf16* Khp = K + (int64_t)hp * N_cap * D + l16 * 8;

  float acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.f;
  for (int j0 = 0; j0 < n; j0 += GROUPS * UPD_UNR) {
    // two round trips per pass: all member ids, then all member rows.  Every load is
    // unconditional (an entry beyond the cluster re-reads its last member and is
    // replaced by zeros): a load under a branch makes the compiler wait for it, and for
    // everything requested before it, ahead of the next one.
    int64_t row[UPD_UNR];
#pragma unroll
    for (int u = 0; u < UPD_UNR; ++u) {
      const int j = j0 + u * GROUPS + grp;
      row[u] = idx[j < n ? j : n - 1];
    }
    uint4 w[UPD_UNR];
#pragma unroll
    for (int u = 0; u < UPD_UNR; ++u) {
      const int64_t r = row[u] < 0 ? 0 : (row[u] >= N_cap ? N_cap - 1 : row[u]);
      w[u] = *reinterpret_cast<const uint4*>(Khp + r * D);
    }
#pragma unroll
    for (int u = 0; u < UPD_UNR; ++u) {
      const bool real = j0 + u * GROUPS + grp < n;
      const uint32_t x = real ? w[u].x : 0u, y = real ? w[u].y : 0u;
      const uint32_t z = real ? w[u].z : 0u, q = real ? w[u].w : 0u;
      acc[0] += lo_bf16(x); acc[1] += hi_bf16(x);
      acc[2] += lo_bf16(y); acc[3] += hi_bf16(y);
      acc[4] += lo_bf16(z); acc[5] += hi_bf16(z);
      acc[6] += lo_bf16(q); acc[7] += hi_bf16(q);
    }
  }
  // groups of one wavefront
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    acc[j] += __shfl_xor(acc[j], 16, WAVE);
    acc[j] += __shfl_xor(acc[j], 32, WAVE);
  }
  if (lane < 16) {
#pragma unroll
    for (int j = 0; j < 8; ++j) part[wave][l16 * 8 + j] = acc[j];
  }
  __syncthreads();
  if (tid < 64) {
    // lane handles channels 2*lane, 2*lane+1
    float m0 = part[0][2 * lane], m1 = part[0][2 * lane + 1];
#pragma unroll
    for (int wv = 1; wv < UPD_WAVES; ++wv) {
      m0 += part[wv][2 * lane];
      m1 += part[wv][2 * lane + 1];
    }
    store_mean(m0, m1, n, hp, c, C_cap, c_begin, c_count, centroids, mu_hat, centroids_f32, metric,
               bias, bias_stride);
  }
}

hipError_t launch_update(const Dims& dm, const bf16* K, const int32_t* offsets,
                         const int32_t* sorted_idx, int c_begin, int c_count, bf16* centroids,
                         bf16* mu_hat, float* centroids_f32, int metric, float* bias,
                         int bias_stride, const int32_t* gate, hipStream_t st) {
  // four wavefronts, eight rows in flight per 16-lane group: measured best of
  // {1, 2, 4 wavefronts} x {4, 8, 16 in flight} (the summation order does not depend on it)
  hipLaunchKernelGGL((k_update<4, 8>), dim3(c_count, dm.HP), dim3(4 * 64), 0, st, K, dm.N_cap,
                     dm.C_cap, offsets, sorted_idx, c_begin, c_count, centroids, mu_hat,
                     centroids_f32, metric, bias, bias_stride, gate);
  return hipGetLastError();
}

// ------------------------------------------------------------------ from the chunk index
// The assignment leaves every chunk's tokens ordered by label (ChunkIndex), so the members of
// a cluster in ascending token order are its runs of chunk 0, chunk 1, ...: no sorted list is
// needed to sum them.  A wavefront scans the run lengths of its cluster over the chunks and
// finds the run that holds the j-th member by binary search in LDS.
struct ChunkRuns {
  const uint32_t* seg;
  const uint16_t* list;
  int n_chunks, chunk_tokens;
  int64_t tok_count;

  const uint32_t* runs;         // this cluster's words of seg, by chunk (LDS)
  const int* upto;              // members up to and including a chunk (LDS)
  const uint16_t* list_hp;
  int n;                        // members

  // All threads of the workgroup; ends with a barrier.  The words of clusters c0 .. c0 + CL,
  // then cluster c0 + cl for this wavefront (the wavefronts of one cluster do the same scan).
  template <int CL, int THREADS>
  __device__ __forceinline__ void stage(uint32_t* lds, int hp, int c0, int cl, int c_count) {
    load<CL, THREADS>(lds, hp, c0, c_count);
    scan(lds, hp, cl);
  }
  template <int CL, int THREADS>
  __device__ __forceinline__ void load(uint32_t* lds, int hp, int c0, int c_count) const {
    constexpr int BATCH = 4;
    const int tid = threadIdx.x;
    const int cpad = (n_chunks + 63) & ~63, stride = seg_stride(c_count);
    const uint32_t* S = seg + (int64_t)hp * n_chunks * stride;
    for (int e0 = tid; e0 < cpad * CL; e0 += BATCH * THREADS) {
      uint32_t v[BATCH];
#pragma unroll
      for (int i = 0; i < BATCH; ++i) {                 // unconditional: one round trip
        const int k = (e0 + i * THREADS) / CL, w = e0 % CL;   // neighbouring clusters share a line
        const bool ok = k < n_chunks && c0 + w < c_count;
        v[i] = S[ok ? (int64_t)k * stride + c0 + w : 0];
        v[i] = ok ? v[i] : 0u;
      }
#pragma unroll
      for (int i = 0; i < BATCH; ++i) {
        const int k = (e0 + i * THREADS) / CL, w = e0 % CL;
        if (k < cpad) lds[(size_t)w * 2 * cpad + k] = v[i];
      }
    }
    __syncthreads();
  }
  __device__ __forceinline__ void scan(uint32_t* lds, int hp, int cl) {
    const int lane = threadIdx.x & 63, cpad = (n_chunks + 63) & ~63;
    uint32_t* r = lds + (size_t)cl * 2 * cpad;
    int* u = reinterpret_cast<int*>(r + cpad);
    n = 0;
    for (int k0 = 0; k0 < cpad; k0 += WAVE) {
      const int v = wave_inclusive_scan((int)(r[k0 + lane] >> 16)) + n;
      u[k0 + lane] = v;
      n = __builtin_amdgcn_readlane(v, WAVE - 1);
    }
    runs = r;
    upto = u;
    list_hp = list + (int64_t)hp * n_chunks * chunk_tokens;
    wave_lds_order();
  }
  // token (offset in the range) of member j, clamped to the last one; n > 0
  __device__ __forceinline__ int member(int j) const {
    j = j < n ? j : n - 1;
    int lo = 0, hi = n_chunks - 1;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (upto[mid] > j) hi = mid; else lo = mid + 1;
    }
    const uint32_t r = runs[lo];
    int at = (int)(r & 0xFFFFu) + j - (upto[lo] - (int)(r >> 16));
    at = at < 0 ? 0 : (at >= chunk_tokens ? chunk_tokens - 1 : at);
    const int64_t t = (int64_t)lo * chunk_tokens + list_hp[(int64_t)lo * chunk_tokens + at];
    return (int)(t < tok_count ? t : tok_count - 1);    // never outside the keys
  }
};

// Update: one workgroup per CL neighbouring clusters, wavefront w summing members 16 s + 4 w + (0..3) of every
// step s, 128 rows in flight.  The additions run in k_update's order (16 member streams, the
// four of a wavefront, then the wavefronts), so both give the same bits.
// Bound: launch, two dependent look-ups (runs, list) and the rows at memory speed.  It takes
// the place of a scan, a scatter and k_update, of which none has enough to do to hide its own
// start; per iteration, assignment included: 8 head-problems x 32768 tokens x 400 clusters
// 53.3 -> 47.0 us (reading those keys once: 10.4 us), 64 x 8163 x 102 58.5 -> 52.3,
// 8 x 131072 x 1600 407 -> 399, 8 x 2985 x 37 15.8 -> 9.9.  One wavefront per cluster with
// four accumulator sets (one to eight clusters per workgroup) is within 2 % on the large
// shapes and 3 us slower on the small one; two wavefronts per cluster are slower everywhere.
// Four clusters share the lines of the run table (a cluster uses 4 bytes of each: lines of 420 MB
// for 13 MB of words at 8 x 131072 x 1600) and one's rows travel while the next one's members
// are looked up; see update_clusters_per_workgroup for where that pays.
constexpr int UPC_WAVES = 4;
constexpr int UPC_STEPS = 8;                            // 16-row steps whose loads are in flight together

template <int CL, bool LOOK>
__global__ __launch_bounds__(UPC_WAVES * 64, CL == 1 ? 7 : 6) void k_update_chunks(
    const bf16* __restrict__ K, const uint32_t* __restrict__ seg,
    const uint16_t* __restrict__ list, int n_chunks, int chunk_tokens, int64_t N_cap,
    int64_t tok_begin, int64_t tok_count, int C_cap, int c_begin, int c_count,
    bf16* __restrict__ centroids, bf16* __restrict__ mu_hat, int32_t* __restrict__ sizes,
    int metric, float* __restrict__ bias, int bias_stride, const TileMap map) {
  constexpr int SPAN = 256;                             // members whose ids a workgroup holds at once
  extern __shared__ uint32_t lds_u[];
  __shared__ __attribute__((aligned(16))) float part[CL][UPC_WAVES][D];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, g4 = lane >> 4;
  int wg, hp;                                           // neighbouring clusters, whose run words share
  if (!map.mine<false, LOOK>(wg, hp)) return;           // cache lines, are on one XCD
  const int c0 = wg * CL;
  CK_FETCH_ARG(centroids);                              // used last, fetched with the others
  CK_FETCH_ARG(metric);
  ChunkRuns cr[CL];
#pragma unroll
  for (int cl = 0; cl < CL; ++cl) cr[cl] = {seg, list, n_chunks, chunk_tokens, tok_count};
  cr[0].template load<CL, UPC_WAVES * 64>(lds_u, hp, c0, c_count);
  if (map.stopped<LOOK>(hp)) return;                          // here the word has travelled with the table
#pragma unroll
  for (int cl = 0; cl < CL; ++cl) {
    cr[cl].scan(lds_u, hp, cl);
    if (tid == 0 && c0 + cl < c_count) sizes[(int64_t)hp * C_cap + c_begin + c0 + cl] = cr[cl].n;
  }
  if (CL == 1 && cr[0].n == 0) return;                  // empty cluster keeps its centroid

  const bf16* Khp = K + ((int64_t)hp * N_cap + tok_begin) * D + l16 * 8;
  const int jl = (lane >> 2) * 16 + wave * 4 + (lane & 3);   // the member whose id this lane holds
  int id = CL == 1 || cr[0].n > 0 ? cr[0].member(jl) : 0;
#pragma unroll
  for (int cl = 0; cl < CL; ++cl) {
    const int n = cr[cl].n;
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    for (int j0 = 0; j0 < n; j0 += SPAN) {
      const int now = id;
#pragma unroll
      for (int s0 = 0; s0 < SPAN / 16; s0 += UPC_STEPS) {
        if (j0 + s0 * 16 >= n) break;                   // uniform
        uint4 r[UPC_STEPS];
#pragma unroll
        for (int s = 0; s < UPC_STEPS; ++s) {
          const int t = __shfl(now, (s0 + s) * 4 + g4, WAVE);
          r[s] = *reinterpret_cast<const uint4*>(Khp + (int64_t)t * D);
        }
        // the members of the next pass, or of the next cluster, are looked up while the first rows
        // of this one travel
        if (s0 == 0) {
          if (j0 + SPAN < n) id = cr[cl].member(j0 + SPAN + jl);
          else if (cl + 1 < CL && cr[cl + 1 < CL ? cl + 1 : cl].n > 0) id = cr[cl + 1 < CL ? cl + 1 : cl].member(jl);
        }
#pragma unroll
        for (int s = 0; s < UPC_STEPS; ++s) {
          const bool real = j0 + (s0 + s) * 16 + wave * 4 + g4 < n;
          const uint32_t x = real ? r[s].x : 0u, y = real ? r[s].y : 0u;
          const uint32_t z = real ? r[s].z : 0u, q = real ? r[s].w : 0u;
          acc[0] += lo_bf16(x); acc[1] += hi_bf16(x);
          acc[2] += lo_bf16(y); acc[3] += hi_bf16(y);
          acc[4] += lo_bf16(z); acc[5] += hi_bf16(z);
          acc[6] += lo_bf16(q); acc[7] += hi_bf16(q);
        }
      }
    }
    if (cl + 1 < CL && n == 0 && cr[cl + 1 < CL ? cl + 1 : cl].n > 0) id = cr[cl + 1 < CL ? cl + 1 : cl].member(jl);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float v = xor32(xor16(acc[j], OpSum()), OpSum());
      if (lane < 16) part[cl][wave][l16 * 8 + j] = v;
    }
  }
  __syncthreads();
  // wavefront w finishes cluster w
  if (wave >= CL) return;
#pragma unroll
  for (int cl = 0; cl < CL; ++cl) {
    const int c = c0 + cl, n = cr[cl].n;
    if (wave != cl || c >= c_count) continue;
    if (n == 0) continue;
    float m0 = part[cl][0][2 * lane], m1 = part[cl][0][2 * lane + 1];
#pragma unroll
    for (int w = 1; w < UPC_WAVES; ++w) {
      m0 += part[cl][w][2 * lane];
      m1 += part[cl][w][2 * lane + 1];
    }
    store_mean(m0, m1, n, hp, c, C_cap, c_begin, c_count, centroids, mu_hat, nullptr, metric, bias,
               bias_stride);
  }
}

// ------------------------------------------------------------------ from the labels
// Short ranges: the workgroup of a cluster reads all labels of its range and keeps the tokens that
// carry its own, in order.  That is one look-up in place of two (runs, then list), the assignment
// need not order its chunks, and the labels below the cluster's own are the tokens in front of its
// segment, so the launch can leave the metadata as well.  Additions in k_update's order.
// Bound: launch, then labels and rows one after the other, and the instructions of looking through the
// labels, which every cluster does: eight wavefronts share that (four: 3 % of the call).
// Ten iterations at 8 x 2985 x 37: 100 us from the chunk index, with an index launch behind it, 92 from the
// labels.
constexpr int UPL_WAVES = 8;                            // look at the labels; UPC_WAVES of them add the rows
constexpr int UPL_ROUNDS = 16;                          // 64 labels each, per wavefront, at most

template <int ROUNDS, bool LOOK>
__global__ __launch_bounds__(UPL_WAVES * 64) void k_update_labels(
    const bf16* __restrict__ K, const int32_t* __restrict__ labels, int64_t N_cap, int64_t tok_begin,
    int tok_count, int C_cap, int c_begin, int c_count, bf16* __restrict__ centroids,
    bf16* __restrict__ mu_hat, int32_t* __restrict__ sizes, int metric, float* __restrict__ bias,
    int bias_stride, int32_t* __restrict__ offsets,
    int32_t* __restrict__ sorted_idx, int32_t* __restrict__ iters_done, int n_iter, const TileMap map) {
  __shared__ uint16_t member[UPL_WAVES * ROUNDS * WAVE];
  __shared__ int found[UPL_WAVES], before[UPL_WAVES];
  __shared__ __attribute__((aligned(16))) float part[UPC_WAVES][D];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, g4 = lane >> 4;
  int c, hp;
  if (!map.mine<false, LOOK>(c, hp)) return;
  CK_FETCH_ARG(centroids);                              // used last, fetched with the others
  CK_FETCH_ARG(metric);
  CK_FETCH_ARG(offsets);
  const int32_t* lab = labels + (int64_t)hp * N_cap + tok_begin;
  const int first = wave * ROUNDS * WAVE + lane, mine = c_begin + c;
  int l[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {                // unconditional: one round trip
    const int t = first + r * WAVE;
    l[r] = lab[t < tok_count ? t : tok_count - 1];
  }
  uint64_t here[ROUNDS];
  int n_here = 0;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    here[r] = __ballot(first + r * WAVE < tok_count && l[r] == mine);
    n_here += __popcll(here[r]);
  }
  if (offsets) {                                        // uniform
    int n_before = 0;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) n_before += __popcll(__ballot(first + r * WAVE < tok_count && l[r] < mine));
    if (lane == 0) before[wave] = n_before;
  }
  if (lane == 0) found[wave] = n_here;
  __syncthreads();
  if (map.stopped<LOOK>(hp)) return;
  int base = 0, n = 0;
#pragma unroll
  for (int w = 0; w < UPL_WAVES; ++w) {
    base += w < wave ? found[w] : 0;
    n += found[w];
  }
  const uint64_t lt = ((uint64_t)1 << lane) - 1;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    if ((here[r] >> lane) & 1) member[base + __popcll(here[r] & lt)] = (uint16_t)(first + r * WAVE);
    base += __popcll(here[r]);
  }
  __syncthreads();
  if (tid == 0) {
    sizes[(int64_t)hp * C_cap + mine] = n;
    if (iters_done && c == 0) iters_done[hp] = n_iter;
  }
  if (offsets) {
    int32_t* off_g = offsets + (int64_t)hp * (C_cap + 1);
    int seg0 = c_begin == 0 ? 0 : off_g[c_begin];
#pragma unroll
    for (int w = 0; w < UPL_WAVES; ++w) seg0 += before[w];
    if (tid == 0) {
      off_g[mine + 1] = seg0 + n;
      if (mine == 0) off_g[0] = 0;
    }
    for (int j = tid; j < n; j += UPL_WAVES * 64) {
      const int64_t pos = (int64_t)seg0 + j;
      if (pos >= 0 && pos < N_cap) sorted_idx[(int64_t)hp * N_cap + pos] = (int32_t)(tok_begin + member[j]);
    }
  }
  if (n == 0) return;                                   // empty cluster keeps its centroid

  const bf16* Khp = K + ((int64_t)hp * N_cap + tok_begin) * D + l16 * 8;
  float acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.f;
  const int stream = wave * 4 + g4;
  for (int j0 = stream; wave < UPC_WAVES && j0 - stream < n; j0 += 16 * UPC_STEPS) {
    uint4 r[UPC_STEPS];
#pragma unroll
    for (int s = 0; s < UPC_STEPS; ++s) {
      const int j = j0 + 16 * s;
      r[s] = *reinterpret_cast<const uint4*>(Khp + (int64_t)member[j < n ? j : n - 1] * D);
    }
#pragma unroll
    for (int s = 0; s < UPC_STEPS; ++s) {
      const bool real = j0 + 16 * s < n;
      const uint32_t x = real ? r[s].x : 0u, y = real ? r[s].y : 0u;
      const uint32_t z = real ? r[s].z : 0u, q = real ? r[s].w : 0u;
      acc[0] += lo_bf16(x); acc[1] += hi_bf16(x);
      acc[2] += lo_bf16(y); acc[3] += hi_bf16(y);
      acc[4] += lo_bf16(z); acc[5] += hi_bf16(z);
      acc[6] += lo_bf16(q); acc[7] += hi_bf16(q);
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float v = xor32(xor16(acc[j], OpSum()), OpSum());
    if (wave < UPC_WAVES && lane < 16) part[wave][l16 * 8 + j] = v;
  }
  __syncthreads();
  if (wave > 0) return;
  float m0 = part[0][2 * lane], m1 = part[0][2 * lane + 1];
#pragma unroll
  for (int w = 1; w < UPC_WAVES; ++w) {
    m0 += part[w][2 * lane];
    m1 += part[w][2 * lane + 1];
  }
  store_mean(m0, m1, n, hp, c, C_cap, c_begin, c_count, centroids, mu_hat, nullptr, metric, bias,
             bias_stride);
}

// Where all workgroups are resident together (four per CU) and the labels read, over all clusters, are
// few.  Ten iterations, chunk index / labels, us (head-problems x tokens x clusters): 8 x 1024 x 13
// 95 / 84, 8 x 4096 x 51 101 / 92, 8 x 4096 x 128 113 / 112, 4 x 8192 x 102 118 / 113, 1 x 8192 x 102
// 114 / 105, 60 x 1024 x 13 113 / 110, 20 x 4096 x 51 127 / 125; more labels: 8 x 8179 x 102 129 / 151,
// 16 x 5000 x 62 125 / 146; more workgroups: 8 x 1024 x 256 154 / 164, 128 x 500 x 25 155 / 187,
// 128 x 1024 x 13 143 / 153.
bool update_labels_fits(const Dims& dm, int64_t tok_count, int c_count) {
  return tok_count <= UPL_WAVES * UPL_ROUNDS * WAVE && (int64_t)dm.HP * c_count <= 1024 &&
         (int64_t)dm.HP * c_count * tok_count <= 1 << 22;
}

hipError_t launch_update_labels(const Dims& dm, const bf16* K, const int32_t* labels,
                                int64_t tok_begin, int64_t tok_count, int c_begin, int c_count,
                                bf16* centroids, bf16* mu_hat, int32_t* sizes, int metric,
                                float* bias, int bias_stride, const Running& running,
                                int32_t* offsets, int32_t* sorted_idx, int32_t* iters_done,
                                int n_iter, hipStream_t st) {
  const TileMap map(c_count, dm.HP, running);
  auto launch = [&](auto look) {
    constexpr bool L = decltype(look)::value;
    const auto kernel = tok_count <= UPL_WAVES * 8 * WAVE ? k_update_labels<8, L> : k_update_labels<UPL_ROUNDS, L>;
    hipLaunchKernelGGL(kernel, map.grid(), dim3(UPL_WAVES * 64), 0, st, K, labels,
                       dm.N_cap, tok_begin, (int)tok_count, dm.C_cap, c_begin, c_count, centroids,
                       mu_hat, sizes, metric, bias, bias_stride, offsets, sorted_idx, iters_done,
                       n_iter, map);
  };
  running.first ? launch(std::true_type()) : launch(std::false_type());
  return hipGetLastError();
}

// Metadata of the final labels: offsets (prefix sum of the sizes the last update wrote) and
// the label-sorted index, one wavefront per cluster.  One launch where the counting sort needs
// two, and the index leaves in coalesced stores: the segments of a workgroup's clusters follow each
// other, so its threads share them whatever their sizes (a wavefront for each cluster took 11.2 us at
// 4 x 24553 x 306 by inner product, where a few clusters hold most keys, now 5.0; 31.6 -> 12.8 at
// 16 x 50000 x 600).
constexpr int EMIT_WAVES = 8;                           // clusters per workgroup

__global__ __launch_bounds__(EMIT_WAVES * 64) void k_emit_index(
    const uint32_t* __restrict__ seg, const uint16_t* __restrict__ list, int n_chunks,
    int chunk_tokens, int64_t N_cap, int64_t tok_begin, int64_t tok_count, int C_cap, int c_begin,
    int c_count, const int32_t* __restrict__ sizes, int32_t* __restrict__ offsets,
    int32_t* __restrict__ sorted_idx, int32_t* __restrict__ iters_done, int n_iter,
    const int32_t* __restrict__ changed) {
  extern __shared__ uint32_t lds_u[];
  __shared__ int below[EMIT_WAVES], own[EMIT_WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int hp = blockIdx.y, c0 = blockIdx.x * EMIT_WAVES, c = c0 + wave;
  int32_t* off_g = offsets + (int64_t)hp * (C_cap + 1);
  const int32_t* sz = sizes + (int64_t)hp * C_cap + c_begin;
  constexpr int PER = CK_MAX_CLUSTERS / (EMIT_WAVES * 64);
  int sum = 0;                                          // sizes of the clusters before this workgroup's
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int b = tid + i * EMIT_WAVES * 64;
    const int v = sz[b < c_count ? b : 0];
    sum += b < c0 ? v : 0;
  }
  const int base0 = c_begin == 0 ? 0 : off_g[c_begin];
  ChunkRuns cr = {seg, list, n_chunks, chunk_tokens, tok_count};
  cr.stage<EMIT_WAVES, EMIT_WAVES * 64>(lds_u, hp, c0, wave, c_count);
  sum = __builtin_amdgcn_readlane(wave_inclusive_scan(sum), WAVE - 1);
  if (lane == 0) {
    below[wave] = sum;
    own[wave] = cr.n;
  }
  __syncthreads();
  int base = base0, total = 0, n_of[EMIT_WAVES];        // base: of the first cluster
  int end = cr.n;                                       // of this wavefront's, relative to it
#pragma unroll
  for (int w = 0; w < EMIT_WAVES; ++w) {
    base += below[w];
    n_of[w] = own[w];                                   // zero behind the last cluster
    total += n_of[w];
    end += w < wave ? n_of[w] : 0;
  }
  if (c < c_count && lane == 0) {
    off_g[c_begin + c + 1] = base + end;
    if (c == 0 && c_begin == 0) off_g[0] = 0;
  }
  if (iters_done && c == 0) {
    const int n = changed ? iterations_run(changed, n_iter, gridDim.y, hp) : n_iter;
    if (lane == 0) iters_done[hp] = n;
  }
  const int cpad = (n_chunks + 63) & ~63;
  int32_t* out = sorted_idx + (int64_t)hp * N_cap;
  for (int j = tid; j < total; j += EMIT_WAVES * 64) {
    int k = j, w = 0;                                   // member k of cluster c0 + w
#pragma unroll
    for (int i = 0; i + 1 < EMIT_WAVES; ++i)
      if (w == i && k >= n_of[i]) {
        k -= n_of[i];
        w = i + 1;
      }
    cr.runs = lds_u + (size_t)w * 2 * cpad;
    cr.upto = reinterpret_cast<const int*>(cr.runs + cpad);
    cr.n = k + 1;
    const int64_t pos = (int64_t)base + j;
    if (pos >= 0 && pos < N_cap) out[pos] = (int32_t)(tok_begin + cr.member(k));
  }
}

bool update_chunks_fits(int chunk_tokens, int64_t tok_count) {
  return (tok_count + chunk_tokens - 1) / chunk_tokens <= CHUNK_RUNS_MAX;
}

static size_t chunk_runs_lds(int clusters, int n_chunks) {
  return (size_t)clusters * 2 * ((n_chunks + 63) & ~63) * sizeof(uint32_t);
}

// Four clusters to a workgroup where the run table weighs as much as the keys.  A cluster on its own
// requests a line of 128 bytes per chunk of 512 tokens (6.28 M requests to the L2s at 8 x 131072 x 1600,
// 3.97 M with four, the same bytes from HBM) and 256 bytes per member, so the table's share grows with
// the clusters: it is three quarters of the rows' at 768.  Below 2M words, launches of about 50 us and
// less, the longer workgroups cost more than they spare, and up to 128 chunks a table is scanned in
// two steps.  One / four, us per launch: 8 x 131072 x 1600 56.8 / 50.9, 16 x 131072 x 819
// 118.3 / 113.2, 12 x 98304 x 1200 68.5 / 63.9, 6 x 196608 x 1012 63.1 / 59.8, 5 x 262144 x 1016
// 77.0 / 69.3, but with few clusters 16 x 131072 x 400 103.9 / 107.9, 9 x 262144 x 510 121.0 / 124.8,
// with few words 4 x 131072 x 1600 26.7 / 28.5, 8 x 131072 x 819 48.9 / 49.8, 4 x 262144 x 1014
// 50.3 / 51.7, and with 128 chunks 24 x 65536 x 800 89.9 / 90.5 and ten iterations of 16 x 65536 x 800
// 2202 / 2221.  With 144 and 160 chunks either is up to 4 % faster.  With tiles by XCD, ten iterations:
// 8 x 131072 x 1600 3655 / 3626, 16 x 131072 x 819 4449 / 4420, 12 x 98304 x 1200 3331 / 3309, 4 x 131072 x 1600
// 1891 / 1908, 8 x 131072 x 819 2216 / 2226, 16 x 65536 x 800 2137 / 2152.
int update_clusters_per_workgroup(int n_chunks, int c_count, int hp) {
  return n_chunks > 128 && c_count >= 768 && (int64_t)n_chunks * c_count * hp >= 1 << 21 ? 4 : 1;
}

hipError_t launch_update_chunks(const Dims& dm, const bf16* K, const ChunkIndex& chunks,
                                int64_t tok_begin, int64_t tok_count, int c_begin, int c_count,
                                bf16* centroids, bf16* mu_hat, int32_t* sizes, int metric,
                                float* bias, int bias_stride, const Running& running, hipStream_t st) {
  const int chunk_tokens = chunks.tokens;
  const int n_chunks = (int)((tok_count + chunk_tokens - 1) / chunk_tokens);
  const int cl = update_clusters_per_workgroup(n_chunks, c_count, dm.HP);
  const TileMap map((c_count + cl - 1) / cl, dm.HP, running);
  auto launch = [&](auto look) {
    constexpr bool L = decltype(look)::value;
    hipLaunchKernelGGL((cl == 4 ? k_update_chunks<4, L> : k_update_chunks<1, L>), map.grid(), dim3(UPC_WAVES * 64),
                       chunk_runs_lds(cl, n_chunks), st, K, chunks.seg, chunks.list, n_chunks,
                       chunk_tokens, dm.N_cap, tok_begin, tok_count, dm.C_cap, c_begin, c_count,
                       centroids, mu_hat, sizes, metric, bias, bias_stride, map);
  };
  running.first ? launch(std::true_type()) : launch(std::false_type());
  return hipGetLastError();
}

hipError_t launch_emit_index(const Dims& dm, const ChunkIndex& chunks, int64_t tok_begin,
                             int64_t tok_count, int c_begin, int c_count, const int32_t* sizes,
                             int32_t* offsets, int32_t* sorted_idx, int32_t* iters_done, int n_iter,
                             const int32_t* changed, hipStream_t st) {
  const int chunk_tokens = chunks.tokens;
  const int n_chunks = (int)((tok_count + chunk_tokens - 1) / chunk_tokens);
  hipLaunchKernelGGL(k_emit_index, dim3((c_count + EMIT_WAVES - 1) / EMIT_WAVES, dm.HP),
                     dim3(EMIT_WAVES * 64), chunk_runs_lds(EMIT_WAVES, n_chunks), st, chunks.seg, chunks.list,
                     n_chunks, chunk_tokens, dm.N_cap, tok_begin, tok_count, dm.C_cap, c_begin,
                     c_count, sizes, offsets, sorted_idx, iters_done, n_iter, changed);
  return hipGetLastError();
}

static ClusterWorkspace carve(const Dims& dm, int64_t tok_count, int c_count, int chunk_tokens, void* base) {
  ClusterWorkspace w;
  const int64_t n_chunks = (tok_count + chunk_tokens - 1) / chunk_tokens;
  size_t mu = (size_t)dm.HP * c_count * D * sizeof(bf16);
  mu = (mu + 255) & ~(size_t)255;
  size_t seg = (size_t)dm.HP * n_chunks * seg_stride(c_count) * sizeof(uint32_t);
  seg = (seg + 255) & ~(size_t)255;
  size_t list = (size_t)dm.HP * n_chunks * chunk_tokens * sizeof(uint16_t);
  list = (list + 255) & ~(size_t)255;
  w.bias_stride = (c_count + 31) / 32 * 32;
  size_t bias = (size_t)dm.HP * w.bias_stride * sizeof(float);
  bias = (bias + 255) & ~(size_t)255;
  size_t chg = (size_t)(KM_MAX_ITER_CONVERGE + 1) * dm.HP * sizeof(int32_t);
  chg = (chg + 255) & ~(size_t)255;
  char* b = reinterpret_cast<char*>(base);
  w.mu_hat = reinterpret_cast<bf16*>(b);
  w.chunks.seg = reinterpret_cast<uint32_t*>(b + mu);
  w.chunks.tokens = chunk_tokens;
  w.chunks.list = reinterpret_cast<uint16_t*>(b + mu + seg);
  w.bias = reinterpret_cast<float*>(b + mu + seg + list);
  w.changed = reinterpret_cast<int32_t*>(b + mu + seg + list + bias);
  w.bytes = mu + seg + list + bias + chg;
  return w;
}

// Chunk size of the counting sort with no assignment in front of it.  Not the one that the assignment
// prefers for small tables: the scan goes through all chunks of a head-problem, and four times as many
// are only longer.
int sort_tile_tokens(const Dims& dm, int64_t tok_count) {
  return tok_count * dm.HP >= 64 * 1024 ? 512 : 128;
}

// Neither chunk size is the larger one for all shapes: 512 tokens save run words, but a range ends in a
// chunk that is filled up (128 head-problems of 600 tokens, 7 clusters: 647680 bytes, 561664 with 128).
size_t cluster_workspace_bytes(const Dims& dm, int64_t tok_count, int c_count) {
  const size_t a = carve(dm, tok_count, c_count, assign_tile_tokens(dm, tok_count, c_count), nullptr).bytes;
  const size_t s = carve(dm, tok_count, c_count, sort_tile_tokens(dm, tok_count), nullptr).bytes;
  return a > s ? a : s;
}

ClusterWorkspace carve_cluster_workspace(const Dims& dm, int64_t tok_count, int c_count, int chunk_tokens,
                                         void* base, size_t have) {
  ClusterWorkspace best = carve(dm, tok_count, c_count, chunk_tokens, base);
  // a workspace that was sized for more tokens holds one of the sizes, and every one of them runs
  for (const int other : {512, 256, 128}) {
    if (best.bytes <= have) break;
    const ClusterWorkspace w = carve(dm, tok_count, c_count, other, base);
    if (w.bytes < best.bytes) best = w;
  }
  return best;
}

}  // namespace ck
