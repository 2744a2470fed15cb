// Label-ordered index of one chunk of tokens, built in the epilogue of the assignment kernels
// (the chunk's labels are in LDS there anyway).
#pragma once
#include "ck_common.hpp"

namespace ck {

// Lanes of a wavefront that hold the same label, as a 64-bit mask (built from one
// ballot per label bit), restricted to `valid` lanes.
__device__ __forceinline__ uint64_t same_label_mask(int label, bool valid, int label_bits) {
  const uint64_t v = __ballot(valid);
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  for (int b = 0; b < label_bits; ++b) {
    const int mine = -((label >> b) & 1);               // all ones where the bit is set
    const uint64_t m = __ballot(mine != 0);
    lo &= ~((uint32_t)m ^ (uint32_t)mine);
    hi &= ~((uint32_t)(m >> 32) ^ (uint32_t)mine);
  }
  return (uint64_t)lo | ((uint64_t)hi << 32);
}

// What a token brings to the sort of its chunk, packed into one word while the labels of its
// group of 64 consecutive tokens are still in the lanes of a wavefront:
//   bit 31 a token exists, bits 0..10 its label, 11..16 how many tokens of the group before it
//   have the same label, 17..22 how many have it in all (minus one), 23..28 the first such lane.
__device__ __forceinline__ uint32_t pack_token(int label, bool valid, int label_bits) {
  const int lane = threadIdx.x & 63;
  const uint64_t peers = same_label_mask(label, valid, label_bits);
  const uint64_t lt = ((uint64_t)1 << lane) - 1;
  const uint32_t rank = (uint32_t)__popcll(peers & lt), n = (uint32_t)__popcll(peers);
  const uint32_t first = (uint32_t)__builtin_ctzll(peers | ((uint64_t)1 << 63));
  return valid ? 0x80000000u | (uint32_t)label | (rank << 11) | ((n - 1) << 17) | (first << 23) : 0u;
}

constexpr int seg_stride(int c_count) { return (c_count + 3) & ~3; }   // words per chunk in seg
constexpr int chunk_sort_cnt_ints(int c_max) { return (c_max + 255) & ~255; }

// Stable counting sort of a chunk of ROUNDS * 64 tokens by label, by W wavefronts of the workgroup
// (W divides ROUNDS; sub is this one's number among them).  To be called by ALL wavefronts of the
// workgroup: it has barriers; active is false where there is no chunk or no part in it.
// tok (LDS): the pack_token words of the chunk, every label below c_count; cnt (LDS, W rows of
// chunk_sort_cnt_ints(CMAX) ints), order (LDS, ROUNDS * 64 entries) and sums (LDS, W ints) are
// 16-byte aligned scratch of the chunk.
// Each wavefront takes ROUNDS / W consecutive groups of 64 and adds their label counts to its row of
// cnt in order, the first lane of every label with one LDS atomic that returns the count of the
// groups before.  Then each scans its share of the labels over all rows, a lane a run of
// consecutive labels, and the rows become first positions.  It runs with the matrix cores idle, so
// what matters is the length of the chain: with one wavefront per chunk of 512 tokens, which takes
// 2.4 us at 1600 labels and 1.9 at 400, ten iterations were 0.6 % longer at 8 x 131072 x 1600 and
// 8 x 32768 x 400.
template <int ROUNDS, int CMAX, int W>
__device__ __forceinline__ void chunk_sort(const uint32_t* tok, int c_count, int sub, bool active,
                                           int* cnt, int* sums, uint16_t* order,
                                           uint32_t* __restrict__ seg, uint16_t* __restrict__ list) {
  static_assert(ROUNDS % W == 0, "whole groups");
  constexpr int ROW = chunk_sort_cnt_ints(CMAX), PER = ROUNDS / W;
  constexpr int QMAX = (ROW / 256 + W - 1) / W;         // quads of labels per lane
  const int lane = threadIdx.x & 63;
  const int quads = (c_count + 256 * W - 1) / (256 * W);
  const int q0 = (sub * WAVE + lane) * quads;           // first quad of this lane
  const int n_quads = (c_count + 3) / 4;
  uint32_t w[PER];
  if (active) {
    int4* row = reinterpret_cast<int4*>(cnt + sub * ROW);
    for (int i = lane; i < n_quads; i += WAVE) row[i] = make_int4(0, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < PER; ++r) w[r] = tok[(sub * PER + r) * WAVE + lane];
  }
  wave_lds_order();
  int before[PER];
  if (active) {
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const bool first = (w[r] >> 31) && ((w[r] >> 11) & 63u) == 0;
      before[r] = 0;
      if (first) before[r] = atomicAdd(&cnt[sub * ROW + (w[r] & 2047u)], (int)((w[r] >> 17) & 63u) + 1);
    }
  }
  if constexpr (W > 1) __syncthreads(); else wave_lds_order();
  // counts of this lane's labels in all rows, and how many tokens come before them
  int4 v[QMAX];
  int run = 0;
  if (active) {
    int sum = 0;
#pragma unroll
    for (int i = 0; i < QMAX; ++i) {
      v[i] = make_int4(0, 0, 0, 0);
      if (i < quads && q0 + i < n_quads) {
#pragma unroll
        for (int r = 0; r < W; ++r) {
          const int4 x = reinterpret_cast<const int4*>(cnt + r * ROW)[q0 + i];
          v[i].x += x.x; v[i].y += x.y; v[i].z += x.z; v[i].w += x.w;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < QMAX; ++i) sum += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    run = wave_inclusive_scan(sum);
    if (W > 1 && lane == WAVE - 1) sums[sub] = run;
    run -= sum;
  }
  if constexpr (W > 1) __syncthreads();
  if (active) {
#pragma unroll
    for (int r = 0; r < W - 1; ++r) run += r < sub ? sums[r] : 0;
#pragma unroll
    for (int i = 0; i < QMAX; ++i)
      if (i < quads && q0 + i < n_quads) {
        int4 e;
        e.x = run;
        e.y = e.x + v[i].x;
        e.z = e.y + v[i].y;
        e.w = e.z + v[i].z;
        run = e.w + v[i].w;
        reinterpret_cast<uint4*>(seg)[q0 + i] =
            make_uint4((uint32_t)e.x | ((uint32_t)v[i].x << 16), (uint32_t)e.y | ((uint32_t)v[i].y << 16),
                       (uint32_t)e.z | ((uint32_t)v[i].z << 16), (uint32_t)e.w | ((uint32_t)v[i].w << 16));
#pragma unroll
        for (int r = 0; r < W; ++r) {                   // first position of row r's tokens
          int4* x = reinterpret_cast<int4*>(cnt + r * ROW) + q0 + i;
          const int4 n = *x;
          *x = e;
          e.x += n.x; e.y += n.y; e.z += n.z; e.w += n.w;
        }
      }
  }
  if constexpr (W > 1) __syncthreads(); else wave_lds_order();
  if (active) {
    int at[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const int b = __shfl(before[r], (int)((w[r] >> 23) & 63u), WAVE);
      at[r] = cnt[sub * ROW + (w[r] & 2047u)] + b + (int)((w[r] >> 11) & 63u);
    }
#pragma unroll
    for (int r = 0; r < PER; ++r)
      if (w[r] >> 31) order[at[r]] = (uint16_t)((sub * PER + r) * WAVE + lane);
  }
  if constexpr (W > 1) __syncthreads(); else wave_lds_order();
  // entries beyond the chunk's tokens are never read back
  if (active)
    for (int i = sub * WAVE + lane; i < ROUNDS * 8; i += W * WAVE)
      reinterpret_cast<uint4*>(list)[i] = reinterpret_cast<const uint4*>(order)[i];
}

}  // namespace ck
