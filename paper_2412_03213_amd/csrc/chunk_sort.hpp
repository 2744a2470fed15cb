// Label-ordered index of one chunk of tokens, built by one wavefront in the epilogue of
// the assignment kernels (the chunk's labels are in LDS there anyway).
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

// Stable counting sort of a chunk of ROUNDS * 64 tokens by label, by one wavefront.  tok
// (LDS): the pack_token words of the chunk, every label below c_count; cnt (LDS, chunk_sort_cnt_ints(CMAX) ints) and
// order (LDS, ROUNDS * 64 entries) are 16-byte aligned scratch of this wavefront.
// The groups of 64 add their label counts to the chunk's in order, the first lane of every
// label with one LDS atomic that returns the count of the groups before; all rounds are
// issued back to back (LDS serves one wavefront in order) and a lane scans a run of
// consecutive labels held in registers, so the chain is a handful of LDS round trips long
// however many rounds and labels there are.  That matters because the epilogue this stands in
// runs with the matrix cores idle: one read-modify-write per round and one pass per 64 labels
// took 6 us per chunk of 512 tokens and 400 labels.
template <int ROUNDS, int CMAX>
__device__ __forceinline__ void chunk_sort(const uint32_t* tok, int c_count, int* cnt,
                                           uint16_t* order, uint32_t* __restrict__ seg,
                                           uint16_t* __restrict__ list) {
  constexpr int QMAX = chunk_sort_cnt_ints(CMAX) / 256; // quads of labels per lane
  const int lane = threadIdx.x & 63;
  const int quads = (c_count + 255) / 256;
  const int q0 = lane * quads;
  int4* mine = reinterpret_cast<int4*>(cnt) + q0;
  for (int i = 0; i < quads; ++i) mine[i] = make_int4(0, 0, 0, 0);
  uint32_t w[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) w[r] = tok[r * WAVE + lane];
  wave_lds_order();
  int before[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const bool first = (w[r] >> 31) && ((w[r] >> 11) & 63u) == 0;
    before[r] = 0;
    if (first) before[r] = atomicAdd(&cnt[w[r] & 2047u], (int)((w[r] >> 17) & 63u) + 1);
  }
  wave_lds_order();
  // counts -> first positions; both together are the words of seg
  int4 v[QMAX];
  int sum = 0;
#pragma unroll
  for (int i = 0; i < QMAX; ++i)
    if (i < quads) v[i] = mine[i];
#pragma unroll
  for (int i = 0; i < QMAX; ++i)
    if (i < quads) sum += (v[i].x + v[i].y) + (v[i].z + v[i].w);
  int run = wave_inclusive_scan(sum) - sum;
#pragma unroll
  for (int i = 0; i < QMAX; ++i)
    if (i < quads) {
      int4 e;
      e.x = run;
      e.y = e.x + v[i].x;
      e.z = e.y + v[i].y;
      e.w = e.z + v[i].z;
      run = e.w + v[i].w;
      mine[i] = e;
      if ((q0 + i) * 4 < c_count)
        reinterpret_cast<uint4*>(seg)[q0 + i] =
            make_uint4((uint32_t)e.x | ((uint32_t)v[i].x << 16), (uint32_t)e.y | ((uint32_t)v[i].y << 16),
                       (uint32_t)e.z | ((uint32_t)v[i].z << 16), (uint32_t)e.w | ((uint32_t)v[i].w << 16));
    }
  wave_lds_order();
  int at[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int b = __shfl(before[r], (int)((w[r] >> 23) & 63u), WAVE);
    at[r] = cnt[w[r] & 2047u] + b + (int)((w[r] >> 11) & 63u);
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
    if (w[r] >> 31) order[at[r]] = (uint16_t)(r * WAVE + lane);
  wave_lds_order();
  // entries beyond the chunk's tokens are never read back
  if constexpr (ROUNDS == 8)
    reinterpret_cast<uint4*>(list)[lane] = reinterpret_cast<const uint4*>(order)[lane];
  else
    for (int i = lane; i < ROUNDS * 32; i += WAVE)
      reinterpret_cast<uint32_t*>(list)[i] = reinterpret_cast<const uint32_t*>(order)[i];
}

}  // namespace ck
