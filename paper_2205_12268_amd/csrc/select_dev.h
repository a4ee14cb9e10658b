// Device code shared by the selection kernels (select.hip, select_two.hip).
#pragma once
#include "strip.h"

namespace wcc {

// lh[digit] += 1 for every valid lane; lanes of a wave that share a digit are counted by one
// LDS atomic (two leader rounds catch the big tie classes, the rest goes lane by lane)
__device__ __forceinline__ void hist_add(uint32_t *lh, uint32_t digit, bool valid) {
  const int lane = threadIdx.x & 63;
  uint64_t todo = __ballot(valid);
#pragma unroll
  for (int round = 0; round < 2; ++round) {
    if (todo == 0) break;
    const int leader = __ffsll((unsigned long long)todo) - 1;
    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)digit, leader);  // leader is wave-uniform
    const uint64_t same = __ballot(valid && digit == d0);
    if (lane == leader) atomicAdd(&lh[d0], (uint32_t)__popcll(same));
    if (digit == d0) valid = false;
    todo &= ~same;
  }
  if (valid) atomicAdd(&lh[digit], 1u);
}

// The same for a workgroup whose digits are spread out: one round, the class of the first
// valid lane is counted by one atomic, every other lane adds for itself.
__device__ __forceinline__ void hist_add_spread(uint32_t *lh, uint32_t digit, bool valid) {
  if (valid) {
    const uint32_t d0 = __builtin_amdgcn_readfirstlane(digit);
    const uint64_t same = __ballot(digit == d0);
    const int first = __ffsll((unsigned long long)same) - 1;
    const uint32_t val = digit != d0 ? 1u : ((int)(threadIdx.x & 63) == first ? (uint32_t)__popcll(same) : 0u);
    if (val) atomicAdd(&lh[digit], val);
  }
}

// Inclusive prefix sum over the 64 lanes of a wave (all of them active), on the data-parallel
// shifts of the vector unit instead of six round trips through the LDS crossbar: shifts by
// 1, 2, 4, 8 inside rows of 16 lanes (a lane shifted in from outside its row adds 0), then lane
// 15 of rows 0 and 2 into rows 1 and 3, then lane 31 into rows 2 and 3.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
  uint32_t v = x;
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// Smallest / largest value over the 64 lanes (all active), every lane gets it: the moves of the
// scan with the operation's identity shifted in; lane 63 ends up with the whole wave's result.
template <bool MAX>
__device__ __forceinline__ uint32_t wave_extreme(uint32_t x) {
  constexpr int id = MAX ? 0 : -1;
  uint32_t v = x;
  auto join = [](uint32_t a, uint32_t b) { return MAX ? max(a, b) : min(a, b); };
  v = join(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x111, 0xf, 0xf, false));
  v = join(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x112, 0xf, 0xf, false));
  v = join(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x114, 0xf, 0xf, false));
  v = join(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x118, 0xf, 0xf, false));
  v = join(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x142, 0xa, 0xf, false));
  v = join(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x143, 0xc, 0xf, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// block-wide sum of v (all threads get it); `tmp` has NW (waves per workgroup) entries
template <int NW>
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t *tmp) {
  v = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(v), 63);
  __syncthreads();  // tmp may still be read from a previous use
  if ((threadIdx.x & 63) == 0) tmp[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t s = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) s += tmp[i];
  return s;
}

// block-wide exclusive scan in thread order; `tmp` has NW (waves per workgroup) entries
template <int NW>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *tmp) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t inc = wave_inclusive_scan(v);
  __syncthreads();
  if (lane == 63) tmp[wv] = inc;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i)
    if (i < wv) before += tmp[i];
  return before + inc - v;
}

// Four keys of this thread.  REDUCE: keys are sums of G partial-norm planes (added in
// increasing group order), and the sums are written to norm.
template <bool REDUCE>
__device__ __forceinline__ uint4 load_keys(const float *__restrict__ src, float *__restrict__ norm,
                                           int G, int64_t BN, int64_t at) {
  float4 v = *reinterpret_cast<const float4 *>(src + at);
  if constexpr (REDUCE) {
    int g = 1;
    for (; g + 4 <= G; g += 4) {  // four loads in flight, added in increasing group order
      float4 t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = *reinterpret_cast<const float4 *>(src + (int64_t)(g + i) * BN + at);
#pragma unroll
      for (int i = 0; i < 4; ++i) { v.x += t[i].x; v.y += t[i].y; v.z += t[i].z; v.w += t[i].w; }
    }
    for (; g < G; ++g) {
      const float4 t = *reinterpret_cast<const float4 *>(src + (int64_t)g * BN + at);
      v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
    }
    *reinterpret_cast<float4 *>(norm + at) = v;
  }
  return make_uint4(__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z),
                    __float_as_uint(v.w));
}

// max over the G channel groups of their largest |coefficient| at this thread's four positions
// (top_part [G, B, N], written by the norm-only transform pass)
__device__ __forceinline__ float4 load_top(const float *__restrict__ top_part, int G, int64_t BN,
                                           int64_t at) {
  float4 m = *reinterpret_cast<const float4 *>(top_part + at);
  int g = 1;
  for (; g + 4 <= G; g += 4) {  // four loads in flight
    float4 t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = *reinterpret_cast<const float4 *>(top_part + (int64_t)(g + i) * BN + at);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      m.x = fmaxf(m.x, t[i].x); m.y = fmaxf(m.y, t[i].y); m.z = fmaxf(m.z, t[i].z); m.w = fmaxf(m.w, t[i].w);
    }
  }
  for (; g < G; ++g) {
    const float4 t = *reinterpret_cast<const float4 *>(top_part + (int64_t)g * BN + at);
    m.x = fmaxf(m.x, t.x); m.y = fmaxf(m.y, t.y); m.z = fmaxf(m.z, t.z); m.w = fmaxf(m.w, t.w);
  }
  return m;
}

// block_top[slot] = the workgroup's largest kept |coefficient| (v >= 0 in every thread, all
// threads of the workgroup call; `tmp` has NW entries).  A plain store per workgroup: the
// consumers take the maximum over all of them.
template <int NW>
__device__ __forceinline__ void publish_top(float v, float *block_top, size_t slot, uint32_t *tmp) {
  const uint32_t w = wave_extreme<true>(__float_as_uint(v));  // (>= 0: floats order like their bits)
  workgroup_lds_barrier();  // tmp may still be read from a previous use (stores keep travelling)
  if ((threadIdx.x & 63) == 0) tmp[threadIdx.x >> 6] = w;
  workgroup_lds_barrier();
  if (threadIdx.x == 0) {
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) mine = max(mine, tmp[i]);
    block_top[slot] = __uint_as_float(mine);
  }
}

// A job of moving 16-byte pieces done beside a kernel that is bound by its own latencies: the first
// piece's load goes out early, its store and the few pieces after it follow at the end.
struct PackOnTheSide {
  uint4 v;
  int e;
  __device__ __forceinline__ PackOnTheSide(const PackJob &job, int first) : v(make_uint4(0, 0, 0, 0)), e(first) {
    if (e < job.total) v = pack_piece(job, e);
  }
  __device__ __forceinline__ void finish(const PackJob &job, int threads) const {
    if (e < job.total) job.out[e] = v;
    for (int i = e + threads; i < job.total; i += threads) job.out[i] = pack_piece(job, i);
  }
};

}  // namespace wcc
