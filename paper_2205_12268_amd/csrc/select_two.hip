// Joint shrinkage of planes too large for one workgroup a sample, in two launches: per sample, the k
// largest of N non-negative fp32 norms, ties toward the lower position, emitted in ascending position
// order (the result of select.hip's passes, bit for bit).
//
// Design.  What a radix selection over the chip pays for is not its keys but its rounds: every round is a
// launch (4-5 us with the chain histogram -> merge -> pick), and three rounds of digits and the compaction
// took 17-19 us on 10^5 keys.  Here the first kernel does for its chunk what later rounds would ask of it:
// it groups the chunk's keys by a digit (counting sort in LDS) and leaves, beside the grouped keys, how many
// of them have that digit or a larger one.  The second kernel's workgroups read these tables -- no histogram
// is merged, nothing has to be cleared before --, find the digit D that holds rank k, collect the keys with
// digit D from all chunks of the sample (a contiguous segment each: half a percent of the keys as norms are
// distributed), find the threshold among them in LDS, and emit their own chunk in position order: how many
// kept positions lie before it follows from the same tables and segments.  Every workgroup of a sample does
// this for itself; none waits for another.
//
// The digit is any monotone function of the key; the exact threshold is found on whole keys.  Taken: zero
// alone, then 64 steps an octave from 2^-32 to 2^32, everything outside in the first or last step.  Where
// the keys with digit D do not fit in LDS (large classes of equal keys, noise over many channels, whose norms
// lie close together, scales outside that range) they are read from memory until those that still matter do.
//
// Such digits are too coarse where norms lie close together (noise over many channels) or are equal (a blank frame): every
// workgroup would read the whole class, which took 131072 equal keys 60 us.  So the first kernel looks at a few hundred
// keys from all over the sample, the same ones in every workgroup: where too many fall into the step that rank k lies in, the
// digits are cut by those keys instead, sorted, with a digit for what equals one of them.
//
// Bound by latency: 5 us for the first kernel, 8-9 for the second (its chain is two table reads and the segments,
// 1 us each, another die wrote them, and a dozen barriers; 256 or 512 threads in place of 1024 take 9-11 us); looking at
// the keys is 0.1-0.7 of it.  Where the norms come as planes of partial norms the look goes to plane 0 first and to the sums only where it finds a
// crowd there (to the sums at once: 12.1 -> 15.3 on 8 x 65536 positions of 16 planes, 58 -> 80 on 44800 of 256; now 12.6).
// Kernel times against the four launches, without the gaps between them, of spread norms: 131072 positions 16.1 -> 12.5 us,
// 4 x 61440 15.8 -> 12.2, 8 x 122880 19.2 -> 13.8, 4 x 524288 26.4 -> 18.3, 1024 x 1024 28.2 -> 18.7.  Crowded: equal norms,
// 131072 of them 16.6 -> 16.4 (60 by the fixed digits), 1024 x 1024 33.0 -> 20.1 (398); norms of noise with a deviation of 3 %, cut
// at the median, 131072 18.0 -> 18.2 (20.3), 512 x 1024 33.6 -> 25.0 (41.5), 1024 x 1024 35.1 -> 29.1 (73).  What it loses: several
// such planes at once, 8 x 122880 22.9 -> 28.0, 4 x 524288 28.3 -> 33.5 (the gaps, 1-2 us each, not counted).
#include "select_dev.h"

namespace wcc {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kCoarse = 64;                  // coarse digits; the tables hold kCoarse + kFine counts a chunk
constexpr int kFine = 64 * kCoarse;          // digits
constexpr uint32_t kBase = (127u - 32u) << 6;  // digit 0 begins at 2^-32: key >> 17 counts 64 steps an octave
constexpr int kStepBits = 17;                // key bits below a step
constexpr uint32_t kListCap = 32768;         // keys of one digit that the second kernel holds in LDS (128 of its 149 KiB)
constexpr int kSteps = 6;                    // of six bits: a whole key
constexpr int kFieldBits = 12;               // bits a pass over memory decides, where the keys do not fit
constexpr int kProbes = 256;                 // most quads of keys that are looked at to see whether a digit is crowded
constexpr int kSplits = kProbes - 1;         // keys that part a crowded sample, then the largest of all
constexpr int kHeader = 4 + kProbes;         // words a sample: whether it is crowded, three unused, those keys

// monotone in the key (as an unsigned number: also for bit patterns that are no norm)
__device__ __forceinline__ uint32_t digit_of(uint32_t key) {
  const int s = (int)(key >> kStepBits) - (int)kBase;
  return key == 0 ? 0u : (uint32_t)min(max(s, 1), kFine - 1);
}

// lh[digit] += 1; returns how many of the digit's keys were counted before this one (an order of arrival).
// The class of the wave's first valid lane is counted by one atomic: smooth maps have many equal digits.
__device__ __forceinline__ uint32_t hist_rank(uint32_t *lh, uint32_t digit, bool valid) {
  uint32_t r = 0;
  if (valid) {
    const uint32_t d0 = __builtin_amdgcn_readfirstlane(digit);
    const uint64_t same = __ballot(digit == d0);
    if (digit == d0) {
      const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
      uint32_t base = 0;
      if (before == 0) base = atomicAdd(&lh[d0], (uint32_t)__popcll(same));
      r = (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + before;  // (the class's first lane)
    } else {
      r = atomicAdd(&lh[digit], 1u);
    }
  }
  return r;
}

// The sums of load_keys<true> at `at`, not written.
__device__ __forceinline__ uint4 sum_of_parts(const float *__restrict__ src, int G, int64_t BN, int64_t at) {
  float4 v = *reinterpret_cast<const float4 *>(src + at);
  int g = 1;
  for (; g + 8 <= G; g += 8) {
    float4 p[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = *reinterpret_cast<const float4 *>(src + (g + i) * BN + at);
#pragma unroll
    for (int i = 0; i < 8; ++i) { v.x += p[i].x; v.y += p[i].y; v.z += p[i].z; v.w += p[i].w; }
  }
  for (; g < G; ++g) {
    const float4 p = *reinterpret_cast<const float4 *>(src + g * BN + at);
    v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
  }
  return make_uint4(__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w));
}

// What the first kernel's workgroups look at to see whether a digit is crowded.
struct Probes {
  int n;           // quads of keys, one of each stretch of
  uint32_t quads;  // so many quads
  uint32_t crowd;  // this many of their keys in one step are too many ...
  int from, to;    // ... if any of them may be the one of rank k: between these of the probes' ranks
};

// First kernel.  grid = (nblk, B), block = 1024; a workgroup takes a chunk of 4096 * SLOTS positions (slot s
// of thread t: the four from (s * 1024 + t) * 4 on).  src: norms, or with REDUCE the partial norms [G, B, N],
// whose sums it writes to norm.  grouped [B, N]: each chunk's keys, largest digit first.  sfx [B, nblk, kFine]: how many of
// the chunk's keys have that digit or a larger one; csfx [B, nblk, kCoarse] the same for digit 64 c.
// hdr [B, kHeader].  Every workgroup of a sample looks at the same keys of it and so comes to the same digits: where too many
// fall into one step that rank k may lie in, 255 of them, sorted, part the sample instead: digit
// 2 j + 1 is what equals the j-th, the even ones lie between two.  REDUCE: first at plane 0, where a digit of any rank counts, then at the
// sums; planes that are crowded only together are not seen, and the second kernel then reads their digit from memory.  (The probes lie anywhere in the plane, so grouped must
// be no plane of src.)
// Also carries out `job`.
template <bool REDUCE, int SLOTS>
__global__ __launch_bounds__(kThreads) void select_group_kernel(const float *__restrict__ src, float *__restrict__ norm, int G,
                                                                int64_t N, int B, uint32_t *__restrict__ grouped,
                                                                uint16_t *__restrict__ sfx, uint16_t *__restrict__ csfx,
                                                                uint32_t *__restrict__ hdr, Probes look, PackJob job) {
  constexpr int kChunk = 4 * kThreads * SLOTS;
  __shared__ __attribute__((aligned(16))) uint32_t lh[kFine];
  __shared__ __attribute__((aligned(16))) uint32_t probed[kFine];
  __shared__ __attribute__((aligned(16))) uint32_t sorted[kChunk];
  __shared__ uint32_t picked[kProbes], runs[kProbes], splits[kProbes], tree[kProbes];
  __shared__ uint32_t tmp[kWaves];
  __shared__ int crowded;
  fetch_args(src, job.total);
  const int b = blockIdx.y, t = threadIdx.x;
  const int64_t c0 = (int64_t)blockIdx.x * kChunk;
  const int n = (int)min((int64_t)kChunk, N - c0);  // (a multiple of 4)
  // (one quad of each stretch of the plane, anywhere in it; by the first waves alone: a few threads of every wave would cost
  // all of them a wait of its own)
  const bool looks = t < look.n;
  const int64_t probe_at = (int64_t)b * N + ((int64_t)t * look.quads + __umulhi(t * 2654435761u, look.quads)) * 4;
  uint4 probe = make_uint4(0, 0, 0, 0);
  if (looks) probe = *reinterpret_cast<const uint4 *>(src + probe_at);  // (REDUCE: of plane 0 alone)
  uint4 k4[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int at = (s * kThreads + t) * 4;
    k4[s] = make_uint4(0, 0, 0, 0);
    if (at < n) k4[s] = load_keys<REDUCE>(src, norm, G, (int64_t)B * N, (int64_t)b * N + c0 + at);
  }
  const PackOnTheSide side(job, (int)((blockIdx.y * gridDim.x + blockIdx.x) * kThreads + t));
  static_assert(kFine == 4 * kThreads, "four digits a thread");
  reinterpret_cast<uint4 *>(lh)[t] = make_uint4(0, 0, 0, 0);
  reinterpret_cast<uint4 *>(probed)[t] = make_uint4(0, 0, 0, 0);
  if (t < kProbes) picked[t] = 0xFFFFFFFFu;
  if (t == 0) crowded = 0;
  __syncthreads();
  uint32_t digit[4 * SLOTS], rank[4 * SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const bool in = (s * kThreads + t) * 4 < n;
    const uint32_t key[4] = {k4[s].x, k4[s].y, k4[s].z, k4[s].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      digit[4 * s + e] = digit_of(key[e]);
      rank[4 * s + e] = hist_rank(lh, digit[4 * s + e], in);
    }
  }
  auto count_probe = [&]() {
    if (!looks) return;
    const uint32_t key[4] = {probe.x, probe.y, probe.z, probe.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      atomicAdd(&probed[digit_of(key[e])], 1u);
      if (e == 0 || 4 * look.n <= kProbes) picked[e * look.n + t] = key[e];
    }
  };
  count_probe();
  __syncthreads();
  const size_t blk = (size_t)b * gridDim.x + blockIdx.x;
  const int low = kFine - 4 - 4 * t;  // four digits a thread, from the top: its lowest one
  // whether one of the thread's digits is crowded: pc of the probes' keys in them, upto above them (anywhere: whatever their rank)
  auto see = [&](const uint4 &pc, int upto, bool anywhere) {
    const uint32_t c[4] = {pc.w, pc.z, pc.y, pc.x};
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // (zero has a digit of its own)
      if (c[i] >= look.crowd && low + 3 - i != 0 && (anywhere || (upto <= look.to && upto + (int)c[i] >= look.from))) crowded = 1;
      upto += (int)c[i];
    }
  };
  // where each digit begins in the grouped chunk, and the tables; LOOK: at the probes as well
  auto place = [&](auto look_c) {
    constexpr bool LOOK = decltype(look_c)::value;
    const uint4 c = reinterpret_cast<const uint4 *>(lh)[low / 4];
    uint4 pc = make_uint4(0, 0, 0, 0);
    if constexpr (LOOK) pc = reinterpret_cast<const uint4 *>(probed)[low / 4];
    // (keys of the chunk | keys of the probes << 16)
    const uint32_t both = block_exclusive_scan<kWaves>((c.x + c.y + c.z + c.w) | (pc.x + pc.y + pc.z + pc.w) << 16, tmp);
    const uint32_t a3 = both & 0xFFFFu, a2 = a3 + c.w, a1 = a2 + c.z, a0 = a1 + c.y, all = a0 + c.x;
    reinterpret_cast<uint4 *>(lh)[low / 4] = make_uint4(a0, a1, a2, a3);
    // (counts of digit d and above: what the next lower digit begins with)
    *reinterpret_cast<uint2 *>(sfx + blk * kFine + low) = make_uint2(all | (a0 << 16), a1 | (a2 << 16));
    if (low % 64 == 0) csfx[blk * kCoarse + low / 64] = (uint16_t)all;
    if constexpr (LOOK) see(pc, (int)(both >> 16), REDUCE);
  };
  place(std::true_type{});
  __syncthreads();
  bool again = __builtin_amdgcn_readfirstlane(crowded) != 0;
  if (REDUCE && __builtin_expect(again, 0)) {  // what is crowded in plane 0 is looked at in the sums
    if (looks) probe = sum_of_parts(src, G, (int64_t)B * N, probe_at);
    reinterpret_cast<uint4 *>(probed)[t] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    if (t == 0) crowded = 0;
    count_probe();
    __syncthreads();
    const uint4 pc = reinterpret_cast<const uint4 *>(probed)[low / 4];
    see(pc, (int)block_exclusive_scan<kWaves>(pc.x + pc.y + pc.z + pc.w, tmp), false);
    __syncthreads();
    again = __builtin_amdgcn_readfirstlane(crowded) != 0;
  }
  if (__builtin_expect(again, 0)) {  // again, by the other digits
    // Sorted: every wave its 64 by counting, then each key its place among the others' runs.
    const int lane = t & 63, wv = t >> 6;
    uint32_t mine = 0, at = 0;
    if (t < kProbes) {
      mine = picked[t];
#pragma unroll 4
      for (int j = 0; j < 64; ++j) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)mine, j);
        at += o < mine || (o == mine && j < lane);
      }
      runs[wv * 64 + at] = mine;
    }
    reinterpret_cast<uint4 *>(lh)[t] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    if (t < kProbes) {
#pragma unroll 1
      for (int r = 1; r < kProbes / 64; ++r) {
        const int other = (wv + r) & (kProbes / 64 - 1);
        const uint32_t *run = runs + other * 64;
        const uint32_t past = other < wv ? 1u : 0u;  // equal keys of earlier runs come first
        int c = 0;
#pragma unroll
        for (int step = 32; step > 0; step >>= 1)
          if (run[c + step - 1] < mine || (past && run[c + step - 1] == mine)) c += step;
        c += run[c] < mine || (past && run[c] == mine);
        at += c;
      }
      splits[at] = at < kSplits ? mine : 0xFFFFFFFFu;
      // (and as a search tree, level by level: the reads of a level hit different banks)
      if (at < kSplits) tree[((at + 1) | kProbes) >> __ffs((int)(at + 1))] = mine;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      const uint32_t key[4] = {k4[s].x, k4[s].y, k4[s].z, k4[s].w};
      uint32_t node[4] = {1, 1, 1, 1};
#pragma unroll 1
      for (int level = kProbes / 2; level > 0; level >>= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) node[e] = 2 * node[e] + (tree[node[e]] < key[e]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t below = node[e] - kProbes;  // keys of `splits` that are smaller
        digit[4 * s + e] = 2 * below + (splits[below] == key[e]);
        rank[4 * s + e] = hist_rank(lh, digit[4 * s + e], (s * kThreads + t) * 4 < n);
      }
    }
    __syncthreads();
    place(std::false_type{});
    __syncthreads();
  }
  if (blockIdx.x == 0) {
    uint32_t *h = hdr + (size_t)b * kHeader;
    if (t == 0) h[0] = (uint32_t)crowded;
    if (t < kProbes) h[4 + t] = splits[t];
  }
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    if ((s * kThreads + t) * 4 < n) {
      const uint32_t key[4] = {k4[s].x, k4[s].y, k4[s].z, k4[s].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) sorted[lh[digit[4 * s + e]] + rank[4 * s + e]] = key[e];
    }
  }
  __syncthreads();
  uint4 *out = reinterpret_cast<uint4 *>(grouped + (int64_t)b * N + c0);
#pragma unroll
  for (int s = 0; s < SLOTS; ++s)
    if ((s * kThreads + t) * 4 < n) out[s * kThreads + t] = reinterpret_cast<const uint4 *>(sorted)[s * kThreads + t];
  side.finish(job, (int)(gridDim.x * gridDim.y * kThreads));
}

// The largest digit of 64 with at least `want` keys in it and above, counts[d] (LDS) of them from digit d on and
// `over` beyond the last digit; and how many keys lie above it.
__device__ __forceinline__ uint32_t pick(const uint32_t *counts, uint32_t want, uint32_t over, uint32_t &above, uint32_t &from) {
  const uint32_t tot = counts[threadIdx.x & 63];
  const uint64_t enough = __ballot(tot >= want);  // (monotone in the lane, and digit 0 has enough)
  const uint32_t digit = 63u - (uint32_t)__builtin_clzll(enough | 1u);
  from = (uint32_t)__builtin_amdgcn_readlane((int)tot, (int)digit);
  above = digit < 63 ? (uint32_t)__builtin_amdgcn_readlane((int)tot, (int)min(digit + 1, 63u)) : over;
  return digit;
}

// Second kernel, same grid.  jmap (nullable) gets the rank of every kept position and -1 for every dropped
// one; top_part, block_top as in select_emit_kernel (one value a workgroup).
// Bound by its chain: two table reads, the segments (1 us each, another die wrote them) and a dozen barriers.
template <int SLOTS>
__global__ __launch_bounds__(kThreads) void select_place_kernel(const float *__restrict__ norm, int64_t N, int64_t k,
                                                                const uint32_t *__restrict__ grouped,
                                                                const uint16_t *__restrict__ sfx,
                                                                const uint16_t *__restrict__ csfx, const uint32_t *__restrict__ hdr,
                                                                int32_t *__restrict__ idx, int32_t *__restrict__ jmap,
                                                                const float *__restrict__ top_part, int G, int B,
                                                                float *block_top) {
  constexpr int kChunk = 4 * kThreads * SLOTS;
  constexpr int kQuads = kSelectTwoBlocks / 64;  // a lane holds the segments of chunks 64 q + lane
  __shared__ __attribute__((aligned(16))) uint32_t lh[1 << kFieldBits];
  __shared__ uint32_t list[kListCap];
  __shared__ uint32_t bins[kSteps][64];
  __shared__ uint32_t counts[2][kCoarse];
  __shared__ uint32_t seg[kSelectTwoBlocks];
  __shared__ uint32_t head[kHeader];
  __shared__ uint32_t tmp[64];
  __shared__ uint32_t sums[2][kWaves];
  __shared__ uint32_t bcast[3];
  static_assert(4 * kWaves == 64, "four turns of the waves are 64 chunks");
  static_assert(kSelectTwoBlocks <= kThreads && kSelectTwoBlocks % 64 == 0, "a thread a chunk");
  const int b = blockIdx.y, t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int nblk = gridDim.x, mine = blockIdx.x;
  const int64_t c0 = (int64_t)mine * kChunk;
  const int n = (int)min((int64_t)kChunk, N - c0);
  const uint32_t *keys = reinterpret_cast<const uint32_t *>(norm) + (size_t)b * N + c0;
  sfx += (size_t)b * nblk * kFine;
  csfx += (size_t)b * nblk * kCoarse;
  grouped += (size_t)b * N;
  hdr += (size_t)b * kHeader;
  const uint32_t head_t = t < kHeader ? hdr[t] : 0u;  // (a scalar load would hold up every access to LDS)

  // rank k's coarse digit: every wave reads the tables of its share of the chunks, lane c the counts of coarse digit
  // c and above
  uint32_t v = 0;
#pragma unroll 8
  for (int i = wv; i < nblk; i += kWaves) v += csfx[(size_t)i * kCoarse + lane];
  // (what does not depend on the threshold travels under its computation)
  uint4 k4[SLOTS];
  float4 top4[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int at = (s * kThreads + t) * 4;
    k4[s] = make_uint4(0, 0, 0, 0);
    top4[s] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (at < n) {
      k4[s] = *reinterpret_cast<const uint4 *>(keys + at);
      if (top_part) top4[s] = load_top(top_part, G, (int64_t)B * N, (int64_t)b * N + c0 + at);
    }
  }
  if (t < kHeader) head[t] = head_t;
  for (int i = t; i < 2 * kCoarse; i += kThreads) (&counts[0][0])[i] = 0;
  for (int i = t; i < kSteps * 64; i += kThreads) (&bins[0][0])[i] = 0;
  workgroup_lds_barrier();
  if (wv < nblk) atomicAdd(&counts[0][lane], v);
  workgroup_lds_barrier();
  uint32_t over, from;
  const uint32_t coarse = pick(counts[0], (uint32_t)k, 0u, over, from);
  v = 0;
#pragma unroll 8
  for (int i = wv; i < nblk; i += kWaves) v += sfx[(size_t)i * kFine + 64 * coarse + lane];
  if (wv < nblk) atomicAdd(&counts[1][lane], v);
  workgroup_lds_barrier();
  const uint32_t D = 64 * coarse + pick(counts[1], (uint32_t)k, over, over, from);
  uint32_t r_take = (uint32_t)k - over;  // rank among the keys with digit D
  const uint32_t M = from - over;        // how many there are

  // every chunk's segment of them: keys above digit D in the chunk | keys with digit D << 16
  if (t < nblk) {
    const uint32_t hi = D + 1 < kFine ? sfx[(size_t)t * kFine + D + 1] : 0u;
    seg[t] = hi | ((uint32_t)sfx[(size_t)t * kFine + D] - hi) << 16;
  }
  workgroup_lds_barrier();
  // ... and where its keys begin among all of digit D (every wave for itself, lane l the chunks 64 q + l)
  uint32_t sg[kQuads], off[kQuads], above = 0, total = 0, off_mine = 0;
#pragma unroll
  for (int q = 0; q < kQuads; ++q) {
    sg[q] = off[q] = 0;
    if (64 * q < nblk) {
      const int i = 64 * q + lane;
      if (i < nblk) sg[q] = seg[i];
      const uint32_t c = sg[q] >> 16, upto = wave_inclusive_scan(c);
      off[q] = total + upto - c;
      if (mine >> 6 == q) off_mine = (uint32_t)__builtin_amdgcn_readlane((int)off[q], mine & 63);
      total += (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
      if (wv == 0 && i < mine) above += sg[q] & 0xFFFFu;  // keys above digit D in the chunks before this one
    }
  }
  // the threshold key: its bits from `hi` up are the same in all keys with digit D; `alone`: digit D is one key
  uint32_t T = 0;
  int hi = 32;
  bool alone = D == 0;
  const uint32_t *splits = head + 4;
  if (head[0] == 0) {
    if (D != 0 && D != 1 && D != kFine - 1) {
      hi = kStepBits;
      T = (D + kBase) << kStepBits;
    }
  } else {
    const uint32_t j = D >> 1;
    alone = D & 1;
    T = splits[j];
    if (!alone) {  // keys in [low, top]
      const uint32_t low = j > 0 ? splits[j - 1] + 1 : 0u, top = j < kSplits ? T - 1 : 0xFFFFFFFFu;
      hi = low == top ? 0 : 32 - __builtin_clz(low ^ top);
      T = hi < 32 ? low >> hi << hi : 0u;
    }
  }
  v = 0;  // keys equal to T in the chunks before this one
  if (!alone) {
    // The list holds the keys that agree with T so far: `before` of chunks before this one at its start, `rest` others
    // from rest_at on.
    uint32_t before = off_mine, rest = M - off_mine, rest_at = off_mine;
    if (M <= kListCap) {
      // (four chunks' loads together: most segments are shorter than a wave)
#pragma unroll
      for (int q = 0; q < kQuads; ++q) {
        if (64 * q >= nblk) continue;
        uint32_t first[4], m[4], to[4];
        const uint32_t *p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = wv + u * kWaves;  // (chunks past the last one have no keys)
          const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)sg[q], i);
          m[u] = w >> 16;
          to[u] = (uint32_t)__builtin_amdgcn_readlane((int)off[q], i);
          p[u] = grouped + (size_t)(64 * q + i) * kChunk + (w & 0xFFFFu);
          first[u] = (uint32_t)lane < m[u] ? p[u][lane] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if ((uint32_t)lane < m[u]) list[to[u] + lane] = first[u];
      }
      // (what is longer, eight loads in flight; one loop for all of it: its instructions are fetched even where it does not run)
      if (__ballot(max(max(sg[0], sg[1]), max(sg[2], sg[3])) >> 16 > 64) != 0) {
        static_assert(kQuads == 4, "");
#pragma unroll 1
        for (int i = wv; i < nblk; i += kWaves) {
          const int q = i >> 6;
          const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)(q < 2 ? (q ? sg[1] : sg[0]) : q == 2 ? sg[2] : sg[3]), i & 63);
          const uint32_t to = (uint32_t)__builtin_amdgcn_readlane((int)(q < 2 ? (q ? off[1] : off[0]) : q == 2 ? off[2] : off[3]), i & 63);
          const uint32_t *p = grouped + (size_t)i * kChunk + (w & 0xFFFFu);
          const uint32_t m = w >> 16;
#pragma unroll 1
          for (uint32_t e0 = 64; e0 < m; e0 += 8 * 64) {
            uint32_t more[8];
#pragma unroll
            for (int x = 0; x < 8; ++x) more[x] = p[min(e0 + x * 64 + lane, m - 1)];
#pragma unroll
            for (int x = 0; x < 8; ++x)
              if (e0 + x * 64 + lane < m) list[to + e0 + x * 64 + lane] = more[x];
          }
        }
      }
      workgroup_lds_barrier();
    } else {
      // f(key, chunk) for every key with digit D in the sample's first `blocks` chunks, from memory
      auto stream = [&](int blocks, auto &&f) {
#pragma unroll
        for (int q = 0; q < kQuads; ++q)
          for (int i = 64 * q + wv; i < min(64 * q + 64, blocks); i += kWaves) {
            // (whole quads, four in flight a lane: bound by the latency of these loads)
            const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)sg[q], i & 63), at = w & 0xFFFFu, end = at + (w >> 16);
            const uint4 *p = reinterpret_cast<const uint4 *>(grouped + (size_t)i * kChunk);
            for (uint32_t e0 = at / 4; e0 * 4 < end; e0 += 4 * 64) {
              uint4 k4s[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) k4s[u] = p[min(e0 + u * 64 + lane, (end - 1) / 4)];
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const uint32_t e = (e0 + u * 64 + lane) * 4;
                const uint32_t key[4] = {k4s[u].x, k4s[u].y, k4s[u].z, k4s[u].w};
#pragma unroll
                for (int x = 0; x < 4; ++x)
                  if (e + x >= at && e + x < end) f(key[x], i);
              }
            }
          }
      };
      uint32_t left = M;
      for (bool first = true; hi > 0 && left > kListCap; first = false) {
        const int lo = max(hi - kFieldBits, 0);
        const uint32_t fmask = (1u << (hi - lo)) - 1u;
        reinterpret_cast<uint4 *>(lh)[t] = make_uint4(0, 0, 0, 0);
        __syncthreads();  // (and bcast has been read)
        stream(nblk, [&](uint32_t key, int) { hist_add_spread(lh, (key >> lo) & fmask, first || (key >> hi) == (T >> hi)); });
        __syncthreads();
        const int low = (1 << kFieldBits) - 4 - 4 * t;
        const uint4 c4 = reinterpret_cast<const uint4 *>(lh)[low / 4];
        const uint32_t c[4] = {c4.w, c4.z, c4.y, c4.x};
        uint32_t upto = block_exclusive_scan<kWaves>(c4.x + c4.y + c4.z + c4.w, tmp);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (upto < r_take && r_take <= upto + c[i]) {  // (1 <= r_take <= keys that agree: one thread's bin)
            bcast[0] = T | ((uint32_t)(low + 3 - i) << lo);
            bcast[1] = r_take - upto;
            bcast[2] = c[i];
          }
          upto += c[i];
        }
        __syncthreads();
        T = bcast[0];
        r_take = bcast[1];
        left = bcast[2];
        hi = lo;
      }
      if (hi > 0) {
        if (t < 2) tmp[t] = 0;
        __syncthreads();
        stream(nblk, [&](uint32_t key, int i) {
          if ((key >> hi) == (T >> hi)) {
            if (i < mine) list[atomicAdd(&tmp[0], 1u)] = key;
            else list[kListCap - 1 - atomicAdd(&tmp[1], 1u)] = key;
          } else if (i < mine) {
            above += key > T;
          }
        });
        __syncthreads();
        before = tmp[0];
        rest = tmp[1];
        rest_at = kListCap - rest;
      } else {
        stream(mine, [&](uint32_t key, int) { above += key > T; v += key == T; });
        before = rest = 0;
      }
    }
    // six bits a step, each step in bins of its own; every wave picks the digit for itself
#pragma unroll 1
    for (int step = 0; hi > 0; ++step) {
      const int lo = max(hi - 6, 0);
      const uint32_t fmask = (1u << (hi - lo)) - 1u;
      for (uint32_t i = t; i < before + rest; i += kThreads) {
        const uint32_t key = list[i < before ? i : rest_at + (i - before)];
        hist_add_spread(bins[step], (key >> lo) & fmask, step == 0 || (key >> hi) == (T >> hi));
      }
      workgroup_lds_barrier();
      const uint32_t c = bins[step][63 - lane];  // from the top
      const uint32_t upto = wave_inclusive_scan(c);
      const int at = __ffsll((unsigned long long)__ballot(upto >= r_take)) - 1;  // (r_take <= keys that agree: a lane has it)
      r_take -= (uint32_t)__builtin_amdgcn_readlane((int)(upto - c), at);
      T |= (63u - (uint32_t)at) << lo;
      hi = lo;
    }
    // what the chunks before this one keep: everything above digit D, and of digit D what is above T or equal
    for (uint32_t i = t; i < before; i += kThreads) {
      const uint32_t key = list[i];
      above += key > T;
      v += key == T;
    }
  } else {
    v = t == 0 ? off_mine : 0u;
  }
  above = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(above), 63);
  v = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(v), 63);
  if (lane == 0) { sums[0][wv] = above; sums[1][wv] = v; }
  workgroup_lds_barrier();  // (tmp is written again below)

  // ordered compaction as in select_small_kernel: slot-major, then thread, then the four keys of a slot; counts
  // packed (above T | equal to T) in 16 + 16 bits
  uint32_t ex[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const uint32_t key[4] = {k4[s].x, k4[s].y, k4[s].z, k4[s].w};
    uint32_t packed = 0;
    if ((s * kThreads + t) * 4 < n) {
#pragma unroll
      for (int e = 0; e < 4; ++e) packed += ((key[e] > T) << 16) + (key[e] == T);
    }
    const uint32_t inc = wave_inclusive_scan(packed);
    ex[s] = inc - packed;
    if (lane == 63) tmp[s * kWaves + wv] = inc;
  }
  workgroup_lds_barrier();
  static_assert(SLOTS * kWaves <= 64, "one wave scans the totals");
  if (t < 64) {
    const uint32_t x = t < SLOTS * kWaves ? tmp[t] : 0u;
    tmp[t] = wave_inclusive_scan(x) - x;
  }
  uint32_t gt0 = 0, eq0 = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) { gt0 += sums[0][i]; eq0 += sums[1][i]; }
  workgroup_lds_barrier();

  float kept_top = 0.f;
  int32_t *out = idx + (size_t)b * k;
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int at = (s * kThreads + t) * 4;
    if (at < n) {
      const uint32_t before = tmp[s * kWaves + wv] + ex[s];
      uint32_t gt = gt0 + (before >> 16), eq = eq0 + (before & 0xFFFFu);
      const uint32_t key[4] = {k4[s].x, k4[s].y, k4[s].z, k4[s].w};
      const float top[4] = {top4[s].x, top4[s].y, top4[s].z, top4[s].w};
      const int64_t q = c0 + at;
      int32_t jm[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool is_gt = key[e] > T, is_eq = key[e] == T;
        const bool keep = is_gt || (is_eq && eq < r_take);
        const uint32_t j = gt + min(eq, r_take);
        if (keep) out[j] = (int32_t)(q + e);
        jm[e] = keep ? (int32_t)j : -1;
        kept_top = fmaxf(kept_top, keep ? top[e] : 0.f);
        gt += is_gt; eq += is_eq;
      }
      if (jmap) *reinterpret_cast<int4 *>(jmap + (size_t)b * N + q) = make_int4(jm[0], jm[1], jm[2], jm[3]);
    }
  }
  if (top_part)  // (uniform over the grid)
    publish_top<kWaves>(kept_top, block_top, (size_t)b * nblk + mine, tmp);
}

// Crowded: a digit with some 16384 keys, half of what the second
// kernel's list takes, but at least what six (three) of the quads hold, which may be neighbours of one value.
Probes probes_of(int64_t N, int64_t k) {
  Probes p{N > 1 << 17 ? kProbes : kProbes / 4, 0, 0, 0, 0};
  p.quads = (uint32_t)(N / 4 / p.n);
  p.crowd = std::max<uint32_t>(std::max(12, p.n * 24 / kProbes), (uint32_t)((int64_t)p.n * 4 * 16384 / N));
  const int rank = (int)((int64_t)p.n * 4 * k / N), slack = p.n / 4;  // (two deviations of the median of 256 quads of equal keys)
  p.from = rank - slack;
  p.to = rank + slack;
  return p;
}

template <int SLOTS>
hipError_t launch(const wcc_desc &d, const float *norm_or_part, int G, float *norm_out, int64_t k, uint32_t *grouped,
                  uint16_t *sfx, uint16_t *csfx, uint32_t *hdr, int nblk, int32_t *idx, int32_t *jmap, const float *top_part,
                  float *block_top, const PackJob &job, hipStream_t s) {
  const int64_t N = (int64_t)d.H * d.W;
  const Probes look = probes_of(N, k);
  const dim3 grid(nblk, d.B), block(kThreads);
  const float *norm = G > 1 ? norm_out : norm_or_part;
  if (G > 1)
    hipLaunchKernelGGL((select_group_kernel<true, SLOTS>), grid, block, 0, s, norm_or_part, norm_out, G, N, d.B, grouped,
                       sfx, csfx, hdr, look, job);
  else
    hipLaunchKernelGGL((select_group_kernel<false, SLOTS>), grid, block, 0, s, norm_or_part, nullptr, 1, N, d.B, grouped,
                       sfx, csfx, hdr, look, job);
  hipLaunchKernelGGL((select_place_kernel<SLOTS>), grid, block, 0, s, norm, N, k, grouped, sfx, csfx, hdr, idx, jmap, top_part,
                     G, d.B, block_top);
  return hipGetLastError();
}

}  // namespace

size_t select_two_bytes(int B, int nblk) { return (size_t)B * nblk * (kFine + kCoarse) * 2 + (size_t)B * kHeader * 4; }
int select_two_chunk(int slots) { return 4 * kThreads * slots; }

hipError_t launch_select_two(const wcc_desc &d, const float *norm_or_part, int G, float *norm_out, int64_t k,
                             void *tables, uint32_t *grouped, int slots, int nblk, int32_t *idx, int32_t *jmap,
                             const float *top_part, float *block_top, const PackJob &job, hipStream_t s) {
  uint16_t *sfx = static_cast<uint16_t *>(tables), *csfx = sfx + (size_t)d.B * nblk * kFine;
  uint32_t *hdr = reinterpret_cast<uint32_t *>(csfx + (size_t)d.B * nblk * kCoarse);
  switch (slots) {
    case 4: return launch<4>(d, norm_or_part, G, norm_out, k, grouped, sfx, csfx, hdr, nblk, idx, jmap, top_part, block_top, job, s);
    case 2: return launch<2>(d, norm_or_part, G, norm_out, k, grouped, sfx, csfx, hdr, nblk, idx, jmap, top_part, block_top, job, s);
    default: return launch<1>(d, norm_or_part, G, norm_out, k, grouped, sfx, csfx, hdr, nblk, idx, jmap, top_part, block_top, job, s);
  }
}

}  // namespace wcc
