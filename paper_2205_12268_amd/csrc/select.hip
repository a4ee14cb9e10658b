// Joint shrinkage (Alg. 1: the index set I holds the k = ceil(gamma n_w n_h) positions whose
// channel vectors have the largest norm):
// per sample, the k largest of N non-negative fp32 norms, ties toward the lower position,
// emitted in ascending position order.
//
// Design.  Non-negative floats order like their bit patterns, so the k-th largest norm is
// found exactly by a most-significant-digit radix select on uint32 keys: three histogram
// passes (11 + 11 + 10 bits) spread over many workgroups per sample, integer atomics only.
// Every workgroup of the NEXT kernel turns the finished histogram of the previous pass into
// the digit to descend into by itself (an 8 KiB read and one block scan): no workgroup waits
// for another and no device-wide fence is needed -- on this chip such a fence writes back a
// whole L2, which costs more than the pass.  The third pass also leaves, per workgroup, the
// suffix sums of its own low-digit histogram; once the threshold key T is known they give every workgroup's count of keys
// above T and equal to T without another pass over the keys.  The last kernel is an ordered
// compaction: a position is kept if key > T, or key == T and fewer than r equal keys precede
// it (r = how many keys equal to T are still needed).  Ordering comes from prefix sums,
// never from the arrival order of atomics, so the result is the same on every run.
// The first pass can take the channel-group partial norms of the forward transform and
// reduce them on the fly (fixed order), writing the final norms as a by-product.
// Planes of middling size take the two launches of select_two.hip instead (the rule is in ws_layout).
#include "select_dev.h"

namespace wcc {
namespace {

constexpr int kThreads = 256;                  // 4 waves
constexpr int kWaves = kThreads / 64;
constexpr int kPer = kSelectChunk / kThreads;  // 4 keys per thread
static_assert(kPer == 4, "one 16-byte load per thread");

__device__ __forceinline__ uint32_t digit_of(uint32_t key, int pass) {
  return pass == 0 ? key >> 21 : pass == 1 ? (key >> 10) & 0x7FFu : key & 0x3FFu;
}
// keys whose bits above the current digit equal those of `prefix`
__device__ __forceinline__ bool matches(uint32_t key, uint32_t prefix, int pass) {
  return pass == 0 ? true : pass == 1 ? (key >> 21) == (prefix >> 21) : (key >> 10) == (prefix >> 10);
}

__global__ __launch_bounds__(256) void select_init_kernel(SelectPrep p, int B) {
  if ((int)blockIdx.x < B) prep_sample(p, blockIdx.x, threadIdx.x, blockDim.x);
}

// Turns the finished histogram of pass P into the digit that holds the remaining rank:
// the digit D with count(> D) < remain <= count(>= D), scanning from the top digit down.
// Every thread returns the same (prefix, remain) for the next pass.
template <int P, int THREADS = kThreads>
__device__ __forceinline__ void pick_digit(const uint32_t *gh, uint32_t &prefix,
                                           uint32_t &remain, uint32_t *tmp, uint32_t *bcast) {
  constexpr int bins = P == 2 ? 1024 : kRadixBins;
  constexpr int per = bins / THREADS;  // consecutive digits per thread, from the top
  const int t = threadIdx.x;
  uint32_t cnt[per], sum = 0;
#pragma unroll
  for (int i = 0; i < per; ++i) {
    cnt[i] = gh[bins - 1 - (t * per + i)];
    sum += cnt[i];
  }
  uint32_t above = block_exclusive_scan<THREADS / 64>(sum, tmp);
#pragma unroll
  for (int i = 0; i < per; ++i) {
    if (above < remain && remain <= above + cnt[i]) {
      const uint32_t digit = bins - 1 - (t * per + i);
      bcast[0] = prefix | (P == 0 ? digit << 21 : P == 1 ? digit << 10 : digit);
      bcast[1] = remain - above;
    }
    above += cnt[i];
  }
  __syncthreads();
  prefix = bcast[0];
  remain = bcast[1];
  __syncthreads();
}

// (prefix, remain) after passes 0..UPTO-1: earlier picks come from the state (stored by a
// previous kernel), the newest one is computed here from the histogram that kernel finished.
template <int UPTO>
__device__ __forceinline__ void current_state(const uint32_t *hist_b, SelectState *s,
                                              uint32_t k, uint32_t &prefix, uint32_t &remain,
                                              uint32_t *tmp, uint32_t *bcast, bool store) {
  prefix = 0;
  remain = k;
  if constexpr (UPTO == 0) return;
  if constexpr (UPTO >= 2) {
    prefix = s->prefix[UPTO - 2];
    remain = s->remain[UPTO - 2];
  }
  if (threadIdx.x == 0) { bcast[0] = prefix; bcast[1] = remain; }  // rank beyond the data: unchanged
  __syncthreads();
  pick_digit<UPTO - 1>(hist_b + (size_t)(UPTO - 1) * kRadixBins, prefix, remain, tmp, bcast);
  if (store && threadIdx.x == 0) {
    s->prefix[UPTO - 1] = prefix;
    s->remain[UPTO - 1] = remain;
  }
}

// One histogram pass.  grid = (nblk, B), block = 256.
// PASS 0 with REDUCE reads partial norms `src` [G, B, N] and writes `norm`; otherwise src is
// the norm array itself.  PASS 2 also writes this workgroup's suffix sums and its count of
// keys above the 22-bit prefix.  PASS 0 also carries out `job`.
// SLOTS: 16-byte loads per thread (a workgroup takes 1024 * SLOTS keys; slot s of thread t
// covers the four positions from (s * 256 + t) * 4 on inside the workgroup's chunk).
template <int PASS, bool REDUCE, int SLOTS>
__global__ __launch_bounds__(kThreads) void select_hist_kernel(const float *__restrict__ src,
                                                               float *__restrict__ norm, int G,
                                                               int64_t N, int B, uint32_t k,
                                                               uint32_t *hist, SelectState *st,
                                                               int nblk,
                                                               uint16_t *__restrict__ block_sfx,
                                                               uint32_t *__restrict__ block_gthi,
                                                               PackJob job) {
  constexpr int bins = PASS == 2 ? 1024 : kRadixBins;
  __shared__ uint32_t lh[kRadixBins];
  __shared__ uint32_t tmp[kWaves];
  __shared__ uint32_t bcast[2];
  const int b = blockIdx.y, t = threadIdx.x;
  uint32_t *hist_b = hist + (size_t)b * 3 * kRadixBins;
  uint32_t *gh = hist_b + (size_t)PASS * kRadixBins;

  for (int i = t; i < bins; i += kThreads) lh[i] = 0;
  // the keys do not depend on the digit picked below: their load travels under it
  const int64_t q0 = (int64_t)blockIdx.x * (kSelectChunk * SLOTS) + (int64_t)t * kPer;
  uint4 k4[SLOTS];
#pragma unroll
  for (int sl = 0; sl < SLOTS; ++sl) {
    const int64_t q = q0 + (int64_t)sl * kSelectChunk;
    k4[sl] = make_uint4(0, 0, 0, 0);  // N is a multiple of 4: a slot's four keys are all in or all out
    if (q < N) k4[sl] = load_keys<REDUCE>(src, norm, G, (int64_t)B * N, (int64_t)b * N + q);
  }
  const int first_piece = (int)((blockIdx.y * gridDim.x + blockIdx.x) * kThreads + t);
  const PackOnTheSide side(job, PASS == 0 ? first_piece : job.total);
  uint32_t prefix, remain;
  current_state<PASS>(hist_b, st + b, k, prefix, remain, tmp, bcast, blockIdx.x == 0);
  __syncthreads();
  uint32_t above = 0;
#pragma unroll
  for (int sl = 0; sl < SLOTS; ++sl) {
    const bool in = q0 + (int64_t)sl * kSelectChunk < N;
    const uint32_t key[4] = {k4[sl].x, k4[sl].y, k4[sl].z, k4[sl].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      hist_add(lh, digit_of(key[e], PASS), in && matches(key[e], prefix, PASS));
      if (PASS == 2) above += (in && (key[e] >> 10) > (prefix >> 10)) ? 1u : 0u;
    }
  }
  __syncthreads();
  for (int i = t; i < bins; i += kThreads) {
    const uint32_t v = lh[i];
    if (v) atomicAdd(&gh[i], v);
  }
  if constexpr (PASS == 0) side.finish(job, (int)(gridDim.x * gridDim.y * kThreads));
  if constexpr (PASS == 2) {
    // sfx[d] = number of this workgroup's matching keys with low digit >= d
    constexpr int per = bins / kThreads;  // 4 digits per thread, from the top
    uint32_t c[per], sum = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
      c[i] = lh[bins - 1 - (t * per + i)];
      sum += c[i];
    }
    uint32_t run = block_exclusive_scan<kWaves>(sum, tmp);
    const size_t blk = (size_t)b * nblk + blockIdx.x;
#pragma unroll
    for (int i = 0; i < per; ++i) {
      run += c[i];
      block_sfx[blk * kSfxStride + (bins - 1 - (t * per + i))] = (uint16_t)run;
    }
    const uint32_t tot_above = block_sum<kWaves>(above, tmp);
    if (t == 0) block_gthi[blk] = tot_above;
  }
}

// Ordered compaction.  grid = (nblk, B), block = 256.  jmap (nullable) gets the rank of
// every kept position and -1 for every dropped one.  top_part (nullable, [G, B, N]): the largest
// |coefficient| over the channels at every position; its maximum over the positions this
// workgroup keeps goes to block_top[b, blockIdx.x] (the largest of those is the layer's clipping
// parameter alpha).
template <int SLOTS>
__global__ __launch_bounds__(kThreads) void select_emit_kernel(const float *__restrict__ norm,
                                                               int64_t N, int64_t k,
                                                               const uint32_t *__restrict__ hist,
                                                               SelectState *st,
                                                               const uint16_t *__restrict__ block_sfx,
                                                               const uint32_t *__restrict__ block_gthi,
                                                               int nblk, int32_t *__restrict__ idx,
                                                               int32_t *__restrict__ jmap,
                                                               const float *__restrict__ top_part,
                                                               int G, int B, float *block_top) {
  __shared__ uint32_t tmp[kWaves];
  __shared__ uint32_t bcast[2];
  const int b = blockIdx.y, t = threadIdx.x;
  const uint32_t *keys = reinterpret_cast<const uint32_t *>(norm) + (size_t)b * N;
  // (the keys do not depend on the threshold: their load travels under its computation)
  const int64_t q0 = (int64_t)blockIdx.x * (kSelectChunk * SLOTS) + (int64_t)t * kPer;
  uint4 k4[SLOTS];
  float4 top4[SLOTS];
#pragma unroll
  for (int sl = 0; sl < SLOTS; ++sl) {
    const int64_t q = q0 + (int64_t)sl * kSelectChunk;
    k4[sl] = make_uint4(0, 0, 0, 0);
    top4[sl] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (q < N) {
      k4[sl] = *reinterpret_cast<const uint4 *>(keys + q);
      if (top_part) top4[sl] = load_top(top_part, G, (int64_t)B * N, (int64_t)b * N + q);
    }
  }
  uint32_t T, r_take;  // threshold key, and how many keys equal to it are still needed
  current_state<3>(hist + (size_t)b * 3 * kRadixBins, st + b, (uint32_t)k, T, r_take, tmp, bcast,
                   blockIdx.x == 0);
  const uint32_t tlow = T & 0x3FFu;

  // keys above / equal to T in the workgroups before this one
  uint32_t gt0 = 0, eq0 = 0;
  for (int i = t; i < (int)blockIdx.x; i += kThreads) {
    const size_t blk = (size_t)b * nblk + i;
    const uint32_t ge = block_sfx[blk * kSfxStride + tlow];
    const uint32_t gtl = tlow + 1 < 1024 ? block_sfx[blk * kSfxStride + tlow + 1] : 0u;
    gt0 += block_gthi[blk] + gtl;
    eq0 += ge - gtl;
  }
  gt0 = block_sum<kWaves>(gt0, tmp);
  eq0 = block_sum<kWaves>(eq0, tmp);

  // Position order inside the workgroup's chunk is slot by slot, thread by thread: one block
  // scan a slot, on top of the totals of the slots before it.  Counts are packed
  // hi16: keys above T, lo16: keys equal to T (each <= 4096 a workgroup).
  float kept_top = 0.f;
  int32_t *out = idx + (size_t)b * k;
#pragma unroll
  for (int sl = 0; sl < SLOTS; ++sl) {
    const int64_t q = q0 + (int64_t)sl * kSelectChunk;
    const bool in = q < N;
    const uint32_t key[4] = {k4[sl].x, k4[sl].y, k4[sl].z, k4[sl].w};
    uint32_t packed = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (in) packed += ((key[e] > T) << 16) + (key[e] == T);
    const uint32_t ex = block_exclusive_scan<kWaves>(packed, tmp);
    uint32_t gt = gt0 + (ex >> 16), eq = eq0 + (ex & 0xFFFFu);
    if (SLOTS > 1) {  // the slot's totals (tmp holds the waves' inclusive sums until the next scan)
      uint32_t tot = 0;
#pragma unroll
      for (int i = 0; i < kWaves; ++i) tot += tmp[i];
      gt0 += tot >> 16;
      eq0 += tot & 0xFFFFu;
    }
    if (in) {
      const float top[4] = {top4[sl].x, top4[sl].y, top4[sl].z, top4[sl].w};
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
    publish_top<kWaves>(kept_top, block_top, (size_t)b * nblk + blockIdx.x, tmp);
}

// ---- small planes: the whole select of one sample in ONE workgroup -------------------------
// For N <= 16384 the kernels above are launch gaps and little else.  Here one workgroup of
// 1024 threads holds all keys of a sample in registers (slot s of thread t covers the four
// positions from (s * 1024 + t) * 4 on: every load is one contiguous 16 KiB row), finds the
// threshold and emits idx and jmap in position order.  Same result, bit for bit.
//
// With all keys in one place the digits need not be raw bit fields: the passes work on
// rel = key - min(keys), whose significant bits (those of max - min) are cut into fields of at
// most 13 bits from the top.  Norms of one plane share their upper exponent bits, so the raw
// top field would put nearly all keys into a handful of bins and the LDS atomics of the 16
// waves would serialise on them; the relative top field spreads them over the whole histogram.
// After a pass the keys that still matter are those of one bin.  They are few (a handful of 2048
// keys in 8192 bins, or one class of equal keys): up to kSmallList of them go to a list in LDS, and
// every entry counts the entries above it; only more than that take another pass.
// Bound by its own chain: the loads, then a barrier behind every step.  Fields of 11 bits, always
// as many passes as there are bits, and loads one slot after the other took 9.5-13 us on the eleven
// small layers of the 16-layer stack (6-9.7 now) and 12.4 us on 16384 positions (10.5).
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallSlots = 4;  // 16-byte loads per thread at most (beyond that the one
                                // workgroup is slower than the spread-out kernels)
static_assert(kSmallMaxN == (int64_t)4 * kSmallSlots * kSmallThreads, "one workgroup's keys");
constexpr int kSmallBits = 13;  // bits of a field
constexpr int kSmallBins = 1 << kSmallBits;
constexpr uint32_t kSmallList = 512;

// The G partial planes summed (and their maxima taken) by the whole chip before the one-workgroup-a-sample kernel below, or
// the two-launch selection: with many groups these would otherwise read G x N values per sample through one or a few
// compute units.  grid = (ceil(N / 1024), B), block = 256.
// The maxima land in group 0's plane of top_part (each position is read and written by one thread).
__global__ __launch_bounds__(256) void combine_parts_kernel(const float *__restrict__ part,
                                                            float *__restrict__ norm, int G, int64_t N,
                                                            int B, float *top_part) {
  const int64_t pos = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (pos >= N) return;
  const int64_t at = (int64_t)blockIdx.y * N + pos;
  load_keys<true>(part, norm, G, (int64_t)B * N, at);
  if (top_part) *reinterpret_cast<float4 *>(top_part + at) = load_top(top_part, G, (int64_t)B * N, at);
}

// The partial planes (sums and maxima) are combined first from this many values a sample on: below
// that the extra launch (5 us) costs more than the one workgroup's reads (16384 positions in 8
// groups, 262144 values: 25 us alone, 5 + 12 us combined first)
constexpr int64_t kCombineValues = 1 << 17;
// ... and in front of the two-launch selection from this many planes on: its few workgroups of 1024 threads read them one after
// another, and the maxima again (44800 positions in 256 planes: 118 us, 68 combined first; 20736 in 128 55 and 41; 18432 in 32 22.3 and
// 20.0; below that it loses, 65536 x 2 in 16 planes 5 us)
constexpr int kCombineTwo = 32;

// grid = B, block = 1024.  SLOTS: loads a thread (1, 2 or 4).  REDUCE as in load_keys.
template <bool REDUCE, int SLOTS>
__global__ __launch_bounds__(kSmallThreads) void select_small_kernel(
    const float *__restrict__ src, int G, int64_t N, int B, uint32_t k,
    int32_t *__restrict__ idx, int32_t *__restrict__ jmap,
    const float *__restrict__ top_part, float *block_top, PackJob job) {
  __shared__ __attribute__((aligned(16))) uint32_t lh[kSmallBins];
  __shared__ __attribute__((aligned(16))) uint32_t list[kSmallList];
  __shared__ uint32_t ends[2 * kSmallWaves];
  __shared__ uint32_t tmp[kSmallSlots * kSmallWaves];
  __shared__ uint32_t bcast[4];  // prefix, remaining rank, keys in the bin, entries in the list
  fetch_args(src, job.total);
  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t BN = (int64_t)B * N;
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < kSmallBins / 4 / kSmallThreads; ++i)
      reinterpret_cast<uint4 *>(lh)[i * kSmallThreads + t] = make_uint4(0, 0, 0, 0);
    if (t == 0) bcast[3] = 0;
  };

  // All loads of all slots go out together, without a branch around any of them: a slot outside
  // the plane (N is a multiple of 4: whole slots) reads the plane's last four values.
  int64_t at[SLOTS];
  uint32_t vmask = 0;  // bit s: slot s of this thread lies inside the plane
  float4 v[SLOTS], m[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int64_t pos = ((int64_t)s * kSmallThreads + t) * 4;
    vmask |= (pos < N ? 1u : 0u) << s;
    at[s] = (int64_t)b * N + min(pos, N - 4);
    v[s] = *reinterpret_cast<const float4 *>(src + at[s]);
  }
  if (top_part) {  // (uniform over the grid)
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) m[s] = *reinterpret_cast<const float4 *>(top_part + at[s]);
  } else {
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) m[s] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const PackOnTheSide side(job, (int)blockIdx.x * kSmallThreads + t);
  clear();
  if constexpr (REDUCE) {
    constexpr int PL = 4 / SLOTS;  // planes a round: four loads in flight of each kind
    for (int g = 1; g < G; g += PL) {
      float4 a[PL][SLOTS], c[PL][SLOTS];
#pragma unroll
      for (int i = 0; i < PL; ++i)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
          a[i][s] = *reinterpret_cast<const float4 *>(src + (int64_t)min(g + i, G - 1) * BN + at[s]);
      if (top_part) {
#pragma unroll
        for (int i = 0; i < PL; ++i)
#pragma unroll
          for (int s = 0; s < SLOTS; ++s)
            c[i][s] = *reinterpret_cast<const float4 *>(top_part + (int64_t)min(g + i, G - 1) * BN + at[s]);
      }
#pragma unroll
      for (int i = 0; i < PL; ++i) {
        if (g + i < G) {  // (uniform) added in increasing group order
#pragma unroll
          for (int s = 0; s < SLOTS; ++s) {
            v[s].x += a[i][s].x; v[s].y += a[i][s].y; v[s].z += a[i][s].z; v[s].w += a[i][s].w;
            if (top_part) {
              m[s].x = fmaxf(m[s].x, c[i][s].x); m[s].y = fmaxf(m[s].y, c[i][s].y);
              m[s].z = fmaxf(m[s].z, c[i][s].z); m[s].w = fmaxf(m[s].w, c[i][s].w);
            }
          }
        }
      }
    }
  }
  uint32_t rel[4 * SLOTS];
  float topv[4 * SLOTS];  // largest |coefficient| over the channels at the key's position
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const uint32_t k4[4] = {__float_as_uint(v[s].x), __float_as_uint(v[s].y), __float_as_uint(v[s].z),
                            __float_as_uint(v[s].w)};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      rel[4 * s + e] = k4[e];
      kmin = min(kmin, k4[e]);  // (the values a slot outside repeats are the plane's own)
      kmax = max(kmax, k4[e]);
    }
    topv[4 * s] = m[s].x; topv[4 * s + 1] = m[s].y; topv[4 * s + 2] = m[s].z; topv[4 * s + 3] = m[s].w;
  }
  // smallest and largest key of the sample
  kmin = wave_extreme<false>(kmin);
  kmax = wave_extreme<true>(kmax);
  if (lane == 0) { ends[wv] = kmin; ends[kSmallWaves + wv] = kmax; }
  __syncthreads();  // (and the histogram is clear)
#pragma unroll
  for (int i = 0; i < kSmallWaves; ++i) {
    kmin = min(kmin, ends[i]);
    kmax = max(kmax, ends[kSmallWaves + i]);
  }
#pragma unroll
  for (int i = 0; i < 4 * SLOTS; ++i) rel[i] -= kmin;

  // T: the threshold (relative key); r_take: how many keys equal to it to take.  The bits of T from
  // `hi` up are fixed.
  uint32_t T = 0, r_take = k;
  int hi = 32 - __clz((int)(kmax - kmin));  // 0 when all keys are equal (clz(0) = 32)
  for (bool first = true; hi > 0; first = false) {
    const int lo = max(hi - kSmallBits, 0);
    const uint32_t fmask = (1u << (hi - lo)) - 1u;
    if (!first) {
      clear();
      __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t r = rel[4 * s + e];
        // (bits above hi: none in the first pass; hi = 32 is a first pass too)
        const bool agrees = first || (r >> hi) == (T >> hi);
        hist_add_spread(lh, (r >> lo) & fmask, ((vmask >> s) & 1u) && agrees);
      }
    __syncthreads();
    // eight consecutive bins per thread, from the top
    constexpr int per = kSmallBins / kSmallThreads;
    uint32_t cnt[per], sum = 0;
    {
      const uint4 *row = reinterpret_cast<const uint4 *>(lh) + (kSmallBins - (t + 1) * per) / 4;
#pragma unroll
      for (int i = 0; i < per / 4; ++i) {
        const uint4 q = row[per / 4 - 1 - i];
        cnt[4 * i] = q.w; cnt[4 * i + 1] = q.z; cnt[4 * i + 2] = q.y; cnt[4 * i + 3] = q.x;
        sum += q.x + q.y + q.z + q.w;
      }
    }
    uint32_t above = block_exclusive_scan<kSmallWaves>(sum, tmp);
#pragma unroll
    for (int i = 0; i < per; ++i) {
      if (above < r_take && r_take <= above + cnt[i]) {  // (1 <= r_take <= keys that agree: one thread's bin)
        bcast[0] = T | ((uint32_t)(kSmallBins - 1 - (t * per + i)) << lo);
        bcast[1] = r_take - above;
        bcast[2] = cnt[i];
      }
      above += cnt[i];
    }
    __syncthreads();
    T = bcast[0];
    r_take = bcast[1];
    const uint32_t left = bcast[2];
    hi = lo;
    if (hi == 0) break;
    if (left <= kSmallList) {  // (uniform)
#pragma unroll
      for (int s = 0; s < SLOTS; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (((vmask >> s) & 1u) && (rel[4 * s + e] >> hi) == (T >> hi)) list[atomicAdd(&bcast[3], 1u)] = rel[4 * s + e];
      __syncthreads();
      if ((uint32_t)t < left) {
        const uint32_t mine = list[t];
        uint32_t gt = 0, ge = 0;
        for (uint32_t i = 0; i < left; ++i) {
          const uint32_t o = list[i];
          gt += o > mine; ge += o >= mine;
        }
        if (gt < r_take && r_take <= ge) { bcast[0] = mine; bcast[1] = r_take - gt; }  // (equal entries write the same)
      }
      __syncthreads();
      T = bcast[0];
      r_take = bcast[1];
      break;
    }
  }

  // Ordered compaction as in select_emit_kernel.  Position order is slot-major, then thread,
  // then the four keys of a slot: a wave scan per slot, then a scan over the 64 (slot, wave)
  // totals.  Counts (above T | equal to T) are packed 16 + 16 bits: N <= 16384.
  uint32_t ex[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    uint32_t packed = 0;
    if ((vmask >> s) & 1u) {
#pragma unroll
      for (int e = 0; e < 4; ++e) packed += ((rel[4 * s + e] > T) << 16) + (rel[4 * s + e] == T);
    }
    const uint32_t inc = wave_inclusive_scan(packed);
    ex[s] = inc - packed;
    if (lane == 63) tmp[s * kSmallWaves + wv] = inc;
  }
  __syncthreads();
  static_assert(kSmallSlots * kSmallWaves == 64, "one wave scans the totals");
  if (t < 64) {  // wave 0: exclusive scan of the totals
    const uint32_t v = t < SLOTS * kSmallWaves ? tmp[t] : 0u;
    tmp[t] = wave_inclusive_scan(v) - v;
  }
  __syncthreads();

  int32_t *out = idx + (size_t)b * k;
  float kept_top = 0.f;  // largest |coefficient| over the channels at a kept position
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    if ((vmask >> s) & 1u) {
      const int e0 = s * kSmallWaves + wv;
      const uint32_t before = tmp[e0] + ex[s];
      uint32_t gt = before >> 16, eq = before & 0xFFFFu;
      const int64_t pos = ((int64_t)s * kSmallThreads + t) * 4;
      int32_t jm[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t ky = rel[4 * s + e];
        const bool is_gt = ky > T, is_eq = ky == T;
        const bool keep = is_gt || (is_eq && eq < r_take);
        const uint32_t j = gt + min(eq, r_take);
        if (keep) out[j] = (int32_t)(pos + e);
        jm[e] = keep ? (int32_t)j : -1;
        kept_top = fmaxf(kept_top, keep ? topv[4 * s + e] : 0.f);
        gt += is_gt; eq += is_eq;
      }
      if (jmap) *reinterpret_cast<int4 *>(jmap + (size_t)b * N + pos) = make_int4(jm[0], jm[1], jm[2], jm[3]);
    }
  }
  side.finish(job, (int)gridDim.x * kSmallThreads);
  if (top_part)  // (uniform over the grid)
    publish_top<kSmallWaves>(kept_top, block_top, (size_t)b, tmp);
}

// jmap from an arbitrary ascending index list: fill with -1, then jmap[b][idx[b][j]] = j
__global__ __launch_bounds__(256) void fill_i32_kernel(int32_t *p, int64_t n, int32_t v, float *alpha,
                                                       float alpha_in) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (alpha && i < kAlphaSlots) alpha[i] = alpha_in > 0.f ? alpha_in : 0.f;
  if (i < n) p[i] = v;
}
__global__ __launch_bounds__(256) void jmap_scatter_kernel(const int32_t *__restrict__ idx,
                                                           int64_t N, int64_t k,
                                                           int32_t *__restrict__ jmap) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (j >= k) return;
  const int32_t q = idx[(size_t)b * k + j];
  if (q >= 0 && q < N) jmap[(size_t)b * N + q] = (int32_t)j;
}

// the index list "first k positions" (coarsest bands first): jmap[b][q] = q < k ? q : -1,
// idx[b][j] = j (idx nullable)
__global__ __launch_bounds__(256) void jmap_prefix_kernel(int64_t N, int64_t k,
                                                          int32_t *__restrict__ jmap,
                                                          int32_t *__restrict__ idx, float *alpha,
                                                          float alpha_in) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (alpha && b == 0 && q < kAlphaSlots) alpha[q] = alpha_in > 0.f ? alpha_in : 0.f;
  if (q >= N) return;
  jmap[(size_t)b * N + q] = q < k ? (int32_t)q : -1;
  if (idx && q < k) idx[(size_t)b * k + q] = (int32_t)q;
}

}  // namespace

hipError_t launch_jmap_prefix(int B, int64_t N, int64_t k, int32_t *jmap, int32_t *idx,
                              float *alpha_slots, float alpha_in, hipStream_t s) {
  hipLaunchKernelGGL(jmap_prefix_kernel, dim3((unsigned)((N + 255) / 256), B), dim3(256), 0, s, N, k,
                     jmap, idx, alpha_slots, alpha_in);
  return hipGetLastError();
}

// Whether the selection merges histograms (select_hist_kernel), which have to be clear before it.
bool select_counts(const WsLayout &L) { return !L.one_wg && L.two_nblk == 0; }

SelectPrep make_prep(void *ws_base, const WsLayout &L, float *alpha_slots, float alpha_in) {
  char *ws = static_cast<char *>(ws_base);
  SelectPrep p;
  p.hist = reinterpret_cast<uint32_t *>(ws + L.hist);
  p.alpha = alpha_slots;
  p.alpha_in = alpha_in;
  return p;
}

// how many partial maxima launch_select leaves in block_top: one per workgroup of its last kernel
int select_top_count(const wcc_desc &d, const WsLayout &L) {
  return L.one_wg ? d.B : d.B * (L.two_nblk > 0 ? L.two_nblk : L.nblk);
}

// Up to four pieces a thread of the first kernel: 16 KiB of weights a 256-thread workgroup.  A layer of
// few select workgroups and many weights is better off with a launch over the whole chip (4 us).
bool select_packs(const wcc_desc &d, const WsLayout &L, const PackJob &job) {
  const int64_t threads = L.one_wg          ? (int64_t)d.B * kSmallThreads
                          : L.two_nblk > 0 ? (int64_t)d.B * L.two_nblk * 1024
                                           : (int64_t)d.B * L.nblk * kThreads;
  return job.total > 0 && job.total <= 4 * threads;
}

hipError_t launch_select_init(const SelectPrep &p, int B, hipStream_t s) {
  hipLaunchKernelGGL(select_init_kernel, dim3(B), dim3(256), 0, s, p, B);
  return hipGetLastError();
}

// the three histogram passes and the compaction, SLOTS 16-byte loads a thread
template <int SLOTS>
static hipError_t launch_passes(const wcc_desc &d, const float *norm_or_part, int G, float *norm_out,
                                int64_t k, uint32_t *hist, SelectState *st, uint16_t *sfx,
                                uint32_t *gthi, int nblk, int32_t *idx, int32_t *jmap,
                                float *top_part, float *block_top, const PackJob &job, hipStream_t s) {
  const int64_t N = (int64_t)d.H * d.W;
  const uint32_t k32 = (uint32_t)k;
  dim3 grid(nblk, d.B), block(kThreads);
  const float *norm = norm_or_part;
  if (G > 1) {
    hipLaunchKernelGGL((select_hist_kernel<0, true, SLOTS>), grid, block, 0, s, norm_or_part, norm_out,
                       G, N, d.B, k32, hist, st, nblk, sfx, gthi, job);
    norm = norm_out;
  } else {
    hipLaunchKernelGGL((select_hist_kernel<0, false, SLOTS>), grid, block, 0, s, norm, nullptr, 1, N,
                       d.B, k32, hist, st, nblk, sfx, gthi, job);
  }
  hipLaunchKernelGGL((select_hist_kernel<1, false, SLOTS>), grid, block, 0, s, norm, nullptr, 1, N, d.B,
                     k32, hist, st, nblk, sfx, gthi, job);
  hipLaunchKernelGGL((select_hist_kernel<2, false, SLOTS>), grid, block, 0, s, norm, nullptr, 1, N, d.B,
                     k32, hist, st, nblk, sfx, gthi, job);
  hipLaunchKernelGGL((select_emit_kernel<SLOTS>), grid, block, 0, s, norm, N, k, hist, st, sfx, gthi,
                     nblk, idx, jmap, top_part, G, d.B, block_top);
  return hipGetLastError();
}

hipError_t launch_select(const wcc_desc &d, const float *norm_or_part, int G, float *norm_out,
                         int64_t k, void *ws_base, const WsLayout &L, int32_t *idx, int32_t *jmap,
                         float *top_part, float *block_top, const PackJob &wanted, hipStream_t s) {
  PackJob job = wanted;
  if (!select_packs(d, L, job)) job.total = 0;
  const int64_t N = (int64_t)d.H * d.W;
  char *ws = static_cast<char *>(ws_base);
  uint32_t *hist = reinterpret_cast<uint32_t *>(ws + L.hist);
  SelectState *st = reinterpret_cast<SelectState *>(ws + L.state);
  uint16_t *sfx = reinterpret_cast<uint16_t *>(ws + L.block_sfx);
  uint32_t *gthi = reinterpret_cast<uint32_t *>(ws + L.block_gthi);
  const int nblk = L.nblk;
  const uint32_t k32 = (uint32_t)k;
  if (L.one_wg) {
    const float *src = norm_or_part;
    int planes = G;
    if (G > 1 && (int64_t)G * N * (top_part ? 2 : 1) >= kCombineValues) {
      hipLaunchKernelGGL(combine_parts_kernel, dim3((unsigned)((N + 1023) / 1024), d.B), dim3(256), 0, s,
                         norm_or_part, norm_out, G, N, d.B, top_part);
      src = norm_out;
      planes = 1;
    }
#define WCC_SMALL(SLOTS)                                                                               \
  do {                                                                                                 \
    if (planes > 1)                                                                                    \
      hipLaunchKernelGGL((select_small_kernel<true, SLOTS>), dim3(d.B), dim3(kSmallThreads), 0, s,     \
                         src, planes, N, d.B, k32, idx, jmap, top_part, block_top, job);                    \
    else                                                                                               \
      hipLaunchKernelGGL((select_small_kernel<false, SLOTS>), dim3(d.B), dim3(kSmallThreads), 0, s,    \
                         src, 1, N, d.B, k32, idx, jmap, top_part, block_top, job);                         \
  } while (0)
    if (N <= 4 * kSmallThreads) WCC_SMALL(1);
    else if (N <= 8 * kSmallThreads) WCC_SMALL(2);
    else WCC_SMALL(4);
#undef WCC_SMALL
    return hipGetLastError();
  }
  if (L.two_nblk > 0) {
    if (G >= kCombineTwo) {
      hipLaunchKernelGGL(combine_parts_kernel, dim3((unsigned)((N + 1023) / 1024), d.B), dim3(256), 0, s,
                         norm_or_part, norm_out, G, N, d.B, top_part);
      norm_or_part = norm_out;
      G = 1;
    }
    return launch_select_two(d, norm_or_part, G, norm_out, k, ws + L.two_tables,
                             reinterpret_cast<uint32_t *>(ws + L.two_grouped), L.two_slots, L.two_nblk, idx, jmap, top_part, block_top, job, s);
  }
  switch (L.sel_slots) {
    case 4: return launch_passes<4>(d, norm_or_part, G, norm_out, k, hist, st, sfx, gthi, nblk, idx, jmap, top_part, block_top, job, s);
    case 2: return launch_passes<2>(d, norm_or_part, G, norm_out, k, hist, st, sfx, gthi, nblk, idx, jmap, top_part, block_top, job, s);
    default: return launch_passes<1>(d, norm_or_part, G, norm_out, k, hist, st, sfx, gthi, nblk, idx, jmap, top_part, block_top, job, s);
  }
}

hipError_t launch_jmap_from_idx(const int32_t *idx, int B, int64_t N, int64_t k, int32_t *jmap,
                                float *alpha_slots, float alpha_in, hipStream_t s) {
  const int64_t n = (int64_t)B * N;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, jmap, n, -1,
                     alpha_slots, alpha_in);
  dim3 grid((unsigned)((k + 255) / 256), B);
  hipLaunchKernelGGL(jmap_scatter_kernel, grid, dim3(256), 0, s, idx, N, k, jmap);
  return hipGetLastError();
}

}  // namespace wcc
