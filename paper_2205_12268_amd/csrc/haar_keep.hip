// Second transform pass of the fused layer: the kept coefficients go straight to their
// compressed place (Eq. T of the joint shrinkage), optionally as 8-bit codes.
#include "strip_io.h"

namespace wcc {
namespace {

// grid = (ceil(units/4), G, B), block = 256.  DWM as in haar_fwd_kernel.  Q8: xc is int8 codes
// for the clipping parameter q_alpha (> 0) or, if alpha_src is given, for the largest of its
// n_alpha entries (what the selection found as max |kept coefficient|); alpha_slots and wg_max must
// be null then.  Otherwise the workgroup's max |kept coefficient| goes to wg_max[its number] (a plain
// store, combined by the consumer) or raises one of the alpha slots (both nullable).
// PREFIX: the first `prefix` positions are kept, each its own rank (jmap unused).  An instance of its own: a branch in the others
// costs the smallest layers 0.1 us of instruction fetches.
template <int D, int V, int PF, int DWM, bool Q8, class XT, bool NT = false, bool PREFIX = false>
__global__ __launch_bounds__(256) void haar_keep_kernel(const XT *__restrict__ x,
                                                        const int32_t *__restrict__ jmap,
                                                        void *__restrict__ xc, float *alpha_slots,
                                                        float *wg_max, Geo g, StripMap m, int C, int Cg, int cstep,
                                                        int64_t k, const float *__restrict__ wdw,
                                                        float q_alpha,
                                                        const float *__restrict__ alpha_src,
                                                        int n_alpha, float *alpha_pub, int64_t prefix) {
  __shared__ float wmax[4];
  fetch_args(jmap, m.units, gridDim.z);
  const int unit = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int grp = blockIdx.y;
  // Samples are taken last to first: what the norm pass has left of x in the memory-side cache is its
  // tail (2 x 128 bf16 channels of 256 x 512: layer 82.2 -> 81.1 us, the 16-layer stack 785 -> 782).
  const int b = gridDim.z - 1 - blockIdx.z;
  LanePos<D> p;
  int row0, col0;
  const bool active = locate<D, V>(m, g, unit, p, row0, col0);
  // the channels of a group: Cg consecutive ones (cstep = 1), or every cstep-th one from grp
  // (cstep = the number of groups)
  const int c0 = cstep == 1 ? grp * Cg : grp;
  const int n_ch = c0 >= C ? 0 : (cstep == 1 ? min(C, c0 + Cg) - c0 : (C - c0 + cstep - 1) / cstep);
  const int64_t kstep = (int64_t)cstep * k;

  using Sink = KeepSink<D, V, Q8>;
  Sink sink(0.f);
  auto ranks = [&](auto &&rank_of) {
    auto fetch = [&](auto Lc, auto Jc) {
      constexpr int L = decltype(Lc)::value, J = decltype(Jc)::value;
      constexpr int CV = cols_at(V, L), S2 = span_at(V, L);
      const bool owner = (S2 == 1) || ((p.lc & (S2 - 1)) == 0);
#pragma unroll
      for (int i = 0; i < rows_at(D, L); ++i)
#pragma unroll
        for (int e = 0; e < CV; ++e) {
          constexpr int base = slot_base(D, V, L, J);
          const int s = base + i * CV + e;
          int j = -1;
          if (active && owner) j = rank_of(J * p.nl[L] + p.off[L] + i * p.rowlen[L] + e);
          sink.at[s] = (uint32_t)j;  // (turned into a byte offset below, once all loads are out)
        }
    };
    auto each_level = [&](auto Lc) {
      constexpr int L = decltype(Lc)::value;
      fetch(Lc, std::integral_constant<int, 1>{});
      fetch(Lc, std::integral_constant<int, 2>{});
      fetch(Lc, std::integral_constant<int, 3>{});
      if constexpr (L == D) fetch(Lc, std::integral_constant<int, 0>{});
    };
    each_level(std::integral_constant<int, 1>{});
    if constexpr (D >= 2) each_level(std::integral_constant<int, 2>{});
    if constexpr (D >= 3) each_level(std::integral_constant<int, 3>{});
    if constexpr (D >= 4) each_level(std::integral_constant<int, 4>{});
  };
  if constexpr (PREFIX) {
    const int first = (int)prefix;
    ranks([&](int at) { return at < first ? at : -1; });
  } else {
    const int32_t *jm = jmap + (size_t)b * g.N;
    ranks([&](int at) { return jm[at]; });
  }
  if constexpr (Q8) {
    // The clipping parameter the selection found: the largest of its workgroups' maxima.  Taken
    // here, behind the rank loads, so that the two round trips to memory overlap.  The first
    // workgroup leaves it as one float for the contraction that follows.
    if (alpha_src != nullptr) {  // (uniform over the grid)
      q_alpha = alpha_max(alpha_src, n_alpha);
      if (alpha_pub != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
        alpha_pub[0] = q_alpha;
    }
    sink.quant = Quant(q_alpha);
  }
  using Out = typename Sink::Out;
  // (lanes outside the plane read the plane's first rows: a valid address whatever the wave
  // does with them; nothing of theirs is ever stored)
  const XT *src = x + ((size_t)b * C + c0) * g.N + (active ? (size_t)row0 * g.W + col0 : (size_t)0);
  Out *plane = static_cast<Out *>(xc) + ((size_t)b * C + c0) * k;
  // walks the group's channels with whichever sink; returns its max |kept coefficient|
  auto walk = [&](auto &sk, auto &&next_channel) {
    sk.vmax = 0.f;
    sk.aim(plane, k);
    if constexpr (DWM == 0) {
      channel_loop<D, V, PF, NT>(src, g.N * cstep, g.W, n_ch, p, sk, next_channel);
    } else {
      const DwLane q = dw_lane<D, V>(g, m, p, row0, col0);
      channel_loop_dw<D, V, DWM == 2, true, false>(src, wdw + (size_t)c0 * 9, g.N, n_ch, q, p, sk,
                                                   next_channel);
    }
    return sk.vmax;
  };

  float mx = 0.f;
  bool done = false;
  // Dense stores pay where a strip keeps at most half of its slots' worth of positions.  With
  // K_dw folded in and fp32 maps the pass is bound by HBM bytes and the staging measured 5-10 %
  // slower than one store per slot; with bf16 maps it is bound by its arithmetic, and taking
  // the maximum and the store offsets over the list rows instead of over every slot makes it
  // 20 % faster (block at keep 1/8: 375 -> 297 us).
  constexpr int NS = slot_count(D, V);
  constexpr bool kStaged = ((V == 4 && (D == 2 || D == 3)) || D == 4) && (DWM == 0 || sizeof(XT) == 2);
  if constexpr (kStaged) {
    __shared__ uint32_t tiles[4][NS * kWave];
    constexpr int kRankBits = 20;  // list entry = rank | tile index << 20
    int count = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) count += __popcll(__ballot((int)sink.at[s] >= 0));
    const int ni = (count + kWave - 1) / kWave;
    // a wave with lanes outside the plane may stage too (their slots are in no list), except
    // with K_dw folded in, whose border handling counts on the lanes' own columns
    const bool whole = DWM == 0 ? __ballot(active) != 0 : __ballot(active) == ~(uint64_t)0;
    if (whole && n_ch > 0 && ni <= NS / 2 && ni <= 16 && k <= ((int64_t)1 << kRankBits)) {
      const int lane = threadIdx.x & (kWave - 1);
      uint32_t *tile = tiles[threadIdx.x >> 6];
      // pack (rank, tile index): slot-major, then lane (a band row's kept positions have
      // consecutive ranks).  The tile is scratch for the list before it becomes the staging area.
      int running = 0;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int j = (int)sink.at[s];
        const uint64_t kept = __ballot(j >= 0);
        const int to = running + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u));
        if (j >= 0) tile[to] = (uint32_t)j | ((uint32_t)(s * kWave + lane) << kRankBits);
        running += __popcll(kept);
      }
      wave_lds_fence();
      auto run = [&](auto ni_c) {
        constexpr int NI = decltype(ni_c)::value;
        KeepStagedSink<D, V, Q8, NI> st(Q8 ? q_alpha : 0.f);
        st.tile = tile;
        st.lane = lane;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const int e = lane + kWave * i;
          const uint32_t packed = e < count ? tile[e] : 0u;
          st.cell[i] = e < count ? packed >> kRankBits : (uint32_t)lane;
          st.at[i] = e < count ? (packed & ((1u << kRankBits) - 1u)) * (uint32_t)sizeof(Out) : Sink::kDropped;
        }
        wave_lds_fence();
        mx = walk(st, [&plane, k, kstep](auto &sk) {
          sk.flush();
          plane += kstep;
          sk.aim(plane, k);
        });
      };
      if (ni <= 4) run(std::integral_constant<int, 4>{});
      else if (ni <= 8) run(std::integral_constant<int, 8>{});
      else run(std::integral_constant<int, 16>{});  // (ni <= 16 is part of the condition above)
      done = true;
    }
  }
  if (!done && active && n_ch > 0) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
      sink.at[s] = (int)sink.at[s] >= 0 ? sink.at[s] * (uint32_t)sizeof(Out) : Sink::kDropped;
    auto next = [&plane, k, kstep](auto &sk) {
      plane += kstep;
      sk.aim(plane, k);
    };
    if constexpr (Q8) {
      // the quantiser's division path is the same for every value of the layer: one look here
      // instead of one a row inside the channel walk
      if (sink.quant.fast) {
        KeepSink<D, V, Q8, 1> fast(sink);
        mx = walk(fast, next);
      } else {
        KeepSink<D, V, Q8, 2> exact(sink);
        mx = walk(exact, next);
      }
    } else {
      mx = walk(sink, next);
    }
  }
  if (alpha_slots == nullptr && wg_max == nullptr) return;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    mx = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    if (wg_max != nullptr) {
      wg_max[((size_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = mx;
      return;
    }
    // integer max on the bit pattern of a non-negative float: exact and order-independent;
    // workgroups spread over the slots because atomics on one address serialise
    unsigned int *a = reinterpret_cast<unsigned int *>(alpha_slots) +
                      ((blockIdx.x + 3u * blockIdx.y + 11u * blockIdx.z) & (kAlphaSlots - 1));
    const unsigned int mine = __float_as_uint(mx);
    if (mine > __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(a, mine);
  }
}


// ---- the same into words ---------------------------------------------------------------------------
// Every lane's coefficients of a channel go into an LDS tile [slot][lane]; the wave picks its kept positions,
// unit by unit (four units a wave, consecutive in the compressed signal), NI rows of 64.  8-bit codes of
// four channels make a word, so that a row of 64 positions and four channels is one store of 256 contiguous bytes.
// Stores of a channel group of four are issued behind the first transform of the next one: between a load and the
// wait for it every path has the same number of memory instructions.
// Bound by its reads of x: 4 x 64 channels of 512 x 1024, an eighth kept, 99 us, where a byte store a code, in short runs
// of lines that several dies write, takes the kernel above 114 (the norm pass reads the same x in 82).
// Three levels, four columns a lane (the last kernel's).
// grid = (ceil(wave units / 4), G, B), block = 256; group y takes the quads of channels y, y + G, ...
struct WordSink {
  static constexpr int D = 3, V = 4;
  uint32_t *tile;  // this lane's column of [slot][lane]
  template <int L, int J>
  __device__ __forceinline__ void put_row(const LanePos<D> &, int i, const float (&v)[cols_at(V, L)], bool) {
    constexpr int CV = cols_at(V, L), base = slot_base(D, V, L, J);
#pragma unroll
    for (int e = 0; e < CV; ++e) tile[(base + i * CV + e) * kWave] = __float_as_uint(v[e]);
  }
};

template <bool Q8, class XT, bool NT>
__global__ __launch_bounds__(256) void haar_keep_words_kernel(const XT *__restrict__ x, const int32_t *__restrict__ jmap,
                                                              const uint32_t *__restrict__ ucount, int upad,
                                                              uint32_t *__restrict__ xw, float *alpha_slots,
                                                              float *wg_max, Geo g, StripMap m, int C, int64_t ks,
                                                              float q_alpha, const float *__restrict__ alpha_src,
                                                              int n_alpha, float *alpha_pub) {
  constexpr int D = WordSink::D, V = WordSink::V, NS = slot_count(D, V), R = 1 << D;
  __shared__ float wmax[4];
  __shared__ uint32_t tiles[4][NS * kWave];
  fetch_args(jmap, m.units, gridDim.z);
  const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = blockIdx.x * 4 + wv, grp = blockIdx.y, G = gridDim.y;
  const int b = gridDim.z - 1 - blockIdx.z;  // (last to first: what the norm pass left in the cache is the tail)
  LanePos<D> p;
  int row0, col0;
  const bool active = locate<D, V>(m, g, unit, p, row0, col0);
  const int quads = (C + 3) / 4, nq = grp < quads ? (quads - grp + G - 1) / G : 0;

  const int32_t *jm = jmap + (size_t)b * g.N;
  int at[NS];
  auto fetch = [&](auto Lc, auto Jc) {
    constexpr int L = decltype(Lc)::value, J = decltype(Jc)::value;
    constexpr int CV = cols_at(V, L), S2 = span_at(V, L);
    const bool owner = (S2 == 1) || ((p.lc & (S2 - 1)) == 0);
#pragma unroll
    for (int i = 0; i < rows_at(D, L); ++i)
#pragma unroll
      for (int e = 0; e < CV; ++e) {
        constexpr int base = slot_base(D, V, L, J);
        int j = -1;
        if (active && owner) j = jm[J * p.nl[L] + p.off[L] + i * p.rowlen[L] + e];
        at[base + i * CV + e] = j;
      }
  };
  auto each_level = [&](auto Lc) {
    constexpr int L = decltype(Lc)::value;
    fetch(Lc, std::integral_constant<int, 1>{});
    fetch(Lc, std::integral_constant<int, 2>{});
    fetch(Lc, std::integral_constant<int, 3>{});
    if constexpr (L == D) fetch(Lc, std::integral_constant<int, 0>{});
  };
  each_level(std::integral_constant<int, 1>{});
  each_level(std::integral_constant<int, 2>{});
  each_level(std::integral_constant<int, 3>{});
  // kept positions in front of this wave's units
  uint32_t before = 0;
  {
    const uint4 *uc = reinterpret_cast<const uint4 *>(ucount + (size_t)b * upad);  // four units: one wave's
    const int n = min(unit, upad / 4);
    for (int i = lane; i < n; i += kWave) {
      const uint4 v = uc[i];
      before += v.x + v.y + v.z + v.w;
    }
  }
  if constexpr (Q8) {
    if (alpha_src != nullptr) {  // (uniform over the grid)
      q_alpha = alpha_max(alpha_src, n_alpha);
      if (alpha_pub != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
        alpha_pub[0] = q_alpha;
    }
  }
  const Quant quant(Q8 ? q_alpha : 0.f);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off, kWave);
  before = (uint32_t)__builtin_amdgcn_readfirstlane((int)before);

  // the wave's list: unit by unit, slot by slot, lane by lane
  uint32_t *tile = tiles[wv];
  const int shift = lane & 16;
  auto mine16 = [&](uint64_t kept) {  // the votes of this lane's unit
    return ((lane & 32 ? (uint32_t)(kept >> 32) : (uint32_t)kept) >> shift) & 0xFFFFu;
  };
  int total = 0;
#pragma unroll
  for (int s = 0; s < NS; ++s) total += __popc(mine16(__ballot(at[s] >= 0)));
  const int t0 = __builtin_amdgcn_readlane(total, 0), t1 = __builtin_amdgcn_readlane(total, 16);
  const int t2 = __builtin_amdgcn_readlane(total, 32), count = t0 + t1 + t2 + __builtin_amdgcn_readlane(total, 48);
  float mx = 0.f;
  if (count > 0 && nq > 0) {
    int running = lane < 16 ? 0 : lane < 32 ? t0 : lane < 48 ? t0 + t1 : t0 + t1 + t2;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const uint32_t kept = mine16(__ballot(at[s] >= 0));
      if (at[s] >= 0) tile[running + __popc(kept & ((1u << (lane & 15)) - 1u))] = (uint32_t)(s * kWave + lane);
      running += __popc(kept);
    }
    wave_lds_fence();
    const int ni = (count + kWave - 1) / kWave;
    // Sixteen of 32 rows a walk over the channels at most: 32 rows take the registers of a second wave.  The cells of
    // the second walk wait two to a register.
    constexpr int kRows = 16;
    static_assert(2 * kRows == V << D, "two walks hold every position of the wave's units");
    auto entry = [&](int i) { return tile[min(lane + kWave * i, count - 1)]; };
    uint32_t later[kRows / 2];
#pragma unroll
    for (int i = 0; i < kRows / 2; ++i) later[i] = entry(kRows + 2 * i) | entry(kRows + 2 * i + 1) << 16;
    // (lanes outside the plane read the plane's first rows; their values are in no list)
    const XT *src = x + (size_t)b * C * g.N + (active ? (size_t)row0 * g.W + col0 : (size_t)0);
    uint32_t *out = xw + (size_t)b * (Q8 ? quads : C) * ks + before;
    // cell: past the end of the list its last entry again (the stores there are dropped); left: entries
    auto walk = [&](auto ni_c, const uint32_t (&cell)[decltype(ni_c)::value], uint32_t *out, int left) {
      constexpr int NI = decltype(ni_c)::value;
      wave_lds_fence();
      WordSink sink{tile + lane};
      uint32_t word[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) word[i] = 0;
      // row of the signal, -1: nothing yet
      auto store = [&](int row) {
        const bool in = row >= 0 && (Q8 || row < C);
        const __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc(out + (size_t)(in ? row : 0) * ks, 0,
                                                                           in ? left * 4 : 0, 0x00020000);
#pragma unroll
        for (int i = 0; i < NI; ++i) __builtin_amdgcn_raw_buffer_store_b32(word[i], to, (lane + kWave * i) * 4, 0, 0);
      };
      auto channel = [&](int i) { return min((grp + (i >> 2) * G) * 4 + (i & 3), C - 1); };
      Row<V, XT> buf[2][R];
      auto load = [&](Row<V, XT> (&to)[R], int i) {
        const XT *nx = src + (size_t)channel(min(i, 4 * nq - 1)) * g.N;
#pragma unroll
        for (int r = 0; r < R; ++r) to[r].template load<NT>(nx + (size_t)r * g.W);
      };
      load(buf[0], 0);
      int pending = -1;
      for (int qd = 0; qd < nq; ++qd) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          load(buf[(u + 1) & 1], 4 * qd + u + 1);
          __builtin_amdgcn_sched_barrier(0);
          float in[R][V];
#pragma unroll
          for (int r = 0; r < R; ++r) buf[u & 1][r].get(in[r]);
          fwd_levels<D, V, 1>(in, p, sink);
          if (!Q8 || u == 0) store(pending);
          wave_lds_fence();
          if constexpr (Q8) {
            float v[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) v[i] = __uint_as_float(tile[cell[i]]);
            auto code = [&](auto fast_c) {  // the new code comes in at the top, the oldest leaves at the bottom
              constexpr bool FAST = decltype(fast_c)::value;
#pragma unroll
              for (int i = 0; i < NI; ++i)
                word[i] = __builtin_amdgcn_alignbyte((uint32_t)(int)quant.template level_as<FAST>(v[i]), word[i], 1);
            };
            if (quant.fast) code(std::true_type{}); else code(std::false_type{});
            if (u == 3) pending = grp + qd * G;
          } else {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
              word[i] = tile[cell[i]];
              mx = fmaxf(mx, fabsf(__uint_as_float(word[i])));
            }
            pending = (grp + qd * G) * 4 + u;  // (channels past the last repeat it, and are not stored)
          }
          wave_lds_fence();
        }
      }
      store(pending);
    };
    auto first = [&](auto ni_c) {
      constexpr int NI = decltype(ni_c)::value;
      uint32_t cell[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) cell[i] = entry(i);
      walk(ni_c, cell, out, count);
    };
    using std::integral_constant;
    if (ni <= 4) first(integral_constant<int, 4>{});
    else if (ni <= 8) first(integral_constant<int, 8>{});
    else {
      first(integral_constant<int, kRows>{});
      if (ni > kRows) {
        uint32_t cell[kRows];
#pragma unroll
        for (int i = 0; i < kRows; ++i) cell[i] = i & 1 ? later[i / 2] >> 16 : later[i / 2] & 0xFFFFu;
        walk(integral_constant<int, kRows>{}, cell, out + kRows * kWave, count - kRows * kWave);
      }
    }
  }
  if (alpha_slots == nullptr && wg_max == nullptr) return;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  if (lane == 0) wmax[wv] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    mx = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    if (wg_max != nullptr) {
      wg_max[((size_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = mx;
      return;
    }
    unsigned int *a = reinterpret_cast<unsigned int *>(alpha_slots) +
                      ((blockIdx.x + 3u * blockIdx.y + 11u * blockIdx.z) & (kAlphaSlots - 1));
    const unsigned int top = __float_as_uint(mx);
    if (top > __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(a, top);
  }
}

// ---- codes of four channels a word, in the order of the ranks ----------------------------------------
// The second pass of layers whose codes are decided in it: four channels' codes of a position leave as one word,
// [B, ceil(C / 4), k], which the contraction reads as it multiplies (four channels of a column are a word of its operand).
// A byte store a code costs the memory pipeline four times the instructions, and lines of 64 bytes at best.  Byte by byte and
// in words: 8 x 256 channels of 256 x 256, a quarter kept, 118 -> 106 us; 8 x 128 of 192 x 640, a sixteenth, 95.6 -> 89; 16 x 256 of
// 128 x 128, a half, 53 -> 50; 256 of 256 x 512 at two levels 25.3 -> 24.4 (its reads alone 20).  Three workgroups a compute
// unit (168 registers, 179 now) lose on the long walks: 113, 90.5.
// Groups take quads of channels y, y + G, ... .  The stores of a quad are issued behind the loads of the next one's
// second channel: between a load and the wait for it every path has the same number of memory instructions.
// grid = (ceil(units / 4), G, B), block = 256.

// A strip that keeps few of its positions: through an LDS tile [slot][lane] and the packed list (see KeepStagedSink).
template <int D, int V, int NI>
struct QuadListSink {
  uint32_t *tile;     // [slot][lane]
  int lane;
  uint32_t cell[NI];  // tile index of the entry's position
  uint32_t at[NI];    // byte offset of the entry's rank, or kRowDropped
  uint32_t word[NI];
  Quant quant;
  __device__ __forceinline__ explicit QuadListSink(const Quant &q) : quant(q) {}
  template <int L, int J>
  __device__ __forceinline__ void put_row(const LanePos<D> &, int i, const float (&v)[cols_at(V, L)], bool) {
    constexpr int CV = cols_at(V, L), base = slot_base(D, V, L, J);
#pragma unroll
    for (int e = 0; e < CV; ++e) tile[(base + i * CV + e) * kWave + lane] = __float_as_uint(v[e]);
  }
  __device__ __forceinline__ void code() {
    wave_lds_fence();
    float v[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) v[i] = __uint_as_float(tile[cell[i]]);
    auto shift_in = [&](auto fast_c) {  // the new code comes in at the top, the oldest leaves at the bottom
      constexpr bool FAST = decltype(fast_c)::value;
#pragma unroll
      for (int i = 0; i < NI; ++i)
        word[i] = __builtin_amdgcn_alignbyte((uint32_t)(int)quant.template level_as<FAST>(v[i]), word[i], 1);
    };
    if (quant.fast) shift_in(std::true_type{}); else shift_in(std::false_type{});
    wave_lds_fence();
  }
  __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t to) const {
#pragma unroll
    for (int i = 0; i < NI; ++i) __builtin_amdgcn_raw_buffer_store_b32(word[i], to, at[i], 0, 0);
  }
};

// Any strip: a word a slot.
template <int D, int V, bool FAST>
struct QuadSlotSink {
  uint32_t at[slot_count(D, V)];  // byte offset of the slot's rank, or kRowDropped
  uint32_t word[slot_count(D, V)];
  Quant quant;
  __device__ __forceinline__ explicit QuadSlotSink(const Quant &q) : quant(q) {}
  template <int L, int J>
  __device__ __forceinline__ void put_row(const LanePos<D> &, int i, const float (&v)[cols_at(V, L)], bool) {
    constexpr int CV = cols_at(V, L), base = slot_base(D, V, L, J);
#pragma unroll
    for (int e = 0; e < CV; ++e) {
      uint32_t &w = word[base + i * CV + e];
      w = __builtin_amdgcn_alignbyte((uint32_t)(int)quant.template level_as<FAST>(v[e]), w, 1);
    }
  }
  __device__ __forceinline__ void code() {}
  __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t to) const {
#pragma unroll
    for (int s = 0; s < slot_count(D, V); ++s) __builtin_amdgcn_raw_buffer_store_b32(word[s], to, at[s], 0, 0);
  }
};

template <int D, int V, class XT, bool NT>
__global__ __launch_bounds__(256) void haar_keep_quads_kernel(const XT *__restrict__ x, const int32_t *__restrict__ jmap,
                                                              uint32_t *__restrict__ xw, Geo g, StripMap m, int C,
                                                              int64_t ks, float q_alpha,
                                                              const float *__restrict__ alpha_src, int n_alpha,
                                                              float *alpha_pub) {
  constexpr int NS = slot_count(D, V), R = 1 << D;
  constexpr bool kStaged = (V == 4 && (D == 2 || D == 3)) || D == 4;
  constexpr int kRankBits = 20;  // list entry = rank | tile index << 20
  __shared__ uint32_t tiles[kStaged ? 4 : 1][kStaged ? NS * kWave : 1];
  const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = blockIdx.x * 4 + wv, grp = blockIdx.y, G = gridDim.y;
  const int b = gridDim.z - 1 - blockIdx.z;  // (last to first: what the norm pass left in the cache is the tail)
  LanePos<D> p;
  int row0, col0;
  const bool active = locate<D, V>(m, g, unit, p, row0, col0);
  const int quads = (C + 3) / 4, nq = (quads - grp + G - 1) / G;  // (G <= quads)

  // ranks of this lane's positions, or -1
  int at[NS];
  const int32_t *jm = jmap + (size_t)b * g.N;
  auto fetch = [&](auto Lc, auto Jc) {
    constexpr int L = decltype(Lc)::value, J = decltype(Jc)::value;
    constexpr int CV = cols_at(V, L), S2 = span_at(V, L);
    const bool owner = (S2 == 1) || ((p.lc & (S2 - 1)) == 0);
#pragma unroll
    for (int i = 0; i < rows_at(D, L); ++i)
#pragma unroll
      for (int e = 0; e < CV; ++e) {
        constexpr int base = slot_base(D, V, L, J);
        int j = -1;
        if (active && owner) j = jm[J * p.nl[L] + p.off[L] + i * p.rowlen[L] + e];
        at[base + i * CV + e] = j;
      }
  };
  auto each_level = [&](auto Lc) {
    constexpr int L = decltype(Lc)::value;
    fetch(Lc, std::integral_constant<int, 1>{});
    fetch(Lc, std::integral_constant<int, 2>{});
    fetch(Lc, std::integral_constant<int, 3>{});
    if constexpr (L == D) fetch(Lc, std::integral_constant<int, 0>{});
  };
  each_level(std::integral_constant<int, 1>{});
  if constexpr (D >= 2) each_level(std::integral_constant<int, 2>{});
  if constexpr (D >= 3) each_level(std::integral_constant<int, 3>{});
  if constexpr (D >= 4) each_level(std::integral_constant<int, 4>{});
  if (alpha_src != nullptr) {  // (uniform over the grid; behind the rank loads)
    q_alpha = alpha_max(alpha_src, n_alpha);
    if (alpha_pub != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
      alpha_pub[0] = q_alpha;
  }
  if (__ballot(active) == 0) return;  // whole waves leave (no barrier below)
  const Quant quant(q_alpha);
  // (lanes outside the plane read the plane's first rows; nothing of theirs is ever stored)
  const XT *src = x + (size_t)b * C * g.N + (active ? (size_t)row0 * g.W + col0 : (size_t)0);
  uint32_t *out = xw + (size_t)b * quads * ks;
  auto walk = [&](auto &sink) {
    // row of the signal, -1: nothing yet
    auto store = [&](int row) {
      sink.store(__builtin_amdgcn_make_buffer_rsrc(out + (size_t)max(row, 0) * ks, 0,
                                                   row >= 0 ? (int)(uint32_t)(ks * 4) : 0, 0x00020000));
    };
    // (channels past the last one repeat it; they meet weights of zero)
    auto channel = [&](int i) { return min((grp + (i >> 2) * G) * 4 + (i & 3), C - 1); };
    Row<V, XT> buf[2][R];
    auto load = [&](Row<V, XT> (&to)[R], int i) {
      const XT *nx = src + (size_t)channel(min(i, 4 * nq - 1)) * g.N;
#pragma unroll
      for (int r = 0; r < R; ++r) to[r].template load<NT>(nx + (size_t)r * g.W);
    };
    load(buf[0], 0);
    int pending = -1;
    for (int qd = 0; qd < nq; ++qd) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        load(buf[(u + 1) & 1], 4 * qd + u + 1);
        if (u == 0) store(pending);
        __builtin_amdgcn_sched_barrier(0);
        float in[R][V];
#pragma unroll
        for (int r = 0; r < R; ++r) buf[u & 1][r].get(in[r]);
        fwd_levels<D, V, 1>(in, p, sink);
        sink.code();
      }
      pending = grp + qd * G;
    }
    store(pending);
  };

  if constexpr (kStaged) {
    int count = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) count += __popcll(__ballot(at[s] >= 0));
    const int ni = (count + kWave - 1) / kWave;
    if (ni <= NS / 2 && ni <= 16 && ks <= ((int64_t)1 << kRankBits)) {
      if (count == 0) return;
      uint32_t *tile = tiles[wv];
      int running = 0;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int j = at[s];
        const uint64_t kept = __ballot(j >= 0);
        const int to = running + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u));
        if (j >= 0) tile[to] = (uint32_t)j | ((uint32_t)(s * kWave + lane) << kRankBits);
        running += __popcll(kept);
      }
      wave_lds_fence();
      auto run = [&](auto ni_c) {
        constexpr int NI = decltype(ni_c)::value;
        QuadListSink<D, V, NI> sink(quant);
        sink.tile = tile;
        sink.lane = lane;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const int e = lane + kWave * i;
          const uint32_t packed = e < count ? tile[e] : 0u;
          sink.cell[i] = e < count ? packed >> kRankBits : (uint32_t)lane;
          sink.at[i] = e < count ? (packed & ((1u << kRankBits) - 1u)) * 4u : kRowDropped;
          sink.word[i] = 0;
        }
        wave_lds_fence();
        walk(sink);
      };
      if (ni <= 4) run(std::integral_constant<int, 4>{});
      else if (ni <= 8) run(std::integral_constant<int, 8>{});
      else if (D == 3 && ni <= 12) run(std::integral_constant<int, 12>{});
      else run(std::integral_constant<int, 16>{});
      return;
    }
  }
  auto slots = [&](auto fast_c) {
    QuadSlotSink<D, V, decltype(fast_c)::value> sink(quant);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      sink.at[s] = at[s] >= 0 ? (uint32_t)at[s] * 4u : kRowDropped;
      sink.word[s] = 0;
    }
    walk(sink);
  };
  if (quant.fast) slots(std::true_type{}); else slots(std::false_type{});
}

// The same with K_dw in front of the transform (fp32 maps), a word a slot: group y takes quads of channels from y * Cq on.
// 16 x 1024 channels of 128 x 128, a half kept: 268 -> 255 us, and the contraction that reads the words 84 -> 78.5.
template <int D, int V, int DWM>
__global__ __launch_bounds__(256) void haar_keep_dw_quads_kernel(const float *__restrict__ x, const int32_t *__restrict__ jmap,
                                                                 uint32_t *__restrict__ xw, Geo g, StripMap m, int C, int Cq,
                                                                 int64_t ks, const float *__restrict__ wdw, float q_alpha,
                                                                 const float *__restrict__ alpha_src, int n_alpha,
                                                                 float *alpha_pub) {
  constexpr int NS = slot_count(D, V);
  fetch_args(jmap, m.units, gridDim.z);
  const int unit = blockIdx.x * 4 + (threadIdx.x >> 6), grp = blockIdx.y;
  const int b = gridDim.z - 1 - blockIdx.z;
  LanePos<D> p;
  int row0, col0;
  const bool active = locate<D, V>(m, g, unit, p, row0, col0);
  const int quads = (C + 3) / 4, c0 = grp * Cq * 4, n_ch = min(C - c0, Cq * 4);
  uint32_t at[NS];
  const int32_t *jm = jmap + (size_t)b * g.N;
  auto fetch = [&](auto Lc, auto Jc) {
    constexpr int L = decltype(Lc)::value, J = decltype(Jc)::value;
    constexpr int CV = cols_at(V, L), S2 = span_at(V, L);
    const bool owner = (S2 == 1) || ((p.lc & (S2 - 1)) == 0);
#pragma unroll
    for (int i = 0; i < rows_at(D, L); ++i)
#pragma unroll
      for (int e = 0; e < CV; ++e) {
        constexpr int base = slot_base(D, V, L, J);
        int j = -1;
        if (active && owner) j = jm[J * p.nl[L] + p.off[L] + i * p.rowlen[L] + e];
        at[base + i * CV + e] = (uint32_t)j;
      }
  };
  auto each_level = [&](auto Lc) {
    constexpr int L = decltype(Lc)::value;
    fetch(Lc, std::integral_constant<int, 1>{});
    fetch(Lc, std::integral_constant<int, 2>{});
    fetch(Lc, std::integral_constant<int, 3>{});
    if constexpr (L == D) fetch(Lc, std::integral_constant<int, 0>{});
  };
  each_level(std::integral_constant<int, 1>{});
  if constexpr (D >= 2) each_level(std::integral_constant<int, 2>{});
  if constexpr (D >= 3) each_level(std::integral_constant<int, 3>{});
  if constexpr (D >= 4) each_level(std::integral_constant<int, 4>{});
  if (alpha_src != nullptr) {  // (uniform over the grid; behind the rank loads)
    q_alpha = alpha_max(alpha_src, n_alpha);
    if (alpha_pub != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
      alpha_pub[0] = q_alpha;
  }
  if (!active || n_ch <= 0) return;
  const Quant quant(q_alpha);
  const float *src = x + ((size_t)b * C + c0) * g.N + (size_t)row0 * g.W + col0;
  uint32_t *out = xw + ((size_t)b * quads + (size_t)grp * Cq) * ks;
  auto walk = [&](auto fast_c) {
    QuadSlotSink<D, V, decltype(fast_c)::value> sink(quant);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      sink.at[s] = (int)at[s] >= 0 ? at[s] * 4u : kRowDropped;
      sink.word[s] = 0;
    }
    const DwLane q = dw_lane<D, V>(g, m, p, row0, col0);
    int pending = -1;  // quad of the group that waits to be stored, -1: none yet
    channel_loop_dw<D, V, DWM == 2, true, false, true>(src, wdw + (size_t)c0 * 9, g.N, n_ch, q, p, sink, [&](auto &sk) {
      sk.store(__builtin_amdgcn_make_buffer_rsrc(out + (size_t)max(pending, 0) * ks, 0,
                                                 pending >= 0 ? (int)(uint32_t)(ks * 4) : 0, 0x00020000));
      ++pending;
    });
  };
  if (quant.fast) walk(std::true_type{}); else walk(std::false_type{});
}

// the lanes of all strips follow each other, 64 a wave: four units
inline StripMap words_map(const wcc_desc &d) {
  StripMap m = make_map(d, lane_cols(d));
  m.flat = true;
  m.units = (int)(((int64_t)m.strips * m.lanes_w + kWave - 1) / kWave);
  return m;
}

int words_groups(const wcc_desc &d, bool late) {
  const StripMap m = words_map(d);
  int G = groups_for(d, m, d.C_in, 2048, 4);
  if (late && (int64_t)((m.units + 3) / 4) * G * d.B > kMaxWgMaxima) G = std::min(G, groups_for(d, m, d.C_in, 1024, 4));
  return G;
}

template <class XT>
hipError_t words_launch(const wcc_desc &d, int64_t ks, const XT *x, const int32_t *jmap, const uint32_t *ucount,
                        uint32_t *xw, float *alpha_slots, float *wg_max, float q_alpha, const float *alpha_src,
                        int n_alpha, float *alpha_pub, hipStream_t s) {
  const Geo g{d.H, d.W, d.levels, (int64_t)d.H * d.W};
  const StripMap m = words_map(d);
  const int upad = unit_pad(unit_map(d));
  const dim3 grid((m.units + 3) / 4, words_groups(d, alpha_slots != nullptr || wg_max != nullptr), d.B);
#define WCC_WORDS(Q8, NT)                                                                                          \
  hipLaunchKernelGGL((haar_keep_words_kernel<Q8, XT, NT>), grid, dim3(256), 0, s, x, jmap, ucount, upad, xw, \
                     alpha_slots, wg_max, g, m, d.C_in, ks, q_alpha, alpha_src, n_alpha, alpha_pub)
  if (q_alpha > 0.f || alpha_src != nullptr) { if (streams(d)) WCC_WORDS(true, true); else WCC_WORDS(true, false); }
  else                                       { if (streams(d)) WCC_WORDS(false, true); else WCC_WORDS(false, false); }
#undef WCC_WORDS
  return hipGetLastError();
}

inline StripMap keep_map(const wcc_desc &d, bool folded) {
  return folded ? make_map(d, lane_cols(d)) : make_flat_map(d, lane_cols(d));
}

constexpr int64_t kQuadWaves = 1024;
constexpr int64_t kQuadRound = 512;  // workgroups, two a compute unit

int keep_groups(const wcc_desc &d, bool folded, bool late) {
  // About two thousand waves, down to two channels each at d <= 2, where a wave has few rows in flight
  // (the 16-layer stack 792 -> 782 us against a thousand waves of four, 256 channels of 256 x 512
  // 123.4 -> 121.3; two channels at d = 3 lose 1-3 %); with K_dw in front as measured there.
  const StripMap m = keep_map(d, folded);
  int G = groups_for(d, m, d.C_in, arithmetic_bound(d, folded) ? 4096 : folded ? 1024 : 2048,
                     !folded && d.levels <= 2 ? 2 : 4);
  // Planes of one to three strip units leave waves of a workgroup idle, so that two thousand waves are as many
  // workgroups: too many to leave a maximum each where alpha is found here, and raising slots costs more than
  // the second thousand gains (15 x 400 bf16 channels of 14 x 10, a fifth kept: 15 us with 960 workgroups, 23 with
  // 1920).
  if (late && (int64_t)((m.units + 3) / 4) * G * d.B > kMaxWgMaxima)
    G = std::min(G, groups_for(d, m, d.C_in, arithmetic_bound(d, folded) ? 4096 : 1024, 4));
  return G;
}

template <int D, int V, class XT>
hipError_t keep_launch_t(const wcc_desc &d, int64_t k, const XT *x, const int32_t *jmap, void *xc,
                         float *alpha_slots, float *wg_max, Plan pl, const float *wdw, float q_alpha,
                         const float *alpha_src, int n_alpha, float *alpha_pub, int64_t prefix, hipStream_t s) {
  const Geo g{d.H, d.W, d.levels, (int64_t)d.H * d.W};
  const StripMap m = keep_map(d, wdw != nullptr);
  const int Cg = (d.C_in + pl.G - 1) / pl.G;
  // Without K_dw in front, group g takes the channels g, g + G, ...: groups running side by
  // side then read neighbouring planes of x and write neighbouring planes of xc (keep pass of
  // workloads 2 and 4 and the stack 2 % faster).  The folded walk indexes its 3x3 weights by
  // consecutive channels and keeps the blocks.
  const int cstep = wdw == nullptr ? pl.G : 1;
  dim3 grid((m.units + 3) / 4, pl.G, d.B);
  const bool q8 = q_alpha > 0.f || alpha_src != nullptr;
  if (jmap == nullptr) {  // the first positions; alpha, if any, is found in this pass
    if (q8 || wdw != nullptr) return hipErrorInvalidValue;
    if (pl.stream)
      hipLaunchKernelGGL((haar_keep_kernel<D, V, 1, 0, false, XT, true, true>), grid, dim3(256), 0, s, x, jmap, xc, alpha_slots,
                         wg_max, g, m, d.C_in, Cg, cstep, k, wdw, 0.f, nullptr, 0, nullptr, prefix);
    else
      hipLaunchKernelGGL((haar_keep_kernel<D, V, 1, 0, false, XT, false, true>), grid, dim3(256), 0, s, x, jmap, xc, alpha_slots,
                         wg_max, g, m, d.C_in, Cg, cstep, k, wdw, 0.f, nullptr, 0, nullptr, prefix);
    return hipGetLastError();
  }
#define WCC_KEEP(PF, DWM)                                                                          \
  do {                                                                                             \
    if (q8)                                                                                        \
      hipLaunchKernelGGL((haar_keep_kernel<D, V, PF, DWM, true, XT>), grid, dim3(256), 0, s, x,   \
                         jmap, xc, nullptr, nullptr, g, m, d.C_in, Cg, cstep, k, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, prefix);                    \
    else                                                                                           \
      hipLaunchKernelGGL((haar_keep_kernel<D, V, PF, DWM, false, XT>), grid, dim3(256), 0, s, x,  \
                         jmap, xc, alpha_slots, wg_max, g, m, d.C_in, Cg, cstep, k, wdw, 0.f, nullptr, 0, nullptr, prefix);                    \
  } while (0)
  if constexpr (V == 4 || D == 4) {
    if (wdw != nullptr) {  // K_dw in front of the transform
      if (dw_needs_edges(m)) WCC_KEEP(1, 2); else WCC_KEEP(1, 1);
      return hipGetLastError();
    }
  }
  if (wdw != nullptr) return hipErrorInvalidValue;
  if (pl.stream) {
    if (q8)
      hipLaunchKernelGGL((haar_keep_kernel<D, V, 1, 0, true, XT, true>), grid, dim3(256), 0, s, x,
                         jmap, xc, nullptr, nullptr, g, m, d.C_in, Cg, cstep, k, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, prefix);
    else
      hipLaunchKernelGGL((haar_keep_kernel<D, V, 1, 0, false, XT, true>), grid, dim3(256), 0, s, x,
                         jmap, xc, alpha_slots, wg_max, g, m, d.C_in, Cg, cstep, k, wdw, 0.f, nullptr, 0, nullptr, prefix);
    return hipGetLastError();
  }
  WCC_KEEP(1, 0);
#undef WCC_KEEP
  return hipGetLastError();
}

template <int D, int V>
hipError_t keep_launch(const wcc_desc &d, int64_t k, const void *x, const int32_t *jmap, void *xc,
                       float *alpha_slots, float *wg_max, Plan pl, const float *wdw, float q_alpha,
                       const float *alpha_src, int n_alpha, float *alpha_pub, int64_t prefix, hipStream_t s) {
  if (d.act_dtype == WCC_BF16)
    return keep_launch_t<D, V>(d, k, static_cast<const bf16_t *>(x), jmap, xc, alpha_slots, wg_max, pl, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, prefix, s);
  return keep_launch_t<D, V>(d, k, static_cast<const float *>(x), jmap, xc, alpha_slots, wg_max, pl, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, prefix, s);
}

}  // namespace

hipError_t keep_dispatch(const wcc_desc &d, int64_t k, const void *x, const int32_t *jmap, void *xc,
                         float *alpha_slots, float *wg_max, Plan pl, const float *wdw, float q_alpha,
                         const float *alpha_src, int n_alpha, float *alpha_pub, int64_t prefix, hipStream_t s) {
  const bool v4 = lane_cols(d) == 4;
  switch (d.levels) {
    case 1: return v4 ? keep_launch<1, 4>(d, k, x, jmap, xc, alpha_slots, wg_max, pl, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, prefix, s)
                      : keep_launch<1, 2>(d, k, x, jmap, xc, alpha_slots, wg_max, pl, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, prefix, s);
    case 2: return keep_launch<2, 4>(d, k, x, jmap, xc, alpha_slots, wg_max, pl, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, prefix, s);
    case 3: return keep_launch<3, 4>(d, k, x, jmap, xc, alpha_slots, wg_max, pl, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, prefix, s);
    case 4: return keep_launch<4, 2>(d, k, x, jmap, xc, alpha_slots, wg_max, pl, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, prefix, s);
  }
  return hipErrorInvalidValue;
}

// Groups of quads of channels, or 0: codes leave byte by byte.  As many groups as the byte-wise launch has, as long as its waves'
// walks, which end with the longest, grow by a tenth at most for going by whole quads (11 x 400 channels of 8 x 608, 64 groups
// of one or two quads, where the byte-wise ones walk 7 channels: layer 62 us, 58.5; in 100 groups of one quad 63.6; 8 x 618 of
// 48 x 332, 18 groups in place of 16, which fill the chip evenly: 65 and 57).  Where there are fewer quads than groups
// they make do with as many waves as the quads give, from a thousand on.
static int quad_groups(const wcc_desc &d) {
  const int G0 = keep_groups(d, false, false), quads = (d.C_in + 3) / 4;
  const int64_t units = keep_map(d, false).units;
  int G = 0;
  if (quads <= G0) G = units * quads * d.B >= kQuadWaves ? quads : 0;
  else if (40 * ((quads + G0 - 1) / G0) <= 11 * ((d.C_in + G0 - 1) / G0)) G = G0;
  if (G == 0) return 0;
  // From three levels on two workgroups of this pass share a compute unit, of the byte-wise one three: a last round of them that is
  // half empty or more costs short walks more than the words give, up to a half kept.  Layers by words and by bytes: 8 x 128 channels of
  // 96 x 160, 768 workgroups of one quad, half kept, 74.0 us and 70.0; 12 x 496 of 80 x 32 at four levels, two quads, 80.6 and 71.3; 4 x 128 of
  // 128 x 320, 640 of one, 76.1 and 73.5, all kept 87.8 and 90.2; in full rounds, and with four quads and more, 0.91 to 1.01.
  const int64_t wgs = (units + 3) / 4 * G * d.B, rounds = (wgs + kQuadRound - 1) / kQuadRound;
  const bool few = 2 * kept_count(d) <= (int64_t)d.H * d.W;
  if (d.levels >= 3 && few && quads <= 3 * G && wgs > kQuadRound && 3 * kQuadRound * rounds >= 4 * wgs) return 0;
  return G;
}

// ... with K_dw in front: quads a group, or 0.  (At three levels, short walks in a second round as above, whatever is kept.  Blocks by words and by
// bytes: 6 x 960 channels of 48 x 56, 720 workgroups of two quads, half kept, 200 us and 188; 7 x 1008 of 16 x 256, 882 of two, all kept, 309 and
// 304; 5 x 512 of 48 x 184, 640 of two, 294 and 291; 7 x 336 of 88 x 184, 588 of three, 355 and 360.)
static int dw_quads_a_group(const wcc_desc &d) {
  const int G0 = keep_groups(d, true, false), quads = (d.C_in + 3) / 4, each = (quads + G0 - 1) / G0;
  if (d.act_dtype != WCC_F32 || quads < G0 || 40 * each > 11 * ((d.C_in + G0 - 1) / G0)) return 0;
  const int64_t wgs = (int64_t)(keep_map(d, true).units + 3) / 4 * ((quads + each - 1) / each) * d.B;
  return d.levels == 3 && each <= 3 && 4 * wgs >= 5 * kQuadRound ? 0 : each;
}

bool keep_in_quads(const wcc_desc &d, bool folded) { return folded ? dw_quads_a_group(d) > 0 : quad_groups(d) > 0; }

template <int D, int V>
static hipError_t dw_quads_launch(const wcc_desc &d, int64_t ks, const float *x, const int32_t *jmap, uint32_t *xw,
                                  const float *wdw, float q_alpha, const float *alpha_src, int n_alpha, float *alpha_pub,
                                  hipStream_t s) {
  const Geo g{d.H, d.W, d.levels, (int64_t)d.H * d.W};
  const StripMap m = keep_map(d, true);
  const int Cq = dw_quads_a_group(d);
  const dim3 grid((m.units + 3) / 4, ((d.C_in + 3) / 4 + Cq - 1) / Cq, d.B);
  if (dw_needs_edges(m))
    hipLaunchKernelGGL((haar_keep_dw_quads_kernel<D, V, 2>), grid, dim3(256), 0, s, x, jmap, xw, g, m, d.C_in, Cq, ks, wdw, q_alpha,
                       alpha_src, n_alpha, alpha_pub);
  else
    hipLaunchKernelGGL((haar_keep_dw_quads_kernel<D, V, 1>), grid, dim3(256), 0, s, x, jmap, xw, g, m, d.C_in, Cq, ks, wdw, q_alpha,
                       alpha_src, n_alpha, alpha_pub);
  return hipGetLastError();
}

template <int D, int V, class XT>
static hipError_t quads_launch(const wcc_desc &d, int64_t ks, const void *x, const int32_t *jmap, uint32_t *xw, float q_alpha,
                               const float *alpha_src, int n_alpha, float *alpha_pub, hipStream_t s) {
  const Geo g{d.H, d.W, d.levels, (int64_t)d.H * d.W};
  const StripMap m = keep_map(d, false);
  const dim3 grid((m.units + 3) / 4, quad_groups(d), d.B);
  if (streams(d))
    hipLaunchKernelGGL((haar_keep_quads_kernel<D, V, XT, true>), grid, dim3(256), 0, s, static_cast<const XT *>(x), jmap, xw, g,
                       m, d.C_in, ks, q_alpha, alpha_src, n_alpha, alpha_pub);
  else
    hipLaunchKernelGGL((haar_keep_quads_kernel<D, V, XT, false>), grid, dim3(256), 0, s, static_cast<const XT *>(x), jmap, xw, g,
                       m, d.C_in, ks, q_alpha, alpha_src, n_alpha, alpha_pub);
  return hipGetLastError();
}

hipError_t launch_haar_keep_quads(const wcc_desc &d, int64_t ks, const void *x, const int32_t *jmap, uint32_t *xw, const float *wdw,
                                  float q_alpha, const float *alpha_src, int n_alpha, float *alpha_pub, hipStream_t s) {
  if (!keep_in_quads(d, wdw != nullptr)) return hipErrorInvalidValue;
  if (wdw != nullptr) {
    const float *xf = static_cast<const float *>(x);
    switch (d.levels) {
      case 1: return lane_cols(d) == 4 ? dw_quads_launch<1, 4>(d, ks, xf, jmap, xw, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, s)
                                       : hipErrorInvalidValue;
      case 2: return dw_quads_launch<2, 4>(d, ks, xf, jmap, xw, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, s);
      case 3: return dw_quads_launch<3, 4>(d, ks, xf, jmap, xw, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, s);
      case 4: return dw_quads_launch<4, 2>(d, ks, xf, jmap, xw, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, s);
    }
    return hipErrorInvalidValue;
  }
#define WCC_QUADS(D, V)                                                                                                 \
  return d.act_dtype == WCC_BF16                                                                                        \
             ? quads_launch<D, V, bf16_t>(d, ks, x, jmap, xw, q_alpha, alpha_src, n_alpha, alpha_pub, s)        \
             : quads_launch<D, V, float>(d, ks, x, jmap, xw, q_alpha, alpha_src, n_alpha, alpha_pub, s)
  switch (d.levels) {
    case 1: if (lane_cols(d) == 4) WCC_QUADS(1, 4); else WCC_QUADS(1, 2);
    case 2: WCC_QUADS(2, 4);
    case 3: WCC_QUADS(3, 4);
    case 4: WCC_QUADS(4, 2);
  }
#undef WCC_QUADS
  return hipErrorInvalidValue;
}

int64_t keep_workgroups(const wcc_desc &d, bool folded) {
  return (int64_t)((keep_map(d, folded).units + 3) / 4) * keep_groups(d, folded, true) * d.B;
}

hipError_t launch_haar_keep(const wcc_desc &d, int64_t k, const void *x, const int32_t *jmap,
                            void *xc, float *alpha_slots, float *wg_max, const float *wdw, float q_alpha,
                            const float *alpha_src, int n_alpha, float *alpha_pub, int64_t prefix, hipStream_t s) {
  const bool late = alpha_slots != nullptr || wg_max != nullptr;
  const Plan pl{keep_groups(d, wdw != nullptr, late), 1, streams(d), 1};
  return keep_dispatch(d, k, x, jmap, xc, alpha_slots, wg_max, pl, wdw, q_alpha, alpha_src, n_alpha, alpha_pub, prefix, s);
}

int64_t keep_words_workgroups(const wcc_desc &d) {
  return (int64_t)((words_map(d).units + 3) / 4) * words_groups(d, true) * d.B;
}

hipError_t launch_haar_keep_words(const wcc_desc &d, int64_t ks, const void *x, const int32_t *jmap,
                                  const uint32_t *ucount, uint32_t *xw, float *alpha_slots, float *wg_max,
                                  float q_alpha, const float *alpha_src, int n_alpha, float *alpha_pub, hipStream_t s) {
  if (d.levels != WordSink::D) return hipErrorInvalidValue;
  return d.act_dtype == WCC_BF16
             ? words_launch(d, ks, static_cast<const bf16_t *>(x), jmap, ucount, xw, alpha_slots, wg_max, q_alpha,
                            alpha_src, n_alpha, alpha_pub, s)
             : words_launch(d, ks, static_cast<const float *>(x), jmap, ucount, xw, alpha_slots, wg_max, q_alpha,
                            alpha_src, n_alpha, alpha_pub, s);
}

}  // namespace wcc
