// Compressed-domain chaining of the inverted residual block (appendix "Inference times",
// paragraph on memory bandwidth and traffic: Haar transform, depthwise convolution and
// gather / scatter applied separately per channel and in parts, with small intermediates, the
// full result kept only in compressed form).
//
// The project layer's input is K_dw t1 with t1 = iHWT(T^T Y_wt) the expand layer's output.  The
// two transform passes of the project layer (channel norms; kept coefficients) take t1 from
// where it already is in compressed form -- the expand layer's Y_wt [B, C, k] and its rank map
// -- instead of from a feature map in memory: per channel a wave rebuilds the 2^d rows of its
// strip and the one row above and below it (inverse transform of the kept values, everything
// else zero), convolves them with the channel's 3x3 kernel and transforms the result again, all
// in registers and LDS.  The expanded feature map, the largest tensor of the block, is neither
// written nor read; the passes read k/N of it, twice.  This is also the mirror fusion "inverse
// transform followed by the depthwise convolution".
//
// The arithmetic is that of the kernels it replaces, operation by operation (synthesis
// butterflies of haar_inv.hip, multiply-adds in the order of depthwise.hip, analysis of strip.h),
// so the values that enter the norms and the quantiser are the same bits.
//
// A row of the plane wider than one wave row (256 columns) is shared by the 2 or 4 waves of a
// workgroup, one 256-column segment each: per channel every wave leaves the first and last
// column of its rebuilt rows in LDS, the workgroup meets at a barrier, and the end lanes take the
// convolution's outside column from the neighbouring segment there.
//
// Limits (the caller falls back to the materialised route otherwise): W % 4 == 0, d <= 3, and
// W <= 256 or a row made of exactly 2 or 4 wave rows (256 < W <= 512, 768 < W <= 1024).
#include "strip_io.h"

namespace wcc {
namespace {

constexpr int V4 = 4;

// ---- slots of ONE row of a strip (the halo rows) -------------------------------------------------
// To rebuild a single image row only the band row that contains it is needed at every level.
__host__ __device__ constexpr int hslot_base(int D, int V, int l, int j) {
  int s = 0;
  for (int m = 1; m < l; ++m) s += 3 * cols_at(V, m);
  return s + (l == D ? j : j - 1) * cols_at(V, l);
}
__host__ __device__ constexpr int hslot_count(int D, int V) {
  return hslot_base(D, V, D, 3) + cols_at(V, D);
}

// (the [lane][slot] tile layout and RegStrip, the source that reads a lane's slots back from
// registers, are in strip_io.h: the inverse transform uses them too)
template <int D, int V, int N>
struct RegRow {
  const float (&c)[N];
  int first;  // the halo row's first slot
  template <int L, int J>
  __device__ __forceinline__ void get(float (&v)[cols_at(V, L)]) const {
    constexpr int CV = cols_at(V, L);
    constexpr int base = hslot_base(D, V, L, J);
#pragma unroll
    for (int e = 0; e < CV; ++e) v[e] = c[first + base + e];
  }
};

// The passes are bound by their vector instructions, so the factors 1/2 of the butterflies are left out where a power of two
// can be carried along instead (scaling by it is exact, so the sums and roundings are those of the transforms of the
// other routes, bit for bit, where nothing is smaller than a normal number): a level of the synthesis returns twice its
// rows, and the level below halves them inside a multiply-add; the convolution's taps take 2^-(D + 1), so that the analysis
// leaves the coefficients of level l scaled by 2^(l - D), at most what they are: nothing overflows that the other
// routes hold, and what lies below 2^-122 may lose bits.  The sinks take the powers off: the norm pass once a walk (of squares before
// they are squared), the keep pass in the multiplication it had.  Vector instructions a channel of the norm pass 709 -> 601.
// With the scale on the coefficients, up to 16 times what they are, and none on the taps it was 591, but the norms
// overflowed from 2^124 on; 8 x 1024 channels of 256 x 256, a quarter kept, in one run: norm pass 335 -> 323 us on smooth maps and 320 -> 332 on
// noise, whose lists are of other lengths, keep pass 441 -> 439 and 436 -> 435.

// 2^-P v for a value that is the same in every lane, on its bits by scalar instructions: there are no scalar multiplications, and the
// vector's put nine taps into registers of every lane.  What falls below the normal numbers becomes zero.  For the keep pass at three
// levels, which is short of registers: 8 x 1024 channels of 256 x 256, a quarter kept, 449 -> 435 us, 2 x 512 of 64 x 64 34.7 -> 32.0; at two
// levels it loses (4 x 384 of 192 x 192 87.5 -> 89.8), and so does the norm pass, which then waits for the taps at once (324 -> 360-474).
template <int P>
__device__ __forceinline__ float scaled_down(float v) {
  const uint32_t bits = __float_as_uint(v);
  return __uint_as_float((bits & 0x7F800000u) > ((uint32_t)P << 23) ? bits - ((uint32_t)P << 23) : bits & 0x80000000u);
}

// Synthesis levels D..L of a strip: twice its rows of level L - 1 (inv_levels without the factors).
template <int D, int V, int L, class Source>
__device__ __forceinline__ void inv_levels_twice(float (&out)[rows_at(D, L - 1)][cols_at(V, L - 1)], const LanePos<D> &p,
                                                 const Source &src) {
  constexpr int R2 = rows_at(D, L), VI = cols_at(V, L - 1), V2 = cols_at(V, L);
  constexpr int SI = span_at(V, L - 1);
  float ll[R2][V2];
  if constexpr (L < D) {
    inv_levels_twice<D, V, L + 1>(ll, p, src);
  } else {
#pragma unroll
    for (int i = 0; i < R2; ++i) src.template get_row<L, 0>(i, ll[i]);
  }
#pragma unroll
  for (int i = 0; i < R2; ++i) {
    float y2[V2], y3[V2], y4[V2];
    src.template get_row<L, 1>(i, y2);
    src.template get_row<L, 2>(i, y3);
    src.template get_row<L, 3>(i, y4);
#pragma unroll
    for (int e = 0; e < V2; ++e) {
      const float s1 = L < D ? fmaf(0.5f, ll[i][e], y3[e]) : ll[i][e] + y3[e];
      const float s2 = L < D ? fmaf(0.5f, ll[i][e], -y3[e]) : ll[i][e] - y3[e];
      const float d1 = y2[e] + y4[e], d2 = y2[e] - y4[e];
      if constexpr (VI >= 2) {
        out[2 * i][2 * e] = s1 + d1; out[2 * i][2 * e + 1] = s1 - d1;
        out[2 * i + 1][2 * e] = s2 + d2; out[2 * i + 1][2 * e + 1] = s2 - d2;
      } else {
        // every lane of the group holds the same (y1..y4); the left half keeps the left pixel
        const bool left = (p.lc & SI) == 0;
        out[2 * i][0] = s1 + (left ? d1 : -d1);
        out[2 * i + 1][0] = s2 + (left ? d2 : -d2);
      }
    }
  }
}

// One image row of a strip: its last one (BOTTOM) or its first one.  The same expressions as
// inv_levels_twice evaluates for that row.
template <int D, int V, int L, bool BOTTOM, class Source>
__device__ __forceinline__ void inv_row_twice(float (&out)[cols_at(V, L - 1)], const LanePos<D> &p,
                                              const Source &src) {
  constexpr int VI = cols_at(V, L - 1), V2 = cols_at(V, L);
  constexpr int SI = span_at(V, L - 1);
  float ll[V2];
  if constexpr (L < D) inv_row_twice<D, V, L + 1, BOTTOM>(ll, p, src);
  else src.template get<L, 0>(ll);
  float y2[V2], y3[V2], y4[V2];
  src.template get<L, 1>(y2);
  src.template get<L, 2>(y3);
  src.template get<L, 3>(y4);
#pragma unroll
  for (int e = 0; e < V2; ++e) {
    const float y3s = BOTTOM ? -y3[e] : y3[e];
    const float s = L < D ? fmaf(0.5f, ll[e], y3s) : ll[e] + y3s;
    const float d = BOTTOM ? y2[e] - y4[e] : y2[e] + y4[e];
    if constexpr (VI >= 2) {
      out[2 * e] = s + d;
      out[2 * e + 1] = s - d;
    } else {
      out[0] = s + (((p.lc & SI) == 0) ? d : -d);
    }
  }
}

// Analysis levels L..D: `in` holds 2^(L - 1 - D) times the rows of level L - 1; the sink gets the coefficients as they are, or
// (Sink::kScaled) 2^(level - D) times them.
template <int D, int V, int L, class Sink>
__device__ __forceinline__ void fwd_levels_scaled(const float (&in)[rows_at(D, L - 1)][cols_at(V, L - 1)],
                                                  const LanePos<D> &p, Sink &sink) {
  constexpr int R2 = rows_at(D, L), VI = cols_at(V, L - 1), V2 = cols_at(V, L);
  constexpr int SI = span_at(V, L - 1), S2 = span_at(V, L);
  constexpr float kScale = Sink::kScaled ? 1.f : (float)(1 << (D - L));
  float ll[R2][V2];
  const bool owner = p.active && ((S2 == 1) || ((p.lc & (S2 - 1)) == 0));
#pragma unroll
  for (int i = 0; i < R2; ++i) {
    float y1[V2], y2[V2], y3[V2], y4[V2];
#pragma unroll
    for (int e = 0; e < V2; ++e) {
      float a, b, c, d;
      if constexpr (VI >= 2) {
        a = in[2 * i][2 * e]; b = in[2 * i][2 * e + 1];
        c = in[2 * i + 1][2 * e]; d = in[2 * i + 1][2 * e + 1];
      } else {
        const float o0 = in[2 * i][0], o1 = in[2 * i + 1][0];
        const float q0 = lane_xor<SI>(o0), q1 = lane_xor<SI>(o1);
        const bool left = (p.lc & SI) == 0;
        a = left ? o0 : q0; b = left ? q0 : o0;
        c = left ? o1 : q1; d = left ? q1 : o1;
      }
      const float s1 = a + b, s2 = c + d, d1 = a - b, d2 = c - d;
      ll[i][e] = s1 + s2;
      y1[e] = kScale * ll[i][e];
      y2[e] = kScale * (d1 + d2);
      y3[e] = kScale * (s1 - s2);
      y4[e] = kScale * (d1 - d2);
    }
    sink.template put_row<L, 1>(p, i, y2, owner);
    sink.template put_row<L, 2>(p, i, y3, owner);
    sink.template put_row<L, 3>(p, i, y4, owner);
    if constexpr (L == D) sink.template put_row<L, 0>(p, i, y1, owner);
  }
  if constexpr (L < D) fwd_levels_scaled<D, V, L + 1>(ll, p, sink);
}

// Sink of the norm pass: per slot the sum of |coefficient| (SQ: of squares) and the largest |coefficient| over the
// channels, of scaled coefficients until finish() (but for the squares).
template <int D, bool SQ>
struct ChainNormSink {
  static constexpr bool kScaled = true;
  float acc[slot_count(D, V4)], top[slot_count(D, V4)];
  template <int L, int J>
  __device__ __forceinline__ void put_row(const LanePos<D> &, int i, const float (&v)[cols_at(V4, L)], bool) {
    constexpr int CV = cols_at(V4, L), base = slot_base(D, V4, L, J);
#pragma unroll
    for (int e = 0; e < CV; ++e) {
      float &a = acc[base + i * CV + e], &t = top[base + i * CV + e];
      const float c = (float)(1 << (D - L)) * v[e];  // (squares leave the normal numbers early enough unscaled)
      a = SQ ? fmaf(c, c, a) : a + fabsf(v[e]);
      // (fmaxf first quiets a value that the compiler does not know to be quiet: a second instruction a slot)
      asm("v_max_f32_e64 %0, %1, |%2|" : "=v"(t) : "v"(t), "v"(v[e]));
    }
  }
  __device__ __forceinline__ void finish() {
    auto level = [&](auto Lc) {
      constexpr int L = decltype(Lc)::value;
      constexpr float kUp = (float)(1 << (D - L));
      constexpr int first = slot_base(D, V4, L, L == D ? 0 : 1), last = L == D ? slot_count(D, V4) : slot_base(D, V4, L, 3) + rows_at(D, L) * cols_at(V4, L);
#pragma unroll
      for (int s = first; s < last; ++s) {
        if constexpr (!SQ) acc[s] *= kUp;
        top[s] *= kUp;
      }
    };
    level(std::integral_constant<int, 1>{});
    if constexpr (D >= 2) level(std::integral_constant<int, 2>{});
    if constexpr (D >= 3) level(std::integral_constant<int, 3>{});
  }
};

// ---- the channel walk ----------------------------------------------------------------------------
constexpr int kChainCap = 2048;  // packed entries per wave (32 a lane)

// What a wave knows about the producer layer's kept positions around its strip.
template <int D>
struct ChainGeo {
  static constexpr int NS = slot_count(D, V4), HS = hslot_count(D, V4), NT = NS + 2 * HS;
  static constexpr int STRIDE = tile_stride(NT);  // words between two lanes' slots in the tile
  uint64_t any;        // wave-uniform: bit s set if some lane keeps slot s (NT <= 64)
  int count;           // kept entries of the wave (wave-uniform)
  bool packed;         // the tile holds the wave's packed list (rank | cell << kInvRankBits)
  int jj[NT];          // rank in the producer's list of the lane's slot, or -1 (used if !packed)
};

// Calls f(slot, position in the producer's rank map, exists) for the lane's NT slots: the strip's
// own NS slots, then the HS slots of the band rows that hold the image row above the strip,
// then those of the row below.
template <int D, class F>
__device__ __forceinline__ void chain_slots(const LanePos<D> &p, bool active, bool up_in, bool dn_in,
                                            F &&f) {
  constexpr int NS = ChainGeo<D>::NS, HS = ChainGeo<D>::HS;
  auto band_rows = [&](auto Lc, auto Jc) {
    constexpr int L = decltype(Lc)::value, J = decltype(Jc)::value;
    constexpr int CV = cols_at(V4, L);
    const int band = J * p.nl[L] + p.off[L];
#pragma unroll
    for (int i = 0; i < rows_at(D, L); ++i)
#pragma unroll
      for (int e = 0; e < CV; ++e) f(slot_base(D, V4, L, J) + i * CV + e, band + i * p.rowlen[L] + e, active);
#pragma unroll
    for (int e = 0; e < CV; ++e) {
      f(NS + hslot_base(D, V4, L, J) + e, band - p.rowlen[L] + e, active && up_in);
      f(NS + HS + hslot_base(D, V4, L, J) + e, band + rows_at(D, L) * p.rowlen[L] + e, active && dn_in);
    }
  };
  auto each_level = [&](auto Lc) {
    constexpr int L = decltype(Lc)::value;
    band_rows(Lc, std::integral_constant<int, 1>{});
    band_rows(Lc, std::integral_constant<int, 2>{});
    band_rows(Lc, std::integral_constant<int, 3>{});
    if constexpr (L == D) band_rows(Lc, std::integral_constant<int, 0>{});
  };
  each_level(std::integral_constant<int, 1>{});
  if constexpr (D >= 2) each_level(std::integral_constant<int, 2>{});
  if constexpr (D >= 3) each_level(std::integral_constant<int, 3>{});
}

// Looks up the lane's slots in the producer's rank map jm1 (one sample) and, if the wave keeps
// at most kChainCap of them (and the ranks fit their bit field), packs (rank, cell) into `tile`:
// slot-major, then lane.
template <int D>
__device__ __forceinline__ ChainGeo<D> chain_setup(const int32_t *__restrict__ jm1, int64_t k1,
                                                   const LanePos<D> &p, bool active, bool up_in,
                                                   bool dn_in, uint32_t *tile) {
  constexpr int NT = ChainGeo<D>::NT;
  static_assert(NT <= 64, "one 64-bit slot mask");
  constexpr int STRIDE = ChainGeo<D>::STRIDE;
  static_assert(STRIDE * kWave <= (1 << (32 - kInvRankBits)), "cell index fits above the rank");
  static_assert(NT % 4 == 0 && STRIDE % 4 == 0, "16-byte reads of a lane's slots");
  const int lane = threadIdx.x & (kWave - 1);
  ChainGeo<D> cg;
  int (&jj)[NT] = cg.jj;
  chain_slots<D>(p, active, up_in, dn_in, [&](int s, int pos, bool exists) {
    int j = -1;
    if (exists) j = jm1[pos];
    jj[s] = j;
  });
  cg.any = 0;
  cg.count = 0;
#pragma unroll
  for (int s = 0; s < NT; ++s) {
    const uint64_t kept = __ballot(jj[s] >= 0);
    if (kept != 0) cg.any |= (uint64_t)1 << s;
    cg.count += __popcll(kept);
  }
  cg.packed = cg.count <= kChainCap && k1 <= ((int64_t)1 << kInvRankBits);
  if (cg.packed) {
    int running = 0;
#pragma unroll
    for (int s = 0; s < NT; ++s) {
      if ((cg.any >> s) & 1) {
        const int j = jj[s];
        const uint64_t kept = __ballot(j >= 0);
        const int at = running + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u));
        if (j >= 0) tile[at] = (uint32_t)j | ((uint32_t)(lane * STRIDE + s) << kInvRankBits);
        running += __popcll(kept);
      }
    }
    wave_lds_fence();
  }
  return cg;
}

// Walks n_ch channels of the producer's compressed output yc1 (first channel at `plane`, channel
// stride k1): per channel the kept values around the strip go into the wave's LDS
// tile (laid out [lane][slot]; its other cells stay zero), the strip's 2^d rows and the rows above and below are
// rebuilt from it, convolved with the channel's 3x3 kernel (wdw: first channel's, 9 floats a
// channel) and transformed into `sink`; after(sink) runs once per channel.
// Waves whose list is packed fetch it with dense loads, one channel ahead; the others
// (strips that keep more than kChainCap positions) load slot by slot from the ranks they hold in
// registers, a channel's loads in flight together.
// NI_FIXED > 0: the packed list is walked with that many rows a wave (the caller has checked that
// it fits); 0: the shortest of 4, 8, 16, 24, 32 rows that holds it.
// SEGS > 1: the plane's row is shared by the SEGS waves of the workgroup (this one holds segment
// `seg`); xchg is the workgroup's exchange buffer (ChainXchg<D, SEGS>::kWords floats).  Every wave
// of the workgroup then runs compute() once per channel, whatever path it takes: one barrier each.
template <int D, int SEGS, int NI_FIXED = 0, class Sink, class After>
__device__ __forceinline__ void chain_walk(const float *__restrict__ plane, int64_t k1, int n_ch,
                                           const float *__restrict__ wdw, const ChainGeo<D> &cg,
                                           uint32_t *tile, const LanePos<D> &p, bool first_lane,
                                           bool last_lane, float *xchg, int seg, Sink &sink,
                                           After &&after) {
  constexpr int R = 1 << D, RR = R + 2, V = V4;
  int parity = 0;  // which half of the exchange buffer this channel uses
  constexpr int NS = ChainGeo<D>::NS, HS = ChainGeo<D>::HS, NT = ChainGeo<D>::NT;
  constexpr int STRIDE = ChainGeo<D>::STRIDE;
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t *mine_row = tile + lane * STRIDE;  // this lane's slots

  // the tile holds a channel's kept values: rebuild, convolve with kw[0..8], transform
  auto compute = [&](const float *kw) {
    float k[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)  // (the rows below are twice what they are)
      k[t] = !Sink::kScaled && D == 3 ? scaled_down<D + 1>(kw[t]) : kw[t] * (1.f / (float)(2 << D));
    wave_lds_fence();
    float six[RR][V + 2];
    {
      float cells[NT];
#pragma unroll
      for (int q = 0; q < NT / 4; ++q) {
        const float4 t = reinterpret_cast<const float4 *>(mine_row)[q];
        cells[4 * q] = t.x; cells[4 * q + 1] = t.y; cells[4 * q + 2] = t.z; cells[4 * q + 3] = t.w;
      }
      const RegStrip<D, V, NT> own{cells};
      const RegRow<D, V, NT> up{cells, NS}, dn{cells, NS + HS};
      float mid[R][V];
      inv_levels_twice<D, V, 1>(mid, p, own);
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int e = 0; e < V; ++e) six[r + 1][e + 1] = mid[r][e];
      float edge[V];
      inv_row_twice<D, V, 1, true>(edge, p, up);
#pragma unroll
      for (int e = 0; e < V; ++e) six[0][e + 1] = edge[e];
      inv_row_twice<D, V, 1, false>(edge, p, dn);
#pragma unroll
      for (int e = 0; e < V; ++e) six[RR - 1][e + 1] = edge[e];
    }
    wave_lds_fence();
    // the column beyond a wave row's end: the plane's zero border, or (SEGS > 1) the neighbouring
    // segment's boundary column.  Two buffers alternate: a wave can be one barrier ahead of
    // another, never two, so the buffer it writes is not the one a slower wave still reads.
    float beyond[RR];
#pragma unroll
    for (int i = 0; i < RR; ++i) beyond[i] = 0.f;
    // (a last segment of a single lane: that lane is first and last at once; `beyond` then holds
    // the column to its left, and to its right lies the plane's border)
    bool left_only = false;
    if constexpr (SEGS > 1) {
      float *ex = xchg + parity * (SEGS * 2 * RR);
      parity ^= 1;
      // (the lane number is computed afresh here, by instructions the compiler may not move out
      // of the loop: kept across the loop it is spilled, and the reload of a spilled register
      // waits for every load in flight, the prefetched channels included)
      int ln;
      asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
      const bool at0 = ln == 0, at63 = ln == kWave - 1;
      if (at0 || at63) {
        float *out = ex + (seg * 2 + (at0 ? 0 : 1)) * RR;
#pragma unroll
        for (int i = 0; i < RR; ++i) out[i] = at0 ? six[i][1] : six[i][V];
      }
      workgroup_lds_barrier();  // (the next channels' values keep travelling)
      if ((at0 && seg > 0) || (at63 && seg < SEGS - 1)) {
        const float *in = ex + (at0 ? (seg - 1) * 2 + 1 : (seg + 1) * 2) * RR;
#pragma unroll
        for (int i = 0; i < RR; ++i) beyond[i] = in[i];
      }
      left_only = at0;
    }
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      // (the neighbouring lanes' columns: through LDS where the vector unit is the bound, by its data-parallel moves in the
      // keep pass, which keeps LDS busy as it is: 455 -> 440 us there, 333 -> 339 in the norm pass, both with the taps unscaled)
      float l, r;
      if constexpr (Sink::kScaled) {
        l = __shfl_up(six[i][V], 1, kWave);
        r = __shfl_down(six[i][1], 1, kWave);
      } else {
        l = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(six[i][V]), 0x138, 0xf, 0xf, true));  // wave_shr:1
        r = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(six[i][1]), 0x130, 0xf, 0xf, true));  // wave_shl:1
      }
      if (first_lane) l = beyond[i];
      if (last_lane) r = left_only ? 0.f : beyond[i];
      six[i][0] = l;
      six[i][V + 1] = r;
    }
    float t1[R][V];
#pragma unroll
    for (int o = 0; o < R; ++o) {
#pragma unroll
      for (int e = 0; e < V; ++e) t1[o][e] = 0.f;
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
          for (int e = 0; e < V; ++e) t1[o][e] = fmaf(k[i * 3 + j], six[o + i][e + j], t1[o][e]);
    }
    fwd_levels_scaled<D, V, 1>(t1, p, sink);
    after(sink);
  };

  if (cg.packed) {
    auto run = [&](auto ni_c) {
      constexpr int NI = decltype(ni_c)::value;
      constexpr uint32_t kRank = (1u << kInvRankBits) - 1u;
      // this lane's share of the list: entries lane + 64 i.  Past the end of the list an entry
      // repeats the list's first one: it fetches the same value and drops it into the same cell,
      // so no load and no LDS write needs a lane mask or a branch.
      uint32_t mine[NI];
      const uint32_t first = tile[0];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int e = lane + kWave * i;
        mine[i] = e < cg.count ? tile[e] : first;
      }
      wave_lds_fence();
#pragma unroll
      for (int s = 0; s < NT; ++s) mine_row[s] = 0u;
      auto fetch = [&](float (&dst)[NI], int ch) {  // (past the last channel: the last again)
        const float *nx = plane + (size_t)min(ch, n_ch - 1) * k1;
#pragma unroll
        for (int i = 0; i < NI; ++i) dst[i] = nx[mine[i] & kRank];
      };
      auto drop = [&](const float (&src)[NI]) {
#pragma unroll
        for (int i = 0; i < NI; ++i) tile[mine[i] >> kInvRankBits] = __float_as_uint(src[i]);
      };
      // One channel of values in flight ahead of the one being worked on.  (Two for short lists double the loops, and with
      // them the code that waves on lists of different lengths run side by side: norm pass 351 us, 336 now.)
      float vn[NI];
      fetch(vn, 0);
      for (int c = 0; c < n_ch; ++c) {
        drop(vn);
        fetch(vn, c + 1);  // travels while this channel is worked on
        __builtin_amdgcn_sched_barrier(0);
        compute(wdw + (size_t)c * 9);
      }
    };
    if (cg.count == 0) {  // nothing kept around this strip: every channel is zero
#pragma unroll
      for (int s = 0; s < NT; ++s) mine_row[s] = 0u;
      for (int c = 0; c < n_ch; ++c) compute(wdw + (size_t)c * 9);
      return;
    }
    if constexpr (NI_FIXED > 0) {
      run(std::integral_constant<int, NI_FIXED>{});
    } else {
      const int ni = (cg.count + kWave - 1) >> 6;
      if (ni <= 4) run(std::integral_constant<int, 4>{});
      else if (ni <= 8) run(std::integral_constant<int, 8>{});
      else if (ni <= 16) run(std::integral_constant<int, 16>{});
      else if (ni <= 24) run(std::integral_constant<int, 24>{});
      else run(std::integral_constant<int, 32>{});
    }
    return;
  }

  // plain path: one load per slot that some lane keeps, all of a channel's loads in flight together
#pragma unroll
  for (int s = 0; s < NT; ++s) mine_row[s] = 0u;
  for (int c = 0; c < n_ch; ++c) {
    const float *pc = plane + (size_t)c * k1;
    float v[NT];
#pragma unroll
    for (int s = 0; s < NT; ++s) v[s] = pc[max(cg.jj[s], 0)];
#pragma unroll
    for (int s = 0; s < NT; ++s) mine_row[s] = cg.jj[s] >= 0 ? __float_as_uint(v[s]) : 0u;
    compute(wdw + (size_t)c * 9);
  }
}

// Sink of the keep pass for a strip that keeps few of its positions (the counterpart of
// KeepStagedSink for the [lane][slot] tile): every lane drops its coefficients into its own
// slots of the tile -- free once the channel's rows have been rebuilt from it --, the wave picks
// the values of the strip's packed list of kept positions from there and stores NI dense rows
// (only those are quantised), and the lane's own slots are cleared again for the next channel.
template <int D, bool Q8, int NI>
struct ChainStagedSink {
  using Out = std::conditional_t<Q8, int8_t, float>;
  static constexpr bool kScaled = false;
  static constexpr uint32_t kDropped = 0xFFFFFFFFu;
  static constexpr int NS = slot_count(D, V4);
  __amdgpu_buffer_rsrc_t xc_c;  // xc[b, c, :]
  uint32_t *tile;               // the wave's tile
  uint32_t *row;                // this lane's slots in it
  uint32_t cell[NI];            // tile index of the entry's position
  uint32_t at[NI];              // byte offset of the entry's rank, or kDropped (list padding)
  float vmax;
  Quant quant;
  __device__ __forceinline__ explicit ChainStagedSink(float alpha) : quant(alpha) {}
  __device__ __forceinline__ void aim(Out *plane, int64_t k) {
    xc_c = __builtin_amdgcn_make_buffer_rsrc(plane, 0, (int)(uint32_t)(k * (int64_t)sizeof(Out)),
                                             0x00020000 /* raw dwords, no swizzle */);
  }
  template <int L, int J>
  __device__ __forceinline__ void put_row(const LanePos<D> &p, int i, const float (&v)[cols_at(V4, L)],
                                          bool owner) {
    constexpr int CV = cols_at(V4, L);
    constexpr int base = slot_base(D, V4, L, J);
    (void)p;
    (void)owner;  // (a value a lane does not own is in no list)
#pragma unroll
    for (int e = 0; e < CV; ++e) row[base + i * CV + e] = __float_as_uint(v[e]);
  }
  // once per channel, after the last level
  __device__ __forceinline__ void flush() {
    wave_lds_fence();
    if constexpr (Q8) {
      // which division the quantiser takes is the same for every value of the layer: chosen
      // once per channel here, not value by value (three branches a value otherwise)
      float v[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) v[i] = __uint_as_float(tile[cell[i]]);
      auto store_codes = [&](auto fast_c) {
        constexpr bool FAST = decltype(fast_c)::value;
#pragma unroll
        for (int i = 0; i < NI; ++i)
          __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(int8_t)(int)quant.template level_as<FAST>(v[i]),
                                               xc_c, at[i], 0, 0);
      };
      if (quant.fast) store_codes(std::true_type{});
      else store_codes(std::false_type{});
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const float v = __uint_as_float(tile[cell[i]]);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), xc_c, at[i], 0, 0);
        vmax = fmaxf(vmax, at[i] != kDropped ? fabsf(v) : 0.f);
      }
    }
    wave_lds_fence();
    // the strip's own slots go back to zero (the slots that round NS up to a multiple of four
    // belong to the row above: zero as well until the next channel's values are dropped in)
#pragma unroll
    for (int q = 0; q < (NS + 3) / 4; ++q) reinterpret_cast<uint4 *>(row)[q] = make_uint4(0u, 0u, 0u, 0u);
    wave_lds_fence();
  }
};

// Waves per workgroup: two (independent of each other when a wave row holds a whole row of the
// plane), so that a workgroup's tiles stay small enough for several workgroups to share a
// compute unit's LDS; with SEGS segments a row, the SEGS waves that share it.
constexpr int kChainWaves = 2;
__host__ __device__ constexpr int chain_waves(int segs) { return segs > 1 ? segs : kChainWaves; }

// the boundary columns of the segments' rebuilt rows: [2 buffers][segment][first | last column][row]
template <int D, int SEGS>
struct ChainXchg {
  static constexpr int kWords = SEGS > 1 ? 2 * SEGS * 2 * ((1 << D) + 2) : 1;
};

// LDS of a workgroup: its waves' [lane][slot] tiles
template <int D>
struct ChainTiles {
  static constexpr int kWords = ChainGeo<D>::STRIDE * kWave;
};

// ---- first pass: channel norms of HWT(K_dw t1) ------------------------------------------------------
// grid = (ceil(units/waves), G, B), block = waves = chain_waves(SEGS) waves.  yc1 [B, C, k1], jmap1 [B, N]: the producer layer's
// compressed output and rank map; wdw [C, 3, 3].  Writes the partial norms (and the partial
// maxima of |coefficient|, nullable) of channel group grp to norm_part / max_part [G, B, N].
template <int D, bool SQ, int SEGS>
__global__ __launch_bounds__(chain_waves(SEGS) * kWave, 4 / chain_waves(SEGS)) void chain_norm_kernel(const float *__restrict__ yc1,
                                                         const int32_t *__restrict__ jmap1,
                                                         int64_t k1, const float *__restrict__ wdw,
                                                         float *__restrict__ norm_part,
                                                         float *__restrict__ max_part, Geo g,
                                                         StripMap m, int C, int Cg, int B,
                                                         SelectPrep prep) {
  constexpr int NS = slot_count(D, V4), WAVES = chain_waves(SEGS);
  __shared__ __attribute__((aligned(16))) uint32_t tiles[WAVES][ChainTiles<D>::kWords];
  __shared__ float xchg[ChainXchg<D, SEGS>::kWords];
  const int wv = threadIdx.x >> 6;
  const int unit = blockIdx.x * WAVES + wv;  // (SEGS > 1: the workgroup's waves share a strip)
  const int grp = blockIdx.y, b = blockIdx.z;
  // one workgroup per sample clears the state of the selection that follows this kernel
  if (blockIdx.x == 0 && grp == 0) prep_sample(prep, b, threadIdx.x, WAVES * kWave);
  LanePos<D> p;
  int row0, col0;
  const bool active = locate<D, V4>(m, g, unit, p, row0, col0);
  const int c0 = grp * Cg, n_ch = min(C, c0 + Cg) - c0;
  // whole waves leave (SEGS > 1: the waves of a workgroup share their strip, and every segment
  // has lanes inside the plane, so they leave or stay together)
  if (__ballot(active) == 0) return;

  const int32_t *jm1 = jmap1 + (size_t)b * g.N;
  const bool up_in = row0 > 0, dn_in = row0 + (1 << D) < g.H;
  const ChainGeo<D> cg = chain_setup<D>(jm1, k1, p, active, up_in, dn_in, tiles[wv]);

  ChainNormSink<D, SQ> sink;
#pragma unroll
  for (int s = 0; s < NS; ++s) sink.acc[s] = sink.top[s] = 0.f;
  // (the last groups have no channels where C does not fill them -- 42 channels in 8 groups of 6 --; their
  // planes are zeros: the selection adds the planes of all groups)
  if (n_ch > 0)
    chain_walk<D, SEGS>(yc1 + ((size_t)b * C + c0) * k1, k1, n_ch, wdw + (size_t)c0 * 9, cg, tiles[wv], p,
                        p.lc == 0, p.lc == m.lpr - 1 || col0 + V4 >= g.W, xchg, wv, sink,
                        [](ChainNormSink<D, SQ> &) {});
  sink.finish();
  if (!active) return;
  write_slots<D, V4>(norm_part + ((size_t)grp * B + b) * g.N, sink.acc, p);
  if (max_part != nullptr) write_slots<D, V4>(max_part + ((size_t)grp * B + b) * g.N, sink.top, p);
}

// ---- second pass: the kept coefficients of HWT(K_dw t1) ---------------------------------------------
// grid = (ceil(units/waves), G, B), block = waves = chain_waves(SEGS) waves.  jmap3: the consumer layer's rank map; xc
// [B, C, k3] fp32, or int8 codes with Q8 (clipping parameter: q_alpha > 0, or the largest of the
// n_alpha floats at alpha_src; the first workgroup leaves it at alpha_pub[0]).  Without Q8 the
// alpha slots (nullable) are raised to max |kept coefficient|.
template <int D, bool Q8, int SEGS>
__global__ __launch_bounds__(chain_waves(SEGS) * kWave, 4 / chain_waves(SEGS)) void chain_keep_kernel(const float *__restrict__ yc1,
                                                         const int32_t *__restrict__ jmap1,
                                                         int64_t k1, const float *__restrict__ wdw,
                                                         const int32_t *__restrict__ jmap3,
                                                         void *__restrict__ xc, int64_t k3,
                                                         float *alpha_slots, Geo g, StripMap m,
                                                         int C, int Cg, float q_alpha,
                                                         const float *__restrict__ alpha_src,
                                                         int n_alpha, float *alpha_pub) {
  constexpr int NS = slot_count(D, V4), WAVES = chain_waves(SEGS);
  __shared__ __attribute__((aligned(16))) uint32_t tiles[WAVES][ChainTiles<D>::kWords];
  __shared__ float xchg[ChainXchg<D, SEGS>::kWords];
  __shared__ float wmax[WAVES];
  const int wv = threadIdx.x >> 6;
  const int unit = blockIdx.x * WAVES + wv;
  const int grp = blockIdx.y, b = blockIdx.z;
  LanePos<D> p;
  int row0, col0;
  const bool active = locate<D, V4>(m, g, unit, p, row0, col0);
  const int c0 = grp * Cg, n_ch = max(min(C, c0 + Cg) - c0, 0);

  using Sink = KeepSink<D, V4, Q8>;
  using Out = typename Sink::Out;
  Sink sink(0.f);
  // the consumer's ranks of this lane's positions (or -1)
  const int32_t *jm3 = jmap3 + (size_t)b * g.N;
  auto fetch = [&](auto Lc, auto Jc) {
    constexpr int L = decltype(Lc)::value, J = decltype(Jc)::value;
    constexpr int CV = cols_at(V4, L), S2 = span_at(V4, L);
    const bool owner = (S2 == 1) || ((p.lc & (S2 - 1)) == 0);
#pragma unroll
    for (int i = 0; i < rows_at(D, L); ++i)
#pragma unroll
      for (int e = 0; e < CV; ++e) {
        int j = -1;
        if (active && owner) j = jm3[J * p.nl[L] + p.off[L] + i * p.rowlen[L] + e];
        sink.at[slot_base(D, V4, L, J) + i * CV + e] = (uint32_t)j;
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

  // The consumer's packed list of kept positions of this strip (rank, cell of the lane's own
  // slot), slot-major, then lane: built in the tile before the producer's list takes it over.
  constexpr int kRankBits = kInvRankBits;
  constexpr int STRIDE = ChainGeo<D>::STRIDE;
  uint32_t *tile = tiles[wv];
  const int lane = threadIdx.x & (kWave - 1);
  int count3 = 0;
#pragma unroll
  for (int s = 0; s < NS; ++s) count3 += __popcll(__ballot((int)sink.at[s] >= 0));
  const bool listed3 = count3 <= 16 * kWave && k3 <= ((int64_t)1 << kRankBits);
  uint32_t cell3[16], at3[16];  // this lane's share: entries lane + 64 i (unused rows fold away)
  if (listed3) {
    int running = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int j = (int)sink.at[s];
      const uint64_t kept = __ballot(j >= 0);
      const int to = running + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u));
      if (j >= 0) tile[to] = (uint32_t)j | ((uint32_t)(lane * STRIDE + s) << kRankBits);
      running += __popcll(kept);
    }
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int e = lane + kWave * i;
      const uint32_t packed = e < count3 ? tile[e] : 0u;
      cell3[i] = e < count3 ? packed >> kRankBits : (uint32_t)(lane * STRIDE);
      at3[i] = e < count3 ? (packed & ((1u << kRankBits) - 1u)) * (uint32_t)sizeof(Out) : Sink::kDropped;
    }
    wave_lds_fence();
  }

  const int32_t *jm1 = jmap1 + (size_t)b * g.N;
  const bool up_in = row0 > 0, dn_in = row0 + (1 << D) < g.H;
  const ChainGeo<D> cg = chain_setup<D>(jm1, k1, p, active, up_in, dn_in, tile);

  if constexpr (Q8) {
    if (alpha_src != nullptr) {  // (uniform over the grid; every thread of the workgroup is here)
      q_alpha = alpha_max(alpha_src, n_alpha);
      if (alpha_pub != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
        alpha_pub[0] = q_alpha;
    }
  }

  float mx = 0.f;  // the wave's largest |kept coefficient| (fp32 output only)
  if (__ballot(active) != 0 && n_ch > 0) {
    Out *plane3 = static_cast<Out *>(xc) + ((size_t)b * C + c0) * k3;
    const float *plane1 = yc1 + ((size_t)b * C + c0) * k1;
    const float *kw = wdw + (size_t)c0 * 9;
    const bool first_lane = p.lc == 0, last_lane = p.lc == m.lpr - 1 || col0 + V4 >= g.W;
    // Both lists short enough: dense stores of the consumer's list (NI3 rows), producer's list
    // walked with NI1 rows.  The two go together (both layers keep the same fraction; the producer's holds the rows
    // above and below as well, and is about twice as long), so four pairs cover the cases instead of every combination.
    // Kept at a quarter, 256 columns, three levels, lists of 8 and 17 rows are the rule, just above a power of two: with 12
    // and 24 rows between 8/16 and 16/32 the pass takes 455-473 us (8x1024 channels, before 476-481), and 4/12 instead of
    // 4/8 takes 3 % off blocks kept at an eighth (at two levels, where 4/8 holds the lists, it costs 1.6 %).  20 rows
    // in place of 16 or 24 were slower, 467-482 us.
    auto staged = [&](auto ni3_c, auto ni1_c) {
      constexpr int NI3 = decltype(ni3_c)::value, NI1 = decltype(ni1_c)::value;
      ChainStagedSink<D, Q8, NI3> st(Q8 ? q_alpha : 0.f);
      st.tile = tile;
      st.row = tile + lane * STRIDE;
#pragma unroll
      for (int i = 0; i < NI3; ++i) { st.cell[i] = cell3[i]; st.at[i] = at3[i]; }
      st.vmax = 0.f;
      st.aim(plane3, k3);
      chain_walk<D, SEGS, NI1>(plane1, k1, n_ch, kw, cg, tile, p, first_lane,
                         last_lane, xchg, wv, st, [&plane3, k3](auto &sk) {
                           sk.flush();
                           plane3 += k3;
                           sk.aim(plane3, k3);
                         });
      mx = st.vmax;
    };
    constexpr int kShort = D == 3 ? 12 : 8;
    const int ni3 = (count3 + kWave - 1) >> 6, ni1 = (cg.count + kWave - 1) >> 6;
    if (listed3 && cg.packed && cg.count > 0 && ni3 <= 4 && ni1 <= kShort) {
      staged(std::integral_constant<int, 4>{}, std::integral_constant<int, kShort>{});
    } else if (listed3 && cg.packed && cg.count > 0 && ni3 <= 8 && ni1 <= 16) {
      staged(std::integral_constant<int, 8>{}, std::integral_constant<int, 16>{});
    } else if (listed3 && cg.packed && cg.count > 0 && ni3 <= 12 && ni1 <= 24) {
      staged(std::integral_constant<int, 12>{}, std::integral_constant<int, 24>{});
    } else if (listed3 && cg.packed && cg.count > 0 && ni3 <= 16 && ni1 <= 32) {
      staged(std::integral_constant<int, 16>{}, std::integral_constant<int, 32>{});
    } else {
      // one store per slot (lanes that keep nothing there aim beyond the vector)
      if constexpr (Q8) sink.quant = Quant(q_alpha);
#pragma unroll
      for (int s = 0; s < NS; ++s)
        sink.at[s] = (int)sink.at[s] >= 0 ? sink.at[s] * (uint32_t)sizeof(Out) : Sink::kDropped;
      sink.vmax = 0.f;
      sink.aim(plane3, k3);
      // (a second sink with the quantiser's division path fixed at compile time, as in
      // haar_keep.hip, was measured here and lost: 761 vs 571 us on 96-wide planes -- this kernel
      // is short of registers as it is)
      chain_walk<D, SEGS>(plane1, k1, n_ch, kw, cg, tile, p, first_lane, last_lane, xchg, wv,
                    sink, [&plane3, k3](Sink &sk) {
                      plane3 += k3;
                      sk.aim(plane3, k3);
                    });
      mx = sink.vmax;
    }
  }
  if constexpr (Q8) return;
  if (alpha_slots == nullptr) return;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  if ((threadIdx.x & 63) == 0) wmax[wv] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    mx = wmax[0];
#pragma unroll
    for (int i = 1; i < WAVES; ++i) mx = fmaxf(mx, wmax[i]);
    unsigned int *a = reinterpret_cast<unsigned int *>(alpha_slots) +
                      ((blockIdx.x + 3u * blockIdx.y + 11u * blockIdx.z) & (kAlphaSlots - 1));
    const unsigned int mine = __float_as_uint(mx);
    if (mine > __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(a, mine);
  }
}

}  // namespace

// How the chained passes tile a plane: as the other strip kernels do where a wave row holds a
// whole row of the plane; else full wave rows side by side (one strip a wave, ceil(W/256) segments).
static StripMap chain_map(const wcc_desc &d) {
  StripMap m = make_map(d, V4);
  if (dw_needs_edges(m)) {
    m.lpr = kWave;
    m.log_lpr = 6;
    m.col_segs = (m.lanes_w + kWave - 1) / kWave;
    m.units = m.strips * m.col_segs;
  }
  return m;
}

// Segments of a row (waves that share it): 1 if a wave row holds the whole row, else 2 or 4;
// 0: a shape the chained passes do not take.
static int chain_segments(const wcc_desc &d) {
  if (d.W % 4 != 0 || d.levels > 3) return 0;
  const StripMap m = chain_map(d);
  if (!dw_needs_edges(m)) return 1;
  return (m.col_segs == 2 || m.col_segs == 4) ? m.col_segs : 0;
}

// Can the project layer d take its input from a producer's compressed output (see the limits at
// the top of this file)?
bool chain_supported(const wcc_desc &d) { return chain_segments(d) != 0; }

hipError_t launch_chain_norm(const wcc_desc &d, const ChainSrc &src, const float *wdw,
                             float *norm_part, float *max_part, int G, const SelectPrep &prep,
                             hipStream_t s) {
  const Geo g{d.H, d.W, d.levels, (int64_t)d.H * d.W};
  const StripMap m = chain_map(d);
  const int Cg = (d.C_in + G - 1) / G;
  const int segs = chain_segments(d), waves = chain_waves(segs);
  if (segs == 0) return hipErrorInvalidValue;
  const dim3 grid((m.units + waves - 1) / waves, G, d.B), block(waves * kWave);
  const bool sq = d.norm == WCC_NORM_L2;
#define WCC_CHAIN_NORM_(D_, SQ_, S_)                                                                   \
  hipLaunchKernelGGL((chain_norm_kernel<D_, SQ_, S_>), grid, block, 0, s, src.yc, src.jmap, src.k, wdw, \
                     norm_part, max_part, g, m, d.C_in, Cg, d.B, prep)
#define WCC_CHAIN_NORM(D_)                                                \
  do {                                                                    \
    if (segs == 1) {                                                      \
      if (sq) WCC_CHAIN_NORM_(D_, true, 1); else WCC_CHAIN_NORM_(D_, false, 1); \
    } else if (segs == 2) {                                               \
      if (sq) WCC_CHAIN_NORM_(D_, true, 2); else WCC_CHAIN_NORM_(D_, false, 2); \
    } else {                                                              \
      if (sq) WCC_CHAIN_NORM_(D_, true, 4); else WCC_CHAIN_NORM_(D_, false, 4); \
    }                                                                     \
  } while (0)
  switch (d.levels) {
    case 1: WCC_CHAIN_NORM(1); break;
    case 2: WCC_CHAIN_NORM(2); break;
    case 3: WCC_CHAIN_NORM(3); break;
    default: return hipErrorInvalidValue;
  }
#undef WCC_CHAIN_NORM
#undef WCC_CHAIN_NORM_
  return hipGetLastError();
}

hipError_t launch_chain_keep(const wcc_desc &d, int64_t k, const ChainSrc &src, const float *wdw,
                             const int32_t *jmap, void *xc, float *alpha_slots, float q_alpha,
                             const float *alpha_src, int n_alpha, float *alpha_pub, hipStream_t s) {
  const Geo g{d.H, d.W, d.levels, (int64_t)d.H * d.W};
  const StripMap m = chain_map(d);
  const int G = groups_for(d, make_map(d, lane_cols(d)), d.C_in, 4096, 8);
  const int Cg = (d.C_in + G - 1) / G;
  const int segs = chain_segments(d), waves = chain_waves(segs);
  if (segs == 0) return hipErrorInvalidValue;
  const dim3 grid((m.units + waves - 1) / waves, G, d.B), block(waves * kWave);
  const bool q8 = q_alpha > 0.f || alpha_src != nullptr;
#define WCC_CHAIN_KEEP_(D_, S_)                                                                     \
  do {                                                                                              \
    if (q8)                                                                                         \
      hipLaunchKernelGGL((chain_keep_kernel<D_, true, S_>), grid, block, 0, s, src.yc, src.jmap,    \
                         src.k, wdw, jmap, xc, k, nullptr, g, m, d.C_in, Cg, q_alpha, alpha_src,    \
                         n_alpha, alpha_pub);                                                       \
    else                                                                                            \
      hipLaunchKernelGGL((chain_keep_kernel<D_, false, S_>), grid, block, 0, s, src.yc, src.jmap,   \
                         src.k, wdw, jmap, xc, k, alpha_slots, g, m, d.C_in, Cg, 0.f, nullptr, 0,   \
                         nullptr);                                                                  \
  } while (0)
#define WCC_CHAIN_KEEP(D_)                     \
  do {                                         \
    if (segs == 1) WCC_CHAIN_KEEP_(D_, 1);     \
    else if (segs == 2) WCC_CHAIN_KEEP_(D_, 2); \
    else WCC_CHAIN_KEEP_(D_, 4);               \
  } while (0)
  switch (d.levels) {
    case 1: WCC_CHAIN_KEEP(1); break;
    case 2: WCC_CHAIN_KEEP(2); break;
    case 3: WCC_CHAIN_KEEP(3); break;
    default: return hipErrorInvalidValue;
  }
#undef WCC_CHAIN_KEEP
#undef WCC_CHAIN_KEEP_
  return hipGetLastError();
}

}  // namespace wcc
