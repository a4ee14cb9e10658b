// The last kernel of a fused layer of few channels and a long kept signal: the 1x1 convolution on the compressed
// signal (Eq. WCC), zero filling and the inverse transform (the last two steps of Alg. 1) in one pass, so that Y_wt
// never is in memory.
//
// A workgroup takes one unit of the plane, 16 lanes of the strip transform (64 columns of a strip of 8 rows), and
// all output channels.  The unit's kept positions are the columns of a small contraction,
//   Y[16 channels x P] = W[16 x K] . X[K x P]
// on 16 x 16 matrix instructions: X staged in LDS once in their order, W block by block.  What comes out fits the
// inverse: register r of a lane's result is channel 4 * (lane / 16) + r at kept position lane % 16 of a column
// block.  The four waves share the column blocks; register r of all of them goes to tile r, from which wave r
// rebuilds four channels, one in each quarter.  No load waits behind a store: the weights of the block after
// next are asked for ahead of this block's stores.
#include "strip_io.h"

namespace wcc {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int intx4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

enum { kOpBf16, kOpI8, kOpF32, kOpI4 };

// three levels, four columns a lane
struct Tail {
  static constexpr int D = 3, V = 4, R = 1 << D;
  static constexpr int NS = slot_count(D, V);
  static constexpr int kOwn = slot_base(D, V, 3, 0);  // slots of levels 1 and 2; those of level 3 are two lanes' together
  static constexpr int PX = kUnitLanes * V << D;      // positions of a unit
  static constexpr int MOST = PX / 16;                // column blocks, all positions kept
  // words between two lanes' slots; the last one is no slot: what has no position is dropped there
  static constexpr int STRIDE = tile_stride((NS + 4) / 4 * 4);
  static constexpr int kTile = STRIDE * kWave;        // words
  static constexpr int kRowW = 128 + 16;              // bytes of a weight row in LDS: 128, and rows on different banks
  // X beside four tiles and W, in KiB (a step of a column block), where two workgroups share a compute unit
  static constexpr int kBlocks = (80 * 1024 - 512 - 16 * kTile - 2 * PX - 16 * kRowW) / 1024;
};
static_assert(Tail::NS < Tail::STRIDE && Tail::kBlocks >= Tail::MOST, "a word that is no slot; a step of every position");

// Two codes (bytes sh / 8 and sh / 8 + 1 of a word) as bf16: an integer |v| <= 127 is exact there, its pattern is
// the float's high half.
__device__ __forceinline__ uint32_t widen2(uint32_t v, int sh) {
  const float lo = (float)((int)(v << (24 - sh)) >> 24), hi = (float)((int)(v << (16 - sh)) >> 24);
  return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

// place of slot s (level, band, row, column of the lane's tile) in the wavelet vector, for all slots; own: whether
// lane l16 of the unit is the one that counts the slot's value
template <class F>
__device__ __forceinline__ void each_slot(F &&f) {
  constexpr int D = Tail::D, V = Tail::V;
  auto band = [&](auto Lc, auto Jc) {
    constexpr int L = decltype(Lc)::value, J = decltype(Jc)::value, CV = cols_at(V, L);
#pragma unroll
    for (int i = 0; i < rows_at(D, L); ++i)
#pragma unroll
      for (int e = 0; e < CV; ++e) f(Lc, Jc, slot_base(D, V, L, J) + i * CV + e, i, e);
  };
  auto level = [&](auto Lc) {
    band(Lc, std::integral_constant<int, 1>{});
    band(Lc, std::integral_constant<int, 2>{});
    band(Lc, std::integral_constant<int, 3>{});
    if constexpr (decltype(Lc)::value == D) band(Lc, std::integral_constant<int, 0>{});
  };
  level(std::integral_constant<int, 1>{});
  level(std::integral_constant<int, 2>{});
  level(std::integral_constant<int, 3>{});
}

// lane l16 of a unit in the plane
__device__ __forceinline__ LanePos<Tail::D> unit_lane(const Geo &g, const UnitMap &um, int unit, int l16, int &row0, int &col0) {
  LanePos<Tail::D> p;
  const int at = unit * kUnitLanes + l16, strip = at / um.lanes_w, cl = at - strip * um.lanes_w;
  row0 = strip << Tail::D;
  col0 = cl * Tail::V;
  p.lc = l16;
#pragma unroll
  for (int l = 1; l <= Tail::D; ++l) {
    p.rowlen[l] = g.W >> l;
    p.nl[l] = (g.H >> l) * (g.W >> l);
    p.off[l] = (row0 >> l) * p.rowlen[l] + (col0 >> l);
  }
  p.active = at < um.lanes;
  return p;
}

// w: rows of at most 128 bytes as the matrix instructions take them (tail_takes).  xw: words [B, ceil(K / 4), ks] of
// codes, or [B, K, ks] fp32 (words_f32), quantised on their way to LDS if alpha is given.
// grid = (units rounded up to 8, 1, B), block = 256.
//
// Bound by its stores: 4 x 64 -> 256 channels of 512 x 1024, an eighth kept, 2.15 GB in 378-395 us = 5.6 TB/s, the
// rate of that store shape (nothing but the same stores: 375 us), where contraction and inverse take 51 and 431 us.
// What a workgroup does before its first store takes 6-8 us, most of it the way to memory and back twice (counts and
// rank map; X), so everything that does not depend on something else goes out together.
template <int OP, class YT>
__global__ __launch_bounds__(256, 2) void layer_tail_kernel(
    const void *__restrict__ w, const float *__restrict__ w_scale, const uint32_t *__restrict__ xw, bool words_f32,
    const float *__restrict__ alpha, int n_alpha, float *alpha_out, const int32_t *__restrict__ jmap,
    const uint32_t *__restrict__ ucount, int upad, YT *__restrict__ y, Geo g, UnitMap um, int M, int K, int64_t ks) {
  using S = Tail;
  using std::integral_constant;
  constexpr int D = S::D, V = S::V, NS = S::NS, NB = S::MOST / 4, NQ = (NS + 3) / 4;
  constexpr bool I8 = OP == kOpI8 || OP == kOpI4, F32 = OP == kOpF32, BF = OP == kOpBf16;
  // LDS holds X in steps of 16 bytes a lane: 64 channels of codes, or 16 of fp32.  Quads of channels a step, and
  // 16-byte fragments of weights a lane and step:
  constexpr int QPS = F32 ? 4 : 16, FPS = BF ? 2 : 1;
  __shared__ __attribute__((aligned(16))) unsigned char bs[S::kBlocks * 1024];  // X
  __shared__ __attribute__((aligned(16))) unsigned char as[16 * S::kRowW];      // W
  __shared__ __attribute__((aligned(16))) float tiles[4][S::kTile];
  __shared__ uint16_t list[S::PX];
  const int t = threadIdx.x, lane = t & 63, q = lane >> 4, l16 = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);  // (a scalar, and with it the planes' descriptors)
  // consecutive units on one die: the lines at their ends are written in one L2
  const int unit = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  const int b = blockIdx.z;
  if (unit >= um.units) return;
  float *tile = tiles[wv];
  int row0, col0;
  const LanePos<D> p = unit_lane(g, um, unit, l16, row0, col0);  // (the wave's quarters stand on the same lanes)

  // kept positions in front of the unit's, and its own
  uint32_t before = 0;
  const uint32_t *uc = ucount + (size_t)b * upad;
  for (int i0 = 0; 4 * i0 < unit; i0 += 4 * kWave) {
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = reinterpret_cast<const uint4 *>(uc)[min(i0 + u * kWave + lane, upad / 4 - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int left = unit - 4 * (i0 + u * kWave + lane);
      before += (left > 0 ? v[u].x : 0u) + (left > 1 ? v[u].y : 0u) + (left > 2 ? v[u].z : 0u) + (left > 3 ? v[u].w : 0u);
    }
  }
  const uint32_t mine = uc[unit];
  // the unit's rank map: wave 0, four slots a load
  int32_t j[NQ];
  if (wv == 0) {
    const int32_t *jm = jmap + (size_t)b * g.N;
    int at[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) at[i] = -1;
    each_slot([&](auto Lc, auto Jc, int s, int i, int e) {
      constexpr int L = decltype(Lc)::value, J = decltype(Jc)::value;
      const bool own = p.active && (l16 & (span_at(V, L) - 1)) == 0;
      at[s / 4] = q == (s & 3) && own ? J * p.nl[L] + p.off[L] + i * p.rowlen[L] + e : at[s / 4];
    });
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      j[i] = jm[max(at[i], 0)];
      if (at[i] < 0) j[i] = -1;
    }
  }

  // W of a block, 16 rows in LDS: 16 bytes a thread (of 128 threads at most), which travel through registers
  const int MB = (M + 15) >> 4, KS = (K + QPS * 4 - 1) / (QPS * 4);  // blocks of channels; steps: 1, or 2 (not bf16)
  const uint32_t row_bytes = BF ? 2u * K : F32 ? 4u * K : OP == kOpI4 ? (uint32_t)K / 2 : (uint32_t)K;
  const __amdgpu_buffer_rsrc_t wdesc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void *>(w), 0, (int)((uint32_t)M * row_bytes), 0x00020000);
  const __amdgpu_buffer_rsrc_t sdesc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(w_scale), 0, I8 ? (int)(uint32_t)(M * 4) : 0, 0x00020000);
  const int pieces_row = KS * FPS * 4, w_row = t / pieces_row, w_pc = t - w_row * pieces_row;
  const uint32_t from_w = (uint32_t)w_row * row_bytes + w_pc * (OP == kOpI4 ? 8u : 16u);
  const int own_w = t < 16 * pieces_row ? ((BF ? 2 * K : F32 ? 4 * K : K) - w_pc * 16) / 4 : -1;  // words that the row has
  const bool ragged = K % (F32 ? 16 : 64) != 0;
  struct Weights { std::conditional_t<OP == kOpI4, u32x2, u32x4> a; u32x4 sc; };
  Weights next;
  auto load_weights = [&](int blk) {  // (rows past the last: zeros)
    const uint32_t at = own_w > 0 && blk < MB ? (uint32_t)(blk * 16) * row_bytes + from_w : kRowDropped;
    if constexpr (OP == kOpI4) next.a = __builtin_amdgcn_raw_buffer_load_b64(wdesc, at, 0, 0);
    else next.a = __builtin_amdgcn_raw_buffer_load_b128(wdesc, at, 0, 0);
    if constexpr (I8) next.sc = __builtin_amdgcn_raw_buffer_load_b128(sdesc, (uint32_t)(blk * 16 + q * 4) * 4u, 0, 0);
  };
  auto put_weights = [&]() {
    u32x4 f;
    if constexpr (OP == kOpI4) {
      auto widen = [](uint32_t hw) {  // four codes in 16 bits -> four bytes
        uint32_t r4 = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) r4 |= ((uint32_t)((int)(hw << (28 - 4 * k)) >> 28) & 0xFFu) << (8 * k);
        return r4;
      };
      f = u32x4{widen(next.a.x & 0xFFFFu), widen(next.a.x >> 16), widen(next.a.y & 0xFFFFu), widen(next.a.y >> 16)};
    } else {
      f = next.a;
    }
    if (ragged) {  // (uniform) what the last load brings in of the next row
      f.x = own_w > 0 ? f.x : 0u;
      f.y = own_w > 1 ? f.y : 0u;
      f.z = own_w > 2 ? f.z : 0u;
      f.w = own_w > 3 ? f.w : 0u;
    }
    if (t < 16 * pieces_row) *reinterpret_cast<u32x4 *>(as + w_row * S::kRowW + w_pc * 16) = f;
  };
  load_weights(0);

  const bool quant = alpha != nullptr;  // (uniform over the grid, like n_alpha)
  float al = 0.f;
  if (quant) {
    al = n_alpha == 1 ? alpha[0] : alpha_max(alpha, n_alpha);
    if (alpha_out && blockIdx.x == 0 && blockIdx.z == 0 && t == 0) alpha_out[0] = al;
  }
#pragma unroll
  for (int i = 0; i < S::kTile / 256; ++i) reinterpret_cast<float4 *>(tile)[i * kWave + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off, kWave);
  before = (uint32_t)__builtin_amdgcn_readfirstlane((int)before);
  const int P = __builtin_amdgcn_readfirstlane((int)mine), nbu = (P + 15) >> 4;  // positions, column blocks
  const Quant qz(al);
  const float sx = quant ? qz.alpha / 127.f : 1.f;

  // X, steps [step0, step0 + steps) of it, to LDS: [step][column block][lane][16 bytes].  A wave takes 64, 32 or 16
  // positions (as many as the list has) of as many quads of channels as that leaves.
  const int c4_end = (K + 3) / 4;
  const __amdgpu_buffer_rsrc_t xdesc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t *>(xw) + (size_t)b * (words_f32 ? (size_t)K : (size_t)c4_end) * ks, 0,
      (int)((uint32_t)(words_f32 ? K : c4_end) * (uint32_t)ks * 4u), 0x00020000);
  const uint32_t ks4 = (uint32_t)ks * 4u;
  const int lg = P > 32 ? 6 : P > 16 ? 5 : 4, per = kWave >> lg, sub = lane >> lg;  // positions (log), quads a wave
  // Codes that meet bf16 weights are widened here where the LDS has room for that, else as they are used.
  const bool resident = KS * nbu <= S::kBlocks, wide = BF && 2 * KS * nbu <= S::kBlocks;
  auto stage_as = [&](int step0, int steps, auto form_c, auto deep_c) {
    constexpr int FORM = decltype(form_c)::value;  // words: 0 codes, 1 fp32, 2, 3 fp32 to be quantised (fast, exact)
    constexpr int U = (FORM == 0 ? 4 : 1) * (decltype(deep_c)::value ? 2 : 1);  // quads in flight
    const int first = step0 * QPS, quads = steps * QPS;
    for (int e0 = 0; e0 < P; e0 += kWave) {
      const int e = e0 + (lane & ((1 << lg) - 1));
      const uint32_t from = (before + (uint32_t)min(e, P - 1)) * 4u;
      unsigned char *dst = bs + ((e >> 4) * 64 + (e & 15)) * 16;
      for (int r0 = wv * per; r0 < quads; r0 += U * 4 * per) {
        uint32_t word[U][FORM == 0 ? 1 : 4];
#pragma unroll
        for (int u = 0; u < U; ++u) {  // (beyond the last channel: zeros)
          const int c4 = first + r0 + u * 4 * per + sub;
          if constexpr (FORM == 0) {
            word[u][0] = __builtin_amdgcn_raw_buffer_load_b32(xdesc, c4 < c4_end ? from + (uint32_t)c4 * ks4 : kRowDropped, 0, 0);
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              word[u][i] = __builtin_amdgcn_raw_buffer_load_b32(
                  xdesc, 4 * c4 + i < K ? from + (uint32_t)(4 * c4 + i) * ks4 : kRowDropped, 0, 0);
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int qd = r0 + u * 4 * per + sub;  // quad of the stage
          if (qd < quads && e < nbu * 16) {
            float f[4];
            if constexpr (FORM != 0 || F32) {
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                if constexpr (FORM == 0) f[i] = (float)((int)(word[u][0] << (24 - 8 * i)) >> 24);
                else f[i] = __uint_as_float(word[u][i]);
                if constexpr (FORM > 1) f[i] = qz.level_as<FORM == 2>(f[i]);
              }
            }
            if constexpr (F32) {
              *reinterpret_cast<float4 *>(dst + ((qd >> 2) * nbu * 64 + (qd & 3) * 16) * 16) = make_float4(f[0], f[1], f[2], f[3]);
            } else {
              uint32_t v = word[u][0];
              if constexpr (FORM != 0)
                v = ((uint32_t)(int)f[0] & 0xFFu) | ((uint32_t)(int)f[1] & 0xFFu) << 8 | ((uint32_t)(int)f[2] & 0xFFu) << 16 |
                    (uint32_t)(int)f[3] << 24;
              if (BF && wide)  // [step][channels 16 q + 0..7, 8..15][column block][lane]
                *reinterpret_cast<uint2 *>(dst + (((qd >> 4) * 2 + ((qd >> 1) & 1)) * nbu * 64 + ((qd & 15) >> 2) * 16) * 16 +
                                           (qd & 1) * 8) = make_uint2(widen2(v, 0), widen2(v, 16));
              else
                *reinterpret_cast<uint32_t *>(dst + ((qd >> 4) * nbu * 64 + ((qd & 15) >> 2) * 16) * 16 + (qd & 3) * 4) = v;
            }
          }
        }
      }
    }
  };
  auto stage = [&](int step0, int steps, auto deep_c) {  // (the choices are the same for the whole grid)
    if (!words_f32) stage_as(step0, steps, integral_constant<int, 0>{}, deep_c);
    else if (F32 && !quant) stage_as(step0, steps, integral_constant<int, 1>{}, deep_c);
    else if (qz.fast) stage_as(step0, steps, integral_constant<int, 2>{}, deep_c);
    else stage_as(step0, steps, integral_constant<int, 3>{}, deep_c);
  };
  if (resident && nbu > 0) stage(0, KS, std::true_type{});

  // the list of kept positions, slot by slot and lane by lane: words of a tile
  if (wv == 0) {
    int running = 0;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const uint64_t kept = __ballot(j[i] >= 0);
      const int to = running + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u));
      if (j[i] >= 0) list[to] = (uint16_t)(l16 * S::STRIDE + 4 * i + q);
      running += __popcll(kept);
    }
    const int e = P + lane;  // up to a whole group of four blocks: a word that is no slot
    if (e < (P + 63) / 64 * 64) list[e] = (uint16_t)(l16 * S::STRIDE + S::STRIDE - 1);
  }
  u32x4 sc4 = next.sc;
  put_weights();
  workgroup_lds_barrier();
  load_weights(1);

  // The wave's column blocks are every fourth one; where a quarter drops its position of each (byte of a tile).
  const int nbw = (nbu - wv + 3) >> 2;
  uint32_t cell[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) cell[i] = (list[(4 * i + wv) * 16 + l16] + q * 16 * S::STRIDE) * 4u;

  const uint32_t plane_bytes = (uint32_t)g.N * (uint32_t)sizeof(YT);
  const uint32_t lane_off =
      p.active ? (uint32_t)(((int64_t)(4 * q) * g.N + (int64_t)row0 * g.W + col0) * (int64_t)sizeof(YT)) : kRowDropped;
  const uint32_t pitch = (uint32_t)(g.W * sizeof(YT));
  YT *yb = y + (size_t)b * M * g.N;
  using Acc = std::conditional_t<I8, intx4, floatx4>;
  Acc acc[NB];
  // runs f(0), f(1), ... for the wave's column blocks; one test behind the last
  auto each_block = [&](auto &&f) {
    auto from = [&](auto n_c, auto &&self) -> void {
      constexpr int N = decltype(n_c)::value;
      if constexpr (N < NB) {
        if (N < nbw) {  // (uniform)
          f(n_c);
          self(integral_constant<int, N + 1>{}, self);
        }
      }
    };
    from(integral_constant<int, 0>{}, from);
  };
  // NSX steps from s on (c0: the first one in LDS)
  auto multiply = [&](auto nsx_c, auto wide_c, int s, int c0) {
    constexpr int NSX = decltype(nsx_c)::value, XPS = decltype(wide_c)::value ? 2 : 1;
    u32x4 f[NSX][FPS];
#pragma unroll
    for (int i = 0; i < NSX; ++i)
#pragma unroll
      for (int h = 0; h < FPS; ++h)
        f[i][h] = *reinterpret_cast<const u32x4 *>(as + l16 * S::kRowW + ((s + i) * 4 + q) * FPS * 16 + h * 16);
    const unsigned char *xs = bs + (((s - c0) * XPS * nbu + wv) * 64 + lane) * 16;
    each_block([&](auto n_c) {
      constexpr int N = decltype(n_c)::value;
      uint4 x[NSX * XPS];
#pragma unroll
      for (int i = 0; i < NSX * XPS; ++i) x[i] = *reinterpret_cast<const uint4 *>(xs + i * nbu * 1024 + N * 4096);
#pragma unroll
      for (int i = 0; i < NSX; ++i) {
        if constexpr (BF) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            u32x4 e;
            if constexpr (XPS == 2) {
              e = __builtin_bit_cast(u32x4, x[2 * i + h]);
            } else {
              const uint32_t lo = h ? x[i].z : x[i].x, hi = h ? x[i].w : x[i].y;
              e = u32x4{widen2(lo, 0), widen2(lo, 16), widen2(hi, 0), widen2(hi, 16)};
            }
            acc[N] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[i][h]), __builtin_bit_cast(bf16x8, e),
                                                             acc[N], 0, 0, 0);
          }
        } else if constexpr (I8) {
          acc[N] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(intx4, f[i][0]), __builtin_bit_cast(intx4, x[i]),
                                                         acc[N], 0, 0, 0);
        } else {
          const uint32_t fa[4] = {f[i][0].x, f[i][0].y, f[i][0].z, f[i][0].w}, xa[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
#pragma unroll
          for (int k = 0; k < 4; ++k)
            acc[N] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(fa[k]), __uint_as_float(xa[k]), acc[N], 0, 0, 0);
        }
      }
    });
  };

  for (int blk = 0; blk < MB; ++blk) {
    each_block([&](auto n_c) { acc[decltype(n_c)::value] = Acc{0, 0, 0, 0}; });
    if (!resident) {  // two steps that the LDS holds one after the other
      for (int s = 0; s < KS; ++s) {
        workgroup_lds_barrier();  // (everyone has read what is replaced)
        stage(s, 1, std::false_type{});
        workgroup_lds_barrier();
        multiply(integral_constant<int, 1>{}, std::false_type{}, s, s);
      }
    } else if constexpr (BF) {
      if (wide) multiply(integral_constant<int, 1>{}, std::true_type{}, 0, 0);
      else multiply(integral_constant<int, 1>{}, std::false_type{}, 0, 0);
    } else {
      if (KS == 2) multiply(integral_constant<int, 2>{}, std::false_type{}, 0, 0);
      else multiply(integral_constant<int, 1>{}, std::false_type{}, 0, 0);
    }
    // register r of every wave's sums goes to tile r, of which wave r makes four channels
    workgroup_lds_barrier();  // (everyone has read the tiles of the last block and the weights of this one)
    each_block([&](auto n_c) {
      constexpr int N = decltype(n_c)::value;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<float *>(reinterpret_cast<char *>(tiles[r]) + cell[N]) =
            (float)acc[N][r] * (I8 ? sx * __uint_as_float(sc4[r]) : sx);
    });
    sc4 = next.sc;
    put_weights();
    workgroup_lds_barrier();
    load_weights(blk + 2);  // ahead of the stores: loads and stores retire in order
    float out[S::R][V];
    {
      float c[NS];
      const float *row = tile + lane * S::STRIDE, *both = tile + (lane & ~1) * S::STRIDE;
#pragma unroll
      for (int s = 0; s + 4 <= S::kOwn; s += 4) {
        const float4 v = *reinterpret_cast<const float4 *>(row + s);
        c[s] = v.x; c[s + 1] = v.y; c[s + 2] = v.z; c[s + 3] = v.w;
      }
#pragma unroll
      for (int s = S::kOwn / 4 * 4; s < S::kOwn; ++s) c[s] = row[s];
#pragma unroll
      for (int s = S::kOwn; s < NS; ++s) c[s] = both[s];
      const RegStrip<D, V, NS> src{c};
      inv_levels<D, V, 1>(out, p, src);
    }
    // Planes blk * 16 + wv and on; what lies past the last channel, and lanes outside the plane, is dropped.  (The
    // range check is against what a row's offset leaves of the size, which is at least a plane.)
    const int m0 = blk * 16 + wv;
    if (m0 < M) {  // (uniform over the wave)
      const __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc(
          yb + (int64_t)m0 * g.N, 0, (int)(plane_bytes * (uint32_t)min(16, M - m0)), 0x00020000);
#pragma unroll
      for (int i = 0; i < S::R; ++i) store_row_buf<V>(to, lane_off, out[i], YT{}, i * pitch);
    }
  }
}

// ucount[b][u] = kept positions of unit u (u < upad).  16 lanes a unit; grid = (upad / 16, B), block = 256.
__global__ __launch_bounds__(256) void unit_count_kernel(const int32_t *__restrict__ jmap, uint32_t *__restrict__ ucount,
                                                         int upad, Geo g, UnitMap um) {
  const int l16 = threadIdx.x & 15, unit = blockIdx.x * 16 + (threadIdx.x >> 4), b = blockIdx.y;
  int row0, col0;
  const LanePos<Tail::D> p = unit_lane(g, um, unit, l16, row0, col0);
  const int32_t *jm = jmap + (size_t)b * g.N;
  int32_t j[Tail::NS];  // (all loads in flight together)
  each_slot([&](auto Lc, auto Jc, int s, int i, int e) {
    constexpr int L = decltype(Lc)::value, J = decltype(Jc)::value;
    const bool own = p.active && (l16 & (span_at(Tail::V, L) - 1)) == 0;
    j[s] = jm[own ? J * p.nl[L] + p.off[L] + i * p.rowlen[L] + e : 0];
    if (!own) j[s] = -1;
  });
  uint32_t n = 0;
#pragma unroll
  for (int s = 0; s < Tail::NS; ++s) n += j[s] >= 0 ? 1u : 0u;
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) n += __shfl_xor(n, off, 16);
  if (l16 == 0) ucount[(size_t)b * upad + unit] = n;
}

template <int OP>
hipError_t tail_launch(const wcc_desc &d, const TailArgs &a, hipStream_t s) {
  const Geo g{d.H, d.W, d.levels, (int64_t)d.H * d.W};
  const UnitMap um = unit_map(d);
  const dim3 grid(((unsigned)um.units + 7) / 8 * 8, 1, d.B), block(256);
#define WCC_TAIL(YT)                                                                                                \
  hipLaunchKernelGGL((layer_tail_kernel<OP, YT>), grid, block, 0, s, a.w, a.w_scale, a.xw, a.words_f32, a.alpha,    \
                     a.n_alpha, a.alpha_out, a.jmap, a.ucount, a.upad, static_cast<YT *>(a.y), g, um, d.C_out,      \
                     d.C_in, a.ks)
  if (d.act_dtype == WCC_BF16) WCC_TAIL(bf16_t); else WCC_TAIL(float);
#undef WCC_TAIL
  return hipGetLastError();
}

}  // namespace

UnitMap unit_map(const wcc_desc &d) {
  UnitMap m;
  m.lanes_w = d.W / Tail::V;
  m.lanes = m.lanes_w * (d.H >> d.levels);
  m.units = (m.lanes + kUnitLanes - 1) / kUnitLanes;
  return m;
}

bool tail_takes(const wcc_desc &d, int64_t ks, size_t count_room) {
  const bool quant = d.act_quant_bits == 8;
  const int K = d.C_in;
  if (d.levels != Tail::D) return false;
  int row;  // bytes of a row of weights as the matrix instructions take it: whole words in memory, 128 at most
  switch (d.w_dtype) {
    case WCC_F32: row = 4 * K; break;
    case WCC_BF16: if (!quant || K % 2) return false; row = 2 * K; break;
    case WCC_I8: if (!quant || K % 4) return false; row = K; break;
    default: if (!quant || K % 8) return false; row = K; break;
  }
  if (row > 128) return false;
  const UnitMap um = unit_map(d);
  // Where it pays: a long Y_wt that need not be written and read (`mb`), workgroups for two rounds of the chip, since a
  // workgroup takes 6-8 us before its first store, and rows of whole 128-byte lines, since units write 256 bytes of a
  // row; where nearly everything is kept, which the inverse on its own takes value by value, any rows.  Layers without and
  // with it, us (X: left to them):
  //   4 x 64 -> 256 channels of 512 x 1024, 1/8 kept, 268 MB of Y_wt, 4096 units: 720 and 617;
  //   48 MB, 512 columns, 1024 units (4 x 16 -> 96): 96 and 94; 53 MB, 416, 1131: 117 and 107; 92 MB, 512, 976: 179 and 149;
  //   126 MB, 224, 1344: 137 and 103; 126 MB, 192, 1152: 190 and 138; all kept: 368 MB, 792, 693: 301 and 223; 759 MB, 280, 945:
  //   576 and 359;
  //   X shorter: 20 MB, 640, 2520: 132 and 143; 26 MB, 688, 1354: 157 and 164; X ragged lines: 186 MB, 744, 1488: 272 and 289;
  //   65 MB, 520, 1040: 155 and 188; 136 MB, 728, 2912: 322 and 360; 106 MB, 424, 1696: 271 and 307; X few units, whole lines:
  //   64 MB, 256, 128: 105 and 134 at 1/4, 83 and 117 at 1/2; 39 MB, 200 (ragged), 188: 58 and 85;
  //   X more channels: 16 x 256 -> 1024 of 128 x 128, half kept: 465 without, 1170 with (conversions of X for every
  //   block of channels); 144 fp32 channels of half kept 192 x 320 maps: 422 and 1400 (X staged again for every block).
  // The line of 900 units is on the safe side: with whole lines 512 to 768 of them measured 0.76..0.97 of the time (2 x 64 ->
  // 256 of 256 x 512, 1/4 kept 123 and 115), with x out of the cache 0.83..1.04.
  // 203 layers drawn from all that the rule takes, lines below included: 0.51..1.01 of the time, 0.78 in the mean; with x out
  // of the cache 0.49..1.03, 0.81.
  const int64_t mb = ((int64_t)d.B * d.C_out * ks * 4) >> 20, units = (int64_t)um.units * d.B;
  const bool whole_lines = (int64_t)d.W * (d.act_dtype == WCC_BF16 ? 2 : 4) % 128 == 0;
  const bool all_kept = ks * 10 >= (int64_t)d.H * d.W * 9;
  if (!(mb >= 48 && units >= 900 && whole_lines) && !(mb >= 256 && units >= 640 && all_kept)) return false;
  // A workgroup's start is paid once a unit, whatever C_out is, and a block of 16 channels costs the same whether all 16
  // are there.  Without and with the one kernel: 8 x 16 -> 4 of 512 x 2048, half kept 427 and 659; 4 x 64 -> 8 of
  // 512 x 1024, all kept 381 and 457; 64 -> 17, half kept 339 and 382; 64 -> 32 375 and 386; 1 x 6 -> 32 of 680 x 1344 112
  // and 128.  Three blocks pay where the unit's share of Y_wt is long enough: 5 x 32 -> 41 of 432 x 608, 1/4 kept 179 and
  // 182, but 13 x 8 -> 35 of 760 x 352, 1/3 kept (154 MB) 305 and 247.
  const int64_t N = (int64_t)d.H * d.W, k = kept_count(d);
  if (d.C_out <= 32 || (d.C_out < 48 && d.C_out * k < 16 * N && mb < 96)) return false;
  // Where the channels take two steps the LDS holds X of 320 of a unit's 512 positions (kBlocks); a unit that keeps more
  // stages X again for every block of channels.  More than half kept: 3 x 80 -> 160 of 376 x 640, the first 3/5 323 us without
  // and 879 with; 10 x 128 -> 224 of 600 x 128, 3/4 576 and 656; 4 x 20 fp32 -> 128 of 256 x 512, 3/4 176 and 215.  Between a
  // third and a half some units do where what is kept stands close together, against which codes need many blocks
  // (15 x 128 -> 66 of 312 x 256 432 and 476, but 8 x 128 -> 404 of 216 x 768 984 and 693); the fp32 contraction that they
  // would take otherwise costs more (5 x 30 -> 61 of 400 x 352 151 and 132).
  const bool two_steps = d.w_dtype != WCC_BF16 && row > 64;
  if (two_steps && (k * 2 > N || (k * 3 > N + 2 && d.w_dtype != WCC_F32 && d.C_out < 96))) return false;
  // Little kept: bf16 maps, whose rows are half as long to write, need a longer Y_wt or more of it a unit (5 x 12 -> 272 of
  // 232 x 768, 1/16 kept 146 without and 151 us with; 2 x 6 -> 89 of 712 x 960, the first sixth 92 and 112; but
  // 6 x 52 -> 144 of 136 x 960, 1/5 166 and 123), and the keep pass into words transforms whole quads of channels
  // (6 x 1 -> 170 of 304 x 480, 1/10 161 and 167; 2 x 6 -> 248 of 456 x 928 227 and 232), which
  // below a twelfth of few channels is not made good either (4 x 8 -> 112 of 624 x 736, 1/16 229 and 235; 14 x 16 -> 373 fp32
  // channels of 360 x 128 238 and 244; but 5 x 38 -> 240 of 344 x 736 312 and 299).
  if (d.act_dtype == WCC_BF16 && mb < 96 && (mb < 64 || d.C_out * k < 24 * N)) return false;
  if (k * 8 < N && K < (k * 12 < N ? 24 : 8)) return false;
  // byte offsets of 32 bits: sixteen planes of the output, the weights, a sample's compressed signal; and the
  // counts that every workgroup adds up
  const int64_t limit = (int64_t)0xFFFFFFF0 - 16;
  if (16 * N * 4 > limit || (int64_t)(d.C_out + 48) * row > limit || (int64_t)(K + 3) * ks * 4 > limit) return false;
  return um.units <= 8192 && (size_t)d.B * unit_pad(um) * 4 <= count_room;
}

hipError_t launch_unit_count(const wcc_desc &d, const int32_t *jmap, uint32_t *ucount, hipStream_t s) {
  const Geo g{d.H, d.W, d.levels, (int64_t)d.H * d.W};
  const UnitMap um = unit_map(d);
  hipLaunchKernelGGL(unit_count_kernel, dim3(unit_pad(um) / 16, d.B), dim3(256), 0, s, jmap, ucount, unit_pad(um), g, um);
  return hipGetLastError();
}

hipError_t launch_layer_tail(const wcc_desc &d, const TailArgs &a, hipStream_t s) {
  switch (d.w_dtype) {
    case WCC_BF16: return tail_launch<kOpBf16>(d, a, s);
    case WCC_F32: return tail_launch<kOpF32>(d, a, s);
    case WCC_I8: return tail_launch<kOpI8>(d, a, s);
    default: return tail_launch<kOpI4>(d, a, s);
  }
}

}  // namespace wcc
