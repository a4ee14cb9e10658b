// The 1x1 convolution on the compressed signal (Eq. WCC: K_1x1 applied between T and T^T;
// output channel i is sum_j k_ij x_j over the length-k compressed channel vectors x_j): per sample a
// [C_out x C_in] . [C_in x k] contraction, k contiguous in memory on both sides.
//
// Matrix-core kernel (int8 activation codes):
//   bf16 weights: v_mfma_f32_32x32x16_bf16.  The codes (|n| <= 127) are exact in bf16 and
//                 every product is exact in fp32; only the fp32 accumulation rounds.
//   int8 weights: v_mfma_i32_32x32x32_i8, exact int32 accumulation.
// At the layer's shapes the contraction is bound by HBM (a few tens of flop per byte), so the
// kernel is built around the activation stream: a workgroup owns BM = 128 or 256 output rows
// (all of C_out when it fits, so every activation is read and quantised once) and BN = 128
// positions; each thread loads its share of a 64-channel chunk of the [C_in x BN] activation
// tile (several chunks going out together was measured at every shape and never paid: it costs
// registers, and with them the second workgroup on the compute unit),
// quantises it in registers, transposes 4(n) x CPT(c) patches into LDS, and the waves (wave w
// owns rows 32w..32w+31 and all BN columns) run the MFMAs 64 channels at a time.  As soon as
// a chunk's registers are in LDS the next chunk's loads (activations and weights) are issued,
// so they travel while the MFMAs of this chunk run.  The n rows are stored permuted
// (row (n%NB)*32 + n/NB, NB = BN/32) so that MFMA column c of column block i is n = NB*c + i:
// after the NB column blocks a lane holds NB adjacent n of one output row and stores them as
// one 16- or 8-byte word.  Layers whose kept signal is short would leave most of the chip
// idle with such tiles and turn the kernel into a chain of memory latencies; they take
// smaller tiles (down to 64 x 64), re-reading the activations once per row tile from L2.
// Everything else (fp32 weights, unquantised activations, rows that no word load can read) runs on
// the fp32 matrix instructions, with both operands widened to fp32.
#include <type_traits>

#include "wcc_internal.h"

namespace wcc {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int intx4;
typedef __attribute__((__vector_size__(16 * sizeof(int)))) int intx16;

constexpr int BK = 64;

// The layer's alpha: the largest of n partial maxima (n = 1: alpha itself).  The first workgroup
// also publishes it to alpha_out (nullable).  Called by every thread of the workgroup.
__device__ __forceinline__ float load_alpha(const float *__restrict__ alpha, int n, float *alpha_out) {
  const float a = alpha_max(alpha, n);
  if (alpha_out && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
    alpha_out[0] = a;
  return a;
}

// In which form the compressed signal comes: int8 codes [K, k], fp32 [K, k] (quantised on load), or codes of four
// channels a word, [ceil(K / 4), k], as the second transform pass of the fused layer writes them: a patch is then a quarter
// of the loads, four times as wide, and transposed as the matrix instructions want it.
enum { kCodes = 0, kFloats = 1, kWords = 2 };
typedef uint32_t word4 __attribute__((ext_vector_type(4)));

// A thread's raw CPT (channels) x 4 (positions) patch of one 64-channel chunk.
template <int FORM, int CPT>
struct Patch {
  static constexpr bool F32 = FORM == kFloats, WORDS = FORM == kWords;
  float4 f[F32 ? CPT : 1];
  uint32_t c[FORM == kCodes ? CPT : 1];
  word4 q[WORDS ? CPT / 4 : 1];
  // Loaded through a buffer descriptor of the sample's compressed signal: off is the byte
  // offset of this thread's four positions in the patch's first channel.  No branch, no lane
  // mask: a load never faults (outside the buffer it returns zeros, a wrapped offset lands
  // inside it); what it returns for channels >= C_in meets zero weights (any finite value will
  // do: fp32 coefficients are clipped by the quantiser, and a NaN quantises to a finite level),
  // and for positions >= k it feeds columns that are never stored.
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t xdesc, uint32_t off, int64_t k) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    if constexpr (WORDS) {
#pragma unroll
      for (int r = 0; r < CPT / 4; ++r)
        q[r] = __builtin_amdgcn_raw_buffer_load_b128(xdesc, off + (uint32_t)r * (uint32_t)k * 4u, 0, 0);
      return;
    }
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
      if constexpr (F32) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(xdesc, off + (uint32_t)r * (uint32_t)k * 4u, 0, 0);
        f[r] = make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
      } else if constexpr (!WORDS) {
        c[r] = __builtin_amdgcn_raw_buffer_load_b32(xdesc, off + (uint32_t)r * (uint32_t)k, 0, 0);
      }
    }
  }
  // level of channel r, position i, as a float holding an integer in [-127, 127]
  template <bool FAST>
  __device__ __forceinline__ float level(int r, int i, const Quant &quant) const {
    if constexpr (F32) {
      const float v = i == 0 ? f[r].x : i == 1 ? f[r].y : i == 2 ? f[r].z : f[r].w;
      return quant.template level_as<FAST>(v);
    } else if constexpr (WORDS) {
      return (float)((int)(q[r >> 2][i] << (24 - 8 * (r & 3))) >> 24);
    } else {
      return (float)((int)(c[r] << (24 - 8 * i)) >> 24);
    }
  }
};

// grid = (ceil(k/BN), ceil(M/BM), B), block = 2*BM threads.  Needs k % 4 == 0 and
// K % 2 == 0 (bf16 weights) or K % 4 == 0 (int8 weights).
// RAG: a weight row is not a whole number of 16-byte loads (K % 8 or K % 16 != 0): what the last load
// of a row brings in of the next one is cleared on its way to LDS.
template <int BM, int BN, int FORM, bool I8W, bool RAG>
__global__ __launch_bounds__(2 * BM) void pointwise_mfma_kernel(
    const void *__restrict__ w, const float *__restrict__ w_scale, const void *__restrict__ xq,
    const float *__restrict__ alpha, int n_alpha, float *alpha_out, float *__restrict__ yc, int M,
    int K, int64_t k, bool stream_out) {
  constexpr bool F32 = FORM == kFloats, WORDS = FORM == kWords;
  constexpr int T = 2 * BM;
  fetch_args(w, k);
  constexpr int NB = BN / 32;                // 32-column blocks of the tile: 4 or 2
  constexpr int NG = BN / 4;                 // groups of four positions
  constexpr int CPT = BK / (T / NG);         // channels of a chunk per thread: 4, 8 or 16
  constexpr int ESZ = I8W ? 1 : 2;           // bytes of an LDS element
  constexpr int LDR = I8W ? BK + 16 : (BK + 8) * 2;  // LDS row bytes: 80 / 144 (16-byte aligned,
                                                      // fragment reads free of bank conflicts)
  constexpr int APT = BK * ESZ / 2 / 16;     // 16-byte weight loads per thread and chunk: 2 / 4
  __shared__ __attribute__((aligned(16))) unsigned char As[BM * LDR];
  __shared__ __attribute__((aligned(16))) unsigned char Bs[BN * LDR];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int b = blockIdx.z;
  const int64_t n0 = (int64_t)blockIdx.x * BN;
  const int64_t xbytes = (WORDS ? (K + 3) / 4 * 4 : K) * k * (F32 ? 4 : 1);  // of a sample
  const void *xb = static_cast<const char *>(xq) + (size_t)b * xbytes;
  const unsigned char *wb = static_cast<const unsigned char *>(w);
  const int a_row = t >> 1, a_half = t & 1;  // weight loader: row, which half of the chunk
  const int g = t % NG, kq = t / NG;         // activation loader: n group (4 n), channel group
  const int nchunks = (K + BK - 1) / BK;

  const float al = load_alpha(alpha, n_alpha, alpha_out);
  const Quant quant(al);
  // Both operands are loaded through buffer descriptors (the host has checked that their byte
  // offsets fit 32 bits): weights of rows >= M lie beyond the end and come back
  // as zeros, those of channels >= C_in are sent there by a wave-uniform choice.
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  constexpr uint32_t kOutside = 0xFFFFFFF0u;
  const __amdgpu_buffer_rsrc_t wdesc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char *>(wb), 0, (int)(uint32_t)((int64_t)M * K * ESZ), 0x00020000);
  const __amdgpu_buffer_rsrc_t xdesc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void *>(xb), 0, (int)(uint32_t)xbytes, 0x00020000);
  // A workgroup takes the row tiles blockIdx.y, blockIdx.y + gridDim.y, ...: with one workgroup
  // per column tile (gridDim.y = 1) the stores of a row tile drain while the next one is being
  // computed, instead of holding the compute unit until they are out.
  for (int m0 = blockIdx.y * BM; m0 < M; m0 += gridDim.y * BM) {
  // accumulators of the NB column blocks: int32 for int8 weights, fp32 for bf16 weights
  using Acc = std::conditional_t<I8W, intx16, floatx16>;
  Acc acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0;

  // weights of chunk kc: wreg <- w[m0 + a_row][kc*64 + this thread's share], zero outside.
  // They are fetched one chunk ahead (while the MFMAs of the previous chunk run).
  uint4 wreg[APT];
  auto load_w = [&](int kc) {
#pragma unroll
    for (int q = 0; q < APT; ++q) {
      const int kk = kc * BK + (a_half * (BK / 2)) + q * (16 / ESZ);  // first element of the load
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(
          wdesc, kk < K ? (uint32_t)(m0 + a_row) * (uint32_t)(K * ESZ) + (uint32_t)kk * ESZ : kOutside, 0, 0);
      wreg[q] = make_uint4(v.x, v.y, v.z, v.w);
    }
  };

  Patch<FORM, CPT> raw;  // the one chunk of activations in flight
  // activations: quantise, transpose the CPT x 4 patch, store with the n rows permuted
  auto stage_patch = [&](const Patch<FORM, CPT> &pt, const Quant &quant, auto fast_c) {
    constexpr bool FAST = decltype(fast_c)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t pk[I8W ? (CPT / 4) : (CPT / 2)];
      if constexpr (I8W && WORDS) {
#pragma unroll
        for (int r = 0; r < CPT; r += 4) pk[r / 4] = pt.q[r / 4][i];
      } else if constexpr (I8W) {
#pragma unroll
        for (int r = 0; r < CPT; r += 4) {
          const uint32_t c0 = (uint32_t)(int)pt.template level<FAST>(r, i, quant) & 0xFFu;
          const uint32_t c1 = (uint32_t)(int)pt.template level<FAST>(r + 1, i, quant) & 0xFFu;
          const uint32_t c2 = (uint32_t)(int)pt.template level<FAST>(r + 2, i, quant) & 0xFFu;
          const uint32_t c3 = (uint32_t)(int)pt.template level<FAST>(r + 3, i, quant) & 0xFFu;
          pk[r / 4] = c0 | (c1 << 8) | (c2 << 16) | (c3 << 24);
        }
      } else {
#pragma unroll
        for (int r = 0; r < CPT; r += 2) {
          // an integer |v| <= 127 is exact in bf16: its bf16 pattern is the float's high half
          const uint32_t lo = __float_as_uint(pt.template level<FAST>(r, i, quant));
          const uint32_t hi = __float_as_uint(pt.template level<FAST>(r + 1, i, quant));
          pk[r / 2] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
        }
      }
      const int nl = 4 * g + i;  // position inside the tile
      unsigned char *dst = &Bs[((nl % NB) * 32 + nl / NB) * LDR + kq * CPT * ESZ];
      constexpr int words = I8W ? CPT / 4 : CPT / 2;
      if constexpr (words == 8) {
        *reinterpret_cast<uint4 *>(dst) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        *reinterpret_cast<uint4 *>(dst + 16) = make_uint4(pk[4], pk[5], pk[6], pk[7]);
      } else if constexpr (words == 4) *reinterpret_cast<uint4 *>(dst) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
      else if constexpr (words == 2) *reinterpret_cast<uint2 *>(dst) = make_uint2(pk[0], pk[1]);
      else *reinterpret_cast<uint32_t *>(dst) = pk[0];
    }
  };

  // this thread's four positions in channel kq * CPT of chunk 0
  constexpr uint32_t XB = F32 ? 4u : 1u;  // bytes of an activation
  const uint32_t xoff = (uint32_t)(kq * CPT) * (uint32_t)k * XB + (uint32_t)(n0 + 4 * g) * (WORDS ? 4u : XB);
  load_w(0);
  raw.load(xdesc, xoff, k);
  for (int kc = 0; kc < nchunks; ++kc) {
    {
      if (quant.fast) stage_patch(raw, quant, std::true_type{});
      else stage_patch(raw, quant, std::false_type{});
      if constexpr (RAG) {
        if (kc == nchunks - 1) {
#pragma unroll
          for (int q = 0; q < APT; ++q) {
            // dwords of this load that belong to the row (K * ESZ is a multiple of 4)
            const int own = (K - (kc * BK + (a_half * (BK / 2)) + q * (16 / ESZ))) * ESZ / 4;
            wreg[q].x = own > 0 ? wreg[q].x : 0u;
            wreg[q].y = own > 1 ? wreg[q].y : 0u;
            wreg[q].z = own > 2 ? wreg[q].z : 0u;
            wreg[q].w = own > 3 ? wreg[q].w : 0u;
          }
        }
      }
#pragma unroll
      for (int q = 0; q < APT; ++q)
        *reinterpret_cast<uint4 *>(&As[a_row * LDR + a_half * (BK / 2) * ESZ + q * 16]) = wreg[q];
      __syncthreads();
      // both register tiles are in LDS now: the next chunk travels while this one is multiplied
      // (past the last chunk: zeros and values nobody uses, no memory traffic to speak of)
      load_w(kc + 1);
      raw.load(xdesc, xoff + (uint32_t)((kc + 1) * BK) * (uint32_t)k * XB, k);
      const int fr = lane & 31, half = lane >> 5;
      if constexpr (I8W) {
#pragma unroll
        for (int ks = 0; ks < BK / 32; ++ks) {
          const intx4 a = __builtin_bit_cast(
              intx4, *reinterpret_cast<const uint4 *>(&As[(wv * 32 + fr) * LDR + ks * 32 + half * 16]));
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const intx4 bb = __builtin_bit_cast(
                intx4, *reinterpret_cast<const uint4 *>(&Bs[(i * 32 + fr) * LDR + ks * 32 + half * 16]));
            acc[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, bb, acc[i], 0, 0, 0);
          }
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
          const bf16x8 a = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const uint4 *>(&As[(wv * 32 + fr) * LDR + (ks * 16 + half * 8) * 2]));
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const bf16x8 bb = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const uint4 *>(&Bs[(i * 32 + fr) * LDR + (ks * 16 + half * 8) * 2]));
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bb, acc[i], 0, 0, 0);
          }
        }
      }
      __syncthreads();
    }
  }
  // epilogue: acc[i][r] is row (r/4)*8 + (lane/32)*4 + r%4, column NB*(lane%32) + i
  const float sx = al / 127.f;
  const int64_t n = n0 + NB * (lane & 31);
  if (n < k) {  // k % 4 == 0: a lane's NB positions are all inside or all outside
    // The two choices that are the same for the whole wave are taken once, outside the loop over
    // the rows: whether all 32 rows of the wave exist (then no store sits under a test) and
    // whether the output is streamed past the caches.
    auto store_rows = [&](auto whole_c, auto stream_c) {
      constexpr bool WHOLE = decltype(whole_c)::value, STREAM = decltype(stream_c)::value;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wv * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        if (WHOLE || m < M) {
          float v[NB];
          const float sc = I8W ? sx * w_scale[m] : sx;
#pragma unroll
          for (int i = 0; i < NB; ++i) v[i] = (float)acc[i][r] * sc;
          float *dst = yc + ((size_t)b * M + m) * k + n;
          if constexpr (STREAM) {  // an output that no cache will hold for its reader
            if constexpr (NB == 4) {
              floatx4 o = {v[0], v[1], v[2], v[3]};
              __builtin_nontemporal_store(o, reinterpret_cast<floatx4 *>(dst));
            } else {
              floatx2 o = {v[0], v[1]};
              __builtin_nontemporal_store(o, reinterpret_cast<floatx2 *>(dst));
            }
          } else {
            if constexpr (NB == 4) *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
            else *reinterpret_cast<float2 *>(dst) = make_float2(v[0], v[1]);
          }
        }
      }
    };
    const bool whole = m0 + wv * 32 + 32 <= M;
    if (whole) {
      if (stream_out) store_rows(std::true_type{}, std::true_type{});
      else store_rows(std::true_type{}, std::false_type{});
    } else {
      if (stream_out) store_rows(std::false_type{}, std::true_type{});
      else store_rows(std::false_type{}, std::false_type{});
    }
  }  // positions inside the signal
  }  // row tiles
}

template <int BM, int BN, bool I8W>
hipError_t mfma_launch(const wcc_desc &d, int64_t k, const void *w, const float *w_scale,
                       const void *xc, int form, const float *alpha, int n_alpha, float *alpha_out,
                       float *yc, hipStream_t s) {
  dim3 grid((unsigned)((k + BN - 1) / BN), (d.C_out + BM - 1) / BM, d.B), block(2 * BM);
  // several row tiles: one workgroup walks them all where the column tiles alone fill the chip
  if (grid.y > 1 && (int64_t)grid.x * grid.z >= 2 * 256) grid.y = 1;
  // The inverse transform reads yc next.  Up to about twice the 256 MB memory-side cache it is
  // better left there (measured); beyond that the output is streamed past it.
  const bool stream_out = (int64_t)d.B * d.C_out * k * 4 > ((int64_t)512 << 20);
  const bool rag = d.C_in % (I8W ? 16 : 8) != 0;
#define WCC_STREAM(FORM, RAG)                                                                         \
  hipLaunchKernelGGL((pointwise_mfma_kernel<BM, BN, FORM, I8W, RAG>), grid, block, 0, s, w, w_scale,   \
                     xc, alpha, n_alpha, alpha_out, yc, d.C_out, d.C_in, k, stream_out)
  if (form == kFloats)     { if (rag) WCC_STREAM(kFloats, true); else WCC_STREAM(kFloats, false); }
  else if (form == kWords) { if (rag) WCC_STREAM(kWords, true); else WCC_STREAM(kWords, false); }
  else                     { if (rag) WCC_STREAM(kCodes, true); else WCC_STREAM(kCodes, false); }
#undef WCC_STREAM
  return hipGetLastError();
}

// ---- the contraction where it is bound by arithmetic (hundreds of channels and more) ------------
// The kernel above is laid out for the memory-bound layers: a wave tile of 32 x 128 re-reads
// every activation fragment in all eight waves (five 16-byte LDS reads per four matrix
// instructions) and one LDS buffer costs two barriers a chunk.  With C_in in the hundreds or
// thousands the matrix cores are what counts, so this variant spends LDS bandwidth and barriers
// sparingly:
//   workgroup tile 128 (rows) x 128 (positions), four waves in a 2 x 2 arrangement, wave tile
//   64 x 64 = 2 x 2 blocks of 32 x 32 (64 accumulator registers, so that two register sets of
//   loads in flight still leave room for three workgroups a compute unit): four fragment reads
//   per four matrix instructions;
//   two LDS stages of 64 bytes of K a row (32 channels of bf16, 64 of int8: the byte addressing
//   of both operand types is the same), 20 KB each: while the matrix instructions of stage s
//   run, the registers loaded two stages earlier are converted and written into the other
//   buffer and the loads of the stage after next are issued; one barrier a stage.
// Activations are int8 codes only (the fused layer's default route).  Positions are stored
// permuted inside a wave's 64 columns (row (n % 2) * 32 + n / 2), so that after the two column
// blocks a lane holds two adjacent positions of one output row and stores 8 bytes.
// Which tile a workgroup takes: the hardware hands consecutive workgroups to the 8 dies in
// turn, each die with an L2 of its own; here die x works through the x-th eighth of the tile
// list (positions fastest, then rows, then samples), so that the tiles a die has in flight share
// their activation columns and walk through neighbouring weight rows in ITS L2.  With the
// natural order every die touches every operand and most fetches come from beyond the L2s
// (1.1 GB at 5 TB/s for 116 GFLOP on 4096 x 1024 weights).
// Needs k % 4 == 0 and C_in % 8 == 0 (bf16 weights) or % 16 == 0 (int8 weights).
constexpr int kDies = 8;
constexpr int kTileM = 128, kTileN = 128, kTileKB = 64, kTileLDR = kTileKB + 16;
constexpr int kTileMinChannels = 256;

// (256-row tiles with 128 x 64 wave tiles, two workgroups a compute unit: measured slower on every layer
// tried, 176 vs 147 us at 1024 -> 4096 channels; three resident workgroups hide more than the halved
// conversion work saves)
// Reached by the stage call, and by fused layers whose compressed signal leaves no room for packed weights.
template <bool I8W>
__global__ __launch_bounds__(256, 3) void pointwise_tile_kernel(
    const void *__restrict__ w, const float *__restrict__ w_scale, const int8_t *__restrict__ xq,
    const float *__restrict__ alpha, int n_alpha, float *alpha_out, float *__restrict__ yc, int M,
    int K, int64_t k, bool stream_out, int gx, int gy, int tiles, int dies) {
  constexpr int ESZ = I8W ? 1 : 2;        // bytes of a weight / of an activation in LDS
  constexpr int KC = kTileKB / ESZ;       // channels a stage: 64 or 32
  constexpr int CPT = KC / 8;             // channels a thread converts: 8 or 4
  constexpr int LDR = kTileLDR;
  __shared__ __attribute__((aligned(16))) unsigned char As[2][kTileM * LDR];
  __shared__ __attribute__((aligned(16))) unsigned char Bs[2][kTileN * LDR];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int wm = wv >> 1, wn = wv & 1;    // the wave's place in the 2 x 2 arrangement
  // grid = 8 * ceil(tiles / 8) workgroups in one dimension
  // (dies = 1: the natural order, for layers whose weights every L2 holds anyway and whose time
  // goes into writing yc: there the dies had better write one neighbourhood together)
  const int tile = (blockIdx.x % dies) * (gridDim.x / dies) + blockIdx.x / dies;
  const int b = tile / (gx * gy), by = (tile / gx) % gy, bx = tile % gx;
  const int64_t n0 = (int64_t)bx * kTileN;
  const int m0 = by * kTileM;
  const int8_t *xb = xq + (size_t)b * K * k;
  const unsigned char *wb = static_cast<const unsigned char *>(w);
  // activation loader: group of four positions, channel group.  A wave takes 8 position groups
  // x all 8 channel groups: the 32 lanes that an LDS write serves together then hit 8 rows
  // (160 bytes apart) x 4 channel groups (8 bytes apart) = 32 different 8-byte bank pairs; with
  // 32 position groups a wave the same write was a four-way bank conflict.
  const int g = wv * 8 + (lane & 7), kq = lane >> 3;
  const int stages = (K + KC - 1) / KC;

  const float al = alpha_max(alpha, n_alpha);  // (every thread of the workgroup is here)
  if (alpha_out && tile == 0 && threadIdx.x == 0) alpha_out[0] = al;
  if (tile >= tiles) return;  // the workgroups that pad the grid to a multiple of 8

  using Acc = std::conditional_t<I8W, intx16, floatx16>;
  Acc acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

  // global -> registers: half a weight row (32 of a stage's 64 bytes of K; two threads a row)
  // and the thread's CPT x 4 activation patch,
  // through buffer descriptors of the weights and of the sample's compressed signal: what lies
  // a load never faults (outside the buffer it returns zeros, and an offset that wraps lands
  // inside it), so there is no branch and no lane mask, a prefetch may run past the last
  // stage, and the compiler can count the loads in flight exactly.  Weights of channels
  // >= C_in are zeros (the offset is sent outside, a wave-uniform choice), so whatever the
  // activation loads return for those channels is multiplied by zero; rows >= M and positions
  // >= k (last tiles) read something, but their rows and columns are never stored and feed
  // no other.
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  struct Regs {
    u32x4 w[2];
    uint32_t x[CPT];
  };
  const __amdgpu_buffer_rsrc_t wdesc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char *>(wb), 0, (int)(uint32_t)((int64_t)M * K * ESZ), 0x00020000);
  const __amdgpu_buffer_rsrc_t xdesc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t *>(xb), 0, (int)(uint32_t)((int64_t)K * k), 0x00020000);
  constexpr uint32_t kOutside = 0xFFFFFFF0u;
  // (two lanes a row: their 16-byte LDS writes collide pairwise with those of other rows, but a
  // row per lane -- conflict-free in LDS -- makes every load touch 64 cache lines instead of 32
  // and was measured slower, 175 vs 147 us)
  const int a_row = t >> 1, a_half = t & 1;
  const uint32_t wrow = (uint32_t)(m0 + a_row) * (uint32_t)(K * ESZ);
  const uint32_t xcol = (uint32_t)(n0 + 4 * g) + (uint32_t)(kq * CPT) * (uint32_t)k;
  auto fetch = [&](Regs &r, int st) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      // first channel of the 16-byte load; a stage is whole or empty in K (C_in is a multiple of
      // what 16 bytes hold), but its two halves may differ: the choice is the lane's
      const int kk = st * KC + (a_half * 2 + q) * (16 / ESZ);
      r.w[q] = __builtin_amdgcn_raw_buffer_load_b128(wdesc, kk < K ? wrow + (uint32_t)kk * ESZ : kOutside, 0, 0);
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c)  // channel st * KC + c (+ kq * CPT, which xcol carries)
      r.x[c] = __builtin_amdgcn_raw_buffer_load_b32(xdesc, xcol + (uint32_t)(st * KC + c) * (uint32_t)k, 0, 0);
  };
  // registers -> LDS stage `buf`: the weight row as it is; the patch transposed (and widened to
  // bf16 for bf16 weights: an integer |v| <= 127 is exact there, its pattern is the float's
  // high half), 8 bytes of K for each of the four positions
  auto stash = [&](const Regs &r, int buf) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
      *reinterpret_cast<u32x4 *>(&As[buf][a_row * LDR + (a_half * 2 + q) * 16]) = r.w[q];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t lo, hi;
      if constexpr (I8W) {
        // byte i of eight channel words -> two words of four channels each
        const uint32_t sel = 0x0C0C0400u + 0x00000101u * i;   // {.., .., b[i], a[i]}
        const uint32_t p01 = __builtin_amdgcn_perm(r.x[1], r.x[0], sel);
        const uint32_t p23 = __builtin_amdgcn_perm(r.x[3], r.x[2], sel);
        const uint32_t p45 = __builtin_amdgcn_perm(r.x[5], r.x[4], sel);
        const uint32_t p67 = __builtin_amdgcn_perm(r.x[7], r.x[6], sel);
        lo = (p01 & 0xFFFFu) | (p23 << 16);
        hi = (p45 & 0xFFFFu) | (p67 << 16);
      } else {
        float f[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) f[c] = (float)((int)(r.x[c] << (24 - 8 * i)) >> 24);
        lo = __builtin_amdgcn_perm(__float_as_uint(f[1]), __float_as_uint(f[0]), 0x07060302u);
        hi = __builtin_amdgcn_perm(__float_as_uint(f[3]), __float_as_uint(f[2]), 0x07060302u);
      }
      const int nl = 4 * g + i;  // position inside the workgroup's tile
      const int row = (nl & 64) + (nl & 1) * 32 + ((nl & 63) >> 1);
      *reinterpret_cast<uint2 *>(&Bs[buf][row * LDR + kq * 8]) = make_uint2(lo, hi);
    }
  };
  const int fr = lane & 31, half = lane >> 5;
  auto multiply = [&](int buf) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      uint4 a[2], bb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        a[i] = *reinterpret_cast<const uint4 *>(&As[buf][(wm * 64 + i * 32 + fr) * LDR + ks * 32 + half * 16]);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        bb[j] = *reinterpret_cast<const uint4 *>(&Bs[buf][(wn * 64 + j * 32 + fr) * LDR + ks * 32 + half * 16]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if constexpr (I8W)
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(intx4, a[i]),
                                                             __builtin_bit_cast(intx4, bb[j]), acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i]),
                                                               __builtin_bit_cast(bf16x8, bb[j]), acc[i][j], 0, 0, 0);
        }
    }
  };

  // Two register sets: the loads of a stage are issued two stages before they are converted,
  // so that they have a whole stage of matrix instructions (and the other workgroup's) to
  // arrive.  r0 carries the odd stages, r1 the even ones.
  Regs r0, r1;
  fetch(r0, 0);
  stash(r0, 0);
  fetch(r0, 1);
  fetch(r1, 2);
  __syncthreads();
  // (an odd number of stages is rounded up: the stage past the end loads zeros and adds them;
  // a way out in the middle of the loop body made the compiler keep two copies of the
  // accumulators and move 64 registers a stage)
  for (int s = 0; s < stages; s += 2) {
    stash(r0, 1);      // stage s + 1 (every wave left buffer 1 at the last barrier)
    fetch(r0, s + 3);
    multiply(0);       // stage s
    __syncthreads();
    // (nothing of the next half moves up across this point: the compiler would start converting
    // r1 here, a stage early, and wait for loads that have another stage to arrive)
    __builtin_amdgcn_sched_barrier(0);
    stash(r1, 0);      // stage s + 2
    fetch(r1, s + 4);
    multiply(1);       // stage s + 1
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
  }

  // acc[i][j][r]: row wm*64 + i*32 + (r/4)*8 + (lane/32)*4 + r%4, position wn*64 + 2*(lane%32) + j
  const float sx = al / 127.f;
  const int64_t n = n0 + wn * 64 + 2 * fr;
  if (n < k) {  // k % 4 == 0 and n even: both positions inside or both outside
    // (what is the same for the whole wave is decided once, outside the loops over the rows)
    auto store_rows = [&](auto whole_c, auto stream_c) {
      constexpr bool WHOLE = decltype(whole_c)::value, STREAM = decltype(stream_c)::value;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + wm * 64 + i * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
          if (WHOLE || m < M) {
            const float sc = I8W ? sx * w_scale[m] : sx;
            const float v0 = (float)acc[i][0][r] * sc, v1 = (float)acc[i][1][r] * sc;
            float *dst = yc + ((size_t)b * M + m) * k + n;
            if constexpr (STREAM) {
              floatx2 o = {v0, v1};
              __builtin_nontemporal_store(o, reinterpret_cast<floatx2 *>(dst));
            } else {
              *reinterpret_cast<float2 *>(dst) = make_float2(v0, v1);
            }
          }
        }
    };
    const bool whole = m0 + wm * 64 + 64 <= M;
    if (whole) {
      if (stream_out) store_rows(std::true_type{}, std::true_type{});
      else store_rows(std::true_type{}, std::false_type{});
    } else {
      if (stream_out) store_rows(std::false_type{}, std::true_type{});
      else store_rows(std::false_type{}, std::false_type{});
    }
  }
}

// ---- the same on weights in the order of the matrix instructions ------------------------------
// What bounds the kernel above is LDS: with 64 x 64 wave tiles every matrix instruction needs one
// 16-byte fragment read, and three workgroups a compute unit keep LDS busy all the time.  Here a
// wave's tile is 64 rows x 128 (or 64) positions and only the activations go through LDS (four
// reads for eight instructions); the weights come straight from memory into registers, reloaded a
// stage ahead as each is used.  A lane's 16 bytes of a row are one of 32 rows' pieces, 32 bytes a
// row and instruction, which cost the address unit as much as the matrix cores had to do
// (1024 -> 256 channels: 110 us); so the weights are first brought into the order of the
// instructions (PackJob), one contiguous KiB a load: 88 us.  The fused calls do that inside the
// selection's first kernel, in memory that the codes leave free; the stage call, which needs no
// workspace unless weights are 4-bit, keeps the kernel above.
// A workgroup's four waves take 64 * WM rows (WM waves) x 32 * CB * 4 / WM positions.  A stage is 128
// bytes of K (64 channels of bf16, 128 of int8), two LDS buffers, one barrier a stage; the
// activations of the stage after next are in flight under the matrix instructions.  The tiles are
// dealt to the dies in contiguous chunks of the list, positions fastest (256 -> 1024 channels
// 125 us, in the natural order 135).
// Measured (8 x 16384 positions): 1024 -> 256 channels 120 -> 88 us with bf16 weights, 94 -> 70
// with int8; 256 -> 1024 158 -> 125 and 142 -> 107; 1024 -> 4096 and back at 6 x 2304: 148 -> 109 and
// 161 -> 107 us (1.08 PFLOP/s).
__global__ __launch_bounds__(256) void pack_weights_kernel(PackJob job) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e < job.total) job.out[e] = pack_piece(job, e);
}

template <bool I8W, int WM, int CB, bool WORDS>
__global__ __launch_bounds__(256, CB == 4 ? 2 : 3) void pointwise_wide_kernel(
    const uint4 *__restrict__ w, const float *__restrict__ w_scale, const int8_t *__restrict__ xq,
    const float *__restrict__ alpha, int n_alpha, float *alpha_out, float *__restrict__ yc, int M,
    int K, int64_t k, bool stream_out, int gx, int gy, int tiles) {
  constexpr int ESZ = I8W ? 1 : 2;
  fetch_args(w, k);
  constexpr int KB = 128, LDR = KB + 16;   // bytes of K a stage, LDS row bytes
  constexpr int KC = KB / ESZ;             // channels a stage: 64 or 128
  constexpr int WN = 4 / WM;               // waves along the positions
  constexpr int TM = 64 * WM, TN = 32 * CB * WN;
  constexpr int NG = TN / 4;               // groups of four positions
  constexpr int DW = NG * KC / 256;        // activation words a thread and stage
  constexpr int CPT = I8W ? (DW >= 16 ? 16 : 8) : (DW >= 8 ? 8 : 4);  // channels of a patch
  constexpr int PT = DW / CPT;             // patches a thread
  constexpr int KQ = KC / CPT;             // channel groups of a stage
  static_assert(PT >= 1 && NG * KQ == 256 * PT, "patches cover the stage");
  __shared__ __attribute__((aligned(16))) unsigned char Bs[2][TN * LDR];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int wm = wv % WM, wn = wv / WM;
  const int tile = (blockIdx.x % kDies) * (gridDim.x / kDies) + blockIdx.x / kDies;
  const float al = alpha_max(alpha, n_alpha);
  if (alpha_out && tile == 0 && threadIdx.x == 0) alpha_out[0] = al;
  if (tile >= tiles) return;
  const int b = tile / (gx * gy);
  const int by = (tile / gx) % gy, bx = tile % gx;
  const int64_t n0 = (int64_t)bx * TN;
  const int m0 = by * TM + wm * 64;
  const int8_t *xb = xq + (size_t)b * K * k;
  const int stages = (K + KC - 1) / KC;

  using Acc = std::conditional_t<I8W, intx16, floatx16>;
  Acc acc[2][CB];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  // (what lies outside returns zeros: blocks of rows past the last one, stages past the last one of
  // the last block; a stage past the end of another block reads the next block's weights, which
  // meet nothing that is used)
  const __amdgpu_buffer_rsrc_t wdesc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint4 *>(w), 0, (int)(uint32_t)((int64_t)((M + 63) / 64 * 64) * stages * KB), 0x00020000);
  const __amdgpu_buffer_rsrc_t xdesc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t *>(xb), 0, (int)(uint32_t)((int64_t)K * k), 0x00020000);
  const int fr = lane & 31, half = lane >> 5;
  // weights of step ks of a stage, for the wave's two blocks of 32 rows
  u32x4 a[4][2];
  const uint32_t wline = (uint32_t)(m0 / 32) * (uint32_t)(stages * 4) * 1024u + (uint32_t)lane * 16u;
  auto load_a = [&](int st, int ks) {
    const uint32_t at = wline + (uint32_t)(st * 4 + ks) * 1024u;
    a[ks][0] = __builtin_amdgcn_raw_buffer_load_b128(wdesc, at, 0, 0);
    a[ks][1] = __builtin_amdgcn_raw_buffer_load_b128(wdesc, at + (uint32_t)stages * 4096u, 0, 0);
  };
  // activations: CPT channels x 4 positions a patch
  uint32_t x[PT][WORDS ? 1 : CPT];
  word4 xw[PT][WORDS ? CPT / 4 : 1];  // (C_in is a multiple of four)
  uint32_t xcol[PT];
#pragma unroll
  for (int p = 0; p < PT; ++p) {
    const int e = t + 256 * p, g = e % NG, kq = e / NG;
    xcol[p] = (uint32_t)(n0 + 4 * g) * (WORDS ? 4u : 1u) + (uint32_t)(kq * CPT) * (uint32_t)k;
  }
  auto load_x = [&](int st) {
#pragma unroll
    for (int p = 0; p < PT; ++p)
#pragma unroll
      for (int c = 0; c < CPT; c += WORDS ? 4 : 1) {
        const uint32_t at = xcol[p] + (uint32_t)(st * KC + c) * (uint32_t)k;
        if constexpr (WORDS) xw[p][c / 4] = __builtin_amdgcn_raw_buffer_load_b128(xdesc, at, 0, 0);
        else x[p][c] = __builtin_amdgcn_raw_buffer_load_b32(xdesc, at, 0, 0);
      }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int p = 0; p < PT; ++p) {
      const int e = t + 256 * p, g = e % NG, kq = e / NG;
      uint32_t o[4][CPT * ESZ / 4];  // [position][words]
      if constexpr (WORDS) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int c = 0; c < CPT; c += 4) {
            const uint32_t four = xw[p][c / 4][i];
            if constexpr (I8W) {
              o[i][c / 4] = four;
            } else {
              float f[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) f[u] = (float)((int)(four << (24 - 8 * u)) >> 24);
              o[i][c / 2] = __builtin_amdgcn_perm(__float_as_uint(f[1]), __float_as_uint(f[0]), 0x07060302u);
              o[i][c / 2 + 1] = __builtin_amdgcn_perm(__float_as_uint(f[3]), __float_as_uint(f[2]), 0x07060302u);
            }
          }
      } else if constexpr (I8W) {
#pragma unroll
        for (int c = 0; c < CPT; c += 4) {
          const uint32_t lo01 = __builtin_amdgcn_perm(x[p][c + 1], x[p][c], 0x05010400u);
          const uint32_t lo23 = __builtin_amdgcn_perm(x[p][c + 3], x[p][c + 2], 0x05010400u);
          const uint32_t hi01 = __builtin_amdgcn_perm(x[p][c + 1], x[p][c], 0x07030602u);
          const uint32_t hi23 = __builtin_amdgcn_perm(x[p][c + 3], x[p][c + 2], 0x07030602u);
          o[0][c / 4] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
          o[1][c / 4] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
          o[2][c / 4] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
          o[3][c / 4] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int c = 0; c < CPT; c += 2) {
            const float f0 = (float)((int)(x[p][c] << (24 - 8 * i)) >> 24);
            const float f1 = (float)((int)(x[p][c + 1] << (24 - 8 * i)) >> 24);
            o[i][c / 2] = __builtin_amdgcn_perm(__float_as_uint(f1), __float_as_uint(f0), 0x07060302u);
          }
      }
      constexpr int WPN = 32 * CB;  // positions of a wave
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int nl = 4 * g + i;
        const int row = (nl / WPN) * WPN + (nl % CB) * 32 + (nl % WPN) / CB;
        unsigned char *dst = &Bs[buf][row * LDR + kq * CPT * ESZ];
        if constexpr (CPT * ESZ == 16) *reinterpret_cast<uint4 *>(dst) = make_uint4(o[i][0], o[i][1], o[i][2], o[i][3]);
        else *reinterpret_cast<uint2 *>(dst) = make_uint2(o[i][0], o[i][1]);
      }
    }
  };

  load_x(0);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) load_a(0, ks);
  stash(0);
  load_x(1);
  __syncthreads();
  for (int s = 0; s < stages; ++s) {
    const unsigned char *bs = &Bs[s & 1][(wn * 32 * CB + fr) * LDR + half * 16];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      uint4 bb[CB];
#pragma unroll
      for (int j = 0; j < CB; ++j) bb[j] = *reinterpret_cast<const uint4 *>(bs + j * 32 * LDR + ks * 32);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) {
          if constexpr (I8W)
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(intx4, a[ks][i]),
                                                             __builtin_bit_cast(intx4, bb[j]), acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[ks][i]),
                                                               __builtin_bit_cast(bf16x8, bb[j]), acc[i][j], 0, 0, 0);
        }
      load_a(s + 1, ks);
    }
    stash((s + 1) & 1);
    load_x(s + 2);
    __syncthreads();
  }

  const float sx = al / 127.f;
  const int64_t n = n0 + wn * 32 * CB + CB * fr;
  if (n < k) {
    auto store_rows = [&](auto whole_c, auto stream_c) {
      constexpr bool WHOLE = decltype(whole_c)::value, STREAM = decltype(stream_c)::value;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + i * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
          if (WHOLE || m < M) {
            const float sc = I8W ? sx * w_scale[m] : sx;
            float *dst = yc + ((size_t)b * M + m) * k + n;
            if constexpr (CB == 4) {
              floatx4 o = {(float)acc[i][0][r] * sc, (float)acc[i][1][r] * sc, (float)acc[i][2][r] * sc,
                           (float)acc[i][3][r] * sc};
              if constexpr (STREAM) __builtin_nontemporal_store(o, reinterpret_cast<floatx4 *>(dst));
              else *reinterpret_cast<floatx4 *>(dst) = o;
            } else {
              floatx2 o = {(float)acc[i][0][r] * sc, (float)acc[i][1][r] * sc};
              if constexpr (STREAM) __builtin_nontemporal_store(o, reinterpret_cast<floatx2 *>(dst));
              else *reinterpret_cast<floatx2 *>(dst) = o;
            }
          }
        }
    };
    const bool whole = m0 + 64 <= M;
    if (whole) {
      if (stream_out) store_rows(std::true_type{}, std::true_type{});
      else store_rows(std::true_type{}, std::false_type{});
    } else {
      if (stream_out) store_rows(std::false_type{}, std::true_type{});
      else store_rows(std::false_type{}, std::false_type{});
    }
  }
}

template <bool I8W, int WM, int CB>
hipError_t wide_launch(const wcc_desc &d, int64_t k, const uint4 *packed, const float *w_scale, const void *xc,
                       bool words, const float *alpha, int n_alpha, float *alpha_out, float *yc, hipStream_t s) {
  constexpr int TM = 64 * WM, TN = 32 * CB * (4 / WM);
  const int64_t gx = (k + TN - 1) / TN, gy = (d.C_out + TM - 1) / TM;
  const int64_t tiles = gx * gy * d.B;
  if (tiles > (int64_t)1 << 30) return hipErrorInvalidValue;
  dim3 grid((unsigned)((tiles + kDies - 1) / kDies * kDies)), block(256);
  const bool stream_out = (int64_t)d.B * d.C_out * k * 4 > ((int64_t)512 << 20);
  if (words)
    hipLaunchKernelGGL((pointwise_wide_kernel<I8W, WM, CB, true>), grid, block, 0, s, packed, w_scale,
                       static_cast<const int8_t *>(xc), alpha, n_alpha, alpha_out, yc, d.C_out, d.C_in, k,
                       stream_out, (int)gx, (int)gy, (int)tiles);
  else
    hipLaunchKernelGGL((pointwise_wide_kernel<I8W, WM, CB, false>), grid, block, 0, s, packed, w_scale,
                       static_cast<const int8_t *>(xc), alpha, n_alpha, alpha_out, yc, d.C_out, d.C_in, k,
                       stream_out, (int)gx, (int)gy, (int)tiles);
  return hipGetLastError();
}

template <bool I8W>
hipError_t tile_launch(const wcc_desc &d, int64_t k, const void *w, const float *w_scale, const void *xc,
                       const float *alpha, int n_alpha, float *alpha_out, float *yc, hipStream_t s) {
  const int64_t gx = (k + kTileN - 1) / kTileN, gy = (d.C_out + kTileM - 1) / kTileM;
  const int64_t tiles = gx * gy * d.B;
  if (tiles > (int64_t)1 << 30) return hipErrorInvalidValue;
  dim3 grid((unsigned)((tiles + kDies - 1) / kDies * kDies)), block(256);
  const bool stream_out = (int64_t)d.B * d.C_out * k * 4 > ((int64_t)512 << 20);
  hipLaunchKernelGGL((pointwise_tile_kernel<I8W>), grid, block, 0, s, w, w_scale,
                     static_cast<const int8_t *>(xc), alpha, n_alpha, alpha_out, yc, d.C_out, d.C_in, k,
                     stream_out, (int)gx, (int)gy, (int)tiles,
                     (int64_t)d.C_out * d.C_in * (I8W ? 1 : 2) >= ((int64_t)1 << 20) ? kDies : 1);
  return hipGetLastError();
}

// Is the layer one for the arithmetic-bound variant?  int8 codes in, enough channels that the
// matrix instructions outweigh the stream (measured crossover), at least a tile of output
// rows, and a workgroup for every compute unit.
static bool wants_tile_kernel(const wcc_desc &d, int64_t k, bool f32) {
  if (f32 || d.C_in < kTileMinChannels || d.C_out < kTileM) return false;
  if (d.C_in % (d.w_dtype == WCC_BF16 ? 8 : 16) != 0) return false;  // (it loads whole 16 bytes of a row)
  // an expansion layer with few input channels spends its time writing yc: the stream kernel's
  // 16-byte stores and its walk over the row tiles do that better (1024 x 256: 170 vs 180 us)
  if (d.C_in < 512 && d.C_out >= 4 * d.C_in) return false;
  const int64_t wgs = ((k + kTileN - 1) / kTileN) * ((d.C_out + kTileM - 1) / kTileM) * (int64_t)d.B;
  // (byte offsets into the weights and into a sample's compressed signal fit 32 bits)
  const int64_t limit = (int64_t)0xFFFFFFF0;
  if ((int64_t)(d.C_out + kTileM) * d.C_in * 2 > limit || (int64_t)d.C_in * k > limit) return false;
  return wgs >= 256 && wgs <= ((int64_t)1 << 30);
}

// Tile choice.  Large tiles first (BM = 256 when C_out needs it: every activation is then read
// once), as long as they give every compute unit a workgroup; otherwise smaller ones.
template <bool I8W>
hipError_t mfma_dispatch(const wcc_desc &d, int64_t k, const void *w, const float *w_scale,
                         const void *xc, int form, const float *alpha, int n_alpha, float *alpha_out,
                         float *yc, hipStream_t s) {
#define WCC_MFMA(BM_, BN_) \
  return mfma_launch<BM_, BN_, I8W>(d, k, w, w_scale, xc, form, alpha, n_alpha, alpha_out, yc, s)
  if (form != kWords && wants_tile_kernel(d, k, form == kFloats))
    return tile_launch<I8W>(d, k, w, w_scale, xc, alpha, n_alpha, alpha_out, yc, s);
  const int64_t want = 256;  // compute units
  auto wgs = [&](int bm, int bn) {
    return ((k + bn - 1) / bn) * ((d.C_out + bm - 1) / bm) * (int64_t)d.B;
  };
  if (d.C_out > 128 && wgs(256, 128) >= want) WCC_MFMA(256, 128);
  if (d.C_out <= 128 && wgs(128, 128) >= want) WCC_MFMA(128, 128);
  // (a quarter of the chip is enough for the 128-row tile: on the short signals of deep layers
  // the smaller tile quantises and stages every activation once more per extra row tile, which
  // costs more than the idle units: 960 -> 320 channels at k = 512, 19.5 -> 17.2 us)
  if (d.C_out > 64 && wgs(128, 64) >= want / 4) WCC_MFMA(128, 64);
  WCC_MFMA(64, 64);
#undef WCC_MFMA
}

// ---- the contraction on the fp32 matrix instructions (any storage types, any shape) ---------------
// Layers with fp32 weights or unquantised activations, and the stage call on a compressed signal
// whose rows no kernel above can load (k % 4 != 0).  v_mfma_f32_32x32x2_f32: fp32 products and
// fp32 sums as a chain of FMAs has them, at twice the rate of the vector unit (157 against
// 79 TFLOP/s), and one instruction keeps the matrix core busy for 64 cycles on two LDS words a
// lane, so operands are staged in LDS as they come: weights by row, activations by channel, no
// transposition.  Bound by the HBM traffic of xc and yc on most layers (2 * C_in * C_out /
// (4 * (C_in + C_out)) flop a byte: 24 at 96 -> 96 channels, 20 at the ratio of the two peaks).
// Measured against the vector-unit tile kernel that stood here (64 x 64 tiles, 16 values of a
// lane): 96 -> 96 channels at 4 x 15360 positions 37.5 -> 19.6 us, 32 -> 32 at 2048 8.2 -> 4.3 us;
// 87 TFLOP/s at 358 -> 570 channels x 38528.
// One LDS stage is filled while the other is multiplied, one barrier a stage; the loads of the
// stage after next travel under the matrix instructions.  With few channels the chain of latencies counts:
// no load is issued past the last stage, the row scales come in with the first loads, and where rows of yc
// are not whole words a store's lanes lie side by side.  (Loads past the end, a scale load in front of every store
// and stores of every other position: 2 -> 79 channels, int8, 3 x 45526 positions 31.4 us, 18.2 now and 19.4 with the
// vector-unit kernel; 8 -> 544, 6 x 5814 44.9, 23.9 and 23.7; 200 -> 544, fp32, 4 x 31103 327, 312 and 544.)
template <int DT> struct WLoad;
template <> struct WLoad<WCC_F32> {
  using T = float;
  static __device__ __forceinline__ float widen(T v) { return v; }
};
template <> struct WLoad<WCC_BF16> {
  using T = uint16_t;
  static __device__ __forceinline__ float widen(T v) { return __uint_as_float((uint32_t)v << 16); }
};
template <> struct WLoad<WCC_I8> {
  using T = int8_t;
  static __device__ __forceinline__ float widen(T v) { return (float)v; }
};

constexpr int FK = 16;  // channels a stage

// WVM: waves along the rows (4 / WVM along the positions); MB, NB: 32 x 32 blocks of a wave, so
// the workgroup's tile is 32 WVM MB rows x 32 (4 / WVM) NB positions.  Channels are accumulated in
// increasing order.  XM: 0 = fp32 activations as they are, 1 = int8 codes, 2 = fp32 activations
// quantised on load.  VEC: k % 4 == 0 (rows of xc and yc are read and written in words of four
// and two positions); otherwise one position at a time.
// grid = (ceil(k / TN), ceil(M / TM), B), block = 256.
template <int WDT, int XM, bool VEC, int WVM, int MB, int NB>
__global__ __launch_bounds__(256) void pointwise_f32_kernel(const void *__restrict__ w,
                                                            const float *__restrict__ w_scale,
                                                            const void *__restrict__ xc,
                                                            const float *__restrict__ alpha,
                                                            int n_alpha, float *alpha_out,
                                                            float *__restrict__ yc, int M, int K,
                                                            int64_t k) {
  constexpr int TM = 32 * WVM * MB, TN = 32 * (4 / WVM) * NB;
  fetch_args(w, k);
  constexpr int LDA = FK + 1, LDB = TN + 32;  // LDS row words: the 64 lanes of a read of Bs hit 64 banks
                                              // (of As 47; FK + 2, which makes that 64, measured the same)
  constexpr int NA = TM * FK / 256;           // weights a thread and stage
  constexpr int XV = VEC ? 4 : 1;             // positions a load
  constexpr int NX = TN * FK / 256 / XV;      // loads of activations a thread and stage
  // Where a lane stores words of two positions the two column blocks of a wave take the even and the
  // odd positions of its 64; else they lie side by side, so that the lanes of a store do.
  constexpr int STEP = VEC ? NB : 1;
  static_assert(TM * FK % 256 == 0 && TN * FK % (256 * XV) == 0, "whole loads");
  using WT = typename WLoad<WDT>::T;
  using XT = std::conditional_t<XM == 1, std::conditional_t<VEC, uint32_t, int8_t>,
                                std::conditional_t<VEC, float4, float>>;
  __shared__ float As[2][TM * LDA];
  __shared__ __attribute__((aligned(16))) float Bs[2][FK * LDB];
  __shared__ __attribute__((aligned(16))) float scales[WDT == WCC_I8 ? TM : 4];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int wm = wv % WVM, wn = wv / WVM;
  const int b = blockIdx.z, m0 = blockIdx.y * TM;
  const int64_t n0 = (int64_t)blockIdx.x * TN;
  const float al = XM != 0 ? load_alpha(alpha, n_alpha, alpha_out) : 0.f;
  const Quant quant(al);
  const WT *wp = static_cast<const WT *>(w);
  const size_t sample = (size_t)b * K * k;

  // Rows and positions outside are read at the last one inside (their results are not stored);
  // channels outside are read at the last channel and count as zero on both sides.
  WT areg[NA];
  XT xreg[NX];
  auto load = [&](int c0) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int e = t + 256 * i, row = min(m0 + e / FK, M - 1), ch = min(c0 + e % FK, K - 1);
      areg[i] = wp[(size_t)row * K + ch];
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int e = t + 256 * i;
      const int ch = min(c0 + e / (TN / XV), K - 1);
      const int64_t n = min(n0 + (int64_t)(e % (TN / XV)) * XV, k - XV);
      const size_t at = sample + (size_t)ch * k + n;
      if constexpr (XM == 1) xreg[i] = *reinterpret_cast<const XT *>(static_cast<const int8_t *>(xc) + at);
      else xreg[i] = *reinterpret_cast<const XT *>(static_cast<const float *>(xc) + at);
    }
  };
  auto stash = [&](int c0, int buf) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int e = t + 256 * i;
      As[buf][(e / FK) * LDA + e % FK] = c0 + e % FK < K ? WLoad<WDT>::widen(areg[i]) : 0.f;
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int e = t + 256 * i, kk = e / (TN / XV);
      const bool in = c0 + kk < K;
      float *dst = &Bs[buf][kk * LDB + (e % (TN / XV)) * XV];
      if constexpr (VEC) {
        float4 v;
        if constexpr (XM == 1) {
          const int c = (int)xreg[i];
          v = make_float4((float)(c << 24 >> 24), (float)(c << 16 >> 24), (float)(c << 8 >> 24), (float)(c >> 24));
        } else {
          v = xreg[i];
          if constexpr (XM == 2) v = make_float4(quant.level(v.x), quant.level(v.y), quant.level(v.z), quant.level(v.w));
        }
        *reinterpret_cast<float4 *>(dst) = in ? v : make_float4(0.f, 0.f, 0.f, 0.f);
      } else {
        float v = (float)xreg[i];
        if constexpr (XM == 2) v = quant.level(v);
        *dst = in ? v : 0.f;
      }
    }
  };
  floatx16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const int fr = lane & 31, half = lane >> 5;
  auto multiply = [&](int buf) {
#pragma unroll
    for (int ks = 0; ks < FK; ks += 2) {
      float a[MB], x[NB];
#pragma unroll
      for (int i = 0; i < MB; ++i) a[i] = As[buf][(wm * 32 * MB + i * 32 + fr) * LDA + ks + half];
      const float *row = &Bs[buf][(ks + half) * LDB + wn * 32 * NB + STEP * fr];
      if constexpr (STEP == 2) {
        const float2 v = *reinterpret_cast<const float2 *>(row);
        x[0] = v.x; x[1] = v.y;
      } else {
#pragma unroll
        for (int j = 0; j < NB; ++j) x[j] = row[32 * j];
      }
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], x[j], acc[i][j], 0, 0, 0);
    }
  };

  const int stages = (K + FK - 1) / FK;
  load(0);
  if constexpr (WDT == WCC_I8) {  // (read behind the barriers below)
    if (t < TM) scales[t] = w_scale[min(m0 + t, M - 1)];
  }
  stash(0, 0);
  if (stages > 1) load(FK);
  __syncthreads();
  for (int s = 0; s < stages; ++s) {
    multiply(s & 1);
    stash((s + 1) * FK, (s + 1) & 1);  // (every wave left that buffer at the last barrier)
    if (s + 2 < stages) load((s + 2) * FK);
    __syncthreads();
  }

  // acc[i][j][r]: row wm*32*MB + i*32 + (r/4)*8 + (lane/32)*4 + r%4, position wn*32*NB + (STEP == 2 ? 2*(lane%32) + j : 32*j + lane%32)
  const float sx = XM != 0 ? al / 127.f : 1.f;
  const int64_t n = n0 + wn * 32 * NB + STEP * fr;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = wm * 32 * MB + i * 32 + q * 8 + half * 4;  // four rows of the lane
      float4 s4 = make_float4(1.f, 1.f, 1.f, 1.f);
      if constexpr (WDT == WCC_I8) s4 = *reinterpret_cast<const float4 *>(&scales[row]);
      const float sw[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + row + e, r = 4 * q + e;
        if (m >= M || n >= k) continue;
        const float sc = sx * sw[e];
        float *dst = yc + ((size_t)b * M + m) * k + n;
        if constexpr (STEP == 2) {
          *reinterpret_cast<float2 *>(dst) = make_float2(acc[i][0][r] * sc, acc[i][1][r] * sc);
        } else {
#pragma unroll
          for (int j = 0; j < NB; ++j)
            if (n + 32 * j < k) dst[32 * j] = acc[i][j][r] * sc;
        }
      }
    }
}

template <int WDT, int XM, bool VEC>
hipError_t f32_launch(const wcc_desc &d, int64_t k, const void *w, const float *w_scale, const void *xc,
                      const float *alpha, int n_alpha, float *alpha_out, float *yc, hipStream_t s) {
#define WCC_F32MM(WVM, MB, NB)                                                                          \
  hipLaunchKernelGGL((pointwise_f32_kernel<WDT, XM, VEC, WVM, MB, NB>),                                 \
                     dim3((unsigned)((k + 32 * (4 / WVM) * NB - 1) / (32 * (4 / WVM) * NB)),            \
                          (d.C_out + 32 * WVM * MB - 1) / (32 * WVM * MB), d.B),                        \
                     dim3(256), 0, s, w, w_scale, xc, alpha, n_alpha, alpha_out, yc, d.C_out, d.C_in, k)
  // Tiles of 128 positions x 128 or 96 rows, whichever pads the rows less (96 -> 96 channels,
  // 4 x 15360 positions: 22.4 and 19.6 us; 358 -> 570, 38528: 182 and 181 us), where they give
  // every compute unit a workgroup; few rows take 32 x 128, the rest 64 x 64 (24.8 and 190 us there).
  auto wgs = [&](int tm) { return ((k + 127) / 128) * ((d.C_out + tm - 1) / tm) * (int64_t)d.B; };
  const bool by96 = (d.C_out + 95) / 96 * 96 < (d.C_out + 127) / 128 * 128;
  if (d.C_out > 64 && wgs(by96 ? 96 : 128) >= 256) {
    if (by96) WCC_F32MM(1, 3, 1); else WCC_F32MM(2, 2, 2);
  } else if (d.C_out <= 32) WCC_F32MM(1, 1, 1);
  else WCC_F32MM(2, 1, 1);
#undef WCC_F32MM
  return hipGetLastError();
}

template <int WDT>
hipError_t f32_dispatch(const wcc_desc &d, int64_t k, const void *w, const float *w_scale,
                        const void *xc, int xm, const float *alpha, int n_alpha, float *alpha_out,
                        float *yc, hipStream_t s) {
#define WCC_F32X(XM)                                                                                    \
  return k % 4 == 0 ? f32_launch<WDT, XM, true>(d, k, w, w_scale, xc, alpha, n_alpha, alpha_out, yc, s) \
                    : f32_launch<WDT, XM, false>(d, k, w, w_scale, xc, alpha, n_alpha, alpha_out, yc, s)
  switch (xm) {
    case 0: WCC_F32X(0);
    case 1: WCC_F32X(1);
    default: WCC_F32X(2);
  }
#undef WCC_F32X
}

}  // namespace

// Layers for the kernel on packed weights: 256 channels and more (128 -> 128 measured 5 % slower than
// the stream kernel, 64 -> 256 the same), more than one 64-row tile, rows of whole 16-byte pieces,
// and byte offsets that fit 32 bits.
PackJob pack_job(const wcc_desc &d, int64_t k, const void *w, void *room, size_t room_bytes) {
  PackJob job{nullptr, nullptr, 0, 0, 0, 0, 0};
  const bool i8 = d.w_dtype == WCC_I8 || d.w_dtype == WCC_I4;
  if (d.act_quant_bits != 8 || k % 4 != 0 || (!i8 && d.w_dtype != WCC_BF16)) return job;
  if (d.C_in < 256 || d.C_out <= 64 || d.C_in % (i8 ? 16 : 8) != 0) return job;
  const int64_t limit = (int64_t)0xFFFFFFF0;
  const int64_t steps = ((int64_t)d.C_in * (i8 ? 1 : 2) + 127) / 128 * 4, rows = ((int64_t)d.C_out + 63) / 64 * 64;
  const int64_t bytes = rows * steps * 32;
  if (bytes > ((int64_t)1 << 30) || (size_t)bytes > room_bytes || (int64_t)d.C_in * k > limit) return job;
  if ((k + 63) / 64 * ((d.C_out + 127) / 128) * (int64_t)d.B > ((int64_t)1 << 30)) return job;
  return PackJob{w, static_cast<uint4 *>(room), d.C_out, d.C_in, (int)steps, (int)(bytes / 16), d.w_dtype};
}

hipError_t launch_pack(const PackJob &job, hipStream_t s) {
  hipLaunchKernelGGL(pack_weights_kernel, dim3((job.total + 255) / 256), dim3(256), 0, s, job);
  return hipGetLastError();
}

hipError_t launch_pointwise_packed(const wcc_desc &d, int64_t k, const PackJob &job, const float *w_scale,
                                   const void *xc, bool words, const float *alpha, int n_alpha, float *alpha_out,
                                   float *yc, hipStream_t s) {
  // The largest tile that still gives a compute unit two workgroups: 256 x 128, or 128 x 128 for layers of up
  // to 128 rows; else 256 x 64, also for those: half its waves then multiply zeros, but it makes twice the
  // workgroups of 128 x 128 (384 -> 96 channels, bf16, 4 x 512 positions: 7.6 us and 9.0; 512 -> 128, 4 x 1024: 8.6
  // and 9.7; 256 -> 80, 8 x 2048: 6.8 and 8.6; 512 -> 96, int8, 4 x 4096: 10.0 and 9.9).
  auto wgs = [&](int tm, int tn) { return (k + tn - 1) / tn * ((d.C_out + tm - 1) / tm) * (int64_t)d.B; };
#define WCC_WIDE(WM, CB)                                                                                          \
  return job.wt == WCC_BF16                                                                                       \
             ? wide_launch<false, WM, CB>(d, k, job.out, w_scale, xc, words, alpha, n_alpha, alpha_out, yc, s)           \
             : wide_launch<true, WM, CB>(d, k, job.out, w_scale, xc, words, alpha, n_alpha, alpha_out, yc, s)
  if (d.C_out > 128 && wgs(256, 128) >= 512) WCC_WIDE(4, 4);
  if (d.C_out <= 128 && wgs(128, 128) >= 512) WCC_WIDE(2, 2);
  WCC_WIDE(4, 2);
#undef WCC_WIDE
}

// The layers of the stream kernel: rows of yc of whole words of four, rows of the weights of whole dwords, and 32-bit byte offsets
// into the activations (xbytes of them a sample) and the weights (more take the fp32 kernel).
static bool wants_stream_kernel(const wcc_desc &d, int64_t k, int64_t xbytes) {
  const int K = d.C_in;
  const int64_t limit = (int64_t)0xFFFFFFF0;
  // (Few channels into few rows leave the stream kernel's large tile, 128 rows x 64 channels, mostly empty: the
  // fp32 kernel's 32 rows x 16 channels fit them.  8 -> 8 channels, int8 weights, 15 x 265760 positions: 205 us
  // there, 94 here; 32 -> 16, 8 x 100000: 52 and 32; 40 -> 32, bf16, 4 x 60000: 17.1 and 16.8; 64 -> 32: 17.9 and
  // 21.7.  The sums of int8 codes are exact either way: 32 * 127 * 127 < 2^24.  Signals too short for that tile stay
  // with the 64 x 64 one: 24 -> 4, quantised on load, 8 x 2688, 5.0 us there and 5.7; 32 -> 16, 4 x 3840, 5.7 and 5.3.)
  const bool few = K <= 32 && d.C_out <= 32 && (k + 127) / 128 * (int64_t)d.B >= 256;
  if (d.act_quant_bits != 8 || k % 4 != 0 || few) return false;
  if ((int64_t)(d.C_out + 256) * K * 2 > limit || xbytes > limit) return false;
  return d.w_dtype == WCC_BF16 ? K % 2 == 0 : (d.w_dtype == WCC_I8 || d.w_dtype == WCC_I4) && K % 4 == 0;
}

bool pointwise_takes_words(const wcc_desc &d, int64_t k) {
  return wants_stream_kernel(d, k, (int64_t)(d.C_in + 3) / 4 * 4 * k) && !wants_tile_kernel(d, k, false);
}

hipError_t launch_pointwise(const wcc_desc &d, int64_t k, const void *w, const float *w_scale,
                            const void *xc, bool xc_is_f32, bool words, const float *alpha, int n_alpha,
                            float *alpha_out, float *yc, hipStream_t s) {
  const bool quant = d.act_quant_bits == 8;
  if (words && !pointwise_takes_words(d, k)) return hipErrorInvalidValue;
  if (wants_stream_kernel(d, k, (int64_t)d.C_in * k * (xc_is_f32 ? 4 : 1))) {
    const int form = words ? kWords : xc_is_f32 ? kFloats : kCodes;
    if (d.w_dtype == WCC_BF16) return mfma_dispatch<false>(d, k, w, w_scale, xc, form, alpha, n_alpha, alpha_out, yc, s);
    if (d.w_dtype == WCC_I8) return mfma_dispatch<true>(d, k, w, w_scale, xc, form, alpha, n_alpha, alpha_out, yc, s);
  }
  const int xm = !quant ? 0 : (xc_is_f32 ? 2 : 1);
  switch (d.w_dtype) {
    case WCC_F32: return f32_dispatch<WCC_F32>(d, k, w, w_scale, xc, xm, alpha, n_alpha, alpha_out, yc, s);
    case WCC_BF16: return f32_dispatch<WCC_BF16>(d, k, w, w_scale, xc, xm, alpha, n_alpha, alpha_out, yc, s);
    case WCC_I8: return f32_dispatch<WCC_I8>(d, k, w, w_scale, xc, xm, alpha, n_alpha, alpha_out, yc, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace wcc
