// First transform pass of the fused layer and the stand-alone analysis (Eq. HaarKernel,
// Eq. wavelet_transform), with the channel norm of Alg. 1 fused in.
#include "strip_io.h"

namespace wcc {
namespace {

// x [B, C, H, W] -> coef [B, C, N]; partial norms over this block's channel group to
// norm_part [G, B, N] (nullable); without STORE also the group's max |coefficient| per position
// to max_part [G, B, N] (nullable).
// WPU = 1: block = 256, grid = (ceil(units/4), G, B); each wave of a workgroup takes its own strip
//          unit and walks all channels of the group.
// WPU > 1: block = 64 * WPU, grid = (units, G, B); the WPU waves of a workgroup share one strip
//          unit and take a share of the group's channels each (WPU times the waves in flight for
//          the same number of partial-norm planes); their |coefficient| sums meet in LDS and are
//          added in wave order.
// split:   STORE with WPU = 1 only; grid.y = G * split.  A group's channels are cut as split waves that
//          share a unit would cut them, each part being a launch row with a plane of partial norms of its
//          own (norm_part [G * split, B, N]), which norm_reduce adds in the order of the shared form.
// DWM: 0 = x is transformed as it is; 1, 2 = K_dw x is (wdw [C, 3, 3]; 2: the outside columns
// of a wave row's first and last lane exist and are read).
// XT: float or bf16_t, the storage type of x.  SQ: sums of squares instead of absolute values.
template <int D, int V, int WPU, bool STORE, int PF, int DWM, class XT, bool SQ = false,
          bool NT = false>
__global__ __launch_bounds__(WPU == 1 ? 256 : 64 * WPU) void haar_fwd_kernel(const XT *__restrict__ x,
                                                       float *__restrict__ coef,
                                                       float *__restrict__ norm_part,
                                                       float *__restrict__ max_part, Geo g,
                                                       StripMap m, int C, int Cg, int B,
                                                       SelectPrep prep,
                                                       const float *__restrict__ wdw, int split) {
  constexpr int NS = slot_count(D, V);
  fetch_args(x, m.units, prep.alpha_in);
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int unit = WPU > 1 ? (int)blockIdx.x : (int)blockIdx.x * 4 + wv;
  constexpr bool kSplit = STORE && WPU == 1;
  const int plane = blockIdx.y, b = blockIdx.z;
  const int grp = kSplit ? plane / split : plane;
  // one workgroup per sample clears the state of the selection that follows this kernel
  if (blockIdx.x == 0 && plane == 0) prep_sample(prep, b, threadIdx.x, blockDim.x);
  LanePos<D> p;
  int row0, col0;
  locate<D, V>(m, g, unit, p, row0, col0);
  (void)coef;
  int c0 = grp * Cg, c1 = min(C, c0 + Cg);
  if constexpr (WPU > 1 || kSplit) {
    const int parts = kSplit ? split : WPU, part = kSplit ? plane - grp * split : wv;
    const int Cw = (c1 - c0 + parts - 1) / parts;
    c0 = c0 + part * Cw;
    c1 = min(c1, c0 + Cw);
  }

  FwdSink<D, V, STORE, SQ> sink;
#pragma unroll
  for (int s = 0; s < NS; ++s) sink.acc[s] = 0.f;
  constexpr bool MX = FwdSink<D, V, STORE, SQ>::MX;
  if constexpr (MX) {
#pragma unroll
    for (int s = 0; s < NS; ++s) sink.top[s] = 0.f;
  }

  if (p.active && c0 < c1) {
    const XT *src = x + ((size_t)b * C + c0) * g.N + (size_t)row0 * g.W + col0;
    sink.plane = STORE ? coef + ((size_t)b * C + c0) * g.N : nullptr;
    const int64_t N = g.N;
    if constexpr (DWM == 0) {
      channel_loop<D, V, PF, NT>(src, N, g.W, c1 - c0, p, sink, [N](FwdSink<D, V, STORE, SQ> &sk) {
        if (STORE) sk.plane += N;
      });
    } else {
      const DwLane q = dw_lane<D, V>(g, m, p, row0, col0);
      channel_loop_dw<D, V, DWM == 2, false, NT>(src, wdw + (size_t)c0 * 9, N, c1 - c0, q, p, sink,
                                             [](FwdSink<D, V, STORE, SQ> &) {});
    }
  }

  if (norm_part == nullptr) return;
  if constexpr (WPU > 1) {
    // Every wave puts its values down, then adds up (takes the largest of) NS / WPU slots over all
    // waves, in wave order; the first wave collects the results.
    __shared__ float comb[WPU][NS][kWave];
    constexpr int SW = (NS + WPU - 1) / WPU;
    auto meet = [&](float (&v)[NS], auto &&join) {
#pragma unroll
      for (int s = 0; s < NS; ++s) comb[wv][s][lane] = v[s];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < SW; ++i) {
        const int s = wv * SW + i;
        if (s < NS) {
          float r = comb[0][s][lane];
#pragma unroll
          for (int u = 1; u < WPU; ++u) r = join(r, comb[u][s][lane]);
          comb[0][s][lane] = r;
        }
      }
      __syncthreads();
      if (wv == 0) {
#pragma unroll
        for (int s = 0; s < NS; ++s) v[s] = comb[0][s][lane];
      }
    };
    meet(sink.acc, [](float a, float c) { return a + c; });
    if constexpr (MX) {
      if (max_part != nullptr) {  // (uniform over the grid)
        __syncthreads();
        meet(sink.top, [](float a, float c) { return fmaxf(a, c); });
      }
    }
    if (wv > 0) return;
  }
  if (!p.active) return;
  write_slots<D, V>(norm_part + ((size_t)plane * B + b) * g.N, sink.acc, p);
  if constexpr (MX) {
    if (max_part != nullptr) write_slots<D, V>(max_part + ((size_t)plane * B + b) * g.N, sink.top, p);
  }
}

// ---- small helpers ----------------------------------------------------------------------------
// norm[i] = sum_g sum_u part[g][u][i], the parts of a group first, then the groups, both in increasing
// order: the order in which the norm-only pass (waves of a unit in LDS) and the selection (groups) add,
// so that the two ways to a layer's norms agree bit for bit.
__global__ __launch_bounds__(256) void norm_reduce_kernel(const float *__restrict__ part, int G, int split,
                                                          int64_t BN4, float4 *__restrict__ norm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= BN4) return;
  const float4 *p = reinterpret_cast<const float4 *>(part) + i;
  const int planes = G * split;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f), r = s;  // (0 + a sum of |values| is that sum)
  int left = split;
  for (int p0 = 0; p0 < planes; p0 += 8) {  // eight loads in flight (past the last plane: it again, unused)
    float4 t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = p[(int64_t)min(p0 + u, planes - 1) * BN4];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (p0 + u >= planes) break;
      r.x += t[u].x; r.y += t[u].y; r.z += t[u].z; r.w += t[u].w;
      if (--left == 0) {
        s.x += r.x; s.y += r.y; s.z += r.z; s.w += r.w;
        r = make_float4(0.f, 0.f, 0.f, 0.f);
        left = split;
      }
    }
  }
  norm[i] = s;
}

// norm[b, q] = sum_c |coef[b, c, q]| (SQ: sum_c coef^2), channels in increasing order.
// grid = (ceil(N/4/256), B)
template <bool SQ>
__global__ __launch_bounds__(256) void channel_norm_kernel(const float *__restrict__ coef, int C,
                                                           int64_t N, float *__restrict__ norm) {
  const int64_t i4 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (i4 * 4 >= N) return;
  const float4 *p = reinterpret_cast<const float4 *>(coef + (size_t)b * C * N) + i4;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int c = 0; c < C; ++c) {
    const float4 t = p[(size_t)c * (N / 4)];
    if constexpr (SQ) {
      s.x = fmaf(t.x, t.x, s.x); s.y = fmaf(t.y, t.y, s.y);
      s.z = fmaf(t.z, t.z, s.z); s.w = fmaf(t.w, t.w, s.w);
    } else {
      s.x += fabsf(t.x); s.y += fabsf(t.y); s.z += fabsf(t.z); s.w += fabsf(t.w);
    }
  }
  reinterpret_cast<float4 *>(norm + (size_t)b * N)[i4] = s;
}

// Most waves that can share a strip unit: the registers of a wave (d = 1: 48, 2: 88, 3: 176) times
// their number fit a compute unit's.
template <int D> constexpr int kMaxWpu = D <= 2 ? 16 : D == 3 ? 8 : 4;
inline int max_wpu(int levels) { return levels <= 2 ? 16 : levels == 3 ? 8 : 4; }
struct FwdShape { int G, wpu; };

// x is fp32, or bf16 when the layer's activations are stored that way (fused calls only)
template <int D, int V, bool STORE>
hipError_t fwd_launch(const wcc_desc &d, const void *x, float *coef, float *norm_part,
                      float *max_part, Plan pl, const SelectPrep &prep, const float *wdw, hipStream_t s);

template <int D, int V, bool STORE, class XT>
hipError_t fwd_launch_t(const wcc_desc &d, const XT *x, float *coef, float *norm_part,
                        float *max_part, Plan pl, const SelectPrep &prep, const float *wdw,
                        hipStream_t s) {
  const Geo g{d.H, d.W, d.levels, (int64_t)d.H * d.W};
  const StripMap m = wdw != nullptr ? make_map(d, V) : make_flat_map(d, V);
  const int Cg = (d.C_in + pl.G - 1) / pl.G;
  // one launch: WPU waves a unit, DWM, and the sink's options
  auto go = [&](auto wpu_c, auto dwm_c, auto sq_c, auto nt_c) {
    constexpr int WPU = decltype(wpu_c)::value, DWM = decltype(dwm_c)::value;
    constexpr bool SQ = decltype(sq_c)::value, NT = decltype(nt_c)::value;
    hipLaunchKernelGGL((haar_fwd_kernel<D, V, WPU, STORE, 1, DWM, XT, SQ, NT>),
                       dim3(WPU > 1 ? m.units : (m.units + 3) / 4, pl.G * (WPU > 1 ? 1 : pl.split), d.B),
                       dim3(WPU > 1 ? 64 * WPU : 256), 0, s, x, coef, norm_part, max_part, g, m, d.C_in, Cg, d.B,
                       prep, wdw, pl.split);
    return hipGetLastError();
  };
  // (a prefetch depth of two channels was measured on every workload and never paid)
  using std::integral_constant;
  auto with_waves = [&](auto dwm_c, auto sq_c) {
    constexpr int DWM = decltype(dwm_c)::value;
    auto with_hint = [&](auto nt_c) {
      if (pl.wpu == 1) return go(integral_constant<int, 1>{}, dwm_c, sq_c, nt_c);
      if constexpr (DWM == 0 && kMaxWpu<D> > 4) {
        if (pl.wpu > 4) return go(integral_constant<int, kMaxWpu<D>>{}, dwm_c, sq_c, nt_c);
      }
      return go(integral_constant<int, 4>{}, dwm_c, sq_c, nt_c);
    };
    if constexpr (!STORE) {
      // An input far larger than the memory-side cache is streamed past it.  Where waves share a unit,
      // only if rows are whole 128-byte lines: otherwise the lines at a unit's ends are wanted by two
      // workgroups (layers of 5, 7, 8 x 128 channels of 192 x 640: 209, 263, 295 us with the hint,
      // 213, 270, 302 without; of 5, 6, 7 x 64 of 376 x 760: 417, 506, 560 with, 396, 482, 546 without).
      const bool whole_lines = d.W * (int)sizeof(XT) % 128 == 0;
      if (pl.stream && (pl.wpu == 1 || (DWM == 0 && whole_lines))) return with_hint(std::true_type{});
    }
    return with_hint(std::false_type{});
  };
  auto with_sums = [&](auto dwm_c) {
    if constexpr (!STORE && std::is_same<XT, float>::value) {
      if (d.norm == WCC_NORM_L2) return with_waves(dwm_c, std::true_type{});
    }
    if (d.norm == WCC_NORM_L2) return hipErrorInvalidValue;  // fp32 maps, norm-only pass
    return with_waves(dwm_c, std::false_type{});
  };
  if (wdw != nullptr) {  // K_dw in front of the transform (norm-only pass)
    if constexpr (!STORE && (V == 4 || D == 4))
      return dw_needs_edges(m) ? with_sums(integral_constant<int, 2>{}) : with_sums(integral_constant<int, 1>{});
    return hipErrorInvalidValue;
  }
  return with_sums(integral_constant<int, 0>{});
}

template <int D, int V, bool STORE>
hipError_t fwd_launch(const wcc_desc &d, const void *x, float *coef, float *norm_part,
                      float *max_part, Plan pl, const SelectPrep &prep, const float *wdw, hipStream_t s) {
  if constexpr (!STORE) {
    if (d.act_dtype == WCC_BF16)
      return fwd_launch_t<D, V, STORE>(d, static_cast<const bf16_t *>(x), coef, norm_part, max_part, pl, prep, wdw, s);
  }
  return fwd_launch_t<D, V, STORE>(d, static_cast<const float *>(x), coef, norm_part, max_part, pl, prep, wdw, s);
}

}  // namespace

// How the norm pass cuts a layer: wpu waves a strip unit and G channel groups (see the kernel).
// About a thousand waves stream best, four thousand at d = 1, where a wave has only two rows of a
// channel in flight.  What the strip units of the layer do not give is made up first by waves that
// share a unit, whose sums meet in LDS, then by groups: every group is a plane of partial norms
// (and one of maxima) that is written here and read by one of the selection's kernels, for a
// small map through a single compute unit.  With groups alone and four waves a unit at most the
// 16-layer stack took 852 us (820 now), 4 x 96 channels of 192 x 320 114 us (108), 2 x 144 of
// 100 x 212 50.4 us (44.6), 8 x 128 of 192 x 640 311 us (305).
static FwdShape fwd_shape(const wcc_desc &d, int front) {
  const bool folded = front == kFrontDw;
  if (front != kFrontNone) {
    // K_dw in front: a wave holds two more rows and the taps; groups, and four waves a unit where
    // there are still too few
    const StripMap m = make_map(d, lane_cols(d));
    FwdShape f{groups_for(d, m, d.C_in, front == kFrontChain || arithmetic_bound(d, folded) ? 4096 : 1024, 4), 1};
    if (folded && (int64_t)m.units * d.B * f.G < 1024 && (d.C_in + f.G - 1) / f.G >= 8) f.wpu = 4;
    return f;
  }
  const StripMap m = make_flat_map(d, lane_cols(d));
  const int64_t units = (int64_t)m.units * d.B;
  const int64_t want = d.levels == 1 ? 4096 : 1024;
  FwdShape f{1, 1};
  if (units >= want) return f;  // enough strips: one wave walks all channels of its own
  // (at least two channels a wave)
  const int top = max_wpu(d.levels);
  f.wpu = units * 4 < want && d.C_in >= 2 * top ? top : d.C_in >= 8 ? 4 : 1;
  // (no more groups than a pass without shared units would take: the planes are the caller's memory, and
  // wcc_forward_static's array holds only so many.  Two groups of a few channels on layers that have the
  // strips for a thousand waves cost more than they gave: 4 -> 32 channels, 4 x 512 x 512, d = 1, layer
  // 84.2 -> 79.8 us without; 2 x 16 -> 96 of 436 x 576 90.8 -> 89.3)
  const int most = groups_for(d, make_map(d, lane_cols(d)), d.C_in, 1024, 4);
  while (units * f.wpu * f.G < want && f.G * 2 <= most && d.C_in / (f.G * 2 * f.wpu) >= 2) f.G *= 2;
  return f;
}

int forward_groups(const wcc_desc &d, int front) { return fwd_shape(d, front).G; }

template <bool STORE>
hipError_t fwd_dispatch(const wcc_desc &d, const void *x, float *coef, float *norm_part,
                        float *max_part, Plan pl, const SelectPrep &prep, const float *wdw,
                        hipStream_t s) {
  const bool v4 = lane_cols(d) == 4;
  switch (d.levels) {
    case 1: return v4 ? fwd_launch<1, 4, STORE>(d, x, coef, norm_part, max_part, pl, prep, wdw, s)
                      : fwd_launch<1, 2, STORE>(d, x, coef, norm_part, max_part, pl, prep, wdw, s);
    case 2: return fwd_launch<2, 4, STORE>(d, x, coef, norm_part, max_part, pl, prep, wdw, s);
    case 3: return fwd_launch<3, 4, STORE>(d, x, coef, norm_part, max_part, pl, prep, wdw, s);
    case 4: return fwd_launch<4, 2, STORE>(d, x, coef, norm_part, max_part, pl, prep, wdw, s);
  }
  return hipErrorInvalidValue;
}

static Plan fwd_plan(const wcc_desc &d, int front) {
  const FwdShape f = fwd_shape(d, front);
  return Plan{f.G, f.wpu, streams(d), 1};
}

// The storing pass writes every coefficient: waves that share a unit write 1 KiB pieces of as many planes
// where the waves of a workgroup otherwise write one run of 4 KiB, and sixteen of them on few units keep as
// few compute units busy.  Where that costs more than the waves' sums as planes of their own, the parts of
// a group become launch rows of the same channels, and norm_reduce adds them as the waves would have: the
// norms are those of the norm-only pass bit for bit.  Measured, shared and apart, the sum over the planes
// included (us; in brackets inputs that are in no cache):
//   large maps, planes at most a sixteenth of the channels: 6 x 432 channels of 56 x 504, d = 3, 293 MB, 165 and 154;
//   1 x 1024 of 192 x 256, d = 2, 201 MB, 120 and 88; with more planes 4 x 96 of 384 x 320, 189 MB, 79 and 85;
//   sixteen waves on fewer than 128 units from 32 MB on, planes at most an eighth: 16 x 512 of 64 x 64, d = 2, 134 MB,
//   63 and 52 (136 and 85); 2 x 512 of 128 x 128, 67 MB, 31 and 27 (76 and 45); 2 x 256, 34 MB, 20 and 17 (39 and 30);
//   with more planes 1 x 400 of 100 x 212, 34 MB, 17 and 21 (35 and 34); on more units 2 x 256 of 128 x 128, d = 1,
//   15 and 20 (25 and 31); on smaller maps 2 x 512 of 64 x 64, 17 MB, 13 and 19 (23 and 26).
StorePlan store_plan(const wcc_desc &d, int64_t planes) {
  const FwdShape f = fwd_shape(d, kFrontNone);
  const int64_t bytes = (int64_t)d.B * d.C_in * d.H * d.W * 4, parts = (int64_t)f.G * f.wpu;
  const int64_t shared_wgs = (int64_t)make_flat_map(d, lane_cols(d)).units * d.B * f.G;
  const bool large = bytes > ((int64_t)128 << 20) && parts * 16 <= d.C_in;
  const bool few = f.wpu == 16 && shared_wgs < 128 && bytes >= ((int64_t)32 << 20) && parts * 8 <= d.C_in;
  return StorePlan{f.G, f.wpu > 1 && parts <= planes && (large || few) ? f.wpu : 1};
}

hipError_t launch_haar_fwd(const wcc_desc &d, const float *x, float *coef, float *norm_part, const StorePlan &sp,
                           const SelectPrep &prep, hipStream_t s) {
  Plan pl = fwd_plan(d, kFrontNone);
  if (sp.split > 1) { pl.split = sp.split; pl.wpu = 1; }
  return fwd_dispatch<true>(d, x, coef, norm_part, nullptr, pl, prep, nullptr, s);
}

hipError_t launch_haar_norm(const wcc_desc &d, const void *x, float *norm_part, float *max_part,
                            const SelectPrep &prep, const float *wdw, hipStream_t s) {
  const Plan pl = fwd_plan(d, wdw ? kFrontDw : kFrontNone);
  return fwd_dispatch<false>(d, x, nullptr, norm_part, max_part, pl, prep, wdw, s);
}

hipError_t launch_norm_reduce(const float *norm_part, const StorePlan &sp, int64_t BN, float *norm, hipStream_t s) {
  const int64_t n4 = BN / 4;
  hipLaunchKernelGGL(norm_reduce_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s,
                     norm_part, sp.G, sp.split, n4, reinterpret_cast<float4 *>(norm));
  return hipGetLastError();
}

hipError_t launch_channel_norm(const float *coef, int B, int C, int64_t N, bool squares,
                               float *norm, hipStream_t s) {
  dim3 grid((unsigned)((N / 4 + 255) / 256), B);
  if (squares)
    hipLaunchKernelGGL(channel_norm_kernel<true>, grid, dim3(256), 0, s, coef, C, N, norm);
  else
    hipLaunchKernelGGL(channel_norm_kernel<false>, grid, dim3(256), 0, s, coef, C, N, norm);
  return hipGetLastError();
}

}  // namespace wcc
