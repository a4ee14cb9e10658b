// Rules of the dispatch that need nothing but a layer's numbers (host code, no HIP).
#pragma once
#include <stdint.h>

#include "wcc.h"

namespace wcc {

// positions that a checked layer keeps: k of Alg. 1
inline int64_t kept_count(const wcc_desc &d) {
  const int64_t N = (int64_t)d.H * d.W;
  return (d.keep_num * N + d.keep_den - 1) / d.keep_den;
}

// Whether the four waves of a workgroup of the inverse share a strip unit (units: those of a plane).  By the count of
// kept positions, not by the row stride of yc, which a layer rounds up: a third kept of 64 x 64 is 1366 positions in rows of
// 1368.
// Sharing takes three quarters of a wave's rank lookups and votes off, which are what a wave starts with; four waves on four
// neighbouring units write runs four times as long, which counts once memory is the bound.  At 1 and 2 levels a strip has
// few slots and sharing measured 0.92..1.27 of the time.
// At 3 levels, apart -> shared: 1x256x128x128 at 1/4 9.8 -> 8.4 us, 1x32x256x512 at 1/4 9.6 -> 7.9, 16x512x64x64 at 1/8
// 34.6 -> 28.5; up to 16 MB of kept values 0.78..1.02 of the time.  From there to 24 MB 0.85..1.01 with up to 512 columns and
// up to 160 MB to be stored (4x96x192x320 at 1/4 25.1 -> 23.1 in the layer), but 39.1 -> 41.2 with 1024 columns and, of 192 MB
// to be stored, 38.8 -> 39.5 and 38.8 -> 40.6 (4x96x256x512 at 1/10 and 1/8); from 24 to 64 MB 1.00..1.12.  Above a third
// kept many units overflow the list and look their ranks up twice: 0.94..1.19; with the residual added sharing pays there
// all the same (8x128x128x128 at 1/2 36.9 -> 34.5, 4x16x192x320 18.0 -> 12.5; at 3/4 38.0 -> 35.0 and 19.2 -> 13.3; all
// kept 0.67..1.01), and from a third on (16x128x128x128, 43 MB, 60.0 -> 55.9; 8x128x192x320, 80 MB, 108.3 -> 109.1).  Below
// 0.71..1.01, at a quarter and more than 24 MB 1.00..1.01, under 8 units (64x64 and smaller) 0.92..1.10.
// At 4 levels the list takes a third workgroup off a compute unit (57 of 160 KiB of LDS), which only the shortest lists make
// good: up to 1/8 kept 0.72..1.00 of the time, at 1/6 0.78..0.97 up to 4 MB but 4x96x96x320 (7.5 MB) 15.0 -> 17.4, at 1/5 and
// above 0.93..1.16, but on planes of half a unit (1024 positions), whose lists are as short, 0.44..0.90 up to a third
// (6x480x16x16 12.4 -> 10.8, 16x256x32x32 20.7 -> 9.3; a whole unit, 8x128x32x64, 11.5 -> 12.0).  With the residual up
// to 1/4 0.72..0.97, then 0.98..1.21 (4x64x256x512 at 1/2 58.8 -> 71.2, at 1/3 58.4 -> 67.0, all kept 68.8 -> 72.2).
inline bool shares_units(const wcc_desc &d, int units, bool residual) {
  if (d.levels < 3 || (residual && units < 8)) return false;
  const int64_t N = (int64_t)d.H * d.W, k = kept_count(d), kept = (int64_t)d.B * d.C_out * k * 4, MB = 1 << 20;
  if (d.levels == 4) {
    if (residual) return k * 4 <= N && kept <= 8 * MB;
    if (kept > 8 * MB) return false;
    return k * 8 <= N || (k * 6 <= N + 5 && kept <= 4 * MB) || (k * 3 <= N + 2 && N <= 1024);
  }
  if (residual && k * 3 >= N) return true;
  const bool long_store = (int64_t)d.B * d.C_out * N > 40 * MB;  // y of more than 160 MB in fp32
  return k * 3 <= N + 2 && kept <= (d.W <= 512 && !long_store ? 24 : 16) * MB;
}

}  // namespace wcc
