// What the kernels of the decoding step (fsvd_decode.hip, fsvd_decode_step.hip) share.
#pragma once
#include "fsvd_common.h"
#include "fsvd_kernels.h"

namespace fsvd {

// ---------------------------------------------------------------------------------------------------------------
// How the keys of the B sequences are dealt to the G = B * nsplit workgroups of the pass over the cache.  Sequences
// differ in length, so an equal number of parts per sequence leaves the workgroups of short sequences idle while the
// longest one finishes.  Instead every sequence gets parts in proportion to its tiles of 32 keys: with `tpw` a (nearly)
// smallest number of tiles per workgroup for which sum_b parts_b <= G, parts_b = clamp(ceil(tiles_b / tpw), 1, 32),
// sequence b owns the slots first_b .. first_b + parts_b - 1 (first = exclusive prefix sum) and its part s the tiles
// s * ceil(tiles_b / parts_b) ...  Computed by every wavefront for itself from n_keys (lane = sequence, B <= 64; the
// core and the merge kernel must agree, and both evaluate exactly this function); for B > 64 every sequence has
// nsplit parts.  All 64 lanes must call it; lane b < B receives its sequence's values.
// ---------------------------------------------------------------------------------------------------------------
// inclusive prefix sum over the lanes in six vector operations (no LDS permutes: a dozen sums in a row start every kernel that uses this)
__device__ __forceinline__ int wave_prefix(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8: within 16 lanes
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast 15: rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast 31: rows 2 and 3
  return x;
}
__device__ __forceinline__ int wave_sum(int x) { return __builtin_amdgcn_readlane(wave_prefix(x), 63); }
__device__ __forceinline__ void decode_parts_of_lane(const int32_t* __restrict__ n_keys, int B, int t_max, int nsplit, int lane,
                                                     int& parts, int& first) {
  if (B > 64) {                           // not balanced: caller indexes by sequence
    parts = nsplit;
    first = 0;
    return;
  }
  const int G = B * nsplit;
  int nt = 0;
  if (lane < B) {
    int n = n_keys[lane];
    n = n < 0 ? 0 : (n > t_max ? t_max : n);
    nt = (n + 31) >> 5;
  }
  const int total = wave_sum(nt);
  // ceil(total / (G - B)) tiles per workgroup always fit (sum_b ceil(tiles_b / tpw) <= total / tpw + B <= G; G >= 4 B here);
  // a few smaller values are tried, the smallest that still fits is kept
  auto parts_at = [&](int t) {
    int q = (nt + t - 1) / t;
    q = q < 1 ? 1 : (q > 32 ? 32 : q);
    return lane < B ? q : 0;
  };
  int tpw = (total + (G - B) - 1) / (G - B);
  tpw = tpw < 1 ? 1 : tpw;
  // (seldom more than one or two tries: all eight at once cost 1.4 us more than they save; no more once every sequence has all the
  // parts it can have)
  int p = parts_at(tpw);
  const int most = lane < B ? (nt < 1 ? 1 : (nt > 32 ? 32 : nt)) : 0;
  for (int it = 0; it < 8 && tpw > 1 && __any(p < most); ++it) {
    const int q = parts_at(tpw - 1);
    if (wave_sum(q) > G) break;
    --tpw;
    p = q;
  }
  parts = p;
  first = wave_prefix(p) - p;
}

}  // namespace fsvd
