// What the two projection kernels (fsvd_gemm.hip, fsvd_gemm_kwave.hip) share: input and output forms, operand conversion.
#pragma once
#include "fsvd_common.h"
#include "fsvd_kernels.h"

namespace fsvd {

enum : int { AM_ROW_F16 = 0, AM_ROW_BF16 = 1, AM_ROW_F32 = 2, AM_FM = 3 };
// output forms: row-major, fragment-major, or the rebuilt Q | K | V of the attention core (every group with its own A; Q and K
// fragment-major, V transposed in operand order)
enum : int { CM_ROW = 0, CM_FM = 1, CM_QKV = 2 };

template <int AM> struct RawAct { u4 v; };
template <> struct RawAct<AM_ROW_F32> { u4 lo, hi; };

template <int AM>
__device__ __forceinline__ h8 cvt_raw_act(const RawAct<AM>& r) {
  if constexpr (AM == AM_ROW_F32) {
    f4v lo = __builtin_bit_cast(f4v, r.lo), hi = __builtin_bit_cast(f4v, r.hi);
    h8 o;
    o[0] = (_Float16)lo[0]; o[1] = (_Float16)lo[1]; o[2] = (_Float16)lo[2]; o[3] = (_Float16)lo[3];
    o[4] = (_Float16)hi[0]; o[5] = (_Float16)hi[1]; o[6] = (_Float16)hi[2]; o[7] = (_Float16)hi[3];
    return o;
  } else if constexpr (AM == AM_ROW_BF16) {
    return raw_to_h8<DT_BF16>(r.v);
  } else {
    return __builtin_bit_cast(h8, r.v);
  }
}

// the kernel whose wavefronts split the contraction (fsvd_gemm_kwave.hip): whether it is the better one, and its launch
bool linear_kwave_pays(const LinearArgs& a);
hipError_t launch_linear_kwave(const LinearArgs& a, hipStream_t s);

}  // namespace fsvd
