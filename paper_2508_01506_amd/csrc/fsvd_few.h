// What the products of few tokens share (fsvd_decode_step.hip, fsvd_gemm_few.hip): activations of 32 tokens as operands in LDS, weights
// through each wavefront's own part of LDS, partial tiles added through LDS.
#pragma once
#include "fsvd_linear.h"

namespace fsvd {

// this wavefront's 64-row chunks of W[K, n0 .. n0 + 32 NT)
template <int WT, int NT>
struct WeightChunks {
  static constexpr int WS = wtile_stride(32 * NT), LPR = 4 * NT, RPP = 64 / LPR, NP = 64 / RPP;
  static constexpr int ST = WT == kWtTiled ? DT_F16 : WT;
  static constexpr int kHalves = kChunkK * WS;   // LDS of one chunk
  const void* W;
  long long total;
  int ldw, n0, ntn, s_r, s_c, tl_col, tr;
  bool ok;
  __device__ __forceinline__ WeightChunks(const void* W_, int K, int N, int ldw_, int n0_, int lane) : W(W_), ldw(ldw_), n0(n0_) {
    s_r = lane / LPR;
    s_c = 8 * (lane % LPR);
    total = WT == kWtTiled ? (long long)tiled_bytes(K, N) : (long long)K * ldw * 2;
    ok = n0 + s_c < N;
    ntn = (N + 127) / 128;
    const int tl_n = (n0 + s_c) & 127;           // tile images: see fsvd_gemm.hip
    tl_col = ((n0 + s_c) >> 7) * kTileImageBytes + ((((tl_n >> 5) ^ (s_r & 3)) << 5) + (tl_n & 31)) * 2;
    tr = tr_lane_off(lane, WS) + 32 * (lane >> 5) * WS;
  }
  // c >= end: zeros (the callers' loops end before they would multiply them)
  __device__ __forceinline__ void load(int c, int end, u4 (&w)[NP]) const {
    if constexpr (WT == kWtTiled) {
      const rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)W, 0, c < end ? (int)total : 0, 0x00020000);
      const int base = (c >> 1) * ntn * kTileImageBytes + (c & 1) * (64 * 256);
#pragma unroll
      for (int p = 0; p < NP; ++p) w[p] = buf_load16(r, ok ? s_r * 256 + tl_col : kOobOffset, base + p * RPP * 256);
    } else {                                     // rows past K: out of range
      const rsrc_t r = rsrc_at(W, c < end ? total : 0, ((long long)c * kChunkK * ldw + n0) * 2);
#pragma unroll
      for (int p = 0; p < NP; ++p) w[p] = buf_load16(r, ok ? ((s_r + p * RPP) * ldw + s_c) * 2 : kOobOffset);
    }
  }
  __device__ __forceinline__ void store(_Float16* mine, const u4 (&w)[NP]) const {
#pragma unroll
    for (int p = 0; p < NP; ++p) stage_store16<ST>(mine + (s_r + p * RPP) * WS + s_c, w[p]);
  }
  __device__ __forceinline__ h8 frag(const _Float16* mine, int kk, int nt) const {
    const _Float16* q = mine + tr + 8 * kk * WS + 32 * nt;
    return tr_frag(q, q + 4 * WS);
  }
};

// activations of up to 32 tokens as operands in LDS: 16-byte units, the unit's place in its row permuted by the row so that the
// eight rows of a phase of the read lie in different banks; `kc` = whole chunks of 64
__device__ __forceinline__ _Float16* act_at(_Float16* tile, int kc, int row, int k) {
  return tile + row * (kc * 64) + ((((k >> 3) ^ (row & 7)) << 3) | (k & 7));
}

// partial tiles of the wavefronts -> sum of one quad (4 output columns x 64 lanes) over `n` of them, `stride` wavefronts apart
template <int NT>
__device__ __forceinline__ void put_partials(f4v* red, int wave, int lane, const f16v (&acc)[NT]) {
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
      red[(wave * 4 * NT + nt * 4 + jj) * 64 + lane] = f4v{acc[nt][4 * jj], acc[nt][4 * jj + 1], acc[nt][4 * jj + 2], acc[nt][4 * jj + 3]};
}
template <int NT, int N, int STRIDE>
__device__ __forceinline__ f4v sum_partials(const f4v* red, int first, int quad, int lane) {
  f4v x = red[(first * 4 * NT + quad) * 64 + lane];
#pragma unroll
  for (int w = 1; w < N; ++w) {
    const f4v y = red[((first + w * STRIDE) * 4 * NT + quad) * 64 + lane];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] += y[e];
  }
  return x;
}

}  // namespace fsvd
