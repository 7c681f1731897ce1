// C[T, N] = A[T, K] W[K, N] (+ bias) (+ residual) for few tokens, K <= 1024: a workgroup makes the fp16 operands of its 32 tokens itself,
// in LDS, from row-major activations, from rows that are to be normalised (LayerNorm), or from the partial sums of the FFN core.
// With few tokens every launch of a layer is a chain of latencies of 4 us or more whatever it does, so the launches that pack,
// normalise or add up cost as much as a product.  us, apart / here: pack + 256 x 768 x 576 4.1 + 5.5 / 6.2; LayerNorm + 256 x 768 x 384
// 4.4 + 5.4 / 8.7; two parts + 256 x 384 x 768 4.3 + 5.0 / 7.0; three parts + 2048 x 192 x 768 4.2 + 8.6 / 8.0; row-major 2048 x 768 x 192
// 7.3 / 6.3.  A layer of 256 tokens, width 768: 79 / 73 with three launches less.
//
// One workgroup = 32 tokens x 32 (8 / KW) columns: KW wavefronts share the contraction of a 32-column tile (64-row chunks, two under way
// each; partial tiles added through LDS in a fixed order), the others have columns of their own.  KW is the largest for which
// the workgroups make one round over the compute units (linear_few_plan): the fewer chunks a wavefront has, the shorter its chain.
#include "fsvd_few.h"

namespace fsvd {

namespace {

// column tiles of a group; a fragment-major output is written up to whole chunks of 64 columns
__host__ __device__ inline int tiles_of(int N, int bn, bool fm) { return ((fm ? (N + 63) / 64 * 64 : N) + bn - 1) / bn; }

// sum over the wavefront, in six vector operations
__device__ __forceinline__ float wave_total(float x) {
  auto add = [&](auto ctrl, auto rows) {
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, decltype(rows)::value, 0xf, false));
  };
  add(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});    // row_shr 1, 2, 4, 8
  add(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
  add(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
  add(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
  add(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});    // row_bcast 15, 31
  add(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

__device__ __forceinline__ void widen8(u4 raw, int dt, float (&x)[8]) {
  const f4v lo = dt == DT_BF16 ? raw_to_f4<DT_BF16>(u2{raw[0], raw[1]}) : raw_to_f4<DT_F16>(u2{raw[0], raw[1]});
  const f4v hi = dt == DT_BF16 ? raw_to_f4<DT_BF16>(u2{raw[2], raw[3]}) : raw_to_f4<DT_F16>(u2{raw[2], raw[3]});
#pragma unroll
  for (int e = 0; e < 4; ++e) { x[e] = lo[e]; x[4 + e] = hi[e]; }
}

// row-major 16-bit rows; a wavefront takes every eighth row, all of them requested at once
__device__ __forceinline__ void gather_row(_Float16* act, int kc, const LinearFewArgs& a, int m0, int wave, int lane) {
  u4 x[4][2];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = m0 + wave + 8 * r, k = 8 * (lane + 64 * i);
      x[r][i] = u4{0u, 0u, 0u, 0u};
      if (row < a.T && k < a.K) x[r][i] = *(const u4*)((const uint16_t*)a.A + (size_t)row * a.K + k);
    }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = 8 * (lane + 64 * i);
      const h8 h = a.a_dt == DT_BF16 ? raw_to_h8<DT_BF16>(x[r][i]) : raw_to_h8<DT_F16>(x[r][i]);
      if (k < kc * 64) *(h8*)act_at(act, kc, wave + 8 * r, k) = h;
    }
}
// normalised rows: mean and biased variance of a row are two sums over the wavefront (layernorm_kernel's arithmetic)
__device__ __forceinline__ void gather_ln(_Float16* act, int kc, const LinearFewArgs& a, int m0, bool first, int wave, int lane) {
  float x[4][2][8], gm[2][8], bt[2][8];
  u4 graw[2], braw[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int k = 8 * (lane + 64 * i);
    graw[i] = braw[i] = u4{0u, 0u, 0u, 0u};
    if (k < a.K) { graw[i] = *(const u4*)((const uint16_t*)a.gamma + k); braw[i] = *(const u4*)((const uint16_t*)a.beta + k); }
  }
  if (a.a_dt == DT_F32) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = m0 + wave + 8 * r, k = 8 * (lane + 64 * i);
        f4v lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
        if (row < a.T && k < a.K) {
          const f4v* const p = (const f4v*)((const float*)a.A + (size_t)row * a.K + k);
          lo = p[0];
          hi = p[1];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[r][i][e] = lo[e]; x[r][i][4 + e] = hi[e]; }
      }
  } else {
    u4 raw[4][2];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = m0 + wave + 8 * r, k = 8 * (lane + 64 * i);
        raw[r][i] = u4{0u, 0u, 0u, 0u};
        if (row < a.T && k < a.K) raw[r][i] = *(const u4*)((const uint16_t*)a.A + (size_t)row * a.K + k);
      }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int i = 0; i < 2; ++i) widen8(raw[r][i], a.a_dt, x[r][i]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) { widen8(graw[i], a.p_dt, gm[i]); widen8(braw[i], a.p_dt, bt[i]); }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = m0 + wave + 8 * r;
    float sum = 0.f, sq = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) sum += x[r][i][e];
    const float mean = wave_total(sum) / (float)a.K;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (8 * (lane + 64 * i) < a.K) {
#pragma unroll
        for (int e = 0; e < 8; ++e) { const float d = x[r][i][e] - mean; sq += d * d; }
      }
    const float rstd = rsqrtf(wave_total(sq) / (float)a.K + a.eps);
    if (first && a.stats && lane == 0 && row < a.T) {
      a.stats[2 * row] = mean;
      a.stats[2 * row + 1] = rstd;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = 8 * (lane + 64 * i);
      h8 h;
#pragma unroll
      for (int e = 0; e < 8; ++e) h[e] = (_Float16)((x[r][i][e] - mean) * rstd * gm[i][e] + bt[i][e]);
      if (k < kc * 64) *(h8*)act_at(act, kc, wave + 8 * r, k) = h;               // (past K: zeros)
    }
  }
}
// sums of the FFN core's parts: lane = token, quads of ranks
__device__ __forceinline__ void gather_ffn_parts(_Float16* act, int kc, const LinearFewArgs& a, int m0) {
  const int t = threadIdx.x & 31, tok = m0 + t < a.T ? m0 + t : a.T - 1;        // (clamped rows are never stored)
  const size_t stride = (size_t)kc * 16 * a.T * 4;
  for (int q0 = threadIdx.x >> 5; q0 < kc * 16; q0 += 64) {
    f4v y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) y[u] = f4v{0.f, 0.f, 0.f, 0.f};
    for (int p = 0; p < a.nparts; p += 2) {                                     // in order
      f4v x[2][4];
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = q0 + 16 * u;
          x[e][u] = f4v{0.f, 0.f, 0.f, 0.f};
          if (q < kc * 16 && p + e < a.nparts) x[e][u] = *(const f4v*)(a.part + (p + e) * stride + ((size_t)q * a.T + tok) * 4);
        }
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) y[u][i] += x[e][u][i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = q0 + 16 * u;
      h4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = (_Float16)y[u][i];
      if (q < kc * 16) *(h4*)act_at(act, kc, t, 4 * q) = o;
    }
  }
}

// fragment-major activations: one unit per lane
__device__ __forceinline__ void gather_fm(_Float16* act, int kc, const LinearFewArgs& a, int m0, int wave, int lane) {
  const h8* const p = (const h8*)a.A + (size_t)(m0 >> 5) * kc * 256 + lane;
  for (int i = wave; i < 4 * kc; i += 32) {      // (chunk, step)
    h8 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = p[(i + 8 * u < 4 * kc ? i + 8 * u : i) * 64];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = i + 8 * u;
      if (j < 4 * kc) *(h8*)act_at(act, kc, lane & 31, 64 * (j >> 2) + 32 * (lane >> 5) + 8 * (j & 3)) = x[u];
    }
  }
}

template <int SRC, int WT, int KW>
__global__ void __launch_bounds__(512, 1) linear_few_kernel(LinearFewArgs a, int tiles_n) {
  typedef WeightChunks<WT, 1> Chunks;
  constexpr int CW = 8 / KW, BN = 32 * CW;
  __shared__ __attribute__((aligned(16))) _Float16 act[32 * 1024];
  __shared__ __attribute__((aligned(16))) _Float16 stage[8 * Chunks::kHalves];  // weights, then partial tiles
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  int tn = wg % tiles_n, gi = 0;
  const int m0 = wg / tiles_n * 32;
  const bool first = tn == 0;
  const bool fm = a.c_layout == LAYOUT_FM;
  for (; gi < a.ngroups - 1; ++gi) {
    const int t = tiles_of(a.g[gi].N, BN, fm);
    if (tn < t) break;
    tn -= t;
  }
  const LinearGroup G = a.g[gi];
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cw = wave % CW, kw = wave / CW;
  const int n0 = tn * BN, kch = (a.K + 63) / 64, T = a.T;
  const Chunks wc(G.W, a.K, G.N, G.ldw, n0 + 32 * cw, lane);
  _Float16* const mine = stage + wave * Chunks::kHalves;
  u4 w[2][Chunks::NP];
  wc.load(kw, kch, w[0]);
  wc.load(kw + KW, kch, w[1]);
  if constexpr (SRC == FEW_ROW) gather_row(act, kch, a, m0, wave, lane);
  else if constexpr (SRC == FEW_LN) gather_ln(act, kch, a, m0, first, wave, lane);
  else if constexpr (SRC == FEW_PARTS) gather_ffn_parts(act, kch, a, m0);
  else gather_fm(act, kch, a, m0, wave, lane);
  __syncthreads();
  f16v acc[1] = {zero16()};
  auto chunk = [&](int c, const u4 (&wd)[Chunks::NP]) {
    wc.store(mine, wd);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      acc[0] = mfma32(wc.frag(mine, kk, 0), *(const h8*)act_at(act, kch, l32, 64 * c + 32 * g + 8 * kk), acc[0]);   // rows n, cols tokens
  };
  for (int c = kw; c < kch; c += 2 * KW) {
    chunk(c, w[0]);
    if (c + KW >= kch) break;
    wc.load(c + 2 * KW, kch, w[0]);
    chunk(c + KW, w[1]);
    wc.load(c + 3 * KW, kch, w[1]);
  }
  // ---- quads (4 output columns x 64 lanes): KW > 1: 4 CW of them, dealt to the wavefronts; else the wavefront's own four
  f4v* const red = (f4v*)stage;
  if constexpr (KW > 1) {
    __syncthreads();
    put_partials<1>(red, wave, lane, acc);
    __syncthreads();
  }
  constexpr int QW = KW == 1 ? 4 : (4 * CW + 7) / 8;
  const int tok = m0 + l32;
#pragma unroll
  for (int i = 0; i < QW; ++i) {
    const int qd = KW == 1 ? 4 * cw + i : wave * QW + i, col = qd >> 2, jj = qd & 3;
    if (KW == 8 && qd >= 4) break;
    f4v x;
    if constexpr (KW == 1) x = f4v{acc[0][4 * i], acc[0][4 * i + 1], acc[0][4 * i + 2], acc[0][4 * i + 3]};
    else x = sum_partials<1, KW, CW>(red, col, jj, lane);
    const int n = n0 + 32 * col + 8 * jj + 4 * g;
    if (tok >= T) continue;
    if (n < G.N) {
      if (G.bias) {
        const f4v b = load4(G.bias, n, a.w_dt);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] += b[e];
      }
      if (a.R) {
        f4v r = load4(a.R, (size_t)tok * a.ldr + n, a.r_dt);
        if (a.r_stats) {
          const float mean = a.r_stats[2 * tok], rstd = a.r_stats[2 * tok + 1];
          const f4v gm = load4(a.gamma, n, a.p_dt), bt = load4(a.beta, n, a.p_dt);
#pragma unroll
          for (int e = 0; e < 4; ++e) r[e] = (r[e] - mean) * rstd * gm[e] + bt[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] += r[e];
      }
    }
    if (!fm) {
      if (n < G.N) store4(G.C, (size_t)tok * G.ldc + n, x, a.c_dt);
    } else {
      const int nch = (G.N + 63) / 64;
      if (n < nch * 64) {                        // columns N .. 64 nch - 1 are zeros (their weights are)
        const size_t unit = ((size_t)((tok >> 5) * nch + (n >> 6)) * 4 + ((n >> 3) & 3)) * 64 + ((n >> 5) & 1) * 32 + (tok & 31);
        h4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (_Float16)x[e];
        *(h4*)((_Float16*)G.C + unit * 8 + 4 * g) = o;
      }
    }
  }
}

template <int SRC, int WT>
hipError_t launch_kw(const LinearFewArgs& a, int kw, hipStream_t s) {
  LinearFewArgs b = a;
  int tiles = 0;
  for (int i = 0; i < a.ngroups; ++i) tiles += tiles_of(a.g[i].N, 256 / kw, a.c_layout == LAYOUT_FM);
  const dim3 grid((a.T + 31) / 32 * tiles), block(512);
  if (kw == 8) hipLaunchKernelGGL((linear_few_kernel<SRC, WT, 8>), grid, block, 0, s, b, tiles);
  else if (kw == 4) hipLaunchKernelGGL((linear_few_kernel<SRC, WT, 4>), grid, block, 0, s, b, tiles);
  else if (kw == 2) hipLaunchKernelGGL((linear_few_kernel<SRC, WT, 2>), grid, block, 0, s, b, tiles);
  else hipLaunchKernelGGL((linear_few_kernel<SRC, WT, 1>), grid, block, 0, s, b, tiles);
  return hipGetLastError();
}
template <int SRC>
hipError_t launch_src(const LinearFewArgs& a, int kw, hipStream_t s) {
  if (a.w_tiled) return launch_kw<SRC, kWtTiled>(a, kw, s);
  return a.w_dt == DT_F16 ? launch_kw<SRC, DT_F16>(a, kw, s) : launch_kw<SRC, DT_BF16>(a, kw, s);
}

}  // namespace

int linear_few_plan(int T, int K, int ngroups, const int* N) {
  if (K > 1024) return 0;
  for (int kw = 8; kw >= 1; kw /= 2) {
    long wgs = 0;
    for (int i = 0; i < ngroups; ++i) wgs += tiles_of(N[i], 256 / kw, true);
    if (kw > 1 && kw * 32 >= K) continue;        // no chunk for half of them
    if (wgs * ((T + 31) / 32) <= 256) return kw;
  }
  return 0;
}

// The product itself takes 1 to 4 us longer here than in the general kernels when it is short (gathering rows, two sums per row, code that is
// fetched once), which has to be less than the launch it saves.  Times of whole calls, us, launches apart / here (T, width, rank):
//   packing: from widths of 128 on never more than 1 % slower, up to 5 us faster (width 64: 38.6 / 39.5);
//   LayerNorm, once: 128, 256, 64 38.1 / 41.0 and 20, 256, 32 38.6 / 39.7, but 176, 512, 96 41.4 / 41.0; 1676, 512, 48 75.0 / 72.2;
//   LayerNorm, and again for the residual of the last product: 2, 256, 48 35.8 / 40.5; 48, 768, 16 53.6 / 54.4, but 24, 768, 272
//     63.4 / 62.5; 3452, 256, 272 113.9 / 110.2;
//   nothing saved (row-major input): 6, 256, 48 14.4 / 15.6; 2, 768, 48 20.0 / 20.6, but 3320, 256, 368 37.0 / 32.7; 2048, 768, 192 7.3 / 6.3
//     for the product alone;
//   adding up parts: 512, 512, 32 50.5 / 52.8; 18, 256, 32 38.9 / 39.8, but 176, 512, 96 41.9 / 41.3; 1792, 768, 160 33.3 / 28.6.
// On 589 layers and feed-forward blocks of 1 to 8192 tokens, widths 64 to 1024, what is taken here is at most 3.6 % slower
// and 470 us faster in all; taking everything that fits would lose 650 us again.
bool linear_few_pays(int use, int T, int K, int rank) {
  switch (use) {
    case FEW_FOR_PACK: return K >= 128;
    case FEW_FOR_NORM: return K >= 512 || (K >= 256 && T >= 1024);
    case FEW_FOR_NORM_TWICE: return (K >= 768 && rank > 64) || (K >= 256 && T >= 1024);
    case FEW_FOR_NOTHING: return (K >= 512 && T > 32) || (K >= 256 && T >= 2048);
    case FEW_FOR_PARTS: return rank > 64 || T > 1024;
  }
  return false;
}

hipError_t launch_linear_few(const LinearFewArgs& a, hipStream_t s) {
  int N[3] = {};
  for (int i = 0; i < a.ngroups; ++i) N[i] = a.g[i].N;
  const int kw = linear_few_plan(a.T, a.K, a.ngroups, N);
  if (kw == 0) return hipErrorInvalidValue;
  if (a.src == FEW_ROW) return launch_src<FEW_ROW>(a, kw, s);
  if (a.src == FEW_LN) return launch_src<FEW_LN>(a, kw, s);
  if (a.src == FEW_PARTS) return launch_src<FEW_PARTS>(a, kw, s);
  return launch_src<FEW_FM>(a, kw, s);
}

}  // namespace fsvd
