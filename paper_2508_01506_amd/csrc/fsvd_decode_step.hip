// The products around the pass over the cache in a decoding step (fsvd_decode.hip): few tokens (one per sequence), so every kernel
// is one chain of latencies - launch, weights, exchange - and the weights' way from memory, and the step is as fast as its launches
// are few and its weights are all under way at once.  Five launches beside the pass itself (project twice):
//   project  x U of q, k and v (and, behind the pass, context U_o): the contraction split over workgroups until the compute units
//            are busy, fp32 partial sums [part][token][column]; whoever needs the product adds the parts up, in order;
//   query    one workgroup per (head, 256 ranks of k): q_h = (p_q V_q + b_q)[head h], then w_h = V_k[:, h] q_h; further workgroups
//            write the new rows of p_k and p_v to the caches;
//   context  one workgroup per (64 columns of a head, some sequences): merges the parts of the pass for its head and sequences
//            (u, rounded to fp16 in LDS as the operand it is) and multiplies by V_v;
//   output   (context U_o) V_o + b_o.
// Instead of nine launches with the append, the query projection, the absorption, the merge and the value product apart (whole step,
// us, nine / six launches; B, cached tokens, width, rank: 1, 3000, 4096, 1024: 73 / 61; 16, 2048 .. 4095: 126 / 107; 32, 1 .. 1023,
// 768, 256: 47 / 37).  Code that a launch runs once is fetched once: 2.5 KiB more of it cost 0.7 us, hence no deeper unrolling.
//
// In every kernel the eight wavefronts of a workgroup take 64-row chunks of the contraction, two under way each: weights to registers,
// through the wavefront's own part of LDS (row by row, read back transposed), partial tiles added through LDS in a fixed order.
#include "fsvd_decode.h"
#include "fsvd_few.h"

namespace fsvd {

namespace {

constexpr float kLog2eS = 1.4426950408889634f;
constexpr int kNT = 2;                           // 64 columns: a workgroup's, or (heads of 128) those of half its wavefronts

__device__ __forceinline__ f4v bias4(const void* b, int n, int dt) {
  return b ? load4(b, (size_t)n, dt) : f4v{0.f, 0.f, 0.f, 0.f};
}

// sum over the parts of 4 consecutive columns
__device__ __forceinline__ f4v sum_parts(const float* p, size_t stride, int ks) {
  f4v x = *(const f4v*)p;
  for (int s = 1; s < ks; ++s) {
    const f4v y = *(const f4v*)(p + s * stride);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] += y[e];
  }
  return x;
}
// rows [m0, m0 + 32) of a product that lies in parts [KS][T][ntot] (columns [0, K), K <= 1024) -> operands, zeros up to a whole chunk.
// A wavefront takes every eighth row and requests 8 to 32 pieces of 256 columns at once: one after the other their latencies made this
// most of the kernel.
template <int KS>
__device__ __forceinline__ void gather_parts_of(_Float16* tile, int kc, const float* part, int T, int ntot, int K, int m0) {
  constexpr int N = KS == 1 ? 8 : 4;             // (at least the 4 pieces of a row)
  const int lane = threadIdx.x & 63;
  const unsigned stride = (unsigned)T * ntot;
  const int rows = T - m0 < 32 ? T - m0 : 32, lq = kc > 8 ? 2 : (kc > 4 ? 1 : 0);            // 1, 2 or 4 pieces a row
  for (int row0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); row0 < rows; row0 += 8 * N >> lq) {
    f4v x[N][KS];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int row = row0 + 8 * (u >> lq), k = 4 * lane + 256 * (u & ((1 << lq) - 1));
      const float* const p = part + (size_t)(m0 + row) * ntot;
#pragma unroll
      for (int t = 0; t < KS; ++t) {
        x[u][t] = f4v{0.f, 0.f, 0.f, 0.f};
        if (row < rows && k < K) x[u][t] = *(const f4v*)(p + t * stride + k);
      }
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int row = row0 + 8 * (u >> lq), k = 4 * lane + 256 * (u & ((1 << lq) - 1));
      f4v y = x[u][0];
#pragma unroll
      for (int t = 1; t < KS; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] += x[u][t][e];
      h4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (_Float16)y[e];
      if (row < rows && k < kc * 64) *(h4*)act_at(tile, kc, row, k) = o;
    }
  }
}
template <int MAX>
__device__ __forceinline__ void gather_parts(_Float16* tile, int kc, const float* part, int ks, int T, int ntot, int K, int m0) {
  if (ks == 1) gather_parts_of<1>(tile, kc, part, T, ntot, K, m0);
  else if (ks == 2) gather_parts_of<2>(tile, kc, part, T, ntot, K, m0);
  else if (MAX == 4 || ks == 4) gather_parts_of<4>(tile, kc, part, T, ntot, K, m0);
  else gather_parts_of<8>(tile, kc, part, T, ntot, K, m0);
}

// ---- project
template <int AM, int WT, int NT>
__global__ void __launch_bounds__(512, 1) decode_project_kernel(DecodeProjectArgs a) {
  typedef WeightChunks<WT, NT> Chunks;
  __shared__ __attribute__((aligned(16))) _Float16 smem[8 * Chunks::kHalves];
  const int mtiles = (a.T + 31) / 32;
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  int tn = wg % a.col_tiles, gi = 0;
  const int tm = wg / a.col_tiles % mtiles, p = wg / a.col_tiles / mtiles;
  for (; gi < a.ngroups - 1; ++gi) {
    const int t = (a.g[gi].N + (32 * NT) - 1) / (32 * NT);
    if (tn < t) break;
    tn -= t;
  }
  const DecodeProjectGroup G = a.g[gi];
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n0 = tn * (32 * NT), m0 = tm * 32, T = a.T, K = a.K;
  const int kch = (K + 63) / 64, c0 = p * kch / a.ks, c1 = (p + 1) * kch / a.ks;
  const Chunks wc(G.W, K, G.N, G.N, n0, lane);
  _Float16* const mine = smem + wave * Chunks::kHalves;
  const int row = m0 + l32 < T ? m0 + l32 : T - 1;             // clamped; their results are never stored
  const int voffA = (row * K + 32 * g) * 2;
  const long long a_total = (long long)T * K * 2;

  f16v acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = zero16();
  u4 w[2][Chunks::NP];
  RawAct<AM> x[2][4];
  auto load = [&](int c, u4 (&wd)[Chunks::NP], RawAct<AM> (&xd)[4]) {
    wc.load(c, c1, wd);
    const rsrc_t r = rsrc_at(a.A, c < c1 ? a_total : 0, (long long)c * kChunkK * 2);
    const int left = K - c * kChunkK;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) xd[kk].v = buf_load16(r, (32 * g + 8 * kk < left ? voffA : kOobOffset) + kk * 16);
  };
  auto chunk = [&](const u4 (&wd)[Chunks::NP], const RawAct<AM> (&xd)[4]) {
    wc.store(mine, wd);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const h8 af = cvt_raw_act<AM>(xd[kk]);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt] = mfma32(wc.frag(mine, kk, nt), af, acc[nt]);     // rows n, cols tokens
    }
  };
  load(c0 + wave, w[0], x[0]);
  load(c0 + wave + 8, w[1], x[1]);
  for (int c = c0 + wave; c < c1; c += 16) {
    chunk(w[0], x[0]);
    load(c + 16, w[0], x[0]);
    if (c + 8 >= c1) break;
    chunk(w[1], x[1]);
    load(c + 24, w[1], x[1]);
  }
  f4v* const red = (f4v*)smem;
  __syncthreads();
  put_partials<NT>(red, wave, lane, acc);
  __syncthreads();
  if (wave >= 4 * NT) return;                                                  // wavefront = quad
  const f4v s = sum_partials<NT, 8, 1>(red, 0, wave, lane);
  const int n = n0 + 32 * (wave >> 2) + 8 * (wave & 3) + 4 * g, tok = m0 + l32;
  if (tok < T && n < G.N) *(f4v*)(a.part + ((size_t)p * T + tok) * a.ntot + G.col0 + n) = s;
}

// ---- query
template <int WT, int DH>
__global__ void __launch_bounds__(512, 1) decode_query_kernel(DecodeQueryArgs a) {
  typedef WeightChunks<WT, kNT> Chunks;
  constexpr int CH = DH / 64, KW = 8 / CH;       // halves of the head's columns; wavefronts that share the contraction
  constexpr int QS = DH + 8;                     // halves per row of the query tile
  __shared__ __attribute__((aligned(16))) _Float16 act[32 * 1024];              // p_q, then the queries
  __shared__ __attribute__((aligned(16))) _Float16 stage[8 * Chunks::kHalves];  // weights, then partial tiles
  const int T = a.B;
  if ((int)blockIdx.x >= a.head_blocks) {        // new rows of the caches, one thread per 8 ranks of p_k, then per rank of p_v
    const int i = ((int)blockIdx.x - a.head_blocks) * 512 + threadIdx.x;
    const int per_seq = a.r_k / 8 + a.r_v;
    if (i >= T * per_seq) return;
    const int b = i / per_seq, j = i % per_seq, t = a.t_len[b];
    if (j == 0) a.n_keys[b] = t + 1;             // the new token is part of its own context
    if (t < 0 || t >= a.t_max) return;
    const size_t stride = (size_t)T * a.ntot;
    const float* const p = a.part + (size_t)b * a.ntot + a.rq;
    if (j < a.r_k / 8) {
      const int rho = 8 * j, kch = (a.r_k + 63) / 64, off = rho & 63;
      const size_t unit = ((size_t)((t >> 5) * kch + (rho >> 6)) * 4 + ((off >> 3) & 3)) * 64 + (off >> 5) * 32 + (t & 31);
      const f4v lo = sum_parts(p + rho, stride, a.ks), hi = sum_parts(p + rho + 4, stride, a.ks);
      h8 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) { o[e] = (_Float16)lo[e]; o[4 + e] = (_Float16)hi[e]; }
      *(h8*)(a.kcache + b * a.k_seq_halves + unit * 8) = o;
    } else {
      const int rho = j - a.r_k / 8, vtl = (a.r_v + 31) / 32, kq = t & 31, o = kq & 15;
      const size_t unit = ((size_t)((t >> 5) * vtl + (rho >> 5)) * 2 + (kq >> 4)) * 64 + ((o >> 2) & 1) * 32 + (rho & 31);
      float s = p[a.r_k + rho];
      for (int q = 1; q < a.ks; ++q) s += p[q * stride + a.r_k + rho];
      a.vcache[b * a.v_seq_halves + unit * 8 + (o & 3) + 4 * (o >> 3)] = (_Float16)s;
    }
    return;
  }
  const int wg = xcd_tile(blockIdx.x, a.head_blocks);
  const int slice = wg % a.nslices, h = wg / a.nslices % a.H, m0 = wg / a.nslices / a.H * 32;
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = wave % CH, kw = wave / CH;
  const int rq = a.rq, D = a.D, kch = (rq + 63) / 64;

  // everything that does not depend on p_q is requested first: all of this wavefront's chunks of V_q and this wavefront's 32 rows of V_k
  const Chunks wc(a.Vq, rq, D, D, h * DH + 64 * half, lane);
  _Float16* const mine = stage + wave * Chunks::kHalves;
  constexpr int PD = 16 / KW;                    // all chunks of a rank up to 1024
  u4 w[PD][Chunks::NP];
#pragma unroll
  for (int i = 0; i < PD; ++i) wc.load(kw + i * KW, kch, w[i]);
  const int tile = 8 * slice + wave, rho = 32 * tile + l32;
  u4 vk[DH / 16];
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) {
    vk[s] = u4{0u, 0u, 0u, 0u};
    if (rho < a.r_k) vk[s] = *(const u4*)((const uint16_t*)a.Vk + (size_t)rho * D + h * DH + 16 * s + 8 * g);
  }
  gather_parts<4>(act, kch, a.part, a.ks, T, a.ntot, rq, m0);
  __syncthreads();
  f16v acc[kNT];
#pragma unroll
  for (int nt = 0; nt < kNT; ++nt) acc[nt] = zero16();
  auto chunk = [&](int c, const u4 (&wd)[Chunks::NP]) {
    wc.store(mine, wd);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const h8 af = *(const h8*)act_at(act, kch, l32, 64 * c + 32 * g + 8 * kk);
#pragma unroll
      for (int nt = 0; nt < kNT; ++nt) acc[nt] = mfma32(wc.frag(mine, kk, nt), af, acc[nt]);
    }
  };
#pragma unroll
  for (int i = 0; i < PD; ++i)
    if (kw + i * KW < kch) chunk(kw + i * KW, w[i]);
  f4v* const red = (f4v*)stage;
  __syncthreads();
  put_partials<kNT>(red, wave, lane, acc);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < CH; ++i) {                 // quad `wave` of column half i
    const f4v s = sum_partials<kNT, KW, CH>(red, i, wave, lane);
    const int n = 64 * i + 32 * (wave >> 2) + 8 * (wave & 3) + 4 * g;
    const f4v b = bias4(a.bq, h * DH + n, a.w_dt);
    h4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (_Float16)(s[e] + b[e]);
    *(h4*)(act + l32 * QS + n) = o;
  }
  __syncthreads();
  if (32 * tile >= a.r_k) return;
  // w_h^T [ranks, tokens] = V_k[ranks, head columns] q_h^T, contiguous along the contraction on both sides
  f16v wacc = zero16();
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) {
    const h8 vf = a.w_dt == DT_BF16 ? raw_to_h8<DT_BF16>(vk[s]) : raw_to_h8<DT_F16>(vk[s]);
    wacc = mfma32(vf, *(const h8*)(act + l32 * QS + 16 * s + 8 * g), wacc);
  }
  const int b = m0 + l32;
  if (b >= T) return;
  const size_t w_seq = (size_t)((a.r_k + 63) / 64) * 2048;                      // halves per sequence
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    const int off = 32 * (tile & 1) + 8 * jj + 4 * g;                           // rank inside the 64-rank chunk
    h4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (_Float16)(wacc[4 * jj + e] * a.qs);
    *(h4*)(a.W + (size_t)b * w_seq + (size_t)(tile >> 1) * 2048 + (((off >> 3) & 3) * 64 + 32 * (off >> 5) + h) * 8 + (off & 7)) = o;
  }
}

// ---- context
constexpr int kSeqs = 16;                        // sequences of a workgroup at most
template <int WT>
__global__ void __launch_bounds__(512, 1) decode_context_kernel(DecodeContextArgs a) {
  typedef WeightChunks<WT, kNT> Chunks;
  __shared__ __attribute__((aligned(16))) _Float16 act[kSeqs * 1024];           // u of this head, rounded: [sequence][rank]
  __shared__ __attribute__((aligned(16))) _Float16 stage[8 * Chunks::kHalves];  // weights, then partial tiles
  __shared__ float wgt[kSeqs][32], inv[kSeqs];
  const int r_v = a.r_v, D = a.D, B = a.B, kch = (r_v + 63) / 64;
  const int tiles = D / 64, wg = xcd_tile(blockIdx.x, gridDim.x);
  const int groups = gridDim.x / tiles;          // (those of one column tile, and the tiles of one head, behind the same L2)
  const int n0 = wg / groups * 64, b0 = wg % groups * a.seqs, h = n0 / (D / a.H);
  const int nb = B - b0 < a.seqs ? B - b0 : a.seqs;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Chunks wc(a.Vv, r_v, D, D, n0, lane);
  _Float16* const mine = stage + wave * Chunks::kHalves;
  u4 w[2][Chunks::NP];
  wc.load(wave, kch, w[0]);
  wc.load(wave + 8, kch, w[1]);

  int parts, first;
  decode_parts_of_lane(a.n_keys, B, a.t_max, a.nsplit, lane, parts, first);
  auto parts_of = [&](int i) { return B > 64 ? a.nsplit : __shfl(parts, b0 + i, 64); };           // of sequence b0 + i
  auto first_of = [&](int i) { return B > 64 ? (b0 + i) * a.nsplit : __shfl(first, b0 + i, 64); };
  // u: 8 ranks per thread and piece; with few pieces up to 4 groups of threads share the parts of one (part s: group s % pg).  The
  // first 8 of a thread's parts are requested ahead of the weights.
  const int octets = kch * 8, pieces = nb * octets;
  const int pg = pieces <= 128 ? 4 : (pieces <= 256 ? 2 : 1);
  const int grp = pg == 4 ? tid >> 7 : (pg == 2 ? tid >> 8 : 0), first_piece = tid & (512 / pg - 1);
  const size_t step = (size_t)32 * r_v;
  int np, rho, seq;
  const _Float16* p;
  auto source = [&](int j) {
    seq = j < pieces ? j / octets : 0;
    rho = 8 * (j - seq * octets);
    np = parts_of(seq);
    p = a.upart + ((size_t)first_of(seq) * 32 + h) * r_v + (rho < r_v ? rho : 0);
  };
  h8 x[8];
  auto request = [&](int s0) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int q = (s0 + s) * pg + grp;
      x[s] = *(const h8*)(p + (size_t)(q < np ? q : 0) * step);
    }
  };
  source(first_piece);
  request(0);
  // weights of the parts: 32 lanes = the parts of one sequence
  {
    const int i = tid >> 5 < nb ? tid >> 5 : 0, s = tid & 31, n = parts_of(i);
    const size_t at = (size_t)(first_of(i) + (s < n ? s : 0)) * 64 + h;
    const float m = a.stats[at], l = s < n ? a.stats[at + 32] : 0.f;
    float top = l > 0.f ? m : -1e30f;
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o, 32));
    const float q = l > 0.f ? l * exp2f(m - top) : 0.f;
    float sum = q;
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 32);
    if (tid >> 5 < nb) {
      wgt[i][s] = q;
      if (s == 0) inv[i] = sum > 0.f ? 1.0f / sum : 0.f;
    }
  }
  __syncthreads();
  // A part without keys has weight 0 and whatever its slot holds is discarded by the select, not multiplied.  Ranks up to the whole
  // chunk are zeros.
  float (*const sums)[512][4] = (float (*)[512][4])stage;                       // [half of the 8 ranks][thread]
  for (int j = first_piece; ; j += 512) {
    float acc[8] = {};
    for (int s0 = 0;; s0 += 8) {
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int t = (s0 + s) * pg + grp;
        const float q = t < np ? wgt[seq][t & 31] : 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += q > 0.f ? q * (float)x[s][e] : 0.f;
      }
      if (!__any((s0 + 8) * pg + grp < np)) break;
      request(s0 + 8);
    }
    if (pg > 1) {
      *(f4v*)sums[0][tid] = f4v{acc[0], acc[1], acc[2], acc[3]};
      *(f4v*)sums[1][tid] = f4v{acc[4], acc[5], acc[6], acc[7]};
      __syncthreads();
      for (int q = 1; grp == 0 && q < pg; ++q) {
        const f4v lo = *(const f4v*)sums[0][tid + q * (512 / pg)], hi = *(const f4v*)sums[1][tid + q * (512 / pg)];
#pragma unroll
        for (int e = 0; e < 4; ++e) { acc[e] += lo[e]; acc[4 + e] += hi[e]; }
      }
    }
    h8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = rho < r_v ? (_Float16)(acc[e] * inv[seq]) : (_Float16)0.0f;
    if (j < pieces && grp == 0) *(h8*)act_at(act, kch, seq, rho) = o;
    if (j - first_piece + 512 >= pieces) break;  // (pg > 1: all pieces are done) the same for the whole workgroup
    source(j + 512);
    request(0);
  }
  __syncthreads();
  f16v acc[kNT];
#pragma unroll
  for (int nt = 0; nt < kNT; ++nt) acc[nt] = zero16();
  const int row = l32 < kSeqs ? l32 : kSeqs - 1;                                // (columns past nb are not stored)
  auto chunk = [&](int c, const u4 (&wd)[Chunks::NP]) {
    wc.store(mine, wd);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const h8 uf = *(const h8*)act_at(act, kch, row, 64 * c + 32 * g + 8 * kk);
#pragma unroll
      for (int nt = 0; nt < kNT; ++nt) acc[nt] = mfma32(wc.frag(mine, kk, nt), uf, acc[nt]);
    }
  };
  if (wave < kch) chunk(wave, w[0]);             // (r_v <= 1024: 16 chunks)
  if (wave + 8 < kch) chunk(wave + 8, w[1]);
  f4v* const red = (f4v*)stage;
  __syncthreads();
  put_partials<kNT>(red, wave, lane, acc);
  __syncthreads();
  const f4v s = sum_partials<kNT, 8, 1>(red, 0, wave, lane);
  const int n = n0 + 32 * (wave >> 2) + 8 * (wave & 3) + 4 * g;
  const f4v b = bias4(a.bv, n, a.w_dt);
  if (l32 < nb) {
    h4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (_Float16)(s[e] + b[e]);
    *(h4*)(a.ctx + (size_t)(b0 + l32) * D + n) = o;
  }
}

// ---- output: 32 columns per workgroup
template <int WT>
__global__ void __launch_bounds__(512, 1) decode_out_kernel(DecodeOutArgs a) {
  typedef WeightChunks<WT, 1> Chunks;
  __shared__ __attribute__((aligned(16))) _Float16 act[32 * 1024];
  __shared__ __attribute__((aligned(16))) _Float16 stage[8 * Chunks::kHalves];
  const int col_tiles = (a.N + 31) / 32, wg = xcd_tile(blockIdx.x, gridDim.x);
  const int n0 = wg % col_tiles * 32, m0 = wg / col_tiles * 32, kch = (a.K + 63) / 64;
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Chunks wc(a.W, a.K, a.N, a.N, n0, lane);
  _Float16* const mine = stage + wave * Chunks::kHalves;
  u4 w[2][Chunks::NP];
  wc.load(wave, kch, w[0]);
  wc.load(wave + 8, kch, w[1]);
  gather_parts<8>(act, kch, a.part, a.ks, a.T, a.K, a.K, m0);
  __syncthreads();
  f16v acc[1] = {zero16()};
  auto chunk = [&](int c, const u4 (&wd)[Chunks::NP]) {
    wc.store(mine, wd);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      acc[0] = mfma32(wc.frag(mine, kk, 0), *(const h8*)act_at(act, kch, l32, 64 * c + 32 * g + 8 * kk), acc[0]);
  };
  if (wave < kch) chunk(wave, w[0]);             // (K <= 1024: 16 chunks)
  if (wave + 8 < kch) chunk(wave + 8, w[1]);
  f4v* const red = (f4v*)stage;
  __syncthreads();
  put_partials<1>(red, wave, lane, acc);
  __syncthreads();
  if (wave >= 4) return;                         // wavefront = quad
  f4v s = sum_partials<1, 8, 1>(red, 0, wave, lane);
  const int n = n0 + 8 * wave + 4 * g, tok = m0 + l32;
  if (tok >= a.T || n >= a.N) return;
  const f4v b = bias4(a.bias, n, a.w_dt);
#pragma unroll
  for (int e = 0; e < 4; ++e) s[e] += b[e];
  store4(a.out, (size_t)tok * a.N + n, s, a.out_dt);
}

template <int AM, int NT>
hipError_t launch_project(DecodeProjectArgs a, hipStream_t s) {
  a.col_tiles = 0;
  for (int i = 0; i < a.ngroups; ++i) a.col_tiles += (a.g[i].N + 32 * NT - 1) / (32 * NT);
  const dim3 grid((a.T + 31) / 32 * a.col_tiles * a.ks);
  if (a.w_tiled) hipLaunchKernelGGL((decode_project_kernel<AM, kWtTiled, NT>), grid, dim3(512), 0, s, a);
  else if (a.w_dt == DT_F16) hipLaunchKernelGGL((decode_project_kernel<AM, DT_F16, NT>), grid, dim3(512), 0, s, a);
  else hipLaunchKernelGGL((decode_project_kernel<AM, DT_BF16, NT>), grid, dim3(512), 0, s, a);
  return hipGetLastError();
}
template <int DH>
hipError_t launch_query(const DecodeQueryArgs& a, dim3 grid, hipStream_t s) {
  if (a.vq_tiled) hipLaunchKernelGGL((decode_query_kernel<kWtTiled, DH>), grid, dim3(512), 0, s, a);
  else if (a.w_dt == DT_F16) hipLaunchKernelGGL((decode_query_kernel<DT_F16, DH>), grid, dim3(512), 0, s, a);
  else hipLaunchKernelGGL((decode_query_kernel<DT_BF16, DH>), grid, dim3(512), 0, s, a);
  return hipGetLastError();
}

}  // namespace

// Up to 64 sequences: with more, every workgroup that needs a product adds up more and more of it, and the projections of
// fsvd_gemm_kwave.hip fill the compute units by themselves.  Ranks of q and of the output up to 1024: the operands of 32 tokens lie in LDS.
bool decode_step_fits(int B, int rq, int ro) { return B <= 64 && rq <= 1024 && ro <= 1024; }

// Parts of a contraction over K for `cols` columns (1, 2, 4 or, for the output's, 8) and the columns of a workgroup.  A part more is
// worth it while wavefronts have several chunks of 64 and compute units are idle, but every workgroup of the consumer reads all parts of
// all its rows: with several sequences 32 columns per workgroup and fewer parts.
DecodeProjectPlan decode_project_plan(int B, int K, int cols, int most) {
  DecodeProjectPlan pl;
  pl.nt = B >= 8 ? 1 : 2;
  const int wgs = (B + 31) / 32 * ((cols + 32 * pl.nt - 1) / (32 * pl.nt));
  pl.ks = 1;
  while (pl.ks < most && pl.ks * 512 < K && 2 * pl.ks * wgs <= 256 && 2 * pl.ks * B <= 64) pl.ks *= 2;
  return pl;
}

hipError_t launch_decode_project(const DecodeProjectArgs& a, hipStream_t s) {
  if (a.nt == 1) return a.a_dt == DT_F16 ? launch_project<AM_ROW_F16, 1>(a, s) : launch_project<AM_ROW_BF16, 1>(a, s);
  return a.a_dt == DT_F16 ? launch_project<AM_ROW_F16, 2>(a, s) : launch_project<AM_ROW_BF16, 2>(a, s);
}

hipError_t launch_decode_query(DecodeQueryArgs a, hipStream_t s) {
  a.nslices = (a.r_k + 255) / 256;
  a.head_blocks = (a.B + 31) / 32 * a.H * a.nslices;
  const int appended = a.B * (a.r_k / 8 + a.r_v);
  const dim3 grid(a.head_blocks + (appended + 511) / 512);
  if (a.rq > 1024 || a.ks > 4) return hipErrorInvalidValue;
  if (a.D / a.H == 64) return launch_query<64>(a, grid, s);
  if (a.D / a.H == 128) return launch_query<128>(a, grid, s);
  return hipErrorInvalidValue;
}

// as many sequences per workgroup as make one round of workgroups over the compute units (more than 64 sequences: as many rounds as it
// takes; whole step, us, merge and value product apart / here: 200 sequences, width 768, rank 256 89 / 72; width 4096, rank 1024, 65, 80 and 200
// sequences 188 / 187, 191 / 193, 249 / 245)
hipError_t launch_decode_context(DecodeContextArgs a, hipStream_t s) {
  if (a.r_v > 1024) return hipErrorInvalidValue;
  const int tiles = a.D / 64;
  int groups = 256 / tiles;
  groups = groups < 1 ? 1 : (groups > a.B ? a.B : groups);
  a.seqs = (a.B + groups - 1) / groups;
  a.seqs = a.seqs > kSeqs ? kSeqs : a.seqs;
  const dim3 grid(tiles * ((a.B + a.seqs - 1) / a.seqs));
  if (a.w_dt == DT_F16) hipLaunchKernelGGL((decode_context_kernel<DT_F16>), grid, dim3(512), 0, s, a);
  else hipLaunchKernelGGL((decode_context_kernel<DT_BF16>), grid, dim3(512), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_decode_out(const DecodeOutArgs& a, hipStream_t s) {
  if (a.K > 1024) return hipErrorInvalidValue;
  const dim3 grid((a.T + 31) / 32 * ((a.N + 31) / 32));
  if (a.w_tiled) hipLaunchKernelGGL((decode_out_kernel<kWtTiled>), grid, dim3(512), 0, s, a);
  else if (a.w_dt == DT_F16) hipLaunchKernelGGL((decode_out_kernel<DT_F16>), grid, dim3(512), 0, s, a);
  else hipLaunchKernelGGL((decode_out_kernel<DT_BF16>), grid, dim3(512), 0, s, a);
  return hipGetLastError();
}

}  // namespace fsvd
