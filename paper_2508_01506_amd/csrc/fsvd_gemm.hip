// C[T, N] = A[T, K] W[K, N] (+ bias) (+ residual): the rank projections P_a = X U_a, the factored
// output projection (C U_o) V_o + b_o and the two GEMMs that bracket the fused FFN kernel
// (Alg. 2 "GEMM 1st" / "GEMM 2nd").
//
// One workgroup = 4 wavefronts stacked along the rows: a 256 x BN output tile, each wavefront a
// 64 x BN slab held as 32x32 MFMA accumulators.  Activation operands go from global memory straight
// into registers (no other wavefront needs them); in the fragment-major layout that is one
// contiguous 1 KiB load per operand.  Weight tiles are copied row by row into a double-buffered LDS
// tile and read back with the LDS's transposing read by all four wavefronts: 0.5 KiB per MFMA.
// A fragment-major output is produced with the operand roles swapped (rows = output columns,
// lanes = tokens), so that each lane owns 4 consecutive output columns of one token and a wavefront
// writes contiguous 512-byte runs of the destination layout.
#include "fsvd_linear.h"

#include <type_traits>

namespace fsvd {

// Narrow tiles when the wide ones would leave compute units idle or unevenly loaded (two wide or four narrow workgroups fit on a
// compute unit).  With a long contraction the wide ones win from one per compute unit on: they read the activations half as often,
// and starting and ending a tile no longer counts (us, narrow / wide: 4096 x 4096 x 3072, 384 wide tiles, 115 / 109; x 2048, 256:
// 78 / 70; x 1024, 128: 46 / 60; but 16384 x 1024 x 768, 384: 33 / 35; 8192 x 768 x 1152, 288: 25 / 29).  Unless their last columns are
// padding and narrow ones would make no more than two a compute unit: 22398 x 3312 x 288, 264 wide, 440 narrow tiles: 112 / 147;
// 14166 x 2528 x 3 x 192, 336, 504: 46 / 66; 5057 x 3360 x 1584, 260, 500: 73 / 87 (52 products of up to 512 narrow tiles: wide 4 % slower
// on average, up to 41; 188 of 513 to 610: 15 % faster).
bool linear_narrow_tiles(long wide, long narrow, int K) {
  return wide < 512 && !(K >= 2048 && (narrow > 512 || (narrow == 512 && wide == 256)));
}

namespace {

template <int AM, int WT, int BN, int CM, int KS>
__global__ void __launch_bounds__(256 * KS, (AM == AM_ROW_F32) ? 1 : 2) linear_kernel(LinearArgs a, int tiles_m, int tiles_n) {
  constexpr int NT = BN / 32;            // 32-column MFMA tiles per wavefront
  constexpr int ESZ = (AM == AM_ROW_F32) ? 4 : 2;
  // Fragment-major activations: a request is a whole contiguous KiB, and the requests keep the order that the loop below gives them.
  // Row-major ones: a lane's four pieces of a chunk are one run of 64 bytes, and with products and weight requests between
  // them the line has left the L1 before the last piece is asked for, so the compiler is left free to put them together
  // (us, kept in order / free; T x K x N, row-major fp16 weights: 11268 x 848 x 400 58 / 47; 4096 x 1024 x 4096 60 / 53; 16384 x 256 x 1024
  // 26.4 / 24.6).
  constexpr bool kOrdered = AM == AM_FM;
  constexpr int WS = wtile_stride(BN);   // halves per LDS tile row
  constexpr int LPR = BN / 8;            // lanes per tile row while staging (16 bytes each)
  constexpr int RPP = 256 / LPR;         // tile rows staged per pass
  constexpr int NP = kChunkK / RPP;      // passes (loads per thread) per chunk
  // KS = 2: two sets of four wavefronts, each with its own weight buffers, take every second chunk of the contraction
  constexpr int kStage = KS * 2 * kChunkK * WS * 2, kSwap = KS == 2 ? 8 * NT * 4096 : 0;      // bytes: weights; exchange at the end
  __shared__ __attribute__((aligned(16))) char smem[kStage > kSwap ? kStage : kSwap];

  const int tile = xcd_tile(blockIdx.x, tiles_m * tiles_n);
  const int tm = tile / tiles_n;
  int tn = tile % tiles_n;
  int gi = 0;
  for (; gi < a.ngroups - 1; ++gi) {
    int t = (a.g[gi].N + BN - 1) / BN;
    if (tn < t) break;
    tn -= t;
  }
  const LinearGroup G = a.g[gi];
  const int n0 = tn * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);   // wave-uniform
  const int set = KS == 2 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
  const int tid = KS == 2 ? threadIdx.x & 255 : threadIdx.x;
  typedef _Float16 wbuf_t[kChunkK * WS];
  wbuf_t* const lds = (wbuf_t*)smem + 2 * set;
  const int l32 = lane & 31, g = lane >> 5;
  const int m0 = tm * 256 + wave * 64;
  const int K = CM == CM_QKV ? G.K : a.K, T = a.T;
  const void* const A = CM == CM_QKV ? G.A : a.A;
  const int kchunks = (K + kChunkK - 1) / kChunkK;

  // ---- activation addressing: one 32-bit offset per 32-row tile
  const long long a_total = (AM == AM_FM) ? (long long)fm_bytes(T, K) : (long long)T * a.lda * ESZ;
  int voffA[2];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    int r = m0 + 32 * mt + l32;
    if constexpr (AM == AM_FM) {
      voffA[mt] = fm_voff(r, kchunks, g);                 // rows past the last tile fall outside the resource
    } else {
      r = r < T ? r : T - 1;                              // clamped; their results are never stored
      voffA[mt] = (r * a.lda + 32 * g) * ESZ;
    }
  }
  // ---- weight staging: thread -> row s_r (+ RPP per pass), 8 columns from s_c
  const int s_r = tid / LPR, s_c = 8 * (tid % LPR);
  const long long w_total = WT == kWtTiled ? (long long)tiled_bytes(K, G.N) : (long long)K * G.ldw * 2;
  const bool s_ok = n0 + s_c < G.N;
  // prepacked weights (tile images): the column part of this thread's byte offset is fixed (chunks start at multiples
  // of 64 rows and RPP is a multiple of 4, so row % 4 == s_r % 4)
  constexpr int ST = WT == kWtTiled ? DT_F16 : WT;        // type of the values as they arrive for staging
  const int tl_ntn = (G.N + 127) / 128, tl_n = (n0 + s_c) & 127;
  const int tl_col = ((n0 + s_c) >> 7) * kTileImageBytes + ((((tl_n >> 5) ^ (s_r & 3)) << 5) + (tl_n & 31)) * 2;
  const int trA = tr_lane_off(lane, WS) + 32 * g * WS;   // transposing-read base of this lane (halves)

  f16v acc[2][NT];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = zero16();

  RawAct<AM> rawA[2][4];      // [row tile][step]; a slot is refilled right after its last use with the next chunk's data
  u4 w_raw[NP];

  // Operand and weight requests never branch (a conditional request inside the MFMA loop would split it into basic blocks with
  // conservative waits).  Past the last chunk the resources have size 0: activations and weights are zeros.  They have to be: with KS = 2
  // and an odd number of chunks the second set's last step multiplies such a chunk.
  auto load_a = [&](int c, int kk, bool live) {
    const rsrc_t r = rsrc_at(A, live ? a_total : 0, kOrdered ? 0 : (long long)c * kChunkK * ESZ);
    const int kleft = K - c * kChunkK;
    const int soff = kOrdered ? c * kFmChunkBytes : 0;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      if constexpr (AM == AM_FM) {
        rawA[mt][kk].v = buf_load16(r, voffA[mt] + kk * kFmStepBytes, soff);   // the k padding of an FM tensor holds zeros
      } else {
        const int v = (32 * g + 8 * kk < kleft) ? voffA[mt] : kOobOffset;
        if constexpr (AM == AM_ROW_F32) {
          rawA[mt][kk].lo = buf_load16(r, v + kk * 32);
          rawA[mt][kk].hi = buf_load16(r, v + kk * 32 + 16);
        } else {
          rawA[mt][kk].v = buf_load16(r, v + kk * 16);
        }
      }
    }
  };
  // chunk c of the weights: a resource that starts there (row-major; rows past K are out of its range), or an offset (images)
  struct WChunk { rsrc_t r; int soff; };
  auto w_chunk = [&](int c) -> WChunk {
    const bool live = c < kchunks;
    if constexpr (WT == kWtTiled) {
      // chunk c = rows 64 (c % 2) .. of tile row c / 2 (zero-padded past K)
      if constexpr (kOrdered) return WChunk{rsrc_at(G.W, live ? w_total : 0, 0), (c >> 1) * tl_ntn * kTileImageBytes + (c & 1) * (64 * 256)};
      else return WChunk{rsrc_at(G.W, live ? w_total : 0, (long long)(c >> 1) * tl_ntn * kTileImageBytes + (c & 1) * (64 * 256)), 0};
    } else {
      return WChunk{rsrc_at(G.W, live ? w_total : 0, ((long long)c * kChunkK * G.ldw + n0) * 2), 0};
    }
  };
  auto load_w_pass = [&](const WChunk& w, int p, u4 (&dst)[NP]) {
    const int off = WT == kWtTiled ? (s_r + p * RPP) * 256 + tl_col : ((s_r + p * RPP) * G.ldw + s_c) * 2;
    dst[p] = buf_load16(w.r, s_ok ? off : kOobOffset, w.soff);   // rows past K: out of range -> 0
  };
  auto store_w_pass = [&](int buf, int p, const u4 (&src)[NP]) { stage_store16<ST>(&lds[buf][(s_r + p * RPP) * WS + s_c], src[p]); };
  auto bias_f4 = [&](u2 raw) -> f4v {
    if constexpr (WT == kWtTiled) return a.w_dt == DT_BF16 ? raw_to_f4<DT_BF16>(raw) : raw_to_f4<DT_F16>(raw);
    else return raw_to_f4<WT>(raw);
  };
  // prologue: the set's first chunk in LDS and in the operand registers, its second chunk's weights in flight.  Both sets make the
  // same number of steps (barriers), and what a step past the end multiplies is zeros.  Those of fragment-major activations go out in the
  // order in which the loop makes them: the compiler's wait counts hold for both ways into the loop, and with the weights requested
  // last here every chunk waited for all of its successor's operands (rebuild of Q, K and V, 4096 tokens, rank 1024, width 4096: 119 us
  // so, 108 like this).
  const int nsteps = (kchunks + KS - 1) / KS;
  {
    const WChunk w0 = w_chunk(set), w1 = w_chunk(set + KS);
    if constexpr (kOrdered) {
      u4 first[NP];
#pragma unroll
      for (int p = 0; p < NP; ++p) load_w_pass(w0, p, first);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        load_a(set, kk, set < kchunks);
        if ((kk * NP) % 4 == 0) load_w_pass(w1, kk * NP / 4, w_raw);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int p = 0; p < NP; ++p) store_w_pass(0, p, first);
    } else {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) load_a(set, kk, set < kchunks);
#pragma unroll
      for (int p = 0; p < NP; ++p) load_w_pass(w0, p, w_raw);
#pragma unroll
      for (int p = 0; p < NP; ++p) { store_w_pass(0, p, w_raw); load_w_pass(w1, p, w_raw); }
    }
  }
  __syncthreads();
  auto sweep = [&](auto tokrows) {
    constexpr bool TOKROWS = decltype(tokrows)::value;
    constexpr bool kAhead = kOrdered && (CM != CM_QKV || BN == 64);      // (the two loops of CM_QKV leave no registers for it with 128 columns)
    for (int i = 0, c = set; i < nsteps; ++i, c += KS) {
      // the next chunk (requested during the previous iteration) is stored to the other buffer and the one after is requested, one
      // staging pass per MFMA step; the activation operands of a step are refilled with the next chunk's right after their use, and a
      // step's weights are read from LDS before the products of the step before it
      const WChunk w2 = w_chunk(c + 2 * KS);
      const bool more = c + KS < kchunks;
      const _Float16* wt = lds[i & 1];
      auto frag_b = [&](int kk, int nt) {
        const _Float16* q = wt + trA + 8 * kk * WS + 32 * nt;
        return tr_frag(q, q + 4 * WS);
      };
      h8 ahead[2][NT];
      if constexpr (kAhead) {
  #pragma unroll
        for (int nt = 0; nt < NT; ++nt) ahead[0][nt] = frag_b(0, nt);
      }
  #pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        h8 now[NT];
        h8 (&bf)[NT] = kAhead ? ahead[kk & 1] : now;
        if constexpr (!kAhead) {
  #pragma unroll
          for (int nt = 0; nt < NT; ++nt) now[nt] = frag_b(kk, nt);
        } else if (kk < 3) {
  #pragma unroll
          for (int nt = 0; nt < NT; ++nt) ahead[(kk + 1) & 1][nt] = frag_b(kk + 1, nt);
        }
        if constexpr (kOrdered) __builtin_amdgcn_sched_barrier(0);
        h8 af[2];
  #pragma unroll
        for (int mt = 0; mt < 2; ++mt) af[mt] = cvt_raw_act<AM>(rawA[mt][kk]);
  #pragma unroll
        for (int mt = 0; mt < 2; ++mt)
  #pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = TOKROWS ? mfma32(af[mt], bf[nt], acc[mt][nt])     // rows tokens, cols n
                                  : mfma32(bf[nt], af[mt], acc[mt][nt]);    // rows n, cols tokens
        load_a(c + KS, kk, more);
        if ((kk * NP) % 4 == 0) {
          const int p = kk * NP / 4;
          store_w_pass((i + 1) & 1, p, w_raw);
          load_w_pass(w2, p, w_raw);
        }
        if constexpr (kOrdered) __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
    }
  };
  if constexpr (CM == CM_QKV) {
    if (G.v_tiles >= 0) sweep(std::true_type{});
    else sweep(std::false_type{});
  } else {
    sweep(std::false_type{});
  }

  // ---- KS = 2: set 0 finishes the first row tile of every slab, set 1 the second one
  constexpr int MTE = KS == 2 ? 1 : 2;          // row tiles finished by a wavefront, kept in acc[0 .. MTE - 1]
  if constexpr (KS == 2) {
    f4v* const xb = (f4v*)smem + (size_t)wave * (NT * 256) + lane;      // [set][wavefront][column tile][quad][lane]
    __syncthreads();
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        f4v x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = set ? acc[0][nt][4 * qd + e] : acc[1][nt][4 * qd + e];
        xb[set * (4 * NT * 256) + (nt * 4 + qd) * 64] = x;
      }
    __syncthreads();
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const f4v x = xb[(1 - set) * (4 * NT * 256) + (nt * 4 + qd) * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0][nt][4 * qd + e] = (set ? acc[1][nt][4 * qd + e] : acc[0][nt][4 * qd + e]) + x[e];
      }
  }
  const int mrow = m0 + (KS == 2 ? 32 * set : 0);

  // ---- epilogue
  if (CM == CM_QKV && G.v_tiles >= 0) {
    // V^T in operand order: accumulator registers 8 t .. 8 t + 7 of lane (column l32) are the tokens that contraction step t of
    // the context product takes from lane group g, so they are one 16-byte unit of [token tile][32 columns][t][lane]
    const rsrc_t rB = rsrc_at(G.bias, G.bias ? (long long)G.N * 2 : 0, 0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int nb = n0 + 32 * nt;
      if (nb >= G.N) continue;
      const f4v b4 = bias_f4(buf_load8(rB, ((nb + l32) & ~3) * 2));
      const float bias = (l32 & 2) ? ((l32 & 1) ? b4[3] : b4[2]) : ((l32 & 1) ? b4[1] : b4[0]);
#pragma unroll
      for (int mt = 0; mt < MTE; ++mt) {
        const int tt = (mrow >> 5) + mt;
        if (32 * tt >= T) continue;
        char* const base = (tt < G.v_tiles ? (char*)G.C + (size_t)tt * G.N * 64 : (char*)G.C2 + (size_t)(tt - G.v_tiles) * G.N * 64) + nb * 64;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          h8 o;
#pragma unroll
          for (int i = 0; i < 8; ++i) o[i] = (_Float16)(acc[mt][nt][8 * t + i] + bias);
          *(h8*)(base + t * 1024 + lane * 16) = o;
        }
      }
    }
  } else if constexpr (CM != CM_ROW) {
    // lane = token, registers = 4 consecutive output columns: 8-byte stores into the fragment-major output
    const int nch = (G.N + 63) / 64;
    const rsrc_t rB = rsrc_at(G.bias, G.bias ? (long long)G.N * 2 : 0, 0);
    _Float16* C = (_Float16*)G.C;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int n = n0 + 32 * nt + 8 * jj + 4 * g;   // first of 4 columns
        if (n >= nch * 64) continue;                   // columns N .. 64*nch-1 are written as zeros (FM padding)
        const f4v bias = bias_f4(buf_load8(rB, n * 2));
#pragma unroll
        for (int mt = 0; mt < MTE; ++mt) {
          const int tok = mrow + 32 * mt + l32;
          if (tok < T) {
            const size_t unit = ((size_t)((tok >> 5) * nch + (n >> 6)) * 4 + jj) * 64 + ((n >> 5) & 1) * 32 + (tok & 31);
            h4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i)
              o[i] = CM == CM_QKV ? (_Float16)((acc[mt][nt][4 * jj + i] + bias[i]) * G.scale) : (_Float16)(acc[mt][nt][4 * jj + i] + bias[i]);
            *(h4*)(C + unit * 8 + 4 * g) = o;
          }
        }
      }
  } else {
    // row-major output: lane = token, registers = 4 consecutive output columns -> one 16-byte (fp32) or 8-byte store
    const rsrc_t rB = rsrc_at(G.bias, G.bias ? (long long)G.N * 2 : 0, 0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      f4v bias[4];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) bias[jj] = bias_f4(buf_load8(rB, (n0 + 32 * nt + 8 * jj + 4 * g) * 2));   // past N: 0
#pragma unroll
      for (int mt = 0; mt < MTE; ++mt) {
        const int tok = mrow + 32 * mt + l32;
        // all residual values of the tile are requested before the first store: the output may alias the residual
        // (in-place update of the residual stream), so a load placed after a store would have to wait for it
        f4v res[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int n = n0 + 32 * nt + 8 * jj + 4 * g;
          res[jj] = (a.R && tok < T && n < G.N) ? load4(a.R, (size_t)tok * a.ldr + n, a.r_dt) : f4v{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int n = n0 + 32 * nt + 8 * jj + 4 * g;
          if (tok < T && n < G.N) {
            f4v x;
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = acc[mt][nt][4 * jj + i] + bias[jj][i] + res[jj][i];
            store4(G.C, (size_t)tok * G.ldc + n, x, a.c_dt);
          }
        }
      }
    }
  }
}

template <int AM, int WT, int CM>
hipError_t launch_bn(const LinearArgs& a, hipStream_t s) {
  const int tiles_m = (a.T + 255) / 256;
  int n128 = 0, n64 = 0;
  for (int i = 0; i < a.ngroups; ++i) { n128 += (a.g[i].N + 127) / 128; n64 += (a.g[i].N + 63) / 64; }
  if (linear_narrow_tiles((long)tiles_m * n128, (long)tiles_m * n64, a.K)) {
    if constexpr (AM == AM_FM && CM == CM_FM) {
      if (linear_two_sets(a)) {
        hipLaunchKernelGGL((linear_kernel<AM, WT, 64, CM, 2>), dim3(tiles_m * n64), dim3(512), 0, s, a, tiles_m, n64);
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((linear_kernel<AM, WT, 64, CM, 1>), dim3(tiles_m * n64), dim3(256), 0, s, a, tiles_m, n64);
  } else {
    hipLaunchKernelGGL((linear_kernel<AM, WT, 128, CM, 1>), dim3(tiles_m * n128), dim3(256), 0, s, a, tiles_m, n128);
  }
  return hipGetLastError();
}

template <int AM, int WT>
hipError_t launch_c(const LinearArgs& a, hipStream_t s) {
  return a.c_layout == LAYOUT_FM ? launch_bn<AM, WT, CM_FM>(a, s) : launch_bn<AM, WT, CM_ROW>(a, s);
}

template <int WT>
hipError_t launch_a(const LinearArgs& a, hipStream_t s) {
  if (a.a_layout == LAYOUT_FM) return launch_c<AM_FM, WT>(a, s);
  if (a.a_dt == DT_F16) return launch_c<AM_ROW_F16, WT>(a, s);
  if (a.a_dt == DT_BF16) return launch_c<AM_ROW_BF16, WT>(a, s);
  return launch_c<AM_ROW_F32, WT>(a, s);
}

}  // namespace

// At most one workgroup per compute unit: one wavefront per SIMD, which waits for every chunk.  A second set of wavefronts
// takes half of the chunks (us, one set / two: 4096 x 4096 x 1024 56 / 48; 2331 x 2048 x 1008 29 / 24 and x 688 28 / 22;
// 8192 x 768 x 384 14.9 / 13.6).  With two workgroups per unit there is nothing to gain (8192 x 768 x 768 20 / 22;
// 4096 x 4096 x 2048 76 / 82), and a contraction of a few chunks does not pay for adding the halves up.
bool linear_two_sets(const LinearArgs& a) {
  long n64 = 0;
  for (int i = 0; i < a.ngroups; ++i) n64 += (a.g[i].N + 63) / 64;
  return a.a_layout == LAYOUT_FM && a.c_layout == LAYOUT_FM && (a.T + 255) / 256 * n64 <= 256 && (a.K + kChunkK - 1) / kChunkK >= 6;
}

hipError_t launch_rebuild_qkv(const LinearArgs& a, hipStream_t s) {
  if (a.w_tiled) return launch_bn<AM_FM, kWtTiled, CM_QKV>(a, s);
  return a.w_dt == DT_F16 ? launch_bn<AM_FM, DT_F16, CM_QKV>(a, s) : launch_bn<AM_FM, DT_BF16, CM_QKV>(a, s);
}

hipError_t launch_linear(const LinearArgs& a, hipStream_t s) {
  if (linear_kwave_pays(a)) return launch_linear_kwave(a, s);
  if (a.w_tiled) return launch_a<kWtTiled>(a, s);
  return a.w_dt == DT_F16 ? launch_a<DT_F16>(a, s) : launch_a<DT_BF16>(a, s);
}

}  // namespace fsvd
