// Fused FFN core (Alg. 2, the on-chip loops) with wavefront-private weight streams, for prepacked and for row-major weights
// (the latter are instantiated in fsvd_ffn_stream_row.hip):
//   Z[T, r2] = phi(P1[T, r1] V_1[r1, F] + b_1) U_2[F, r2],  hidden activation only on chip.
//
// One workgroup = 32 TT tokens x one slice of 64-rank groups x one part of F; accumulator Z^T in registers over the
// whole sweep, the tokens' P1 operands in LDS (fragment-major, copied as they lie; all of them, or in pieces if r1 is too
// large).  F is swept in chunks of 512 features:
//   phase A  Y^T[512 f, tok] = b_1 + V_1[:, chunk]^T P1^T: wavefront w owns features 64 w .. 64 w + 63 for all tokens;
//   phase B  twice per chunk (first, then second 32 features of every wavefront): phi, fp16, publish 256 features as operands
//            in LDS; Z^T[rank, tok] += U_2[those features, :]^T Y^T, every wavefront its own 64-rank groups.
// Order: A(c), B over the second half of c - 1, B over the first half of c; the activations that the next publish needs are
// evaluated between the products of the B before it (matrix cores and vector unit busy at the same time).
// Every weight element a workgroup uses is used by exactly one of its wavefronts, so the weights need no workgroup
// barrier at all: each wavefront copies its own 64 columns straight into its own LDS ring (four slots of 16 rows x 64
// columns, one slot = one step of 2 TT products), waits for them by its own counter and reads them back with the transposing
// read.  Barriers remain only where the activated features change hands (four per chunk).  A copy moves 8 rows x 128
// bytes: with 64-byte row segments (32 columns per wavefront) the same loads deliver 18 TB/s instead of 30 TB/s.
// When the slice has fewer than eight groups, the sum over the published features is split over KS sets of wavefronts
// and added up through LDS once, at the end of the sweep.
//
// What bounds it: with 64 tokens a step moves 2 KiB per wavefront for 4 products, 64 FLOP per byte out of the L2, which is
// about where copies (30 TB/s) and products meet; on real data the part is at its power limit there (clock 1.9 of 2.4 GHz;
// T 16384, r 256, F 4096: 78 us on random data).  With 32 tokens the copies bind (r1 = r2 = 2048, F 16384, T 4096: 711 .. 770
// us, by the card, for 18 GB out of the L2s; matrix cores busy 38 % of the cycles, wavefronts waiting 37 %).  32 tokens serve
// whatever does not fit at 64: more than 512 output ranks per workgroup without repeating phase A, and token counts that would
// leave compute units idle.  Row-major fp16 weights cost the same (their rows are copied as the image's are, 128 bytes at a
// time); bf16 weights are widened after the LDS read, 12 vector operations per operand (us prepacked / row-major fp16 / bf16:
// r1 = r2 = 688, F 8192, T 2331: 127 / 130 / 149; 2048, 16384, 4096: 711 / 750 / 866).
// Against the kernel with loader wavefronts (fsvd_ffn.hip) see ffn_core_plan().
#include "fsvd_common.h"
#include "fsvd_kernels.h"

#include <type_traits>

namespace fsvd {

namespace {

constexpr int kSF = 512;                       // features per chunk
constexpr int kUnit = 2048;                    // ring slot: 16 contraction rows x 64 columns
constexpr int kRing = 4 * kUnit;               // per wavefront
constexpr int kStreamLds = 160 * 1024;

typedef uint32_t u8v __attribute__((ext_vector_type(8)));

__device__ __forceinline__ void lds_wait_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// WT: kWtTiled, or the storage type (DT_F16, DT_BF16) of row-major weights
template <int TT, int NR, int KS, bool PS, bool ERF, int WT>
__global__ void __launch_bounds__(512, 1) ffn_core_stream_kernel(FfnCoreArgs a, int nslices, int slice_g, int fsplit) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kStreamLds];
  constexpr int kG = TT * 16384;               // activated operands of 256 features
  unsigned char* const gx = smem + 8 * kRing;
  unsigned char* const p1 = gx + kG;           // [token tile][64-rank chunk][step][lane]

  const int tid = threadIdx.x;
  const int lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  const int slice = wg % nslices;
  const int ntile = (a.T + 32 * TT - 1) / (32 * TT);
  const int tb = (wg / nslices) % ntile;
  const int fs = wg / (nslices * ntile);
  const int r1 = a.r1, r2 = a.r2, F = a.F, T = a.T;
  const int nA = (r1 + 63) / 64;               // 64-rank chunks of P1 = blocks of phase A
  const int ptiles = (T + 31) / 32;
  const int ntF = (F + 127) / 128, ntR2 = (r2 + 127) / 128, ng_all = (r2 + 63) / 64;
  const int nch_all = (F + kSF - 1) / kSF;
  const int c_begin = fs * nch_all / fsplit, c_end = (fs + 1) * nch_all / fsplit;

  // ---- this wavefront's rank groups: wavefront wi of the W that share part ks of the features owns groups
  // wr, wr + W of the slice (rotated so that uneven counts add up evenly over the four SIMDs)
  constexpr int W = 8 / KS;
  const int ks = w / W, wi = w % W;
  const int g0 = slice * slice_g;              // even: slices are whole 128-rank tiles
  const int ng = (g0 + slice_g < ng_all) ? slice_g : ng_all - g0;
  const int wr = (wi + ks * (ng % W)) % W;
  bool act[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) act[i] = wr + W * i < ng;
  constexpr int kFSteps = 16 / KS;             // 16-feature steps of a half chunk this wavefront sums over
  constexpr int nB = kFSteps * NR / 4;         // blocks (four ring slots) per half chunk: 2, 4, 8 or 16
  const int f_lo = ks * kFSteps;
  // P1 that does not stay in LDS (PS) is used in pieces of kPC 64-rank chunks.  The workgroups of one XCD sweep the same
  // weights in step, and a line that is not in that XCD's L2 yet costs all of them its latency.  With weights larger than
  // that L2 (which is when PS is used) each workgroup therefore starts its contractions at another place: most of what one
  // asks for has just been fetched for another (decoder shape inside a layer, weights from HBM: 1010 -> 800 us; with the
  // weights in the last-level cache, and for ranks up to 768, no difference).  The order of the fp32 sums depends on the
  // workgroup's index only.
  constexpr int kPC = 8 / TT;
  const int nP = PS ? (nA + kPC - 1) / kPC : 1;
  const int rot = PS ? (blockIdx.x >> 3) & 31 : 0;
  const int rotP = PS ? (rot >> 3) % nP : 0, rotB = rot & (nB - 1);
  const int tail = nA - (nP - 1) * kPC;                  // chunks of the last piece
  auto piece_len = [&](int p) { return !PS ? nA : (p + 1 < nP ? kPC : tail); };
  auto piece_start = [&](int len) { return PS ? rot % kPC < len ? rot % kPC : 0 : 0; };

  // ---- copies of weights into the ring.  Slot row 8 j + s (j = 0, 1: the two copies of a slot) holds contraction rows
  // in the order in which the operands want them: phase A 64 c + 32 j + 8 kk + s (fragment-major steps of P1), phase B
  // 16 f + 4 j + s % 4 + 8 (s / 4) (the order in which the activated accumulators are published).  The two 32-column tiles of
  // a row trade places with bits 0 and 1 of the row, so that four rows of a tile lie in disjoint LDS banks.
  const int s_ = lane >> 3;
  const int cc = ((lane >> 2) & 1) ^ (s_ & 1) ^ ((s_ >> 1) & 1);
  auto lane_seg = [&](int h) { return (((2 * h + cc) ^ (s_ & 3)) << 6) + (lane & 3) * 16; };
  // Row-major weights: the same pieces, addressed by row and column.  Only the per-lane part of an address is checked against the
  // matrix, so the row goes there, and rows past it (rank padding, features >= F) deliver zeros, as the tile images do: P1 may
  // hold anything finite in its padded ranks.  (Offsets stay below 2^32: the matrix is smaller than 1 GiB, and rows are clamped
  // to the first one past it.)  V_1's columns past the matrix are replaced by its last eight (features that are zeroed when they
  // are published), U_2's are zeros: the padded ranks of Z are written.
  constexpr bool kRow = WT != kWtTiled;
  const int col = 32 * cc + 8 * (lane & 3);              // this lane's first column inside the 64
  const int voffA = kRow ? s_ * F * 2 : s_ * 256 + lane_seg(w & 1);
  int voffB[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int rank = 64 * (g0 + wr + W * i) + col;
    const int off = kRow ? ((s_ & 3) + 8 * (s_ >> 2)) * r2 * 2 + rank * 2
                         : ((s_ & 3) + 8 * (s_ >> 2)) * 256 + lane_seg(wr & 1);
    voffB[i] = act[i] && (!kRow || rank < r2) ? off : kOobOffset;
  }
  const u4 rV1 = lds_dma_rsrc(uniform_ptr(a.V1), kRow ? (unsigned)r1 * F * 2 : (unsigned)tiled_bytes(r1, F));
  const u4 rU2 = lds_dma_rsrc(uniform_ptr(a.U2), kRow ? (unsigned)F * r2 * 2 : (unsigned)tiled_bytes(F, r2));
  const unsigned ring0 = lds_addr_of(smem) + w * kRing;
  // Block about to be requested: resource, per-lane offsets, offset of its first slot and the increments of its slots.  The stream
  // is A(c) B1(c - 1) B0(c) for every chunk c (B1 of the chunk before the first one is copied but not used) and B1 of the last chunk
  // (B1, B0: second and first half of a chunk's features).  begin_a / begin_b set the first block of a phase, next_a / next_b step
  // to the one after it; each wavefront runs them once per four steps, between its products, so they are kept to a few scalar
  // operations (with one function that worked every block out from its place in the stream a step had 22 scalar
  // instructions and the decoder shape took 805 us).
  u4 rq_r = rV1;
  int rq_v[NR], rq_off = 0, rq_s1 = 0, rq_s2 = 0, rq_sj = 0;   // rq_off, rq_s*: bytes; rows if the weights are row-major
  int rq_ld = 0, rq_lim = 0;                              // row-major: bytes per row, rows
  int rq_a0 = 0, rq_da = 0;                               // phase A: offset of rank 0 of the chunk's columns; step to the next block
  int nq_p = 0, nq_len = 0, nq_j = 0, nq_n = 0;           // phase A, PS: piece, its length, place, blocks left
  int nq_i = 0, nq_f = 0;                                 // phase B: block; first feature (row-major) or 128-feature tile of the chunk
  int nq_h = 0;                                           // phase B: 32 rows for the second half
  const int spanA = ntF * kTileImageBytes;                // 128 rows of V_1's image
  auto place_a = [&](int ra) { return kRow ? 64 * ra : rq_a0 + (ra >> 1) * spanA + (ra & 1) * 16384; };
  auto begin_a = [&](int c) {
    rq_r = rV1;
    if constexpr (kRow) {
      int f = kSF * c + 64 * w + col;
      f = f < F ? f : F - 8;
#pragma unroll
      for (int i = 0; i < NR; ++i) rq_v[i] = voffA + f * 2;
      rq_s1 = 8; rq_s2 = 16; rq_sj = 32;
      rq_ld = F * 2;
      rq_lim = r1;
    } else {
      int nt = 4 * c + (w >> 1);
      nt = nt < ntF ? nt : ntF - 1;                        // features >= F: any tile, their activations are zeroed
      rq_a0 = nt * kTileImageBytes;
#pragma unroll
      for (int i = 0; i < NR; ++i) rq_v[i] = voffA;
      rq_s1 = 2048; rq_s2 = 4096; rq_sj = 8192 - 1024;     // slots 1, 3 against 0, 2; slots 2, 3 against 0, 1; second copy of a slot (its LDS part is 1024)
    }
    if constexpr (PS) {
      nq_p = rotP;
      nq_n = nq_len = piece_len(nq_p);
      nq_j = piece_start(nq_len);
      rq_off = place_a(nq_p * kPC + nq_j);
    } else {
      rq_off = place_a(0);
      rq_da = 16384;
    }
  };
  auto next_a = [&]() {
    if constexpr (PS) {
      nq_j = nq_j + 1 == nq_len ? 0 : nq_j + 1;
      if (--nq_n == 0) {
        nq_p = nq_p + 1 == nP ? 0 : nq_p + 1;
        nq_n = nq_len = piece_len(nq_p);
        nq_j = piece_start(nq_len);
      }
      rq_off = place_a(nq_p * kPC + nq_j);
    } else if constexpr (kRow) {
      rq_off += 64;
    } else {                                               // blocks alternate between the halves of a tile
      rq_off += rq_da;
      rq_da = spanA - rq_da;
    }
  };
  auto place_b = [&]() {
    const int f0 = f_lo + ((nq_i + rotB) & (nB - 1)) * (4 / NR);   // first 16-feature step of the block
    if constexpr (kRow) {
      rq_off = nq_f + 128 * (f0 >> 2) + 64 * ((f0 >> 1) & 1) + nq_h + 16 * (f0 & 1);
    } else {
      int ft = nq_f + (f0 >> 2);
      ft = ft < ntF ? ft : ntF - 1;
      rq_off = (ft * ntR2 + ((g0 + wr) >> 1)) * kTileImageBytes + (64 * ((f0 >> 1) & 1) + nq_h + 16 * (f0 & 1)) * 256;
    }
  };
  auto begin_b = [&](int c, int half) {
    c = c < c_begin ? c_begin : c;                         // before this workgroup's part: a valid block, multiplied by the zeros in G
    rq_r = rU2;
#pragma unroll
    for (int i = 0; i < NR; ++i) rq_v[i] = voffB[i];
    nq_i = 0;
    nq_h = 32 * half;
    if constexpr (kRow) {
      nq_f = kSF * c;
      rq_s1 = NR == 1 ? 16 : 0; rq_s2 = NR == 1 ? 64 : (NR == 2 ? 16 : 0); rq_sj = 4;
      rq_ld = r2 * 2;
      rq_lim = F;
    } else {
      nq_f = 4 * c;
      rq_s1 = NR == 1 ? 4096 : (W / 2) * kTileImageBytes;
      rq_s2 = NR == 1 ? 16384 : (NR == 2 ? 4096 : W * kTileImageBytes);
      rq_sj = 0;
    }
    place_b();
  };
  auto next_b = [&]() {
    ++nq_i;
    place_b();
  };
  auto request = [&](int u) {                            // slot u of the block that has been set up
    const unsigned dst = ring0 + u * kUnit;
    const int off = rq_off + (u & 1) * rq_s1 + (u >> 1) * rq_s2;
    if constexpr (kRow) {
      const int offj = off + rq_sj;
      const unsigned v = (unsigned)rq_v[u % NR];
      lds_dma16(rq_r, dst, (int)(v + (unsigned)((off < rq_lim ? off : rq_lim) * rq_ld)), 0);
      lds_dma16(rq_r, dst + 1024, (int)(v + (unsigned)((offj < rq_lim ? offj : rq_lim) * rq_ld)), 0);
    } else {
      lds_dma16x2(rq_r, dst, rq_v[u % NR], off, off + rq_sj);
    }
  };

  // ---- operand reads
  const int ri = (lane & 15) >> 2;
  const int tr0 = (8 * g + ri) * 64 + (((ri & 1) ^ (ri >> 1)) << 5) + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);   // halves, column tile 0
  const _Float16* const ringp = (const _Float16*)smem + w * (kRing / 2);
  const _Float16* const rp0 = ringp + tr0;
  const _Float16* const rp1 = ringp + (tr0 ^ 32);
  auto read_w = [&](int u, h8 (&d)[2]) {
    d[0] = tr_frag(rp0 + u * (kUnit / 2), rp0 + u * (kUnit / 2) + 4 * 64);
    d[1] = tr_frag(rp1 + u * (kUnit / 2), rp1 + u * (kUnit / 2) + 4 * 64);
  };
  h8 wf[2][2];                                            // operands of this and the next slot
  // Step u: this slot's operands have been read (a step ago), so its place is refilled with the same slot of the next block; then
  // the next slot has landed and is read.  (Refilled after the products, a slot less is under way while they run.)
  auto step_begin = [&](int u) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    request(u);
    asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    read_w((u + 1) & 3, wf[(u + 1) & 1]);
  };
  // bf16 weights arrive as they are stored and are widened where they are used
  auto widen = [&](h8 x) -> h8 {
    if constexpr (WT == DT_BF16) return raw_to_h8<DT_BF16>(__builtin_bit_cast(u4, x));
    else return x;
  };
  const h8* const p1v = (const h8*)p1;
  const h8* const gv = (const h8*)gx;

  f16v z[NR][2][TT], y[2][TT];
#pragma unroll
  for (int i = 0; i < NR; ++i)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) z[i][c][tt] = zero16();

  // ---- P1.  PS = false: all of it stays in LDS.  PS = true (it does not fit): pieces of kPC 64-rank chunks pass through
  // two buffers of 32 KiB once per chunk of F; piece `pnext` is requested while the one before it is in use.
  const u4 rP = lds_dma_rsrc(uniform_ptr(a.P1), (unsigned)fm_bytes(T, r1));
  const unsigned pl = lds_addr_of(p1);
  int pnext = rotP, pbuf = 0;                              // piece to be requested next; buffer it goes to
  auto request_p = [&](int kk) {                         // four per wavefront and piece
    const int j = kk * 8 + w;                            // 1 KiB: token tile j / (4 kPC), chunk (j / 4) % kPC, step j % 4
    int tile = tb * TT + j / (4 * kPC), ch = pnext * kPC + (j >> 2) % kPC;
    tile = tile < ptiles ? tile : ptiles - 1;            // past the end: anything valid (never used or never written out)
    ch = ch < nA ? ch : nA - 1;
    lds_dma16(rP, pl + pbuf * 32768 + j * 1024, lane * 16, ((tile * nA + ch) * 4 + (j & 3)) * 1024);
  };
  auto piece_requested = [&]() {
    pnext = pnext + 1 < nP ? pnext + 1 : 0;
    pbuf ^= 1;
  };
  {
    if constexpr (PS) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) request_p(kk);
      piece_requested();
    } else {
      for (int i = w; i < TT * nA * 4; i += 8) {         // 1 KiB pieces
        int tile = tb * TT + i / (nA * 4);
        tile = tile < ptiles ? tile : ptiles - 1;
        lds_dma16(rP, pl + i * 1024, lane * 16, (tile * nA * 4 + i % (nA * 4)) * 1024);
      }
    }
    // B1 of the chunk before the first one runs on an empty G: zeros
    for (int i = tid; i < TT * 1024; i += 512) ((u4*)gx)[i] = u4{0u, 0u, 0u, 0u};
    begin_a(c_begin);
#pragma unroll
    for (int u = 0; u < 4; ++u) request(u);
    asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)\n\ts_barrier" ::: "memory");     // P1 (its first piece) and slot 0
  }
  read_w(0, wf[0]);

  auto phi = [&](float x) {
    if constexpr (ERF) return gelu_erf_f(x);
    else return a.act == 1 ? gelu_tanh_f(x) : fmaxf(x, 0.f);
  };

  // Accumulators of phase A start as b_1 of their features.  b_1 comes through the scalar unit (its loads are not counted
  // with the copies), requested ahead of a barrier that is waited for anyway.  Words past F are not used (those features
  // are zeroed when they are published), so addresses are clamped instead of tested.
  const uint32_t bias_on = a.b1 != nullptr ? 0xffffffffu : 0u;
  const char* const bias_p = uniform_ptr(a.b1 != nullptr ? a.b1 : a.V1);
  u8v bwd[2][2];
  auto bias_barrier = [&](int c) {
    const char* p[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int f = c * kSF + 64 * w + 16 * q;
      f = f < F - 16 ? f : F - 16;
      p[q] = bias_p + 2 * f;
    }
    asm volatile("s_load_dwordx8 %0, %4, 0\n\ts_load_dwordx8 %1, %5, 0\n\ts_load_dwordx8 %2, %6, 0\n\ts_load_dwordx8 %3, %7, 0\n\t"
                 "s_waitcnt lgkmcnt(0)\n\ts_barrier"
                 : "=&s"(bwd[0][0]), "=&s"(bwd[0][1]), "=&s"(bwd[1][0]), "=&s"(bwd[1][1])
                 : "s"(p[0]), "s"(p[1]), "s"(p[2]), "s"(p[3]) : "memory");
  };
  auto start_y = [&]() {
    auto fill = [&](auto widen) {
#pragma unroll
      for (int fi = 0; fi < 2; ++fi)
#pragma unroll
        for (int q = 0; q < 8; ++q) {                     // accumulators 2 q, 2 q + 1: features 8 (q / 2) + 4 g + 2 (q % 2) + {0, 1}
          const int d0 = 4 * (q >> 1) + (q & 1);          // word of lanes g = 0; g = 1: two further on
          const uint32_t w0 = bwd[fi][d0 >> 3][d0 & 7], w1 = bwd[fi][d0 >> 3][(d0 & 7) + 2];
          float lo, hi;
          widen((g ? w1 : w0) & bias_on, lo, hi);
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) { y[fi][tt][2 * q] = lo; y[fi][tt][2 * q + 1] = hi; }
        }
    };
    if (a.w_dt == DT_BF16)
      fill([](uint32_t x, float& lo, float& hi) { lo = __uint_as_float(x << 16); hi = __uint_as_float(x & 0xffff0000u); });
    else
      fill([](uint32_t x, float& lo, float& hi) { const h2 p = __builtin_bit_cast(h2, x); lo = (float)p[0]; hi = (float)p[1]; });
  };
  auto phase_a = [&](int c) {
    h8 pf[2][TT];
    const int pstride = PS ? kPC * 256 : nA * 256;                  // between token tiles
    int p = rotP, before = kPC;
    for (int q = 0; q < nP; ++q) {
      const int len = piece_len(p);
      const h8* pbase = p1v + lane;
      if constexpr (PS) {
        // The piece requested last has landed: every wavefront has waited for later copies since, unless the piece before it
        // was a single block.  Everyone has read that piece; its buffer is filled again during this piece's first block.
        if (before < 2) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_wait_barrier();
        pbase += (pbuf ^ 1) * 2048;
      }
      int j = piece_start(len);
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) pf[0][tt] = pbase[tt * pstride + j * 256];
      for (int ab = 0; ab < len; ++ab) {
        if (ab + 1 < len || (PS && q + 1 < nP)) next_a();
        else begin_b(c - 1, 1);
        const h8* const pb = pbase + j * 256;
        j = j + 1 == len ? 0 : j + 1;
        const h8* const pn = pbase + j * 256;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          step_begin(kk);
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) pf[(kk + 1) & 1][tt] = kk < 3 ? pb[tt * pstride + (kk + 1) * 64] : pn[tt * pstride];
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int fi = 0; fi < 2; ++fi) {
            const h8 wv = widen(wf[kk & 1][fi]);
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) y[fi][tt] = mfma32(wv, pf[kk & 1][tt], y[fi][tt]);   // rows features, cols tokens
          }
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (PS) {
            if (ab == 0) request_p(kk);
          }
        }
        if constexpr (PS) {
          if (ab == 0) piece_requested();
        }
      }
      before = len;
      p = p + 1 == nP ? 0 : p + 1;
    }
  };
  // one half of phase B; with ACTIVATE the first two blocks also turn the accumulators yy of the features published next
  // into operands o, two accumulator rows per slot, so that the vector unit works beside the matrix cores
  auto phase_b = [&](auto activate, f16v (&yy)[TT], u4 (&o)[TT][2], auto next_phase) {
    constexpr bool kAct = decltype(activate)::value;
    constexpr int FB = 4 / NR;                                      // feature steps per block
    h8 gf[2][TT];
    int f = f_lo + rotB * FB;
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) gf[0][tt] = gv[(f * TT + tt) * 64 + lane];
    auto block = [&](int b, auto part) {
      constexpr int kPart = decltype(part)::value;
      if (b + 1 < nB) next_b();
      else next_phase();
      const int fn = f_lo + ((b + 1 + rotB) & (nB - 1)) * FB;                      // the next block's first step
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = u % NR, fb = u / NR;
        step_begin(u);
        if (i == 0) {
          const int f2 = fb + 1 < FB ? f + fb + 1 : fn;
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) gf[(fb + 1) & 1][tt] = gv[(f2 * TT + tt) * 64 + lane];
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kPart >= 0) {
          // one activation after every product: about as many cycles of the vector unit as the product takes of the matrix
          // core.  No test for inactive groups here: their weights are zeros (copies out of range).
          constexpr int kBase = 8 * (kPart < 0 ? 0 : kPart);
          const int v = kBase + 2 * u;
          float r[2][TT];
#pragma unroll
          for (int ct = 0; ct < 2; ++ct) {
            const h8 wv = widen(wf[u & 1][ct]);
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
              z[i][ct][tt] = mfma32(wv, gf[fb & 1][tt], z[i][ct][tt]);   // rows ranks, cols tokens
              __builtin_amdgcn_sched_barrier(0);
              r[ct][tt] = phi(yy[tt][v + ct]);
              asm volatile("" : "+v"(r[ct][tt]));
              __builtin_amdgcn_sched_barrier(0);
            }
          }
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) {
            h2 p;
            p[0] = (_Float16)r[0][tt];
            p[1] = (_Float16)r[1][tt];
            o[tt][v >> 3][(v & 7) >> 1] = __builtin_bit_cast(uint32_t, p);
          }
        } else if (act[i]) {
#pragma unroll
          for (int ct = 0; ct < 2; ++ct) {
            const h8 wv = widen(wf[u & 1][ct]);
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) z[i][ct][tt] = mfma32(wv, gf[fb & 1][tt], z[i][ct][tt]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (FB == 1) {
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) gf[0][tt] = gf[1][tt];
      }
      f = fn;
    };
    if constexpr (kAct) {
      block(0, std::integral_constant<int, 0>{});
      block(1, std::integral_constant<int, 1>{});
      for (int b = 2; b < nB; ++b) block(b, std::integral_constant<int, -1>{});
    } else {
      for (int b = 0; b < nB; ++b) block(b, std::integral_constant<int, -1>{});
    }
  };
  // activated features (fp16 operands) -> LDS; features >= F are zeroed here (the weight tiles behind them are others, not zeros)
  auto publish = [&](u4 (&o)[TT][2], int f0, auto first_barrier) {
    if (f0 + 32 > F) {
#pragma unroll
      for (int q = 0; q < 8; ++q)                        // F is a multiple of 16: both halves of a word or none
        if (f0 + 8 * (q >> 1) + 4 * g + 2 * (q & 1) >= F) {
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) o[tt][q >> 2][q & 3] = 0u;
        }
    }
    first_barrier();                                                // everyone has read the previous half
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) ((u4*)gx)[((2 * w + t) * TT + tt) * 64 + lane] = o[tt][t];
    lds_wait_barrier();
  };

  if (c_begin < c_end) {
    u4 o[TT][2];
    bias_barrier(c_begin);
    for (int c = c_begin; c < c_end; ++c) {
      start_y();
      phase_a(c);
      phase_b(std::true_type{}, y[0], o, [&]() { begin_b(c, 0); });                           // second half of c - 1; activates the first half of c
      publish(o, c * kSF + 64 * w, lds_wait_barrier);
      phase_b(std::true_type{}, y[1], o, [&]() {                    // first half of c; activates the second
        if (c + 1 < c_end) begin_a(c + 1);
        else begin_b(c, 1);
      });
      publish(o, c * kSF + 64 * w + 32, [&]() { bias_barrier(c + 1); });
    }
    phase_b(std::false_type{}, y[0], o, []() {});                   // (its last block requests itself again: no loop is left to read it)
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                  // nothing may still be writing LDS

  // ---- add the KS partial sums of a group (fixed order), through LDS
  for (int k = 1; k < KS; ++k) {
    lds_wait_barrier();
    f4v* const xb = (f4v*)smem + (size_t)wr * (NR * 2 * TT * 4 * 64);
    if (ks == k) {
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
          for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              xb[(((i * 2 + ct) * TT + tt) * 4 + j) * 64 + lane] =
                  f4v{z[i][ct][tt][4 * j], z[i][ct][tt][4 * j + 1], z[i][ct][tt][4 * j + 2], z[i][ct][tt][4 * j + 3]};
    }
    lds_wait_barrier();
    if (ks == 0) {
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
          for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const f4v v = xb[(((i * 2 + ct) * TT + tt) * 4 + j) * 64 + lane];
#pragma unroll
              for (int e = 0; e < 4; ++e) z[i][ct][tt][4 * j + e] += v[e];
            }
    }
  }
  if (ks != 0) return;

  // ---- write Z (or this part's fp32 partial sums)
  const int zch = (r2 + 63) / 64;
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    const int tok = (tb * TT + tt) * 32 + l32;
    if (tok >= T) continue;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      if (!act[i]) continue;
      const int gr = g0 + wr + W * i;                    // 64-rank group = chunk of Z
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          if (fsplit == 1) {
            const size_t unit = ((size_t)((tok >> 5) * zch + gr) * 4 + jj) * 64 + ct * 32 + (tok & 31);
            h4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (_Float16)z[i][ct][tt][4 * jj + e];
            *(h4*)((_Float16*)a.Z + unit * 8 + 4 * g) = o;
          } else {
            const int r = 64 * gr + 32 * ct + 8 * jj + 4 * g;
            f4v o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = z[i][ct][tt][4 * jj + e];
            *(f4v*)(a.Zpart + (((size_t)fs * (zch * 16) + (r >> 2)) * T + tok) * 4) = o;
          }
        }
    }
  }
}

template <int TT, int NR, int KS, int WT>
hipError_t launch_weights(const FfnCoreArgs& a, const FfnCorePlan& pl, hipStream_t s) {
  const dim3 grid(((a.T + 32 * TT - 1) / (32 * TT)) * pl.nslices * pl.fsplit), block(512);
  const int sg = pl.slice_w / 64;
  if (ffn_stream_resident(TT, a.r1)) {
    if (a.act == 0) hipLaunchKernelGGL((ffn_core_stream_kernel<TT, NR, KS, false, true, WT>), grid, block, 0, s, a, pl.nslices, sg, pl.fsplit);
    else hipLaunchKernelGGL((ffn_core_stream_kernel<TT, NR, KS, false, false, WT>), grid, block, 0, s, a, pl.nslices, sg, pl.fsplit);
  } else {
    if (a.act == 0) hipLaunchKernelGGL((ffn_core_stream_kernel<TT, NR, KS, true, true, WT>), grid, block, 0, s, a, pl.nslices, sg, pl.fsplit);
    else hipLaunchKernelGGL((ffn_core_stream_kernel<TT, NR, KS, true, false, WT>), grid, block, 0, s, a, pl.nslices, sg, pl.fsplit);
  }
  return hipGetLastError();
}
template <int TT, int NR, int KS>
hipError_t launch_shape(const FfnCoreArgs& a, const FfnCorePlan& pl, hipStream_t s) {
#ifndef FSVD_FFN_STREAM_ROW
  return launch_weights<TT, NR, KS, kWtTiled>(a, pl, s);
#else
  return a.w_dt == DT_F16 ? launch_weights<TT, NR, KS, DT_F16>(a, pl, s) : launch_weights<TT, NR, KS, DT_BF16>(a, pl, s);
#endif
}

}  // namespace

#ifndef FSVD_FFN_STREAM_ROW
bool ffn_stream_resident(int tt, int r1) { return 8 * kRing + tt * 16384 + tt * ((r1 + 63) / 64) * 4096 <= kStreamLds; }

hipError_t launch_ffn_core_stream(const FfnCoreArgs& a, const FfnCorePlan& pl, hipStream_t s) {
  if (!a.tiled) return launch_ffn_core_stream_row(a, pl, s);
#else
hipError_t launch_ffn_core_stream_row(const FfnCoreArgs& a, const FfnCorePlan& pl, hipStream_t s) {
#endif
  switch (pl.stream_tt * 16 + pl.stream_nr * 2 + pl.ks) {
    case 1 * 16 + 1 * 2 + 1: return launch_shape<1, 1, 1>(a, pl, s);
    case 1 * 16 + 1 * 2 + 2: return launch_shape<1, 1, 2>(a, pl, s);
    case 1 * 16 + 2 * 2 + 1: return launch_shape<1, 2, 1>(a, pl, s);
    case 1 * 16 + 2 * 2 + 2: return launch_shape<1, 2, 2>(a, pl, s);
    case 1 * 16 + 4 * 2 + 1: return launch_shape<1, 4, 1>(a, pl, s);
    case 2 * 16 + 1 * 2 + 1: return launch_shape<2, 1, 1>(a, pl, s);
    case 2 * 16 + 1 * 2 + 2: return launch_shape<2, 1, 2>(a, pl, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace fsvd
