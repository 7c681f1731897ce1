// Up-projection fused with the residual add and the LayerNorm that follows it (the H3 -> H4 and H7 -> H8 hand-offs of
// a post-LN layer):   Y = LN(A W + bias + R),  A [T, K] fragment-major fp16 (rank space), W [K, D] prepacked tile images.
// The paper only notes that the residual add and the normalisation remain once the two blocks are fused; done as
// separate passes they cost a write and a read of the [T, D] fp32 stream each, more than the projection itself when
// the rank is small.  Here one workgroup owns 32 MT tokens and ALL D columns (D <= 1024, D % 256 == 0), so the row
// statistics are available on chip: a wavefront accumulates D / 8 columns for all tokens
// (accumulators: lane = token, registers = columns, as in linear_kernel), per-lane partial sums are combined through LDS,
// and the normalised row is written once - fp32 / 16-bit row-major and / or the fragment-major fp16 copy that feeds the
// next projection.
// Every weight element is used by one wavefront, so the weights need no workgroup barrier: a wavefront copies its own columns of
// the tile images straight into its own LDS ring (slots of 16 contraction rows, the two 8-row groups an MFMA step of the
// fragment-major slot order touches), waits for them by its own counter and reads operands one step ahead of the products.
// The tokens' operands are shared: blocks of 128 ranks in two LDS buffers, one barrier a block.  (With the weights shared
// and a barrier every 16 ranks: 8192 tokens, width 768: rank 768 32.5 against 28.9 us, rank 384 25.0 against 23.6; with 64 tokens per
// workgroup or width 1024 within 2 %.  What remains is the [T, D] traffic at both ends, which no wavefront overlaps with its
// products.)  The main loop has no compiler-tracked vector loads.
// Bias, gamma and beta of a wavefront's columns are staged as floats in LDS before the loop; the 32 x 32 patches of the
// epilogue reuse the weight ring.
#include "fsvd_common.h"
#include "fsvd_kernels.h"

namespace fsvd {

namespace {

// at most n of this wavefront's vector-memory operations outstanding (n a constant after unrolling; other values wait for all)
__device__ __forceinline__ void wait_vm(int n) {
  switch (n) {
    case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
    case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
    case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
    case 8: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
    case 12: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
  }
}

template <int NT, int MT>   // NT = D / 256: 32-column tiles per wavefront; MT: 32-token tiles per workgroup
__global__ void __launch_bounds__(512, 1) linear_ln_kernel(LinearLnArgs a) {
  // Ring slots of a wavefront (NT KiB each), and the blocks of 4 KiB that the epilogue keeps where ring and operands were.  With up to
  // 512 columns (but for 64 tokens of 512) all of it is kept below 80 KiB, so that two workgroups share a compute unit: there is
  // often more than one round of them, and one's [T, D] traffic then overlaps the other's products (us, one / two per unit: width
  // 256, 24000 tokens, rank 192 20.0 / 16.2; width 512, 12000 tokens 20.4 / 16.7).
  constexpr bool kSplit = NT == 2 && MT == 1;       // the second block lies in two places
  constexpr int NB = NT == 4 || kSplit ? 3 : 4;
  constexpr int kRing = NB * NT * 1024;             // bytes per wavefront
  constexpr int NSLOT = NT == 1 ? MT : (NT < 4 ? NT : 3);
  constexpr int kPatch = 32 * 36 * 4;               // the padded fp32 patch
  constexpr int kOwn = kSplit ? 6144 : (NT == 1 ? 5120 : NSLOT * 4096);        // the epilogue's part of a wavefront's share
  static_assert(kOwn >= kPatch, "");
  constexpr int kShare = kRing > kOwn ? kRing : kOwn;                          // per wavefront: ring, then epilogue blocks
  __shared__ __attribute__((aligned(1024))) char wbuf[8 * kShare];
  __shared__ __attribute__((aligned(1024))) h8 abuf[2][MT][8][64];             // [buffer][token tile][step of the block][lane]
  __shared__ float red[8][32 * MT];
  __shared__ __attribute__((aligned(16))) float prm[8][3][32 * NT];            // per wavefront: bias, gamma, beta of its columns

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = a.T, K = a.K, D = a.D;
  const int kch = (K + 63) / 64, nsteps = 4 * kch;
  const int tile0 = blockIdx.x * MT, ntiles = (T + 31) / 32;
  const unsigned lds_a0 = lds_addr_of(&abuf[0][0][0][0]);
  const u4 rW = lds_dma_rsrc(uniform_ptr(a.W), (unsigned)tiled_bytes(K, D));
  const u4 rA = lds_dma_rsrc(uniform_ptr(a.A), (unsigned)fm_bytes(T, K));

  // This wavefront's 32-column tiles.  Copies move whole 256-byte image rows (NT = 4: 128 columns), 128-byte pairs of tiles, or
  // 64-byte single tiles (NT odd), so for NT = 3 the pairs come first: columns 64 w .. of the first 512, then 32 w .. of the last 256.
  const int colw = (NT == 3 ? 64 : 32 * NT) * wave;
  auto col_of = [&](int j) { return NT == 3 && j == 2 ? 512 + 32 * wave : colw + 32 * j; };

  // step s = (chunk c = s / 4, MFMA step kk = s % 4): contraction rows 64 c + 8 kk + {0..7} and 64 c + 32 + 8 kk + {0..7} are rows
  // 0..7 and 8..15 of a slot.  The segments of an image row are permuted by (row % 4); a pair's two tiles additionally trade
  // places with bits 0 and 1 of the row, so that four rows of a tile lie in disjoint banks in every form.
  constexpr int NTD = 2 * NT;                       // 128-column tile images across D
  char* const mine = &wbuf[wave * kShare];
  const unsigned lds_w0 = lds_addr_of(mine);
  const int pr = lane >> 3, pt = ((lane >> 2) & 1) ^ (pr & 1) ^ ((pr >> 1) & 1);
  const int voff4 = (lane >> 4) * 256 + (lane & 15) * 16;                                               // 4 rows of 256 bytes
  const int voff2 = pr * 256 + ((((colw & 127) >> 5) + pt) ^ (pr & 3)) * 64 + (lane & 3) * 16;          // 8 rows of 128
  const int sr = lane >> 2, scol = NT == 3 ? 512 + 32 * wave : colw;
  const int voff1 = (32 * (sr >> 3) + (sr & 7)) * 256 + (((scol & 127) >> 5) ^ (sr & 3)) * 64 + (lane & 3) * 16;   // 16 rows of 64
  // `nq`: the step to be requested next, `base` the offset of its first row; past the end: the last step again (the loop makes
  // nsteps steps, so it is read at most, never multiplied)
  int nq = 0, base = 0;
  auto request = [&](int slot) {
    const unsigned dst = lds_w0 + slot * NT * 1024;
    if constexpr (NT == 4) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {                   // 4 + 4 rows
        const int at = base + wave * kTileImageBytes + 32 * i * 256;
        lds_dma16x2(rW, dst + 2 * i * 1024, voff4, at, at + 4 * 256 - 1024);
      }
    }
    if constexpr (NT == 2 || NT == 3) {
      const int at = base + (colw >> 7) * kTileImageBytes;
      lds_dma16x2(rW, dst, voff2, at, at + 32 * 256 - 1024);
    }
    if constexpr (NT == 1 || NT == 3) lds_dma16(rW, dst + (NT - 1) * 1024, voff1, base + (scol >> 7) * kTileImageBytes);
    if (++nq < nsteps) base += (nq & 3) ? 8 * 256 : ((nq & 7) ? 64 * 256 - 24 * 256 : NTD * kTileImageBytes - 88 * 256);
  };
  // operands of 128 ranks of the tokens: MT requests per wavefront (step `wave` of the block)
  auto request_a = [&](int b) {
    int c = 2 * b + (wave >> 2);
    c = c < kch ? c : kch - 1;                      // second half of the last block, odd number of chunks: past step nsteps - 1, never read
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      int tile = tile0 + mt;
      tile = tile < ntiles ? tile : ntiles - 1;     // token tiles past the end: any valid one (their rows are not stored)
      lds_dma16(rA, lds_a0 + (((b & 1) * MT + mt) * 8 + wave) * 1024, lane * 16, ((tile * kch + c) * 4 + (wave & 3)) * 1024);
    }
  };

  f16v acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[mt][j] = zero16();

  // operand reads of tile j of a slot: 256-byte rows, 128-byte rows of a pair, 64-byte rows of a single tile
  const int ri = (lane & 15) >> 2, rc = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  auto read_w = [&](int slot, h8 (&bf)[NT]) {
    const _Float16* const p = (const _Float16*)(mine + slot * NT * 1024);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      if constexpr (NT == 4) {
        const _Float16* q = p + 8 * g * 128 + tr_lane_off_swz(lane, j);
        bf[j] = tr_frag(q, q + 4 * 128);
      } else if (NT == 1 || j == 2) {
        const _Float16* q = p + j * 512 + (8 * g + ri) * 32 + rc;
        bf[j] = tr_frag(q, q + 4 * 32);
      } else {
        const _Float16* q = p + (8 * g + ri) * 64 + (((ri & 1) ^ (ri >> 1) ^ j) << 5) + rc;
        bf[j] = tr_frag(q, q + 4 * 64);
      }
    }
  };
  auto read_a = [&](int s, h8 (&af)[MT]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) af[mt] = abuf[(s >> 3) & 1][mt][s & 7][lane];
  };

  // the per-column parameters of this wavefront's columns, as floats, where the epilogue reads them with LDS latency
  {
    float* const pw = &prm[wave][0][0];
#pragma unroll
    for (int c = lane; c < 32 * NT; c += 64) {
      const int col = col_of(c >> 5) + (c & 31);
      pw[c] = a.bias ? load_param(a.bias, col, a.w_dt) : 0.f;
      pw[32 * NT + c] = load_param(a.gamma, col, a.p_dt);
      pw[64 * NT + c] = load_param(a.beta, col, a.p_dt);
    }
  }

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the parameters: from here on the counter is the copies'
  request_a(0);
#pragma unroll
  for (int i = 0; i < NB; ++i) request(i);
  lds_dma_wait_barrier<(NB - 1) * NT>();             // everybody's share of block 0, this wavefront's slot 0
  if (nsteps > 8) request_a(1);
  h8 bf[2][NT], af[2][MT];
  read_w(0, bf[0]);
  read_a(0, af[0]);
  int slot = 0;
  auto step = [&](int s, h8 (&b0)[NT], h8 (&a0)[MT], h8 (&b1)[NT], h8 (&a1)[MT]) {
    const int nslot = slot + 1 == NB ? 0 : slot + 1;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this slot's operands have been read: refill it, ahead of the products
    request(slot);
    if ((s & 7) == 7 && s + 1 < nsteps) {            // the next step opens a block, requested a block ago
      lds_dma_wait_barrier<(NB - 1) * NT>();         // (all operand reads of the block before are complete: its buffer is free)
      if (s + 9 < nsteps) request_a((s >> 3) + 2);
    } else {
      asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NB - 1) * NT) : "memory");      // slot s + 1 has landed
    }
    read_w(nslot, b1);
    read_a(s + 1 < nsteps ? s + 1 : s, a1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[mt][j] = mfma32(b0[j], a0[mt], acc[mt][j]);   // rows columns, cols tokens
    __builtin_amdgcn_sched_barrier(0);
    slot = nslot;
  };
  for (int s = 0; s < nsteps; s += 2) {              // nsteps is a multiple of 4
    step(s, bf[0], af[0], bf[1], af[1]);
    step(s + 1, bf[1], af[1], bf[0], af[0]);
  }
  lds_dma_wait_barrier<0>();                         // every wavefront's requests past the end have landed: LDS is quiet

  // ---- epilogue: + bias + residual, row statistics over all D columns, normalise, write.
  // The accumulators have lane = token; row-major tensors want lane = column (a wavefront then touches whole row
  // segments).  Both directions pass through this wavefront's share of the (now free) weight ring:
  //  - the residual's 32 x 32 blocks are requested straight into LDS, as they are stored (row-major, 64 or 128 bytes
  //    per row), up to NSLOT blocks ahead, and picked up per token from there;
  //  - the normalised block is written per token into a padded fp32 patch and read back along the rows.
  char* const ring = mine;
  const float* const pw = &prm[wave][0][0];
  // place of KiB d of a block: all in the ring's share, but with NT = 1 the second block, and with kSplit its upper half, where the
  // operands were (nobody reads those any more)
  const unsigned lds_ring = lds_addr_of(ring);
  auto place = [&](int slot, int d) -> unsigned {
    if (NT == 1 && slot == 1) return lds_a0 + wave * 4096 + d * 1024;
    if (kSplit && slot == 1 && d >= 2) return lds_a0 + wave * 2048 + (d - 2) * 1024;
    return lds_ring + slot * 4096 + d * 1024;
  };
  const bool r32 = a.r_dt == DT_F32;
  const int res = r32 ? 4 : 2;                                // bytes per residual element
  const u4 rR = lds_dma_rsrc(uniform_ptr(a.R), a.R ? (unsigned)((size_t)T * D * res) : 0u);
  const int rrow = r32 ? lane >> 3 : lane >> 2;               // one request covers 8 (fp32) or 16 (16-bit) rows of a block
  // this lane's 16 bytes inside the row's 128 or 64: the 16-byte pieces of a row change places with its number, so that the lanes of a
  // read (one row each) meet all banks.  As they lie, eight rows met the same ones (us, as they lie / so, with the refill ahead of the
  // products: 16384 tokens of width 1024, rank 256, 40.4 / 38.2 and, 16-bit residual, 35.2 / 33.5; width 768 within 2 %).
  const int rcol = r32 ? 16 * ((lane & 7) ^ (rrow & 7)) : 16 * ((lane & 3) ^ ((rrow >> 1) & 3));
  auto request_block = [&](int mt, int j, int slot) {         // rows past T: the last row again (never stored)
    const int tok0 = (tile0 + mt) * 32;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      if (d < res) {
        int tok = tok0 + rrow + (r32 ? 8 : 16) * d;
        tok = tok < T ? tok : T - 1;
        lds_dma16(rR, place(slot, d), tok * D * res + rcol, col_of(j) * res);
      }
    }
  };
  constexpr int NBLK = MT * NT;
  if (a.R) {
#pragma unroll
    for (int i = 0; i < NSLOT && i < NBLK; ++i) request_block(i / NT, i % NT, i);
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int i = mt * NT + j, slot = i % NSLOT;
      f4v rv[4];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) rv[jj] = f4v{0.f, 0.f, 0.f, 0.f};
      if (a.R) {
        // requests complete in order: all but the blocks requested after this one have landed
        const int after = (i + NSLOT < NBLK ? i + NSLOT : NBLK) - 1 - i;
        if (r32) wait_vm(4 * after); else wait_vm(2 * after);
        const char* sp = ring + slot * 4096;
        if (NT == 1 && slot == 1) sp = (const char*)abuf + wave * 4096;
        if (kSplit && slot == 1 && r32 && l32 >= 16) sp = (const char*)abuf + wave * 2048 - 2048;      // rows 16 .. 31 of 128 bytes
        if (r32) {
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) rv[jj] = *(const f4v*)(sp + 128 * l32 + 16 * ((2 * jj + g) ^ (l32 & 7)));
        } else {
          u2 raw[4];
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) raw[jj] = *(const u2*)(sp + 64 * l32 + 16 * (jj ^ ((l32 >> 1) & 3)) + 8 * g);
#pragma unroll
          for (int jj = 0; jj < 4; ++jj)
            rv[jj] = a.r_dt == DT_BF16 ? raw_to_f4<DT_BF16>(raw[jj]) : raw_to_f4<DT_F16>(raw[jj]);
        }
        if (i + NSLOT < NBLK) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read before it is requested into again
          request_block((i + NSLOT) / NT, (i + NSLOT) % NT, slot);
        }
      }
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const f4v b = *(const f4v*)(pw + 32 * j + 8 * jj + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[mt][j][4 * jj + e] += b[e] + rv[jj][e];
          sum += acc[mt][j][4 * jj + e];
        }
      }
    }
    sum = halves_sum(sum);
    if (g == 0) red[wave][32 * mt + l32] = sum;
  }
  __syncthreads();
  float mean[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    float t = 0.f;
#pragma unroll
    for (int w2 = 0; w2 < 8; ++w2) t += red[w2][32 * mt + l32];
    mean[mt] = t / (float)D;
  }
  __syncthreads();
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    float sq = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float dlt = acc[mt][j][v] - mean[mt];
        sq = fmaf(dlt, dlt, sq);
      }
    sq = halves_sum(sq);
    if (g == 0) red[wave][32 * mt + l32] = sq;
  }
  __syncthreads();

  // stores go through buffer resources: a lane whose token lies past T passes an out-of-range offset and writes nothing
  float* const po = (float*)ring;                             // [32 tokens][36]: 16-byte accesses from both sides
  const int prow = lane >> 3, pc4 = 4 * (lane & 7);           // row-major side: rows prow + 8 i, 4 columns from pc4
  const bool y32 = a.yrow_dt == DT_F32;
  const int yes = y32 ? 4 : 2;
  const rsrc_t rY = rsrc_at(a.Yrow, a.Yrow ? (long long)T * D * yes : 0, 0);
  const rsrc_t rF = rsrc_at(a.Yfm, a.Yfm ? (long long)fm_bytes(T, D) : 0, 0);
  const int cch = D / 64;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    float t = 0.f;
#pragma unroll
    for (int w2 = 0; w2 < 8; ++w2) t += red[w2][32 * mt + l32];
    const float rstd = rsqrtf(t / (float)D + a.eps);
    const int tok0 = (tile0 + mt) * 32;
    // fragment-major unit of (token, column n = col_of(j) + 8 jj + 4 g): chunk n / 64, step jj, lane (n / 32) % 2 * 32 + token % 32
    const int fm_off = tok0 + l32 < T ? ((tile0 + mt) * cch * 256 + l32) * 16 + 8 * g : kOobOffset;
    int yoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tk = tok0 + prow + 8 * i;
      yoff[i] = tk < T ? (tk * D + colw + pc4) * yes : kOobOffset;
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int n0 = col_of(j), dn = n0 - colw;
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const f4v gm = *(const f4v*)(pw + 32 * NT + 32 * j + 8 * jj + 4 * g);
        const f4v bt = *(const f4v*)(pw + 64 * NT + 32 * j + 8 * jj + 4 * g);
        f4v y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (acc[mt][j][4 * jj + e] - mean[mt]) * rstd * gm[e] + bt[e];
        if (a.Yfm) {
          h4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (_Float16)y[e];
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, o), rF, fm_off,
                                                (((n0 >> 6) * 4 + jj) * 64 + ((n0 >> 5) & 1) * 32) * 16, 0);
        }
        if (a.Yrow) *(f4v*)(po + l32 * 36 + 8 * jj + 4 * g) = y;
      }
      if (a.Yrow) {
        f4v yy[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) yy[i] = *(const f4v*)(po + (prow + 8 * i) * 36 + pc4);
        if (y32) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, yy[i]), rY, yoff[i], dn * 4, 0);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            u2 raw;
            if (a.yrow_dt == DT_F16) {
              h4 h;
#pragma unroll
              for (int e = 0; e < 4; ++e) h[e] = (_Float16)yy[i][e];
              raw = __builtin_bit_cast(u2, h);
            } else {
              raw[0] = (uint32_t)float_to_bf16_bits(yy[i][0]) | ((uint32_t)float_to_bf16_bits(yy[i][1]) << 16);
              raw[1] = (uint32_t)float_to_bf16_bits(yy[i][2]) | ((uint32_t)float_to_bf16_bits(yy[i][3]) << 16);
            }
            __builtin_amdgcn_raw_buffer_store_b64(raw, rY, yoff[i], dn * 2, 0);
          }
        }
      }
    }
  }
}

template <int NT>
hipError_t launch_nt(const LinearLnArgs& a, hipStream_t s) {
  // 64-token workgroups when that still gives one per compute unit, else 32-token ones
  if ((a.T + 63) / 64 >= 256) hipLaunchKernelGGL((linear_ln_kernel<NT, 2>), dim3((a.T + 63) / 64), dim3(512), 0, s, a);
  else hipLaunchKernelGGL((linear_ln_kernel<NT, 1>), dim3((a.T + 31) / 32), dim3(512), 0, s, a);
  return hipGetLastError();
}

}  // namespace

bool linear_ln_supported(int D) { return D % 256 == 0 && D >= 256 && D <= 1024; }

// the residual and the row-major output are addressed with 32-bit byte offsets below the out-of-range marker
bool linear_ln_fits(long long T, int D) { return T > 0 && T * D * 4 < (long long)kOobOffset; }

hipError_t launch_linear_ln(const LinearLnArgs& a, hipStream_t s) {
  if (!linear_ln_supported(a.D) || !linear_ln_fits(a.T, a.D)) return hipErrorInvalidValue;
  switch (a.D / 256) {
    case 1: return launch_nt<1>(a, s);
    case 2: return launch_nt<2>(a, s);
    case 3: return launch_nt<3>(a, s);
    default: return launch_nt<4>(a, s);
  }
}

}  // namespace fsvd
