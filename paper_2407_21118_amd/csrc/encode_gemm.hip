// Cache-append side for many tokens at once: the prompt-sized down-projection
// h = x A (Sec. 3.1), optionally quantized as it is stored (Sec. 3.4, Appendix A).
//
// This file is a translation unit of its own: encode_gemm_kernel keeps up to 256
// accumulators per lane in the accumulation registers, while the rest of the library is
// compiled with the matrix instructions writing ordinary vector registers, an option that
// applies to a whole compilation and that this kernel does not fit.

#include <type_traits>

#include "encode_quant.hip"

namespace palu {

// A tiled GEMM on the matrix cores, C[n_tok, R] = X[n_tok, d] A[d, R].  Workgroup = TM x TN outputs, four wavefronts (WM rows of
// them) on v_mfma_f32_32x32x16, with 256 accumulator registers per lane in the 256 x 256 tile.
// k advances in stages of KS rows through a ring of NBUF stages in LDS, filled by LDS-direct loads: no staging
// registers, NBUF - 1 stages of memory requests in flight, one barrier per stage.
//
// X is k-contiguous, which is what a matrix operand wants: 16-byte reads.  A is column-contiguous: its rows lie in LDS as
// they are and the operand is read with the transposing LDS read, 4 k of 16 columns per 16 lanes.  LDS-direct loads fill
// consecutive 16-byte slots, so the swizzle that keeps the reads free of bank conflicts is in which chunk a lane requests.
//
// G k-steps of 16 make a step: the operands of a step are read while the previous one is multiplied (one wavefront
// per SIMD: nobody else hides them), its reads and the stage's requests dealt out between the matrix instructions.  The
// hand-over to the next stage (its loads waited for, one barrier, the finished stage's buffer requested anew) lies
// inside the last step of a stage, whose operands are in registers by then.
//
// Bound by the matrix pipe at the power limit from about 4096 tokens on; below, by how fast one compute unit takes its
// tile's operands in (70 .. 85 GB/s each here) over 64 k-stages, hence small tiles.  Measured, R = 2048 per side, against the
// form this replaces (two LDS buffers filled through registers, A transposed there with byte permutes): both sides of 64 / 500 / 1024 /
// 4096 tokens 35 / 39 / 63 / 128 -> 17 / 26 / 41 / 120 us; one side quantized of 64 / 500 / 2048 tokens 33 / 39 / 67 -> 15 / 22 / 43 us.
// (Wavefronts that split k instead of the tile, to read every byte from LDS once, were slower: 27 us where this takes 22.)
//
// Workgroups are numbered so that each of the 8 XCDs (workgroup id mod 8) owns a contiguous range of the tiles, columns
// fastest (the column tiles of a token row share their X rows through that XCD's L2) or, where X is smaller than A, rows
// fastest (the row tiles share a column slice of A, which then comes from memory once and not once per XCD).
constexpr int gemm_buffers(int tm, int tn, int ks) {             // stages in LDS: as many as fit 144 KiB, at most 6
  const int n = 144 * 1024 / ((tm + tn) * ks * 2);
  return n < 6 ? n : 6;
}
constexpr size_t gemm_lds_bytes(int tm, int tn, int ks) {
  const size_t stages = (size_t)gemm_buffers(tm, tn, ks) * (tm + tn) * ks * 2, out = (size_t)tm * (tn + 8) * 2;
  return stages > out ? stages : out;
}

struct GemmGrid {
  int n_col_tiles, n_row_tiles, n_tiles, per_xcd;     // tiles: sides x row tiles x column tiles
  int rows_fastest;
};

// QUANT: every 128 columns of the tile are exactly one quantization block per token, so the
// workgroup quantizes its rounded outputs in place of storing them (Sec. 3.4 applied
// while the cache is filled): codes, scales and zero-points are the ones quant_kernel
// gives for the latents the plain kernel stores.
// grid (8 * per_xcd), 256 threads, gemm_lds_bytes(TM, TN, KS) of LDS.
template <typename T, bool QUANT, int TM, int TN, int KS, int G, int WM>
__global__ __launch_bounds__(256) void encode_gemm_kernel(EncodeArgs a, GemmGrid gg) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gemm_lds[];
  constexpr int NBUF = gemm_buffers(TM, TN, KS);
  static_assert(NBUF >= 3, "the schedule keeps at least one stage in flight beyond the next");
  constexpr int WN = 4 / WM, MI = TM / WM / 32, NJ = TN / WN / 32;       // wavefronts: WM rows of WN, each MI x NJ tiles of 32 x 32
  constexpr int SPS = KS / 16 / G;                                       // steps per stage
  static_assert(SPS == 1 || SPS % 2 == 0, "register sets alternate step by step");
  constexpr int kOutPitch = TN + 8;                                      // halfs per row of the output tile
  constexpr int kXB = TM * KS * 2, kStageB = (TM + TN) * KS * 2;
  constexpr int kXOps = kXB / 4096, kAOps = TN * KS * 2 / 4096, kOps = kXOps + kAOps;      // LDS-direct requests per wavefront and stage
  static_assert(kXB % 4096 == 0 && (TN * KS * 2) % 4096 == 0 && (NBUF - 1) * kOps < 64, "whole requests, counted by the wait");
  constexpr int kCh = KS / 8;                                            // 16-byte chunks per X row and stage
  uint16_t* lds16 = reinterpret_cast<uint16_t*>(gemm_lds);

  const int tile = (blockIdx.x & 7) * gg.per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= gg.per_xcd || tile >= gg.n_tiles) return;          // uniform
  const int per_side = gg.n_col_tiles * gg.n_row_tiles;
  const int side = tile / per_side, in_side = tile - side * per_side;
  const int row_tile = gg.rows_fastest ? in_side % gg.n_row_tiles : in_side / gg.n_col_tiles;
  const int col_tile = gg.rows_fastest ? in_side / gg.n_row_tiles : in_side % gg.n_col_tiles;
  const EncodeSide sd = a.side[side];
  const int n0 = col_tile * TN, m0 = row_tile * TM;
  if (n0 >= sd.R) return;                                                // uniform
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane_lo = lane & 31, lane_hi = lane >> 5;
  const int wm = wave / WN * (TM / WM), wn = wave % WN * (TN / WN);     // this wavefront's corner of the tile

  // ---- requests.  X: slot p of row r holds chunk p ^ x_swz(r), so that 16 rows' reads of one chunk fall on distinct
  // banks.  A: slot p of row k holds chunk p ^ 4 (k mod 4) (rows of 128 bytes: p ^ 4 (k / 2 mod 2)), i.e. the four rows of a
  // transposing read lie in different 64-byte quarters of the 256-byte bank space.  Rows past the last token re-read it and columns past R the
  // last chunk (R is a multiple of 32): their products are never stored.
  auto x_swz = [](int r) { return (r / (16 / kCh)) & (kCh - 1); };
  auto a_swz = [](int k) { return TN >= 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2; };
  unsigned x_off[kXOps], a_off[kAOps];
#pragma unroll
  for (int x = 0; x < kXOps; ++x) {
    const int o = (wave * kXOps + x) * 1024 + lane * 16, r = o / (KS * 2), p = (o % (KS * 2)) / 16;
    x_off[x] = ((unsigned)min(r, a.n_tok - 1 - m0) * (unsigned)a.d + (unsigned)((p ^ x_swz(r)) * 8)) * 2u;
  }
#pragma unroll
  for (int x = 0; x < kAOps; ++x) {
    const int o = (wave * kAOps + x) * 1024 + lane * 16, k = o / (TN * 2), p = (o % (TN * 2)) / 16;
    a_off[x] = ((unsigned)k * (unsigned)sd.R + (unsigned)min(n0 + (p ^ a_swz(k)) * 8, sd.R - 8)) * 2u;
  }
  const unsigned char* x_base = uniform_ptr(reinterpret_cast<const unsigned char*>(a.x + (size_t)m0 * a.d));
  const unsigned char* a_base = uniform_ptr(reinterpret_cast<const unsigned char*>(sd.A));
  const unsigned lds_base = __builtin_amdgcn_readfirstlane((unsigned)(size_t)gemm_lds);
  const unsigned a_stage_bytes = (unsigned)KS * 2u * (unsigned)sd.R;
  const int n_stages = a.d / KS;                                         // even: d is a multiple of 128
  struct Req {
    const unsigned char *xs, *as;
    unsigned m0;
  };
  auto request_stage = [&](int stage, unsigned buf_off) __attribute__((always_inline)) {       // past the last stage: that one again, unused
    const int st = min(stage, n_stages - 1);
    Req r;
    r.xs = uniform_ptr(x_base + (size_t)st * (KS * 2));
    r.as = uniform_ptr(a_base + (size_t)st * a_stage_bytes);
    r.m0 = __builtin_amdgcn_readfirstlane(lds_base + buf_off);
    return r;
  };
  auto request_op = [&](const Req& r, int x) __attribute__((always_inline)) {
    const unsigned m0v = r.m0 + (x < kXOps ? (unsigned)((wave * kXOps + x) * 1024) : (unsigned)(kXB + (wave * kAOps + x - kXOps) * 1024));
    if (x < kXOps) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(m0v), "v"(x_off[x]), "s"(r.xs) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(m0v), "v"(a_off[x - kXOps]), "s"(r.as) : "memory");
  };

  // ---- operand reads, byte offsets inside a stage.  X: row wm + 32 i + lane_lo, k-octet 2 ks + lane_hi.  A: k = 16 ks +
  // 8 lane_hi + 4 q + 0..3 of columns wn + 32 j + 16 (lane bit 4) + 0..15: the lane hands in row (lane / 4) % 4, columns
  // 4 (lane % 4) .. + 3 of that block and receives column lane % 16.
  int x_rd[KS / 16], a_rd[NJ];
#pragma unroll
  for (int ks = 0; ks < KS / 16; ++ks) {
    const int r = wm + lane_lo;
    x_rd[ks] = r * (KS * 2) + (((2 * ks + lane_hi) ^ x_swz(r)) * 16);
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int kr = (lane >> 2) & 3, c = (wn >> 3) + 4 * j + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    a_rd[j] = kXB + (8 * lane_hi + kr) * (TN * 2) + ((c ^ a_swz(kr)) * 16) + (lane & 1) * 8;
  }
  using Vec = typename T::vec8;
  Vec xa[2][G][MI], ab[2][G][NJ];
  constexpr int kRd = G * (MI + NJ);                                     // operands per step
  auto read_op = [&](int set, unsigned buf_off, int p, int x) __attribute__((always_inline)) {      // operand x of step p of the stage at buf_off
    const int g = x / (MI + NJ), y = x % (MI + NJ), ks = p * G + g;
    if (y < MI) {
      xa[set][g][y] = *reinterpret_cast<const Vec*>(gemm_lds + buf_off + x_rd[ks] + y * (32 * KS * 2));
    } else {
      typedef short short4v __attribute__((ext_vector_type(4)));
      using LdsV = __attribute__((address_space(3))) short4v;
      const unsigned char* src = gemm_lds + buf_off + a_rd[y - MI] + ks * (16 * TN * 2);
      const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsV*)src);
      const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsV*)(src + 4 * TN * 2));
      ab[set][g][y - MI] = __builtin_bit_cast(Vec, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };

  float16v acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // Step P of stage s (its operands in register set SET).  buf / next_buf: the stage's buffer and the next one's.
  constexpr int kMma = G * MI * NJ;
  constexpr int kHand = SPS == 1 ? 0 : kMma / 2;                         // matrix instruction before which the hand-over of the last step lies
  auto step = [&](auto p_c, auto set_c, int s, unsigned buf, unsigned next_buf) __attribute__((always_inline)) {
    constexpr int P = decltype(p_c)::value, SET = decltype(set_c)::value;
    constexpr bool last = P == SPS - 1;
    constexpr int from = last ? kHand : 0, span = kMma - from;
    Req req;
#pragma unroll
    for (int mi = 0; mi < kMma; ++mi) {
      if (last && mi == from) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NBUF - 2) * kOps));       // stage s + 1 has landed (this wavefront's share)
        __syncthreads();                                                 // ... everybody's; and stage s has been read by everybody
        req = request_stage(s + NBUF, buf);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (mi >= from) {
#pragma unroll
        for (int x = (mi - from) * kRd / span; x < (mi - from + 1) * kRd / span; ++x)
          read_op(SET ^ 1, last ? next_buf : buf, last ? 0 : P + 1, x);
        if (last) {
#pragma unroll
          for (int x = (mi - from) * kOps / span; x < (mi - from + 1) * kOps / span; ++x) request_op(req, x);
        }
      }
      const int g = mi / (MI * NJ), i = mi / NJ % MI, j = mi % NJ;
      acc[i][j] = T::mfma(xa[SET][g][i], ab[SET][g][j], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // ---- start-up: the whole ring requested, stage 0 landed, its first operands read
#pragma unroll
  for (int b = 0; b < NBUF; ++b) {
    const Req r = request_stage(b, (unsigned)(b * kStageB));
#pragma unroll
    for (int x = 0; x < kOps; ++x) request_op(r, x);
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm((NBUF - 1) * kOps));
  __syncthreads();
#pragma unroll
  for (int x = 0; x < kRd; ++x) read_op(0, 0, 0, x);
  unsigned buf = 0;
  auto after = [](unsigned b) { return b + kStageB == (unsigned)(NBUF * kStageB) ? 0u : b + kStageB; };
  for (int s = 0; s < n_stages; s += SPS == 1 ? 2 : 1) {
    const unsigned b1 = after(buf);
    if constexpr (SPS == 1) {
      const unsigned b2 = after(b1);
      step(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, s, buf, b1);
      step(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{}, s + 1, b1, b2);
      buf = b2;
    } else {
      step(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, s, buf, b1);
      step(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, s, buf, b1);
      if constexpr (SPS == 4) {
        step(std::integral_constant<int, 2>{}, std::integral_constant<int, 0>{}, s, buf, b1);
        step(std::integral_constant<int, 3>{}, std::integral_constant<int, 1>{}, s, buf, b1);
      }
      buf = b1;
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));       // the ring becomes the output tile: no request may still write it, nobody still read it
  __syncthreads();

  // accumulator element e of tile (i, j): token m0 + wm + 32 i + mfma_row(e), column n0 + wn + 32 j + lane_lo.
  // LDS becomes the rounded output tile [TM][kOutPitch].
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        lds16[(wm + 32 * i + mfma_row(e, lane_hi)) * kOutPitch + wn + 32 * j + lane_lo] = T::from_float(acc[i][j][e]);
  __syncthreads();

  if constexpr (QUANT) {
    const int n_blocks = sd.R / 128;
    constexpr int NB = TN / 128;                     // quantization blocks per token in the tile
    // threads per (token, block): up to 16 where the tile has few blocks (every thread at work; a block's parameters,
    // two divisions, are computed by each of them)
    constexpr int TPB = 1024 / (TM * NB) < 16 ? 1024 / (TM * NB) : 16, CH8 = 16 / TPB;
#pragma unroll 1
    for (int item = tid; item < TM * NB * TPB; item += 256) {
      const int tr = item / (NB * TPB), bl = (item / TPB) % NB, part = item % TPB;
      uint4v v[CH8];                                 // channels 8 CH8 part .. of the block
#pragma unroll
      for (int i = 0; i < CH8; ++i) v[i] = *reinterpret_cast<const uint4v*>(lds16 + tr * kOutPitch + bl * 128 + (part * CH8 + i) * 8);
      float mn = T::to_float((uint16_t)(v[0][0] & 0xffffu)), mx = mn;
#pragma unroll
      for (int i = 0; i < CH8; ++i)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float x0 = T::to_float((uint16_t)(v[i][w] & 0xffffu)), x1 = T::to_float((uint16_t)(v[i][w] >> 16));
          mn = fminf(mn, fminf(x0, x1));
          mx = fmaxf(mx, fmaxf(x0, x1));
        }
#pragma unroll
      for (int off = 1; off < TPB; off <<= 1) {
        mn = fminf(mn, __shfl_xor(mn, off, 64));
        mx = fmaxf(mx, __shfl_xor(mx, off, 64));
      }
      const int t = m0 + tr, blk = col_tile * NB + bl;
      if (t >= a.n_tok || blk >= n_blocks) continue;
      const QuantParams qp = quant_params(mn, mx);
      const size_t orow = a.dst_row ? (size_t)a.dst_row[t] : (size_t)t;
      uint32_t word[CH8];
#pragma unroll
      for (int i = 0; i < CH8; ++i) {
        word[i] = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          word[i] |= (quant_code(T::to_float((uint16_t)(v[i][c] & 0xffffu)), qp) | (quant_code(T::to_float((uint16_t)(v[i][c] >> 16)), qp) << 4)) << (8 * c);
      }
      uint8_t* dst = sd.codes + orow * (size_t)(sd.R / 2) + blk * 64 + part * (4 * CH8);
      if constexpr (CH8 >= 4) {
#pragma unroll
        for (int i = 0; i < CH8; i += 4) *reinterpret_cast<uint4v*>(dst + 4 * i) = uint4v{word[i], word[i + 1], word[i + 2], word[i + 3]};
      } else if constexpr (CH8 == 2) {
        *reinterpret_cast<uint2v*>(dst) = uint2v{word[0], word[1]};
      } else {
        *reinterpret_cast<uint32_t*>(dst) = word[0];
      }
      if (part == 0) {
        sd.scale[orow * n_blocks + blk] = qp.s16;
        sd.zero[orow * n_blocks + blk] = qp.z16;
      }
    }
    return;
  }
  // rows leave in 16-byte pieces where the destination allows it (4-byte alignment is all the interface asks for)
  const bool wide = ((reinterpret_cast<uintptr_t>(sd.latent) & 15) == 0) && ((sd.row_stride & 7) == 0);
#pragma unroll 4
  for (int id = tid; id < TM * (TN / 8); id += 256) {
    const int tr = id / (TN / 8), c8 = (id % (TN / 8)) * 8;
    const int t = m0 + tr;
    if (t >= a.n_tok || n0 + c8 >= sd.R) continue;
    const uint4v v = *reinterpret_cast<const uint4v*>(lds16 + tr * kOutPitch + c8);
    const long long row = a.dst_row ? a.dst_row[t] : t;
    uint16_t* dst = sd.latent + row * sd.row_stride + n0 + c8;
    if (wide) {
      *reinterpret_cast<uint4v*>(dst) = v;
    } else {
      uint32_t* d32 = reinterpret_cast<uint32_t*>(dst);
      d32[0] = v[0]; d32[1] = v[1]; d32[2] = v[2]; d32[3] = v[3];
    }
  }
}

namespace {

template <typename K>
int allow_gemm_lds(K kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return PALU_OK;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes) == hipSuccess ? PALU_OK : PALU_ERR_HIP;
}

// The tiles in use and what one costs: microseconds per 4096 inputs of a workgroup with every compute unit busy (measured,
// R = 2048 per side).  A launch takes the tile whose rounds of workgroups cost least: a larger one reads fewer bytes
// per product, a smaller one leaves no compute unit idle.
struct GemmTile {
  int tm, tn, ks;
  float us;
};
constexpr GemmTile kGemmTiles[] = {{256, 256, 32, 119.f}, {128, 256, 64, 70.f}, {128, 128, 64, 41.f}, {64, 128, 64, 25.f}, {32, 128, 64, 21.f}, {64, 64, 64, 16.f}};
constexpr int kNumGemmTiles = sizeof(kGemmTiles) / sizeof(kGemmTiles[0]);

template <typename T, bool Q>
int launch_gemm_t(const EncodeArgs& a, int max_R, int n_sides, int tile_opt, int n_cu, hipStream_t s) {
  auto ceil_div = [](int x, int y) { return (x + y - 1) / y; };
  auto tiles = [&](const GemmTile& g) { return ceil_div(max_R, g.tn) * ceil_div(a.n_tok, g.tm) * n_sides; };
  int best = 0;
  for (int i = 1; i < kNumGemmTiles; ++i) {
    if (Q && kGemmTiles[i].tn % 128 != 0) continue;                      // whole quantization blocks
    if (ceil_div(tiles(kGemmTiles[i]), n_cu) * kGemmTiles[i].us < ceil_div(tiles(kGemmTiles[best]), n_cu) * kGemmTiles[best].us) best = i;
  }
  // option: the first tile of that many rows (32: the smallest tile)
  for (int i = kNumGemmTiles - 1; tile_opt > 0 && i >= 0; --i)
    if (kGemmTiles[i].tm == tile_opt && !(Q && kGemmTiles[i].tn % 128 != 0)) best = i;
  const GemmTile& g = kGemmTiles[best];
  GemmGrid gg;
  gg.n_col_tiles = ceil_div(max_R, g.tn);
  gg.n_row_tiles = ceil_div(a.n_tok, g.tm);
  gg.n_tiles = tiles(g);
  gg.per_xcd = ceil_div(gg.n_tiles, 8);
  gg.rows_fastest = a.n_tok < max_R;
  const size_t lds = gemm_lds_bytes(g.tm, g.tn, g.ks);
  using Fn = void (*)(EncodeArgs, GemmGrid);
  // (a quantized call takes no tile of 64 columns; the entry repeats its neighbour)
  static const Fn fns[kNumGemmTiles] = {encode_gemm_kernel<T, Q, 256, 256, 32, 1, 2>, encode_gemm_kernel<T, Q, 128, 256, 64, 1, 2>,
                                        encode_gemm_kernel<T, Q, 128, 128, 64, 1, 2>, encode_gemm_kernel<T, Q, 64, 128, 64, 4, 2>,
                                        encode_gemm_kernel<T, Q, 32, 128, 64, 4, 1>,
                                        encode_gemm_kernel<T, Q, Q ? 32 : 64, Q ? 128 : 64, 64, 4, Q ? 1 : 2>};
  const Fn fn = fns[best];
  if (allow_gemm_lds(fn, lds) != PALU_OK) return PALU_ERR_HIP;
  hipLaunchKernelGGL(fn, dim3((unsigned)(8 * gg.per_xcd)), dim3(256), lds, s, a, gg);
  return hipGetLastError() == hipSuccess ? PALU_OK : PALU_ERR_HIP;
}

}  // namespace

int launch_encode_gemm_tiles(int act, const EncodeArgs& a, int max_R, int n_sides, bool quant, int tile_opt, int n_cu,
                             hipStream_t s) {
  if (act == PALU_F16) {
    return quant ? launch_gemm_t<F16, true>(a, max_R, n_sides, tile_opt, n_cu, s)
                 : launch_gemm_t<F16, false>(a, max_R, n_sides, tile_opt, n_cu, s);
  }
  return quant ? launch_gemm_t<BF16, true>(a, max_R, n_sides, tile_opt, n_cu, s)
               : launch_gemm_t<BF16, false>(a, max_R, n_sides, tile_opt, n_cu, s);
}

}  // namespace palu
