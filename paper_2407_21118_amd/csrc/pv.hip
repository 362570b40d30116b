// Softmax partials and the value contraction in latent space on the matrix cores
// (Eq. 4: softmax(q K^T) (H_v B_v) evaluated as (p H_v) B_v; Sec. 3.1.1):
//   per (sequence, split of the sequence, unit of heads x latent columns)
//     p_t = exp2(score_t - m),  l = sum_t p_t,  o[c] = sum_t p_t H_v[t, c].
//
// One wavefront owns one split and shares nothing with the others: no workgroup
// barrier anywhere.  It walks its tokens in sets of 32 with an online softmax
// (running maximum m, accumulators rescaled when m grows) and contracts each
// set with v_mfma_f32_16x16x32_f16: A = probabilities (rows = heads, k = tokens),
// B = latents (k = tokens, columns = latent channels).  The cache is token-major,
// so a 16-byte load brings 8 channels of one token, while the matrix cores want
// 8 tokens of one channel per lane: each lane loads the same 8-channel chunk of
// 8 consecutive tokens and transposes the 8x8 block in registers with byte
// permutes (one per operand register); channel e of every chunk then forms the
// B operand of the e-th of 8 accumulator sets.  The vector ALU only does the
// softmax (a few operations per token and head) and the transposes, so the
// kernel stays bound by the latent stream for every head-group size (a latent
// shared by all 32 heads goes in two blocks of 16 heads, side by side in a
// workgroup, so that the second read of a row comes from the cache).
//
// 4-bit latents: while transposing, a code c is masked in place into the low mantissa bits of an fp16 zero,
// i.e. becomes the subnormal number c 2^-24 (codes in bits 0 .. 3) or c 2^-20 (bits 4 .. 7): the matrix cores
// take subnormal fp16 operands exactly, so one AND per operand register (and one shift per four) dequantizes.
// The per-(token, 128-channel block) scale is folded into the probabilities (one probability tile per block,
// a = p s), the power of two into the write-out, and the zero-points into one scalar per (head, block):
// sum_t a (c - z) = 2^24 sum_t a (c 2^-24) - sum_t a z.
//
// The running maximum is lazy: it only rises (and the accumulators are only rescaled) when a set's maximum
// exceeds it by more than 8 (scores are base-2 logarithms), so probabilities reach 256 at most; the (max, sum)
// pair a split reports is consistent with its accumulators, which is all the combination needs.

#include "launch.h"
#include "softmax_dev.h"

#include <type_traits>

#ifndef PALU_PV_PAIR_DEPTH
#define PALU_PV_PAIR_DEPTH 2
#endif

namespace palu {

// scores[0] += scores[1] + ... + scores[n_parts-1] for heads with more than two
// partial planes (ranks contracted in slices); the value kernel then reads one.
__global__ __launch_bounds__(256) void plane_sum_kernel(PlaneSumArgs a) {
  const int h = blockIdx.y, b = blockIdx.z;
  const int np = a.n_parts[h];
  if (np <= 2) return;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= a.seq_len) return;
  float* p = a.scores + ((size_t)b * a.n_heads + h) * a.lpad + t;
  float s = p[0];
  for (int pl = 1; pl < np; ++pl) s += p[(size_t)pl * a.part_stride];
  p[0] = s;
}

// T:  storage type of unquantized latents (bfloat16 is converted to fp16 in registers: exact in the fp16 range)
// HS: score slots per lane: the unit has at most 2*HS heads (built: 2 and 8; above 8 the code takes two 16-row tiles)
// NG: 128-column blocks per unit (16 lanes x 8 channels each)
// QB: latents are QB-bit codes (4, 3 or 2; 0: unquantized); every 128-column block of the unit is one
//     quantization block.  In the body I4 = "quantized": 3- and 2-bit codes are spread into the
//     4-bit register layout when they are consumed and then follow the 4-bit arithmetic.
// TWO: some head of the launch has two score planes (the kernel then requests both planes of every head; with one
//     plane everywhere the second request, an instruction per head slot and set, is left out)
// QK: non-RoPE attention in one pass: the scores of a set are made from its key latents and the folded queries (the arithmetic of qk_kernel, same
//     units and columns of at most 256) instead of being read; nothing goes through memory in between.  Bound like the two kernels
//     it replaces, by the latent streams and, with codes, by the instructions beside them; what it saves is a launch and the scores' way
//     through memory.  us a step, two launches -> one: 1 x 65536 tokens 129 -> 119, in 4 bits 76.9 -> 71.7; 16 x 8192 236 -> 218, in 4
//     bits 108.5 -> 96.8; 1 x 1024 34.6 -> 33.2; rank 64 per head, 4 x 8000 80.8 -> 70.5.
template <typename T, int HS, int NG, int QB, bool TWO, bool QK>
__device__ __forceinline__ void pv_body(const std::conditional_t<QK, StreamArgs, PvArgs>& a) {
  constexpr bool I4 = QB != 0;
  constexpr bool kIsBf16 = !__is_same(T, F16);
  constexpr int MT = HS > 8 ? 2 : 1;
  constexpr int NA = I4 ? NG : 1;                  // scaled probabilities: one set per quantization block
  // Quantized latents, four heads, two blocks: a lane takes two neighbouring 8-channel chunks with one load (8 bytes
  // of 4-bit codes: a load instruction then covers whole 128-byte rows; 4 bytes of 2-bit fields, plus 2 bytes of
  // third bits), and a set needs half the requests.  The chunks of lanes
  // n < 8 lie in block 0 and those of lanes n >= 8 in block 1, so one matrix instruction serves both blocks:
  // the probability tile has rows (block, head) - 8 of its 16 - and a lane keeps the rows of its own block.
  constexpr bool kPair = I4 && NG == 2 && HS == 2;
  constexpr int NT = kPair ? 1 : NA;               // probability tiles
  constexpr int kPitch = 40;                       // halfs per head row: 80-byte pitch, 16-byte reads of 16 rows hit distinct banks
  __shared__ __attribute__((aligned(16))) _Float16 p_lds[4][NT][MT * 16 * kPitch];
  __shared__ __attribute__((aligned(16))) float x_lds[4][MT * 16 * NA];
  constexpr int kScPitch = 33;                     // floats per score row: the 16 tokens of two rows fall on distinct banks
  __shared__ float sc_lds[QK ? 4 : 1][QK ? 2 * HS * kScPitch : 1];
  extern __shared__ __attribute__((aligned(16))) unsigned char qk_lds_all[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, kq = lane >> 4;         // matrix-core roles: column (B, D) or head row (A); token quarter
  const int tl = lane & 31, hp = lane >> 5;        // softmax roles: token of the set; head parity
  const Meta& m = a.meta;

  // grid (groups of units_per_wg units, groups of 4 / units_per_wg splits, batch); the wavefronts of a
  // workgroup take neighbouring units of the same split first: they read neighbouring columns of the same
  // rows, and the scales and zero-points of a token's blocks, which lie side by side, come into this
  // compute unit's cache once instead of once per unit.
  const int upw = a.units_per_wg;
  const int unit = blockIdx.x * upw + (wave & (upw - 1)), b = blockIdx.z;
  const int split = blockIdx.y * (4 / upw) + wave / upw;
  if constexpr (QK) {
    // folded queries of the workgroup's units (one behind the other), in the order of channels that the quantized operands have
    for (int j = 0; j < upw; ++j) {
      const int uj = blockIdx.x * upw + j;
      if (uj >= a.units.n_units) break;              // uniform
      const int rows = (I4 ? 1 : 2) * a.units.u[uj].nh;
      const uint16_t* src = a.qt + (size_t)blockIdx.z * a.qt_bstride + a.keys[uj].q_off;
      unsigned char* dst = qk_lds_all + j * a.lds_unit_stride;
      for (int i = threadIdx.x; i < rows * 32; i += 256) {
        const int r = i >> 5, cc = i & 31;
        uint4v v = *reinterpret_cast<const uint4v*>(src + r * 256 + cc * 8);
        if constexpr (I4)
          v = uint4v{__builtin_amdgcn_perm(v.z, v.x, 0x05040100u), __builtin_amdgcn_perm(v.z, v.x, 0x07060302u),
                     __builtin_amdgcn_perm(v.w, v.y, 0x05040100u), __builtin_amdgcn_perm(v.w, v.y, 0x07060302u)};
        *reinterpret_cast<uint4v*>(dst + (r * kStreamPitch + cc * 8) * 2) = v;
      }
      if constexpr (I4) {                            // their block sums behind the rows
        const float* qs_src = a.qsum + (size_t)blockIdx.z * a.qs_bstride + a.keys[uj].qs_off;
        float* qs_dst = reinterpret_cast<float*>(dst + rows * kStreamPitch * 2);
        for (int i = threadIdx.x; i < rows * 2; i += 256) qs_dst[i] = qs_src[i];
      }
    }
    __syncthreads();
  }
  if (unit >= a.units.n_units) return;             // whole wavefront; nothing below synchronises wavefronts
  const int L = a.seq_lens ? min(a.seq_lens[b], a.seq_len) : a.seq_len;
  const int s0 = split * a.split_tokens;
  if (split >= a.n_split || s0 >= L) return;       // whole wavefront; nothing below synchronises wavefronts
  const int ntok = min(a.split_tokens, L - s0);
  const int n_sets = (ntok + 31) >> 5;
  const int last = ntok - 1;

  const PvUnit u = a.units.u[unit];
  asm volatile("" :: "s"(a.hv), "s"(a.scores), "s"(a.seq_lens), "s"(a.o_part), "s"(a.ml_part), "s"(a.row_elems), "s"(a.max_seq),
               "s"(a.part_stride), "s"(a.seq_len), "s"(a.lpad), "s"(a.split_tokens), "s"(a.n_split), "s"(a.o_stride),
               "s"(u.c0), "s"((int)u.h0), "s"((int)u.ncols), "s"((int)u.nh));      // all in registers here: one round trip
  const int h0 = u.h0, nh = u.nh, c0 = u.c0;
  const int lpt = u.ncols >> 3;                    // 8-channel chunks per row of the unit

  const size_t row0 = (size_t)b * a.max_seq + s0;
  // quantized latents: 4-bit codes, or 2-bit fields followed (3 bits) by a plane of third bits at R/4 bytes
  constexpr int bits = I4 ? QB : 16;
  const unsigned row_bytes = (unsigned)a.row_elems * (unsigned)bits / 8u;
  const unsigned char* base = (const unsigned char*)a.hv + row0 * row_bytes + (I4 ? (bits == 4 ? c0 / 2 : c0 / 4) : c0 * 2);
  const unsigned hi_plane = (unsigned)a.row_elems / 4u + (unsigned)c0 / 8u - (unsigned)c0 / 4u;   // from `base` to the third bits
  unsigned coff[NG];
#pragma unroll
  for (int ng = 0; ng < NG; ++ng) coff[ng] = (unsigned)min(ng * 16 + n, lpt - 1) * (I4 ? (bits == 4 ? 4u : 2u) : 16u);
  if constexpr (kPair) coff[0] = (unsigned)min(n, (lpt >> 1) - 1) * (bits == 4 ? 8u : 4u);      // chunks 2n and 2n + 1 (a unit has a multiple of 4 chunks)
  // byte offset of the row of the lane's token j in set 0; a set further on is 32 rows further, clamped to the last row
  unsigned roff[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) roff[j] = (unsigned)(8 * kq + j) * row_bytes;
  const unsigned last_off = (unsigned)last * row_bytes, set_bytes = 32u * row_bytes;

  const float* sc_ptr[HS];
  bool two[HS];
  int lim[HS];                                     // tokens of this split the head's query attends (its own row limit)
#pragma unroll
  for (int i = 0; i < HS; ++i) {
    const int h = h0 + min(hp + 2 * i, nh - 1);
    if constexpr (!QK) {
      sc_ptr[i] = a.scores + ((size_t)b * m.n_heads + h) * a.lpad + s0;
      two[i] = a.n_parts[h] > 1;
    }
    lim[i] = a.q_len ? a.q_len[b * m.nq + q_token(m, h)] - s0 : 0x7fffffff;
  }
  const size_t sz_idx0 = I4 ? row0 * a.n_blocks_q + (c0 >> 7) : 0;
  const int n_blk = (u.ncols + 127) >> 7;          // 128-column blocks the unit really has

  // QK: the key side, requests of a set and scores from it as in qk_kernel (one chunk of at most 256 columns)
  constexpr int kKeyLoads = I4 ? 2 : 8;            // 16-byte loads per 16 tokens: one per 128-column block of codes, else one per 32 columns
  unsigned k_row_bytes = 0, k_hi_plane = 0;
  const unsigned char* k_base = nullptr;
  size_t k_sz0 = 0;
  int k_cols = 256, k_blk = 2;
  const unsigned char* qk_lds = nullptr;
  uint32_t fp16_ones = 0;
  if constexpr (QK) {
    const StreamKeys ku = a.keys[unit];
    k_row_bytes = (unsigned)a.k_row_elems * (unsigned)bits / 8u;
    k_base = (const unsigned char*)a.hk + row0 * k_row_bytes + (I4 ? (bits == 4 ? ku.c0 / 2 : ku.c0 / 4) : ku.c0 * 2);
    k_hi_plane = (unsigned)a.k_row_elems / 4u + (unsigned)ku.c0 / 8u - (unsigned)ku.c0 / 4u;
    k_sz0 = I4 ? row0 * a.k_blocks_q + (ku.c0 >> 7) : 0;
    k_cols = ku.ncols;
    k_blk = (k_cols + 127) >> 7;
    qk_lds = qk_lds_all + (wave & (upw - 1)) * a.lds_unit_stride;
    fp16_ones = per_lane_constant(0x3c003c00u);
  }
  struct Keys {
    uint4v h[QK ? 2 : 1][QK ? kKeyLoads : 1];      // [16-token tile][load]
    uint16_t sz[2];                                // quantized: the lane's share of the set's scales and zero-points
  };
  auto issue_keys = [&](Keys& st, int k) {
    if constexpr (QK) {
      if constexpr (I4) {
        const unsigned t = (unsigned)min(k * 32 + (kq >> 1) * 16 + n, last);
        const uint16_t* arr = (kq & 1) ? a.hk_zero : a.hk_scale;
#pragma unroll
        for (int x = 0; x < 2; ++x) st.sz[x] = arr[k_sz0 + (size_t)t * a.k_blocks_q + min(x, k_blk - 1)];
      }
#pragma unroll
      for (int tau = 0; tau < 2; ++tau) {
        const unsigned t = (unsigned)min(k * 32 + tau * 16 + n, last);
#pragma unroll
        for (int x = 0; x < kKeyLoads; ++x) {
          const unsigned off = I4 ? (unsigned)min(x, k_blk - 1) * 64u + (unsigned)kq * 16u : (unsigned)min(x * 32 + kq * 8, k_cols - 8) * 2u;
          const unsigned char* p = k_base + (size_t)(t * k_row_bytes);
          if constexpr (!I4 || bits == 4) {
            st.h[tau][x] = *reinterpret_cast<const uint4v*>(p + off);
          } else {
            const uint2v lo = *reinterpret_cast<const uint2v*>(p + (off >> 1));
            st.h[tau][x].x = lo.x;
            st.h[tau][x].y = lo.y;
            if constexpr (bits == 3) st.h[tau][x].z = *reinterpret_cast<const uint32_t*>(p + k_hi_plane + (off >> 2));
          }
        }
      }
    }
  };
  // the set's scores of all heads to sc_lds [head][token]
  auto make_scores = [&](const Keys& st) {
    if constexpr (QK) {
      const int qrow = min(n, nh - 1) * kStreamPitch * 2;
      float4v d2[2] = {};
      if constexpr (!I4) {
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const half8 af = *reinterpret_cast<const half8*>(qk_lds + qrow + (x * 32 + kq * 8) * 2);
          const half8 al = *reinterpret_cast<const half8*>(qk_lds + nh * kStreamPitch * 2 + qrow + (x * 32 + kq * 8) * 2);
#pragma unroll
          for (int tau = 0; tau < 2; ++tau) {
            uint4v hw = st.h[tau][x];
            if constexpr (kIsBf16) {
#pragma unroll
              for (int e = 0; e < 4; ++e)
                hw[e] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__builtin_bit_cast(float, hw[e] << 16),
                                                                                __builtin_bit_cast(float, hw[e] & 0xffff0000u)));
            }
            const half8 bop = __builtin_bit_cast(half8, hw);
            d2[tau] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af, bop, d2[tau], 0, 0, 0);
            d2[tau] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, bop, d2[tau], 0, 0, 0);
          }
        }
      } else {
        uint32_t szv[4];                           // [2 tau + (0: scales, 1: zero-points)], block x in bits 16 x ..
        const int own = (int)((uint32_t)st.sz[0] | ((uint32_t)st.sz[1] << 16));
#pragma unroll
        for (int k4 = 0; k4 < 4; ++k4) szv[k4] = (uint32_t)__builtin_amdgcn_ds_bpermute((n + 16 * k4) * 4, own);
        const float* qs_base = reinterpret_cast<const float*>(qk_lds + nh * kStreamPitch * 2);
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          half8 af[4];
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) af[jj] = *reinterpret_cast<const half8*>(qk_lds + qrow + (x * 128 + kq * 32 + jj * 8) * 2);
          float qs[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) qs[r] = qs_base[min(4 * kq + r, nh - 1) * 2 + min(x, k_blk - 1)];
#pragma unroll
          for (int tau = 0; tau < 2; ++tau) {
            float4v d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
              uint32_t w = st.h[tau][x][jj];
              if constexpr (bits != 4) w = expand_low_bits(st.h[tau][x][jj >> 1] >> (16 * (jj & 1)), st.h[tau][x][2] >> (8 * jj), bits == 3);
              const NibblePairs np = nibbles_to_fp16_pairs(w, fp16_ones);
              const uint4v bw = {np.p[0], np.p[1], np.p[2], np.p[3]};
              d = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[jj], __builtin_bit_cast(half8, bw), d, 0, 0, 0);
            }
            const float sc = x < k_blk ? F16::to_float((uint16_t)(szv[2 * tau] >> (16 * x))) : 0.f;
            const float zp = F16::to_float((uint16_t)(szv[2 * tau + 1] >> (16 * x)));
#pragma unroll
            for (int r = 0; r < 4; ++r) d2[tau][r] = fmaf(sc, fmaf(-(zp + 64.f), qs[r], 64.f * d[r]), d2[tau][r]);
          }
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (4 * kq + r >= nh) continue;            // accumulator row = head
#pragma unroll
        for (int tau = 0; tau < 2; ++tau) sc_lds[wave][(4 * kq + r) * kScPitch + tau * 16 + n] = d2[tau][r] * a.scale;
      }
      wave_lds_fence();
    }
  };

  struct Blk {
    uint32_t h[8][I4 ? (QB == 3 ? 2 : 1) : 4];     // [token j of the lane's quarter][dword]; quantized: codes, third bits (3-bit only)
  };
  struct Set {
    Blk blk[NG];
    float sc[QK ? 1 : HS][TWO ? 2 : 1];
    Keys keys;
    uint16_t sz[NA];                               // quantized: scales (lanes 0 .. 31) or zero-points (32 .. 63) of the lane's softmax token, as loaded
  };

  // every load is unconditional and in bounds (clamped to the last token / chunk / head);
  // what a clamped load returns is given zero weight or never stored
  auto issue = [&](Set& st, int k) {
    const int tb = k * 32;
    issue_keys(st.keys, k);
#pragma unroll
    for (int ng = 0; ng < (kPair ? 1 : NG); ++ng) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const unsigned char* p = base + (size_t)(min(roff[j] + (unsigned)k * set_bytes, last_off) + coff[ng]);
        if constexpr (kPair && bits == 4) {
          const uint2v v = *reinterpret_cast<const uint2v*>(p);
          st.blk[0].h[j][0] = v.x;
          st.blk[1].h[j][0] = v.y;
        } else if constexpr (kPair) {
          const uint32_t v = *reinterpret_cast<const uint32_t*>(p);                 // two chunks' two-bit fields
          st.blk[0].h[j][0] = v;
          st.blk[1].h[j][0] = v >> 16;
          if constexpr (QB == 3) {
            const uint32_t pl = *reinterpret_cast<const uint16_t*>(p + hi_plane - (coff[0] >> 1));   // their two bytes of third bits
            st.blk[0].h[j][1] = pl;
            st.blk[1].h[j][1] = pl >> 8;
          }
        } else if constexpr (I4) {
          if constexpr (bits == 4) {
            st.blk[ng].h[j][0] = *reinterpret_cast<const uint32_t*>(p);
          } else {
            st.blk[ng].h[j][0] = *reinterpret_cast<const uint16_t*>(p);
            if constexpr (QB == 3) st.blk[ng].h[j][1] = p[hi_plane - (coff[ng] >> 1)];      // the chunk's byte of the third-bit plane
          }
        } else {
          const uint4v v = *reinterpret_cast<const uint4v*>(p);
          st.blk[ng].h[j][0] = v.x; st.blk[ng].h[j][1] = v.y; st.blk[ng].h[j][2] = v.z; st.blk[ng].h[j][3] = v.w;
        }
      }
    }
    const int ts = min(tb + tl, last);
    if constexpr (!QK) {
#pragma unroll
      for (int i = 0; i < HS; ++i) {
        st.sc[i][0] = sc_ptr[i][ts];
        if constexpr (TWO) st.sc[i][1] = sc_ptr[i][ts + a.part_stride];
      }
    }
    if constexpr (I4) {
      // the two lanes of a token split its scales and zero-points (2-byte requests cost the memory pipeline as much
      // as the 8-byte latent ones) and swap them in process()
      const uint16_t* arr = hp ? a.hv_zero : a.hv_scale;
#pragma unroll
      for (int ng = 0; ng < NG; ++ng)
        st.sz[ng] = arr[sz_idx0 + (size_t)ts * a.n_blocks_q + min(ng, n_blk - 1)];     // a narrow unit's idle block re-reads block 0
    }
  };

  constexpr float kLazy = 8.f;
  float mx[HS], lsum[HS], lz[HS][NA];
#pragma unroll
  for (int i = 0; i < HS; ++i) {
    mx[i] = -INFINITY;
    lsum[i] = 0.f;
#pragma unroll
    for (int g = 0; g < NA; ++g) lz[i][g] = 0.f;
  }
  float4v acc[MT][NG][8];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ng = 0; ng < NG; ++ng)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[mt][ng][e] = float4v{0.f, 0.f, 0.f, 0.f};

  _Float16* pw = &p_lds[wave][0][0];
  float* xw = &x_lds[wave][0];

  auto process = [&](Set& st, int k) {
    const bool tok_ok = k * 32 + tl < ntok;
    make_scores(st.keys);
    // ---- online softmax statistics of the 32 tokens
    float s[HS], bm[HS];
    bool grew = false;
    // lazy maximum: probabilities up to 2^kLazy.  Quantized latents carry the scale in the fp16 weights a = p s:
    // with a scale above 128 somewhere in the set the maximum is exact (p <= 1) and a stays in range as before.
    float lazy = kLazy;
    uint16_t qs[NA], qz[NA];                                   // scales and zero-points of the lane's token
    if constexpr (I4) {
      uint32_t own = st.sz[0];
      if constexpr (NA > 1) own |= (uint32_t)st.sz[1] << 16;
      const uint32_t other = (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ 32) * 4, (int)own);
      const uint32_t sv = hp ? other : own, zv = hp ? own : other;
      bool big = false;
#pragma unroll
      for (int g = 0; g < NA; ++g) {
        qs[g] = (uint16_t)(sv >> (16 * g));
        qz[g] = (uint16_t)(zv >> (16 * g));
        big |= qs[g] > (uint16_t)0x5800;                       // fp16 bits of 128 (a negative or NaN scale also lands here)
      }
      if (__builtin_amdgcn_ballot_w64(big) != 0) lazy = 0.f;
    }
#pragma unroll
    for (int i = 0; i < HS; ++i) {
      float v;
      if constexpr (QK) v = sc_lds[wave][min(hp + 2 * i, nh - 1) * kScPitch + tl];
      else v = st.sc[i][0];
      if constexpr (TWO) v += two[i] ? st.sc[i][1] : 0.f;
      s[i] = (tok_ok && hp + 2 * i < nh && k * 32 + tl < lim[i]) ? v : -INFINITY;
      bm[i] = half_wave_max(s[i]);
      grew |= bm[i] > mx[i] + lazy;
    }
    if (__builtin_amdgcn_ballot_w64(grew) != 0) {             // uniform: some head's running maximum rises
#pragma unroll
      for (int i = 0; i < HS; ++i) {
        const float mn = fmaxf(mx[i], bm[i]);
        const float al = mx[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mx[i] - mn);
        mx[i] = mn;
        lsum[i] *= al;
#pragma unroll
        for (int g = 0; g < NA; ++g) lz[i][g] *= al;
        if (tl == 0) {
          xw[hp + 2 * i] = al;
          if constexpr (kPair) xw[4 + hp + 2 * i] = al;       // rows 4 .. 7: the same heads under block 1
        }
      }
      wave_lds_fence();
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const float4v al = *reinterpret_cast<const float4v*>(xw + mt * 16 + 4 * kq);   // accumulator rows 4*kq + 0..3
#pragma unroll
        for (int ng = 0; ng < NG; ++ng)
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[mt][ng][e] *= al;
      }
      wave_lds_fence();
    }
#pragma unroll
    for (int i = 0; i < HS; ++i) {
      const float p = s[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(s[i] - mx[i]);
      const int slot = (hp + 2 * i) * kPitch + tl;
      if constexpr (!I4) {
        const _Float16 ph = (_Float16)p;
        lsum[i] += (float)ph;                                  // the weights that enter the contraction
        pw[slot] = ph;
      } else {
        lsum[i] += p;
#pragma unroll
        for (int g = 0; g < NA; ++g) {
          const float sc = F16::to_float(qs[g]);
          const float zp = F16::to_float(qz[g]);
          const _Float16 ah = (_Float16)(p * sc);
          lz[i][g] = fmaf((float)ah, zp, lz[i][g]);
          pw[kPair ? slot + g * 4 * kPitch : g * (MT * 16 * kPitch) + slot] = ah;
        }
      }
    }
    wave_lds_fence();
    half8 pa[NT][MT];
#pragma unroll
    for (int g = 0; g < NT; ++g)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        pa[g][mt] = *reinterpret_cast<const half8*>(pw + g * (MT * 16 * kPitch) + (mt * 16 + n) * kPitch + 8 * kq);
    wave_lds_fence();

    // ---- transposed latents as B operands, 8 accumulator sets per 128-column block
#pragma unroll
    for (int ng = 0; ng < NG; ++ng) {
      const Blk& bl = st.blk[ng];
      uint32_t o[8][4];                                        // [channel e of the chunk][token pair]
#pragma unroll
      for (int jp = 0; jp < 4; ++jp) {
        if constexpr (!I4) {
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            // perm(hi_src, lo_src, sel): selector bytes 0-3 pick from lo_src, 4-7 from hi_src
            uint32_t lo = __builtin_amdgcn_perm(bl.h[2 * jp + 1][d], bl.h[2 * jp][d], 0x05040100u);
            uint32_t hi = __builtin_amdgcn_perm(bl.h[2 * jp + 1][d], bl.h[2 * jp][d], 0x07060302u);
            if constexpr (kIsBf16) {
              lo = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__builtin_bit_cast(float, lo << 16),
                                                                           __builtin_bit_cast(float, lo & 0xffff0000u)));
              hi = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__builtin_bit_cast(float, hi << 16),
                                                                           __builtin_bit_cast(float, hi & 0xffff0000u)));
            }
            o[2 * d][jp] = lo;
            o[2 * d + 1][jp] = hi;
          }
        } else {
          uint32_t ca = bl.h[2 * jp][0], cb = bl.h[2 * jp + 1][0];
          if constexpr (bits != 4) {
            ca = expand_low_bits(ca, bl.h[2 * jp][QB == 3 ? 1 : 0], QB == 3);
            cb = expand_low_bits(cb, bl.h[2 * jp + 1][QB == 3 ? 1 : 0], QB == 3);
          }
          // Four channels of both tokens side by side (token a's 16 bits of codes below token b's): the codes of
          // channel u of the two tokens are then 16 bits apart, i.e. in the two halves of one operand register.
          // Masked in place they are the subnormal fp16 numbers c 2^-24 (channels 0 and 2 of the four, after a
          // shift by 8 for the latter) and c 2^-20 (channels 1 and 3); the powers of two are undone at the write-out.
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const uint32_t x = __builtin_amdgcn_perm(cb, ca, half ? 0x07060302u : 0x05040100u), x8 = x >> 8;
            o[4 * half + 0][jp] = x & 0x000f000fu;
            o[4 * half + 1][jp] = x & 0x00f000f0u;
            o[4 * half + 2][jp] = x8 & 0x000f000fu;
            o[4 * half + 3][jp] = x8 & 0x00f000f0u;
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint4v bw = {o[e][0], o[e][1], o[e][2], o[e][3]};
        const half8 bop = __builtin_bit_cast(half8, bw);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt][ng][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa[NT > 1 ? ng : 0][mt], bop, acc[mt][ng][e], 0, 0, 0);
      }
    }
  };

  // ---- kDepth register sets in turn: the loads of the next kDepth - 1 sets are in flight while one is
  // consumed.  Every request is unconditional (past the last set the clamped addresses re-read the last
  // token, and nothing consumes them): with a request under a branch the wait in front of process() would
  // have to cover both ways of reaching it, i.e. every load in flight, and nothing would be prefetched.
  // (Three and four sets for quantized latents, whose sets are a quarter of the bytes, measured 5 - 10 % slower,
  // and 2-bit codes take as long as 4-bit ones: that kernel is bound by its instruction stream, not by bytes in flight.)
  constexpr int kDepth = kPair ? PALU_PV_PAIR_DEPTH : 2;
  Set ring[kDepth];
#pragma unroll
  for (int d = 0; d < kDepth - 1; ++d) issue(ring[d], d);
  for (int k = 0; k < n_sets; k += kDepth) {
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
      issue(ring[(d + kDepth - 1) % kDepth], k + d + kDepth - 1);
      if (d == 0 || k + d < n_sets) process(ring[d], k + d);      // uniform
    }
  }

  // ---- results of the split
#pragma unroll
  for (int i = 0; i < HS; ++i) {
    const float ls = half_wave_sum(lsum[i]);
    const int hh = hp + 2 * i;
    if (tl == 0 && hh < nh && u.write_ml) {
      float* ml = a.ml_part + (((size_t)b * a.n_split + split) * m.n_heads + h0 + hh) * 2;
      ml[0] = mx[i];
      ml[1] = ls;
    }
    if constexpr (I4) {
#pragma unroll
      for (int g = 0; g < NA; ++g) {
        const float zs = half_wave_sum(lz[i][g]);
        if (tl == 0) xw[hh * NA + g] = zs;
      }
    }
  }
  if constexpr (I4) wave_lds_fence();

  float* op = a.o_part + ((size_t)b * a.n_split + split) * a.o_stride;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (kPair && kq != (n >> 3)) continue;                  // rows 4 kq + r: block kq's scale; the lane's chunks are in block n / 8
      const int hh = kPair ? r : mt * 16 + 4 * kq + r;        // accumulator row = head of the unit
      if (hh >= nh) continue;
      const int h = h0 + hh;
      const int j = group_of(m, h);
      const int lo = m.v_off[j], hi = m.v_off[j + 1];
      float* oh = op + o_head_off(m, h) - lo;
#pragma unroll
      for (int ng = 0; ng < NG; ++ng) {
        const int chunk = kPair ? 2 * n + ng : ng * 16 + n;
        const int col = c0 + chunk * 8;
        if (chunk >= lpt || col < lo || col >= hi) continue;   // a head keeps the columns of its own group
        // quantized: acc = sum a c 2^-24 (even channels of the chunk) or sum a c 2^-20 (odd), zt = sum a z
        const float zt = I4 ? xw[hh * NA + (kPair ? n >> 3 : ng)] : 0.f;
        const float g0 = I4 ? 16777216.f : 1.f, g1 = I4 ? 1048576.f : 1.f;
        float4v v0, v1;
        v0.x = fmaf(g0, acc[mt][ng][0][r], -zt); v0.y = fmaf(g1, acc[mt][ng][1][r], -zt);
        v0.z = fmaf(g0, acc[mt][ng][2][r], -zt); v0.w = fmaf(g1, acc[mt][ng][3][r], -zt);
        v1.x = fmaf(g0, acc[mt][ng][4][r], -zt); v1.y = fmaf(g1, acc[mt][ng][5][r], -zt);
        v1.z = fmaf(g0, acc[mt][ng][6][r], -zt); v1.w = fmaf(g1, acc[mt][ng][7][r], -zt);
        *reinterpret_cast<float4v*>(oh + col) = v0;
        *reinterpret_cast<float4v*>(oh + col + 4) = v1;
      }
    }
  }
}

template <typename T, int HS, int NG, int QB, bool TWO>
__global__ __launch_bounds__(256, (QB != 0 && HS <= 2) ? 2 : 1) void pv_kernel(PvArgs a) {
  pv_body<T, HS, NG, QB, TWO, false>(a);
}
template <typename T, int HS, int NG, int QB>
__global__ __launch_bounds__(256, (QB != 0 && HS <= 2) ? 2 : 1) void stream_kernel(StreamArgs a) {
  pv_body<T, HS, NG, QB, false, true>(a);
}

namespace {

// units of more than 4 heads: unquantized only (nullptr otherwise)
template <typename T, int QB>
StreamFn stream_fn_t(int cls) {
  if (cls == 0) return stream_kernel<T, 2, 1, QB>;
  if (cls == 1) return stream_kernel<T, 2, 2, QB>;
  if constexpr (QB == 0) return cls == 2 ? stream_kernel<T, 8, 1, QB> : stream_kernel<T, 8, 2, QB>;
  return nullptr;
}

template <typename T, int QB, bool TWO>
PvFn pv_fn_t(int cls) {
  switch (cls) {
    case 0: return pv_kernel<T, 2, 1, QB, TWO>;
    case 1: return pv_kernel<T, 2, 2, QB, TWO>;
    case 2: return pv_kernel<T, 8, 1, QB, TWO>;
    default: return pv_kernel<T, 8, 2, QB, TWO>;
  }
}
template <bool TWO>
PvFn pv_fn_p(int act, int bits, int cls) {
  if (bits == 4) return pv_fn_t<F16, 4, TWO>(cls);
  if (bits == 3) return pv_fn_t<F16, 3, TWO>(cls);
  if (bits == 2) return pv_fn_t<F16, 2, TWO>(cls);
  return act == PALU_F16 ? pv_fn_t<F16, 0, TWO>(cls) : pv_fn_t<BF16, 0, TWO>(cls);
}
}  // namespace

PvFn pv_fn(int act, int bits, int cls, bool two_planes) {
  return two_planes ? pv_fn_p<true>(act, bits, cls) : pv_fn_p<false>(act, bits, cls);
}

StreamFn stream_fn(int act, int bits, int cls) {
  if (bits == 4) return stream_fn_t<F16, 4>(cls);
  if (bits == 3) return stream_fn_t<F16, 3>(cls);
  if (bits == 2) return stream_fn_t<F16, 2>(cls);
  return act == PALU_F16 ? stream_fn_t<F16, 0>(cls) : stream_fn_t<BF16, 0>(cls);
}

int launch_plane_sum(const PlaneSumArgs& a, int batch, hipStream_t s) {
  hipLaunchKernelGGL(plane_sum_kernel, dim3((unsigned)((a.seq_len + 255) / 256), (unsigned)a.n_heads, (unsigned)batch), dim3(256), 0, s, a);
  return hipGetLastError() == hipSuccess ? PALU_OK : PALU_ERR_HIP;
}

}  // namespace palu
