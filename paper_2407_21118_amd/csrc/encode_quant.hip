// Cache-append side: down-projection h = x A (Sec. 3.1) for a handful of new
// tokens, and the 4-bit asymmetric quantizer of Appendix A.
//
// At decode time the projection reads all of A (d x R) for n_tok = batch
// tokens: a weight-streaming problem.  Up to 63 tokens it is a split-K product on the
// matrix cores (the weights are read once whatever the number of tokens), followed by a
// small reduction that rounds once and scatters the rows.

#pragma once

#include "palu_dev.h"

namespace palu {

constexpr int kEncRows = 256;     // rows of A per workgroup, a quarter of them per wavefront (two k-steps of 32)
constexpr int kEncCols = 128;     // columns of A per workgroup

struct EncodeSide {
  const uint16_t* A;       // [d, R]
  float* partial;          // [k_splits][n_tok][R]
  uint16_t* latent;
  long long row_stride;
  int R;
  uint8_t* codes;          // fused quantization (GEMM path only): packed codes, rows of R/2 bytes ...
  uint16_t* scale;         // ... and the fp16 (scale, zero) pairs, rows of R/128
  uint16_t* zero;
};
// Memory that the next launch begins by reading (a decode step: B_k, which every workgroup of the score kernel loads before it
// can do anything): each thread of the projection's first launch requests 16 bytes of it and drops them, so that the
// next launch finds them in the caches.  That is 4 KiB a workgroup, from the start of B_k on: with equal ranks on both sides all of it for
// groups of 4 heads, half of it for groups of 8, an eighth for one group of 32.  Worth 0.2 .. 1.9 us a step with B_k out of the caches
// (rank 256 in groups of 4: 1 x 512 tokens 39.0 -> 37.5, 8 x 700 56.3 -> 54.4), 0 .. 1.0 for one group of 32, nothing (+-0.4) with B_k in them.
// n_words: 16-byte words, 0: nothing to fetch.
struct WarmArgs {
  const uint4v* p;
  unsigned n_words;
};
__device__ __forceinline__ uint4v warm_request(const WarmArgs& w, unsigned wg) {
  uint4v v = {0, 0, 0, 0};
  const unsigned i = wg * 256 + threadIdx.x;
  if (i < w.n_words) v = w.p[i];
  return v;
}
__device__ __forceinline__ void warm_done(const uint4v& v) { asm volatile("" :: "v"(v)); }

struct EncodeArgs {
  const uint16_t* x;       // [n_tok, d]
  const int32_t* dst_row;
  EncodeSide side[2];      // key and value caches; blockIdx.z selects (one launch may cover both)
  int n_tok, d, k_splits;
};

// The prompt-sized projection (encode_gemm.hip, compiled on its own): C[n_tok, R] = X A on the matrix
// cores for the one or two sides of `a`, quantized in place of stored when `quant`.
// tile_opt: token rows per workgroup (0 = by the number of tokens); n_cu: compute units of the device.
int launch_encode_gemm_tiles(int act, const EncodeArgs& a, int max_R, int n_sides, bool quant, int tile_opt, int n_cu,
                             hipStream_t s);

// Split-K projection of up to 16 MT tokens.  Bound by the HBM stream of A: 32 MiB for a 7B-shaped layer whatever the
// number of tokens.  (The vector-ALU form this replaces took 8 tokens per pass over weights kept in registers and wrote
// 64 partial sums per output: 48 tokens of a 7B-shaped layer took 40 us + 9 us for the sums, 16 tokens 19 + 5 us.)
//
// A workgroup takes 256 rows of A (k) x 128 columns, a wavefront 64 of the rows.  A is column-contiguous while the
// matrix cores want 8 consecutive k of one column per lane: a lane loads the same 8-column chunk of 8 consecutive rows
// and transposes the 8 x 8 block in registers (one byte permute per operand register, as the value kernel does with its
// latents), so that column e of every chunk is the operand of the e-th of 8 accumulator sets.  All 16 loads of a
// wavefront (16 KiB) go out before anything else; a 7B-shaped layer is 512 workgroups, two to a compute unit, i.e. all
// of A is in flight at once.  The four wavefronts' sums meet in LDS, so that a workgroup writes one partial sum per
// output: d / 256 of them per output in all, summed in a fixed order by encode_finish_kernel.
//
// grid (ceil(max R / 128), ceil(d / 256), sides), 256 threads.
// (bx, by, bz): the workgroup's position in that grid (the kernel below passes blockIdx; the fused
// first launch of a decode step runs the same body next to the query fold)
// while_loading(): work of the whole workgroup that is independent of the projection, run after the
// weight loads have been issued, in the shadow of their latency (the fused decode step folds the query there)
struct NoExtraWork {
  __device__ __forceinline__ void operator()() const {}
};
template <typename T, int MT, typename Extra = NoExtraWork>
__device__ __forceinline__ void encode_partial_body(const EncodeArgs& a, int bx, int by, int bz, Extra while_loading = Extra{}) {
  constexpr int kPitch = kEncCols + 4;            // floats per token row: the 8-float stores of the four token quads hit distinct banks
  __shared__ __attribute__((aligned(16))) float red[4][16 * kPitch];
  const EncodeSide sd = a.side[bz];
  if (bx * kEncCols >= sd.R) {                    // uniform
    while_loading();
    return;
  }
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 15, kq = lane >> 4;        // column chunk (B), token (A) or accumulator column; k-octet or token quad
  const int k0 = by * kEncRows + wave * (kEncRows / 4);
  const bool k_ok = k0 < a.d;                     // wavefront-uniform: d is a multiple of 128, a wavefront's 64 rows are all in or all out
  const int kw = k_ok ? k0 : 0;
  const int c0 = bx * kEncCols + n * 8;
  const int cc = min(c0, sd.R - 8);               // R is a multiple of 32: a chunk is all in or all out; clamped ones are never stored

  // activations (A operand: token 16 mt + n, k-octet kq of the step) ahead of the weights, which are the long stream
  typename T::vec8 xa[MT][2];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int s = 0; s < 2; ++s)
      xa[mt][s] = *reinterpret_cast<const typename T::vec8*>(a.x + (size_t)min(16 * mt + n, a.n_tok - 1) * a.d + kw + 32 * s + 8 * kq);
  uint4v w[2][8];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int j = 0; j < 8; ++j)
      w[s][j] = *reinterpret_cast<const uint4v*>(sd.A + (size_t)(kw + 32 * s + 8 * kq + j) * sd.R + cc);
  while_loading();

  float4v acc[MT][8];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[mt][e] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      uint4v t;                                   // column e of the chunk over the 8 rows, as four (k, k + 1) pairs
#pragma unroll
      for (int jp = 0; jp < 4; ++jp)
        t[jp] = __builtin_amdgcn_perm(w[s][2 * jp + 1][e >> 1], w[s][2 * jp][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
      const typename T::vec8 b = __builtin_bit_cast(typename T::vec8, t);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        if constexpr (__is_same(T, F16)) acc[mt][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[mt][s], b, acc[mt][e], 0, 0, 0);
        else acc[mt][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[mt][s], b, acc[mt][e], 0, 0, 0);
      }
    }
  }

  // accumulator e, entry r: token 16 mt + 4 kq + r, column c0 + e.  The wavefronts' tiles meet in LDS, 16 tokens at a time.
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    if (mt > 0) __syncthreads();                  // the previous 16 tokens have been summed
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float* dst = &red[wave][(4 * kq + r) * kPitch + n * 8];
      // a wavefront without rows contributes zeros, selected: its sums over the rows it re-read may be infinite
      const float4v none = {0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<float4v*>(dst) = k_ok ? float4v{acc[mt][0][r], acc[mt][1][r], acc[mt][2][r], acc[mt][3][r]} : none;
      *reinterpret_cast<float4v*>(dst + 4) = k_ok ? float4v{acc[mt][4][r], acc[mt][5][r], acc[mt][6][r], acc[mt][7][r]} : none;
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int id = x * 256 + tid, tok = id >> 5, c4 = (id & 31) * 4;
      float4v s = *reinterpret_cast<const float4v*>(&red[0][tok * kPitch + c4]);
#pragma unroll
      for (int v = 1; v < 4; ++v) s += *reinterpret_cast<const float4v*>(&red[v][tok * kPitch + c4]);
      const int t = 16 * mt + tok, col = bx * kEncCols + c4;
      if (t < a.n_tok && col < sd.R) *reinterpret_cast<float4v*>(sd.partial + ((size_t)by * a.n_tok + t) * sd.R + col) = s;
    }
  }
}

template <typename T, int MT>
__global__ __launch_bounds__(256, MT <= 2 ? 2 : 1) void encode_partial_kernel(EncodeArgs a, WarmArgs w) {
  const uint4v warm = warm_request(w, blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z));
  encode_partial_body<T, MT>(a, blockIdx.x, blockIdx.y, blockIdx.z);
  warm_done(warm);
}

// Sums the split-K partials in a fixed order, rounds once, scatters the rows.
// Workgroup = 256 columns of one token; thread = (quarter of the splits, 4 columns).
// grid (ceil(max R / 256), n_tok, sides), 256 threads.
template <typename T>
__global__ __launch_bounds__(256) void encode_finish_kernel(EncodeArgs a) {
  __shared__ __attribute__((aligned(16))) float part[4][256];
  const EncodeSide sd = a.side[blockIdx.z];
  if ((int)blockIdx.x * 256 >= sd.R) return;      // uniform
  const int tid = threadIdx.x;
  const int c = blockIdx.x * 256 + (tid & 63) * 4, t = blockIdx.y, sub = tid >> 6;
  const int per = (a.k_splits + 3) / 4;
  asm volatile("" :: "s"(sd.partial), "s"(sd.latent), "s"(sd.row_stride), "s"(sd.R), "s"(a.dst_row), "s"(a.n_tok), "s"(a.k_splits));      // one round trip
  const long long row = a.dst_row ? a.dst_row[t] : t;      // ... and this beside the sums, not behind them
  float4v s = {0.f, 0.f, 0.f, 0.f};
  if (c < sd.R) {
    const float* p = sd.partial + (size_t)t * sd.R + c;
#pragma unroll 4
    for (int ks = sub * per; ks < min((sub + 1) * per, a.k_splits); ++ks)
      s += *reinterpret_cast<const float4v*>(p + (size_t)ks * a.n_tok * sd.R);
  }
  *reinterpret_cast<float4v*>(&part[sub][(tid & 63) * 4]) = s;
  __syncthreads();
  const int cc = tid * 2;
  if (tid < 128 && (int)blockIdx.x * 256 + cc < sd.R) {
    const float s0 = (part[0][cc] + part[1][cc]) + (part[2][cc] + part[3][cc]);
    const float s1 = (part[0][cc + 1] + part[1][cc + 1]) + (part[2][cc + 1] + part[3][cc + 1]);
    uint32_t* dst = reinterpret_cast<uint32_t*>(sd.latent + row * sd.row_stride + blockIdx.x * 256 + cc);
    *dst = (uint32_t)T::from_float(s0) | ((uint32_t)T::from_float(s1) << 16);
  }
}

// ---- the same projection from transposed weights At [R, d] (column c of A contiguous): a wavefront owns
// kTCols columns and all of k, so a column's sum is finished inside the wavefront, in one launch, with no
// partial sums in memory.  Workgroup = 4 wavefronts = 4 kTCols columns of one side; every weight load of
// the wavefront (kTCols x 8 chunks of 1 KiB) goes out before anything else.
constexpr int kTCols = 2;          // columns per wavefront (4 for passes of 4 or 8 tokens was slower: half the workgroups)
constexpr int kTBlock = 4096;      // k per batch of loads: 8 chunks of 64 lanes x 8
struct EncodeTArgs {
  const uint16_t* x;               // [n_tok, d]
  const int32_t* dst_row;
  const uint16_t* At[2];           // [R, d]
  uint16_t* latent[2];
  long long row_stride[2];
  int R[2];
  int n_tok, d, wg_side1;          // workgroups below wg_side1 work on side 0
};
// acc + sum of the 8 products of two packed 16-byte operands
template <typename T>
__device__ __forceinline__ float dot8(const uint4v& w, const uint4v& x, float acc) {
  if constexpr (__is_same(T, F16)) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t we = w[e], xe = x[e];                       // named copies: a bit cast applied to a vector element reads element 0
      acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(h2, we), __builtin_bit_cast(h2, xe), acc, false);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc = fmaf(T::to_float((uint16_t)(x[e] & 0xffffu)), T::to_float((uint16_t)(w[e] & 0xffffu)), acc);
      acc = fmaf(T::to_float((uint16_t)(x[e] >> 16)), T::to_float((uint16_t)(w[e] >> 16)), acc);
    }
  }
  return acc;
}

// wg_id: the workgroup's index in the projection's grid of wg_side1 + ceil(R_v / (4 kTCols)) workgroups
// while_loading(): as for encode_partial_body
template <typename T, int TOK, typename Extra = NoExtraWork>
__device__ __forceinline__ void encode_t_body(const EncodeTArgs& a, int wg_id, Extra while_loading = Extra{}) {
  extern __shared__ __attribute__((aligned(16))) unsigned char enct_lds[];
  uint16_t* xs = reinterpret_cast<uint16_t*>(enct_lds);          // [TOK][d]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int side = wg_id >= a.wg_side1 ? 1 : 0;
  const int wg = wg_id - (side ? a.wg_side1 : 0);
  const int R = a.R[side];
  const int c0 = (wg * 4 + wave) * kTCols;                       // R is a multiple of 32: a wavefront's columns are all in or all out
  const bool cols_ok = c0 < R;
  const uint16_t* At = a.At[side] + (size_t)min(c0, R - kTCols) * a.d;
  for (int tb = 0; tb < a.n_tok; tb += TOK) {
    int dst[TOK];                                                // where the rows go, known before the sums are
#pragma unroll
    for (int t = 0; t < TOK; ++t) dst[t] = a.dst_row ? a.dst_row[min(tb + t, a.n_tok - 1)] : tb + t;
    float acc[kTCols][TOK];
#pragma unroll
    for (int c = 0; c < kTCols; ++c)
#pragma unroll
      for (int t = 0; t < TOK; ++t) acc[c][t] = 0.f;
    for (int kb = 0; kb < a.d; kb += kTBlock) {
      // One or two tokens: a lane needs only its own k of x, the same for every column, and takes them straight
      // from memory ahead of the weights (loads return in order: behind the weights they would cost a second
      // round trip).  More tokens would not fit the registers and go through LDS.
      constexpr bool kDirect = TOK <= 2;
      uint4v xd[kDirect ? TOK : 1][8];
      if constexpr (kDirect) {
#pragma unroll
        for (int t = 0; t < TOK; ++t)
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int k = kb + (i * 64 + lane) * 8;
            xd[t][i] = (k < a.d && tb + t < a.n_tok) ? *reinterpret_cast<const uint4v*>(a.x + (size_t)(tb + t) * a.d + k) : uint4v{0, 0, 0, 0};
          }
      }
      uint4v w[kTCols][8];
#pragma unroll
      for (int c = 0; c < kTCols; ++c)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int k = kb + (i * 64 + lane) * 8;
          w[c][i] = k < a.d ? *reinterpret_cast<const uint4v*>(At + (size_t)c * a.d + k) : uint4v{0, 0, 0, 0};
        }
      if (kb == 0) {
        if (tb == 0) while_loading();
        if constexpr (!kDirect) {
          __syncthreads();                                       // the previous pass has read xs
          const int nt = min(TOK, a.n_tok - tb);
          for (int i = tid; i < TOK * (a.d >> 3); i += 256) {
            const int t = i / (a.d >> 3), k8 = i - t * (a.d >> 3);
            reinterpret_cast<uint4v*>(xs)[i] = t < nt ? reinterpret_cast<const uint4v*>(a.x + (size_t)(tb + t) * a.d)[k8] : uint4v{0, 0, 0, 0};
          }
          __syncthreads();
        }
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = kb + (i * 64 + lane) * 8;
        if (k >= a.d) continue;
#pragma unroll
        for (int t = 0; t < TOK; ++t) {
          uint4v xv;
          if constexpr (kDirect) xv = xd[t][i];
          else xv = *reinterpret_cast<const uint4v*>(xs + (size_t)t * a.d + k);
#pragma unroll
          for (int c = 0; c < kTCols; ++c) acc[c][t] = dot8<T>(w[c][i], xv, acc[c][t]);
        }
      }
    }
#pragma unroll
    for (int c = 0; c < kTCols; ++c)
#pragma unroll
      for (int t = 0; t < TOK; ++t) {
        float v = acc[c][t];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0 && cols_ok && tb + t < a.n_tok) {
          a.latent[side][(long long)dst[t] * a.row_stride[side] + c0 + c] = T::from_float(v);
        }
      }
  }
}

template <typename T, int TOK>
__global__ __launch_bounds__(256) void encode_t_kernel(EncodeTArgs a, WarmArgs w) {
  const uint4v warm = warm_request(w, blockIdx.x);
  encode_t_body<T, TOK>(a, blockIdx.x);
  warm_done(warm);
}

// The quantizer of Appendix A with B = 4 (s = (max-min)/(2^B-1), z = round(-min/s),
// code = clamp(round(x/s) + z, 0, 2^B-1)) for one (token, 128-channel block).
// Every arithmetic step is a single IEEE float32 operation so the integer codes are
// reproducible bit for bit; scale and zero are stored as fp16 and used as stored.
struct QuantParams {
  float sf, zf, top;
  uint16_t s16, z16;
};
// top = 2^B - 1: 15 for the 4-bit cache, 7 and 3 for the 3- and 2-bit settings of Sec. 4.4
__device__ __forceinline__ QuantParams quant_params(float mn, float mx, float top = 15.0f) {
  QuantParams p;
  p.top = top;
  const float s32 = __fdiv_rn(__fsub_rn(mx, mn), top);
  p.s16 = F16::from_float(s32);
  if ((p.s16 & 0x7fffu) == 0) p.s16 = 0x3c00u;                  // s == 0 -> 1
  p.sf = F16::to_float(p.s16);
  float z = rintf(__fdiv_rn(-mn, p.sf));
  z = fminf(fmaxf(z, -65504.0f), 65504.0f);
  p.z16 = F16::from_float(z);
  p.zf = F16::to_float(p.z16);
  return p;
}
__device__ __forceinline__ uint32_t quant_code(float x, const QuantParams& p) {
  return (uint32_t)fminf(fmaxf(__fadd_rn(rintf(__fdiv_rn(x, p.sf)), p.zf), 0.0f), p.top);
}

struct QuantArgs {
  const uint16_t* latent;
  uint8_t* codes;
  uint16_t* scale;
  uint16_t* zero;
  const int32_t* dst_row;     // output row of token t (NULL: t)
  long long row_stride;
  int n_tok, R, n_blocks;     // n_blocks = R / 128
  int bits;                   // 4, 3 or 2
};

// One wavefront per (token, 128-channel block); lane l owns channels 2l, 2l+1.
template <typename T>
__global__ __launch_bounds__(256) void quant_kernel(QuantArgs a) {
  asm volatile("" :: "s"(a.latent), "s"(a.codes), "s"(a.scale), "s"(a.zero), "s"(a.dst_row), "s"(a.row_stride), "s"(a.n_tok), "s"(a.R), "s"(a.n_blocks),
               "s"(a.bits));                      // one round trip
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const long long item = (long long)blockIdx.x * 4 + wave;
  if (item >= (long long)a.n_tok * a.n_blocks) return;
  int t, blk;                                     // items beyond 32 bits take the long division
  if ((long long)a.n_tok * a.n_blocks < (1LL << 31)) {
    t = (int)((unsigned)item / (unsigned)a.n_blocks);
    blk = (int)item - t * a.n_blocks;
  } else {
    t = (int)(item / a.n_blocks);
    blk = (int)(item - (long long)t * a.n_blocks);
  }
  const size_t orow = a.dst_row ? (size_t)a.dst_row[t] : (size_t)t;      // beside the latents, not behind their block's parameters
  const uint32_t raw = *reinterpret_cast<const uint32_t*>(a.latent + (size_t)t * a.row_stride + blk * 128 + lane * 2);
  const float x0 = T::to_float((uint16_t)(raw & 0xffffu));
  const float x1 = T::to_float((uint16_t)(raw >> 16));
  float mn = fminf(x0, x1), mx = fmaxf(x0, x1);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    mn = fminf(mn, __shfl_xor(mn, off, 64));
    mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  }
  const QuantParams qp = quant_params(mn, mx, (float)((1 << a.bits) - 1));
  const uint32_t c0 = quant_code(x0, qp), c1 = quant_code(x1, qp);
  if (a.bits == 4) {
    a.codes[orow * (a.R / 2) + blk * 64 + lane] = (uint8_t)(c0 | (c1 << 4));
  } else {
    // 2 bits: byte k of a row holds channels 4k .. 4k+3 (lanes 2k, 2k+1).  3 bits: the low two bits of every
    // code in that layout, then the third bits, byte k holding channels 8k .. 8k+7 (lanes 4k .. 4k+3).
    uint8_t* row = a.codes + orow * (size_t)(a.R * a.bits / 8);
    const uint32_t lo = (c0 & 3u) | ((c1 & 3u) << 2);
    const uint32_t lo_n = __shfl_xor(lo, 1, 64);
    if ((lane & 1) == 0) row[blk * 32 + (lane >> 1)] = (uint8_t)(lo | (lo_n << 4));
    if (a.bits == 3) {
      uint32_t hi = (c0 >> 2) | ((c1 >> 2) << 1);                  // 2 bits: this lane's channels
      hi |= __shfl_xor(hi, 1, 64) << 2;                            // even lanes: 4 bits
      hi |= __shfl_xor(hi, 2, 64) << 4;                            // lanes 4k: 8 bits
      if ((lane & 3) == 0) row[a.R / 4 + blk * 16 + (lane >> 2)] = (uint8_t)hi;
    }
  }
  if (lane == 0) {
    a.scale[orow * a.n_blocks + blk] = qp.s16;
    a.zero[orow * a.n_blocks + blk] = qp.z16;
  }
}

}  // namespace palu
