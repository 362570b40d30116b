// Scores and values of a run of tiles in one workgroup: score16_kernel (score16.hip) with the softmax partials and the value
// contraction of pv.hip (Eq. 4, (p H_v) B_v in latent space) behind its last tile, for unquantized latents.
//
// The two kernels use a compute unit alike (four wavefronts, one per SIMD), and the score units of whole groups are value
// units too, so the workgroup that has a run's scores can go on to its values: no launch in between (its start, the wait for the
// slowest score workgroup), and its four wavefronts, which split the run's tokens, merge their results in LDS, so that one partial result per
// run is written and merged later instead of four.  The scores are handed over through the XCD's cache (one 128-byte line
// per head and tile).  The registers are the score phase's first and the value phase's afterwards; nothing of either is kept for the other.
//
// Bound by the matrix pipe first and by the memory then (64 MiB of value latents in 12.8 us, what a plain read takes); of the
// second part each wavefront's first set of tokens is requested during the last tiles of the first, into the ring buffers of
// the tiles past the end (see kValues in score16_body.inc): 1 x 16384 tokens 65.1 -> 63.7 us a step, 1 x 65536 174.4 -> 171.0, 4 x 16384 grouped
// queries 74.6 -> 73.4.  (Touching all values a line to a lane during the whole score phase, or the last eight tiles' worth, so that
// they come from a nearer cache later, took 3 to 9 us more.)  Two launches -> this, us a step: 1 x 1024 tokens of 8 heads 21.1 -> 18.1, 1 x 16384
// 69.1 -> 63.7, 1 x 65536 in bf16 178.1 -> 171.0, 4 x 16384 of 8 key/value heads with 4 queries 81.6 -> 73.4; four queries over
// 2 x 8190, rank 128 / 384, 70.0 -> 65.5.

#pragma once

#include "score16.hip"
#include "softmax_dev.h"

namespace palu {

// LDS of the value phase behind the score phase's ring (offsets from its end); the wavefronts' partial results go into the ring
constexpr int kAttPitch = 40;                                   // halfs per probability row, see pv_kernel
constexpr int kAttX = 4 * 16 * kAttPitch * 2;                   // behind the probabilities [wavefront][16 rows]: rescaling factors
constexpr int kAttMl = kAttX + 4 * 16 * 4;                      // (max, sum) of every wavefront's rows
constexpr int kAttLim = kAttMl + 4 * 16 * 2 * 4;                // row limits of up to 32 query rows
constexpr int kAttScratch = kAttLim + 32 * 4;
constexpr int attend_lds_bytes(int width) { return score16_lds_bytes(width) + kAttScratch; }
constexpr size_t attend_partials_lds(int hs, int ng) { return (size_t)4 * 2 * hs * ng * 128 * 4; }

// HS: score slots per lane (at most 2 HS heads at a time); NG: 128-column blocks at a time.
// n_rows heads from query head row0 on (a wavefront half takes every other one), columns of the unit from block to block; rows
// 0 .. last of the run, whose first row is row0_tok of the cache (sequence b) and tok0 of the sequence.
template <typename T, int HS, int NG>
__device__ __forceinline__ void value_of_run(const AttendArgs& a, const int unit, const int n_rows, const int h_first, const int rows_per_group,
                                             const int groups, const int b, const int wg, const size_t cache_row0, const int tok0, const int last,
                                             unsigned char* lds, unsigned char* scratch, const unsigned half0, const unsigned half1) {
  constexpr bool kIsBf16 = !__is_same(T, F16);
  const AttendValue uv = a.val[unit];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, kq = lane >> 4;                      // matrix-core roles, as in pv_kernel
  const int tl = lane & 31, hp = lane >> 5;                     // softmax roles
  _Float16* pw = reinterpret_cast<_Float16*>(scratch) + wave * 16 * kAttPitch;
  float* xw = reinterpret_cast<float*>(scratch + kAttX) + wave * 16;
  float* ml_lds = reinterpret_cast<float*>(scratch + kAttMl);   // [wavefront][16][2]
  int* lim_lds = reinterpret_cast<int*>(scratch + kAttLim);         // [n_rows], counted from the run's first row
  float* o_lds = reinterpret_cast<float*>(lds);                 // [wavefront][2 HS][NG * 128]
  constexpr int kORow = NG * 128, kOWave = 2 * HS * kORow;

  // this wavefront's share of the run: whole sets of 32 tokens
  const int n_sets_run = (last >> 5) + 1;
  const int set0 = n_sets_run * wave / 4, n_sets = n_sets_run * (wave + 1) / 4 - set0;
  const unsigned row_bytes = (unsigned)a.v_row_elems * 2u;
  const unsigned last_off = (unsigned)last * row_bytes, set_bytes = 32u * row_bytes;
  const unsigned char* run_base = (const unsigned char*)a.hv + cache_row0 * row_bytes + (size_t)uv.c0 * 2;
  const int cols = groups * uv.rv;                              // of the unit

  struct Set {
    uint32_t h[NG][8][4];
    float sc[HS];
  };
  Set ring[2];
  const unsigned roff = (unsigned)(8 * kq) * row_bytes;
  const float* sc_base = a.scores + ((size_t)b * a.n_heads + h_first) * a.lpad + tok0;
  int min_lim = 0x7fffffff;                                     // smallest row limit of the unit's queries

  for (int r0 = 0; r0 < n_rows; r0 += 2 * HS) {
    const int nh = min(n_rows - r0, 2 * HS);
    for (int cb = 0; cb < cols; cb += NG * 128) {
      const int lpt = min(cols - cb, NG * 128) >> 3;            // 8-channel chunks per row
      const unsigned char* base = run_base + (size_t)cb * 2;
      unsigned coff[NG];
#pragma unroll
      for (int ng = 0; ng < NG; ++ng) coff[ng] = (unsigned)min(ng * 16 + n, lpt - 1) * 16u;
      // every request is unconditional and in bounds, as in pv_kernel
      auto issue_latents = [&](Set& st, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int ng = 0; ng < NG; ++ng)
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const uint4v v = *reinterpret_cast<const uint4v*>(base + (size_t)(min(roff + ((unsigned)j * row_bytes + (unsigned)(set0 + k) * set_bytes), last_off) + coff[ng]));
            st.h[ng][j][0] = v.x; st.h[ng][j][1] = v.y; st.h[ng][j][2] = v.z; st.h[ng][j][3] = v.w;
          }
      };
      unsigned sc_off[HS];                                      // the lane's score rows (the host keeps 32 of them below 2^32 bytes)
#pragma unroll
      for (int i = 0; i < HS; ++i) sc_off[i] = (unsigned)(r0 + min(hp + 2 * i, nh - 1)) * (unsigned)a.lpad;
      auto issue_scores = [&](Set& st, int k) __attribute__((always_inline)) {
        const unsigned ts = (unsigned)min((set0 + k) * 32 + tl, last);
#pragma unroll
        for (int i = 0; i < HS; ++i) st.sc[i] = sc_base[sc_off[i] + ts];
      };
      const bool begin = r0 == 0 && cb == 0;
      int own_lim = 0;
      if (begin && a.q_len != nullptr) {                        // each thread one query row's limit
        Meta mq;
        mq.qpk = a.m_qpk; mq.nq = a.m_nq;
        own_lim = a.q_len[b * a.m_nq + q_token(mq, h_first + min(tid, n_rows - 1))] - tok0;
      }
      if (begin) {
        // the scores of all four wavefronts, and this one's share of the values requested in place of tiles past the end
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      } else {
        issue_latents(ring[0], 0);
      }
      issue_scores(ring[0], 0);
      if (begin && a.q_len != nullptr) {
        if (tid < n_rows) lim_lds[tid] = own_lim;
        __syncthreads();
        min_lim = lim_lds[min(lane, n_rows - 1)];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) min_lim = min(min_lim, __shfl_xor(min_lim, d, 64));
        min_lim = __builtin_amdgcn_readfirstlane(min_lim);
      }
      if (begin) {                                              // set 0: half 0, and half 1 where a row has more than 128 columns
#pragma unroll
        for (int ng = 0; ng < NG; ++ng)
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const uint4v v = *reinterpret_cast<const uint4v*>(lds + (ng ? half1 : half0) + wave * 8192 + (8 * kq + j) * 256 + n * 16);
            ring[0].h[ng][j][0] = v.x; ring[0].h[ng][j][1] = v.y; ring[0].h[ng][j][2] = v.z; ring[0].h[ng][j][3] = v.w;
          }
      }

      constexpr float kLazy = 8.f;
      float mx[HS], lsum[HS];
#pragma unroll
      for (int i = 0; i < HS; ++i) {
        mx[i] = -INFINITY;
        lsum[i] = 0.f;
      }
      float4v acc[NG][8];
#pragma unroll
      for (int ng = 0; ng < NG; ++ng)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[ng][e] = float4v{0.f, 0.f, 0.f, 0.f};

      // the arithmetic of pv_kernel
      auto process = [&](Set& st, int k) __attribute__((always_inline)) {
        const int t0 = (set0 + k) * 32, t = t0 + tl;
        float s[HS], bm[HS];
        bool grew = false;
#pragma unroll
        for (int i = 0; i < HS; ++i) s[i] = (t <= last && hp + 2 * i < nh) ? st.sc[i] : -INFINITY;
        if (t0 + 32 > min_lim) {                                // uniform: some query's row limit lies in this set or before
#pragma unroll
          for (int i = 0; i < HS; ++i)
            if (t >= lim_lds[r0 + min(hp + 2 * i, nh - 1)]) s[i] = -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < HS; ++i) {
          bm[i] = half_wave_max(s[i]);
          grew |= bm[i] > mx[i] + kLazy;
        }
        if (__builtin_amdgcn_ballot_w64(grew) != 0) {           // uniform: some head's running maximum rises
#pragma unroll
          for (int i = 0; i < HS; ++i) {
            const float mn = fmaxf(mx[i], bm[i]);
            bm[i] = mx[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mx[i] - mn);
            mx[i] = mn;
            lsum[i] *= bm[i];
          }
          if (tl == 0) {
#pragma unroll
            for (int i = 0; i < HS; ++i) xw[hp + 2 * i] = bm[i];
          }
          wave_lds_fence();
          const float4v al = *reinterpret_cast<const float4v*>(xw + 4 * kq);
#pragma unroll
          for (int ng = 0; ng < NG; ++ng)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[ng][e] *= al;
          wave_lds_fence();
        }
#pragma unroll
        for (int i = 0; i < HS; ++i) {
          const float p = s[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(s[i] - mx[i]);
          const _Float16 ph = (_Float16)p;
          lsum[i] += (float)ph;                                 // the weights that enter the contraction
          pw[(hp + 2 * i) * kAttPitch + tl] = ph;
        }
        wave_lds_fence();
        const half8 pa = *reinterpret_cast<const half8*>(pw + n * kAttPitch + 8 * kq);
        wave_lds_fence();
#pragma unroll
        for (int ng = 0; ng < NG; ++ng) {
          uint32_t o[8][4];                                     // [channel e of the chunk][token pair]
#pragma unroll
          for (int jp = 0; jp < 4; ++jp)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
              uint32_t lo = __builtin_amdgcn_perm(st.h[ng][2 * jp + 1][d], st.h[ng][2 * jp][d], 0x05040100u);
              uint32_t hi = __builtin_amdgcn_perm(st.h[ng][2 * jp + 1][d], st.h[ng][2 * jp][d], 0x07060302u);
              if constexpr (kIsBf16) {
                lo = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__builtin_bit_cast(float, lo << 16), __builtin_bit_cast(float, lo & 0xffff0000u)));
                hi = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__builtin_bit_cast(float, hi << 16), __builtin_bit_cast(float, hi & 0xffff0000u)));
              }
              o[2 * d][jp] = lo;
              o[2 * d + 1][jp] = hi;
            }
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint4v bw = {o[e][0], o[e][1], o[e][2], o[e][3]};
            acc[ng][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa, __builtin_bit_cast(half8, bw), acc[ng][e], 0, 0, 0);
          }
        }
      };
      // rows of the probability tile that no head fills: zeros, so that their products are (rows 2 HS .. 15 are in nobody's slot)
      if constexpr (HS < 8) {
        for (int i = 2 * HS * kAttPitch + lane; i < 16 * kAttPitch; i += 64) pw[i] = (_Float16)0.f;
        wave_lds_fence();
      }
      for (int k = 0; k < n_sets; k += 2) {
        issue_latents(ring[1], k + 1);
        issue_scores(ring[1], k + 1);
        process(ring[0], k);
        issue_latents(ring[0], k + 2);
        issue_scores(ring[0], k + 2);
        if (k + 1 < n_sets) process(ring[1], k + 1);            // uniform
      }

      // ---- merge of the four wavefronts
#pragma unroll
      for (int i = 0; i < HS; ++i) lsum[i] = half_wave_sum(lsum[i]);
      if (tl == 0) {
#pragma unroll
        for (int i = 0; i < HS; ++i) *reinterpret_cast<float2*>(ml_lds + (wave * 16 + hp + 2 * i) * 2) = float2{mx[i], lsum[i]};
      }
      __syncthreads();
      {                                                         // lane = row
        const int row = lane & 15;
        float m = -INFINITY, l = 0.f, own = 0.f;
        float2 w4[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          w4[x] = *reinterpret_cast<const float2*>(ml_lds + (x * 16 + row) * 2);
          m = fmaxf(m, w4[x].x);
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const float f = w4[x].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(w4[x].x - m);
          l = fmaf(w4[x].y, f, l);
          own = x == wave ? f : own;
        }
        if (lane < 16) xw[lane] = own;
        if (cb == 0 && wave == 0 && lane < nh)
          *reinterpret_cast<float2*>(a.ml_part + (((size_t)b * a.n_split + wg) * a.n_heads + h_first + r0 + lane) * 2) = float2{m, l};
      }
      wave_lds_fence();
      const float4v fac = *reinterpret_cast<const float4v*>(xw + 4 * kq);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (4 * kq + r >= nh) continue;                         // accumulator row = head
#pragma unroll
        for (int ng = 0; ng < NG; ++ng) {
          float* dst = o_lds + wave * kOWave + (4 * kq + r) * kORow + (ng * 16 + n) * 8;
          *reinterpret_cast<float4v*>(dst) = float4v{acc[ng][0][r], acc[ng][1][r], acc[ng][2][r], acc[ng][3][r]} * fac[r];
          *reinterpret_cast<float4v*>(dst + 4) = float4v{acc[ng][4][r], acc[ng][5][r], acc[ng][6][r], acc[ng][7][r]} * fac[r];
        }
      }
      __syncthreads();
      float* op = a.o_part + ((size_t)b * a.n_split + wg) * a.o_stride + uv.o0;
      for (int id = tid; id < nh * (kORow / 4); id += 256) {
        const int row = id / (kORow / 4), col = (id % (kORow / 4)) * 4;
        if (col >= 8 * lpt) continue;
        const int head = r0 + row, c = cb + col - (groups == 1 ? 0 : head / rows_per_group * uv.rv);      // column inside the head's own group
        if (c < 0 || c >= uv.rv) continue;                      // a head keeps the columns of its own group
        float4v v = *reinterpret_cast<const float4v*>(o_lds + row * kORow + col);
#pragma unroll
        for (int x = 1; x < 4; ++x) v += *reinterpret_cast<const float4v*>(o_lds + x * kOWave + row * kORow + col);
        *reinterpret_cast<float4v*>(op + (size_t)head * uv.rv + c) = v;
      }
      __syncthreads();                                          // LDS is the next block's
    }
  }
}

// T, NK, G, NQ: as in score16_kernel.  grid (runs per unit and sequence, units, sequences), 256 threads, score16_lds_bytes of LDS.
#undef SCORE16_DRAIN
#define SCORE16_DRAIN (void)0                                   // value_of_run waits for them
template <typename T, int NK, int G, int NQ>
__global__ __launch_bounds__(256) void attend16_kernel(AttendArgs a) {
  constexpr int QB = 0;
  constexpr bool FLAT = false, kValues = true;
  const int wg = blockIdx.x, n_wg = a.n_wg, unit = blockIdx.y, seq = blockIdx.z, run = a.run, run_more = a.run_more;
#include "score16_body.inc"
  // at most 4 heads with a query each, else 4 NQ query rows, 16 at a time
  constexpr int HS = NQ == 1 ? 2 : (NQ == 2 ? 4 : 8);
  static_assert(attend_partials_lds(HS, 2) <= (size_t)score16_lds_bytes(kWidth), "the partial results live in the score phase's ring");
  const int qpk = NQ == 1 ? 1 : a.m_qpk;
  const int rows_per_group = (G == 1 ? u.nh : u.s) * qpk;
  if (G * a.val[unit].rv > 128) value_of_run<T, HS, 2>(a, unit, u.nh * qpk, u.h0 * qpk, rows_per_group, G, b, wg, row0, off * kTile, rel_last, lds, lds + score16_lds_bytes(kWidth),
                                                     ring[1], ring[2]);
  else value_of_run<T, HS, 1>(a, unit, u.nh * qpk, u.h0 * qpk, rows_per_group, G, b, wg, row0, off * kTile, rel_last, lds, lds + score16_lds_bytes(kWidth),
                                                     ring[1], ring[2]);
}
#undef SCORE16_DRAIN
#define SCORE16_DRAIN __builtin_amdgcn_s_waitcnt(vmcnt_imm(0))

}  // namespace palu
