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
// second part each wavefront's first latents are requested during the last tiles of the first, into the ring buffers of
// the tiles past the end (see kValues in score16_body.inc): 1 x 16384 tokens 65.1 -> 63.7 us a step, 1 x 65536 174.4 -> 171.0, 4 x 16384 grouped
// queries 74.6 -> 73.4.  (Touching all values a line to a lane during the whole score phase, or the last eight tiles' worth, so that
// they come from a nearer cache later, took 3 to 9 us more.)  The rest goes through LDS as well, four halves of 8 KiB per wavefront in turn:
// through registers, two sets in turn, the first set's successor could be asked for only behind the hand-over of the scores, and the
// weights of a run through several sequences did not fit beside them (1 x 16384 63.7 -> 60, 4 x 16384 grouped queries 73.4 -> 69).
//
// Two launches -> this, us a step: 1 x 1024 tokens of 8 heads 21.7 -> 18.2, 1 x 16384 68 -> 61, 1 x 65536 in bf16 179 -> 173, 4 x 16384 of
// 8 key/value heads with 4 queries 80.5 -> 69.5, four queries over 2 x 8190, rank 128 / 384, 69.9 -> 66.5; runs through all sequences: 48
// sequences of 1022 .. 2043 tokens 233 -> 207, 8 of 8191 .. 16384, rank 64 per head, 198 -> 193 (segments of at most 32 / 16 tiles instead of 64, so that more
// of the chip reads while the rest multiplies: 207 -> 210 / 218 and 193 -> 199 / 211: a change of segment costs more than that gives).

#pragma once

#include "score16.hip"
#include "softmax_dev.h"

namespace palu {

// LDS of the value phase behind the score phase's ring (offsets from its end); latents and partial results lie in the ring
constexpr int kAttPitch = 40;                                   // halfs per probability row, see pv_kernel
constexpr int kAttX = 4 * 16 * kAttPitch * 2;                   // behind the probabilities [wavefront][16 rows]: rescaling factors
constexpr int kAttMl = kAttX + 4 * 16 * 4;                      // (max, sum) of every wavefront's rows
constexpr int kAttLim = kAttMl + 4 * 16 * 2 * 4;                // row limits of up to 32 query rows
constexpr int kAttRun = kAttLim + 32 * 4;                       // (max, sum) so far of up to 32 query rows, and the factors of what they had
constexpr int kAttSc = kAttRun + 32 * 2 * 4 + 16 * 4;           // scores of two sets of every wavefront
constexpr int attend_scratch_bytes(int hs) { return kAttSc + 4 * 2 * hs * 256; }
// Score slots per lane: 2 HS query rows at a time.  Units of one head, or two with two queries, have no more than 4 rows, as many as four heads with a query
// each, and the slots decide what the softmax costs (eight for 4 rows: 11 us over 64 tiles): 4 queries over 64 tiles, one head of rank 64 to
// a unit, 64 / 96 / 160 value columns 112 / 112 / 121 -> 98 / 99 / 109 us a step (two launches 101 / 104 / 117), rank 256 178 / 177 / 188 -> 169 / 168 / 178.
constexpr int attend_hs(int nq, int rows) { return nq == 1 || rows <= 4 ? 2 : (nq == 2 ? 4 : 8); }
constexpr int attend_lds_bytes(int width, int hs) { return score16_lds_bytes(width) + attend_scratch_bytes(hs); }
constexpr size_t attend_partials_lds(int hs, int ng) { return (size_t)4 * 2 * hs * ng * 128 * 4; }

// A segment (tiles of one sequence) and the unit whose values it is about
struct ValueSegment {
  int n_rows, h_first;             // query heads, the first of them
  int rows_per_group, groups;
  int c0, rv, o0;                  // AttendValue
  int b, tok0, last;               // sequence, its first row here, last row counted from that
  bool more;                       // the workgroup's partial result of this sequence is added to
  size_t slot, cache_row0;         // place of the partial result; row of the cache
};

// Heads r0 .. r0 + 2 HS - 1 of the unit and columns cb .. cb + 128 NG - 1 of its latents (HS: score slots per lane).
//
// A wavefront takes whole sets of 32 tokens; it shares nothing until the merge.  Latents and scores come by LDS-direct requests: a half (32 tokens
// of 128 columns, eight requests) to one of four 8 KiB places, halves in turn, the first PRE of them requested by the score phase in place
// of tiles past the segment's end.  So 16 .. 32 KiB are in flight per wavefront, and the registers hold only what is being
// multiplied: the weights keep theirs where more segments follow.
template <typename T, int HS, int NG, int PRE>
__device__ __forceinline__ void value_block(const AttendArgs& a, const ValueSegment& v, const int r0, const int cb, unsigned char* lds,
                                            unsigned char* scratch, const unsigned (&ring)[4]) {
  constexpr bool kIsBf16 = !__is_same(T, F16);
  const int last = v.last;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, kq = lane >> 4;                      // matrix-core roles, as in pv_kernel
  const int tl = lane & 31, hp = lane >> 5;                     // softmax roles
  _Float16* pw = reinterpret_cast<_Float16*>(scratch) + wave * 16 * kAttPitch;
  float* xw = reinterpret_cast<float*>(scratch + kAttX) + wave * 16;
  float* ml_lds = reinterpret_cast<float*>(scratch + kAttMl);   // [wavefront][16][2]
  int* lim_lds = reinterpret_cast<int*>(scratch + kAttLim);     // [n_rows], counted from the segment's first row
  float* run_lds = reinterpret_cast<float*>(scratch + kAttRun); // [n_rows][2]
  float* old_lds = run_lds + 64;                                // [16]
  const float* sc_lds = reinterpret_cast<const float*>(scratch + kAttSc) + wave * 2 * HS * 64;      // [2 sets][HS][lane]
  float* o_lds = reinterpret_cast<float*>(lds);                 // [wavefront][2 HS][NG * 128]
  constexpr int kORow = NG * 128, kOWave = 2 * HS * kORow;
  const unsigned lds_base = (unsigned)(size_t)lds, sc_base = (unsigned)(size_t)scratch + (unsigned)(kAttSc + wave * 2 * HS * 256);

  // this wavefront's share of the segment: whole sets of 32 tokens
  const int n_sets_run = (last >> 5) + 1;
  const int set0 = n_sets_run * wave / 4, n_sets = n_sets_run * (wave + 1) / 4 - set0;
  const unsigned pitch = (unsigned)a.v_row_elems * 2u;
  const unsigned last_off = (unsigned)last * pitch, row_off = (unsigned)kq * pitch;
  const unsigned char* base = uniform_ptr((const unsigned char*)a.hv + v.cache_row0 * pitch + (size_t)(v.c0 + cb) * 2);
  const unsigned char* sc_row0 = uniform_ptr((const unsigned char*)(a.scores + ((size_t)v.b * a.n_heads + v.h_first) * a.lpad + v.tok0));
  const int cols = v.groups * v.rv, n_rows = v.n_rows;          // of the unit
  const bool begin = r0 == 0 && cb == 0;

  const int nh = min(n_rows - r0, 2 * HS);
  const int lpt = min(cols - cb, NG * 128) >> 3;            // 16-byte chunks per row
  // places of the halves in turn, this wavefront's: the next one first
  unsigned place[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) place[i] = ring[(1 + i) & 3] + (unsigned)(wave * 8192);
  auto request_half = [&](int h, unsigned at) __attribute__((always_inline)) {       // rows past the last one and chunks past the row's end: the last ones
    const unsigned col = (unsigned)min((NG == 2 ? (h & 1) * 16 : 0) + n, lpt - 1) * 16u;
    const unsigned row0 = (unsigned)((set0 + (NG == 2 ? h >> 1 : h)) * 32) * pitch;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const unsigned voff = min(row0 + (unsigned)(4 * i) * pitch + row_off, last_off) + col;
      const unsigned m0v = __builtin_amdgcn_readfirstlane(lds_base + at + (unsigned)(i * 1024));
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(m0v), "v"(voff), "s"(base) : "memory");
    }
  };
  unsigned sc_off[HS];                                      // bytes; the host keeps 32 rows below 2^32
#pragma unroll
  for (int i = 0; i < HS; ++i) sc_off[i] = (unsigned)(r0 + min(hp + 2 * i, nh - 1)) * (unsigned)a.lpad * 4u;
  auto request_scores = [&](int k) __attribute__((always_inline)) {
    const unsigned ts = (unsigned)min((set0 + k) * 32 + tl, last) * 4u;
#pragma unroll
    for (int i = 0; i < HS; ++i) {
      const unsigned m0v = __builtin_amdgcn_readfirstlane(sc_base + (unsigned)(((k & 1) * HS + i) * 256));
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" :: "s"(m0v), "v"(sc_off[i] + ts), "s"(sc_row0) : "memory");
    }
  };
  int min_lim = 0x7fffffff;                                     // smallest row limit of the unit's queries
  if (begin) {
    int own_lim = 0;
    if (a.q_len != nullptr) {                               // each thread one query row's limit
      Meta mq;
      mq.qpk = a.m_qpk; mq.nq = a.m_nq;
      own_lim = a.q_len[v.b * a.m_nq + q_token(mq, v.h_first + min(tid, n_rows - 1))] - v.tok0;
      if (tid < n_rows) lim_lds[tid] = own_lim;
    }
    // the scores of all four wavefronts have reached the cache; nobody reads the ring's tiles any more
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0) & ~0x0F00);     // ... and lgkmcnt 0
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  } else {
#pragma unroll
    for (int h = 0; h < PRE; ++h) request_half(h, place[h]);
  }
  if (a.q_len != nullptr) {
    min_lim = lim_lds[min(lane, n_rows - 1)];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) min_lim = min(min_lim, __shfl_xor(min_lim, d, 64));
    min_lim = __builtin_amdgcn_readfirstlane(min_lim);
  }
  request_scores(0);
#pragma unroll
  for (int h = PRE; h < 4; ++h) request_half(h, place[h]);
  request_scores(1);

  // The lazy maximum of pv_kernel (probabilities up to 2^8), which lets all heads of a unit catch up where one of them rises.  Blocks of fewer
  // rows than its units merge (4) keep the exact one instead: catching up less often, they rounded more (16 units of two heads, 1 x 4096
  // tokens, queries of four times N(0, 1): 1.05 of pv_kernel's error against 64 bits; one head each, 1 x 2000: 1.09).
  const float lazy = nh < 4 ? 0.f : 8.f;
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
  // rows of the probability tile that no head fills: zeros
  if constexpr (HS < 8) {
    for (int i = 2 * HS * kAttPitch + lane; i < 16 * kAttPitch; i += 64) pw[i] = (_Float16)0.f;
    wave_lds_fence();
  }
  // the arithmetic of pv_kernel
  for (int k = 0; k < n_sets; ++k) {
    // set k and its scores have landed: what is younger are the scores of set k + 1 and the halves requested with them
    constexpr int kNext = 8 * NG + HS;
    if (k + (NG == 1 ? 3 : 1) >= n_sets) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    else if (k == 0) __builtin_amdgcn_s_waitcnt(vmcnt_imm(8 * (4 - PRE) + HS));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(kNext));
    asm volatile("" ::: "memory");
    const int t0 = (set0 + k) * 32, t = t0 + tl;
    float s[HS], bm[HS];
    bool grew = false;
#pragma unroll
    for (int i = 0; i < HS; ++i) {
      const float v = sc_lds[((k & 1) * HS + i) * 64 + lane];
      s[i] = (t <= last && hp + 2 * i < nh) ? v : -INFINITY;
    }
    if (t0 + 32 > min_lim) {                                // uniform: some query's row limit lies in this set or before
#pragma unroll
      for (int i = 0; i < HS; ++i)
        if (t >= lim_lds[r0 + min(hp + 2 * i, nh - 1)]) s[i] = -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < HS; ++i) {
      bm[i] = half_wave_max(s[i]);
      grew |= bm[i] > mx[i] + lazy;
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
      uint4v row[8];                                        // the lane's chunk of tokens 8 kq .. + 7
#pragma unroll
      for (int j = 0; j < 8; ++j) row[j] = *reinterpret_cast<const uint4v*>(lds + place[ng] + (8 * kq + j) * 256 + n * 16);
      uint32_t o[8][4];                                     // [channel e of the chunk][token pair]
#pragma unroll
      for (int jp = 0; jp < 4; ++jp)
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          uint32_t lo = __builtin_amdgcn_perm(row[2 * jp + 1][d], row[2 * jp][d], 0x05040100u);
          uint32_t hi = __builtin_amdgcn_perm(row[2 * jp + 1][d], row[2 * jp][d], 0x07060302u);
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
    // the places just read are requested anew: their reads, and those of the scores, are done
    if (k + (NG == 1 ? 4 : 2) < n_sets) {
      __builtin_amdgcn_s_waitcnt(0xC07F);                   // lgkmcnt 0
      asm volatile("" ::: "memory");
#pragma unroll
      for (int ng = 0; ng < NG; ++ng) request_half((k + 1) * NG + 4 - NG + ng, place[ng]);
    }
    if (k + 2 < n_sets) {
      __builtin_amdgcn_s_waitcnt(0xC07F);
      asm volatile("" ::: "memory");
      request_scores(k + 2);
    }
#pragma unroll
    for (int r = 0; r < NG; ++r) {
      const unsigned p0 = place[0];
      place[0] = place[1]; place[1] = place[2]; place[2] = place[3]; place[3] = p0;
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                 // nothing requested may land in what LDS holds next
  asm volatile("" ::: "memory");

  // ---- merge of the four wavefronts
#pragma unroll
  for (int i = 0; i < HS; ++i) lsum[i] = half_wave_sum(lsum[i]);
  if (tl == 0) {
#pragma unroll
    for (int i = 0; i < HS; ++i) *reinterpret_cast<float2*>(ml_lds + (wave * 16 + hp + 2 * i) * 2) = float2{mx[i], lsum[i]};
  }
  __syncthreads();
  float m, l = 0.f;                                         // of row lane & 15, this segment included
  {
    const int row = lane & 15;
    float own = 0.f, old = 0.f;
    float2 w4[4], before = {-INFINITY, 0.f};
    if (v.more && row < nh) before = *reinterpret_cast<const float2*>(run_lds + (r0 + row) * 2);
    m = before.x;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      w4[x] = *reinterpret_cast<const float2*>(ml_lds + (x * 16 + row) * 2);
      m = fmaxf(m, w4[x].x);
    }
    if (before.x != -INFINITY) {
      old = __builtin_amdgcn_exp2f(before.x - m);
      l = before.y * old;
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const float f = w4[x].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(w4[x].x - m);
      l = fmaf(w4[x].y, f, l);
      own = x == wave ? f : own;
    }
    if (lane < 16) xw[lane] = own;
    if (wave == 0 && lane < 16) old_lds[lane] = old;
    if (wave == 0 && cb == 0 && lane < nh) *reinterpret_cast<float2*>(a.ml_part + (v.slot * a.n_heads + v.h_first + r0 + lane) * 2) = float2{m, l};
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
  if (wave == 0 && lane < nh && cb + NG * 128 >= cols) *reinterpret_cast<float2*>(run_lds + (r0 + lane) * 2) = float2{m, l};
  float* op = a.o_part + v.slot * a.o_stride + v.o0;
  for (int id = tid; id < nh * (kORow / 4); id += 256) {
    const int row = id / (kORow / 4), col = (id % (kORow / 4)) * 4;
    if (col >= 8 * lpt) continue;
    const int head = r0 + row, c = cb + col - (v.groups == 1 ? 0 : head / v.rows_per_group * v.rv);      // column inside the head's own group
    if (c < 0 || c >= v.rv) continue;                      // a head keeps the columns of its own group
    float4v o = *reinterpret_cast<const float4v*>(o_lds + row * kORow + col);
#pragma unroll
    for (int x = 1; x < 4; ++x) o += *reinterpret_cast<const float4v*>(o_lds + x * kOWave + row * kORow + col);
    float4v* dst = reinterpret_cast<float4v*>(op + (size_t)head * v.rv + c);
    if (v.more) o += *dst * old_lds[row];                     // this workgroup's own sum so far, written by the same thread
    *dst = o;
  }
  __syncthreads();                                          // LDS is the next block's
}

// T, NK, G, NQ, FLAT: as in score16_kernel; HS: attend_hs.  FLAT: a workgroup's run goes through the tiles of all sequences; the values of a segment follow
// its scores, up to a.seg_tiles tiles at a time.  Workgroups then are at different places of their segments at any time: the matrix
// pipes of some work while others read values.
// grid as score16_kernel's, 256 threads, attend_lds_bytes of LDS.
#undef SCORE16_DRAIN
#define SCORE16_DRAIN values_of_segment()                        // value_block waits for them
#define SCORE16_VALUES                                                                                                              \
  constexpr int kHalves = kAheadTiles * kDmaIssues / 8;                                                                             \
  static_assert(attend_partials_lds(HS, 2) <= (size_t)score16_lds_bytes(kWidth), "the partial results live in the score phase's ring"); \
  int sequence_before = -1;                                                                                                         \
  auto values_of_segment = [&]() __attribute__((always_inline)) {                                                                   \
    const int qpk = NQ == 1 ? 1 : a.m_qpk;                                                                                          \
    const int rows_per_group = (G == 1 ? u.nh : u.s) * qpk;                                                                         \
    const bool more = FLAT && b == sequence_before;                                                                                 \
    sequence_before = b;                                                                                                            \
    const size_t slot = FLAT ? (size_t)(wg + b) : (size_t)b * a.n_split + wg;                                                       \
    if (a.slots != nullptr && wave == 0 && lane < u.nh * qpk) {                                                                     \
      int* sl = a.slots + ((size_t)b * a.n_heads + u.h0 * qpk + lane) * 2;                                                          \
      if (off == 0) sl[0] = (int)slot;                                                                                              \
      if (off + n_tiles >= (FLAT ? seq_tiles : (seq_rows + kTile - 1) / kTile)) sl[1] = (int)slot;                                  \
    }                                                                                                                               \
    const AttendValue uv = a.val[unit];                                                                                             \
    const ValueSegment v{u.nh * qpk, u.h0 * qpk, rows_per_group, G, uv.c0, uv.rv, uv.o0, b, off * kTile, rel_last, more, slot, row0}; \
    unsigned char* scratch = lds + score16_lds_bytes(kWidth);                                                                       \
    for (int r0 = 0; r0 < v.n_rows; r0 += 2 * HS)                                                                                   \
      for (int cb = 0; cb < G * v.rv; cb += 256) {                                                                                  \
        if (G * v.rv - cb > 128) value_block<T, HS, 2, kHalves>(a, v, r0, cb, lds, scratch, ring);                                  \
        else value_block<T, HS, 1, kHalves>(a, v, r0, cb, lds, scratch, ring);                                                      \
      }                                                                                                                             \
  };
template <typename T, int NK, int G, int NQ, bool FLAT, int HS>
__global__ __launch_bounds__(256) void attend16_kernel(AttendArgs a) {
  constexpr int QB = 0;
  constexpr bool kValues = true;
  const int wg = blockIdx.x, n_wg = a.n_wg, unit = blockIdx.y, seq = blockIdx.z, run = a.run, run_more = a.run_more;
#include "score16_body.inc"
}

// The same body for a launch over units of several key ranks (see score16_mixed_kernel), runs inside one sequence: every unit has its own number of
// workgroups, chosen by the host so that all end at about the same time.  grid (sum over units of workgroups and sequences).
// Ranks 64 .. 256 by group, 32 heads, us a step, two launches -> this: 1 x 16384 tokens 50.7 -> 46.1, 2 x 5000 37.6 -> 34.8.  (Runs through all sequences, whose
// weights stay in registers across the values, spill 63 of them in this kernel: 4 x 16384 156.5 -> 168, 8 of 2000 .. 4000 66.8 -> 84.)
template <typename T, int NK>
__device__ __forceinline__ void attend16_body(const AttendArgs& a, const int wg, const int n_wg, const int unit, const int seq, const int run, const int run_more) {
  constexpr int G = 1, NQ = 1, QB = 0, HS = 2;
  constexpr bool FLAT = false, kValues = true;
#include "score16_body.inc"
}
template <typename T>
__global__ __launch_bounds__(256) void attend16_mixed_kernel(AttendArgs a) {
  int unit = 0;
  for (int i = 1; i < a.units.n_units; ++i)
    if ((int)blockIdx.x >= a.mix.first[i]) unit = i;
  const int local = (int)blockIdx.x - a.mix.first[unit], n_wg = (a.mix.first[unit + 1] - a.mix.first[unit]) / a.batch;
  const int seq = local / n_wg, wg = local - seq * n_wg, run = a.mix.run[unit], run_more = a.mix.run_more[unit];
  switch (a.mix.nk[unit]) {
    case 2: attend16_body<T, 2>(a, wg, n_wg, unit, seq, run, run_more); break;
    case 3: attend16_body<T, 3>(a, wg, n_wg, unit, seq, run, run_more); break;
    case 4: attend16_body<T, 4>(a, wg, n_wg, unit, seq, run, run_more); break;
    case 5: attend16_body<T, 5>(a, wg, n_wg, unit, seq, run, run_more); break;
    case 6: attend16_body<T, 6>(a, wg, n_wg, unit, seq, run, run_more); break;
    case 7: attend16_body<T, 7>(a, wg, n_wg, unit, seq, run, run_more); break;
    default: attend16_body<T, 8>(a, wg, n_wg, unit, seq, run, run_more); break;
  }
}
#undef SCORE16_VALUES
#undef SCORE16_DRAIN
#define SCORE16_DRAIN __builtin_amdgcn_s_waitcnt(vmcnt_imm(0))

}  // namespace palu
