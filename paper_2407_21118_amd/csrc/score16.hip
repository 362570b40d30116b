// The score kernel of score.hip (key reconstruction + RoPE + query product in float32, Sec. 3.1.2,
// Sec. 2.1 Eq. 2, Appendix B) for its most common case: unquantized fp16 / bf16 latents, ranks up
// to 256, one query per head.  Same LDS layout and LDS-direct staging; a different use of the CU:
//
//   * four wavefronts, one per SIMD, each owning ONE WHOLE HEAD: B_k^T of the head (128 x r) stays in
//     its registers (256 at rank 256).  A head's two features of a rotation pair sit in the same lane,
//     so a wavefront reads the angles of a (token, pair) once for both, sums a token's 128 products
//     with ONE lane exchange sequence per head (the half-head wavefronts of score.hip: two), and each
//     16-byte latent read from LDS feeds 8 matrix instructions (there: 2 of twice the size);
//   * v_mfma_f32_16x16x32: 16 tokens x 16 features per instruction.  An accumulator set of a 16-token
//     sub-tile is 32 registers, so two sets fit beside the weights: the vector ALU rotates and
//     multiplies sub-tile s-1 (6 operations per token and pair, dealt out between the matrix
//     instructions of sub-tile s) while the matrix pipe works on s.  The lane exchange that sums a
//     token's products runs inside the 16 lanes of a DPP row: 11 operations for the 4 tokens a lane holds.
//
// Per 32-token tile and CU this moves 160 KiB through the LDS where the ping-pong schedule moves 225,
// and issues 0.75 as many vector instructions.
//
// Several queries per key/value head (grouped-query layers, several query tokens per sequence; NQ = 2, 4, 8, other
// counts in passes with idle rows): the
// wavefront's head is a key/value head; its key tile is rebuilt once, each key pair rotated once in float32 and
// multiplied by each of the NQ rotated queries.  NQ = 2: on the vector ALU (8 operations per token and pair instead of 12), then one
// lane exchange and one score row per query.  NQ = 4, 8 (kMx): vector work of 4 + 2 NQ operations per pair would
// take longer than the matrix instructions (which leave room for two vector operations each: 16.8 cycles alone or
// with two, 21.6 with three, 33.8 with six), so the products go to v_mfma_f32_4x4x1_16b, exact float32 at twice the
// vector rate.  It wants tokens across lanes, so the operands of the key product are exchanged (a lane then holds one token of 16
// pairs), and the angles are read token by token from the same tile.  The 32 (64) products of a sub-tile are issued in
// one go behind its rotations: alone each takes 8.8 cycles, but one between two 16-bit matrix instructions 28 (one
// at a time they were no faster than the vector form).  What is left to sum lies in the four quarters of the wavefront: three lane
// swaps and adds for four queries instead of eleven operations each.  us a call, vector form -> this: 4 queries over 2 x 8190
// tokens of 32 heads, rank 128 75.1 -> 69.5, 256 74.5 -> 68.5, 64 120.8 -> 94.8; 4 x 16384 tokens of 8 heads 76.6 -> 74.1;
// 8 queries, rank 256 89.6 -> 77.1, and at the ranks that took passes of four before, 128 99.9 -> 66.6, 64 225 -> 123.

#pragma once
#include <type_traits>

#include "score.hip"

namespace palu {

// Columns a latent tile row takes in LDS: the rows of unquantized latents (at most 256 columns: groups x rank) are
// laid out in the 32 slots of a 256-column row, whatever their width, and requested two per instruction.
constexpr int score16_lds_width(int width, bool staged) { return staged ? width : 256; }
// LDS bytes of score16_kernel for unquantized latents (shared with the host)
constexpr int score16_lds_bytes(int width) { return score_lds_bytes(score16_lds_width(width, false), true, true, false); }

// part[j], j = 0..3, belongs to token 4 (lane / 16) + j of a 16-token sub-tile and to the feature this lane
// owns (lane % 16).  Returns the sum over the 16 lanes of the row of ONE of the lane's tokens:
//   token 4 (lane / 16) + 2 L2 + L0    (Lk = bit k of the lane number),
// the same value in the four lanes that differ in bits 1 and 3.
__device__ __forceinline__ float sum_quad_over_row(const float (&p)[4], int lane) {
  const bool l0 = lane & 1, l2 = lane & 4;
  float v2[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) v2[j] = (l2 ? p[2 + j] : p[j]) + dpp_lane_move<0x141>(l2 ? p[j] : p[2 + j]);      // row_half_mirror
  float v = (l0 ? v2[1] : v2[0]) + dpp_lane_move<0xB1>(l0 ? v2[0] : v2[1]);                                     // quad_perm [1,0,3,2]
  v += dpp_lane_move<0x4E>(v);                                                                                  // quad_perm [2,3,0,1]
  return v + dpp_lane_move<0x128>(v);                                                                           // row_ror 8
}

// The value latents of a unit, where they are contracted in the same workgroup (attend16_kernel): the unit's first column in the cache's
// first row, bytes between rows, 16-byte chunks of a row (at most 32: the first 256 columns)
struct ValueView {
  const unsigned char* base;
  unsigned pitch;
  int chunks;
};
__device__ __forceinline__ ValueView value_view(const ScoreArgs&, int, int) { return ValueView{nullptr, 0, 1}; }
__device__ __forceinline__ ValueView value_view(const AttendArgs& a, int unit, int groups) {
  return ValueView{(const unsigned char*)a.hv + (size_t)a.val[unit].c0 * 2, (unsigned)a.v_row_elems * 2u, min(groups * a.val[unit].rv, 256) >> 3};
}

// T:  storage type of the weights and latents (the matrix instruction of that type)
// NK: k-steps of 32: the rank of every head of the workgroup is 32 * NK (NK <= 8)
// G:  groups spanned by the workgroup's heads (1, 2 or 4 adjacent groups of equal rank): the staged
//     latent row is G * 32 * NK columns wide
// FLAT: a workgroup's run goes through the tiles of all sequences, else it lies in one
// grid (workgroups per unit and sequence, units, sequences; FLAT: per unit, units), 256 threads.
// NQ: queries that share the wavefront's key/value head (grouped-query layers, several query tokens per sequence):
//     the unit's heads are then key/value heads with a.m_qpk query rows each; this launch takes rows a.sk_row0 ..
//     + a.sk_rows - 1 (at most NQ) of every key/value head: the key tile is rebuilt once, rotated once in float32
//     and multiplied by each rotated query (NQ = 1: the head's own query)
// QB: 4: the key latents are 4-bit codes (Sec. 3.4, Appendix A; fp16 layers).  Their tiles go through registers: codes,
//     scales and zero-points are requested two tiles ahead, dequantized to fp16 ((code - zero) * scale, one rounding; see
//     dequant8_packed) between the matrix instructions of the tile before and written to LDS in the layout these
//     read; only the angle tiles stay LDS-direct.  16 x 8192 tokens of a 7B-shaped layer, rank 256: 327 .. 370 us on
//     score_kernel (two half-head wavefronts per SIMD), 257 .. 288 us here.
//
// One wavefront per SIMD issues in order, so the kernel's time is its instruction count where that exceeds the matrix
// pipe's (128 matrix instructions of 16 cycles per 32-token tile at rank 256).  Two things keep the count down: the
// weights are pinned to the accumulation registers, which the matrix instructions read in place (left to
// itself the compiler kept part of them as spilled copies, up to four moves per matrix instruction), and the loop
// has no branch inside a sub-tile.  Instructions per tile at rank 256: one query 519 -> 500, four queries (vector form) 1300 -> 790
// (4 x 16384 tokens, 8 key/value heads: 65 -> 45 us).  LDS offsets that move on with the tile instead of being computed from
// its number: 500 -> 492, 4-bit keys 627 -> 603, with four queries 922 -> 904.
// Waits count as well: the first angles of a sub-tile, requested by the body that needs them, cost about 100 cycles each; requested in
// the last slots of the body before, and with a hand-over barrier that waits for no LDS read (unquantized latents), they
// are gone from the tile: a step of ranks 96 .. 416 over 4 x 16384 tokens 226.2 -> 223.5 us, of rank 64 per head over 8 x 16384
// 202.8 -> 201.1; 16 x 8192 in 4 bits and 1 x 65536, at the power limit, level.
//
// The weights come from B_k as the caller has it.  A launch of its own used to lay them out (5 us, or 3 us more for the
// projection that it rode in); transposing them in registers, 64 byte permutes per k-step of which all but the first are
// dealt out between the first sub-tile's matrix instructions (FLAT, 4-bit keys: ahead of them), adds about 1 us to the
// kernel: one sequence of 1024 / 16384 tokens 22.9 / 64.7 -> 20.8 / 62.5 us a step, 28.0 / 83.0 -> 25.5 / 79.1 with all inputs out of the
// caches; 16 x 8192 in 4 bits 302 -> 298, four queries over 2 x 8190 70.6 -> 67.4; long launches, at the power limit, level.
#define SCORE16_DRAIN __builtin_amdgcn_s_waitcnt(vmcnt_imm(0))      // no LDS-direct load may outlive the workgroup's LDS allocation
template <typename T, int NK, int G, int NQ, int QB, bool FLAT>
__global__ __launch_bounds__(256) void score16_kernel(ScoreArgs a) {
  constexpr bool kValues = false;
  const int wg = blockIdx.x, n_wg = a.n_wg, unit = blockIdx.y, seq = blockIdx.z, run = a.run, run_more = a.run_more;
#include "score16_body.inc"
}

// The same body with its place in the launch as arguments (workgroup wg of n_wg of the unit), so that a launch over
// several rank classes can hand each workgroup the body of its unit's class.
template <typename T, int NK, int G, bool FLAT>
__device__ __forceinline__ void score16_body(const ScoreArgs& a, const int wg, const int n_wg, const int unit, const int seq, const int run, const int run_more) {
  constexpr int NQ = 1, QB = 0;
  constexpr bool kValues = false;
#include "score16_body.inc"
}

// One launch for a layer whose groups have different ranks (the ranks a search assigns per group, Sec. 3.3):
// a.mix lists the rank classes, heaviest first, each with its own number of workgroups per unit (chosen by the host so
// that workgroups of different classes take about as long) and its units, which lie side by side in a.units.
// grid (sum over classes of workgroups x units, and x sequences where a run lies in one), 256 threads; the workgroups of a
// class are consecutive.
template <typename T, bool FLAT>
__global__ __launch_bounds__(256) void score16_mixed_kernel(ScoreArgs a) {
  int c = 0;
#pragma unroll
  for (int i = 1; i < kMaxMixClasses; ++i)
    if (i < a.mix.n_cls && (int)blockIdx.x >= a.mix.first[i]) c = i;
  const int local = (int)blockIdx.x - a.mix.first[c];
  const int n_wg = a.mix.n_wg[c], wg = local % n_wg, rest = local / n_wg;
  const int unit = a.mix.unit0[c] + (FLAT ? rest : rest % a.mix.n_units[c]), seq = FLAT ? 0 : rest / a.mix.n_units[c];
  const int run = a.mix.run[c], run_more = a.mix.run_more[c];
  switch (a.mix.nk[c]) {
    case 2: score16_body<T, 2, 1, FLAT>(a, wg, n_wg, unit, seq, run, run_more); break;
    case 3: score16_body<T, 3, 1, FLAT>(a, wg, n_wg, unit, seq, run, run_more); break;
    case 4: score16_body<T, 4, 1, FLAT>(a, wg, n_wg, unit, seq, run, run_more); break;
    case 5: score16_body<T, 5, 1, FLAT>(a, wg, n_wg, unit, seq, run, run_more); break;
    case 6: score16_body<T, 6, 1, FLAT>(a, wg, n_wg, unit, seq, run, run_more); break;
    case 7: score16_body<T, 7, 1, FLAT>(a, wg, n_wg, unit, seq, run, run_more); break;
    default: score16_body<T, 8, 1, FLAT>(a, wg, n_wg, unit, seq, run, run_more); break;
  }
}

}  // namespace palu
