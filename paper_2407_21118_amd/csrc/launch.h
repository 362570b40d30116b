// What the host side (api.hip) needs of the kernels that are compiled as translation units of their own: their
// argument structures and the functions that pick or launch an instantiation.
#pragma once

#include "palu_dev.h"

namespace palu {

// ---- score kernels (score_forms.hip, score16_forms.hip)
using ScoreFn = void (*)(ScoreArgs);
// 4-bit keys (i4) of ranks 384 and 512 that are not sliced, rank 32 and the forced schedules: class id = rank class * 3 + log2(groups per workgroup);
// w8: four heads as 8 half-head wavefronts (two per SIMD) instead of 4 whole-head ones
ScoreFn score_fn(int act, bool i4, int cls_id, bool w8);
// 3- and 2-bit key latents
ScoreFn score_fn_lowbit(int rc);
// fp16 shared-key form (option shared_key_fp16): at most 4, else at most 16 queries per key/value head
ScoreFn score_fn_shared(int rc, bool four);
// unquantized latents, ranks 64 .. 256, one whole head per wavefront.  FLAT: runs through the tiles of all sequences
// (each value is a translation unit of its own, also of the forms below)
template <bool FLAT> ScoreFn score16_fn(int act, int rc, int lg);
// one launch over several rank classes of the above
template <bool FLAT> ScoreFn score16_mixed_fn(int act);
// several queries per key/value head, the key rebuilt once per pass of nq rows (NULL: not compiled)
template <bool FLAT> ScoreFn score16q_fn(int act, int rc, int nq);
// the same with 4-bit key latents (rank classes 128 and 256, also slices of larger ranks); one query per head (nq = 1): also 2 or 4
// groups per workgroup (lg)
template <bool FLAT> ScoreFn score16q4_fn(int rc, int nq, int lg);
// score16_kernel's runs of tiles with the value contraction behind them, one launch for both (attend16.hip); nq: query rows per
// key/value head (1, or up to 8); FEW: at most four rows to a unit
using AttendFn = void (*)(AttendArgs);
template <bool FLAT> AttendFn attend16_fn(int act, int rc, int lg);
template <bool FEW> AttendFn attend16q_fn(int act, int rc, int nq);
AttendFn attend16_mixed_fn(int act);
// option score_fp8
ScoreFn score8_fn(int rc, int lg);
struct Fold8Args {
  const uint16_t* Bk;
  unsigned char* w8;         // per head r * 128 bytes at byte offset (bk_off[group] + head in group * r * 128)
  float* scale;              // [n_heads][128]
  Meta meta;
};
int launch_fold8(const Fold8Args& a, hipStream_t s);

// ---- value kernel (pv.hip)
struct PvUnit {
  int32_t c0;         // first column of the value-latent row
  uint16_t h0;        // first head
  uint16_t ncols;     // columns (multiple of 32, at most 128 * NG)
  uint8_t nh;         // heads (at most 16 in the built forms); a head only keeps the columns of its own group
  uint8_t write_ml;   // this unit stores the (max, sum) pair of its heads
};
constexpr int kMaxPvUnits = 128;
struct PvUnits {
  int n_units;
  PvUnit u[kMaxPvUnits];
};

struct PvCommon {
  const void* hv;
  const uint16_t* hv_scale;
  const uint16_t* hv_zero;
  const float* scores;       // [parts][batch][n_heads][lpad]; planes 0 and 1 are read
  const int32_t* seq_lens;
  const int32_t* q_len;      // several queries per sequence: rows attended by query j of sequence b at [b * nq + j]; or NULL
  float* o_part;             // [batch][n_split][o_stride]
  float* ml_part;            // [batch][n_split][n_heads][2]
  long long row_elems;       // R_v
  long long max_seq;
  long long part_stride;
  int seq_len;
  int lpad;
  int batch;
  int split_tokens;          // tokens per wavefront (multiple of 32)
  int n_split;
  int o_stride;
  int n_blocks_q;
  int units_per_wg;          // 1, 2 or 4: the wavefronts of a workgroup take this many units of the same splits
  Meta meta;
};
struct PvArgs : PvCommon {
  uint8_t n_parts[PALU_MAX_HEADS];   // 1 or 2 score planes per head
  PvUnits units;
};

// Non-RoPE attention in one pass (pv.hip): every wavefront makes its split's scores itself, from the folded queries (qk.hip).  The units are
// the value units; of each its key side:
struct StreamKeys {
  int32_t c0, q_off, qs_off;         // as in QkUnit
  int32_t ncols;                     // at most 256
};
constexpr int kMaxStreamUnits = 32;
struct StreamUnits {
  int n_units;
  PvUnit u[kMaxStreamUnits];
};
struct StreamArgs : PvCommon {
  const void* hk;
  const uint16_t* hk_scale;
  const uint16_t* hk_zero;
  const uint16_t* qt;
  const float* qsum;
  long long qt_bstride, qs_bstride;
  long long k_row_elems;             // R_k
  int k_blocks_q;
  int lds_unit_stride;               // bytes of LDS per unit's folded queries
  float scale;                       // log2(e) / sqrt(d_h)
  StreamUnits units;
  StreamKeys keys[kMaxStreamUnits];
};
static_assert(sizeof(PvArgs) <= 4096 && sizeof(StreamArgs) <= 4096, "kernel arguments");

struct PlaneSumArgs {
  float* scores;
  long long part_stride;
  int lpad;
  int seq_len;
  int n_heads;
  uint8_t n_parts[PALU_MAX_HEADS];
};


using PvFn = void (*)(PvArgs);
// bits: 4, 3 or 2 for quantized value latents, else 0; two_planes: some head's scores lie in two planes
PvFn pv_fn(int act, int bits, int cls, bool two_planes);
// ... of the one-pass form, both sides of the same latent dtype; LDS per unit: stream_unit_lds
using StreamFn = void (*)(StreamArgs);
StreamFn stream_fn(int act, int bits, int cls);
constexpr int kStreamPitch = 256 + 8;      // halfs per folded query: 16 bytes of padding keep the head rows on distinct banks
constexpr int stream_unit_lds(bool quantized, int nh) { return quantized ? nh * kStreamPitch * 2 + nh * 2 * 4 : 2 * nh * kStreamPitch * 2; }
int launch_plane_sum(const PlaneSumArgs& a, int batch, hipStream_t s);

}  // namespace palu
