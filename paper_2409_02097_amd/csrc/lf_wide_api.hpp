// Host-side interface between the two translation units of the library: linfusion.hip (boundary, planning,
// head widths up to 64) and linfusion_wide.hip (the kernels for head widths above 64).
#pragma once
#include <hip/hip_runtime.h>

#include "lf_common.hpp"

namespace lfw {

// launch shape of the wide kernels for one problem size (from the forward plan)
struct WidePlan {
  int splits, blk_reduce, apply_wgs, blk_apply;
  int apply_waves;            // waves per apply workgroup: 4 or 8 (apply16_wide)
  bool wave_apply;            // apply16_wave (a wave per tile, the whole state in its registers) instead
  int short_parts;            // > 0: the whole forward call in one launch (lf_short16.hpp), that many workgroups per group of
  bool short_half;            // value channels: 32 of a head, or half of the head's
};

// state reduction + combine:  state[bh] = {S = sum_t phi(k_t)^T v_t, z = sum_t phi(k_t)}, fp32 [d*d + d]
struct WideReduceArgs {
  const void *k, *v;
  int B, H;
  long long N;
  int d, dtype, fm;           // dtype: LINFUSION_DTYPE_F16 or _BF16
  lf::Layout lk, lv;          // the two tensors may be laid out differently
  float *partials, *state;    // [B*H][splits][d*d + d] and [B*H][d*d + d], fp32
  WidePlan plan;
  hipStream_t st;
};

// out_t = phi(q_t) S / (phi(q_t) z + eps)   (unnorm: phi(q_t) S)
struct WideApplyArgs {
  const void* q;
  void* out;
  int B, H;
  long long N;
  int d, dtype, fm;
  float eps;
  bool unnorm;
  lf::Layout lq, lo;
  const float* state;         // [B*H][d*d + d]
  unsigned char* packed;      // wide_packed_bytes(d, dtype) per head: scratch for the state as apply operands
  WidePlan plan;
  hipStream_t st;
};

struct WideArgs {
  const void *q, *k, *v;
  void* out;                  // null: stop after the combine (state only)
  int B, H;
  long long N;
  int d, dtype, fm;           // dtype: LINFUSION_DTYPE_F16 or _BF16
  float eps;
  bool unnorm;
  lf::Layout lq, lkv, lo;
  float *partials, *state;    // [B*H][splits][d*d + d] and [B*H][d*d + d], fp32
  unsigned char* packed;      // wide_packed_bytes(d, dtype) per head: the state as apply operands
  WidePlan plan;
  hipStream_t st;
  hipEvent_t* ev;             // null, or four events: before reduce, after it, after combine, after apply
};

// State-reduction workgroups of a problem, given what fills the chip.  Each adds a partial of 4 (d^2 + d) bytes per head that
// is written and read again, about 0.5 us per MB over all heads, and takes its share of about 1.5 us per tile from the
// others, so the sum is least at sqrt(3 tiles / MB) per head.  (One partial per two tiles, as two workgroups per CU gave,
// against this, us per call: fp16 12 x 8 x 256 x 160 39.6 -> 33.7; 2 x 8 x 1024 x 160 35.6 -> 29.5; bf16 4 x 16 x 512 x 128
// 36.6 -> 30.7.)  From three quarters of a workgroup per CU on, whole rounds: with 1.1 to 1.7 per CU some CUs have two and
// the others wait (us at the least of the sum -> one per CU: fp16 4 x 8 x 4096 x 160 70.6 -> 62.4, 12 x 8 x 1024 x 160
// 62.4 -> 56.4, bf16 2 x 8 x 4096 x 160 52.8 -> 46.3, 4 x 16 x 2048 x 128 60.9 -> 56.2; near two per CU -> two: 2 x 8 x
// 16384 x 160 108 -> 98 to 105).  Long streams stay at what fills the chip.
// `ratio`: a tile's time over that of a partial's MB, 3 for the mixer alone.  The MLP-fed reduction's tiles have a third
// stream and the branch sum to form, and it has to reach two workgroups per CU sooner: with 3 it lost to the two per CU that
// it always had before at bf16 4 x 8 x 4096 x 160 (112.7 -> 121.7 us per call), 1 x 8 x 16384 x 160 (104.5 -> 117.0), fp16 1 x 10
// x 4096 x 128 (47.9 -> 53.2); kMlpTileRatio gives those their two and keeps what fewer gain (4 x 8 x 256 x 160 44.8 -> 43.1,
// 2 x 8 x 1024 x 160 47.9 -> 45.3, 4 x 8 x 1024 x 160 64.4 -> 59.2, 4 x 16 x 512 x 128 51.2 -> 46.2).
constexpr double kMlpTileRatio = 11.0;
inline int wide_reduce_wgs(long long heads, long long tiles, int d, int fill, int cus, double ratio = 3.0) {
  const double mb = (double)heads * ((double)d * d + d) * 4e-6;
  const double s = __builtin_sqrt(ratio * (double)tiles / mb) + 0.5;
  const long long want = (s < 1.0 ? 1 : (s > 1e6 ? 1000000 : (long long)s)) * heads;
  if (want >= fill) return fill;
  if (4 * want >= 7 * (long long)cus) return want > 2 * cus ? (int)want : 2 * cus;   // (`fill` is two per CU or more)
  return 4 * want >= 3 * (long long)cus ? cus : (int)want;
}
// head widths the wide kernels are built for
bool wide_supported(int d);
// whether apply16_wave is built for this width and dtype (its state operands must fit one wave's registers)
bool wave_apply_supported(int d, int dtype);
// bytes per head of the operand-ready state between the pack and apply kernels (0 if unsupported)
size_t wide_packed_bytes(int d, int dtype);
// enqueues state reduction, combine and (if out) pack and apply; returns LINFUSION_OK or a LINFUSION_ERR_* code
int run_wide(const WideArgs& a);
// the forward plan's launch shape for a wide width (linfusion.hip), and the bytes its partial states take;
// LINFUSION_ERR_UNSUPPORTED for other widths
int wide_launch_plan(int B, int H, long long N, int d, int dtype, WidePlan* wp, size_t* partial_bytes);
// For the backward pass of these widths: the forward state of k and v (one layout) in a.state, with the bits that the forward
// call of these tensors leaves in its workspace; the reduction by itself -- the summed state in a.state, or the partials as
// they are (a single one is the state, in a.state) -- and the apply kernel of one wave per tile on operands that lie packed
// (PackWave's layout) already; a.state is not read.
int run_wide_state(const WideReduceArgs& a);
int run_wide_reduce(const WideReduceArgs& a);
int run_wide_reduce_partials(const WideReduceArgs& a);
int run_wide_apply_packed(const WideApplyArgs& a);

}  // namespace lfw
