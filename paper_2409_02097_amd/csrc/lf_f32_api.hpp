// Host-side interface between the translation units: the fp32 three-kernel path and backward pass (linfusion_f32.hip),
// the launch plan they take from the forward planner (linfusion.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "lf_common.hpp"

namespace lf32 {

// launch shape from the forward plan of the same problem size
struct Plan32 {
  int splits, blk_reduce, apply_wgs, blk_apply;
};
// LINFUSION_OK, or the forward plan's error code; `partial_bytes`: what the partial states of one pass take
int launch_plan32(int B, int H, long long N, int d, Plan32* p, size_t* partial_bytes);

// out = mixer(q, k, v); with out == null only the state.  The head states are left in `state` either way.
struct Fwd32Args {
  const void *q, *k, *v;
  void* out;
  long long BH, N;
  int d, fm;
  float eps;
  bool unnorm;
  lf::Layout lq, lkv, lo;
  float *partials, *state;    // [B*H][splits][d*d + d] and [B*H][d*d + d]
  Plan32 plan;
  hipStream_t st;
  hipEvent_t* ev;             // null, or four events around the kernels
};
int run_fwd32(const Fwd32Args& a);
const char* apply32_name(int d);   // the kernel that its apply step takes

// gradients of q, k, v
struct Bwd32Args {
  const float* saved_state;   // the forward state of the same q, k, v, or null: recompute it from k, v
  const void *q, *k, *v, *g;
  void *dq, *dk, *dv;
  int B, H;
  long long N;
  int d, fm;
  float eps;
  bool unnorm;
  lf::Layout lq, lkv, lg, ldq, ldkv;   // q; k and v; dout; dq; dk and dv
  unsigned char* ws;                   // bwd32_workspace_bytes
  hipStream_t st;
};
bool bwd32_supported(int d);
size_t bwd32_workspace_bytes(int B, int H, long long N, int d);   // 0 for unsupported shapes
int run_bwd32(const Bwd32Args& a);

}  // namespace lf32
