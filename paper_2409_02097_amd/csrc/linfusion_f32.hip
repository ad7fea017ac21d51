// Translation unit of the library: the fp32 three-kernel path and the fp32 backward pass (kernels in lf_ring32.hpp).
#include "../../include/linfusion.h"

#include "lf_f32_api.hpp"
#include "lf_host_api.hpp"
#include "lf_ring32.hpp"

namespace lf32 {

namespace {

#define LF_FOR_D(X) X(8) X(16) X(24) X(32) X(40) X(48) X(56) X(64)

constexpr int ne_of(int d) { return d * d + d; }

// Up to 24 channels the apply step on the fp32 instruction (apply32) stays the faster one: there a tile's products are
// few and splitting its values costs more (8 heads, 2^20 tokens: d = 8 205 against 230 us per call, d = 24 equal).
constexpr bool narrow_apply(int d) { return d <= 24; }

// Whether the consumers of a state sum its partials themselves (see lf_ring32.hpp): every workgroup then reads
// parts * (d^2 + d) floats, which up to 64 KB is cheaper than the launch it saves (96 heads of 40 channels, five partials
// each: training step 200.7 -> 197.7 us), beyond that not (20 heads of 64, 25 partials of 16 KB: 83 -> 90 us).
// (LINFUSION_FOLD = 2 under tuning: never)
bool fold(int parts, int d) {
  return parts <= lf::kFoldParts && lfh::env_int("LINFUSION_FOLD", 1) == 1 &&
         (long long)parts * ne_of(d) * 4 <= (long long)lfh::env_int("LINFUSION_F32_FOLD_KB", 64) * 1024;
}
// the forward state's partials: the same answer in the forward and in the backward pass, so that the state (and with it
// every result) has the same bits whether it is handed over or computed again
bool fold_fwd(int parts, int d) { return !narrow_apply(d) && fold(parts, d); }

unsigned heads_of(const lf::Layout& l) { return (unsigned)l.H | (unsigned)l.H << 16; }   // lf::HeadAt

template <int D, int FM>
int launch_reduce(const void* k, const void* v, lf::Layout l, float* partials, long long N,
                  const Plan32& p, long long BH, hipStream_t st) {
  using namespace lf;
  constexpr int lds = Sum32<D>::kBytes;
  // the plan counts 16-token tiles; this kernel's are 32 or 64 tokens
  constexpr int per = Reduce32s<D>::kTokens / kTile32;
  const lfh::Share sh = lfh::even_share((N + Reduce32s<D>::kTokens - 1) / Reduce32s<D>::kTokens, p.splits, kWavesPerWG,
                                        p.blk_reduce / per);
  state_reduce32s<D, FM><<<dim3(p.splits, (unsigned)BH), dim3(kThreads), lds, st>>>(
      (const float*)k, (const float*)v, l.batch, l.head, l.row, heads_of(l), sh.blk, N, partials);
  return LINFUSION_OK;
}

void launch_combine(const float* partials, int parts, int d, float* state, long long BH, hipStream_t st) {
  const int ne = ne_of(d);
  lf::combine_state<0><<<dim3((ne + lf::kCombineElems - 1) / lf::kCombineElems, (unsigned)BH),
                         dim3(lf::kCombineThreads), 0, st>>>(partials, parts, ne, state);
}

template <int D, int FM, bool NORM>
int fwd(const Fwd32Args& a) {
  using namespace lf;
  const Plan32& p = a.plan;
  if (a.ev) (void)hipEventRecord(a.ev[0], a.st);
  if (int rc = launch_reduce<D, FM>(a.k, a.v, a.lkv, a.partials, a.N, p, a.BH, a.st)) return rc;
  if (a.ev) (void)hipEventRecord(a.ev[1], a.st);
  const bool folded = a.out && fold_fwd(p.splits, D);
  if (!folded) launch_combine(a.partials, p.splits, D, a.state, a.BH, a.st);
  if (a.ev) (void)hipEventRecord(a.ev[2], a.st);
  if (a.out && narrow_apply(D)) {
    apply32<D, FM, NORM><<<dim3(p.apply_wgs, (unsigned)a.BH), dim3(kThreads), apply32_lds_bytes<D>(), a.st>>>(
        (const f32x4*)a.q, a.lq, (f32x4*)a.out, a.lo, a.state, a.eps, a.N, p.blk_apply);
  } else if (a.out) {
    constexpr int lds = consume32_lds_bytes<D, 1>();
    if (!lfh::allow_lds(apply32s<D, FM, NORM>, lds)) return LINFUSION_ERR_HIP;
    apply32s<D, FM, NORM><<<dim3(p.apply_wgs, (unsigned)a.BH), dim3(kThreads), lds, a.st>>>(
        (const f32x4*)a.q, a.lq.batch, a.lq.head, a.lq.row, heads_of(a.lq), p.blk_apply, a.N, folded ? a.partials : a.state,
        folded ? p.splits : 1, a.eps, folded ? a.state : nullptr, (f32x4*)a.out, a.lo.batch, a.lo.head, a.lo.row);
  }
  if (a.ev) (void)hipEventRecord(a.ev[3], a.st);
  return hipGetLastError() == hipSuccess ? LINFUSION_OK : LINFUSION_ERR_HIP;
}

size_t up(size_t x) { return (x + 255) & ~(size_t)255; }

struct Regions {
  Plan32 plan;
  size_t fpart, state, dpart, dstate, total;   // byte offsets: partials and sum of the forward state, of its gradient
};

int make_regions(int B, int H, long long N, int d, Regions* r) {
  size_t pbytes = 0;
  const int rc = launch_plan32(B, H, N, d, &r->plan, &pbytes);
  if (rc != LINFUSION_OK) return rc;
  const size_t st = up((size_t)B * H * ne_of(d) * sizeof(float));
  size_t o = 0;
  r->fpart = o; o += up(pbytes);
  r->state = o; o += st;
  r->dpart = o; o += up(pbytes);
  r->dstate = o; o += st;
  r->total = o;
  return LINFUSION_OK;
}

template <int D, int FM, bool NORM>
int bwd(const Bwd32Args& a, const Regions& r) {
  using namespace lf;
  const Plan32& p = r.plan;
  const long long BH = (long long)a.B * a.H;
  float* dpart = reinterpret_cast<float*>(a.ws + r.dpart);
  const float* state = a.saved_state;
  int parts = 1;
  if (!state) {
    float* fpart = reinterpret_cast<float*>(a.ws + r.fpart);
    if (int rc = launch_reduce<D, FM>(a.k, a.v, a.lkv, fpart, a.N, p, BH, a.st)) return rc;
    if (fold_fwd(p.splits, D)) {
      state = fpart;
      parts = p.splits;
    } else {
      float* whole = reinterpret_cast<float*>(a.ws + r.state);
      launch_combine(fpart, p.splits, D, whole, BH, a.st);
      state = whole;
    }
  }
  constexpr int lds_q = qs32_lds_bytes<D>(), lds_k = consume32_lds_bytes<D, 2>();
  if (!lfh::allow_lds(bwd_qs32<D, FM, NORM>, lds_q) || !lfh::allow_lds(bwd_kv32<D, FM>, lds_k)) return LINFUSION_ERR_HIP;
  bwd_qs32<D, FM, NORM><<<dim3(p.splits, (unsigned)BH), dim3(kThreads), lds_q, a.st>>>(
      (const f32x4*)a.q, a.lq, (const f32x4*)a.g, a.lg, (f32x4*)a.dq, a.ldq, state, parts, dpart, a.eps, a.N, p.blk_reduce);
  const float* dstate = dpart;
  int dparts = p.splits;
  if (!fold(p.splits, D)) {
    float* whole = reinterpret_cast<float*>(a.ws + r.dstate);
    launch_combine(dpart, p.splits, D, whole, BH, a.st);
    dstate = whole;
    dparts = 1;
  }
  bwd_kv32<D, FM><<<dim3(p.apply_wgs, (unsigned)BH), dim3(kThreads), lds_k, a.st>>>(
      (const f32x4*)a.k, (const f32x4*)a.v, a.lkv, (f32x4*)a.dk, (f32x4*)a.dv, a.ldkv, dstate, dparts, a.N, p.blk_apply);
  return hipGetLastError() == hipSuccess ? LINFUSION_OK : LINFUSION_ERR_HIP;
}

template <int D>
int fwd_fm(const Fwd32Args& a) {
  switch (a.fm) {
    case 0: return a.unnorm ? fwd<D, 0, false>(a) : fwd<D, 0, true>(a);
    case 1: return a.unnorm ? fwd<D, 1, false>(a) : fwd<D, 1, true>(a);
    default: return a.unnorm ? fwd<D, 2, false>(a) : fwd<D, 2, true>(a);
  }
}

template <int D>
int bwd_fm(const Bwd32Args& a, const Regions& r) {
  switch (a.fm) {
    case 0: return a.unnorm ? bwd<D, 0, false>(a, r) : bwd<D, 0, true>(a, r);
    case 1: return a.unnorm ? bwd<D, 1, false>(a, r) : bwd<D, 1, true>(a, r);
    default: return a.unnorm ? bwd<D, 2, false>(a, r) : bwd<D, 2, true>(a, r);
  }
}

}  // namespace

const char* apply32_name(int d) { return narrow_apply(d) ? "apply32" : "apply32s"; }

int run_fwd32(const Fwd32Args& a) {
  switch (a.d) {
#define X(DD) case DD: return fwd_fm<DD>(a);
    LF_FOR_D(X)
#undef X
  }
  return LINFUSION_ERR_UNSUPPORTED;
}

bool bwd32_supported(int d) { return d >= 8 && d <= 64 && d % 8 == 0; }

size_t bwd32_workspace_bytes(int B, int H, long long N, int d) {
  Regions r;
  if (!bwd32_supported(d) || make_regions(B, H, N, d, &r) != LINFUSION_OK) return 0;
  return r.total;
}

int run_bwd32(const Bwd32Args& a) {
  if (!bwd32_supported(a.d)) return LINFUSION_ERR_UNSUPPORTED;
  Regions r;
  const int rc = make_regions(a.B, a.H, a.N, a.d, &r);
  if (rc != LINFUSION_OK) return rc;
  switch (a.d) {
#define X(DD) case DD: return bwd_fm<DD>(a, r);
    LF_FOR_D(X)
#undef X
  }
  return LINFUSION_ERR_UNSUPPORTED;
}

}  // namespace lf32
