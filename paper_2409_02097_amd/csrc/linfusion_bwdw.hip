// Translation unit of the library: the fp16 backward pass at head widths above 80 (lf_backward_wide.hpp), on its own two
// kernels and the forward's wide state reduction and apply.
#include "../../include/linfusion.h"

#include "lf_backward_wide.hpp"
#include "lf_bwd_short16.hpp"
#include "lf_bwdw_api.hpp"
#include "lf_host_api.hpp"
#include "lf_wide_api.hpp"

namespace lfbw {

namespace {

size_t up(size_t x) { return (x + 255) & ~(size_t)255; }

struct Regions {
  lfw::WidePlan plan;         // the wide kernels' launch shape
  int wgs;                    // workgroups per head of bwdw_q and bwdw_k: one per CU, every wave a tile
  size_t partials, state, dstate, packed, packed_t, dzpart, gp, total;   // byte offsets
};

int make_regions(int B, int H, long long N, int d, int dtype, Regions* r) {
  size_t pbytes = 0;
  const int rc = lfw::wide_launch_plan(B, H, N, d, dtype, &r->plan, &pbytes);
  if (rc != LINFUSION_OK) return rc;
  const size_t BH = (size_t)B * H;
  const long long tiles = (N + 15) / 16, most = (tiles + lf::kWavesPerWG - 1) / lf::kWavesPerWG;
  long long wgs = lfh::env_int("LINFUSION_BWDW_WGS", lfh::num_cu()) / (long long)BH;
  r->wgs = (int)(wgs > most ? most : (wgs < 1 ? 1 : wgs));
  {   // dv: the forward's one-wave-per-tile apply, whatever the forward plan takes; 32-token tiles
    const long long t32 = ((N + lf::kTile - 1) / lf::kTile + lf::kWavesPerWG - 1) / lf::kWavesPerWG;
    r->plan.wave_apply = true;
    r->plan.apply_wgs = (int)(wgs > t32 ? t32 : (wgs < 1 ? 1 : wgs));
    r->plan.blk_apply = lf::kWavesPerWG;
  }
  const size_t st = up(BH * ((size_t)d * d + d) * sizeof(float));
  const size_t pk = up(BH * lfw::wide_packed_bytes(d, dtype));
  size_t o = 0;
  r->partials = o; o += up(pbytes);
  r->state = o; o += st;
  r->dstate = o; o += st;
  r->packed = o; o += pk;
  r->packed_t = o; o += pk;
  r->dzpart = o; o += up(BH * r->wgs * d * sizeof(float));
  r->gp = o; o += up(BH * (size_t)N * d * 2);
  r->total = o;
  return LINFUSION_OK;
}

// Longest stream that the one launch (lf_bwd_short16.hpp) takes.  It costs 4 to 5.5 us per 64 tokens whatever the heads up to
// 128, where its workgroups fill the chip; the launches below cost a chain of 30 to 45 us, and what their packed states and
// partials move, which grows with the heads.  us per call with the state given, these launches / that one, fp16:
//   4 heads of 160:   64 tokens 40.0 / 13.4, 256 42.8 / 28.2, 448 44.9 / 44.2, 512 44.7 / 49.7
//   16 heads of 96:   64 28.7 / 10.7, 192 30.9 / 17.1, 512 34.2 / 34.7, 640 37.0 / 42.3
//   100 heads of 128: 512 74.4 / 42.6, 1100 123 / 86.9
//   128 heads of 160: 1100 164 / 119;  of 96: 1100 100 / 77.2
// More heads: it runs a round of workgroups per 128 heads, these a round per 256, and both step where one begins.
//   129 heads, 1100 tokens: of 160 244 / 223, of 128 186 / 171, of 96 146 / 145;  385 of 160 468 / 462, 4096 of 160 3992 / 3720
// At 96 channels these are the faster ones from a length on that depends on the rounds:
//   3 rounds: 257 heads 1000 tokens 202 / 196, 1100 214 / 216      4: 385 heads 384 108 / 107, 448 121 / 122, 1100 238 / 288
//   5: 513 heads 512 184 / 174, 800 264 / 265                      6: 641 heads 320 145 / 141, 384 160 / 163
//   8: 1024 heads 320 195 / 188, 384 216 / 219                     16: 2048 heads 192 272 / 258, 256 314 / 316
int bwd_short_tokens(int d, long long heads) {
  if (lfh::env_int("LINFUSION_BWDW_SHORT", 1) == 2) return 0;   // never
  int line = 400 + 7 * (heads > 100 ? 100 : (int)heads);
  const long long cus = lfh::num_cu(), rounds = (2 * heads + cus - 1) / cus;
  if (d == 96 && rounds > 2) line = rounds == 3 ? 1024 : rounds == 4 ? 384 : rounds == 5 ? 768 : rounds <= 8 ? 320 : 192;
  return lfh::env_int("LINFUSION_BWDW_SHORT_TOKENS", line);
}

template <int D, int FM, bool NORM>
int run(const BwdWideArgs& a, const Regions& r) {
  using namespace lf;
  constexpr int CPR = D / 8, lds = BwdWaveShape<D>::kLdsBytes;
  const long long BH = (long long)a.B * a.H;
  hipStream_t st = a.st;
  unsigned char* ws = a.ws;
  float* partials = reinterpret_cast<float*>(ws + r.partials);
  float* whole = reinterpret_cast<float*>(ws + r.state);
  float* dwhole = reinterpret_cast<float*>(ws + r.dstate);
  unsigned char *packed = ws + r.packed, *packed_t = ws + r.packed_t;
  float* dzpart = reinterpret_cast<float*>(ws + r.dzpart);
  void* GP = ws + r.gp;
  const Layout dense{(long long)a.H * a.N * CPR, a.N * CPR, CPR, a.H};   // [B, H, N, D], in 16-byte units
  const dim3 blk(kThreads), grid(r.wgs, (unsigned)BH);
  const int splits = r.plan.splits;
  int rc;
  if (!lfh::allow_lds(bwdw_q<D, FM, NORM>, lds) || !lfh::allow_lds(bwdw_k<D, FM>, lds)) return LINFUSION_ERR_HIP;

  // the forward state, unless the caller kept it
  const float* state = a.saved_state;
  if (!state) {
    const lfw::WideReduceArgs x{a.k, a.v, a.B, a.H, a.N, a.d, a.dtype, FM, a.lkv, a.lkv, partials, whole, r.plan, st};
    if ((rc = lfw::run_wide_state(x)) != LINFUSION_OK) return rc;
    state = whole;
  }
  if constexpr (NORM) {   // (the un-normalized form has no ratio in which the scale of a query row cancels)
    if (a.N <= bwd_short_tokens(D, BH)) {
      using C = BwdShortCfg<D>;
      if (!lfh::allow_lds(bwd_short16<D, FM>, C::kLdsBytes)) return LINFUSION_ERR_HIP;
      bwd_short16<D, FM><<<dim3((unsigned)(2 * BH)), dim3(C::kThreads), C::kLdsBytes, st>>>(
          (const u32x4*)a.q, a.lq, (const u32x4*)a.g, a.lg, state, (int)a.N, a.eps, (const u32x4*)a.k, (const u32x4*)a.v, a.lkv,
          (u32x4*)a.dq, a.ldq, (u32x4*)a.dk, (u32x4*)a.dv, a.ldkv);
      return hipGetLastError() == hipSuccess ? LINFUSION_OK : LINFUSION_ERR_HIP;
    }
  }
  const float* z = NORM ? state + D * D : nullptr;
  bwdw_pack<D><<<dim3(D / 16, (unsigned)BH, 1), blk, 0, st>>>(state, 1, z, packed, packed_t, 1);
  bwdw_q<D, FM, NORM><<<grid, blk, lds, st>>>((const u32x4*)a.q, a.lq, (const u32x4*)a.g, a.lg, (u32x4*)a.dq, a.ldq,
                                              (u32x4*)GP, packed_t, z, dzpart, a.eps, a.N, kWavesPerWG);
  // dS' = sum phi(q)^T gp: as partials where the packing sums them (see kPackParts)
  const bool sum_first = splits > kPackParts;
  const lfw::WideReduceArgs x{a.q, GP, a.B, a.H, a.N, a.d, a.dtype, FM, a.lq, dense, partials, dwhole, r.plan, st};
  if ((rc = sum_first ? lfw::run_wide_reduce(x) : lfw::run_wide_reduce_partials(x)) != LINFUSION_OK) return rc;
  const bool parts = !sum_first && splits > 1;   // (one partial: the reduction wrote the state itself)
  bwdw_pack<D><<<dim3(D / 16, (unsigned)BH, 2), blk, 0, st>>>(parts ? partials : dwhole, parts ? splits : 1, z, packed,
                                                              packed_t, 0);
  // dv = dS^T phi(k)
  const lfw::WideApplyArgs y{a.k, a.dv, a.B, a.H, a.N, a.d, a.dtype, FM, 0.0f, true, a.lkv, a.ldkv, nullptr, packed, r.plan, st};
  if ((rc = lfw::run_wide_apply_packed(y)) != LINFUSION_OK) return rc;
  // dk = (dS v + dz) phi'(k)
  bwdw_k<D, FM><<<grid, blk, lds, st>>>((const u32x4*)a.k, (const u32x4*)a.v, a.lkv, (u32x4*)a.dk, a.ldkv, packed_t, dzpart,
                                        r.wgs, a.N, kWavesPerWG);
  return hipGetLastError() == hipSuccess ? LINFUSION_OK : LINFUSION_ERR_HIP;
}

template <int D>
int run_fm(const BwdWideArgs& a, const Regions& r) {
  switch (a.fm) {
    case 0: return a.unnorm ? run<D, 0, false>(a, r) : run<D, 0, true>(a, r);
    case 1: return a.unnorm ? run<D, 1, false>(a, r) : run<D, 1, true>(a, r);
    default: return a.unnorm ? run<D, 2, false>(a, r) : run<D, 2, true>(a, r);
  }
}

}  // namespace

bool bwd_wide_supported(int d, int dtype) { return dtype == LINFUSION_DTYPE_F16 && lfw::wide_supported(d); }

size_t bwd_wide_workspace_bytes(int B, int H, long long N, int d, int dtype) {
  Regions r;
  if (!bwd_wide_supported(d, dtype) || make_regions(B, H, N, d, dtype, &r) != LINFUSION_OK) return 0;
  return r.total;
}

int run_bwd_wide(const BwdWideArgs& a) {
  if (!bwd_wide_supported(a.d, a.dtype)) return LINFUSION_ERR_UNSUPPORTED;
  if ((a.N + 3) / 4 > 0x7fffffffLL) return LINFUSION_ERR_INVALID;   // (what has always been refused; no launch needs it)
  Regions r;
  const int rc = make_regions(a.B, a.H, a.N, a.d, a.dtype, &r);
  if (rc != LINFUSION_OK) return rc;
  switch (a.d) {
    case 96: return run_fm<96>(a, r);
    case 128: return run_fm<128>(a, r);
    case 160: return run_fm<160>(a, r);
  }
  return LINFUSION_ERR_UNSUPPORTED;
}

}  // namespace lfbw
