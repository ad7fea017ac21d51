// Second translation unit of the library: launches of the kernels for head widths above 64
// (lf_wide16.hpp).  Kept apart from linfusion.hip so that the two compile side by side.
#include "../../include/linfusion.h"

#include "lf_short16.hpp"
#include "lf_wave16.hpp"
#include "lf_host_api.hpp"
#include "lf_wide_api.hpp"

namespace lfw {

namespace {

using lfh::allow_lds;

// apply16_wave holds the (d + 2) x d fp16 operands of a head in one wave's registers, for both storage types
// (query rows are scaled into fp16's range as they are read): built for every wide width.
template <typename T, int D> constexpr bool wave_ok() { return true; }

// `combine`: leave the summed state in a.state; otherwise only the partials are left (one of them: the state itself, in
// a.state)
template <typename T, int D>
int reduce(const WideReduceArgs& a, hipEvent_t* ev, bool combine) {
  using namespace lf;
  constexpr int NE = D * D + D;
  const long long BH = (long long)a.B * a.H;
  const dim3 blk(kThreads);
  const u32x4* K = (const u32x4*)a.k;
  const u32x4* V = (const u32x4*)a.v;
  hipStream_t st = a.st;
  constexpr int lds1 = reduce16_wide_lds_bytes<T, D>();
  const dim3 g1(a.plan.splits, (unsigned)BH);
  // one workgroup per head: its partial is the state (same layout), and there is nothing to combine
  const bool direct = a.plan.splits == 1;
  float* part = direct ? a.state : a.partials;
  if (ev) (void)hipEventRecord(ev[0], st);
#define LFW_REDUCE(FM)                                                                       \
  {                                                                                          \
    if (!allow_lds(state_reduce16_wide<T, D, FM>, lds1)) return LINFUSION_ERR_HIP;           \
    state_reduce16_wide<T, D, FM><<<g1, blk, lds1, st>>>(K, a.lk, V, a.lv, part, a.N, a.plan.blk_reduce); \
  }
  switch (a.fm) {
    case 0: LFW_REDUCE(0) break;
    case 1: LFW_REDUCE(1) break;
    default: LFW_REDUCE(2) break;
  }
#undef LFW_REDUCE
  if (ev) (void)hipEventRecord(ev[1], st);
  if (!direct && combine)
    combine_state<0><<<dim3((NE + kCombineElems - 1) / kCombineElems, (unsigned)BH), dim3(kCombineThreads), 0, st>>>(
        a.partials, a.plan.splits, NE, a.state);
  if (ev && combine) (void)hipEventRecord(ev[2], st);
  return hipGetLastError() == hipSuccess ? LINFUSION_OK : LINFUSION_ERR_HIP;
}

// `parts`: a.state holds that many partials per head; with `keep` their sum goes there (0: packed already).  `ev`: recorded between packing
// and apply.
template <typename T, int D>
int apply(const WideApplyArgs& a, int parts = 1, float* keep = nullptr, hipEvent_t* ev = nullptr) {
  using namespace lf;
  const long long BH = (long long)a.B * a.H;
  const dim3 blk(kThreads);
  const u32x4* Q = (const u32x4*)a.q;
  u32x4* O = (u32x4*)a.out;
  const unsigned all = (unsigned)a.H | (unsigned)a.H << 16;   // HeadAt
  hipStream_t st = a.st;
  const dim3 g2(a.plan.apply_wgs, (unsigned)BH);
#define LFW_APPLY_W(FM, NORM, WW)                                                                            \
  {                                                                                                          \
    constexpr int lds2 = apply16_wide_lds_bytes<T, D, WW>();                                                 \
    if (!allow_lds(apply16_wide<T, D, FM, NORM, WW>, lds2)) return LINFUSION_ERR_HIP;                        \
    pack_state_wide<T, D, WW><<<dim3(ApplyWideShape<D, WW>::kKS, (unsigned)BH), dim3(64 * WW), 0, st>>>(     \
        a.state, a.packed, NORM ? 1 : 0);                                                                    \
    apply16_wide<T, D, FM, NORM, WW><<<g2, dim3(64 * WW), lds2, st>>>(Q, a.lq, O, a.lo, a.packed, a.eps, \
                                                                      a.N, a.plan.blk_apply);                \
  }
#define LFW_APPLY_WAVE(FM, NORM)                                                                             \
  if constexpr (wave_ok<T, D>()) {                                                                          \
    constexpr int lds2 = apply16_wave_lds_bytes<D>();                                                        \
    if (!allow_lds(apply16_wave<T, D, FM, NORM>, lds2)) return LINFUSION_ERR_HIP;                            \
    if (parts > 0) launch_pack_wave<D>(a.state, parts, keep, a.packed, NORM, (unsigned)BH, st);              \
    if (ev) (void)hipEventRecord(*ev, st);                                                                   \
    apply16_wave<T, D, FM, NORM><<<g2, blk, lds2, st>>>(Q, a.lq.batch, a.lq.head, a.lq.row, all,              \
                                                        a.plan.blk_apply, a.N, a.packed, a.eps, O, a.lo.batch, \
                                                        a.lo.head, a.lo.row);                                \
  } else {                                                                                                   \
    return LINFUSION_ERR_UNSUPPORTED;                                                                        \
  }
#define LFW_APPLY(FM, NORM)                                        \
  if (a.plan.wave_apply) { LFW_APPLY_WAVE(FM, NORM) }              \
  else if (a.plan.apply_waves == 8) LFW_APPLY_W(FM, NORM, 8) else LFW_APPLY_W(FM, NORM, 4)
  switch (a.fm) {
    case 0: if (a.unnorm) { LFW_APPLY(0, false) } else { LFW_APPLY(0, true) } break;
    case 1: if (a.unnorm) { LFW_APPLY(1, false) } else { LFW_APPLY(1, true) } break;
    default: if (a.unnorm) { LFW_APPLY(2, false) } else { LFW_APPLY(2, true) } break;
  }
#undef LFW_APPLY
#undef LFW_APPLY_WAVE
#undef LFW_APPLY_W
  return hipGetLastError() == hipSuccess ? LINFUSION_OK : LINFUSION_ERR_HIP;
}

// the whole call in one launch
template <typename T, int D, int CB, bool DEEP>
int launch_short_as(const WideArgs& a, dim3 grid, int parts) {
  using namespace lf;
  using C = Short16Cfg<T, D, CB, DEEP>;
  if (a.ev) (void)hipEventRecord(a.ev[0], a.st);
#define LFW_SHORT(FM, NORM)                                                                                       \
  {                                                                                                               \
    if (!allow_lds(short16<T, D, CB, FM, NORM, DEEP>, C::kLdsBytes)) return LINFUSION_ERR_HIP;                              \
    short16<T, D, CB, FM, NORM, DEEP><<<grid, dim3(C::kThreads), C::kLdsBytes, a.st>>>(                                     \
        (const u32x4*)a.k, (const u32x4*)a.v, a.lkv.batch, a.lkv.head, a.lkv.row,                                 \
        (unsigned)a.H | (unsigned)a.H << 16, (int)a.N, parts, (const u32x4*)a.q, a.lq.batch, a.lq.head, \
        a.lq.row, a.eps, a.state, (u32x4*)a.out, a.lo.batch, a.lo.head, a.lo.row);                                \
  }
  switch (a.fm) {
    case 0: if (a.unnorm) LFW_SHORT(0, false) else LFW_SHORT(0, true) break;
    case 1: if (a.unnorm) LFW_SHORT(1, false) else LFW_SHORT(1, true) break;
    default: if (a.unnorm) LFW_SHORT(2, false) else LFW_SHORT(2, true) break;
  }
#undef LFW_SHORT
  if (a.ev) { (void)hipEventRecord(a.ev[1], a.st); (void)hipEventRecord(a.ev[2], a.st); (void)hipEventRecord(a.ev[3], a.st); }
  return hipGetLastError() == hipSuccess ? LINFUSION_OK : LINFUSION_ERR_HIP;
}

// Several rounds of tokens between two barriers (DEEP) rather than one, where the call's workgroups take two thirds of the CUs at most:
// such a workgroup fills its CU's LDS, so that with more of them two calls on two streams would go one after the other.  us per call,
// alone / beside another on a second stream, one round -> several:
//   bf16 1 x 8 x 400 x 96 (120 workgroups) 12.0 / 13.7 -> 11.6 / 12.0,  2 x 8 x 256 x 128 (128) 9.9 / 11.5 -> 9.6 / 10.2,
//        1 x 8 x 512 x 128 (128) 14.2 / 16.3 -> 13.5 / 13.9,  2 x 8 x 256 x 160 (160) 12.3 / 14.7 -> 12.1 / 14.9
//   fp16 2 x 8 x 256 x 96 (144) 8.6 / 10.1 -> 8.4 / 10.2,  2 x 8 x 256 x 128 (128) 9.4 / 10.0 -> 9.2 / 9.8
//   too many: bf16 2 x 8 x 500 x 128 (256) 14.5 / 19.5 -> 13.9 / 25.0, of 96 (240) 13.8 / 19.9 -> 13.3 / 21.4, fp16 (256) 12.3 / 20.9 -> 12.3 / 21.8
// Not for fp16 of 160 channels (2 x 8 x 256 12.0 / 14.4 -> 12.0 / 14.8, four registers spilled), and not with half of a head's
// channels, whose sums leave no registers for it: fp16 12 x 8 x 256 x 160 forward and backward 50.4 -> 54.6 (58 spilled; two rounds
// 54.0, 27), bf16 forward 19.5 -> 20.6.
template <typename T, int D, int CB>
int launch_short(const WideArgs& a) {
  const int parts = a.out ? a.plan.short_parts : 1;
  const long long wgs = (long long)a.B * a.H * (D / (16 * CB)) * parts;
  const dim3 grid((unsigned)wgs);
  if constexpr (CB == 2 && (lf::NSplit<T>::value == 2 || D < 160)) {
    if (3 * wgs <= 2 * (long long)lfh::num_cu()) return launch_short_as<T, D, CB, true>(a, grid, parts);
  }
  return launch_short_as<T, D, CB, false>(a, grid, parts);
}

template <typename T, int D>
int run_short(const WideArgs& a) {
  return a.plan.short_half ? launch_short<T, D, D / 32>(a) : launch_short<T, D, 2>(a);
}

// The state of a problem whose call is one launch, with the bits that this launch leaves: summed by the same kernel, or
// by the state reduction where one workgroup of it sums a whole head -- the same products in the same order -- and the
// one-launch kernel's workgroups, which repeat phi(K), would be more than run at once, or in fp16 a head is one tile (us per
// state-only call, that kernel / the reduction, fp16: 128 heads of 128 x 160 8.7 / 9.5, 160 heads 14.3 / 9.7, 512 heads
// 30.4 / 15.9, 160 heads of 128 x 128 11.3 / 8.0; 128 heads of 32 x 160 7.9 / 6.3, in bf16 6.9 / 6.7 and 8 heads 6.1 / 6.4).
template <typename T, int D>
int state_of_short(const WideReduceArgs& a, hipEvent_t* ev) {
  const long long wgs = (long long)a.B * a.H * (a.plan.short_half ? 2 : D / 32);
  const bool one_tile = lf::NSplit<T>::value == 1 && a.N <= lf::kTile;
  if (a.plan.splits == 1 && (wgs > lfh::num_cu() || one_tile)) return reduce<T, D>(a, ev, true);
  return run_short<T, D>(WideArgs{nullptr, a.k, a.v, nullptr, a.B, a.H, a.N, a.d, a.dtype, a.fm, 0.0f, true, a.lk, a.lk, a.lk,
                                  a.partials, a.state, nullptr, a.plan, a.st, ev});
}

template <typename T, int D>
int run(const WideArgs& a) {
  const WideReduceArgs r{a.k, a.v, a.B, a.H, a.N, a.d, a.dtype, a.fm, a.lkv, a.lkv, a.partials, a.state, a.plan, a.st};
  if (a.plan.short_parts > 0) {
    if (a.out && a.out != a.q) return run_short<T, D>(a);
    if (!a.out) return state_of_short<T, D>(r, a.ev);
    // In place a workgroup of the one launch would read query rows that others have written a part of.  Where the room for
    // partial states, which this launch does not use, holds the queries, it reads a copy of them, unless heads of more than
    // 128 tokens take it a second round (us per call, the split path / the same state, then the apply kernel / a copy:
    // bf16 1 x 5 x 439 x 96 15.9 / 19.1 / 15.3, fp16 2 x 8 x 256 x 160 22.9 / 20.5 / 15.1, 12 x 8 x 256 x 160 31.4 / 28.3 / 28.2,
    // 25 x 8 x 100 x 160 31.8 / 32.0 / 29.8, 20 x 8 x 200 x 160 38.2 / 38.2 / 42.8).
    constexpr int CPR = D / 8;
    const bool rounds = (long long)a.B * a.H * (a.plan.short_half ? 2 : D / 32) > lfh::num_cu();
    if ((!rounds || a.N <= 128) && (long long)a.plan.splits * (D * D + D) * 4 >= a.N * D * 2) {
      if (a.ev) (void)hipEventRecord(a.ev[0], a.st);
      lf::u32x4* copy = (lf::u32x4*)a.partials;
      const unsigned chunks = (unsigned)(a.N * CPR);
      lf::copy_rows<CPR><<<dim3((chunks + lf::kThreads - 1) / lf::kThreads, (unsigned)((long long)a.B * a.H)), dim3(lf::kThreads),
                           0, a.st>>>((const lf::u32x4*)a.q, a.lq.batch, a.lq.head, a.lq.row,
                                      (unsigned)a.H | (unsigned)a.H << 16, chunks, copy);
      WideArgs b = a;
      b.q = copy;
      b.lq = lf::Layout{(long long)a.H * chunks, (long long)chunks, CPR, a.H};
      b.ev = nullptr;
      const int rc = run_short<T, D>(b);
      if (a.ev) { (void)hipEventRecord(a.ev[1], a.st); (void)hipEventRecord(a.ev[2], a.st); (void)hipEventRecord(a.ev[3], a.st); }
      return rc;
    }
    // Else the same state, then the apply of a wave per tile, whose arithmetic is the same.
    int rc = state_of_short<T, D>(r, a.ev);
    if (rc != LINFUSION_OK) return rc;
    const WideApplyArgs p{a.q, a.out, a.B, a.H, a.N, a.d, a.dtype, a.fm, a.eps, a.unnorm, a.lq, a.lo, a.state, a.packed,
                          a.plan, a.st};
    rc = apply<T, D>(p, 1, nullptr, a.ev ? a.ev + 2 : nullptr);
    if (a.ev) (void)hipEventRecord(a.ev[3], a.st);
    return rc;
  }
  const bool fuse = a.out && a.plan.wave_apply;   // the partials are summed where the operands are packed
  int rc = reduce<T, D>(r, a.ev, !fuse);
  if (rc != LINFUSION_OK) return rc;
  if (a.out) {
    const bool partials = fuse && a.plan.splits > 1;
    const WideApplyArgs p{a.q, a.out, a.B, a.H, a.N, a.d, a.dtype, a.fm, a.eps, a.unnorm, a.lq, a.lo,
                          partials ? a.partials : a.state, a.packed, a.plan, a.st};
    rc = apply<T, D>(p, partials ? a.plan.splits : 1, partials ? a.state : nullptr, fuse && a.ev ? a.ev + 2 : nullptr);
  }
  if (a.ev) (void)hipEventRecord(a.ev[3], a.st);
  return rc;
}

}  // namespace

#define LFW_FOR_D(X) X(96) X(128) X(160)

// room for the operands of any of the apply kernels
template <typename T, int D>
constexpr size_t pack_bytes() {
  size_t b = lf::PackWide<T, D, 4>::kHeadBytes > lf::PackWide<T, D, 8>::kHeadBytes ? lf::PackWide<T, D, 4>::kHeadBytes
                                                                                   : lf::PackWide<T, D, 8>::kHeadBytes;
  if (wave_ok<T, D>() && (size_t)lf::PackWave<D>::kHeadBytes > b) b = lf::PackWave<D>::kHeadBytes;
  return b;
}

bool wide_supported(int d) {
  switch (d) {
#define X(DD) case DD:
    LFW_FOR_D(X)
#undef X
    return true;
  }
  return false;
}

bool wave_apply_supported(int d, int dtype) {
  switch (d) {
#define X(DD) \
  case DD: return dtype == LINFUSION_DTYPE_F16 ? wave_ok<lf::F16, DD>() : wave_ok<lf::BF16, DD>();
    LFW_FOR_D(X)
#undef X
  }
  return false;
}

size_t wide_packed_bytes(int d, int dtype) {
  switch (d) {
#define X(DD) \
  case DD: return dtype == LINFUSION_DTYPE_F16 ? pack_bytes<lf::F16, DD>() : pack_bytes<lf::BF16, DD>();
    LFW_FOR_D(X)
#undef X
  }
  return 0;
}

int run_wide_reduce(const WideReduceArgs& a) {
  switch (a.d) {
#define X(DD) \
  case DD: return a.dtype == LINFUSION_DTYPE_F16 ? reduce<lf::F16, DD>(a, nullptr, true) : reduce<lf::BF16, DD>(a, nullptr, true);
    LFW_FOR_D(X)
#undef X
  }
  return LINFUSION_ERR_UNSUPPORTED;
}

int run_wide_state(const WideReduceArgs& a) {
  if (a.plan.short_parts == 0) return run_wide_reduce(a);
  switch (a.d) {
#define X(DD) \
  case DD: return a.dtype == LINFUSION_DTYPE_F16 ? state_of_short<lf::F16, DD>(a, nullptr) : state_of_short<lf::BF16, DD>(a, nullptr);
    LFW_FOR_D(X)
#undef X
  }
  return LINFUSION_ERR_UNSUPPORTED;
}

int run_wide_reduce_partials(const WideReduceArgs& a) {
  switch (a.d) {
#define X(DD) \
  case DD: return a.dtype == LINFUSION_DTYPE_F16 ? reduce<lf::F16, DD>(a, nullptr, false) : reduce<lf::BF16, DD>(a, nullptr, false);
    LFW_FOR_D(X)
#undef X
  }
  return LINFUSION_ERR_UNSUPPORTED;
}

int run_wide_apply_packed(const WideApplyArgs& a) {
  if (!a.plan.wave_apply || a.dtype != LINFUSION_DTYPE_F16) return LINFUSION_ERR_UNSUPPORTED;
  switch (a.d) {
#define X(DD) case DD: return apply<lf::F16, DD>(a, 0);
    LFW_FOR_D(X)
#undef X
  }
  return LINFUSION_ERR_UNSUPPORTED;
}

int run_wide(const WideArgs& a) {
  switch (a.d) {
#define X(DD) \
  case DD: return a.dtype == LINFUSION_DTYPE_F16 ? run<lf::F16, DD>(a) : run<lf::BF16, DD>(a);
    LFW_FOR_D(X)
#undef X
  }
  return LINFUSION_ERR_UNSUPPORTED;
}

}  // namespace lfw
