// fp32 kernels of the three-kernel path and of the backward pass, on the bf16 matrix-core instructions.
//
// The fp32 matrix instruction (16x16x4) shares its unit with the vector instructions: measured on MI355X, a loop of 16
// of them takes 233 ns, eight phi 181 ns, both together 419 ns -- the times add up, also with two waves per SIMD, and at
// d = 64 the products alone are two thirds of the time the bytes need.  The bf16 instructions run beside the vector
// unit.  Every fp32 value is therefore split into three bf16 terms, x = x1 + x2 + x3 (each the bf16 rounding of what the
// terms before it left: 24 bits), and a product is the sum of the six partial products
// whose weight is 2^-16 of the leading one or more (a1 b1, a1 b2, a2 b1, a2 b2, a1 b3, a3 b1; the three dropped ones are
// below 2^-24, fp32's own rounding), accumulated in fp32, smallest first.
//
// The three terms hold 0 and every value from 2^-110 up to below 2^127 exactly.  Smaller ones lose bits, since the third term
// runs into bf16's subnormals (phi of a key below -76 is such a value), and just above 2^127 the first term may round to
// infinity; an infinity leaves NaN as its second term.  A tile with such a value, or a head whose state has one, is
// therefore multiplied on the fp32 instruction, from the same registers: the operands and results of both instructions lie
// alike in the lanes; the state reduction goes on with it from the first such tile of a wave.  The test (Low) costs half an
// instruction per value, one in bwd_qs32: 20 heads of 64 channels and 16384 tokens 83.3 -> 84.4 us per call, forward and backward
// of 96 heads of 40 and 4096 tokens 187.8 -> 193.7.  (The matrix instructions keep subnormal operands, products and sums: measured on MI355X.)
//
//   state_reduce32s  S, z partials        reads K, V                       (Prop. 2: g'(X)^T X; Eq. 5: Z)
//   apply32s         out                  reads Q, writes out
//   bwd_qs32         dQ and dS, dz partials   reads Q, g, writes dQ        (formulas: lf_backward16.hpp)
//   bwd_kv32         dK, dV               reads K, V, writes both
//
// state_reduce32s contracts over tokens: lane (m = lane % 16, kq = lane / 16) loads the CPL = ceil(d / 16) channels
// from CPL m on of tokens 4 j + kq, j = 0 .. 7, straight from memory (four neighbouring rows per instruction), which is
// the operand layout (any assignment of tokens to the contraction index does): block i of the state holds channels CPL row + i.  No LDS before the end, no transposition.
//
// The other three stream 16-token tiles through a ring of LDS slots per wave, filled by asynchronous global->LDS
// copies; no workgroup barrier in the loop.  A tile is read from LDS in two forms:
//   row form     lane (m, kq) reads the 16-byte chunks 4 T + kq of token m: the operand whose contraction runs over
//                channels (in the order 16 T + 4 kq + e), and at the same time the layout of the products' results
//                (row 4 kq + r of output block T is channel 16 T + 4 kq + r of token m), so everything elementwise
//                happens in place;
//   column form  lane (m, kq) reads channel 16 i + m of tokens 4 u + kq: the operand whose contraction runs over
//                tokens (the state's gradient).
// Chunks of a row are rotated by a row-dependent amount so that both forms are (nearly) free of bank conflicts.
// The waves' priorities follow their progress (Pace; us per call without / with): 96 heads of 40 channels and 4096 tokens, forward and
// backward 180.3 / 175.0, 700 tokens 60.9 / 59.9, 16 heads, forward, 20.9 / 20.6; 20 heads of 64 and 16384 tokens, forward, 80.4 / 79.2.
// The state is loaded before the first tiles are requested rather than behind them: 175.1 -> 174.4, 20.8 -> 20.6, 79.3 -> 79.2 us.  Up to
// 24 channels neither holds for short streams (forward and backward of 96 heads of 24: 300 tokens 29.9 -> 29.4 without, 700 tokens 41.6 ->
// 41.2, of 16 700 tokens 28.6 -> 28.2): there the state comes behind the tiles, and a wave of few tiles keeps its priority.
// They take a state as `parts` partial states and sum them while they stage it (parts = 1: a finished
// state): where the partials are few that is cheaper than a launch of combine_state in between.
#pragma once
#include "lf_common.hpp"
#include "lf_fp32.hpp"       // kTile32, wait_vmcnt32
#include "lf_reduce16.hpp"   // kWavesPerWG, kThreads

namespace lf {

// x = h + m + l, each term the bf16 rounding of what was left; four values, packed in pairs
struct Split4 { u32x2 t[3]; };
LF_DEV Split4 split3(f32x4 x) {
  Split4 s;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    s.t[k] = u32x2{pack2<BF16>(x[0], x[1]), pack2<BF16>(x[2], x[3])};
    if (k < 2) {
      float t0, t1, t2, t3;
      unpack2<BF16>(s.t[k][0], t0, t1);
      unpack2<BF16>(s.t[k][1], t2, t3);
      x[0] -= t0; x[1] -= t1; x[2] -= t2; x[3] -= t3;
    }
  }
  return s;
}
// eight values: the operand of one lane of v_mfma_f32_16x16x32_bf16, three terms
struct Split8 { u32x4 t[3]; };
LF_DEV Split8 join(const Split4& a, const Split4& b) {
  Split8 s;
#pragma unroll
  for (int k = 0; k < 3; ++k) s.t[k] = u32x4{a.t[k][0], a.t[k][1], b.t[k][0], b.t[k][1]};
  return s;
}
LF_DEV f32x4 mfma_split(const Split8& a, const Split8& b, f32x4 c) {
  c = mfma_16x16x32<BF16>(a.t[2], b.t[0], c);
  c = mfma_16x16x32<BF16>(a.t[0], b.t[2], c);
  c = mfma_16x16x32<BF16>(a.t[1], b.t[1], c);
  c = mfma_16x16x32<BF16>(a.t[1], b.t[0], c);
  c = mfma_16x16x32<BF16>(a.t[0], b.t[1], c);
  return mfma_16x16x32<BF16>(a.t[0], b.t[0], c);
}
// the same on four values per lane (contraction over 16)
LF_DEV f32x4 mfma_16x16x16_bf16(u32x2 a, u32x2 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
}
LF_DEV f32x4 mfma_split(const Split4& a, const Split4& b, f32x4 c) {
  c = mfma_16x16x16_bf16(a.t[2], b.t[0], c);
  c = mfma_16x16x16_bf16(a.t[0], b.t[2], c);
  c = mfma_16x16x16_bf16(a.t[1], b.t[1], c);
  c = mfma_16x16x16_bf16(a.t[1], b.t[0], c);
  c = mfma_16x16x16_bf16(a.t[0], b.t[1], c);
  return mfma_16x16x16_bf16(a.t[0], b.t[0], c);
}

// The same products on the fp32 instruction, for operands that three terms do not hold: lane (m, kq) gives one value of the
// contraction's index kq at a time, so any order in which both operands' values are taken does.
LF_DEV f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
LF_DEV f32x4 mfma_f32(f32x4 a, f32x4 b, f32x4 c) {
#pragma unroll
  for (int e = 0; e < 4; ++e) c = mfma_f32(a[e], b[e], c);
  return c;
}
// x, for a path that is hardly ever taken: the empty statement keeps the compiler from working out ahead of the branch, or of
// the loop around it, what only that path needs (d = 64: the state's fp32 values, 96 registers)
template <typename X> LF_DEV X rarely(X x) {
  asm volatile("" : "+v"(x));
  return x;
}
// x1 + x2 + x3 of what join put together: exact where the terms hold the value
LF_DEV f32x4 joined(const Split8& a, int half) {
  f32x4 x;
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    float h0, h1, m0, m1, l0, l1;
    unpack2<BF16>(rarely(a.t[0][2 * half + w]), h0, h1);
    unpack2<BF16>(rarely(a.t[1][2 * half + w]), m0, m1);
    unpack2<BF16>(rarely(a.t[2][2 * half + w]), l0, l1);
    x[2 * w] = h0 + (m0 + l0);
    x[2 * w + 1] = h1 + (m1 + l1);
  }
  return x;
}

// Whether three bf16 terms hold every value that a wave is about to split.
constexpr float kSplitLow = 0x1p-110f, kSplitHigh = 0x1p127f;
LF_DEV bool splits_exactly(float x) {   // (a NaN does as well as any: either instruction gives NaN)
  const float a = fabsf(x);
  return !((a < kSplitLow) & (a > 0.0f)) & !(a >= kSplitHigh);
}
LF_DEV bool all_lanes(bool x) { return __builtin_amdgcn_ballot_w64(!x) == 0; }
// What a wave tests before it splits: the smallest magnitude.  (The three terms of an infinity, or of a value that the first
// term rounds to one, end in a NaN, which every product with them shows afterwards: nothing has to look for those first.)
// Passes only where no value is 0; splits_exactly decides where this does not.
struct Low {
  float lo = 1.0f;
  // (written out: left to itself the compiler quiets every operand of a minimum first)
  LF_DEV void add(float a, float b) { asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(lo) : "v"(a), "v"(b)); }
  LF_DEV bool passes() const { return all_lanes(lo >= kSplitLow); }
};
// the same for phi of the values that are given: elu + 1 is e^x below 0, and e^-76 above 2^-110
template <int FM> struct PhiLow : Low {
  LF_DEV void add(float a, float b) {
    if constexpr (FM == kPhiEluPlusOne) asm("v_min3_f32 %0, %1, %2, %0" : "+v"(lo) : "v"(a), "v"(b));
    else Low::add(a, b);
  }
  LF_DEV bool passes() const {
    if constexpr (FM == kPhiEluPlusOne) return all_lanes(lo >= -76.0f);
    else return Low::passes();
  }
};
// with the largest magnitude too, where nothing is looked at afterwards
template <typename L> struct Both : L {
  float hi = 1.0f;
  LF_DEV void add(float a, float b) {
    L::add(a, b);
    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(hi) : "v"(a), "v"(b));
  }
  LF_DEV bool passes() const { return L::passes() && all_lanes(hi < 0.5f * kSplitHigh); }   // (half: x + 1 may round up)
};
// A value that did not pass, for phi below: elu + 1 of anything from -200 down is 0.  (A NaN stays one.)
template <int FM> LF_DEV float unmasked(float x) { return FM == kPhiEluPlusOne && x < -200.0f ? -200.0f : x; }
// phi of a value that passed or has been unmasked
template <int FM> LF_DEV float phi32(float x) { return phi<FM, true, false>(x); }

template <int D> struct Tile32 {
  static constexpr int kCH = D / 4;                        // 16-byte chunks per token row
  static constexpr int kMT = (D + 15) / 16;                // 16-channel blocks
  static constexpr int kNL = (kTile32 * kCH + 63) / 64;    // copy instructions per tile
  static constexpr int kTB = kNL * 1024;                   // bytes per tile (whole 1 KiB deposits)
  static constexpr int kG = (kCH % 16 == 0) ? 16 : ((kCH % 8 == 0) ? 8 : ((kCH % 4 == 0) ? 4 : 2));
  static_assert(D % 8 == 0 && D <= 64, "widths of the fp32 kernels");
  // rotation of row r in chunks.  16 rows at the same chunk (row form) need kG different rotations; four
  // consecutive rows at the same four chunks (column form) need rotations four chunks apart where the row stride is a
  // multiple of the bank count (kG = 16) or of half of it (kG = 8).
  static LF_DEV int rot(int r) {
    if constexpr (kG == 16) return ((r & 3) << 2) | (r >> 2);
    else if constexpr (kG == 8) return (((r >> 1) & 1) << 2) | (r >> 2);
    else return ((r * kG) >> 4) & (kG - 1);
  }
  static LF_DEV int place(int r, int c) {                  // byte offset of chunk c of row r
    int x = c + rot(r);
    if (x >= kCH) x -= kCH;
    return (r * kCH + x) * 16;
  }
};

// NT: tensors per slot.  R: slots (R - 1 tiles in flight).
// Priorities by progress: in narrow heads not below 64 tokens per wave, where what comes behind the loop is as long as the loop.
template <int D> LF_DEV bool paced(long long N) { return D > 24 || N >= (long long)gridDim.x * (kWavesPerWG * 64); }

template <int D, int NT, int R_>
struct Ring32 {
  using TC = Tile32<D>;
  static constexpr int CH = TC::kCH, MT = TC::kMT, KS = (MT + 1) / 2, NL = TC::kNL, TB = TC::kTB, R = R_, NE = D * D + D;
  static constexpr int kSlot = NT * TB;
  static constexpr int kRingBytes = R * kWavesPerWG * kSlot;
  static constexpr int kStageOffset = (R - 1) * kWavesPerWG * kSlot;   // free until the stream loop starts
  static constexpr bool kWhole = D % 16 == 0;
  static_assert(R >= 2 && R <= 3, "ring depths the wait counts are written for");
  static_assert(MT * 4 <= 16, "row form: chunk 4 T + kq");

  const f32x4* X[NT];
  int off[NT][NL];
  long long N;
  unsigned char* smem;
  int lane, wave, m, kq;
  int rs[NT];
  int trow[NL], tpos[NL], sbyte[NL];
  TileIter it, ahead;

  LF_DEV Ring32(const f32x4* const (&x)[NT], const int (&rs_)[NT], long long N_, int tiles_per_block, int wg, int nwg,
                unsigned char* smem_)
      : N(N_), smem(smem_), lane(threadIdx.x & 63), wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)),
        it(wg, nwg, wave, tiles_per_block, (N_ + kTile32 - 1) / kTile32), ahead(it) {
    m = lane & 15;
    kq = lane >> 4;
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int P = u * 64 + lane, r = P / CH, pos = P % CH;
      int c = pos - TC::rot(r & 15);      // position pos of row r receives chunk c
      if (c < 0) c += CH;
      trow[u] = r;
      tpos[u] = pos;
      sbyte[u] = TC::place(r & 15, pos);   // where the chunk that leaves for position pos lies
#pragma unroll
      for (int t = 0; t < NT; ++t) off[t][u] = r * rs_[t] + c;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      X[t] = x[t];
      rs[t] = rs_[t];
    }
  }

  LF_DEV unsigned char* tile_ptr(int slot, int which) const { return smem + (slot * kWavesPerWG + wave) * kSlot + which * TB; }
  LF_DEV int lim_of(long long tile) const {
    const long long rem = N - tile * kTile32;
    return rem < kTile32 ? (int)rem : kTile32;
  }
  // always NT NL vector memory instructions, issued by every lane (rows past N and the padding re-read chunk 0)
  LF_DEV void issue_copy(long long tile, int slot) {
    const int lim = lim_of(tile);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const f32x4* p = X[t] + tile * kTile32 * rs[t];
      unsigned char* sl = tile_ptr(slot, t);
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        const int c = trow[u] < lim ? off[t][u] : 0;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(p + c),
                                         (LF_LDS void*)(sl + u * 1024), 16, 0, 2 /* nt */);
      }
    }
  }
  LF_DEV void prefetch() {
#pragma unroll
    for (int s = 0; s < R - 1; ++s) {
      if (ahead.valid()) issue_copy(ahead.t, s);
      ahead.next();
    }
  }
  // The tile about to be used has landed.  Issued after its copies: those of the R - 1 tiles behind it and the SN
  // stores of each of the up to R - 1 tiles finished since.
  template <int SN>
  LF_DEV void wait_tile(int iter, bool more) {
    constexpr int C = (R - 1) * NT * NL;
    static_assert(C + (R - 1) * SN <= 63, "the counter of outstanding vector memory operations has six bits");
    if (!more) wait_vmcnt32<0>();
    else if (iter == 0) wait_vmcnt32<C>();
    else if (iter == 1 || R == 2) wait_vmcnt32<C + SN>();
    else wait_vmcnt32<C + (R - 1) * SN>();
  }
  // coalesced stores of tile part `which` to rows of `Oh` in memory order: always NL instructions
  LF_DEV void store_tile(long long tile, int slot, int which, f32x4* Oh, int rso) {
    const unsigned char* sl = tile_ptr(slot, which);
    const int lim = lim_of(tile);
    f32x4* op = Oh + tile * kTile32 * rso;   // (rso is the same for every tile: the products below leave the loop)
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const f32x4 w = *reinterpret_cast<const f32x4*>(sl + sbyte[u]);
      if (trow[u] < lim) __builtin_nontemporal_store(w, op + trow[u] * rso + tpos[u]);
    }
  }

  // ---- row form ------------------------------------------------------------------------------------------
  LF_DEV bool has(int T) const { return kWhole || 4 * T + 3 < CH || 4 * T + kq < CH; }
  LF_DEV void read_rows(int slot, int which, f32x4 (&x)[MT]) const {
#pragma unroll
    for (int T = 0; T < MT; ++T) {
      x[T] = f32x4{1, 1, 1, 1};   // (past d: multiplied by zeros of the state, and no 0 that would not pass)
      if (has(T)) x[T] = *reinterpret_cast<const f32x4*>(tile_ptr(slot, which) + TC::place(m, 4 * T + kq));
    }
  }
  LF_DEV void write_rows(int slot, int which, const f32x4 (&x)[MT]) const {
#pragma unroll
    for (int T = 0; T < MT; ++T)
      if (has(T)) *reinterpret_cast<f32x4*>(tile_ptr(slot, which) + TC::place(m, 4 * T + kq)) = x[T];
  }
  // ---- column form: channel 16 i + m of token 4 u + kq (past d: some value inside the tile, whose row or column of
  // the products nobody reads)
  LF_DEV float read_col(int slot, int which, int u, int i) const {
    int c = 4 * i + (m >> 2);
    if (!kWhole && 4 * i + 3 >= CH) c = c < CH ? c : 0;
    return *reinterpret_cast<const float*>(tile_ptr(slot, which) + TC::place(4 * u + kq, c) + (m & 3) * 4);
  }

  // ---- the head's state ------------------------------------------------------------------------------------
  static constexpr int kStageBytes = NE * 4 + kWavesPerWG * 4;   // the state, and a word per wave
  // The sum of `parts` partial states, this thread's share of it: before the first tiles are requested, since a request that
  // waits behind the chip's first two tiles comes two microseconds later; in narrow heads behind them (kLate), since there the tiles
  // are small and it is they that wait for the sums.
  static constexpr bool kLate = D <= 24;
  static constexpr int kPer = (NE / 4 + kThreads - 1) / kThreads;
  static LF_DEV int share(int i) {   // (past the state's end: its last element again)
    const int e = i * kThreads + (int)threadIdx.x;
    return e < NE / 4 ? e : NE / 4 - 1;
  }
  static LF_DEV void load_state(const float* src, int parts, f32x4 (&s)[kPer]) {
    const f32x4* p = reinterpret_cast<const f32x4*>(src);
    if (parts == 1) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) s[i] = p[share(i)];
    } else if (parts <= 4) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) s[i] = sum_up_to<4>(p + share(i), parts, NE / 4);
    } else {
#pragma unroll
      for (int i = 0; i < kPer; ++i) s[i] = sum_up_to<kFoldParts>(p + share(i), parts, NE / 4);
    }
  }
  // -> LDS (and, by one workgroup of the head, -> `keep`); raw: three terms do not hold S
  LF_DEV const float* stage_state(const f32x4 (&s)[kPer], float* keep, bool& raw) {
    f32x4* st = reinterpret_cast<f32x4*>(smem + kStageOffset);
    int* flags = reinterpret_cast<int*>(smem + kStageOffset + NE * 4);
    bool ok = true;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = share(i);   // (the last element is written by several threads, with one value)
      if (!kLate || i * kThreads + (int)threadIdx.x < NE / 4) {   // (narrow: by one, where most threads would have it)
        st[e] = s[i];
        if (keep) reinterpret_cast<f32x4*>(keep)[e] = s[i];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) ok &= splits_exactly(s[i][k]) | (4 * e >= D * D);
    }
    const bool exact = all_lanes(ok);
    if (lane == 0) flags[wave] = !exact;
    __syncthreads();
    raw = __builtin_amdgcn_readfirstlane((flags[0] | flags[1]) | (flags[2] | flags[3])) != 0;
    return reinterpret_cast<const float*>(st);
  }
  // operands of  out[o] = sum_c M'[o][c] x[c]:  element M[o][c], or (TRANSPOSED) M[c][o], at output channel
  // 16 t + m and input channels 16 T + 4 kq + e, T = 2 s and 2 s + 1; zero outside d.  raw (stage_state): A keeps the fp32
  // values as they are, those of T = 2 s in t[0] and of 2 s + 1 in t[1].
  template <bool TRANSPOSED>
  LF_DEV f32x4 state_values(const float* st, int t, int T) const {
    f32x4 x = f32x4{0, 0, 0, 0};
    if (T < MT) {
      const int o = 16 * t + m;
      const bool ok = (kWhole || 16 * t + 15 < D || o < D) && has(T);
      const int oo = ok ? o : 0, cc = ok ? 16 * T + 4 * kq : 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float y = TRANSPOSED ? st[(cc + e) * D + oo] : st[oo * D + cc + e];
        x[e] = ok ? y : 0.0f;
      }
    }
    return x;
  }
  template <bool TRANSPOSED>
  LF_DEV void build_A(const float* st, bool raw, Split8 (&A)[MT][KS]) const {
    if (__builtin_expect(raw, 0)) {
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          A[t][s].t[0] = __builtin_bit_cast(u32x4, state_values<TRANSPOSED>(st, t, 2 * s));
          A[t][s].t[1] = __builtin_bit_cast(u32x4, state_values<TRANSPOSED>(st, t, 2 * s + 1));
          A[t][s].t[2] = u32x4{0, 0, 0, 0};
        }
      return;
    }
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int s = 0; s < KS; ++s)
        A[t][s] = join(split3(state_values<TRANSPOSED>(st, t, 2 * s)), split3(state_values<TRANSPOSED>(st, t, 2 * s + 1)));
  }
  LF_DEV void load_vec(const float* st, f32x4 (&z)[MT]) const {
#pragma unroll
    for (int T = 0; T < MT; ++T) {
      z[T] = f32x4{0, 0, 0, 0};
      if (has(T)) z[T] = *reinterpret_cast<const f32x4*>(st + D * D + 16 * T + 4 * kq);
    }
  }
  template <typename L>
  static LF_DEV L seen(const f32x4 (&x)[MT]) {
    L sp;
#pragma unroll
    for (int T = 0; T < MT; ++T) {
      sp.add(x[T][0], x[T][1]);
      sp.add(x[T][2], x[T][3]);
    }
    return sp;
  }
  template <int FM>
  static LF_DEV void unmask(f32x4 (&x)[MT]) {
#pragma unroll
    for (int T = 0; T < MT; ++T)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[T][e] = unmasked<FM>(x[T][e]);
  }
  static LF_DEV bool exact(const f32x4 (&x)[MT]) {   // of this lane's values
    bool ok = true;
#pragma unroll
    for (int T = 0; T < MT; ++T)
#pragma unroll
      for (int e = 0; e < 4; ++e) ok &= splits_exactly(rarely(x[T][e]));
    return ok;
  }
  // x in row form, finite past d; A from build_A.  A NaN among a token's terms is in all of its results.
  LF_DEV void products(const Split8 (&A)[MT][KS], const f32x4 (&x)[MT], f32x4 (&acc)[MT]) const {
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const Split8 b = join(split3(x[2 * s]), 2 * s + 1 < MT ? split3(x[2 * s + 1 < MT ? 2 * s + 1 : 0]) : Split4{});
#pragma unroll
      for (int t = 0; t < MT; ++t) acc[t] = mfma_split(A[t][s], b, acc[t]);
    }
  }
  static LF_DEV bool sound(const f32x4 (&acc)[MT]) { return acc[0][0] == acc[0][0]; }
  // the same whatever the state and the values: A and raw from build_A
  LF_DEV void products_any(const Split8 (&A)[MT][KS], bool raw, const f32x4 (&x)[MT], f32x4 (&acc)[MT]) const {
    if (!raw && all_lanes(exact(x))) {
      products(A, x, acc);
      return;
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = f32x4{0, 0, 0, 0};
    if (raw) {
#pragma unroll
      for (int T = 0; T < MT; ++T)
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[t] = mfma_f32(__builtin_bit_cast(f32x4, A[t][T / 2].t[T % 2]), x[T], acc[t]);
    } else {
#pragma unroll
      for (int T = 0; T < MT; ++T)
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[t] = mfma_f32(joined(A[t][T / 2], T % 2), x[T], acc[t]);
    }
  }
  // over the four lanes that share a token
  static LF_DEV float token_sum(float x) {
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
  }

};

// The workgroup's partial: the four waves' sums meet in LDS in a fixed order, (w0 + w2) + (w1 + w3), and leave as 16-byte
// stores.  `put(copy, add)` stores one wave's sums into (adds them to) a copy of the state.
template <int D> struct Sum32 {
  static constexpr int NE = D * D + D;
  static constexpr int kCopies = 4 * NE * 4 <= 32768 ? 4 : 2;
  static constexpr int kBytes = kCopies * NE * 4;
  template <typename Put>
  static LF_DEV void write(unsigned char* smem, Put put, float* dst) {
    float* red = reinterpret_cast<float*>(smem);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    __syncthreads();   // nobody uses the LDS for anything else any more
#pragma unroll
    for (int round = 0; round < kWavesPerWG / kCopies; ++round) {
      if (wave / kCopies == round) put(red + (wave % kCopies) * NE, round != 0);
      __syncthreads();
    }
    for (int i = threadIdx.x; i < NE / 4; i += kThreads) {
      const f32x4* q = reinterpret_cast<const f32x4*>(red) + i;
      constexpr int S = NE / 4;
      f32x4 v;
      if constexpr (kCopies == 4) v = (q[0] + q[2 * S]) + (q[S] + q[3 * S]);
      else v = q[0] + q[S];
      reinterpret_cast<f32x4*>(dst)[i] = v;
    }
  }
};

// Ring depths: two workgroups of four waves per CU (160 KB of LDS); at 56 and 64 channels two slots of two tensors.
template <int D, int NT> constexpr int ring32_depth() { return NT == 2 && D > 48 ? 2 : 3; }
template <int D, int NT> using Ring32For = Ring32<D, NT, ring32_depth<D, NT>()>;

constexpr int max32(int a, int b) { return a > b ? a : b; }
template <int D, int NT> constexpr int consume32_lds_bytes() {
  using RG = Ring32For<D, NT>;
  return max32(RG::kRingBytes, RG::kStageOffset + RG::kStageBytes);
}
// bwd_qs32 at 56 and 64 channels: 280-300 registers, so one workgroup per CU and the deeper ring
template <int D> using RingQs32 = Ring32<D, 2, 3>;
template <int D> constexpr int qs32_lds_bytes() {
  using RG = RingQs32<D>;
  return max32(max32(RG::kRingBytes, RG::kStageOffset + RG::kStageBytes), Sum32<D>::kBytes);
}

// grid = (splits, B*H), block = 256, dynamic LDS Sum32<D>::kBytes.  partials: [B*H][splits][D*D + D].
// A tile is Reduce32s<D>::kTokens tokens.
template <int D> struct Reduce32s {
  static constexpr int kCPL = D == 24 ? 3 : (D + 15) / 16;   // channels per lane
  typedef float Row __attribute__((ext_vector_type(kCPL == 3 ? 3 : (kCPL == 1 ? 2 : kCPL)), aligned(4)));
  // d = 8 and 24: eight lanes cover a row, and the sixteen rows of a block are those of two groups of 32 tokens (their
  // sums are the block's two diagonal quarters), so that no lane loads in vain
  static constexpr int kGroups = D == 8 || D == 24 ? 2 : 1;
  static constexpr int kTokens = kTile * kGroups;   // tokens per tile
  // first channel of lane m (the lanes past the row repeat its end)
  static LF_DEV int first(int m) {
    if constexpr (kGroups == 2) return kCPL * (m & 7);
    else return kCPL * m < D - kCPL ? kCPL * m : D - kCPL;
  }
};
template <int D, int FM>
__global__ void __launch_bounds__(kThreads, 2)
state_reduce32s(const float* __restrict__ K, const float* __restrict__ V, long long batch, long long head, int row,
                unsigned heads, int tiles_per_block, long long N, float* __restrict__ partials) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using C = Reduce32s<D>;
  constexpr int CPL = C::kCPL, TOK = C::kTokens;
  const int lane = threadIdx.x & 63, m = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long bh = blockIdx.y;
  const int c0 = C::first(m);
  // the lane's eight tokens t0 + kStep j: one load instruction reads kStep neighbouring rows (of eight
  // rows apart every 128-byte line would be fetched by several instructions: 8 x 40 at 2^20 tokens 609 us, d = 8 173 us)
  constexpr int kStep = 4 * C::kGroups;
  const int t0 = kq + (C::kGroups == 2 ? (m >> 3) * 4 : 0);
  const long long off = HeadAt(blockIdx.y, heads).slice(batch, head) * 4;
  const float *Kh = K + off, *Vh = V + off;
  const int rs = row * 4;
  TileIter it(blockIdx.x, gridDim.x, wave, tiles_per_block, (N + TOK - 1) / TOK);

  float kr[8][CPL], vr[8][CPL];   // this lane's channels of its eight tokens: the next tile's
  auto load_row = [](const float* p, float (&x)[CPL]) {
    if constexpr (CPL == 1) {
      x[0] = __builtin_nontemporal_load(p);
    } else {
      const typename C::Row w = __builtin_nontemporal_load(reinterpret_cast<const typename C::Row*>(p));
#pragma unroll
      for (int i = 0; i < CPL; ++i) x[i] = w[i];
    }
  };
  auto lim_of = [&](long long tile) {
    const long long rem = N - tile * TOK;
    return rem < TOK ? (int)rem : TOK;
  };
  // (an offset is 63 rows of floats at most: unsigned, since it may exceed an int)
  static_assert((TOK - 1) * 4 * (kMaxRowStride - 1) + D <= 0xffffffffLL, "row offsets of a tile fit 32 bits");
  auto issue_loads = [&](long long tile, int lim) {   // rows past N: the tile's first row instead
    const float* kp = Kh + tile * TOK * rs;
    const float* vp = Vh + tile * TOK * rs;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const unsigned r = t0 + kStep * j < lim ? t0 + kStep * j : 0;
      load_row(kp + (r * (unsigned)rs + c0), kr[j]);
      load_row(vp + (r * (unsigned)rs + c0), vr[j]);
    }
  };

  f32x4 acc[CPL][CPL];
  float z[CPL];
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    z[i] = 0.0f;
#pragma unroll
    for (int j = 0; j < CPL; ++j) acc[i][j] = f32x4{0, 0, 0, 0};
  }
  auto test = [&](const float (&k)[8][CPL], const float (&v)[8][CPL]) __attribute__((always_inline)) {
    Low vs;
    PhiLow<FM> ks;
#pragma unroll
    for (int j = 0; j < 8; j += 2)
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        ks.add(k[j][i], k[j + 1][i]);
        vs.add(v[j][i], v[j + 1][i]);
      }
    return ks.passes() && vs.passes();
  };
  // the tile that has been loaded.  True: it passes the test, though what stands for rows past the end would not.
  auto take = [&](float (&k)[8][CPL], float (&v)[8][CPL], int lim) {
    bool passes = false;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        k[j][i] = kr[j][i];
        v[j][i] = vr[j][i];
      }
    if (lim < TOK) {   // rows past the end (the tile's first so far) add nothing
      passes = test(k, v);
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
          const bool ok = t0 + kStep * j < lim;
          k[j][i] = ok ? k[j][i] : (FM == kPhiIdentity ? 0.0f : -1.0e4f);   // phi = 0
          v[j][i] = ok ? v[j][i] : 0.0f;
        }
    }
    return passes;
  };
  auto phi_of = [&](int i, const float (&k)[8][CPL], float (&p)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = phi32<FM>(k[j][i]);
    z[i] += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
  };
  const TileIter first = it;
  int lim = 0;
  if (it.valid()) {
    lim = lim_of(it.t);
    issue_loads(it.t, lim);
  }
  Pace pace((N + TOK - 1) / TOK, (long long)gridDim.x * kWavesPerWG, paced<D>(N));
  while (it.valid()) {
    float k[8][CPL], v[8][CPL];
    const bool passes = take(k, v, lim);
    const TileIter cur = it;
    it.next();
    if (it.valid()) {
      lim = lim_of(it.t);
      issue_loads(it.t, lim);
    }
    if (__builtin_expect(!(test(k, v) || passes), 0)) {
      bool exact = true;
#pragma unroll
      for (int i = 0; i < CPL; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          k[j][i] = unmasked<FM>(k[j][i]);
          exact &= splits_exactly(phi32<FM>(rarely(k[j][i]))) & splits_exactly(rarely(v[j][i]));
        }
      if (!all_lanes(exact)) {
        it = cur;
        break;
      }
    }
    Split8 b[CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j)
      b[j] = join(split3(f32x4{v[0][j], v[1][j], v[2][j], v[3][j]}), split3(f32x4{v[4][j], v[5][j], v[6][j], v[7][j]}));
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      float p[8];
      phi_of(i, k, p);
      const Split8 a = join(split3(f32x4{p[0], p[1], p[2], p[3]}), split3(f32x4{p[4], p[5], p[6], p[7]}));
#pragma unroll
      for (int j = 0; j < CPL; ++j) acc[i][j] = mfma_split(a, b[j], acc[i][j]);
    }
    pace.tile_done();
  }
  {   // a NaN among a row's or a column's terms is in every sum of that row or column: all tiles again
    bool sound = true;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      sound &= acc[0][i][0] == acc[0][i][0];
#pragma unroll
      for (int r = 0; r < 4; ++r) sound &= acc[i][0][r] == acc[i][0][r];
    }
    if (__builtin_expect(!all_lanes(sound), 0)) {
      it = first;
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        z[i] = 0.0f;
#pragma unroll
        for (int j = 0; j < CPL; ++j) acc[i][j] = f32x4{0, 0, 0, 0};
      }
    }
  }
  // from the first tile on that three terms do not hold: the fp32 instruction (a loop of its own for the registers' sake)
  while (it.valid()) {
    lim = lim_of(it.t);
    issue_loads(it.t, lim);
    float k[8][CPL], v[8][CPL];
    (void)take(k, v, lim);
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
#pragma unroll
      for (int j = 0; j < 8; ++j) k[j][i] = unmasked<FM>(k[j][i]);
      float p[8];
      phi_of(i, k, p);
#pragma unroll
      for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int j = 0; j < CPL; ++j) acc[i][j] = mfma_f32(p[t], v[t][j], acc[i][j]);
    }
    it.next();
  }
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    z[i] += __shfl_xor(z[i], 16);
    z[i] += __shfl_xor(z[i], 32);
  }
  if constexpr (C::kGroups == 2) {   // the second group's sums: row + 8, column + 8
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
#pragma unroll
      for (int j = 0; j < CPL; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] += __shfl_xor(acc[i][j][r], 40);
      z[i] += __shfl_xor(z[i], 8);
    }
  }
  Sum32<D>::write(smem, [&](float* st, bool add) {
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int col = c0 + j;
      if (col / CPL != m) continue;   // a repeated channel
#pragma unroll
      for (int i = 0; i < CPL; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = C::first(4 * kq + r) + i;
          if (row / CPL == 4 * kq + r) {
            float* p = st + row * D + col;
            *p = add ? *p + acc[i][j][r] : acc[i][j][r];
          }
        }
      if (kq == 0) {
        float* p = st + D * D + col;
        *p = add ? *p + z[j] : z[j];
      }
    }
  }, partials + (bh * gridDim.x + blockIdx.x) * (long long)Sum32<D>::NE);
}

// out_i = phi(q_i) S / (phi(q_i).z + eps).  grid = (wgs, B*H), block = 256, dynamic LDS consume32_lds_bytes<D, 1>().
// state: [B*H][parts][D*D + D]; with `keep` the summed state goes there too ([B*H][D*D + D]).
template <int D, int FM, bool NORM>
__global__ void __launch_bounds__(kThreads, 2)
apply32s(const f32x4* __restrict__ Q, long long qbatch, long long qhead, int qrow, unsigned heads, int tiles_per_block,
         long long N, const float* __restrict__ state, int parts, float eps, float* __restrict__ keep, f32x4* __restrict__ O,
         long long obatch, long long ohead, int orow) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using RG = Ring32For<D, 1>;
  constexpr int MT = RG::MT, R = RG::R, NE = RG::NE;
  const long long bh = blockIdx.y;
  const HeadAt at(blockIdx.y, heads);
  const f32x4* const src[1] = {Q + at.slice(qbatch, qhead)};
  const int rs[1] = {qrow};
  RG rg(src, rs, N, tiles_per_block, blockIdx.x, gridDim.x, smem);
  f32x4* Oh = O + at.slice(obatch, ohead);
  f32x4 whole[RG::kPer];
  if constexpr (!RG::kLate) RG::load_state(state + bh * parts * (long long)NE, parts, whole);
  rg.prefetch();
  if constexpr (RG::kLate) RG::load_state(state + bh * parts * (long long)NE, parts, whole);
  bool raw;
  const float* st = rg.stage_state(whole, keep && blockIdx.x == 0 ? keep + bh * NE : nullptr, raw);
  Split8 A[MT][RG::KS];
  rg.template build_A<true>(st, raw, A);
  f32x4 z[MT];
  if constexpr (NORM) rg.load_vec(st, z);
  __syncthreads();   // the staged state is dead
  Pace pace((N + kTile32 - 1) / kTile32, (long long)gridDim.x * kWavesPerWG, paced<D>(N));
  int slot = 0, iter = 0;
  while (rg.it.valid()) {
    const long long tile = rg.it.t;
    int aslot = slot + (R - 1);
    if (aslot >= R) aslot -= R;
    const bool more = rg.ahead.valid();
    if (more) rg.issue_copy(rg.ahead.t, aslot);
    rg.template wait_tile<RG::NL>(iter, more);
    iter = iter < 2 ? iter + 1 : 2;
    f32x4 r[MT], acc[MT];
    rg.read_rows(slot, 0, r);
    float den = 0.0f;
    auto form = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int T = 0; T < MT; ++T)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          r[T][e] = phi32<FM>(r[T][e]);
          if constexpr (NORM) den = __builtin_fmaf(r[T][e], z[T][e], den);
        }
    };
    bool split = !raw && RG::template seen<PhiLow<FM>>(r).passes();
    if (split) {   // (one straight piece: phi beside the matrix steps)
      form();
      rg.products(A, r, acc);
      split = all_lanes(RG::sound(acc));
    }
    if (__builtin_expect(!split, 0)) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (read again, not kept)
      rg.read_rows(slot, 0, r);
      RG::template unmask<FM>(r);
      den = 0.0f;
      form();
      rg.products_any(A, raw, r, acc);
    }
    if constexpr (NORM) {
      const float scale = 1.0f / (RG::token_sum(den) + eps);
#pragma unroll
      for (int T = 0; T < MT; ++T) acc[T] *= scale;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    rg.write_rows(slot, 0, acc);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    rg.store_tile(tile, slot, 0, Oh, orow);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    pace.tile_done();
    rg.it.next();
    rg.ahead.next();
    slot = slot + 1 == R ? 0 : slot + 1;
  }
}

// dQ, and dS, dz as partials.  grid = (wgs, B*H), block = 256, dynamic LDS qs32_lds_bytes<D>().  state, parts, keep: as
// apply32s; partials: [B*H][gridDim.x][D*D + D], another buffer than `state`.
template <int D, int FM, bool NORM>
__global__ void __launch_bounds__(kThreads, D > 48 ? 1 : 2)
bwd_qs32(const f32x4* __restrict__ Q, Layout lq, const f32x4* __restrict__ G, Layout lg, f32x4* __restrict__ dQ,
         Layout ldq, const float* __restrict__ state, int parts, float* __restrict__ partials, float eps, long long N,
         int tiles_per_block) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using RG = RingQs32<D>;
  constexpr int MT = RG::MT, R = RG::R, NE = RG::NE;
  const long long bh = blockIdx.y;
  const f32x4* const src[2] = {Q + lq.slice(bh), G + lg.slice(bh)};
  const int rs[2] = {lq.row, lg.row};
  RG rg(src, rs, N, tiles_per_block, blockIdx.x, gridDim.x, smem);
  f32x4* dQh = dQ + ldq.slice(bh);
  f32x4 whole[RG::kPer];
  if constexpr (!RG::kLate) RG::load_state(state + bh * parts * (long long)NE, parts, whole);
  rg.prefetch();
  if constexpr (RG::kLate) RG::load_state(state + bh * parts * (long long)NE, parts, whole);
  bool raw;
  const float* st = rg.stage_state(whole, nullptr, raw);
  Split8 A[MT][RG::KS];
  rg.template build_A<false>(st, raw, A);       // u = S g
  f32x4 z[MT];
  if constexpr (NORM) rg.load_vec(st, z);
  __syncthreads();                          // the staged state is dead
  f32x4 acc[MT][MT], dz[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    dz[i] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[i][j] = f32x4{0, 0, 0, 0};
  }
  Pace pace((N + kTile32 - 1) / kTile32, (long long)gridDim.x * kWavesPerWG, paced<D>(N));
  int slot = 0, iter = 0;
  while (rg.it.valid()) {
    const long long tile = rg.it.t;
    const int lim = rg.lim_of(tile);
    int aslot = slot + (R - 1);
    if (aslot >= R) aslot -= R;
    const bool more = rg.ahead.valid();
    if (more) rg.issue_copy(rg.ahead.t, aslot);
    rg.template wait_tile<RG::NL>(iter, more);
    iter = iter < 2 ? iter + 1 : 2;
    f32x4 x[MT], g[MT], u[MT];
    rg.read_rows(slot, 1, g);
    rg.read_rows(slot, 0, x);
    const auto gs = RG::template seen<Both<Low>>(g);
    f32x4 r[MT];
    float den = 0.0f, ru = 0.0f;
    auto form = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int T = 0; T < MT; ++T)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          r[T][e] = phi32<FM>(x[T][e]);
          if constexpr (NORM) {
            den = __builtin_fmaf(r[T][e], z[T][e], den);   // z and u are zero past d
            ru = __builtin_fmaf(r[T][e], u[T][e], ru);
          }
          if constexpr (FM == kPhiEluPlusOne) x[T][e] = x[T][e] > 0.0f ? 1.0f : r[T][e];     // phi'(q)
          else if constexpr (FM == kPhiRelu) x[T][e] = x[T][e] > 0.0f ? 1.0f : 0.0f;
          else x[T][e] = 1.0f;
        }
    };
    // (in three pieces, unlike the other two kernels: in one it takes some ten registers more than there are)
    if (__builtin_expect(!raw && gs.passes(), 1)) rg.products(A, g, u);
    else rg.products_any(A, raw, g, u);
    const bool pass = RG::template seen<Both<PhiLow<FM>>>(x).passes();
    if (__builtin_expect(!pass, 0)) RG::template unmask<FM>(x);
    form();
    float invden = 1.0f, go = 0.0f;
    if constexpr (NORM) {
      invden = 1.0f / (RG::token_sum(den) + eps);
      go = RG::token_sum(ru) * invden;
    }
    const bool on = rg.m < lim;             // rows past the end add nothing
    const float e_i = on ? -go * invden : 0.0f;
#pragma unroll
    for (int T = 0; T < MT; ++T)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (NORM) u[T][e] = (u[T][e] - go * z[T][e]) * invden;
        x[T][e] *= u[T][e];                                            // dq
        r[T][e] = on ? r[T][e] : 0.0f;
        g[T][e] = on ? g[T][e] * invden : 0.0f;
        if constexpr (NORM) dz[T][e] = __builtin_fmaf(r[T][e], e_i, dz[T][e]);
      }
    // (g / den lies within what its tile's extremes divided by den span, so those need not be sought again)
    const float by = fabsf(invden);
    const bool split = (pass && all_lanes(!on || (gs.lo * by >= kSplitLow && gs.hi * by < kSplitHigh))) ||
                       all_lanes(RG::exact(r) & RG::exact(g));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    rg.write_rows(slot, 0, r);
    rg.write_rows(slot, 1, g);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    float pc[4][MT], gc[4][MT];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        pc[k][i] = rg.read_col(slot, 0, k, i);
        gc[k][i] = rg.read_col(slot, 1, k, i);
      }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    rg.write_rows(slot, 0, x);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    rg.store_tile(tile, slot, 0, dQh, ldq.row);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (__builtin_expect(split, 1)) {
      Split4 b[MT];
#pragma unroll
      for (int j = 0; j < MT; ++j) b[j] = split3(f32x4{gc[0][j], gc[1][j], gc[2][j], gc[3][j]});
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const Split4 a = split3(f32x4{pc[0][i], pc[1][i], pc[2][i], pc[3][i]});
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[i][j] = mfma_split(a, b[j], acc[i][j]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
          acc[i][j] = mfma_f32(f32x4{pc[0][i], pc[1][i], pc[2][i], pc[3][i]}, f32x4{gc[0][j], gc[1][j], gc[2][j], gc[3][j]},
                               acc[i][j]);
    }
    pace.tile_done();
    rg.it.next();
    rg.ahead.next();
    slot = slot + 1 == R ? 0 : slot + 1;
  }
#pragma unroll
  for (int T = 0; T < MT; ++T)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) dz[T][e] += __shfl_xor(dz[T][e], o);   // over the sixteen tokens
  Sum32<D>::write(smem, [&](float* sd, bool add) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * i + 4 * rg.kq + r;
        if (RG::kWhole || 16 * i + 15 < D || row < D) {
#pragma unroll
          for (int j = 0; j < MT; ++j) {
            const int col = 16 * j + rg.m;
            if (RG::kWhole || 16 * j + 15 < D || col < D) {
              float* p = sd + row * D + col;
              *p = add ? *p + acc[i][j][r] : acc[i][j][r];
            }
          }
        }
      }
#pragma unroll
    for (int T = 0; T < MT; ++T)
      if (rg.m == 0 && rg.has(T)) {
        f32x4* p = reinterpret_cast<f32x4*>(sd + D * D + 16 * T + 4 * rg.kq);
        *p = add ? *p + dz[T] : dz[T];
      }
  }, partials + (bh * gridDim.x + blockIdx.x) * (long long)NE);
}

// dK, dV.  Both orientations of dS as operands: one workgroup per CU from 56 channels on.  grid = (wgs, B*H), block = 256, dynamic LDS consume32_lds_bytes<D, 2>().  state: dS, dz as `parts` partials.
template <int D, int FM>
__global__ void __launch_bounds__(kThreads, D > 48 ? 1 : 2)
bwd_kv32(const f32x4* __restrict__ K, const f32x4* __restrict__ V, Layout lkv, f32x4* __restrict__ dK,
         f32x4* __restrict__ dV, Layout ldkv, const float* __restrict__ state, int parts, long long N,
         int tiles_per_block) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using RG = Ring32For<D, 2>;
  constexpr int MT = RG::MT, R = RG::R, NE = RG::NE;
  const long long bh = blockIdx.y;
  const f32x4* const src[2] = {K + lkv.slice(bh), V + lkv.slice(bh)};
  const int rs[2] = {lkv.row, lkv.row};
  RG rg(src, rs, N, tiles_per_block, blockIdx.x, gridDim.x, smem);
  f32x4 *dKh = dK + ldkv.slice(bh), *dVh = dV + ldkv.slice(bh);
  f32x4 whole[RG::kPer];
  if constexpr (!RG::kLate) RG::load_state(state + bh * parts * (long long)NE, parts, whole);
  rg.prefetch();
  if constexpr (RG::kLate) RG::load_state(state + bh * parts * (long long)NE, parts, whole);
  bool raw;
  const float* st = rg.stage_state(whole, nullptr, raw);
  Split8 A[MT][RG::KS], At[MT][RG::KS];
  rg.template build_A<false>(st, raw, A);       // dS v
  rg.template build_A<true>(st, raw, At);       // dS^T p
  f32x4 dz[MT];
  rg.load_vec(st, dz);
  __syncthreads();                          // the staged state is dead
  Pace pace((N + kTile32 - 1) / kTile32, (long long)gridDim.x * kWavesPerWG, paced<D>(N));
  int slot = 0, iter = 0;
  while (rg.it.valid()) {
    const long long tile = rg.it.t;
    int aslot = slot + (R - 1);
    if (aslot >= R) aslot -= R;
    const bool more = rg.ahead.valid();
    if (more) rg.issue_copy(rg.ahead.t, aslot);
    rg.template wait_tile<2 * RG::NL>(iter, more);
    iter = iter < 2 ? iter + 1 : 2;
    f32x4 k[MT], v[MT], t[MT], dv[MT], p[MT];
    rg.read_rows(slot, 1, v);
    rg.read_rows(slot, 0, k);
    auto form = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int T = 0; T < MT; ++T)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p[T][e] = phi32<FM>(k[T][e]);
          if constexpr (FM == kPhiEluPlusOne) k[T][e] = k[T][e] > 0.0f ? 1.0f : p[T][e];     // phi'(k)
          else if constexpr (FM == kPhiRelu) k[T][e] = k[T][e] > 0.0f ? 1.0f : 0.0f;
          else k[T][e] = 1.0f;
        }
    };
    bool split = !raw && RG::template seen<Low>(v).passes() && RG::template seen<PhiLow<FM>>(k).passes();
    if (split) {
      rg.products(A, v, t);
      form();
      rg.products(At, p, dv);
      split = all_lanes(RG::sound(t) && RG::sound(dv));
    }
    if (__builtin_expect(!split, 0)) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (read again, not kept)
      rg.read_rows(slot, 1, v);
      rg.read_rows(slot, 0, k);
      RG::template unmask<FM>(k);
      rg.products_any(A, raw, v, t);
      form();
      rg.products_any(At, raw, p, dv);
    }
#pragma unroll
    for (int T = 0; T < MT; ++T) k[T] *= t[T] + dz[T];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    rg.write_rows(slot, 0, k);
    rg.write_rows(slot, 1, dv);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    rg.store_tile(tile, slot, 0, dKh, ldkv.row);
    rg.store_tile(tile, slot, 1, dVh, ldkv.row);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    pace.tile_done();
    rg.it.next();
    rg.ahead.next();
    slot = slot + 1 == R ? 0 : slot + 1;
  }
}

}  // namespace lf
