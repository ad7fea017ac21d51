// Shared device-side helpers for the gfx950 LinFusion kernels: vector types, 16-bit
// conversions, the feature map phi (Sec. 2.3: non-negative activation on Q and K), and the
// shape constants that the state-reduction, combine and apply kernels must agree on.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lf {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kPhiEluPlusOne = 0;
constexpr int kPhiRelu = 1;
constexpr int kPhiIdentity = 2;

struct F16 {};   // tag: IEEE binary16 storage
struct BF16 {};  // tag: bfloat16 storage

#define LF_DEV __device__ __forceinline__
#define LF_LDS __attribute__((address_space(3)))

// ---- feature map -------------------------------------------------------------------------
// elu(x)+1 = x+1 for x > 0, exp(x) otherwise.  exp(x) = 2^(x*log2 e) on the hardware exp2
// unit; `Precise` adds the rounding error of the product back as a first-order correction
// (used on the fp32 path, whose tolerance is 1e-5).  `Masked`: so that keys masked with the type's lowest value or
// -infinity give 0; without it a Precise x must not lie below about -1e4 (the correction would become infinite, and 0
// times it NaN).
template <int FM, bool Precise = false, bool Masked = Precise>
LF_DEV float phi(float x) {
  if constexpr (FM == kPhiEluPlusOne) {
    constexpr float kLog2e = 1.44269504088896340736f;
    if constexpr (Precise) {
      // from -200 on, where exp(x) is 0 already; the branch above 0 does not use it
      const float y = Masked ? __builtin_amdgcn_fmed3f(x, -200.0f, 0.0f) : x;
      const float t = y * kLog2e;
      const float e = __builtin_amdgcn_exp2f(t);
      // t_err = y*log2e - t (exactly, via fma) plus the part of log2e that fp32 drops.
      const float terr = __builtin_fmaf(y, kLog2e, -t) + y * 1.92596299112661746e-8f;
      const float ex = __builtin_fmaf(e, terr * 0.69314718055994530942f, e);
      if constexpr (Masked) return x <= 0.0f ? ex : x + 1.0f;   // (a NaN stays one)
      return x > 0.0f ? x + 1.0f : ex;
    }
    const float e = __builtin_amdgcn_exp2f(x * kLog2e);
    return x > 0.0f ? x + 1.0f : e;
  } else if constexpr (FM == kPhiRelu) {
    return x > 0.0f ? x : 0.0f;   // NaN maps to 0 like fmax(x, 0)
  } else {
    return x;
  }
}

// phi(x) to the same bits with elu(x) + 1 chosen by the sign bit (both branches give 1 at +-0 and keep a NaN one): two vector
// instructions that write no condition code, where a compare and a select of its result have a wait between them.  For kernels
// bound by their vector work that do not need the compare again (the gradient kernels take phi'(x) from it, and they are short of
// registers: with this in the dQ kernel on row pieces 29 registers spilled, 43 -> 62 us).  Kernel times in a trace, both sides on one box,
// with the remainders of pack2_split: bf16 12 x 8 x 4096 x 40 token-major apply16_rows 23.0 -> 21.9 us, state_reduce16_rows 20.3 -> 19.9;
// 2 x 10 x 16384 x 64 state_reduce16_mlph 35.5 -> 33.3, fused16 50.4 -> 49.3.  Calls gain less (2 x 8 x 36503 x 40 51.1 -> 50.3, the
// first and the last of those above nothing that can be told from noise).
template <int FM>
LF_DEV float phi_by_sign(float x) {
  if constexpr (FM == kPhiEluPlusOne) {
    constexpr float kLog2e = 1.44269504088896340736f;
    uint32_t neg;
    asm("v_ashrrev_i32 %0, 31, %1" : "=v"(neg) : "v"(x));   // (left to itself the compiler turns the mask back into a compare)
    const uint32_t e = __builtin_bit_cast(uint32_t, __builtin_amdgcn_exp2f(x * kLog2e)), lin = __builtin_bit_cast(uint32_t, x + 1.0f);
    return __builtin_bit_cast(float, lin ^ ((lin ^ e) & neg));   // (one instruction; as (e & neg) | (lin & ~neg) four)
  } else {
    return phi<FM>(x);
  }
}

// elu(x)+1 of a value whose exponential branch is evaluated as exp(x + c / log2 e), i.e. scaled by 2^c: used
// where a whole row (or a whole stream) of inputs is negative and so small that exp(x) itself would leave the
// normal range of fp16; the caller divides the factor out again (or it cancels in a ratio).  c = 0: phi itself.
template <int FM>
LF_DEV float phi_scaled(float x, float c) {
  if constexpr (FM == kPhiEluPlusOne) {
    constexpr float kLog2e = 1.44269504088896340736f;
    const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(x, kLog2e, c));
    return x > 0.0f ? x + 1.0f : e;
  } else {
    return phi<FM>(x);
  }
}

// ---- 16-bit storage <-> fp32 ----------------------------------------------------------------
template <typename T> LF_DEV void unpack2(uint32_t w, float& lo, float& hi);
template <> LF_DEV void unpack2<F16>(uint32_t w, float& lo, float& hi) {
  f16x2 h = __builtin_bit_cast(f16x2, w);
  lo = (float)h[0];
  hi = (float)h[1];
}
template <> LF_DEV void unpack2<BF16>(uint32_t w, float& lo, float& hi) {
  lo = __builtin_bit_cast(float, w << 16);
  hi = __builtin_bit_cast(float, w & 0xffff0000u);
}

// round-to-nearest-even pack of two floats into one 32-bit word (element 0 in the low half)
template <typename T> LF_DEV uint32_t pack2(float lo, float hi);
template <> LF_DEV uint32_t pack2<F16>(float lo, float hi) {
  f16x2 h = {(_Float16)lo, (_Float16)hi};
  return __builtin_bit_cast(uint32_t, h);
}
template <> LF_DEV uint32_t pack2<BF16>(float lo, float hi) {
  bf16x2 h = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, h);
}

// phi of a stored pair, rounded to the storage type again: the word a matrix-core operand takes; the _scaled form
// is phi_scaled on both halves.  fp16 elu(x)+1 goes a shorter way to the same bits: x + 1 in packed fp16 arithmetic
// (the exact sum rounded once, as the fp32 sum rounded to fp16 is: it is exact in fp32 wherever it is not 1 anyway),
// the exponential through fp32 as in phi(), and the choice between them by the sign bit (both give 1 at +-0, and
// callers scale by 2^c only rows or streams without a non-negative element; a NaN stays a NaN on either side) --
// 6 + 2 instructions per pair instead of 11 + 2.
template <typename T, int FM> struct PhiPack2 {
  static LF_DEV uint32_t run(uint32_t w) {
    float x0, x1;
    unpack2<T>(w, x0, x1);
    return pack2<T>(phi<FM>(x0), phi<FM>(x1));
  }
  static LF_DEV uint32_t run_scaled(uint32_t w, float c) {
    float x0, x1;
    unpack2<T>(w, x0, x1);
    return pack2<T>(phi_scaled<FM>(x0, c), phi_scaled<FM>(x1, c));
  }
};
template <> struct PhiPack2<F16, kPhiEluPlusOne> {
  static LF_DEV uint32_t run_scaled(uint32_t w, float c) {
    const float kLog2e = 1.44269504088896340736f;
    const f16x2 x = __builtin_bit_cast(f16x2, w);
    const f16x2 one = {(_Float16)1.0f, (_Float16)1.0f};
    const uint32_t lin = __builtin_bit_cast(uint32_t, x + one);
    // (written out: left to itself the compiler turns the mask into two compares and selects, and converts before
    //  it multiplies)  t = fma(half, log2 e, c) in one rounding, as the fp32 fma of the converted half is
    float t0, t1;
    uint32_t neg;
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(t0) : "v"(w), "v"(kLog2e), "v"(c));
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(t1) : "v"(w), "v"(kLog2e), "v"(c));
    // 0xffff in every negative half (op_sel_hi: the upper half takes its shift count from the constant's lower half too)
    asm("v_pk_ashrrev_i16 %0, 15, %1 op_sel_hi:[0,1]" : "=v"(neg) : "v"(w));
    const uint32_t e = pack2<F16>(__builtin_amdgcn_exp2f(t0), __builtin_amdgcn_exp2f(t1));
    return (e & neg) | (lin & ~neg);
  }
  static LF_DEV uint32_t run(uint32_t w) { return run_scaled(w, 0.0f); }
};
template <typename T, int FM> LF_DEV uint32_t phi_pack2(uint32_t w) { return PhiPack2<T, FM>::run(w); }
template <typename T, int FM> LF_DEV uint32_t phi_pack2_scaled(uint32_t w, float c) { return PhiPack2<T, FM>::run_scaled(w, c); }

// value of a packed pair after rounding, back in fp32 (for hi/lo operand splitting).  ONCE: the remainders come from the packed
// word; left to itself the compiler rounds the lower half a second time for its remainder, off the chain through the word.  The same bits
// either way; us per call, ONCE false / true: bf16 forward 2 x 8 x 36503 x 40 token-major 51.4 / 50.2, forward and backward 4 x 8 x 4096
// x 64 85.1 / 83.7, 12 x 8 x 2048 x 24 48.9 / 48.2, 4 x 8 x 8192 x 40 token-major 84.4 / 83.6; but the row-piece MLP-fed forward 2 x 8 x
// 16384 x 40 49.3 / 50.7, 2 x 8 x 4096 x 40 24.8 / 25.1, and forward 2 x 8 x 8000 x 128 54.3 / 55.3 (96 and 160 channels the same).
template <typename T, bool ONCE = true> LF_DEV void pack2_split(float lo, float hi, uint32_t& w_hi, uint32_t& w_lo) {
  w_hi = pack2<T>(lo, hi);
  if constexpr (ONCE) asm("" : "+v"(w_hi));
  float rl, rh;
  unpack2<T>(w_hi, rl, rh);
  w_lo = pack2<T>(lo - rl, hi - rh);
}

// ---- matrix-core wrappers (operands carried as raw 128-bit words) ---------------------------
template <typename T> LF_DEV f32x4 mfma_16x16x32(u32x4 a, u32x4 b, f32x4 c);
template <> LF_DEV f32x4 mfma_16x16x32<F16>(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <> LF_DEV f32x4 mfma_16x16x32<BF16>(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
template <typename T> LF_DEV f32x16 mfma_32x32x16(u32x4 a, u32x4 b, f32x16 c);
template <> LF_DEV f32x16 mfma_32x32x16<F16>(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <> LF_DEV f32x16 mfma_32x32x16<BF16>(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// LDS transposing read: the 16 lanes of a group each name 8 bytes (4 x 16-bit, lane i = row
// i/4, columns 4*(i%4)..+3 of a 4 x 16 block); afterwards lane j of the group holds column j
// of the 4 rows.  Two of them give the 8 contraction-index elements a 16x16x32 operand needs.
LF_DEV u32x2 lds_read_tr16(const uint16_t* p) {
  s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LF_LDS s16x4*)(p));
  return __builtin_bit_cast(u32x2, r);
}

// Workgroup barrier that orders LDS traffic only: the wave's LDS operations are complete before it arrives,
// while its outstanding global loads, stores and LDS copies stay in flight (before __syncthreads() the
// compiler drains every memory counter, which would expose the latency of loads issued just before it).
LF_DEV void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Zeros in `elems` 16-bit elements of LDS, by thread t of nt: 16 bytes per store.  (Two at a time, with a division per element
// to find the ones column, the fill of state_reduce16_rows took 7 of that kernel's 26 us at 12 x 8 x 4096 x 40.)
LF_DEV void lds_zero(uint16_t* p, int elems, int t, int nt) {
  for (int i = t; i < elems / 8; i += nt) reinterpret_cast<u32x4*>(p)[i] = u32x4{0, 0, 0, 0};
}

// streaming 128-bit global load / store (non-temporal: the tensors are touched once)
LF_DEV u32x4 ld_stream(const u32x4* p) { return __builtin_nontemporal_load(p); }
LF_DEV void st_stream(u32x4* p, u32x4 v) { __builtin_nontemporal_store(v, p); }
LF_DEV void st_stream(u32x2* p, u32x2 v) { __builtin_nontemporal_store(v, p); }

// Loads / stores of the small fp32 partial states and states that other workgroups (on other XCDs,
// each with its own L2) consume inside the same launch: device-scope relaxed atomics, which go
// through to the device-coherent level instead of staying in the issuing XCD's L2.
LF_DEV void st_agent(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
LF_DEV float ld_agent(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// ---- shape constants of the 16-bit path ---------------------------------------------------
// State reduction tiles the d x d state in 16 x 16 blocks; apply tiles the output in 32-row
// blocks with the two normalizer rows (z hi, z lo) appended after each half of the channels.
template <int D> struct Shape16 {
  static_assert(D % 8 == 0 && D >= 8 && D <= 80, "head width must be a multiple of 8 up to 80");
  static constexpr int kChunksPerRow = D / 8;          // 16-byte chunks per token row
  static constexpr int kMT = (D + 15) / 16;            // 16-wide tiles across d
  static constexpr int kDP = kMT * 16;
  static constexpr bool kSpareCol = (D % 16) != 0;     // a free padded column carries the ones
  // apply: k-steps of 16 channels (lanes 0-31 supply the first 8, lanes 32-63 the second 8)
  static constexpr int kKS = (kChunksPerRow + 1) / 2;
  static constexpr int kHalf = D / 2;                  // output channels held by one half-wave
  static constexpr int kMT2 = (kHalf + 2 + 15) / 16;   // 32-row output tiles incl. normalizer rows
};

// ---- where a (batch, head) slice of a tensor starts and how far apart its token rows are ------
// All in units of one vector access (16 bytes): [B, H, N, d] contiguous has row = d * s / 16,
// head = N * row, batch = H * head; the token-major [B, N, H * d] layout of the UNet has
// row = H * d * s / 16, head = d * s / 16, batch = N * row.  Inside a row the d channels are contiguous.
constexpr long long kMaxRowStride = 1LL << 24;   // token strides stay below this: 32 rows in units of 16 bytes fit an int
struct Layout {
  long long batch, head;   // strides between batches / heads
  int row;                 // stride between consecutive tokens of one head
  int H;                   // heads per batch
  // (bh < 2^16 always: divided in 32 bits -- a 64-bit division by a variable is 130 dependent scalar instructions at
  // the start of every workgroup)
  LF_DEV long long slice(long long bh) const {
    const unsigned b = (unsigned)bh / (unsigned)H, h = (unsigned)bh - b * (unsigned)H;
    return (long long)b * batch + (long long)h * head;
  }
};

// The head of grid row y, in kernels whose arguments come first to last in the order in which a workgroup needs them, all as
// plain numbers: the library is built so that the first fourteen 32-bit words of a kernel's arguments are in scalar registers
// when it starts (a structure would end that), and a workgroup's first loads need not wait for the arguments to be read from
// memory (500 calls drawn from 0.25 to 3 MB per tensor, with the words preloaded against the same kernels without: forward calls of
// less than 16 us 2.2 %, in place 2 to 3 %, the state alone 1.2 %, backward 1.5 %).
// `heads`: heads per batch of this launch, and << 16 those of the arrays that are indexed by head (a launch on some of a
// batch's heads is given their first one's addresses).
struct HeadAt {
  unsigned b, h, index;
  LF_DEV HeadAt(unsigned y, unsigned heads) {
    const unsigned per = heads & 0xffffu;
    b = y / per;
    h = y - b * per;
    index = b * (heads >> 16) + h;
  }
  LF_DEV long long slice(long long batch, long long head) const { return (long long)b * batch + (long long)h * head; }
};

// ---- which tiles a wave processes -----------------------------------------------------------
// The tiles of a head are cut into blocks of `blk` consecutive tiles (blk a multiple of the
// waves per workgroup); workgroup g of G takes blocks g, g + G, g + 2G, ... and inside a block its
// waves take tiles round-robin.  blk = ceil(n_tiles / G) gives every workgroup one contiguous
// chunk; a small blk keeps all workgroups of the chip inside one moving window of memory.
// `stride` = 4 with `wave_` = the wave's index is that round-robin; `stride` = 1 with `wave_` = 0 makes a
// wave visit every tile of the workgroup's blocks (used when each wave of a workgroup works on a
// different head over the same token range).
struct TileIter {
  long long t, blk_end, blk_first, n_tiles, step;
  int blk, wave, stride;
  LF_DEV TileIter(int g, int G, int wave_, int blk_, long long n_tiles_, int stride_ = 4)
      : n_tiles(n_tiles_), step((long long)G * blk_), blk(blk_), wave(wave_), stride(stride_) {
    blk_first = (long long)g * blk;
    t = blk_first + wave;
    blk_end = blk_first + blk < n_tiles ? blk_first + blk : n_tiles;
  }
  LF_DEV bool valid() const { return t < n_tiles; }
  LF_DEV void next() {
    t += stride;
    if (t >= blk_end) {
      blk_first += step;
      t = blk_first + wave;
      blk_end = blk_first + blk < n_tiles ? blk_first + blk : n_tiles;
    }
  }
};

// A wave's priority on its SIMD, by how far it has come: 3 for the first half of its tiles, 2 for the next quarter, 1 for
// the next eighth, then 0.  A SIMD serves its waves oldest first, so that of two workgroups on a CU the one that came
// first runs ahead and the other one ends alone, with nobody to hide its waits behind (96 heads of 40 fp32 channels and 4096
// tokens, time in the loop over tiles, first and second workgroup of a CU: state_reduce32s 19 and 27 us, apply32s 26 and 31,
// bwd_qs32 53 and 65, bwd_kv32 40 and 45; with this 22 and 24, 27 and 27, 52 and 55, 42 and 42).
struct Pace {
  int left, next, level;   // tiles left, how many are left when the priority falls next, the priority
  // a wave takes one of `per_round` tiles, n_tiles in all
  LF_DEV Pace(long long n_tiles, long long per_round, bool on) {
    if (!on) {
      left = 0;
      next = 1;   // (never reached)
      level = 0;
      return;
    }
    const unsigned n = n_tiles < 0x7fffffff ? (unsigned)n_tiles : 0x7fffffffu;
    const unsigned r = per_round < 0x7fffffff ? (unsigned)per_round : 0x7fffffffu;
    left = __builtin_amdgcn_readfirstlane((int)((n + r - 1) / r));
    next = left / 2;
    level = 3;
    __builtin_amdgcn_s_setprio(3);
  }
  LF_DEV void tile_done() {
    if (--left == next) {
      next = --level > 0 ? left / 2 : -1;
      if (level == 2) __builtin_amdgcn_s_setprio(2);
      else if (level == 1) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(0);
    }
  }
};

template <typename T> struct NSplit;                 // operand levels needed to hold an fp32 value
template <> struct NSplit<F16> { static constexpr int value = 1; };
template <> struct NSplit<BF16> { static constexpr int value = 2; };

// Bit pattern of the most negative finite value of the storage type.  Rows past the end of a head are given this
// value instead of a per-element mask: elu(x)+1 and relu map it to exactly 0 (exp underflows), so such rows add
// nothing to the state; only the identity map (a test aid) still needs the mask.
template <typename T> struct LowestBits;
template <> struct LowestBits<F16> { static constexpr uint32_t value = 0xFBFFFBFFu; };    // -65504
template <> struct LowestBits<BF16> { static constexpr uint32_t value = 0xFF7FFF7Fu; };   // -3.39e38
template <int FM> constexpr bool kPhiKillsLowest = FM != kPhiIdentity;

template <typename T> struct OneBits;                // bit pattern of 1.0 in the storage type
template <> struct OneBits<F16> { static constexpr uint16_t value = 0x3C00; };
template <> struct OneBits<BF16> { static constexpr uint16_t value = 0x3F80; };

}  // namespace lf
