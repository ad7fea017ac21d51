// Backward pass for fp16 at head widths above 80.  Same derivative as lf_backward16.hpp (of Eq. 5 applied to Prop. 2's
// state; Sec. 2.5 (Training Objectives) differentiates through every module), evaluated in units of a power of two beta
// near sum(z) so that every 16-bit operand is of order one whatever N is:
//   S' = S / beta, z' = z / beta, eps' = eps / beta            (exact)
//   u'_i  = S' g_i
//   den'_i = phi(q_i) . z' + eps',  go_i = phi(q_i) . u'_i / den'_i
//   dq_i = (u'_i - go_i z') / den'_i * phi'(q_i),   gp_i = g_i / den'_i,   dz' = sum_i phi(q_i) (-go_i / den'_i)
//   dS' = sum_i phi(q_i)^T gp_i
//   dS = dS' / beta, dz = dz' / beta                           (exact)
//   dv_j = dS^T phi(k_j),   dk_j = (dS v_j + dz) * phi'(k_j)
// Without the normalizer: den' = 1, go = 0, beta = 1.  Launches:
//   bwdw_pack (S transposed)      the head's state as operands of u' = S' g
//   bwdw_q                        reads q, g: writes dq, gp (fp16, a temporary) and partials of dz'
//   the forward's wide reduction  with q in K's place and gp in V's: dS' partials
//   bwdw_pack (dS, both ways)     summed partials as operands of the next two
//   the forward's wide apply      dv = dS^T phi(k)
//   bwdw_k                        reads k, v: writes dk
// Short streams go another way (lf_bwd_short16.hpp).
// bwdw_q and bwdw_k are apply16_wave with a second tensor in every ring slot: a wave holds the whole operand-ready state of
// its head in registers (200 of the 512 a lone wave per SIMD has, at d = 160) and streams 16-token tiles through a ring of
// its own; a product's results lie channels-of-my-token, so everything elementwise happens where they land, in fp32.
// Before, the pass was composed of the forward's kernels with u', t = dS v and per-token scalars as tensors in memory,
// thirteen launches besides the state: at 12 x 8 x 256 x 160, where launches and passes over the states are what costs,
// the training step took 185 us and took 131 after it (108 with fewer state partials, 100 with the reduction by quarters).
#pragma once
#include "lf_wave16.hpp"
#include "lf_backward16.hpp"

namespace lf {

template <int D> struct BwdWaveShape {
  using Sw = ApplyWaveShape<D>;
  static constexpr int kTok = 16;                              // tokens per tile
  static_assert((kTok * Sw::kCPR) % 64 == 0, "whole 1 KiB deposits per tile");
  static constexpr int kNL = kTok * Sw::kCPR / 64;             // deposits per tensor and tile
  static constexpr int kTensorBytes = kNL * 1024;
  static constexpr int kSlotBytes = 2 * kTensorBytes;
  static constexpr int kRing = 3;
  static constexpr int kWaves = 4;
  static constexpr int kTabOffset = kRing * kWaves * kSlotBytes;   // a vector of the head: D floats
  static constexpr int kLdsBytes = kTabOffset + D * 4;
  static_assert(kLdsBytes <= 160 * 1024, "workgroup LDS limit of the device");
};

// power of two near the sum of the head's normalizer state; every thread of the workgroup calls it (red: one float per wave)
template <int D, int NT>
LF_DEV void bwdw_beta(const float* z, float* red, float& beta, float& inv_beta) {
  float zs = 0.0f;
  for (int i = threadIdx.x; i < D; i += NT) zs += z[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) zs += __shfl_xor(zs, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = zs;
  __syncthreads();
  zs = 0.0f;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) zs += red[w];
  beta = inv_beta = 1.0f;
  if (zs > 0.0f && zs < 3.0e38f) {
    int ex;
    (void)__builtin_frexpf(zs, &ex);
    ex = ex > 100 ? 100 : (ex < -100 ? -100 : ex);
    beta = __builtin_ldexpf(1.0f, ex);
    inv_beta = __builtin_ldexpf(1.0f, -ex);
  }
}

// The sum of the head's `parts` partial states over beta as operands (PackWave's layout, without the normalizer's block).
// grid = (d / 16, heads, n), block = 256: workgroup b handles the 16 output channels of block b; blockIdx.z + first picks
// the orientation: 0 = S[ch][m] (out = S^T x) into `packed`, 1 = S[m][ch] (out = S x) into `packed_t`.
// header: [b] = 1 / (alpha_b beta), [d / 16] = 1 / beta.  z: the head's forward normalizer state (stride D*D + D), or null:
// beta = 1.
template <int D>
__global__ void __launch_bounds__(kThreads)
bwdw_pack(const float* __restrict__ src, int parts, const float* __restrict__ z, unsigned char* __restrict__ packed,
          unsigned char* __restrict__ packed_t, int first) {
  using Sw = ApplyWaveShape<D>;
  constexpr int KS = Sw::kKS, CB = Sw::kCB, NE = D * D + D, PER = D / 16, RS = 17;
  __shared__ float tile[D * RS];       // [ch][m]
  __shared__ float red[2][kThreads / 64];
  const int tid = threadIdx.x, b = blockIdx.x;
  const long long bh = blockIdx.y;
  const bool transposed = (int)blockIdx.z + first == 1;
  const float* st = src + bh * parts * (long long)NE;
  unsigned char* out = (transposed ? packed_t : packed) + bh * PackWave<D>::kHeadBytes;
  float beta = 1.0f, inv_beta = 1.0f;
  if (z) bwdw_beta<D, kThreads>(z + bh * NE, red[0], beta, inv_beta);
  // element i of this thread: normal: row 16 i + tid / 16, column 16 b + tid % 16; transposed: the 16 rows from 16 b on are
  // one run of 16 D floats, of which it takes every 256th
  const float* sp = transposed ? st + 16 * b * D + tid : st + (tid >> 4) * D + 16 * b + (tid & 15);
  const int step = transposed ? kThreads : 16 * D;
  float acc[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) acc[i] = 0.0f;
#pragma unroll 4
  for (int p = 0; p < parts; ++p) {
#pragma unroll
    for (int i = 0; i < PER; ++i) acc[i] += sp[(long long)p * NE + i * step];
  }
  float mS = 0.0f;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    mS = fmaxf(mS, fabsf(acc[i]));
    int ch, m;
    if (transposed) {
      const int e = tid + i * kThreads;
      m = e / D;
      ch = e % D;
    } else {
      ch = 16 * i + (tid >> 4);
      m = tid & 15;
    }
    tile[ch * RS + m] = acc[i];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mS = fmaxf(mS, __shfl_xor(mS, o));
  if ((tid & 63) == 0) red[1][tid >> 6] = mS;
  __syncthreads();
  mS = 0.0f;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) mS = fmaxf(mS, red[1][w]);
  const float aS = pow2_scale_for(mS);
  if (tid == 0) {
    float* scales = reinterpret_cast<float*>(out);
    scales[b] = inv_beta / aS;
    if (b == 0) scales[CB] = inv_beta;
  }
  u32x4* frag = reinterpret_cast<u32x4*>(out + PackWave<D>::kHeaderBytes);
  for (int f = tid; f < KS * 64; f += kThreads) {
    const int s = f >> 6, l = f & 63, ch = 32 * s + 8 * (l >> 4), m = l & 15;
    u32x4 w4;
#pragma unroll
    for (int w = 0; w < 4; ++w)
      w4[w] = pack2<F16>(tile[(ch + 2 * w) * RS + m] * aS, tile[(ch + 2 * w + 1) * RS + m] * aS);
    frag[(b * KS + s) * 64 + l] = w4;
  }
}

// A wave's stream of 16-token tiles of two tensors: X, the operand, and Y.  NST: tensors stored per tile.
template <int D, int NST>
struct BwdWave {
  using Sw = ApplyWaveShape<D>;
  using Sm = BwdWaveShape<D>;
  static constexpr int CPR = Sw::kCPR, KS = Sw::kKS, CB = Sw::kCB, NL = Sm::kNL, R = Sm::kRing, W = Sm::kWaves, TOK = Sm::kTok;
  static constexpr int C = 2 * NL, S = NST * NL;   // vector memory instructions of a tile's copies and stores
  static_assert(R == 3, "the wait counts below are written for a ring of three slots");
  static_assert(2 * C + 2 * S <= 63, "the vector-memory counter has six bits");

  const u32x4 *Xh, *Yh;
  int rsx, rsy;
  long long N;
  unsigned char* smem;
  int lane, wave, g;
  int trow[NL], cpos[NL];    // position u * 64 + lane of a tile image: token row, chunk it holds
  int rowb, x0;              // byte offset of this lane's token row in a tile image, its swizzle
  TileIter it, ahead;
  u32x4 A[CB][KS];
  float c1[CB], inv_beta;

  LF_DEV BwdWave(const u32x4* Xh_, int rsx_, const u32x4* Yh_, int rsy_, long long N_, int tiles_per_block, int wg, int nwg,
                 unsigned char* smem_)
      : Xh(Xh_), Yh(Yh_), rsx(rsx_), rsy(rsy_), N(N_), smem(smem_), lane(threadIdx.x & 63),
        wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)),
        it(wg, nwg, wave, tiles_per_block, (N_ + TOK - 1) / TOK, W), ahead(it) {
    g = lane >> 4;
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int P = u * 64 + lane, r = P / CPR;
      trow[u] = r;
      cpos[u] = (P % CPR) ^ Sw::swz(r);
    }
    rowb = (lane & 15) * CPR * 16;
    x0 = Sw::swz(lane & 15);
  }

  LF_DEV unsigned char* tile_ptr(int slot, int which) const {
    return smem + (slot * W + wave) * Sm::kSlotBytes + which * Sm::kTensorBytes;
  }
  LF_DEV int chunk_off(int chunk) const { return rowb + ((chunk ^ x0) << 4); }
  // where channels 16 b + 4 g .. + 3 of this lane's token lie: eight bytes
  LF_DEV int piece_off(int b) const { return chunk_off(2 * b + (g >> 1)) + 8 * (g & 1); }
  LF_DEV float* table() const { return reinterpret_cast<float*>(smem + Sm::kTabOffset); }
  LF_DEV int lim_of(long long tile) const {
    const long long rem = N - tile * TOK;
    return rem < TOK ? (int)rem : TOK;
  }

  // always C vector memory instructions, issued by every lane (rows past N re-read chunk 0 and are never stored)
  LF_DEV void issue_copy(long long tile, int slot) {
    const int lim = lim_of(tile);
#pragma unroll
    for (int which = 0; which < 2; ++which) {
      const int rs = which ? rsy : rsx;
      const u32x4* p = (which ? Yh : Xh) + tile * TOK * rs;
      unsigned char* sl = tile_ptr(slot, which);
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        const int c = trow[u] < lim ? trow[u] * rs + cpos[u] : 0;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(p + c),
                                         (LF_LDS void*)(sl + u * 1024), 16, 0, 2 /* nt */);
      }
    }
  }
  LF_DEV void prefetch() {
#pragma unroll
    for (int i = 0; i < R - 1; ++i) {
      if (ahead.valid()) issue_copy(ahead.t, i);
      ahead.next();
    }
  }
  // always NL vector memory instructions for a full tile (only a head's last tile is ragged; nothing is counted after it)
  LF_DEV void store_tile(long long tile, int slot, int which, u32x4* Oh, int rso) {
    const unsigned char* sl = tile_ptr(slot, which);
    const int lim = lim_of(tile);
    u32x4* op = Oh + tile * TOK * rso;
    u32x4 w[NL];
#pragma unroll
    for (int u = 0; u < NL; ++u) w[u] = *reinterpret_cast<const u32x4*>(sl + u * 1024 + lane * 16);
    if (lim == TOK) {   // (a branch per store would pull each read behind it, one LDS round trip each)
#pragma unroll
      for (int u = 0; u < NL; ++u) st_stream(op + trow[u] * rso + cpos[u], w[u]);
    } else {
#pragma unroll
      for (int u = 0; u < NL; ++u)
        if (trow[u] < lim) st_stream(op + trow[u] * rso + cpos[u], w[u]);
    }
  }
  // this head's operands as bwdw_pack wrote them
  LF_DEV void load_packed(const unsigned char* packed) {
    const u32x4* frag = reinterpret_cast<const u32x4*>(packed + PackWave<D>::kHeaderBytes);
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
      for (int s = 0; s < KS; ++s) A[b][s] = frag[(b * KS + s) * 64 + lane];
    const float* scales = reinterpret_cast<const float*>(packed);
#pragma unroll
    for (int b = 0; b < CB; ++b) c1[b] = scales[b];
    inv_beta = scales[CB];
  }

  // this lane's chunks of its token of X, raw
  LF_DEV void read_operand(int slot, u32x4 (&raw)[KS]) const {
#pragma unroll
    for (int s = 0; s < KS; ++s) raw[s] = *reinterpret_cast<const u32x4*>(tile_ptr(slot, 0) + chunk_off(4 * s + g));
  }
  // acc[b][i] = sum_ch M[16 b + 4 g + i][ch] x[ch] (beta and the packing scales taken out) for this lane's token.  The row is
  // scaled by a power of two so that its largest channel lies in [1, 2) as an fp16 operand, as in apply16_wave.
  LF_DEV void multiply(const u32x4 (&raw)[KS], f32x4 (&acc)[CB]) const {
    float m = 0.0f;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        float a, b;
        unpack2<F16>(raw[s][w], a, b);
        m = fmaxf(m, fmaxf(fabsf(a), fabsf(b)));
      }
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    uint32_t f = (__builtin_bit_cast(uint32_t, m) >> 23) & 0xffu;
    f = f < 1u ? 1u : (f > 253u ? 253u : f);
    const float mult = __builtin_bit_cast(float, (254u - f) << 23), post = __builtin_bit_cast(float, f << 23);
#pragma unroll
    for (int b = 0; b < CB; ++b) acc[b] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      u32x4 B;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        float a, b;
        unpack2<F16>(raw[s][w], a, b);
        B[w] = pack2<F16>(a * mult, b * mult);
      }
#pragma unroll
      for (int b = 0; b < CB; ++b) acc[b] = mfma_16x16x32<F16>(A[b][s], B, acc[b]);
    }
#pragma unroll
    for (int b = 0; b < CB; ++b) acc[b] *= c1[b] * post;
  }
  static LF_DEV float token_sum(float x) {   // over the four lanes that share a token
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
  }
  LF_DEV f32x4 read_piece(int slot, int which, int b) const {
    const u32x2 w = *reinterpret_cast<const u32x2*>(tile_ptr(slot, which) + piece_off(b));
    f32x4 x;
    float t0, t1;
    unpack2<F16>(w[0], t0, t1);
    x[0] = t0;
    x[1] = t1;
    unpack2<F16>(w[1], t0, t1);
    x[2] = t0;
    x[3] = t1;
    return x;
  }
  LF_DEV void write_piece(int slot, int which, int b, f32x4 x) const {
    *reinterpret_cast<u32x2*>(tile_ptr(slot, which) + piece_off(b)) = u32x2{pack2<F16>(x[0], x[1]), pack2<F16>(x[2], x[3])};
  }

  template <int NS, int NC> LF_DEV void wait_group() { wait_vmcnt<NS * S + NC * C>(); }
  LF_DEV void wait_mix(int ns, int nc) {   // at most ns tiles' stores and nc tiles' copies outstanding
    switch (ns * 3 + nc) {
      case 0: wait_group<0, 0>(); break;
      case 1: wait_group<0, 1>(); break;
      case 2: wait_group<0, 2>(); break;
      case 3: wait_group<1, 0>(); break;
      case 4: wait_group<1, 1>(); break;
      case 5: wait_group<1, 2>(); break;
      case 6: wait_group<2, 0>(); break;
      case 7: wait_group<2, 1>(); break;
      default: wait_group<2, 2>(); break;
    }
  }
  // Issue order per wave:  C0 C1 [state] | C2 K0 | S0 C3 K1 | S1 C4 K2 | ...  (see ApplyWave::stream).
  // compute(slot, lim) leaves the finished tensors in the slot; store(tile, slot) sends them.
  template <typename Compute, typename Store>
  LF_DEV void stream(Compute compute, Store store) {
    int slot = 0, prev_slot = 0, j = 0;
    long long prev_tile = -1;
    bool next_copied = false;   // C(j+1) exists
    {
      TileIter second = it;
      second.next();
      next_copied = second.valid();
    }
    while (it.valid()) {
      const long long tile = it.t;
      const bool have_prev = prev_tile >= 0;
      if (have_prev) store(prev_tile, prev_slot);
      const bool copied = ahead.valid();
      if (copied) issue_copy(ahead.t, have_prev ? prev_slot : R - 1);
      wait_mix(j >= 2 ? 2 : j, (next_copied ? 1 : 0) + (copied ? 1 : 0));
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      compute(slot, lim_of(tile));
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      it.next();
      ahead.next();
      next_copied = copied;
      prev_tile = tile;
      prev_slot = slot;
      slot = slot + 1 == R ? 0 : slot + 1;
      ++j;
    }
    if (prev_tile >= 0) store(prev_tile, prev_slot);
  }
};

// grid = (wgs, heads), block = 256, dynamic LDS BwdWaveShape<D>::kLdsBytes.  packed: S' transposed (bwdw_pack); z: the
// forward normalizer state.  GP: dense [B*H][N][D].  dzpart: [B*H][gridDim.x][D].
template <int D, int FM, bool NORM>
__global__ void __launch_bounds__(kThreads, 1)
bwdw_q(const u32x4* __restrict__ Q, Layout lq, const u32x4* __restrict__ G, Layout lg, u32x4* __restrict__ DQ, Layout ldq,
       u32x4* __restrict__ GP, const unsigned char* __restrict__ packed, const float* __restrict__ z,
       float* __restrict__ dzpart, float eps, long long N, int tiles_per_block) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using RG = BwdWave<D, 2>;
  constexpr int KS = RG::KS, CB = RG::CB, CPR = RG::CPR, NE = D * D + D;
  const long long bh = blockIdx.y;
  RG rg(G + lg.slice(bh), lg.row, Q + lq.slice(bh), lq.row, N, tiles_per_block, blockIdx.x, gridDim.x, smem);
  u32x4* DQh = DQ + ldq.slice(bh);
  u32x4* GPh = GP + bh * N * CPR;
  rg.prefetch();
  rg.load_packed(packed + bh * PackWave<D>::kHeadBytes);
  for (int i = threadIdx.x; i < D; i += kThreads) rg.table()[i] = NORM ? z[bh * NE + i] * rg.inv_beta : 0.0f;
  __syncthreads();
  const float eps_b = eps * rg.inv_beta;
  f32x4 dz[CB];
#pragma unroll
  for (int b = 0; b < CB; ++b) dz[b] = f32x4{0, 0, 0, 0};

  rg.stream(
      [&](int slot, int lim) {
        u32x4 raw[KS];
        rg.read_operand(slot, raw);
        f32x4 u[CB];
        rg.multiply(raw, u);
        float den = 0.0f, ru = 0.0f;
        if constexpr (NORM) {   // (phi(q) is worked out again below rather than kept: 40 registers at d = 160)
#pragma unroll
          for (int b = 0; b < CB; ++b) {
            const f32x4 x = rg.read_piece(slot, 1, b);
            const f32x4 zz = *reinterpret_cast<const f32x4*>(rg.table() + 16 * b + 4 * rg.g);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float r = phi<FM>(x[i]);
              den = __builtin_fmaf(r, zz[i], den);
              ru = __builtin_fmaf(r, u[b][i], ru);
            }
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        float invden = 1.0f, go = 0.0f;
        if constexpr (NORM) {
          invden = 1.0f / (RG::token_sum(den) + eps_b);
          go = RG::token_sum(ru) * invden;
        }
        const float e = (rg.lane & 15) < lim ? -go * invden : 0.0f;   // rows past the end add nothing
#pragma unroll
        for (int b = 0; b < CB; ++b) {
          const f32x4 x = rg.read_piece(slot, 1, b);
          const f32x4 zz = *reinterpret_cast<const f32x4*>(rg.table() + 16 * b + 4 * rg.g);
          f32x4 o;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float r = phi<FM>(x[i]);
            if constexpr (NORM) {
              dz[b][i] = __builtin_fmaf(r, e, dz[b][i]);
              o[i] = (u[b][i] - go * zz[i]) * invden * phi_prime_from<FM>(x[i], r);
            } else {
              o[i] = u[b][i] * phi_prime_from<FM>(x[i], r);
            }
          }
          rg.write_piece(slot, 1, b, o);
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) {   // gp = g / den'
          u32x4 w;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            float a, b;
            unpack2<F16>(raw[s][k], a, b);
            w[k] = pack2<F16>(a * invden, b * invden);
          }
          *reinterpret_cast<u32x4*>(rg.tile_ptr(slot, 0) + rg.chunk_off(4 * s + rg.g)) = w;
        }
      },
      [&](long long tile, int slot) {
        rg.store_tile(tile, slot, 1, DQh, ldq.row);
        rg.store_tile(tile, slot, 0, GPh, CPR);
      });

  // dz': over the sixteen tokens of a wave, then over the waves in order
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) dz[b][i] += __shfl_xor(dz[b][i], o);
  __syncthreads();
  float* part = reinterpret_cast<float*>(smem);
  if ((rg.lane & 15) == 0) {
#pragma unroll
    for (int b = 0; b < CB; ++b) *reinterpret_cast<f32x4*>(part + rg.wave * D + 16 * b + 4 * rg.g) = dz[b];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < D; i += kThreads)
    dzpart[(bh * gridDim.x + blockIdx.x) * D + i] = ((part[i] + part[D + i]) + part[2 * D + i]) + part[3 * D + i];
}

// grid = (wgs, heads), block = 256, dynamic LDS BwdWaveShape<D>::kLdsBytes.  packed: dS transposed (bwdw_pack); dzpart:
// `dzparts` partials of dz' per head.
template <int D, int FM>
__global__ void __launch_bounds__(kThreads, 1)
bwdw_k(const u32x4* __restrict__ K, const u32x4* __restrict__ V, Layout lkv, u32x4* __restrict__ DK, Layout ldkv,
       const unsigned char* __restrict__ packed, const float* __restrict__ dzpart, int dzparts, long long N,
       int tiles_per_block) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using RG = BwdWave<D, 1>;
  constexpr int KS = RG::KS, CB = RG::CB;
  const long long bh = blockIdx.y;
  RG rg(V + lkv.slice(bh), lkv.row, K + lkv.slice(bh), lkv.row, N, tiles_per_block, blockIdx.x, gridDim.x, smem);
  u32x4* DKh = DK + ldkv.slice(bh);
  rg.prefetch();
  rg.load_packed(packed + bh * PackWave<D>::kHeadBytes);
  for (int i = threadIdx.x; i < D; i += kThreads) {
    float s = 0.0f;
#pragma unroll 4
    for (int p = 0; p < dzparts; ++p) s += dzpart[(bh * dzparts + p) * D + i];
    rg.table()[i] = s * rg.inv_beta;
  }
  __syncthreads();
  rg.stream(
      [&](int slot, int) {
        u32x4 raw[KS];
        rg.read_operand(slot, raw);
        f32x4 t[CB];
        rg.multiply(raw, t);
#pragma unroll
        for (int b = 0; b < CB; ++b) {
          const f32x4 x = rg.read_piece(slot, 1, b);
          const f32x4 dz = *reinterpret_cast<const f32x4*>(rg.table() + 16 * b + 4 * rg.g);
          f32x4 o;
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] = (t[b][i] + dz[i]) * phi_prime_from<FM>(x[i], phi<FM>(x[i]));
          rg.write_piece(slot, 1, b, o);
        }
      },
      [&](long long tile, int slot) { rg.store_tile(tile, slot, 1, DKh, ldkv.row); });
}

}  // namespace lf
