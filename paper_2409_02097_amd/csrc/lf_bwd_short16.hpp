// Backward pass of short fp16 token streams at head widths above 80 in one launch: the derivative of lf_backward_wide.hpp
// (same units: S' = S / beta, z' = z / beta), nothing of it in memory but the four tensors, the state and the gradients.
//   grid = 2 x heads, block = 64 x 2 x d / 32 threads
// One workgroup of a head does dq and dk, the other dv; both sum the state gradient (a workgroup that did all would be a third
// longer, and 96 heads leave 160 of 256 CUs idle).  No workgroup waits for another.
//
// Queries, rounds of 64 tokens in LDS (a wave: 32 feature channels x half of the round's tokens):
//   u' = S' g          S' lies in LDS as operand rows; a lane ends up with 16 channels of one token of u' and reads the same
//                      channels of q: everything elementwise happens there, in fp32
//   den', go           summed over the waves through LDS
//   dq                 leaves from registers;  dz' is summed in registers
//   r, gp              phi(q) and g / den' replace q and g in LDS
//   dS'^T = gp^T r     (a wave: 32 feature channels x half of the value channels) in fp32 registers
// As the outer product r_i gp_i^T does not change when a row of one is scaled up and that of the other down, rows of phi(q) whose
// largest value is below one are scaled up to it, as the apply kernels do (lf_wave16.hpp: wave_operands): rows far below zero keep
// their bits, and gp = g / den' loses no headroom, since den' is below one with them.  Rows of large values are scaled down only
// as far as den' is above one (by all of their largest phi, gp would be up to phi_max / den' times g: for one query channel of 300
// among ordinary ones and dout of 1000 that is beyond fp16, and with it all of the head's dk and dv).  So |gp| is at most the larger
// of |g| and |g / den'|, and phi(q) at most itself.
// Then dS' turns into operands through LDS, with a scale per 16 output channels, and the keys follow, a round after the other:
// dk = (dS v + dz) phi'(k) or dv = dS^T phi(k).
//
// What bounds it: the chain of rounds between two barriers, 4.3 us per 64 queries and 2 us per 64 keys at d = 160: ten waves on
// four SIMDs, of which the fuller ones issue vector instructions 58 % of the time (conversions, phi, the elementwise part), LDS
// busy 40 %, matrix units 13 %; a wave alone on its part of the chain waits for LDS.  12 x 8 x 256 x 160 with the state given: 33
// us, against 68 of the seven launches before (lf_backward_wide.hpp), two of which only pack states; the training step 88.7 -> 50.0
// us.  At d = 160 a few registers go to scratch before the query rounds and come back behind them.
#pragma once
#include "lf_backward_wide.hpp"
#include "lf_solo.hpp"   // solo_unit

namespace lf {

template <int D> struct BwdShortCfg {
  static constexpr int kCB = D / 32, kWaves = 2 * kCB, kThreads = 64 * kWaves;
  static constexpr int kTokens = 64;                              // per round
  static constexpr int kCPR = D / 8, kKS = D / 16;
  static constexpr int kNL = kTokens * kCPR / kThreads;           // chunks per thread, tensor and round
  static_assert(kNL * kThreads == kTokens * kCPR, "whole rounds of chunks");
  static constexpr int kLow = (kCB + 1) / 2;                      // value-channel blocks of the first half of the waves
  // Rows in LDS, in elements: token rows of a tile and rows of the operand matrices.  20 (d = 96: 52) dwords modulo 64: reads of
  // one chunk of 16 rows meet every bank group once, transposing reads of 64 bytes of four neighbouring rows nearly so; and
  // every place is a constant away from a few registers (places swizzled without padding took 80 more of them).
  static constexpr int kRS = D == 96 ? 104 : 168;
  static_assert(kRS >= D, "a row must hold the channels");
  static constexpr int kTensorBytes = kTokens * kRS * 2, kSlotBytes = 2 * kTensorBytes;
  static constexpr int kMatrixBytes = D * kRS * 2;
  // a slot for the round that the waves work on, one for the next; the state, later the state gradient, as operand rows
  static constexpr int kMatrixOffset = 2 * kSlotBytes;
  static constexpr int kRedOffset = kMatrixOffset + kMatrixBytes;      // float4 per feature block and token of a round
  static constexpr int kTabOffset = kRedOffset + kCB * kTokens * 16;   // z' and dz: D floats each
  static constexpr int kScaleOffset = kTabOffset + 2 * D * 4;          // per 16 feature channels: the state's scale; maxima of
  static constexpr int kLdsBytes = kScaleOffset + (2 * kCB + 2 * kCB * 2 + 2 * kCB * kCB) * 4;   // the gradient, by half, by block
  static_assert(kLdsBytes <= 160 * 1024, "workgroup LDS limit of the device");
};

// fp32 products rounded once to a pair of halves: one instruction less per pair than products, then a conversion.  (Never
// straight on what a matrix instruction leaves: the compiler does not see through the assembly that it has to wait for it.)
LF_DEV uint32_t mul2_f16(float a0, float b0, float a1, float b1) {
  uint32_t w;
  asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(w) : "v"(a0), "v"(b0));
  asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(w) : "v"(a1), "v"(b1));
  return w;
}
// both halves of x times b
LF_DEV uint32_t scale2_f16(uint32_t x, float b) {
  uint32_t w;
  asm("v_fma_mixlo_f16 %0, %1, %2, 0 op_sel_hi:[1,0,0]" : "=v"(w) : "v"(x), "v"(b));
  asm("v_fma_mixhi_f16 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(w) : "v"(x), "v"(b));
  return w;
}
// phi of a stored pair in fp32 (elu + 1: the conversions are part of the multiplication and the addition)
template <int FM>
LF_DEV void phi2(uint32_t w, float& r0, float& r1) {
  if constexpr (FM == kPhiEluPlusOne) {
    const float kLog2e = 1.44269504088896340736f;
    float t0, t1, l0, l1;
    asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,0,0]" : "=v"(t0) : "v"(w), "v"(kLog2e));
    asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(t1) : "v"(w), "v"(kLog2e));
    asm("v_fma_mix_f32 %0, %1, 1.0, 1.0 op_sel_hi:[1,0,0]" : "=v"(l0) : "v"(w));
    asm("v_fma_mix_f32 %0, %1, 1.0, 1.0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(l1) : "v"(w));
    t0 = __builtin_amdgcn_exp2f(t0);
    t1 = __builtin_amdgcn_exp2f(t1);
    r0 = l0 > 1.0f ? l0 : t0;
    r1 = l1 > 1.0f ? l1 : t1;
  } else {
    unpack2<F16>(w, r0, r1);
    r0 = phi<FM>(r0);
    r1 = phi<FM>(r1);
  }
}
// phi' from phi: under elu + 1 phi itself up to 1, and 1 above; of relu 1 where phi is positive
template <int FM>
LF_DEV float phi_prime_of(float r) {
  if constexpr (FM == kPhiEluPlusOne) return fminf(r, 1.0f);
  else if constexpr (FM == kPhiRelu) return r > 0.0f ? 1.0f : 0.0f;
  else return 1.0f;
}
// over lanes l and l + 32
LF_DEV float halves_sum(float x) {
  const auto s = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
  const uint32_t a = s[0], b = s[1];
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
LF_DEV float halves_max(float x) {
  const auto s = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
  const uint32_t a = s[0], b = s[1];
  return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
// over lanes l and l ^ 16
LF_DEV float rows_max(float x) {
  const auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
  const uint32_t a = s[0], b = s[1];
  return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
LF_DEV float rows_sum(float x) {
  const auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
  const uint32_t a = s[0], b = s[1];
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
// over the sixteen lanes of a row, on the vector unit: lane ^ 1, lane ^ 2, then mirrored in eight and in sixteen
template <int CTRL> LF_DEV float dpp_of(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
LF_DEV float row16_sum(float x) {
  x += dpp_of<0xb1>(x);
  x += dpp_of<0x4e>(x);
  x += dpp_of<0x141>(x);
  return x + dpp_of<0x140>(x);
}
LF_DEV float row16_max(float x) {
  x = fmaxf(x, dpp_of<0xb1>(x));
  x = fmaxf(x, dpp_of<0x4e>(x));
  x = fmaxf(x, dpp_of<0x141>(x));
  return fmaxf(x, dpp_of<0x140>(x));
}

// One workgroup's work on a head: its gradients of q and k, or (VALUES) of v.  S: the head's forward state, D*D + D floats.
template <int D, int FM, bool VALUES>
LF_DEV void bwd_short_head(const u32x4* Qh, int qrow, const u32x4* Gh, int grow, const float* S, int N, float eps,
                           const u32x4* Kh, const u32x4* Vh, int kvrow, u32x4* DQh, int dqrow, u32x4* DKVh, int dkvrow,
                           unsigned char* smem) {
  using C = BwdShortCfg<D>;
  constexpr bool do_k = !VALUES, do_v = VALUES;
  constexpr int CB = C::kCB, NT = C::kThreads, TOK = C::kTokens, CPR = C::kCPR, KS = C::kKS, NL = C::kNL;
  constexpr int LOW = C::kLow, RS = C::kRS;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = wave >= CB ? 1 : 0, cb = wave - half * CB;
  const int rounds = (N + TOK - 1) / TOK;
  f32x4* red = reinterpret_cast<f32x4*>(smem + C::kRedOffset);
  float* ztab = reinterpret_cast<float*>(smem + C::kTabOffset);
  float* dztab = ztab + D;
  float* c1tab = reinterpret_cast<float*>(smem + C::kScaleOffset);
  float* maxc = c1tab + 2 * CB;          // [feature group of 16][half]
  float* maxe = maxc + 4 * CB;           // [value group of 16][feature block]
  uint16_t* M = reinterpret_cast<uint16_t*>(smem + C::kMatrixOffset);   // [feature channel][value channel]

  // ---- copies of a round: chunk u * NT + tid of either tensor, column ccol of row crow + u * kStep ----
  constexpr int kStep = NT / CPR;
  static_assert(NT % CPR == 0, "a thread's chunks lie in one column");
  const int crow = tid / CPR, ccol = tid % CPR;
  auto issue = [&](const u32x4* X, int rx, const u32x4* Y, int ry, int rd, u32x4 (&x)[NL], u32x4 (&y)[NL]) {
    const int lim = N - rd * TOK;      // (rows past it: the round's first; they add nothing and are never stored)
    const u32x4 *xp = X + (long long)rd * TOK * rx, *yp = Y + (long long)rd * TOK * ry;
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int r = crow + u * kStep < lim ? crow + u * kStep : 0;
      x[u] = xp[r * rx + ccol];
      y[u] = yp[r * ry + ccol];
    }
  };
  auto deposit = [&](unsigned char* slot, const u32x4 (&x)[NL], const u32x4 (&y)[NL]) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      unsigned char* p = slot + ((crow + u * kStep) * RS + ccol * 8) * 2;
      *reinterpret_cast<u32x4*>(p) = x[u];
      *reinterpret_cast<u32x4*>(p + C::kTensorBytes) = y[u];
    }
  };

  // ---- this lane's token of a round, and where its pieces lie ----
  const int tok = 32 * half + l32;
  const int operand_at = (tok * RS + 8 * h) * 2, pieces_at = (tok * RS + 32 * cb + 4 * h) * 2;
  auto piece_at = [&](int q) { return pieces_at + 16 * q; };   // channels 32 cb + 8 q + 4 h .. + 3
  auto read_pieces = [&](const unsigned char* t, u32x2 (&x)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = *reinterpret_cast<const u32x2*>(t + piece_at(q));
  };
  auto packed = [](f32x4 x) { return u32x2{pack2<F16>(x[0], x[1]), pack2<F16>(x[2], x[3])}; };
  // out[i] = sum over the contraction of 32 operand rows with this lane's token row of the tile
  auto multiply = [&](auto operand, const unsigned char* t) {
    f32x16 o;
#pragma unroll
    for (int i = 0; i < 16; ++i) o[i] = 0.0f;
#pragma unroll
    for (int s = 0; s < KS; ++s) o = mfma_32x32x16<F16>(operand(s), *reinterpret_cast<const u32x4*>(t + operand_at + 32 * s), o);
    return o;
  };
  const int m_at = (32 * cb + l32) * RS + 8 * h;
  auto operand_row = [&](int s) { return *reinterpret_cast<const u32x4*>(M + m_at + 16 * s); };
  // w[q]: channels 8 q + 4 h .. + 3 of the lane's token (q = 0..3 of the wave's 32), lanes l and l + 32 between them a chunk each
  auto store = [&](u32x4* Oh, int row, int rd, const u32x2 (&w)[4]) {
    u32x4 c[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const auto s0 = __builtin_amdgcn_permlane32_swap(w[2 * p][0], w[2 * p + 1][0], false, false);   // upper half against lower half
      const auto s1 = __builtin_amdgcn_permlane32_swap(w[2 * p][1], w[2 * p + 1][1], false, false);
      c[p] = u32x4{s0[0], s1[0], s0[1], s1[1]};
    }
    const int t = rd * TOK + tok;
    if (t < N) {
      u32x4* p = Oh + (long long)t * row + 4 * cb + h;
      p[0] = c[0];
      p[2] = c[1];
    }
  };
  // transposing reads: a lane's place in an operand of 32 channels x 16 rows; rows 8 h + lane / 4 % 4 and four further on
  const int tr_at = ((8 * h + ((lane & 15) >> 2)) * RS + 16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
  auto read_tr = [&](const unsigned char* t, int step, int block) {
    const uint16_t* p = reinterpret_cast<const uint16_t*>(t + tr_at) + 16 * step * RS + 32 * block;
    const u32x2 a = lds_read_tr16(p), b = lds_read_tr16(p + 4 * RS);
    return u32x4{a[0], a[1], b[0], b[1]};
  };

  // ---- the first round, the state ----
  u32x4 x[NL], y[NL];
  // rounds of queries, then rounds of keys: round i's chunks are in registers while round i - 1 is worked on, slot i % 2 takes them
  auto issue_round = [&](int i) {
    if (i < rounds) issue(Qh, qrow, Gh, grow, i, x, y);
    else if (i < 2 * rounds) issue(Kh, kvrow, Vh, kvrow, i - rounds, x, y);
  };
  auto slot_of = [&](int i) { return smem + (i & 1) * C::kSlotBytes; };
  issue_round(0);
  f32x4 raw[KS];   // the 16 feature rows of group 2 cb + half, scaled as one; as they follow one another in memory
  if (do_k) {
#pragma unroll
    for (int s = 0; s < KS; ++s) raw[s] = reinterpret_cast<const f32x4*>(S + 16 * (2 * cb + half) * D)[64 * s + lane];
  }
  float inv_beta;   // as bwdw_beta, every wave for itself
  {
    float zs = 0.0f;
#pragma unroll
    for (int i = 0; i < (D + 63) / 64; ++i) {
      const int c = 64 * i + lane;
      const float z = S[D * D + (c < D ? c : 0)];
      if (c < D) zs += z;
    }
    zs = halves_sum(rows_sum(row16_sum(zs)));
    inv_beta = 1.0f;
    if (zs > 0.0f && zs < 3.0e38f) {
      int ex;
      (void)__builtin_frexpf(zs, &ex);
      ex = ex > 100 ? 100 : (ex < -100 ? -100 : ex);
      inv_beta = __builtin_ldexpf(1.0f, -ex);
    }
  }
  for (int i = tid; i < D; i += NT) ztab[i] = S[D * D + i] * inv_beta;
  if (do_k) {
    float m = 0.0f;
#pragma unroll
    for (int s = 0; s < KS; ++s) m = fmaxf(m, fmaxf(fmaxf(fabsf(raw[s][0]), fabsf(raw[s][1])), fmaxf(fabsf(raw[s][2]), fabsf(raw[s][3]))));
    const float aS = pow2_scale_for(halves_max(rows_max(row16_max(m))));
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int p = 64 * s + lane, r = p / (D / 4), c = 4 * (p % (D / 4));
      *reinterpret_cast<u32x2*>(M + (16 * (2 * cb + half) + r) * RS + c) = packed(raw[s] * aS);
    }
    if (lane == 0) c1tab[2 * cb + half] = inv_beta / aS;
  }
  const float eps_b = eps * inv_beta;
  const f32x4* zz4 = reinterpret_cast<const f32x4*>(ztab + 32 * cb + 4 * h);     // + 2 q
  f32x16 acc[LOW];
#pragma unroll
  for (int e = 0; e < LOW; ++e)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[e][i] = 0.0f;
  f32x4 dz[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) dz[q] = f32x4{0, 0, 0, 0};
  const int eb0 = half * LOW, ebn = half ? CB - LOW : LOW;
  constexpr float kLog2e = 1.44269504088896340736f;

  // The power of two (or, for a row of negative channels under elu + 1, exp of minus the largest) that brings the row's largest
  // operand into [1, 2), from its largest channel (wave_operands, there on phi's argument: here phi itself is in fp32 first,
  // so that the factor ends where that has underflowed), and its inverse.  The inverse exceeds 2^most only where it is below one.
  auto row_scale = [&](float m, int most, float& mult, float& post) {
    if constexpr (FM == kPhiEluPlusOne) {
      int ex = __builtin_amdgcn_frexp_expf(m + 1.0f) - 1;
      ex = ex < most ? ex : most;
      const float c = m < 0.0f ? fminf(-m * kLog2e, 120.0f) : (float)-ex;
      mult = __builtin_amdgcn_exp2f(c);
      post = __builtin_amdgcn_exp2f(-c);
    } else {
      const float top = FM == kPhiRelu ? fmaxf(m, 0.0f) : m;
      int f = (int)(__builtin_bit_cast(uint32_t, top) >> 23) & 0xff;
      f = f < 127 + most ? f : 127 + most;
      f = f < 1 ? 1 : (f > 253 ? 253 : f);
      mult = __builtin_bit_cast(float, (uint32_t)(254 - f) << 23);
      post = __builtin_bit_cast(float, (uint32_t)f << 23);
    }
  };
  auto row_max = [&](const u32x2 (&raw)[4]) {   // of the wave's 32 channels
    f16x2 m = __builtin_bit_cast(f16x2, FM == kPhiIdentity ? 0u : 0xfc00fc00u);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint32_t w = raw[q][k];
        m = __builtin_elementwise_max(m, __builtin_bit_cast(f16x2, FM == kPhiIdentity ? w & 0x7fff7fffu : w));
      }
    return halves_max(fmaxf((float)m[0], (float)m[1]));
  };
  auto phi_all = [&](const u32x2 (&raw)[4], float (&r)[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      phi2<FM>(raw[q][0], r[4 * q], r[4 * q + 1]);
      phi2<FM>(raw[q][1], r[4 * q + 2], r[4 * q + 3]);
    }
  };
  auto write_phi = [&](unsigned char* t, const float (&r)[16], float mult) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<u32x2*>(t + piece_at(q)) =
          u32x2{mul2_f16(r[4 * q], mult, r[4 * q + 1], mult), mul2_f16(r[4 * q + 2], mult, r[4 * q + 3], mult)};
  };

  // ---- queries ----
  deposit(slot_of(0), x, y);
  issue_round(1);
  lds_barrier();
  for (int rd = 0; rd < rounds; ++rd) {
    unsigned char* qt = slot_of(rd);
    unsigned char* gt = qt + C::kTensorBytes;
    f32x16 u;
    if (do_k) u = multiply(operand_row, gt);
    float r[16], mrow;
    {
      u32x2 qx[4];
      read_pieces(qt, qx);
      mrow = row_max(qx);
      phi_all(qx, r);
    }
    float den = 0.0f, ru = 0.0f;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      float part = 0.0f;
#pragma unroll
      for (int q = 2 * p; q < 2 * p + 2; ++q) {
        const f32x4 zz = zz4[2 * q];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          den = __builtin_fmaf(r[4 * q + i], zz[i], den);
          if (do_k) part = __builtin_fmaf(r[4 * q + i], u[4 * q + i], part);
        }
      }
      if (do_k) ru = __builtin_fmaf(part, c1tab[2 * cb + p], ru);
    }
    den = halves_sum(den);
    if (do_k) ru = halves_sum(ru);
    if (h == 0) red[cb * TOK + tok] = f32x4{den, ru, mrow, 0.0f};
    lds_barrier();
    den = ru = 0.0f;
    float m = -__builtin_inff();
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const f32x4 p = red[b * TOK + tok];
      den += p[0];
      ru += p[1];
      m = fmaxf(m, p[2]);
    }
    const float invden = 1.0f / (den + eps_b);
    const bool in = rd * TOK + tok < N;      // rows past the end add nothing
    float mult, post;
    const int above = -__builtin_amdgcn_frexp_expf(invden);   // den' is 2^above and some, at most twice that
    row_scale(m, above > 0 ? above : 0, mult, post);
    const float gs = invden * post;
    write_phi(qt, r, mult);
    u32x2 gx[4];
    read_pieces(gt, gx);
    if (!in) {
#pragma unroll
      for (int q = 0; q < 4; ++q) gx[q] = u32x2{0, 0};
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<u32x2*>(gt + piece_at(q)) =
          in ? u32x2{scale2_f16(gx[q][0], gs), scale2_f16(gx[q][1], gs)} : u32x2{0, 0};   // (0 times an infinite gs)
    if (do_k) {
      const float e = -(ru * invden) * invden, ein = in ? e : 0.0f;
      u32x2 w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 zz = zz4[2 * q];
        const float cu = c1tab[2 * cb + (q >> 1)] * invden;
        float o[4], dp[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = 4 * q + i;
          dz[q][i] = __builtin_fmaf(r[k], ein, dz[q][i]);
          o[i] = __builtin_fmaf(u[k], cu, e * zz[i]);
          dp[i] = phi_prime_of<FM>(r[k]);
        }
        w[q] = u32x2{mul2_f16(o[0], dp[0], o[1], dp[1]), mul2_f16(o[2], dp[2], o[3], dp[3])};
      }
      store(DQh, dqrow, rd, w);
    }
    deposit(slot_of(rd + 1), x, y);   // (every wave has left round rd - 1, which this slot held, before the last barrier)
    issue_round(rd + 2);
    lds_barrier();
#pragma unroll
    for (int s = 0; s < TOK / 16; ++s) {
      const u32x4 b = read_tr(qt, s, cb);
#pragma unroll
      for (int e = 0; e < CB - LOW; ++e) acc[e] = mfma_32x32x16<F16>(read_tr(gt, s, eb0 + e), b, acc[e]);
    }
    if (CB % 2 == 1 && half == 0) {
#pragma unroll
      for (int s = 0; s < TOK / 16; ++s) acc[LOW - 1] = mfma_32x32x16<F16>(read_tr(gt, s, LOW - 1), read_tr(qt, s, cb), acc[LOW - 1]);
    }
  }

  // ---- the state gradient as operands ----
  float mc = 0.0f;
#pragma unroll
  for (int e = 0; e < LOW; ++e) {
    if (e < ebn) {
      float me[2] = {0.0f, 0.0f};
#pragma unroll
      for (int i = 0; i < 16; ++i) me[i >> 3] = fmaxf(me[i >> 3], fabsf(acc[e][i]));
      mc = fmaxf(mc, fmaxf(me[0], me[1]));
      if (do_v) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const float x = halves_max(rows_max(row16_max(me[p])));
          if (lane == 0) maxe[(2 * (eb0 + e) + p) * CB + cb] = x;
        }
      }
    }
  }
  if (do_k) {
    mc = halves_max(row16_max(mc));
    if (lane == 0 || lane == 16) maxc[(2 * cb + (lane >> 4)) * 2 + half] = mc;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int i = 0; i < 4; ++i) dz[q][i] = rows_sum(row16_sum(dz[q][i]));
    }
  }
  f32x4* dz4 = reinterpret_cast<f32x4*>(dztab + 32 * cb + 4 * h);   // + 2 q
  if (half == 0 && l32 == 0 && do_k) {
#pragma unroll
    for (int q = 0; q < 4; ++q) dz4[2 * q] = dz[q];
  }
  lds_barrier();   // the maxima are there, and every wave has left the last round
  if (half == 1 && l32 == 0 && do_k) {
#pragma unroll
    for (int q = 0; q < 4; ++q) dz4[2 * q] = (dz4[2 * q] + dz[q]) * inv_beta;
  }
  auto scale_k = [&](int group) { return pow2_scale_for(fmaxf(maxc[2 * group], maxc[2 * group + 1])); };
  auto scale_v = [&](int group) {
    float m = maxe[group * CB];
#pragma unroll
    for (int b = 1; b < CB; ++b) m = fmaxf(m, maxe[group * CB + b]);
    return pow2_scale_for(m);
  };
  {
    const float sk = scale_k(2 * cb + ((lane >> 4) & 1));
    const int at = (32 * cb + l32) * RS;
#pragma unroll
    for (int e = 0; e < LOW; ++e) {
      if (e < ebn) {
        const float sv[2] = {scale_v(2 * (eb0 + e)), scale_v(2 * (eb0 + e) + 1)};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float a0 = acc[e][4 * q], a1 = acc[e][4 * q + 1], a2 = acc[e][4 * q + 2], a3 = acc[e][4 * q + 3];
          const int to = at + 32 * (eb0 + e) + 8 * q + 4 * h;
          if (do_k)
            *reinterpret_cast<u32x2*>(M + to) = u32x2{pack2<F16>(a0 * sk, a1 * sk), pack2<F16>(a2 * sk, a3 * sk)};
          const float s = sv[q >> 1];
          if (do_v) *reinterpret_cast<u32x2*>(M + to) = u32x2{pack2<F16>(a0 * s, a1 * s), pack2<F16>(a2 * s, a3 * s)};
        }
      }
    }
  }
  lds_barrier();
  u32x4 B[KS];
  float cm[2];
  if (do_k) {
#pragma unroll
    for (int s = 0; s < KS; ++s) B[s] = operand_row(s);
    cm[0] = inv_beta / scale_k(2 * cb);
    cm[1] = inv_beta / scale_k(2 * cb + 1);
  }
  if (do_v) {
#pragma unroll
    for (int s = 0; s < KS; ++s) B[s] = read_tr(smem + C::kMatrixOffset, s, cb);
    cm[0] = inv_beta / scale_v(2 * cb);
    cm[1] = inv_beta / scale_v(2 * cb + 1);
  }

  // ---- keys ----
  for (int rd = 0; rd < rounds; ++rd) {
    unsigned char* kt = slot_of(rounds + rd);
    unsigned char* vt = kt + C::kTensorBytes;
    float r[16], mrow;
    {
      u32x2 kx[4];
      read_pieces(kt, kx);
      if (do_v) mrow = row_max(kx);
      phi_all(kx, r);
    }
    u32x2 w[4];
    if (do_v) {
      if (h == 0) red[cb * TOK + tok][0] = mrow;
      lds_barrier();
      float m = red[tok][0];
#pragma unroll
      for (int b = 1; b < CB; ++b) m = fmaxf(m, red[b * TOK + tok][0]);
      float mult, post;
      row_scale(m, 127, mult, post);   // (dv takes the inverse in fp32: no bound)
      write_phi(kt, r, mult);
      if (rd + 1 < rounds) deposit(slot_of(rounds + rd + 1), x, y);
      issue_round(rounds + rd + 2);
      lds_barrier();
      const f32x16 o = multiply([&](int s) { return B[s]; }, kt);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float c = cm[q >> 1] * post;
        w[q] = packed(f32x4{o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]} * c);
      }
    } else {
      const f32x16 o = multiply([&](int s) { return B[s]; }, vt);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 dzk = dz4[2 * q];
        float t[4], dp[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          t[i] = __builtin_fmaf(o[4 * q + i], cm[q >> 1], dzk[i]);
          dp[i] = phi_prime_of<FM>(r[4 * q + i]);
        }
        w[q] = u32x2{mul2_f16(t[0], dp[0], t[1], dp[1]), mul2_f16(t[2], dp[2], t[3], dp[3])};
      }
    }
    store(DKVh, dkvrow, rd, w);
    if (do_k && rd + 1 < rounds) {
      deposit(slot_of(rounds + rd + 1), x, y);
      issue_round(rounds + rd + 2);
      lds_barrier();
    }
  }
}

// state: [B*H][D*D + D], the forward state
template <int D, int FM>
__global__ void __launch_bounds__((BwdShortCfg<D>::kThreads), 1)
bwd_short16(const u32x4* __restrict__ Q, Layout lq, const u32x4* __restrict__ G, Layout lg, const float* __restrict__ state,
            int N, float eps, const u32x4* __restrict__ K, const u32x4* __restrict__ V, Layout lkv, u32x4* __restrict__ DQ,
            Layout ldq, u32x4* __restrict__ DK, u32x4* __restrict__ DV, Layout ldkv) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int unit = solo_unit((int)blockIdx.x, (int)gridDim.x);   // a head's workgroups share an XCD's L2
  const int bh = unit >> 1;
  const u32x4 *Qh = Q + lq.slice(bh), *Gh = G + lg.slice(bh), *Kh = K + lkv.slice(bh), *Vh = V + lkv.slice(bh);
  const float* S = state + (long long)bh * (D * D + D);
  if (unit & 1)
    bwd_short_head<D, FM, true>(Qh, lq.row, Gh, lg.row, S, N, eps, Kh, Vh, lkv.row, nullptr, 0, DV + ldkv.slice(bh), ldkv.row, smem);
  else
    bwd_short_head<D, FM, false>(Qh, lq.row, Gh, lg.row, S, N, eps, Kh, Vh, lkv.row, DQ + ldq.slice(bh), ldq.row,
                                 DK + ldkv.slice(bh), ldkv.row, smem);
}

}  // namespace lf
