// One launch for short token streams at head widths above 80: no partial states, no exchange between workgroups.
//   grid = heads x (d / (16 CB)) x parts, block = 4 d threads (one wave per 16 feature channels); CB = 2 or d / 32.
// A workgroup takes 16 CB value channels of one head and a part of its query tokens.  It computes the columns of the state
// that belong to the channels from all of the head's tokens, S[:, cols] = phi(K)^T V[:, cols], and z (Prop. 2, Eq. 5's
// normalizer), lays them out in LDS as matrix-core operands, and applies them to its query tokens, out[:, cols].  No workgroup
// waits for another; what is repeated for that is phi(K) and z, once per group of value channels and part, and the columns of
// the state once per part.
//
// What bounds such a call otherwise is three dependent launches, each with its fill, its round trips to memory and its drain
// (fp16 2 x 8 x 256 x 160: 8.4 + 6.3 + 8.7 us; per call 22.1 us, one launch 12.4).  Here K and V come to LDS through
// registers, four rounds of 64 tokens on their way, so that up to 256 tokens are one round trip, and a wave's first query
// tokens behind them; what bounds it is the chain of phi(K), LDS round trip and barrier between the launch and the operands
// (a graph of such calls takes as long as calls one by one, whose host part is 7.1 us).  1.3 us a round while each had a
// barrier of its own; where a call leaves CUs to others a workgroup takes four rounds (bf16 above 96 channels: two) in one (2 x 8 x 256 x
// 128 bf16 9.9 -> 9.6 us, 1 x 8 x 512 x 128 14.2 -> 13.5).
//
// Reduction: a round's phi(K) and V rows are written to LDS by all threads; after a barrier wave w multiplies feature block w
// with all column blocks (transposing LDS reads, 16x16x32 products, bf16: phi(K) in two terms) and with ones for z.  A wave
// holds its rows for all tokens: no sum across waves.
// Apply: as apply16_wave (fp16 operands for both storage types, query rows scaled into fp16's range, a power of two for each 16
// value channels), a wave taking 16 tokens at a time straight from memory: lane (token l % 16, chunks 4 s + l / 16).
#pragma once
#include "lf_solo.hpp"   // solo_unit
#include "lf_wave16.hpp"

namespace lf {

// CB: blocks of 16 value channels per workgroup; DEEP: several rounds between two barriers, the only workgroup of its CU
template <typename T, int D, int CB, bool DEEP> struct Short16Cfg {
  static constexpr int kWaves = D / 16, kThreads = 64 * kWaves;
  static constexpr int kCols = 16 * CB, kGroups = D / kCols;
  static_assert(D % kCols == 0, "whole groups of value channels");
  static constexpr int kTokens = 64;                 // per round
  static constexpr int kNS = NSplit<T>::value;
  static constexpr int kCPR = D / 8, kKS = D / 32;
  static constexpr int kNL = kTokens * kCPR / kThreads;   // K chunks per thread and round
  static_assert(kNL * kThreads == kTokens * kCPR && kThreads >= kTokens * kCols / 8, "whole rounds of chunks");
  // row strides in elements that spread the four rows of a transposing read over the banks
  static constexpr int kRS = D + 16, kVS = kCols + (kCols % 64 == 48 ? 8 : 16);
  static constexpr int kLevel = kTokens * kRS, kBuf = kNS * kLevel + kTokens * kVS;
  static constexpr int kAhead = 4;                   // rounds on their way
  // A CU's only workgroup takes as many rounds between two barriers as its LDS holds (4 or 2); where a CU has two workgroups,
  // they are each other's company: one round at a time, two buffers (fp16) or one (two of bf16 would leave one workgroup per CU).
  static constexpr int kTogether = !DEEP ? 1 : (kAhead * kBuf * 2 <= 156 * 1024 ? kAhead : 2);
  static constexpr int kBuffers = DEEP ? kTogether : (kNS == 1 ? 2 : 1);
  static constexpr int kOS = D + 8;                  // operand rows: [32 value channels, z', its remainder][d]
  static constexpr int kTileBytes = kBuffers * kBuf * 2;
  static constexpr int kOperandBytes = (kCols + 2) * kOS * 2;
  // (DEEP: the operands take the place of the tiles, which every wave has left by then)
  static constexpr int kOperandsAt = DEEP ? 0 : kTileBytes;
  static constexpr int kLdsBytes = DEEP ? (kTileBytes > kOperandBytes ? kTileBytes : kOperandBytes) : kTileBytes + kOperandBytes;
  static_assert(kLdsBytes <= 159 * 1024 && kAhead % kTogether == 0, "workgroup LDS limit of the device");
};

// keep: null, or where the heads' states go ([B*H][D*D + D]); O = null: nothing else is wanted (Q is not read).
// parts: workgroups that share a head's query tokens.
template <typename T, int D, int CB, int FM, bool NORM, bool DEEP>
__global__ void __launch_bounds__((Short16Cfg<T, D, CB, DEEP>::kThreads))
short16(const u32x4* __restrict__ K, const u32x4* __restrict__ V, long long kbatch, long long khead, int rs, unsigned heads,
        int N, int parts, const u32x4* __restrict__ Q, long long qbatch, long long qhead, int qrow, float eps,
        float* __restrict__ keep, u32x4* __restrict__ O, long long obatch, long long ohead, int orow) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using C = Short16Cfg<T, D, CB, DEEP>;
  constexpr int W = C::kWaves, NT = C::kThreads, NS = C::kNS, NL = C::kNL, KS = C::kKS, CPR = C::kCPR;
  constexpr int RS = C::kRS, VS = C::kVS, OS = C::kOS, TOK = C::kTokens, AH = C::kAhead;
  __shared__ float red[CB + 1][W];
  const int tid = threadIdx.x, lane = tid & 63, j16 = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int unit = solo_unit((int)blockIdx.x, (int)gridDim.x);   // a head's workgroups share an XCD's L2
  const int per_head = C::kGroups * parts;
  const int bh = unit / per_head, rem = unit - bh * per_head;
  const HeadAt head((unsigned)bh, heads);
  const int part = rem / C::kGroups, grp = rem - part * C::kGroups;
  uint16_t* lds = reinterpret_cast<uint16_t*>(smem);
  uint16_t* ops = reinterpret_cast<uint16_t*>(smem + C::kOperandsAt);

  // ---- query tokens: block t of 16 ---------------------------------------------------------------------------
  const u32x4* Qh = Q + head.slice(qbatch, qhead);
  auto load_q = [&](int t, u32x4 (&B)[KS]) {
    const int tok = 16 * t + j16;
    const u32x4* p = Qh + (long long)(tok < N ? tok : 0) * qrow + g4;   // (rows past the end are never stored)
#pragma unroll
    for (int s = 0; s < KS; ++s) B[s] = p[4 * s];
  };
  const int blocks = O ? (N + 15) / 16 : 0;
  int t = part * W + wave;
  u32x4 B[KS];

  // ---- state columns -------------------------------------------------------------------------------------------
  const u32x4* Kh = K + head.slice(kbatch, khead);
  const u32x4* Vh = V + head.slice(kbatch, khead) + grp * (C::kCols / 8);
  const int rounds = (N + TOK - 1) / TOK;
  int krow[NL], kcol[NL];
#pragma unroll
  for (int u = 0; u < NL; ++u) {
    const int p = u * NT + tid;
    krow[u] = p / CPR;
    kcol[u] = p % CPR;
  }
  const int vrow = tid / (C::kCols / 8), vcol = tid % (C::kCols / 8);
  const bool has_v = tid < TOK * C::kCols / 8;
  // rows past the end: a key that phi maps to 0 (the identity map: 0 itself), and no value
  constexpr uint32_t kPad = kPhiKillsLowest<FM> ? LowestBits<T>::value : 0u;
  u32x4 kr[AH][NL], vr[AH];
  auto issue = [&](int rd, u32x4 (&k)[NL], u32x4& v) {
    const int lim = N - rd * TOK;      // (rows past it: the round's first, replaced below)
    const u32x4* kp = Kh + (long long)rd * TOK * rs;
    const u32x4* vp = Vh + (long long)rd * TOK * rs;
#pragma unroll
    for (int u = 0; u < NL; ++u) k[u] = kp[(krow[u] < lim ? krow[u] : 0) * rs + kcol[u]];
    if (has_v) v = vp[(vrow < lim ? vrow : 0) * rs + vcol];
    if (lim < TOK) {
#pragma unroll
      for (int u = 0; u < NL; ++u)
        if (krow[u] >= lim) k[u] = u32x4{kPad, kPad, kPad, kPad};
      if (vrow >= lim) v = u32x4{0, 0, 0, 0};
    }
  };

  f32x4 acc[CB], accz;
  const uint32_t one2 = (uint32_t)OneBits<T>::value * 0x10001u;
  const u32x4 ones = {one2, one2, one2, one2};
  const int a_at = (8 * g4 + (j16 >> 2)) * RS + 16 * wave + 4 * (j16 & 3);
  const int v_at = (8 * g4 + (j16 >> 2)) * VS + 4 * (j16 & 3);

  // fp16 with elu + 1: keys far below zero, whose exponentials leave fp16's normal range, are summed a second time relative
  // to the largest key (see reduce16_phase: the same test and the same remedy; here all of a head's tokens together)
  constexpr bool kRescan = NS == 1 && FM == kPhiEluPlusOne;
  constexpr float kRescanBelow = -5.0f, kShiftFloor = -64.0f, kLog2e = 1.44269504088896340736f;
  auto workgroup_max = [&](float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
    __syncthreads();
    if (lane == 0) red[0][wave] = x;
    __syncthreads();
    x = red[0][0];
#pragma unroll
    for (int w = 1; w < W; ++w) x = fmaxf(x, red[0][w]);
    return x;
  };
  float kc = 0.0f;
  for (int pass = 0;; ++pass) {
#pragma unroll
    for (int b = 0; b < CB; ++b) acc[b] = f32x4{0, 0, 0, 0};
    accz = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < AH; ++s)
      if (s < rounds) issue(s, kr[s], vr[s]);
    // round base + s, from the registers to a buffer; its registers take the round four ahead
    auto convert = [&](int base, int s, uint16_t* buf) {
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        u32x4 ph, pl;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          if constexpr (NS == 1) {
            ph[w] = kRescan ? phi_pack2_scaled<T, FM>(kr[s][u][w], kc) : phi_pack2<T, FM>(kr[s][u][w]);
          } else {
            float x0, x1;
            unpack2<T>(kr[s][u][w], x0, x1);
            uint32_t h, l;
            pack2_split<T>(phi<FM>(x0), phi<FM>(x1), h, l);
            ph[w] = h;
            pl[w] = l;
          }
        }
        *reinterpret_cast<u32x4*>(buf + krow[u] * RS + kcol[u] * 8) = ph;
        if constexpr (NS == 2) *reinterpret_cast<u32x4*>(buf + C::kLevel + krow[u] * RS + kcol[u] * 8) = pl;
      }
      if (has_v) *reinterpret_cast<u32x4*>(buf + NS * C::kLevel + vrow * VS + vcol * 8) = vr[s];
      if (base + s + AH < rounds) issue(base + s + AH, kr[s], vr[s]);
      if (base + s == (rounds > 1 ? 1 : 0) && pass == 0 && t < blocks) load_q(t, B);   // the wave's first block
    };
    auto multiply = [&](const uint16_t* buf) {
#pragma unroll
      for (int ks = 0; ks < TOK / 32; ++ks) {
        u32x4 bv[CB];
#pragma unroll
        for (int b = 0; b < CB; ++b) {
          const uint16_t* p = buf + NS * C::kLevel + v_at + 32 * ks * VS + 16 * b;
          const u32x2 r0 = lds_read_tr16(p), r1 = lds_read_tr16(p + 4 * VS);
          bv[b] = u32x4{r0[0], r0[1], r1[0], r1[1]};
        }
#pragma unroll
        for (int l = 0; l < NS; ++l) {
          const uint16_t* p = buf + l * C::kLevel + a_at + 32 * ks * RS;
          const u32x2 r0 = lds_read_tr16(p), r1 = lds_read_tr16(p + 4 * RS);
          const u32x4 a = u32x4{r0[0], r0[1], r1[0], r1[1]};
#pragma unroll
          for (int b = 0; b < CB; ++b) acc[b] = mfma_16x16x32<T>(a, bv[b], acc[b]);
          accz = mfma_16x16x32<T>(a, ones, accz);
        }
      }
    };
    constexpr int G = C::kTogether;
    for (int base = 0; base < rounds; base += AH) {
#pragma unroll
      for (int first = 0; first < AH; first += G) {
        if (base + first >= rounds) break;
        uint16_t* bufs = lds + (G == 1 && C::kBuffers == 2 ? (first & 1) : 0) * C::kBuf;
#pragma unroll
        for (int i = 0; i < G; ++i) {
          if (base + first + i >= rounds) break;
          convert(base, first + i, bufs + i * C::kBuf);
        }
        lds_barrier();   // the rounds are complete in LDS; with two buffers of one the other one is free to be rewritten
        if (base + first + G <= rounds) {   // (all of them without a branch between: operands are read ahead)
#pragma unroll
          for (int i = 0; i < G; ++i) multiply(bufs + i * C::kBuf);
        } else {
#pragma unroll
          for (int i = 0; i < G - 1; ++i) {
            if (base + first + i >= rounds) break;
            multiply(bufs + i * C::kBuf);
          }
        }
        if (G == 1 ? C::kBuffers == 1 : base + first + G < rounds) lds_barrier();
      }
    }
    if constexpr (!kRescan) {
      break;
    } else {
      if (pass == 1) {
        const float back = __builtin_amdgcn_exp2f(-kc);      // the rescanned sums carry 2^kc
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[b] *= back;
        accz *= back;
        break;
      }
      const float zm = workgroup_max(fmaxf(fmaxf(accz[0], accz[1]), fmaxf(accz[2], accz[3])));
      if (!(zm < (float)N * 0x1p-11f)) break;                // ordinary data, NaNs
      f16x2 kmax2 = __builtin_bit_cast(f16x2, LowestBits<F16>::value);
      for (int p = tid; p < N * CPR; p += NT) {
        const u32x4 k = Kh[(long long)(p / CPR) * rs + p % CPR];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t word = k[w];
          kmax2 = __builtin_elementwise_max(kmax2, __builtin_bit_cast(f16x2, word));
        }
      }
      const float m = workgroup_max(fmaxf((float)kmax2[0], (float)kmax2[1]));
      // (not small after all -- many tokens of middling keys -- or nothing but the most negative value: keep the sums)
      if (!(m < kRescanBelow && m > -65504.0f)) break;
      kc = fmaxf(m, kShiftFloor) * -kLog2e;
      __syncthreads();   // (every wave has left the first pass's last round)
    }
  }

  // ---- this wave's 16 feature channels of the state columns: lane (rows 16 wave + 4 g4 + i, column 16 b + j16) ----
  if (keep && part == 0) {
    float* dst = keep + (long long)bh * (D * D + D);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 16 * wave + 4 * g4 + i;
#pragma unroll
      for (int b = 0; b < CB; ++b) dst[row * D + grp * C::kCols + 16 * b + j16] = acc[b][i];
      if (grp == 0 && j16 == 0) dst[D * D + row] = accz[i];
    }
  }
  if (!O) return;
  float m[CB + 1];
#pragma unroll
  for (int b = 0; b <= CB; ++b) {
    const f32x4 x = b < CB ? acc[b < CB ? b : 0] : accz;
    m[b] = fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3])));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m[b] = fmaxf(m[b], __shfl_xor(m[b], o));
  }
  __syncthreads();   // (workgroup_max's readers are done)
  if (lane == 0) {
#pragma unroll
    for (int b = 0; b <= CB; ++b) red[b][wave] = m[b];
  }
  __syncthreads();
  float scale[CB + 1];
#pragma unroll
  for (int b = 0; b <= CB; ++b) {
    float x = red[b][0];
#pragma unroll
    for (int w = 1; w < W; ++w) x = fmaxf(x, red[b][w]);
    scale[b] = b < CB || NORM ? pow2_scale_for(x) : 1.0f;
  }
#pragma unroll
  for (int b = 0; b < CB; ++b) {
    const f32x4 x = acc[b] * scale[b];
    *reinterpret_cast<u32x2*>(ops + (16 * b + j16) * OS + 16 * wave + 4 * g4) =
        u32x2{pack2<F16>(x[0], x[1]), pack2<F16>(x[2], x[3])};
  }
  if (NORM && j16 == 0) {
    const f32x4 z = accz * scale[CB];
    const u32x2 hi = {pack2<F16>(z[0], z[1]), pack2<F16>(z[2], z[3])};
    float h0, h1, h2, h3;
    unpack2<F16>(hi[0], h0, h1);
    unpack2<F16>(hi[1], h2, h3);
    *reinterpret_cast<u32x2*>(ops + C::kCols * OS + 16 * wave + 4 * g4) = hi;
    *reinterpret_cast<u32x2*>(ops + (C::kCols + 1) * OS + 16 * wave + 4 * g4) =
        u32x2{pack2<F16>(z[0] - h0, z[1] - h1), pack2<F16>(z[2] - h2, z[3] - h3)};
  }
  __syncthreads();
  // (rows 2 to 15 of the normalizer's block repeat its two rows: nobody reads those results)
  auto operand = [&](const uint16_t* at, const uint16_t* at_z, int b, int s) {
    return *reinterpret_cast<const u32x4*>((b < CB ? at + 16 * b * OS : at_z) + 32 * s);
  };
  int at = j16 * OS + 8 * g4, at_z = (C::kCols + (j16 & 1)) * OS + 8 * g4;
  const float eps_s = eps * scale[CB];
  float c1[CB];
#pragma unroll
  for (int b = 0; b < CB; ++b) c1[b] = scale[CB] / scale[b];

  // ---- out^T = S'^T phi(q)^T, 16 tokens at a time ------------------------------------------------------------------
  u32x2* Oh = reinterpret_cast<u32x2*>(O + head.slice(obatch, ohead)) + grp * (C::kCols / 4);
  while (t < blocks) {
    const int next = t + parts * W;
    u32x4 Bn[KS];
    if (next < blocks) load_q(next, Bn);
    asm volatile("" : "+v"(at), "+v"(at_z));   // read anew for each block: kept, the operands would spill
    float eps_tok, post;
    wave_operands<T, FM>(B, eps_s, eps_tok, post);
    f32x4 o[CB + 1];
#pragma unroll
    for (int b = 0; b <= CB; ++b) o[b] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int b = 0; b <= CB; ++b)
        if (b < CB || NORM) o[b] = mfma_16x16x32<F16>(operand(ops + at, ops + at_z, b, s), B[s], o[b]);
    float inv = post;
    if constexpr (NORM) inv = __builtin_amdgcn_rcpf(__shfl(o[CB][0] + o[CB][1], j16) + eps_tok);
    const int tok = 16 * t + j16;
    if (tok < N) {
      u32x2* p = Oh + 2LL * tok * orow;
#pragma unroll
      for (int b = 0; b < CB; ++b) {
        const f32x4 x = o[b] * (c1[b] * inv);
        p[4 * b + g4] = u32x2{pack2<T>(x[0], x[1]), pack2<T>(x[2], x[3])};
      }
    }
    t = next;
#pragma unroll
    for (int s = 0; s < KS; ++s) B[s] = Bn[s];
  }
}

// Rows of CPR 16-byte chunks of every head, one after the other.  grid = (whole rows / 256 chunks, heads), block = 256;
// `chunks`: of one head.
template <int CPR>
__global__ void __launch_bounds__(kThreads)
copy_rows(const u32x4* __restrict__ X, long long batch, long long head, int row, unsigned heads, unsigned chunks,
          u32x4* __restrict__ Y) {
  const unsigned c = blockIdx.x * kThreads + threadIdx.x;
  if (c >= chunks) return;
  const HeadAt at(blockIdx.y, heads);
  Y[(long long)at.index * chunks + c] = X[at.slice(batch, head) + (long long)(c / CPR) * row + c % CPR];
}

}  // namespace lf
