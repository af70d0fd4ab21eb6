// Fused evaluation of the paper's deployed network on CDNA4 matrix cores
// (gfx950): 160-channel residual tower with global-pooling blocks, from-to
// policy head and WDL value head (Section 3.5 "Chess representation and
// outputs", Section 4.3 "Convolution, attention, and global context", "Three
// policy representations", "Value and training-only heads", Appendix D).
//
// Kernels.  az_dep_kernel1 (int8, large batches): one wave per board, four such
// workgroups per compute unit (one per SIMD); the wave owns every output channel
// (five 32-channel MFMA blocks), so global pooling, the heads and both softmaxes
// need no exchange with other waves and no wave waits for another.  az_dep_kernel
// (everything else): four waves, one per SIMD, evaluate one board (small batches) or
// two, which share every weight fragment; they meet at a barrier per layer and share
// the heads, or with two boards run one board's heads per wave.
//
// Tower.  Every 3x3 convolution is an implicit GEMM D[ch][sq] = sum_k
// W[ch][k] X[k][sq] with weights as the A operand (streamed from L2 in pre-packed
// fragment order through a ring of prefetched groups) and the boards' activations
// as the B operand, read from LDS.  A 32-column block is whole board rows (row j of
// two boards and row j + 4 of each, or rows j, j + 2, j + 4, j + 6 of one), so the
// fragments of one horizontal tap and channel step serve all three vertical taps:
// the K steps run over (dx, channel step) with the three dy inside.
//
// What bounds it.  Large int8 batches: the wave's own instruction stream; its
// float64 requantisation and the float64 conversions of it (2 to 3 times a plain
// instruction) run with the matrix pipe idle, and beside 160 accumulators a lane the
// registers have room for a ring of three weight steps (5 KB each, 32 channels of a
// tap).  Small batches: that and the layers' chain of barriers.  Measured on 14x160
// against one-tap-at-a-time K loops and one board per workgroup, both on one box (us
// per batch): int8 64 boards 143 -> 139, 256 146 -> 142, 333 285 -> 197, 512 289 ->
// 212, 1,024 383 -> 366; bf16 64 boards 211 -> 203, 333 437 -> 293, 1,024 925 -> 713.
// Four int8 boards per workgroup were slower than a wave per board (1,024 boards 463
// against 365: the epilogue of 160 values a lane behind one barrier; its registers
// spill in the pooling layers).
//
// Global pooling (every pool_every-th block).  After the first convolution's
// K loop, the pooled channels (the last F/4) are transposed through LDS (int8:
// the exact accumulators; bf16: their activations); one lane per pooled
// channel activates (int8, in float64) and reduces its row to a board sum
// (fp64) and maximum, and the projection c = Wg [mean, max] runs in fp64.  c is
// added to the regular channels' bias (int8: in code units, in float64), so the
// epilogue that writes them takes it with the bias.  The second convolution leaves
// out the channel steps that hold pooled channels only.
//
// bf16 networks carry the residual stream h as hi + lo: hi = bf16(h) is the
// convolution operand in LDS, lo = bf16(h - hi) stays in the registers of the
// lane that produces it (a 16-bit significand for the running sum).
//
// Heads.  The final tensor h (int8 codes, or the bf16 hi + lo parts) feeds one
// bf16 GEMM whose rows are the 128 token rows and
// the value rows.  The token, query and key products then run from registers:
// each accumulator tile is split into bf16 hi + lo parts and used directly as
// an MFMA operand, with the next weight matrix packed in the order the
// accumulator registers hold their rows (a permutation of the K dimension
// applied to both operands of the product); with four waves per board the
// tiles that cross waves go through LDS as those same fragments.  Query-key
// logits are written to LDS once, gathered through the action table, and
// soft-maxed over the legal actions in fp32; the WDL head runs on the vector
// ALUs.
#pragma once

#include "az_internal.h"
#include "az_mfma_common.h"

#include <math.h>

namespace {

constexpr int DF = 160;                         // filters
constexpr int DNMB = DF / 32;                   // 32-channel blocks
constexpr int DG = DF / 4;                      // pooled channels
constexpr int DFR = DF - DG;                    // regular channels of a pooling block
constexpr int DCP = AZ_DEP_MAX_IN_PLANES;       // stem input channels (padded)
constexpr int DD = AZ_DEP_TOKEN;                // token width
constexpr int DEMB = AZ_DEP_EMB_ROWS / 32;      // embedding row blocks (tokens + value rows)
constexpr int DTB = DD / 32;                    // token row blocks

typedef __attribute__((ext_vector_type(4))) float f32x4;

// LDS geometry of a tensor with RB bytes per square of BPG boards: [row][board]
// [column], a square every CS bytes (an odd number of 16-byte units, so the 16
// squares of a ds_read_b128 group hit 16 different bank groups), every row ending
// in a zero pad that stands for the columns left and right of a board, read at the
// bank slot the virtual square would use.  A 32-column MFMA block j takes row
// j + i * NBK of each board, i < RPB, so a vertical tap of block j is block j +- 1;
// with one board a read group holds two rows, whose stride is half the banks.
template <int RB, int BPG>
struct DGeo {
  static constexpr int CS = RB + 16;
  static_assert(CS / 16 % 2 == 1, "odd square stride");
  static constexpr int PAD = BPG * 8 * CS;
  static constexpr int ZP0 = 256 + RB;
  static constexpr int ZP = BPG == 1 ? ZP0 + (12 - (PAD + ZP0) / 16 % 8) % 8 * 16 : ZP0;
  static constexpr int RS = PAD + ZP;
  static_assert(BPG != 1 || RS / 16 % 8 == 4, "two rows of a read group half the banks apart");
  static constexpr int NBK = 2 * BPG, RPB = 8 / NBK;
  static constexpr bool EDGE = RPB > 1;  // blocks -1 and NBK hold rows inside the board
  static constexpr int X0 = EDGE ? 1 : 0, NX = NBK + 2 * X0;
  static constexpr int BUF = 8 * RS;
  static __device__ __forceinline__ int at(int row, int board, int col) { return row * RS + (board * 8 + col) * CS; }
};

// Lane addresses, relative to the buffer, of the B fragments of one horizontal tap:
// channel step cs of block x is at row + x * RS + 32 * cs; blocks -1 and NBK have
// rows of their own (the pad where a row is outside the board).
template <int RB, int BPG>
struct DTaps {
  using G = DGeo<RB, BPG>;
  int row, lo, hi;
  __device__ __forceinline__ void init(int dx, int l32, int lhi) {
    const int i = l32 / (8 * BPG), v = l32 % (8 * BPG) + dx, c = (l32 & 7) + dx;
    const int pad = G::PAD + ((v * G::CS) & 255) + 16 * lhi;
    row = i * G::NBK * G::RS + ((unsigned)c < 8u ? v * G::CS + 16 * lhi : pad);
    lo = i > 0 ? row - G::RS : pad;
    hi = i < G::RPB - 1 ? row + G::NBK * G::RS : pad;
  }
  __device__ __forceinline__ void opaque() { asm volatile("" : "+v"(row), "+v"(lo), "+v"(hi)); }
  template <class Frag, int X>
  __device__ __forceinline__ Frag get(const uint8_t* buf, int cs) const {
    const uint8_t* q = X < 0 ? buf + lo : X >= G::NBK ? buf + hi : buf + X * G::RS + row;
    return *reinterpret_cast<const Frag*>(q + 32 * cs);
  }
};

// LDS writes before, reads after, across every wave of the workgroup
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
// the same ordering within one wave (LDS writes by its lanes, reads by others)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Board maximum (x) and sum (y) of pooled row pc of a pooling layer (first conv
// n_conv), read from LDS rows [pooled channel][square] with 16-byte chunks
// XOR-swizzled by the row.  int8 rows hold the exact accumulators, activated
// here in float64: act(acc * a[n] * s_w[f] + b1[f]); bf16 rows hold the
// activations.
template <bool QUANT>
__device__ __forceinline__ double2 pool_row(const AzDevNet& p, const float* pt, int pc, int n_conv) {
  double sum = 0.0, mx = 0.0;  // activations are >= 0
  // values made opaque to the compiler so that they are formed here, in the
  // pooling layer, not hoisted out of the block loop and held across the tower
  asm volatile("" : "+v"(pc));
  if constexpr (QUANT) {
    const size_t o = (size_t)n_conv * DF + DFR + pc;
    double cap = p.act_cap;
    asm volatile("" : "+v"(cap));
    const double pm = p.pool_m[o], pb = p.pool_b[o];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int4 v = *reinterpret_cast<const int4*>(pt + pc * 64 + ((j ^ (pc & 15)) << 2));
      const int vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double a = clamp_d(__builtin_fma((double)vv[r], pm, pb), cap);
        sum += a;
        mx = __builtin_fmax(mx, a);
      }
    }
  } else {
    float mxf = 0.0f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const float4 v = *reinterpret_cast<const float4*>(pt + pc * 64 + ((j ^ (pc & 15)) << 2));
      sum += (double)v.x;
      sum += (double)v.y;
      sum += (double)v.z;
      sum += (double)v.w;
      mxf = fmaxf(mxf, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
    }
    mx = mxf;
  }
  return make_double2(mx, sum);
}

// Folds the projected context c of a pooling layer into regular channel o's bias in
// an int8 layer's constant slot: it holds qbias = b / a[n+1] in float64, so c enters
// in code units (c / a[n+1]).
__device__ __forceinline__ void add_context(const AzDevNet& p, float* kslot, int o, double c, int n_conv) {
  reinterpret_cast<double*>(kslot)[o] += c * p.pool_cinv[n_conv];
}

// bf16 hi and lo parts of eight fp32 values: x = hi + lo within 2^-16 |x|.
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8& hi, bf16x8& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = x[2 * i], b = x[2 * i + 1];
    h[i] = pack_bf16x2(a, b);
    l[i] = pack_bf16x2(a - bf16_round(a), b - bf16_round(b));
  }
  hi = __builtin_bit_cast(bf16x8, make_uint4(h[0], h[1], h[2], h[3]));
  lo = __builtin_bit_cast(bf16x8, make_uint4(l[0], l[1], l[2], l[3]));
}

__device__ __forceinline__ f32x16 mma_bf16(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

template <int MK, int BPG_>
struct DepCfg {
  using T = Mk<MK>;
  static constexpr int BPG = BPG_;                    // boards per workgroup
  static constexpr bool QUANT = MK != MK_BF16;
  static constexpr int RB = DF * T::ES;               // bytes per square, tower tensors
  using GT = DGeo<RB, BPG>;                           // tower tensors
  using GS = DGeo<2 * DCP, BPG>;                      // stem input
  static_assert(GS::BUF <= GT::BUF, "stem input fits in the T buffer");
  static constexpr int BUF = GT::BUF;
  static constexpr int OFF_H = 0, OFF_T = BUF;
  // per-layer epilogue constants: [bias F] floats, or for int8 [qbias F | qmul F
  // | qres, qhi] doubles (the float64 requantisation; the layer's two scalars
  // ride along so that the epilogue reads them from LDS: a load from global
  // memory there would wait behind the weight stream)
  static constexpr int KE = QUANT ? 8 : 4;            // bytes of a bias
  static constexpr int KSLOT = QUANT ? 16 * DF + 16 : 4 * DF;
  static constexpr int OFF_K = 2 * BUF;
  static constexpr int OFF_PB = OFF_K + 2 * KSLOT;    // a pooling layer's biases, [board][F]
  static constexpr int OFF_PG = OFF_PB + BPG * DF * KE;  // pooled statistics, [board][2g] doubles
  static constexpr int TOWER_END = OFF_PG + BPG * 2 * DG * 8;
  static_assert(BPG * DG * 64 * 4 <= BUF, "pooled activations fit in the T buffer");
  static constexpr int OFF_X = OFF_T;                 // heads' bf16 input: the lo part (bf16 networks)
  // heads, per board (past every use of H and X)
  static constexpr int OFF_S = 0;                     // query-key logits [64][64] f32
  static constexpr int OFF_U = 64 * 64 * 4;           // value features [V][64] f32
  static constexpr int OFF_O = OFF_U + 32 * 64 * 4;   // promotion offsets [8][4] f32
  static constexpr int HEAD = OFF_O + 32 * 4;
  static constexpr int OFF_HC = (cmax(TOWER_END, BPG * HEAD) + 15) & ~15;  // head constants
  static constexpr int OFF_Q4 = (OFF_HC + (2 * AZ_DEP_EMB_ROWS + 2 * DD) * 4 + 255) & ~255;
  // one board: operand fragments shared by the heads' waves (four planes of 16 KB)
  static constexpr int SMEM = OFF_Q4 + (BPG == 1 ? 4 * 16384 : 0);
  static_assert(SMEM <= 160 * 1024, "LDS");
  static constexpr int CPT = DF / T::KS;              // channel steps
  static constexpr int NS = 3 * CPT;                  // (dx, channel step) groups per layer
  static constexpr int GROUP_BYTES = 3 * DNMB * 64 * T::FB;  // [dy][channel block] fragments
  static constexpr size_t LAYER_BYTES = (size_t)NS * GROUP_BYTES;
};

// WDL value head of one board, one wave (lane = 0..63), from the value
// features U[c][sq] in LDS: y = relu(W1 u + b1), z = W2 y + b2, softmax over
// (win, draw, loss), value = W - L.
__device__ __forceinline__ void dep_wdl(const AzDevNet& p, const float* U, float* __restrict__ value,
                                        float* __restrict__ wdl, int b, int lane) {
  {
    const int H = p.value_hidden, NU = p.value_channels * 64;
    float z0 = 0.0f, z1 = 0.0f, z2 = 0.0f;
    for (int k0 = 0; k0 < H; k0 += 64) {
      const int k = k0 + lane;
      const bool ok = k < H;
      const int kk = ok ? k : 0;
      float y = p.wdl_fc1_b[kk];
      // fc1 row of unit kk in chunks of 16 inputs, the next chunk in flight
      // (NU is a multiple of 64)
      float wa[16], wb[16];
      auto ld = [&](float(&d)[16], int i0) {
#pragma unroll
        for (int t = 0; t < 16; ++t) d[t] = p.wdl_fc1_t[(size_t)(i0 + t) * H + kk];
      };
      ld(wa, 0);
      for (int i0 = 0; i0 < NU; i0 += 32) {
        ld(wb, i0 + 16);
#pragma unroll
        for (int t = 0; t < 16; ++t) y = __builtin_fmaf(wa[t], U[i0 + t], y);
        if (i0 + 32 < NU) ld(wa, i0 + 32);
#pragma unroll
        for (int t = 0; t < 16; ++t) y = __builtin_fmaf(wb[t], U[i0 + 16 + t], y);
      }
      y = ok ? fmaxf(y, 0.0f) : 0.0f;
      z0 = __builtin_fmaf(p.wdl_fc2_w[kk], y, z0);
      z1 = __builtin_fmaf(p.wdl_fc2_w[H + kk], y, z1);
      z2 = __builtin_fmaf(p.wdl_fc2_w[2 * H + kk], y, z2);
    }
    z0 = wave_sum(z0) + p.wdl_fc2_b[0];
    z1 = wave_sum(z1) + p.wdl_fc2_b[1];
    z2 = wave_sum(z2) + p.wdl_fc2_b[2];
    const float m = fmaxf(z0, fmaxf(z1, z2));
    const float e0 = expf(z0 - m), e1 = expf(z1 - m), e2 = expf(z2 - m);
    const float is = 1.0f / (e0 + e1 + e2);
    if (lane == 0) {
      const float pw = e0 * is, pd = e1 * is, pl = e2 * is;
      value[b] = pw - pl;
      if (wdl) {
        wdl[3 * (size_t)b + 0] = pw;
        wdl[3 * (size_t)b + 1] = pd;
        wdl[3 * (size_t)b + 2] = pl;
      }
    }
  }
}

// Heads of one board (bd of the workgroup's, position b of the batch), run by one
// wave (lane = 0..63) once the final tower output h is in LDS (int8: codes in H;
// bf16: hi parts in H, lo parts in X): embedding, tokens, query-key logits and
// promotion offsets, legal-action softmax, WDL value head.  Every wave of the
// workgroup meets the one barrier inside, and does nothing else if it has no
// position (live: it has one).
template <int MK, int BPG>
__device__ __forceinline__ void dep_heads(const AzDevNet& p, uint8_t* smem_all, const uint8_t* __restrict__ legal,
                                          float* __restrict__ policy, float* __restrict__ value,
                                          float* __restrict__ wdl, int b, int bd, bool live, int lane_in) {
  using C = DepCfg<MK, BPG>;
  using GT = typename C::GT;
  uint8_t* const smem = smem_all + bd * C::HEAD;  // this board's logits, features, offsets
  constexpr bool QUANT = C::QUANT;
  constexpr int OFF_H = C::OFF_H;
  // the lane index, opaque to the compiler here, so that the heads' lane-dependent
  // addresses are computed in the heads instead of being shared with the stem's
  // and held (or spilled) across the tower
  int lane = lane_in;
  asm volatile("" : "+v"(lane));
  const int l32 = lane & 31, lhi = lane >> 5;

  // ---- embedding: E[row][sq] = sum_f Wemb[row][f] h[f][sq], rows = tokens then value channels
  f32x16 tok[DTB][2];   // token rows (accumulators, then values)
  f32x16 uacc[2];       // value rows 128..159
  if (live) {
    const uint8_t* ew = static_cast<const uint8_t*>(p.emb_w) + (size_t)lane * 16;
    // A fragments of K step s in ring slot s % 4, loaded three steps ahead
    constexpr int ES = DF / 16, ER = 4;
    bf16x8 awr[ER][DEMB];
    auto load_e = [&](int st) {
#pragma unroll
      for (int m = 0; m < DEMB; ++m) awr[st % ER][m] = g_frag<MK_BF16>(ew + (st * DEMB + m) * 64 * 16);
    };
#pragma unroll
    for (int st = 0; st < ER - 1; ++st) load_e(st);
#pragma unroll
    for (int s = 0; s < ES; ++s) {
      if (s + ER - 1 < ES) load_e(s + ER - 1);
      const bf16x8(&aw)[DEMB] = awr[s % ER];
      bf16x8 bx[2], bh[2];
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int j = n * 32 + l32;
        if constexpr (QUANT) {
          // eight codes of channels 16 s + 8 lhi .. + 7, exact in bf16
          const uint2 v = *reinterpret_cast<const uint2*>(smem_all + OFF_H + GT::at(j >> 3, bd, j & 7) + 16 * s + 8 * lhi);
          bx[n] = __builtin_bit_cast(
              bf16x8, make_uint4(pack_bf16x2(code_value<MK, 0>(v.x), code_value<MK, 1>(v.x)),
                                 pack_bf16x2(code_value<MK, 2>(v.x), code_value<MK, 3>(v.x)),
                                 pack_bf16x2(code_value<MK, 0>(v.y), code_value<MK, 1>(v.y)),
                                 pack_bf16x2(code_value<MK, 2>(v.y), code_value<MK, 3>(v.y))));
        } else {
          bx[n] = *reinterpret_cast<const bf16x8*>(smem_all + C::OFF_X + GT::at(j >> 3, bd, j & 7) + 32 * s + 16 * lhi);
          bh[n] = *reinterpret_cast<const bf16x8*>(smem_all + OFF_H + GT::at(j >> 3, bd, j & 7) + 32 * s + 16 * lhi);
        }
      }
#pragma unroll
      for (int n = 0; n < 2; ++n) {
#pragma unroll
        for (int m = 0; m < DTB; ++m) {
          tok[m][n] = mma_bf16(aw[m], bx[n], s == 0 ? f32x16{} : tok[m][n]);
          if constexpr (!QUANT) tok[m][n] = mma_bf16(aw[m], bh[n], tok[m][n]);
        }
        uacc[n] = mma_bf16(aw[DTB], bx[n], s == 0 ? f32x16{} : uacc[n]);
        if constexpr (!QUANT) uacc[n] = mma_bf16(aw[DTB], bh[n], uacc[n]);
      }
    }
  }
  wave_lds_sync();  // H and X are dead from here on
  if (!live) return;

  // token values relu(acc * scale + bias); value features u[c][sq] to LDS
  const float* HC = reinterpret_cast<const float*>(smem_all + C::OFF_HC);
  {
#pragma unroll
    for (int m = 0; m < DTB; ++m)
#pragma unroll
      for (int jq = 0; jq < 4; ++jq) {
        const int r0 = 32 * m + 8 * jq + 4 * lhi;
        const float4 sc = *reinterpret_cast<const float4*>(HC + r0);
        const float4 bc = *reinterpret_cast<const float4*>(HC + AZ_DEP_EMB_ROWS + r0);
        const float sv[4] = {sc.x, sc.y, sc.z, sc.w}, bv[4] = {bc.x, bc.y, bc.z, bc.w};
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int r = 0; r < 4; ++r) tok[m][n][4 * jq + r] = fmaxf(__builtin_fmaf(tok[m][n][4 * jq + r], sv[r], bv[r]), 0.0f);
      }
    float* U = reinterpret_cast<float*>(smem + C::OFF_U);
    const int V = p.value_channels;
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
      const int r0 = DD + 8 * jq + 4 * lhi;
      const float4 sc = *reinterpret_cast<const float4*>(HC + r0);
      const float4 bc = *reinterpret_cast<const float4*>(HC + AZ_DEP_EMB_ROWS + r0);
      const float sv[4] = {sc.x, sc.y, sc.z, sc.w}, bv[4] = {bc.x, bc.y, bc.z, bc.w};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ch = 8 * jq + 4 * lhi + r;
        if (ch < V) {
#pragma unroll
          for (int n = 0; n < 2; ++n) {
            float u = __builtin_fmaf(uacc[n][4 * jq + r], sv[r], bv[r]);
            if (p.value_conv_relu) u = fmaxf(u, 0.0f);
            U[ch * 64 + n * 32 + l32] = u;
          }
        }
      }
    }
  }

  // The token values as split bf16 operand fragments: K step s (0..7) of the
  // products below holds positions 8s .. 8s+7 of the lane's 64 token values
  // (the accumulators' register order), as x = hi + lo.
  bf16x8 tkh[DD / 16][2], tkl[DD / 16][2];
#pragma unroll
  for (int st = 0; st < DD / 16; ++st)
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      float x[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) x[t] = tok[(8 * st + t) / 16][n][(8 * st + t) % 16];
      split8(x, tkh[st][n], tkl[st][n]);
    }

  // action table entries and legal-mask words of the softmax, in flight during
  // the last query / key block's products
  constexpr int NA = AZ_FROMTO_ACTIONS, NIT = (NA + 255) / 256;
  uint4 tbl[NIT];
  uint32_t mkw[NIT];
  auto load_actions = [&]() {
    const uint8_t* lg = legal + (size_t)b * NA;
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
      const int a0 = 256 * i + 4 * lane;
      const bool in = a0 < NA;
      tbl[i] = *reinterpret_cast<const uint4*>(p.actions + (in ? a0 : 0));
      const uint32_t mk0 = *reinterpret_cast<const uint32_t*>(lg + (in ? a0 : 0));  // clamped, unconditional
      mkw[i] = in ? mk0 : 0u;
    }
  };

  // Per 32-row block m of Q^T = Wq tok^T + bq and K^T = Wk tok^T + bk (rows in
  // the token accumulators' register order), then the two K steps 2m, 2m+1 of
  //   S[f][t] = sum_d Q[f][d] K[t][d]      (hi*hi + hi*lo + lo*hi)
  //   O^T[k][t] = sum_d Wp[k][d] K[t][d]   (promotion offsets, last row's destinations)
  // that block holds.  Every accumulator runs the same chain of products as
  // when all blocks are computed at once (the four-wave heads do that), with
  // only one block of Q and K live at a time.
  f32x16 Sa[2][2], Oa;
  {
    const uint8_t* qp = static_cast<const uint8_t*>(p.q_w) + (size_t)lane * 16;
    const uint8_t* kp = static_cast<const uint8_t*>(p.k_w) + (size_t)lane * 16;
    const uint8_t* pw = static_cast<const uint8_t*>(p.p_w) + (size_t)lane * 16;
    constexpr int QS = DD / 16, QR = 2;
#pragma unroll
    for (int m = 0; m < DTB; ++m) {
      if (m == DTB - 1) load_actions();
      const bf16x8 apw0 = g_frag<MK_BF16>(pw + (2 * m) * 64 * 16), apw1 = g_frag<MK_BF16>(pw + (2 * m + 1) * 64 * 16);
      f32x16 Qm[2], Km[2];
      // A fragments of K step s in ring slot s % 2, loaded one step ahead
      bf16x8 aqr[QR], akr[QR];
      auto load_qk = [&](int st) {
        aqr[st % QR] = g_frag<MK_BF16>(qp + (st * DTB + m) * 64 * 16);
        akr[st % QR] = g_frag<MK_BF16>(kp + (st * DTB + m) * 64 * 16);
      };
      load_qk(0);
#pragma unroll
      for (int st = 0; st < QS; ++st) {
        if (st + 1 < QS) load_qk(st + 1);
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          Qm[n] = mma_bf16(aqr[st % QR], tkh[st][n], st == 0 ? f32x16{} : Qm[n]);
          Qm[n] = mma_bf16(aqr[st % QR], tkl[st][n], Qm[n]);
          Km[n] = mma_bf16(akr[st % QR], tkh[st][n], st == 0 ? f32x16{} : Km[n]);
          Km[n] = mma_bf16(akr[st % QR], tkl[st][n], Km[n]);
        }
      }
#pragma unroll
      for (int jq = 0; jq < 4; ++jq) {
        const int r0 = 32 * m + 8 * jq + 4 * lhi;
        const float4 bq = *reinterpret_cast<const float4*>(HC + 2 * AZ_DEP_EMB_ROWS + r0);
        const float4 bk = *reinterpret_cast<const float4*>(HC + 2 * AZ_DEP_EMB_ROWS + DD + r0);
        const float qv[4] = {bq.x, bq.y, bq.z, bq.w}, kv[4] = {bk.x, bk.y, bk.z, bk.w};
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            Qm[n][4 * jq + r] += qv[r];
            Km[n][4 * jq + r] += kv[r];
          }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int s = 2 * m + h;
        bf16x8 qh[2], ql[2], kh[2], kl[2];
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          float xq[8], xk[8];
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            xq[t] = Qm[n][8 * h + t];
            xk[t] = Km[n][8 * h + t];
          }
          split8(xq, qh[n], ql[n]);
          split8(xk, kh[n], kl[n]);
        }
#pragma unroll
        for (int mf = 0; mf < 2; ++mf)
#pragma unroll
          for (int nt = 0; nt < 2; ++nt) {
            Sa[mf][nt] = mma_bf16(qh[mf], kh[nt], s == 0 ? f32x16{} : Sa[mf][nt]);
            Sa[mf][nt] = mma_bf16(qh[mf], kl[nt], Sa[mf][nt]);
            Sa[mf][nt] = mma_bf16(ql[mf], kh[nt], Sa[mf][nt]);
          }
        Oa = mma_bf16(h ? apw1 : apw0, kh[1], s == 0 ? f32x16{} : Oa);
        Oa = mma_bf16(h ? apw1 : apw0, kl[1], Oa);
      }
    }
  }
  // logits pre-scaled by log2(e) for the exp2 softmax
  {
    const float log2e = 1.4426950408889634f;
    const float ss = log2e / sqrtf((float)DD);
    float* S = reinterpret_cast<float*>(smem + C::OFF_S);
#pragma unroll
    for (int mf = 0; mf < 2; ++mf)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int f = 32 * mf + 8 * (v / 4) + 4 * lhi + v % 4, t = 32 * nt + l32;
          S[f * 64 + t] = Sa[mf][nt][v] * ss;
        }
    float* O = reinterpret_cast<float*>(smem + C::OFF_O);
    if (lhi == 0 && l32 >= 24) {
#pragma unroll
      for (int k = 0; k < 4; ++k) O[(l32 - 24) * 4 + k] = Oa[k] * log2e;
    }
  }
  wave_sync();

  // ---- legal-action softmax: lane owns the runs of 4 actions at 256 i + 4 lane
  {
    const float* S = reinterpret_cast<const float*>(smem + C::OFF_S);
    const float* O = reinterpret_cast<const float*>(smem + C::OFF_O);
    float e[NIT][4];
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
      const int a0 = 256 * i + 4 * lane;
      const bool in = a0 < NA;  // NA is a multiple of 4
      const uint4 tb = tbl[i];
      const uint32_t mk = mkw[i];
      const uint32_t te[4] = {tb.x, tb.y, tb.z, tb.w};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t x = te[r], pr = x >> 12;
        const float z = S[x & 4095u] + (pr ? O[pr - 1] : 0.0f);
        const bool ok = in && ((mk >> (8 * r)) & 0xffu);
        e[i][r] = ok ? z : -INFINITY;
        mx = fmaxf(mx, e[i][r]);
      }
    }
    mx = wave_max(mx);
    const float msub = mx == -INFINITY ? 0.0f : mx;
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < NIT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        e[i][r] = __builtin_amdgcn_exp2f(e[i][r] - msub);  // exp2(-inf) = 0
        sum += e[i][r];
      }
    sum = wave_sum(sum);
    const float inv = sum > 0.0f ? 1.0f / sum : 0.0f;
    float* pol = policy + (size_t)b * NA;
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
      const int a0 = 256 * i + 4 * lane;
      if (a0 < NA)
        *reinterpret_cast<float4*>(pol + a0) = make_float4(e[i][0] * inv, e[i][1] * inv, e[i][2] * inv, e[i][3] * inv);
    }
  }

  // ---- WDL head
  dep_wdl(p, reinterpret_cast<const float*>(smem + C::OFF_U), value, wdl, b, lane);
}

// Heads of a workgroup's only board shared by its four waves (wave = 0..3,
// lane = 0..63), once the final tower output h is in LDS.  The arithmetic is
// dep_heads' operation for operation: every accumulator tile runs the same
// chain of products, split operands are split the same way, and the softmax
// normaliser is summed in the same order, so the outputs are bitwise the same.
// The work is spread as the tower's is: wave w owns token / query / key block w
// and one 32x32 tile of the logits S; operands that cross waves go through LDS
// as the very fragments a single wave would have taken from its registers
// (fragment set [square block][K step][lane] of 16 bytes).
template <int MK>
__device__ __forceinline__ void dep_heads4(const AzDevNet& p, uint8_t* smem, const uint8_t* __restrict__ legal,
                                           float* __restrict__ policy, float* __restrict__ value,
                                           float* __restrict__ wdl, int b, int wave, int lane) {
  using C = DepCfg<MK, 1>;
  using GT = typename C::GT;
  constexpr bool QUANT = C::QUANT;
  constexpr int OFF_H = C::OFF_H;
  constexpr int FS = 64 * 16;                   // bytes of one fragment set
  static_assert(DTB == 4, "one token block per wave");
  const int l32 = lane & 31, lhi = lane >> 5;
  const float* HC = reinterpret_cast<const float*>(smem + C::OFF_HC);
  uint8_t* const q4 = smem + C::OFF_Q4;
  // fragment set of K step s (0..7) of square block n in one of the four 16 KB planes
  auto fset = [&](int plane, int n, int s) { return q4 + plane * 16384 + ((n * 8 + s) * 64 + lane) * 16; };

  // action table entries and legal-mask words of this wave's two groups of 256
  // actions (actions 256 i + 4 lane .. + 3), in flight during the products
  constexpr int NA = AZ_FROMTO_ACTIONS, NIT = (NA + 255) / 256, GW = NIT / 4;
  static_assert(NIT % 4 == 0, "action groups per wave");
  uint4 tbl[GW];
  uint32_t mkw[GW];
  {
    const uint8_t* lg = legal + (size_t)b * NA;
#pragma unroll
    for (int g = 0; g < GW; ++g) {
      const int a0 = 256 * (wave * GW + g) + 4 * lane;
      const bool in = a0 < NA;
      tbl[g] = *reinterpret_cast<const uint4*>(p.actions + (in ? a0 : 0));
      const uint32_t mk0 = *reinterpret_cast<const uint32_t*>(lg + (in ? a0 : 0));  // clamped, unconditional
      mkw[g] = in ? mk0 : 0u;
    }
  }

  // every weight fragment of the wave's embedding rows and query / key rows,
  // issued at once: the heads then wait for one load latency, not one per step
  constexpr int ES = DF / 16, QS = DD / 16;
  bf16x8 awe[ES][2], aq[QS], ak[QS];
  {
    const uint8_t* ew = static_cast<const uint8_t*>(p.emb_w) + (size_t)lane * 16;
    const uint8_t* qp = static_cast<const uint8_t*>(p.q_w) + (size_t)lane * 16;
    const uint8_t* kp = static_cast<const uint8_t*>(p.k_w) + (size_t)lane * 16;
#pragma unroll
    for (int st = 0; st < ES; ++st) {
      awe[st][0] = g_frag<MK_BF16>(ew + (st * DEMB + wave) * FS);
      awe[st][1] = g_frag<MK_BF16>(ew + (st * DEMB + DTB) * FS);
    }
#pragma unroll
    for (int st = 0; st < QS; ++st) {
      aq[st] = g_frag<MK_BF16>(qp + (st * DTB + wave) * FS);
      ak[st] = g_frag<MK_BF16>(kp + (st * DTB + wave) * FS);
    }
  }

  // ---- embedding: token rows of block wave (both square blocks) and the value
  // rows on square block wave & 1 (kept by waves 0 and 1)
  const int nv = wave & 1;
  f32x16 tk[2], ua;
  {
#pragma unroll
    for (int s = 0; s < ES; ++s) {
      const bf16x8(&aw)[2] = awe[s];
      bf16x8 bx[2], bh[2];
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int j = n * 32 + l32;
        if constexpr (QUANT) {
          const uint2 v = *reinterpret_cast<const uint2*>(smem + OFF_H + GT::at(j >> 3, 0, j & 7) + 16 * s + 8 * lhi);
          bx[n] = __builtin_bit_cast(
              bf16x8, make_uint4(pack_bf16x2(code_value<MK, 0>(v.x), code_value<MK, 1>(v.x)),
                                 pack_bf16x2(code_value<MK, 2>(v.x), code_value<MK, 3>(v.x)),
                                 pack_bf16x2(code_value<MK, 0>(v.y), code_value<MK, 1>(v.y)),
                                 pack_bf16x2(code_value<MK, 2>(v.y), code_value<MK, 3>(v.y))));
        } else {
          bx[n] = *reinterpret_cast<const bf16x8*>(smem + C::OFF_X + GT::at(j >> 3, 0, j & 7) + 32 * s + 16 * lhi);
          bh[n] = *reinterpret_cast<const bf16x8*>(smem + OFF_H + GT::at(j >> 3, 0, j & 7) + 32 * s + 16 * lhi);
        }
      }
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        tk[n] = mma_bf16(aw[0], bx[n], s == 0 ? f32x16{} : tk[n]);
        if constexpr (!QUANT) tk[n] = mma_bf16(aw[0], bh[n], tk[n]);
      }
      const bf16x8 bxv = nv ? bx[1] : bx[0];
      ua = mma_bf16(aw[1], bxv, s == 0 ? f32x16{} : ua);
      if constexpr (!QUANT) {
        const bf16x8 bhv = nv ? bh[1] : bh[0];
        ua = mma_bf16(aw[1], bhv, ua);
      }
    }
  }
  wave_lds_sync();  // H and X are dead from here on

  // token values relu(acc * scale + bias), as the query / key products' B
  // fragments of K steps 2 wave and 2 wave + 1; value features u[c][sq] to LDS
  {
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
      const int r0 = 32 * wave + 8 * jq + 4 * lhi;
      const float4 sc = *reinterpret_cast<const float4*>(HC + r0);
      const float4 bc = *reinterpret_cast<const float4*>(HC + AZ_DEP_EMB_ROWS + r0);
      const float sv[4] = {sc.x, sc.y, sc.z, sc.w}, bv[4] = {bc.x, bc.y, bc.z, bc.w};
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) tk[n][4 * jq + r] = fmaxf(__builtin_fmaf(tk[n][4 * jq + r], sv[r], bv[r]), 0.0f);
    }
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float x[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t] = tk[n][8 * h + t];
        bf16x8 hi, lo;
        split8(x, hi, lo);
        *reinterpret_cast<bf16x8*>(fset(0, n, 2 * wave + h)) = hi;
        *reinterpret_cast<bf16x8*>(fset(1, n, 2 * wave + h)) = lo;
      }
    if (wave < 2) {
      float* U = reinterpret_cast<float*>(smem + C::OFF_U);
      const int V = p.value_channels;
#pragma unroll
      for (int jq = 0; jq < 4; ++jq) {
        const int r0 = DD + 8 * jq + 4 * lhi;
        const float4 sc = *reinterpret_cast<const float4*>(HC + r0);
        const float4 bc = *reinterpret_cast<const float4*>(HC + AZ_DEP_EMB_ROWS + r0);
        const float sv[4] = {sc.x, sc.y, sc.z, sc.w}, bv[4] = {bc.x, bc.y, bc.z, bc.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ch = 8 * jq + 4 * lhi + r;
          if (ch < V) {
            float u = __builtin_fmaf(ua[4 * jq + r], sv[r], bv[r]);
            if (p.value_conv_relu) u = fmaxf(u, 0.0f);
            U[ch * 64 + nv * 32 + l32] = u;
          }
        }
      }
    }
  }
  wave_lds_sync();

  // query and key block wave: Q^T = Wq tok^T + bq, K^T = Wk tok^T + bk over the
  // eight token K steps (hi, then lo)
  f32x16 Qa[2], Ka[2];
  {
#pragma unroll
    for (int s = 0; s < QS; ++s) {
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const bf16x8 xh = *reinterpret_cast<const bf16x8*>(fset(0, n, s));
        const bf16x8 xl = *reinterpret_cast<const bf16x8*>(fset(1, n, s));
        Qa[n] = mma_bf16(aq[s], xh, s == 0 ? f32x16{} : Qa[n]);
        Qa[n] = mma_bf16(aq[s], xl, Qa[n]);
        Ka[n] = mma_bf16(ak[s], xh, s == 0 ? f32x16{} : Ka[n]);
        Ka[n] = mma_bf16(ak[s], xl, Ka[n]);
      }
    }
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
      const int r0 = 32 * wave + 8 * jq + 4 * lhi;
      const float4 bq = *reinterpret_cast<const float4*>(HC + 2 * AZ_DEP_EMB_ROWS + r0);
      const float4 bk = *reinterpret_cast<const float4*>(HC + 2 * AZ_DEP_EMB_ROWS + DD + r0);
      const float qv[4] = {bq.x, bq.y, bq.z, bq.w}, kv[4] = {bk.x, bk.y, bk.z, bk.w};
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          Qa[n][4 * jq + r] += qv[r];
          Ka[n][4 * jq + r] += kv[r];
        }
    }
  }
  wave_lds_sync();  // token fragments dead
  // the logits' A (query) and B (key) fragments of K steps 2 wave, 2 wave + 1
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float x[8], y[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        x[t] = Qa[n][8 * h + t];
        y[t] = Ka[n][8 * h + t];
      }
      bf16x8 qh, ql, kh, kl;
      split8(x, qh, ql);
      split8(y, kh, kl);
      *reinterpret_cast<bf16x8*>(fset(0, n, 2 * wave + h)) = qh;
      *reinterpret_cast<bf16x8*>(fset(1, n, 2 * wave + h)) = ql;
      *reinterpret_cast<bf16x8*>(fset(2, n, 2 * wave + h)) = kh;
      *reinterpret_cast<bf16x8*>(fset(3, n, 2 * wave + h)) = kl;
    }
  wave_lds_sync();

  // S tile (mf, nt) = (wave >> 1, wave & 1): S[f][t] = sum_d Q[f][d] K[t][d]
  // (hi*hi + hi*lo + lo*hi); the promotion offsets O^T = Wp K^T of the last row's
  // destinations (square block 1, written by wave 3)
  {
    const int mf = wave >> 1, nt = wave & 1;
    const uint8_t* pw = static_cast<const uint8_t*>(p.p_w) + (size_t)lane * 16;
    bf16x8 apw[DD / 16];
#pragma unroll
    for (int s = 0; s < DD / 16; ++s) apw[s] = g_frag<MK_BF16>(pw + s * FS);
    f32x16 Sa, Oa;
#pragma unroll
    for (int s = 0; s < DD / 16; ++s) {
      const bf16x8 qh = *reinterpret_cast<const bf16x8*>(fset(0, mf, s));
      const bf16x8 ql = *reinterpret_cast<const bf16x8*>(fset(1, mf, s));
      const bf16x8 kh = *reinterpret_cast<const bf16x8*>(fset(2, nt, s));
      const bf16x8 kl = *reinterpret_cast<const bf16x8*>(fset(3, nt, s));
      Sa = mma_bf16(qh, kh, s == 0 ? f32x16{} : Sa);
      Sa = mma_bf16(qh, kl, Sa);
      Sa = mma_bf16(ql, kh, Sa);
      Oa = mma_bf16(apw[s], kh, s == 0 ? f32x16{} : Oa);
      Oa = mma_bf16(apw[s], kl, Oa);
    }
    // logits pre-scaled by log2(e) for the exp2 softmax
    const float log2e = 1.4426950408889634f;
    const float ss = log2e / sqrtf((float)DD);
    float* S = reinterpret_cast<float*>(smem + C::OFF_S);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int f = 32 * mf + 8 * (v / 4) + 4 * lhi + v % 4, t = 32 * nt + l32;
      S[f * 64 + t] = Sa[v] * ss;
    }
    float* O = reinterpret_cast<float*>(smem + C::OFF_O);
    if (wave == 3 && lhi == 0 && l32 >= 24) {
#pragma unroll
      for (int k = 0; k < 4; ++k) O[(l32 - 24) * 4 + k] = Oa[k] * log2e;
    }
  }
  wave_lds_sync();  // query / key fragments dead

  // ---- legal-action softmax: wave w gathers and exponentiates groups 2w, 2w + 1;
  // the maximum is exact in any order, the normaliser is summed by wave 0 over all
  // groups in the one-wave order
  float* E = reinterpret_cast<float*>(q4);            // numerators, 2048 slots
  float* MX = reinterpret_cast<float*>(q4 + 8192);    // per-wave maxima, then 1 / sum
  {
    const float* S = reinterpret_cast<const float*>(smem + C::OFF_S);
    const float* O = reinterpret_cast<const float*>(smem + C::OFF_O);
    float e[GW][4];
    float mx = -INFINITY;
#pragma unroll
    for (int g = 0; g < GW; ++g) {
      const int a0 = 256 * (wave * GW + g) + 4 * lane;
      const bool in = a0 < NA;  // NA is a multiple of 4
      const uint4 tb = tbl[g];
      const uint32_t mk = mkw[g];
      const uint32_t te[4] = {tb.x, tb.y, tb.z, tb.w};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t x = te[r], pr = x >> 12;
        const float z = S[x & 4095u] + (pr ? O[pr - 1] : 0.0f);
        const bool ok = in && ((mk >> (8 * r)) & 0xffu);
        e[g][r] = ok ? z : -INFINITY;
        mx = fmaxf(mx, e[g][r]);
      }
    }
    mx = wave_max(mx);
    if (lane == 0) MX[wave] = mx;
    wave_lds_sync();
    mx = fmaxf(fmaxf(MX[0], MX[1]), fmaxf(MX[2], MX[3]));
    const float msub = mx == -INFINITY ? 0.0f : mx;
#pragma unroll
    for (int g = 0; g < GW; ++g) {
#pragma unroll
      for (int r = 0; r < 4; ++r) e[g][r] = __builtin_amdgcn_exp2f(e[g][r] - msub);  // exp2(-inf) = 0
      *reinterpret_cast<float4*>(E + 256 * (wave * GW + g) + 4 * lane) = make_float4(e[g][0], e[g][1], e[g][2], e[g][3]);
    }
    wave_lds_sync();
    if (wave == 0) {
      float sum = 0.0f;
#pragma unroll
      for (int i = 0; i < NIT; ++i) {
        const float4 v = *reinterpret_cast<const float4*>(E + 256 * i + 4 * lane);
        sum += v.x;
        sum += v.y;
        sum += v.z;
        sum += v.w;
      }
      sum = wave_sum(sum);
      if (lane == 0) MX[4] = sum > 0.0f ? 1.0f / sum : 0.0f;
    }
    wave_lds_sync();
    const float inv = MX[4];
    float* pol = policy + (size_t)b * NA;
#pragma unroll
    for (int g = 0; g < GW; ++g) {
      const int a0 = 256 * (wave * GW + g) + 4 * lane;
      if (a0 < NA)
        *reinterpret_cast<float4*>(pol + a0) = make_float4(e[g][0] * inv, e[g][1] * inv, e[g][2] * inv, e[g][3] * inv);
    }
  }

  // ---- WDL head (wave 1): y = relu(W1 u + b1), z = W2 y + b2, softmax, value = W - L
  if (wave == 1) dep_wdl(p, reinterpret_cast<const float*>(smem + C::OFF_U), value, wdl, b, lane);
}

// One wave evaluates one board (int8): four such workgroups share a compute unit,
// one per SIMD, and none waits for another.  The wave owns all five channel blocks
// and both square blocks.
template <int MK>
__global__ __attribute__((amdgpu_flat_work_group_size(64, 64), amdgpu_waves_per_eu(1, 1))) void
az_dep_kernel1(AzDevNet p, const float* __restrict__ planes, const uint8_t* __restrict__ legal,
              float* __restrict__ policy, float* __restrict__ value, float* __restrict__ wdl) {
  using C = DepCfg<MK, 1>;
  using GT = typename C::GT;
  using GS = typename C::GS;
  using T = typename C::T;
  using frag_t = typename T::frag;
  using acc_t = typename T::acc;
  constexpr bool QUANT = C::QUANT;
  static_assert(QUANT, "bf16 boards are evaluated by four waves");
  constexpr int OFF_H = C::OFF_H, OFF_T = C::OFF_T;

  __shared__ __attribute__((aligned(16))) uint8_t smem[C::OFF_Q4];
  static_assert(4 * C::OFF_Q4 <= 160 * 1024, "four workgroups per compute unit");

  constexpr int NBW = GT::NBK;  // square blocks (the wave owns the whole board)
  const int lane = threadIdx.x;
  const int l32 = lane & 31, lhi = lane >> 5, lr0 = l32 / 8 * GT::NBK;
  const int b = blockIdx.x;
  const int Cin = p.in_planes;

  // ---- ingest: zero pads, planes -> bf16 [square][64 channels] at OFF_T
  auto zero_pads = [&](auto geo, int off) {
    using G = decltype(geo);
    constexpr int PC = G::ZP / 16;
    for (int i = lane; i < 8 * PC; i += 64)
      *reinterpret_cast<i32x4*>(smem + off + i / PC * G::RS + G::PAD + i % PC * 16) = i32x4{0, 0, 0, 0};
  };
  zero_pads(GT{}, OFF_H);
  zero_pads(GS{}, OFF_T);
  {
    // item k = planes 8k..8k+7: lane = square, eight coalesced loads, one
    // 16-byte store
    constexpr int KI = DCP / 8;
    float pv[KI][8];
#pragma unroll
    for (int ki = 0; ki < KI; ++ki)
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int c = 8 * ki + t;
        const bool ok = c < Cin;
        const float x = planes[((size_t)b * Cin + (ok ? c : 0)) * 64 + lane];
        pv[ki][t] = ok ? x : 0.0f;
      }
#pragma unroll
    for (int ki = 0; ki < KI; ++ki) {
      const int k = ki;
      *reinterpret_cast<uint4*>(smem + OFF_T + GS::at(lane >> 3, 0, lane & 7) + 16 * k) =
          make_uint4(pack_bf16x2(pv[ki][0], pv[ki][1]), pack_bf16x2(pv[ki][2], pv[ki][3]),
                     pack_bf16x2(pv[ki][4], pv[ki][5]), pack_bf16x2(pv[ki][6], pv[ki][7]));
    }
  }

  // tower weights: a ring of one group, the three dy of a (dx, channel step), each
  // loaded two steps ahead.  The stream is read through a buffer resource: the
  // lane's offset is a constant VGPR, the step's byte offset a scalar, so a step's
  // five loads cost no vector address arithmetic.
  constexpr int STEP_BYTES = C::GROUP_BYTES / 3;
  const __amdgpu_buffer_rsrc_t twr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.tower_w), (short)0, (int)(2 * p.blocks * C::LAYER_BYTES), 0x00020000);
  const int tvoff = lane * T::FB;
  frag_t A[3][DNMB];
  auto load_step = [&](frag_t(&dst)[DNMB], int soff) {
#pragma unroll
    for (int m = 0; m < DNMB; ++m)
      dst[m] = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(twr, tvoff, soff + m * 64 * T::FB, 0));
  };
  // per-layer epilogue constants of conv index k (0 = stem), [qbias F | qmul F | qres,
  // qhi] doubles, as lane-held 16-byte chunks loaded at the start of a layer and
  // parked in LDS before its barrier
  constexpr int KV = C::KSLOT / 16;                  // 16-byte chunks per slot
  constexpr int KPL = (KV + 63) / 64;                // per lane
  auto load_consts = [&](int k, float4(&dst)[KPL]) {
#pragma unroll
    for (int t = 0; t < KPL; ++t) {
      const int i = lane + 64 * t;
      const double* src = i < DF / 2 ? p.qbias + (size_t)k * DF + 2 * i
                          : i < DF   ? p.qmul + (size_t)k * DF + 2 * (i - DF / 2)
                                     : p.qext + 2 * (size_t)k;
      dst[t] = i < KV ? *reinterpret_cast<const float4*>(src) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  auto store_consts = [&](int slot, const float4(&v)[KPL]) {
    float4* dst = reinterpret_cast<float4*>(smem + C::OFF_K + slot * C::KSLOT);
#pragma unroll
    for (int t = 0; t < KPL; ++t)
      if (lane + 64 * t < KV) dst[lane + 64 * t] = v[t];
  };
  // head constants, staged once: embedding row scale and bias, query and key biases
  {
    float* hc = reinterpret_cast<float*>(smem + C::OFF_HC);
    for (int i = lane; i < AZ_DEP_EMB_ROWS; i += 64) {
      hc[i] = p.emb_sc[i];
      hc[AZ_DEP_EMB_ROWS + i] = p.emb_bc[i];
    }
    for (int i = lane; i < DD; i += 64) {
      hc[2 * AZ_DEP_EMB_ROWS + i] = p.q_b[i];
      hc[2 * AZ_DEP_EMB_ROWS + DD + i] = p.k_b[i];
    }
  }
  {
    float4 k0[KPL];
    load_consts(1, k0);
    store_consts(0, k0);
  }
  __syncthreads();

  // ---- stem: bf16 3x3 conv over 64 (padded) input channels, K = 576, its fp32 sums
  // in the order (dy, dx, channel step)
  {
    constexpr int SSTEP = DNMB * 64 * 16;  // bytes per K step of the stem stream
    const uint8_t* sw8 = static_cast<const uint8_t*>(p.stem_w) + (size_t)lane * 16;
    f32x16 sacc[DNMB][NBW];
    // A fragments in a ring of SR steps, B fragments one step ahead
    constexpr int SR = 4, CS4 = DCP / 16, NST = 9 * CS4;
    bf16x8 a[SR][DNMB];
    auto load_a = [&](int st) {
      const int tap = st / CS4, f = (tap % 3 * CS4 + st % CS4) * 3 + tap / 3;
#pragma unroll
      for (int m = 0; m < DNMB; ++m) a[st % SR][m] = g_frag<MK_BF16>(sw8 + f * SSTEP + m * 64 * 16);
    };
    auto load_b = [&](auto st_c, bf16x8(&dst)[NBW]) {
      constexpr int st = decltype(st_c)::value, tap = st / CS4, dy = tap / 3 - 1;
      DTaps<2 * DCP, 1> t;
      t.init(tap % 3 - 1, l32, lhi);
      dst[0] = t.template get<bf16x8, dy>(smem + OFF_T, st % CS4);
      dst[1] = t.template get<bf16x8, 1 + dy>(smem + OFF_T, st % CS4);
    };
#pragma unroll
    for (int st = 0; st < SR - 1; ++st) load_a(st);
    bf16x8 bcur[NBW], bnext[NBW];
    load_b(std::integral_constant<int, 0>{}, bcur);
    static_for<0, NST>([&](auto st_c) {
      constexpr int st = decltype(st_c)::value;
      if constexpr (st + SR - 1 < NST) load_a(st + SR - 1);
      if constexpr (st + 1 < NST) load_b(std::integral_constant<int, (st + 1 < NST ? st + 1 : st)>{}, bnext);
#pragma unroll
      for (int m = 0; m < DNMB; ++m)
#pragma unroll
        for (int n = 0; n < NBW; ++n)
          sacc[m][n] = mma_bf16(a[st % SR][m], bcur[n], st == 0 ? f32x16{} : sacc[m][n]);
#pragma unroll
      for (int n = 0; n < NBW; ++n) bcur[n] = bnext[n];
    });
    // the tower's first weight steps, in flight during the stem's epilogue
    load_step(A[0], 0);
    load_step(A[1], STEP_BYTES);
    // epilogue: bias, activation, codes stored at OFF_H
#pragma unroll
    for (int m = 0; m < DNMB; ++m)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ch0 = m * 32 + 8 * q + 4 * lhi;
        double mq[4], bq[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          mq[r] = p.qmul[ch0 + r];
          bq[r] = p.qbias[ch0 + r];
        }
#pragma unroll
        for (int n = 0; n < NBW; ++n) {
          const f32x16& v = sacc[m][n];
          // fp32 sum of the bf16 matrix instruction; rescale and rounding in float64
          *reinterpret_cast<uint32_t*>(smem + OFF_H + GT::at(lr0 + n, 0, l32 & 7) + ch0) =
              pack_codes_d<MK>(__builtin_fma((double)v[4 * q + 0], mq[0], bq[0]),
                               __builtin_fma((double)v[4 * q + 1], mq[1], bq[1]),
                               __builtin_fma((double)v[4 * q + 2], mq[2], bq[2]),
                               __builtin_fma((double)v[4 * q + 3], mq[3], bq[3]), p.qhi[0]);
        }
      }
  }
  __syncthreads();
  zero_pads(GT{}, OFF_T);

  // ---- residual tower
  {
    constexpr int CPT = C::CPT;
    acc_t c[DNMB][NBW];
    const int nconv = 2 * p.blocks;

    const int l32_ = l32, lhi_ = lhi;
    // POOL: first convolution of a pooling block; SHORT: its second one, whose
    // pooled input channels have zero weights: it leaves out the groups past the
    // last regular one
    auto conv = [&](auto second_c, auto pool_c, int n_conv) {
      constexpr bool SECOND = decltype(second_c)::value, PB = decltype(pool_c)::value;
      constexpr bool POOL = PB && !SECOND, SHORT = PB && SECOND;
      // lane coordinates, opaque to the compiler per layer, so that the layer's
      // many lane-dependent addresses are computed in the layer instead of being
      // hoisted out of the block loop and held (or spilled) across it
      int l32 = l32_, lhi = lhi_;
      asm volatile("" : "+v"(l32), "+v"(lhi));
      const int lr0 = l32 / 8 * GT::NBK;
      const int wl = n_conv * (int)C::LAYER_BYTES;  // byte offset of the layer in the stream
      const bool has_next = n_conv + 1 < nconv;
      constexpr int in_off = SECOND ? OFF_T : OFF_H;
      constexpr int out_off = SECOND ? OFF_H : OFF_T;
      float* kslot = reinterpret_cast<float*>(smem + C::OFF_K + (n_conv & 1) * C::KSLOT);
      // the next layer's epilogue constants, in flight during this layer
      float4 kn[KPL];
      if (has_next) load_consts(n_conv + 2, kn);
      // groups visited, in order: visit v is group v (SHORT: the last channel step of
      // a tap left out)
      constexpr int CPV = SHORT ? (DFR + T::KS - 1) / T::KS : CPT, NV = 3 * CPV;
      DTaps<C::RB, 1> taps[3];
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) taps[dx].init(dx - 1, l32, lhi);
      frag_t x[GT::NX], xn[GT::NX];
      auto load_x = [&](auto v_c, frag_t(&dst)[GT::NX]) {
        constexpr int v = decltype(v_c)::value;
        static_for<0, GT::NX>([&](auto i_c) {
          constexpr int i = decltype(i_c)::value;
          dst[i] = taps[v / CPV].template get<frag_t, i - GT::X0>(smem + in_off, v % CPV);
        });
      };
      load_x(std::integral_constant<int, 0>{}, x);
      static_for<0, NV>([&](auto v_c) {
        constexpr int v = decltype(v_c)::value;
        static_for<0, 3>([&](auto d_c) {
          constexpr int d = decltype(d_c)::value, s2 = 3 * v + d + 2, v2 = s2 / 3;  // two steps ahead
          // past the layer's end the next layer's first steps (past the network's last
          // layer this layer is re-read and never used)
          constexpr int g2 = v2 < NV ? v2 / CPV * CPT + v2 % CPV : v2 - NV;
          load_step(A[(d + 2) % 3], (v2 < NV ? wl : has_next ? wl + (int)C::LAYER_BYTES : wl) + (3 * g2 + s2 % 3) * STEP_BYTES);
          if constexpr (d == 0 && v + 1 < NV) load_x(std::integral_constant<int, (v + 1 < NV ? v + 1 : v)>{}, xn);
#pragma unroll
          for (int m = 0; m < DNMB; ++m)
#pragma unroll
            for (int n = 0; n < NBW; ++n)
              c[m][n] = T::mma(A[d][m], x[n + d], (v == 0 && d == 0) ? acc_t{} : c[m][n]);
          // each MFMA followed by one of the next group's LDS reads, then by one of
          // the prefetched step's weight loads
          static_for<0, DNMB * 2>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value;
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if constexpr (d == 0 && i < GT::NX && v + 1 < NV) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            if constexpr (i < DNMB) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
          });
          __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (v + 1 < NV) {
#pragma unroll
          for (int i = 0; i < GT::NX; ++i) x[i] = xn[i];
        }
      });

      // global pooling: pooled channels' board mean and maximum, projected to a
      // context term that is folded into the regular channels' bias (in place in
      // this layer's constant slot)
      if constexpr (POOL) {
        // (1) the pooled channels to LDS as [pooled channel][square] in the T
        //     buffer (written by this layer's epilogue only afterwards); rows of
        //     256 bytes with 16-byte chunks XOR-swizzled by the row: the exact
        //     accumulators, activated in float64 in (2)
        float* pt = reinterpret_cast<float*>(smem + OFF_T);
        static_assert(DG * 64 * 4 <= C::BUF, "pooled activations fit in the T buffer");
        static_for<0, DNMB * 4>([&](auto k_c) {
          constexpr int k = decltype(k_c)::value, m = k / 4, q = k % 4;
          if constexpr (32 * m + 8 * q >= DFR) {
            const int ch0 = 32 * m + 8 * q + 4 * lhi;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int pc = ch0 + r - DFR;
#pragma unroll
              for (int n = 0; n < NBW; ++n) {
                const int sq = (lr0 + n) * 8 + (l32 & 7), idx = pc * 64 + (((sq >> 2) ^ (pc & 15)) << 2) + (sq & 3);
                reinterpret_cast<int*>(pt)[idx] = c[m][n][4 * q + r];
              }
            }
          }
        });
        wave_lds_sync();
        // (2) lane pc < g: board sum (fp64) and maximum of its row; g = [mean, max]
        double* pg = reinterpret_cast<double*>(smem + C::OFF_PG);
        if (lane < DG) {
          const double2 mx_sum = pool_row<QUANT>(p, pt, lane, n_conv);
          pg[lane] = mx_sum.y * (1.0 / 64.0);
          pg[DG + lane] = mx_sum.x;
        }
        wave_lds_sync();
        // (3) c[o] = sum_i Wg[o][i] g[i] in fp64 (fp32 weights are exact): lane L
        //     takes outputs L and L + 64; the weights, [i/4][o][4] floats, stream
        //     in chunks of 16 inputs with the next chunk in flight
        const float4* wt = reinterpret_cast<const float4*>(p.pool_wt) +
                           (size_t)(n_conv / 2 / p.pool_every) * (2 * DG / 4) * AZ_DEP_POOL_OPAD;
        constexpr int NCH = 2 * DG / 16;
        float4 wbuf[2][2][4];
        auto load_chunk = [&](float4(&dst)[2][4], int chk) {
#pragma unroll
          for (int k4 = 0; k4 < 4; ++k4) {
            dst[0][k4] = wt[(size_t)(4 * chk + k4) * AZ_DEP_POOL_OPAD + lane];
            dst[1][k4] = wt[(size_t)(4 * chk + k4) * AZ_DEP_POOL_OPAD + 64 + lane];
          }
        };
        load_chunk(wbuf[0], 0);
        double c0 = 0.0, c1 = 0.0;
#pragma unroll
        for (int chk = 0; chk < NCH; ++chk) {
          if (chk + 1 < NCH) load_chunk(wbuf[(chk + 1) & 1], chk + 1);
#pragma unroll
          for (int k4 = 0; k4 < 4; ++k4) {
            const float4 w0 = wbuf[chk & 1][0][k4], w1 = wbuf[chk & 1][1][k4];
            const double* gi = pg + 16 * chk + 4 * k4;
            c0 = __builtin_fma((double)w0.x, gi[0], c0);
            c1 = __builtin_fma((double)w1.x, gi[0], c1);
            c0 = __builtin_fma((double)w0.y, gi[1], c0);
            c1 = __builtin_fma((double)w1.y, gi[1], c1);
            c0 = __builtin_fma((double)w0.z, gi[2], c0);
            c1 = __builtin_fma((double)w1.z, gi[2], c1);
            c0 = __builtin_fma((double)w0.w, gi[3], c0);
            c1 = __builtin_fma((double)w1.w, gi[3], c1);
          }
        }
        // regular channel o's bias takes c[o] (int8: in code units, c[o] / a[n+1])
        add_context(p, kslot, lane, c0, n_conv);
        if (lane + 64 < DFR) add_context(p, kslot, lane + 64, c1, n_conv);
        zero_pads(GT{}, OFF_T);  // (1) wrote over them
        wave_lds_sync();
      }

      // epilogue: per run of 4 channels; LDS reads of constants (and residual
      // codes) issued two runs ahead
      const double* kd = reinterpret_cast<const double*>(kslot);
      const float hi = (float)kd[2 * DF + 1];
      const double rq = SECOND ? kd[2 * DF] : 0.0;
      constexpr int NRUN = DNMB * 4, EP_AHEAD = 2, EP_RING = EP_AHEAD + 1;
      // qbias and qmul of the run's four channels, float64, and (second convolutions)
      // the residual codes, read in place
      struct KQ { double b[4], m[4]; };
      KQ kq[EP_RING];
      uint32_t rcode[SECOND ? EP_RING : 1][NBW];
      auto ep_addr = [&](int m, int q, int n) {
        return out_off + GT::at(lr0 + n, 0, l32 & 7) + m * 32 + 8 * q + 4 * lhi;
      };
      auto ep_load = [&](auto k_c) {
        constexpr int k = decltype(k_c)::value, m = k / 4, q = k % 4, slot = k % EP_RING;
        const int ch0 = m * 32 + 8 * q + 4 * lhi;
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          const double2 b2 = *reinterpret_cast<const double2*>(kd + ch0 + r);
          const double2 m2 = *reinterpret_cast<const double2*>(kd + DF + ch0 + r);
          kq[slot].b[r] = b2.x;
          kq[slot].b[r + 1] = b2.y;
          kq[slot].m[r] = m2.x;
          kq[slot].m[r + 1] = m2.y;
        }
        if constexpr (SECOND) {
#pragma unroll
          for (int n = 0; n < NBW; ++n) rcode[slot][n] = *reinterpret_cast<const uint32_t*>(smem + ep_addr(m, q, n));
        }
      };
      static_for<0, EP_AHEAD>([&](auto k_c) { ep_load(k_c); });
      static_for<0, NRUN>([&](auto k_c) {
        constexpr int k = decltype(k_c)::value, m = k / 4, q = k % 4, slot = k % EP_RING;
        if constexpr (k + EP_AHEAD < NRUN) ep_load(std::integral_constant<int, k + EP_AHEAD>{});
#pragma unroll
        for (int n = 0; n < NBW; ++n) {
          const acc_t& v = c[m][n];
          // float64 requantisation: z = acc * qmul + qbias (+ residual code * qres)
          const KQ& kk = kq[slot];
          double z[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) z[r] = __builtin_fma((double)v[4 * q + r], kk.m[r], kk.b[r]);
          if constexpr (SECOND) {
            const uint32_t rc = rcode[slot][n];
            z[0] = __builtin_fma(code_value_d<MK, 0>(rc), rq, z[0]);
            z[1] = __builtin_fma(code_value_d<MK, 1>(rc), rq, z[1]);
            z[2] = __builtin_fma(code_value_d<MK, 2>(rc), rq, z[2]);
            z[3] = __builtin_fma(code_value_d<MK, 3>(rc), rq, z[3]);
          }
          *reinterpret_cast<uint32_t*>(smem + ep_addr(m, q, n)) = pack_codes_d<MK>(z[0], z[1], z[2], z[3], hi);
        }
      });
      if (has_next) store_consts((n_conv + 1) & 1, kn);
      __syncthreads();
    };

    for (int blk = 0; blk < p.blocks; ++blk) {
      const bool pool = p.pool_every > 0 && blk % p.pool_every == p.pool_every - 1;
      if (pool) {
        conv(std::false_type{}, std::true_type{}, 2 * blk);
        conv(std::true_type{}, std::true_type{}, 2 * blk + 1);
      } else {
        conv(std::false_type{}, std::false_type{}, 2 * blk);
        conv(std::true_type{}, std::false_type{}, 2 * blk + 1);
      }
    }
  }
  dep_heads<MK, 1>(p, smem, legal, policy, value, wdl, b, 0, true, lane);
}

// Four waves evaluate the workgroup's BPG boards (1 or 2).  Wave w owns every square
// block of channel block w (0..3) and a share of channel block 4: with two boards
// square block w, with one (two blocks) waves 0 and 1 have one each.  NBUF: weight
// ring in groups, SR: the stem's in steps.  Measured (us, NBUF 3 / 5): int8 one
// board 141 / 140, bf16 one board 204 / 207, two boards 294 / 299.
template <int MK, int BPG, int NBUF, int SR>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(1, 1))) void
az_dep_kernel(AzDevNet p, const float* __restrict__ planes, const uint8_t* __restrict__ legal, int B,
              float* __restrict__ policy, float* __restrict__ value, float* __restrict__ wdl) {
  using C = DepCfg<MK, BPG>;
  using T = typename C::T;
  using GT = typename C::GT;
  using GS = typename C::GS;
  using frag_t = typename T::frag;
  using acc_t = typename T::acc;
  constexpr bool QUANT = C::QUANT;
  constexpr int OFF_H = C::OFF_H, OFF_T = C::OFF_T, NBK = GT::NBK;
  constexpr int NWV = 4, NT = 64 * NWV;
  static_assert(DNMB == NWV + 1, "four waves, five channel blocks");
  static_assert(BPG == 1 || BPG == 2, "boards per workgroup");

  __shared__ __attribute__((aligned(16))) uint8_t smem[C::SMEM];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int b0 = blockIdx.x * BPG;
  const int Cin = p.in_planes;
  const float cap = p.act_cap;
  // this lane's column of a square block: place v in a row, first row r0
  const int lv = l32 % (8 * BPG), lr0 = l32 / (8 * BPG) * NBK;

  // ---- ingest: zero pads, planes -> bf16 [square][64 channels] at OFF_T.  The T
  // buffer's own pads, some inside the stem input, are cleared after the stem.
  auto zero_pads = [&](auto geo, int off) {
    using G = decltype(geo);
    constexpr int PC = G::ZP / 16;
    for (int i = tid; i < 8 * PC; i += NT)
      *reinterpret_cast<i32x4*>(smem + off + i / PC * G::RS + G::PAD + i % PC * 16) = i32x4{0, 0, 0, 0};
  };
  zero_pads(GT{}, OFF_H);
  zero_pads(GS{}, OFF_T);
  {
    // item = planes 8k..8k+7 of one board: lane = square, eight coalesced loads,
    // one 16-byte store; unconditional loads (clamped to plane 0 of board 0)
    constexpr int KI = DCP / 8, ITEMS = BPG * KI, PER = ITEMS / NWV;
    static_assert(ITEMS % NWV == 0, "ingest items per wave");
    float pv[PER][8];
#pragma unroll
    for (int it = 0; it < PER; ++it)
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int item = wave + NWV * it, b = b0 + item / KI, c = 8 * (item % KI) + t;
        const bool ok = b < B && c < Cin;
        const float x = planes[ok ? ((size_t)b * Cin + c) * 64 + lane : (size_t)lane];
        pv[it][t] = ok ? x : 0.0f;
      }
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int item = wave + NWV * it;
      *reinterpret_cast<uint4*>(smem + OFF_T + GS::at(lane >> 3, item / KI, lane & 7) + 16 * (item % KI)) =
          make_uint4(pack_bf16x2(pv[it][0], pv[it][1]), pack_bf16x2(pv[it][2], pv[it][3]),
                     pack_bf16x2(pv[it][4], pv[it][5]), pack_bf16x2(pv[it][6], pv[it][7]));
    }
  }

  // tower weight stream, read through a buffer resource: the lane's offsets (its
  // own block, and block 4) are constant VGPRs and a fragment's byte offset a
  // scalar, so the loads cost no vector address arithmetic.  Group g of a layer
  // (the three dy of one (dx, channel step)) lives in ring slot g % NBUF, loaded
  // NBUF - 1 groups ahead, across layers.
  const __amdgpu_buffer_rsrc_t twr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.tower_w), (short)0, (int)(2 * p.blocks * C::LAYER_BYTES), 0x00020000);
  const int tvoff = (wave * 64 + lane) * T::FB, tvoffx = ((DNMB - 1) * 64 + lane) * T::FB;
  // per-layer epilogue constants of conv index k (0 = stem), one 16-byte chunk per
  // thread, loaded at the start of a layer and parked in LDS before its barrier
  constexpr int KV = C::KSLOT / 16;
  static_assert(KV <= NT, "constant staging");
  auto load_consts = [&](int k) -> float4 {
    if (tid >= KV) return make_float4(0.f, 0.f, 0.f, 0.f);
    const void* src;
    if constexpr (QUANT)
      src = tid < DF / 2 ? p.qbias + (size_t)k * DF + 2 * tid
            : tid < DF   ? p.qmul + (size_t)k * DF + 2 * (tid - DF / 2)
                         : p.qext + 2 * (size_t)k;
    else src = p.bias + (size_t)k * DF + 4 * tid;
    return *reinterpret_cast<const float4*>(src);
  };
  auto store_consts = [&](int slot, const float4& v) {
    if (tid < KV) *reinterpret_cast<float4*>(smem + C::OFF_K + slot * C::KSLOT + 16 * tid) = v;
  };
  // head constants, staged once: embedding row scale and bias, query and key biases
  {
    float* hc = reinterpret_cast<float*>(smem + C::OFF_HC);
    if (tid < AZ_DEP_EMB_ROWS) {
      hc[tid] = p.emb_sc[tid];
      hc[AZ_DEP_EMB_ROWS + tid] = p.emb_bc[tid];
    }
    if (tid < DD) {
      hc[2 * AZ_DEP_EMB_ROWS + tid] = p.q_b[tid];
      hc[2 * AZ_DEP_EMB_ROWS + DD + tid] = p.k_b[tid];
    }
  }
  store_consts(0, load_consts(1));

  // ---- stem and tower of one wave.  XB: its square blocks of channel block 4 (the
  // second tile set); with one board XN is that block's index, else the blocks are
  // wave * XB ..  Every wave meets the same sequence of workgroup barriers.
  auto trunk = [&](auto xb_c, auto xn_c) {
    constexpr int XB = decltype(xb_c)::value, XN = decltype(xn_c)::value;
    constexpr int NAF = XB > 0 ? 2 : 1;  // weight fragments per K step
    constexpr int XBn = XB > 0 ? XB : 1;
    const int xfirst = BPG == 1 ? XN : wave * XB;
    // lane rows of the second set's fragments of one horizontal tap (several boards):
    // blocks xfirst - 1, xfirst .., xfirst + XB
    struct XRows { int lo, mid, hi; };
    auto x_rows = [&](const auto& t) {
      using G = typename std::decay_t<decltype(t)>::G;
      XRows r;
      r.mid = t.row + xfirst * G::RS;
      r.lo = xfirst == 0 ? t.lo : r.mid - G::RS;
      r.hi = xfirst + XBn == NBK ? t.hi : r.mid + XBn * G::RS;
      return r;
    };

    // residual stream of the boards (bf16 networks): h = hi + lo, hi = bf16(h) in
    // the H buffer (the convolution operand), lo = bf16(h - hi) packed here, two
    // per register: [square block][run of 4 channels][2]
    uint32_t rlo[QUANT ? 1 : NBK][QUANT ? 1 : 8], rlox[QUANT ? 1 : XBn][QUANT ? 1 : 8];

    // B fragments of one (dx, channel step): every block's, and the second set's
    // with several boards (its blocks differ by wave, so they have no fixed place
    // among the first)
    constexpr bool XF = XB > 0 && BPG > 1;
    auto load_x = [&](const auto& t, const XRows& xr, const uint8_t* buf, int cs, auto& x, auto& xx) {
      using G = typename std::decay_t<decltype(t)>::G;
      using Frag = std::decay_t<decltype(x[0])>;
      static_for<0, G::NX>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        x[i] = t.template get<Frag, i - G::X0>(buf, cs);
      });
      if constexpr (XF) {
        xx[0] = *reinterpret_cast<const Frag*>(buf + xr.lo + 32 * cs);
#pragma unroll
        for (int k = 0; k < XB; ++k) xx[1 + k] = *reinterpret_cast<const Frag*>(buf + k * G::RS + xr.mid + 32 * cs);
        xx[1 + XB] = *reinterpret_cast<const Frag*>(buf + xr.hi + 32 * cs);
      }
    };
    // every product of one (dx, channel step), each accumulator in the order of dy
    auto products = [&](auto mk_c, auto first_c, const auto& a, const auto& x, const auto& xx, auto& acc, auto& accx) {
      using M = Mk<decltype(mk_c)::value>;
      constexpr bool FIRST = decltype(first_c)::value;
      constexpr int X0 = GT::X0, NX = GT::NX;
      static_for<0, 3>([&](auto d_c) {
        constexpr int d = decltype(d_c)::value;
        static_for<0, NBK>([&](auto j_c) {
          constexpr int j = decltype(j_c)::value, xi = j + d - 1 + X0;
          if constexpr (xi >= 0 && xi < NX) {
            constexpr bool zero = FIRST && (d == 0 || (X0 == 0 && d == 1 && j == 0));
            acc[j] = M::mma(a[d][0], x[xi], zero ? typename M::acc{} : acc[j]);
          }
        });
        if constexpr (XB > 0) {
#pragma unroll
          for (int k = 0; k < XB; ++k) {
            constexpr int xn = XN + (GT::X0 - 1);
            if constexpr (XF) accx[k] = M::mma(a[d][NAF - 1], xx[k + d], FIRST && d == 0 ? typename M::acc{} : accx[k]);
            else accx[k] = M::mma(a[d][NAF - 1], x[xn + d], FIRST && d == 0 ? typename M::acc{} : accx[k]);
          }
        }
      });
    };
    constexpr int NXX = XF ? XB + 2 : 1;
    constexpr int NMF = 3 * NBK - (GT::EDGE ? 0 : 2) + 3 * XB, NDS = GT::NX + (XF ? XB + 2 : 0), NVM = 3 * NAF;
    auto interleave = [&](auto lds_c, auto vm_c) {
      // each MFMA is followed by one of the next step's LDS reads, then by one of
      // the prefetched group's weight loads; a step is one scheduling region
      constexpr bool LDS = decltype(lds_c)::value, VM = decltype(vm_c)::value;
      static_for<0, NMF>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (LDS && i < NDS) __builtin_amdgcn_sched_group_barrier(0x100, i + 1 == NMF ? NDS - i : 1, 0);
        if constexpr (VM && i < NVM) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      });
      __builtin_amdgcn_sched_barrier(0);
    };
    // the lane's coordinates in the epilogues, opaque to the compiler in every layer:
    // hoisted out of the block loop, the epilogues' addresses would spill
    int elh = lhi, elv = lv, elr = lr0;
    // first channel of run q (four channels 8q + 4 lhi ..) of tile set m
    auto ch_of = [&](int m, int q) { return (m == 0 ? wave : DNMB - 1) * 32 + 8 * q + 4 * elh; };
    // LDS address of a run of square block n
    auto run_addr = [&](int off, int ch0, int n) { return off + (elr + n) * GT::RS + elv * GT::CS + ch0 * T::ES; };

    frag_t A[NBUF][3][NAF];
    auto load_group = [&](frag_t(&dst)[3][NAF], int soff) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int o = soff + d * DNMB * 64 * T::FB;
        dst[d][0] = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(twr, tvoff, o, 0));
        if constexpr (NAF > 1) dst[d][1] = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(twr, tvoffx, o, 0));
      }
    };

    // ---- stem: bf16 3x3 conv over 64 (padded) input channels.  Its fp32 sums run
    // in the order (dy, dx, channel step): the unnormalised count planes round in
    // them, and another order moves a stem code in about every second batch of
    // 1,024.  36 K steps, each reading its own fragments (4% of the products).
    {
      constexpr int CS4 = DCP / 16, SN = 9 * CS4;
      const uint8_t* sw8 = static_cast<const uint8_t*>(p.stem_w) + (size_t)lane * 16;
      // A fragments in a ring of SR steps, the first ones loaded before the barrier
      bf16x8 a[SR][NAF];
      auto load_a = [&](int st) {
        const int tap = st / CS4, f = (tap % 3 * CS4 + st % CS4) * 3 + tap / 3;
#pragma unroll
        for (int m = 0; m < NAF; ++m)
          a[st % SR][m] = g_frag<MK_BF16>(sw8 + (f * DNMB + (m == 0 ? wave : DNMB - 1)) * 64 * 16);
      };
#pragma unroll
      for (int st = 0; st < SR - 1; ++st) load_a(st);
      __syncthreads();  // the ingest's planes and constants are in LDS
      f32x16 sacc[NBK], saccx[XBn];
      bf16x8 x[NBK], xx[XBn], xn[NBK], xxn[XBn];
      auto load_s = [&](auto st_c, auto& d0, auto& d1) {
        constexpr int st = decltype(st_c)::value, dx = st / CS4 % 3, dy = st / CS4 / 3 - 1, cs = st % CS4;
        DTaps<2 * DCP, BPG> t;
        t.init(dx - 1, l32, lhi);
        const uint8_t* buf = smem + OFF_T;
        static_for<0, NBK>([&](auto j_c) {
          constexpr int j = decltype(j_c)::value;
          d0[j] = t.template get<bf16x8, j + dy>(buf, cs);
        });
        if constexpr (XB > 0 && BPG == 1) d1[0] = t.template get<bf16x8, XN + dy>(buf, cs);
        if constexpr (XF) {
          const XRows xr = x_rows(t);
#pragma unroll
          for (int k = 0; k < XB; ++k) {
            const int r = k + dy < 0 ? xr.lo : k + dy >= XB ? xr.hi : xr.mid + (k + dy) * GS::RS;
            d1[k] = *reinterpret_cast<const bf16x8*>(buf + r + 32 * cs);
          }
        }
      };
      load_s(std::integral_constant<int, 0>{}, x, xx);
      static_for<0, SN>([&](auto st_c) {
        constexpr int st = decltype(st_c)::value;
        if constexpr (st + SR - 1 < SN) load_a(st + SR - 1);
        if constexpr (st + 1 < SN) load_s(std::integral_constant<int, st + 1>{}, xn, xxn);
#pragma unroll
        for (int j = 0; j < NBK; ++j) sacc[j] = mma_bf16(a[st % SR][0], x[j], st == 0 ? f32x16{} : sacc[j]);
#pragma unroll
        for (int k = 0; k < XB; ++k) saccx[k] = mma_bf16(a[st % SR][NAF - 1], xx[k], st == 0 ? f32x16{} : saccx[k]);
        if constexpr (st + 1 < SN) {
#pragma unroll
          for (int j = 0; j < NBK; ++j) x[j] = xn[j];
#pragma unroll
          for (int k = 0; k < XBn; ++k) xx[k] = xxn[k];
        }
        if constexpr (st % CS4 == CS4 - 1) __builtin_amdgcn_sched_barrier(0);
      });
      // the tower's first weight groups, in flight during the stem's epilogue
      static_for<0, NBUF - 1>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        load_group(A[i], i * C::GROUP_BYTES);
      });
      // epilogue: bias, activation (codes for int8), store in the tower format at OFF_H
      auto put = [&](int m, int q, int n, const f32x16& v, uint32_t(&rl)[QUANT ? 1 : 8], const float4& bb,
                     const double(&mq)[4], const double(&bq)[4]) {
        const int addr = run_addr(OFF_H, ch_of(m, q), n);
        if constexpr (!QUANT) {
          const float y0 = act_fn(v[4 * q + 0] + bb.x, cap), y1 = act_fn(v[4 * q + 1] + bb.y, cap);
          const float y2 = act_fn(v[4 * q + 2] + bb.z, cap), y3 = act_fn(v[4 * q + 3] + bb.w, cap);
          rl[2 * q + 0] = pack_bf16x2(y0 - bf16_round(y0), y1 - bf16_round(y1));
          rl[2 * q + 1] = pack_bf16x2(y2 - bf16_round(y2), y3 - bf16_round(y3));
          *reinterpret_cast<uint2*>(smem + addr) = make_uint2(pack_bf16x2(y0, y1), pack_bf16x2(y2, y3));
        } else {
          // fp32 sum of the bf16 matrix instruction; rescale and rounding in float64
          *reinterpret_cast<uint32_t*>(smem + addr) =
              pack_codes_d<MK>(__builtin_fma((double)v[4 * q + 0], mq[0], bq[0]),
                               __builtin_fma((double)v[4 * q + 1], mq[1], bq[1]),
                               __builtin_fma((double)v[4 * q + 2], mq[2], bq[2]),
                               __builtin_fma((double)v[4 * q + 3], mq[3], bq[3]), p.qhi[0]);
        }
      };
#pragma unroll
      for (int m = 0; m < NAF; ++m)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int ch0 = ch_of(m, q);
          const float4 bb = *reinterpret_cast<const float4*>(p.bias + ch0);
          double mq[4] = {}, bq[4] = {};
          if constexpr (QUANT) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              mq[r] = p.qmul[ch0 + r];
              bq[r] = p.qbias[ch0 + r];
            }
          }
          if (m == 0) {
#pragma unroll
            for (int n = 0; n < NBK; ++n) put(m, q, n, sacc[n], rlo[QUANT ? 0 : n], bb, mq, bq);
          } else {
#pragma unroll
            for (int k = 0; k < XB; ++k) put(m, q, xfirst + k, saccx[k], rlox[QUANT ? 0 : k], bb, mq, bq);
          }
        }
    }
    __syncthreads();
    zero_pads(GT{}, OFF_T);  // read after the first layer's barrier

    // ---- residual tower
    {
      constexpr int CPT = C::CPT;
      acc_t c[NBK], cx[XBn];
      const int nconv = 2 * p.blocks;
      DTaps<C::RB, BPG> taps[3];
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) taps[dx].init(dx - 1, l32, lhi);

      // pool (wave-uniform): the layer is in a pooling block.  One code for both kinds
      // of block: the four kinds of layer unrolled would pass the instruction cache.
      auto conv = [&](auto second_c, int n_conv, bool pool) {
        constexpr bool SECOND = decltype(second_c)::value;
        constexpr int NS = C::NS;
        static_assert(NS % NBUF == 0, "every layer starts at ring slot 0");
        const int wl = n_conv * (int)C::LAYER_BYTES;  // byte offset of the layer in the stream
        const bool has_next = n_conv + 1 < nconv;
        constexpr int in_off = SECOND ? OFF_T : OFF_H;
        constexpr int out_off = SECOND ? OFF_H : OFF_T;
        uint8_t* kslot = smem + C::OFF_K + (n_conv & 1) * C::KSLOT;
        // the next layer's epilogue constants, in flight during this layer
        const float4 kn = has_next ? load_consts(n_conv + 2) : make_float4(0.f, 0.f, 0.f, 0.f);
        // a pooling layer's projection weights: thread t's output t % 128, all 2g
        // inputs as [i/4] float4s; with one board in flight during the K loop
        constexpr int NWP = SECOND ? 1 : 2 * DG / 4;
        const int po = tid & 127;
        float4 wpool[NWP];
        auto load_pool = [&]() {
          const float4* wt = reinterpret_cast<const float4*>(p.pool_wt) +
                             (size_t)(n_conv / 2 / p.pool_every) * (2 * DG / 4) * AZ_DEP_POOL_OPAD + po;
#pragma unroll
          for (int i4 = 0; i4 < NWP; ++i4) wpool[i4] = wt[(size_t)i4 * AZ_DEP_POOL_OPAD];
        };
        if constexpr (!SECOND && BPG == 1) {
          if (pool) load_pool();
        }
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) taps[dx].opaque();
        asm volatile("" : "+v"(elh), "+v"(elv), "+v"(elr));
        XRows xr[3];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) xr[dx] = x_rows(taps[dx]);

        frag_t x[GT::NX], xx[NXX], xn[GT::NX], xxn[NXX];
        auto load_s = [&](auto s_c, auto& d0, auto& d1) {
          constexpr int s = decltype(s_c)::value;
          load_x(taps[s / CPT], xr[s / CPT], smem + in_off, s % CPT, d0, d1);
        };
        load_s(std::integral_constant<int, 0>{}, x, xx);
        static_for<0, NS>([&](auto s_c) {
          constexpr int s = decltype(s_c)::value, gi = s + NBUF - 1;
          // group s + NBUF-1 of this layer, or of the next one past its end; past the
          // network's last layer this layer is re-read and never used
          if constexpr (gi < NS) load_group(A[gi % NBUF], wl + gi * C::GROUP_BYTES);
          else load_group(A[gi % NBUF], has_next ? wl + (int)C::LAYER_BYTES + (gi - NS) * C::GROUP_BYTES : wl);
          if constexpr (s + 1 < NS) load_s(std::integral_constant<int, s + 1>{}, xn, xxn);
          // the second convolution of a pooling block has zero weights for the pooled
          // channels: its steps past the last regular one only pass the ring on
          constexpr bool REGULAR = !SECOND || s % CPT * T::KS < DFR;
          if (REGULAR || !pool) {
            products(std::integral_constant<int, MK>{}, std::integral_constant<bool, s == 0>{}, A[s % NBUF], x, xx, c, cx);
            interleave(std::integral_constant<bool, (REGULAR && s + 1 < NS)>{}, std::integral_constant<bool, REGULAR>{});
          }
          if constexpr (s + 1 < NS) {
#pragma unroll
            for (int i = 0; i < GT::NX; ++i) x[i] = xn[i];
#pragma unroll
            for (int i = 0; i < NXX; ++i) xx[i] = xxn[i];
          }
        });

        // global pooling: per board the pooled channels' mean and maximum, projected
        // to a context term that joins the regular channels' bias (OFF_PB)
        if constexpr (!SECOND) {
         if (pool) {
          if constexpr (BPG > 1) load_pool();
          // (1) the pooled channels to LDS as [board][pooled channel][square] in the T
          //     buffer (written by this layer's epilogue only afterwards); rows of
          //     256 bytes with 16-byte chunks XOR-swizzled by the row.  int8: the
          //     exact accumulators, activated in float64 in (2); bf16: act(acc + b1)
          float* pt = reinterpret_cast<float*>(smem + OFF_T);
          auto put_pool = [&](int m, int q, int n, const acc_t& v) {
            const int ch0 = ch_of(m, q);
            float4 bb = make_float4(0.f, 0.f, 0.f, 0.f);
            if constexpr (!QUANT) bb = *reinterpret_cast<const float4*>(kslot + 4 * ch0);
            const float bv[4] = {bb.x, bb.y, bb.z, bb.w};
            float* ptb = pt + (elv >> 3) * DG * 64;
            const int sq = (elr + n) * 8 + (elv & 7);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int pc = ch0 + r - DFR, idx = pc * 64 + (((sq >> 2) ^ (pc & 15)) << 2) + (sq & 3);
              if constexpr (QUANT) reinterpret_cast<int*>(ptb)[idx] = (int)v[4 * q + r];
              else ptb[idx] = med3(v[4 * q + r] + bv[r], 0.0f, cap);
            }
          };
          constexpr int Q0 = (DFR - 32 * (DNMB - 2)) / 8;  // block 3's first pooled run
          if (wave == DNMB - 2) {
#pragma unroll
            for (int q = Q0; q < 4; ++q)
#pragma unroll
              for (int n = 0; n < NBK; ++n) put_pool(0, q, n, c[n]);
          }
          if constexpr (XB > 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int k = 0; k < XB; ++k) put_pool(1, q, xfirst + k, cx[k]);
          }
          wave_lds_sync();
          // (2) thread r < BPG * g: board sum (fp64) and maximum of row r; statistics
          //     [mean g | max g] per board
          double* pg = reinterpret_cast<double*>(smem + C::OFF_PG);
          static_assert(BPG * DG <= NT, "a thread per pooled row");
          // with one board ten rows per wave, else in thread order
          const int pr = BPG == 1 ? (lane < DG / 4 ? (DG / 4) * wave + lane : DG) : tid;
          if (pr < BPG * DG) {
            const int bd = pr / DG, pc = pr % DG;
            const double2 mx_sum = pool_row<QUANT>(p, pt + bd * DG * 64, pc, n_conv);
            pg[bd * 2 * DG + pc] = mx_sum.y * (1.0 / 64.0);
            pg[bd * 2 * DG + DG + pc] = mx_sum.x;
          }
          wave_lds_sync();
          // (3) c[o] = sum_i Wg[o][i] g[i] in fp64 (fp32 weights are exact): thread
          //     t takes output t % 128 of board t / 128; the pooled channels keep
          //     their bias (their codes are read by nothing)
          {
            const int bd = tid >> 7;
            if (bd < BPG) {
              const double* gi = pg + bd * 2 * DG;
              double co = 0.0;
#pragma unroll
              for (int i4 = 0; i4 < NWP; ++i4) {
                const float4 w = wpool[i4];
                co = __builtin_fma((double)w.x, gi[4 * i4 + 0], co);
                co = __builtin_fma((double)w.y, gi[4 * i4 + 1], co);
                co = __builtin_fma((double)w.z, gi[4 * i4 + 2], co);
                co = __builtin_fma((double)w.w, gi[4 * i4 + 3], co);
              }
              if constexpr (QUANT) {
                const double* kb = reinterpret_cast<const double*>(kslot);
                double* pb = reinterpret_cast<double*>(smem + C::OFF_PB) + bd * DF;
                pb[po] = po < DFR ? kb[po] + co * p.pool_cinv[n_conv] : kb[po];
                if (po < DF - 128) pb[128 + po] = kb[128 + po];
              } else {
                const float* kb = reinterpret_cast<const float*>(kslot);
                float* pb = reinterpret_cast<float*>(smem + C::OFF_PB) + bd * DF;
                pb[po] = po < DFR ? kb[po] + (float)co : kb[po];
                if (po < DF - 128) pb[128 + po] = kb[128 + po];
              }
            }
          }
          zero_pads(GT{}, OFF_T);  // (1) wrote over them
          wave_lds_sync();
         }
        }

        // epilogue: per run of 4 channels; LDS reads of constants (and residual codes
        // or hi parts, read in place) issued two runs ahead
        const uint8_t* kbias = !SECOND && pool ? smem + C::OFF_PB + (elv >> 3) * DF * C::KE : kslot;
        float hi = 0.0f;
        double rq = 0.0;
        if constexpr (QUANT) {
          const double* kd = reinterpret_cast<const double*>(kslot);
          hi = (float)kd[2 * DF + 1];
          rq = SECOND ? kd[2 * DF] : 0.0;
        }
        constexpr int NRUN = NAF * 4, EP_AHEAD = 2, EP_RING = EP_AHEAD + 1;
        constexpr int NMAX = cmax(NBK, XBn);
        struct KQ { double b[QUANT ? 4 : 1], m[QUANT ? 4 : 1]; float4 f; };
        KQ kq[EP_RING];
        using rin_t = std::conditional_t<QUANT, uint32_t, uint2>;  // codes, or hi parts
        rin_t rin[SECOND ? EP_RING : 1][SECOND ? NMAX : 1];
        auto ep_load = [&](auto k_c) {
          constexpr int k = decltype(k_c)::value, m = k / 4, q = k % 4, slot = k % EP_RING;
          const int ch0 = ch_of(m, q);
          if constexpr (QUANT) {
            const double* kb = reinterpret_cast<const double*>(kbias);
            const double* kd = reinterpret_cast<const double*>(kslot);
#pragma unroll
            for (int r = 0; r < 4; r += 2) {
              const double2 b2 = *reinterpret_cast<const double2*>(kb + ch0 + r);
              const double2 m2 = *reinterpret_cast<const double2*>(kd + DF + ch0 + r);
              kq[slot].b[r] = b2.x;
              kq[slot].b[r + 1] = b2.y;
              kq[slot].m[r] = m2.x;
              kq[slot].m[r + 1] = m2.y;
            }
          } else {
            kq[slot].f = *reinterpret_cast<const float4*>(kbias + 4 * ch0);
          }
          if constexpr (SECOND) {
#pragma unroll
            for (int n = 0; n < (m == 0 ? NBK : XB); ++n) {
              const uint8_t* a = smem + run_addr(out_off, ch0, m == 0 ? n : xfirst + n);
              rin[slot][n] = *reinterpret_cast<const rin_t*>(a);
            }
          }
        };
        auto ep_run = [&](int q, const KQ& kk, const acc_t& v, int addr, rin_t hv, uint32_t(&rl)[QUANT ? 1 : 8]) {
          if constexpr (!QUANT) {
            float y0 = v[4 * q + 0] + kk.f.x, y1 = v[4 * q + 1] + kk.f.y;
            float y2 = v[4 * q + 2] + kk.f.z, y3 = v[4 * q + 3] + kk.f.w;
            if constexpr (SECOND) {
              // block input h = hi + lo (exact in fp32)
              const uint32_t l01 = rl[2 * q], l23 = rl[2 * q + 1];
              y0 = act_fn(y0 + (__uint_as_float(hv.x << 16) + __uint_as_float(l01 << 16)), cap);
              y1 = act_fn(y1 + (__uint_as_float(hv.x & 0xffff0000u) + __uint_as_float(l01 & 0xffff0000u)), cap);
              y2 = act_fn(y2 + (__uint_as_float(hv.y << 16) + __uint_as_float(l23 << 16)), cap);
              y3 = act_fn(y3 + (__uint_as_float(hv.y & 0xffff0000u) + __uint_as_float(l23 & 0xffff0000u)), cap);
              rl[2 * q + 0] = pack_bf16x2(y0 - bf16_round(y0), y1 - bf16_round(y1));
              rl[2 * q + 1] = pack_bf16x2(y2 - bf16_round(y2), y3 - bf16_round(y3));
            } else {
              y0 = act_fn(y0, cap);
              y1 = act_fn(y1, cap);
              y2 = act_fn(y2, cap);
              y3 = act_fn(y3, cap);
            }
            *reinterpret_cast<uint2*>(smem + addr) = make_uint2(pack_bf16x2(y0, y1), pack_bf16x2(y2, y3));
          } else {
            // float64 requantisation: z = acc * qmul + qbias (+ residual code * qres)
            double z[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) z[r] = __builtin_fma((double)v[4 * q + r], kk.m[r], kk.b[r]);
            if constexpr (SECOND) {
              z[0] = __builtin_fma(code_value_d<MK, 0>(hv), rq, z[0]);
              z[1] = __builtin_fma(code_value_d<MK, 1>(hv), rq, z[1]);
              z[2] = __builtin_fma(code_value_d<MK, 2>(hv), rq, z[2]);
              z[3] = __builtin_fma(code_value_d<MK, 3>(hv), rq, z[3]);
            }
            *reinterpret_cast<uint32_t*>(smem + addr) = pack_codes_d<MK>(z[0], z[1], z[2], z[3], hi);
          }
        };
        static_for<0, EP_AHEAD>([&](auto k_c) { ep_load(k_c); });
        static_for<0, NRUN>([&](auto k_c) {
          constexpr int k = decltype(k_c)::value, m = k / 4, q = k % 4, slot = k % EP_RING;
          if constexpr (k + EP_AHEAD < NRUN) ep_load(std::integral_constant<int, k + EP_AHEAD>{});
          const int ch0 = ch_of(m, q);
          if constexpr (m == 0) {
#pragma unroll
            for (int n = 0; n < NBK; ++n)
              ep_run(q, kq[slot], c[n], run_addr(out_off, ch0, n), SECOND ? rin[SECOND ? slot : 0][SECOND ? n : 0] : rin_t{},
                     rlo[QUANT ? 0 : n]);
          } else {
#pragma unroll
            for (int n = 0; n < XB; ++n)
              ep_run(q, kq[slot], cx[n], run_addr(out_off, ch0, xfirst + n),
                     SECOND ? rin[SECOND ? slot : 0][SECOND ? n : 0] : rin_t{}, rlox[QUANT ? 0 : n]);
          }
        });
        if (has_next) store_consts((n_conv + 1) & 1, kn);
        __syncthreads();
      };

      for (int blk = 0; blk < p.blocks; ++blk) {
        const bool pool = p.pool_every > 0 && blk % p.pool_every == p.pool_every - 1;
        conv(std::false_type{}, 2 * blk, pool);
        conv(std::true_type{}, 2 * blk + 1, pool);
      }
    }

    // ---- heads input (bf16 networks): the low part h - bf16(h) of the residual in
    // the tower's layout at OFF_X, H holding bf16(h); int8 networks read the final
    // codes from H and convert them in registers
    if constexpr (!QUANT) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int n = 0; n < NBK; ++n)
          *reinterpret_cast<uint2*>(smem + run_addr(C::OFF_X, ch_of(0, q), n)) = make_uint2(rlo[n][2 * q], rlo[n][2 * q + 1]);
#pragma unroll
        for (int k = 0; k < XB; ++k)
          *reinterpret_cast<uint2*>(smem + run_addr(C::OFF_X, ch_of(1, q), xfirst + k)) =
              make_uint2(rlox[k][2 * q], rlox[k][2 * q + 1]);
      }
    }
  };
  using std::integral_constant;
  if constexpr (BPG > 1) {
    trunk(integral_constant<int, NBK / NWV>{}, integral_constant<int, 0>{});
  } else {
    if (wave == 0) trunk(integral_constant<int, 1>{}, integral_constant<int, 0>{});
    else if (wave == 1) trunk(integral_constant<int, 1>{}, integral_constant<int, 1>{});
    else trunk(integral_constant<int, 0>{}, integral_constant<int, 0>{});
  }
  __syncthreads();
  // ---- heads: one board shared by the four waves, or a wave per board
  if constexpr (BPG == 1) {
    dep_heads4<MK>(p, smem, legal, policy, value, wdl, b0, wave, lane);
  } else {
    dep_heads<MK, BPG>(p, smem, legal, policy, value, wdl, b0 + wave, wave, wave < BPG && b0 + wave < B, lane);
  }
}

template <int MK, int BPG, int NBUF, int SR>
hipError_t launch_dep(const AzDevNet& n, const float* planes, const uint8_t* legal, int B, float* policy, float* value,
                      float* wdl, hipStream_t s) {
  (void)hipGetLastError();
  if (n.filters != DF || B <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL((az_dep_kernel<MK, BPG, NBUF, SR>), dim3((B + BPG - 1) / BPG), dim3(256), 0, s, n, planes, legal, B,
                     policy, value, wdl);
  return hipGetLastError();
}

}  // namespace
