// Fused policy/value network evaluation in fp32 (AZ_F32), on the bf16 matrix
// cores.
//
// Every fp32 operand x is the exact sum of three bf16 parts, x = h + m + l with
// h = bf16(x), m = bf16(x - h), l = x - h - m (8 + 8 + 8 significant bits), and a
// product w * x is taken as the six part products of weight 2^-16 or more: hw hx
// into one fp32 accumulator, lw hx, hw lx, mw mx, mw hx and hw mx into another.
// Each is exact in fp32.  What is left out, m l + l m + l l of parts of at most
// 2^-8 (m) and 2^-17 (l) of their operand's power of two, is at most 2^-24 of the
// product (random operands in [1, 2) reach 2^-24.3): about the rounding of one fp32
// multiply-add.  The sums gain: the leading accumulator is rounded once per 32
// channels where the multiply-add chain was once per channel.  Operands below 2^-110
// lose low bits of l to bf16's range, and a sum whose leading products overflow is
// infinite within 2^-8 of the largest float.  Distance from float64 (2-norm, policy /
// value; in brackets fp32 multiply-adds on the vector
// ALUs, which this replaces): 2x32 1.3e-7 / 2.1e-7 (3.6e-7 / 4.1e-7), 20x128 3.2e-7 /
// 9.2e-7 (7.3e-7 / 2.3e-6), 2x256 2.0e-7 / 5.6e-7 (5.9e-7 / 1.2e-6).  With all six
// in one accumulator it was no better than the chain.  The bf16 instruction runs at
// 16 times the rate of the fp32 one, so six products cost 0.38 of it.
//
// One workgroup of eight waves (two per SIMD, to cover each other's latencies)
// evaluates one board.  A convolution is an implicit GEMM of 16x16 blocks: 16
// output channels by 16 squares, block b = rows b and b + 4 of the board, so that
// the LDS fragments of one horizontal tap and channel step serve all three
// vertical taps (block b's neighbour rows are block b +- 1).  A wave owns MB
// channel blocks x NB square blocks, chosen so that one pass covers the layer:
// 1 x 1 up to 16 filters, 1 x 2 up to 64, 1 x 4 up to 128, 2 x 4 up to 256 (32
// filters: 1 x 1 20.7 us, 1 x 2 19.3 us; 64: 1 x 2 33 us, 1 x 4 36 us: the waves that
// share a channel block each stream its weights through the L1).  The 2 x 4 tile does
// not fit the 256 registers two waves a SIMD leave each: 53 of them spill, 216 bytes
// of scratch a lane, on every network above 128 filters.
//
// LDS holds one activation buffer: [square slot][part h, m, l][channel].  Slots
// are 9 to a row with zero rows above and below the board and one zero column
// between rows, so no tap needs a bounds check; a slot is an odd number of
// 16-byte units.  A layer keeps its outputs in registers until every wave has
// read the buffer, then overwrites it; the residual stream stays in registers in
// fp32.  Weights stream from L2 through a ring of the three vertical taps.
//
// What bounds it: the six products (27.6k MFMA cycles a 128-filter convolution on
// the one compute unit a board has, 0.46 ms for 20x128) and, on small networks, the
// latency of the layers' chain.  20x128, 64 boards: 13.5 ms -> 0.68 ms; 2x32, 16
// boards: 102 -> 19.3 us; 1,024 boards: 355 -> 78 us; 2x256, 16 boards: 5.7 -> 0.27 ms.
#include "az_internal.h"
#include "az_mfma_common.h"

#include <float.h>
#include <math.h>

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int NW = 8, NT = 64 * NW;
constexpr int SLOTS = 91;  // (8 + 2) rows x 9 columns, and the last row's right neighbour
constexpr int CELLS = AZ_MAX_POLICY * 64;

struct Split { bf16x8 h, m, l; };

// x = h + m + l; a finite x that rounds past the largest bf16 takes that as its h.
// Of a non-finite x, h is x and the others are zero.
__device__ __forceinline__ void split3(float x, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = bf16_bits(x);
  const bool finite = fabsf(x) < INFINITY;
  if (finite && (h & 0x7fffu) == 0x7f80u) --h;
  const float r = finite ? x - __uint_as_float(h << 16) : 0.0f;
  m = bf16_bits(r);
  l = bf16_bits(r - __uint_as_float(m << 16));
}
// The same for 0 <= x < BIG.
constexpr float BIG = 0x1.fep127f;  // the largest bf16
__device__ __forceinline__ void split3_small(float x, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = bf16_bits(x);
  const float r = x - __uint_as_float(h << 16);
  m = bf16_bits(r);
  l = bf16_bits(r - __uint_as_float(m << 16));
}

__device__ __forceinline__ f32x4 mma16(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// A X over one K step of 32: the leading product into c, the others, at most
// 2^-7 of it, into an accumulator of their own
__device__ __forceinline__ void mma_split(const Split& a, const Split& x, f32x4& c, f32x4& small) {
  c = mma16(a.h, x.h, c);
  small = mma16(a.l, x.h, small);
  small = mma16(a.h, x.l, small);
  small = mma16(a.m, x.m, small);
  small = mma16(a.m, x.h, small);
  small = mma16(a.h, x.m, small);
}

// The sum of the two accumulators.  Where an operand or the sum is infinite the
// leading products alone give what a chain of multiply-adds gives; the small ones (a
// zero or negative part times the infinity) are infinite or NaN, and the median is
// then a finite value.
__device__ __forceinline__ float mma_sum(float c, float small) { return c + med3(small, -FLT_MAX, FLT_MAX); }

__device__ __forceinline__ bf16x8 frag_at(const uint8_t* p) { return *reinterpret_cast<const bf16x8*>(p); }

// Block-wide reduction of one value per thread (every thread gets the result);
// waves are combined in order.
__device__ __forceinline__ float block_reduce(float v, bool is_max, float* scratch) {
  v = is_max ? wave_max(v) : wave_sum(v);
  if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = scratch[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) r = is_max ? fmaxf(r, scratch[i]) : r + scratch[i];
  return r;
}

// LDS: activations [SLOTS][3][Fp] bf16 + 16 bytes a slot (logits overlay them after
// the tower) | scratch
template <int MB, int NB>
__global__ __launch_bounds__(NT) void az_net_f32_kernel(AzDevNet p, const float* __restrict__ planes,
                                                        const uint8_t* __restrict__ legal,
                                                        float* __restrict__ policy, float* __restrict__ value,
                                                        int scratch_off) {
  extern __shared__ __attribute__((aligned(16))) uint8_t sm[];
  const int F = p.filters, Cin = p.in_planes, P = p.policy_planes, H = p.value_hidden;
  const int M16 = (F + 15) / 16, CP = (F + 31) / 32;  // output channel blocks, input channel steps
  const int RB = CP * 64, CS = 3 * RB + 16, RS = 9 * CS;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = lane >> 4, col = lane & 7, hi4 = (lane >> 3) & 1;  // K quarter; column and half of a block's square
  constexpr int NU = 4 / NB;                                        // waves per channel block
  const int mb0 = w / NU * MB, nb0 = w % NU * NB;
  const bool busy = mb0 < M16;
  const float cap = p.act_cap;
  float* scratch = reinterpret_cast<float*>(sm + scratch_off);

  // weights: fragment (dx, channel step, dy, channel block, part) of 1 KB each.  A
  // wave whose second channel block is past the last one multiplies the last again
  // and drops it.
  Split A[3][MB];
  auto load_a = [&](const uint8_t* g, int d) {  // g: the (dx, channel step) group
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      const int mb = mb0 + m < M16 ? mb0 + m : M16 - 1;
      const uint8_t* q = g + ((size_t)(d * M16 + mb) * 3) * 1024 + lane * 16;
      A[d][m].h = frag_at(q);
      A[d][m].m = frag_at(q + 1024);
      A[d][m].l = frag_at(q + 2048);
    }
  };
  const size_t group = (size_t)9 * M16 * 1024;
  const uint8_t* sw = static_cast<const uint8_t*>(p.stem_w);
#pragma unroll
  for (int d = 0; d < 3; ++d) load_a(sw, d);

  // ---- ingest: clear the buffer (zero borders and padding channels), then the
  // input planes as channels 0..31 (eight planes of a square per wave item)
  float pv[8];
  if (w < 4) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int c = 8 * w + t;
      const float x = planes[((size_t)b * Cin + (c < Cin ? c : 0)) * 64 + lane];
      pv[t] = c < Cin ? x : 0.0f;
    }
  }
  for (int i = tid; i < SLOTS * CS / 16; i += NT) *reinterpret_cast<i32x4*>(sm + i * 16) = i32x4{0, 0, 0, 0};
  __syncthreads();
  if (w < 4) {
    uint32_t h[8], m[8], l[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) split3(pv[t], h[t], m[t], l[t]);
    uint8_t* dst = sm + (((lane >> 3) + 1) * 9 + (lane & 7) + 1) * CS + w * 16;
    auto put = [&](int part, const uint32_t(&v)[8]) {
      *reinterpret_cast<uint4*>(dst + part * RB) =
          make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16);
    };
    put(0, h);
    put(1, m);
    put(2, l);
  }
  __syncthreads();

  // ---- the stem and the residual convolutions
  const uint8_t* xb = sm + ((nb0 + 4 * hi4 + 1) * 9 + col + 1) * CS + kq * 16;  // block nb0, dx = 0
  float res[MB][NB][4];
  // cp channel steps; next: the following layer's first group
  auto conv = [&](const uint8_t* wl, int cp, const uint8_t* next, const float* bias, bool residual, bool last) {
    f32x4 acc[MB][NB], sml[MB][NB];
    float4 bb[MB];
    if (busy) {
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        bb[m] = make_float4(0.f, 0.f, 0.f, 0.f);
        const int ch = (mb0 + m) * 16 + 4 * kq;
        if (ch < F) bb[m] = *reinterpret_cast<const float4*>(bias + ch);  // F is a multiple of 8
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[m][n] = sml[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      const uint8_t* g = wl;
      for (int dx = 0; dx < 3; ++dx) {
        for (int cs = 0; cs < cp; ++cs) {
          g = dx == 2 && cs + 1 == cp ? next : g + group;
          Split X[NB + 2];  // blocks nb0 - 1 .. nb0 + NB
          const uint8_t* q = xb + (dx - 1) * CS + cs * 64 - RS;
#pragma unroll
          for (int x = 0; x < NB + 2; ++x) {
            X[x].h = frag_at(q + x * RS);
            X[x].m = frag_at(q + x * RS + RB);
            X[x].l = frag_at(q + x * RS + 2 * RB);
          }
#pragma unroll
          for (int d = 0; d < 3; ++d) {
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
              for (int n = 0; n < NB; ++n) mma_split(A[d][m], X[n + d], acc[m][n], sml[m][n]);
            load_a(g, d);  // the next group's, two vertical taps ahead
          }
        }
      }
    }
    __syncthreads();  // every wave has read the buffer
    if (busy) {
      float most = 0.0f;
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const float bv[4] = {bb[m].x, bb[m].y, bb[m].z, bb[m].w};
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float y = mma_sum(acc[m][n][r], sml[m][n][r]) + bv[r];
            if (residual) y += res[m][n][r];
            y = act_fn(y, cap);
            if (residual || last) res[m][n][r] = y;
            acc[m][n][r] = y;
            most = fmaxf(most, y);
          }
      }
      auto store = [&](auto split) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int n = 0; n < NB; ++n) {
            uint32_t h[4], md[4], l[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) split(acc[m][n][r], h[r], md[r], l[r]);
            if (mb0 + m < M16) {
              uint8_t* dst = sm + ((nb0 + n + 4 * hi4 + 1) * 9 + col + 1) * CS + (mb0 + m) * 32 + kq * 8;
              *reinterpret_cast<uint2*>(dst) = make_uint2(h[0] | h[1] << 16, h[2] | h[3] << 16);
              *reinterpret_cast<uint2*>(dst + RB) = make_uint2(md[0] | md[1] << 16, md[2] | md[3] << 16);
              *reinterpret_cast<uint2*>(dst + 2 * RB) = make_uint2(l[0] | l[1] << 16, l[2] | l[3] << 16);
            }
          }
      };
      // checked once for the wave's values, off the stores' path: a check in every
      // split costs 2 to 4% of the network
      store([](float x, uint32_t& h, uint32_t& m, uint32_t& l) { split3_small(x, h, m, l); });
      if (__builtin_expect(__any(most >= BIG), 0))
        store([](float x, uint32_t& h, uint32_t& m, uint32_t& l) { split3(x, h, m, l); });
    }
    __syncthreads();
  };
  // the heads' first weight step, in flight during the tower where the registers
  // allow
  constexpr bool EARLY = MB == 1 && NB <= 2;
  const int RBK = (P + 16) / 16, hrb0 = w >> 2;
  const uint8_t* hw = static_cast<const uint8_t*>(p.head_w) + lane * 16;
  Split ha[3];
  auto load_head = [&](int cs) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int rb = hrb0 + 2 * i < RBK ? hrb0 + 2 * i : RBK - 1;
      const uint8_t* a = hw + (size_t)(cs * RBK + rb) * 3 * 1024;
      ha[i] = Split{frag_at(a), frag_at(a + 1024), frag_at(a + 2048)};
    }
  };
  if constexpr (EARLY) load_head(0);
  const uint8_t* tw = static_cast<const uint8_t*>(p.tower_w);
  const size_t layer = (size_t)3 * CP * group;
  conv(sw, 1, tw, p.bias, false, true);
  if (M16 == 1 && tid < 64 * 3) {
    // one channel block: the stem input's channels 16..31 give way to zeros
    uint8_t* dst = sm + (((tid & 63) / 8 + 1) * 9 + (tid & 7) + 1) * CS + tid / 64 * RB + 32;
    *reinterpret_cast<i32x4*>(dst) = i32x4{0, 0, 0, 0};
    *reinterpret_cast<i32x4*>(dst + 16) = i32x4{0, 0, 0, 0};
  }
  if (M16 == 1) __syncthreads();
  for (int n = 0; n < 2 * p.blocks; ++n) {
    const uint8_t* wl = tw + n * layer;
    // past the last layer the last one's start is re-read (never used)
    conv(wl, CP, n + 1 < 2 * p.blocks ? wl + layer : wl, p.bias + (size_t)(n + 1) * F, n & 1, false);
  }

  // ---- heads: rows 0..P-1 policy planes, row P the value 1x1 conv.  Wave w takes
  // square block w % 4 and row blocks w / 4, w / 4 + 2, w / 4 + 4.  The legal mask
  // and fc1 (hidden unit tid) are in flight meanwhile.
  const int NM = P * 64;
  constexpr int UN = (CELLS / 4 + NT - 1) / NT;  // 4-cell units of a thread
  const uint8_t* lg = legal + (size_t)b * NM;
  uint32_t mk[UN];
#pragma unroll
  for (int i = 0; i < UN; ++i) {
    const int c = 4 * (tid + i * NT);
    const uint32_t x = *reinterpret_cast<const uint32_t*>(lg + (c < NM ? c : 0));
    mk[i] = c < NM ? x : 0u;
  }
  const bool unit = tid < H;
  float4 f1[16];
#pragma unroll
  for (int s = 0; s < 16; ++s) f1[s] = reinterpret_cast<const float4*>(p.fc1_t)[(size_t)s * H + (unit ? tid : 0)];
  const float f1b = p.fc1_b[unit ? tid : 0], f2 = unit ? p.fc2_w[tid] : 0.0f;
  {
    const int nb = w & 3, rb0 = hrb0;
    const uint8_t* q = sm + ((nb + 4 * hi4 + 1) * 9 + col + 1) * CS + kq * 16;
    f32x4 acc[3], sml[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) acc[i] = sml[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (!EARLY) load_head(0);
    for (int cs = 0; cs < CP; ++cs) {
      const Split x = {frag_at(q + cs * 64), frag_at(q + cs * 64 + RB), frag_at(q + cs * 64 + 2 * RB)};
#pragma unroll
      for (int i = 0; i < 3; ++i) mma_split(ha[i], x, acc[i], sml[i]);
      load_head(cs + 1 < CP ? cs + 1 : cs);
    }
    __syncthreads();
    float* L = reinterpret_cast<float*>(sm);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = (rb0 + 2 * i) * 16 + 4 * kq + r;
        if (row <= P) L[row * 64 + (nb + 4 * hi4) * 8 + col] = mma_sum(acc[i][r], sml[i][r]) + p.head_b[row];
      }
  }
  __syncthreads();

  // ---- legal-move softmax and value head
  const float* L = reinterpret_cast<const float*>(sm);
  float e[UN][4], mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < UN; ++i) {
    const int c = 4 * (tid + i * NT);
    const float4 z = c < NM ? *reinterpret_cast<const float4*>(L + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float zz[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      e[i][t] = (mk[i] >> (8 * t)) & 0xffu ? zz[t] : -INFINITY;
      mx = fmaxf(mx, e[i][t]);
    }
  }
  float g = f1b;
  const float* u = L + NM;
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    float4 us = *reinterpret_cast<const float4*>(u + 4 * s);
    if (p.value_conv_relu) us = make_float4(fmaxf(us.x, 0.f), fmaxf(us.y, 0.f), fmaxf(us.z, 0.f), fmaxf(us.w, 0.f));
    g = fmaf(f1[s].x, us.x, g);
    g = fmaf(f1[s].y, us.y, g);
    g = fmaf(f1[s].z, us.z, g);
    g = fmaf(f1[s].w, us.w, g);
  }
  mx = block_reduce(mx, true, scratch);
  const float msub = mx == -INFINITY ? 0.0f : mx;
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < UN; ++i)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      e[i][t] = e[i][t] == -INFINITY ? 0.0f : expf(e[i][t] - msub);
      sum += e[i][t];
    }
  sum = block_reduce(sum, false, scratch + NW);
  const float part = block_reduce(f2 * (unit ? fmaxf(g, 0.0f) : 0.0f), false, scratch + 2 * NW);
  const float inv = sum > 0.0f ? 1.0f / sum : 0.0f;
  float* pol = policy + (size_t)b * NM;
#pragma unroll
  for (int i = 0; i < UN; ++i) {
    const int c = 4 * (tid + i * NT);
    if (c < NM) *reinterpret_cast<float4*>(pol + c) = make_float4(e[i][0] * inv, e[i][1] * inv, e[i][2] * inv, e[i][3] * inv);
  }
  if (tid == 0) value[b] = tanhf(part + p.fc2_b);
}

template <int MB, int NB>
hipError_t launch(const AzDevNet& n, const float* planes, const uint8_t* legal, int B, float* policy, float* value,
                  hipStream_t s) {
  const int slot = 3 * 64 * ((n.filters + 31) / 32) + 16;
  const int act = SLOTS * slot, logits = (n.policy_planes + 1) * 64 * 4;
  const int scratch_off = act > logits ? act : logits;  // multiples of 16
  const int lds = scratch_off + 3 * NW * 4;
  static_assert(SLOTS * (3 * 64 * (256 / 32) + 16) + 3 * NW * 4 == 141328, "LDS at 256 filters, of 160 KB");
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&az_net_f32_kernel<MB, NB>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((az_net_f32_kernel<MB, NB>), dim3(B), dim3(NT), lds, s, n, planes, legal, policy, value,
                     scratch_off);
  return hipGetLastError();
}

}  // namespace

hipError_t az_launch_f32(const AzDevNet& n, const float* planes, const uint8_t* legal, int B,
                         float* policy, float* value, hipStream_t s) {
  (void)hipGetLastError();
  const int M16 = (n.filters + 15) / 16;  // 16-channel blocks: eight waves cover the layer's blocks once
  if (M16 > 8) return launch<2, 4>(n, planes, legal, B, policy, value, s);
  if (M16 > 4) return launch<1, 4>(n, planes, legal, B, policy, value, s);
  if (M16 > 1) return launch<1, 2>(n, planes, legal, B, policy, value, s);
  return launch<1, 1>(n, planes, legal, B, policy, value, s);
}
