// Fused policy/value network evaluation on CDNA4 matrix cores (gfx950).
//
// One kernel evaluates the whole network for a tile of boards: stem, every
// residual block, the policy and value heads, the legal-move softmax and the
// tanh value.  Activations never leave the workgroup's LDS; the only HBM
// traffic is the input planes, the legal mask, the outputs and the weight
// stream (which stays resident in L2 / the Infinity Cache across workgroups).
//
// Every 3x3 convolution is an implicit GEMM per board:
//   D[ch][sq] = sum_k W[ch][k] * X[k][sq],  k = tap * C_in + c,
//   X[tap*C_in + c][sq] = act[c][sq shifted by tap]   (zero outside the board)
// with output channels as the MFMA M dimension (A operand = weights, streamed
// from global memory in pre-packed fragment order) and board squares as the N
// dimension (B operand = activations, read from LDS).  A 32x32 MFMA block
// covers 32 channels x 32 squares (half a board).  The tap loop is the K loop:
// no im2col is materialised; a shifted window is just a different LDS row per
// lane, and out-of-board taps read a zero row.
//
// Column mapping.  A 32-column MFMA block takes its squares from BPG boards, and
// the blocks of a wave's boards are whole board rows: with four boards block j is
// row j of each; with two, rows j and j + 4; with one, rows j, j + 2, j + 4 and
// j + 6.  A vertical tap (dy) of block j is then block j + dy, so the fragments
// read from LDS for one horizontal tap (dx) and one channel step serve all three
// dy: the K loop runs over (dx, channel step) and does every (dy, block) product
// inside.  That reads LDS a third as often with four boards (half, two thirds
// with two, one), streams each weight fragment once per workgroup (waves differ
// in channels, not in squares), and with four boards leaves out the products
// whose rows lie wholly outside the board (2 of 24).  Only the blocks -1 and NBK
// of the mappings with fewer boards, partly outside, are fragments of their own.
//
// The K loop is unrolled with compile-time register indices: weight fragments
// stream through a ring of groups (a group: the three dy of one (dx, channel
// step)) that crosses layers, and the LDS fragments of the next step are read
// while the MFMAs of this one run.  The epilogue (bias, residual, activation,
// requantisation) runs once per layer, followed by one workgroup barrier; its
// per-channel constants are staged through LDS one layer ahead.
//
// What bounds it.  With every compute unit busy (1,024 boards) the chip's clock: at
// 20x128 int8 the batch takes 254 us against 235 us for 768 boards, the same work
// per compute unit, on one box (281 against 238 on a box that clocks lower); a loop of
// nothing but these MFMAs runs at 1.93 GHz on all 256 compute units, 2.3 GHz on half
// of them.  Below that, the float64 epilogue: a wave has a SIMD to itself and issues
// it between products of the next block (the tail) or after the loop.  Against the K
// loop in tap order (each fragment read for one product, two waves streaming the same
// weights), both on one box, us: 20x128 int8 64 boards 90 -> 85, 1,024 299 -> 254;
// bf16 32 boards 143 -> 130, 256 182 -> 161, 1,024 553 -> 465; 24x256 bf16 64 boards
// 920 -> 540, 1,024 2,500 -> 2,338.
//
// Activation layout in LDS: [board group][row][board][column][channel], one run
// of F channels per square, stored in 16-byte chunks whose position is
// XOR-swizzled by the square's place in its row so that the 16 lanes of a
// ds_read_b128 group hit 16 different bank groups.  Every row of a group ends in
// a zero pad: the columns left and right of a board are read there, at the bank
// slot the virtual square would use, so one lane address serves every row.
//
// bf16 networks keep the residual stream (every block input h) in fp32 in the
// registers of the wave that produces it: each wave owns the same output tile
// in every layer, so the residual of an output element lives in the lane that
// computes it.  LDS holds bf16(h), the convolution operand.  The heads read h
// as bf16(h) + bf16(h - bf16(h)).
//
// MFMA output layout (32x32 blocks): lane l holds column l%32 and rows
// 8*(v/4) + 4*(l/32) + v%4 of its 16 accumulators v, i.e. four runs of four
// consecutive channels of one square, which the epilogue packs and stores with
// one LDS write per run.
#include "az_internal.h"
#include "az_mfma_common.h"

#include <math.h>

#include <type_traits>

namespace {

// LDS geometry of a tensor with RB bytes per square, boards in groups of BPG.
template <int RB, int BPG>
struct Geo {
  static constexpr int ZP = cmax(RB, 256);          // zero pad: a 256-byte bank window at least
  static constexpr int PAD = BPG * 8 * RB;          // its place in a row
  static constexpr int RS = PAD + ZP;               // row stride
  static constexpr int GS = 8 * RS;                 // group stride
  static constexpr int NBK = 2 * BPG;               // 32-column blocks of a group
  static constexpr int RPB = 8 / NBK;               // rows of a board in one block
  static constexpr bool EDGE = RPB > 1;             // blocks -1 and NBK hold rows inside the board
  static constexpr int NX = NBK + (EDGE ? 2 : 0);   // fragments of one (dx, channel step)
  static_assert(RS % 256 == 0 && (NBK - 1) * RS < 65536, "row offsets are immediates");
  // swizzle of the square at (row, place v = 8 * board + column); with one board a
  // 16-lane group holds two rows, told apart by their place in the block
  static __device__ __forceinline__ int sw(int row, int v) {
    return swz<RB>(BPG == 1 ? ((row >> 1) & 1) * 8 + v : v);
  }
  // byte offset of a square's run of channels
  static __device__ __forceinline__ int at(int group, int row, int board, int col) {
    return group * GS + row * RS + (board * 8 + col) * RB;
  }
};

// Lane addresses of the B fragments of one horizontal tap dx: channel step cs of
// block j is at row + j * RS + (sw ^ cs * step), in a buffer whose offset the
// caller adds; blocks -1 and NBK have rows and swizzles of their own.  They are
// computed once; `opaque` redefines them to the compiler, once per layer: hoisted
// out of the block loop, the addresses of every step would take (and, at 256
// filters, spill) over a hundred registers.
template <int MK, int RB, int BPG>
struct Taps {
  using G = Geo<RB, BPG>;
  static constexpr int STEP = 2 * Mk<MK>::FB;  // bytes of one channel step
  int row, sw, row_lo, sw_lo, row_hi, sw_hi;
  __device__ __forceinline__ void init(int base, int dx, int l32, int lhi) {
    const int i = l32 / (8 * BPG), v = l32 % (8 * BPG) + dx, c = (l32 & 7) + dx;
    const bool ok = (unsigned)c < 8u;
    const int pad = base + G::PAD + ((v * RB) & 255), r0 = i * G::NBK, ch = lhi * (STEP / 32);
    row = (ok ? base + v * RB : pad) + r0 * G::RS;
    sw = (G::sw(r0, v) ^ ch) << 4;
    row_lo = i > 0 ? row - G::RS : pad;
    sw_lo = (G::sw(r0 - 2, v) ^ ch) << 4;  // row r0 - 1
    row_hi = i < G::RPB - 1 ? row + G::NBK * G::RS : pad;
    sw_hi = (G::sw(r0 + G::NBK, v) ^ ch) << 4;
  }
  __device__ __forceinline__ void opaque() {
    asm volatile("" : "+v"(row), "+v"(sw));
    if constexpr (G::EDGE) asm volatile("" : "+v"(row_lo), "+v"(row_hi));
    if constexpr (G::EDGE && BPG == 1) asm volatile("" : "+v"(sw_lo), "+v"(sw_hi));
  }
  // the fragment of channel step cs, block x (-1 .. NBK)
  template <int X>
  __device__ __forceinline__ typename Mk<MK>::frag get(const uint8_t* buf, int cs) const {
    constexpr bool LO = X < 0, HI = X >= G::NBK;
    const int r = LO ? row_lo : HI ? row_hi : row;
    const int w = BPG == 1 ? (LO ? sw_lo : HI ? sw_hi : sw) : sw;  // row parity matters with one board only
    const uint8_t* q = buf + (LO || HI ? 0 : X * G::RS);
    if constexpr (MK == MK_F8) {
      const i32x4 lo = *reinterpret_cast<const i32x4*>(q + (w ^ cs * STEP) + r);
      const i32x4 hi = *reinterpret_cast<const i32x4*>(q + (w ^ (cs * STEP + 16)) + r);
      return i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    } else {
      return *reinterpret_cast<const typename Mk<MK>::frag*>(q + (w ^ cs * STEP) + r);
    }
  }
  // all fragments of channel step cs, in the order of blocks
  __device__ __forceinline__ void load(const uint8_t* buf, int cs, typename Mk<MK>::frag (&dst)[G::NX]) const {
    static_for<0, G::NX>([&](auto x_c) {
      constexpr int x = decltype(x_c)::value;
      dst[x] = get<x - (G::EDGE ? 1 : 0)>(buf, cs);
    });
  }
};

// Tile shape: the wave owns MBW 32-channel blocks x the NBK 32-square blocks of
// BPG boards; the workgroup is WM x WN waves; OCC workgroups share a compute unit.
template <int MK, int F, int MBW, int BPG, int WM, int WN, int OCC, int NBUF_, int TAIL_>
struct Cfg {
  using T = Mk<MK>;
  static constexpr int NW = WM * WN, NT = 64 * NW;
  static constexpr int BPW = BPG * WN;  // boards per workgroup
  static constexpr int NMB = F / 32;
  static_assert(NMB == MBW * WM, "channel tiling");
  static constexpr int RB = F * T::ES;  // bytes per square, tower tensors
  using GeoT = Geo<RB, BPG>;            // tower tensors
  using GeoS = Geo<64, BPG>;            // stem input: 32 bf16 channels
  static constexpr int NBK = GeoT::NBK;
  static constexpr int BUF = WN * GeoT::GS;
  static constexpr int OFF_H = 0, OFF_T = BUF;
  static_assert(GeoS::GS <= GeoT::GS, "the stem input lies in the T buffer");
  static constexpr int RBX = 2 * F;  // bf16 row bytes of the heads' input
  static constexpr int OFF_X = OFF_T;
  static constexpr int LBMAX = (AZ_MAX_POLICY + 1) * 64;  // floats per board, logits + u
  // per-layer epilogue constants, double-buffered: [2 slots][bias F] floats, or
  // for quantised nets [2 slots][qbias F | qmul F | qres, qhi] doubles (the layer's
  // two scalars ride along: a load from global memory in the epilogue would wait
  // for the whole weight stream in flight, 1,000 cycles and more per layer)
  static constexpr int OFF_K = 2 * BUF;
  static constexpr int KSLOT = MK == MK_BF16 ? 4 * F : 16 * F + 16;
  // head row constants (scale, bias) and the softmax / value reductions sit past
  // every other region: they are written at the start and read at the end
  static constexpr int OFF_HC = (cmax(cmax(OFF_K + 2 * KSLOT, OFF_X + BPW * 64 * RBX), BPW * LBMAX * 4) + 15) & ~15;
  static constexpr int RED_PER_BOARD = 32;  // floats: [0,8) sum groups, [8,12) max per wave, [16,24) value groups
  static constexpr int OFF_RED = OFF_HC + 2 * AZ_HEAD_ROWS * 4;
  static constexpr int SMEM = OFF_RED + BPW * RED_PER_BOARD * 4;
  static_assert(SMEM * OCC <= 160 * 1024, "LDS");
  static_assert(NW % BPW == 0, "every board gets a whole number of waves at the end");
  static constexpr int CPT = F / T::KS;  // channel steps
  static constexpr int NS = 3 * CPT;     // (dx, channel step) groups per layer
  static constexpr int NBUF = NBUF_;     // weight prefetch ring depth (groups)
  // The layer's last TAIL groups are done block by block, each block's epilogue
  // under the next one's products.  Its constants stay in registers meanwhile:
  // not with two channel blocks of float64 ones (0: the epilogue follows the loop).
  static constexpr int TAIL = MK != MK_BF16 && MBW > 1 ? 0 : TAIL_;
  static_assert(TAIL < NBUF_ && TAIL < NS, "the tail's weights are in the ring");
  static_assert((2 * NS) % NBUF == 0, "every block's first conv starts at ring slot 0");
  static constexpr int FRAG_BYTES = 64 * T::FB;
  static constexpr int GROUP_BYTES = 3 * NMB * FRAG_BYTES;  // [dy][channel block] fragments
  static constexpr size_t LAYER_BYTES = (size_t)NS * GROUP_BYTES;
  static constexpr int NBH = (2 * BPW + NW - 1) / NW;  // head N-blocks per wave
};

// Product acc[m] += A[m] X of output block J for dy = D - 1, one (dx, channel
// step), x its fragments in block order.  With whole-row blocks (no EDGE) the rows
// above and below the board are left out.  FIRST: the layer's first step, whose
// first product of a block starts its accumulators.
template <class T, class G, int MBW, int J, int D, bool FIRST, class A_, class X_, class C_>
__device__ __forceinline__ void tap_product(const A_& a, const X_& x, C_& acc) {
  constexpr int xi = J + D - 1 + (G::EDGE ? 1 : 0);
  if constexpr (xi >= 0 && xi < G::NX) {
    constexpr bool zero = FIRST && (D == 0 || (!G::EDGE && D == 1 && J == 0));
#pragma unroll
    for (int m = 0; m < MBW; ++m)
      acc[m][J] = T::mma(a[D][m], x[xi], zero ? typename T::acc{} : acc[m][J]);
  }
}
// Every product of one (dx, channel step); each accumulator in the order of dy,
// whatever the mapping.
template <class T, class G, int MBW, bool FIRST, class A_, class X_, class C_>
__device__ __forceinline__ void tap_products(const A_& a, const X_& x, C_& acc) {
  static_for<0, 3>([&](auto d_c) {
    static_for<0, G::NBK>([&](auto j_c) {
      tap_product<T, G, MBW, decltype(j_c)::value, decltype(d_c)::value, FIRST>(a, x, acc);
    });
  });
}

template <int MK, int F, int MBW, int BPG, int WM, int WN, int OCC, int NBUF_, int TAIL_>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WM * WN, 64 * WM * WN),
                          amdgpu_waves_per_eu(OCC, OCC))) void
az_net_kernel(AzDevNet p, const float* __restrict__ planes, const uint8_t* __restrict__ legal, int B,
              float* __restrict__ policy, float* __restrict__ value) {
  using C = Cfg<MK, F, MBW, BPG, WM, WN, OCC, NBUF_, TAIL_>;
  using T = typename C::T;
  using SB = Mk<MK_BF16>;
  using GT = typename C::GeoT;
  using GS = typename C::GeoS;
  using frag_t = typename T::frag;
  using acc_t = typename T::acc;
  constexpr bool QUANT = MK != MK_BF16;
  constexpr int NW = C::NW, NT = C::NT, BPW = C::BPW, NMB = C::NMB, RB = C::RB, NBK = C::NBK;
  constexpr int OFF_H = C::OFF_H, OFF_T = C::OFF_T;

  __shared__ __attribute__((aligned(16))) uint8_t smem[C::SMEM];

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w % WM, wn = w / WM;
  const int l32 = lane & 31, lhi = lane >> 5;
  const int mb0 = wm * MBW;
  const int b0 = blockIdx.x * BPW;
  const int Cin = p.in_planes;
  const float cap = p.act_cap;
  // this lane's column: place v in a row of its group, first row r0 of its blocks
  const int lv = l32 % (8 * BPG), lr0 = l32 / (8 * BPG) * NBK;

  // fp32 residual stream of the wave's output tile (bf16 networks)
  float res[QUANT ? 1 : MBW][QUANT ? 1 : NBK][16];

  // The multi-board tilings with one workgroup per CU have registers to spare
  // outside the tower: they load the stem's and the heads' weights early.
  constexpr bool ROOMY = OCC == 1 && BPG >= 2;
  // Stem weights (bf16, six (dx, channel step) groups of three dy): a ring of SR
  // groups, the first SR - 1 loaded here, ahead of the input planes, so that their
  // latency overlaps the ingest: all six (up to F = 128), or double-buffered.
  constexpr int SN = 6, SR = ROOMY && F <= 128 ? SN : 2;
  const uint8_t* sw8 = static_cast<const uint8_t*>(p.stem_w) + (size_t)(mb0 * 64 + lane) * 16;
  SB::frag sa[SR][3][MBW];
  auto load_stem = [&](int g, SB::frag(&dst)[3][MBW]) {
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int m = 0; m < MBW; ++m) dst[d][m] = g_frag<MK_BF16>(sw8 + ((g * 3 + d) * NMB + m) * 64 * 16);
  };
  static_for<0, SR - 1>([&](auto t_c) { load_stem(decltype(t_c)::value, sa[decltype(t_c)::value]); });

  // ---- ingest: zero pads, planes -> bf16 [square][32 channels] at OFF_T.  The T
  // buffer's own pads, some of them inside the stem input, are cleared after the stem.
  auto zero_pads = [&](auto geo, int off) {
    using G = decltype(geo);
    constexpr int PC = G::ZP / 16;  // 16-byte chunks of a pad
    for (int i = tid; i < WN * 8 * PC; i += NT)
      *reinterpret_cast<i32x4*>(smem + off + i / PC * G::RS + G::PAD + i % PC * 16) = i32x4{0, 0, 0, 0};
  };
  zero_pads(GT{}, OFF_H);
  zero_pads(GS{}, OFF_T);
  // One item = 8 input planes of one board: lane = square, eight plane loads (each
  // coalesced over the wave), one 16-byte LDS store.  Items are wave-uniform and
  // every load is issued before the first is used.
  {
    constexpr int ITEMS = BPW * 4, PER = (ITEMS + NW - 1) / NW;
    float pv[PER][8];
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int item = w + it * NW, bl = item >> 2, k = item & 3, b = b0 + bl;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        // unconditional load (clamped to plane 0 of board 0) so that no branch
        // separates a load from the next one
        const int c = 8 * k + t;
        const bool ok = item < ITEMS && b < B && c < Cin;
        const float x = planes[ok ? ((size_t)b * Cin + c) * 64 + lane : (size_t)lane];
        pv[it][t] = ok ? x : 0.0f;
      }
    }
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int item = w + it * NW, bl = item >> 2, k = item & 3;
      if (item < ITEMS)
        *reinterpret_cast<uint4*>(smem + OFF_T + GS::at(bl / BPG, lane >> 3, bl % BPG, lane & 7) +
                                  ((k ^ GS::sw(lane >> 3, bl % BPG * 8 + (lane & 7))) << 4)) =
            make_uint4(pack_bf16x2(pv[it][0], pv[it][1]), pack_bf16x2(pv[it][2], pv[it][3]),
                       pack_bf16x2(pv[it][4], pv[it][5]), pack_bf16x2(pv[it][6], pv[it][7]));
    }
  }

  // first weight group of the tower, in flight during the stem
  // Weight fragments: a ring of NBUF prefetch groups; group g of a layer lives in
  // buffer g % NBUF and is loaded NBUF - 1 groups before its use.
  // The stream is read through a buffer resource: the lane's offset is a
  // constant VGPR and a group's byte offset a scalar, so weight loads cost no
  // vector address arithmetic in the K loop.
  constexpr int NBUF = C::NBUF;
  const __amdgpu_buffer_rsrc_t twr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.tower_w), (short)0, (int)(2 * p.blocks * C::LAYER_BYTES), 0x00020000);
  const int tvoff = (mb0 * 64 + lane) * T::FB;
  frag_t A[NBUF][3][MBW];
  auto load_group = [&](frag_t(&dst)[3][MBW], int soff) {
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int m = 0; m < MBW; ++m) {
        const int o = soff + (d * NMB + m) * C::FRAG_BYTES;
        if constexpr (T::FB == 16) {
          dst[d][m] = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(twr, tvoff, o, 0));
        } else {
          const i32x4 lo = __builtin_amdgcn_raw_buffer_load_b128(twr, tvoff, o, 0);
          const i32x4 hi = __builtin_amdgcn_raw_buffer_load_b128(twr, tvoff, o + 16, 0);
          dst[d][m] = __builtin_bit_cast(frag_t, i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
        }
      }
  };
  static_for<0, NBUF - 1>([&](auto i_c) {
    constexpr int i = decltype(i_c)::value;
    load_group(A[i], i * C::GROUP_BYTES);
  });
  // per-layer epilogue constants: thread t < KSLOT/16 carries 16-byte chunk t of
  // the slot ([bias] floats, or [qbias | qmul | qres, qhi] doubles); with 256
  // filters the last chunk has no thread left and thread 0 carries it as well
  constexpr int KCH = C::KSLOT / 16;
  struct Consts { float4 a, b; };
  auto load_consts = [&](int k) -> Consts {  // k = 1 + conv index (0 = stem)
    Consts r = {};
    if constexpr (QUANT) {
      if (tid < KCH) {
        const double* src = tid < F / 2 ? p.qbias + (size_t)k * F + 2 * tid
                            : tid < F   ? p.qmul + (size_t)k * F + 2 * (tid - F / 2)
                                        : p.qext + 2 * k;
        r.a = *reinterpret_cast<const float4*>(src);
      }
      if constexpr (KCH > NT) {
        if (tid == 0) r.b = *reinterpret_cast<const float4*>(p.qext + 2 * k);
      }
    } else {
      if (tid < KCH) r.a = *reinterpret_cast<const float4*>(p.bias + (size_t)k * F + tid * 4);
    }
    return r;
  };
  auto store_consts = [&](int slot, const Consts& v) {
    uint8_t* dst = smem + C::OFF_K + slot * C::KSLOT;
    if (tid < KCH) *reinterpret_cast<float4*>(dst + tid * 16) = v.a;
    if constexpr (KCH > NT) {
      if (tid == 0) *reinterpret_cast<float4*>(dst + NT * 16) = v.b;
    }
  };
  static_assert(NT + 1 >= KCH, "constant staging");
  store_consts(0, load_consts(1));
  if (tid < AZ_HEAD_ROWS / 2)  // [scale 96 | bias 96] floats
    *reinterpret_cast<float4*>(smem + C::OFF_HC + tid * 16) =
        *reinterpret_cast<const float4*>(tid < AZ_HEAD_ROWS / 4 ? p.head_sc + tid * 4 : p.head_bc + (tid - AZ_HEAD_ROWS / 4) * 4);
  static_assert(NT >= AZ_HEAD_ROWS / 2, "head constant staging");
  __syncthreads();

  // ---- stem: bf16 3x3 conv over 32 (padded) input channels, K = 288
  {
    f32x16 sacc[MBW][NBK];
    SB::frag xc[GS::NX], xn[GS::NX];
    auto load_x = [&](auto g_c, SB::frag(&dst)[GS::NX]) {
      constexpr int g = decltype(g_c)::value;
      Taps<MK_BF16, 64, BPG> t;
      t.init(wn * GS::GS, g / 2 - 1, l32, lhi);
      t.load(smem + OFF_T, g % 2, dst);
    };
    load_x(std::integral_constant<int, 0>{}, xc);
    static_for<0, SN>([&](auto g_c) {
      constexpr int g = decltype(g_c)::value;
      if constexpr (g + SR - 1 < SN) load_stem(g + SR - 1, sa[(g + SR - 1) % SR]);
      if constexpr (g + 1 < SN) load_x(std::integral_constant<int, g + 1>{}, xn);
      tap_products<SB, GS, MBW, g == 0>(sa[g % SR], xc, sacc);
      if constexpr (g + 1 < SN) {
#pragma unroll
        for (int x = 0; x < GS::NX; ++x) xc[x] = xn[x];
      }
    });
    // epilogue: bias, activation, store in the tower format at OFF_H
#pragma unroll
    for (int m = 0; m < MBW; ++m)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ch0 = (mb0 + m) * 32 + 8 * q + 4 * lhi;
        const float4 bb = *reinterpret_cast<const float4*>(p.bias + ch0);
        double mq[4] = {}, bq[4] = {};
        if constexpr (QUANT) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            mq[r] = p.qmul[ch0 + r];
            bq[r] = p.qbias[ch0 + r];
          }
        }
#pragma unroll
        for (int n = 0; n < NBK; ++n) {
          const f32x16& v = sacc[m][n];
          const int rowo = OFF_H + wn * GT::GS + (lr0 + n) * GT::RS + lv * RB, swo = GT::sw(lr0 + n, lv);
          if constexpr (!QUANT) {
            const float y0 = act_fn(v[4 * q + 0] + bb.x, cap), y1 = act_fn(v[4 * q + 1] + bb.y, cap);
            const float y2 = act_fn(v[4 * q + 2] + bb.z, cap), y3 = act_fn(v[4 * q + 3] + bb.w, cap);
            res[m][n][4 * q + 0] = y0;
            res[m][n][4 * q + 1] = y1;
            res[m][n][4 * q + 2] = y2;
            res[m][n][4 * q + 3] = y3;
            *reinterpret_cast<uint2*>(smem + rowo + (((ch0 >> 3) ^ swo) << 4) + 8 * lhi) =
                make_uint2(pack_bf16x2(y0, y1), pack_bf16x2(y2, y3));
          } else {
            // the stem's sum comes from the bf16 matrix instruction in fp32; the
            // rescale and rounding of its code are taken in float64
            const float hi = p.qhi[0];
            *reinterpret_cast<uint32_t*>(smem + rowo + (((ch0 >> 4) ^ swo) << 4) + (ch0 & 15)) =
                pack_codes_d<MK>(__builtin_fma((double)v[4 * q + 0], mq[0], bq[0]),
                                 __builtin_fma((double)v[4 * q + 1], mq[1], bq[1]),
                                 __builtin_fma((double)v[4 * q + 2], mq[2], bq[2]),
                                 __builtin_fma((double)v[4 * q + 3], mq[3], bq[3]), hi);
          }
        }
      }
  }
  __syncthreads();

  // ---- residual tower: per block conv1 (H -> T) and conv2 (T -> H, + residual)
  {
    constexpr int CPT = C::CPT, NS = C::NS;
    acc_t c[MBW][NBK];
    const int nconv = 2 * p.blocks;
    zero_pads(GT{}, OFF_T);  // read after the first layer's barrier
    Taps<MK, RB, BPG> taps[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) taps[dx].init(wn * GT::GS, dx - 1, l32, lhi);

    auto conv = [&](auto second_c, auto lb_c, int n_conv) {
      constexpr bool SECOND = decltype(second_c)::value;
      constexpr int LB = decltype(lb_c)::value;  // ring slot of the layer's first group
      const int wl = n_conv * (int)C::LAYER_BYTES;  // byte offset of the layer in the stream
      const bool has_next = n_conv + 1 < nconv;
      constexpr int in_off = SECOND ? OFF_T : OFF_H;
      constexpr int out_off = SECOND ? OFF_H : OFF_T;
      // the next layer's epilogue constants, parked in LDS before this layer's barrier
      const Consts kn = has_next ? load_consts(n_conv + 2) : Consts{};
      const float* kslot = reinterpret_cast<const float*>(smem + C::OFF_K + (n_conv & 1) * C::KSLOT);
      // B fragments of one (dx, channel step)
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) taps[dx].opaque();
      frag_t xc[GT::NX], xn[GT::NX];
      auto load_x = [&](auto s_c, frag_t(&dst)[GT::NX]) {
        constexpr int s = decltype(s_c)::value;
        taps[s / CPT].load(smem + in_off, s % CPT, dst);
      };
      // group s + NBUF-1 of this layer, i.e. of the next layer past the end (layers
      // are contiguous); past the network's last layer this layer's start is
      // re-read (never used)
      auto prefetch = [&](auto s_c) {
        constexpr int s = decltype(s_c)::value, gi = s + NBUF - 1;
        load_group(A[(LB + gi) % NBUF], wl + ((gi < NS || has_next) ? gi * C::GROUP_BYTES : 0));
      };

      // Epilogue of the 4-channel run q of block n, channel block m: float32 bias,
      // residual and activation (bf16), or the float64 requantisation z = acc * qmul
      // + qbias (+ residual code * qres), rounded to the code grid and clamped.  The
      // run's constants and residual codes were read from LDS before (the codes in
      // place, by the lane that then overwrites them).
      constexpr bool RCODE = QUANT && SECOND;
      struct KQ { double b[QUANT ? 4 : 1], m[QUANT ? 4 : 1]; float4 f; };
      float hi = 0.0f;
      double rq = 0.0;
      auto ep_addr = [&](int m, int q, int n) {
        const int ch0 = (mb0 + m) * 32 + 8 * q + 4 * lhi;
        const int rowo = out_off + wn * GT::GS + (lr0 + n) * GT::RS + lv * RB, swo = GT::sw(lr0 + n, lv);
        if constexpr (QUANT) return rowo + (((ch0 >> 4) ^ swo) << 4) + (ch0 & 15);
        else return rowo + (((ch0 >> 3) ^ swo) << 4) + 8 * lhi;
      };
      auto ep_scalars = [&]() {
        if constexpr (QUANT) {
          const double* kd = reinterpret_cast<const double*>(kslot);
          rq = kd[2 * F];
          hi = (float)kd[2 * F + 1];
        }
      };
      auto ep_consts = [&](int m, int q, KQ& k) {
        const int ch0 = (mb0 + m) * 32 + 8 * q + 4 * lhi;
        if constexpr (QUANT) {
          const double* kd = reinterpret_cast<const double*>(kslot);
#pragma unroll
          for (int r = 0; r < 4; r += 2) {
            const double2 b2 = *reinterpret_cast<const double2*>(kd + ch0 + r);
            const double2 m2 = *reinterpret_cast<const double2*>(kd + F + ch0 + r);
            k.b[r] = b2.x;
            k.b[r + 1] = b2.y;
            k.m[r] = m2.x;
            k.m[r + 1] = m2.y;
          }
        } else {
          k.f = *reinterpret_cast<const float4*>(kslot + ch0);
        }
      };
      auto ep_code = [&](int m, int q, int n) { return *reinterpret_cast<const uint32_t*>(smem + ep_addr(m, q, n)); };
      auto ep_run = [&](int m, int q, int n, const KQ& k, uint32_t rc) {
        const int addr = ep_addr(m, q, n);
        const acc_t& v = c[m][n];
        if constexpr (!QUANT) {
          float y0 = v[4 * q + 0] + k.f.x, y1 = v[4 * q + 1] + k.f.y;
          float y2 = v[4 * q + 2] + k.f.z, y3 = v[4 * q + 3] + k.f.w;
          if constexpr (SECOND) {
            y0 = act_fn(y0 + res[m][n][4 * q + 0], cap);
            y1 = act_fn(y1 + res[m][n][4 * q + 1], cap);
            y2 = act_fn(y2 + res[m][n][4 * q + 2], cap);
            y3 = act_fn(y3 + res[m][n][4 * q + 3], cap);
            res[m][n][4 * q + 0] = y0;
            res[m][n][4 * q + 1] = y1;
            res[m][n][4 * q + 2] = y2;
            res[m][n][4 * q + 3] = y3;
          } else {
            y0 = act_fn(y0, cap);
            y1 = act_fn(y1, cap);
            y2 = act_fn(y2, cap);
            y3 = act_fn(y3, cap);
          }
          *reinterpret_cast<uint2*>(smem + addr) = make_uint2(pack_bf16x2(y0, y1), pack_bf16x2(y2, y3));
        } else {
          double z[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) z[r] = __builtin_fma((double)v[4 * q + r], k.m[r], k.b[r]);
          if constexpr (SECOND) {
            z[0] = __builtin_fma(code_value_d<MK, 0>(rc), rq, z[0]);
            z[1] = __builtin_fma(code_value_d<MK, 1>(rc), rq, z[1]);
            z[2] = __builtin_fma(code_value_d<MK, 2>(rc), rq, z[2]);
            z[3] = __builtin_fma(code_value_d<MK, 3>(rc), rq, z[3]);
          }
          *reinterpret_cast<uint32_t*>(smem + addr) = pack_codes_d<MK>(z[0], z[1], z[2], z[3], hi);
        }
      };

      constexpr int TAIL = C::TAIL, MAIN = NS - TAIL, PER = MK == MK_F8 ? 2 : 1;  // instructions per fragment
      constexpr int X0 = GT::EDGE ? 1 : 0;  // index of block 0 among the fragments
      frag_t xt[TAIL > 0 ? TAIL : 1][GT::NX];
      auto tail_x = [&](auto x_c) {  // fragment x of every tail group
        constexpr int x = decltype(x_c)::value;
        static_for<0, TAIL>([&](auto t_c) {
          constexpr int t = decltype(t_c)::value, s = MAIN + t;
          xt[t][x] = taps[s / CPT].template get<x - X0>(smem + in_off, s % CPT);
        });
      };
      load_x(std::integral_constant<int, 0>{}, xc);
      static_for<0, MAIN>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value;
        prefetch(s_c);
        if constexpr (s + 1 < MAIN) load_x(std::integral_constant<int, s + 1>{}, xn);
        else if constexpr (TAIL > 0) static_for<0, X0 + 2>(tail_x);
        tap_products<T, GT, MBW, s == 0>(A[(LB + s) % NBUF], xc, c);
        if constexpr (s + 1 < MAIN) {
#pragma unroll
          for (int x = 0; x < GT::NX; ++x) xc[x] = xn[x];
        }
        // interleave: each MFMA is followed by one of the next step's LDS reads,
        // then by one of the prefetched group's weight loads
        constexpr int NDS = PER * (s + 1 < MAIN ? GT::NX : TAIL * (X0 + 2)), NVM = 3 * MBW * PER;
        constexpr int NMF = MBW * (3 * NBK - (GT::EDGE ? 0 : 2));
        static_for<0, NMF>([&](auto i_c) {
          constexpr int i = decltype(i_c)::value;
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if constexpr (i < NDS) __builtin_amdgcn_sched_group_barrier(0x100, i + 1 == NMF ? NDS - i : 1, 0);
          if constexpr (i < NVM) __builtin_amdgcn_sched_group_barrier(0x020, i + 1 == NMF ? NVM - i : 1, 0);
        });
        __builtin_amdgcn_sched_barrier(0);  // a step is one scheduling region
      });

      if constexpr (TAIL > 0) {
        KQ kq[MBW][4];
        uint32_t rc[2][MBW][4];
        static_for<0, NBK + 1>([&](auto j_c) {
          constexpr int j = decltype(j_c)::value;
          if constexpr (j == 0) {
            prefetch(std::integral_constant<int, MAIN>{});
            ep_scalars();
#pragma unroll
            for (int m = 0; m < MBW; ++m)
#pragma unroll
              for (int q = 0; q < 4; ++q) ep_consts(m, q, kq[m][q]);
          }
          if constexpr (j < NBK) {
            if constexpr (j + 2 + X0 < GT::NX) tail_x(std::integral_constant<int, j + 2 + X0>{});
            if constexpr (RCODE) {
#pragma unroll
              for (int m = 0; m < MBW; ++m)
#pragma unroll
                for (int q = 0; q < 4; ++q) rc[j % 2][m][q] = ep_code(m, q, j);
            }
            static_for<0, TAIL>([&](auto t_c) {
              constexpr int t = decltype(t_c)::value;
              static_for<0, 3>([&](auto d_c) {
                tap_product<T, GT, MBW, j, decltype(d_c)::value, false>(A[(LB + MAIN + t) % NBUF], xt[t], c);
              });
              // the last block frees the group: its slot takes the next load
              if constexpr (j + 1 == NBK && t + 1 < TAIL) prefetch(std::integral_constant<int, MAIN + t + 1>{});
            });
          }
          if constexpr (j > 0) {
#pragma unroll
            for (int m = 0; m < MBW; ++m)
#pragma unroll
              for (int q = 0; q < 4; ++q) ep_run(m, q, j - 1, kq[m][q], RCODE ? rc[(j - 1) % 2][m][q] : 0u);
          }
          if constexpr (j < NBK) {
            // a block's products with the reads ahead and the previous block's epilogue
            constexpr int NMF = 3 * TAIL * MBW, VPM = QUANT ? 8 : 6;
            static_for<0, NMF>([&](auto i_c) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
              if constexpr (j > 0) __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
            });
          }
          __builtin_amdgcn_sched_barrier(0);
        });
      } else {
        // Epilogue after the loop: runs k = (m, q), their LDS reads issued EP_AHEAD
        // runs ahead of their arithmetic in a ring of EP_AHEAD + 1 slots, so that no
        // read latency is exposed.
        constexpr int NRUN = MBW * 4, EP_AHEAD = QUANT ? (BPG >= 2 ? 2 : 1) : 0, EP_RING = EP_AHEAD + 1;
        KQ kq[EP_RING];
        uint32_t rc[EP_RING][NBK];
        ep_scalars();
        auto ep_load = [&](auto k_c) {
          constexpr int k = decltype(k_c)::value, slot = k % EP_RING;
          ep_consts(k / 4, k % 4, kq[slot]);
#pragma unroll
          for (int n = 0; n < NBK; ++n) rc[slot][n] = RCODE ? ep_code(k / 4, k % 4, n) : 0u;
        };
        static_for<0, EP_AHEAD>([&](auto k_c) { ep_load(k_c); });
        static_for<0, NRUN>([&](auto k_c) {
          constexpr int k = decltype(k_c)::value, slot = k % EP_RING;
          if constexpr (k + EP_AHEAD < NRUN) ep_load(std::integral_constant<int, k + EP_AHEAD>{});
#pragma unroll
          for (int n = 0; n < NBK; ++n) ep_run(k / 4, k % 4, n, kq[slot], rc[slot][n]);
        });
      }
      if (has_next) store_consts((n_conv + 1) & 1, kn);
      __syncthreads();
    };

    for (int blk = 0; blk < p.blocks; ++blk) {
      conv(std::false_type{}, std::integral_constant<int, 0>{}, 2 * blk);
      conv(std::true_type{}, std::integral_constant<int, NS % NBUF>{}, 2 * blk + 1);
    }
  }

  // ---- heads: 1x1 convs F -> (P policy planes + 1 value row) as one bf16 GEMM
  const int P = p.policy_planes;
  const int NMV = P * 64;
  // Softmax and value: WPB waves per board.  The board's cells form groups g of
  // 1024; in group g lane l owns the four runs of 4 cells at g*1024 + u*256 + 4l
  // (u = 0..3), so that a wave's LDS reads, mask loads and policy stores are
  // contiguous.  Wave part p of the board takes groups p, p + WPB, ...  Its
  // legal mask is loaded here, in flight during the heads.
  constexpr int WPB = NW / BPW;
  constexpr int NGRP = (AZ_MAX_POLICY * 64 + 1023) / 1024;  // cell groups
  constexpr int NGW = (NGRP + WPB - 1) / WPB;               // groups per wave
  const int sbl = w / WPB, spart = w % WPB;
  const int sb = b0 + sbl;
  const bool svalid = sb < B;
  uint32_t mk0[NGW][4];
#pragma unroll
  for (int ii = 0; ii < NGW; ++ii)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = 1024 * (spart + WPB * ii) + 256 * u + 4 * lane;
      const bool ok = svalid && c < NMV;
      const uint32_t x = *reinterpret_cast<const uint32_t*>(legal + (ok ? (size_t)sb * NMV + c : (size_t)0));
      mk0[ii][u] = ok ? x : 0u;
    }
  {
    constexpr int HS = F / 16, RBX = C::RBX, OFF_X = C::OFF_X, NBH = C::NBH;
    // head weights: in flight during the conversion below where the registers
    // allow, else loaded after it
    SB::frag ha[HS][3];
    auto load_head_w = [&]() {
      const uint8_t* hw = static_cast<const uint8_t*>(p.head_w) + (size_t)lane * 16;
#pragma unroll
      for (int s = 0; s < HS; ++s)
#pragma unroll
        for (int m = 0; m < 3; ++m) ha[s][m] = g_frag<MK_BF16>(hw + ((s * 3 + m) * 64) * 16);
    };
    if constexpr (ROOMY) load_head_w();
    if constexpr (QUANT) {
      // codes -> exact bf16 values (int8 and e4m3 values are bf16-representable)
      for (int idx = tid; idx < BPW * 64 * (F / 8); idx += NT) {
        const int k = idx % (F / 8), sq = (idx / (F / 8)) & 63, bl = idx / (64 * (F / 8));
        const uint2 v = *reinterpret_cast<const uint2*>(
            smem + OFF_H + GT::at(bl / BPG, sq >> 3, bl % BPG, sq & 7) +
            (((k >> 1) ^ GT::sw(sq >> 3, bl % BPG * 8 + (sq & 7))) << 4) + (k & 1) * 8);
        const uint4 o = make_uint4(pack_bf16x2(code_value<MK, 0>(v.x), code_value<MK, 1>(v.x)),
                                   pack_bf16x2(code_value<MK, 2>(v.x), code_value<MK, 3>(v.x)),
                                   pack_bf16x2(code_value<MK, 0>(v.y), code_value<MK, 1>(v.y)),
                                   pack_bf16x2(code_value<MK, 2>(v.y), code_value<MK, 3>(v.y)));
        *reinterpret_cast<uint4*>(smem + OFF_X + (bl * 64 + sq) * RBX + ((k ^ swz<RBX>(sq)) << 4)) = o;
      }
    } else {
      // low half of the fp32 residual: bf16(h - bf16(h)), same layout at OFF_X
#pragma unroll
      for (int m = 0; m < MBW; ++m)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int ch0 = (mb0 + m) * 32 + 8 * q + 4 * lhi;
#pragma unroll
          for (int n = 0; n < NBK; ++n) {
            const int bl = wn * BPG + (lv >> 3), j = (lr0 + n) * 8 + (lv & 7);
            float lo[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) lo[r] = res[m][n][4 * q + r] - bf16_round(res[m][n][4 * q + r]);
            *reinterpret_cast<uint2*>(smem + OFF_X + (bl * 64 + j) * RBX + (((ch0 >> 3) ^ swz<RBX>(j)) << 4) +
                                      8 * lhi) = make_uint2(pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]));
          }
        }
    }
    if constexpr (!ROOMY) load_head_w();
    __syncthreads();

    f32x16 hacc[NBH][3];
#pragma unroll
    for (int k = 0; k < NBH; ++k) {
#pragma unroll
      for (int m = 0; m < 3; ++m) hacc[k][m] = f32x16{};
      const int nb = w + k * NW;
      if (nb < 2 * BPW) {
        const int bl = nb >> 1, j = ((nb & 1) << 5) + l32;
        const int rowx = OFF_X + (bl * 64 + j) * RBX, swx = swz<RBX>(j);
#pragma unroll
        for (int s = 0; s < HS; ++s) {
          const SB::frag bfr = lds_frag<MK_BF16>(smem, rowx, swx, 2 * s + lhi);
#pragma unroll
          for (int m = 0; m < 3; ++m) hacc[k][m] = SB::mma(ha[s][m], bfr, hacc[k][m]);
        }
        if constexpr (!QUANT) {
          const int rowh = OFF_H + GT::at(bl / BPG, j >> 3, bl % BPG, j & 7);
          const int swh = GT::sw(j >> 3, bl % BPG * 8 + (j & 7));
#pragma unroll
          for (int s = 0; s < HS; ++s) {
            const SB::frag bfr = lds_frag<MK_BF16>(smem, rowh, swh, 2 * s + lhi);
#pragma unroll
            for (int m = 0; m < 3; ++m) hacc[k][m] = SB::mma(ha[s][m], bfr, hacc[k][m]);
          }
        }
      }
    }
    __syncthreads();
    // every row of every board: fma(acc, scale, bias) with the row constants
    // (policy rows leave pre-scaled by log2(e), rows past P are never read)
    float* L = reinterpret_cast<float*>(smem);
    const float* HC = reinterpret_cast<const float*>(smem + C::OFF_HC);
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r0 = m * 32 + 8 * q + 4 * lhi;
        const float4 sc = *reinterpret_cast<const float4*>(HC + r0);
        const float4 bc = *reinterpret_cast<const float4*>(HC + AZ_HEAD_ROWS + r0);
#pragma unroll
        for (int k = 0; k < NBH; ++k) {
          const int nb = w + k * NW;
          if (nb < 2 * BPW) {
            const int bl = nb >> 1, j = ((nb & 1) << 5) + l32;
            float* dst = L + bl * C::LBMAX + r0 * 64 + j;
            dst[0] = __builtin_fmaf(hacc[k][m][4 * q + 0], sc.x, bc.x);
            dst[64] = __builtin_fmaf(hacc[k][m][4 * q + 1], sc.y, bc.y);
            dst[128] = __builtin_fmaf(hacc[k][m][4 * q + 2], sc.z, bc.z);
            dst[192] = __builtin_fmaf(hacc[k][m][4 * q + 3], sc.w, bc.w);
          }
        }
      }
  }
  __syncthreads();

  // ---- legal-move softmax and value head: WPB waves per board (board sbl, part spart)
  // Sums are taken in an order that does not depend on WPB, so every tiling
  // returns the same bits: each 64-chunk group (policy) or 64-unit group (value
  // hidden layer) is reduced across the lanes of one wave, and the group sums
  // are added in group order.
  {
    const float* L = reinterpret_cast<const float*>(smem);
    float* red = reinterpret_cast<float*>(smem + C::OFF_RED) + sbl * C::RED_PER_BOARD;
    const float* Lb = L + sbl * C::LBMAX;
    float* pol = policy + (size_t)sb * NMV;
    const int H = p.value_hidden;
    // logits are stored as z * log2(e): p_i = 2^(zl_i - max zl) / sum over legal cells.
    // Illegal cells carry -inf through the max and contribute exactly 0.
    float e[NGW][16];
    float mx = -INFINITY;
#pragma unroll
    for (int ii = 0; ii < NGW; ++ii)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = 1024 * (spart + WPB * ii) + 256 * u + 4 * lane;
        const bool in = c < NMV;
        const float4 z4 = in ? *reinterpret_cast<const float4*>(Lb + c) : make_float4(0.f, 0.f, 0.f, 0.f);
        const float zz[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const bool ok = in && ((mk0[ii][u] >> (8 * t)) & 0xffu);
          e[ii][4 * u + t] = ok ? zz[t] : -INFINITY;
          mx = fmaxf(mx, e[ii][4 * u + t]);
        }
      }
    mx = wave_max(mx);
    if (lane == 0) red[8 + spart] = mx;
    __syncthreads();
    float bmx = red[8];
#pragma unroll
    for (int t = 1; t < WPB; ++t) bmx = fmaxf(bmx, red[8 + t]);
    const float msub = bmx == -INFINITY ? 0.0f : bmx;
#pragma unroll
    for (int ii = 0; ii < NGW; ++ii) {
      float gsum = 0.0f;
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        e[ii][t] = __builtin_amdgcn_exp2f(e[ii][t] - msub);  // exp2(-inf) = 0
        gsum += e[ii][t];
      }
      gsum = wave_sum(gsum);
      if (lane == 0 && spart + WPB * ii < NGRP) red[spart + WPB * ii] = gsum;
    }
    // value head inputs and hidden-unit groups r (unit 64 r + lane) of this wave
    float u[64];
#pragma unroll
    for (int s4 = 0; s4 < 64; s4 += 4) {
      const float4 t4 = *reinterpret_cast<const float4*>(Lb + NMV + s4);
      u[s4] = t4.x;
      u[s4 + 1] = t4.y;
      u[s4 + 2] = t4.z;
      u[s4 + 3] = t4.w;
    }
    if (p.value_conv_relu) {
#pragma unroll
      for (int s4 = 0; s4 < 64; ++s4) u[s4] = fmaxf(u[s4], 0.0f);
    }
    const int ngv = (H + 63) >> 6;  // hidden-unit groups (H <= 512: at most 8)
    for (int r = spart; r < ngv; r += WPB) {
      const int k = 64 * r + lane;
      const bool ok = k < H;
      const float4* src = reinterpret_cast<const float4*>(p.fc1_t) + (ok ? k : 0);
      float4 wr[16];
#pragma unroll
      for (int s4 = 0; s4 < 16; ++s4) wr[s4] = src[(size_t)s4 * H];
      const float gb = p.fc1_b[ok ? k : 0], w2r = p.fc2_w[ok ? k : 0];
      float g = ok ? gb : 0.0f;
      const float w2 = ok ? w2r : 0.0f;
#pragma unroll
      for (int s4 = 0; s4 < 16; ++s4)
        g += wr[s4].x * u[4 * s4] + wr[s4].y * u[4 * s4 + 1] + wr[s4].z * u[4 * s4 + 2] + wr[s4].w * u[4 * s4 + 3];
      const float vsum = wave_sum(w2 * fmaxf(g, 0.0f));
      if (lane == 0) red[16 + r] = vsum;
    }
    __syncthreads();
    float tot = 0.0f;
#pragma unroll
    for (int g = 0; g < NGRP; ++g) tot += (1024 * g < NMV) ? red[g] : 0.0f;
    const float inv = tot > 0.0f ? 1.0f / tot : 0.0f;
    if (svalid) {
#pragma unroll
      for (int ii = 0; ii < NGW; ++ii)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int c = 1024 * (spart + WPB * ii) + 256 * u + 4 * lane;
          if (c < NMV)
            *reinterpret_cast<float4*>(pol + c) =
                make_float4(e[ii][4 * u] * inv, e[ii][4 * u + 1] * inv, e[ii][4 * u + 2] * inv, e[ii][4 * u + 3] * inv);
        }
      if (spart == 0 && lane == 0) {
        float vs = 0.0f;
        for (int r = 0; r < ngv; ++r) vs += red[16 + r];
        value[sb] = tanhf(vs + p.fc2_b);
      }
    }
  }
}

template <int MK, int F, int MBW, int BPG, int WM, int WN, int OCC, int NBUF, int TAIL>
hipError_t launch_cfg(const AzDevNet& n, const float* planes, const uint8_t* legal, int B,
                      float* policy, float* value, hipStream_t s) {
  using C = Cfg<MK, F, MBW, BPG, WM, WN, OCC, NBUF, TAIL>;
  const int grid = (B + C::BPW - 1) / C::BPW;
  hipLaunchKernelGGL((az_net_kernel<MK, F, MBW, BPG, WM, WN, OCC, NBUF, TAIL>), dim3(grid), dim3(C::NT), 0, s,
                     n, planes, legal, B, policy, value);
  return hipGetLastError();
}

// Deepest weight ring of at most `want` groups that tiles two layers of `ns` groups.
constexpr int ring_depth(int want, int ns) {
  return want <= 2 ? 2 : ((2 * ns) % want == 0 ? want : ring_depth(want - 1, ns));
}

// Weight ring depth N (groups of three dy) and tail T per tiling.  A group is 704
// MFMA cycles in the large tiling, 384 in the medium and 192 in the small one; the
// ring covers a load from the Infinity Cache (about 1,000 cycles) where the
// registers allow.  Measured on 20x128, us per batch:
//   int8 large, 768 boards: (N, T) = (8, 0) 251, (8, 4) 238, (8, 6) 241, (12, 8) 270
//     (the tail hides half the epilogue; past six groups its registers crowd out
//     the prefetch); 1,024 boards, where the clock gives way: 286, 281, 281, 298
//   int8 medium, 512 boards: (4, 0) 166, (4, 2) 164; small, 64: (8, 0) 86, (12, 0) 88
//   bf16 large, 768 boards: (4, 0) 411, (4, 2) 393, (3, 2) 395; small, 256: (8, 0)
//     163, (6, 0) 160, (6, 3) 157; medium, 512: two workgroups per compute unit
//     with (2, 0) 313, one with (6, 3) 272 (the fp32 residual needs the registers)
//   24x256 bf16, 1,024 boards: (3, 0) 2,385, (3, 1) 2,364, (2, 1) 2,351
template <int MK, int F>
struct Sched {
  static constexpr int NS = 3 * (F / Mk<MK>::KS);
  static constexpr bool BF = MK == MK_BF16, I8 = MK == MK_I8;
  static constexpr int NL = ring_depth(BF ? (F <= 128 ? 4 : 2) : (I8 ? (F <= 128 ? 8 : 4) : (F <= 128 ? 3 : 2)), NS);
  static constexpr int OM = BF && F == 128 ? 1 : 2;  // medium: workgroups per compute unit
  static constexpr int NM = ring_depth(BF ? (OM == 1 ? 6 : 2) : (I8 ? 4 : 2), NS);
  static constexpr int NSM = ring_depth(BF ? 6 : (I8 ? (F <= 128 ? 8 : 6) : 3), NS);
  static constexpr int TL = NL / 2, TM = NM / 2, TSM = BF ? NSM / 2 : 0;
};

// Tilings (wave tile = MBW*32 channels x BPG boards):
//   1 large:  4 boards per workgroup (2 for F = 256)
//   2 small:  1 board per workgroup
//   3 medium: 2 boards per workgroup (F = 64, 128), two workgroups per compute unit
//             but for bf16 with 128 filters
template <int MK, int F>
hipError_t launch_f(int tiling, const AzDevNet& n, const float* planes, const uint8_t* legal, int B,
                    float* policy, float* value, hipStream_t s) {
  using S = Sched<MK, F>;
  if constexpr (F == 128) {
    if (tiling == 1) return launch_cfg<MK, 128, 1, 4, 4, 1, 1, S::NL, S::TL>(n, planes, legal, B, policy, value, s);
    if (tiling == 3) return launch_cfg<MK, 128, 1, 2, 4, 1, S::OM, S::NM, S::TM>(n, planes, legal, B, policy, value, s);
    return launch_cfg<MK, 128, 1, 1, 4, 1, 2, S::NSM, S::TSM>(n, planes, legal, B, policy, value, s);
  } else if constexpr (F == 256) {
    if (tiling == 1) return launch_cfg<MK, 256, 2, 2, 4, 1, 1, S::NL, S::TL>(n, planes, legal, B, policy, value, s);
    return launch_cfg<MK, 256, 2, 1, 4, 1, 1, S::NSM, S::TSM>(n, planes, legal, B, policy, value, s);
  } else {
    static_assert(F == 64, "filters");
    if (tiling == 1) return launch_cfg<MK, 64, 1, 2, 2, 2, 1, S::NL, S::TL>(n, planes, legal, B, policy, value, s);
    if (tiling == 3) return launch_cfg<MK, 64, 1, 1, 2, 2, 2, S::NM, S::TM>(n, planes, legal, B, policy, value, s);
    return launch_cfg<MK, 64, 1, 1, 2, 1, 2, S::NSM, S::TSM>(n, planes, legal, B, policy, value, s);
  }
}

template <int MK>
hipError_t launch_mk(int tiling, const AzDevNet& n, const float* planes, const uint8_t* legal, int B,
                     float* policy, float* value, hipStream_t s) {
  switch (n.filters) {
    case 64: return launch_f<MK, 64>(tiling, n, planes, legal, B, policy, value, s);
    case 128: return launch_f<MK, 128>(tiling, n, planes, legal, B, policy, value, s);
    case 256: return launch_f<MK, 256>(tiling, n, planes, legal, B, policy, value, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool az_mfma_supported(int dtype, int filters) {
  return (dtype >= 1 && dtype <= 3) && (filters == 64 || filters == 128 || filters == 256);
}

bool az_mfma_tiling_valid(int filters, int tiling) {
  return tiling == 1 || tiling == 2 || (tiling == 3 && filters != 256);
}

hipError_t az_launch_mfma(int dtype, int tiling, const AzDevNet& n, const float* planes,
                          const uint8_t* legal, int B, float* policy, float* value,
                          hipStream_t s) {
  (void)hipGetLastError();
  switch (dtype) {
    case 1: return launch_mk<MK_BF16>(tiling, n, planes, legal, B, policy, value, s);
    case 2: return launch_mk<MK_I8>(tiling, n, planes, legal, B, policy, value, s);
    case 3: return launch_mk<MK_F8>(tiling, n, planes, legal, B, policy, value, s);
    default: return hipErrorInvalidValue;
  }
}
