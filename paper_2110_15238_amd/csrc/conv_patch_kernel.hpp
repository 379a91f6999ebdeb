// Thin convolutions over many pixels: a 3x3 of at most 64 channels into at most 64, alone or with the 1x1 convolution behind it,
// and pairs of 1x1 convolutions whose first has at most 128 channels.  All weights of the first op stay in REGISTERS, output
// pixels stream through independent waves.
//
// The tiled kernels let all workgroups load, multiply and store in lockstep, and read every weight fragment from LDS once per
// 32 or 64 pixels: 64 x 64 wave tiles take 128 bytes per cycle of a compute unit's LDS, all that it has.  Here
//   * a compute unit has four waves, one per SIMD with 512 registers.  A wave keeps the whole W0 as matrix-core operands (64 x
//     9 x 64: 288 registers, 240 of them accumulation registers) and walks units of 4 x 8 output pixels of one image from end to
//     end.  LDS serves activations (once per product of 32 x 64) and W1 only: half the bytes;
//   * a unit's input patch lies in LDS as it is needed: pixels padded to an odd number of 16-byte chunks, rows to the pitch
//     that spreads a fragment over all banks, so a filter tap is a constant offset.  A patch row is loaded through a buffer descriptor
//     of that image row: what lies outside the image, on any side, is out of range and reads as zeros, without a mask;
//   * no barrier in the loop.  The next unit's patch is in flight, and op1, the output's way through a piece of LDS of the wave's
//     own and its stores go between the products of the next unit's op0 (3x3 of stride 1);
//   * bias in the accumulators from the start, ReLU on packed halves: one vector instruction per output value.  One wave per SIMD
//     issues one instruction every 4 cycles, so instructions are what the loop is short of (a first form with 1740 per unit
//     took 13400 cycles for it; 700 are left).
// What bounds it: the chain of one wave per SIMD, neither memory nor a pipe.  64 -> 64 -> 256 at 56 x 56, batch 32, moves its 64 MB at 3.3 to 3.5 TB/s
// (a large copy: 4.9; the 1x1 pairs here: 4.5), the matrix cores are busy for 31 % of the SIMDs' cycles, vector instructions for 16 % and
// LDS for 31 %; a wave waits for loads, LDS and the places of its stores for 42 % of its life, and its 3584 units of 7 columns are 3.5 rounds.  Below 8
// images, the fill: weights, first patch and a unit's chain of products take 5 us (64 channels) beside the launch.
// Its residual: single ops fetch it one unit ahead of the output.  Other activations than ReLU and alpha != 1 run without the overlap (GEN).
// Measured under a HIP graph, best tiled instance -> this one, us: 3x3 -> 1x1 at 56 x 56, 64 -> 64 -> 256, batch 32 24.4 -> 19.8, with a
// residual 35.0 -> 28.9, batch 8 12.9 -> 7.7; 32 -> 32 -> 128 with a residual 30.5 -> 14.3; 112 x 112, 32 -> 32 -> 128 93 -> 23.4;
// stride 2, 64 -> 64 -> 256 13.6 -> 9.2; 1x1 -> 1x1 at 56 x 56, 64 -> 64 -> 256 26.1 -> 14.4 (4.5 TB/s).  The single 3x3 at 56 x 56,
// 64 -> 64: batch 32 12.8 -> 12.0, 16 9.3 -> 7.1, 8 7.9 -> 5.2; with a residual, 15.4 -> 12.7 and 9.0 -> 5.9 at batch 32 and 8.
// Widths end at 64: the weights of 96 -> 96 would take 648 of a SIMD's 512 registers.
#pragma once
#include <algorithm>
#include <cmath>

#include "b2b_dma_kernel.hpp"

namespace bolt {

struct ConvPatchParams : B2bParams {
  int tq;        // columns of a unit
  int uq, per_img, units;     // units per row of units, per image, in all
  unsigned rcp_uq, rcp_img;   // (2^32 - 1) / uq and / per_img: quotients from them are exact or one too small
};

// RS: filter extent, 3 or 1.  ST: stride of a 3x3 filter in LDS (the pixels that a strided 1x1 filter samples lie side by side).
template <int CP, int N0T, int RS, int ST, bool PAIR>
struct ConvPatchTraits {
  static constexpr int NW = 4, NT = 64 * NW;
  static constexpr int TP = 4, TQ = 8;  // a wave's unit: TP x (at most) TQ output pixels of one image
  static constexpr int CH = CP / 8, PIT = CH | 1;  // 16-byte chunks of one pixel, and its pitch in LDS
  static constexpr int ROWS = (TP - 1) * ST + RS, COLS = (TQ - 1) * ST + RS;
  static constexpr int RI = (COLS * PIT + 63) / 64;  // load instructions of a patch row
  static constexpr bool MASK = ST == 2;  // the last one is cut short where whole ones do not fit LDS
  static constexpr int TAIL = COLS * PIT - (RI - 1) * 64;
  // Chunks from one patch row to the next.  The 16 pixels of a half fragment are in two rows, 8 pixels next to each other in
  // each: with this pitch they fall into 16 (stride 2: 8) different 16-byte bank groups.
  static constexpr int row_pitch() {
    int r = MASK ? COLS * PIT : RI * 64;
    while (ST == 1 ? r % 16 != 8 : r % 8 != 4) ++r;
    return r;
  }
  static constexpr int RP = row_pitch();
  static constexpr int PATCH = (ROWS * RP * 16 + 1023) / 1024 * 1024;
  // Weights of op0 in LDS: blocks of [output channel][CHW chunks], one per tap and 64 channels
  static constexpr int CHW = CP > 32 || N0T == 32 ? 8 : 4, KT = (CH + CHW - 1) / CHW;
  static constexpr int IPT = N0T * CHW / 64 / NW;  // load instructions of a block per wave
  static constexpr int W0_BYTES = RS * RS * KT * N0T * CHW * 16;
  static constexpr int KC = CP / 16, KS = RS * RS * KC, FN0 = N0T / 32;
  static constexpr int NC = 64;      // columns of op1 per step
  static constexpr int W1I = NC * N0T / 8 / 64 / NW;  // load instructions of those per wave
  static constexpr int OUT = 32 * NC * 2;  // staged output of one wave
  static constexpr int BIAS = (N0T + 256) * 4;
  // A unit's op1 and output go beside the next unit's op0 where that is long enough; its patch then needs a second buffer.
  static constexpr bool OVERLAP = RS == 3 && ST == 1;
  static constexpr int NBUF = OVERLAP ? 2 : 1;
  // LDS: biases, W1, then the waves' part: first patches, second patches, staged outputs.  W0 passes through the place of the
  // latter two, and of the first patches where there is no room otherwise (those are then requested behind it).
  static constexpr int WAVES_BYTES = NW * (NBUF * PATCH + OUT);
  static constexpr bool EARLY = BIAS + (PAIR ? 256 * N0T * 2 : 0) + NW * PATCH + W0_BYTES <= 160 * 1024;
  static constexpr int W0_AT = EARLY ? NW * PATCH : 0;  // (relative to the waves' part)
  static constexpr int DYN = WAVES_BYTES > W0_AT + W0_BYTES ? WAVES_BYTES : W0_AT + W0_BYTES;
  static_assert(CP % 16 == 0 && (N0T == 32 || N0T == 64) && (ST == 1 || (ST == 2 && RS == 3)) && (RS == 1 || RS == 3), "instance");
  static_assert(IPT >= 1 && W1I >= 1, "weights split evenly over the waves");
  static_assert(BIAS + (PAIR ? 256 * N0T * 2 : 0) + DYN <= 160 * 1024, "LDS");
  static_assert(EARLY || !OVERLAP, "the overlapped form reads the first weights beside the first unit's products");
  // chunk slot of patch column c inside a patch row: with stride 2 the even columns come first, so that the pixels of a
  // fragment are neighbours again
  static constexpr int col_slot(int c) { return ST == 1 ? c : (c & 1) * ((COLS + 1) / 2) + (c >> 1); }

  static int lds_bytes_n(int n1) { return BIAS + (PAIR ? (n1 + NC - 1) / NC * NC * N0T * 2 : 0) + DYN; }
  static void plan(const B2bParams& p, int tq, ConvPatchParams& q) {
    q.tq = tq;
    q.uq = (p.cg.Q + tq - 1) / tq;
    q.per_img = q.uq * ((p.cg.P + TP - 1) / TP);
    q.units = p.M / (p.cg.P * p.cg.Q) * q.per_img;
    q.rcp_uq = 0xffffffffu / (unsigned)q.uq;
    q.rcp_img = 0xffffffffu / (unsigned)q.per_img;
  }
  static constexpr int MOST_WGS = 256;  // one per compute unit
  // Columns of a unit: as many rounds as the units take on the chip's waves, each at half a full unit's cost plus the columns'
  // share (56 x 56 at batch 32: 3136 units of 8 columns are 3.06 per wave, four rounds with the last one empty; of 7, 3.5).
  static ConvPatchParams plan(const B2bParams& p) {
    ConvPatchParams best{}, q{};
    static_cast<B2bParams&>(best) = p;
    int best_cost = 0;
    for (int tq = TQ; tq >= 6; --tq) {
      plan(p, tq, q);
      const int cost = (q.units + MOST_WGS * NW - 1) / (MOST_WGS * NW) * (TQ + tq);
      if (tq == TQ || cost < best_cost) { plan(p, tq, best); best_cost = cost; }
    }
    return best;
  }
  // What the overlapped loop computes: ReLU or nothing, the products as they are.  Everything else runs on the general form of the
  // kernel if a config says so; the pick rule's costs are those of the plain one.
  static bool plain(const B2bParams& p) { return p.act0 <= ACT_RELU && p.act1 <= ACT_RELU && p.alpha0 == 1.f && p.alpha1 == 1.f; }
  static bool plain_single(const FpropParams& f) { return plain(from_single(f)); }
  static bool supports(const B2bParams& p) {
    const ConvGeom& g = p.cg;
    if (g.R != RS || g.S != RS || g.stride_h != g.stride_w || g.pad_h > 2 || g.pad_w > 2 || g.C % 8 != 0) return false;
    if (RS == 3 ? g.stride_h != ST : g.stride_h > 2) return false;
    return g.C <= CP && p.N0 <= N0T && p.N1 <= 256 && lds_bytes_n(p.N1) <= 160 * 1024;
  }
  static int lds_bytes(const B2bParams& p) { return lds_bytes_n(p.N1); }
  // the single op: its epilogue is op0's, and so is its residual
  static B2bParams from_single(const FpropParams& f) {
    B2bParams p{};
    p.X = f.X; p.W0 = f.W; p.b0 = f.bias; p.b0_on = f.bias_on; p.Y = f.Y; p.res = f.res; p.ldr = f.ldr; p.gamma = f.gamma;
    p.M = f.M; p.N0 = p.N1 = f.N; p.K0 = f.K; p.ldw0 = f.ldw; p.ldy = f.ldy;
    p.alpha0 = f.alpha; p.beta0 = f.beta; p.act0 = f.act; p.alpha1 = 1.f; p.cg = f.cg;
    return p;
  }
  static bool supports_single(const FpropParams& f) { return supports(from_single(f)); }
  static int lds_bytes_single(const FpropParams&) { return lds_bytes_n(0); }
  // Pick rule, us of a pair: the fill, then rounds of units, each with its products of 32 x 32 x 16, the load instructions of a patch, and
  // per 64 columns of op1 the store, the residual and the products; and what memory moves.  A unit that an image does not fill costs
  // as much as a full one.  (3998 pairs, images of 1 x 1 to 112 x 112, 1000 to 300000 pixels, with and without a residual: 6 % off, nine of
  // ten within 9 %.)
  static double estimate_pair(const B2bParams& p, bool residual) {
    if (!plain(p)) return HUGE_VAL;
    const int rounds = (plan(p).units + MOST_WGS * NW - 1) / (MOST_WGS * NW), chunks = (p.N1 + NC - 1) / NC;
    const double round = 0.07 + 0.018 * (KS * FN0) + 0.033 * (ROWS * RI) + chunks * (0.38 + 0.075 * FN0 + (residual ? 0.42 : 0.0));
    return 3.2 + rounds * round + 0.049 * b2b_conv_mbytes(p, residual);
  }
  // Pick rule, us: the fill with the first unit, then a round per unit and wave (from 28 problems, 1 to 7 rounds).  A single round
  // takes 3.7 or 4.9 too, but stands against the kernels for small problems, whose estimates are up to 1.1 us too high here: of 83
  // problems that the two numbers took from them, 32 ran 1.02 to 1.14 times as long (550 pixels, 8 -> 32: 3.6 -> 4.1 us).
  static double estimate(const FpropParams& f) {
    const int rounds = (plan(from_single(f)).units + MOST_WGS * NW - 1) / (MOST_WGS * NW);
    if (rounds == 1) return CP > 32 ? 5.2 : 4.6;
    return CP > 32 ? 4.9 + 2.3 * (rounds - 1) : 3.7 + 1.5 * (rounds - 1);
  }
};

#if defined(__HIP_DEVICE_COMPILE__)
// max(v, lo) of two halves; lo = NaN: v
__device__ __forceinline__ half2v pk_max(half2v v, unsigned lo) {
  half2v r;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(v), "s"(lo));
  return r;
}
#endif

// GEN: any activation and any alpha, the epilogues in single precision and one unit after the other.
template <int CP, int N0T, int RS, int ST, bool PAIR, bool RES, bool GEN, bool SHARE = false>
__global__ __launch_bounds__(256, 1) void conv_patch_kernel(const ConvPatchParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
  using T = ConvPatchTraits<CP, N0T, RS, ST, PAIR>;
  constexpr int NW = T::NW, RI = T::RI, KC = T::KC, KS = T::KS, FN0 = T::FN0, CHW = T::CHW, PIT = T::PIT, RP = T::RP, NC = T::NC;
  extern __shared__ __attribute__((aligned(16))) half_t lds[];
  const ConvGeom& cg = p.cg;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* const bias0 = reinterpret_cast<float*>(lds);  // beta * bias, zeros beyond the columns
  float* const bias1 = bias0 + N0T;
  const int nch = PAIR ? (p.N1 + NC - 1) / NC : 1;
  half_t* const W1s = lds + T::BIAS / 2;
  half_t* const dyn = W1s + (PAIR ? nch * NC * N0T : 0);
  half_t* const W0s = dyn + T::W0_AT / 2;
  half_t* const patch0 = dyn + wave * (T::PATCH / 2);
  half_t* const out = dyn + (T::NBUF * NW * T::PATCH + wave * T::OUT) / 2;

  // ---- biases to registers, weights of op0 to LDS: [tap][output channel][CHW chunks], XOR-swizzled ---------------------------------
  float hb0 = 0.f, hb1 = 0.f;  // (256 threads: one column each)
  if (tid < p.N0) hb0 = p.beta0 * (float)p.b0[tid * p.b0_on];
  if (PAIR && tid < p.N1) hb1 = p.beta1 * (float)p.b1[tid * p.b1_on];
  {
    // a tap is an offset of the whole instruction, so a lane has one offset per group of rows
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.W0, (unsigned)(((p.N0 - 1) * p.ldw0 + p.K0) * 2));
    constexpr int RPI = 64 / CHW;
#pragma unroll
    for (int i = 0; i < T::IPT; ++i)
#pragma unroll
      for (int kt = 0; kt < T::KT; ++kt) {
        const int row = (i * NW + wave) * RPI + lane / CHW, ch = kt * CHW + ((lane % CHW) ^ dma_swizzle<CHW * 8>(row));
        const unsigned off = ((row < p.N0) & (ch * 8 < cg.C)) ? (unsigned)(row * p.ldw0 + ch * 8) * 2u : kInvalidOffset;
#pragma unroll
        for (int tap = 0; tap < RS * RS; ++tap)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, BOLT_LDS_PTR(W0s + (tap * T::KT + kt) * N0T * CHW * 8 + (i * NW + wave) * 512), 16, off,
                                                   tap * cg.C * 2, 0, 0);
      }
  }

  // ---- units of this wave: every XCD (ids are dealt round-robin over 8) takes a contiguous run ---------------------------------
  struct Unit {
    int img, p0, q0;
  };
  auto unit_at = [&](int u) {
    Unit t;
    t.img = (int)__umulhi((unsigned)u, p.rcp_img);
    int r = u - t.img * p.per_img;
    if (r >= p.per_img) { r -= p.per_img; ++t.img; }
    int pp = (int)__umulhi((unsigned)r, p.rcp_uq), q = r - pp * p.uq;
    if (q >= p.uq) { q -= p.uq; ++pp; }
    t.p0 = pp * T::TP;
    t.q0 = q * p.tq;
    return t;
  };
  const int grid = (int)gridDim.x, nx = grid < 8 ? grid : 8;
  const int xcd = grid < 8 ? (int)blockIdx.x : (int)blockIdx.x & 7, wg = grid < 8 ? 0 : (int)blockIdx.x >> 3;
  const int per = p.units / nx, rem = p.units - per * nx;
  const int u_end = __builtin_amdgcn_readfirstlane(per * (xcd + 1) + (xcd + 1 < rem ? xcd + 1 : rem));
  const int step = grid < 8 ? NW : ((grid - xcd + 7) >> 3) * NW;
  const int u_first = per * xcd + (xcd < rem ? xcd : rem);
  int u = __builtin_amdgcn_readfirstlane(u_first + wg * NW + wave);
  // SHARE: the units behind the last whole round, where there are some for half of the waves at most, are taken by two to four waves
  // together, each with its share of the columns of op1 (op0 they all compute).  They would be all that runs for a while, and the residual
  // makes their outputs long.  64 -> 64 -> 256 with a skip connection, not shared -> shared, us: 56 x 56, 32 images, 3584 units for 1024 waves, by two
  // 31.3 -> 30.3; 28 x 8, 217 images, 1519 units, by two 16.7 -> 15.2; 192 images, by three 15.7 -> 14.3; 147 and 300 images, by four 13.5 -> 12.1
  // and 23.8 -> 21.1; stride 2 by four 18.4 -> 16.4; 1 x 1 by four 11.2 -> 9.3.  (Without a residual nothing was won at 56 x 56, by two, 21.0 us either
  // way; shares of three and four were not measured without one.  Where no unit is shared the code cost 0 to 3 %.)
  constexpr int WAVES = T::MOST_WGS / 8 * NW;  // of an XCD in a launch whose waves have several units
  static_assert((WAVES & (WAVES - 1)) == 0, "whole rounds by a mask");
  const int left = (u_end - u_first) & (WAVES - 1), tail = u_end - left;
  int share = 1;
  if (SHARE && step == WAVES && tail > u_first && nch > 1) share = left * 4 <= WAVES && nch > 3 ? 4 : left * 3 <= WAVES && nch > 2 ? 3 : left * 2 <= WAVES ? 2 : 1;
  const int rcp_share = share == 1 ? 1 << 17 : share == 2 ? 1 << 16 : share == 3 ? 43691 : 1 << 15;  // (exact below 2^15)
  int c_first = 0, c_end = nch;  // columns of the last unit, in 64s
  auto next_of = [&](int at) {  // this wave's unit behind unit `at`
    int n = at + step;
    if (SHARE && share > 1 && n >= tail) n = at >= tail ? u_end : tail + ((n - tail) * rcp_share >> 17);
    return n;
  };
  auto part_of_last = [&](int at) {
    if (SHARE && share > 1 && at >= tail) {
      const int w = wg * NW + wave, part = w - (w * rcp_share >> 17) * share;
      c_first = part * nch * rcp_share >> 17;
      c_end = (part + 1) * nch * rcp_share >> 17;
    }
  };

  // ---- patches: one row at a time through a descriptor of that image row, so that whatever lies outside the image, on any
  // side, is beyond the buffer and reads as zeros ---------------------------------------------------------------------------------
  const int row_bytes = cg.Wi * cg.C * 2, gst = RS == 1 ? cg.stride_h : 1;  // gst: image rows and columns per patch row and column
  unsigned pat[RI];  // byte offset of this lane's chunk in a row, from the patch's first column
#pragma unroll
  for (int h = 0; h < RI; ++h) {
    const int j = h * 64 + lane, slot = (int)(__umul24((unsigned)j, 65536u / PIT + 1) >> 16), ch = j - slot * PIT;
    const int col = ST == 1 ? slot : slot < (T::COLS + 1) / 2 ? 2 * slot : 2 * (slot - (T::COLS + 1) / 2) + 1;
    const bool ok = (slot < T::COLS) & (col < (p.tq - 1) * ST + RS) & (ch * 8 < cg.C);
    pat[h] = ok ? (unsigned)(__umul24(col * gst, cg.C) + ch * 8) * 2u : kInvalidOffset;
  }
  struct Patch {
    const char* row0;  // the image row of the patch's first row (it may lie outside the image)
    int h0;
    unsigned at[RI];
  };
  auto patch_of = [&](const Unit& t, bool on) {  // (off: all of it outside the image, no traffic)
    Patch s;
    s.h0 = t.p0 * ST * gst - cg.pad_h;
    s.row0 = reinterpret_cast<const char*>(p.X) + (int64_t)(t.img * cg.H + s.h0) * row_bytes;
#pragma unroll
    for (int h = 0; h < RI; ++h) s.at[h] = pat[h] + (unsigned)((t.q0 * ST * gst - cg.pad_w) * cg.C * 2);
    if (!on) s.h0 = -(1 << 20);
    return s;
  };
  auto issue_row = [&](const Patch& s, int r, half_t* dst) {
    const bool ok = (unsigned)(s.h0 + r * gst) < (unsigned)cg.H;
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(s.row0 + (int64_t)(r * gst) * row_bytes, ok ? (unsigned)row_bytes : 0u);
#pragma unroll
    for (int h = 0; h < RI; ++h)
      if (!T::MASK || h + 1 < RI || lane < T::TAIL)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, BOLT_LDS_PTR(dst + (r * RP + h * 64) * 8), 16, s.at[h], 0, 0, 0);
  };
  auto issue_patch = [&](const Patch& s, half_t* dst) {
#pragma unroll
    for (int r = 0; r < T::ROWS; ++r) issue_row(s, r, dst);
  };
  const Unit first = unit_at(u);
  const Patch first_patch = patch_of(first, u < u_end);
  if constexpr (T::EARLY) issue_patch(first_patch, patch0);

  // ---- weights of op1: [64 columns][output channel][input channels], XOR-swizzled --------------------------------------------------
  if constexpr (PAIR) {
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.W1, (unsigned)(((p.N1 - 1) * p.ldw1 + p.N0) * 2));
    constexpr int CH1 = N0T / 8, RPI = 64 / CH1;
    const int row = wave * RPI + lane / CH1, ch = (lane % CH1) ^ dma_swizzle<N0T>(row);
    unsigned off = ch * 8 < p.N0 ? (unsigned)(row * p.ldw1 + ch * 8) * 2u : kInvalidOffset;
    for (int i = 0; i < nch * T::W1I; ++i) {  // (rows past N1 lie beyond the buffer)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, BOLT_LDS_PTR(W1s + (i * NW + wave) * 512), 16, off, 0, 0, 0);
      off += ch * 8 < p.N0 ? (unsigned)(RPI * NW * p.ldw1) * 2u : 0u;
    }
  }
  if (tid < N0T) bias0[tid] = hb0;
  if (PAIR && tid < nch * NC) bias1[tid] = hb1;
  // W0 and this wave's patch have landed (W1 may be on its way)
  if (!PAIR || nch == 1) barrier_after_reads_and_loads<PAIR ? T::W1I : 0>();
  else if (nch == 2) barrier_after_reads_and_loads<2 * T::W1I>();
  else if (nch == 3) barrier_after_reads_and_loads<3 * T::W1I>();
  else barrier_after_reads_and_loads<4 * T::W1I>();

  // Fragment (tap, 16 channels) of 32 output channels of W0.  Row i of a fragment is output channel i with bits 2
  // and 3 exchanged: a lane's accumulators 8t .. 8t + 7 are then channels 16t + 8g .. + 7, in order, which is both the
  // operand order of op1 and a 16-byte chunk of the output.
  const int n32 = (l32 & 0x13) | (l32 & 4) << 1 | (l32 & 8) >> 1;
  half8 wf[KS][FN0];
  auto read_wf = [&](int k) {
#pragma unroll
    for (int a = 0; a < FN0; ++a)
      wf[k][a] = *(const half8*)(W0s + ((k / KC) * T::KT + (k % KC) * 2 / CHW) * N0T * CHW * 8 +
                                 dma_chunk_offset<CHW * 8>(a * 32 + n32, (k % KC) * 2 % CHW + g));
#pragma unroll
    for (int a = 0; a < FN0; ++a)
      if (k * FN0 + a < 60) asm volatile("" : "+a"(wf[k][a]));
  };
  // ---- op0 of one unit, in steps of 16 channels of one tap; fragments of the activations are read D steps ahead --------------------
  constexpr int D = KS < 4 ? KS : 4;
  const int x_at = ((l32 >> 3) * ST * RP + (l32 & 7) * PIT + g) * 8;  // this lane's pixel inside the patch
  floatx16 acc0[FN0];
  half8 xq[D];
  auto set_bias = [&](floatx16& acc, const float* bias) {  // 32 columns: the accumulators start from the bias
    if constexpr (GEN) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = 0.f;
      return;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const floatx4 b = *(const floatx4*)(bias + t * 16 + g * 8 + h * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t * 8 + h * 4 + e] = b[e];
      }
  };
  auto read_x = [&](const half_t* xs, int k) {
    const int tap = k / KC, r = tap / RS, s = tap % RS;
    xq[k % D] = *(const half8*)(xs + (r * RP + T::col_slot(s) * PIT + (k % KC) * 2) * 8);
  };
  auto op0_start = [&](const half_t* xs) {
#pragma unroll
    for (int k = 0; k < D; ++k) read_x(xs, k);
#pragma unroll
    for (int a = 0; a < FN0; ++a) set_bias(acc0[a], bias0 + a * 32);
  };
  auto op0_step = [&](const half_t* xs, int k) {
#pragma unroll
    for (int a = 0; a < FN0; ++a) acc0[a] = mfma_32x32x16(wf[k][a], xq[k % D], acc0[a]);
    if (k + D < KS) read_x(xs, k + D);
  };
  const unsigned lo0 = p.act0 == ACT_RELU ? 0u : 0x7e007e00u, lo1 = p.act1 == ACT_RELU ? 0u : 0x7e007e00u;
  constexpr bool RES1 = RES && PAIR, RES0 = RES && !PAIR;  // the op that the residual goes to
  auto stage_at = [&](int row, int chunk) { return out + row * NC + ((chunk ^ ((row >> 1) & 7)) << 3); };
  // act(alpha acc + beta bias + gamma res) of accumulators 8t .. 8t + 7
  auto general = [&](const floatx16& acc, int t, const float* bias, half8 rs, float gamma, float alpha, int act) {
    half8 o;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const floatx4 b = *(const floatx4*)(bias + t * 16 + g * 8 + h * 4);
      floatx4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = alpha * acc[t * 8 + h * 4 + e] + b[e] + gamma * (float)rs[h * 4 + e];
      if (act > ACT_RELU) {
        v = apply_act_slow4_inline(v, act);
      } else {
        const float lo = relu_bound(act);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = at_least(v[e], lo);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) o[h * 4 + e] = (half_t)v[e];
    }
    return o;
  };
  half8 d[FN0 * 2];
  auto make_d = [&]() {  // the hand-over: op0's output as op1's operand
#pragma unroll
    for (int a = 0; a < FN0; ++a)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        half8 rs = {0, 0, 0, 0, 0, 0, 0, 0};
        if constexpr (RES0) rs = *(const half8*)stage_at(l32, a * 4 + t * 2 + g);
        if constexpr (GEN) {
          d[a * 2 + t] = general(acc0[a], t, bias0 + a * 32, rs, RES0 ? p.gamma : 0.f, p.alpha0, p.act0);
          continue;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float v0 = acc0[a][t * 8 + 2 * e], v1 = acc0[a][t * 8 + 2 * e + 1];
          if constexpr (RES0) {
            v0 += p.gamma * (float)rs[2 * e];
            v1 += p.gamma * (float)rs[2 * e + 1];
          }
          const half2v v = pk_max(half2v{(half_t)v0, (half_t)v1}, lo0);
          d[a * 2 + t][2 * e] = v[0];
          d[a * 2 + t][2 * e + 1] = v[1];
        }
      }
  };

  // ---- 64 columns of op1 out, through this wave's piece of LDS (one wave's LDS accesses are served in order) ------------------------
  __amdgpu_buffer_rsrc_t yr, rr;
  unsigned y_at, r_at;     // this lane's 16 bytes of the unit's first output row: lanes 8j .. 8j + 7 take pixel j
  int rows_out, rows_res;  // output rows of the unit
  // 16 bytes per lane of an [M][ld] matrix at a unit: its descriptor, and this lane's offset in the first row
  auto set_rows = [&](const Unit& t, const half_t* base, int ld, __amdgpu_buffer_rsrc_t& desc, unsigned& at, int& rows) {
    const int64_t m_at = ((int64_t)t.img * cg.P + t.p0) * cg.Q + t.q0;
    const int64_t rem = ((int64_t)(p.M - m_at - 1) * ld + p.N1) * 2;
    desc = make_rsrc(base + m_at * ld, (unsigned)(rem < 0x7fffffff ? rem : 0x7fffffff));
    rows = cg.P - t.p0;
    const int j = lane >> 3;
    at = ((t.q0 + j < cg.Q) & (j < p.tq)) ? (unsigned)(j * ld + (lane & 7) * 8) * 2u : kInvalidOffset;
  };
  auto set_res = [&](const Unit& t) { set_rows(t, p.res, p.ldr, rr, r_at, rows_res); };
  auto set_out = [&](const Unit& t) {
    set_rows(t, p.Y, p.ldy, yr, y_at, rows_out);
    if constexpr (RES1) set_res(t);
  };
  auto row_offset = [&](int i, int c, unsigned at, int ld, int rows) {
    const bool ok = (i < rows) & (c * NC + (lane & 7) * 8 < p.N1);
    return ok ? at + (unsigned)(i * cg.Q * ld + c * NC) * 2u : kInvalidOffset;
  };
  uintx4 rv[RES ? 4 : 1];
  auto fetch_res = [&](int c) {
    if constexpr (RES) {
#pragma unroll
      for (int i = 0; i < 4; ++i) rv[i] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(rr, row_offset(i, c, r_at, p.ldr, rows_res), 0, 0));
    }
  };
  auto stage_res = [&]() {
    if constexpr (RES) {
#pragma unroll
      for (int i = 0; i < 4; ++i) *(uintx4*)stage_at(i * 8 + (lane >> 3), lane & 7) = rv[i];
      asm volatile("" ::: "memory");
    }
  };
  floatx16 acc1[2];
  auto octet_out = [&](int i, int c) {  // octet i = 0 .. 3 of this lane's 32 values of the 64 columns
    const int a = i >> 1, t = i & 1;
    half8* const slot = (half8*)stage_at(l32, a * 4 + t * 2 + g);
    if constexpr (!PAIR) {
      *slot = d[i];
      return;
    }
    half8 rs = {0, 0, 0, 0, 0, 0, 0, 0}, o;
    if constexpr (RES1) rs = *slot;
    if constexpr (GEN) {
      *slot = general(acc1[a], t, bias1 + c * NC + a * 32, rs, RES1 ? p.gamma : 0.f, p.alpha1, p.act1);
      return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v0 = acc1[a][t * 8 + 2 * e], v1 = acc1[a][t * 8 + 2 * e + 1];
      if constexpr (RES1) {
        v0 += p.gamma * (float)rs[2 * e];
        v1 += p.gamma * (float)rs[2 * e + 1];
      }
      const half2v v = pk_max(half2v{(half_t)v0, (half_t)v1}, lo1);
      o[2 * e] = v[0];
      o[2 * e + 1] = v[1];
    }
    *slot = o;
  };
  const bool whole_lines = p.ldy % 64 == 0;
  auto store_out = [&](int c) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uintx4 v = *(const uintx4*)stage_at(i * 8 + (lane >> 3), lane & 7);
      // non-temporal, except where a cache line is shared by columns that are stored at different times
      if (whole_lines) __builtin_amdgcn_raw_buffer_store_b128(v, yr, row_offset(i, c, y_at, p.ldy, rows_out), 0, 2);
      else __builtin_amdgcn_raw_buffer_store_b128(v, yr, row_offset(i, c, y_at, p.ldy, rows_out), 0, 0);
    }
    asm volatile("" ::: "memory");
  };
  auto op1 = [&](int c) {
    if constexpr (!PAIR) return;
    const half_t* const ws = W1s + c * NC * N0T;
    half8 w1f[FN0 * 2][2];
#pragma unroll
    for (int t = 0; t < FN0 * 2; ++t)
#pragma unroll
      for (int a = 0; a < 2; ++a) w1f[t][a] = *(const half8*)(ws + dma_chunk_offset<N0T>(a * 32 + n32, 2 * t + g));
#pragma unroll
    for (int a = 0; a < 2; ++a) set_bias(acc1[a], bias1 + c * NC + a * 32);
#pragma unroll
    for (int t = 0; t < FN0 * 2; ++t)
#pragma unroll
      for (int a = 0; a < 2; ++a) acc1[a] = mfma_32x32x16(w1f[t][a], d[t], acc1[a]);
  };

  auto all_out = [&]() {  // op1 and output of the unit in d
    if constexpr (RES1) fetch_res(c_first);
    for (int c = c_first; c < c_end; ++c) {
      if constexpr (RES1) stage_res();
      op1(c);
#pragma unroll
      for (int q = 0; q < 4; ++q) octet_out(q, c);
      store_out(c);
      if constexpr (RES1)
        if (c + 1 < c_end) fetch_res(c + 1);
    }
  };
  auto wait_patch = [&]() {
    // the next patch has landed: it is older than the stores of all columns
    if (nch == 1) __builtin_amdgcn_s_waitcnt(0x0F70 | 4);
    else if (nch == 2) __builtin_amdgcn_s_waitcnt(0x0F70 | 8);
    else if (nch == 3) __builtin_amdgcn_s_waitcnt(0x0F70 | 12);
    else __builtin_amdgcn_s_waitcnt(0x0F70 | 1 << 14);
    asm volatile("" ::: "memory");
  };

  if constexpr (T::OVERLAP && !GEN) {
    // ---- first unit: the weights go to registers on the way
#pragma unroll
    for (int k = 0; k < D; ++k) read_wf(k);
    op0_start(patch0 + x_at);
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      __builtin_amdgcn_sched_barrier(0);
      if (k + D < KS) read_wf(k + D);
      op0_step(patch0 + x_at, k);
    }
    barrier_after_reads_and_loads<0>();  // W0's place is free, W1 is there
    if (u >= u_end) return;              // (no barrier follows)

    int buf = 0;
    Unit cur = first;
    int un = next_of(u);
    Unit nxt = unit_at(un);
    if constexpr (RES0) {
      set_res(cur);
      fetch_res(0);
    }
    issue_patch(patch_of(nxt, un < u_end), patch0 + NW * T::PATCH / 2);
    if constexpr (RES0) stage_res();
    make_d();
    __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("" ::: "memory");
    while (un < u_end) {
      // d: the unit cur, its op1 and output in up to four segments, each beside a quarter of the next unit's op0
      const int un2 = next_of(un);
      const Unit nxt2 = unit_at(un2);
      const Patch np = patch_of(nxt2, un2 < u_end);
      half_t* const x_next = patch0 + buf * (NW * T::PATCH / 2);
      buf ^= 1;
      const half_t* const xs = patch0 + buf * (NW * T::PATCH / 2) + x_at;
      set_out(cur);
      if constexpr (RES0) set_res(nxt);  // (one unit ahead of the output: it goes to op0's results)
      if constexpr (RES) fetch_res(0);
      op0_start(xs);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k0 = KS * s / 4, k1 = KS * (s + 1) / 4;
        auto segment = [&](auto with_out) {
          constexpr bool OUT_TOO = decltype(with_out)::value;
          if constexpr (OUT_TOO) {
            if constexpr (RES1) stage_res();
            op1(s);
          }
          int q = 0, r = 0;
#pragma unroll
          for (int k = k0; k < k1; ++k) {
            __builtin_amdgcn_sched_barrier(0);
            op0_step(xs, k);
            if (s == 0) {  // all of the next patch's loads are older than this unit's stores
#pragma unroll
              for (; r < ((k - k0 + 1) * T::ROWS) / (k1 - k0); ++r) issue_row(np, r, x_next);
            }
            if constexpr (OUT_TOO) {  // (two products of op0 and more stand between those of op1 and the use of their results)
              if (k > k0) {
#pragma unroll
                for (; q < ((k - k0) * 4) / (k1 - k0 - 1); ++q) octet_out(q, s);
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (OUT_TOO) {
            store_out(s);
            if constexpr (RES1)
              if (s + 1 < nch) fetch_res(s + 1);
          }
        };
        if (s == 0 || s < nch) segment(std::true_type{});
        else segment(std::false_type{});
      }
      if constexpr (RES0) stage_res();  // (the stored unit has left the place)
      make_d();
      wait_patch();
      cur = nxt;
      u = un;
      un = un2;
      nxt = nxt2;
    }
    set_out(cur);
    part_of_last(u);
    all_out();
  } else {
    // ---- one unit after the other: the next patch is requested as soon as op0 has read the last one
#pragma unroll
    for (int k = 0; k < KS; ++k) read_wf(k);
    barrier_after_reads_and_loads<0>();  // W0's place is free, W1 is there
    if (u >= u_end) return;              // (no barrier follows)
    if constexpr (!T::EARLY) {
      issue_patch(first_patch, patch0);
      __builtin_amdgcn_s_waitcnt(0x0F70);
      asm volatile("" ::: "memory");
    }
    Unit cur = first;
    for (;;) {
      op0_start(patch0 + x_at);
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        __builtin_amdgcn_sched_barrier(0);
        op0_step(patch0 + x_at, k);
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);  // the patch has been read
      asm volatile("" ::: "memory");
      const int un = next_of(u);
      const Unit nxt = unit_at(un);
      issue_patch(patch_of(nxt, un < u_end), patch0);
      if constexpr (RES0) {
        set_res(cur);
        fetch_res(0);
        stage_res();
      }
      make_d();
      set_out(cur);
      part_of_last(u);
      all_out();
      if (un >= u_end) break;
      wait_patch();
      u = un;
      cur = nxt;
    }
  }
#endif
}

template <int CP, int N0T, int RS, int ST, bool PAIR>
hipError_t launch_conv_patch(const B2bParams& p, int /*grid*/, int lds_bytes, hipStream_t stream) {
  using T = ConvPatchTraits<CP, N0T, RS, ST, PAIR>;
  static LdsOptIn opt_in[4];
  const bool res = p.res != nullptr, gen = !T::plain(p);
  auto kern = gen ? (res ? conv_patch_kernel<CP, N0T, RS, ST, PAIR, true, true> : conv_patch_kernel<CP, N0T, RS, ST, PAIR, false, true>)
                  : (res ? conv_patch_kernel<CP, N0T, RS, ST, PAIR, true, false> : conv_patch_kernel<CP, N0T, RS, ST, PAIR, false, false>);
  if (hipError_t e = opt_in[gen * 2 + res].ensure((const void*)kern, 160 * 1024); e != hipSuccess) return e;
  const ConvPatchParams q = T::plan(p);
  // (every XCD, ids are dealt round-robin over 8, has the same number of waves for its eighth of the units)
  int grid = std::min((q.units + T::NW - 1) / T::NW, T::MOST_WGS);
  if (grid > 8) grid = (grid + 7) / 8 * 8;
  if constexpr (PAIR) {
    // an XCD's units behind the last whole round of its waves; XCDs differ by one unit at most
    const int waves = T::MOST_WGS / 8 * T::NW, left = (q.units + 7) / 8 % waves;
    if (res && p.N1 > 64 && grid == T::MOST_WGS && q.units >= 8 * waves && left > 0 && left * 2 <= waves) {
      kern = gen ? conv_patch_kernel<CP, N0T, RS, ST, true, true, true, true> : conv_patch_kernel<CP, N0T, RS, ST, true, true, false, true>;
      static LdsOptIn shared[2];
      if (hipError_t e = shared[gen].ensure((const void*)kern, 160 * 1024); e != hipSuccess) return e;
    }
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(T::NT), lds_bytes, stream, q);
  return hipGetLastError();
}

template <int CP, int RS, int ST>
hipError_t launch_conv_patch_single(const FpropParams& f, hipStream_t stream) {
  using T = ConvPatchTraits<CP, 64, RS, ST, false>;
  return launch_conv_patch<CP, 64, RS, ST, false>(T::from_single(f), 0, T::lds_bytes_n(0), stream);
}

#define BOLT_CONV_PATCH_INSTANCE(CP, RS, ST)                                                                    \
  {                                                                                                            \
    "patch_c" #CP "_r" #RS "_st" #ST, 128, 64, 64, 4, 1, 1, 0, 2, 0, &bolt::launch_conv_patch_single<CP, RS, ST>, \
        &bolt::ConvPatchTraits<CP, 64, RS, ST, false>::supports_single,                                          \
        &bolt::ConvPatchTraits<CP, 64, RS, ST, false>::lds_bytes_single, 0, 0, true, false, false,               \
        &bolt::ConvPatchTraits<CP, 64, RS, ST, false>::estimate, &bolt::ConvPatchTraits<CP, 64, RS, ST, false>::plain_single, true \
  }

#define BOLT_CONV_PATCH_PAIR_INSTANCE(CP, N0T, RS, ST)                                                          \
  {                                                                                                            \
    "b2bpatch_c" #CP "_n" #N0T "_r" #RS "_st" #ST, 0, 128, CP, 4, 1, N0T, 256, 1, 0, 256, 1, nullptr,            \
        &bolt::launch_conv_patch<CP, N0T, RS, ST, true>, &bolt::ConvPatchTraits<CP, N0T, RS, ST, true>::supports,            \
        &bolt::ConvPatchTraits<CP, N0T, RS, ST, true>::lds_bytes, true, 0.f,         \
        &bolt::ConvPatchTraits<CP, N0T, RS, ST, true>::estimate_pair                                              \
  }

}  // namespace bolt
