// 3x3 convolutions of stride 1 and "same" padding with 128, 256 or 512 input channels: the reduction is split over four waves that
// work on their own, each on a quarter of the channels.
//
// The tiled kernels spend such a problem (25 to 400 tiles, 18 to 72 k-tiles each) on a chain of barriers: every k-tile of 64
// waits for its loads, with all waves of the workgroup.  Here
//   * a wave owns the whole tile of BM output pixels x BN channels and a quarter of the input channels, with a SIMD and its
//     registers to itself.  There is no barrier before the sum over the waves, in which each finishes a quarter of the pixels;
//   * the tile's input pixels (BM consecutive ones and the rows above and below, see conv_halo_kernel.hpp), the wave's quarter of
//     the channels, go to LDS once for all nine taps.  A tap is a shift by whole pixels; taps outside the image read a pixel of zeros;
//   * the wave's weights pass through a ring of its own in LDS, D steps of 32 channels deep.  (Straight to registers in the matrix
//     core's order, 16 rows of 64 bytes with neighbouring lanes in different rows, they arrive at 16 bytes per cycle: 22 us
//     instead of 13 for 512 channels.)
//   * the workgroups of an XCD first touch all weights of their column band between them, one load per 64 lines: the ring looks 0.5
//     to 1 us ahead, memory takes longer (batch 32, caches cold: 512 channels 18.2 -> 13.2 us, 256 13.4 -> 13.2).
// What bounds it: products, at 20 cycles of the 16 that the instruction takes under the power limit (LDS: 64 x 64 tiles take the
// 128 bytes per cycle that there are), 55 % of a tile's time; loads of the input and instruction fetch in front of them, 25 %; the sum
// over the waves and the store behind them, 20 %.
// Measured with cold / warm caches, best other instance -> this one, us, batch 32: 28 x 28 x 128 -> 128 15.4 / 14.2 -> 13.9 / 13.0; 14 x 14 x 256
// -> 256 17.7 / 15.2 -> 13.2 / 11.4; 7 x 7 x 512 -> 512 22.8 / 17.0 -> 13.2 / 10.9; batch 8: 12.7 / 10.9 -> 6.2 / 5.7, 11.8 / 10.8 -> 9.5 / 7.1,
// 16.2 / 13.8 -> 12.8 / 10.0.  A residual, whose rows are on their way while the sums go round, costs 0.3 to 0.7 us (batch 32, warm: 14.8 -> 13.3,
// 15.7 -> 12.0, 17.7 -> 12.2 against the other kernels).
// Channels are 128, 256 and 512 because a wave's quarter is unrolled in whole steps of 32 and its pixels lie in LDS at a power of two of chunks:
// 96, 192 and 320 do not split so, 384 would need a bank order of its own; each count costs up to three kernels of 13 to 22 KB.
#pragma once
#include "fprop_dma_kernel.hpp"

namespace bolt {

struct ConvSliceParams : FpropParams {
  unsigned rcp_hw, rcp_w, rcp_tiles;  // (2^32 - 1) / (H W), / W and / tiles_m: quotients from them are exact or one too small
};

template <int BM, int BN, int CWS>
struct ConvSliceTraits {
  static constexpr int NW = 4, NT = 64 * NW;
  static constexpr int FM = BM / 16, FN = BN / 16;  // fragments of pixels and output channels
  static constexpr int C = 32 * CWS * NW, CW = 32 * CWS;  // input channels, and those of a wave
  static constexpr int CH = CW / 8;                       // 16-byte chunks of a pixel of one wave
  static constexpr int STEPS = 9 * CWS;                   // steps of 32 channels of one tap
  static constexpr int D = 4 * 64 / BN + (CWS == 1 ? 1 : 0);  // steps of weights in flight
  static constexpr int W_BYTES = BN * 64;                 // weights of a step
  // Steps whose weights have been requested before step t starts: two in front of the loop, where loads are all that a wave
  // waits for, then two per step until D are ahead
  static constexpr int requested(int t) { return t + D < 2 * t + 2 ? (t + D < STEPS ? t + D : STEPS) : 2 * t + 2; }
  static constexpr int FQ = FM / NW;                      // pixel fragments that a wave finishes
  // The sum over the waves passes through LDS, in two halves of the columns where the whole does not fit
  static constexpr int PH = BM * BN * 4 * (NW - 1) > 150 * 1024 ? 2 : 1;
  static constexpr int SUM_BYTES = BM * BN * 4 * (NW - 1) / PH;
  static_assert(FM % NW == 0 && FN % PH == 0 && D >= 3 && D * FN < 64, "instance");

  static __host__ __device__ int halo_pixels(const ConvGeom& g) { return BM + 2 * (g.Wi + 1); }
  static __host__ __device__ int load_instructions(const ConvGeom& g) { return (halo_pixels(g) * CH + 63) / 64; }
  static __host__ __device__ int input_bytes(const ConvGeom& g) { return (load_instructions(g) + 1) * 1024; }  // the last: zeros
  static __host__ __device__ int wave_bytes(const ConvGeom& g) { return input_bytes(g) + D * W_BYTES; }
  static int lds_bytes(const FpropParams& p) {
    const int pipe = NW * wave_bytes(p.cg) + 1024;  // and a place that is never read, see the kernel
    return pipe > SUM_BYTES ? pipe : SUM_BYTES;
  }
  // The chunk of a pixel that a logical one lies in: 16 pixels side by side, at one logical chunk, fall into 16 bank groups
  static __device__ int swizzle(int px) { return CH == 16 ? px & 15 : CH == 8 ? (px >> 1) & 7 : (px >> 2) & 3; }
  static bool supports(const FpropParams& p) {
    const ConvGeom& g = p.cg;
    return g.C == C && g.R == 3 && g.S == 3 && g.stride_h == 1 && g.stride_w == 1 && g.pad_h == 1 && g.pad_w == 1 &&
           lds_bytes(p) <= 160 * 1024;
  }
  // Pick rule, us: a round of tiles is fill, sum and launch of 2.7, then 1.9 per 64 x 64 outputs and 128 channels (hot, from 18 problems).
  // (One round of more than one column of tiles: 0.4 more, what the kernels for small problems, against which it stands, are estimated
  // too high there; 480 pixels, 128 -> 152: 5.5 us there, 5.9 here; 1500 pixels, 128 -> 64: 5.6 and 5.4.)
  static double estimate(const FpropParams& p) {
    const int rounds = ((p.M + BM - 1) / BM * ((p.N + BN - 1) / BN) + 255) / 256;
    return (rounds == 1 && p.N > BN ? 1.0 : 0.6) + rounds * (2.7 + 1.9 * (BM / 64 * (BN / 64) * CWS) + 2.0 * (PH - 1));
  }
};

template <int BM, int BN, int CWS, bool RES>
__global__ __launch_bounds__(256, 1) void conv_slice_kernel(const ConvSliceParams p) {
#if defined(__HIP_DEVICE_COMPILE__)
  using T = ConvSliceTraits<BM, BN, CWS>;
  constexpr int NW = T::NW, FM = T::FM, FN = T::FN, CH = T::CH, STEPS = T::STEPS, D = T::D, FQ = T::FQ, PH = T::PH;
  extern __shared__ __attribute__((aligned(16))) half_t lds[];
  const ConvGeom& cg = p.cg;
  const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // Every XCD (ids are dealt round-robin over 8) takes a contiguous run of tiles, rows of one column band after the other: its
  // workgroups share their weights in its L2.
  auto divide = [](unsigned n, unsigned d, unsigned rcp, unsigned& rem) {
    unsigned q = __umulhi(n, rcp);
    rem = n - q * d;
    if (rem >= d) { rem -= d; ++q; }
    return (int)q;
  };
  int tm, tn, pos, cnt;  // pos, cnt: this workgroup among those of its XCD with the same weights
  {
    const int total = (int)gridDim.x, xcd = (int)blockIdx.x & 7, per = total >> 3, rem = total & 7;
    const int first = xcd * per + (xcd < rem ? xcd : rem), end = first + per + (xcd < rem ? 1 : 0), t = first + ((int)blockIdx.x >> 3);
    unsigned rem_t;
    tn = __builtin_amdgcn_readfirstlane(divide((unsigned)t, (unsigned)p.tiles_m, p.rcp_tiles, rem_t));
    tm = __builtin_amdgcn_readfirstlane((int)rem_t);
    const int band = tn * p.tiles_m, lo = first > band ? first : band, hi = end < band + p.tiles_m ? end : band + p.tiles_m;
    pos = t - lo;
    cnt = hi - lo;
  }
  const int m0 = tm * BM, n0 = tn * BN;

  char* const lds0 = reinterpret_cast<char*>(lds);
  // this tile's rows of the weights; the whole matrix may be larger than a descriptor's 4 GiB
  const int w_rows = p.N - n0 < BN ? p.N - n0 : BN;
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.W + (int64_t)n0 * p.ldw, (unsigned)(((w_rows - 1) * p.ldw + p.K) * 2));
  // ---- the weights of this column band into the L2, each workgroup of the XCD a share: in a network they come from memory, and
  // the ring below looks ahead for less than that takes.  One load touches 64 lines of 128 bytes; its data goes nowhere. ----------
  {
    const unsigned bytes = (unsigned)(w_rows * p.ldw * 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned at = (unsigned)(((i * cnt + pos) * T::NT + (int)threadIdx.x) * 128);
      if (((i * cnt + pos) * T::NT + wave * 64) * 128u < bytes)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, BOLT_LDS_PTR(lds0 + NW * T::wave_bytes(cg) + wave * 256), 4, at, 0, 0, 0);
    }
  }

  // what the epilogue needs, now: a scalar load that misses takes as long as the whole of its arithmetic
  EpilogueArgs ep{p.bias, p.bias_on, p.N, p.alpha, p.beta, p.act, RES ? p.gamma : 0.f};
  half_t* y = p.Y;
  int ldy = p.ldy;
  asm volatile("" : "+s"(ep.alpha), "+s"(ep.beta), "+s"(ep.act), "+s"(ep.N), "+s"(y), "+s"(ldy));

  // ---- input pixels m0 - (W + 1) .. m0 + BM + W, this wave's channels, to LDS ------------------------------------------------
  const int halo = cg.Wi + 1, n_load = T::load_instructions(cg);
  const int xs = wave * T::wave_bytes(cg);
  const int zero_at = xs + n_load * 1024;  // a pixel of zeros: what lanes read for taps outside the image
  {
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.X, (unsigned)((int64_t)p.M * T::C * 2));
    const int end = m0 + BM + halo < p.M ? m0 + BM + halo : p.M;
    int row = lane / CH;  // pixel of the chunk that this lane's slot of the first instruction holds
    for (int i = 0; i < n_load; ++i) {
      const int px = m0 - halo + row, ch = lane % CH ^ T::swizzle(row);
      const unsigned off = ((px >= 0) & (px < end)) ? (unsigned)(px * T::C + wave * T::CW + ch * 8) * 2u : kInvalidOffset;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, BOLT_LDS_PTR(lds0 + xs + i * 1024), 16, off, 0, 0, 0);
      row += 64 / CH;
    }
    *(half8*)(lds0 + zero_at + lane * 16) = half8{0, 0, 0, 0, 0, 0, 0, 0};
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  // ---- weights: a step is [output channel][32 input channels], XOR-swizzled; 16 rows per load instruction ------------------------
  half_t* const ws = reinterpret_cast<half_t*>(lds0 + xs + T::input_bytes(cg));
  unsigned w_at[FN];
#pragma unroll
  for (int a = 0; a < FN; ++a) {
    const int n = a * 16 + (lane >> 2), ch = (lane & 3) ^ dma_swizzle<32>(n);
    w_at[a] = n < w_rows ? (unsigned)(n * p.ldw + wave * T::CW + ch * 8) * 2u : kInvalidOffset;
  }
  auto load_w = [&](int a, int t) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, BOLT_LDS_PTR(ws + t % D * (T::W_BYTES / 2) + a * 512), 16, w_at[a],
                                             (t / CWS * T::C + t % CWS * 32) * 2, 0, 0);
  };
  // which taps of a lane's pixels lie inside the image; between the first loads, which keep the wave waiting for their turn anyway
  unsigned taps[FM];
  const unsigned hw = (unsigned)(cg.H * cg.Wi);
#pragma unroll
  for (int i = 0; i < T::requested(0) * FN; ++i) {
    load_w(i % FN, i / FN);
#pragma unroll
    for (int b = i * FM / (T::requested(0) * FN); b < (i + 1) * FM / (T::requested(0) * FN); ++b) {
      const int m = m0 + b * 16 + l16;
      unsigned rem, col;
      (void)divide((unsigned)m, hw, p.rcp_hw, rem);
      const int h = divide(rem, (unsigned)cg.Wi, p.rcp_w, col), w = (int)col;
      const unsigned row = (w > 0 ? 1u : 0u) | 2u | (w < cg.Wi - 1 ? 4u : 0u);
      taps[b] = m < p.M ? (h > 0 ? row : 0u) | row << 3 | (h < cg.H - 1 ? row << 6 : 0u) : 0u;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  half4 bias[FN];  // of this lane's output channels
#pragma unroll
  for (int a = 0; a < FN; ++a) {
    const int n = n0 + a * 16 + g * 4;
    bias[a] = *(const half4*)(p.bias + (n < p.N ? n : 0) * p.bias_on);
  }
  half8 wf[2][FN], xf[2][FM];
  const half_t* const w_lane = ws + dma_chunk_offset<32>(l16, g);
  auto read_w = [&](int a, int t) { wf[t & 1][a] = *(const half8*)(w_lane + t % D * (T::W_BYTES / 2) + a * 512); };

  floatx4 acc[FN][FM];
#pragma unroll
  for (int a = 0; a < FN; ++a)
#pragma unroll
    for (int b = 0; b < FM; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};

  // LDS addresses of this lane's part of the pixels' fragments under the tap that is being read
  int x_at[FM], tap_at = 0;
  auto set_tap = [&](int t) {  // of step t
    const int row = l16 + t / CWS / 3 * cg.Wi + t / CWS % 3;
    tap_at = xs + row * T::CW * 2 + ((g ^ T::swizzle(row)) << 4);
  };
  auto read_x = [&](int b, int t) {
    if (t % CWS == 0) x_at[b] = (taps[b] >> (t / CWS) & 1u) ? tap_at + b * 16 * T::CW * 2 : zero_at + g * 16;
    xf[t & 1][b] = *(const half8*)(lds0 + (x_at[b] ^ t % CWS * 64));
  };
  // all but the newest n loads have landed (they retire in order)
  auto wait_loads = [](auto n) {
    constexpr int N = decltype(n)::value;
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4) << 14);
    asm volatile("" ::: "memory");
  };

  wait_loads(std::integral_constant<int, (T::requested(0) - 1) * FN>{});
  set_tap(0);
#pragma unroll
  for (int a = 0; a < FN; ++a) read_w(a, 0);
#pragma unroll
  for (int b = 0; b < FM; ++b) read_x(b, 0);

  // ---- a step's products stand beside the reads of the next step's operands, in the order of their use -----------------------------
  for_constants<T::STEPS>([&](auto tc) __attribute__((always_inline)) {
    constexpr int t = decltype(tc)::value;
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (t + 1 < T::STEPS) {
      wait_loads(std::integral_constant<int, (T::requested(t) - t - 2) * FN>{});  // weights of step t + 1 have landed
      if ((t + 1) % CWS == 0) set_tap(t + 1);
    }
#pragma unroll
    for (int b = 0; b < FM; ++b) {
      __builtin_amdgcn_sched_barrier(0);
      if (t + 1 < T::STEPS) {
        constexpr int R = FN + FM, G = FM - FM / 4;  // reads of a step, in the first three quarters of its products
#pragma unroll
        for (int i = b * R / G; i < (b + 1) * R / G && i < R; ++i) {
          if (i < FN) read_w(i, t + 1);
          else read_x(i - FN, t + 1);
        }
      }
#pragma unroll
      for (int a = 0; a < FN; ++a) acc[a][b] = mfma_16x16x32(wf[t & 1][a], xf[t & 1][b], acc[a][b]);
      // (the first products had to wait for step t's weights: their place is free)
      constexpr int from = T::requested(t) * FN, loads = T::requested(t + 1) * FN - from;  // (step by step: the waits count them)
#pragma unroll
      for (int i = b * loads / FM; i < (b + 1) * loads / FM; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        load_w((from + i) % FN, (from + i) / FN);
      }
    }
  });
  __builtin_amdgcn_sched_barrier(0);

  // ---- the sum over the waves: wave q finishes the pixel fragments q FQ .. q FQ + FQ - 1.  Its own part stays in registers, the
  // others' come through LDS, [wave q][source][fragment][lane] ----------------------------------------------------------------------
  floatx4* const sums = reinterpret_cast<floatx4*>(lds);
  constexpr int AP = FN / PH, NF = AP * FQ;  // column fragments of a half, fragments of a part
#pragma unroll
  for (int ph = 0; ph < PH; ++ph) {
    floatx4 own[AP][FQ];
    constexpr int BP = AP * 16, CPR = BP / 8, PASSES = FQ * 16 * CPR / 64;  // columns of a half, their chunks, instructions for a wave's rows
    const int n_half = n0 + ph * BP;
    // the residual's rows as the stores write them, on their way while the sums go round
    half8 rv[RES ? PASSES : 1];
    if constexpr (RES) {
#pragma unroll
      for (int i = 0; i < PASSES; ++i) {
        const int m = m0 + wave * FQ * 16 + (i * 64 + lane) / CPR, n = n_half + (i * 64 + lane) % CPR * 8;
        rv[i] = half8{0, 0, 0, 0, 0, 0, 0, 0};
        if ((m < p.M) & (n < ep.N)) rv[i] = *(const half8*)(p.res + (int64_t)m * p.ldr + n);
      }
    }
    barrier_after_lds_writes();  // all waves are done with what the sums overwrite
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      if (q == wave) {
#pragma unroll
        for (int a = 0; a < AP; ++a)
#pragma unroll
          for (int b = 0; b < FQ; ++b) own[a][b] = acc[ph * AP + a][q * FQ + b];
      } else {
        floatx4* const to = sums + ((q * (NW - 1) + (wave < q ? wave : wave - 1)) * NF) * 64 + lane;
#pragma unroll
        for (int a = 0; a < AP; ++a)
#pragma unroll
          for (int b = 0; b < FQ; ++b) to[(a * FQ + b) * 64] = acc[ph * AP + a][q * FQ + b];
      }
    }
    barrier_after_lds_writes();
    floatx4* const mine = sums + wave * (NW - 1) * NF * 64;
#pragma unroll
    for (int a = 0; a < AP; ++a)
#pragma unroll
      for (int b = 0; b < FQ; ++b)
#pragma unroll
        for (int s = 0; s < NW - 1; ++s) own[a][b] += mine[(s * NF + a * FQ + b) * 64 + lane];
    asm volatile("" ::: "memory");
    // ---- epilogue; the halves pass through this wave's part of the sums, so that stores write whole rows ----------------------------
    half_t* const out = reinterpret_cast<half_t*>(mine);
    if constexpr (RES) {
#pragma unroll
      for (int i = 0; i < PASSES; ++i) {
        const int row = (i * 64 + lane) / CPR, chunk = (i * 64 + lane) % CPR;
        *(half8*)(out + row * BP + ((chunk ^ ctile_swizzle<CPR>(row)) << 3)) = rv[i];
      }
      asm volatile("" ::: "memory");
    }
    auto finish = [&](auto slow) {
#pragma unroll
      for (int a = 0; a < AP; ++a)
#pragma unroll
        for (int b = 0; b < FQ; ++b) {
          const int n = a * 16 + g * 4, row = b * 16 + l16;
          half4* const slot = (half4*)(out + row * BP + (((n >> 3) ^ ctile_swizzle<CPR>(row)) << 3) + (n & 4));
          *slot = epilogue_quad4_values<decltype(slow)::value, RES>(own[a][b], bias[ph * AP + a], ep, RES ? *slot : half4{0, 0, 0, 0});
        }
    };
    if (ep.act > ACT_RELU) finish(std::true_type{});
    else finish(std::false_type{});
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      const int row = (i * 64 + lane) / CPR, chunk = (i * 64 + lane) % CPR;
      const int m = m0 + wave * FQ * 16 + row, n = n_half + chunk * 8;
      if ((m < p.M) & (n < ep.N))
        __builtin_nontemporal_store(*(const half8*)(out + row * BP + ((chunk ^ ctile_swizzle<CPR>(row)) << 3)), (half8*)(y + (int64_t)m * ldy + n));
    }
  }
#endif
}

template <int BM, int BN, int CWS>
hipError_t launch_conv_slice(const FpropParams& p, hipStream_t stream) {
  using T = ConvSliceTraits<BM, BN, CWS>;
  static LdsOptIn opt_in[2];
  auto kern = p.res ? conv_slice_kernel<BM, BN, CWS, true> : conv_slice_kernel<BM, BN, CWS, false>;
  if (hipError_t e = opt_in[p.res ? 1 : 0].ensure((const void*)kern, 160 * 1024); e != hipSuccess) return e;
  ConvSliceParams q{p};
  q.rcp_hw = 0xffffffffu / (unsigned)(p.cg.H * p.cg.Wi);
  q.rcp_w = 0xffffffffu / (unsigned)p.cg.Wi;
  q.rcp_tiles = 0xffffffffu / (unsigned)p.tiles_m;
  hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n), dim3(T::NT), T::lds_bytes(p), stream, q);
  return hipGetLastError();
}

#define BOLT_CONV_SLICE_INSTANCE(BM, BN, CWS)                                                                   \
  {                                                                                                            \
    "slice_" #BM "x" #BN "_c" #CWS, BM, BN, 32, 4, 1, 1, 0, 2, 0, &bolt::launch_conv_slice<BM, BN, CWS>,          \
        &bolt::ConvSliceTraits<BM, BN, CWS>::supports, &bolt::ConvSliceTraits<BM, BN, CWS>::lds_bytes, 0, 16,    \
        true, false, false, &bolt::ConvSliceTraits<BM, BN, CWS>::estimate, nullptr, true                   \
  }

}  // namespace bolt
