// Convolution of a tensor whose channel count is even but no multiple of 8 (the "unpadded" layers of Table 3), without a
// padding pass: the padding happens on the way to LDS.
//
// The general alignment-2 kernel (fprop_kernel, x mode 2) gathers an im2col tile in 4-byte pieces, R * S times over,
// with its index arithmetic per piece, and stages it through registers: 28 us for 128 images of 14 x 19 x 46, 5 x 7
// filter without padding, 32 output channels, of which the matrix cores need 1 us.  Here a workgroup
//   * copies the input patch its TP x TQ output pixels of ONE image need to LDS once, every pixel's channels zero-padded
//     to a multiple of 8 (16-byte loads at 4-byte alignment, the halves behind the last channel masked), pixels outside
//     the image as zeros.  Filter taps are then plain LDS offsets: 16-byte aligned reads of one pixel's 8 channels.  A
//     pixel takes an odd number of 16-byte units, so that 16 neighbouring pixels fall into 16 different bank groups;
//   * splits the REDUCTION over its waves: wave w takes a contiguous run of the k-steps of 32 = 4 chunks (tap, 8
//     channels), for all pixels and channels of the tile.  A weight is then read by exactly one wave of the workgroup,
//     so weights go straight from global memory to registers, in the order of the matrix core's operand, without LDS and
//     without a barrier in the loop;
//   * sums the waves' partial tiles through LDS in a fixed order, FP32, and applies the epilogue.
// A table in LDS holds every chunk's offsets (pixel-relative LDS offset, weight offset, valid halves).
// What bounds it: latency, of the patch, the first weights and the sum over the waves.  On the problem above waves wait for 41 % of
// their life, vector instructions take 39 % of the SIMD-cycles, matrix ones 14 %, the LDS is active in 24 %, a third of that in
// bank conflicts (a fragment's 16 pixels span two tile rows).
// Measured back to back under the tuner's picks, old -> new: the problem above 28 -> 7.5 us (230 TFLOP/s; the host needs 4
// per call); 128 images of 20 x 26 x 174, 5 x 5, 64 channels 252 -> 73 us (510 TFLOP/s); over 85 problems of
// those ranges nothing was slower (10 input channels, 3 x 3: 5.8 -> 5.5 us, the least gain).
// Without requests past a wave's last step: 7.2 -> 6.8 us, 10 images of 12 x 20 x 170, 5 x 5, 56 channels 8.7 -> 7.9, 38 of 15 x 22 x 146,
// 5 x 7, 24 channels 10.0 -> 9.1 (25 problems, best instance: 0.90 to 1.01, 0.97 on average).
#pragma once
#include <algorithm>
#include <cmath>

#include "fprop_dma_kernel.hpp"

namespace bolt {

// How a problem is cut: output tile TP x TQ pixels, input patch ph x pw pixels of `pitch` 16-byte units.
struct ConvEvenPlan {
  int tp, tq, tiles_p, tiles_q;
  int ph, pw, c8, pitch;
  int chunks, steps, steps_per_wave;
  int patch_at;   // byte offset of the patch in LDS (behind one chunk of zeros and the table)
  int lds_bytes;  // 0: the problem does not fit
};

template <int NW, int FM, int FN>
struct ConvEvenTraits {
  static constexpr int NT = 64 * NW, BM = 16 * FM, BN = 16 * FN;
  // n-fragments reduced per pass: the partial tiles of all waves in at most 80 KB, half a compute unit's LDS
  static constexpr int PF = NW * FM * FN <= 80 ? FN : NW * FM * 2 <= 80 && FN % 2 == 0 ? 2 : 1;
  static constexpr int REDUCE_BYTES = NW * FM * PF * 1024;
  static_assert(REDUCE_BYTES <= 80 * 1024, "partial tiles of one pass");

  static ConvEvenPlan plan(const ConvGeom& g) {
    ConvEvenPlan t{};
    t.c8 = (g.C + 7) / 8;
    t.pitch = t.c8 | 1;
    const int64_t chunks = (int64_t)g.R * g.S * t.c8;
    // (the small divisions in the kernel are exact up to 2^16 / 2^10; 9 bits of the pixel pitch are far beyond LDS)
    if (chunks > 8192 || t.pitch >= 512) return t;
    t.chunks = (int)chunks;
    t.steps = (t.chunks + 3) / 4;
    t.steps_per_wave = (t.steps + NW - 1) / NW;
    t.patch_at = 16 + t.steps * 4 * 8;
    auto split = [](int n, int most, int& tile, int& tiles) {  // n into equal tiles of at most `most`
      tiles = (n + most - 1) / most;
      tile = (n + tiles - 1) / tiles;
      tiles = (n + tile - 1) / tile;
    };
    int most_q = g.Q < BM ? g.Q : BM;
    for (;;) {
      split(g.Q, most_q, t.tq, t.tiles_q);
      int most_p = BM / t.tq < g.P ? BM / t.tq : g.P;
      for (; most_p >= 1; --most_p) {
        split(g.P, most_p, t.tp, t.tiles_p);
        t.ph = (t.tp - 1) * g.stride_h + g.R;
        t.pw = (t.tq - 1) * g.stride_w + g.S;
        const int64_t bytes = t.patch_at + (int64_t)t.ph * t.pw * t.pitch * 16;
        if (bytes <= 160 * 1024 && t.pw < 1024) {
          t.lds_bytes = (int)bytes > REDUCE_BYTES ? (int)bytes : REDUCE_BYTES;
          return t;
        }
        most_p = t.tp;  // (equal tiles may already be smaller)
      }
      if (most_q == 1) return t;
      most_q = (t.tq + 1) / 2;
      if (t.tq == 1) return t;
    }
  }
  static bool supports(const FpropParams& p) {
    const ConvGeom& g = p.cg;
    if (g.C < 10 || (g.C & 1) || (int64_t)p.N * p.ldw * 2 >= (1ll << 31)) return false;
    const ConvEvenPlan t = plan(g);
    return t.lds_bytes > 0 && (int64_t)(p.M / (g.P * g.Q)) * t.tiles_p * t.tiles_q * ((p.N + BN - 1) / BN) < (1ll << 31);
  }
  static int lds_bytes(const FpropParams& p) { return plan(p.cg).lds_bytes; }
  // Pick rule: estimated time in us.  A filter of one tap gives nothing to the copy of the patch (with a stride it holds pixels
  // that nobody reads): with more than 32 output channels over more than 16000 input pixels the alignment-2 kernels take 0.8 to 1.05
  // of this one's time (80 images of 30 x 28 x 98, 1x1 / 2, 40 channels 6.3 against 7.7 us), below either line 0.52 to 1.09 the other way.
  static double estimate(const FpropParams& p) {
    const ConvEvenPlan t = plan(p.cg);
    const double wgs = (double)(p.M / (p.cg.P * p.cg.Q)) * t.tiles_p * t.tiles_q * ((p.N + BN - 1) / BN);
    const double by_lds = 160.0 * 1024 / t.lds_bytes, by_regs = (FM * FN > 12 ? 8.0 : 16.0) / NW;
    const double per_cu = std::max(1.0, std::floor(std::min(by_lds, by_regs)));
    const double seq = std::ceil(wgs / 256), rounds = std::ceil(wgs / (256 * per_cu));
    const double thru = seq * t.steps * (std::max(FM / 262.0, FM * FN / 525.0) + FN / 131.0);
    const bool one_tap = p.cg.R * p.cg.S == 1 && p.N > 32 && (double)p.M * p.cg.stride_h * p.cg.stride_w > 16000;
    return 2.85 + thru + rounds * (1.5 + t.steps_per_wave * 0.1) + (one_tap ? 1.0 : 0.0);
  }
};

template <int NW, int FM, int FN, bool RES>
__global__ __launch_bounds__(64 * NW, 2) void conv_even_kernel(const FpropParams p, const ConvEvenPlan t) {
  using Tr = ConvEvenTraits<NW, FM, FN>;
  constexpr int NT = Tr::NT;
  constexpr int D = 3;  // k-steps of weights in flight per wave
  extern __shared__ __attribute__((aligned(16))) half_t lds[];
  unsigned char* const lds_b = reinterpret_cast<unsigned char*>(lds);
  const ConvGeom& cg = p.cg;
  const int tid = threadIdx.x, lane = tid & 63, g4 = lane >> 4, l16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // small exact divisions: v / d = (int)((v + 0.5f) * (1 / d)) for v < 2^16, d < 2^10
  auto fdiv = [](int v, float rcp) { return (int)(((float)v + 0.5f) * rcp); };

  // Workgroup -> (image, rows, columns, channels), channels fastest.  Every XCD (ids are dealt round-robin over 8) takes
  // a contiguous run: tiles of one image share their halo, all of them the weights, through one L2.
  int id;
  {
    const int total = (int)gridDim.x, xcd = (int)blockIdx.x & 7, per = total >> 3, rem = total & 7;
    id = xcd * per + (xcd < rem ? xcd : rem) + ((int)blockIdx.x >> 3);
  }
  const int tiles_n = (p.N + Tr::BN - 1) / Tr::BN;
  const int tn = id % tiles_n;
  id /= tiles_n;
  const int tqi = id % t.tiles_q;
  id /= t.tiles_q;
  const int tpi = id % t.tiles_p, img = id / t.tiles_p;
  const int n0 = tn * Tr::BN, p0 = tpi * t.tp, q0 = tqi * t.tq;
  const int npix = t.tp * t.tq;

  // ---- input patch: global -> registers -> LDS, 16 bytes (8 channels of one pixel) per item -------------------------
  {
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.X, (unsigned)((int64_t)(p.M / (cg.P * cg.Q)) * cg.H * cg.Wi * cg.C * 2));
    const int ih0 = p0 * cg.stride_h - cg.pad_h, iw0 = q0 * cg.stride_w - cg.pad_w;
    const int items = t.ph * t.pw * t.pitch;  // at most 10240
    const float rcp_pitch = 1.0f / (float)t.pitch, rcp_pw = 1.0f / (float)t.pw;
    constexpr int NB = 4;  // loads in flight per thread
    for (int i0 = tid; i0 < items; i0 += NB * NT) {
      uintx4 v[NB];
      int left[NB];  // channels of the pixel from this chunk on
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        const int i = i0 + k * NT;
        const int pix = fdiv(i, rcp_pitch), c = (i - pix * t.pitch) * 8;
        const int y = fdiv(pix, rcp_pw), x = pix - y * t.pw;
        const int ih = ih0 + y, iw = iw0 + x;
        left[k] = cg.C - c;
        const bool ok = i < items && left[k] > 0 && (unsigned)ih < (unsigned)cg.H && (unsigned)iw < (unsigned)cg.Wi;
        const auto got = __builtin_amdgcn_raw_buffer_load_b128(
            xr, ok ? (unsigned)(((img * cg.H + ih) * cg.Wi + iw) * cg.C + c) * 2u : kInvalidOffset, 0, 0);
        v[k] = uintx4{got[0], got[1], got[2], got[3]};
      }
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        const int i = i0 + k * NT;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[k][e] = 2 * e < left[k] ? v[k][e] : 0u;
        if (i < items) *(uintx4*)(lds_b + t.patch_at + i * 16) = v[k];
      }
    }
  }
  // ---- table of chunks: {LDS byte offset from a pixel's first byte or -1, weight byte offset << 3 | valid dwords} ----
  // (chunks past the last one read the 16 zero bytes in front of the table and no weights)
  if (tid == 0) *(uintx4*)lds_b = uintx4{0, 0, 0, 0};
  {
    const float rcp_c8 = 1.0f / (float)t.c8, rcp_s = 1.0f / (float)cg.S;
    for (int ch = tid; ch < t.steps * 4; ch += NT) {
      const int tap = fdiv(ch, rcp_c8), c = ch - tap * t.c8;
      const int r = fdiv(tap, rcp_s), s = tap - r * cg.S;
      const int left = (cg.C - c * 8) >> 1;
      int2 e = {-1, 0};
      if (ch < t.chunks) e = int2{((r * t.pw + s) * t.pitch + c) * 16, ((tap * cg.C + c * 8) * 2) << 3 | (left < 4 ? left : 4)};
      *(int2*)(lds_b + 16 + ch * 8) = e;
    }
  }

  // ---- this lane's pixels and weight rows ----------------------------------------------------------------------------
  const float rcp_tq = 1.0f / (float)t.tq;
  int pix_at[FM];  // LDS byte offset of the window's first pixel
#pragma unroll
  for (int b = 0; b < FM; ++b) {
    const int j = b * 16 + l16, jj = j < npix ? j : 0;
    const int ty = fdiv(jj, rcp_tq), tx = jj - ty * t.tq;
    pix_at[b] = t.patch_at + (ty * cg.stride_h * t.pw + tx * cg.stride_w) * t.pitch * 16;
  }
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.W, (unsigned)((int64_t)p.N * p.ldw * 2));
  unsigned row_at[FN];  // byte offset of the weight row, far beyond the buffer for a row past N
#pragma unroll
  for (int a = 0; a < FN; ++a) {
    const int n = n0 + a * 16 + l16;
    row_at[a] = n < p.N ? (unsigned)(n * p.ldw * 2) : kInvalidOffset;
  }
  floatx4 acc[FN][FM];
#pragma unroll
  for (int a = 0; a < FN; ++a)
#pragma unroll
    for (int b = 0; b < FM; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();

  // ---- main loop: this wave's k-steps, weights D steps ahead ---------------------------------------------------------
  const int s0 = wave * t.steps_per_wave;
  int n_steps = t.steps - s0 < t.steps_per_wave ? t.steps - s0 : t.steps_per_wave;
  if (n_steps < 0) n_steps = 0;
  uintx4 wv[D][FN];
  int2 ent[D];
  auto fetch = [&](int i, int set, bool on) {  // entry and weights of this wave's k-step i (off: nothing)
    ent[set] = *(const int2*)(lds_b + 16 + (on ? (s0 + i) * 4 + g4 : 0) * 8);
    const bool ok = on && ent[set].x >= 0;
    const unsigned off = ok ? (unsigned)ent[set].y >> 3 : kInvalidOffset;
#pragma unroll
    for (int a = 0; a < FN; ++a) {
      const auto got = __builtin_amdgcn_raw_buffer_load_b128(wr, ok ? row_at[a] + off : kInvalidOffset, 0, 0);
      wv[set][a] = uintx4{got[0], got[1], got[2], got[3]};
    }
  };
#pragma unroll
  for (int k = 0; k < D; ++k) fetch(k, k, k < n_steps);  // (without branches, for the waits behind them)
  auto step = [&](int k) {  // the products of set k
    half8 xf[FM];
#pragma unroll
    for (int b = 0; b < FM; ++b) xf[b] = *(const half8*)(lds_b + (ent[k].x >= 0 ? pix_at[b] + ent[k].x : 0));
    const int nv = ent[k].y & 7;
#pragma unroll
    for (int a = 0; a < FN; ++a) {
#pragma unroll
      for (int e = 1; e < 4; ++e) wv[k][a][e] = e < nv ? wv[k][a][e] : 0u;  // the halves behind belong to the next tap
#pragma unroll
      for (int b = 0; b < FM; ++b) acc[a][b] = mfma_16x16x32(__builtin_bit_cast(half8, wv[k][a]), xf[b], acc[a][b]);
    }
  };
  // A request past the wave's last step would bring zeros, and would cost the address unit (16 rows of 64 bytes) as much as any: of
  // 7 steps per wave D = 3 more.  Whole rounds stand apart, and a fence keeps each request behind the step whose registers it takes, so
  // that a step waits for its own set only.  Weights are masked where they lie and requested behind the products: a copy beside them is 9 to
  // 13 registers, a workgroup per compute unit for the narrow tiles.  (Requests ahead of the products without the fence, all three of a round behind
  // its last product as compiled, -> this: 274 images of 32 x 20 x 36, 3 x 3, 32 channels, 17.1 -> 16.4 us, its 6 x 1 fragments on 8 waves 37.6
  // -> 31.9; 186 of 33 x 36 x 42, 5 x 7, 24 channels 35.7 -> 33.6.  40 problems, best instance: 0.973.)
  int i = 0;
  for (; i + 2 * D <= n_steps; i += D) {
#pragma unroll
    for (int k = 0; k < D; ++k) {
      step(k);
      fetch(i + k + D, k, true);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  for (; i < n_steps; i += D) {
#pragma unroll
    for (int k = 0; k < D; ++k) {
      if (i + k < n_steps) {
        step(k);
        if (i + k + D < n_steps) fetch(i + k + D, k, true);
      }
    }
  }

  // ---- sum over the waves through LDS, epilogue, store ---------------------------------------------------------------
  const EpilogueArgs ep{p.bias, p.bias_on, p.N, p.alpha, p.beta, p.act, p.gamma};
  floatx4* const red = reinterpret_cast<floatx4*>(lds);  // [wave][PF * FM fragments][64 lanes]
  constexpr int PFR = Tr::PF * FM;
#pragma unroll
  for (int a0 = 0; a0 < FN; a0 += Tr::PF) {
    __syncthreads();  // every wave has finished with what the partial tiles overwrite
#pragma unroll
    for (int a = 0; a < Tr::PF; ++a)
#pragma unroll
      for (int b = 0; b < FM; ++b)
        if (a0 + a < FN) red[(wave * PFR + a * FM + b) * 64 + lane] = acc[a0 + a < FN ? a0 + a : 0][b];
    __syncthreads();
    for (int f = wave; f < PFR; f += NW) {
      floatx4 s = red[f * 64 + lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += red[(w * PFR + f) * 64 + lane];  // fixed order
      const int a = f / FM, j = (f - a * FM) * 16 + l16, n = n0 + (a0 + a) * 16 + g4 * 4;
      const int ty = fdiv(j, rcp_tq), tx = j - ty * t.tq;
      if (j < npix && p0 + ty < cg.P && q0 + tx < cg.Q && n < p.N) {
        const int64_t m = ((int64_t)img * cg.P + p0 + ty) * cg.Q + q0 + tx;
        half4 res = {0, 0, 0, 0};
        if constexpr (RES) res = *(const half4*)(p.res + m * p.ldr + n);
        const half4 o = p.act > ACT_RELU ? epilogue_quad4_impl<true, RES>(s, n, ep, res) : epilogue_quad4_impl<false, RES>(s, n, ep, res);
        *(half4*)(p.Y + m * p.ldy + n) = o;
      }
    }
  }
}

template <int NW, int FM, int FN>
hipError_t launch_conv_even(const FpropParams& p, hipStream_t stream) {
  using Tr = ConvEvenTraits<NW, FM, FN>;
  const ConvEvenPlan t = Tr::plan(p.cg);
  auto kern = p.res ? conv_even_kernel<NW, FM, FN, true> : conv_even_kernel<NW, FM, FN, false>;
  static LdsOptIn opt_in[2];
  if (hipError_t e = opt_in[p.res ? 1 : 0].ensure((const void*)kern, 160 * 1024); e != hipSuccess) return e;
  const int tiles = p.M / (p.cg.P * p.cg.Q) * t.tiles_p * t.tiles_q * ((p.N + Tr::BN - 1) / Tr::BN);
  hipLaunchKernelGGL(kern, dim3(tiles, 1, 1), dim3(Tr::NT), t.lds_bytes, stream, p, t);
  return hipGetLastError();
}

// In the instance table: x mode and w mode 2 (even channel counts), tile = 16 FM pixels x 16 FN channels, stated as the
// multiple of 32 that holds it (the unit of every tile in the table), tile K = the 32 of one matrix instruction, NW
// waves as k-groups of 4.
#define BOLT_CONV_EVEN_INSTANCE(NW, FM, FN)                                                                      \
  {                                                                                                              \
    "even_" #NW "w_" #FM "x" #FN, (16 * FM + 31) / 32 * 32, (16 * FN + 31) / 32 * 32, 32, 4, 1, 2, 2, 2, 0,       \
        &bolt::launch_conv_even<NW, FM, FN>, &bolt::ConvEvenTraits<NW, FM, FN>::supports,                        \
        &bolt::ConvEvenTraits<NW, FM, FN>::lds_bytes, NW / 4, 16, false, false, false,                           \
        &bolt::ConvEvenTraits<NW, FM, FN>::estimate                                                              \
  }

}  // namespace bolt
