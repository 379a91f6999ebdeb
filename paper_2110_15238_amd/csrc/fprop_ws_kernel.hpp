// Small problems: GEMM / implicit-GEMM convolution whose REDUCTION is split over the waves of a workgroup, with operands
// that go straight from global memory to registers.
//
// A problem with few output tiles (a convolution of one image, a classifier's 32 rows) leaves most compute units idle
// under the tiled kernels, and each of the few workgroups walks its whole reduction through LDS in turn: load, barrier,
// read, multiply, a fixed latency per 64-wide k-tile.  Here
//   * the output tile is small (16 FM x 16 FN, from 16 x 16), so that there are workgroups for more compute units;
//   * wave w of NW takes a contiguous run of the reduction, in units of 64, for the WHOLE tile.  Every operand element is
//     then used by one wave of the workgroup only, so nothing is staged for others: a wave loads its units to registers, D
//     ahead, 8 neighbouring lanes one 128-byte row, and passes them through a piece of LDS of its own into the matrix core's
//     operand order.  There is no barrier in the loop.  (Loads in operand order, 16 rows per 16 lanes, touch a cache line
//     per lane: 64 x 64 x 8192 took 16.9 us so, 8.1 now.);
//   * the waves' partial tiles are summed through LDS in a fixed order, in FP32, and the epilogue is applied once.  Bias and
//     residual are requested before the loop.
// Row-major weights ([K][N]) lie in LDS as in memory and are read with the transposing read.
// What bounds it: launch (2.3 us), one round trip to memory and the sum over the waves (waves wait for 46 to 77 % of their life).  With several units per
// wave it matters how they are requested: the conditions of a request's offsets split the wave, a load stands on either side, and both write
// the same registers.  As compiled, the forms of 8 and 16 waves (256 and 128 registers, no accumulation registers) wait for everything in flight in
// between, so their units come one round trip after the other whatever D is; those of 4 waves don't wait.  (Held to 128 registers, 4 waves of
// 1 x 2 fragments wait so too: 365 x 112 x 4032 8.5 -> 10.3 us, 2 images of 45 x 33 x 832, 3 x 3, 16.0 -> 19.6.)
// A wave has few units (1 to 9 in a
// network of one image), so no request is made past the last one: requests that bring only zeros take their turn in the address
// unit like any other, and D of them per wave cost 0.1 to 0.6 us (1024 -> 256 at 14 x 14 3.99 -> 3.84 us, 3 x 3 256 -> 256 5.94 -> 5.5,
// 128 -> 512 with a skip connection at 28 x 28 4.3 -> 3.7, 32 x 1000 x 2048 row-major 5.8 -> 5.65; the network's 52 layers 248 -> 221).  D = 4 to 6 was 2 to 20 %
// slower, but measured on requests that wait as described.
// Measured back to back under the tuner's picks, tiled kernels -> this one (first form): 32 x 1000 x 2048 row-major 8.1 -> 5.0 us,
// 256 x 256 x 256 4.1 -> 3.2; convolutions of one image: 14 x 14, 3 x 3, 256 -> 256 9.5 -> 5.5, 1024 -> 256 6.1 -> 3.8,
// 7 x 7, 3 x 3, 512 -> 512 10.5 -> 7.2, 2048 -> 512 8.0 -> 4.5.
#pragma once
#include <algorithm>
#include <cmath>

#include "fprop_dma_kernel.hpp"

namespace bolt {

template <int NW, int FM, int FN>
struct FpropWsTraits {
  static constexpr int NT = 64 * NW, BM = 16 * FM, BN = 16 * FN;
  static constexpr int PITCH = BN + 4;  // floats per row of a partial tile: 16 rows fall into 16 different bank groups
  // of one wave: its rows on their way into operand order, then its partial tile
  static constexpr int STAGE_BYTES = (FM + FN) * 2048, PART_BYTES = BM * PITCH * 4;
  static constexpr int WAVE_BYTES = STAGE_BYTES > PART_BYTES ? STAGE_BYTES : PART_BYTES;
  static constexpr int LDS_BYTES = NW * WAVE_BYTES;
  static constexpr int QUADS = BM * BN / 4, QPT = (QUADS + NT - 1) / NT;  // output quads, per thread
  static_assert(LDS_BYTES <= 160 * 1024, "partial tiles of all waves");

  static int64_t workgroups(const FpropParams& p) {
    return (((int64_t)p.M + BM - 1) / BM) * (((int64_t)p.N + BN - 1) / BN);
  }
  // (The small divisions in the kernel are exact up to 2^20; a launch has fewer than 2^32 threads.)
  static bool supports(const FpropParams& p) { return p.K <= (1 << 20) && workgroups(p) * NT < (1ll << 32); }
  // Up to 512 tiles, two per compute unit: with more of them the kernels with larger tiles and LDS staging read less (over
  // 70 problems of 1 to 8 images the last win was at 392 tiles of 32 x 32, 7.6 against 7.7 us; at 784 it was 29 against 14).
  static bool worth_trying(const FpropParams& p) { return workgroups(p) <= 512; }
  static int lds_bytes(const FpropParams&) { return LDS_BYTES; }
  // Pick rule: estimated time in us.  A fit to 612 timings of 76 problems (rms 16 %): operand traffic of the tiles a compute
  // unit runs in turn; per round of co-resident workgroups one latency, the units of a wave, the sum over the waves and,
  // for a convolution, the addresses; no faster than every tensor once from memory.  Rows run fastest over the tiles, so the
  // activations are read again for every column of tiles: from memory where they are more than the L2s keep (half of 32 MB).
  // (Without the activations 7 of 106 tall problems, 1024 to 16384 rows x 8 to 64 x 512 to 8192, went from the tiled kernels
  // to slower ones: 8192 x 64 x 2048 10.0 -> 14.2 us, 16384 x 32 x 8192 42.1 -> 44.8.  The 0.02 ranks the tiles among each other.)
  // A deep reduction over more than one tile per compute unit is a second round of nothing but operand traffic: the fit errs by
  // up to 45 % to this side there and the tiled kernels are close, so a quarter on top, 15 % for filter windows.  The depth where
  // that begins, of 107 problems with 257 to 512 tiles (time against the tiled pick): GEMM and 1x1 up to 600 0.77-1.09, from 1224
  // on 0.94-1.46 (4677 x 40 x 3272 13.0 -> 18.5 us); windows up to 3024 0.75-1.12, beyond 0.97-1.48.
  static double estimate(const FpropParams& p) {
    const bool window = p.cg.R > 0 && p.ldx == 0;
    const double wgs = (double)workgroups(p), units = (p.K + 63) / 64, upw = std::ceil(units / NW);
    const double seq = std::ceil(wgs / 256);
    const double per_cu = std::max(1, std::min(160 * 1024 / LDS_BYTES, 16 / NW));
    const double fill = seq * units * 128.0 * (BM + BN) / 6.06e4;
    const double chain = std::ceil(wgs / (256 * per_cu)) * (1.41 + upw * 0.105 + NW * FM * FN * 0.0274 + (window ? 0.89 : 0.0)) +
                         (seq - 1) * 0.66;
    double x = (double)p.M * (window ? std::min<double>(p.K, (double)p.cg.C * p.cg.stride_h * p.cg.stride_w) : p.K);
    if (x * 2 > (16 << 20)) x *= (p.N + BN - 1) / BN;
    const double mem = 2.0 * (x + (double)p.N * p.K + (double)p.M * p.N) / 5.0e6 + 0.02 * fill;
    const double second_round = wgs <= 256 ? 1.0 : window ? (p.K > 3200 ? 1.15 : 1.0) : p.K > 1200 ? 1.25 : 1.0;
    return (2.0 + std::max(std::sqrt(fill * fill + chain * chain), mem)) * second_round;
  }
};

// 8 reduction indices of one column out of two row segments per 4 lanes (ds_read_b64_tr_b16: within 16 lanes, lanes 4r ..
// 4r + 3 address the quarters of a 16-half row segment, lane i receives element i of the four segments).
__device__ __forceinline__ half8 ws_transposed_read(const unsigned char* lo_at, const unsigned char* hi_at) {
  typedef short short4v __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) short4v lds_short4;
  const half4 lo = __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)lo_at));
  const half4 hi = __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)hi_at));
  return half8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}

template <int NW, int FM, int FN, int XMODE, bool WKN, bool RES>
__global__ __launch_bounds__(64 * NW) void fprop_ws_kernel(const FpropParams p) {
  using Tr = FpropWsTraits<NW, FM, FN>;
  constexpr int NT = Tr::NT, BM = Tr::BM, BN = Tr::BN, PITCH = Tr::PITCH;
  constexpr int D = FM + FN <= 3 ? 3 : 2;  // units in flight per wave, within the registers
  static_assert(!WKN || FN == 1 || FN == 2 || FN == 4, "swizzle of row-major weights");
  static_assert(XMODE == 0 || !WKN, "convolution weights are [K][R][S][C]");
  extern __shared__ __attribute__((aligned(16))) half_t lds[];
  float* const part = reinterpret_cast<float*>(lds);  // [NW][BM][PITCH], waves WAVE_BYTES apart
  const int tid = threadIdx.x, lane = tid & 63, g4 = lane >> 4, l16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto fdiv = [](int v, float rcp) { return (int)(((float)v + 0.5f) * rcp); };  // exact for v < 2^20, also if rcp is an ulp off

  // Workgroup -> tile, rows fastest; every XCD (ids are dealt round-robin over 8) takes a contiguous run, so a stripe of
  // weights is read into one or two L2s only.
  int tm, tn;
  {
    const int tiles_m = (p.M + BM - 1) / BM;
    const int total = (int)gridDim.x, xcd = (int)blockIdx.x & 7, per = total >> 3, rem = total & 7;
    const int id = xcd * per + (xcd < rem ? xcd : rem) + ((int)blockIdx.x >> 3);
    tn = id / tiles_m;
    tm = id - tn * tiles_m;
  }
  const int m0 = tm * BM, n0 = tn * BN;

  // ---- this lane's rows of both operands ------------------------------------------------------------------------------
  // A unit is 64 reduction indices = 128 bytes of a K-contiguous row: 8 neighbouring lanes read one row's unit, two load
  // instructions the 16 rows of a fragment.
  const ConvGeom& cg = p.cg;
  const int lrow = lane >> 3, lk = (lane & 7) * 8;
  __amdgpu_buffer_rsrc_t xr;
  unsigned x_at[2 * FM];               // XMODE 0: byte offset of the row, far beyond the buffer past M
  int x_px[2 * FM], ihw0[2 * FM];      // XMODE 1: the window's first pixel: element offset; row << 16 | column + 2^15
  float rcp_c = 0.f, rcp_s = 0.f;
  if constexpr (XMODE == 0) {
    const int rows = p.M - m0 < BM ? p.M - m0 : BM;
    xr = make_rsrc(p.X + (int64_t)m0 * p.ldx, (unsigned)(((rows - 1) * p.ldx + p.K) * 2));
#pragma unroll
    for (int b = 0; b < 2 * FM; ++b)
      x_at[b] = b * 8 + lrow < rows ? (unsigned)((b * 8 + lrow) * p.ldx + lk) * 2u : kInvalidOffset;
  } else {
    xr = make_rsrc(p.X, (unsigned)((int64_t)(p.M / (cg.P * cg.Q)) * cg.H * cg.Wi * cg.C * 2));
    rcp_c = __builtin_amdgcn_rcpf((float)cg.C);
    rcp_s = __builtin_amdgcn_rcpf((float)cg.S);
    // Quotients of integers are 30 to 40 vector instructions, and up to four waves of a workgroup share a SIMD: only the tile's
    // first pixel is divided so, once for all lanes; its others are less than BM behind it.  (3 x 3 of one image: 14 x 14 256 -> 256 4.91 -> 4.80 us,
    // 56 x 56 64 -> 64 4.28 -> 4.19; 14 problems in every instance 0.988 of the time on average, 0.976 to 1.002 by instance.)
    const float rcp_q = __builtin_amdgcn_rcpf((float)cg.Q), rcp_p = __builtin_amdgcn_rcpf((float)cg.P);
    const int row0 = m0 / cg.Q, q0 = m0 - row0 * cg.Q, img0 = row0 / cg.P, pp0 = row0 - img0 * cg.P;
#pragma unroll
    for (int b = 0; b < 2 * FM; ++b) {
      const int j = b * 8 + lrow, m = m0 + j;
      const int rows = fdiv(q0 + j, rcp_q), q = q0 + j - rows * cg.Q;
      const int imgs = fdiv(pp0 + rows, rcp_p), img = img0 + imgs, pp = pp0 + rows - imgs * cg.P;
      const int ih = m < p.M ? pp * cg.stride_h - cg.pad_h : -(1 << 15), iw = q * cg.stride_w - cg.pad_w;
      ihw0[b] = (int)((unsigned)ih << 16 | (unsigned)(iw + (1 << 15)));
      x_px[b] = ((img * cg.H + pp * cg.stride_h - cg.pad_h) * cg.Wi + iw) * cg.C;
    }
  }
  const int w_rows = p.N - n0 < BN ? p.N - n0 : BN;
  __amdgpu_buffer_rsrc_t wr;
  // [N][K]: byte offset of the lane's 16 bytes of a weight row.  [K][N]: (only w_at[0]) of its 8 columns in its reduction
  // row of a load instruction: a tile row is 2 FN chunks wide, an instruction covers KROWS rows.
  constexpr int CH = 2 * FN, KROWS = 64 / CH;
  const int krow = lane / CH, kch = lane % CH;
  unsigned w_at[2 * FN];
  if constexpr (WKN) {
    wr = make_rsrc(p.W + n0, (unsigned)(((int64_t)(p.K - 1) * p.ldw + w_rows) * 2));
    w_at[0] = kch * 8 < w_rows ? ((unsigned)krow * (unsigned)p.ldw + kch * 8) * 2u : kInvalidOffset;
  } else {
    wr = make_rsrc(p.W + (int64_t)n0 * p.ldw, (unsigned)(((int64_t)(w_rows - 1) * p.ldw + p.K) * 2));
#pragma unroll
    for (int a = 0; a < 2 * FN; ++a)
      w_at[a] = a * 8 + lrow < w_rows ? ((unsigned)(a * 8 + lrow) * (unsigned)p.ldw + lk) * 2u : kInvalidOffset;
  }

  // ---- main loop: this wave's units, D of them in flight ---------------------------------------------------------------
  const int units = (p.K + 63) >> 6, upw = (units + NW - 1) / NW, u0 = wave * upw;
  const int n_units = units - u0 < upw ? units - u0 : upw;  // (may be negative: no work)
  uintx4 xv[D][2 * FM], wv[D][2 * FN];
  auto fetch = [&](int i, int set) {  // operands of this wave's unit i
    const int k0 = (u0 + i) * 64, k = k0 + lk;
    const bool on = k < p.K;
    if constexpr (XMODE == 0) {
#pragma unroll
      for (int b = 0; b < 2 * FM; ++b) {
        const unsigned off = on && x_at[b] != kInvalidOffset ? x_at[b] + (unsigned)k0 * 2u : kInvalidOffset;
        xv[set][b] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0));
      }
    } else {
      const int tap = fdiv(k, rcp_c), c = k - tap * cg.C;
      const int r = fdiv(tap, rcp_s), s = tap - r * cg.S;
      const int delta = (r * cg.Wi + s) * cg.C + c;
#pragma unroll
      for (int b = 0; b < 2 * FM; ++b) {
        const int ih = (ihw0[b] >> 16) + r, iw = (ihw0[b] & 0xffff) - (1 << 15) + s;
        const bool ok = on && (unsigned)ih < (unsigned)cg.H && (unsigned)iw < (unsigned)cg.Wi;
        const unsigned off = ok ? (unsigned)(x_px[b] + delta) * 2u : kInvalidOffset;
        xv[set][b] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0));
      }
    }
    if constexpr (WKN) {
#pragma unroll
      for (int a = 0; a < 2 * FN; ++a) {
        const bool ok = k0 + a * KROWS + krow < p.K && w_at[0] != kInvalidOffset;
        const unsigned off = ok ? (unsigned)(k0 + a * KROWS) * (unsigned)p.ldw * 2u + w_at[0] : kInvalidOffset;
        wv[set][a] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(wr, off, 0, 0));
      }
    } else {
#pragma unroll
      for (int a = 0; a < 2 * FN; ++a) {
        const unsigned off = on && w_at[a] != kInvalidOffset ? w_at[a] + (unsigned)k0 * 2u : kInvalidOffset;
        wv[set][a] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(wr, off, 0, 0));
      }
    }
  };
#pragma unroll
  for (int k = 0; k < D; ++k)
    if (k < n_units) fetch(k, k);

  // bias and residual of this thread's output quads, while the operands are on their way
  half4 hb[Tr::QPT], res[Tr::QPT];
#pragma unroll
  for (int i = 0; i < Tr::QPT; ++i) {
    const int quad = tid + i * NT, row = quad / (BN / 4), n = n0 + (quad - row * (BN / 4)) * 4;
    const bool ok = quad < Tr::QUADS && n < p.N;
    hb[i] = *(const half4*)(p.bias + (ok ? n : 0) * p.bias_on);
    if (!ok) hb[i] = half4{0, 0, 0, 0};
    res[i] = half4{0, 0, 0, 0};
    if constexpr (RES) {
      if (ok && m0 + row < p.M) res[i] = *(const half4*)(p.res + (int64_t)(m0 + row) * p.ldr + n);
    }
  }

  floatx4 acc[FN][FM];
#pragma unroll
  for (int a = 0; a < FN; ++a)
#pragma unroll
    for (int b = 0; b < FM; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  // The rows pass through a piece of LDS of the wave's own to get into operand order (a wave's LDS accesses are executed
  // in order, so no barrier): 128 bytes per row, 16-byte chunks XOR-swizzled by the row (bank conflicts: 1 to
  // 12 % of the LDS-active cycles).
  // Row-major weights stay [k][n]; the transposing read gathers 8 reduction indices of a column.  Its half-waves read
  // rows {0..3, 8..11} of 32 bytes, which the swizzle (kn_at) spreads over all banks.
  unsigned char* const stage = reinterpret_cast<unsigned char*>(lds) + wave * Tr::WAVE_BYTES;
  unsigned char* const wstage = stage + FM * 2048;
  auto kn_at = [](int k, int frag) {  // byte offset of the 16 columns of fragment `frag` in reduction row k
    if constexpr (FN == 1) return (k ^ ((k >> 1) & 4)) * 32;
    else if constexpr (FN == 2) return k * 64 + ((frag ^ (k >> 3)) & 1) * 32;
    else return k * 128 + ((frag ^ ((k >> 1) & 1) ^ ((k >> 2) & 2)) & 3) * 32;
  };
  unsigned put[2], get[2];  // rows lrow and lrow + 8 of a fragment; this lane's operand of indices 0 .. 31 and 32 .. 63
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = h * 8 + lrow;
    put[h] = row * 128 + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    get[h] = l16 * 128 + (((h * 4 + g4) ^ ((l16 >> 1) & 7)) << 4);
  }
  for (int i = 0; i < n_units; i += D) {
#pragma unroll
    for (int k = 0; k < D; ++k) {
      if (i + k < n_units) {
#pragma unroll
        for (int b = 0; b < 2 * FM; ++b) *(uintx4*)(stage + (b >> 1) * 2048 + put[b & 1]) = xv[k][b];
#pragma unroll
        for (int a = 0; a < 2 * FN; ++a) {
          if constexpr (WKN) *(uintx4*)(wstage + kn_at(a * KROWS + krow, kch >> 1) + (kch & 1) * 16) = wv[k][a];
          else *(uintx4*)(wstage + (a >> 1) * 2048 + put[a & 1]) = wv[k][a];
        }
        asm volatile("" ::: "memory");  // reads of what other lanes wrote stay behind the writes (and the next unit's writes behind them)
        if (i + k + D < n_units) fetch(i + k + D, k);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          half8 xf[FM], wf[FN];
#pragma unroll
          for (int b = 0; b < FM; ++b) xf[b] = *(const half8*)(stage + b * 2048 + get[h]);
#pragma unroll
          for (int a = 0; a < FN; ++a) {
            if constexpr (WKN) {
              const int r = h * 32 + g4 * 8 + (l16 >> 2);
              wf[a] = ws_transposed_read(wstage + kn_at(r, a) + (l16 & 3) * 8, wstage + kn_at(r + 4, a) + (l16 & 3) * 8);
            } else {
              wf[a] = *(const half8*)(wstage + a * 2048 + get[h]);
            }
          }
#pragma unroll
          for (int a = 0; a < FN; ++a)
#pragma unroll
            for (int b = 0; b < FM; ++b) acc[a][b] = mfma_16x16x32(wf[a], xf[b], acc[a][b]);
        }
        asm volatile("" ::: "memory");
      }
    }
  }

  // ---- sum over the waves through LDS, epilogue, store -------------------------------------------------------------------
#pragma unroll
  for (int b = 0; b < FM; ++b) {
    float* const row = part + wave * (Tr::WAVE_BYTES / 4) + (b * 16 + l16) * PITCH;
#pragma unroll
    for (int a = 0; a < FN; ++a) *(floatx4*)(row + a * 16 + g4 * 4) = acc[a][b];
  }
  barrier_after_lds_writes();
  const EpilogueArgs ep{p.bias, p.bias_on, p.N, p.alpha, p.beta, p.act, p.gamma};
#pragma unroll
  for (int i = 0; i < Tr::QPT; ++i) {
    const int quad = tid + i * NT, row = quad / (BN / 4), col = (quad - row * (BN / 4)) * 4;
    if (quad < Tr::QUADS && m0 + row < p.M && n0 + col < p.N) {
      floatx4 s = *(const floatx4*)(part + row * PITCH + col);
#pragma unroll
      for (int w = 1; w < NW; ++w) s += *(const floatx4*)(part + w * (Tr::WAVE_BYTES / 4) + row * PITCH + col);  // fixed order
      const half4 o = p.act > ACT_RELU ? epilogue_quad4_values<true, RES>(s, hb[i], ep, res[i])
                                       : epilogue_quad4_values<false, RES>(s, hb[i], ep, res[i]);
      *(half4*)(p.Y + (int64_t)(m0 + row) * p.ldy + n0 + col) = o;
    }
  }
}

template <int NW, int FM, int FN, int XMODE, bool WKN>
hipError_t launch_fprop_ws(const FpropParams& p, hipStream_t stream) {
  using Tr = FpropWsTraits<NW, FM, FN>;
  auto kern = p.res ? fprop_ws_kernel<NW, FM, FN, XMODE, WKN, true> : fprop_ws_kernel<NW, FM, FN, XMODE, WKN, false>;
  static LdsOptIn opt_in[2];
  if (hipError_t e = opt_in[p.res ? 1 : 0].ensure((const void*)kern, Tr::LDS_BYTES); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)Tr::workgroups(p), 1, 1), dim3(Tr::NT), Tr::LDS_BYTES, stream, p);
  return hipGetLastError();
}

// Tile extents as multiples of 32 that hold them (the unit of every tile in the table), waves as k-groups of 4.
#define BOLT_FPROP_WS_INSTANCE(NW, FM, FN, XMODE, WKN)                                                              \
  {                                                                                                                \
    "ws_" #NW "w_" #FM "x" #FN, (16 * FM + 31) / 32 * 32, (16 * FN + 31) / 32 * 32, 32, 4, 1, XMODE, WKN ? 1 : 0, 2, \
        bolt::FpropWsTraits<NW, FM, FN>::LDS_BYTES, &bolt::launch_fprop_ws<NW, FM, FN, XMODE, WKN>,                \
        &bolt::FpropWsTraits<NW, FM, FN>::supports, &bolt::FpropWsTraits<NW, FM, FN>::lds_bytes, NW / 4, 16, true, \
        false, WKN, &bolt::FpropWsTraits<NW, FM, FN>::estimate, &bolt::FpropWsTraits<NW, FM, FN>::worth_trying      \
  }

}  // namespace bolt
