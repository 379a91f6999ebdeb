// First-layer convolution for 3 or 4 input channels (an image's colour planes), NHWC without channel padding or NCHW: the
// layout transformation and the padding to 4 channels happen on the way to LDS.
//
// conv_smallc_kernel (any C <= 4) keeps the channels unpadded in LDS: it spends most of its vector instructions and LDS
// accesses on 2-byte granularity (8 2-byte LDS writes per 16 bytes of an NCHW plane, four 4-byte reads and four masks per
// fragment, all weights re-read from LDS per 32 pixels), stages every input row of a filter again for each output row, and
// always computes 128 columns.  Here
//   * a workgroup (4 waves) takes a strip of TP output rows x up to 128 columns x 64 channels and stages the strip's
//     (TP - 1) stride + R input rows once, as pixels of 4 channels (8 bytes; the 4th zero for C = 3).  A work item is 8
//     pixels of a row: aligned loads of the runs that hold them (C planes, or one NHWC run), shifted into place and
//     interleaved in registers, four 16-byte LDS writes;
//   * the reduction is ordered (r, s, c) with the taps of a filter row padded to an even number: a fragment of 8 halves is
//     two neighbouring taps, for a pixel ONE aligned 16-byte LDS read (two of 8 bytes for stride 1).  The odd tap behind a
//     filter row reads a real pixel: it is masked (its weights are zero as well, but 0 * inf is not 0);
//   * each wave keeps all 64 channels' weights in registers (T k-steps x 4 fragments, 112 registers for 7 x 7) and walks over
//     its share of the strip's 16-pixel blocks.
// TP is chosen so that the strips fill the chip's 512 workgroup slots in whole rounds (plan()).
// What bounds it: instruction issue.  Vector instructions take 54 % of the SIMD-cycles, matrix ones 26 %, two waves share a SIMD;
// the output leaves at 2.3 TB/s; 39 % of the LDS-active cycles are bank conflicts, with the LDS active in 28 % of all (counters
// of the first of these).  Measured, 32 images of 224 x 224 x 3, 7 x 7 / 2, 64 channels, NCHW, conv_smallc_kernel -> this one: 29 -> 21.5 us (NHWC 24.3 -> 19.7), 3 x 3 / 2 24.5 -> 14.5; 32 of 96 x 96, 7 x 7 / 2,
// 32 channels 15.0 -> 8.7; 1 of 224 x 224 7.5 -> 6.2.
#pragma once
#include "conv_smallc_kernel.hpp"

namespace bolt {

struct ConvFirstPlan {
  int tp, tiles_p;    // output rows of a strip, strips along P
  int tq, tiles_q;    // output columns of a strip (a multiple of 16 or all of them), strips along Q
  int rows, items;    // staged input rows, 8-pixel items of a row
  int lds_bytes;      // 0: does not fit
  int grid;           // workgroups per block of 64 channels
};

template <int T, int SW>
struct ConvFirstTraits {
  static constexpr int NT = 256, BN = 64, MAX_Q = 128, SLOTS = 512, MAX_LDS = 78 * 1024;  // two workgroups per compute unit
  // in front of the pixels: the weights on their way to registers, later a block's outputs of every wave (4 x 2 KB)
  static constexpr int FRONT_BYTES = T * 4096 > 8192 ? T * 4096 : 8192;
  static ConvFirstPlan plan(const FpropParams& p) {
    const ConvGeom& g = p.cg;
    ConvFirstPlan t{};
    t.tiles_q = (g.Q + MAX_Q - 1) / MAX_Q;
    t.tq = ((g.Q + t.tiles_q - 1) / t.tiles_q + 15) / 16 * 16;
    if (t.tq > g.Q) t.tq = g.Q;
    t.tiles_q = (g.Q + t.tq - 1) / t.tq;
    const int blocks = (t.tq + 15) / 16;
    // columns that the blocks' fragments read, in whole items
    t.items = ((blocks * 16 - 1) * SW + (g.S + 1) / 2 * 2 + 7) / 8;
    const int64_t images = p.M / (g.P * g.Q);
    const int slots = std::max(8, SLOTS / ((p.N + BN - 1) / BN) / 8 * 8);  // of one block of channels
    double best = 0;
    for (int tp = 1; tp <= g.P && tp <= 32; ++tp) {
      const int rows = (tp - 1) * g.stride_h + g.R, bytes = FRONT_BYTES + rows * t.items * 64;
      if (bytes > MAX_LDS) break;
      const int64_t tiles_p = (g.P + tp - 1) / tp, strips = images * tiles_p * t.tiles_q;
      if (strips >= (1ll << 31)) continue;
      // clocks: blocks of a wave, staging items of a thread, two barriers and a memory latency per strip
      const double cost = (double)((strips + slots - 1) / slots) * ((tp * blocks + 3) / 4 * (60.0 + 64.0 * T) + (rows * t.items + NT - 1) / NT * 500.0 + 2000.0);
      if (t.lds_bytes == 0 || cost < best) {
        best = cost;
        t.tp = tp;
        t.tiles_p = (int)tiles_p;
        t.rows = rows;
        t.lds_bytes = bytes;
        t.grid = (int)(strips < slots ? strips : slots);
      }
    }
    return t;
  }
  static bool supports(const FpropParams& p) {
    const ConvGeom& g = p.cg;
    // No call runs only here: which first layers are accepted stays what bolt.h says (conv_smallc_kernel's limits; 4 channels
    // from NHWC to NHWC also run on the alignment-2 kernels).
    if (!(g.C == 4 && !p.x_nchw && !p.y_nchw) && !ConvSmallCTraits<6, SW>::supports(p)) return false;
    return (g.C == 3 || g.C == 4) && g.stride_w == SW && g.R * ((g.S + 1) / 2) <= 4 * T && (int64_t)p.N * p.ldw * 2 < (1ll << 31) &&
           plan(p).lds_bytes > 0;
  }
  static int lds_bytes(const FpropParams& p) { return plan(p).lds_bytes; }
  // Pick rule: wherever one of these can run it is the fastest (24 problems: 1.2 to 1.9 times conv_smallc_kernel, 1 to 32
  // images of 32 to 500 pixels, both layouts), the shorter k loop first.
  static double estimate(const FpropParams&) { return 0.01 * T; }
};

template <int T, int SW, int C, bool NCHW>
__global__ __launch_bounds__(256, 2) void conv_first_kernel(const FpropParams p, const ConvFirstPlan pl) {
  using Tr = ConvFirstTraits<T, SW>;
  constexpr int NT = Tr::NT;
  // dwords that cover an item's runs: NCHW: C runs of 8 halves at any 2-byte boundary; NHWC: one run of 8 C halves (at
  // any 2-byte boundary for C = 3, at 8 bytes for C = 4)
  constexpr int RUNS = NCHW ? C : 1, RUN_DWORDS = NCHW ? 5 : C == 3 ? 13 : 16, NV = RUNS * RUN_DWORDS;
  extern __shared__ __attribute__((aligned(16))) half_t lds[];
  unsigned char* const out = reinterpret_cast<unsigned char*>(lds);  // [4 waves][16 pixels][64 channels]
  unsigned char* const px = out + Tr::FRONT_BYTES;                    // [rows][items * 8 pixels][4 channels]
  const ConvGeom& cg = p.cg;
  const int tid = threadIdx.x, lane = tid & 63, kg = lane >> 4, l16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NF = (cg.S + 1) / 2, nfrag = cg.R * NF, row_bytes = pl.items * 64;
  const float rcp_nf = 1.0f / (float)NF;  // (small exact divisions)

  // strips, columns fastest, then rows, images; every XCD (ids are dealt round-robin over 8) takes a contiguous run
  const int images = p.M / (cg.P * cg.Q), n0 = blockIdx.y * Tr::BN;
  const int total = images * pl.tiles_p * pl.tiles_q;
  int first = blockIdx.x, step = gridDim.x, end = total;
  if ((gridDim.x & 7) == 0) {
    const int band = (total + 7) >> 3, xcd = blockIdx.x & 7;
    first = xcd * band + (int)(blockIdx.x >> 3);
    step = gridDim.x >> 3;
    end = (xcd + 1) * band < total ? (xcd + 1) * band : total;
  }
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.W, (unsigned)((int64_t)p.N * p.ldw * 2));
  // (rounded up to whole dwords: the last element of a tensor with an odd element count shares its dword with two bytes
  // that still lie inside the caller's allocation - x is 16-byte aligned and allocations are multiples of 4)
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.X, ((unsigned)((int64_t)images * cg.H * cg.Wi * C * 2) + 3u) & ~3u);
  // weights of the lane's output channel in block b: 32 (b / 2) + 8 (i / 4) + 4 (b % 2) + i % 4 for operand row i, so that
  // a lane ends up with two runs of 8 consecutive channels of its pixel
  half8 wf[T][4];
  int f_at[T];                  // LDS byte offset of this lane's fragment of a k-step, from the block's first pixel
  unsigned lo_on = 0, hi_on = 0;  // bit t: its first, its second tap exists
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int f = t * 4 + kg, r = (int)(((float)f + 0.5f) * rcp_nf), sp = f - r * NF;
    f_at[t] = (f < nfrag ? r * row_bytes + sp * 16 : 0) + l16 * (SW * 8);
    lo_on |= (f < nfrag ? 1u : 0u) << t;
    hi_on |= (f < nfrag && 2 * sp + 1 < cg.S ? 1u : 0u) << t;
  }
  const bool tail = (nfrag & 3) != 0 || nfrag < 4 * T;  // some fragments have no tap at all
  // A thread fetches every fourth fragment of one channel, so that four lanes read one run of a weight row; the fragments
  // go through LDS once (each lane fetching its own from memory would touch 64 cache lines per load).
  const int w_chl = tid >> 2, w_sub = tid & 3;
  const int w_dst = ((2 * (w_chl >> 5) + ((w_chl >> 2) & 1)) * 64 + w_sub * 16 + 4 * ((w_chl >> 3) & 3) + (w_chl & 3)) * 16;
  uintx4 w_raw[T];
  auto fetch_weights = [&] {
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int f = t * 4 + w_sub, r = (int)(((float)f + 0.5f) * rcp_nf), sp = f - r * NF, ch = n0 + w_chl;
      const int h0 = ch * p.ldw + (r * cg.S + 2 * sp) * C;
      w_raw[t] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(
                                                wr, f < nfrag && ch < p.N ? (unsigned)(h0 >> 1) * 4u : kInvalidOffset, 0, 0));
    }
  };
  auto stage_weights = [&] {
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int f = t * 4 + w_sub, r = (int)(((float)f + 0.5f) * rcp_nf), sp = f - r * NF;
      const bool lo = f < nfrag, hi = lo && 2 * sp + 1 < cg.S;
      const uintx4 v = w_raw[t];
      uintx4 o = v;
      if constexpr (C == 3) {
        const unsigned sh = (unsigned)(((n0 + w_chl) * p.ldw + (r * cg.S + 2 * sp) * C) & 1) * 16u;
        const unsigned c0 = __builtin_amdgcn_alignbit(v[1], v[0], sh), c1 = __builtin_amdgcn_alignbit(v[2], v[1], sh),
                       c2 = __builtin_amdgcn_alignbit(v[3], v[2], sh);  // halves 0 .. 5
        o = uintx4{c0, c1 & 0xffffu, __builtin_amdgcn_alignbit(c2, c1, 16), c2 >> 16};
      }
      *(uintx4*)(out + t * 4096 + w_dst) = uintx4{lo ? o[0] : 0u, lo ? o[1] : 0u, hi ? o[2] : 0u, hi ? o[3] : 0u};
    }
    barrier_after_lds_writes();
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int b = 0; b < 4; ++b) wf[t][b] = *(const half8*)(out + t * 4096 + (b * 64 + lane) * 16);
  };
  floatx4 bias_f[4];  // beta * bias of the lane's channels
#pragma unroll
  for (int hb = 0; hb < 2; ++hb) {
    const int n = n0 + 32 * hb + 8 * kg;
    const half8 got = *(const half8*)(p.bias + (n < p.N ? n : 0) * p.bias_on);
#pragma unroll
    for (int e = 0; e < 8; ++e) bias_f[2 * hb + e / 4][e % 4] = n < p.N && p.bias_on ? p.beta * (float)got[e] : 0.f;
  }
  int img, p0, q0, ih0, iw0;
  auto locate = [&](int strip) {
    const int row = strip / pl.tiles_q;
    q0 = (strip - row * pl.tiles_q) * pl.tq;
    img = row / pl.tiles_p;
    p0 = (row - img * pl.tiles_p) * pl.tp;
    ih0 = p0 * cg.stride_h - cg.pad_h;
    iw0 = q0 * SW - cg.pad_w;
  };

  // ---- staging -------------------------------------------------------------------------------------------------------
  const int n_items = pl.rows * pl.items;
  const float rcp_items = 1.0f / (float)pl.items;
  // v: an item's dwords; at: the first half of its (first) run in the tensor; col: the image column of its first pixel
  auto fetch = [&](int i, unsigned(&v)[NV], int& at, int& col) {
    const int row = (int)(((float)i + 0.5f) * rcp_items), x0 = (i - row * pl.items) * 8;  // (exact: i < 2^16)
    const int ih = ih0 + row;
    col = iw0 + x0;
    at = NCHW ? (img * C * cg.H + ih) * cg.Wi + col : ((img * cg.H + ih) * cg.Wi + col) * C;
    const bool ok = i < n_items && (unsigned)ih < (unsigned)cg.H && col < cg.Wi;
#pragma unroll
    for (int u = 0; u < RUNS; ++u) {
      const int a4 = ((at + u * cg.H * cg.Wi) >> 1) * 4;
      unsigned* const d = v + u * RUN_DWORDS;
      // an item that starts in front of the tensor (left of the first image's rows) takes single dwords: those in front
      // hold only columns that are zeroed below
      if (a4 >= 0) {
#pragma unroll
        for (int n = 0; n + 4 <= RUN_DWORDS; n += 4) {
          const auto got = __builtin_amdgcn_raw_buffer_load_b128(xr, ok ? (unsigned)a4 + 4u * n : kInvalidOffset, 0, 0);
          d[n] = got[0]; d[n + 1] = got[1]; d[n + 2] = got[2]; d[n + 3] = got[3];
        }
        if constexpr (RUN_DWORDS % 4 == 1)
          d[RUN_DWORDS - 1] = __builtin_amdgcn_raw_buffer_load_b32(xr, ok ? (unsigned)a4 + 4u * (RUN_DWORDS - 1) : kInvalidOffset, 0, 0);
      } else {
#pragma unroll
        for (int n = 0; n < RUN_DWORDS; ++n) {
          const int off = a4 + 4 * n;
          d[n] = __builtin_amdgcn_raw_buffer_load_b32(xr, ok ? (unsigned)(off > 0 ? off : 0) : kInvalidOffset, 0, 0);
        }
      }
    }
  };
  auto scatter = [&](int i, const unsigned(&v)[NV], int at, int col) {
    uintx4 o[4];  // 8 pixels of 4 channels
    if constexpr (NCHW) {
      unsigned c[4][4];  // [channel][pixel pair]
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const unsigned sh = u < C ? (unsigned)((at + u * cg.H * cg.Wi) & 1) * 16u : 0u;
#pragma unroll
        for (int n = 0; n < 4; ++n)
          c[u][n] = u < C ? __builtin_amdgcn_alignbit(v[(u < C ? u : 0) * RUN_DWORDS + n + 1], v[(u < C ? u : 0) * RUN_DWORDS + n], sh) : 0u;
      }
#pragma unroll
      for (int n = 0; n < 4; ++n) {  // pixels 2n, 2n + 1: low halves, high halves of two channels
        o[n][0] = __builtin_amdgcn_perm(c[1][n], c[0][n], 0x05040100u);
        o[n][1] = C == 4 ? __builtin_amdgcn_perm(c[3][n], c[2][n], 0x05040100u) : c[2][n] & 0xffffu;
        o[n][2] = __builtin_amdgcn_perm(c[1][n], c[0][n], 0x07060302u);
        o[n][3] = C == 4 ? __builtin_amdgcn_perm(c[3][n], c[2][n], 0x07060302u) : c[2][n] >> 16;
      }
    } else if constexpr (C == 3) {
      const unsigned sh = (unsigned)(at & 1) * 16u;
      unsigned s[12];
#pragma unroll
      for (int n = 0; n < 12; ++n) s[n] = __builtin_amdgcn_alignbit(v[n + 1], v[n], sh);
#pragma unroll
      for (int n = 0; n < 4; ++n)  // pixels 2n, 2n + 1 = halves 6n .. 6n + 5
        o[n] = uintx4{s[3 * n], s[3 * n + 1] & 0xffffu, __builtin_amdgcn_alignbit(s[3 * n + 2], s[3 * n + 1], 16), s[3 * n + 2] >> 16};
    } else {
#pragma unroll
      for (int n = 0; n < 4; ++n) o[n] = uintx4{v[4 * n], v[4 * n + 1], v[4 * n + 2], v[4 * n + 3]};
    }
    if (col < 0 || col + 8 > cg.Wi) {  // on the image's edge: zero the pixels outside
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const bool e = (unsigned)(col + 2 * n) < (unsigned)cg.Wi, f = (unsigned)(col + 2 * n + 1) < (unsigned)cg.Wi;
        o[n] = uintx4{e ? o[n][0] : 0u, e ? o[n][1] : 0u, f ? o[n][2] : 0u, f ? o[n][3] : 0u};
      }
    }
    if (i < n_items) {
#pragma unroll
      for (int n = 0; n < 4; ++n) *(uintx4*)(px + i * 64 + n * 16) = o[n];
    }
  };
  if (first >= end) return;
  // (one item of a thread in flight at a time: with three, 45 registers and a call of all of them for the smallest strips,
  // every size was slower)
  unsigned v[NV];
  int at, col;
  fetch_weights();
  locate(first);
  fetch(tid, v, at, col);
  stage_weights();

  for (int strip = first; strip < end; strip += step) {
    scatter(tid, v, at, col);
    for (int i = tid + NT; i < n_items; i += NT) {
      fetch(i, v, at, col);
      scatter(i, v, at, col);
    }
    __syncthreads();

    // ---- the strip's blocks of 16 pixels, dealt over the waves ------------------------------------------------------------
    const int blocks = (pl.tq + 15) / 16;
    const int rows_here = cg.P - p0 < pl.tp ? cg.P - p0 : pl.tp, n_blocks = rows_here * blocks;
    const float rcp_blocks = 1.0f / (float)blocks;
    for (int u = wave; u < n_blocks; u += 4) {
      const int ty = __builtin_amdgcn_readfirstlane((int)(((float)u + 0.5f) * rcp_blocks));
      const int qb = (u - ty * blocks) * 16, prow = p0 + ty;
      const unsigned src = ty * cg.stride_h * row_bytes + qb * (SW * 8);
      floatx4 acc[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[b] = floatx4{0.f, 0.f, 0.f, 0.f};
      uintx4 x[2];  // the fragment of this k-step and of the next
      auto read = [&](int t) {
        const unsigned char* const at = px + (src + f_at[t]);
        if constexpr (SW == 2) {
          x[t & 1] = *(const uintx4*)at;
        } else {
          const uint2 a = *(const uint2*)at, z = *(const uint2*)(at + 8);
          x[t & 1] = uintx4{a.x, a.y, z.x, z.y};
        }
      };
      read(0);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        if (t + 1 < T) read(t + 1);
        __builtin_amdgcn_sched_barrier(0);  // (k-steps are kept apart: all reads in front would need 28 registers)
        const unsigned hi = (unsigned)((int)(hi_on << (31 - t)) >> 31);
        uintx4 v = x[t & 1];
        v[2] &= hi;
        v[3] &= hi;
        if (tail) {
          const unsigned lo = (unsigned)((int)(lo_on << (31 - t)) >> 31);
          v[0] &= lo;
          v[1] &= lo;
        }
        const half8 xf = __builtin_bit_cast(half8, v);
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[b] = mfma_16x16x32(wf[t][b], xf, acc[b]);
      }
      // this lane holds channels n0 + 8 kg + [0, 8) and n0 + 32 + 8 kg + [0, 8) of its pixel
      auto store = [&](auto act) {
        constexpr int ACT = decltype(act)::value;  // none, ReLU or any of the others
        const int q = q0 + qb + l16;
        half8 o[2];
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
          for (int b2 = 0; b2 < 2; ++b2) {
            floatx4 s;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              s[e] = p.alpha * acc[2 * hb + b2][e] + bias_f[2 * hb + b2][e];
              if constexpr (ACT == ACT_RELU) s[e] = s[e] > 0.f ? s[e] : 0.f;
            }
            if constexpr (ACT > ACT_RELU) s = apply_act_slow4_inline(s, p.act);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[hb][4 * b2 + e] = (half_t)s[e];
          }
        if (!p.y_nchw) {
          // through LDS (the wave's own 2 KB: its accesses are executed in order), so that a store instruction writes whole
          // runs: 8 lanes the 128 bytes of one pixel, chunks XOR-swizzled by the pixel
          unsigned char* const mine = out + wave * (16 * Tr::BN * 2);
          auto place = [](int pix, int ch) { return pix * 128 + ((ch ^ ((pix >> 1) & 7)) << 4); };
#pragma unroll
          for (int hb = 0; hb < 2; ++hb) *(half8*)(mine + place(l16, hb * 4 + kg)) = o[hb];
          asm volatile("" ::: "memory");  // reads of what other lanes wrote stay behind the writes, the next block's writes behind them
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int pix = h * 8 + (lane >> 3), ch = lane & 7;
            const half8 v = *(const half8*)(mine + place(pix, ch));
            half_t* const y = p.Y + (((int64_t)img * cg.P + prow) * cg.Q + q0 + qb) * p.ldy + n0;  // (the same in all lanes)
            if (n0 + ch * 8 < p.N && q0 + qb + pix < cg.Q) __builtin_nontemporal_store(v, (half8*)(y + (unsigned)(pix * p.ldy + ch * 8)));
          }
          asm volatile("" ::: "memory");
        } else if (q < cg.Q) {  // [N][K][P][Q]: 8 channel planes, 16 consecutive pixels of each
#pragma unroll
          for (int hb = 0; hb < 2; ++hb) {
            const int n = n0 + 32 * hb + 8 * kg;
            half_t* y = p.Y + (((int64_t)img * p.N + n) * cg.P + prow) * cg.Q + q;
            if (n < p.N) {
#pragma unroll
              for (int k = 0; k < 8; ++k) y[(int64_t)k * cg.P * cg.Q] = o[hb][k];
            }
          }
        }
      };
      if (p.act == ACT_RELU) store(std::integral_constant<int, ACT_RELU>{});
      else if (p.act == ACT_NONE) store(std::integral_constant<int, ACT_NONE>{});
      else store(std::integral_constant<int, ACT_GELU>{});
    }
    if (strip + step < end) {
      locate(strip + step);
      fetch(tid, v, at, col);
      raw_barrier();  // every wave has read its pixels: they may be overwritten
    }
  }
}

template <int T, int SW>
hipError_t launch_conv_first(const FpropParams& p, hipStream_t stream) {
  using Tr = ConvFirstTraits<T, SW>;
  const ConvFirstPlan t = Tr::plan(p);
  const int which = (p.cg.C == 4 ? 2 : 0) + (p.x_nchw ? 1 : 0);
  void (*const kernels[4])(FpropParams, ConvFirstPlan) = {conv_first_kernel<T, SW, 3, false>, conv_first_kernel<T, SW, 3, true>,
                                                          conv_first_kernel<T, SW, 4, false>, conv_first_kernel<T, SW, 4, true>};
  static LdsOptIn opt_in[4];
  if (hipError_t e = opt_in[which].ensure((const void*)kernels[which], Tr::MAX_LDS); e != hipSuccess) return e;
  hipLaunchKernelGGL(kernels[which], dim3((unsigned)t.grid, (unsigned)((p.N + Tr::BN - 1) / Tr::BN), 1), dim3(Tr::NT), t.lds_bytes, stream, p, t);
  return hipGetLastError();
}

// In the instance table as conv_smallc_kernel: x mode 4, tile = 128 columns x 64 channels.
#define BOLT_CONV_FIRST_INSTANCE(T, SW)                                                                                  \
  {                                                                                                                      \
    "first_t" #T "_sw" #SW, 128, 64, 32, 4, 1, 4, 0, 1, 0, &bolt::launch_conv_first<T, SW>,                               \
        &bolt::ConvFirstTraits<T, SW>::supports, &bolt::ConvFirstTraits<T, SW>::lds_bytes, 0, 16, true, false, false,     \
        &bolt::ConvFirstTraits<T, SW>::estimate                                                                          \
  }

}  // namespace bolt
