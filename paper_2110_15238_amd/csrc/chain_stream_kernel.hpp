// GEMM chains and pairs with a thin first op: rows stream through independent waves, all weights resident in LDS.
// Instantiated in a file of its own (inst_chain_stream.hip): the out-of-line activation is compiled once per file, for the
// register budget of all its callers there, so that these kernels beside the tiled chains changed the latters' code.
#pragma once
#include "b2b_chain_kernel.hpp"

namespace bolt {

// The GEMM chain, and pair (N2T = 0), for thin first ops (K0 <= KT): rows stream through waves that share nothing but the weights.
// All three weight matrices stay in LDS; a wave owns 32 rows of the chain from end to end.  It loads its activations in
// matrix-core operand order straight to registers, requests the next 32 rows as soon as op0 has used them, and takes its
// output tile through a piece of LDS of its own, so the loop has no workgroup barrier and no operand staging: with a
// reduction of one or two k-tiles the pipeline of b2b_chain_kernel is all fill and drain, every workgroup loading, computing
// and storing in lockstep.
// What bounds it: below 32768 rows the fill (weights and first rows, one round trip) and the chain of the three products;
// above, issue and latency as much as memory: at 128320 rows and 3.5 TB/s vector instructions take 45 % of the SIMD-cycles, matrix
// ones 11 %, and waves wait for 46 % of their life.  Two waves per SIMD: at three the prefetched rows spill (56 registers).
// Measured, best tiled instance -> this one, ReLU, us (HIP-graph replay): 128320 x 96 -> 32 -> 96 -> 32 13.6 -> 10.8 (3.0 TB/s), 128 -> 64 -> 128 -> 64 27.8 -> 16.5,
// 104 -> 56 -> 64 -> 128 27.9 -> 15.4, 128 -> 64 -> 64 -> 64 15.7 -> 13.3; 65536 x 104 -> 56 -> 64 -> 128 14.9 -> 10.2, but
// 65536 x 128 -> 64 -> 64 -> 64 8.5 -> 9.0 and 8192 x 128 -> 64 -> 128 -> 64 7.5 -> 8.5: see the pick rule of the chains.
// The pair: 131072 x 96 -> 64 -> 32 10.1 -> 7.8 us, 128 -> 64 -> 128 17.5 -> 14.4, 128 -> 64 -> 64 12.3 -> 10.9.
template <int NW, int KT, int N0T, int N1T, int N2T>
struct ChainStreamTraits {
  static constexpr int BM = 32 * NW;
  static constexpr int NLT = N2T ? N2T : N1T;  // width of the last op
  static constexpr int WEIGHT_HALVES = KT * N0T + N0T * N1T + N1T * N2T, OUT_HALVES = 32 * NLT;  // OUT: per wave
  static constexpr int BIAS_HALVES = N0T + N1T + N2T;
  static constexpr int LDS_BYTES = (WEIGHT_HALVES + NW * OUT_HALVES + BIAS_HALVES) * 2;
  static constexpr int WGS_PER_CU = 160 * 1024 / LDS_BYTES < 8 / NW ? 160 * 1024 / LDS_BYTES : 8 / NW;  // 2 waves per SIMD
  static_assert(KT % 64 == 0 && N0T % 32 == 0 && N1T % 32 == 0 && (NLT == 32 || NLT == 64 || NLT == 128), "tile shape");
  static_assert(WGS_PER_CU >= 1, "LDS");
  static bool supports(const B2bParams& p) { return p.K0 <= KT; }
  static int lds_bytes(const B2bParams&) { return LDS_BYTES; }
  static int grid(const B2bParams& p) {  // every wave the same number of 32-row tiles, give or take one
    const int64_t tiles = ((int64_t)p.M + 31) / 32, most = 256 * WGS_PER_CU * NW;
    const int64_t rounds = (tiles + most - 1) / most;
    return (int)((tiles + rounds * NW - 1) / (rounds * NW));
  }
};

// b2b_make_d with the bias of the op in LDS, zeros for columns beyond N.  (A bias read from memory behind the request for the
// next rows waits for those rows too, loads return in order: 1.5 to 2.5 us per launch, whatever M.)
template <int FN>
__device__ __forceinline__ void chain_stream_make_d(const EpilogueArgs& ep, const half_t* bias, const floatx16 (&acc)[FN][1],
                                                    half8 (&d)[FN * 2][1], int g) {
  const half4 z = {0, 0, 0, 0};
  auto make = [&](auto slow) {
#pragma unroll
    for (int a = 0; a < FN; ++a)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        half4 o[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int q = 2 * h + u, c = a * 32 + q * 8 + g * 4;
          const floatx4 a4 = {acc[a][0][q * 4], acc[a][0][q * 4 + 1], acc[a][0][q * 4 + 2], acc[a][0][q * 4 + 3]};
          o[u] = epilogue_quad4_values<decltype(slow)::value, false>(a4, *(const half4*)(bias + c), ep, z);
          if (c >= ep.N) o[u] = z;
        }
        d[a * 2 + h][0] = half8{o[0][0], o[0][1], o[0][2], o[0][3], o[1][0], o[1][1], o[1][2], o[1][3]};
      }
  };
  if (ep.act > ACT_RELU) make(std::true_type{});
  else make(std::false_type{});
}

// KU, NU: reduction indices of the first op and columns of a 128-wide one that are computed, of KT and 128 that the layouts are made for.
template <int NW, int KT, int N0T, int N1T, int N2T, int KU, int NU, bool RES, bool WKN>
__global__ __launch_bounds__(64 * NW, 2) void chain_stream_kernel(const B2bParams p) {
  using T = ChainStreamTraits<NW, KT, N0T, N1T, N2T>;
  constexpr int NLT = T::NLT, CPR = NLT / 8;
  constexpr int N0U = N0T < NU ? N0T : NU, N1U = N1T < NU ? N1T : NU, NLU = NLT < NU ? NLT : NU;
  constexpr int KS = KU / 16, FN0 = N0U / 32, FNL = NLU / 32;
  extern __shared__ __attribute__((aligned(16))) half_t lds[];
  half_t* const W0s = lds;
  half_t* const W1s = W0s + KT * N0T;
  half_t* const W2s = W1s + N0T * N1T;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  half_t* const out = W2s + N1T * N2T + wave * T::OUT_HALVES;
  half_t* const bias0 = W2s + N1T * N2T + NW * T::OUT_HALVES;
  half_t* const bias1 = bias0 + N0T;
  half_t* const bias2 = bias1 + N1T;
  const int step = (int)gridDim.x * NW;
  const int tiles = (p.M - 1) / 32 + 1;
  int t = __builtin_amdgcn_readfirstlane((int)blockIdx.x * NW + wave);

  b2b_issue_weights<N0T, KT, NW, WKN>(p.W0, p.ldw0, p.N0, p.K0, W0s, p.cg, wave, lane);
  b2b_issue_weights<N1T, N0T, NW, WKN>(p.W1, p.ldw1, p.N1, p.N0, W1s, p.cg, wave, lane);
  if constexpr (N2T > 0) b2b_issue_weights<N2T, N1T, NW, WKN>(p.W2, p.ldw2, p.N2, p.N1, W2s, p.cg, wave, lane);

  half8 x[KS];
  auto load_rows = [&](int tile) {  // lane: row l32, reduction indices 16 ks + 8 g ..; zeros past M and K0
    const int m0 = tile * 32;
    const int64_t rem = ((int64_t)(p.M - m0 - 1) * p.ldx + p.K0) * 2;
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.X + (int64_t)m0 * p.ldx, (unsigned)(rem < 0x7fffffff ? rem : 0x7fffffff));
    const bool row_ok = m0 + l32 < p.M;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int k = ks * 16 + g * 8;
      const unsigned off = row_ok && k < p.K0 ? (unsigned)(l32 * p.ldx + k) * 2u : kInvalidOffset;
      x[ks] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0));
    }
  };
  if (t < tiles) load_rows(t);
  for (int i = tid; i < N0T; i += 64 * NW) bias0[i] = i < p.N0 ? p.b0[i * p.b0_on] : (half_t)0;
  for (int i = tid; i < N1T; i += 64 * NW) bias1[i] = i < p.N1 ? p.b1[i * p.b1_on] : (half_t)0;
  if constexpr (N2T > 0)
    for (int i = tid; i < N2T; i += 64 * NW) bias2[i] = i < p.N2 ? p.b2[i * p.b2_on] : (half_t)0;
  barrier_after_loads<0>();  // the weights ...
  __syncthreads();           // ... and the biases; no barrier after this one

  int w0off[WKN ? FN0 : 1];
  if constexpr (WKN) {
#pragma unroll
    for (int a = 0; a < FN0; ++a) w0off[a] = kn_frag_offset<N0T>(a * 32, lane);
  }
  // last epilogue: quads -> this wave's [32][NLT] tile in LDS -> 16-byte row stores.  One wave's LDS accesses are served
  // in order, so no barrier; the empty asm keeps the compiler from moving accesses between the layouts across each other.
  auto tile_out = [&](int tile, const floatx16 (&acc)[FNL][1], const EpilogueArgs& ep, const half_t* bias) {
    const int m0 = tile * 32;
    asm volatile("" ::: "memory");
    if constexpr (RES) {  // the residual takes the slots that the output will; C may be the output: these rows are this wave's
#pragma unroll
      for (int i = 0; i < CPR / 2; ++i) {
        const int row = i * (64 / CPR) + lane / CPR, chunk = lane % CPR;
        half8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (m0 + row < p.M && chunk * 8 < ep.N) v = *(const half8*)(p.res + (int64_t)(m0 + row) * p.ldr + chunk * 8);
        *(half8*)(out + row * NLT + ((chunk ^ ctile_swizzle<CPR>(row)) << 3)) = v;
      }
      asm volatile("" ::: "memory");
    }
    auto to_lds = [&](auto slow) {
#pragma unroll
      for (int a = 0; a < FNL; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int nl = a * 32 + q * 8 + g * 4;
          half4* const slot = (half4*)(out + l32 * NLT + (((nl >> 3) ^ ctile_swizzle<CPR>(l32)) << 3) + (nl & 4));
          const floatx4 a4 = {acc[a][0][q * 4], acc[a][0][q * 4 + 1], acc[a][0][q * 4 + 2], acc[a][0][q * 4 + 3]};
          half4 res = {0, 0, 0, 0};
          if constexpr (RES) res = *slot;
          *slot = epilogue_quad4_values<decltype(slow)::value, RES>(a4, *(const half4*)(bias + nl), ep, res);
        }
    };
    if (ep.act > ACT_RELU) to_lds(std::true_type{});
    else to_lds(std::false_type{});
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < CPR / 2; ++i) {
      const int row = i * (64 / CPR) + lane / CPR, chunk = lane % CPR;
      const half8 v = *(const half8*)(out + row * NLT + ((chunk ^ ctile_swizzle<CPR>(row)) << 3));
      if (m0 + row < p.M && chunk * 8 < ep.N) __builtin_nontemporal_store(v, (half8*)(p.Y + (int64_t)(m0 + row) * p.ldy + chunk * 8));
    }
    asm volatile("" ::: "memory");
  };
  for (; t < tiles; t += step) {
    floatx16 acc0[FN0][1];
#pragma unroll
    for (int a = 0; a < FN0; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc0[a][0][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int a = 0; a < FN0; ++a) {
        half8 w;
        if constexpr (WKN) w = kn_frag_read<N0T>(W0s, w0off[a], ks * 16);
        else w = *(const half8*)(W0s + (ks / 4) * N0T * 64 + dma_chunk_offset<64>(a * 32 + l32, (ks & 3) * 2 + g));
        acc0[a][0] = mfma_32x32x16(w, x[ks], acc0[a][0]);
      }
    if (t + step < tiles) load_rows(t + step);
    __builtin_amdgcn_sched_barrier(0);

    half8 d0[N0U / 16][1];
    chain_stream_make_d<FN0>(EpilogueArgs{p.b0, p.b0_on, p.N0, p.alpha0, p.beta0, p.act0}, bias0, acc0, d0, g);
    floatx16 acc1[N1U / 32][1];
    b2b_rf_gemm<N0T, N1T, 1, WKN, N0U, N1U>(W1s, d0, acc1, l32, g);
    if constexpr (N2T > 0) {
      half8 d1[N1U / 16][1];
      chain_stream_make_d<N1U / 32>(EpilogueArgs{p.b1, p.b1_on, p.N1, p.alpha1, p.beta1, p.act1}, bias1, acc1, d1, g);
      floatx16 acc2[FNL][1];
      b2b_rf_gemm<N1T, NLT, 1, WKN, N1U, NLU>(W2s, d1, acc2, l32, g);
      tile_out(t, acc2, EpilogueArgs{p.b2, p.b2_on, p.N2, p.alpha2, p.beta2, p.act2, RES ? p.gamma : 0.f}, bias2);
    } else {
      tile_out(t, acc1, EpilogueArgs{p.b1, p.b1_on, p.N1, p.alpha1, p.beta1, p.act1, RES ? p.gamma : 0.f}, bias1);
    }
  }
}

template <int NW, int KT, int N0T, int N1T, int N2T, int KU, int NU, bool WKN>
hipError_t launch_chain_stream_as(const B2bParams& p, hipStream_t stream) {
  static LdsOptIn opt_in[2];
  using T = ChainStreamTraits<NW, KT, N0T, N1T, N2T>;
  if (p.res)
    return b2b_launch_common(chain_stream_kernel<NW, KT, N0T, N1T, N2T, KU, NU, true, WKN>, opt_in[1], p, T::grid(p), 64 * NW,
                             T::LDS_BYTES, stream);
  return b2b_launch_common(chain_stream_kernel<NW, KT, N0T, N1T, N2T, KU, NU, false, WKN>, opt_in[0], p, T::grid(p), 64 * NW,
                           T::LDS_BYTES, stream);
}
// What of the compiled widths is only padding is not computed: loads, products and epilogues of it take the issue slots that bound
// the kernel.  (32 at a time of 128: up to 96 and above, of the reduction and of the 128-wide op.  128320 x 96 -> 32 -> 96 -> 32 11.8 -> 10.6 us,
// 70992 x 88 -> 48 -> 72 12.2 -> 10.7, 56016 x 16 -> 40 -> 72 7.9 -> 7.1, 98632 x 32 -> 32 -> 56 -> 16 10.6 -> 10.0, 41440 x 88 -> 64 -> 32 5.7 -> 5.5.  A
// reduction of up to 64 as a third form would save another quarter of the loads, for half as many kernels again.)
template <int NW, int KT, int N0T, int N1T, int N2T, bool WKN>
hipError_t launch_chain_stream(const B2bParams& p, hipStream_t stream) {
  static_assert(KT == 128 && N0T <= 128 && N1T <= 128 && N2T <= 128, "widths that the rule below knows");
  const bool narrow = (N0T < 128 || p.N0 <= 96) && (N1T < 128 || p.N1 <= 96) && (N2T < 128 || p.N2 <= 96);
  if constexpr (N0T == 128 || N1T == 128 || N2T == 128) {
    if (narrow)
      return p.K0 <= 96 ? launch_chain_stream_as<NW, KT, N0T, N1T, N2T, 96, 96, WKN>(p, stream)
                        : launch_chain_stream_as<NW, KT, N0T, N1T, N2T, KT, 96, WKN>(p, stream);
  }
  return p.K0 <= 96 ? launch_chain_stream_as<NW, KT, N0T, N1T, N2T, 96, 128, WKN>(p, stream)
                    : launch_chain_stream_as<NW, KT, N0T, N1T, N2T, KT, 128, WKN>(p, stream);
}

// The GEMM pair on the same kernel: N2T = 0.
template <int NW, int KT, int N0T, int N1T, bool WKN>
hipError_t launch_pair_stream(const B2bParams& p, int /*grid*/, int /*lds_bytes*/, hipStream_t stream) {
  return launch_chain_stream<NW, KT, N0T, N1T, 0, WKN>(p, stream);
}
#define BOLT_PAIR_STREAM_INSTANCE(NW, KT, N0T, N1T, WKN)                                                      \
  {                                                                                                          \
    "pairstream_k" #KT "_w" #NW "_n" #N0T "_" #N1T, 0, 32 * NW, 64, NW, 1, N0T, N1T, 0, WKN ? 1 : 0, 64 * NW, 1, \
        nullptr, &bolt::launch_pair_stream<NW, KT, N0T, N1T, WKN>,                                             \
        &bolt::ChainStreamTraits<NW, KT, N0T, N1T, 0>::supports,                                               \
        &bolt::ChainStreamTraits<NW, KT, N0T, N1T, 0>::lds_bytes, true, 0.f                                    \
  }

#define BOLT_CHAIN_STREAM_INSTANCE(NW, KT, N0T, N1T, N2T, WKN)                                                  \
  {                                                                                                            \
    "chainstream_k" #KT "_w" #NW "_n" #N0T "_" #N1T "_" #N2T, 32 * NW, 64, NW, N0T, N1T, N2T, 0, 1, 0,           \
        &bolt::launch_chain_stream<NW, KT, N0T, N1T, N2T, WKN>,                                                  \
        &bolt::ChainStreamTraits<NW, KT, N0T, N1T, N2T>::supports,                                               \
        &bolt::ChainStreamTraits<NW, KT, N0T, N1T, N2T>::lds_bytes, WKN ? 1 : 0                                  \
  }

}  // namespace bolt
