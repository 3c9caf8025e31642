// W4A4 GEMM for one to a few hundred token rows (gfx950, v_mfma_i32_16x16x64_i8):
// decode steps, and the shapes whose large output tiles would leave most of the
// chip idle.
//
//   acc_b[m,n] = sum_{k in group b} q_a[m,k] q_w[n,k]                 (int32)
//   Y[m,n]     = sw[n] * sum_b s[m,b] * (acc_b[m,n] - z[m,b] * colsum[b,n])
//
// What bounds it: at these sizes the chip is filled by splitting K, not by
// the output. A workgroup of P waves owns a small tile (16 MT tokens x 16 T
// channels) and its waves take 1/P of K each, straight from global memory
// (no LDS stage, no barrier in the loop): a wave's weight load is one 1 KB
// block of the blocked layout and its activation load 16 rows of 64 bytes, so
// every cache line is used whole, and NB steps of 128 k are in flight per
// wave. The P fp32 partial tiles meet in LDS at the end. What is left is
// latency: at 333 x 4096 x 14336 (384 tiles of 64 x 64 by four waves, one step in
// flight, two waves per SIMD) the waves wait 45 % of their cycles, with the matrix
// cores busy 18 % of the time, the VALU 26 % and the address units 44 %; decode
// products wait 47 to 64 %, address units 9 to 46 %.
//
// Every accumulator holds 16 acc exactly (weight nibbles widened to 16 q);
// per group F += (s / 16) acc; the zero-point terms are a rank-G product that
// runs on the fp32 matrix cores after the loop, a share of the groups per wave.
#include "common.h"
#include "gemm_common.h"
#include "internal.h"

namespace offq {
namespace {

using namespace gemm;

typedef float ks_f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int ks_u32x2 __attribute__((ext_vector_type(2)));

constexpr int KS_STEP = 128;  // k per step (64 packed bytes per row)

// dynamic LDS: scale and zero-point of the tile's tokens (one word each) and
// column sums of its channels per group, or the partial tiles at the end
template <int MT, int T, int P>
constexpr int64_t ks_lds_bytes(int64_t G) {
  const int64_t par = (16 * MT * (G | 1) + G * 16 * T) * 4;
  const int64_t red = (int64_t)P * MT * T * 64 * 16;
  return par > red ? par : red;
}

template <int MT, int T, int P, int NB, bool G128, bool DBG>
__global__ __launch_bounds__(64 * P, 2) void w4a4_ksplit_kernel(
    const uint8_t* __restrict__ A, const uint16_t* __restrict__ a_scale,
    const int16_t* __restrict__ a_zero, const uint8_t* __restrict__ W,
    const uint16_t* __restrict__ w_scale, const int32_t* __restrict__ w_colsum, int M, int N,
    int K, int log2g, uint16_t* __restrict__ Y, int64_t ldy, int32_t* __restrict__ acc_dbg) {
  constexpr int NT = 64 * P;
  extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];
  __shared__ __attribute__((aligned(16))) float sSW[16 * T];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kb = lane >> 4;
  // Workgroups of one channel tile (all its token tiles) follow each other on
  // one XCD, whose L2 then serves the weights to all but the first. Weights of
  // 64 or 128 MB put the eight XCDs' runs so far apart that they meet on the same
  // memory channels; with one token tile, which shares nothing, they are read front to
  // back instead (16 x 16384 x 16384 33.3 -> 29.0 us, 8 x 32768 x 8192 30.1 -> 25.5;
  // 32 MB 16 x 16384 x 4096 the same, 256 MB 1 x 16384 x 32768 48 -> 56).
  const int tiles_m = (M + 16 * MT - 1) / (16 * MT);
  const int nwg = (int)gridDim.x;
  int L = (int)blockIdx.x;
  const int64_t wbytes = (int64_t)N * (K >> 1);
  const bool camps = tiles_m == 1 && (wbytes == (64 << 20) || wbytes == (128 << 20));
  if ((nwg & 7) == 0 && !camps) L = (L & 7) * (nwg >> 3) + (L >> 3);
  const int m0 = (L % tiles_m) * (16 * MT), n0 = (L / tiles_m) * (16 * T);
  const int ldk = K >> 1;
  const int G = K >> log2g;
  const int GS = G | 1;  // odd row stride of the token parameters: no bank conflicts
  const int ns = K / KS_STEP;
  const int s_lo = (int)((int64_t)wave * ns / P), s_hi = (int)((int64_t)(wave + 1) * ns / P);
  uint32_t* const sAZ = dyn;                                              // [16 MT][GS]
  float* const sCS = reinterpret_cast<float*>(dyn + 16 * MT * GS);        // [G][16 T]

  // rows past N (weights) and past M (tokens) read as zero; the padding rows of
  // the last band hold zero codes
  const int wrows = min(16 * T, ((N - n0) + 15) & ~15), arows = min(16 * MT, M - m0);
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(W + (int64_t)n0 * ldk), 0, wrows * ldk, 0x00020000);
  const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(A + (int64_t)m0 * ldk), 0, arows * ldk, 0x00020000);
  const int a_off = r16 * ldk + 16 * kb, w_off = r16 * 64 + 16 * kb;

  v4i acc[MT][T];
  ks_f32x4 F[MT][T];
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int t = 0; t < T; ++t) {
      acc[a][t] = v4i{};
      F[a][t] = ks_f32x4{};
    }

  uint4 wa[NB][T], aa[NB][MT];
  auto load = [&](int s, uint4 (&w)[T], uint4 (&a)[MT]) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < T; ++t)
      w[t] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                           wrsrc, w_off + t * 16 * ldk, s * 1024, 0));
#pragma unroll
    for (int i = 0; i < MT; ++i)
      a[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                           arsrc, a_off + i * 16 * ldk, s * 64, 0));
  };
#pragma unroll
  for (int u = 0; u < NB; ++u)
    if (s_lo + u < s_hi) load(s_lo + u, wa[u], aa[u]);

  // group parameters of the tile
  for (int e = tid; e < arows * G; e += NT) {
    const int m = e / G, b = e - m * G;
    const int64_t src = (int64_t)m0 * G + e;
    sAZ[m * GS + b] = (uint32_t)a_scale[src] | ((uint32_t)(uint16_t)a_zero[src] << 16);
  }
  for (int e = tid; e < (16 * MT - arows) * GS; e += NT) sAZ[arows * GS + e] = 0;
  for (int e = tid; e < G * 16 * T; e += NT) {
    const int b = e / (16 * T), c = e % (16 * T);
    sCS[e] = n0 + c < N ? (float)w_colsum[(int64_t)b * N + n0 + c] : 0.0f;
  }
  for (int c = tid; c < 16 * T; c += NT)
    sSW[c] = n0 + c < N ? fp16_bits_to_f32(w_scale[n0 + c]) : 0.0f;
  __syncthreads();

  // Register i of (a, t) is channel n0 + 16 t + 4 kb + i, token m0 + 16 a + r16.
  auto fold = [&](int b) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < MT; ++a) {
      if constexpr (DBG) {
        const int m = m0 + 16 * a + r16;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int n = n0 + 16 * t + 4 * kb + i;
            if (m < M && n < N)
              atomicAdd(&acc_dbg[((int64_t)b * M + m) * N + n], acc[a][t][i] >> 4);
          }
      } else {
        const float s = fp16_bits_to_f32((uint16_t)sAZ[(16 * a + r16) * GS + b]) * 0.0625f;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) F[a][t][i] = __builtin_fmaf(s, (float)acc[a][t][i], F[a][t][i]);
      }
      if constexpr (!G128) {
#pragma unroll
        for (int t = 0; t < T; ++t) acc[a][t] = v4i{};
      }
    }
  };
  const int lgs = log2g - 7;
  const int gmask = (1 << lgs) - 1;  // steps per group - 1
  for (int s0 = s_lo; s0 < s_hi; s0 += NB) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int s = s0 + u;
      if (s >= s_hi) break;
      v4i alo[MT], ahi[MT];
#pragma unroll
      for (int a = 0; a < MT; ++a) {
        alo[a] = act_lo(aa[u][a]);
        ahi[a] = act_hi(aa[u][a]);
      }
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const v4i wlo = wgt_lo16(wa[u][t]), whi = wgt_hi16(wa[u][t]);
        // (g = 128: every step is a group and starts from zero)
#pragma unroll
        for (int a = 0; a < MT; ++a)
          acc[a][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wlo, alo[a], G128 ? v4i{} : acc[a][t], 0, 0, 0);
#pragma unroll
        for (int a = 0; a < MT; ++a)
          acc[a][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(whi, ahi[a], acc[a][t], 0, 0, 0);
      }
      if (s + NB < s_hi) load(s + NB, wa[u], aa[u]);
      // the step ends a group, or the wave's part of it
      if (G128 || (s & gmask) == gmask || s == s_hi - 1) fold(s >> lgs);
    }
  }
  if constexpr (DBG) return;

  // zero-point terms of this wave's part of the groups, four
  // at a time: F += sum_b colsum[b, n] (-s z)[m, b]
  const int b_lo = (int)((int64_t)wave * G / P), b_hi = (int)((int64_t)(wave + 1) * G / P);
  for (int b0 = b_lo; b0 < b_hi; b0 += 4) {
    const int b = b0 + kb;
    const bool in = b < b_hi;
    float sz[MT];
#pragma unroll
    for (int a = 0; a < MT; ++a) {
      const uint32_t p = in ? sAZ[(16 * a + r16) * GS + b] : 0u;
      sz[a] = -(fp16_bits_to_f32((uint16_t)p) * (float)(int16_t)(p >> 16));
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const float cs = in ? sCS[b * 16 * T + 16 * t + r16] : 0.0f;
#pragma unroll
      for (int a = 0; a < MT; ++a)
        F[a][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(cs, sz[a], F[a][t], 0, 0, 0);
    }
  }

  // ---- sum the P parts of K and store: wave w finishes tiles w, w + P, ... ----
  const bool vec = (ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(Y) & 7) == 0;
  if constexpr (P > 1) {
    __syncthreads();  // the parameters are done with
    ks_f32x4* const red = reinterpret_cast<ks_f32x4*>(dyn);  // [P][MT * T][64]
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int t = 0; t < T; ++t) red[(wave * (MT * T) + a * T + t) * 64 + lane] = F[a][t];
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < MT; ++a) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int q = a * T + t;
      if (q % P != wave) continue;
      const int m = m0 + 16 * a + r16, c = 16 * t + 4 * kb, n = n0 + c;
      if (m >= M) continue;
      ks_f32x4 f = F[a][t];
      if constexpr (P > 1) {
        const ks_f32x4* const red = reinterpret_cast<const ks_f32x4*>(dyn);
        f = red[q * 64 + lane];
#pragma unroll
        for (int w = 1; w < P; ++w) {
          const ks_f32x4 o = red[(w * (MT * T) + q) * 64 + lane];
#pragma unroll
          for (int i = 0; i < 4; ++i) f[i] += o[i];
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) f[i] *= sSW[c + i];
      uint16_t* const yp = Y + (int64_t)m * ldy + n;
      if (vec && n + 3 < N) {
        const ks_u32x2 v = {bf16x2_rne(f[0], f[1]), bf16x2_rne(f[2], f[3])};
        *reinterpret_cast<ks_u32x2*>(yp) = v;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < N) yp[i] = f32_to_bf16_rne(f[i]);
      }
    }
  }
}

// (a kernel, not a memset node: the call may be captured into a graph)
__global__ void ks_zero(int32_t* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0;
}

template <int MT, int T, int P, int NB>
hipError_t launch_ks(const uint8_t* a_codes, const uint16_t* a_scale, const int16_t* a_zero,
                     const uint8_t* w_codes, const uint16_t* w_scale, const int32_t* w_colsum,
                     int64_t M, int64_t N, int64_t K, int log2g, uint16_t* y, int64_t ldy,
                     int32_t* acc_debug, hipStream_t stream) {
  const int64_t tiles = ((M + 16 * MT - 1) / (16 * MT)) * ((N + 16 * T - 1) / (16 * T));
  const dim3 grid((unsigned)tiles), block(64 * P);
  const int64_t lds = ks_lds_bytes<MT, T, P>(K >> log2g);
#define OFFQ_KS_GO(G1, D)                                                                       \
  hipLaunchKernelGGL((w4a4_ksplit_kernel<MT, T, P, NB, G1, D>), grid, block, (size_t)lds, stream, \
                     a_codes, a_scale, a_zero, w_codes, w_scale, w_colsum, (int)M, (int)N, (int)K, \
                     log2g, y, ldy, acc_debug)
  // A debug request runs an accumulator-only pass (the waves' parts added
  // atomically into the zeroed buffer), then the regular kernel.
  if (acc_debug) {
    hipLaunchKernelGGL(ks_zero, dim3(1024), dim3(256), 0, stream, acc_debug, (K >> log2g) * M * N);
    if (log2g == 7) OFFQ_KS_GO(true, true); else OFFQ_KS_GO(false, true);
  }
  if (log2g == 7) OFFQ_KS_GO(true, false); else OFFQ_KS_GO(false, false);
#undef OFFQ_KS_GO
  return hipGetLastError();
}

// Tile and split, from sweeps over M = 17 ... 1000, N = 1000 ... 28672, K = 4096 ... 14336
// (us of the product alone, weights cycled beyond the 256 MB last-level cache; best of
// eighteen shapes). The kernel wants about 256 workgroups of
// eight waves or 384 of four; larger tiles reload less, more parts of K fill
// the chip where the output is small:
//   64 x 64 tiles by 4 waves from 384 tiles (64 x 28672 x 4096: 27.0, by 8 waves 32.0;
//     512 x 4096 x 4096: 19.4 / 24.7), 32 x 64 tiles where M <= 32; from 192 where a
//     wave of eight has one step of K or none (1280 x 1024 x 1024: 9.0, by 8 waves 13.1;
//     1280 x 1024 x 512: 7.7 / 11.7; 17 x 14336 x 256, 32 x 64 tiles, 4.8, 64 x 32 by 8
//     waves 8.1);
//   by 8 waves from 256 tiles (1000 x 1000 x 8192: 20.0, by 4 waves 24.5);
//   32 x 32 tiles by 16 waves up to 256 of them (64 x 4096 x 14336: 19.3; 64 x 32 by
//     8 waves 31), 32 x 16 by 8 waves up to 64 (17 x 1024 x 4096: 6.4 / 7.3);
//   64 x 32 tiles by 8 waves between (64 x 6144 x 4096: 12.5; 32 x 32 tiles 14.1).
// Up to 16 rows the weights' stream bounds it, and waves in flight (per byte) carry
// it; the activations are read again by every channel tile, which counts from about
// five rows. Sweeps over M = 1 ... 16, N = 64 ... 57344, K = 128 ... 32768:
//   one to four waves for a short K: more of them only add to the reduction (8 x 10240 x
//     128 2.8, by 16 waves 4.7; 5 x 10240 x 512 3.9 / 5.1; 1 x 14336 x 768 4.3, by 8 waves
//     5.0);
//   narrow outputs 16 channels by 8 waves, by 16 from K = 5120 (16 x 4096 x 4096: 5.2;
//     1 x 4096 x 14336: 9.2, by 8 waves 10.5; 1 x 1000 x 6144 4.6 / 5.1);
//   wider ones with M <= 4 the same by 8 waves (1 x 9216 x 12288 13.6, by 16 waves 15.3),
//     up to 8192 channels by 16 where that leaves whole batches (1 x 5120 x 6144 7.4 /
//     7.8), and by 4 from N = 16384 up to K = 6144 (1 x 28672 x 4096: 13.5, by 8 waves
//     15.0; 1 x 16384 x 8192 18.5 / 15.4);
//   with more rows 32 channels by 16 waves (16 x 14336 x 4096: 10.2; 16 channels by 8
//     waves 11.5), by 8 below K = 4096 and, from 6145 channels, from K = 6144 to 10240, where
//     16 have too few steps (16 x 8192 x 8192 10.2 / 10.9; 16 x 5120 x 8192 stays: 0.98 of
//     it); there 16 channels where 32 leave 320 to 416 workgroups (5 x 10240 x 1536 4.9,
//     32 channels 5.4; 16 x 16368 x 2048, 32 channels, 0.91 of it);
//   from N = 16384 by 8 waves (5 x 20480 x 8192 17.7, 64 channels by 8 20.5), by 4 at
//     K = 4096 (16 x 28672 x 4096: 16.6 / 17.4), 64 channels by 8 where rows and
//     channels are most (16 x 28672 x 8192: 24.4 / 25.9), and 16 from K = 10240 to 13312
//     (16 x 16384 x 12288 21.5 / 23.2; at 14336 33.1 / 31.4 for 18432 channels) and above
//     16384 except at its multiples, whose sixteenths are a power of two apart (16 x
//     20480 x 28672 64 / 66; 16 x 16384 x 16384 36.8, by 8 waves 33.2; below 16384
//     channels and up to 8 rows 16 channels by 8: 5 x 16368 x 16384 38.5 / 25.2).
struct KsShape { int mt, t, p; };
KsShape ks_shape(int64_t M, int64_t N, int64_t K) {
  if (M <= 16) {
    if (K <= 256) return {1, 1, 1};
    if (K < 1024) return {1, 1, N < 16384 ? 4 : 2};
    if (N < 5120) return {1, 1, K < 5120 ? 8 : 16};
    const bool middle = K > 6144 && K <= 10240;
    if (N >= 16384) {
      if (M <= 4) return {1, 1, K <= 6144 ? 4 : 8};
      if (K <= 1536) return {1, 1, 4};
      if (K > 3072 && K <= 4096) return {1, 2, 4};
      if (K > 4096 && K < 16384 && M > 8 && N >= 28672) return {1, 4, 8};
      return {1, 2, (K > 10240 && K < 13312) || (K > 16384 && K % 16384 != 0) ? 16 : 8};
    }
    if (M <= 4) return {1, 1, N > 8192 || K < 5120 || middle ? 8 : 16};
    if (K % 16384 == 0 && M <= 8 && N >= 10240) return {1, 1, 8};
    if (K < 4096 || (middle && N > 6144)) return {1, N >= 10240 && N < 13312 ? 1 : 2, 8};
    return {1, 2, 16};
  }
  auto tiles = [&](int mt, int t) { return ((M + 16 * mt - 1) / (16 * mt)) * ((N + 16 * t - 1) / (16 * t)); };
  const int four = K <= 1024 ? 192 : 384;
  if (M <= 32 && tiles(2, 4) >= four) return {2, 4, 4};
  if (tiles(4, 4) >= four) return {4, 4, 4};
  if (M > 32 && tiles(4, 4) >= 256) return {4, 4, 8};
  if (tiles(2, 2) <= 64) return {2, 1, 8};
  if (tiles(2, 2) <= 256) return {2, 2, 16};
  return {4, 2, 8};
}

}  // namespace

bool gemm_ksplit_supported(int64_t M, int64_t N, int64_t K, int log2g) {
  // whole steps of 128 k inside one group; 32-bit offsets within a tile; the
  // group parameters (or the partial tiles) in LDS
  if (log2g < 7 || K % KS_STEP || 64 * (K / 2) >= (int64_t(1) << 31)) return false;
  const KsShape c = ks_shape(M, N, K);
  const int64_t G = K >> log2g, rows = 16 * c.mt, cols = 16 * c.t;
  return (rows * (G | 1) + G * cols) * 4 <= 160 * 1024 - 1024;
}

int gemm_ksplit_form(int64_t M, int64_t N, int64_t K) {
  const KsShape c = ks_shape(M, N, K);
  return 10000 * c.mt + 100 * c.t + c.p;
}

hipError_t launch_w4a4_gemm_ksplit(const uint8_t* a_codes, const uint16_t* a_scale,
                                   const int16_t* a_zero, const uint8_t* w_codes,
                                   const uint16_t* w_scale, const int32_t* w_colsum, int64_t M,
                                   int64_t N, int64_t K, int log2g, uint16_t* y, int64_t ldy,
                                   int32_t* acc_debug, hipStream_t stream) {
#define OFFQ_KS(MT, T, P, NB)                                                                   \
  case 10000 * MT + 100 * T + P:                                                                \
    return launch_ks<MT, T, P, NB>(a_codes, a_scale, a_zero, w_codes, w_scale, w_colsum, M, N, K, \
                                   log2g, y, ldy, acc_debug, stream)
  switch (gemm_ksplit_form(M, N, K)) {
    OFFQ_KS(1, 1, 1, 1);
    OFFQ_KS(1, 1, 2, 4);
    OFFQ_KS(1, 1, 4, 4);
    OFFQ_KS(1, 1, 8, 4);
    OFFQ_KS(1, 1, 16, 2);
    OFFQ_KS(1, 2, 4, 4);
    OFFQ_KS(1, 2, 8, 2);
    OFFQ_KS(1, 2, 16, 2);
    OFFQ_KS(1, 4, 8, 2);
    OFFQ_KS(2, 1, 8, 4);
    OFFQ_KS(2, 2, 16, 2);
    OFFQ_KS(2, 4, 4, 2);
    OFFQ_KS(4, 2, 8, 1);
    OFFQ_KS(4, 4, 4, 1);
    OFFQ_KS(4, 4, 8, 1);
  }
#undef OFFQ_KS
  return hipErrorInvalidValue;
}

}  // namespace offq
