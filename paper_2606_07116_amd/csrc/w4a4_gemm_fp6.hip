// W4A4 GEMM on the 6-bit matrix format (gfx950,
// v_mfma_f32_32x32x64_f8f6f4 with e2m3 operands), one or several
// quantization groups per row.
//
//   acc_b[m,n] = sum_{k in group b} q_a[m,k] q_w[n,k]
//   Y[m,n]     = sw[n] * sum_b s[m,b] * (acc_b[m,n] - z[m,b] * colsum[b,n])
//
// Why this format: a 4-bit code c = 0..15 with two zero bits above it is the
// e2m3 value c / 8 (subnormals up to 7, then the first binade), so unsigned
// codes enter the matrix cores exactly, at twice the i8 rate, and the products
// are summed in fp32: multiples of 1/64, exact while a group's sum stays below
// 2^24 / 64, which 225 g does up to the largest group (8192). The accumulators
// need no conversion before the per-group fold.
//   * Sixteen nibbles become three words of 6-bit fields in eight VALU
//     operations (expand16; the field order is a permutation of k, the same
//     for both operands).
//   * Weight codes are signed: q + 8 goes in, and the excess 8 sum_k q_a comes
//     out again with the zero-point term, as one fp32 MFMA per group and tile
//     (k = 2: (asum, 8) and (z, colsum), integers in units of 1/64). acc - z colsum is
//     exact while all of it stays below 2^24; where z colsum is larger (|z| above
//     16384 at g = 128) the sum rounds at 2^-24 of that term, as the fp32 fold of exact
//     integers does (largest error beyond the bf16 rounding with z over all of int16 and
//     columns of -8, terms that cancel between groups: 78 units of acc, by that fold 72;
//     the mean is the same).
//
// What bounds it: per stage of 128 k a wave issues 135 (one group, 128 x 64) or 190
// (g = 128, 64 x 64; 286 for 128 x 64) VALU instructions beside its 12 to 24 matrix
// instructions, and LDS takes stores at 64 bytes a clock (it returns 128-bit reads at
// 229). An operand byte is expanded once per workgroup, on its way into LDS, and the
// tiles are as large as the registers allow. No unit is busy more than about half the time
// (one group, 4096 x 28672 x 4096: matrix cores 38 %, VALU 39 %, LDS 51 %; g = 128, 1777 x
// 10240 x 8192: 27, 40 and 34 %), and matrix cores and VALU together only 3 to 12 %: with
// two LDS buffers and one barrier per stage the waves go through the same phase at the
// same time, and a stage takes nearly the sum of its parts.
//   * 256 x 256 by eight waves of 128 x 64 (FM = 4): two operand bytes expanded per
//     256 products. At g = 128 the running sums take 128 registers and each
//     fragment row is folded right after the next row's reads and expansion were
//     issued. 4096 x 28672 x 4096: 400 -> 304 us with one group (3.16 POP/s),
//     673 -> 502 us at g = 128, against i8 tiles of 256 x 256 and 256 x 128.
//   * 128 x 128 by four waves of 64 x 64 (FM = 2), g = 128: two workgroups per CU,
//     where the larger tiles would not fill whole rounds of the 256 CUs:
//     1777 x 10240 x 8192 279 -> 218 us (256 x 256: 284).
// Stages go global memory -> registers -> one of two LDS buffers, one LDS-only
// barrier per stage; loads take whole 64-byte rows.
#include <type_traits>

#include "common.h"
#include "gemm_common.h"
#include "internal.h"

namespace offq {
namespace {

using namespace gemm;

typedef int f6_v8i __attribute__((ext_vector_type(8)));
typedef float f6_v16f __attribute__((ext_vector_type(16)));
typedef unsigned int f6_u32x4 __attribute__((ext_vector_type(4)));

// One operand of R rows in LDS: a row's 128 k of a stage are four chunks of 32
// (24 bytes each), the first 16 bytes of a chunk in plane X, the other 8 in
// plane Y; the pads put the four chunks' writes of a wave on different banks.
template <int R>
struct F6Oper {
  static constexpr int XC = R * 16 + 64, YC = R * 8 + 32;  // chunk strides
  static constexpr int Y = 4 * XC, BYTES = 4 * XC + 4 * YC;
};

// nibbles of d, e (in order) -> 16 fields of 6 bits, zero-extended
__device__ __forceinline__ void expand16(uint32_t d, uint32_t e, uint32_t* w) {
  const uint32_t x = __builtin_amdgcn_alignbit(e, d, 2), x1 = e >> 2;
  w[0] = (d & 0x0f00f00fu) | (x & 0xc03c03c0u);
  w[1] = (d & 0xf00f00f0u) | (x1 & 0x03c03c03u);
  w[2] = (e & 0x00f00f00u) | (x1 & 0x3c03c03cu);
}

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// FOLD: 0 one group per row, 1 every stage is a group (g = 128). FM: fragments of
// 32 token rows per wave; NWM x NWN waves.
template <int FM, int NWM, int NWN, int FOLD, bool DBG>
__global__ __launch_bounds__(64 * NWM * NWN, 2) void w4a4_gemm_fp6_kernel(
    const uint8_t* __restrict__ A, const uint16_t* __restrict__ a_scale,
    const int16_t* __restrict__ a_zero, const uint8_t* __restrict__ W,
    const uint16_t* __restrict__ w_scale, const int32_t* __restrict__ w_colsum, int M, int N,
    int K, int log2g, uint16_t* __restrict__ Y, int64_t ldy, int32_t* __restrict__ acc_dbg) {
  constexpr int WROWS = 32 * FM, BM = NWM * WROWS;
  constexpr int BN = 64 * NWN, THREADS = 64 * NWM * NWN;
  constexpr int RS = THREADS / 4, ASETS = BM / RS, WSETS = BN / RS;  // rows staged at a time
  constexpr int NSET = FM == 2 ? 2 : 1;  // stages in registers on their way to LDS
  using OA = F6Oper<BM>;
  using OW = F6Oper<BN>;
  constexpr int STAGE = OA::BYTES + OW::BYTES;
  __shared__ __attribute__((aligned(16))) char ring[2 * STAGE];
  __shared__ __attribute__((aligned(16))) float pT[2][3][BM];    // asum / 8, z, 64 s
  __shared__ __attribute__((aligned(16))) float pC[2][BN];  // -colsum / 64
  __shared__ __attribute__((aligned(16))) float sSW[BN];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, fr = lane & 31;
  const int wm = wave % NWM, wn = wave / NWM;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  // each XCD takes a run of tiles: groups of 1024 token rows, column by column
  int ti, tj;
  {
    const int nwg = (int)gridDim.x, bid = (int)blockIdx.x;
    const int q = nwg >> 3, r = nwg & 7, xcd = bid & 7;
    const int L = xcd * q + min(xcd, r) + (bid >> 3);
    constexpr int GM = 1024 / BM;
    const int per = GM * tiles_n, grp = L / per, first = grp * GM, gm = min(tiles_m - first, GM);
    const int o = L - grp * per;
    ti = first + o % gm;
    tj = o / gm;
  }
  const int tm = ti * BM, tn = tj * BN;
  const int ldk = K >> 1, nst = K >> 7, G = K >> log2g;

  // ---- staging: thread = (row, chunk) of each set of 64 rows, so that four
  // lanes read a row's 64 bytes. Rows past M or N read as zero.
  const int srow = tid >> 2, sch = tid & 3;
  const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(A + (int64_t)tm * ldk), 0, min(BM, M - tm) * ldk, 0x00020000);
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(W + (int64_t)tn * ldk), 0, min(BN, (N - tn + 15) & ~15) * ldk, 0x00020000);
  const int a_off = srow * ldk + sch * 16;
  const int w_off = (srow >> 4) * 16 * ldk + (srow & 15) * 64 + sch * 16;
  // group parameters: the first half of the threads a row's scale, the second its
  // zero-point; a column's sum twice over. They are wanted with the group's last
  // stage only (for the others the buffers are empty: no access, no branch).
  static_assert(THREADS == 2 * BM && BN <= THREADS, "one parameter per thread");
  const bool zp_wave = wave >= NWM * NWN / 2;
  const int prow = tid & (BM - 1), pcol = tid & (BN - 1);
  const int rbytes = min(BM, M - tm) * G * 2;
  const int cbytes = min(BN, N - tn) * 4;  // (columns past N read as zero)
  const void* const par0 = !zp_wave ? (const void*)(a_scale + (int64_t)tm * G)
                                  : (const void*)(a_zero + (int64_t)tm * G);

  struct Regs {
    uint4 a[ASETS], w[WSETS];
    uint32_t p0;
    int pc;
  };
  auto gload = [&](int st, Regs& r) __attribute__((always_inline)) {
    const int s = min(st, nst - 1);  // (past the end: loaded again, never used)
#pragma unroll
    for (int i = 0; i < ASETS; ++i)
      r.a[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(arsrc, a_off + i * RS * ldk, s * 64, 0));
#pragma unroll
    for (int i = 0; i < WSETS; ++i)
      r.w[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, w_off + i * RS * ldk, s * 1024, 0));
    const int b = FOLD == 1 ? s : 0;
    const bool last = FOLD == 1 || s == nst - 1;
    const __amdgpu_buffer_rsrc_t srsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)par0, 0, last ? rbytes : 0, 0x00020000);
    r.p0 = __builtin_amdgcn_raw_buffer_load_b16(srsrc, prow * G * 2, b * 2, 0);
    const __amdgpu_buffer_rsrc_t crsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(w_colsum + (int64_t)b * N + tn), 0, last ? cbytes : 0, 0x00020000);
    r.pc = (int)__builtin_amdgcn_raw_buffer_load_b32(crsrc, pcol * 4, 0, 0);
  };
  char* const sax = ring + sch * OA::XC + srow * 16;
  char* const say = ring + OA::Y + sch * OA::YC + srow * 8;
  char* const swx = ring + OA::BYTES + sch * OW::XC + srow * 16;
  char* const swy = ring + OA::BYTES + OW::Y + sch * OW::YC + srow * 8;
  auto put = [&](char* x, char* y, int off, int i, const uint4& c) __attribute__((always_inline)) {
    uint32_t w[6];
    expand16(c.x, c.y, w);
    expand16(c.z, c.w, w + 3);
    *reinterpret_cast<uint4*>(x + off + i * RS * 16) = make_uint4(w[0], w[1], w[2], w[3]);
    *reinterpret_cast<uint2*>(y + off + i * RS * 8) = make_uint2(w[4], w[5]);
  };
  int asum[ASETS] = {};  // sums of the thread's codes in the current group
  auto put_a = [&](int buf, int i, const uint4& c) __attribute__((always_inline)) {
    put(sax, say, buf * STAGE, i, c);
    int t = FOLD == 1 ? 0 : asum[i];
    t = (int)__builtin_amdgcn_udot8(c.x, 0x11111111u, t, false);
    t = (int)__builtin_amdgcn_udot8(c.y, 0x11111111u, t, false);
    t = (int)__builtin_amdgcn_udot8(c.z, 0x11111111u, t, false);
    t = (int)__builtin_amdgcn_udot8(c.w, 0x11111111u, t, false);
    asum[i] = t;
  };
  auto put_sums = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < ASETS; ++i) {
      // the row's four chunks (quad_perm [1, 0, 3, 2], then [2, 3, 0, 1])
      int t = asum[i];
      t += __builtin_amdgcn_update_dpp(0, t, 0xB1, 0xF, 0xF, true);
      t += __builtin_amdgcn_update_dpp(0, t, 0x4E, 0xF, 0xF, true);
      pT[buf][0][srow + RS * i] = 0.125f * (float)t;
    }
  };
  auto put_w = [&](int buf, int i, const uint4& c) __attribute__((always_inline)) {
    const uint32_t X = 0x88888888u;
    put(swx, swy, buf * STAGE, i, make_uint4(c.x ^ X, c.y ^ X, c.z ^ X, c.w ^ X));
  };
  auto put_p = [&](int buf, const Regs& r) __attribute__((always_inline)) {
    const float sc = 64.0f * fp16_bits_to_f32((uint16_t)r.p0), z = DBG ? 0.0f : (float)(int16_t)r.p0;
    pT[buf][zp_wave ? 1 : 2][prow] = zp_wave ? z : sc;
    pC[buf][pcol] = -0.015625f * (float)r.pc;
  };
  auto lstore = [&](int buf, const Regs& r) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < ASETS; ++i) put_a(buf, i, r.a[i]);
#pragma unroll
    for (int i = 0; i < WSETS; ++i) put_w(buf, i, r.w[i]);
    put_sums(buf);
    put_p(buf, r);
  };

  // ---- fragments: lane row fr, half h; fragment f is 32 rows further; k-step j
  // takes chunk 2 j + h
  struct Frag {
    uint4 x[2];
    uint2 y[2];
  };
  const char* const rax = ring + h * OA::XC + (wm * WROWS + fr) * 16;
  const char* const ray = ring + OA::Y + h * OA::YC + (wm * WROWS + fr) * 8;
  const char* const rwx = ring + OA::BYTES + h * OW::XC + (wn * 64 + fr) * 16;
  const char* const rwy = ring + OA::BYTES + OW::Y + h * OW::YC + (wn * 64 + fr) * 8;
  auto fread = [&](const char* x, const char* y, int xs, int ys, int off, int f, Frag& v)
      __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      v.x[j] = *reinterpret_cast<const uint4*>(x + off + j * 2 * xs + f * 512);
      v.y[j] = *reinterpret_cast<const uint2*>(y + off + j * 2 * ys + f * 256);
    }
  };
  auto op = [](const Frag& v, int j) __attribute__((always_inline)) {
    return f6_v8i{(int)v.x[j].x, (int)v.x[j].y, (int)v.x[j].z, (int)v.x[j].w, (int)v.y[j].x, (int)v.y[j].y, 0, 0};
  };

  f6_v16f acc[FM][2], F[FM][2];
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if constexpr (FOLD != 1) acc[a][b] = f6_v16f{};
      if constexpr (FOLD != 0) F[a][b] = f6_v16f{};
    }

  // acc (in units of 1/64) minus the weights' excess and the zero-point term
  auto correct = [&](int buf, int fm, int fn, f6_v16f c) __attribute__((always_inline)) {
    const float tk = pT[buf][h][wm * WROWS + fm * 32 + fr];
    const float cs = pC[buf][wn * 64 + fn * 32 + fr];
    return __builtin_amdgcn_mfma_f32_32x32x2f32(h ? cs : -1.0f, tk, c, 0, 0, 0);
  };
  auto dump = [&](int b, int fm, int fn) __attribute__((always_inline)) {  // debug: acc of group b
    const int row = tm + wm * WROWS + fm * 32 + fr;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int col = tn + wn * 64 + fn * 32 + 8 * (i >> 2) + 4 * h + (i & 3);
      if (row < M && col < N) acc_dbg[((int64_t)b * M + row) * N + col] = (int)(64.0f * acc[fm][fn][i]);
    }
  };
#define F6_MMA(w, a, c) __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w, a, c, 2, 2, 0, 0, 0, 0)

  auto scale64 = [&](int buf, int fm) __attribute__((always_inline)) {
    return pT[buf][2][wm * WROWS + fm * 32 + fr];
  };
  auto fold = [&](int st, int buf, int fm) __attribute__((always_inline)) {
    const float s = scale64(buf, fm);
#pragma unroll
    for (int fn = 0; fn < 2; ++fn) {
      if constexpr (DBG) dump(st, fm, fn);
#pragma unroll
      for (int i = 0; i < 16; ++i) F[fm][fn][i] = __builtin_fmaf(s, acc[fm][fn][i], F[fm][fn][i]);
    }
  };

  // One stage: its fragments are requested first and the next stage's operands
  // expanded and stored between the products, so that LDS latency, expansion and
  // the stores' drain run beside them. FM = 2 folds a fragment row beside the next
  // one's products; FM = 4 has no registers for a second row of accumulators at
  // g = 128 and folds a row after its share of the expansion instead (fold first,
  // 4096 x 28672 x 4096: 515 us; this order 503; the next row's products first, with
  // spills: 549).
  auto stage = [&](int st, auto BUFC, Regs& nxt) __attribute__((always_inline)) {
    constexpr int buf = decltype(BUFC)::value;
    constexpr int off = buf * STAGE;
    Frag wf[2], af;
    fread(rwx, rwy, OW::XC, OW::YC, off, 0, wf[0]);
    fread(rwx, rwy, OW::XC, OW::YC, off, 1, wf[1]);
    auto puts = [&](int fm) __attribute__((always_inline)) {
#pragma unroll
      for (int q = fm * (ASETS + WSETS) / FM; q < (fm + 1) * (ASETS + WSETS) / FM; ++q) {
        if (q < ASETS) put_a(buf ^ 1, q < ASETS ? q : 0, nxt.a[q < ASETS ? q : 0]);
        else put_w(buf ^ 1, q - ASETS, nxt.w[q >= ASETS ? q - ASETS : 0]);
      }
      if (fm == FM - 1) {
        if (FOLD == 1 || st + 1 == nst - 1) {  // (one group: its last stage carries them)
          put_sums(buf ^ 1);
          put_p(buf ^ 1, nxt);
        }
        gload(st + 1 + NSET, nxt);
      }
    };
    auto products = [&](int fm) __attribute__((always_inline)) {
      if constexpr (FOLD == 1) {
        acc[fm][0] = correct(buf, fm, 0, f6_v16f{});
        acc[fm][1] = correct(buf, fm, 1, f6_v16f{});
      }
      acc[fm][0] = F6_MMA(op(wf[0], 0), op(af, 0), acc[fm][0]);
      acc[fm][1] = F6_MMA(op(wf[1], 0), op(af, 0), acc[fm][1]);
      acc[fm][0] = F6_MMA(op(wf[0], 1), op(af, 1), acc[fm][0]);
      acc[fm][1] = F6_MMA(op(wf[1], 1), op(af, 1), acc[fm][1]);
    };
    if constexpr (FM == 4 && FOLD == 1) {
      fread(rax, ray, OA::XC, OA::YC, off, 0, af);
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) {
        products(fm);
        __builtin_amdgcn_sched_barrier(0);
        if (fm + 1 < FM) fread(rax, ray, OA::XC, OA::YC, off, fm + 1, af);
        puts(fm);
        __builtin_amdgcn_sched_barrier(0);
        fold(st, buf, fm);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) {
        fread(rax, ray, OA::XC, OA::YC, off, fm, af);
        puts(fm);
        __builtin_amdgcn_sched_barrier(0);
        products(fm);
        if (FOLD == 1 && fm > 0) fold(st, buf, fm - 1);
      }
      if constexpr (FOLD == 1) fold(st, buf, FM - 1);
    }
    lds_barrier();
  };

  // stage 0 into LDS, the next NSET in registers (stage s in r[s mod NSET])
  Regs r[NSET];
  gload(0, r[0]);
  if constexpr (NSET == 2) gload(1, r[1]);
  if (tid < BN) sSW[tid] = tn + tid < N ? fp16_bits_to_f32(w_scale[tn + tid]) : 0.0f;
  lstore(0, r[0]);
  gload(NSET, r[0]);
  lds_barrier();
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  int st = 0;
  for (; st + 2 <= nst; st += 2) {
    stage(st, B0{}, r[NSET - 1]);
    stage(st + 1, B1{}, r[0]);
  }
  if (st < nst) stage(st, B0{}, r[NSET - 1]);
  if constexpr (DBG && FOLD != 0) return;

  // ---- Y = sw F, one fragment row at a time through a private LDS area per
  // wave (rows of 16 8-byte units, unit u of row r at u ^ (r & 15)) for 16-byte
  // stores
  static_assert(NWM * NWN * 32 * 128 <= 2 * STAGE, "the waves' areas fit in the ring");
  uint32_t* const ot = reinterpret_cast<uint32_t*>(ring) + wave * (32 * 32);
  const bool vec = (tm + BM <= M) && (tn + BN <= N) && (ldy % 8 == 0) &&
                   ((reinterpret_cast<uintptr_t>(Y) & 15) == 0);
  const int lastbuf = (nst - 1) & 1;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
#pragma unroll
    for (int fn = 0; fn < 2; ++fn) {
      if constexpr (FOLD == 0) {
        acc[fm][fn] = correct(lastbuf, fm, fn, acc[fm][fn]);
        if constexpr (DBG) dump(0, fm, fn);
        const float s = scale64(lastbuf, fm);
#pragma unroll
        for (int i = 0; i < 16; ++i) F[fm][fn][i] = s * acc[fm][fn][i];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 sw = *reinterpret_cast<const float4*>(&sSW[wn * 64 + fn * 32 + q * 8 + h * 4]);
        const f6_v16f& f = F[fm][fn];
        const int u = fn * 8 + q * 2 + h;
        *reinterpret_cast<uint2*>(ot + fr * 32 + ((u ^ (fr & 15)) * 2)) =
            make_uint2(bf16x2_rne(sw.x * f[q * 4 + 0], sw.y * f[q * 4 + 1]),
                       bf16x2_rne(sw.z * f[q * 4 + 2], sw.w * f[q * 4 + 3]));
      }
    }
    if constexpr (DBG) continue;
    wave_lds_fence();
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int r = 8 * p + (lane >> 3);
      const int k = lane & 7;
      const int pu = (2 * k) ^ (r & 15);
      uint4 d = *reinterpret_cast<const uint4*>(ot + r * 32 + (pu & ~1) * 2);
      if (pu & 1) d = make_uint4(d.z, d.w, d.x, d.y);
      const int row = tm + wm * WROWS + fm * 32 + r;
      const int col = tn + wn * 64 + 8 * k;
      if (vec) {
        const f6_u32x4 dv = {d.x, d.y, d.z, d.w};
        __builtin_nontemporal_store(dv, reinterpret_cast<f6_u32x4*>(Y + (int64_t)row * ldy + col));
      } else if (row < M) {
        const uint32_t w4[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (col + e < N) Y[(int64_t)row * ldy + col + e] = (uint16_t)(w4[e >> 1] >> (16 * (e & 1)));
      }
    }
    wave_lds_fence();
  }
#undef F6_MMA
}

template <int FM, int NWM, int NWN, int FOLD>
hipError_t launch_f6(const uint8_t* a_codes, const uint16_t* a_scale, const int16_t* a_zero,
                     const uint8_t* w_codes, const uint16_t* w_scale, const int32_t* w_colsum,
                     int64_t M, int64_t N, int64_t K, int log2g, uint16_t* y, int64_t ldy,
                     int32_t* acc_debug, hipStream_t stream) {
  constexpr int BM = 32 * FM * NWM, BN = 64 * NWN;
  const dim3 grid((unsigned)(((M + BM - 1) / BM) * ((N + BN - 1) / BN))), block(64 * NWM * NWN);
#define OFFQ_F6(D)                                                                            \
  hipLaunchKernelGGL((w4a4_gemm_fp6_kernel<FM, NWM, NWN, FOLD, D>), grid, block, 0, stream,   \
                     a_codes, a_scale, a_zero, w_codes, w_scale, w_colsum, (int)M, (int)N,    \
                     (int)K, log2g, y, ldy, acc_debug)
  // A debug request runs an accumulator-only pass, then the regular kernel.
  if (acc_debug) OFFQ_F6(true);
  OFFQ_F6(false);
#undef OFFQ_F6
  return hipGetLastError();
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Large tiles at g = 128? A stage of a full round of the 256 CUs takes 2.25 us with
// one 256 x 256 tile per CU and 1.36 us with two of 128 x 128; a last round of at
// most one small tile per CU 0.92 us (4096 x 28672 x 4096, 2048 x 4096 x 4096,
// 512 x 6144 x 4096).
bool f6_large(int64_t M, int64_t N) {
  const int64_t t256 = ceil_div(M, 256) * ceil_div(N, 256), t128 = ceil_div(M, 128) * ceil_div(N, 128);
  const int64_t rest = t128 % 512;
  return 225 * ceil_div(t256, 256) < 136 * (t128 / 512) + (rest == 0 ? 0 : rest <= 256 ? 92 : 136);
}

}  // namespace

bool gemm_fp6_one_group(int64_t M, int64_t N, int64_t K) {
  // One group per row: a round of 256 x 256 tiles takes 1.36 us a stage, one of the
  // i8 kernel's 256 x 128 tiles 1.1 us (4096 x 28672 x 4096 and 2048 x 4096 x 4096).
  // With two stages they are the smaller part, and the i8 kernel is ahead (2500 x 8192
  // x 256 32.5, here 34.6; 2500 x 8192 x 512 37.0 / 37.8).
  const int64_t f6 = ceil_div(ceil_div(M, 256) * ceil_div(N, 256), 256);
  const int64_t i8 = ceil_div(ceil_div(M, 256) * ceil_div(N, 128), 256);
  return K > 256 && 5 * f6 < 4 * i8;
}

int gemm_fp6_form(int64_t M, int64_t N, int log2g) {
  return log2g != 7 ? 0 : f6_large(M, N) ? 1 : 2;
}

hipError_t launch_w4a4_gemm_fp6(const uint8_t* a_codes, const uint16_t* a_scale,
                                const int16_t* a_zero, const uint8_t* w_codes,
                                const uint16_t* w_scale, const int32_t* w_colsum, int64_t M,
                                int64_t N, int64_t K, int log2g, uint16_t* y, int64_t ldy,
                                int32_t* acc_debug, hipStream_t stream) {
#define OFFQ_F6_GO(FM, NWM, NWN, FOLD)                                                       \
  return launch_f6<FM, NWM, NWN, FOLD>(a_codes, a_scale, a_zero, w_codes, w_scale, w_colsum, \
                                       M, N, K, log2g, y, ldy, acc_debug, stream)
  switch (gemm_fp6_form(M, N, log2g)) {
    case 0: OFFQ_F6_GO(4, 2, 4, 0);
    case 1: OFFQ_F6_GO(4, 2, 4, 1);
    default: OFFQ_F6_GO(2, 2, 2, 1);
  }
#undef OFFQ_F6_GO
}

}  // namespace offq
