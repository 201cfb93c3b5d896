// The ASP GEMM for a few hundred tokens (more than kSmallM, too few 128 x 128
// tiles to fill the chip): the arithmetic of the large-tile kernel (exact
// integer group partials on v_mfma_scale_f32_32x32x64_f8f6f4, scale products
// on the bf16 matrix cores, one float32 FMA per output and group) in small
// tiles whose K is split over the workgroup's waves:
//
//   * a workgroup of MW waves (eight, or four with two workgroups on a CU)
//     owns 32 TB tokens x 64 output channels; wave w takes the w-th contiguous
//     range of the 64-channel spans and all of the tile, so a tile keeps its
//     operand reuse (TB + 2 fragment reads for 2 TB integer blocks) while its
//     latency is divided by MW;
//   * each wave copies its own operands into its own part of LDS
//     (buffer_load ... lds, stages of four spans: one cache line of every row,
//     eight lanes per line) and waits only for its own copies: the main loop
//     has no barrier.  A stage is read into registers at once and its buffer
//     requested again before the stage is multiplied;
//   * the waves' partial tiles are summed in LDS in wave order
//     (deterministic); each wave finishes 32 TB / MW result registers (branch,
//     bias, rounding, 8- or 16-byte stores).
//
// What bounds it (M = 415, K = 14336, N = 3072, 64 x 64 tiles: 35.7 us, the
// large tiles 75.7 us on 96 of 256 CUs): 24 us with no multiplication at all
// (the copies run at about 85 B/ns per CU), 28.6 us with no copies.  Measured
// and not kept: stages of two spans in two buffers (half lines: 36.3 us, 32 x
// 64 tiles 44.5 us), a ring shared by the waves with a barrier per stage and
// one span per wave and stage (38.7 us), 64 x 64 tiles by eight waves (42 us).
#include "qwam_device.h"
#include "qwam_internal.h"
#include "qwam_mfma.h"

namespace qwam {

namespace {

constexpr int KC = 4;              // spans per stage: one 128-byte line of every packed row
constexpr int ROWB = KC * 32;      // bytes of one packed row per stage

template <int GS, int TB, int WB>
struct MidShape {
  static constexpr int NS = kGroup / GS;                        // scale groups per span
  static constexpr int GPS = KC * NS;                           // scale groups per stage
  static constexpr int TM = 32 * TB, TN = 32 * WB;
  static constexpr int STAGE = (TM + TN) * (ROWB + GPS * 4);    // codes and scales, per wave
};

// 16-byte chunk slot permutation of a 128-byte row: 16 consecutive rows reading
// the same chunk hit 16 different 16-byte columns of the banks
__device__ __forceinline__ int mid_swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

}  // namespace

template <int RANK, int GS, int TB, int WB, int MW>
__global__ __launch_bounds__(64 * MW, 8 / MW) void asp_gemm_mid_kernel(
    const uint8_t* __restrict__ xq, const float* __restrict__ xs, const uint16_t* __restrict__ t,
    const uint8_t* __restrict__ wq, const uint32_t* __restrict__ wsp, const uint16_t* __restrict__ L2t,
    const uint16_t* __restrict__ bias, uint16_t* __restrict__ y, int M, int N, int K) {
  using S = MidShape<GS, TB, WB>;
  constexpr int NS = S::NS, GPS = S::GPS, TM = S::TM, TN = S::TN;
  static_assert(WB == 2 && (TB == 1 || TB == 2), "two weight blocks, one or two token blocks");
  static_assert(TB * WB * 16 * 256 <= S::STAGE, "a wave's partial tile fits in its stage buffer");
  __shared__ __attribute__((aligned(16))) uint8_t st0[MW][S::STAGE];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int G = K / kGroup;
  const int GSC = K / GS;
  const int KB = K / 2;

  // XCD-major (hardware places workgroup b on XCD b % 8): each XCD takes a
  // contiguous range of tiles, token blocks fastest, so it reads its own part
  // of the weights once and the activations of every token block
  const int tiles_m = (M + TM - 1) / TM;
  const int total = static_cast<int>(gridDim.x);
  const int per = total / 8, rem = total % 8;
  const int xcd = static_cast<int>(blockIdx.x) % 8, idx = static_cast<int>(blockIdx.x) / 8;
  const int logical = (xcd < rem) ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
  const int m0 = (logical % tiles_m) * TM, n0 = (logical / tiles_m) * TN;

  // this wave's spans [g_lo, g_hi), in whole stages except for the last range
  const int gpw = ((G + MW - 1) / MW + KC - 1) / KC * KC;
  const int g_lo = min(G, wave * gpw), g_hi = min(G, g_lo + gpw);
  const int ns = (g_hi - g_lo + KC - 1) / KC;

  const int frow = lane & 31;
  const int fhalf = lane >> 5;

  // rows / columns past M / N read as zero
  const buf_rsrc a_rsrc = make_rsrc(xq + static_cast<int64_t>(m0) * KB, static_cast<uint32_t>(min(TM, M - m0)) * KB);
  const buf_rsrc b_rsrc = make_rsrc(wq + static_cast<int64_t>(n0) * KB, static_cast<uint32_t>(min(TN, N - n0)) * KB);
  const buf_rsrc xs_rsrc = make_rsrc(xs, static_cast<uint32_t>(GSC) * M * 4u);
  const buf_rsrc ws_rsrc = make_rsrc(wsp, static_cast<uint32_t>(GSC) * N * 4u);
  // copy i of a tile: rows 8 i + lane/8, slot lane%8 (chunk (lane%8) ^ swz(row))
  const int crow = lane >> 3;
  const uint32_t c_off[2] = {static_cast<uint32_t>(crow * KB + (((lane & 7) ^ mid_swz(crow)) * 16)),
                             static_cast<uint32_t>((crow + 8) * KB + (((lane & 7) ^ mid_swz(crow + 8)) * 16))};
  // scale copies: 64 consecutive rows of one group, or 32 rows of two
  const uint32_t sx_off = TB == 2 ? static_cast<uint32_t>(m0 + lane) * 4u
                                  : (static_cast<uint32_t>(fhalf) * M + static_cast<uint32_t>(m0 + frow)) * 4u;
  const uint32_t sw_off = static_cast<uint32_t>(n0 + lane) * 4u;

  // a wave's stage: tokens' codes [TM][64] | weights' codes [TN][64] | token scales [GPS][TM] | weight pieces [GPS][TN]
  constexpr int OFF_B = TM * ROWB, OFF_SX = OFF_B + TN * ROWB, OFF_SW = OFF_SX + GPS * TM * 4;
  auto issue = [&](int s, uint8_t* st) __attribute__((always_inline)) {
    const int g = g_lo + s * KC;
    const uint32_t ko[2] = {c_off[0] + static_cast<uint32_t>(g) * 32u, c_off[1] + static_cast<uint32_t>(g) * 32u};
#pragma unroll
    for (int i = 0; i < TM / 8; ++i)
      buf_load16_lds(a_rsrc, ko[i & 1] + static_cast<uint32_t>(16 * (i >> 1)) * KB, st + i * 1024);
#pragma unroll
    for (int i = 0; i < TN / 8; ++i)
      buf_load16_lds(b_rsrc, ko[i & 1] + static_cast<uint32_t>(16 * (i >> 1)) * KB, st + OFF_B + i * 1024);
    const uint32_t gs = static_cast<uint32_t>(NS * g);
    constexpr int XG = 2 / TB;                   // scale groups per copy of the token scales
#pragma unroll
    for (int i = 0; i < GPS / XG; ++i)
      buf_load4_lds(xs_rsrc, sx_off + (gs + XG * i) * static_cast<uint32_t>(M) * 4u, st + OFF_SX + i * 256);
#pragma unroll
    for (int i = 0; i < GPS; ++i)
      buf_load4_lds(ws_rsrc, sw_off + (gs + i) * static_cast<uint32_t>(N) * 4u, st + OFF_SW + i * 256);
  };

  struct GroupData {
    uint4 a[WB], b[TB];                       // packed codes: weights (A operand), tokens (B operand)
    uint32_t sw[TB == 2 ? WB : 1][NS];        // weight-scale pieces (A operand of the scale products)
    float sx[NS];                             // token scale (B operand)
  };
  const int fslot = fhalf ^ mid_swz(frow);
  auto load_group = [&](const uint8_t* st, int q) __attribute__((always_inline)) {
    GroupData d;
    const int c = ((2 * q) ^ fslot) * 16;
#pragma unroll
    for (int i = 0; i < WB; ++i) d.a[i] = *reinterpret_cast<const uint4*>(st + OFF_B + (32 * i + frow) * ROWB + c);
#pragma unroll
    for (int j = 0; j < TB; ++j) d.b[j] = *reinterpret_cast<const uint4*>(st + (32 * j + frow) * ROWB + c);
#pragma unroll
    for (int h = 0; h < NS; ++h) {
      const float* sx = reinterpret_cast<const float*>(st + OFF_SX) + (NS * q + h) * TM;
      const uint32_t* sw = reinterpret_cast<const uint32_t*>(st + OFF_SW) + (NS * q + h) * TN;
      // two token blocks: lane half b takes token block b, and both halves the
      // weight block of the product; one token block: both halves its tokens,
      // lane half b weight block b
      if constexpr (TB == 2) {
        d.sx[h] = sx[lane];
#pragma unroll
        for (int i = 0; i < WB; ++i) d.sw[i][h] = sw[32 * i + frow];
      } else {
        d.sx[h] = sx[frow];
        d.sw[0][h] = sw[lane];
      }
    }
    return d;
  };

  // result layout of block (i, j) (i: weight block, j: token block): lane l
  // holds token l%32 and columns 8*(v/4) + 4*(l/32) + v%4, v = 0..15
  v16f acc[WB][TB];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = v16f{};
  auto update = [&](v16f& a, const v16f& p, const v32f& sc, int blk) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 16; ++v) a[v] = __builtin_fmaf(p[v], sc[16 * blk + v], a[v]);
  };
  auto group = [&](const GroupData& d) __attribute__((always_inline)) {
    v8i af[WB], bf[TB];
#pragma unroll
    for (int i = 0; i < WB; ++i) af[i] = codes_to_fp6(d.a[i]);
#pragma unroll
    for (int j = 0; j < TB; ++j) bf[j] = codes_to_fp6(d.b[j]);
#pragma unroll
    for (int h = 0; h < NS; ++h) {
      // group 32: the other lane half's channels are masked by scales of 2^-127
      int e = kE8M0Code;
      if constexpr (GS == 32) e = fhalf == h ? kE8M0Code : 0;
      if constexpr (TB == 2) {
#pragma unroll
        for (int i = 0; i < WB; ++i) {
          const v32f sc = scale_outer(d.sw[i][h], d.sx[h]);
          const v16f p0 = fp6_partial(af[i], bf[0], e, e);
          const v16f p1 = fp6_partial(af[i], bf[1], e, e);
          update(acc[i][0], p0, sc, 0);
          update(acc[i][1], p1, sc, 1);
        }
      } else {
        const v32f sc = scale_outer(d.sw[0][h], d.sx[h]);
        const v16f p0 = fp6_partial(af[0], bf[0], e, e);
        const v16f p1 = fp6_partial(af[1], bf[0], e, e);
        update(acc[0][0], p0, sc, 0);
        update(acc[1][0], p1, sc, 1);
      }
    }
  };

  uint8_t* const my0 = st0[wave];
  // stage s: wait for its copies, read all of it into registers, request stage
  // s + 1 into the same buffer, multiply
  if (ns > 0) issue(0, my0);
  for (int s = 0; s < ns; ++s) {
    wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    GroupData d[KC];
#pragma unroll
    for (int q = 0; q < KC; ++q) d[q] = load_group(my0, q);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (s + 1 < ns) issue(s + 1, my0);
#pragma unroll
    for (int q = 0; q < KC; ++q)
      if (q == 0 || g_lo + s * KC + q < g_hi) group(d[q]);
  }

  // the epilogue's operands of this wave's block, requested before the reduction
  constexpr int NREG = TB * WB * 16 / MW;       // result registers finished per wave
  constexpr int WPB = 16 / NREG;                // waves per block
  constexpr int KSTEPS = RANK / 16;
  const int blk = wave / WPB, v0 = (wave % WPB) * NREG;
  const int bi = blk / TB, bj = blk % TB;       // weight block, token block
  const int mt = m0 + 32 * bj + frow;
  const buf_rsrc t_rsrc = make_rsrc(t + static_cast<int64_t>(m0) * RANK, static_cast<uint32_t>(min(TM, M - m0)) * RANK * 2u);
  const buf_rsrc l_rsrc = make_rsrc(L2t + static_cast<int64_t>(n0) * RANK, static_cast<uint32_t>(min(TN, N - n0)) * RANK * 2u);
  uint4 tv[KSTEPS], lv[KSTEPS];
#pragma unroll
  for (int k = 0; k < KSTEPS; ++k) {
    tv[k] = buf_load16(t_rsrc, static_cast<uint32_t>((32 * bj + frow) * RANK + k * 16 + fhalf * 8) * 2u);
    lv[k] = buf_load16(l_rsrc, static_cast<uint32_t>((32 * bi + frow) * RANK + k * 16 + fhalf * 8) * 2u);
  }

  // partial tiles -> the waves' own stage buffers (all copies have landed):
  // registers r = 16 block + v
  auto part = [&](int w, int r) __attribute__((always_inline)) {
    return reinterpret_cast<float*>(st0[w]) + r * 64 + lane;
  };
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) *part(wave, (i * TB + j) * 16 + v) = acc[i][j][v];
  __syncthreads();
  float c2[NREG];
#pragma unroll
  for (int e = 0; e < NREG; ++e) c2[e] = 0.0f;
#pragma unroll
  for (int w = 0; w < MW; ++w)
#pragma unroll
    for (int e = 0; e < NREG; ++e) c2[e] += *part(w, blk * 16 + v0 + e);
  // branch t . L2 on the matrix cores (the block's other registers are not used)
  v16f c;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    c[v] = 0.0f;
#pragma unroll
    for (int u = 0; u < WPB; ++u)
      if (v / NREG == u && wave % WPB == u) c[v] = c2[v % NREG];
  }
#pragma unroll
  for (int k = 0; k < KSTEPS; ++k)
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, lv[k]), __builtin_bit_cast(v8bf, tv[k]), c, 0,
                                                0, 0);
  float out[NREG];
#pragma unroll
  for (int e = 0; e < NREG; ++e) {
    out[e] = c[e];
#pragma unroll
    for (int u = 1; u < WPB; ++u)
      if (wave % WPB == u) out[e] = c[u * NREG + e];
  }
  // bias of the four columns of each register quad, then bf16
  const buf_rsrc bias_rsrc = make_rsrc(bias, bias != nullptr ? static_cast<uint32_t>(N) * 2u : 0u);
  const int n_blk = n0 + 32 * bi;
  constexpr int NQ = NREG / 4;
  uint32_t w2[NQ][2];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int n = n_blk + 8 * (v0 / 4 + q) + 4 * fhalf;
    const uint2 b = buf_load8(bias_rsrc, static_cast<uint32_t>(n) * 2u);
    w2[q][0] = bf16_pair(out[4 * q] + bf16_to_f32(b.x & 0xFFFFu), out[4 * q + 1] + bf16_to_f32(b.x >> 16));
    w2[q][1] = bf16_pair(out[4 * q + 2] + bf16_to_f32(b.y & 0xFFFFu), out[4 * q + 3] + bf16_to_f32(b.y >> 16));
  }
  if constexpr (NQ >= 2) {
    // per pair of quads, the upper half-wave's words of the first trade places
    // with the lower half-wave's of the second: 8 consecutive columns per lane
#pragma unroll
    for (int p = 0; p < NQ / 2; ++p) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const auto r = __builtin_amdgcn_permlane32_swap(w2[2 * p][e], w2[2 * p + 1][e], false, false);
        w2[2 * p][e] = r[0];
        w2[2 * p + 1][e] = r[1];
      }
      const int n = n_blk + 2 * v0 + 16 * p + 8 * fhalf;
      if (mt < M && n < N)
        *reinterpret_cast<uint4*>(y + static_cast<int64_t>(mt) * N + n) =
            make_uint4(w2[2 * p][0], w2[2 * p][1], w2[2 * p + 1][0], w2[2 * p + 1][1]);
    }
  } else {
    const int n = n_blk + 2 * v0 + 4 * fhalf;
    if (mt < M && n < N) *reinterpret_cast<uint2*>(y + static_cast<int64_t>(mt) * N + n) = make_uint2(w2[0][0], w2[0][1]);
  }
}

template <int GS, int TB, int MW>
static hipError_t launch_mid(int M, int N, int K, int r, const uint8_t* xq, const float* xs, const uint16_t* t,
                             const uint8_t* wq, const uint32_t* wsp, const uint16_t* L2t, const uint16_t* bias,
                             uint16_t* y, hipStream_t stream) {
  constexpr int WB = 2;
  const dim3 grid(static_cast<unsigned>((M + 32 * TB - 1) / (32 * TB)) * static_cast<unsigned>((N + 32 * WB - 1) / (32 * WB)));
  const dim3 block(64 * MW);
#define QWAM_MID_CASE(R)                                                                                             \
  case R:                                                                                                            \
    hipLaunchKernelGGL((asp_gemm_mid_kernel<R, GS, TB, WB, MW>), grid, block, 0, stream, xq, xs, t, wq, wsp, L2t, bias, y, \
                       M, N, K);                                                                                     \
    break;
  switch (r) {
    QWAM_MID_CASE(16)
    QWAM_MID_CASE(32)
    QWAM_MID_CASE(48)
    QWAM_MID_CASE(64)
    default:
      return hipErrorInvalidValue;
  }
#undef QWAM_MID_CASE
  return hipGetLastError();
}

hipError_t launch_asp_gemm_mid(GemmForm form, int M, int N, int K, int r, int group, const uint8_t* xq,
                               const float* xs, const uint16_t* t, const uint8_t* wq, const uint32_t* wsp,
                               const uint16_t* L2t, const uint16_t* bias, uint16_t* y, hipStream_t stream) {
#define QWAM_MID_FORM(TB, MW)                                                                                 \
  return group == 32 ? launch_mid<32, TB, MW>(M, N, K, r, xq, xs, t, wq, wsp, L2t, bias, y, stream)           \
                     : launch_mid<64, TB, MW>(M, N, K, r, xq, xs, t, wq, wsp, L2t, bias, y, stream);
  switch (form) {
    case GemmForm::k32x64Waves8: QWAM_MID_FORM(1, 8)
    case GemmForm::k32x64Waves4: QWAM_MID_FORM(1, 4)
    case GemmForm::k64x64Waves4: QWAM_MID_FORM(2, 4)
    default: return hipErrorInvalidValue;
  }
#undef QWAM_MID_FORM
}

}  // namespace qwam
