// Weight pack (offline) and the fused activation kernel of the ASP layer.
//
//  pack:  R [N][K] f32 -> wq [N][K/2] packed codes, ws [G][N] scales (Eq. 2, App. B.1),
//         and each scale as two bf16 pieces for the GEMM's scale products
//  act:   x [M][K] bf16 -> x~ = x * (1/lambda) (Eq. 3), per-token group-64
//         codes xq [M][K/2] and scales xs [G][M] (Eq. 2), and the rank-r
//         down-projection t = bf16(x~) . L1 on bf16 matrix cores (V^T x~ of
//         Eq. 9), all in one pass over x.
#include <algorithm>

#include "qwam_act.h"
#include "qwam_device.h"
#include "qwam_internal.h"

namespace qwam {

// ---------------------------------------------------------------------------
// Weight pack: 4 lanes per (row, 64-channel span); each lane owns 16
// consecutive floats, i.e. one code block.  A workgroup takes 16 rows x 4 spans:
// whole lines of R and of the codes, and 16 neighbours of each scale array
// row, whose 4-byte stores then meet in one L2 (rows of spans dealt out one
// after another left every such line to all eight XCDs' L2s in pieces: 14336 x
// 3072 47.9 -> 39.9 us, i.e. 5.1 of the 5.2 TB/s that a large copy reaches;
// 9216 x 3072, group 32 38.3 -> 28.3 us).  Where the spans are no multiple of
// four the remaining ones are dealt out in the same way, so that no lane idles.
// The first `inv_blocks` workgroups write 1/lambda instead (a launch of its own
// took 4.8 us behind the pack).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_weights_kernel(const float* __restrict__ R,
                                                           const float* __restrict__ smooth,
                                                           uint8_t* __restrict__ wq,
                                                           float* __restrict__ ws, uint32_t* __restrict__ wsp,
                                                           float* __restrict__ inv_smooth, int N, int K, int g32,
                                                           int inv_blocks) {
  if (static_cast<int>(blockIdx.x) < inv_blocks) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < K) inv_smooth[k] = 1.0f / smooth[k];
    return;
  }
  const int G = K / kGroup;
  const int sub = threadIdx.x & 3;
  // (row, span) number of the four lanes: bands of 16 rows, in a band four spans
  // at a time (the last ones: G % 4), row by row
  const int team = (static_cast<int>(blockIdx.x) - inv_blocks) * 64 + (threadIdx.x >> 2);
  const int band = team / (16 * G), v16 = team % (16 * G);
  const int w = min(4, G - 4 * (v16 >> 6));
  const int n = 16 * band + (v16 & 63) / w;
  const int g = 4 * (v16 >> 6) + (v16 & 63) % w;
  const bool active = n < N;

  float v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = 0.0f;
  if (active) {
    const v4f* src = reinterpret_cast<const v4f*>(R + static_cast<int64_t>(n) * K + g * kGroup + sub * 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const v4f a = src[i];
      v[4 * i] = a.x; v[4 * i + 1] = a.y; v[4 * i + 2] = a.z; v[4 * i + 3] = a.w;
    }
  }
  float amax = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) amax = __builtin_fmaxf(amax, __builtin_fabsf(v[i]));
  // the 4 lanes of a 64-channel span; with group 32 lanes 0-1 and 2-3 separately
  amax = __builtin_fmaxf(amax, __shfl_xor(amax, 1));
  if (!g32) amax = __builtin_fmaxf(amax, __shfl_xor(amax, 2));
  const float s = q4_scale(amax);
  const float inv = q4_inv(s);
  float x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = v[i] * inv;
  uint32_t d0, d1, d2;
  codes_fp6_16(x, d0, d1, d2);
  if (active) {
    *reinterpret_cast<uint2*>(wq + static_cast<int64_t>(n) * (K / 2) + g * (kGroup / 2) + sub * 8) =
        fp6_code_block(d0, d1, d2);
    if (g32 ? (sub & 1) == 0 : sub == 0) {
      const int64_t at = static_cast<int64_t>(g32 ? 2 * g + (sub >> 1) : g) * N + n;
      ws[at] = s;
      // hi = bf16(s), lo = bf16(s - hi): s - hi is exact in float32
      const uint32_t hi = f32_to_bf16_rne(s);
      wsp[at] = hi | (f32_to_bf16_rne(s - bf16_to_f32(hi)) << 16);
    }
  }
}

// ---------------------------------------------------------------------------
// Fused activation kernel.
//
// A workgroup owns 16 tokens and all of K; its waves split the K groups into
// contiguous ranges, in the lane layout of qwam_act.h (lane l: token l % 16,
// channels 16*(l/16) .. +15 of the current group), so the smoothed values feed
// the down-projection on the bf16 matrix cores straight from registers.  Each
// wave prefetches the next group (x, L1 fragments) while it quantizes the current one;
// x is read with buffer loads and the codes / scales are written with buffer
// stores, so rows past M need no branches.  From K = 4096 on, a wave's code
// blocks of four consecutive groups (one 128-byte line of each of its 16 rows)
// are gathered in a 2 KB LDS line buffer of its own and written out as whole
// lines, 16 bytes per lane and 8 lines per instruction, instead of 32-byte
// pieces of 16 lines per group (the wave ranges are then whole line chunks);
// below, the 16 waves keep their ranges and store each group's blocks.  The
// per-wave partial t tiles are summed in LDS in wave order (deterministic) and
// rounded to bf16 once.
//
// With few token blocks (act_split) the workgroup takes a part of K instead,
// and its sums of t go to a workspace that split_t_kernel adds up: one
// workgroup's reads of x and L1 (32 + 2 r bytes per channel) are what a call
// of a few tokens waits for, at about 50 B/ns per CU
// (33 tokens, K = 14336: 26.3 us in three workgroups, 7.7 us in 168).  SPLIT
// kernels are instances of their own: the part's bounds and the choice of where
// the sums go cost a call with the whole K 0.1 us (1-4% up to K = 2752).
// ---------------------------------------------------------------------------
template <int RANK, bool INV_LDS, bool SPLIT>
__global__ __launch_bounds__(64 * act_waves<RANK>()) void quantize_act_kernel(
    const uint16_t* __restrict__ x, const float* __restrict__ inv_smooth,
    const uint16_t* __restrict__ L1f, uint8_t* __restrict__ xq, float* __restrict__ xs,
    uint16_t* __restrict__ t, float* __restrict__ part, int M, int K, int groups_per_wg, int groups_per_wave, int g32) {
  constexpr int RB = RANK / 16;
  // dynamic LDS: [nwaves][16][RANK] partial t, then (INV_LDS) [nwaves][groups_per_wave * 64] 1/lambda,
  // then [nwaves][16 rows][128 bytes] code lines
  extern __shared__ float red[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwaves = blockDim.x >> 6;
  const int row = lane & 15;
  const int chunk = lane >> 4;
  const int m0 = blockIdx.x * 16;
  const int rows = min(16, M - m0);
  const int G = K / kGroup;
  // the workgroup's groups (all of K, or split blockIdx.y), then the wave's
  const int wg_begin = SPLIT ? static_cast<int>(blockIdx.y) * groups_per_wg : 0;
  const int wg_end = SPLIT ? min(G, wg_begin + groups_per_wg) : G;
  const int g_begin = wg_begin + wave * groups_per_wave;
  const int g_end = min(wg_end, g_begin + groups_per_wave);

  // the workgroup's 16 rows of x, xq; out-of-range rows read as zero / are dropped
  const buf_rsrc x_rsrc = make_rsrc(x + static_cast<int64_t>(m0) * K, static_cast<uint32_t>(rows) * K * 2u);
  const buf_rsrc q_rsrc = make_rsrc(xq + static_cast<int64_t>(m0) * (K / 2), static_cast<uint32_t>(rows) * (K / 2));
  const uint32_t x_off = static_cast<uint32_t>(row * K + chunk * 16) * 2u;
  const uint32_t q_off = static_cast<uint32_t>(row * (K / 2) + chunk * 8);

  // the wave's slice of 1/lambda goes to LDS once (a per-group float4 load by
  // every lane would move 16x more bytes through the address unit than it uses)
  float* inv_w = red + nwaves * 16 * RANK + wave * groups_per_wave * kGroup;
  if (INV_LDS && g_begin < g_end) {
    const int n4 = (g_end - g_begin) * (kGroup / 4);
    const float4* src = reinterpret_cast<const float4*>(inv_smooth + g_begin * kGroup);
    for (int i = lane; i < n4; i += 64) reinterpret_cast<float4*>(inv_w)[i] = src[i];
  }

  auto fetch = [&](int g, ActFetch<RANK>& f) __attribute__((always_inline)) {
    const uint32_t go = static_cast<uint32_t>(g) * kGroup * 2u;
    f.xa = buf_load16(x_rsrc, x_off + go);
    f.xb = buf_load16(x_rsrc, x_off + go + 16u);
    load_l1_fragments<RB>(L1f, g, lane, f.l1);
  };

  v4f acc[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) acc[rb] = v4f{0.f, 0.f, 0.f, 0.f};

  uint8_t* line = reinterpret_cast<uint8_t*>(red + nwaves * 16 * RANK + (INV_LDS ? nwaves * groups_per_wave * kGroup : 0)) +
                  wave * 2048;
  // the launcher gives whole line chunks per wave from 64 groups on
  const bool lines = groups_per_wave % 4 == 0;
  // writes the staged blocks of groups max(g_begin, g & ~3) .. g (one line
  // chunk): lane l takes row 8h + l/8 and the 16-byte piece l%8 of its line
  auto flush = [&](int g) __attribute__((always_inline)) {
    const int q0 = g & ~3;
    const int p_lo = 2 * (max(g_begin, q0) - q0), p_hi = 2 * (g - q0 + 1);
    const int piece = lane & 7;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = 8 * h + (lane >> 3);
      if (piece >= p_lo && piece < p_hi) {
        const uint4 d = *reinterpret_cast<const uint4*>(line + r * 128 + piece * 16);
        buf_store16(d, q_rsrc, static_cast<uint32_t>(r * (K / 2) + q0 * (kGroup / 2) + piece * 16));
      }
    }
  };

  auto work = [&](int g, const ActFetch<RANK>& f) __attribute__((always_inline)) {
    const float4* ip = INV_LDS ? reinterpret_cast<const float4*>(inv_w + (g - g_begin) * kGroup + chunk * 16)
                               : reinterpret_cast<const float4*>(inv_smooth + g * kGroup + chunk * 16);
    float v[16];
    smooth16(f.xa, f.xb, ip, v);
    float s;
    const uint2 blk = quantize_block(v, g32, s);
    // the block goes to the row's line at its group's 32-byte slot (or, when
    // the wave's range is not made of line chunks, straight out); every lane
    // of a row (of a 32-channel half with group 32) holds the same scale and
    // writes it at the row's slot (letting one lane of each write it instead
    // measured 2-3 us slower at K = 3072)
    if (lines) *reinterpret_cast<uint2*>(line + row * 128 + (g & 3) * 32 + chunk * 8) = blk;
    else buf_store8(blk, q_rsrc, q_off + static_cast<uint32_t>(g) * (kGroup / 2));
    if (float* p = xs_slot(xs, g, M, m0, row, rows, chunk, g32)) *p = s;
    t_step_bf16<RB>(v, f.l1, acc);
    if (lines && ((g & 3) == 3 || g == g_end - 1)) flush(g);
  };

  // software pipeline, two groups per trip so the fetch registers are named statically;
  // the prefetch past the wave's last group re-reads that group (harmless, in bounds)
  if (g_begin < g_end) {
    ActFetch<RANK> fa, fb;
    fetch(g_begin, fa);
    int g = g_begin;
    for (; g + 1 < g_end; g += 2) {
      fetch(g + 1, fb);
      work(g, fa);
      fetch(min(g + 2, g_end - 1), fa);
      work(g + 1, fb);
    }
    if (g < g_end) work(g, fa);
  }

  store_t_partials<RB>(red, wave, lane, acc);
  __syncthreads();
  if constexpr (SPLIT) store_split_t<RANK>(red, nwaves, m0, part);
  else reduce_t<RANK>(red, nwaves, rows, t + static_cast<int64_t>(m0) * RANK, static_cast<float*>(nullptr));
}

// t of a call whose K was split over workgroups: the splits' partial sums
// (part [splits][stride], stride = padded tokens x r) added in split order.
__global__ __launch_bounds__(64) void split_t_kernel(const float* __restrict__ part, uint16_t* __restrict__ t, int n,
                                                     int splits, int stride) {
  const int e = blockIdx.x * 64 + threadIdx.x;
  if (e >= n) return;
  float sum = 0.0f;
#pragma unroll 8
  for (int s = 0; s < splits; ++s) sum += part[static_cast<int64_t>(s) * stride + e];
  t[e] = static_cast<uint16_t>(f32_to_bf16_rne(sum));
}

// ---------------------------------------------------------------------------
// Deflated activation kernel: the 4-bit path quantizes x~_perp = x~ - L1 t
// (Eq. 8 / Eq. 9) instead of x~.  Deflation needs t before any token of the
// workgroup is quantized, and it needs t's exact bits (every code depends on
// them), so the workgroup of 16 tokens runs two phases:
//
//  1. t = bf16(sum_k bf16(x~_k) L1[k, :]) on the FP64 matrix cores
//     (t_step_f64): the products are exact in double and the double sum is
//     within ~1e-13 of the exact one, far inside bf16's half ulp, so the
//     single rounding to bf16 gives the bf16 of the exact sum.  The per-wave
//     partial tiles are summed in LDS in wave order.
//  2. every wave walks its groups again: the re-read, re-smoothed x~ goes
//     through r rank-1 updates on the FP32 matrix cores (deflate_step), whose
//     result is in the quantizer's lane layout.
// With few token blocks the phases are launches of their own, each over parts
// of K (Phase::kSums, kCodes): the second adds the first one's sums in split
// order (33 tokens, K = 14336: 117 us in one launch, 15 us in two).
// ---------------------------------------------------------------------------
template <int RANK, bool INV_LDS, Phase PHASE>
__global__ __launch_bounds__(64 * act_waves<RANK>()) void quantize_act_deflated_kernel(
    const uint16_t* __restrict__ x, const float* __restrict__ inv_smooth,
    const uint16_t* __restrict__ L1f, const uint16_t* __restrict__ L1, uint8_t* __restrict__ xq, float* __restrict__ xs,
    uint16_t* __restrict__ t, double* __restrict__ part, int M, int K, int groups_per_wg, int groups_per_wave,
    int g32) {
  constexpr int RB = RANK / 16;
  // dynamic LDS: [nwaves][16][RANK] double partial t (not in kCodes) | [16][RANK] float -t |
  // (INV_LDS) [nwaves][groups_per_wave * 64] 1/lambda
  extern __shared__ double red64[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwaves = blockDim.x >> 6;
  const int row = lane & 15;
  const int chunk = lane >> 4;
  const int m0 = blockIdx.x * 16;
  const int rows = min(16, M - m0);
  const int G = K / kGroup;
  const int wg_begin = PHASE == Phase::kAll ? 0 : static_cast<int>(blockIdx.y) * groups_per_wg;
  const int wg_end = PHASE == Phase::kAll ? G : min(G, wg_begin + groups_per_wg);
  const int g_begin = wg_begin + wave * groups_per_wave;
  const int g_end = min(wg_end, g_begin + groups_per_wave);

  const buf_rsrc x_rsrc = make_rsrc(x + static_cast<int64_t>(m0) * K, static_cast<uint32_t>(rows) * K * 2u);
  const buf_rsrc q_rsrc = make_rsrc(xq + static_cast<int64_t>(m0) * (K / 2), static_cast<uint32_t>(rows) * (K / 2));
  const uint32_t x_off = static_cast<uint32_t>(row * K + chunk * 16) * 2u;
  const uint32_t q_off = static_cast<uint32_t>(row * (K / 2) + chunk * 8);

  float* tneg = reinterpret_cast<float*>(red64 + (PHASE == Phase::kCodes ? 0 : nwaves * 16 * RANK));
  float* inv_w = tneg + 16 * RANK + wave * groups_per_wave * kGroup;
  if (INV_LDS && g_begin < g_end) {
    const int n4 = (g_end - g_begin) * (kGroup / 4);
    const float4* src = reinterpret_cast<const float4*>(inv_smooth + g_begin * kGroup);
    for (int i = lane; i < n4; i += 64) reinterpret_cast<float4*>(inv_w)[i] = src[i];
  }
  auto inv_ptr = [&](int g) __attribute__((always_inline)) {
    return INV_LDS ? reinterpret_cast<const float4*>(inv_w + (g - g_begin) * kGroup + chunk * 16)
                   : reinterpret_cast<const float4*>(inv_smooth + g * kGroup + chunk * 16);
  };

  // ---- phase 1: t in double ----
  if constexpr (PHASE != Phase::kCodes) {
    auto fetch1 = [&](int g, ActFetch<RANK>& f) __attribute__((always_inline)) {
      const uint32_t go = static_cast<uint32_t>(g) * kGroup * 2u;
      f.xa = buf_load16(x_rsrc, x_off + go);
      f.xb = buf_load16(x_rsrc, x_off + go + 16u);
      load_l1_fragments<RB>(L1f, g, lane, f.l1);
    };
    v4d acc[RB];
  #pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[rb] = v4d{0.0, 0.0, 0.0, 0.0};
    auto work1 = [&](int g, const ActFetch<RANK>& f) __attribute__((always_inline)) {
      float v[16];
      smooth16(f.xa, f.xb, inv_ptr(g), v);
      t_step_f64<RB>(v, f.l1, acc);
    };
    if (g_begin < g_end) {
      ActFetch<RANK> fa, fb;
      fetch1(g_begin, fa);
      int g = g_begin;
      for (; g + 1 < g_end; g += 2) {
        fetch1(g + 1, fb);
        work1(g, fa);
        fetch1(min(g + 2, g_end - 1), fa);
        work1(g + 1, fb);
      }
      if (g < g_end) work1(g, fa);
    }
    store_t_partials<RB>(red64, wave, lane, acc);
    __syncthreads();
    if constexpr (PHASE == Phase::kSums) {
      store_split_t<RANK>(red64, nwaves, m0, part);
      return;
    }
    reduce_t<RANK>(red64, nwaves, rows, t + static_cast<int64_t>(m0) * RANK, tneg);
  } else {
    combine_split_t<RANK>(part, gridDim.y, m0, rows, t + static_cast<int64_t>(m0) * RANK, tneg);
  }
  __syncthreads();

  // ---- phase 2: deflate with r rank-1 updates, then quantize ----
  const int a_ch = deflate_channel(lane);
  auto fetch2 = [&](int g, DeflFetch<RANK>& f) __attribute__((always_inline)) {
    const uint32_t go = static_cast<uint32_t>(g) * kGroup * 2u;
    f.xa = buf_load16(x_rsrc, x_off + go);
    f.xb = buf_load16(x_rsrc, x_off + go + 16u);
    load_l1_row<RANK>(L1, g * kGroup + a_ch, f.l1);
  };
  const float* tn_row = tneg + row * RANK;
  auto work2 = [&](int g, const DeflFetch<RANK>& f) __attribute__((always_inline)) {
    float v[16];
    smooth16(f.xa, f.xb, inv_ptr(g), v);
    deflate_step<RANK>(v, f.l1, tn_row);
    quantize_pack_store(v, q_rsrc, q_off + static_cast<uint32_t>(g) * (kGroup / 2),
                        xs_slot(xs, g, M, m0, row, rows, chunk, g32), g32);
  };
  if (g_begin < g_end) {
    DeflFetch<RANK> fa, fb;
    fetch2(g_begin, fa);
    int g = g_begin;
    for (; g + 1 < g_end; g += 2) {
      fetch2(g + 1, fb);
      work2(g, fa);
      fetch2(min(g + 2, g_end - 1), fa);
      work2(g + 1, fb);
    }
    if (g < g_end) work2(g, fa);
  }
}

// ---------------------------------------------------------------------------
hipError_t launch_pack_weights(int K, int N, int group, const float* R, const float* smooth, uint8_t* wq,
                               float* ws, uint32_t* wsp, float* inv_smooth, hipStream_t stream) {
  const int64_t blocks = (static_cast<int64_t>(N) * (K / kGroup) + 63) / 64;
  const int inv_blocks = (K + 255) / 256;
  hipLaunchKernelGGL(pack_weights_kernel, dim3(static_cast<unsigned>(blocks + inv_blocks)), dim3(256), 0, stream, R,
                     smooth, wq, ws, wsp, inv_smooth, N, K, group == 32 ? 1 : 0, inv_blocks);
  return hipGetLastError();
}

// Splits of K over workgroups, and groups per split, for few token blocks: as
// many splits as fill the chip once, in whole line chunks of four groups (0
// splits: K stays whole).
ActSplit act_split(int M, int K, int unit_groups, int min_units) {
  const int blocks = (M + 15) / 16;
  const int units = (K / kGroup + unit_groups - 1) / unit_groups;
  if (blocks > kSplitBlocks || units < min_units) return {0, 0};
  const int want = 256 / blocks;                       // >= 2
  // units per split; at most 128 groups, so that a split's 1/lambda fits in LDS
  const int per = std::min((units + want - 1) / want, 128 / unit_groups);
  return {(units + per - 1) / per, per * unit_groups};
}

int plain_min_units(int M, int r) {
  return r <= 32 && 256 / ((M + 15) / 16) <= 2 ? kMinUnitsTwo : kMinUnits;
}

static int64_t split_bytes(const ActSplit& s, int M, int r, size_t elem) {
  return static_cast<int64_t>(s.splits) * ((M + 15) / 16 * 16) * r * static_cast<int64_t>(elem);
}

int64_t act_workspace_bytes(int M, int K, int r, int B, bool deflate) {
  const ActSplit s = B != 0 ? rotated_split(M, K, r, B, deflate)
                            : act_split(M, K, 4, deflate ? kMinUnitsDeflated : plain_min_units(M, r));
  return s.splits > 1 ? split_bytes(s, M, r, deflate ? sizeof(double) : sizeof(float)) : 0;
}

hipError_t launch_split_t(int M, int r, int splits, const float* part, uint16_t* t, hipStream_t stream) {
  const int n = M * r, stride = (M + 15) / 16 * 16 * r;
  hipLaunchKernelGGL(split_t_kernel, dim3((n + 63) / 64), dim3(64), 0, stream, part, t, n, splits, stride);
  return hipGetLastError();
}

hipError_t launch_quantize_act(int M, int K, int r, int group, const uint16_t* x, const float* inv_smooth,
                               const uint16_t* L1f, uint8_t* xq, float* xs, uint16_t* t, void* workspace,
                               hipStream_t stream) {
  const int g32 = group == 32 ? 1 : 0;
  const ActSplit split = workspace != nullptr ? act_split(M, K, 4, plain_min_units(M, r)) : ActSplit{0, 0};
  float* part = split.splits > 1 ? static_cast<float*>(workspace) : nullptr;
  const int nsplit = part != nullptr ? split.splits : 1;
  const int G = part != nullptr ? split.groups : K / kGroup;     // groups per workgroup
  // 1/lambda is staged in LDS when the slice fits (16384 channels); a longer one is read from global memory
  const bool inv_lds = G * kGroup <= 16384;
  auto go = [&](auto kernel, int max_waves) {
    int nwaves = G < max_waves ? G : max_waves;
    int gpw = (G + nwaves - 1) / nwaves;
    if (G >= 64) {   // wave ranges of whole 4-group line chunks (below, the waves keep one group or more each)
      gpw = (gpw + 3) & ~3;
      nwaves = (G + gpw - 1) / gpw;
    }
    // the code-line buffers (2 KB per wave) only where the kernel uses them
    const size_t lds = static_cast<size_t>(nwaves) * (16 * r + (inv_lds ? gpw * kGroup : 0)) * sizeof(float) +
                       (gpw % 4 == 0 ? static_cast<size_t>(nwaves) * 2048 : 0);
    if (lds > 64 * 1024) {   // opt in to more than 64 KB of dynamic LDS
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((M + 15) / 16, nsplit), dim3(64 * nwaves), lds, stream,
                       x, inv_smooth, L1f, xq, xs, t, part, M, K, G, gpw, g32);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || part == nullptr ? e : launch_split_t(M, r, nsplit, part, t, stream);
  };
#define QWAM_ACT_CASE(R)                                                                  \
  case R:                                                                                 \
    /* a split's slice of 1/lambda always fits in LDS */                                  \
    if (part != nullptr) return go(quantize_act_kernel<R, true, true>, act_waves<R>());   \
    return inv_lds ? go(quantize_act_kernel<R, true, false>, act_waves<R>())              \
                   : go(quantize_act_kernel<R, false, false>, act_waves<R>());
  switch (r) {
    QWAM_ACT_CASE(16)
    QWAM_ACT_CASE(32)
    QWAM_ACT_CASE(48)
    QWAM_ACT_CASE(64)
    default: return hipErrorInvalidValue;
  }
#undef QWAM_ACT_CASE
}

hipError_t launch_quantize_act_deflated(int M, int K, int r, int group, const uint16_t* x,
                                        const float* inv_smooth, const uint16_t* L1f, const uint16_t* L1,
                                        uint8_t* xq, float* xs, uint16_t* t, void* workspace, hipStream_t stream) {
  const int g32 = group == 32 ? 1 : 0;
  const ActSplit split = workspace != nullptr ? act_split(M, K, 4, kMinUnitsDeflated) : ActSplit{0, 0};
  double* part = split.splits > 1 ? static_cast<double*>(workspace) : nullptr;
  const int nsplit = part != nullptr ? split.splits : 1;
  const int G = part != nullptr ? split.groups : K / kGroup;     // groups per workgroup
  const bool inv_lds = G * kGroup <= 16384;
  auto go = [&](auto kernel, int max_waves, bool sums) {
    const int nwaves = G < max_waves ? G : max_waves;
    const int gpw = (G + nwaves - 1) / nwaves;
    const size_t lds = (sums ? static_cast<size_t>(nwaves) * 16 * r * sizeof(double) : 0) + 16 * r * sizeof(float) +
                       (inv_lds ? static_cast<size_t>(nwaves) * gpw * kGroup * sizeof(float) : 0);
    if (lds > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((M + 15) / 16, nsplit), dim3(64 * nwaves), lds, stream, x, inv_smooth, L1f, L1, xq,
                       xs, t, part, M, K, G, gpw, g32);
    return hipGetLastError();
  };
#define QWAM_DEFL_CASE(R)                                                                                          \
  case R: {                                                                                                        \
    if (part == nullptr)                                                                                           \
      return inv_lds ? go(quantize_act_deflated_kernel<R, true, Phase::kAll>, act_waves<R>(), true)                \
                     : go(quantize_act_deflated_kernel<R, false, Phase::kAll>, act_waves<R>(), true);              \
    /* a split's slice of 1/lambda always fits in LDS */                                                           \
    const hipError_t e = go(quantize_act_deflated_kernel<R, true, Phase::kSums>, act_waves<R>(), true);            \
    return e != hipSuccess ? e : go(quantize_act_deflated_kernel<R, true, Phase::kCodes>, act_waves<R>(), false);  \
  }
  switch (r) {
    QWAM_DEFL_CASE(16)
    QWAM_DEFL_CASE(32)
    QWAM_DEFL_CASE(48)
    QWAM_DEFL_CASE(64)
    default: return hipErrorInvalidValue;
  }
#undef QWAM_DEFL_CASE
}

}  // namespace qwam
