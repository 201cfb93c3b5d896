// Activation kernels with the block Hadamard rotation of Eq. 3:
//     x~ = H diag(lambda)^-1 x,
// H block-diagonal with Hadamard blocks of size B (the largest power of two
// dividing K, at most 1024, App. B.1), applied online with the fast
// Walsh-Hadamard transform (the weights were rotated offline).  The transform
// runs in float32, one rounding per butterfly, stages on element bit 0, 1, ..
// in that order, then one multiply by fl32(1/sqrt(B)).
//
// A block spans several groups, so a workgroup (16 tokens) works in tiles of
// T channels (a multiple of B and of 64 dividing K, at most 1024):
//   rotate:   pass p of a tile is 1024 consecutive elements of the [16][T]
//             tile; a lane holds 16 consecutive channels of one token, so
//             butterfly stages 0-3 run in registers and the others between
//             lanes (fwht16: DPP operands and the permlane swaps of gfx950).
//             The rotated tile goes to LDS (rows padded by 4 floats and
//             swizzled against bank conflicts).
//   quantize: each wave reads its groups of the tile back in the lane layout
//             of qwam_act.h and runs the plain kernel's per-group steps (or,
//             deflated, the two phases of the deflated kernel, rotating the
//             tiles again in phase 2).
// With few token blocks a workgroup takes some of the tiles (rotated_split):
// the sums of t are then added by a second launch, which for the deflated
// variant is the one that deflates and quantizes (Phase::kCodes).
#include <cmath>
#include <type_traits>

#include "qwam_act.h"
#include "qwam_device.h"
#include "qwam_internal.h"

namespace qwam {

namespace {

constexpr int kTilePad = 4;   // floats of padding per LDS tile row

// A tile row keeps float4 q of its 16-channel chunk c in slot q ^ tile_swz(c).
// The rotation writes one float4 per lane, 64 bytes apart: unswizzled, 16
// lanes fall on 16 of the 64 banks.  The reads (16 rows, one chunk) are
// conflict-free either way, by the padding.
__device__ __forceinline__ int tile_swz(int c) { return (c >> 2) & 3; }

// The 1024 elements of a rotation pass are indexed by 10 bits.  Lane l holds
// 16 consecutive ones, chunk rot_chunk(l) (bits 4-9), register = bits 0-3.
// Within 8 lanes the chunks are ordered so that chunk bit 2 (element bit 6)
// pairs lanes l and l ^ 7, which a DPP modifier can reach (row_half_mirror);
// bits 0, 1, 3 pair l ^ 1, l ^ 2 (quad permutes) and l ^ 8 (row_ror:8).
__device__ __forceinline__ int rot_chunk(int lane) { return lane ^ ((lane & 4) ? 3 : 0); }

// Fast Walsh-Hadamard transform of blocks of 2^logB elements (stages on
// element bit 0, 1, .., one rounding per butterfly), times `scale`.  What it
// costs is vector instructions, so each stage takes as few as it can:
//   bits 0-3   between the lane's registers, one add or subtraction each;
//   bits 4-7   between lanes, one v_fmac_f32 with a DPP operand each
//              (EXACT: two): v <- v + s p, s = -1 in the lane whose element
//              has the bit set, which so holds b - a instead of a - b.  A lane's
//              values thus change sign together; the final multiply undoes it.
//              Negation commutes with rounding, except that the sign of a zero
//              result is lost: fma(v, scale, +0) makes every zero +0, which is
//              what the true stages give unless an input is -0 (a -0 comes from -0s only).  EXACT keeps
//              a - b itself and is for passes that hold a -0;
//   bits 8, 9  v_permlane16/32_swap of registers i and i + 4 (i + 8): the
//              lower lanes then hold both halves of register i's pairs and
//              the upper ones those of register i + 4, so one add and one
//              subtraction serve two elements.  Register bit 2 (3) and lane bit
//              4 (5) trade places; rot_element gives the resulting element.
// 11 vector instructions per element (18 and an LDS swizzle with a separate
// exchange per element): M = 4096, r = 32, rotated 20.1 -> 15.9 us (K = 3072)
// and 79 -> 66 us (K = 14336), rotated and deflated 50 -> 41 and 224 -> 179 us;
// where every pass holds a -0, 18.0, 71, 45 and 201 us.
//
// v <- v + s (v of the lane that `ctrl` names), for eight registers in one
// instruction each (the compiler keeps the exchange and the multiply-add
// apart).  The leading s_nop separates a register's last write from its use as
// a DPP source, the trailing one the last writes from a lane swap.
#define QWAM_FMAC1_DPP(N, CTRL) "v_fmac_f32_dpp %" #N ", %" #N ", %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"
#define QWAM_FMAC8_DPP(a, b, c, d, e, f, g, h, s, CTRL)                                                              \
  asm("s_nop 1\n\t" QWAM_FMAC1_DPP(0, CTRL) QWAM_FMAC1_DPP(1, CTRL) QWAM_FMAC1_DPP(2, CTRL) QWAM_FMAC1_DPP(3, CTRL)  \
          QWAM_FMAC1_DPP(4, CTRL) QWAM_FMAC1_DPP(5, CTRL) QWAM_FMAC1_DPP(6, CTRL) QWAM_FMAC1_DPP(7, CTRL) "s_nop 1"  \
      : "+v"(a), "+v"(b), "+v"(c), "+v"(d), "+v"(e), "+v"(f), "+v"(g), "+v"(h)                                       \
      : "v"(s))
template <bool EXACT>
__device__ __forceinline__ void fwht16(float (&v)[16], int lane, int logB, float scale) {
#pragma unroll
  for (int h = 1; h < 16; h <<= 1)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (!(i & h)) {
        const float a = v[i], b = v[i + h];
        v[i] = a + b;
        v[i + h] = a - b;
      }
  const int c = rot_chunk(lane);
  float total = scale;
#define QWAM_DPP_STAGE(BIT, CTRL, TEXT)                                                                              \
  if (logB > 4 + BIT) {                                                                                              \
    const float s = ((c >> BIT) & 1) != 0 ? -1.0f : 1.0f;                                                            \
    if constexpr (EXACT) {                                                                                           \
      _Pragma("unroll") for (int i = 0; i < 16; ++i) {                                                               \
        const int u = __float_as_int(v[i]);                                                                          \
        v[i] = __builtin_fmaf(v[i], s, __int_as_float(__builtin_amdgcn_update_dpp(0, u, CTRL, 0xF, 0xF, false)));    \
      }                                                                                                              \
    } else {                                                                                                         \
      QWAM_FMAC8_DPP(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], s, TEXT);                                       \
      QWAM_FMAC8_DPP(v[8], v[9], v[10], v[11], v[12], v[13], v[14], v[15], s, TEXT);                                 \
      total *= s;                                                                                                    \
    }                                                                                                                \
  }
  QWAM_DPP_STAGE(0, 0xB1, "quad_perm:[1,0,3,2]")     // l ^ 1
  QWAM_DPP_STAGE(1, 0x4E, "quad_perm:[2,3,0,1]")     // l ^ 2
  QWAM_DPP_STAGE(2, 0x141, "row_half_mirror")        // l ^ 7
  QWAM_DPP_STAGE(3, 0x128, "row_ror:8")              // l ^ 8
#undef QWAM_DPP_STAGE
  auto swap_stage = [&](auto hc, auto swap) __attribute__((always_inline)) {
    constexpr int h = decltype(hc)::value;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (!(i & h)) {
        const auto r = swap(__float_as_uint(v[i]), __float_as_uint(v[i + h]));
        const float a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
        v[i] = a + b;
        v[i + h] = a - b;
      }
  };
  if (logB > 8)
    swap_stage(std::integral_constant<int, 4>{},
               [](unsigned x, unsigned y) { return __builtin_amdgcn_permlane16_swap(x, y, false, false); });
  if (logB > 9)
    swap_stage(std::integral_constant<int, 8>{},
               [](unsigned x, unsigned y) { return __builtin_amdgcn_permlane32_swap(x, y, false, false); });
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = EXACT ? v[i] * scale : __builtin_fmaf(v[i], total, 0.0f);
}

#undef QWAM_FMAC8_DPP
#undef QWAM_FMAC1_DPP

// The element of the pass that register 4 q (q = 0..3) holds after fwht16
// (registers 4 q + 1 .. + 3: the next three).
__device__ __forceinline__ int rot_element(int lane, int q, int logB) {
  const int c = rot_chunk(lane);
  const int b2 = q & 1, b3 = q >> 1, l4 = (c >> 4) & 1, l5 = c >> 5;
  return 16 * (c & 15) + (logB > 8 ? 4 * l4 + 256 * b2 : 4 * b2 + 256 * l4) +
         (logB > 9 ? 8 * l5 + 512 * b3 : 8 * b3 + 512 * l5);
}

// Smoothed inputs of a pass that include a -0 (the transform's exact form).
__device__ __forceinline__ bool any_negative_zero(const float (&v)[16]) {
  int least = __float_as_int(v[0]);
#pragma unroll
  for (int i = 1; i < 16; ++i) least = min(least, __float_as_int(v[i]));
  return __any(least == INT32_MIN);      // -0 is the least float bit pattern as an integer
}

}  // namespace

// Registers of one rotation pass: 16 bf16 of x and the matching 1/lambda.
struct RotFetch {
  uint4 xa, xb;
  float4 inv[4];
};

// Rotation passes (= groups) of a tile per wave: a tile of at most 1024
// channels has at most 16, spread over act_waves<RANK>() waves.
template <int RANK>
constexpr int per_wave() { return 16 / act_waves<RANK>(); }

// Barrier for LDS hand-offs between the waves: waits for this wave's LDS
// operations only, so prefetched global loads stay in flight across it.
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Row of the [16][T] tile that holds 16-element chunk c: c / (T / 16), as one
// multiplication and a shift.  T is no constant and often no power of two; a
// division and a remainder per tile address, five pairs a pass, cost up to 1 us a
// tile (M = 300, K = 320, r = 16, deflated: 7.9 us, as it is 6.1).  Every chunk of
// every width is checked below.
constexpr int tile_row_mul(int T) { return (65536 + T / 16 - 1) / (T / 16); }
constexpr int tile_row(int c, int mul) { return (c * mul) >> 16; }
constexpr bool tile_rows_exact() {
  for (int T = 64; T <= 1024; T += 64)
    for (int c = 0; c < T; ++c)
      if (tile_row(c, tile_row_mul(T)) != c / (T / 16)) return false;
  return true;
}
static_assert(tile_rows_exact(), "the multiplication gives the quotient");

template <int RANK, bool DEFLATE, Phase PHASE>
__global__ __launch_bounds__(64 * act_waves<RANK>()) void quantize_act_rotated_kernel(
    const uint16_t* __restrict__ x, const float* __restrict__ inv_smooth,
    const uint16_t* __restrict__ L1f, const uint16_t* __restrict__ L1, uint8_t* __restrict__ xq, float* __restrict__ xs,
    uint16_t* __restrict__ t, std::conditional_t<DEFLATE, double, float>* __restrict__ part, int M, int K, int logB,
    int T, int row_mul, float hscale, int g32, int red_off, int tiles_per_wg) {
  static_assert(DEFLATE || PHASE == Phase::kAll, "one launch without deflation");
  constexpr int RB = RANK / 16;
  constexpr int kMaxPerWave = per_wave<RANK>();
  using Acc = std::conditional_t<DEFLATE, double, float>;
  // dynamic LDS: two tiles [16][T + pad] float (tile tb in buffer tb % 2) |
  // partial t [nwaves][16][RANK] Acc at float offset red_off (after the tiles,
  // or, when both do not fit, over the buffer the last tile does not use) |
  // (DEFLATE) -t [16][RANK] float after both
  extern __shared__ double lds_raw[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwaves = blockDim.x >> 6;
  const int row = lane & 15;
  const int chunk = lane >> 4;
  const int m0 = blockIdx.x * 16;
  const int rows = min(16, M - m0);
  const int TS = T + kTilePad;
  const int tile0 = static_cast<int>(blockIdx.y) * tiles_per_wg;   // the workgroup's tiles (all of them, or a split)
  const int ntiles = PHASE == Phase::kOneTile ? 1 : min(K / T - tile0, tiles_per_wg);
  const int npass = T / kGroup;          // 1024-element passes per tile = groups per tile

  float* tiles = reinterpret_cast<float*>(lds_raw);
  Acc* red = reinterpret_cast<Acc*>(tiles + red_off);
  float* tneg = reinterpret_cast<float*>(red + (PHASE == Phase::kCodes ? 0 : nwaves * 16 * RANK));
  if (red_off < 2 * 16 * TS) tneg = tiles + 2 * 16 * TS;   // red over a tile buffer

  const buf_rsrc x_rsrc = make_rsrc(x + static_cast<int64_t>(m0) * K, static_cast<uint32_t>(rows) * K * 2u);
  const buf_rsrc q_rsrc = make_rsrc(xq + static_cast<int64_t>(m0) * (K / 2), static_cast<uint32_t>(rows) * (K / 2));
  const uint32_t q_off = static_cast<uint32_t>(row * (K / 2) + chunk * 8);

  // pass k of this wave in a tile covers elements (wave + k nwaves) * 1024 + 16 lane .. +15
  auto fetch_tile = [&](int tb, RotFetch (&rf)[kMaxPerWave]) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < kMaxPerWave; ++k) {
      const int p = wave + k * nwaves;
      if (p < npass) {
        const int c = p * 64 + rot_chunk(lane);
        const int r = tile_row(c, row_mul);
        const int ch = (tile0 + tb) * T + 16 * c - r * T;
        const uint32_t xo = static_cast<uint32_t>(r * K + ch) * 2u;
        rf[k].xa = buf_load16(x_rsrc, xo);
        rf[k].xb = buf_load16(x_rsrc, xo + 16u);
        const float4* ip = reinterpret_cast<const float4*>(inv_smooth + ch);
#pragma unroll
        for (int q = 0; q < 4; ++q) rf[k].inv[q] = ip[q];
      }
    }
  };
  // smooth, transform and scale the fetched passes into the LDS tile (tokens past M are zero)
  auto rotate_tile = [&](const RotFetch (&rf)[kMaxPerWave], float* tile) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < kMaxPerWave; ++k) {
      const int p = wave + k * nwaves;
      if (p < npass) {
        // The lane's signs and addresses do not change from tile to tile.  Kept
        // in registers (128 at 16 waves) they make the variant without
        // deflation spill, which then takes 83 instead of 74 us at M = 4096,
        // K = 14336; the deflated one keeps them (178 against 189 us), except
        // where there is only one tile (kOneTile: the set-up ahead of the loop
        // took longer than it saved, M = 300, K = 320, r = 16 6.7 us).
        int ln = lane;
        if constexpr (!DEFLATE) asm volatile("" : "+v"(ln));
        float v[16];
        smooth16_regs(rf[k].xa, rf[k].xb, rf[k].inv, v);
        if (any_negative_zero(v)) fwht16<true>(v, ln, logB, hscale);
        else fwht16<false>(v, ln, logB, hscale);
        // float offsets of the four quads in the tile; blocks of up to 256 keep
        // a lane's elements in one chunk, whose row is computed once
        int off[4];
        if (logB > 8) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int e = p * 1024 + rot_element(ln, q, logB);
            const int r = tile_row(e >> 4, row_mul);
            const int ch = e - r * T;
            off[q] = r * TS + (ch & ~15) + 4 * (((ch >> 2) & 3) ^ tile_swz(ch >> 4));
          }
        } else {
          const int c = p * 64 + rot_chunk(ln);
          const int r = tile_row(c, row_mul);
          const int ch = 16 * c - r * T;
          const int sw = tile_swz(ch >> 4);
#pragma unroll
          for (int q = 0; q < 4; ++q) off[q] = r * TS + ch + 4 * (q ^ sw);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(tile + off[q]) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
      }
    }
  };
  auto read_group = [&](const float* tile, int gl, float (&v)[16]) __attribute__((always_inline)) {
    const float* src = tile + row * TS + gl * kGroup + chunk * 16;
    const int sw = tile_swz(4 * gl + chunk);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 f = *reinterpret_cast<const float4*>(src + 4 * (q ^ sw));
      v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
    }
  };
  auto store_codes = [&](int g, const float (&v)[16]) __attribute__((always_inline)) {
    quantize_pack_store(v, q_rsrc, q_off + static_cast<uint32_t>(g) * (kGroup / 2),
                        xs_slot(xs, g, M, m0, row, rows, chunk, g32), g32);
  };

  std::conditional_t<DEFLATE, v4d, v4f> acc[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) acc[rb] = {};

  RotFetch rf[kMaxPerWave];
  fetch_tile(0, rf);
  // pass over the tiles: t partials (and, without deflation, the codes).  The
  // next tile's x and 1/lambda are requested as soon as this tile's are in LDS.
  // Tile tb goes to buffer tb % 2, so one barrier per tile suffices: a wave
  // writes buffer tb % 2 only after the barrier of tile tb - 1, which every
  // wave reaches after its reads of tile tb - 2 from that buffer.
  if constexpr (PHASE != Phase::kCodes) {
    for (int tb = 0; tb < ntiles; ++tb) {
      float* tile = tiles + (tb & 1) * 16 * TS;
      rotate_tile(rf, tile);
      if (tb + 1 < ntiles) fetch_tile(tb + 1, rf);
      v8s l1[kMaxPerWave][RB][2];
  #pragma unroll
      for (int k = 0; k < kMaxPerWave; ++k) {
        const int gl = wave + k * nwaves;
        if (gl < npass) load_l1_fragments<RB>(L1f, (tile0 + tb) * npass + gl, lane, l1[k]);
      }
      lds_sync();
  #pragma unroll
      for (int k = 0; k < kMaxPerWave; ++k) {
        const int gl = wave + k * nwaves;
        if (gl < npass) {
          float v[16];
          read_group(tile, gl, v);
          if constexpr (DEFLATE) {
            t_step_f64<RB>(v, l1[k], acc);
          } else {
            store_codes((tile0 + tb) * npass + gl, v);
            t_step_bf16<RB>(v, l1[k], acc);
          }
        }
      }
    }
    // the second pass takes the last tile first, still in LDS from the first
    // pass, then tiles 0 .. ntiles - 2 again; tile 0's x is requested here
    if constexpr (DEFLATE && PHASE == Phase::kAll)
      if (ntiles > 1) fetch_tile(0, rf);
    lds_sync();                                   // the partials may overwrite a tile buffer
    store_t_partials<RB>(red, wave, lane, acc);
    lds_sync();
    if (PHASE == Phase::kSums || (!DEFLATE && part != nullptr)) {
      store_split_t<RANK>(red, nwaves, m0, part);
      return;
    }
    reduce_t<RANK>(red, nwaves, rows, t + static_cast<int64_t>(m0) * RANK, DEFLATE ? tneg : nullptr);
  } else {
    combine_split_t<RANK>(part, gridDim.y, m0, rows, t + static_cast<int64_t>(m0) * RANK, tneg);
  }

  if constexpr (DEFLATE) {
    lds_sync();
    // second pass: deflate and quantize.  Step 0 reads the last tile where
    // the first pass left it (buffer Lb; the partial t tiles, if they were
    // placed over a tile, went to the other buffer); step i >= 1 rotates tile
    // i - 1 again into buffer (Lb + i) % 2, which every wave last read at
    // step i - 2, before the previous barrier.
    const int a_ch = deflate_channel(lane);
    const float* tn_row = tneg + row * RANK;
    // (A launch of its own for the codes, kCodes, has no tile in LDS: it
    // rotates tiles 0, 1, .. in order.)
    constexpr bool kept = PHASE != Phase::kCodes;
    const int Lb = (ntiles - 1) & 1;
    for (int i = 0; i < ntiles; ++i) {
      const int tb = !kept ? i : i == 0 ? ntiles - 1 : i - 1;
      float* tile = tiles + ((Lb + i) & 1) * 16 * TS;
      if (!kept || i > 0) {
        rotate_tile(rf, tile);
        if (tb + 1 < (kept ? ntiles - 1 : ntiles)) fetch_tile(tb + 1, rf);
      }
      uint32_t l1w[kMaxPerWave][RANK / 2];
#pragma unroll
      for (int k = 0; k < kMaxPerWave; ++k) {
        const int gl = wave + k * nwaves;
        if (gl < npass) load_l1_row<RANK>(L1, ((tile0 + tb) * npass + gl) * kGroup + a_ch, l1w[k]);
      }
      lds_sync();
#pragma unroll
      for (int k = 0; k < kMaxPerWave; ++k) {
        const int gl = wave + k * nwaves;
        if (gl < npass) {
          float v[16];
          read_group(tile, gl, v);
          deflate_step<RANK>(v, l1w[k], tn_row);
          store_codes((tile0 + tb) * npass + gl, v);
        }
      }
    }
  }
}

// Few tokens (M <= kFewTokens, K <= KMAX): one 256-thread workgroup per
// token, so that a call of a few tokens spreads over as many CUs as tokens
// instead of running on one.  The same arithmetic as above, laid out for one
// token:
//   rotate:   wave w < ceil(K / 1024) transforms channels 1024 w .. + 1023,
//             16 per lane, in registers (fwht16) into an LDS row of K floats, and
//             bf16(x~) as doubles into a second row;
//   t:        thread i sums column j = i % r over its range of CH = KMAX r /
//             256 consecutive channels in double, from its L1t row segment
//             (requested at the start); the 256 / r range sums of a column
//             are then added in range order and rounded once to bf16 (the
//             sum is exact up to double rounding, as in the oracle's float64
//             sum);
//   deflate:  thread i takes channels i, i + 256, .. (CPT = KMAX / 256) and
//             removes the r directions from them, j ascending, with its L1
//             rows: cur <- fma(L1[c][j], -t_j, cur) (an exact product, one
//             rounding: the oracle's step);
//   quantize: the rotation waves read their 16 channels per lane back and
//             quantize per group (lanes l, l^1 share a group of 32; l .. l^3
//             one of 64), one code block per lane.
constexpr int kFewTokens = 64;

template <int RANK, int KMAX, bool DEFLATE>
__global__ __launch_bounds__(256) void quantize_act_rotated_few_kernel(
    const uint16_t* __restrict__ x, const float* __restrict__ inv_smooth, const uint16_t* __restrict__ L1t,
    const uint16_t* __restrict__ L1, uint8_t* __restrict__ xq, float* __restrict__ xs, uint16_t* __restrict__ t,
    int M, int K, int logB, float hscale, int group) {
  constexpr int Q = 256 / RANK;                 // channel ranges per column of t
  constexpr int CH = KMAX / Q;                  // channels per range
  constexpr int CPT = KMAX / 256;               // channels per thread in the deflation
  // LDS: bf16(x~) row [K] double | range sums [Q][RANK] double | x~ row [K] float | -t [RANK] float
  extern __shared__ double lds_raw[];
  double* xd = lds_raw;
  double* sums = xd + K;
  float* xt = reinterpret_cast<float*>(sums + Q * RANK);
  float* tn = xt + K;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = blockIdx.x;
  const int npass = (K + 1023) / 1024;
  const int e = wave * 1024 + 16 * rot_chunk(lane);   // first channel of this lane's slice before the rotation
  const bool rot_wave = wave < npass;
  const bool rot_lane = rot_wave && e < K;
  const int tj = tid % RANK;                    // column of t
  const int c0 = (tid / RANK) * CH;             // first channel of the range

  // requests: the lane's x and 1/lambda (rotation waves), the thread's L1t
  // segment and (deflated) its L1 rows, all issued unconditionally as buffer
  // loads (bytes past each array read as zero), so that the rotation waits
  // for its own two requests only and not for the L1t and L1 ones behind them
  const buf_rsrc x_rsrc = make_rsrc(x + static_cast<int64_t>(m) * K, static_cast<uint32_t>(K) * 2u);
  const buf_rsrc inv_rsrc = make_rsrc(inv_smooth, static_cast<uint32_t>(K) * 4u);
  const buf_rsrc lt_rsrc = make_rsrc(L1t, static_cast<uint32_t>(RANK * K) * 2u);
  RotFetch rf;
  rf.xa = buf_load16(x_rsrc, static_cast<uint32_t>(e) * 2u);
  rf.xb = buf_load16(x_rsrc, static_cast<uint32_t>(e) * 2u + 16u);
#pragma unroll
  for (int q = 0; q < 4; ++q)
    rf.inv[q] = __builtin_bit_cast(float4, buf_load16(inv_rsrc, static_cast<uint32_t>(e) * 4u + 16u * q));
  uint4 lt[CH / 8];
#pragma unroll
  for (int k = 0; k < CH / 8; ++k) {
    // a segment past K would read the next row: zero it (its terms are skipped too)
    const uint4 w = buf_load16(lt_rsrc, static_cast<uint32_t>(tj * K + c0 + 8 * k) * 2u);
    lt[k] = c0 + 8 * k < K ? w : make_uint4(0, 0, 0, 0);
  }
  uint32_t l1w[DEFLATE ? CPT : 1][RANK / 2];
  if constexpr (DEFLATE) {
    const buf_rsrc l1_rsrc = make_rsrc(L1, static_cast<uint32_t>(K * RANK) * 2u);
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
#pragma unroll
      for (int q = 0; q < RANK / 8; ++q) {
        const uint4 w = buf_load16(l1_rsrc, static_cast<uint32_t>((tid + 256 * i) * RANK + 8 * q) * 2u);
        l1w[i][4 * q] = w.x;
        l1w[i][4 * q + 1] = w.y;
        l1w[i][4 * q + 2] = w.z;
        l1w[i][4 * q + 3] = w.w;
      }
    }
  }

  // rotate into the LDS rows (lanes past K stay out of every block: B divides K);
  // the other waves rotate zeros and store nothing (a branch around the
  // rotation would let the compiler move the x and 1/lambda requests into it,
  // behind the L1t and L1 ones, and the rotation would wait for all of them)
  {
    float v[16];
    smooth16_regs(rf.xa, rf.xb, rf.inv, v);
    if (any_negative_zero(v)) fwht16<true>(v, lane, logB, hscale);
    else fwht16<false>(v, lane, logB, hscale);
    if (rot_lane) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int to = wave * 1024 + rot_element(lane, q, logB);
        const float4 f = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        *reinterpret_cast<float4*>(xt + to) = f;
        double2* dd = reinterpret_cast<double2*>(xd + to);
        dd[0] = make_double2(bf16_to_f32(f32_to_bf16_rne(f.x)), bf16_to_f32(f32_to_bf16_rne(f.y)));
        dd[1] = make_double2(bf16_to_f32(f32_to_bf16_rne(f.z)), bf16_to_f32(f32_to_bf16_rne(f.w)));
      }
    }
  }
  __syncthreads();

  // column tj of t over the thread's channel range, in double
  {
    // four interleaved partial sums (a quarter of the dependent chain each):
    // the products are exact in double and each sum is within ~1e-14 of the
    // exact one, so the order does not reach the single rounding to bf16
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < CH / 8; ++k) {
      if (c0 + 8 * k < K) {
        const uint32_t w[4] = {lt[k].x, lt[k].y, lt[k].z, lt[k].w};
        const double2* xp = reinterpret_cast<const double2*>(xd + c0 + 8 * k);
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const double2 a = xp[h];
          s[h] = __builtin_fma(a.x, static_cast<double>(__uint_as_float(w[h] << 16)), s[h]);
          s[h] = __builtin_fma(a.y, static_cast<double>(__uint_as_float(w[h] & 0xFFFF0000u)), s[h]);
        }
      }
    }
    sums[(tid / RANK) * RANK + tj] = (s[0] + s[1]) + (s[2] + s[3]);
  }
  __syncthreads();
  if (tid < RANK) {
    double s = 0.0;
    for (int q = 0; q < Q; ++q) s += sums[q * RANK + tid];
    const uint32_t b = f64_to_bf16_rne(s);
    t[static_cast<int64_t>(m) * RANK + tid] = static_cast<uint16_t>(b);
    tn[tid] = -bf16_to_f32(b);
  }

  if constexpr (DEFLATE) {
    __syncthreads();
    // -t and the thread's channels into registers first (the stores into xt
    // would otherwise make every read of tn wait for them); each channel
    // still takes its r updates one after another, j ascending
    float tr[RANK], v[CPT];
#pragma unroll
    for (int j = 0; j < RANK; ++j) tr[j] = tn[j];
#pragma unroll
    for (int i = 0; i < CPT; ++i) v[i] = tid + 256 * i < K ? xt[tid + 256 * i] : 0.0f;
#pragma unroll
    for (int j = 0; j < RANK; j += 2) {
#pragma unroll
      for (int i = 0; i < CPT; ++i) {
        const uint32_t w = l1w[i][j / 2];
        v[i] = __builtin_fmaf(__uint_as_float(w << 16), tr[j], v[i]);
        v[i] = __builtin_fmaf(__uint_as_float(w & 0xFFFF0000u), tr[j + 1], v[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < CPT; ++i)
      if (tid + 256 * i < K) xt[tid + 256 * i] = v[i];
    __syncthreads();
  }

  // quantize the lane's 16 channels; one code block per lane
  if (rot_wave) {
    float v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = 0.0f;
    if (rot_lane) {
      const float4* src = reinterpret_cast<const float4*>(xt + e);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 f = src[q];
        v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
      }
    }
    float amax = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; ++q) amax = __builtin_fmaxf(amax, __builtin_fabsf(v[q]));
    // lanes of one group: l, l^1 (32 channels), and l^2, l^3 (64)
    amax = __builtin_fmaxf(amax, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(amax), 0xB1, 0xF, 0xF, false)));
    if (group == kGroup)
      amax = __builtin_fmaxf(amax, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(amax), 0x4E, 0xF, 0xF, false)));
    const float sc = q4_scale(amax);
    const float inv = q4_inv(sc);
    float xs16[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) xs16[q] = v[q] * inv;
    uint32_t d0, d1, d2;
    codes_fp6_16(xs16, d0, d1, d2);
    if (rot_lane) {
      *reinterpret_cast<uint2*>(xq + static_cast<int64_t>(m) * (K / 2) + e / 2) = fp6_code_block(d0, d1, d2);
      if (e % group == 0) xs[static_cast<int64_t>(e / group) * M + m] = sc;
    }
  }
}

// LDS of a workgroup of the tile kernel: two tiles, then the partial t tiles
// (`sums`: not in the launch of the codes alone), or those over a tile buffer
// when all of it would not fit (and they fit in a tile), then -t (deflated).
constexpr size_t kLdsBytes = 160 * 1024;
struct RotLds {
  size_t tile, total;
  bool over;                    // partial t tiles over a tile buffer
};
static RotLds rotate_lds(int T, int r, bool deflate, bool sums) {
  const int nwaves = r <= 32 ? act_waves<32>() : act_waves<64>();
  RotLds l;
  l.tile = static_cast<size_t>(16) * (T + kTilePad) * sizeof(float);
  const size_t red = sums ? static_cast<size_t>(nwaves) * 16 * r * (deflate ? sizeof(double) : sizeof(float)) : 0;
  const size_t tneg = deflate ? 16 * r * sizeof(float) : 0;
  l.over = 2 * l.tile + red + tneg > kLdsBytes && red <= l.tile;
  l.total = 2 * l.tile + (l.over ? 0 : red) + tneg;
  return l;
}

// Tile width: the largest multiple of max(B, 64) that divides K, is at most
// 1024 and fits in LDS with the partial t tiles (deflated at r = 32 and 64,
// widths of 768 to 960 do not: 64 KB of double partials, larger than a tile of
// them and too large beside two; B itself, at most 512 or 1024, always fits).
static int rotate_tile_width(int K, int B, int r, bool deflate) {
  const int base = B > kGroup ? B : kGroup;
  for (int c = 1024 / base; c > 1; --c)
    if ((K / base) % c == 0 && rotate_lds(base * c, r, deflate, true).total <= kLdsBytes) return base * c;
  return base;
}

// few tokens: one workgroup per token (r = 16 up to K = 2048, r = 32 up to K = 1024)
static bool rotate_few(int M, int K, int r) { return M <= kFewTokens && (r == 16 || r == 32) && K * r <= 256 * 128; }

ActSplit rotated_split(int M, int K, int r, int B, bool deflate) {
  if (rotate_few(M, K, r)) return {0, 0};
  const int T = rotate_tile_width(K, B, r, deflate);
  return act_split(M, K, T / kGroup, kMinTiles);
}

hipError_t launch_quantize_act_rotated(int M, int K, int r, int group, int B, bool deflate, const uint16_t* x,
                                       const float* inv_smooth, const uint16_t* L1t, const uint16_t* L1f,
                                       const uint16_t* L1, uint8_t* xq, float* xs, uint16_t* t, void* workspace,
                                       hipStream_t stream) {
  int logB = 0;
  while ((1 << logB) < B) ++logB;
  if ((1 << logB) != B || B < 16 || B > 1024 || K % B != 0) return hipErrorInvalidValue;
  const int T = rotate_tile_width(K, B, r, deflate);
  // a tile has at most 16 passes / groups: per_wave<r>() per wave
  if (T / kGroup > 16) return hipErrorInvalidValue;
  const float hscale = static_cast<float>(1.0 / std::sqrt(static_cast<double>(B)));
  if (rotate_few(M, K, r)) {
    auto few = [&](auto kernel) {
      const size_t lds = static_cast<size_t>(K + 256) * sizeof(double) + static_cast<size_t>(K + r) * sizeof(float);
      hipLaunchKernelGGL(kernel, dim3(M), dim3(256), lds, stream, x, inv_smooth, L1t, L1, xq, xs, t, M, K, logB,
                         hscale, group);
      return hipGetLastError();
    };
    const int kmax = K <= 256 ? 256 : K <= 512 ? 512 : K <= 1024 ? 1024 : 2048;
#define QWAM_FEW(R, KM)                                                                             \
  if (r == R && kmax == KM)                                                                         \
    return deflate ? few(quantize_act_rotated_few_kernel<R, KM, true>)                              \
                   : few(quantize_act_rotated_few_kernel<R, KM, false>);
    QWAM_FEW(16, 256) QWAM_FEW(16, 512) QWAM_FEW(16, 1024) QWAM_FEW(16, 2048)
    QWAM_FEW(32, 256) QWAM_FEW(32, 512) QWAM_FEW(32, 1024)
#undef QWAM_FEW
  }
  const ActSplit split = workspace != nullptr ? rotated_split(M, K, r, B, deflate) : ActSplit{0, 0};
  const bool splits = split.splits > 1;
  const int tiles_per_wg = splits ? split.groups * kGroup / T : K / T;
  auto go = [&](auto kernel, int nwaves, auto* part, bool sums) {
    const RotLds l = rotate_lds(T, r, deflate, sums);
    // over a tile: the buffer the last tile does not use (the deflated
    // variant's second pass reads that tile again)
    const int last_buf = (tiles_per_wg - 1) & 1;
    const int red_off = static_cast<int>((l.over ? 1 - last_buf : 2) * l.tile / sizeof(float));
    const size_t lds = l.total;
    if (lds > kLdsBytes) return hipErrorInvalidValue;
    if (lds > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((M + 15) / 16, splits ? split.splits : 1), dim3(64 * nwaves), lds, stream, x, inv_smooth,
                       L1f, L1, xq, xs, t, splits ? part : nullptr, M, K, logB, T, tile_row_mul(T),
                       hscale, group == 32 ? 1 : 0, red_off,
                       tiles_per_wg);
    return hipGetLastError();
  };
  double* pd = static_cast<double*>(workspace);
  float* pf = static_cast<float*>(workspace);
#define QWAM_ROT_CASE(R)                                                                                            \
  case R: {                                                                                                         \
    if (!deflate) {                                                                                                 \
      const hipError_t e = go(quantize_act_rotated_kernel<R, false, Phase::kAll>, act_waves<R>(), pf, true);        \
      return e != hipSuccess || !splits ? e : launch_split_t(M, R, split.splits, pf, t, stream);                    \
    }                                                                                                               \
    if (!splits)                                                                                                    \
      return T == K ? go(quantize_act_rotated_kernel<R, true, Phase::kOneTile>, act_waves<R>(), pd, true)           \
                    : go(quantize_act_rotated_kernel<R, true, Phase::kAll>, act_waves<R>(), pd, true);              \
    const hipError_t e = go(quantize_act_rotated_kernel<R, true, Phase::kSums>, act_waves<R>(), pd, true);          \
    return e != hipSuccess ? e : go(quantize_act_rotated_kernel<R, true, Phase::kCodes>, act_waves<R>(), pd, false);  \
  }
  switch (r) {
    QWAM_ROT_CASE(16)
    QWAM_ROT_CASE(32)
    QWAM_ROT_CASE(48)
    QWAM_ROT_CASE(64)
    default:
      return hipErrorInvalidValue;
  }
#undef QWAM_ROT_CASE
}

}  // namespace qwam
