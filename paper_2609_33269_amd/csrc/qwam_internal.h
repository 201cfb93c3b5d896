// Host-side launchers of the ASP kernels (internal to libqwam).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qwam {

hipError_t launch_pack_weights(int K, int N, int group, const float* R, const float* smooth, uint8_t* wq,
                               float* ws, uint32_t* wsp, float* inv_smooth, hipStream_t stream);

// L1f: the fragment-ordered copy of L1 (qwam_layer) that the activation
// kernels' down-projection reads
hipError_t launch_quantize_act(int M, int K, int r, int group, const uint16_t* x, const float* inv_smooth,
                               const uint16_t* L1f, uint8_t* xq, float* xs, uint16_t* t, void* workspace,
                               hipStream_t stream);

// the 4-bit path quantizes the deflated activation x~ - L1 t (Eq. 8 / Eq. 9);
// L1 is [K][r] bf16 (the deflation's rows), L1t the same factor as [r][K]
hipError_t launch_quantize_act_deflated(int M, int K, int r, int group, const uint16_t* x,
                                        const float* inv_smooth, const uint16_t* L1f, const uint16_t* L1,
                                        uint8_t* xq, float* xs, uint16_t* t, void* workspace, hipStream_t stream);

// the same two activation kernels with the block Hadamard rotation of Eq. 3
// (block B, a power of two with 16 <= B <= 1024 dividing K)
hipError_t launch_quantize_act_rotated(int M, int K, int r, int group, int B, bool deflate, const uint16_t* x,
                                       const float* inv_smooth, const uint16_t* L1t, const uint16_t* L1f,
                                       const uint16_t* L1, uint8_t* xq, float* xs, uint16_t* t, void* workspace,
                                       hipStream_t stream);

// Few token blocks: K split over workgroups (`splits` of `groups` 64-channel
// groups each), their partial sums of t in a workspace of act_workspace_bytes
// (0: the call does not split); the launchers above do so when they get one.
struct ActSplit {
  int splits, groups;
};
// Split from two workgroups per block on (at most kSplitBlocks blocks), where
// K is long enough to pay for the second launch (units of four groups; tiles
// of the rotated kernels).  Graph replays, r = 32, 33 tokens, unsplit / split:
// plain K = 2048 7.4 us (kept), K = 5120 11.9 / 6.9 us, K = 14336 26.3 / 7.7
// us; deflated K = 1024 11.8 us (kept), K = 2048 20.5 / 9.5 us, K = 14336 117 /
// 14.8 us; rotated K = 2048 10.9 / 8.9 us, K = 14336 57.8 / 10.3 us; rotated and
// deflated K = 2048 27.8 / 20.2 us, K = 14336 173 / 22.2 us.  2048 tokens (two
// splits), K = 14336: 29.8 / 21.6, 119 / 68, 61 / 36 and 177 / 104 us.  As many
// splits as one round of 256 workgroups holds: 384 to 768 took 10-30% longer.
// Plain calls of 16 waves a workgroup (r <= 32) that only get two splits (above
// 1360 tokens) need a longer K: 12-13 units 9.0 / 9.8 us, 14-15 units 10.2 /
// 10.4, 16 units 11.2 / 10.8 us (of 8 waves, r = 48 and 64: 11.6 / 10.7 us at 12).
constexpr int kSplitBlocks = 128;
constexpr int kMinUnits = 12, kMinUnitsTwo = 16, kMinUnitsDeflated = 6;
constexpr int kMinTiles = 2;
int plain_min_units(int M, int r);
ActSplit act_split(int M, int K, int unit_groups, int min_units);
ActSplit rotated_split(int M, int K, int r, int B, bool deflate);
int64_t act_workspace_bytes(int M, int K, int r, int B, bool deflate);
hipError_t launch_split_t(int M, int r, int splits, const float* part, uint16_t* t, hipStream_t stream);

hipError_t launch_asp_gemm(int M, int N, int K, int r, int group, const uint8_t* xq, const float* xs,
                           const uint16_t* t, const uint8_t* wq, const float* ws, const uint32_t* wsp,
                           const uint16_t* L2t, const uint16_t* bias, uint16_t* y,
                           hipStream_t stream);

hipError_t launch_group_partials(int M, int N, int K, int group, const uint8_t* xq, const uint8_t* wq,
                                 int32_t* P, hipStream_t stream);

// AOG accumulation: A [d][d] += gT gT^T, gT bf16 [d][n], n % 64 == 0
hipError_t launch_aog_accumulate(int d, int n, const uint16_t* gT, float* A, hipStream_t stream);

// top-r eigenvectors of G~ = scale H diag(lam) A diag(lam) H by subspace
// iteration with a block of kEigBlock vectors; r <= kEigMaxRank, d % 64 == 0
constexpr int kEigBlock = 64;
constexpr int kEigMaxRank = 48;
int64_t eig_workspace_bytes(int d, int r);
hipError_t launch_aog_eig(int d, int r, int iters, const float* A, float scale, const float* lam, int B, float* V,
                          float* evals, void* workspace, hipStream_t stream);

// the few-token GEMM (one wave per 32 x 32 block), used for M <= kSmallM
constexpr int kSmallM = 64;

hipError_t launch_asp_gemm_small(int M, int N, int K, int r, int group, const uint8_t* xq, const float* xs,
                                 const uint16_t* t, const uint8_t* wq, const float* ws,
                                 const uint16_t* L2t, const uint16_t* bias, uint16_t* y,
                                 hipStream_t stream);

bool small_staged(int K);

// Forms of the GEMM for more than kSmallM tokens: 128 x 128 tiles by four
// waves, the same by eight with K in two halves, and tiles of 32 or 64 tokens
// x 64 channels with K split over the workgroup's waves (for a few hundred
// tokens)
enum class GemmForm { kLarge = 0, kLargeSplit = 1, k32x64Waves8 = 2, k32x64Waves4 = 3, k64x64Waves4 = 4 };
GemmForm gemm_form(int M, int N, int K, int group);
hipError_t launch_asp_gemm_mid(GemmForm form, int M, int N, int K, int r, int group, const uint8_t* xq,
                               const float* xs, const uint16_t* t, const uint8_t* wq, const uint32_t* wsp,
                               const uint16_t* L2t, const uint16_t* bias, uint16_t* y, hipStream_t stream);

// the whole layer for M <= kSmallM in one launch (r = 16 or 32, group 64, no
// rotation); xq / xs / t are optional outputs (all null or none)
hipError_t launch_asp_layer_small(int M, int N, int K, int r, const uint16_t* x, const float* inv_smooth,
                                  const uint16_t* L1t, const uint8_t* wq, const float* ws, const uint16_t* L2t,
                                  const uint16_t* bias, uint16_t* y, uint8_t* xq, float* xs, uint16_t* t,
                                  hipStream_t stream);

hipError_t launch_group_partials_small(int M, int N, int K, int group, const uint8_t* xq, const uint8_t* wq,
                                       int32_t* P, hipStream_t stream);

}  // namespace qwam
