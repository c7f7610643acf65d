// The convolutions of a training step on wide tiles, in fp32: the sums of
// conv_kernel, bit for bit, so that a pre-activation near 0 stays on its side
// of the activation's kink whichever kernel a layer's shape selects.  An fp32
// MFMA is a chain of fused multiply-adds in k order (checked against fmaf,
// 16x16x4 and 32x32x2 alike), so a tile shape is free as long as every output
// takes its k in conv_kernel's order: 16-deep blocks in turn and, in a block,
// k = u, 4 + u, 8 + u, 12 + u for u = 0 .. 3.
//
// A 256-thread workgroup (4 wave64, 2 x 2) owns a TM x TN tile, 64 x 64 (or
// 64 x 32, 32 x 32) per wave, on v_mfma_f32_32x32x2f32: half of conv_kernel's
// LDS traffic and address arithmetic per product, and the MFMA with the higher
// measured rate (one wave per SIMD: 151 TFLOP/s against 138 for 16x16x4).
// 32-deep slices, two LDS stages, operands straight into LDS (buffer_load ...
// lds, 16 bytes per lane; taps outside the image are loads past the extent,
// which write zeros).  What bounds it is the matrix cores; loads through
// registers and ds_write held them up (a loop of the same LDS traffic and
// MFMAs: 135 - 138 TFLOP/s through registers, 146 straight into LDS), and so
// did address arithmetic between the MFMAs.  Measured, 16 cells x 128 images,
// 137 GFLOP per launch: D's 128 -> 256 convolution 1391 us on conv_kernel, 1073
// here (128 TFLOP/s); its input gradient and weight gradient 2717 us in one
// launch of conv_kernel, 1047 + 1065 here.
#include <hip/hip_ext.h>

#include "conv_wide_tile.h"

namespace lipz {

namespace {

template <int TM, int TN, int MODE, int BT, bool TAP1>
__global__ __launch_bounds__(NT, 2) void conv_wide_kernel(const ConvProb* __restrict__ probs, ConvGroups grp,
                                                          float slope) {
  __shared__ __align__(16) float stage0[STAGE_FLOATS<TM, TN>];
  __shared__ __align__(16) float stage1[STAGE_FLOATS<TM, TN>];
  const int b = blockIdx.x;
  int gi = 0;
#pragma unroll
  for (int q = 1; q < GEMM_MAX_GROUPS; ++q)
    if (q < grp.n && b >= grp.first_block[q]) gi = q;
  // first_block is a multiple of 8, so (b - first_block) % 8 is still the XCD
  const int rel = xcd_remap(b - grp.first_block[gi], grp.blocks[gi]);
  if (rel >= grp.real_tiles[gi]) return;
  const ConvProb P = probs[grp.first_prob[gi] + rel / grp.tiles_per_prob[gi]];
  const int lt = rel % grp.tiles_per_prob[gi];
  const int tiles_mn = P.tiles_m * P.tiles_n;
  const int split = lt / tiles_mn;
  const int rem = lt - split * tiles_mn;
  const int m0 = (rem / P.tiles_n) * TM, n0 = (rem % P.tiles_n) * TN;
  int kbeg = 0, kend = P.K;
  if (MODE == CONV_WG) {
    kbeg = split * P.ksplit;
    kend = min(P.K, kbeg + P.ksplit);
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  wide_tile<TM, TN, MODE, BT, TAP1>(P, m0, n0, split, kbeg, kend, slope, wave, stage0, stage1);
}

}  // namespace

hipError_t launch_conv_wide(const ConvProb* d_probs, const ConvGroups& grp, int total_blocks, const ConvVariant& v,
                            float slope, hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (grp.n <= 0 || total_blocks <= 0) return hipSuccess;
#define LIPZ_CW(TM, TN, MODE, BT, T1)                                                                           \
  hipExtLaunchKernelGGL((conv_wide_kernel<TM, TN, MODE, BT, T1>), dim3(total_blocks), dim3(NT), 0, s, ev_start, \
                        ev_stop, 0, d_probs, grp, slope)
#define LIPZ_CW_MODE(TM, TN)                                   \
  if (v.mode == CONV_WG) LIPZ_CW(TM, TN, CONV_WG, 0, false);   \
  else if (v.bt && v.tap1) LIPZ_CW(TM, TN, CONV_FWD, 1, true); \
  else if (v.bt) LIPZ_CW(TM, TN, CONV_FWD, 1, false);          \
  else if (v.tap1) LIPZ_CW(TM, TN, CONV_FWD, 0, true);         \
  else LIPZ_CW(TM, TN, CONV_FWD, 0, false)
  if (v.tm == 128 && v.tn == 128) { LIPZ_CW_MODE(128, 128); }
  else if (v.tm == 128 && v.tn == 64) { LIPZ_CW_MODE(128, 64); }
  else if (v.tm == 64 && v.tn == 64) { LIPZ_CW_MODE(64, 64); }
  else return hipErrorInvalidValue;
#undef LIPZ_CW_MODE
#undef LIPZ_CW
  return hipGetLastError();
}

}  // namespace lipz
