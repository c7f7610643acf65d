// Grouped fp32 GEMM on CDNA4 matrix cores (v_mfma_f32_16x16x4f32) with fused
// epilogues.  One launch computes every (cell, slot) problem of one dependent
// phase of a generation: each cell's networks are small (M = 100..600 rows,
// K = 64..784), so they are only worth a GPU when all of them run side by side.
// Problems of one launch are described in device memory (GemmProb) and grouped
// by shape and depth (GemmGroups, passed as scalar kernel arguments that the
// hardware preloads); blockIdx is remapped so that each group is split into
// eight contiguous shares, one per XCD: the tiles of one problem share an L2
// and the long tiles of a launch are spread over every XCD.
//
// Stores: a template parameter WT selects device-scope (write-through) buffer
// stores for the epilogues' outputs, or write-back; the library picks one per
// grid, by the size of its state.
//
// Tiling: a 256-thread workgroup (4 wave64) owns a BM x 64 output tile; wave w
// owns the (BM / 2) x 32 block (w / 2, w % 2).  BM = 64: one MFMA 32 x 32 x 2
// block per wave; BM = 32: two 16 x 16 x 4 blocks.
//
// Main loop: 32-deep K slices in two LDS stages, filled by buffer_load ... lds
// (16 bytes per lane, straight into LDS) one slice ahead; one barrier per
// slice.  A slice's loads need no vector instruction: lanes keep fixed
// offsets, and the buffer resource's base and extent advance in scalar
// registers.  Nothing is asked of the alignment of rows (a dword-aligned
// 16-byte load reads the same bytes) or of the sizes: dwords past an operand's
// extent are zeros in LDS.
//
// Order of sums: MFMAs are chains of fused multiply-adds in k order.  An output
// takes 16-deep k blocks in turn and, in a block, k = u, 4 + u, 8 + u, 12 + u
// for u = 0 .. 3.  CH = 4 keeps four such chains, of the k blocks 0, 1, 2, 3
// (mod 4), and adds them at the end, (0 + 1) + (2 + 3).
//
// Before the epilogue every wave passes its block through LDS, so that a lane
// holds four consecutive columns and eight lanes a row's 32: C, the Adam
// moments and the auxiliary operand move in full 128-byte lines, 16 bytes per
// lane.
//
// Epilogues: plain store; bias + activation (forward), optionally with the
// tile's partial dot product against a 1-wide output layer; activation
// derivative (input gradient); Adam on the weight gradient in registers.  What
// an epilogue reads is requested before the main loop.
//
// What bounds it: on large phases the matrix cores are 70 % busy, while the
// tiles' operands come out of L2 at about 9 TB/s (a 32 x 64 tile takes 96 floats
// per k for 2048 products); which of the waits between holds them up is not
// shown (64-row tiles move a third less and gain 4 - 8 %, on the largest
// products only).  Phases of a tile or two per CU are bound by the launch and
// the chain of a tile's slices; weight gradients with Adam by the 24 bytes per
// parameter and the vector instructions of its divisions.  Measured, against
// operands staged through registers and element-wise epilogues: 16 cells'
// 784 -> 256 weight gradient with Adam (200 samples) and its neighbour 41.1 ->
// 36.4 us; 32 cells' 81 -> 68; a forward of 600 rows, 256 -> 256, for 80
// pairs 83.6 -> 77.4 us; and against element-wise loads of rows that are not
// 16-byte aligned, six cells of 301 -> 203 -> 97 units: 1960 -> 1100 us for 10
// steps.  64-row tiles were no faster on phases of 256 to 8960 tiles of 32
// rows, four LDS stages neither.  Larger single products do run faster on them
// (LIPZ_GEMM_TILE64_MIN).
#include <string.h>

#include <hip/hip_ext.h>

#include "lipz_internal.h"

namespace lipz {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

namespace {

#ifndef LIPZ_GEMM_TILE64_MIN
// Phases with at least this many 64 x 64 tiles (outputs of 1.6 GB) use 64-row
// tiles: one product of 102400 of them, time against 32-row tiles: K = 32 0.75 -
// 0.89, 64 0.87 - 0.92, 128 0.92 - 0.96, 256 0.94 - 0.96, 384 0.93 - 0.96.  The line
// is not where they begin to gain: products of 8192 to 65536 tiles have the
// same ratios, grouped phases of that size were not measured.
#define LIPZ_GEMM_TILE64_MIN 100000
#endif
#ifndef LIPZ_GEMM_CHAINS4_MIN_K
#define LIPZ_GEMM_CHAINS4_MIN_K 512  // phases of aligned problems at least this deep sum in four chains
#endif
#ifndef LIPZ_GEMM_WAVE_MAX_TILES
// ... on the wave-split kernel up to this many tiles (two per CU: 512 tiles of
// K = 784 take 20.3 us there and 21.1 on the other, 672 take 27.8 and 21.7)
#define LIPZ_GEMM_WAVE_MAX_TILES 512
#endif
#ifndef LIPZ_GEMM_WAVE_MIN_K
// ... and from this depth on at any number of tiles, where no problem reads B
// transposed: one product of 256 columns, K = 4096, 520 to 4096 tiles: 0.94 -
// 0.96 of the other kernel's time, 8960 tiles 1.00; of 2048 columns, 4096 to
// 32768 tiles 0.94 - 0.97; K = 8192 0.92 - 0.98.  At K = 2048 the two are even
// (0.97 - 1.11), at K = 784 it takes 1.05 - 1.15, and with B transposed 1.2 - 1.4
// at every depth (its columns are rows there, K apart).
#define LIPZ_GEMM_WAVE_MIN_K 4096
#endif

constexpr int BN = GEMM_BN;
constexpr int BK = 32;        // K depth of an LDS stage
constexpr int NT = 256;
constexpr uint32_t FAR = 0x80000000u;  // an offset past every extent

template <int BM>
struct Tile {
  static constexpr int WM = BM / 2;   // rows per wave
  static constexpr int NQ = WM / 8;   // epilogue passes of 8 rows
  static constexpr int NA = BM / 32, NB = 2, NL = NA + NB;  // 1024-byte loads of a slice per wave
  static constexpr int A_FLOATS = BM * BK, FLOATS = (BM + BN) * BK;
};

typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  // dword 3 = 0x00020000: raw 32-bit data format on gfx9-family parts
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)bytes, 0x00020000);
}

// Elements through a buffer resource: the epilogues address C, the Adam
// moments and the auxiliary operand with 32-bit element offsets from the
// descriptor's base (no 64-bit address per element).
//
// Store policy (WT, a template parameter of the kernels, chosen per grid).
// With WT the epilogues' element stores (outputs, Adam's p, m, v), the head
// partials and the minibatch rows are device-scope stores (cache policy
// sc1): written through the XCD's L2 towards memory, so that the next
// dependent launch, which reads them from whichever XCD its tiles run on,
// does not wait for an end-of-kernel writeback of dirty L2 lines.  Without
// it they are write-back stores.  (The folded loss head's per-row side
// outputs and partial dot products are write-back stores in either case.)
constexpr uint32_t kWholeBuffer = 0x7FFFFFFFu;  // element offsets of a problem stay below 2^31 (planning checks)
constexpr int kStoreDevice = 16;                // buffer-store cache policy: sc1 (device scope)
__device__ __forceinline__ float bld1(__amdgpu_buffer_rsrc_t r, uint32_t off_elems) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)(off_elems * 4u), 0, 0));
}
template <bool WT>
__device__ __forceinline__ void bst1(__amdgpu_buffer_rsrc_t r, uint32_t off_elems, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)(off_elems * 4u), 0, WT ? kStoreDevice : 0);
}

// Four elements in a row.  A load of the last row's end may run past the row;
// the resource's extent bounds it (zeros).  A store writes the first n.
__device__ __forceinline__ v4f bld4(__amdgpu_buffer_rsrc_t r, uint32_t off_elems) {
  return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(off_elems * 4u), 0, 0));
}
template <bool WT>
__device__ __forceinline__ void bst4(__amdgpu_buffer_rsrc_t r, uint32_t off_elems, int n, v4f v) {
  if (n >= 4) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), r, (int)(off_elems * 4u), 0,
                                           WT ? kStoreDevice : 0);
  } else {
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (u < n) bst1<WT>(r, off_elems + u, v[u]);
  }
}

// The loss head's dL/da of a row, from its partial logits, formed as the
// separate head kernel forms it.  With four partial sums per row (a 129..256-
// wide last hidden layer) the row's load is issued together with the
// epilogue's other loads.
__device__ __forceinline__ float head_row_dl(const GemmProb& P, int row) {
  const LIPZ_GLOBAL float* pr = as_global(P.rs_part) + (size_t)(row < P.M ? row : 0) * P.rs_tn;
  float a;
  if (P.rs_tn == 4) {
    const v4f v = *reinterpret_cast<const LIPZ_GLOBAL v4f*>(pr);
    a = ((v[0] + v[1]) + v[2]) + v[3];
  } else {
    a = 0.f;
    for (int t = 0; t < P.rs_tn; ++t) a += pr[t];
  }
  return head_dl(P.loss_kind, a, P.rs_mode == 2 || row < P.rs_B, 1.f / (float)P.rs_B);
}

// Workgroup q of a sampling job: SAMPLE_ROWS minibatch rows of one unit,
// drawn exactly as sample_kernel draws them.
template <bool WT>
__device__ __forceinline__ void sample_rows(const SampleJob& sj, int q) {
  const int per = (sj.B + SAMPLE_ROWS - 1) / SAMPLE_ROWS;
  const int u = sj.u0 + q / per, b0 = (q % per) * SAMPLE_ROWS;
  const int nr = sj.B - b0 < SAMPLE_ROWS ? sj.B - b0 : SAMPLE_ROWS;
  const int tid = threadIdx.x;
  for (int rr = 0; rr < nr; ++rr) {
    const int b = b0 + rr;
    const uint4 wi = stream_block(sj.key, (uint32_t)(b >> 2), (uint32_t)u, sj.gen, sj.sf, LIPZ_TAG_IDX);
    const int64_t row = (int64_t)(((uint64_t)word_of(wi, b & 3) * (uint64_t)sj.N) >> 32);
    const float* src = sj.data + row * sj.xd;
    const __amdgpu_buffer_rsrc_t rd = make_rsrc(sj.X + u * sj.x_stride + (int64_t)b * sj.xd, kWholeBuffer);
    if ((sj.xd & 3) == 0) {
      for (int k = tid; k < (sj.xd >> 2); k += NT) {
        const float4 v = reinterpret_cast<const float4*>(src)[k];
        __builtin_amdgcn_raw_buffer_store_b128(
            v4u{__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)}, rd,
            k * 16, 0, WT ? kStoreDevice : 0);
      }
    } else {
      for (int k = tid; k < sj.xd; k += NT) bst1<WT>(rd, (uint32_t)k, src[k]);
    }
  }
  const __amdgpu_buffer_rsrc_t rz = make_rsrc(sj.Z + u * sj.z_stride + (int64_t)b0 * sj.zd, kWholeBuffer);
  for (int k = tid; k < nr * sj.zd; k += NT) {
    const int64_t e = (int64_t)b0 * sj.zd + k;
    const uint4 w = stream_block(sj.key, (uint32_t)(e >> 2), (uint32_t)u, sj.gen, sj.sf, LIPZ_TAG_Z);
    bst1<WT>(rz, (uint32_t)k, (float)normal_of(w, (int)(e & 3)));
  }
}

// The output layer's weight gradient of the discriminator step, in pieces of
// 32 rows: column sums of dL/da[i] * hsrc[i][j] over a piece's rows (and, in
// column 0, of dL/da[i]), summed over 16 rows' lane groups and then over the
// two 16-row halves, in a fixed order.  Rows past M and columns past hp_w add
// nothing.  dlr[q]: dL/da of row 8 q + lane / 8 of the wave's.
template <int BM, bool WT>
__device__ __forceinline__ void head_partials(const GemmProb& P, const float (&dlr)[Tile<BM>::NQ], int m0, int n0,
                                              int tile_n, float (*red)[BM]) {
  using T = Tile<BM>;
  constexpr int H = T::WM / 16;  // 16-row halves of a piece in the wave
  __shared__ float dsum;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * T::WM, wn = (wave & 1) * 32;
  const int li = lane & 15, lg = lane >> 4;
  const bool wgan = P.loss_kind == LIPZ_LOSS_WASSERSTEIN;
  const __amdgpu_buffer_rsrc_t rH = make_rsrc(P.hsrc, kWholeBuffer);
  float hv[H][2][4];
#pragma unroll
  for (int i = 0; i < H; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm + 16 * i + 4 * lg + r, col = n0 + wn + 16 * j + li;
        const bool in = row < P.M && col < P.hp_w;
        const float x = bld1(rH, in ? (uint32_t)(row * P.hp_w + col) : 0u);
        hv[i][j][r] = in ? x : 0.f;
      }
  float cs[H][2] = {}, ds[H] = {};
#pragma unroll
  for (int i = 0; i < H; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = m0 + wm + 16 * i + 4 * lg + r;
      const int src = ((4 * lg + r) & 7) * 8;
      const float d0 = __shfl(dlr[2 * i], src, 64), d1 = __shfl(dlr[2 * i + 1], src, 64);
      const float d = row < P.M ? (wgan ? (row < P.rs_B ? -1.f : 1.f) : (lg >= 2 ? d1 : d0)) : 0.f;
      ds[i] += d;
#pragma unroll
      for (int j = 0; j < 2; ++j) cs[i][j] = fmaf(d, hv[i][j][r], cs[i][j]);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      cs[i][j] += __shfl_xor(cs[i][j], 16, 64);
      cs[i][j] += __shfl_xor(cs[i][j], 32, 64);
    }
    ds[i] += __shfl_xor(ds[i], 16, 64);
    ds[i] += __shfl_xor(ds[i], 32, 64);
  }
  float c2[2], d2 = 0.f;  // the second halves' sums
  if (H == 2) {
    c2[0] = cs[H - 1][0];
    c2[1] = cs[H - 1][1];
    d2 = ds[H - 1];
  } else {
    if (wm != 0 && lane < 16) {
      red[wave & 1][li] = cs[0][0];
      red[wave & 1][16 + li] = cs[0][1];
      if (wn == 0 && lane == 0) dsum = ds[0];
    }
    __syncthreads();
    c2[0] = red[wave & 1][li];
    c2[1] = red[wave & 1][16 + li];
    d2 = dsum;
    if (wm != 0) return;
  }
  if (lane >= 16 || m0 + wm >= P.M) return;
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(P.hpart + (size_t)((m0 + wm) / 32) * P.hp_ld, kWholeBuffer);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = n0 + wn + 16 * j + li;
    if (col < P.hp_w) bst1<WT>(ro, (uint32_t)col, cs[0][j] + c2[j]);
  }
  if (tile_n == 0 && wn == 0 && lane == 0) bst1<WT>(ro, (uint32_t)P.hp_w, ds[0] + d2);
}

// Kernel arguments.  The descriptor pointer, the
// tile groups of the launch and the step index come first, as 14 scalar
// words that the hardware preloads into scalar registers (the library is
// built with -mllvm -amdgpu-kernarg-preload-count=14), so that a GEMM
// workgroup's first memory access is its problem descriptor; only the
// sampling workgroups read their SampleJob from kernel-argument memory.
// Group q of the launch: tiles first_tile[q] .. (first_tile[q + 1] or
// total) - 1, problems first_prob[q] on, tiles_per_prob[q] tiles each;
// first_tile[0] = first_prob[0] = 0, and a group past the launch's last one
// has first_tile = total.
#define LIPZ_GEMM_ARGS                                                                              \
  const GemmProb *__restrict__ probs, int32_t g_total, int32_t g_ft1, int32_t g_ft2, int32_t g_ft3, \
      int32_t g_fp1, int32_t g_fp2, int32_t g_fp3, int32_t g_tp0, int32_t g_tp1, int32_t g_tp2,     \
      int32_t g_tp3, int32_t step_local, SampleJob sj
#define LIPZ_GEMM_GROUPS g_total, g_ft1, g_ft2, g_ft3, g_fp1, g_fp2, g_fp3, g_tp0, g_tp1, g_tp2, g_tp3

// This workgroup's problem (index pi into the launch's descriptors) and tile
// of it (lt), from the XCD-balanced block-to-tile map.  No array is indexed
// at run time, so the groups stay in scalar registers.
__device__ __forceinline__ void locate_tile(int total, int ft1, int ft2, int ft3, int fp1, int fp2, int fp3, int tp0,
                                            int tp1, int tp2, int tp3, int& pi, int& lt) {
  GemmGroups grp;
  grp.n = 1 + (ft1 < total) + (ft2 < total) + (ft3 < total);
  grp.total = total;
  grp.first_tile[0] = 0;
  grp.first_tile[1] = ft1;
  grp.first_tile[2] = ft2;
  grp.first_tile[3] = ft3;
  const int t = xcd_group_tile(blockIdx.x, total, grp);
  int ft = 0, fp = 0, tp = tp0;
  if (t >= ft1) ft = ft1, fp = fp1, tp = tp1;
  if (t >= ft2) ft = ft2, fp = fp2, tp = tp2;
  if (t >= ft3) ft = ft3, fp = fp3, tp = tp3;
  pi = fp + (t - ft) / tp;
  lt = (t - ft) % tp;
}

// A lane's share of the epilogue: pass q takes row row0 + 8 q, columns col ..
// col + 3, of which n lie inside C.
template <int BM>
struct EpiPos {
  int row0, col, n;
  uint32_t c_bytes;  // extent of C
  __device__ __forceinline__ EpiPos(const GemmProb& P, int m0, int n0) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    row0 = m0 + (wave >> 1) * Tile<BM>::WM + (lane >> 3);
    col = n0 + (wave & 1) * 32 + 4 * (lane & 7);
    n = P.N - col;
    c_bytes = ((uint32_t)(P.M - 1) * (uint32_t)P.ldc + (uint32_t)P.N) * 4u;
  }
  __device__ __forceinline__ bool ok(const GemmProb& P, int q) const { return row0 + 8 * q < P.M && n > 0; }
  __device__ __forceinline__ uint32_t off(const GemmProb& P, int q) const {
    return ok(P, q) ? (uint32_t)((row0 + 8 * q) * P.ldc + col) : 0u;
  }
};

// What a lane's epilogue reads, requested before the main loop: the operands'
// first slices come behind it, so its latency is hidden.
template <int BM>
struct EpiIn {
  v4f x[Tile<BM>::NQ];  // EPI_ADAM: p; EPI_DACT: aux
  v4f m[Tile<BM>::NQ], v[Tile<BM>::NQ];
};

template <int BM>
__device__ __forceinline__ void epi_load(const GemmProb& P, const EpiPos<BM>& E, EpiIn<BM>& in) {
  const bool adam = P.epi == EPI_ADAM;
  if (!adam && P.epi != EPI_DACT) return;
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(adam ? P.C : P.aux, E.c_bytes);
#pragma unroll
  for (int q = 0; q < Tile<BM>::NQ; ++q) in.x[q] = bld4(rx, E.off(P, q));
  if (!adam) return;
  const __amdgpu_buffer_rsrc_t rm = make_rsrc(P.m, E.c_bytes), rv = make_rsrc(P.v, E.c_bytes);
#pragma unroll
  for (int q = 0; q < Tile<BM>::NQ; ++q) {
    in.m[q] = bld4(rm, E.off(P, q));
    in.v[q] = bld4(rv, E.off(P, q));
  }
}

// Adam's update of the lane's elements.  The moments' sums b1 m + (1 - b1) g
// (and v's) are fused one way or the other: OLD_FIRST rounds the old moment's
// product first, else the gradient's.  Which is GemmProb::vec's to say: a
// network of given sizes trains to the same bits whichever kernel runs it.
//
// Where it can, with the divisions and the square root without the scaling and special
// cases of their IEEE sequences (LLVM's for this target: a reciprocal refined once, the
// quotient twice; a square root moved by an ulp where its residuals say so), for
// operands in the range where those do nothing: the same bits in 35 vector
// instructions per element instead of 58 (a training step of 16 MNIST cells:
// 191 us without, 188 with; of four 2-D cells 69 and 66).
__device__ __forceinline__ float refined_rcp(float d) {
  const float y = __builtin_amdgcn_rcpf(d);
  return fmaf(fmaf(-d, y, 1.f), y, y);
}
__device__ __forceinline__ float div_by(float n, float d, float y) {  // y = refined_rcp(d)
  float q = n * y;
  q = fmaf(fmaf(-d, q, n), y, q);
  return fmaf(fmaf(-d, q, n), y, q);
}
__device__ __forceinline__ float root(float x) {
  const float s = __builtin_amdgcn_sqrtf(x);
  const float lo = __uint_as_float(__float_as_uint(s) - 1u), hi = __uint_as_float(__float_as_uint(s) + 1u);
  const float r = fmaf(-lo, s, x) <= 0.f ? lo : s;
  return fmaf(-hi, s, x) > 0.f ? hi : r;
}
// +0, or of magnitude 2^lo .. 2^hi: of the bits with the sign moved to the low
// end, the smallest of bits - 1 (+0 wraps to the largest, -0 is the smallest)
// and the largest.  -0 stays with the full sequences: its short quotient is +0,
// which takes the sign off a parameter of -0.
struct Range {
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
  __device__ __forceinline__ void take(float v) {
    const uint32_t b = __builtin_rotateleft32(__float_as_uint(v), 1);
    lo = min(lo, b - 1u);
    hi = max(hi, b);
  }
  __device__ __forceinline__ bool inside(int lo_exp, int hi_exp) const {
    return lo >= ((uint32_t)(127 + lo_exp) << 24) - 1u && hi <= ((uint32_t)(127 + hi_exp) << 24) + 1u;
  }
};

template <int BM, bool WT, bool OLD_FIRST>
__device__ __forceinline__ void adam(const GemmProb& P, const v4f (&acc)[Tile<BM>::NQ], const EpiPos<BM>& E,
                                     const EpiIn<BM>& in, const float* bc) {
  const AdamConsts& ac = P.ac;
  const __amdgpu_buffer_rsrc_t rC = make_rsrc(P.C, kWholeBuffer);
  const __amdgpu_buffer_rsrc_t rM = make_rsrc(P.m, kWholeBuffer);
  const __amdgpu_buffer_rsrc_t rV = make_rsrc(P.v, kWholeBuffer);
  const float lr = *as_global(P.lr);
  const float bc1 = bc[0], bc2 = bc[1];
  // with these and m, v in the ranges below every quotient, root and reciprocal
  // is a normal number (or 0), about 2^-120 at least.  The residuals need not be: of a
  // numerator of 2^-100 they go down to 2^-147.  They are exact all the same,
  // multiples of 2^-149, as long as subnormal numbers are kept (the target's
  // default for fp32).
  const bool plain = lr >= 0x1p-20f && lr <= 1.f && bc1 >= 0x1p-20f && bc2 >= 0x1p-20f && ac.eps >= 0x1p-30f && ac.eps <= 1.f;
  const float y1 = refined_rcp(bc1), y2 = refined_rcp(bc2);
#pragma unroll
  for (int q = 0; q < Tile<BM>::NQ; ++q) {
    v4f pn, mn, vn;
    Range rm, rv;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float g = P.gscale != 0.f ? acc[q][r] * P.gscale : acc[q][r];
      const float g2 = ac.one_minus_beta2 * g;
      mn[r] = OLD_FIRST ? fmaf(ac.one_minus_beta1, g, ac.beta1 * in.m[q][r])
                        : fmaf(ac.beta1, in.m[q][r], ac.one_minus_beta1 * g);
      vn[r] = OLD_FIRST ? fmaf(g2, g, ac.beta2 * in.v[q][r]) : fmaf(ac.beta2, in.v[q][r], g2 * g);
      rm.take(mn[r]);
      rv.take(vn[r]);
    }
    if (__all(plain && rm.inside(-80, 20) && rv.inside(-100, 20))) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float den = root(div_by(vn[r], bc2, y2)) + ac.eps;
        pn[r] = in.x[q][r] - div_by(lr * div_by(mn[r], bc1, y1), den, refined_rcp(den));
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        pn[r] = in.x[q][r] - lr * (mn[r] / bc1) / (sqrtf(vn[r] / bc2) + ac.eps);
    }
    if (P.clip > 0.f) {
#pragma unroll
      for (int r = 0; r < 4; ++r) pn[r] = pn[r] > P.clip ? P.clip : (pn[r] < -P.clip ? -P.clip : pn[r]);  // keeps NaN
    }
    if (E.ok(P, q)) {
      const uint32_t o = E.off(P, q);
      bst4<WT>(rM, o, E.n, mn);
      bst4<WT>(rV, o, E.n, vn);
      bst4<WT>(rC, o, E.n, pn);
    }
  }
}

// Bias + activation (optionally with the per-tile partial dot product of the
// next 1-wide layer), the activation-derivative product, or the fused Adam
// update; then stores.  bc: Adam's bias corrections of this step (in LDS,
// written before the main loop's first barrier).
template <int BM, bool WT>
__device__ __forceinline__ void epilogue(const GemmProb& P, const v4f (&acc)[Tile<BM>::NQ], const EpiPos<BM>& E,
                                         const EpiIn<BM>& in, int m0, int n0, int tile_n, const float* bc,
                                         float (*red)[BM]) {
  using T = Tile<BM>;
  typedef v4f v4f_any __attribute__((aligned(4)));
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * T::WM, wn = (wave & 1) * 32;
  const float slope = P.slope;
  const __amdgpu_buffer_rsrc_t rC = make_rsrc(P.C, kWholeBuffer);
  if (P.epi == EPI_ADAM) {
    if (P.vec & GEMM_ADAM_OLD_FIRST) adam<BM, WT, true>(P, acc, E, in, bc);
    else adam<BM, WT, false>(P, acc, E, in, bc);
    return;
  }
  if (P.epi == EPI_DACT) {
    float dl[T::NQ];
    if (P.rs_mode != 0) {
#pragma unroll
      for (int q = 0; q < T::NQ; ++q) dl[q] = head_row_dl(P, E.row0 + 8 * q);
    }
    LIPZ_GLOBAL float* gSide = as_global(P.side);
#pragma unroll
    for (int q = 0; q < T::NQ; ++q) {
      v4f y;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        y[r] = acc[q][r] * act_deriv_from_out(P.act, in.x[q][r], slope);
        if (P.rs_mode != 0) y[r] = dl[q] * y[r];
      }
      if (!E.ok(P, q)) continue;
      bst4<WT>(rC, E.off(P, q), E.n, y);
      if (P.rs_mode != 0 && P.side) {
        LIPZ_GLOBAL float* o = gSide + (size_t)(E.row0 + 8 * q) * P.side_ld + E.col;
        if (E.n >= 4) {
          *reinterpret_cast<LIPZ_GLOBAL v4f_any*>(o) = dl[q] * in.x[q];
        } else {
          for (int r = 0; r < E.n; ++r) o[r] = dl[q] * (r == 0 ? in.x[q][0] : r == 1 ? in.x[q][1] : in.x[q][2]);
        }
      }
    }
    if (P.rs_mode == 0) return;
    if (P.rs_mode == 1 && P.hpart) head_partials<BM, WT>(P, dl, m0, n0, tile_n, red);
    // column 0 of the problem: the per-row extras
    if (P.side && tile_n == 0 && wn == 0 && (lane & 7) == 0) {
      LIPZ_GLOBAL float* gDl = as_global(P.dlout);
#pragma unroll
      for (int q = 0; q < T::NQ; ++q) {
        const int row = E.row0 + 8 * q;
        if (row < P.M) {
          LIPZ_GLOBAL float* sr = gSide + (size_t)row * P.side_ld + P.N;
          sr[0] = dl[q];
          sr[1] = 0.f;
          sr[2] = 0.f;
          sr[3] = 0.f;
          LIPZ_GLOBAL float* o = gDl + (size_t)row * 4;
          o[0] = P.loss_kind == LIPZ_LOSS_WASSERSTEIN ? (row < P.rs_B ? -1.f : 1.f) : dl[q];
          o[1] = 0.f;
          o[2] = 0.f;
          o[3] = 0.f;
        }
      }
    }
    return;
  }
  if (P.epi != EPI_BIAS_ACT) {
#pragma unroll
    for (int q = 0; q < T::NQ; ++q)
      if (E.ok(P, q)) bst4<WT>(rC, E.off(P, q), E.n, acc[q]);
    return;
  }
  // bias + activation, optional partial dot product with the next layer's weights
  const bool dot = P.dot_out != nullptr;
  const uint32_t c0 = E.n > 0 ? (uint32_t)E.col : 0u, nbytes = (uint32_t)P.N * 4u;
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  const v4f bias = P.bias ? bld4(make_rsrc(P.bias, nbytes), c0) : zero;
  const v4f dw = dot ? bld4(make_rsrc(P.dotw, nbytes), c0) : zero;
#pragma unroll
  for (int q = 0; q < T::NQ; ++q) {
    v4f y;
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = act_fwd(P.act, acc[q][r] + bias[r], slope);
    if (E.ok(P, q)) {
      bst4<WT>(rC, E.off(P, q), E.n, y);
      if (dot && P.gout) {
        v4f gy;
#pragma unroll
        for (int r = 0; r < 4; ++r) gy[r] = dw[r] * act_deriv_from_out(P.act, y[r], slope);
        bst4<WT>(make_rsrc(P.gout, kWholeBuffer), E.off(P, q), E.n, gy);
      }
    }
    if (dot) {
      // a row's 32 columns: column c + 16's product onto column c's, then a
      // tree over the 16; then the two column halves of the tile (waves wn =
      // 0 and 32), in a fixed order
      float s[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float t = E.ok(P, q) && r < E.n ? y[r] * dw[r] : 0.f;
        const float low = __shfl_xor(t, 4, 64);
        s[r] = E.ok(P, q) && r < E.n ? fmaf(y[r], dw[r], low) : low;
      }
      float v = (s[0] + s[1]) + (s[2] + s[3]);
      v += __shfl_xor(v, 1, 64);
      v += __shfl_xor(v, 2, 64);
      if ((lane & 7) == 4) red[wave & 1][wm + 8 * q + (lane >> 3)] = v;
    }
  }
  if (dot) {
    __syncthreads();
    const float b = (tile_n == 0 && P.dot_bias) ? *as_global(P.dot_bias) : 0.f;
    for (int r = tid; r < BM; r += NT) {
      const int row = m0 + r;
      if (row < P.M) as_global(P.dot_out)[(size_t)row * P.dot_ld + tile_n] = (red[0][r] + red[1][r]) + b;
    }
  }
}

// LDS stage of an operand slice (32 k), as the loads write it: 64 lanes x 16
// bytes in a row per instruction, 16-byte chunk q = 64 (4 c + wave) + lane.
//
// Rows of k (A [M][K], B [N][K]): row r is chunks 8 r .. 8 r + 7, its k quad x
// at place x ^ (r % 8).
// k rows of 64 columns (B [K][N], A [K][M] with BM = 64): row k is chunks 16 k
// .. 16 k + 15, column quad x at place x ^ 8 ((k / 4) % 2) (BM = 64) or x ^ 4
// ((k / 4) % 4) (BM = 32).
// k rows of 32 columns (A [K][M] with BM = 32): row k at chunk row s = 2 (k % 4)
// + (k / 4) % 2 + 8 (k / 8), column quad x at place x ^ 4 ((k / 8) % 2).
// The lane groups of a fragment read then lie on different banks.
template <int BM, int W, bool ROWS>
struct Opnd {
  static constexpr int N = W / 32;  // loads of a slice per wave
  const char* base;                 // the next slice
  int64_t step;                     // bytes per slice
  int bytes;                        // ROWS: extent from base; else the columns before r0, in bytes
  uint32_t row;                     // a row, in bytes
  uint32_t off[N];                  // of the lane's chunks, from base
  int k4;                           // ROWS: first k of the lane's chunks in the slice (the same in all of them)
  __device__ __forceinline__ void init(const float* p, int rows, int ld, int r0, int wave, int lane) {
    // ROWS: rows r0 .. of [rows][ld]; else columns r0 .. of [K][ld]
    base = (const char*)(p + (ROWS ? (int64_t)r0 * ld : (int64_t)r0));
    step = ROWS ? BK * 4 : (int64_t)ld * (BK * 4);
    row = (uint32_t)ld * 4u;
    bytes = ROWS ? min(max(rows - r0, 0), W) * (int)row : r0 * 4;
    k4 = 4 * ((lane & 7) ^ ((lane >> 3) & 7));
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const int q = 64 * (4 * c + wave) + lane;
      if (ROWS) {
        off[c] = (uint32_t)((q >> 3) * ld + k4) * 4u;
      } else if (W == 64) {
        const int k = q >> 4, x = (q & 15) ^ (BM == 64 ? (k & 4) << 1 : k & 12);
        off[c] = (uint32_t)(k * ld + 4 * x) * 4u;
      } else {
        const int s = q >> 3, k = (s & 24) | ((s >> 1) & 3) | ((s & 1) << 2), x = (q & 7) ^ ((k >> 1) & 4);
        off[c] = (uint32_t)(k * ld + 4 * x) * 4u;
      }
    }
  }
  // Loads the next slice; kleft: k left from its first one.
  __device__ __forceinline__ void load(float* st, int wave, int kleft) {
    // (no saturating difference: that is a vector instruction, and with its
    // result in the resource every load becomes a loop over lanes)
    uint32_t e;
    if (ROWS) {
      e = (uint32_t)max(bytes, 0);
      bytes -= BK * 4;
    } else {
      const int n = min(kleft, BK);
      e = n > 0 ? (uint32_t)n * row - (uint32_t)bytes : 0u;
    }
    const __amdgpu_buffer_rsrc_t r = make_rsrc(base, e);
    if (ROWS && kleft < BK) {
#pragma unroll
      for (int c = 0; c < N; ++c)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(st + (4 * c + wave) * 256), 16,
                                                 (int)(k4 >= kleft ? FAR : off[c]), 0, 0, 0);
    } else {
#pragma unroll
      for (int c = 0; c < N; ++c)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(st + (4 * c + wave) * 256), 16, (int)off[c], 0, 0, 0);
    }
    base += step;
  }
  // The lane's chunks of a slice with kleft k left, landed: elements past K
  // that came with them (of the next row) become 0.
  __device__ __forceinline__ void clear_tail(float* st, int wave, int lane, int kleft) const {
    if (!ROWS || k4 >= kleft || k4 + 4 <= kleft) return;
#pragma unroll
    for (int c = 0; c < N; ++c)
#pragma unroll
      for (int e = 1; e < 4; ++e)
        if (k4 + e >= kleft) st[(4 * c + wave) * 256 + 4 * lane + e] = 0.f;
  }
};

// A wave's products of one 16-deep k block.  BM = 32: two 16 x 16 x 4 MFMA
// blocks side by side; lane l supplies row (column) l % 16 and k = 4 (l / 16)
// + u.  BM = 64: one 32 x 32 x 2 block; row (column) l % 32 and k = 8 e + 4 (l /
// 32) + u.
template <int BM>
struct Block;

template <>
struct Block<32> {
  struct A { float v[4]; };
  struct B { float v[2][4]; };
  struct Acc { v4f v[2]; };
  template <bool ROWS>
  static __device__ __forceinline__ void read_a(const float* st, int r0, int kb, int lane, A& F) {
    const int li = lane & 15, lg = lane >> 4, r = r0 + li;
    if (ROWS) {
      const v4f v = *reinterpret_cast<const v4f*>(st + r * 32 + (((4 * kb + lg) ^ (li & 7)) << 2));
#pragma unroll
      for (int u = 0; u < 4; ++u) F.v[u] = v[u];
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        F.v[u] = st[(16 * kb + 8 * (lg >> 1) + 2 * u + (lg & 1)) * 32 + (r ^ (16 * (lg >> 1)))];
    }
  }
  template <bool ROWS>
  static __device__ __forceinline__ void read_b(const float* st, int c0, int kb, int lane, B& F) {
    const int li = lane & 15, lg = lane >> 4;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = c0 + 16 * j + li;
      if (ROWS) {
        const v4f v = *reinterpret_cast<const v4f*>(st + c * 32 + (((4 * kb + lg) ^ (li & 7)) << 2));
#pragma unroll
        for (int u = 0; u < 4; ++u) F.v[j][u] = v[u];
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) F.v[j][u] = st[(16 * kb + 4 * lg + u) * 64 + (c ^ (16 * lg))];
      }
    }
  }
  static __device__ __forceinline__ void zero(Acc& c) { c.v[0] = c.v[1] = v4f{0.f, 0.f, 0.f, 0.f}; }
  static __device__ __forceinline__ void fill(A& a, bool real, float x) {
#pragma unroll
    for (int u = 0; u < 4; ++u) a.v[u] = real ? a.v[u] : x;
  }
  static __device__ __forceinline__ void mma(const A& a, const B& b, Acc& c) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int j = 0; j < 2; ++j) c.v[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[u], b.v[j][u], c.v[j], 0, 0, 0);
  }
  static __device__ __forceinline__ void add(Acc& c, const Acc& d) {
    c.v[0] += d.v[0];
    c.v[1] += d.v[1];
  }
  // to the wave's block in LDS: register r of lane l is row 4 (l / 16) + r, column 16 j + l % 16
  static __device__ __forceinline__ void store(const Acc& c, float* st, int lane) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 4 * (lane >> 4) + r, n = 16 * j + (lane & 15);
        st[32 * m + ((((n >> 2) ^ (m & 7)) << 2) | (n & 3))] = c.v[j][r];
      }
  }
};

template <>
struct Block<64> {
  struct A { float v[2][4]; };
  typedef A B;
  typedef v16f Acc;
  template <bool ROWS>
  static __device__ __forceinline__ void read_a(const float* st, int r0, int kb, int lane, A& F) {
    const int h = lane >> 5, r = r0 + (lane & 31);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if (ROWS) {
        const v4f v = *reinterpret_cast<const v4f*>(st + r * 32 + (((4 * kb + 2 * e + h) ^ (lane & 7)) << 2));
#pragma unroll
        for (int u = 0; u < 4; ++u) F.v[e][u] = v[u];
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) F.v[e][u] = st[(16 * kb + 8 * e + 4 * h + u) * 64 + (r ^ (32 * h))];
      }
    }
  }
  template <bool ROWS>
  static __device__ __forceinline__ void read_b(const float* st, int c0, int kb, int lane, B& F) {
    read_a<ROWS>(st, c0, kb, lane, F);
  }
  static __device__ __forceinline__ void zero(Acc& c) {
#pragma unroll
    for (int r = 0; r < 16; ++r) c[r] = 0.f;
  }
  static __device__ __forceinline__ void fill(A& a, bool real, float x) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int u = 0; u < 4; ++u) a.v[e][u] = real ? a.v[e][u] : x;
  }
  static __device__ __forceinline__ void mma(const A& a, const B& b, Acc& c) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 2; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[e][u], b.v[e][u], c, 0, 0, 0);
  }
  static __device__ __forceinline__ void add(Acc& c, const Acc& d) { c += d; }
  // register r of lane l is row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
  static __device__ __forceinline__ void store(const Acc& c, float* st, int lane) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), n = lane & 31;
      st[32 * m + ((((n >> 2) ^ (m & 7)) << 2) | (n & 3))] = c[r];
    }
  }
};

// s_waitcnt vmcnt(0) lgkmcnt(0): this wave's loads into LDS have landed and
// its LDS accesses are done; lgkmcnt(0) alone.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0070); }
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// A barrier alone (the waits before it are the callers').
__device__ __forceinline__ void barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// K loop: acc = this lane's elements of the tile's product (EpiPos), by way of
// the wave's part of stage 0: element (m, n) of its block at 32 m + (4 (n / 4 ^
// m % 8) | n % 4).  FILL: the tile has rows past a_rows of a [K][M] operand: row
// ones_row is 1, the others 0.
template <int BM, int CH, bool AT, bool BT, bool FILL>
__device__ __forceinline__ void mainloop(const GemmProb& P, int m0, int n0, float* stage0, float* stage1,
                                         v4f (&acc)[Tile<BM>::NQ]) {
  using T = Tile<BM>;
  using X = Block<BM>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave >> 1) * T::WM, wn = (wave & 1) * 32;
  Opnd<BM, BM, !AT> A;
  Opnd<BM, BN, BT> B;
  A.init(P.A, P.a_rows, P.lda, m0, wave, lane);
  B.init(P.B, P.N, P.ldb, n0, wave, lane);
  typename X::Acc p[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) X::zero(p[c]);
  const int m = m0 + wm + (lane & (T::WM - 1));
  const bool real = m < P.a_rows;
  const float fill = m == P.ones_row ? 1.f : 0.f;
  const int n_it = (P.K + BK - 1) / BK;
  int it0 = 0, loaded = 1;  // slices begun, slices asked for
  A.load(stage0, wave, P.K);
  B.load(stage0 + T::A_FLOATS, wave, P.K);
  // Steady state of four chains (deep products): full slices with another one
  // behind them, half a slice at a time: the second k block's fragments are read
  // before the first one's MFMAs, and the next slice's first ones before the
  // second's.  No branches: with one, the compiler no longer sees which stage a
  // load in flight goes to, and waits for all of them before it reads either.
  // (8960 tiles of K = 784: 283 us, 292 with whole slices; 672 tiles 21.7 and 23.3.)
  const int steady = n_it - 1 - (P.K & 3 ? 1 : 0);
  if (CH == 4 && steady >= 2) {
    wait_loads();
    barrier();
    A.load(stage1, wave, P.K - BK);
    B.load(stage1 + T::A_FLOATS, wave, P.K - BK);
    if (m0 + wm < P.M) {
      typename X::A a0, a1;
      typename X::B b0, b1;
      X::template read_a<!AT>(stage0, wm, 0, lane, a0);
      X::template read_b<BT>(stage0 + T::A_FLOATS, wn, 0, lane, b0);
      for (; it0 + 2 <= steady; it0 += 2) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          float* st = s == 0 ? stage0 : stage1;
          float* next = s == 0 ? stage1 : stage0;
          X::template read_a<!AT>(st, wm, 1, lane, a1);
          X::template read_b<BT>(st + T::A_FLOATS, wn, 1, lane, b1);
          __builtin_amdgcn_sched_barrier(0);
          if (FILL) X::fill(a0, real, fill);
          X::mma(a0, b0, p[(2 * s) % CH]);
          __builtin_amdgcn_sched_barrier(0);
          wait_loads();
          barrier();  // the next slice is in LDS, and every wave has read this one
          A.load(st, wave, P.K - (it0 + s + 2) * BK);
          B.load(st + T::A_FLOATS, wave, P.K - (it0 + s + 2) * BK);
          X::template read_a<!AT>(next, wm, 0, lane, a0);
          X::template read_b<BT>(next + T::A_FLOATS, wn, 0, lane, b0);
          __builtin_amdgcn_sched_barrier(0);
          if (FILL) X::fill(a1, real, fill);
          X::mma(a1, b1, p[(2 * s + 1) % CH]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else {  // rows past M: the loads and barriers alone
      for (; it0 + 2 <= steady; it0 += 2) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          wait_loads();
          barrier();
          A.load(s == 0 ? stage0 : stage1, wave, P.K - (it0 + s + 2) * BK);
          B.load((s == 0 ? stage0 : stage1) + T::A_FLOATS, wave, P.K - (it0 + s + 2) * BK);
        }
      }
    }
    loaded = it0 + 2;
  }
  for (; it0 < n_it; it0 += 2) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int it = it0 + s;
      if (it >= n_it) break;
      const int kleft = P.K - it * BK;
      float* st = s == 0 ? stage0 : stage1;
      float* next = s == 0 ? stage1 : stage0;
      // this wave's loads of the slice have landed, then every wave's; and
      // every wave has read the slice before
      wait_loads();
      if ((!AT || BT) && kleft < BK && (kleft & 3)) {
        A.clear_tail(st, wave, lane, kleft);
        B.clear_tail(st + T::A_FLOATS, wave, lane, kleft);
        wait_lds();
      }
      barrier();
      if (it + 1 < n_it && it + 1 >= loaded) {
        A.load(next, wave, kleft - BK);
        B.load(next + T::A_FLOATS, wave, kleft - BK);
      }
      // a wave whose rows all lie past M and a k block past K have no MFMAs
      if (m0 + wm >= P.M) continue;
      const bool two = kleft > 16;
      typename X::A a[2];
      typename X::B b[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        if (kb == 1 && !two) break;
        X::template read_a<!AT>(st, wm, kb, lane, a[kb]);
        X::template read_b<BT>(st + T::A_FLOATS, wn, kb, lane, b[kb]);
      }
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        if (kb == 1 && !two) break;
        if (FILL) X::fill(a[kb], real, fill);
        X::mma(a[kb], b[kb], p[(2 * s + kb) % CH]);
      }
    }
  }
  if (CH == 4) {
    X::add(p[0], p[1 % CH]);
    X::add(p[2 % CH], p[3 % CH]);
    X::add(p[0], p[2 % CH]);
  }
  wait_lds();
  barrier();  // every wave has read its last slice
  float* blk = stage0 + wave * (T::WM * 32);
  X::store(p[0], blk, lane);
  // a wave reads its own block back: LDS runs a wave's accesses in order
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int q = 0; q < T::NQ; ++q)
    acc[q] = *reinterpret_cast<const v4f*>(blk + 256 * q + 32 * (lane >> 3) + 4 * ((lane & 7) ^ (lane >> 3)));
}

// The bias corrections 1 - beta^t of Adam's step, into bc: by one wave (not the
// same one in every tile: each has its SIMD), lane 0 beta1's and lane 1 beta2's.
__device__ __forceinline__ void bias_corrections(const GemmProb& P, int lt, int step_local, float* bc) {
  if (P.epi != EPI_ADAM || (int)(threadIdx.x >> 6) != (lt & 3)) return;
  const int lane = threadIdx.x & 63;
  const int tt = *as_global(P.t) + step_local + 1;
  const float c = (float)(1.0 - pow((double)(lane == 0 ? P.ac.beta1 : P.ac.beta2), (double)tt));
  if (lane < 2) bc[lane] = c;
  wait_lds();
}

template <int BM, int CH, bool WT>
__global__ __launch_bounds__(NT, BM == 32 ? 4 : 3) void gemm_kernel(LIPZ_GEMM_ARGS) {
  using T = Tile<BM>;
  if ((int)blockIdx.x >= g_total) {
    sample_rows<WT>(sj, (int)blockIdx.x - g_total);
    return;
  }
  int pi, lt;
  locate_tile(LIPZ_GEMM_GROUPS, pi, lt);
  const GemmProb P = probs[pi];
  const int tile_n = lt % P.tiles_n;
  const int m0 = (lt / P.tiles_n) * BM;
  const int n0 = tile_n * BN;

  // arrays of their own, not one: a load into one stage is then seen not to
  // touch the other, and reads of that one do not wait for it
  __shared__ __align__(16) float st0[T::FLOATS];
  __shared__ __align__(16) float st1[T::FLOATS];
  __shared__ float red[2][BM];
  __shared__ float bc[2];

  const EpiPos<BM> E(P, m0, n0);
  EpiIn<BM> in;
  if (CH == 1) epi_load<BM>(P, E, in);  // with four chains registers are short
  bias_corrections(P, lt, step_local, bc);
  v4f acc[T::NQ];
  if (CH == 1 && P.a_trans && P.b_trans) {  // no phase of the library; never in four chains (gemm_fast_ok)
    mainloop<BM, 1, true, true, true>(P, m0, n0, st0, st1, acc);
  } else if (P.a_trans) {
    if (m0 + BM > P.a_rows) mainloop<BM, CH, true, false, true>(P, m0, n0, st0, st1, acc);
    else mainloop<BM, CH, true, false, false>(P, m0, n0, st0, st1, acc);
  } else if (P.b_trans) {
    mainloop<BM, CH, false, true, false>(P, m0, n0, st0, st1, acc);
  } else {
    mainloop<BM, CH, false, false, false>(P, m0, n0, st0, st1, acc);
  }
  if (CH != 1) epi_load<BM>(P, E, in);
  epilogue<BM, WT>(P, acc, E, in, m0, n0, tile_n, bc, red);
}

// ---------------------------------------------------------------------------
// Four chains on few tiles: the four waves of a workgroup each compute the
// whole 32 x 64 tile over every fourth 16-deep k block.  Each wave streams its
// operands from global memory (L2) straight into registers in the MFMA
// fragment layout, two k blocks ahead of its MFMAs, with no LDS traffic and no
// barriers, and the four partial tiles are summed through LDS at the end.
// ---------------------------------------------------------------------------
__device__ __forceinline__ v4f bld4b(__amdgpu_buffer_rsrc_t r, uint32_t off_bytes) {
  return __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off_bytes, 0, 0));
}

struct WFrag {
  float a[2][4];   // A rows 16 i + (l % 16), k = kb + 4 (l / 16) + s
  float b[4][4];         // B cols 16 j + (l % 16), same k
};

template <int AT, int BT>
__device__ __forceinline__ void wave_load(const GemmProb& P, __amdgpu_buffer_rsrc_t ra,
                                          __amdgpu_buffer_rsrc_t rb, int m0, int n0, int kb, int li,
                                          int lg, WFrag& F) {
  const int k = kb + 4 * lg;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + 16 * i + li;
    if (AT == 0) {
      const v4f v = bld4b(ra, (uint32_t)(m * P.lda + k) * 4u);
      F.a[i][0] = v[0]; F.a[i][1] = v[1]; F.a[i][2] = v[2]; F.a[i][3] = v[3];
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s)
        F.a[i][s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, (int)((uint32_t)((k + s) * P.lda + m) * 4u), 0, 0));
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int n = n0 + 16 * j + li;
    if (BT == 1) {
      const v4f v = bld4b(rb, (uint32_t)(n * P.ldb + k) * 4u);
      F.b[j][0] = v[0]; F.b[j][1] = v[1]; F.b[j][2] = v[2]; F.b[j][3] = v[3];
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s)
        F.b[j][s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, (int)((uint32_t)((k + s) * P.ldb + n) * 4u), 0, 0));
    }
  }
}

// MFMAs of one k block.  TAIL: zero k >= K (the problem's last, partial
// block).  ONES: the tile holds the bias row of a [K][M] operand: set row
// ones_row to 1 (0 past K) and the other rows past a_rows to 0.
template <bool TAIL, bool ONES>
__device__ __forceinline__ void wave_mma(const GemmProb& P, int m0, int kb, int li, int lg, WFrag& F,
                                         v4f (&acc)[2][4]) {
  const int k = kb + 4 * lg;
  if (TAIL) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool ok = k + s < P.K;
#pragma unroll
      for (int i = 0; i < 2; ++i) F.a[i][s] = ok ? F.a[i][s] : 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) F.b[j][s] = ok ? F.b[j][s] : 0.f;
    }
  }
  if (ONES) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = m0 + 16 * i + li;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float one = (TAIL && k + s >= P.K) ? 0.f : 1.f;
        F.a[i][s] = m < P.a_rows ? F.a[i][s] : (m == P.ones_row ? one : 0.f);
      }
    }
  }
  // a 16-row block wholly past M has no MFMA work (uniform); each
  // accumulator still takes its four k steps in order
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (i == 0 || m0 + 16 * i < P.M)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(F.a[i][s], F.b[j][s], acc[i][j], 0, 0, 0);
}

template <int AT, int BT, bool ONES>
__device__ __forceinline__ void wave_mainloop(const GemmProb& P, int m0, int n0, v4f (&acc)[2][4]) {
  constexpr int PD = 2;
  // the wave index is uniform across the wave: keep it (and every k-block
  // index and loop bound derived from it) in scalar registers
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(P.A, P.a_bytes);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(P.B, P.b_bytes);
  const int nkb = (P.K + 15) / 16;                          // k blocks of the problem
  const int mine = nkb > wave ? (nkb - wave + 3) / 4 : 0;   // blocks wave, wave + 4, ...
  WFrag F[PD];
  // every prologue load issued (past the wave's blocks they read zeros or
  // values no MFMA uses), so that the steady-state loop below starts from
  // the same outstanding loads on every path
#pragma unroll
  for (int p = 0; p < PD; ++p) wave_load<AT, BT>(P, ra, rb, m0, n0, 16 * (wave + 4 * p), li, lg, F[p]);
  // steady state: every block full, every prefetch needed, no branches on
  // the loads, so the compiler can count outstanding loads exactly
  int q = 0;
  for (; q + 2 * PD <= mine; q += PD) {
#pragma unroll
    for (int p = 0; p < PD; ++p) {
      wave_mma<false, ONES>(P, m0, 16 * (wave + 4 * (q + p)), li, lg, F[p], acc);
      wave_load<AT, BT>(P, ra, rb, m0, n0, 16 * (wave + 4 * (q + p + PD)), li, lg, F[p]);
    }
  }
  // drain: the last PD .. 2 PD - 1 blocks, the problem's partial block among them
  for (; q < mine; q += PD) {
#pragma unroll
    for (int p = 0; p < PD; ++p) {
      if (q + p < mine) {
        const int kb = 16 * (wave + 4 * (q + p));
        if (kb + 16 > P.K) wave_mma<true, ONES>(P, m0, kb, li, lg, F[p], acc);
        else wave_mma<false, ONES>(P, m0, kb, li, lg, F[p], acc);
        if (q + p + PD < mine)
          wave_load<AT, BT>(P, ra, rb, m0, n0, 16 * (wave + 4 * (q + p + PD)), li, lg, F[p]);
      }
    }
  }
}

template <bool WT>
__global__ __launch_bounds__(NT, 2) void gemm_wave_kernel(LIPZ_GEMM_ARGS) {
  constexpr int BM = 32, RS = BN + 4;  // row stride of the partial tiles in LDS
  if ((int)blockIdx.x >= g_total) {
    sample_rows<WT>(sj, (int)blockIdx.x - g_total);
    return;
  }
  int pi, lt;
  locate_tile(LIPZ_GEMM_GROUPS, pi, lt);
  const GemmProb P = probs[pi];
  const int tile_n = lt % P.tiles_n;
  const int m0 = (lt / P.tiles_n) * BM;
  const int n0 = tile_n * BN;

  __shared__ __align__(16) float part[4][BM * RS];
  __shared__ float red[2][BM];
  __shared__ float bc[2];

  const EpiPos<BM> E(P, m0, n0);
  EpiIn<BM> in;
  epi_load<BM>(P, E, in);
  bias_corrections(P, lt, step_local, bc);
  v4f pacc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) pacc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  if (P.a_trans) {
    if (m0 + BM > P.a_rows) wave_mainloop<1, 0, true>(P, m0, n0, pacc);
    else wave_mainloop<1, 0, false>(P, m0, n0, pacc);
  } else if (P.b_trans) {
    wave_mainloop<0, 1, false>(P, m0, n0, pacc);
  } else {
    wave_mainloop<0, 0, false>(P, m0, n0, pacc);
  }

  // partial tiles to LDS (MFMA D layout: row 16 i + 4 (l / 16) + r, col 16 j + l % 16)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lg = lane >> 4;
  float* mine = part[wave];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) mine[(16 * i + 4 * lg + r) * RS + 16 * j + li] = pacc[i][j][r];
  __syncthreads();
  v4f acc[Tile<BM>::NQ];
#pragma unroll
  for (int q = 0; q < Tile<BM>::NQ; ++q) {
    const int o = (E.row0 - m0 + 8 * q) * RS + E.col - n0;
    const v4f p0 = *reinterpret_cast<const v4f*>(part[0] + o), p1 = *reinterpret_cast<const v4f*>(part[1] + o);
    const v4f p2 = *reinterpret_cast<const v4f*>(part[2] + o), p3 = *reinterpret_cast<const v4f*>(part[3] + o);
    acc[q] = (p0 + p1) + (p2 + p3);
  }
  epilogue<BM, WT>(P, acc, E, in, m0, n0, tile_n, bc, red);
}

}  // namespace

int gemm_tile_rows(int tiles64) { return tiles64 < LIPZ_GEMM_TILE64_MIN ? 32 : 64; }

void gemm_set_extents(GemmProb& p) {
  const uint64_t a = (uint64_t)(p.a_trans ? p.K : p.a_rows) * (uint64_t)p.lda * 4u;
  const uint64_t b = (uint64_t)(p.b_trans ? p.N : p.K) * (uint64_t)p.ldb * 4u;
  p.a_bytes = a < 0x7FFFFFF0u ? (uint32_t)a : 0u;
  p.b_bytes = b < 0x7FFFFFF0u ? (uint32_t)b : 0u;
}

bool gemm_fast_ok(const GemmProb& p) {
  // the three operand layouts the library uses:
  // (A, B) = (row, row) forward, (row, W^T) input gradient, (X^T, row) weight gradient
  return !(p.a_trans && p.b_trans) && (p.vec & 3) == 3 && p.a_bytes > 0 && p.b_bytes > 0 && p.a_bytes < 0x7FFFFFF0u &&
         p.b_bytes < 0x7FFFFFF0u;
}

hipError_t launch_gemm_grouped(const GemmProb* d_probs, const GemmGroups& grp, int total_tiles,
                               int tile_rows, int kernel, int step_local, bool write_through, hipStream_t s,
                               hipEvent_t ev_start, hipEvent_t ev_stop, const SampleJob* job) {
  if (grp.n <= 0 || total_tiles <= 0) return hipSuccess;
  SampleJob sj;
  memset(&sj, 0, sizeof(sj));
  if (job) sj = *job;
  // the groups as the kernels take them (see LIPZ_GEMM_ARGS)
  if (grp.n > GEMM_MAX_GROUPS || grp.first_tile[0] != 0 || grp.first_prob[0] != 0) return hipErrorInvalidValue;
  int ft[GEMM_MAX_GROUPS], fp[GEMM_MAX_GROUPS];
  for (int q = 0; q < GEMM_MAX_GROUPS; ++q) {
    ft[q] = q < grp.n ? grp.first_tile[q] : total_tiles;
    fp[q] = q < grp.n ? grp.first_prob[q] : 0;
    if (q > 0 && q < grp.n && !(ft[q - 1] < ft[q] && ft[q] < total_tiles)) return hipErrorInvalidValue;
  }
  const dim3 g(total_tiles + sj.blocks), b(NT);
  // the events (may be null) are stamped by the kernel's own dispatch packet,
  // so their difference is the kernel's execution time alone
#define LIPZ_LAUNCH(K)                                                                                          \
  hipExtLaunchKernelGGL(K, g, b, 0, s, ev_start, ev_stop, 0, d_probs, total_tiles, ft[1], ft[2], ft[3], fp[1], \
                        fp[2], fp[3], grp.tiles_per_prob[0], grp.tiles_per_prob[1], grp.tiles_per_prob[2],    \
                        grp.tiles_per_prob[3], step_local, sj)
#define LIPZ_LAUNCH_WT(BMV, CHV) \
  if (write_through) LIPZ_LAUNCH((gemm_kernel<BMV, CHV, true>)); else LIPZ_LAUNCH((gemm_kernel<BMV, CHV, false>))
  if (kernel == GEMM_K_WAVE) {
    if (tile_rows != 32) return hipErrorInvalidValue;
    if (write_through) LIPZ_LAUNCH((gemm_wave_kernel<true>)); else LIPZ_LAUNCH((gemm_wave_kernel<false>));
  } else if (kernel == GEMM_K_CHAINS4) {
    if (tile_rows == 32) { LIPZ_LAUNCH_WT(32, 4); } else { LIPZ_LAUNCH_WT(64, 4); }
  } else {
    if (tile_rows == 32) { LIPZ_LAUNCH_WT(32, 1); } else { LIPZ_LAUNCH_WT(64, 1); }
  }
#undef LIPZ_LAUNCH_WT
#undef LIPZ_LAUNCH
  return hipGetLastError();
}

int gemm_choose_kernel(bool aligned, bool b_trans, int max_k, int tiles, int tile_rows) {
  if (!aligned || max_k < LIPZ_GEMM_CHAINS4_MIN_K) return GEMM_K_CHAIN;
  const bool wave = tiles <= LIPZ_GEMM_WAVE_MAX_TILES || (max_k >= LIPZ_GEMM_WAVE_MIN_K && !b_trans);
  return tile_rows == 32 && wave ? GEMM_K_WAVE : GEMM_K_CHAINS4;
}

}  // namespace lipz
