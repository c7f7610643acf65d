// The forward convolutions of the evaluation on the bf16 matrix cores, at fp32
// accuracy (split.h): the same implicit GEMMs, position maps and taps as
// conv_kernel, for problems whose operand rows are read as float4 (ConvProb::gen
// == 0), with row-major weights and outputs wider than 16.  (Training keeps the
// fp32 sums: conv_wide.hip.)
//
// A 256-thread workgroup (4 wave64, 2 x 2) owns a TM x TN output tile.  K
// advances in 32-deep slices: the fp32 operands of the next slice are in
// registers while the current one is multiplied; a slice is split into its
// three bf16 pieces on the way into LDS (single buffer, two barriers per
// slice; the two or three workgroups of a CU fill each other's barriers), and
// the six piece products go through v_mfma_f32_32x32x16_bf16.
//
// PRE: the weights were split by split_weights_kernel into the order of the
// MFMA's operand.  The waves read them from L2 straight into registers, half a
// slice ahead, and only the gathered operand goes through LDS: the LDS traffic
// of a slice, which comes between its MFMAs and the next one's, is halved.
//
// What bounds it: the bf16 matrix rate the card holds on real data (a large
// bf16 product of the math library: 1.21 PFLOP/s, 202 for six products; the
// clock drops to 1.9 GHz).  Measured, 80 problems of 98304 x 128 x 1024 (2.06
// TFLOP): 11.5 ms (179 TFLOP/s) with PRE, 12.2 without, 15.8 on fp32 MFMAs
// (conv_wide_kernel) and 20.9 on conv_kernel; 6144 x 512 x 4096: 9.9 ms (208)
// with PRE, 10.2 without; all weights of 16 cells (44 million) are split in
// 0.10 ms.  Splitting the weights ahead but staging them in LDS gained nothing.
//
// A tile with a non-finite sum (split.h) is multiplied again in fp32, as 64 x 64
// tiles of conv_wide_kernel's loop: conv_kernel's sums, bit for bit, for its
// finite outputs too.  A 64 x 64 tile's registers and LDS fit in what the bf16
// loop holds anyway.  (4x4 grid of 64x64 images, evaluation 44.0 ms: 48.5 with
// one discriminator all NaN, 59.5 when such tiles took two more bf16 passes and
// were noticed at their end only; with every network NaN 66 and 115, on
// conv_kernel 83.)
//
// TAP1: the channels per tap are a multiple of 32, so a slice lies within one
// tap and its shift and weight row are scalars; otherwise every float4
// carries its own (tap, channel), advanced without divisions.
#include <hip/hip_ext.h>

#include "conv_wide_tile.h"

namespace lipz {

namespace {

constexpr int max3(int a, int b, int c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }

template <int TM, int TN>
struct SplitTile {
  static constexpr int A_PIECE = TM * RK_PITCH, B_PIECE = SK_DEEP * km_pitch(TN);
  static constexpr int A_F4 = TM / 32, B_F4 = TN / 32;  // float4 of a slice per thread
  static constexpr int TI = TM / 64, TJ = TN / 64;      // 32 x 32 MFMA tiles per wave
  // A's pieces, then the stores' strips; B's pieces.  Tiles with non-finite sums
  // use the two as the stages of 64 x 64 fp32 tiles.
  static constexpr int STAGE = 4 * STAGE_FLOATS<64, 64>, STRIPS = 4 * 16 * (TN / 2 + 4) * 4;
  static constexpr int LDS0 = max3(3 * A_PIECE, STRIPS, STAGE), LDS1 = max3(3 * B_PIECE, 0, STAGE);
};

// Operand loads of a slice.  A: thread t takes k 8 (t % 4) .. + 7 of rows
// t / 4 + 64 h; B (k rows): one column quad of k rows t / (TN / 4) +
// (1024 / TN) h.
template <int TM, int TN, bool TAP1>
struct SplitCtx {
  __amdgpu_buffer_rsrc_t ra, rb, rp;
  int pb[TN / 64];                           // byte offsets of the wave's column blocks in the split weights
  int y[TM / 64], x[TM / 64], off[TM / 64];  // source coordinates and element offset of the thread's rows
  uint32_t va[TM / 64];                      // TAP1: byte offsets of the rows under the slice's tap
  KPos ka[2], kb[TN / 32];                   // not TAP1
  int dt, dc;                                // not TAP1: 32 = dt * cs + dc
  int t, c;                                  // TAP1: the slice's tap and first channel
  uint32_t bcol;                             // byte offset of the thread's B columns (TAP1: and k row), FAR past N
};

template <int TM, int TN, bool TAP1, bool PRE>
__device__ __forceinline__ void split_setup(const ConvProb& P, int m0, int n0, SplitCtx<TM, TN, TAP1>& X) {
  const int tid = threadIdx.x;
  X.ra = rsrc(P.S, P.s_bytes);
  if (PRE) {
    X.rp = rsrc(reinterpret_cast<const float*>(P.Wp), (uint32_t)((P.N + 31) / 32) * (uint32_t)(P.wp_k * 192));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int j = 0; j < TN / 64; ++j) {
      // a block past N repeats the last one, for columns that are not stored: the extent of
      // a resource does not bound a scalar offset past it
      const int blk = min((n0 + (wave & 1) * (TN / 2)) / 32 + j, (P.N + 31) / 32 - 1);
      X.pb[j] = blk * (P.wp_k * 192);
    }
  } else {
    X.rb = rsrc(P.W, P.w_bytes);
  }
#pragma unroll
  for (int h = 0; h < TM / 64; ++h) {
    const int p = m0 + (tid >> 2) + 64 * h;
    const Pos q = grid_pos(p < P.M ? p : 0, P.gh_log, P.gw_log);
    X.y[h] = q.y * P.smap.sy;
    X.x[h] = q.x * P.smap.sx;
    X.off[h] = ((((q.img << P.smap.h_log) + X.y[h]) << P.smap.w_log) + X.x[h]) * P.smap.ld;
    if (p >= P.M) X.y[h] = 0x40000000;  // no tap brings it inside
  }
  const int kr = tid / (TN / 4);
  const int n = n0 + ((tid % (TN / 4)) << 2);
  X.bcol = n < P.N ? (uint32_t)(n + (TAP1 ? kr * P.N : 0)) * 4u : FAR;
  X.t = 0;
  X.c = 0;
  if (!TAP1) {
    X.dt = P.taps > 1 ? 32 / P.cs : 0;
    X.dc = P.taps > 1 ? 32 - X.dt * P.cs : 32;
    X.ka[0] = kpos(P, (tid & 3) << 3);
    X.ka[1] = kpos(P, ((tid & 3) << 3) + 4);
#pragma unroll
    for (int h = 0; h < TN / 32; ++h) X.kb[h] = kpos(P, kr + (1024 / TN) * h);
  }
}

// Byte offset of row h's source pixel under tap d, channel ch; FAR outside.
template <int TM, int TN, bool TAP1>
__device__ __forceinline__ uint32_t split_row(const ConvProb& P, const SplitCtx<TM, TN, TAP1>& X, int h, Tap d, int ch) {
  const bool ok = ((unsigned)(X.y[h] + d.dy) < (1u << P.smap.h_log)) & ((unsigned)(X.x[h] + d.dx) < (1u << P.smap.w_log));
  return ok ? (uint32_t)(X.off[h] + ((d.dy << P.smap.w_log) + d.dx) * P.smap.ld + ch) * 4u : FAR;
}

__device__ __forceinline__ float4 ld4s(__amdgpu_buffer_rsrc_t r, uint32_t off_bytes, uint32_t scalar_bytes) {
  const v4u v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off_bytes, (int)scalar_bytes, 0);
  return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
}

// kw: the slice's first weight row (TAP1).
template <int TM, int TN, bool TAP1, bool PRE>
__device__ __forceinline__ void split_load(const ConvProb& P, SplitCtx<TM, TN, TAP1>& X, int k0,
                                           float4 (&fa)[TM / 32], float4 (&fb)[TN / 32], int& kw) {
  const int tid = threadIdx.x, kg = (tid & 3) << 3;
  if (TAP1) {
    // within a tap only the scalar offsets move
    const Tap d = tap_of(P, X.t);
    if (X.c == 0) {
#pragma unroll
      for (int h = 0; h < TM / 64; ++h) X.va[h] = split_row<TM, TN, TAP1>(P, X, h, d, kg);
    }
#pragma unroll
    for (int h = 0; h < TM / 64; ++h) {
      fa[2 * h] = ld4s(X.ra, X.va[h], (uint32_t)X.c * 4u);
      fa[2 * h + 1] = ld4s(X.ra, X.va[h], (uint32_t)X.c * 4u + 16u);
    }
    const int r0 = d.wt * P.cs + X.c;
    kw = r0;
    if (!PRE)
#pragma unroll
    for (int h = 0; h < TN / 32; ++h) fb[h] = ld4s(X.rb, X.bcol, (uint32_t)((r0 + (1024 / TN) * h) * P.N) * 4u);
    X.c += SK_DEEP;
    if (X.c >= P.cs) {
      X.c = 0;
      ++X.t;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const bool kok = k0 + kg + 4 * e < P.K;
      const Tap d = tap_of(P, X.ka[e].t);
#pragma unroll
      for (int h = 0; h < TM / 64; ++h) {
        const uint32_t o = split_row<TM, TN, TAP1>(P, X, h, d, X.ka[e].c);
        fa[2 * h + e] = ld4(X.ra, kok ? o : FAR);
      }
      advance(P, X.ka[e], X.dt, X.dc);
    }
#pragma unroll
    for (int h = 0; h < TN / 32; ++h) {
      const uint32_t o = X.bcol + (uint32_t)((tap_of(P, X.kb[h].t).wt * P.cs + X.kb[h].c) * P.N) * 4u;
      fb[h] = ld4(X.rb, k0 + tid / (TN / 4) + (1024 / TN) * h < P.K ? o : FAR);
      advance(P, X.kb[h], X.dt, X.dc);
    }
  }
}

// The operand slices, split, into their three LDS tiles each.
template <int TM, int TN, bool PRE>
__device__ __forceinline__ void split_store(const float4 (&fa)[TM / 32], const float4 (&fb)[TN / 32], char* At, char* Bt) {
  using T = SplitTile<TM, TN>;
  const int tid = threadIdx.x;
#pragma unroll
  for (int h = 0; h < TM / 64; ++h) {
    const float4 u = fa[2 * h], v = fa[2 * h + 1];
    uint4 p[3];
    split2(u.x, u.y, p[0].x, p[1].x, p[2].x);
    split2(u.z, u.w, p[0].y, p[1].y, p[2].y);
    split2(v.x, v.y, p[0].z, p[1].z, p[2].z);
    split2(v.z, v.w, p[0].w, p[1].w, p[2].w);
    const int o = rk_off((tid >> 2) + 64 * h, tid & 3);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<uint4*>(At + q * T::A_PIECE + o) = p[q];
  }
  if (PRE) return;
#pragma unroll
  for (int h = 0; h < TN / 32; ++h) {
    uint2 p[3];
    split2(fb[h].x, fb[h].y, p[0].x, p[1].x, p[2].x);
    split2(fb[h].z, fb[h].w, p[0].y, p[1].y, p[2].y);
    const int o = (tid / (TN / 4) + (1024 / TN) * h) * km_pitch(TN) + ((tid % (TN / 4)) << 3);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(Bt + q * T::B_PIECE + o) = p[q];
  }
}

// The K loop: acc = the tile's products.  Ends after the first slice where
// that has an infinity or NaN in some wave's last rows, as it does all over for
// a network that has diverged: the caller multiplies such a tile by fp32 MFMAs.
template <int TM, int TN, bool TAP1, bool PRE>
__device__ __forceinline__ void split_products(const ConvProb& P, int m0, int n0, char* At, char* Bt,
                                               v16f (&acc)[TM / 64][TN / 64]) {
  using T = SplitTile<TM, TN>;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave >> 1) * (TM / 2), wn = (wave & 1) * (TN / 2);
  SplitCtx<TM, TN, TAP1> X;
  split_setup<TM, TN, TAP1, PRE>(P, m0, n0, X);
  v16f low[T::TI][T::TJ];  // the five smaller piece products
#pragma unroll
  for (int i = 0; i < T::TI; ++i)
#pragma unroll
    for (int j = 0; j < T::TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = low[i][j][r] = 0.f;
  float4 fa[T::A_F4], fb[T::B_F4];
  int kw = 0;
  auto products = [&](const v8bf (&a)[T::TI][3], const v8bf (&b)[T::TJ][3]) {
#pragma unroll
    for (int s = 2; s >= 0; --s)
#pragma unroll
      for (int q = 0; q <= s; ++q)
#pragma unroll
        for (int i = 0; i < T::TI; ++i)
#pragma unroll
          for (int j = 0; j < T::TJ; ++j) {
            v16f& to = s ? low[i][j] : acc[i][j];
            to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][q], b[j][s - q], to, 0, 0, 0);
          }
  };
  auto a_frags = [&](int kk, v8bf (&a)[T::TI][3]) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int i = 0; i < T::TI; ++i) a[i][q] = rk_frag(At + q * T::A_PIECE, wm + 32 * i, kk, lane);
  };
  // Every wave has read the previous slice; true: no further slice.
  auto enough = [&](int k0) {
    if (k0 != SK_DEEP) {
      __syncthreads();
      return false;
    }
    bool bad = false;
#pragma unroll
    for (int i = 0; i < T::TI; ++i)
#pragma unroll
      for (int j = 0; j < T::TJ; ++j) bad |= non_finite(acc[i][j][15]);
    return __syncthreads_or(bad) != 0;
  };
  if (PRE) {
    // split weights: fragments as they are used, straight from memory, half a
    // slice ahead; past the last slice those loads repeat it
    auto b_frags = [&](int row, v8bf (&b)[T::TJ][3]) {
#pragma unroll
      for (int j = 0; j < T::TJ; ++j)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          b[j][q] = __builtin_bit_cast(v8bf, __builtin_amdgcn_raw_buffer_load_b128(X.rp, lane * 16,
                                                                                  X.pb[j] + row * 192 + q * 1024, 0));
    };
    v8bf a[T::TI][3], b0[T::TJ][3], b1[T::TJ][3];
    split_load<TM, TN, TAP1, PRE>(P, X, 0, fa, fb, kw);
    b_frags(kw, b0);
    for (int k0 = 0; k0 < P.K; k0 += SK_DEEP) {
      if (enough(k0)) break;
      split_store<TM, TN, PRE>(fa, fb, At, Bt);
      b_frags(kw + 16, b1);
      if (k0 + SK_DEEP < P.K) split_load<TM, TN, TAP1, PRE>(P, X, k0 + SK_DEEP, fa, fb, kw);
      __syncthreads();
      a_frags(0, a);
      products(a, b0);
      a_frags(1, a);
      b_frags(kw, b0);
      products(a, b1);
    }
  } else {
    split_load<TM, TN, TAP1, PRE>(P, X, 0, fa, fb, kw);
    for (int k0 = 0; k0 < P.K; k0 += SK_DEEP) {
      if (enough(k0)) break;
      split_store<TM, TN, PRE>(fa, fb, At, Bt);
      if (k0 + SK_DEEP < P.K) split_load<TM, TN, TAP1, PRE>(P, X, k0 + SK_DEEP, fa, fb, kw);
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        v8bf a[T::TI][3], b[T::TJ][3];
        a_frags(kk, a);
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
          for (int j = 0; j < T::TJ; ++j) b[j][q] = km_frag<TN>(Bt + q * T::B_PIECE, wn + 32 * j, kk, lane);
        products(a, b);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < T::TI; ++i)
#pragma unroll
    for (int j = 0; j < T::TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = (acc[i][j][r] + low[i][j][r]) * SPLIT_UNSCALE;
}

// The lane's index in its wave; no register holds it over the K loop.
__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// The descriptor, read again, into scalar registers: kept in them over the K
// loop, it would spill.
__device__ __forceinline__ ConvProb read_again(const ConvProb* p) {
  typedef const __attribute__((address_space(4))) uint32_t* Words;
  static_assert(sizeof(ConvProb) % 4 == 0, "whole words");
  struct {
    uint32_t w[sizeof(ConvProb) / 4];
  } v;
  uintptr_t a = (uintptr_t)p;
  asm volatile("" : "+s"(a));
#pragma unroll
  for (size_t i = 0; i < sizeof(ConvProb) / 4; ++i) v.w[i] = ((Words)a)[i];
  return __builtin_bit_cast(ConvProb, v);
}

template <int TM, int TN, bool TAP1, bool PRE>
__global__ __launch_bounds__(NT, 2) void conv_split_kernel(const ConvProb* __restrict__ probs, ConvGroups grp,
                                                           float slope) {
  using T = SplitTile<TM, TN>;
  __shared__ __align__(16) float lds0[T::LDS0 / 4];
  __shared__ __align__(16) float lds1[T::LDS1 / 4];
  const int b = blockIdx.x;
  int gi = 0;
#pragma unroll
  for (int q = 1; q < GEMM_MAX_GROUPS; ++q)
    if (q < grp.n && b >= grp.first_block[q]) gi = q;
  // first_block is a multiple of 8, so (b - first_block) % 8 is still the XCD
  const int rel = xcd_remap(b - grp.first_block[gi], grp.blocks[gi]);
  if (rel >= grp.real_tiles[gi]) return;
  const int pi = grp.first_prob[gi] + rel / grp.tiles_per_prob[gi];
  const int lt = rel % grp.tiles_per_prob[gi];
  const ConvProb P = probs[pi];
  const int m0 = (lt / P.tiles_n) * TM, n0 = (lt % P.tiles_n) * TN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  v16f acc[T::TI][T::TJ];
  split_products<TM, TN, TAP1, PRE>(P, m0, n0, reinterpret_cast<char*>(lds0), reinterpret_cast<char*>(lds1), acc);
  bool bad = false;
#pragma unroll
  for (int i = 0; i < T::TI; ++i)
#pragma unroll
    for (int j = 0; j < T::TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) bad |= non_finite(acc[i][j][r]);
  if (__builtin_expect(__syncthreads_or(bad) == 0, 1)) {
    wide_write<TM, TN, CONV_FWD>(read_again(probs + pi), acc, m0, n0, 0, slope, wave, lane_id(), lds0);
    return;
  }
#pragma unroll 1
  for (int q = 0; q < TM / 64 * (TN / 64); ++q) {
    const ConvProb A = read_again(probs + pi);
    const int m = m0 + q / (TN / 64) * 64, n = n0 + q % (TN / 64) * 64;
    if (m >= A.M || n >= A.N) continue;
    wide_tile<64, 64, CONV_FWD, 0, TAP1>(A, m, n, 0, 0, A.K, slope, wave, lds0, lds1);
    __syncthreads();
  }
}

// 32 x 32 elements of W per workgroup and step, transposed through LDS.
__global__ __launch_bounds__(NT) void split_weights_kernel(const SplitWProb* __restrict__ probs) {
  __shared__ float t[32][33];
  const SplitWProb P = probs[blockIdx.y];
  const int tid = threadIdx.x, r = tid >> 3, q = (tid & 7) << 2;
  const int tk = P.K / 32, tiles = tk * ((P.N + 31) / 32);
  for (int b = blockIdx.x; b < tiles; b += gridDim.x) {
    const int k0 = 32 * (b % tk), nb = b / tk;
    __syncthreads();
    const bool ok = 32 * nb + q < P.N;
    const float4 v = ok ? *reinterpret_cast<const float4*>(P.W + (size_t)(k0 + r) * P.N + 32 * nb + q)
                        : make_float4(0.f, 0.f, 0.f, 0.f);
    t[r][q] = v.x;
    t[r][q + 1] = v.y;
    t[r][q + 2] = v.z;
    t[r][q + 3] = v.w;
    __syncthreads();
    // column r, k rows q .. q + 3 of the tile: lane r + 32 ((q / 8) % 2) of k
    // block q / 16, half of its 16 bytes
    uint2 p[3];
    split2(t[q][r], t[q + 1][r], p[0].x, p[1].x, p[2].x);
    split2(t[q + 2][r], t[q + 3][r], p[0].y, p[1].y, p[2].y);
    char* o = reinterpret_cast<char*>(P.out) + ((size_t)nb * (P.K / 16) + k0 / 16 + (q >> 4)) * 3072 +
              (r + 32 * ((q >> 3) & 1)) * 16 + (q & 4) * 2;
#pragma unroll
    for (int e = 0; e < 3; ++e) *reinterpret_cast<uint2*>(o + e * 1024) = p[e];
  }
}

}  // namespace

hipError_t launch_split_weights(const SplitWProb* d_probs, int count, int64_t max_elems, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const int64_t tiles = (max_elems + 1023) / 1024;
  hipLaunchKernelGGL(split_weights_kernel, dim3(tiles < 1024 ? (unsigned)tiles : 1024u, count), dim3(NT), 0, s, d_probs);
  return hipGetLastError();
}

hipError_t launch_conv_split(const ConvProb* d_probs, const ConvGroups& grp, int total_blocks, const ConvVariant& v,
                             float slope, hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (grp.n <= 0 || total_blocks <= 0) return hipSuccess;
  if (v.mode != CONV_FWD || v.bt) return hipErrorInvalidValue;
#define LIPZ_CS1(TM, TN, T1, PR)                                                                                  \
  hipExtLaunchKernelGGL((conv_split_kernel<TM, TN, T1, PR>), dim3(total_blocks), dim3(NT), 0, s, ev_start, ev_stop, \
                        0, d_probs, grp, slope)
#define LIPZ_CS(TM, TN)                          \
  if (v.pre) LIPZ_CS1(TM, TN, true, true);       \
  else if (v.tap1) LIPZ_CS1(TM, TN, true, false); \
  else LIPZ_CS1(TM, TN, false, false)
  if (v.pre && !v.tap1) return hipErrorInvalidValue;
  if (v.tm == 128 && v.tn == 128) { LIPZ_CS(128, 128); }
  else if (v.tm == 128 && v.tn == 64) { LIPZ_CS(128, 64); }
  else if (v.tm == 64 && v.tn == 64) { LIPZ_CS(64, 64); }
  else return hipErrorInvalidValue;
#undef LIPZ_CS
#undef LIPZ_CS1
  return hipGetLastError();
}

}  // namespace lipz
