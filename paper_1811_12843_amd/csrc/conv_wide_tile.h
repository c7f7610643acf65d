// The wide fp32 tiles: operand loads into LDS, K loop and stores of a TM x TN
// output tile (conv_wide.hip has the layouts' reasons and what they measured).
// conv_wide_kernel is this loop; conv_split_kernel multiplies tiles with
// non-finite sums by it.
#pragma once

#include "conv_tile.h"

namespace lipz {

namespace {

typedef __attribute__((address_space(3))) void lds_void;

// LDS stage of an operand slice, as the loads write it (64 lanes x 16 bytes in
// a row per instruction).
//
// Rows of k ("RK": gathered rows, transposed weights): 128 bytes per row, k
// quad q at place q ^ (row % 8), so that the 8 rows of a ds_read_b128 phase lie
// on different banks.  k rows ("KM": weights of a forward layer, both operands
// of a weight gradient): row k holds the operand's columns, column quad q at
// place q ^ (8 ((k / 4) % 2)), which puts the two k rows of a fragment read on
// different halves of the banks.
template <int ROWS, bool RK>
struct Stage {
  static constexpr int FLOATS = ROWS * SK_DEEP;
  static constexpr int LOADS = FLOATS / 1024;  // per wave and slice
};
__device__ __forceinline__ int km_col(int col, int k) { return (((col >> 2) ^ ((k & 4) << 1)) << 2) | (col & 3); }

// MFMA fragments of one 16-deep k block: sub-step (u, e) multiplies k
// 8 e + 4 (l / 32) + u.
template <int T>
struct WideFrag {
  float v[T][2][4];  // [32-row tile][e][u]
};
template <int ROWS, bool RK, int T>
__device__ __forceinline__ void wide_frags(const float* s, int row0, int kb, int lane, WideFrag<T>& F) {
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const int r = row0 + 32 * i + (lane & 31);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if (RK) {
        const float4 v = *reinterpret_cast<const float4*>(s + r * SK_DEEP + ((((kb >> 2) + 2 * e + (lane >> 5)) ^ (r & 7)) << 2));
        F.v[i][e][0] = v.x;
        F.v[i][e][1] = v.y;
        F.v[i][e][2] = v.z;
        F.v[i][e][3] = v.w;
      } else {
        const int k = kb + 8 * e + 4 * (lane >> 5);
#pragma unroll
        for (int u = 0; u < 4; ++u) F.v[i][e][u] = s[(k + u) * ROWS + km_col(r, k)];
      }
    }
  }
}

// What a lane's loads need.  Every load is lane offset + scalar offset; within
// a tap only the scalar one moves from slice to slice (VALU instructions between
// the MFMAs keep the matrix cores waiting).
//
// Row of load c of an operand for this lane: an RK operand's row (eight rows of
// eight k quads per instruction), a KM operand's k row.
template <int ROWS, bool RK>
__device__ __forceinline__ int load_row(int c, int wave, int lane) {
  return RK ? 8 * (4 * c + wave) + (lane >> 3) : (256 / ROWS) * (4 * c + wave) + lane / (ROWS / 4);
}
// KM: first column of the lane's column quad (the swizzle bit (k / 4) % 2 of
// its k rows is the same for all c).
template <int ROWS>
__device__ __forceinline__ int load_col(int wave, int lane) {
  return ((lane % (ROWS / 4)) ^ ((load_row<ROWS, false>(0, wave, lane) & 4) << 1)) << 2;
}

template <int TM, int TN, int MODE, int BT, bool TAP1>
struct WideCtx {
  static constexpr bool FWD = MODE == CONV_FWD;
  static constexpr bool A_RK = FWD, B_RK = FWD && BT == 1;
  static constexpr int NA = Stage<TM, A_RK>::LOADS, NB = Stage<TN, B_RK>::LOADS;
  __amdgpu_buffer_rsrc_t ra, rb;
  uint32_t va[NA], vb[NB];  // lane offsets in bytes (FAR: zeros) of the slice at k
  uint32_t sa, sb;          // scalar offsets
  int k;
  uint32_t nb[NB];          // lane offsets of B's rows (RK) or column quad, FAR past N
  // FWD: source coordinates and element offset of the lane's rows (a row past
  // M has coordinates that no tap brings inside) and its k within a slice
  int y[FWD ? NA : 1], x[FWD ? NA : 1], off[FWD ? NA : 1], kq;
  int t, c;                 // TAP1: the slice's tap and first channel
  KPos ka, kb[NB];          // not TAP1: (tap, channel) of k + kq, and of a KM B's k rows
  int dt, dc;               // not TAP1: 32 = dt * cs + dc
  // WG (grids at most 32 wide: a slice is whole grid rows, so a lane keeps its x):
  // offsets of A at the first slice, grid row of the lane's positions, and the
  // grid row on which the tap leaves the image (-1: none)
  uint32_t ab[FWD ? 1 : NA];
  int gy[FWD ? 1 : NA], gy_bad;
};

template <int TM, int TN, int MODE, int BT, bool TAP1>
__device__ __forceinline__ void wide_setup(const ConvProb& P, int m0, int n0, int kbeg, int wave, int lane,
                                           WideCtx<TM, TN, MODE, BT, TAP1>& X) {
  using C = WideCtx<TM, TN, MODE, BT, TAP1>;
  X.ra = rsrc(P.S, P.s_bytes);
  X.rb = C::FWD ? rsrc(P.W, P.w_bytes) : rsrc(P.P, P.p_bytes);
  X.sa = X.sb = 0;
  X.k = kbeg;
  const int n = n0 + load_col<TN>(wave, lane);  // a KM B's columns
  if (C::FWD) {
    X.kq = ((lane & 7) ^ (lane >> 3)) << 2;
#pragma unroll
    for (int c = 0; c < C::NA; ++c) {
      const int p = m0 + load_row<TM, true>(c, wave, lane);
      const Pos q = grid_pos(p < P.M ? p : 0, P.gh_log, P.gw_log);
      X.y[c] = q.y * P.smap.sy;
      X.x[c] = q.x * P.smap.sx;
      X.off[c] = ((((q.img << P.smap.h_log) + X.y[c]) << P.smap.w_log) + X.x[c]) * P.smap.ld;
      if (p >= P.M) X.y[c] = 0x40000000;
    }
    X.t = 0;
    X.c = 0;
    if (!TAP1) {
      X.dt = P.taps > 1 ? 32 / P.cs : 0;
      X.dc = P.taps > 1 ? 32 - X.dt * P.cs : 32;
      X.ka = kpos(P, X.kq);
    }
#pragma unroll
    for (int c = 0; c < C::NB; ++c) {
      const int r = load_row<TN, C::B_RK>(c, wave, lane);
      if (C::B_RK) {
        X.nb[c] = n0 + r < P.N ? (uint32_t)((n0 + r) * P.wsn + (TAP1 ? X.kq : 0)) * 4u : FAR;
      } else {
        X.nb[c] = n < P.N ? (uint32_t)(n + (TAP1 ? r * P.N : 0)) * 4u : FAR;
        if (!TAP1) X.kb[c] = kpos(P, r);
      }
      X.vb[c] = X.nb[c];
    }
  } else {
    const int m = m0 + load_col<TM>(wave, lane);
    const bool mok = m < P.taps * P.cs;
    int t = 0, ch = 0;
    if (mok) split_k(P, m, t, ch);
    const Tap d = tap_of(P, t);
    const int gh = 1 << P.gh_log;
    X.gy_bad = d.dy < 0 ? 0 : ((gh - 1) * P.smap.sy + d.dy >= (1 << P.smap.h_log) ? gh - 1 : -1);
#pragma unroll
    for (int c = 0; c < C::NA; ++c) {
      const int p = kbeg + load_row<TM, false>(c, wave, lane);
      const Pos q = grid_pos(p, P.gh_log, P.gw_log);
      const int x = q.x * P.smap.sx + d.dx;
      X.gy[c] = q.y;
      const int o = ((((q.img << P.smap.h_log) + q.y * P.smap.sy + d.dy) << P.smap.w_log) + x) * P.smap.ld + ch;
      X.ab[c] = mok && (unsigned)x < (1u << P.smap.w_log) ? (uint32_t)o * 4u : FAR;
    }
#pragma unroll
    for (int c = 0; c < C::NB; ++c) {
      const int p = kbeg + load_row<TN, false>(c, wave, lane);
      X.nb[c] = n < P.N ? (uint32_t)(map_off(P.pmap, grid_pos(p, P.gh_log, P.gw_log)) + n) * 4u : FAR;
      X.vb[c] = X.nb[c];
    }
  }
}

// The offsets of the slice at X.k, once before its loads.
template <int TM, int TN, int MODE, int BT, bool TAP1>
__device__ __forceinline__ void wide_offsets(const ConvProb& P, int kend, int wave, int lane,
                                             WideCtx<TM, TN, MODE, BT, TAP1>& X) {
  using C = WideCtx<TM, TN, MODE, BT, TAP1>;
  if (C::FWD) {
    const Tap d = tap_of(P, TAP1 ? X.t : X.ka.t);
    const bool kok = TAP1 || X.k + X.kq < kend;
    if (!TAP1 || X.c == 0) {  // the rows under the tap's shift
      const int sh = ((d.dy << P.smap.w_log) + d.dx) * P.smap.ld + (TAP1 ? X.kq : X.ka.c);
#pragma unroll
      for (int c = 0; c < C::NA; ++c) {
        const bool ok = kok & ((unsigned)(X.y[c] + d.dy) < (1u << P.smap.h_log)) &
                        ((unsigned)(X.x[c] + d.dx) < (1u << P.smap.w_log));
        X.va[c] = ok ? (uint32_t)(X.off[c] + sh) * 4u : FAR;
      }
    }
    if (TAP1) {
      X.sa = (uint32_t)X.c * 4u;
      X.sb = (uint32_t)(C::B_RK ? d.wt * P.cs * P.N + X.c : (d.wt * P.cs + X.c) * P.N) * 4u;
    } else {
      const uint32_t w = (uint32_t)(d.wt * P.cs * P.N + X.ka.c) * 4u;
#pragma unroll
      for (int c = 0; c < C::NB; ++c) {
        if (C::B_RK) {
          X.vb[c] = kok ? X.nb[c] + w : FAR;
        } else {
          const bool in = X.k + load_row<TN, false>(c, wave, lane) < kend;
          X.vb[c] = in ? X.nb[c] + (uint32_t)((tap_of(P, X.kb[c].t).wt * P.cs + X.kb[c].c) * P.N) * 4u : FAR;
        }
      }
    }
  } else {
#pragma unroll
    for (int c = 0; c < C::NA; ++c) X.va[c] = X.gy[c] == X.gy_bad ? FAR : X.ab[c];
    if (X.k + SK_DEEP > kend) {  // a last slice that is not whole
#pragma unroll
      for (int c = 0; c < C::NA; ++c)
        if (X.k + load_row<TM, false>(c, wave, lane) >= kend) X.va[c] = FAR;
#pragma unroll
      for (int c = 0; c < C::NB; ++c)
        if (X.k + load_row<TN, false>(c, wave, lane) >= kend) X.vb[c] = FAR;
    }
  }
}
// On to the next slice, after the loads.
template <int TM, int TN, int MODE, int BT, bool TAP1>
__device__ __forceinline__ void wide_next(const ConvProb& P, WideCtx<TM, TN, MODE, BT, TAP1>& X) {
  using C = WideCtx<TM, TN, MODE, BT, TAP1>;
  X.k += SK_DEEP;
  if (C::FWD && TAP1) {
    X.c += SK_DEEP;
    if (X.c >= P.cs) {
      X.c = 0;
      ++X.t;
    }
  } else if (C::FWD) {
    advance(P, X.ka, X.dt, X.dc);
    if (!C::B_RK) {
#pragma unroll
      for (int c = 0; c < C::NB; ++c) advance(P, X.kb[c], X.dt, X.dc);
    }
  } else {
    // 32 / 2^gw_log grid rows on: both maps are linear in the grid row, across
    // images too (2^gh_log grid rows of sy source rows are an image).  A's
    // offsets advance per lane: a tap may start above the first image.
    const int rows = SK_DEEP >> P.gw_log;
    const uint32_t da = (uint32_t)(((rows * P.smap.sy) << P.smap.w_log) * P.smap.ld) * 4u;
    X.sb += (uint32_t)(((rows * P.pmap.sy) << P.pmap.w_log) * P.pmap.ld) * 4u;
#pragma unroll
    for (int c = 0; c < C::NA; ++c) {
      X.gy[c] = (X.gy[c] + rows) & ((1 << P.gh_log) - 1);
      X.ab[c] += da;
    }
  }
}

// Load `part` (A's, then B's) of the slice, into the stage at sa.
template <int TM, int TN, int MODE, int BT, bool TAP1>
__device__ __forceinline__ void wide_load(const WideCtx<TM, TN, MODE, BT, TAP1>& X, int part, int wave, float* sa,
                                          float* sb) {
  using C = WideCtx<TM, TN, MODE, BT, TAP1>;
  const bool is_a = part < C::NA;
  const int c = is_a ? part : part - C::NA;
  __builtin_amdgcn_raw_ptr_buffer_load_lds(is_a ? X.ra : X.rb, (lds_void*)((is_a ? sa : sb) + (4 * c + wave) * 256), 16,
                                           (int)(is_a ? X.va[c] : X.vb[c]), (int)(is_a ? X.sa : X.sb), 0, 0);
}

// LDS of a tile: two stages of this many floats.
template <int TM, int TN>
constexpr int STAGE_FLOATS = (TM + TN) * SK_DEEP;

// Stores of the tile: 16-row strips through the wave's own part of LDS (lds:
// 4 x 16 rows of TN / 2 + 4 floats).  Register r of lane l of a 32 x 32 tile is
// row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
template <int TM, int TN, int MODE>
__device__ __forceinline__ void wide_write(const ConvProb& P, const v16f (&acc)[TM / 64][TN / 64], int m0, int n0, int split,
                                           float slope, int wave, int lane, float* lds) {
  constexpr int W = TN / 2, PITCH = W + 4;
  static_assert(4 * 16 * PITCH <= STAGE_FLOATS<TM, TN>, "a stage holds the waves' strips");
  const int wm = (wave >> 1) * (TM / 2), wn = (wave & 1) * W;
  float* st = lds + wave * 16 * PITCH;
#pragma unroll
  for (int i = 0; i < TM / 64; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // the previous strip's reads are issued before these writes, and LDS runs
      // a wave's accesses in order
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < TN / 64; ++j)
#pragma unroll
        for (int r = 0; r < 8; ++r)
          st[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * PITCH + 32 * j + (lane & 31)] = acc[i][j][8 * h + r];
      __builtin_amdgcn_wave_barrier();
      store_strip<16, W, MODE>(P, m0 + wm + 32 * i + 16 * h, n0 + wn, split, slope, lane, st);
    }
}

// The tile: its sums over k kbeg .. kend - 1, in conv_kernel's order, and their
// stores.  stage0 and stage1 are two arrays, not one: a load into one stage is then seen not to
// touch the other, and reads of that one do not wait for it.  (wave: the
// wave's index, in a scalar register.)
template <int TM, int TN, int MODE, int BT, bool TAP1>
__device__ __forceinline__ void wide_tile(const ConvProb& P, int m0, int n0, int split, int kbeg, int kend, float slope,
                                          int wave, float* stage0, float* stage1) {
  using C = WideCtx<TM, TN, MODE, BT, TAP1>;
  constexpr int TI = TM / 64, TJ = TN / 64;  // 32 x 32 MFMA tiles per wave
  constexpr int AF = Stage<TM, C::A_RK>::FLOATS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wm = (wave >> 1) * (TM / 2), wn = (wave & 1) * (TN / 2);
  C X;
  wide_setup<TM, TN, MODE, BT, TAP1>(P, m0, n0, kbeg, wave, lane, X);
  v16f acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // WG: the bias gradient (the ones row of conv_kernel's product) by the first
  // row tile, one column per thread, in the products' order
  const bool sums = MODE == CONV_WG && m0 == 0 && P.ones_row >= 0 && tid < TN;
  float csum = 0.f;
  WideFrag<TI> A0, A1;
  WideFrag<TJ> B0, B1;
  constexpr int NL = C::NA + C::NB;
  static_assert(NL <= 8, "a load after each of a block's eight MFMA groups");
  auto frags = [&](const float* st, int kb, WideFrag<TI>& FA, WideFrag<TJ>& FB) {
    wide_frags<TM, C::A_RK, TI>(st, wm, kb, lane, FA);
    wide_frags<TN, C::B_RK, TJ>(st + AF, wn, kb, lane, FB);
  };
  auto mma = [&](const WideFrag<TI>& FA, const WideFrag<TJ>& FB, auto between) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(FA.v[i][e][u], FB.v[j][e][u], acc[i][j], 0, 0, 0);
        between(2 * u + e);
      }
  };
  // One slice, in stage cur; its first block's fragments are in A0, B0, the
  // next slice is on its way into stage nxt.  The barrier comes after the first
  // block's MFMAs: from there on every wave holds the second block's fragments
  // in registers, so the slice after the next may overwrite cur.
  auto step = [&](float* cur, float* nxt, int k0) {
    frags(cur, 16, A1, B1);
    if (MODE == CONV_WG && sums)
#pragma unroll
      for (int kb = 0; kb < SK_DEEP; kb += 16)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int g = 0; g < 4; ++g) csum += cur[AF + (kb + 4 * g + u) * TN + km_col(tid, 4 * g)];
    __builtin_amdgcn_sched_barrier(0);
    mma(A0, B0, [](int) {});
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's loads of the next slice have landed
    __syncthreads();
    if (k0 + SK_DEEP < kend) frags(nxt, 0, A0, B0);
    __builtin_amdgcn_sched_barrier(0);
    if (k0 + 2 * SK_DEEP < kend) {
      wide_offsets<TM, TN, MODE, BT, TAP1>(P, kend, wave, lane, X);
      mma(A1, B1, [&](int c) {
        __builtin_amdgcn_sched_barrier(0);
        if (c < NL) wide_load<TM, TN, MODE, BT, TAP1>(X, c, wave, cur, cur + AF);
        __builtin_amdgcn_sched_barrier(0);
      });
      wide_next<TM, TN, MODE, BT, TAP1>(P, X);
    } else {
      mma(A1, B1, [](int) {});
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto fill = [&](float* st) {
    wide_offsets<TM, TN, MODE, BT, TAP1>(P, kend, wave, lane, X);
#pragma unroll
    for (int c = 0; c < NL; ++c) wide_load<TM, TN, MODE, BT, TAP1>(X, c, wave, st, st + AF);
    wide_next<TM, TN, MODE, BT, TAP1>(P, X);
  };
  fill(stage0);
  if (kbeg + SK_DEEP < kend) fill(stage1);
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();
  frags(stage0, 0, A0, B0);
  for (int k0 = kbeg; k0 < kend; k0 += 2 * SK_DEEP) {
    step(stage0, stage1, k0);
    if (k0 + SK_DEEP < kend) step(stage1, stage0, k0 + SK_DEEP);
  }
  if (MODE == CONV_WG && sums && n0 + tid < P.N)
    as_global(P.C)[(int64_t)split * P.split_stride + (int64_t)P.brow * P.ldc + n0 + tid] = csum;
  __syncthreads();
  wide_write<TM, TN, MODE>(P, acc, m0, n0, split, slope, wave, lane, stage0);
}

}  // namespace

}  // namespace lipz
