// Device code shared by the convolution kernels (conv.hip, conv_wide.hip, conv_split.hip):
// bounded loads, position maps and tap shifts of a ConvProb; the stores of
// the wide tiles.
#pragma once

#include "lipz_internal.h"
#include "split.h"

namespace lipz {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

namespace {

constexpr int NT = 256;
// A byte offset past every operand extent the host accepts: such a buffer
// load returns 0.
constexpr uint32_t OOB = 0x7FFFFFF0u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const float* p, uint32_t bytes) {
  // dword 3 = 0x00020000: raw 32-bit data format on gfx9-family parts
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float4 ld4(__amdgpu_buffer_rsrc_t r, uint32_t off_bytes) {
  const v4u v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off_bytes, 0, 0);
  return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]),
                     __uint_as_float(v[3]));
}
__device__ __forceinline__ float ld1(__amdgpu_buffer_rsrc_t r, uint32_t off_bytes) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off_bytes, 0, 0));
}

// Blocks are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous range of logical tiles so neighbouring tiles share its L2.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
  const int q = nb >> 3, r = nb & 7;
  const int x = b & 7, i = b >> 3;
  return x * q + (x < r ? x : r) + i;
}

struct Pos {
  int img, y, x;
};
__device__ __forceinline__ Pos grid_pos(int p, int gh, int gw) {
  return {p >> (gh + gw), (p >> gw) & ((1 << gh) - 1), p & ((1 << gw) - 1)};
}

// Tap t -> (row shift, column shift) of the gathered operand, and its
// weight-tap index kh * kw_full + kw.
struct Tap {
  int dy, dx, wt;
};
__device__ __forceinline__ Tap tap_of(const ConvProb& P, int t) {
  const int a = t >> P.tw_log, b = t & ((1 << P.tw_log) - 1);
  return {a * P.tys + P.ty0, b * P.tys + P.tx0, (a * P.khs + P.kh0) * P.kw_full + (b * P.khs + P.kw0)};
}

// k index of the tap-expanded operand -> (tap, channel).
__device__ __forceinline__ void split_k(const ConvProb& P, int k, int& t, int& c) {
  if (P.cs_log >= 0) {
    t = k >> P.cs_log;
    c = k & (P.cs - 1);
  } else if (P.taps <= 1) {
    t = 0;
    c = k;
  } else {
    t = k / P.cs;
    c = k - t * P.cs;
  }
}

// Byte offset of channel c of S at grid position q shifted by tap d, or OOB.
__device__ __forceinline__ uint32_t src_off(const ConvProb& P, Pos q, Tap d, int c) {
  const int sy = q.y * P.smap.sy + d.dy;
  const int sx = q.x * P.smap.sx + d.dx;
  if ((unsigned)sy >= (1u << P.smap.h_log) || (unsigned)sx >= (1u << P.smap.w_log)) return OOB;
  const int pos = (((q.img << P.smap.h_log) + sy) << P.smap.w_log) + sx;
  return (uint32_t)(pos * P.smap.ld + c) * 4u;
}

// Element offset (floats) of grid position q under a position map.
__device__ __forceinline__ int map_off(const PosMap& m, Pos q) {
  const int y = q.y * m.sy + m.y0, x = q.x * m.sx + m.x0;
  return ((((q.img << m.h_log) + y) << m.w_log) + x) * m.ld;
}

// The wide tiles (conv_wide.hip, conv_split.hip) run K in 32-deep slices of
// whole float4s.
constexpr int SK_DEEP = 32;              // K of one slice
constexpr uint32_t FAR = 0x80000000u;    // a byte offset that stays past every extent when an extent is added

// (tap, channel) of one float4, advanced by 32 k per slice.
struct KPos {
  int t, c;
};
__device__ __forceinline__ KPos kpos(const ConvProb& P, int k) {
  KPos q;
  split_k(P, k, q.t, q.c);
  return q;
}
__device__ __forceinline__ void advance(const ConvProb& P, KPos& q, int dt, int dc) {
  q.t += dt;
  q.c += dc;
  if (q.c >= P.cs) {
    q.c -= P.cs;
    ++q.t;
  }
}

// Stores of a strip of ROWS rows of a wave's part of the tile, from the wave's
// own part of LDS (rows of W + 4 floats), where the caller put its sums: as
// float4, whole rows of the strip per instruction.  The wave takes rows
// m0 .. m0 + ROWS - 1, columns n0 .. n0 + W - 1.
template <int ROWS, int W, int MODE>
__device__ __forceinline__ void store_strip(const ConvProb& P, int m0, int n0, int split, float slope, int lane, const float* st) {
  constexpr int PITCH = W + 4;
  constexpr int RQ = 64 / (W / 4);                    // rows one float4 pass of the wave covers
  const int c4 = (lane % (W / 4)) * 4, rq = lane / (W / 4);
  const int n = n0 + c4;
  LIPZ_GLOBAL float* gC = as_global(P.C);
  float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
  int coff[4];
  if (MODE == CONV_WG) {
    gC += (int64_t)split * P.split_stride;
#pragma unroll
    for (int e = 0; e < 4; ++e) coff[e] = P.n_inner ? ((n + e) / P.n_inner) * P.n_tap_stride + (n + e) % P.n_inner : n + e;
  } else if (P.epi == EPI_BIAS_ACT && P.bias && n < P.N) {
    const LIPZ_GLOBAL float* gb = as_global(P.bias) + n;
    bias = make_float4(gb[0], gb[1], gb[2], gb[3]);
  }
#pragma unroll 2
  for (int q = 0; q < ROWS / RQ; ++q) {
    const int row = m0 + RQ * q + rq;
    float4 v = *reinterpret_cast<const float4*>(st + (RQ * q + rq) * PITCH + c4);
    if (MODE == CONV_WG) {
      if (row < P.taps * P.cs && n < P.N) {
        int t, c;
        split_k(P, row, t, c);
        LIPZ_GLOBAL float* o = gC + (int64_t)(tap_of(P, t).wt * P.cs + c) * P.ldc;
        if (P.n_inner) {
          o[coff[0]] = v.x;
          o[coff[1]] = v.y;
          o[coff[2]] = v.z;
          o[coff[3]] = v.w;
        } else {
          *reinterpret_cast<LIPZ_GLOBAL v4f*>(o + n) = v4f{v.x, v.y, v.z, v.w};
        }
      }
    } else if (row < P.M && n < P.N) {
      const int64_t o = (int64_t)map_off(P.omap, grid_pos(row, P.gh_log, P.gw_log)) + n;
      if (P.epi == EPI_BIAS_ACT) {
        v = make_float4(act_fwd(P.act, v.x + bias.x, slope), act_fwd(P.act, v.y + bias.y, slope),
                        act_fwd(P.act, v.z + bias.z, slope), act_fwd(P.act, v.w + bias.w, slope));
      } else if (P.epi == EPI_DACT) {
        const v4f x = *reinterpret_cast<const LIPZ_GLOBAL v4f*>(as_global(P.aux) + o);
        v = make_float4(v.x * act_deriv_from_out(P.act, x[0], slope), v.y * act_deriv_from_out(P.act, x[1], slope),
                        v.z * act_deriv_from_out(P.act, x[2], slope), v.w * act_deriv_from_out(P.act, x[3], slope));
      }
      *reinterpret_cast<LIPZ_GLOBAL v4f*>(gC + o) = v4f{v.x, v.y, v.z, v.w};
    }
  }
}

}  // namespace

}  // namespace lipz
