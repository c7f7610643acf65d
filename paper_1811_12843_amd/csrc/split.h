// fp32 products on the bf16 matrix cores.
//
// An fp32 value is the sum of three bf16 values, x = x0 + x1 + x2: x0 is x
// rounded to nearest, x1 the remainder rounded to nearest, x2 what is left,
// which fits bf16's 8 significand bits (|x1| <= 2^-8 |x|, |x2| <= 2^-17 |x|).
// A product is the six piece products x_i y_j with i + j <= 2, each exact in
// fp32, summed into fp32 accumulators; the three left out are together at most
// (2^-24 + 2^-34) |x y|, what rounding the product to fp32 may take.  Six bf16
// MFMAs take 6/16 of the matrix-core time of the fp32 MFMAs for the same product.
//
// Operands are scaled by 2^16 before they are split, and sums by 2^-32: bf16's
// smallest subnormal is 2^-133, so a scaled operand's pieces hold all its bits
// down to fp32's smallest subnormal (unscaled, those of |x| < 2^-110 do not: with
// operands of 2^-120 the results' rms error was 3.5e-5).  Operands and sums too
// large for the scale come out as non-finite ones do.
//
// x0 y0 has accumulators of its own, added to those of the five smaller
// products at the end: a bf16 MFMA drops product bits below its accumulator's
// last place, towards minus infinity, and in one accumulator for all six that
// is a bias on every sum.  Measured, one wave's 32 x 32 tiles of normal data, K =
// 1024, against fp64, relative to the rms result: fp32 MFMAs rms error
// 5.8e-7, mean error 1e-9; six products into one accumulator 4.9e-7, -5.6e-8;
// two accumulators 1.9e-7, -1e-9.  On sums of one sign, K = 16384, rms and mean
// of fp32 MFMAs 1.7e-6 and 8e-8, of two accumulators 6.0e-7 and -6e-8.
//
// A non-finite operand, and a finite one that the scale or the rounding takes
// past bf16's largest value, give non-finite pieces and NaN sums where fp32
// products may give an infinity or a number.  Kernels test their accumulators;
// a tile with a non-finite one is multiplied again, by fp32 MFMAs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lipz {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// (a, b) rounded to bf16, a in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef float v2f __attribute__((ext_vector_type(2)));
  typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{a, b}), v2bf));
}

// True when v is an infinity or NaN (also under finite-math assumptions).
__device__ __forceinline__ bool non_finite(float v) { return (__float_as_uint(v) & 0x7F800000u) == 0x7F800000u; }

constexpr float SPLIT_SCALE = 0x1p16f, SPLIT_UNSCALE = 0x1p-32f;

// The three pieces of two scaled values, packed.
__device__ __forceinline__ void split2(float a, float b, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
  a *= SPLIT_SCALE;
  b *= SPLIT_SCALE;
  p0 = pack_bf16(a, b);
  const float a1 = a - __uint_as_float(p0 << 16), b1 = b - __uint_as_float(p0 & 0xFFFF0000u);
  p1 = pack_bf16(a1, b1);
  p2 = pack_bf16(a1 - __uint_as_float(p1 << 16), b1 - __uint_as_float(p1 & 0xFFFF0000u));
}

// LDS tiles of one bf16 piece of an operand slice, 32 k deep.
//
// RK ("row, k"): row r holds its 32 k in four 16-byte chunks of 8 k, chunk
// g stored at place g ^ ((r / 2) % 4): the 8 rows that one phase of a
// ds_read_b128 touches then lie on 8 different 16-byte bank groups.
//
// KM ("k, column"): row k holds the operand's columns; pitch 2 C + 32 bytes,
// so the four k rows x 32 bytes that 16 lanes of a transposing read touch lie
// on different banks.
constexpr int RK_PITCH = 64;
__device__ __forceinline__ int rk_off(int row, int g) { return row * RK_PITCH + ((g ^ ((row >> 1) & 3)) << 4); }
constexpr int km_pitch(int cols) { return 2 * cols + 32; }

// v_mfma_f32_32x32x16_bf16 operand fragment of lane l: row (or column)
// l % 32, k 8 (l / 32) .. + 7.  From an RK tile: one 16-byte read.
__device__ __forceinline__ v8bf rk_frag(const char* tile, int row0, int kk, int lane) {
  return *reinterpret_cast<const v8bf*>(tile + rk_off(row0 + (lane & 31), 2 * kk + (lane >> 5)));
}
// From a KM tile: two transposing reads.  In each, lane i of a group of 16
// gives the address of 4 columns (4 (i % 4)) of k row i / 4 and receives
// column i of the group's four k rows.
template <int COLS>
__device__ __forceinline__ v8bf km_frag(const char* tile, int col0, int kk, int lane) {
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef short v8s __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) v4s lds_v4s;
  constexpr int PITCH = km_pitch(COLS);
  const int i = lane & 15;
  const char* p = tile + (16 * kk + 8 * (lane >> 5) + (i >> 2)) * PITCH + (col0 + 16 * ((lane >> 4) & 1) + 4 * (i & 3)) * 2;
  const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)p);
  const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(p + 4 * PITCH));
  return __builtin_bit_cast(v8bf, (v8s{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]}));
}

}  // namespace lipz
