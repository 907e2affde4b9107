// Shared pieces of the FP64 matrix-core kernels: the k-tile and its layout in LDS, and the
// address forms that keep the vector ALU (whose pipe the matrix instructions share) free.
#pragma once
#include "common.hpp"

namespace xtc {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int GK = 16;    // tile K

// Element (k, row) of a BT-row operand tile in LDS. Counted in 8-byte slots modulo the 32
// of one LDS pass, row 0 of k sits at 16 (k & 1) + 2 (k >> 1): the 16 rows by 2 k's that
// half a wave reads as MFMA fragments, the 16 k's by 2 rows that it stores of a
// k-contiguous operand and the 32 rows of one k that it stores of the others each fall
// into 32 different slots.
template <int BT>
__host__ __device__ __forceinline__ constexpr int lds_at(int k, int row) {
  return k * BT + (k >> 1) * 34 + (k & 1) * 16 + row;
}
template <int BT>
constexpr int LDS_TILE = GK * BT + (GK / 2) * 34;

// Pins a value to scalar registers, or a vector one as the base that constant offsets are
// added to: without them the compiler folds the scalar part of an address into a vector
// multiply-add per load, and a vector add per LDS store.
typedef const __attribute__((address_space(1))) char* GlobalBytes;
typedef const __attribute__((address_space(1))) double* GlobalF64;
__device__ __forceinline__ void keep_scalar(GlobalBytes& p) { asm("" : "+s"(p)); }
template <class T>
__device__ __forceinline__ void keep_vector(T& x) { asm("" : "+v"(x)); }

}  // namespace xtc
