// The operand tiles of the FP64 matrix-core products whose operands lie in memory, on their
// way through registers to LDS.
#pragma once
#include <type_traits>
#include "mfma_f64.hpp"

namespace xtc {

// One operand's share of a thread: BT / 16 elements of each BT x 16 tile, in registers
// between the load and the store to LDS.
//   KCONT:  element i is (row tid / 16 + 16 i, k tid % 16);
//   else:   element i is (row tid % BT, k tid / BT + (256 / BT) i), k uniform over a wave.
// Rows past the operand's end read its last row (their products are not stored); k's past
// K read K - 1 and are zeroed before the store (mask), tiles past the last one read it again.
// The matrix instructions share their pipe with the vector ALU, so the addresses are kept
// off it: a scalar pointer that moves with k plus per-thread byte offsets that stay, 32-bit
// (WIDE: 64-bit, for row strides of 2^22 elements and more).
template <int BT, bool KCONT, bool WIDE, int DEPTH>
struct TileLoader {
  static constexpr int N = BT / 16;
  static constexpr int G = 256 / BT;
  using Off = typename std::conditional<WIDE, unsigned long, unsigned>::type;
  GlobalBytes base;   // the tile's first row, k = 0
  GlobalBytes next;   // the first element of the next whole tile for this thread's wave
  long sk, K, step;
  Off off[KCONT ? N : 1];
  int k_first;
  double v[DEPTH][N];

  __device__ __forceinline__ TileLoader(const double* X, long s_row, long s_k, long r0, long rows,
                                        long K_, int tid)
      : base((GlobalBytes)(X + r0 * s_row)), sk(8 * s_k), K(K_) {
    if constexpr (KCONT) {
      k_first = tid & 15;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        long r = (tid >> 4) + 16 * i;
        if (r > rows - 1 - r0) r = rows - 1 - r0;
        off[i] = (Off)(8 * (r * s_row + k_first));
      }
      next = base;
      step = 0;
    } else {
      long r = tid % BT;
      if (r > rows - 1 - r0) r = rows - 1 - r0;
      off[0] = (Off)(8 * r * s_row);
      k_first = __builtin_amdgcn_readfirstlane(tid / BT);
      next = base + k_first * sk;
      step = G * sk;
    }
  }
  __device__ __forceinline__ int k_of(int i) const {   // k of element i within the tile
    return KCONT ? k_first : k_first + G * i;
  }
  // The next tile, all of whose k's are below K; tiles come in order.
  __device__ __forceinline__ void load_whole(int q) {
    GlobalBytes p = next;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      keep_scalar(p);
      Off o = off[KCONT ? i : 0];
      if constexpr (!WIDE) keep_vector(o);
      v[q][i] = *(GlobalF64)(p + o);
      if constexpr (!KCONT) p += step;
    }
    next += GK * sk;
  }
  // The tile from k0: k's past K read K - 1.
  __device__ __forceinline__ void load_any(int q, long k0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const long k = k0 + k_of(i) < K ? k0 + k_of(i) : K - 1;
      v[q][i] = *(GlobalF64)(base + (KCONT ? off[KCONT ? i : 0] + 8 * (k - k_first) : k * sk + off[0]));
    }
  }
  __device__ __forceinline__ void mask(int q, long k0) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (k0 + k_of(i) >= K) v[q][i] = 0.0;
  }
  __device__ __forceinline__ void store(int q, double* lds, int at) const {   // at: store_at + buffer
    keep_vector(at);
#pragma unroll
    for (int i = 0; i < N; ++i) lds[at + (KCONT ? 16 * i : lds_at<BT>(G * i, 0))] = v[q][i];
  }
  __device__ __forceinline__ int store_at(int tid) const {
    return lds_at<BT>(k_first, KCONT ? tid >> 4 : tid % BT);
  }
};

}  // namespace xtc
