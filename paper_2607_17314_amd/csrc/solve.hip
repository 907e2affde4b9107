// Triangular solves of the fit, L Y = R and L^T X = Y for many columns, with the inverses of
// L's 64 x 64 diagonal blocks: one launch per solve. A workgroup keeps its columns from the
// first block row to the last, two block rows (128 rows) at a time:
//   acc = L_{i,<i} Y_{<i}                    (back: (L^T)_{i,>i} X_{>i}), FP64 MFMA products
//   T_1 = R_1 - acc_1,  Y_1 = inv(L_11) T_1  for the first of the two block rows
//   acc_2 += L_21 Y_1,  T_2 = R_2 - acc_2,  Y_2 = inv(L_22) T_2  for the second.
// Every wave owns 16 NI columns and all 128 rows, so that the last two lines stay in its
// registers: the four registers of an MFMA result are the B operands of four MFMA steps. The
// products' operands go global -> registers -> LDS in the pipeline of gemm_f64.hip, L shared by
// the four waves.
//
// Bound: the FP64 matrix rate. As one product and one 64 x 64 product per block row, 48
// launches, the results so far were read again for every 64 rows and the remainder went
// through memory between the two: 1,500 rows, 58,200 columns, forward and back 6.85 ms
// (38 TFLOP/s over n^2 products a column and solve), here 5.16 (51; 64 at 65,536 columns,
// which are two whole rounds of workgroups).
#include "fit.hpp"
#include "tile_f64.hpp"

namespace xtc {

constexpr int SB64 = 64;          // rows of a diagonal block
constexpr int SM = 2 * SB64;      // rows of a step

// The row of a 16-row block at position p of an MFMA's A operand: turned so that a lane's four
// results (positions l / 16 + 4 r) are the consecutive rows 4 (l / 16) + r, and the matrix
// that they are multiplied by is read in 32-byte runs of its rows.
__device__ __forceinline__ int row_at(int p) { return 4 * (p & 3) + (p >> 2); }

template <bool BACK, int NI>
__global__ __launch_bounds__(256, 2) void k_solve(const double* __restrict__ L,
                                                  const double* __restrict__ linv, long n, long cn,
                                                  const double* C, long ldc, double* out, long ldo) {
  constexpr int MI = SM / 16, BN = 64 * NI;
  constexpr int SA = LDS_TILE<SM>, SBt = LDS_TILE<BN>;
  __shared__ __align__(16) double As[2 * SA];
  __shared__ __align__(16) double Bs[2 * SBt];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const long n0 = (long)blockIdx.x * BN, nw = n0 + 16 * NI * wave;   // first column, the wave's
  const int ra = lds_at<SM>(lk, row_at(li)), rb = lds_at<BN>(lk, 16 * NI * wave + li);
  d4 acc[MI][NI];

  // acc = the K products of rows i0 .. i0 + 127 of L (L^T) from A and the columns from B
  auto products = [&](const double* A, const double* B, long rows, long K) {
    int tp = tid;
    asm volatile("" : "+v"(tp));   // opaque: no offsets kept, as live registers, for the next step
    TileLoader<SM, !BACK, false, 1> la(A, BACK ? 1 : n, BACK ? n : 1, 0, rows, K, tp);
    TileLoader<BN, false, false, 1> lb(B, 1, ldo, n0, cn, K, tp);
    const int wa = la.store_at(tp), wb = lb.store_at(tp);
    double fa[2][MI], fb[2][NI];
    auto load = [&](auto whole, long k0) {
      if constexpr (whole.value) {
        la.load_whole(0);
        lb.load_whole(0);
      } else {
        la.load_any(0, k0);
        lb.load_any(0, k0);
      }
    };
    auto store = [&](auto whole, int buf, long k0) {   // the loaded tile, whose first k is k0
      if (!whole.value && k0 + GK > K) {
        la.mask(0, k0);
        lb.mask(0, k0);
      }
      la.store(0, As, wa + buf * SA);
      lb.store(0, Bs, wb + buf * SBt);
    };
    auto read = [&](int buf, int s) {
      int pa = ra + buf * SA, pb = rb + buf * SBt;
      keep_vector(pa);
      keep_vector(pb);
#pragma unroll
      for (int i = 0; i < MI; ++i) fa[s & 1][i] = As[pa + lds_at<SM>(4 * s, 0) + 16 * i];
#pragma unroll
      for (int j = 0; j < NI; ++j) fb[s & 1][j] = Bs[pb + lds_at<BN>(4 * s, 0) + 16 * j];
    };
    auto multiply = [&](int s) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s & 1][i], fb[s & 1][j], acc[i][j], 0, 0, 0);
    };
    auto reads_first = [&]() {   // the step's fragment reads go ahead of its MFMAs
      __builtin_amdgcn_sched_group_barrier(0x100, MI + NI, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, MI * NI, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    int buf = 0;
    // multiplies tile k0 - GK, stores tile k0 from the registers, requests tile k0 + GK
    auto tile = [&](auto w, long k0) {
      read(buf, 1);
      store(w, buf ^ 1, k0);
      load(w, k0 + GK);
      multiply(0);
      __builtin_amdgcn_sched_group_barrier(0x100, MI + NI, 0);
#pragma unroll
      for (int i = 0; i < MI * NI; ++i) {   // one LDS store and one load beside each MFMA
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      read(buf, 2);
      multiply(1);
      reads_first();
      read(buf, 3);
      multiply(2);
      reads_first();
      __builtin_amdgcn_s_waitcnt(0xc07f);   // LDS stores done before the barrier
      __syncthreads();
      buf ^= 1;
      read(buf, 0);
      multiply(3);
      reads_first();
    };
    constexpr std::true_type whole{};
    constexpr std::false_type any{};
    auto first = [&](auto w) {
      load(w, 0);
      store(w, 0, 0);
      load(w, GK);
    };
    if (2 * GK <= K) first(whole);
    else first(any);
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __syncthreads();
    read(0, 0);
    long k0 = GK;
    for (; k0 + 2 * GK <= K; k0 += GK) tile(whole, k0);
    for (; k0 < K; k0 += GK) tile(any, k0);
    read(buf, 1);
    multiply(0);
    read(buf, 2);
    multiply(1);
    read(buf, 3);
    multiply(2);
    multiply(3);
  };

  // to[i][j] += (fresh: =) the 64 x 64 matrix A (element (m, k) at m sm + k, back: m + k sk;
  // past mmax, kmax the last one) times from, whose registers are the B operands of the 16
  // MFMA steps as they are: step 4 b + r takes the k's 16 b + 4 lk + r. A is read two steps at
  // a time, the next two while two multiply.
  auto apply = [&](auto fresh, int el, int ek, const double* A, unsigned ld, int mmax, int kmax,
                   auto&& from, auto&& to) {
    const d4 zero = {0.0, 0.0, 0.0, 0.0};
    double f[2][4][2];
    unsigned row[4];
    asm volatile("" : "+v"(el), "+v"(ek));   // no addresses kept from one product for the next
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = 16 * i + row_at(el);
      row[i] = (unsigned)(m < mmax ? m : mmax) * (BACK ? 1 : ld);
    }
    auto fetch = [&](int s) {   // steps s and s + 1, s even
      const int k = 16 * (s / 4) + 4 * ek + s % 4;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if constexpr (BACK) {
#pragma unroll
          for (int e = 0; e < 2; ++e)
            f[s / 2 % 2][i][e] = A[row[i] + (unsigned)(k + e < kmax ? k + e : kmax) * ld];
        } else {
          __builtin_memcpy(f[s / 2 % 2][i], A + row[i] + k, 16);
        }
    };
    fetch(0);
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      if (s % 2 == 0 && s + 2 < 16) fetch(s + 2);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
          to(i, j) = __builtin_amdgcn_mfma_f64_16x16x4f64(f[s / 2 % 2][i][s % 2], from(s / 4, j)[s % 4],
                                                          fresh.value && s == 0 ? zero : to(i, j), 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  const long steps = (n + SM - 1) / SM;
  d4 y[4][NI];
  auto y_at = [&](int i, int j) -> d4& { return y[i][j]; };
  for (long st = 0; st < steps; ++st) {
    const long p = BACK ? steps - 1 - st : st, i0 = p * SM;
    const long kb = BACK ? i0 + SM : 0, K = BACK ? n - kb : i0;
    const bool two = i0 + SB64 < n;   // the second block row is there
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = (d4){0.0, 0.0, 0.0, 0.0};
    if (K > 0)
      products(BACK ? L + kb * n + i0 : L + i0 * n, out + kb * ldo, n - i0, K);
    // the lane's row and column go through an opaque move, so that the addresses below are
    // formed here and not hoisted, as live registers, out of the loop over the steps
    int el = li, ek = lk;
    asm volatile("" : "+v"(el), "+v"(ek));
    const double* L21 = L + (i0 + SB64) * n + i0;
    // block row h: acc = its right-hand sides less acc (zero past the matrix, for the product
    // that follows), y = inv(L_hh) acc, stored
    auto finish = [&](auto half) {
      constexpr int h = half.value;
      const long r0 = i0 + SB64 * h;
      const int left = (int)(n - r0 < SB64 ? n - r0 : SB64) - 4 * ek;   // this lane's rows: 16 i + r < left
      auto acc_at = [&](int i, int j) -> d4& { return acc[4 * h + i][j]; };
      long at[NI];
      bool in[NI];
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        in[j] = nw + el + 16 * j < cn;
        at[j] = (in[j] ? nw + el + 16 * j : cn - 1) + 4 * ek * ldc;
      }
      auto rhs = [&](auto full) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          double d[NI][4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const double* row = C + (r0 + 16 * i + r) * ldc;
#pragma unroll
            for (int j = 0; j < NI; ++j)
              d[j][r] = full.value || 16 * i + r < left ? row[at[j]] : 0.0;
          }
#pragma unroll
          for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              acc_at(i, j)[r] = full.value || 16 * i + r < left ? d[j][r] - acc_at(i, j)[r] : 0.0;
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      if (r0 + SB64 <= n) rhs(std::true_type{});
      else rhs(std::false_type{});
      apply(std::true_type{}, el, ek, linv + (2 * p + h) * SB64 * SB64, SB64, SB64 - 1, SB64 - 1, acc_at,
            y_at);
#pragma unroll
      for (int j = 0; j < NI; ++j) at[j] = nw + el + 16 * j + 4 * ek * ldo;
      auto put = [&](auto full) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            double* row = out + (r0 + 16 * i + r) * ldo;
#pragma unroll
            for (int j = 0; j < NI; ++j)
              if (full.value || (in[j] && 16 * i + r < left)) row[at[j]] = y[i][j][r];
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      if (r0 + SB64 <= n && nw + 16 * NI <= cn) put(std::true_type{});
      else put(std::false_type{});
    };
    const int last = (int)(n - 1 - (i0 + SB64));   // L21's last row within the matrix
    if constexpr (BACK) {
      if (two) {
        finish(std::integral_constant<int, 1>{});
        apply(std::false_type{}, el, ek, L21, (unsigned)n, SB64 - 1, last < SB64 - 1 ? last : SB64 - 1, y_at,
              [&](int i, int j) -> d4& { return acc[i][j]; });
      }
      finish(std::integral_constant<int, 0>{});
    } else {
      finish(std::integral_constant<int, 0>{});
      if (two) {
        apply(std::false_type{}, el, ek, L21, (unsigned)n, last < SB64 - 1 ? last : SB64 - 1, SB64 - 1, y_at,
              [&](int i, int j) -> d4& { return acc[4 + i][j]; });
        finish(std::integral_constant<int, 1>{});
      }
    }
    // the rows are read back by all four waves
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0)
    __syncthreads();
  }
}

xtc_status solve_columns(const double* L, const double* linv, long n, long cn, const double* C,
                         long ldc, double* out, long ldo, bool back, hipStream_t st) {
  XTC_REQUIRE(n > 0 && n < (1L << 22), "fit solve: bad number of rows");   // 32-bit offsets
  if (cn <= 0) return XTC_OK;
  // Whole rounds of workgroups per CU, a round of 64-column ones taking 0.58 of the time of a
  // round of 128-column ones. A fit of xi alone, 128- and 64-column workgroups: 1,500 rows,
  // 16,384 columns 4.31, 3.36 ms; 32,768: 4.74, 4.97; 40,000: 7.12, 6.59; 58,200: 7.68, 8.25;
  // 3,000 rows, 32,768: 14.9, 15.7. Up to 300 rows the two are within 7% of each other.
  const double wide = 1.0 * cdiv(cdiv(cn, 128), 256), narrow = 0.58 * cdiv(cdiv(cn, 64), 256);
  auto go = [&](auto B, auto NI) {
    hipLaunchKernelGGL((k_solve<B.value, NI.value>), dim3(cdiv(cn, 64 * NI.value)), dim3(256), 0, st, L,
                       linv, n, cn, C, ldc, out, ldo);
  };
  auto pick = [&](auto B) {
    if (wide <= narrow) go(B, std::integral_constant<int, 2>{});
    else go(B, std::integral_constant<int, 1>{});
  };
  if (back) pick(std::true_type{});
  else pick(std::false_type{});
  XTC_CHECK_LAUNCH();
  return XTC_OK;
}

}  // namespace xtc
