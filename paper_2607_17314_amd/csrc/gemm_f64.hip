// Generic FP64 GEMM on CDNA4 matrix cores (v_mfma_f64_16x16x4f64) and small
// deterministic reductions. Used by the orbital GEMM, the fit (Gram, RHS,
// Cholesky updates, blocked triangular solves) and stage 2 of the contraction.
//
// Tiles of 128 x 128, 64 x 128 or 64 x 64 by 16, 256 threads = 4 wave64s arranged 2 x 2.
// Bound: the FP64 matrix rate (77.6 TFLOP/s measured in registers), and with it the issue
// slots: the matrix instructions share their pipe with the vector ALU and are issued in
// program order, so every address instruction between two of them counts. Operands go
// global -> registers -> LDS with one k-tile (64 x 64: two) in registers, one being
// multiplied and one being stored, one barrier per k-tile; fragments are double-buffered
// in registers so no MFMA waits for LDS. 8192 x 8192 x 4096: 55.5 -> 69.3 TFLOP/s (MFMA
// busy 92% of the cycles), 22,500 x 1,500 x 4,500: 51 -> 60, 64 x 58,200 x 1,408: 36.7 -> 46.
// Each output sums its products in the same order in every shape.
//
// MFMA 16x16x4 f64 register layout (per lane l of the wave):
//   A operand: A[l % 16][l / 16]      B operand: B[l / 16][l % 16]
//   D (4 doubles): D[(l / 16) + 4 r][l % 16], r = 0..3  (measured on gfx950)
#include "tile_f64.hpp"

namespace xtc {

// M tiles of one group: the 64 tiles in flight on an XCD then cover 8 row and 8 column panels
constexpr long GROUP_M = 8;

// The products of one launch (blockIdx.y), all of the same shape.
struct GemmList {
  GemmArgs g[GEMM_LIST];
};

// BM x BN output tile per workgroup, four waves 2 x 2.
template <int BM, int BN, bool A_KCONT, bool B_KCONT, bool SCALE, bool WIDE>
__global__ __launch_bounds__(256, 2) void k_gemm_f64(GemmList list) {
  const GemmArgs& g = list.g[blockIdx.y];
  constexpr int MI = BM / 32, NI = BN / 32;   // 16 x 16 blocks per wave
  constexpr int SA = LDS_TILE<BM>, SB = LDS_TILE<BN>;
  __shared__ __align__(16) double As[2 * SA];
  __shared__ __align__(16) double Bs[2 * SB];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  // Tile order: groups of GROUP_M M tiles, the M tile fastest within one, so the
  // workgroups that read the same panels of A and B run at the same time, and
  // consecutive workgroup ids (which the hardware deals to the 8 XCDs in turn) are
  // spread so that each XCD takes a contiguous run of tiles and shares those panels in
  // its own L2.
  const long n_mt = (g.M + BM - 1) / BM, n_nt = (g.N + BN - 1) / BN, n_tiles = n_mt * n_nt;
  const long per_xcd = (n_tiles + 7) / 8;
  const long t = (long)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (t >= n_tiles) return;   // the whole workgroup, before any barrier
  const long in_group = GROUP_M * n_nt, group = t / in_group, tg = t % in_group;
  const long gm = n_mt - group * GROUP_M < GROUP_M ? n_mt - group * GROUP_M : GROUP_M;
  const long m0 = (group * GROUP_M + tg % gm) * BM;
  const long n0 = (tg / gm) * BN;
  if (g.lower_only && m0 + BM - 1 < n0) return;

  constexpr int DEPTH = BM == 64 && BN == 64 ? 2 : 1;
  TileLoader<BM, A_KCONT, WIDE, DEPTH> la(g.A, g.a_sm, g.a_sk, m0, g.M, g.K, tid);
  TileLoader<BN, B_KCONT, WIDE, DEPTH> lb(g.B, g.b_sn, g.b_sk, n0, g.N, g.K, tid);
  const int wa = la.store_at(tid), wb = lb.store_at(tid);
  constexpr int NS = A_KCONT ? 1 : BM / 16;
  double sv[DEPTH][NS];
  auto load = [&](auto whole, int q, long k0) {
    if constexpr (whole.value) {
      la.load_whole(q);
      lb.load_whole(q);
    } else {
      la.load_any(q, k0);
      lb.load_any(q, k0);
    }
    if constexpr (SCALE) {
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const long k = k0 + la.k_of(i);
        sv[q][i] = g.s[whole.value || k < g.K ? k : g.K - 1];
      }
    }
  };
  auto store = [&](auto whole, int q, int buf, long k0) {   // the loaded tile, whose first k is k0
    if constexpr (SCALE) {
#pragma unroll
      for (int i = 0; i < BM / 16; ++i) la.v[q][i] *= sv[q][A_KCONT ? 0 : i];
    }
    if (!whole.value && k0 + GK > g.K) {
      la.mask(q, k0);
      lb.mask(q, k0);
    }
    la.store(q, As, wa + buf * SA);
    lb.store(q, Bs, wb + buf * SB);
  };

  d4 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = (d4){0.0, 0.0, 0.0, 0.0};

  const int li = lane & 15, lk = lane >> 4;
  const int ra = lds_at<BM>(lk, (BM / 2) * wm + li);
  const int rb = lds_at<BN>(lk, (BN / 2) * wn + li);
  // Fragments of MFMA step s (k = 4 s .. 4 s + 3) of a buffer, double-buffered in registers:
  // step s + 1's are read while step s multiplies, step 0 of the next tile's during step 3.
  double fa[2][MI], fb[2][NI];
  auto read = [&](int buf, int s) {
    int pa = ra + buf * SA, pb = rb + buf * SB;
    keep_vector(pa);
    keep_vector(pb);
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[s & 1][i] = As[pa + lds_at<BM>(4 * s, 0) + 16 * i];
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
  // DEPTH k-tiles in registers beside the one being multiplied: during step 0 the next tile goes
  // from registers to the other LDS buffer and the one DEPTH after it is requested, so the loads
  // have DEPTH tiles' time to arrive and the stores are long done at the barrier before step 3.
  constexpr std::true_type whole{};
  constexpr std::false_type any{};
  int buf = 0;
  auto reads_first = [&]() {   // the step's fragment reads go ahead of its MFMAs
    __builtin_amdgcn_sched_group_barrier(0x100, MI + NI, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, MI * NI, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // multiplies tile k0 - GK, stores tile k0 (from registers q), requests tile k0 + DEPTH GK
  auto tile = [&](auto w, int q, long k0) {
    read(buf, 1);
    store(w, q, buf ^ 1, k0);
    load(w, q, k0 + DEPTH * GK);
    multiply(0);
    // step 0: the fragment reads, then one LDS store and one load beside each MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, MI + NI, 0);
#pragma unroll
    for (int i = 0; i < MI * NI; ++i) {
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
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __syncthreads();
    buf ^= 1;
    read(buf, 0);
    multiply(3);
    reads_first();
  };
  long k0 = GK;
  auto first = [&](auto w) {
    load(w, 0, 0);
    store(w, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < DEPTH; ++q) load(w, q, (1 + q) * GK);
  };
  if ((DEPTH + 1) * GK <= g.K) first(whole);
  else first(any);
  __builtin_amdgcn_s_waitcnt(0xc07f);   // LDS stores done before the barrier
  __syncthreads();
  read(0, 0);
  for (; k0 + 2 * DEPTH * GK <= g.K; k0 += DEPTH * GK)
#pragma unroll
    for (int q = 0; q < DEPTH; ++q) tile(whole, q, k0 + q * GK);
  for (; k0 < g.K; k0 += DEPTH * GK)
#pragma unroll
    for (int q = 0; q < DEPTH; ++q)
      if (k0 + q * GK < g.K) tile(any, q, k0 + q * GK);
  read(buf, 1);
  multiply(0);
  read(buf, 2);
  multiply(1);
  read(buf, 3);
  multiply(2);
  multiply(3);
  // Epilogue, 16 rows at a time: the C (or D) and E values that the rows need are all
  // requested before the first is used. Whole tiles skip the bounds checks; offsets are a
  // per-thread part plus a scalar one.
  const long mt = m0 + (BM / 2) * wm, nt = n0 + (BN / 2) * wn;   // the wave's first row, column
  const double* D = g.D ? g.D : g.C;
  const long c0 = (mt + lk) * g.c_sm + (nt + li) * g.c_sn;
  const long e0 = (mt + lk) * g.e_sm + (nt + li) * g.e_sn;
  auto emit = [&](auto full) {
#pragma unroll
    for (int bi = 0; bi < MI; ++bi) {
      double d[NI][4], e[NI][4];
      auto in = [&](int bj, int r) {
        return full.value || (mt + lk + 16 * bi + 4 * r < g.M && nt + li + 16 * bj < g.N);
      };
      if (g.beta != 0.0)
#pragma unroll
        for (int bj = 0; bj < NI; ++bj)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (in(bj, r)) d[bj][r] = D[c0 + ((16 * bi + 4 * r) * g.c_sm + 16 * bj * g.c_sn)];
      if (g.epi == EPI_MUL_E)
#pragma unroll
        for (int bj = 0; bj < NI; ++bj)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (in(bj, r)) e[bj][r] = g.E[e0 + ((16 * bi + 4 * r) * g.e_sm + 16 * bj * g.e_sn)];
#pragma unroll
      for (int bj = 0; bj < NI; ++bj) {
        double sn = 1.0;
        if (g.sn && in(bj, 0)) sn = g.sn[nt + li + 16 * bj];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double v = g.alpha * acc[bi][bj][r];
          if (g.sn) v *= sn;
          if (g.beta != 0.0) v += g.beta * d[bj][r];
          if (g.epi == EPI_MUL_E) v *= e[bj][r];
          if (in(bj, r)) g.C[c0 + ((16 * bi + 4 * r) * g.c_sm + 16 * bj * g.c_sn)] = v;
        }
      }
    }
  };
  if (m0 + BM <= g.M && n0 + BN <= g.N) emit(whole);
  else emit(any);
}

template <int BM, int BN, bool WIDE = false>
static xtc_status launch_gemm(const GemmList& list, int n, hipStream_t st) {
  const GemmArgs& g = list.g[0];
  const long n_tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  const long n_wg = 8 * ((n_tiles + 7) / 8);
  if (n_wg > 0x7fffffffL) {
    set_error("gemm_f64: too many tiles for one launch");
    return XTC_ERR_INVALID_ARG;
  }
  const dim3 grid((unsigned)n_wg, (unsigned)n);
  const bool ak = (g.a_sk == 1), bk = (g.b_sk == 1);
  auto go = [&](auto A, auto B) {
    if (g.s)
      hipLaunchKernelGGL((k_gemm_f64<BM, BN, A.value, B.value, true, WIDE>), grid, dim3(256), 0, st, list);
    else
      hipLaunchKernelGGL((k_gemm_f64<BM, BN, A.value, B.value, false, WIDE>), grid, dim3(256), 0, st, list);
  };
  if (ak && bk) go(std::true_type{}, std::true_type{});
  else if (ak) go(std::true_type{}, std::false_type{});
  else if (bk) go(std::false_type{}, std::true_type{});
  else go(std::false_type{}, std::false_type{});
  XTC_CHECK_LAUNCH();
  return XTC_OK;
}

xtc_status gemm_f64(const GemmArgs& g, hipStream_t st) { return gemm_f64_list(&g, 1, st); }

xtc_status gemm_f64_list(const GemmArgs* gs, int count, hipStream_t st) {
  const GemmArgs& g = gs[0];
  XTC_REQUIRE(count >= 1 && count <= GEMM_LIST, "gemm_f64: bad number of products");
  // 32-bit offsets within a tile of at most 128 rows
  constexpr long FAR = 1L << 22;
  bool wide = false;
  GemmList list;
  for (int i = 0; i < count; ++i) {
    const GemmArgs& h = gs[i];
    XTC_REQUIRE(h.A32 == nullptr, "gemm_f64: FP32 operands are for the split GEMM only");
    XTC_REQUIRE(h.M == g.M && h.N == g.N && h.K == g.K && (h.a_sk == 1) == (g.a_sk == 1) &&
                    (h.b_sk == 1) == (g.b_sk == 1) && !h.s == !g.s && h.lower_only == g.lower_only,
                "gemm_f64: the products of one launch must have one shape");
    wide = wide || h.a_sm >= FAR || h.b_sn >= FAR;
    list.g[i] = h;
  }
  if (g.M <= 0 || g.N <= 0) return XTC_OK;
  if (g.K <= 0) {
    set_error("gemm_f64: K must be positive");
    return XTC_ERR_INVALID_ARG;
  }
  // Time of a shape, in units of one element at the full rate of one of the 256 CUs: whole
  // rounds of tiles per CU (one workgroup alone keeps a CU's matrix pipes about as busy as
  // several) over the rate that the shape reaches at 8192 x 8192 x 4096.
  auto tiles = [&](long bm, long bn) {
    const long mt = (g.M + bm - 1) / bm, nt = (g.N + bn - 1) / bn;
    return count * (g.lower_only ? (mt * nt + (mt > nt ? mt : nt)) / 2 : mt * nt);
  };
  auto cost = [&](long bm, long bn, double rate) {
    return (double)((tiles(bm, bn) + 255) / 256 * bm * bn) / rate;
  };
  if (wide) return launch_gemm<64, 64, true>(list, count, st);
  // up to two tiles per CU the smallest shape ends first: its tiles are in flight together
  // (60 x 17,200 x 60: 11.5 us against 13.4 with 64 x 128 tiles)
  if (tiles(64, 64) <= 512) return launch_gemm<64, 64>(list, count, st);
  const double c1 = cost(128, 128, 69.0), c2 = cost(64, 128, 66.0), c3 = cost(64, 64, 64.0);
  if (c1 <= c2 && c1 <= c3) return launch_gemm<128, 128>(list, count, st);
  if (c2 <= c3) return launch_gemm<64, 128>(list, count, st);
  return launch_gemm<64, 64>(list, count, st);
}

// ---------------------------------------------------------------------------
// Deterministic FP64 sum: 256-thread blocks, each block sums a contiguous
// stretch in a fixed shuffle/LDS tree; a second single-block pass sums the
// partials in order.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

__device__ double block_sum_256(double v) {
  __shared__ double part[4];
  v = wave_sum(v);
  int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) part[wave] = v;
  __syncthreads();
  double r = (part[0] + part[1]) + (part[2] + part[3]);
  return r;
}

__global__ __launch_bounds__(256) void k_reduce_stage(const double* x, long n, long per_block,
                                                      double* out) {
  long b0 = (long)blockIdx.x * per_block;
  long b1 = b0 + per_block < n ? b0 + per_block : n;
  double v = 0.0;
  for (long i = b0 + threadIdx.x; i < b1; i += 256) v += x[i];
  v = block_sum_256(v);
  if (threadIdx.x == 0) out[blockIdx.x] = v;
}

xtc_status reduce_sum_f64(const double* x, long n, double* out, double* scratch, hipStream_t st) {
  // scratch must hold 1024 doubles
  long per = (n + 1023) / 1024;
  if (per < 256) per = 256;
  unsigned nb = cdiv(n, per);
  if (nb == 0) nb = 1;
  hipLaunchKernelGGL(k_reduce_stage, dim3(nb), dim3(256), 0, st, x, n, per, scratch);
  XTC_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_reduce_stage, dim3(1), dim3(256), 0, st, (const double*)scratch, (long)nb,
                     (long)nb, out);
  XTC_CHECK_LAUNCH();
  return XTC_OK;
}

}  // namespace xtc
