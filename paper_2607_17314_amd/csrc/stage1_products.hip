// FP64 stage 1 of the grid-pair contraction (see stage1_f64.hip) as matrix products
//   panel[ch][row][g] (+)= sum_g' A[row][g'] K_ch(g, g'),  A = [w xi ; w rho ; w rhot],
// in the pipeline of the FP64 GEMM (gemm_f64.hip): the B tile of 16 kets by NCH channels of
// 32 bra points is made in registers beside the MFMAs (EE form) or read from the pair-value
// buffer (BH form), and goes to LDS with the A tile of the same kets.
//
// Workgroup tile: 32 MI rows x 32 bra points, 256 threads = 4 waves 2 x 2, each 16 MI rows
// x 16 bra points of every channel. Bound: the FP64 pipe, which the matrix instructions and
// the pair generation (two pairs per thread and 16-ket step, ~65 vector instructions each)
// share: at MI = 4 the generation adds ~1/8 to the matrix instructions' time, against ~1/4
// at 64 rows. Every panel element sums its products in ket order. The Laplacian's fifth
// channel takes the registers of a fourth row block, so it runs with MI = 3.
// One of four bra shards of a ten-atom chain (58,200 points, N_mu 1,500, four channels):
// stage 1 314 -> 173 ms (32 -> 59 TFLOP/s of products alone; MFMA alone reaches 77.6); five
// channels, 17,200 points, N_mu 600: 80.5 -> 35.7 ms.
#include <type_traits>
#include "ee_pair.hpp"
#include "mfma_f64.hpp"

namespace xtc {

typedef __attribute__((address_space(1))) const double GlobalD;

// The A operand's share of a thread: rows m0 + tid / 16 + 16 i of ket k0 + tid % 16, times
// the ket's weight; rows n_mu and n_mu + 1 are rho and rhot, later ones (unused) rhot.
template <int N>
struct RowLoader {
  GlobalD* p[N];
  GlobalD* w;
  long n_g;
  int kf;
  double v[N], wv;

  __device__ __forceinline__ RowLoader(const double* w_, const double* xi, const double* rho,
                                       const double* rhot, long n_g_, int n_mu, long m0, int tid)
      : w((GlobalD*)w_), n_g(n_g_), kf(tid & 15) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const long r = m0 + (tid >> 4) + 16 * i;
      p[i] = (GlobalD*)(r < n_mu ? xi + r * n_g : (r == n_mu ? rho : rhot));
    }
  }
  __device__ __forceinline__ void load(bool whole, long k0) {
    long k = k0 + kf;
    if (!whole && k > n_g - 1) k = n_g - 1;
    wv = w[k];
    if (!whole && k0 + kf > n_g - 1) wv = -1.0;   // past the grid: no point's weight
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = p[i][k];
  }
  // kets past the grid are stored as zero; 0 * x of a point of weight zero is what it is
  template <int RT>
  __device__ __forceinline__ void store(bool whole, double* lds, int at) {
    keep_vector(at);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      double x = wv * v[i];
      if (!whole && wv < 0.0) x = 0.0;
      lds[at + 16 * i] = x;
    }
  }
};

// EE pair values: each thread makes the channels of bra tid % 32 with kets tid / 32 and
// tid / 32 + 8 of a 16-ket step (kets past the grid repeat its last point).
template <int NCH, int NQ, bool C1>
struct EEPairs {
  static constexpr bool BUFFER = false;
  struct Args {
    const double* xyz; long n_g; long b0; long bn; EECoef cf;
  };
  const Args& a;
  GlobalD* xyz;
  double q1[NQ], q2[NQ], q3[NQ];
  double bx, by, bz, kx[2], ky[2], kz[2];

  __device__ __forceinline__ EEPairs(const Args& a_, long bt, int tid) : a(a_), xyz((GlobalD*)a_.xyz) {
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      q1[j] = j < a.cf.n1 ? a.cf.q1[j] : 0.0;
      q2[j] = j < a.cf.n2 ? a.cf.q2[j] : 0.0;
      q3[j] = j < a.cf.n3 ? a.cf.q3[j] : 0.0;
    }
    long b = a.b0 + bt * 32 + (tid & 31);
    if (b > a.b0 + a.bn - 1) b = a.b0 + a.bn - 1;
    bx = xyz[b];
    by = xyz[a.n_g + b];
    bz = xyz[2 * a.n_g + b];
  }
  __device__ __forceinline__ void load(bool whole, long k0, int tid) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      long k = k0 + (tid >> 5) + 8 * h;
      if (!whole && k > a.n_g - 1) k = a.n_g - 1;
      kx[h] = xyz[k];
      ky[h] = xyz[a.n_g + k];
      kz[h] = xyz[2 * a.n_g + k];
    }
  }
  __device__ __forceinline__ void make(int h, double* out) const {
    const double dx = bx - kx[h], dy = by - ky[h], dz = bz - kz[h], d = a.cf.d;
    double r, rinv;
    sqrt_rsqrt(fma(dx, dx, fma(dy, dy, dz * dz)), r, rinv);
    const double t = recip(fma(d, r, 1.0));
    const double e = d * r * t;
    const double t2 = t * t;
    const double p1 = horner_fixed(q1, e);
    const double up = d * t2 * p1;
    const double f3 = d * d * t2 * t;
    double f = f3 * horner_fixed(q2, e);
    if (C1) f = fma(a.cf.c1 * d * t2, rinv, f);   // the o = 1 term; 0 at r = 0
    out[0] = f * dx;
    out[1] = f * dy;
    out[2] = f * dz;
    out[3] = up * up;
    if (NCH > 4) {
      double upp = d * d * t2 * t2 * horner_fixed(q3, e) - 2.0 * f3 * p1;
      if (C1 && r == 0.0) upp += 2.0 * f3 * a.cf.c1;   // the o = 1 term dropped at r = 0
      out[NCH - 1] = upp + 2.0 * f;
    }
  }
};

// BH pair values of one ket launch from the buffer pv64[64-bra tile][step][q][c][gk][gb], the
// pair (bra gb, ket 4 gk + q): two kets (tid / 32 and + 8) of one bra point per thread.
struct BHPairs {
  static constexpr bool BUFFER = true;
  struct Args {
    const double* pv64; long nsteps; long kbeg;
  };
  GlobalBytes next;
  unsigned off;
  double v[2][4];

  __device__ __forceinline__ BHPairs(const Args& a, long bt, int tid)
      : next((GlobalBytes)(a.pv64 + (bt >> 1) * a.nsteps * 4096)) {
    const int kq = tid >> 5;
    off = 8u * ((kq & 3) * 1024 + (kq >> 2) * 64 + (int)(bt & 1) * 32 + (tid & 31));
  }
  // the next step's values (steps come in order; `last` repeats the current one)
  __device__ __forceinline__ void load(bool advance) {
    GlobalBytes p = next;
    keep_scalar(p);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        unsigned o = off;
        keep_vector(o);
        v[h][c] = *(GlobalF64)(p + o + 8 * (c * 256 + h * 128));
      }
    if (advance) next += 8 * 4096;
  }
  __device__ __forceinline__ void make(int h, double* out) const {
#pragma unroll
    for (int c = 0; c < 4; ++c) out[c] = v[h][c];
  }
};

struct S1Args {
  const double* w; const double* xi; const double* rho; const double* rhot;
  long n_g; int n_mu; long bn; double* panel; long rows_pad; long bp;
  long kbeg; long kend;   // kets [kbeg, kend), kend - kbeg a multiple of 16 unless it is n_g
  int first;              // the panel is written, else added to
};

template <int NCH, int MI, class Pairs>
__global__ __launch_bounds__(256, 2) void k_stage1_products(S1Args s, typename Pairs::Args pa) {
  constexpr int RT = 32 * MI, BN = 32 * NCH;
  constexpr int SA = LDS_TILE<RT>, SB = LDS_TILE<BN>;
  __shared__ __align__(16) double As[2 * SA];
  __shared__ __align__(16) double Bs[2 * SB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const long m0 = (long)blockIdx.y * RT, bt = blockIdx.x;
  RowLoader<2 * MI> la(s.w, s.xi, s.rho, s.rhot, s.n_g, s.n_mu, m0, tid);
  Pairs pr(pa, bt, tid);
  const int wa = lds_at<RT>(tid & 15, tid >> 4);
  const int wb = lds_at<BN>(tid >> 5, tid & 31);   // ket tid / 32; ket + 8 is 8 BN + 136 on

  d4 acc[MI][NCH];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int c = 0; c < NCH; ++c) acc[i][c] = (d4){0.0, 0.0, 0.0, 0.0};
  const int li = lane & 15, lk = lane >> 4;
  const int ra = lds_at<RT>(lk, (RT / 2) * wm + li);
  const int rb = lds_at<BN>(lk, 16 * wn + li);
  double fa[2][MI], fb[2][NCH];
  auto read = [&](int buf, int st) {
    int oa = ra + buf * SA, ob = rb + buf * SB;
    keep_vector(oa);
    keep_vector(ob);
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[st & 1][i] = As[oa + lds_at<RT>(4 * st, 0) + 16 * i];
#pragma unroll
    for (int c = 0; c < NCH; ++c) fb[st & 1][c] = Bs[ob + lds_at<BN>(4 * st, 0) + 32 * c];
  };
  auto multiply = [&](int st) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int c = 0; c < NCH; ++c)
        acc[i][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[st & 1][i], fb[st & 1][c], acc[i][c], 0, 0, 0);
  };
  auto put = [&](int buf, int h) {   // one pair's channels to LDS
    double o[NCH];
    pr.make(h, o);
    int at = wb + buf * SB;
    keep_vector(at);
#pragma unroll
    for (int c = 0; c < NCH; ++c) Bs[at + lds_at<BN>(8 * h, 0) + 32 * c] = o[c];
  };
  auto load_pairs = [&](bool whole, long k0) {
    if constexpr (Pairs::BUFFER) pr.load(k0 + GK < s.kend);
    else pr.load(whole, k0, tid);
  };
  constexpr std::true_type whole{};
  constexpr std::false_type any{};
  int buf = 0;
  // multiplies tile k0 - GK, makes and stores tile k0, requests tile k0 + GK
  auto tile = [&](auto w, long k0) {
    read(buf, 1);
    la.template store<RT>(w.value, As, wa + (buf ^ 1) * SA);
    la.load(w.value, k0 + GK);
    multiply(0);
    __builtin_amdgcn_sched_group_barrier(0x100, MI + NCH, 0);
#pragma unroll
    for (int i = 0; i < MI * NCH; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      read(buf, 2 + h);
      put(buf ^ 1, h);
      multiply(1 + h);
      __builtin_amdgcn_sched_group_barrier(0x100, MI + NCH, 0);
#pragma unroll
      for (int i = 0; i < MI * NCH; ++i) {   // one pair's vector instructions beside the MFMAs
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);   // LDS stores and reads done before the barrier
    __syncthreads();
    buf ^= 1;
    read(buf, 0);
    load_pairs(w.value, k0 + GK);
    multiply(3);
    __builtin_amdgcn_sched_group_barrier(0x100, MI + NCH, 0);
    __builtin_amdgcn_sched_group_barrier(0x020, 8, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, MI * NCH, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  la.load(false, s.kbeg);
  load_pairs(false, s.kbeg);
  la.template store<RT>(false, As, wa);
  put(0, 0);
  put(0, 1);
  la.load(false, s.kbeg + GK);
  load_pairs(false, s.kbeg + GK);
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __syncthreads();
  read(0, 0);
  long k0 = s.kbeg + GK;
  const long kw = s.kend < s.n_g ? s.kend : s.n_g;
  for (; k0 + 2 * GK <= kw; k0 += GK) tile(whole, k0);
  for (; k0 < s.kend; k0 += GK) tile(any, k0);
  read(buf, 1);
  multiply(0);
  read(buf, 2);
  multiply(1);
  read(buf, 3);
  multiply(2);
  multiply(3);
  const long col = bt * 32 + 16 * wn + li;
  if (col >= s.bn) return;
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const long row = m0 + (RT / 2) * wm + 16 * i + lk;
      double* p = s.panel + ((long)c * s.rows_pad + row) * s.bp + col;
      double old[4] = {0.0, 0.0, 0.0, 0.0};
      if (!s.first)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row + 4 * r <= s.n_mu + 1) old[r] = p[4 * r * s.bp];
#pragma unroll
      for (int r = 0; r < 4; ++r)   // D[(l/16) + 4r][l%16]
        if (row + 4 * r <= s.n_mu + 1) p[4 * r * s.bp] = s.first ? acc[i][c][r] : old[r] + acc[i][c][r];
    }
}

xtc_status stage1_ee_f64(const Stage1Args& a, const EECoef& cf, hipStream_t st) {
  const S1Args s{a.w, a.xi, a.rho, a.rhot, a.n_g, a.n_mu, a.bn, a.panel, a.rows_pad, a.bp,
                 0, a.n_g, 1};
  auto go = [&](auto NCH, auto MI, auto NQ, auto C1) {
    using P = EEPairs<NCH.value, NQ.value, C1.value>;
    const typename P::Args pa{a.xyz, a.n_g, a.b0, a.bn, cf};
    const dim3 grid(cdiv(a.bn, 32), cdiv(a.n_mu + 2, 32 * MI.value));
    hipLaunchKernelGGL((k_stage1_products<NCH.value, MI.value, P>), grid, dim3(256), 0, st, s, pa);
  };
  auto with_c1 = [&](auto NCH, auto MI, auto NQ) {
    if (cf.c1 != 0.0) go(NCH, MI, NQ, std::true_type{});
    else go(NCH, MI, NQ, std::false_type{});
  };
  auto with_nq = [&](auto NCH, auto MI) {
    if (cf.n1 <= 8) with_c1(NCH, MI, std::integral_constant<int, 8>{});
    else with_c1(NCH, MI, std::integral_constant<int, MAXQ>{});
  };
  if (a.nch == 4) with_nq(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
  else with_nq(std::integral_constant<int, 5>{}, std::integral_constant<int, 3>{});
  XTC_CHECK_LAUNCH();
  return XTC_OK;
}

xtc_status stage1_pv_f64(const Stage1Args& a, long nsteps, long kbeg, hipStream_t st) {
  const S1Args s{a.w, a.xi, a.rho, a.rhot, a.n_g, a.n_mu, a.bn, a.panel, a.rows_pad, a.bp,
                 kbeg, kbeg + 16 * nsteps, kbeg == 0 ? 1 : 0};
  const BHPairs::Args pa{a.pv64, nsteps, kbeg};
  const dim3 grid(cdiv(a.bn, 32), cdiv(a.n_mu + 2, 128));
  hipLaunchKernelGGL((k_stage1_products<4, 4, BHPairs>), grid, dim3(256), 0, st, s, pa);
  XTC_CHECK_LAUNCH();
  return XTC_OK;
}

}  // namespace xtc
