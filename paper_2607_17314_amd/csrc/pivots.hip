// Interpolation-point selection: weight-scaled fixed-rank pivoted Cholesky
// (ISDF section, Alg. 1; matrix-free pivot search) for the scalar and gradient
// channels, fused by the fill-to-target rule.
//
// The pivots are Alg. 1's greedy ones; what is reorganised is how the residual
// column of each pivot is formed. A plain step reads the orbital rows (N_orb, or
// 4 N_orb for the gradient channel) and every earlier factor row L[0..mu) at all
// grid points, so a channel of n steps streams ~n (4 N_orb + n / 2) rows of N_g
// doubles from HBM. Here the steps run in batches around a speculative candidate
// set: at a batch start with mu0 pivots, C = the 64 points of largest residual
// diagonal d (ties to the lowest index), and one set of FP64 matrix-core GEMMs
// forms their columns against every grid point,
//   R[c][g] = S(g, c) - sum_{l < mu0} L[l][g] L[l][c],
// from the orbitals at the candidates and the factor rows gathered there. While the
// exact argmax g* of d over all points is a candidate, its factor row needs only R[g*]
// and the rows made in this batch,
//   L[mu][g] = (R[g*][g] - sum_{mu0 <= l < mu} L[l][g] L[l][g*]) / sqrt(d_g*),
// and the first pivot outside C ends the batch (the next batch's C holds it, as
// the largest d). The selected points, the stop rules and the fused order are
// those of the plain algorithm; the sums are grouped differently, so the factor
// agrees with a plain step's to rounding.
//
// The steps of a batch are not launched one by one (a pick and a column launch of ~4 us
// each, whatever their work): the greedy sequence among the candidates needs only the
// 64 x 64 values R[c][c'] and is made in advance, then replayed at every point:
//   k_top_local / k_top_merge  the previous batch's accepted rows taken off d, and the
//                  64 largest d with their points;
//   k_plan   (one block)  the greedy sequence among the candidates: pivots g_t, their d_t
//                  and the factor entries L[l][g_t], up to NPLAN steps or the
//                  rank-deficiency stop;
//   k_replay (grid)  the factor rows of all planned steps at every point; a point whose
//                  d exceeds d_t before step t marks that step: the argmax was not g_t.
// The steps before the first marked one are the plain algorithm's; the host, which reads
// the plan and the marks once per batch, records them. Ties go to the lowest grid index
// and every sum has a fixed order, so repeated runs select identical pivots.
// 1,733 steps of an eight-atom chain (46,560 points) in 79 batches: 34.2 -> 17.1 ms, of
// which the products 7.1, plan and replay 4.5, candidate search 2.0 (9.0 with LDS sorts).
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <utility>
#include "common.hpp"
#include "plans.hpp"
#include "timing.hpp"

namespace xtc {

constexpr int PIV_BLOCK = 256;
constexpr double RANK_TOL = 1e-14;
constexpr int NCAND = 64;      // candidates per batch (one 64-row GEMM tile)
constexpr int NPLAN = 48;      // steps planned per batch: a factor entry per VGPR pair in the
                               // replay, and about twice the 20-30 steps a batch accepts
constexpr int TOP_PTS = 512;   // points per block of the candidate search

// The planned steps of a batch (k_plan) and what the replay found (k_replay).
struct PivPlan {
  int steps;              // planned steps T
  int stop;               // 1: the best candidate after them is at or below the rank tolerance
  int mark[NPLAN + 1];    // step t (or the stop after T steps): some point's d is larger
  int slot[NPLAN];        // candidate slot of step t's pivot
  long g[NPLAN + 1];      // step t's pivot (entry T: the best candidate left at a stop)
  double d[NPLAN + 1];    // its residual diagonal before the step
  double lstar[NPLAN][NPLAN];   // lstar[t][l] = L[mu0 + l][g_t], l < t
};

struct Cand {
  double d;
  long g;
};

__device__ __forceinline__ Cand better(Cand a, Cand b) {
  if (a.d > b.d) return a;
  if (b.d > a.d) return b;
  return a.g <= b.g ? a : b;
}

// channel: 0 scalar, 1 gradient. A point whose d is NaN gets the d = 0 that its first factor
// entry would leave it: the search below compares d's and would lose others to a NaN.
__global__ __launch_bounds__(PIV_BLOCK) void k_diag(const double* __restrict__ phi4,
                                                    const double* __restrict__ w, long n_g,
                                                    int n_orb, int channel,
                                                    double* __restrict__ d) {
  long g = (long)blockIdx.x * PIV_BLOCK + threadIdx.x;
  if (g < n_g) {
    double n2 = 0.0, g2 = 0.0;
    for (int p = 0; p < n_orb; ++p) {
      double v = phi4[(long)p * n_g + g];
      n2 += v * v;
    }
    double dd;
    if (channel == 0) {
      dd = w[g] * w[g] * n2 * n2;
    } else {
      for (int q = 0; q < 3 * n_orb; ++q) {
        double v = phi4[(long)(n_orb + q) * n_g + g];
        g2 += v * v;
      }
      dd = w[g] * w[g] * n2 * g2;
    }
    d[g] = dd == dd ? dd : 0.0;
  }
}

// --- the candidate search: the NCAND best (d, index) pairs -----------------------
// A wave holds one sorted list of 64, best first (larger d, then lower index).
constexpr Cand NO_CAND{-1.0, 0x7fffffffffffffffL};   // below every residual diagonal (d >= 0)

__device__ __forceinline__ Cand shfl_cand(Cand c, int lane) {
  return Cand{__shfl(c.d, lane, 64), __shfl(c.g, lane, 64)};
}

// one compare-exchange with lane ^ j; the lower lane keeps the better entry if best_first
__device__ __forceinline__ Cand exchange(Cand c, int lane, int j, bool best_first) {
  const Cand o = shfl_cand(c, lane ^ j);
  const bool other = o.d > c.d || (o.d == c.d && o.g < c.g);
  return other == (((lane & j) == 0) == best_first) ? o : c;
}

__device__ __forceinline__ Cand sort64(Cand c, int lane) {
#pragma unroll
  for (int k = 2; k <= 64; k <<= 1)
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) c = exchange(c, lane, j, (lane & k) == 0);
  return c;
}

// the 64 best of two sorted lists, sorted
__device__ __forceinline__ Cand merge64(Cand a, Cand b, int lane) {
  a = better(a, shfl_cand(b, 63 - lane));
#pragma unroll
  for (int j = 32; j > 0; j >>= 1) a = exchange(a, lane, j, true);
  return a;
}

// whether any entry of list c would enter the sorted list `kept`
__device__ __forceinline__ bool enters(Cand kept, Cand c) {
  const Cand last = shfl_cand(kept, 63);
  return __any(c.d > last.d || (c.d == last.d && c.g < last.g));
}

// merges the lists of a block's waves (W a power of two) in LDS; wave 0 returns the result
template <int W>
__device__ __forceinline__ Cand block_merge(Cand c, double (*sd)[64], long (*sg)[64], int lane,
                                            int wave) {
  for (int h = W / 2; h > 0; h >>= 1) {
    if (wave >= h && wave < 2 * h) {
      sd[wave][lane] = c.d;
      sg[wave][lane] = c.g;
    }
    __syncthreads();
    if (wave < h) c = merge64(c, Cand{sd[wave + h][lane], sg[wave + h][lane]}, lane);
    __syncthreads();
  }
  return c;
}

// Points [TOP_PTS blockIdx.x, ...): the previous batch's n_acc accepted rows L[mu0 ..] are
// taken off d, then the 64 best points of the block.
__global__ __launch_bounds__(256) void k_top_local(double* __restrict__ d, long n_g,
                                                   const double* __restrict__ L, long mu0,
                                                   int n_acc, const PivPlan* __restrict__ plan,
                                                   double* __restrict__ out_d,
                                                   long* __restrict__ out_g) {
  __shared__ double sd[4][64];
  __shared__ long sg[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Cand kept = NO_CAND;
  for (int i = 0; i < TOP_PTS / 256; ++i) {
    const long g = (long)blockIdx.x * TOP_PTS + 256 * i + threadIdx.x;
    Cand c = NO_CAND;
    if (g < n_g) {
      double dn = d[g];
      if (n_acc > 0) {
        for (int t0 = 0; t0 < n_acc; t0 += 8) {   // eight rows' loads in flight
          double col[8];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            col[u] = L[(mu0 + (t0 + u < n_acc ? t0 + u : n_acc - 1)) * n_g + g];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            if (t0 + u >= n_acc) break;
            dn = dn - col[u] * col[u];
            dn = dn > 0.0 ? dn : 0.0;
            if (g == plan->g[t0 + u]) dn = 0.0;
          }
        }
        d[g] = dn;
      }
      c = Cand{dn, g};
    }
    if (i == 0) kept = sort64(c, lane);
    else if (enters(kept, c)) kept = merge64(kept, sort64(c, lane), lane);
  }
  kept = block_merge<4>(kept, sd, sg, lane, wave);
  if (wave == 0) {
    out_d[(long)blockIdx.x * NCAND + lane] = kept.d;
    out_g[(long)blockIdx.x * NCAND + lane] = kept.g;
  }
}

// The 64 best of the blocks' lists: the candidates, best first (-1 where there are fewer).
__global__ __launch_bounds__(1024) void k_top_merge(const double* __restrict__ in_d,
                                                    const long* __restrict__ in_g, int n_lists,
                                                    long n_g, long* __restrict__ cand) {
  __shared__ double sd[16][64];
  __shared__ long sg[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Cand kept = NO_CAND;
  for (int l = wave; l < n_lists; l += 16) {
    const Cand c{in_d[(long)l * NCAND + lane], in_g[(long)l * NCAND + lane]};
    if (enters(kept, c)) kept = merge64(kept, c, lane);
  }
  kept = block_merge<16>(kept, sd, sg, lane, wave);
  if (wave == 0) cand[lane] = kept.g >= 0 && kept.g < n_g ? kept.g : -1;
}

// Every factor entry, planned or replayed, sums x[l] y[l], l < t, in one order: four
// accumulators over whole groups of sixteen and the rest in the first.
template <class F, int... I>
__device__ __forceinline__ void for_each_int(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

// max over the wave by row shifts and broadcasts (no LDS round trips); NaNs are passed over
__device__ __forceinline__ double wave_max(double v) {
  auto shifted = [](double x, auto ctrl) {
    const long b = __builtin_bit_cast(long, x);
    const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, ctrl.value, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), ctrl.value, 0xf, 0xf, false);
    return __builtin_bit_cast(double, (long)(unsigned)lo | ((long)hi << 32));
  };
  v = fmax(v, shifted(v, std::integral_constant<int, 0x111>{}));   // row_shr 1, 2, 4, 8
  v = fmax(v, shifted(v, std::integral_constant<int, 0x112>{}));
  v = fmax(v, shifted(v, std::integral_constant<int, 0x114>{}));
  v = fmax(v, shifted(v, std::integral_constant<int, 0x118>{}));
  v = fmax(v, shifted(v, std::integral_constant<int, 0x142>{}));   // row_bcast 15, 31
  v = fmax(v, shifted(v, std::integral_constant<int, 0x143>{}));
  const long b = __builtin_bit_cast(long, v);
  const int lo = __builtin_amdgcn_readlane((int)b, 63), hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
  return __builtin_bit_cast(double, (long)(unsigned)lo | ((long)hi << 32));
}

// The greedy sequence among the candidates, at most `lim` steps; d0max <= 0: the channel's
// first batch, whose first pivot sets the rank tolerance. One wave, compile-time steps.
__global__ __launch_bounds__(256) void k_plan(const double* __restrict__ R,
                                              const double* __restrict__ d, long n_g,
                                              const long* __restrict__ cand, int lim,
                                              double d0max, PivPlan* __restrict__ plan) {
  __shared__ double Rc[NCAND][NCAND + 1];
  __shared__ double Lb[NPLAN][NCAND + 1];
  for (int e = threadIdx.x; e < NCAND * NCAND; e += 256) {
    const long g = cand[e % NCAND];
    Rc[e / NCAND][e % NCAND] = g >= 0 ? R[(long)(e / NCAND) * n_g + g] : 0.0;
  }
  if (threadIdx.x <= NPLAN) plan->mark[threadIdx.x] = 0;
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  const long gc = cand[lane];
  double dc = gc >= 0 ? d[gc] : -1.0;
  double col[NPLAN];
  int T = 0, stop = 0;
  auto step = [&](auto tc) {
    constexpr int t = tc.value;
    if (t >= lim || stop) return;
    const double bd = wave_max(dc);
    // the lowest grid index among the lanes that hold the maximum (one, but for ties)
    unsigned long hold = __ballot(dc == bd);
    int bs = hold ? __builtin_ctzl(hold) : 0;   // none: NaN, which stops below
    long bg = __shfl(gc, bs, 64);
    for (hold &= hold - 1; hold; hold &= hold - 1) {
      const int o = __builtin_ctzl(hold);
      const long og = __shfl(gc, o, 64);
      if (og < bg) {
        bg = og;
        bs = o;
      }
    }
    bs = __builtin_amdgcn_readfirstlane(bs);
    if (t == 0 && d0max <= 0.0) d0max = bd;
    if (lane == 0) {
      plan->g[t] = bg;
      plan->d[t] = bd;
    }
    if (!(bd > RANK_TOL * d0max)) {
      stop = 1;
      return;
    }
    if (lane == 0) plan->slot[t] = bs;
    if (lane < t) plan->lstar[t][lane] = Lb[lane][bs];
    const double inv = 1.0 / sqrt(bd);
    double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int l = 0; l < t; ++l) {
      const int q = l < (t & ~15) ? l & 3 : 0;
      a[q] = fma(col[l], Lb[l][bs], a[q]);
    }
    col[t] = (Rc[bs][lane] - ((a[0] + a[1]) + (a[2] + a[3]))) * inv;
    Lb[t][lane] = col[t];
    __builtin_amdgcn_s_waitcnt(0xc07f);   // one wave: the store is done before the next reads
    double dn = dc - col[t] * col[t];
    dn = dn > 0.0 ? dn : 0.0;
    if (gc >= 0) dc = lane == bs ? 0.0 : dn;
    T = t + 1;
  };
  for_each_int(step, std::make_integer_sequence<int, NPLAN>{});
  if (lane == 0) {
    plan->steps = T;
    plan->stop = stop;
  }
}

// The planned steps at every point: the factor rows L[mu0 + t], and a mark on each step
// before which the point's d is larger than the planned pivot's.
__global__ __launch_bounds__(PIV_BLOCK) void k_replay(const double* __restrict__ R, long n_g,
                                                      const double* __restrict__ d,
                                                      double* __restrict__ L, long mu0,
                                                      PivPlan* __restrict__ plan_rw,
                                                      const PivPlan* __restrict__ plan) {
  const long g = (long)blockIdx.x * PIV_BLOCK + threadIdx.x;
  const bool in = g < n_g;
  const long gg = in ? g : n_g - 1;
  double dn = d[gg];
  double col[NPLAN];
  const int T = plan->steps, stop = plan->stop;
  constexpr int AHEAD = 8;   // R loads in flight ahead of their step
  double r[AHEAD];
  auto request = [&](int t) {
    return R[(long)plan->slot[t < T ? t : (T > 0 ? T - 1 : 0)] * n_g + gg];
  };
  if (T > 0)
#pragma unroll
    for (int t = 0; t < AHEAD; ++t) r[t] = request(t);
  auto check = [&](int t) {
    const double dt = plan->d[t];
    const long gt = plan->g[t];
    if (__any(in && (dn > dt || (dn == dt && g < gt))) && (threadIdx.x & 63) == 0)
      plan_rw->mark[t] = 1;
  };
  auto step = [&](auto tc) {   // compile-time t: the point's factor entries stay in registers
    constexpr int t = tc.value;
    if (t >= T) return;
    if (t > 0) check(t);   // the first pivot is the largest d by construction
    const double rt = r[t % AHEAD];
    r[t % AHEAD] = request(t + AHEAD);
    const double inv = 1.0 / sqrt(plan->d[t]);
    double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int l = 0; l < t; ++l) {
      const int q = l < (t & ~15) ? l & 3 : 0;
      a[q] = fma(col[l], plan->lstar[t][l], a[q]);
    }
    col[t] = (rt - ((a[0] + a[1]) + (a[2] + a[3]))) * inv;
    if (in) L[(mu0 + t) * n_g + g] = col[t];
    dn = dn - col[t] * col[t];
    dn = dn > 0.0 ? dn : 0.0;
    if (g == plan->g[t]) dn = 0.0;
  };
  for_each_int(step, std::make_integer_sequence<int, NPLAN>{});
  if (stop && T > 0) check(T);
}

// The orbital values and factor entries at the candidates, candidate-major:
// Ac[m][k] = phi4 row k at cand[m] (k < nrows), Lc[m][l] = L[l][cand[m]] (l < mu0),
// wc[m] = w[cand[m]]; rows of missing candidates are zero.
__global__ __launch_bounds__(256) void k_gather_cand(const double* __restrict__ phi4,
                                                     const double* __restrict__ w, long n_g,
                                                     int nrows, const double* __restrict__ L,
                                                     int mu0, int ldl,
                                                     const long* __restrict__ cand,
                                                     double* __restrict__ Ac,
                                                     double* __restrict__ Lc,
                                                     double* __restrict__ wc) {
  const long per = (long)nrows + mu0;
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= NCAND * per) return;
  const int m = (int)(i / per);
  const long k = i % per;
  const long g = cand[m];
  if (k < nrows) {
    Ac[(long)m * nrows + k] = g >= 0 ? phi4[k * n_g + g] : 0.0;
    if (k == 0) wc[m] = g >= 0 ? w[g] : 0.0;
  } else {
    const long l = k - nrows;
    Lc[(long)m * ldl + l] = g >= 0 ? L[l * n_g + g] : 0.0;
  }
}

// S(g, c) from the orbital dot products: scalar w_g w_c a^2, gradient w_g w_c a b,
// with a = R2 (gradient) or R (scalar) and b = R (gradient).
__global__ __launch_bounds__(256) void k_pair_values(double* __restrict__ R,
                                                     const double* __restrict__ R2,
                                                     const double* __restrict__ w,
                                                     const double* __restrict__ wc, long n_g,
                                                     int channel) {
  const long g = (long)blockIdx.x * 256 + threadIdx.x;
  const int m = blockIdx.y;
  if (g >= n_g) return;
  double* r = R + (long)m * n_g + g;
  if (channel == 0) {
    const double a = *r;
    *r = w[g] * wc[m] * a * a;
  } else {
    const double a = R2[(long)m * n_g + g];
    *r = w[g] * wc[m] * a * *r;
  }
}

struct SelLayout {
  double* d; double* L; PivPlan* plan; long* cand; double* R; double* R2; double* Ac; double* Lc;
  double* wc; double* td; long* tg;
  int n_lists, ldl;
};

static SelLayout layout_sel(Arena& ar, int64_t n_g, int n_orb, int n_mu) {
  SelLayout S;
  S.n_lists = (int)cdiv(n_g, TOP_PTS);
  S.ldl = n_mu > 0 ? n_mu : 1;
  S.d = ar.take<double>(n_g);
  S.L = ar.take<double>((size_t)n_mu * n_g);
  S.plan = ar.take<PivPlan>(1);
  S.cand = ar.take<long>(NCAND);
  S.R = ar.take<double>((size_t)NCAND * n_g);
  S.R2 = ar.take<double>((size_t)NCAND * n_g);
  S.Ac = ar.take<double>((size_t)NCAND * 4 * n_orb);
  S.Lc = ar.take<double>((size_t)NCAND * S.ldl);
  S.wc = ar.take<double>(NCAND);
  S.td = ar.take<double>((size_t)S.n_lists * NCAND);
  S.tg = ar.take<long>((size_t)S.n_lists * NCAND);
  return S;
}

size_t ws_select(int64_t n_g, int n_orb, int n_mu, int mode) {
  (void)mode;
  Arena ar(nullptr, 0);
  layout_sel(ar, n_g, n_orb, n_mu);
  return ar.used;
}

// XTC_PROGRESS set in the environment: long host loops report their progress on stderr
// at the points where they synchronise anyway.
static bool progress_enabled() {
  static const bool on = getenv("XTC_PROGRESS") != nullptr;
  return on;
}

// Opens a batch: the previous batch's n_acc accepted rows (before mu0) taken off d, the
// candidate search, and the candidates' columns R against every point (GEMMs on the
// orbitals and the mu0 factor rows).
static xtc_status open_batch(const double* phi4, const double* w, long n_g, int n_orb,
                             int channel, int mu0, int n_acc, SelLayout& S, hipStream_t st) {
  hipLaunchKernelGGL(k_top_local, dim3(S.n_lists), dim3(256), 0, st, S.d, n_g,
                     (const double*)S.L, (long)(mu0 - n_acc), n_acc, (const PivPlan*)S.plan, S.td,
                     S.tg);
  XTC_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_top_merge, dim3(1), dim3(1024), 0, st, (const double*)S.td,
                     (const long*)S.tg, S.n_lists, n_g, S.cand);
  XTC_CHECK_LAUNCH();
  const int nrows = channel == 0 ? n_orb : 4 * n_orb;
  hipLaunchKernelGGL(k_gather_cand, dim3(cdiv((long)NCAND * (nrows + mu0), 256)), dim3(256), 0, st,
                     phi4, w, n_g, nrows, S.L, mu0, S.ldl, S.cand, S.Ac, S.Lc, S.wc);
  XTC_CHECK_LAUNCH();
  // a[c][g] = sum_p phi_p(c) phi_p(g) (into R2 for the gradient channel)
  GemmArgs g{};
  g.M = NCAND; g.N = n_g; g.K = n_orb;
  g.A = S.Ac; g.a_sm = nrows; g.a_sk = 1;
  g.B = phi4; g.b_sk = n_g; g.b_sn = 1;
  g.C = channel == 0 ? S.R : S.R2; g.c_sm = n_g; g.c_sn = 1;
  XTC_TRY(gemm_f64(g, st));
  if (channel != 0) {
    // b[c][g] = sum_{x, p} d_x phi_p(c) d_x phi_p(g)
    GemmArgs h{};
    h.M = NCAND; h.N = n_g; h.K = 3L * n_orb;
    h.A = S.Ac + n_orb; h.a_sm = nrows; h.a_sk = 1;
    h.B = phi4 + (long)n_orb * n_g; h.b_sk = n_g; h.b_sn = 1;
    h.C = S.R; h.c_sm = n_g; h.c_sn = 1;
    XTC_TRY(gemm_f64(h, st));
  }
  hipLaunchKernelGGL(k_pair_values, dim3(cdiv(n_g, 256), NCAND), dim3(256), 0, st, S.R, S.R2, w,
                     S.wc, n_g, channel);
  XTC_CHECK_LAUNCH();
  if (mu0 > 0) {
    // R -= Lc L: what the mu0 earlier pivots already explain
    GemmArgs l{};
    l.M = NCAND; l.N = n_g; l.K = mu0;
    l.A = S.Lc; l.a_sm = S.ldl; l.a_sk = 1;
    l.B = S.L; l.b_sk = n_g; l.b_sn = 1;
    l.C = S.R; l.c_sm = n_g; l.c_sn = 1;
    l.alpha = -1.0; l.beta = 1.0;
    XTC_TRY(gemm_f64(l, st));
  }
  return XTC_OK;
}

// Runs one channel: its pivots to `piv` in order, at most max_steps. target > 0: stops after
// the pivot with which the union with `mark` (an entry per grid point, updated) holds target
// points. *deficient: the channel ended at the rank tolerance.
static xtc_status run_channel(const double* phi4, const double* w, long n_g, int n_orb, int channel,
                              int max_steps, SelLayout& S, std::vector<char>& mark, int target,
                              std::vector<long>& piv, hipStream_t st, int* deficient) {
  hipLaunchKernelGGL(k_diag, dim3(cdiv(n_g, PIV_BLOCK)), dim3(PIV_BLOCK), 0, st, phi4, w, n_g,
                     n_orb, channel, S.d);
  XTC_CHECK_LAUNCH();
  PivPlan h;
  int done = 0, n_acc = 0, batches = 0, stop = 0, guess = NPLAN;
  int in_union = 0;
  for (char m : mark) in_union += m;
  double d0max = 0.0;
  while (done < max_steps && !stop) {
    ++batches;
    XTC_TRY(open_batch(phi4, w, n_g, n_orb, channel, done, n_acc, S, st));
    // steps past the last accepted one are made for nothing: plan a few more than the
    // previous batch accepted
    const int lim = max_steps - done < guess ? max_steps - done : guess;
    hipLaunchKernelGGL(k_plan, dim3(1), dim3(256), 0, st, (const double*)S.R, (const double*)S.d,
                       n_g, (const long*)S.cand, lim, d0max, S.plan);
    XTC_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_replay, dim3(cdiv(n_g, PIV_BLOCK)), dim3(PIV_BLOCK), 0, st,
                       (const double*)S.R, n_g, (const double*)S.d, S.L, (long)done, S.plan,
                       (const PivPlan*)S.plan);
    XTC_CHECK_LAUNCH();
    XTC_HIP(hipMemcpyAsync(&h, S.plan, offsetof(PivPlan, lstar), hipMemcpyDeviceToHost, st));
    XTC_HIP(hipStreamSynchronize(st));
    n_acc = 0;
    while (n_acc < h.steps && !h.mark[n_acc] && !stop) {
      const long g = h.g[n_acc++];
      XTC_REQUIRE(g >= 0 && g < n_g, "isdf_select_points: the pivot search left the grid "
                                     "(non-finite orbital values or weights?)");
      piv.push_back(g);
      if (!mark[g]) {
        mark[g] = 1;
        ++in_union;
      }
      if (target > 0 && in_union >= target) stop = 2;   // the completing pivot is recorded
    }
    if (!stop && h.stop && n_acc == h.steps && !h.mark[h.steps]) stop = 1;
    // the batch's first pick is the largest d, its first candidate: no progress and no
    // stop means the search and the plan disagree, which only non-finite values cause
    if (n_acc == 0 && !stop) {
      set_error("isdf_select_points: the pivot search made no progress (non-finite orbital "
                "values or weights?)");
      return XTC_ERR_INVALID_ARG;
    }
    if (d0max <= 0.0) d0max = h.d[0];
    guess = n_acc + 12 < NPLAN ? n_acc + 12 : NPLAN;
    if (progress_enabled() && (done + n_acc) / 1024 != done / 1024)
      fprintf(stderr, "isdf_select_points: %s channel, %d steps done (%d batches)\n",
              channel == 0 ? "scalar" : "gradient", done + n_acc, batches);
    done += n_acc;
  }
  *deficient = stop == 1;
  return XTC_OK;
}

}  // namespace xtc

using namespace xtc;

xtc_status xtc_select_qr(const double* phi4, const xtc_grid* grid, int n_orb, int n_mu,
                         int64_t* pivots, int32_t* n_mu_out, double* info, Arena& ar,
                         hipStream_t st);
xtc_status xtc_select_learned(const double* phi4, const xtc_grid* grid, int n_orb, int n_occ,
                              int n_mu, int mode, const xtc_mlp* mlp, double fallback_factor,
                              int64_t* pivots, int32_t* n_mu_out, double* info, Arena& ar,
                              hipStream_t st);

xtc_status xtc_select_qr(const double* phi4, const xtc_grid* grid, int n_orb, int n_mu,
                         int64_t* pivots, int32_t* n_mu_out, double* info, Arena& ar,
                         hipStream_t st) {
  const long n_g = grid->n_g;
  const size_t mark = ar.used;
  SelLayout S = layout_sel(ar, n_g, n_orb, n_mu);
  XTC_TRY(need_ws(ar));
  // gradient channel to ceil(n_mu / 2) pivots, then the scalar channel until the union
  // reaches n_mu
  std::vector<char> in_union(n_g, 0);
  std::vector<long> hg, hs;
  int defg = 0, defs = 0;
  XTC_TRY(run_channel(phi4, grid->w, n_g, n_orb, 1, (n_mu + 1) / 2, S, in_union, 0, hg, st, &defg));
  const int ng = (int)hg.size();
  if (ng < n_mu)
    XTC_TRY(run_channel(phi4, grid->w, n_g, n_orb, 0, n_mu, S, in_union, n_mu, hs, st, &defs));
  const int ns = (int)hs.size();
  // fused order: scalar pivots in selection order, then gradient-only pivots
  std::vector<char> in_s(n_g, 0);
  int n = 0;
  for (int i = 0; i < ns; ++i) {
    pivots[n++] = hs[i];
    in_s[hs[i]] = 1;
  }
  for (int i = 0; i < ng && n < n_mu; ++i)
    if (!in_s[hg[i]]) pivots[n++] = hg[i];
  *n_mu_out = n;
  if (info) {
    info[0] = ns;
    info[1] = ng;
  }
  ar.used = mark;
  return n < n_mu ? XTC_WARN_RANK_DEFICIENT : XTC_OK;
}

extern "C" xtc_status isdf_select_points(const double* phi4, const xtc_grid* grid, int32_t n_orb,
                                         int32_t n_occ, int32_t n_mu_target, int32_t mode,
                                         const xtc_mlp* mlp, double fallback_factor,
                                         int64_t* pivots, int32_t* n_mu_out, double* info,
                                         void* ws, size_t ws_bytes, void* stream);

extern "C" xtc_status isdf_select_points(const double* phi4, const xtc_grid* grid, int32_t n_orb,
                                         int32_t n_occ, int32_t n_mu_target, int32_t mode,
                                         const xtc_mlp* mlp, double fallback_factor,
                                         int64_t* pivots, int32_t* n_mu_out, double* info,
                                         void* ws, size_t ws_bytes, void* stream) {
  XTC_REQUIRE(phi4 && grid && pivots && n_mu_out, "isdf_select_points: null argument");
  XTC_REQUIRE(grid->n_g > 0 && grid->w, "isdf_select_points: empty grid");
  XTC_REQUIRE(n_orb > 0 && n_mu_target > 0 && n_mu_target <= grid->n_g,
              "isdf_select_points: bad sizes");
  XTC_REQUIRE(mode == XTC_SELECT_QR || mode == XTC_SELECT_LEARNED ||
                  mode == XTC_SELECT_LEARNED_JUDGED,
              "isdf_select_points: unknown mode");
  XTC_REQUIRE(mode == XTC_SELECT_QR || mlp, "isdf_select_points: learned modes need an mlp");
  if (info)
    for (int i = 0; i < 8; ++i) info[i] = 0.0;
  XTC_TRY(check_weights(grid, ws, ws_bytes, as_stream(stream), "isdf_select_points"));
  Arena ar(ws, ws_bytes);
  size_t tk = timing_begin(TM_SELECT, as_stream(stream));
  xtc_status s = mode == XTC_SELECT_QR
                     ? xtc_select_qr(phi4, grid, n_orb, n_mu_target, pivots, n_mu_out, info, ar,
                                     as_stream(stream))
                     : xtc_select_learned(phi4, grid, n_orb, n_occ, n_mu_target, mode, mlp,
                                          fallback_factor, pivots, n_mu_out, info, ar,
                                          as_stream(stream));
  timing_end(tk, as_stream(stream));
  return s;
}
