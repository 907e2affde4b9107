// The split path's pair values of the BH correlator (bh.hpp) with their nuclear sums on the
// FP64 matrix cores. For a pair (bra g, ket g')
//   F_o = sum_I sum_m a_I(g)^m gamma_{I,o,m}(g'),  d_c F_o = sum_I sum_{m>0} m a_I^{m-1} d_c a_I gamma_{I,o,m}
// are products over k = (I, m), m = 1..3, of four bra operands (a^m and m a^{m-1} d_c a) with
// four ket operands (gamma_o), plus the m = 0 terms, which depend on the ket alone: per bra
// and ket point 16 sums, one MFMA block of 16 kets x 16 bra points each, so a lane ends with
// every sum of its four pairs (one bra point, kets lane / 16 + 4 r) and finishes them in
// registers, with one bra point's density sums to carry.
//
// Workgroup: 8 waves over 32 bra points (2 halves) x 64 kets (4 steps of 16), for the GCH ket
// chunks of its group. The bra operand of the tile stays in LDS; the ket operand goes through
// two LDS buffers of four nuclei (three MFMA steps) each, the next four made while the current
// ones multiply. Bound: the FP64 pipe, which the matrix instructions (16 per four k's, 3 n_nuc
// k's) share with the finish (~170 vector instructions a pair: square root, reciprocal, the
// channels, their splits and the density sums). Against one thread per two pairs walking the
// nuclei over LDS tables (96 bytes of LDS per pair and nucleus), ten nuclei, 58,200 points,
// mean of launches of up to 16,384 x 16,384 pairs: 9.09 -> 5.85 ms (10.0 ms with the bra points along a
// lane's rows, whose four points' density sums no longer fit the registers; 7.23 ms with the
// compiler's FP64 to FP16 conversion).
#include "bh.hpp"
#include "ee_pair.hpp"
#include "half_round.hpp"
#include "stage1_split.hpp"
#include "stage1_split_bh.hpp"

namespace xtc {

constexpr int BPN = 4;         // nuclei per ket buffer
constexpr int BPK = 3 * BPN;   // its k's
constexpr int BPT = 64;        // kets per group
constexpr long KT_BUF = 4L * BPK * BPT;            // doubles per ket buffer [o][k][ket]
constexpr long ST_DOUBLES = 4L * 4096 / 4;         // staged halves of four k-steps
constexpr long KT_DOUBLES = 2 * KT_BUF > ST_DOUBLES ? 2 * KT_BUF : ST_DOUBLES;

static int bra_k(int nn) { return (3 * nn + 3) / 4 * 4; }

// LDS: ket buffers (the staged fragments and, at the end, the density sums over them), bra
// operand [type][k][32 bras], the m = 0 sums [4][3 o][64 kets], ket coordinates and density
// weights [5][64 kets]
static size_t bh_pairs_lds_bytes(int nn) {
  return sizeof(double) * (size_t)(KT_DOUBLES + 4L * bra_k(nn) * SB + 4 * 3 * BPT + 5 * BPT);
}

// Column of a point in an LDS row of operand k: rows are multiples of 32 slots long, so odd
// k's are turned by 16 and the two k's that half a wave reads fall into different banks.
__device__ __forceinline__ int turned(int k, int point) { return point ^ ((k & 1) * 16); }

__global__ __launch_bounds__(512, 2) void k_bh_pairs(
    const double* __restrict__ xyz, const double* __restrict__ w, const double* __restrict__ rho,
    const double* __restrict__ rhot, long n_g, long b0, long bn, long c0, long nloc, EECoef cf,
    const BHTable* __restrict__ T, int eg, int es, h8* __restrict__ pv, double* __restrict__ part,
    long bp, int first) {
  extern __shared__ __align__(16) double sm[];
  const int nn = T->n_nuc, bk = (3 * nn + 3) / 4 * 4;
  double* KT = sm;
  double* BR = sm + KT_DOUBLES;
  double* P0 = BR + 4L * bk * SB;
  double* KX = P0 + 4 * 3 * BPT;
  unsigned* ST = (unsigned*)sm;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wb = wave & 1, wk = wave >> 1;   // bra half, 16-ket step of the group
  const int li = lane & 15, lk = lane >> 4;
  const long bt = blockIdx.x, blast = b0 + bn - 1;
  // the bra operand: k = 3 I + m - 1, zero past the nuclei
  for (int e = tid; e < (bk + 2) / 3 * SB; e += 512) {
    const int I = e / SB, bb = e % SB;
    long b = b0 + bt * SB + bb;
    if (b > blast) b = blast;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (I < nn) bh_nuc_point(T, I, xyz[b], xyz[n_g + b], xyz[2 * n_g + b], v);
    const double a = v[0], pw[3] = {a, a * a, a * a * a}, dp[3] = {1.0, 2.0 * a, 3.0 * a * a};
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      const int k = 3 * I + m;
      if (k >= bk) continue;
      BR[k * SB + turned(k, bb)] = pw[m];
#pragma unroll
      for (int c = 0; c < 3; ++c) BR[((1 + c) * bk + k) * SB + turned(k, bb)] = dp[m] * v[1 + c];
    }
  }
  long bra = b0 + bt * SB + 16 * wb + li;
  if (bra > blast) bra = blast;
  const double bx = xyz[bra], by = xyz[n_g + bra], bz = xyz[2 * n_g + bra];
  const double sg = ldexp(1.0, eg), ss = ldexp(1.0, es);
  // this thread's share of the ket operand: ket tid % 64, nucleus 4 ch + fj, powers 2 fh, 2 fh + 1
  const int fj = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
  const int fh = __builtin_amdgcn_readfirstlane(tid >> 8);
  const int nch = (nn + BPN - 1) / BPN;
  double fx, fy, fz, p0[2];
  auto fill = [&](int ch) {
    const int I = BPN * ch + fj;
    double g[2][BH_NP] = {};
    if (I < nn) {
      const double dx = fx - T->nuc[I][0], dy = fy - T->nuc[I][1], dz = fz - T->nuc[I][2];
      const double b = T->nuc[I][3];
      double r, rinv;
      sqrt_rsqrt(fma(dx, dx, fma(dy, dy, dz * dz)), r, rinv);
      const double a = b * r * recip(fma(b, r, 1.0));
      const double* c = &T->csym[T->type[I]][0][0][2 * fh];   // [m][n][o]
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int m = 0; m < BH_NP; ++m) {
          const double* cm = c + m * BH_NP * BH_NO + q;
          g[q][m] = fma(fma(fma(cm[3 * BH_NO], a, cm[2 * BH_NO]), a, cm[BH_NO]), a, cm[0]);
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      p0[q] += g[q][0];
#pragma unroll
      for (int m = 1; m < BH_NP; ++m) {
        const int k = 3 * fj + m - 1;
        KT[(ch & 1) * KT_BUF + ((2 * fh + q) * BPK + k) * BPT + turned(k, lane)] = g[q][m];
      }
    }
  };
  double s[4] = {}, h[4] = {};   // density sums of this lane's bra point
  const long cl0 = (long)blockIdx.y * GCH;
  const long cl1 = cl0 + GCH < nloc ? cl0 + GCH : nloc;
  for (long cg = 2 * cl0; cg < 2 * cl1; ++cg) {   // groups of 64 kets, half a chunk
    const long kg = (c0 * SKC) + cg * BPT;
    const long gf = kg + lane < n_g ? kg + lane : n_g - 1;
    fx = xyz[gf];
    fy = xyz[n_g + gf];
    fz = xyz[2 * n_g + gf];
    p0[0] = p0[1] = 0.0;
    const double wf = kg + lane < n_g ? w[gf] : 0.0;   // padding kets: finite values, zero weight
    const double rf = rho[gf], rtf = rhot[gf];
    __syncthreads();   // the staged fragments of the previous group are out; the bra operand in
    if (wave == 0) {
      KX[lane] = fx;
      KX[BPT + lane] = fy;
      KX[2 * BPT + lane] = fz;
      KX[3 * BPT + lane] = wf * rf;
      KX[4 * BPT + lane] = wf * rtf;
    }
    fill(0);
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __syncthreads();
    d4 acc[4][BH_NO];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int o = 0; o < BH_NO; ++o) acc[x][o] = (d4){0.0, 0.0, 0.0, 0.0};
    for (int ch = 0; ch < nch; ++ch) {
      if (ch + 1 < nch) fill(ch + 1);
      const int left = 3 * nn - BPK * ch, ns = left >= BPK ? BPK / 4 : (left + 3) / 4;
      int oa = (BPK * ch + lk) * SB + turned(lk, 16 * wb + li);
      int ob = (ch & 1) * (int)KT_BUF + lk * BPT + turned(lk, 16 * wk + li);
      for (int st = 0; st < ns; ++st) {
        double fa[4], fb[BH_NO];
#pragma unroll
        for (int x = 0; x < 4; ++x) fa[x] = BR[oa + x * bk * SB];
#pragma unroll
        for (int o = 0; o < BH_NO; ++o) fb[o] = KT[ob + o * BPK * BPT];
        oa += 4 * SB;
        ob += 4 * BPT;
#pragma unroll
        for (int o = 0; o < BH_NO; ++o)
#pragma unroll
          for (int x = 0; x < 4; ++x)
            if (x > 0 || o > 0)   // F_0 is not needed
              acc[x][o] = __builtin_amdgcn_mfma_f64_16x16x4f64(fb[o], fa[x], acc[x][o], 0, 0, 0);
      }
      if (ch + 1 == nch) {   // the m = 0 sums of this thread's nuclei
        if (fh == 0) {
          P0[(fj * 3 + 0) * BPT + lane] = p0[1];
        } else {
          P0[(fj * 3 + 1) * BPT + lane] = p0[0];
          P0[(fj * 3 + 2) * BPT + lane] = p0[1];
        }
      }
      __builtin_amdgcn_s_waitcnt(0xc07f);
      __syncthreads();
    }
    // finish: lane holds the pairs (bra 16 wb + li, kets 16 wk + lk + 4 r); its split values go
    // to the staging (over the ket buffers) in the B-fragment order
    const bool odd = lk & 1;
#pragma unroll
    for (int r2 = 0; r2 < 4; r2 += 2) {
      unsigned pk[2][4];   // per ket and channel: (hi, lo) halves of the scaled value
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int r = r2 + v, kt = 16 * wk + lk + 4 * r;
        const double dx = bx - KX[kt], dy = by - KX[BPT + kt], dz = bz - KX[2 * BPT + kt];
        const double ar = KX[3 * BPT + kt], at = KX[4 * BPT + kt];
        double f0[3];
#pragma unroll
        for (int o = 0; o < 3; ++o)
          f0[o] = (P0[o * BPT + kt] + P0[(3 + o) * BPT + kt]) +
                  (P0[(6 + o) * BPT + kt] + P0[(9 + o) * BPT + kt]);
        double rr, rinv;
        sqrt_rsqrt(fma(dx, dx, fma(dy, dy, dz * dz)), rr, rinv);
        const double t = recip(fma(cf.d, rr, 1.0));
        const double e = cf.d * rr * t, e2 = e * e, e3 = e2 * e;
        double N[3];
#pragma unroll
        for (int c = 0; c < 3; ++c)
          N[c] = fma(e3, acc[1 + c][3][r], fma(e2, acc[1 + c][2][r], fma(e, acc[1 + c][1][r], acc[1 + c][0][r])));
        // U'_ee(rbar), the pure electron-electron part (coefficients past the degree are zero)
        double q = 0.0;
#pragma unroll
        for (int j = MAXQ - 1; j >= 0; --j) q = fma(q, e, cf.q1[j]);
        const double S = cf.d * t * t *
                         (fma(3.0 * e2, acc[0][3][r] + f0[2], fma(2.0 * e, acc[0][2][r] + f0[1], acc[0][1][r] + f0[0])) + q);
        const double sr = S * rinv;   // 0 at r = 0: the rhat part is dropped there
        double o[4];
        o[0] = fma(sr, dx, N[0]);
        o[1] = fma(sr, dy, N[1]);
        o[2] = fma(sr, dz, N[2]);
        o[3] = fma(o[0], o[0], fma(o[1], o[1], o[2] * o[2]));
        if (!(rr > 0.0)) o[3] = fma(S, S, o[3]);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          s[c] = fma(ar, o[c], s[c]);
          h[c] = fma(at, o[c], h[c]);
          const double x = o[c] * (c < 3 ? sg : ss);
          const _Float16 hi = half_of(x), lo = half_of(x - (double)(float)hi);
          pk[v][c] = (unsigned)__builtin_bit_cast(unsigned short, hi) |
                     ((unsigned)__builtin_bit_cast(unsigned short, lo) << 16);
        }
      }
      // lanes lk = 2p and 2p + 1 hold adjacent kets and trade values so that each stores whole
      // 32-bit words: the even one those of block r2, the odd one those of block r2 + 1
      const int kk = (lk & 2) + 4 * (r2 + (odd ? 1 : 0));   // the first of the word's two kets
      const int slot = 16 * wb + li + 32 * (kk >> 3);
      unsigned* dw = ST + wk * 2048 + slot * 4 + (kk & 6) / 2;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const unsigned mine = odd ? pk[1][c] : pk[0][c];
        const unsigned other = (unsigned)__shfl_xor((int)(odd ? pk[0][c] : pk[1][c]), 16);
        const unsigned e0 = odd ? other : mine, e1 = odd ? mine : other;   // kets kk, kk + 1
        dw[(c * 2 + 0) * 256] = (e0 & 0xffffu) | (e1 << 16);
        dw[(c * 2 + 1) * 256] = (e0 >> 16) | (e1 & 0xffff0000u);
      }
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __syncthreads();
    h8* out = pv + (bt * nloc + (cg >> 1)) * PV_CHUNK + (cg & 1) * 2048;
#pragma unroll
    for (int i = 0; i < 4; ++i) out[tid + 512 * i] = ((const h8*)sm)[tid + 512 * i];
  }
  // the density sums of each bra point: over the wave's four lanes of it, then the ket steps
  __syncthreads();
  double* red = sm;   // [wk][8][32 bras]
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    double v = c < 4 ? s[c & 3] : h[c & 3];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (lk == 0) red[(wk * 8 + c) * SB + 16 * wb + li] = v;
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __syncthreads();
  if (tid < 8 * SB) {
    const int qq = tid / SB, bb = tid % SB;
    const double v = (red[qq * SB + bb] + red[(8 + qq) * SB + bb]) +
                     (red[(16 + qq) * SB + bb] + red[(24 + qq) * SB + bb]);
    const long tb = bt * SB + bb;
    if (tb < bn) {
      double* p = part + ((long)blockIdx.y * 8 + qq) * bp + tb;
      *p = first ? v : *p + v;
    }
  }
}

xtc_status bh_pair_values_split(const Stage1Args& a, const EECoef& cf, long c0, long nloc, int eg,
                                int es, h8* pv, double* part, int first, hipStream_t st) {
  hipLaunchKernelGGL(k_bh_pairs, dim3(cdiv(a.bn, SB), cdiv(nloc, GCH)), dim3(512),
                     bh_pairs_lds_bytes(a.bh_host->n_nuc), st, a.xyz, a.w, a.rho, a.rhot, a.n_g,
                     a.b0, a.bn, c0, nloc, cf, a.bh, eg, es, pv, part, a.bp, first);
  XTC_CHECK_LAUNCH();
  return XTC_OK;
}

}  // namespace xtc
