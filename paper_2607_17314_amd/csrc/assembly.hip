// Four-index assembly of the transcorrelated two-body corrections and the xTC
// one-body pieces from the ISDF intermediates (K-kernel section, eq.
// K-recombine-final with eqs. K1-isdf and K3-isdf; xTC section, eq.
// delta-u-dx-kernels and the final assembly; Hamiltonian assembly section, eqs.
// xtc-deltah, xtc-fock, xtc-const).
//
// With the pair factors C_mu(p,r) = phi_p phi_r (r_mu) (symmetric in p, r) and
// A^c_mu(p,r) = phi_p d_c phi_r - phi_r d_c phi_p (r_mu) (antisymmetric):
//   K1 - K1swap + K3 = sum_nu PK_nu(p,r) C_nu(q,s),  PK_nu = sum_mu [sum_c A^c_mu u1^c_{mu nu} + C_mu u3_{mu nu}]
//   C D C - C X      = sum_nu PU_nu(p,r) C_nu(q,s) - sum_mu C_mu(p,r) X_mu(q,s),  PU_nu = sum_mu C_mu D_{mu nu}
// and P12 T^{pq}_{rs} = T^{pq}_{rs} + T^{qp}_{sr}, so every output is
//   out[(p,r),(q,s)] = a sum_nu [P(p,r) C(q,s) + C(p,r) P(q,s)] + b sum_mu [C(p,r) X(q,s) + X(p,r) C(q,s)]
//                    = sum_nu [F(p,r) C(q,s) + C(p,r) F(q,s)],  F = a P + b X,
// with (P, a, b) = (PK, 1/2, 0) for K, (PU, -1, 1) for dU and (PW = PK/2 + PU, -1, 1) for
// W = -K + dU: with F formed once by the preparation, a panel is two FP64 MFMA products
// instead of four. In all but small problems P is split into the projections of the
// antisymmetric A (PA) and of the symmetric C (PC), each formed for p <= r only. The one-body
// pieces need only partial traces over the occupied orbitals, formed from the same factors
// without the four-index tensors.
// Ten atoms (150 orbitals, N_mu 1,500), a panel of 20 orbitals with its preparation:
// 29.7 -> 10.5 ms (panel 20.7 -> 6.6, 61 TFLOP/s; preparation 9.2 -> 4.7).
#include "common.hpp"
#include "plans.hpp"
#include "timing.hpp"

namespace xtc {

struct AsmLayout {
  bool packed;   // the projections run over the pairs p <= r, else over all
  double* A3;    // [x, y, z][n_mu][np]: A^c_mu(p,r)
  double* Cp;    // [n_mu][np]: C_mu(p,r), when packed
  double* C;     // [n_mu][n_orb^2]: C_mu(p,r); when not packed right behind A3
  double* Xm;    // [n_mu][n_orb^2] = X2 + X3 transposed
  double* PA; double* PC;  // [n_mu][np]: the projections of A3 and Cp, when packed
  double* FK; double* FU; double* FW;   // [n_mu][n_orb^2] each (when requested)
  double* U4;    // [4][n_mu][n_mu] stacked right factors of the projection GEMMs
  double* vec;   // [2][n_mu]: g, phi of the one-body traces
  double* J; double* Kx;   // [n_orb][n_orb] one-body partial traces
  double* dhd;   // [n_orb] diagonal of dh
  long nn;       // n_orb^2
  long np;       // pairs: n_orb (n_orb + 1) / 2 when packed, else n_orb^2
};

// Packed pairs halve the projections' work but take two launches more per output (the
// symmetric part's product and the unpacking): from more 64 x 64 tiles than CUs on. W of one
// orbital's panel with its preparation, packed and not: 44 orbitals, N_mu 440 (217 tiles) 189,
// 179 us; 48, 480 (288 tiles) 203, 244 us; 4 orbitals, N_mu 16: 59, 50 us.
static bool packed_pairs(int n_orb, int n_mu) {
  return (long)cdiv(n_mu, 64) * cdiv((long)n_orb * n_orb, 64) > 256;
}

static AsmLayout layout_asm(Arena& ar, int n_orb, int n_mu, uint32_t outputs, bool one_body) {
  AsmLayout L{};
  L.nn = (long)n_orb * n_orb;
  L.packed = packed_pairs(n_orb, n_mu);
  L.np = L.packed ? (long)n_orb * (n_orb + 1) / 2 : L.nn;
  const size_t blk = (size_t)n_mu * L.nn, half = (size_t)n_mu * L.np;
  if (L.packed) {
    L.A3 = ar.take<double>(3 * half);
    L.Cp = ar.take<double>(half);
    L.C = ar.take<double>(blk);
    L.PA = ar.take<double>(half);
    L.PC = ar.take<double>(half);
  } else {
    L.A3 = ar.take<double>(4 * blk);
    L.C = L.A3 + 3 * blk;
  }
  L.Xm = ar.take<double>(blk);
  if (outputs & XTC_ASM_K) L.FK = ar.take<double>(blk);
  if (outputs & XTC_ASM_DU) L.FU = ar.take<double>(blk);
  if (outputs & XTC_ASM_W) L.FW = ar.take<double>(blk);
  L.U4 = ar.take<double>((size_t)4 * n_mu * n_mu);
  L.vec = ar.take<double>((size_t)2 * n_mu);
  if (one_body) {
    L.J = ar.take<double>(L.nn);
    L.Kx = ar.take<double>(L.nn);
    L.dhd = ar.take<double>(n_orb);
  }
  return L;
}

size_t ws_assembly(int n_orb, int n_mu, uint32_t outputs) {
  Arena ar(nullptr, 0);
  layout_asm(ar, n_orb, n_mu, outputs, false);
  return ar.used;
}

size_t ws_one_body(int n_orb, int n_mu) {
  Arena ar(nullptr, 0);
  layout_asm(ar, n_orb, n_mu, XTC_ASM_DU | XTC_ASM_W, true);
  return ar.used;
}

// Index of the pair p <= r among the packed ones.
__device__ __forceinline__ long packed(int p, int r, int n) {
  return (long)p * n - (long)p * (p - 1) / 2 + (r - p);
}

// C[mu][p n + r] = C_mu(p,r) and A3[c] = A^c_mu(p,r); with Cp packed: A3 and Cp for p <= r
__global__ void k_pair_factors(const double* __restrict__ phi4, int n, int n_mu, long np,
                               double* __restrict__ A3, double* __restrict__ Cp,
                               double* __restrict__ C) {
  const long t = (long)blockIdx.x * 256 + threadIdx.x;
  const long nn = (long)n * n;
  if (t >= (long)n_mu * nn) return;
  const long pr = t % nn;
  const int mu = (int)(t / nn);
  const int p = (int)(pr / n), r = (int)(pr % n);
  const long sp = (long)p * n_mu + mu, sr = (long)r * n_mu + mu, comp = (long)n * n_mu;
  const double fp = phi4[sp], fr = phi4[sr];
  C[t] = fp * fr;
  if (Cp && r < p) return;
  const long o = Cp ? mu * np + packed(p, r, n) : t;
  if (Cp) Cp[o] = fp * fr;
#pragma unroll
  for (int c = 0; c < 3; ++c)
    A3[(long)c * n_mu * np + o] = fp * phi4[(1 + c) * comp + sr] - fr * phi4[(1 + c) * comp + sp];
}

// F[nu][p n + r] = a (PC(p,r) + PA(p,r)) + X, PC symmetric and PA (or null) antisymmetric
__global__ void k_unpack_f(const double* __restrict__ PC, const double* __restrict__ PA,
                           const double* __restrict__ X, int n, int n_mu, long np, double a,
                           double* __restrict__ F) {
  const long t = (long)blockIdx.x * 256 + threadIdx.x;
  const long nn = (long)n * n;
  if (t >= (long)n_mu * nn) return;
  const int p = (int)(t % nn / n), r = (int)(t % n);
  const long o = t / nn * np + (p <= r ? packed(p, r, n) : packed(r, p, n));
  double v = PC[o];
  if (PA) v += p <= r ? PA[o] : -PA[o];
  v *= a;
  F[t] = X ? v + X[t] : v;
}

// U4[seg][mu][nu] = s1 * M1[seg] + s2 * M2 (a scaled copy, M2 only in the last segment)
__global__ void k_stack_u(const double* __restrict__ u1, const double* __restrict__ u3,
                          const double* __restrict__ Da, const double* __restrict__ Db, int n_mu,
                          double su, double s3, double sa, double sb, double* __restrict__ U4) {
  const long t = (long)blockIdx.x * 256 + threadIdx.x;
  const long m2 = (long)n_mu * n_mu;
  if (t >= 4 * m2) return;
  const int seg = (int)(t / m2);
  const long i = t % m2;
  double v;
  if (seg < 3) {
    v = su * u1[seg * m2 + i];
  } else {
    v = s3 * u3[i];
    if (Da) v += sa * Da[i];
    if (Db) v += sb * Db[i];
  }
  U4[t] = v;
}

// Xm[mu][q n + s] = X2[q][s][mu] + X3[q][s][mu] (64 x 64 tiles through LDS)
__global__ __launch_bounds__(256) void k_x_transpose(const double* __restrict__ X2,
                                                     const double* __restrict__ X3, long nn,
                                                     int n_mu, double* __restrict__ Xm) {
  __shared__ double tile[64][65];
  const long qs0 = (long)blockIdx.x * 64;
  const int mu0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int r = ty; r < 64; r += 4) {
    const long qs = qs0 + r;
    const int mu = mu0 + tx;
    double v = 0.0;
    if (qs < nn && mu < n_mu) {
      const long i = qs * n_mu + mu;
      if (X2) v += X2[i];
      if (X3) v += X3[i];
    }
    tile[r][tx] = v;
  }
  __syncthreads();
  for (int r = ty; r < 64; r += 4) {
    const int mu = mu0 + r;
    const long qs = qs0 + tx;
    if (mu < n_mu && qs < nn) Xm[(long)mu * nn + qs] = tile[tx][r];
  }
}

// g[k] = sum_o C_k(o,o); phi[k] = sum_o F_k(o,o) (o < n_occ)
__global__ void k_occ_diag(const double* __restrict__ C, const double* __restrict__ F, int n,
                           int n_occ, int n_mu, double* __restrict__ vec) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= n_mu) return;
  const long nn = (long)n * n;
  double g = 0.0, phi = 0.0;
  for (int o = 0; o < n_occ; ++o) {
    const long i = (long)k * nn + (long)o * n + o;
    g += C[i];
    phi += F[i];
  }
  vec[k] = g;
  vec[n_mu + k] = phi;
}

__global__ void k_one_body_mix(const double* __restrict__ J, const double* __restrict__ Kx,
                               long nn, double cj, double ck, const double* __restrict__ base,
                               double* __restrict__ out) {
  const long t = (long)blockIdx.x * 256 + threadIdx.x;
  if (t >= nn) return;
  out[t] = (base ? base[t] : 0.0) + cj * J[t] + ck * Kx[t];
}

__global__ void k_diag(const double* __restrict__ M, int n, double* __restrict__ d) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) d[i] = M[(long)i * n + i];
}

static xtc_status check_asm(const xtc_assembly* a) {
  XTC_REQUIRE(a, "assembly: null argument");
  XTC_REQUIRE(a->n_orb > 0 && a->n_mu > 0, "assembly: bad sizes");
  XTC_REQUIRE(a->phi4_piv && a->u1 && a->u3 && a->D1 && a->D4,
              "assembly: null phi4_piv, u1, u3, D1 or D4");
  XTC_REQUIRE((long)a->n_orb * a->n_orb <= (1L << 31), "assembly: n_orb too large");
  return XTC_OK;
}

// The factors every panel reads (see the file comment).
static xtc_status prepare(const xtc_assembly* a, uint32_t outputs, const AsmLayout& L,
                          hipStream_t st) {
  const int n = a->n_orb, n_mu = a->n_mu;
  const long nn = L.nn, np = L.np, blk = (long)n_mu * nn;
  const bool has_x = a->X2 || a->X3;
  hipLaunchKernelGGL(k_pair_factors, dim3(cdiv(blk, 256)), dim3(256), 0, st, a->phi4_piv, n, n_mu,
                     np, L.A3, L.Cp, L.C);
  XTC_CHECK_LAUNCH();
  if (has_x && (outputs & (XTC_ASM_DU | XTC_ASM_W))) {
    hipLaunchKernelGGL(k_x_transpose, dim3(cdiv(nn, 64), cdiv(n_mu, 64)), dim3(256), 0, st, a->X2,
                       a->X3, nn, n_mu, L.Xm);
    XTC_CHECK_LAUNCH();
  }
  const long m2 = (long)n_mu * n_mu;
  // P[nu][pr] = alpha sum_{seg, mu} U4[seg][mu][nu] B[seg - seg0][mu][pr] + X (or nothing)
  auto project = [&](double* P, const double* B, int seg0, int nseg, double alpha, const double* X) {
    GemmArgs g{};
    g.M = n_mu; g.N = np; g.K = (long)nseg * n_mu;
    g.A = L.U4 + (long)seg0 * m2; g.a_sm = 1; g.a_sk = n_mu;
    g.B = B; g.b_sk = np; g.b_sn = 1;
    g.C = P; g.c_sm = np; g.c_sn = 1;
    g.alpha = alpha;
    g.D = X;
    g.beta = X ? 1.0 : 0.0;
    return gemm_f64(g, st);
  };
  // U4 from su u1, s3 u3 + sd (D4 + 2 D1), then F = coef (PC + PA) + X
  auto factor = [&](double su, double s3, double sd, double coef, bool x, double* F) -> xtc_status {
    hipLaunchKernelGGL(k_stack_u, dim3(cdiv(4 * m2, 256)), dim3(256), 0, st, a->u1, a->u3,
                       sd != 0.0 ? a->D4 : nullptr, sd != 0.0 ? a->D1 : nullptr, n_mu, su, s3, sd,
                       2.0 * sd, L.U4);
    XTC_CHECK_LAUNCH();
    if (!L.packed) {
      const int seg0 = su != 0.0 ? 0 : 3;   // A3, C or C alone
      return project(F, L.A3 + (long)seg0 * blk, seg0, 4 - seg0, coef, x ? L.Xm : nullptr);
    }
    if (su != 0.0) XTC_TRY(project(L.PA, L.A3, 0, 3, 1.0, nullptr));
    XTC_TRY(project(L.PC, L.Cp, 3, 1, 1.0, nullptr));
    hipLaunchKernelGGL(k_unpack_f, dim3(cdiv(blk, 256)), dim3(256), 0, st, (const double*)L.PC,
                       su != 0.0 ? (const double*)L.PA : nullptr,
                       x ? (const double*)L.Xm : nullptr, n, n_mu, np, coef, F);
    XTC_CHECK_LAUNCH();
    return XTC_OK;
  };
  if (outputs & XTC_ASM_K) XTC_TRY(factor(1.0, 1.0, 0.0, 0.5, false, L.FK));
  if (outputs & XTC_ASM_DU) XTC_TRY(factor(0.0, 0.0, 1.0, -1.0, has_x, L.FU));
  if (outputs & XTC_ASM_W) XTC_TRY(factor(0.5, 0.5, 1.0, -1.0, has_x, L.FW));
  return XTC_OK;
}

// Partial traces of out = F C + C F:
//   J[p][q] = sum_o out[(p,q),(o,o)],  Kx[p][q] = sum_o out[(p,o),(o,q)]
static xtc_status partial_traces(const AsmLayout& L, const double* F, int n, int n_occ, int n_mu,
                                 hipStream_t st) {
  const long nn = L.nn;
  hipLaunchKernelGGL(k_occ_diag, dim3(cdiv(n_mu, 256)), dim3(256), 0, st, (const double*)L.C, F, n,
                     n_occ, n_mu, L.vec);
  XTC_CHECK_LAUNCH();
  // J = F g + C phi, as products [n^2 x n_mu] [n_mu x 1]
  const double* left[2] = {F, L.C};
  const double* right[2] = {L.C, F};
  for (int i = 0; i < 2; ++i) {
    GemmArgs q{};
    q.M = nn; q.N = 1; q.K = n_mu;
    q.A = left[i]; q.a_sm = 1; q.a_sk = nn;
    q.B = L.vec + i * n_mu; q.b_sk = 1; q.b_sn = 1;
    q.C = L.J; q.c_sm = 1; q.c_sn = 1;
    q.beta = i == 0 ? 0.0 : 1.0;
    XTC_TRY(gemm_f64(q, st));
  }
  // Kx = sum_o [F(p,o) C(o,q) + C(p,o) F(o,q)]
  for (int o = 0; o < n_occ; ++o)
    for (int i = 0; i < 2; ++i) {
      GemmArgs q{};
      q.M = n; q.N = n; q.K = n_mu;
      q.A = left[i] + o; q.a_sm = n; q.a_sk = nn;           // A[p][k] = L_k(p, o)
      q.B = right[i] + (long)o * n; q.b_sk = nn; q.b_sn = 1;  // B[k][q] = R_k(o, q)
      q.C = L.Kx; q.c_sm = n; q.c_sn = 1;
      q.beta = o == 0 && i == 0 ? 0.0 : 1.0;
      XTC_TRY(gemm_f64(q, st));
    }
  return XTC_OK;
}

}  // namespace xtc

using namespace xtc;

extern "C" xtc_status xtc_assembly_prepare(const xtc_assembly* a, uint32_t outputs, void* ws,
                                           size_t ws_bytes, void* stream) {
  XTC_TRY(check_asm(a));
  XTC_REQUIRE(outputs != 0 && (outputs & ~7u) == 0, "assembly: outputs must be a mask of K, DU, W");
  Arena ar(ws, ws_bytes);
  AsmLayout L = layout_asm(ar, a->n_orb, a->n_mu, outputs, false);
  XTC_TRY(need_ws(ar));
  return prepare(a, outputs, L, as_stream(stream));
}

extern "C" xtc_status xtc_assembly_panel(const xtc_assembly* a, uint32_t outputs, int32_t p0,
                                         int32_t p1, double* K, double* dU, double* W, void* ws,
                                         size_t ws_bytes, void* stream) {
  XTC_TRY(check_asm(a));
  XTC_REQUIRE(outputs != 0 && (outputs & ~7u) == 0, "assembly: outputs must be a mask of K, DU, W");
  XTC_REQUIRE(0 <= p0 && p0 <= p1 && p1 <= a->n_orb, "assembly: panel outside the orbital range");
  XTC_REQUIRE(!(outputs & XTC_ASM_K) || K, "assembly: K output NULL");
  XTC_REQUIRE(!(outputs & XTC_ASM_DU) || dU, "assembly: dU output NULL");
  XTC_REQUIRE(!(outputs & XTC_ASM_W) || W, "assembly: W output NULL");
  Arena ar(ws, ws_bytes);
  AsmLayout L = layout_asm(ar, a->n_orb, a->n_mu, outputs, false);
  XTC_TRY(need_ws(ar));
  if (p1 == p0) return XTC_OK;
  hipStream_t st = as_stream(stream);
  const int n = a->n_orb;
  const long M = (long)(p1 - p0) * n, N = L.nn;
  struct Out { uint32_t bit; const double* F; double* dst; };
  const Out outs[3] = {{XTC_ASM_K, L.FK, K}, {XTC_ASM_DU, L.FU, dU}, {XTC_ASM_W, L.FW, W}};
  for (const Out& o : outs) {
    if (!(outputs & o.bit)) continue;
    const size_t tk = timing_begin(TM_ASM_PANEL, st);
    const double* left[2] = {o.F, L.C};
    const double* right[2] = {L.C, o.F};
    for (int i = 0; i < 2; ++i) {   // out = F C, then += C F
      GemmArgs g{};
      g.M = M; g.N = N; g.K = a->n_mu;
      g.A = left[i] + (long)p0 * n; g.a_sm = 1; g.a_sk = N;
      g.B = right[i]; g.b_sk = N; g.b_sn = 1;
      g.C = o.dst; g.c_sm = N; g.c_sn = 1;
      g.beta = i == 0 ? 0.0 : 1.0;
      XTC_TRY(gemm_f64(g, st));
    }
    timing_end(tk, st);
  }
  return XTC_OK;
}

extern "C" xtc_status xtc_one_body(const xtc_assembly* a, int32_t n_occ, double e_nuc, double* dh,
                                   double* f, double* e0, void* ws, size_t ws_bytes,
                                   void* stream) {
  XTC_TRY(check_asm(a));
  XTC_REQUIRE(n_occ > 0 && n_occ <= a->n_orb, "one-body: bad n_occ");
  XTC_REQUIRE(dh || f || e0, "one-body: no output requested");
  Arena ar(ws, ws_bytes);
  AsmLayout L = layout_asm(ar, a->n_orb, a->n_mu, XTC_ASM_DU | XTC_ASM_W, true);
  XTC_TRY(need_ws(ar));
  hipStream_t st = as_stream(stream);
  const int n = a->n_orb;
  XTC_TRY(prepare(a, XTC_ASM_DU | XTC_ASM_W, L, st));
  // dh = -1/2 (2 J[dU] - Kx[dU])   (eq. xtc-deltah)
  XTC_TRY(partial_traces(L, L.FU, n, n_occ, a->n_mu, st));
  double* dhb = dh ? dh : L.J;   // dh is needed for f and E0 even when not returned
  const unsigned gb = cdiv(L.nn, 256);
  if (!dh) {
    // keep J, Kx of dU apart from the buffers reused below
    hipLaunchKernelGGL(k_one_body_mix, dim3(gb), dim3(256), 0, st, (const double*)L.J,
                       (const double*)L.Kx, L.nn, -1.0, 0.5, (const double*)nullptr, L.Kx);
    XTC_CHECK_LAUNCH();
    dhb = L.Kx;
  } else {
    hipLaunchKernelGGL(k_one_body_mix, dim3(gb), dim3(256), 0, st, (const double*)L.J,
                       (const double*)L.Kx, L.nn, -1.0, 0.5, (const double*)nullptr, dh);
    XTC_CHECK_LAUNCH();
  }
  if (e0) {
    hipLaunchKernelGGL(k_diag, dim3(cdiv(n, 256)), dim3(256), 0, st, (const double*)dhb, n, L.dhd);
    XTC_CHECK_LAUNCH();
    std::vector<double> d(n);
    XTC_HIP(hipMemcpyAsync(d.data(), L.dhd, sizeof(double) * n, hipMemcpyDeviceToHost, st));
    XTC_HIP(hipStreamSynchronize(st));
    double tr = 0.0;
    for (int i = 0; i < n_occ; ++i) tr += d[i];
    *e0 = -2.0 / 3.0 * tr + e_nuc;   // eq. xtc-const
  }
  if (f) {
    // the dh buffer must survive the W traces: copy it into f first
    hipLaunchKernelGGL(k_one_body_mix, dim3(gb), dim3(256), 0, st, (const double*)dhb,
                       (const double*)dhb, L.nn, 1.0, 0.0, (const double*)nullptr, f);
    XTC_CHECK_LAUNCH();
    // f = dh + 2 J[W] - Kx[W]   (eq. xtc-fock)
    XTC_TRY(partial_traces(L, L.FW, n, n_occ, a->n_mu, st));
    hipLaunchKernelGGL(k_one_body_mix, dim3(gb), dim3(256), 0, st, (const double*)L.J,
                       (const double*)L.Kx, L.nn, 2.0, -1.0, (const double*)f, f);
    XTC_CHECK_LAUNCH();
  }
  return XTC_OK;
}
