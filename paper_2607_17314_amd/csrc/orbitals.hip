// Orbital and orbital-gradient values on the grid (Alg. 2, grid step).
// One thread per grid point and shell group evaluates the AO values and Cartesian gradients
// of a grid chunk into an SoA buffer ao4[4][n_ao][chunk]; the MO values follow as
// four FP64 MFMA GEMMs phi4[c] = C_mo^T ao4[c] in one launch; rho_gamma is a per-point sum
// over the occupied orbitals.
#include <cstring>
#include "common.hpp"
#include "plans.hpp"
#include "timing.hpp"

namespace xtc {

constexpr int ORB_CHUNK = 32768;
constexpr int MAX_L = 6;

struct BasisDev {
  const double* atom_xyz;
  const int* shell_center;
  const int* shell_l;   // l | first function << 4
  const int* shell_prim_start;
  const double* prim_exp;
  const double* prim_coef;
  const double* comp;
  int n_shell, n_ao;
};

// The values and gradients of one shell of angular momentum L at (x, y, z) from its centre,
// to o, o + chunk, ... per function and at o + plane, ... per direction
template <int L>
__device__ __forceinline__ void put_shell(const double* __restrict__ comp, double x, double y,
                                          double z, double rad, double drad, double* o, long chunk,
                                          long plane) {
  double xp[L + 2], yp[L + 2], zp[L + 2];
  xp[0] = yp[0] = zp[0] = 1.0;
#pragma unroll
  for (int n = 1; n <= L + 1; ++n) {
    xp[n] = xp[n - 1] * x;
    yp[n] = yp[n - 1] * y;
    zp[n] = zp[n - 1] * z;
  }
  int a = 0;
#pragma unroll
  for (int i = L; i >= 0; --i) {
#pragma unroll
    for (int j = L - i; j >= 0; --j, ++a) {
      const int k = L - i - j;
      const double f = comp[a];
      const double ang = xp[i] * yp[j] * zp[k];
      const double dxi = i > 0 ? i * xp[i - 1] : 0.0;
      const double dyj = j > 0 ? j * yp[j - 1] : 0.0;
      const double dzk = k > 0 ? k * zp[k - 1] : 0.0;
      o[0] = f * ang * rad;
      o[plane] = f * yp[j] * zp[k] * (dxi * rad + xp[i + 1] * drad);
      o[2 * plane] = f * xp[i] * zp[k] * (dyj * rad + yp[j + 1] * drad);
      o[3 * plane] = f * xp[i] * yp[j] * (dzk * rad + zp[k + 1] * drad);
      o += chunk;
    }
  }
}

// Workgroup (x, y): 256 points, the shells y, y + gridDim.y, ... Bound: for a grid of a few
// ten thousand points by latency (a chain of exponentials per shell), so the shells are spread
// over as many workgroups as it takes to fill the chip, and each angular momentum has a body
// of its own whose powers stay in registers. 60 functions, 17,200 points: 32 -> 12 us.
__global__ __launch_bounds__(256) void k_eval_ao(BasisDev b, const double* __restrict__ xyz,
                                                 long n_g, long g0, long chunk,
                                                 double* __restrict__ ao4) {
  long t = (long)blockIdx.x * 256 + threadIdx.x;
  if (t >= chunk) return;
  long g = g0 + t;
  if (g >= n_g) return;
  const double px = xyz[g], py = xyz[n_g + g], pz = xyz[2 * n_g + g];
  const long plane = (long)b.n_ao * chunk;
  for (int s = blockIdx.y; s < b.n_shell; s += gridDim.y) {
    const int cen = b.shell_center[s];
    const int l = b.shell_l[s] & 15, a = b.shell_l[s] >> 4;
    const double x = px - b.atom_xyz[3 * cen], y = py - b.atom_xyz[3 * cen + 1],
                 z = pz - b.atom_xyz[3 * cen + 2];
    const double r2 = x * x + y * y + z * z;
    double rad = 0.0, drad = 0.0;
    for (int p = b.shell_prim_start[s]; p < b.shell_prim_start[s + 1]; ++p) {
      double e = b.prim_coef[p] * exp(-b.prim_exp[p] * r2);
      rad += e;
      drad -= 2.0 * b.prim_exp[p] * e;
    }
    const double* f = b.comp + a;
    double* o = ao4 + (long)a * chunk + t;
    switch (l) {
      case 0: put_shell<0>(f, x, y, z, rad, drad, o, chunk, plane); break;
      case 1: put_shell<1>(f, x, y, z, rad, drad, o, chunk, plane); break;
      case 2: put_shell<2>(f, x, y, z, rad, drad, o, chunk, plane); break;
      case 3: put_shell<3>(f, x, y, z, rad, drad, o, chunk, plane); break;
      case 4: put_shell<4>(f, x, y, z, rad, drad, o, chunk, plane); break;
      case 5: put_shell<5>(f, x, y, z, rad, drad, o, chunk, plane); break;
      default: put_shell<6>(f, x, y, z, rad, drad, o, chunk, plane); break;
    }
  }
}
static_assert(MAX_L == 6, "one body per angular momentum in k_eval_ao");

__global__ __launch_bounds__(256) void k_density(const double* __restrict__ phi, long n_g,
                                                 int n_occ, double* __restrict__ rho) {
  long g = (long)blockIdx.x * 256 + threadIdx.x;
  if (g >= n_g) return;
  double s = 0.0;
  for (int i = 0; i < n_occ; ++i) {
    double v = phi[(long)i * n_g + g];
    s += v * v;
  }
  rho[g] = s;
}

struct OrbLayout {
  double* atom_xyz; int* ints; double* prim; double* comp; double* ao4;
  long chunk;
};

static OrbLayout layout_orb(Arena& ar, int64_t n_g, int n_ao, int n_atom, int n_shell, int n_prim) {
  OrbLayout L;
  L.chunk = n_g < ORB_CHUNK ? n_g : ORB_CHUNK;
  L.atom_xyz = ar.take<double>(3 * (size_t)n_atom);
  L.ints = ar.take<int>(3 * (size_t)n_shell + 1);
  L.prim = ar.take<double>(2 * (size_t)n_prim);
  L.comp = ar.take<double>(n_ao);
  L.ao4 = ar.take<double>(4 * (size_t)n_ao * L.chunk);
  return L;
}

size_t ws_eval_orbitals(int64_t n_g, int n_orb, int n_ao) {
  (void)n_orb;
  Arena ar(nullptr, 0);
  // basis tables are tiny; reserve generously for up to 4096 shells / primitives / atoms
  layout_orb(ar, n_g, n_ao, 4096, 4096, 16384);
  return ar.used;
}

}  // namespace xtc

using namespace xtc;

extern "C" xtc_status xtc_eval_orbitals(const xtc_basis* basis, const xtc_grid* grid,
                                        const double* C_mo, int32_t n_orb, int32_t n_occ,
                                        double* phi4, double* rho, void* ws, size_t ws_bytes,
                                        void* stream) {
  XTC_REQUIRE(basis && grid && C_mo && phi4, "xtc_eval_orbitals: null argument");
  XTC_REQUIRE(grid->n_g > 0 && grid->xyz, "xtc_eval_orbitals: empty grid");
  XTC_REQUIRE(n_orb > 0 && n_occ >= 0 && n_occ <= n_orb, "xtc_eval_orbitals: bad n_orb/n_occ");
  XTC_REQUIRE(basis->n_shell > 0 && basis->n_atom > 0 && basis->n_atom <= 4096 &&
                  basis->n_shell <= 4096,
              "xtc_eval_orbitals: bad basis sizes");
  XTC_REQUIRE(basis->atom_xyz && basis->shell_center && basis->shell_l &&
                  basis->shell_prim_start && basis->prim_exp && basis->prim_coef &&
                  basis->comp_factor,
              "xtc_eval_orbitals: null basis table");
  int n_ao = 0;
  for (int s = 0; s < basis->n_shell; ++s) {
    int l = basis->shell_l[s];
    XTC_REQUIRE(l >= 0 && l <= MAX_L, "xtc_eval_orbitals: angular momentum out of range");
    XTC_REQUIRE(basis->shell_center[s] >= 0 && basis->shell_center[s] < basis->n_atom,
                "xtc_eval_orbitals: shell centre out of range");
    XTC_REQUIRE(basis->shell_prim_start[s + 1] > basis->shell_prim_start[s],
                "xtc_eval_orbitals: shell without primitives");
    n_ao += (l + 1) * (l + 2) / 2;
  }
  int n_prim = basis->shell_prim_start[basis->n_shell];
  XTC_REQUIRE(basis->shell_prim_start[0] == 0 && n_prim <= 16384,
              "xtc_eval_orbitals: bad primitive table");
  XTC_REQUIRE(n_ao == basis->n_ao, "xtc_eval_orbitals: n_ao does not match the shells");
  hipStream_t st = as_stream(stream);
  Arena ar(ws, ws_bytes);
  OrbLayout L = layout_orb(ar, grid->n_g, n_ao, basis->n_atom, basis->n_shell, n_prim);
  XTC_TRY(need_ws(ar));

  // the tables as they lie in the workspace, uploaded as one
  const char* base = (const char*)L.atom_xyz;
  std::vector<char> host((const char*)(L.comp + n_ao) - base);
  auto at = [&](const void* dev) { return host.data() + ((const char*)dev - base); };
  memcpy(at(L.atom_xyz), basis->atom_xyz, sizeof(double) * 3 * basis->n_atom);
  int* ints = (int*)at(L.ints);
  for (int s = 0, first = 0; s < basis->n_shell; ++s) {
    const int l = basis->shell_l[s];
    ints[s] = basis->shell_center[s];
    ints[basis->n_shell + s] = l | first << 4;
    first += (l + 1) * (l + 2) / 2;
  }
  memcpy(ints + 2 * basis->n_shell, basis->shell_prim_start, sizeof(int) * (basis->n_shell + 1));
  memcpy(at(L.prim), basis->prim_exp, sizeof(double) * n_prim);
  memcpy(at(L.prim + n_prim), basis->prim_coef, sizeof(double) * n_prim);
  memcpy(at(L.comp), basis->comp_factor, sizeof(double) * n_ao);
  XTC_HIP(hipMemcpyAsync(L.atom_xyz, host.data(), host.size(), hipMemcpyHostToDevice, st));
  XTC_HIP(hipStreamSynchronize(st));   // the host copy ends with this call
  BasisDev b{L.atom_xyz, L.ints, L.ints + basis->n_shell, L.ints + 2 * basis->n_shell,
             L.prim, L.prim + n_prim, L.comp, basis->n_shell, n_ao};
  const long n_g = grid->n_g;
  size_t tk = timing_begin(TM_ORBITALS, st);
  for (long g0 = 0; g0 < n_g; g0 += L.chunk) {
    long cn = (n_g - g0) < L.chunk ? (n_g - g0) : L.chunk;
    // about four workgroups per CU, shells permitting
    const unsigned wg = cdiv(cn, 256), rounds = cdiv(1024, wg);
    const unsigned split = rounds < (unsigned)basis->n_shell ? rounds : (unsigned)basis->n_shell;
    hipLaunchKernelGGL(k_eval_ao, dim3(wg, split), dim3(256), 0, st, b, grid->xyz, n_g, g0, L.chunk,
                       L.ao4);
    XTC_CHECK_LAUNCH();
    GemmArgs gs[4];
    for (int c = 0; c < 4; ++c) {
      GemmArgs& g = gs[c];
      g = GemmArgs{};
      g.M = n_orb; g.N = cn; g.K = n_ao;
      g.A = C_mo; g.a_sm = 1; g.a_sk = n_orb;
      g.B = L.ao4 + (long)c * n_ao * L.chunk; g.b_sk = L.chunk; g.b_sn = 1;
      g.s = nullptr;
      g.C = phi4 + (long)c * n_orb * n_g + g0; g.c_sm = n_g; g.c_sn = 1;
    }
    XTC_TRY(gemm_f64_list(gs, 4, st));
  }
  if (rho) {
    hipLaunchKernelGGL(k_density, dim3(cdiv(n_g, 256)), dim3(256), 0, st, phi4, n_g, n_occ, rho);
    XTC_CHECK_LAUNCH();
  }
  timing_end(tk, st);
  return XTC_OK;
}
