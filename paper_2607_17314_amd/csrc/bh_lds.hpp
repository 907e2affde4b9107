// LDS of the Boys-Handy pair-value kernels (stage1_split_bh.hip) and the rule that depends on
// it, in plain constexpr so that a host program can check them.
#pragma once

namespace xtc {

constexpr int BH_MAXNUC = 24;   // nuclei
constexpr int BH_MAXTYPE = 2;   // nucleus types
constexpr int BH_NP = 4;        // powers 0..3 of a_iI in the nuclear terms
constexpr int BH_NO = 4;        // powers 0..3 of rbar12 in the nuclear terms
constexpr int BH_BRAS = 32;     // bra points per workgroup of the pair-value kernels

// Doubles per ket in the LDS ket tables: the 16 kets of a wave read at once sit 2 doubles
// (4 banks) apart modulo the 64 banks, instead of all in one bank.
constexpr int bh_ket_stride(int nn) { return nn * BH_NO * BH_NP + 2; }

// LDS tables of the pair-value kernels, in doubles: bra tables [nn][a, grad a][32 bras], one
// ket table [16 kets][bh_ket_stride(nn)] (two: 1 + ahead), as many tables a_I [nn][16 kets],
// csym [t][m][n][o]
constexpr long bh_tables_lds_doubles(int nn, int ahead) {
  return (long)nn * 4 * BH_BRAS + (1 + ahead) * (16L * bh_ket_stride(nn) + 16L * nn) +
         BH_MAXTYPE * BH_NP * BH_NP * BH_NO;
}

// What a kernel's workgroups take beside the tables, and how many of them its registers let run
// on a CU.
struct BHKernel {
  long staged;      // doubles of LDS beside the tables
  int workgroups;
};
constexpr BHKernel BH_PAIRS{2 * 4096 / 4, 2};   // half-precision fragments, two k-steps' worth
constexpr BHKernel BH_PAIRS_F64{0, 3};

// Workgroups of a kernel on a CU (160 KB of LDS).
constexpr int bh_resident(BHKernel k, int nn, int ahead) {
  const long fit = 160 * 1024 / (8 * (bh_tables_lds_doubles(nn, ahead) + k.staged));
  return fit < k.workgroups ? (int)fit : k.workgroups;
}

// Whether a workgroup keeps the next step's ket tables beside the current one's: yes, unless
// that costs the CU a workgroup. Per launch of 16,384 x 16,384 pairs, with them and without:
//   k_bh_pairs      4 nuclei 4.57, 4.81 ms; 11: 8.42, 8.68; 20: 19.8, 14.1 (the second
//                   workgroup); 22: 20.5, 21.1 (one either way)
//   k_bh_pairs_f64  4 nuclei 3.76, 3.86 ms; 10: 7.72, 7.12 and 13: 9.45, 8.60 (the third);
//                   22: 21.1, 14.9 and 24: 23.0, 16.1 (the second)
constexpr int bh_tables_ahead(BHKernel k, int nn) {
  return bh_resident(k, nn, 1) == bh_resident(k, nn, 0) ? 1 : 0;
}

}  // namespace xtc
