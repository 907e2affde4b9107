// Layout of the split path's BH pair-value buffer and the launch that fills it.
#pragma once
#include "stage1_split.hpp"

namespace xtc {

constexpr int GCH = 8;                // ket chunks per generation workgroup
constexpr int PV_CHUNK = 8 * 4 * 2 * 64;   // h8 per (bra tile, ket chunk): [ks][ch][hl][lane]

// The pair values of ket chunks [c0, c0 + nloc) for the bra tiles of `a`, scaled by 2^eg (2^es
// the squared norm) and split into FP16 pairs, to pv [bra tile][chunk][PV_CHUNK]; the density-
// row sums of each bra to part[group][8][bp] (written if `first`, else added).
xtc_status bh_pair_values_split(const Stage1Args& a, const EECoef& cf, long c0, long nloc, int eg,
                                int es, h8* pv, double* part, int first, hipStream_t st);

}  // namespace xtc
