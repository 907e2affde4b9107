// How many walkers of the e-e local energies share a SIMD, in plain constexpr so that a host
// program can check it.
#pragma once

namespace xtc {

// Whether two walkers share a SIMD, `lds` bytes each: where that saves a round of walkers over
// four on a CU, one per SIMD. Rounds of four are the shorter ones, and where five or six fit
// by LDS, the fifth and sixth load two SIMDs double. 20 atoms (five by LDS), one and two per
// SIMD: 1,280 walkers 390, 277 us; 2,048 walkers (two rounds either way) 401, 450; 4,096 (four
// rounds) 738, 759; 8,192 (eight, seven) 1,402, 1,303.
constexpr bool vmc_two_per_simd(long lds, long n_walkers) {
  constexpr long cu = 160 * 1024, n_cu = 256;
  const long fit = cu / lds < 8 ? cu / lds : 8;
  const long per_cu = (n_walkers + n_cu - 1) / n_cu;
  return fit > 4 && (per_cu + fit - 1) / fit < (per_cu + 3) / 4;
}

}  // namespace xtc
