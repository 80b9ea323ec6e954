// lf2_rules.hpp -- rules that choose a launch's shape on the host, free of HIP
// so that they are checked without a GPU.
#pragma once
#include <stddef.h>

namespace lf2 {

// Blocks of a binned z pass over lines of `len` points (reg: in register
// tiles): one round of what 256 CUs hold at `lds` bytes and `waves` waves a
// block, at most 16 waves a CU.  More blocks than that only repeat the tables'
// set-up.  With 1024 blocks and with a round (us): Poisson with 32 bins at 256^3
// 153 and 149, 400^3 594 and 556, 600^3 2590 and 2482 (300^3 295 and 298), P(k)
// at 256^3 87 and 83, 512^3 538 and 530; the fused register tile over 256
// points alone 42.0 and 38.6 at 256^3, 127 and 124 over 512 x 512 x 256, over 64
// points 44.6 and 43.2, over 128 points 79.7 and 78.5 (512 x 512 planes).
// Longer lines take long enough a tile that the balance of 1024 blocks is
// worth more: the register tile over 512 points 275 and 280 at 512^3 and 73
// and 76 over 256 x 256 x 512 (equal over 320 x 320 x 512 and 384 x 256 x 512),
// the LDS tile from 640 points on (P(k) at 640^3 1287 and 1293, 768^3 2223 and
// 2269, 1024^3 5634 and 5801).
inline int binning_blocks(int len, int cap, size_t lds, int waves, bool reg = false)
{
    if (len >= (reg ? 512 : 640)) return cap;
    const int by_lds = (int)(160 * 1024 / lds), by_waves = 16 / waves;
    const int n = by_lds < by_waves ? by_lds : by_waves, r = 256 * (n < 1 ? 1 : n);
    return cap < r ? cap : r;
}

}  // namespace lf2
