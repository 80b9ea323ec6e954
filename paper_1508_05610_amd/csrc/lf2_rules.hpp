// lf2_rules.hpp -- rules that choose a launch's shape on the host, free of HIP
// so that they are checked without a GPU.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <vector>

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

// Planes per block of the derivative: most, or 4.  waves: of the grid with most
// (32) planes a block; full: its rows leave no lane idle.  A block marches
// through its planes one memory latency at a time, so a lattice's few blocks of
// 32 planes leave most of the chip idle, or the last of them run alone; with
// blocks of 4 (every march reads one plane more than it writes) 64^3 takes 6.6
// us of 25.2, 128^3 9.0 of 28.2, 256^3 60 of 75, 384^3 214 of 256, 200^3 with 3
// components 84 of 101.  Blocks of 32 stay where their waves fill the chip's 8192
// half to three quarters in one round with no idle lane: 640 x 640 x 96 133 us
// (147 with 4), 384 x 384 x 256 141 (144), 256^3 with 3 components 160 (166); and
// past one and a half rounds (512^3 with 3 the same with either).
inline int gradient_planes(int64_t waves, bool full, int most)
{
    const bool round = full && waves >= 4096 && waves <= 6144;
    return waves >= 12288 || round ? most : 4;
}

// A setting of a strided pass that the autotuner timed: microseconds of the
// forward and of the backward pass (below 0: not measured).
struct TileTime {
    int variant, chunk;
    double fwd, bwd;
};
// The chosen variants of the two directions, their common chunk, and the sum of
// the two passes' microseconds of the default and of the choice.
struct TileChoice {
    int fwd, bwd, chunk;
    double us_default, us;
};
// From the timed settings: per direction and chunk the default's variant, or
// one that beats the best so far by 3 %, so that noise does not flip the choice
// from run to run; of the chunks the default's, or one whose two passes
// together beat the best so far by 3 %.  d: the default setting.
inline TileChoice choose_tiles(const std::vector<TileTime> &t, TileChoice d)
{
    auto pick = [&](int chunk, int def, double TileTime::*us, int &variant) {
        double best = -1.0;
        for (int pass = 0; pass < 2; ++pass)  // the default first
            for (const TileTime &x : t) {
                if (x.chunk != chunk || (x.variant == def) != (pass == 0) || x.*us < 0) continue;
                if (best < 0 || x.*us < 0.97 * best) {
                    best = x.*us;
                    variant = x.variant;
                }
            }
        return best;
    };
    TileChoice out = d;
    out.us_default = out.us = -1.0;
    double f0 = -1.0, b0 = -1.0;
    std::vector<int> chunks{d.chunk};
    for (const TileTime &x : t) {
        if (x.chunk == d.chunk && x.variant == d.fwd) f0 = x.fwd;
        if (x.chunk == d.chunk && x.variant == d.bwd) b0 = x.bwd;
        bool seen = false;
        for (int c : chunks) seen = seen || c == x.chunk;
        if (!seen) chunks.push_back(x.chunk);
    }
    if (f0 >= 0 && b0 >= 0) out.us_default = f0 + b0;
    for (int c : chunks) {
        int vf = d.fwd, vb = d.bwd;
        const double f = pick(c, d.fwd, &TileTime::fwd, vf), b = pick(c, d.bwd, &TileTime::bwd, vb);
        if (f < 0 || b < 0) continue;
        if (out.us < 0 || f + b < 0.97 * out.us) {
            out.us = f + b;
            out.fwd = vf;
            out.bwd = vb;
            out.chunk = c;
        }
    }
    return out;
}

}  // namespace lf2
