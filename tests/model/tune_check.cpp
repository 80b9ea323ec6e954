// Host check of the autotuner's choice (choose_tiles): a direction's winner is
// chosen by that direction's times, the default setting stays within 3 %, and
// the chunk, which the directions share, by both together.
#include <stdio.h>

#include "../../paper_1508_05610_amd/csrc/lf2_rules.hpp"

using lf2::TileChoice;
using lf2::TileTime;

static int check(const char *what, const TileChoice &c, int fwd, int bwd, int chunk, double us0, double us)
{
    if (c.fwd == fwd && c.bwd == bwd && c.chunk == chunk && c.us_default == us0 && c.us == us) return 0;
    printf("FAIL %s: %d/%d chunk %d, %g -> %g; want %d/%d chunk %d, %g -> %g\n", what, c.fwd, c.bwd,
           c.chunk, c.us_default, c.us, fwd, bwd, chunk, us0, us);
    return 1;
}

int main()
{
    int bad = 0;
    // a 512^3 real z pass: nontemporal wins backward alone, and is the default there
    const std::vector<TileTime> z = {{2, 16, 198, 208}, {3, 16, 219, 229}, {0, 16, 194, 229}, {1, 16, 219, 237}};
    bad += check("default kept", lf2::choose_tiles(z, {0, 2, 16, -1, -1}), 0, 2, 16, 402, 402);
    // the same times with a default of normal accesses both ways
    bad += check("backward found", lf2::choose_tiles(z, {0, 0, 16, -1, -1}), 0, 2, 16, 423, 402);
    // the default is another tile than the first timed, within 3 % of it
    const std::vector<TileTime> w = {{2, 16, 99, 99}, {0, 16, 98, 98}, {1, 16, 100, 100}};
    bad += check("tie goes to the default", lf2::choose_tiles(w, {1, 1, 16, -1, -1}), 1, 1, 16, 200, 200);
    // chunk 4 wins together although its forward pass loses
    const std::vector<TileTime> c = {{0, 16, 100, 100}, {0, 4, 102, 80}, {0, 64, 97.5, 97.5}};
    bad += check("chunk", lf2::choose_tiles(c, {0, 0, 16, -1, -1}), 0, 0, 4, 200, 182);
    // a setting that failed one way is not chosen that way
    const std::vector<TileTime> f = {{2, 16, 50, -1}, {0, 16, 100, 100}};
    bad += check("failed", lf2::choose_tiles(f, {0, 0, 16, -1, -1}), 2, 0, 16, 200, 150);
    // nothing measured: the default, unmeasured
    bad += check("none", lf2::choose_tiles({{0, 16, -1, -1}}, {0, 3, 16, -1, -1}), 0, 3, 16, -1, -1);
    if (!bad) printf("ok\n");
    return bad != 0;
}
