// Host check of the grids of the binned z passes (binning_blocks): a round of
// the blocks that 256 CUs hold up to the lengths where one was measured
// faster, the partial rows' whole number past them, never more rows than
// those, and a multiple of 8 (one virtual block id walk per XCD); and of the
// derivative's planes per block (gradient_planes).
#include <stdio.h>

#include "../../paper_1508_05610_amd/csrc/lf2_rules.hpp"

int main()
{
    const int cap = 1024;
    struct {
        int len;
        size_t lds;
        int waves;
        bool reg;
        int want;
    } c[] = {
        {256, 80 * 1024, 8, true, 512},    // two blocks a CU by LDS and by waves
        {256, 81 * 1024, 8, true, 256},    // one by LDS
        {64, 20 * 1024, 8, true, 512},     // two by waves
        {512, 70 * 1024, 8, true, cap},    // the register tile from 512 points on
        {1024, 150 * 1024, 8, true, cap},
        {512, 70 * 1024, 8, false, 512},   // the LDS tile up to 639
        {216, 50 * 1024, 4, false, 768},
        {640, 70 * 1024, 8, false, cap},
        {400, 158 * 1024, 8, false, 256},
    };
    for (const auto &k : c) {
        const int g = lf2::binning_blocks(k.len, cap, k.lds, k.waves, k.reg);
        if (g != k.want || g > cap || g % 8) {
            printf("FAIL len %d lds %zu waves %d reg %d: %d blocks, want %d\n", k.len, k.lds, k.waves,
                   (int)k.reg, g, k.want);
            return 1;
        }
    }
    struct {
        int64_t waves;
        bool full;
        int want;
    } d[] = {
        {32, true, 4},     {4095, true, 4},   {4096, true, 32},  // one round, no idle lane
        {4800, true, 32},  {6144, true, 32},  {6145, true, 4},
        {4800, false, 4},  {12287, true, 4},  {12288, false, 32}, {49152, true, 32},
    };
    for (const auto &k : d)
        if (lf2::gradient_planes(k.waves, k.full, 32) != k.want) {
            printf("FAIL %lld waves full %d\n", (long long)k.waves, (int)k.full);
            return 1;
        }
    printf("ok\n");
    return 0;
}
