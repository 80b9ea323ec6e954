// lf2_kst.hip -- instantiations and launcher of the z pass between the natural
// order and the c2c (k_z, k_x, k_y) order (k_strided_t).  In a unit of their
// own: three blocks fit a CU's LDS up to 640 points but 128, 256 and 512, and
// their registers leave room for them (80 at most) but at 384.  Compiled beside
// the binning kernels the compiler gave the same code 83 to 90 registers at 160,
// 192, 320 and 640 points, and a bound of 80 made it spill two at 192 and 640:
// c2c z pass over 320^3 with three components (us, forward and back) 460 and
// 548, with the bound 419 and 455, here 416 and 446; 192^3 with three 94 and
// 122, 84 and 104, 82 and 101; 640^3 back 1917, 1547 and 1515.
#include "lf2_kernels.hpp"
#include "lf2_lengths.hpp"

namespace lf2 {

hipError_t launch_transposed(int len, int sign, const SArgs &a, int grid_cap, hipStream_t s,
                             int *grid_used)
{
#define LF2_CASE(L)                                                                          \
    case L: {                                                                                \
        int64_t ntiles = (a.ncols + s_b(L) - 1) / s_b(L);                                    \
        int g = (int)(ntiles < grid_cap ? ntiles : grid_cap);                                \
        if (grid_used) *grid_used = g;                                                       \
        if (sign < 0)                                                                        \
            hipLaunchKernelGGL((k_strided_t<L, -1>), dim3(g), dim3(kSThreads), 0, s, a);     \
        else                                                                                 \
            hipLaunchKernelGGL((k_strided_t<L, 1>), dim3(g), dim3(kSThreads), 0, s, a);      \
        return hipGetLastError();                                                            \
    }
    switch (len) {
        LF2_S_LENGTHS(LF2_CASE)
    default:
        return hipErrorInvalidValue;
    }
#undef LF2_CASE
}

}  // namespace lf2
