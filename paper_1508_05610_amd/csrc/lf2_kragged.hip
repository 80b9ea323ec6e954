// lf2_kragged.hip -- the strided (y / z) pass and the fused last-axis pass
// over the line lengths of LF2_RAGGED_LENGTHS: the narrow tile's code, with
// lines, radices and thread counts fixed at compile time.  LF2_KR_PART
// selects the list (0: A, 1: B), so that the two build in parallel.
#include "lf2_kernels.hpp"
#include "lf2_lengths.hpp"

namespace lf2 {

#ifndef LF2_KR_PART
#define LF2_KR_PART 0
#endif
#if LF2_KR_PART == 0
#define LF2_KR_LENGTHS LF2_RAGGED_LENGTHS_A
#else
#define LF2_KR_LENGTHS LF2_RAGGED_LENGTHS_B
#endif

template <int L, bool NTM>
static void plain(int sign, int g, const SArgs &a, hipStream_t s)
{
    if (sign < 0)
        hipLaunchKernelGGL((k_strided<L, -1, false, NTM>), dim3(g), dim3(s_nt<L>), 0, s, a);
    else
        hipLaunchKernelGGL((k_strided<L, 1, false, NTM>), dim3(g), dim3(s_nt<L>), 0, s, a);
}

#if LF2_KR_PART == 0
hipError_t ragged_strided_a(
#else
hipError_t ragged_strided_b(
#endif
    int len, int sign, const SArgs &a, int grid_cap, size_t shm, bool ntm, hipStream_t s,
    int *grid_used)
{
    const bool epi = (a.epi & (EPI_PK | EPI_PK_AFTER | EPI_POISSON)) != 0;
    if (epi && (sign > 0 || ntm)) return hipErrorInvalidValue;
#define LF2_CASE(L)                                                                          \
    case L: {                                                                                \
        const int grid = s_grid<L>(a, grid_cap, shm);                                        \
        if (grid_used) *grid_used = grid;                                                    \
        if (epi && a.mt.k2z_unit > 0.0)                                                      \
            hipLaunchKernelGGL((k_strided<L, -1, true, true, 1>), dim3(grid), dim3(e_nt<L>), \
                               shm, s, a);                                                   \
        else if (epi)                                                                        \
            hipLaunchKernelGGL((k_strided<L, -1, true, true, 2>), dim3(grid), dim3(e_nt<L>), \
                               shm, s, a);                                                   \
        else if (ntm)                                                                        \
            plain<L, true>(sign, grid, a, s);                                                \
        else                                                                                 \
            plain<L, false>(sign, grid, a, s);                                               \
        return hipGetLastError();                                                            \
    }
    switch (len) {
        LF2_KR_LENGTHS(LF2_CASE)
    default:
        return hipErrorInvalidValue;
    }
#undef LF2_CASE
}

}  // namespace lf2
