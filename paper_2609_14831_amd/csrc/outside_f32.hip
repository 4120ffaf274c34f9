// Outside-space tiles for float operands.
#include "triples_kernel.h"

namespace cut {

template <>
void launch_outside_t<float>(const TriArgs& a, int nops, int sq, dim3 grid, hipStream_t s) {
    switch (nops) {
        case 1: launch_outside_n<1, float>(a, sq, grid, s); break;
        case 2: launch_outside_n<2, float>(a, sq, grid, s); break;
        case 3: launch_outside_n<3, float>(a, sq, grid, s); break;
        case 4: launch_outside_n<4, float>(a, sq, grid, s); break;
        default: launch_outside_n<5, float>(a, sq, grid, s); break;
    }
}

}  // namespace cut
