// Outside-space tiles for double operands.
#include "triples_kernel.h"

namespace cut {

template <>
void launch_outside_t<double>(const TriArgs& a, int nops, int sq, dim3 grid, hipStream_t s) {
    switch (nops) {
        case 1: launch_outside_n<1, double>(a, sq, grid, s); break;
        case 2: launch_outside_n<2, double>(a, sq, grid, s); break;
        default: launch_outside_n<3, double>(a, sq, grid, s); break;
    }
}

}  // namespace cut
