// The triple-space contraction for double operands.
#include "triples_kernel.h"

namespace cut {

template <>
void launch_triples_t<double>(const TriArgs& a, int nops, int sq, int ti, dim3 grid, hipStream_t s) {
    switch (nops) {
        case 1: launch_triples_n<1, double>(a, sq, ti, grid, s); break;
        case 2: launch_triples_n<2, double>(a, sq, ti, grid, s); break;
        default: launch_triples_n<3, double>(a, sq, ti, grid, s); break;
    }
}

}  // namespace cut
