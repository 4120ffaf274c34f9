// The triple-space contraction for float operands.
#include "triples_kernel.h"

namespace cut {

template <>
void launch_triples_t<float>(const TriArgs& a, int nops, int sq, int ti, dim3 grid, hipStream_t s) {
    switch (nops) {
        case 1: launch_triples_n<1, float>(a, sq, ti, grid, s); break;
        case 2: launch_triples_n<2, float>(a, sq, ti, grid, s); break;
        case 3: launch_triples_n<3, float>(a, sq, ti, grid, s); break;
        case 4: launch_triples_n<4, float>(a, sq, ti, grid, s); break;
        default: launch_triples_n<5, float>(a, sq, ti, grid, s); break;
    }
}

}  // namespace cut
