// Instantiation of the sublattice apply kernels for states wider than 32 bits.
#include "apply_impl.hpp"

namespace xdg {

int launch_sub_wide(bool single, bool acc64, bool cplx, int nv, const ApplyArgs &A, unsigned grid,
                    unsigned block, size_t lds, hipStream_t st) {
    return launch_width<uint64_t, K_SUB>(single, acc64, cplx, nv, A, grid, block, lds, st);
}

}  // namespace xdg
