// Instantiation of the apply / count kernels for sublattice coding
// (32-bit states; the wide ones are in apply_sub_wide.hip).
#include "apply_impl.hpp"

namespace xdg {

template <>
int launch_kind<K_SUB>(bool wide, bool single, bool acc64, bool cplx, int nv, const ApplyArgs &A,
                    unsigned grid, unsigned block, size_t lds, hipStream_t st) {
    return wide ? launch_sub_wide(single, acc64, cplx, nv, A, grid, block, lds, st)
                : launch_width<uint32_t, K_SUB>(single, acc64, cplx, nv, A, grid, block, lds, st);
}

template <>
int launch_count_kind<K_SUB>(bool wide, const ApplyArgs &A, unsigned grid, unsigned block, size_t lds,
                          hipStream_t st) {
    return launch_count_impl<K_SUB>(wide, A, grid, block, lds, st);
}

}  // namespace xdg
