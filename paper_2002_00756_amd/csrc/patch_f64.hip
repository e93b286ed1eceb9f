// The small levels' V-cycle legs in float64 (patch.hpp).
#include "patch.hpp"

namespace hh {
template <>
void launch_patch<double>(int kind, int leg, bool nine, bool weighted, const PatchArgs<double>& A,
                         hipStream_t s) {
    launch_patch_impl<double>(kind, leg, nine, weighted, A, s);
}
}  // namespace hh
