// The small levels' V-cycle legs in float32 (patch.hpp).
#include "patch.hpp"

namespace hh {
template <>
void launch_patch<float>(int kind, int leg, bool nine, bool weighted, const PatchArgs<float>& A,
                         hipStream_t s) {
    launch_patch_impl<float>(kind, leg, nine, weighted, A, s);
}
}  // namespace hh
