// Instantiations of the inner-state kernel (see inner_impl.hpp).
#include "inner_impl.hpp"

namespace qaoa {

hipError_t launch_inner_k7_8(int kin, bool grad, const InArgs& a, hipStream_t st) {
    switch (kin) {
        case 7: return launch_inner_k<7>(grad, a, st);
        case 8: return launch_inner_k<8>(grad, a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace qaoa
