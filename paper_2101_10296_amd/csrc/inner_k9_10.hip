// Instantiations of the inner-state kernel (see inner_impl.hpp).
#include "inner_impl.hpp"

namespace qaoa {

hipError_t launch_inner_k9_10(int kin, bool grad, const InArgs& a, hipStream_t st) {
    switch (kin) {
        case 9: return launch_inner_k<9>(grad, a, st);
        case 10: return launch_inner_k<10>(grad, a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace qaoa
