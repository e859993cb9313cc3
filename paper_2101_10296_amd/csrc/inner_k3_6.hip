// Instantiations of the inner-state kernel (see inner_impl.hpp).
#include "inner_impl.hpp"

namespace qaoa {

hipError_t launch_inner_k3_6(int kin, bool grad, const InArgs& a, hipStream_t st) {
    switch (kin) {
        case 3: return launch_inner_k<3>(grad, a, st);
        case 4: return launch_inner_k<4>(grad, a, st);
        case 5: return launch_inner_k<5>(grad, a, st);
        case 6: return launch_inner_k<6>(grad, a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace qaoa
