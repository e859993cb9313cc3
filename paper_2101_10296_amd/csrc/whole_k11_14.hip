// Instantiations of the shared-state kernel (see whole_impl.hpp).
#include "whole_impl.hpp"

namespace qaoa {

hipError_t launch_whole_k11_14(int K, bool grad, const WhArgs& a, hipStream_t st) {
    switch (K) {
        case 11: return launch_whole_k<11>(grad, a, st);
        case 12: return launch_whole_k<12>(grad, a, st);
        case 13: return launch_whole_k<13>(grad, a, st);
        case 14: return launch_whole_k<14>(grad, a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace qaoa
