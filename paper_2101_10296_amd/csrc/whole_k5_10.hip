// Instantiations of the shared-state kernel (see whole_impl.hpp).
#include "whole_impl.hpp"

namespace qaoa {

hipError_t launch_whole_k5_10(int K, bool grad, const WhArgs& a, hipStream_t st) {
    switch (K) {
        case 5: return launch_whole_k<5>(grad, a, st);
        case 6: return launch_whole_k<6>(grad, a, st);
        case 7: return launch_whole_k<7>(grad, a, st);
        case 8: return launch_whole_k<8>(grad, a, st);
        case 9: return launch_whole_k<9>(grad, a, st);
        case 10: return launch_whole_k<10>(grad, a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace qaoa
