#pragma once

namespace qaoa {

constexpr int ZL_W = 4;   // different couplings of the leaves of one inner qubit

}  // namespace qaoa
