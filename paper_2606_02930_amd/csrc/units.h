// Work units of the batched kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace ite {

// Problem of unit u in a range split by the per-problem first units
// (start(g) increasing; G small): the last g with start(g) <= u.
template <typename F>
__device__ inline int unit_problem(int u, int G, F start) {
    int g = 0;
    while (g + 1 < G && start(g + 1) <= u) ++g;
    return g;
}

}  // namespace ite
