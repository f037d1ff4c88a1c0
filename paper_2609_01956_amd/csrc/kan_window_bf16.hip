// kan_window_bf16.hip -- the bf16 instantiations of the window kernel.
#include "kan_window_kernel.h"

namespace kan {

hipError_t launch_window_bf16(const WinGeom& g, const WinArgs& a, hipStream_t s) {
    return win::launch_ns<1>(g, a, s);
}

}  // namespace kan
