// kan_window_f32.hip -- the f32 instantiations of the window kernel.
#include "kan_window_kernel.h"

namespace kan {

hipError_t launch_window_f32(const WinGeom& g, const WinArgs& a, hipStream_t s) {
    return win::launch_ns<2>(g, a, s);
}

}  // namespace kan
