// Batched one-dimensional implicit viscous solver: launches for 257 to 512
// unknowns.  The row tiles of a group go to eight wavefronts, two on a SIMD, and
// not to four of up to eight tiles: those keep more vectors live than one
// register file holds, and moved every accumulator to the other file and back at
// each k tile (RMR at 384 unknowns 82 us an iteration with four, 57 with eight).
// 20 and 28 row tiles do not divide by eight: ten wavefronts of two tiles and
// seven of four give the busiest SIMD the work of 24 and 32.
#include "visc1d_kernel.hpp"

namespace vd {

hipError_t visc1d_launch_large(const Visc1dArgs& a, hipStream_t st) {
  switch (visc1d_tpw(a.ni)) {
    case 5: return launch_tpw<2, 10, OP1D_VISC>(a, st);
    case 6: return launch_tpw<3, 8, OP1D_VISC>(a, st);
    case 7: return launch_tpw<4, 7, OP1D_VISC>(a, st);
    case 8: return launch_tpw<4, 8, OP1D_VISC>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace vd
