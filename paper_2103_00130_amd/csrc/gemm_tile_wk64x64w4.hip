// K split among wavefronts: 64x64 tile, four wavefronts.
#include "gemm_tile_wk.h"

namespace abft {
hipError_t launch_gemm_wk64x64w4(bool whole_a, bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s) {
    return wktile::launch_cfg<2, 2, 4, false>(whole_a, check, want_c, want_q, p, s);
}
}  // namespace abft
