// K split among wavefronts: 32x32 tile, eight wavefronts.
#include "gemm_tile_wk.h"

namespace abft {
hipError_t launch_gemm_wk32x32w8(bool whole_a, bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s) {
    return wktile::launch_cfg<1, 1, 8, false>(whole_a, check, want_c, want_q, p, s);
}
}  // namespace abft
