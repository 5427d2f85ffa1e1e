// Tiled checked GEMM for A of any alignment, leading dimension and K (loads through registers): 64x64 workgroup tile,
// 2x2 wavefronts, a double buffer in LDS and two register sets ahead of it.
// Bound by the loads of A: sixteen bytes per lane from an address that is no multiple of four take about twice the time
// of aligned ones (10.7 against 22 TB/s out of the L2s).  2000x1000x479 with both outputs: 33-41 us with A put
// together from single bytes, 10.8 us now; 7.7 us for the aligned kernel at K = 480 (that grid has gone to
// gemm_tile_wk.h, 9.4 us).  Two register sets rather than four:
// 8 % faster there, 7.6 against 8.0 us at 256x512x1023 (three workgroups per compute unit instead of two); long loops, where
// four sets are the better ones (1000x1000x4097: 18.8 against 20.2 us), are realigned first (realign_plan in abft_internal.h).
#include "gemm_tile_async.h"

namespace abft {
hipError_t launch_gemm_tile_g64(bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s) {
    return atile::launch_cfg<64, 64, 2, 2, 2, 2>(check, want_c, want_q, p, s);
}
}  // namespace abft
