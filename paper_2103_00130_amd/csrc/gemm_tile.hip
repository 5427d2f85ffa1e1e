// Dispatch of the tiled checked GEMM over its compiled tile shapes.
#include "abft_internal.h"

namespace abft {
#define ABFT_DECL(name) hipError_t launch_gemm_tile_##name(bool, bool, bool, const GemmParams&, hipStream_t)
ABFT_DECL(a256);
ABFT_DECL(a256w24);
ABFT_DECL(a256w42);
ABFT_DECL(a128);
ABFT_DECL(a64);
ABFT_DECL(a64r4);
ABFT_DECL(a64s);
ABFT_DECL(g64);
#undef ABFT_DECL
#define ABFT_DECL(name) hipError_t launch_gemm_##name(bool, bool, bool, bool, const GemmParams&, hipStream_t)
ABFT_DECL(wk32x32w4);
ABFT_DECL(wk32x32w8);
ABFT_DECL(wk32x32w8s);
ABFT_DECL(wk32x64w4);
ABFT_DECL(wk32x64w8);
ABFT_DECL(wk64x64w4);
#undef ABFT_DECL

namespace {
// direct-to-LDS loads take whole, aligned 16-byte chunks of A (and 32-bit byte offsets into it)
bool whole_chunks(const GemmParams& p) { return p.a_vec_ok && p.K % 16 == 0 && (int64_t)(p.M - 1) * p.lda + p.K <= 0x7fffffffll; }
}  // namespace

hipError_t launch_gemm_wk(WkForm form, bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s) {
    const bool whole_a = whole_chunks(p);
    if (!whole_a && (p.mod127 || p.K < 16)) return hipErrorNotSupported;
    switch (form) {
        case kWk32x32w4: return launch_gemm_wk32x32w4(whole_a, check, want_c, want_q, p, s);
        case kWk32x32w8: {
            // (the launcher refuses when no split is planned or the caller's workspace has no room for the parts)
            const hipError_t e = launch_gemm_wk32x32w8s(whole_a, check, want_c, want_q, p, s);
            if (e != hipErrorNotSupported) return e;
            return launch_gemm_wk32x32w8(whole_a, check, want_c, want_q, p, s);
        }
        case kWk32x64w4: return launch_gemm_wk32x64w4(whole_a, check, want_c, want_q, p, s);
        case kWk32x64w8: return launch_gemm_wk32x64w8(whole_a, check, want_c, want_q, p, s);
        case kWk64x64w4: return launch_gemm_wk64x64w4(whole_a, check, want_c, want_q, p, s);
        default: return hipErrorNotSupported;
    }
}

hipError_t launch_gemm_split64(bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s) {
    if (split64_plan(p.M, p.N, p.KB2).z < 2 || !whole_chunks(p)) return hipErrorNotSupported;
    return launch_gemm_tile_a64s(check, want_c, want_q, p, s);
}

hipError_t launch_gemm_tile(int variant, bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s) {
    const bool fast_a = whole_chunks(p);
    if (!fast_a && p.mod127) return hipErrorNotSupported;
    // The row words of more than about kWsRows rows reach into the scratch that earlier calls on this workspace may have left
    // a K split's partial tiles or a padded copy of A in, so that part of them is zeroed first (one small launch, 2 us).
    if (check && ws_base_ints(p.M) > kWsScratchOff) {
        const hipError_t e = launch_fill_zero(p.ws + kWsScratchOff, ws_base_ints(p.M) - kWsScratchOff, s);
        if (e != hipSuccess) return e;
    }
    if (!fast_a) return launch_gemm_tile_g64(check, want_c, want_q, p, s);   // (whichever tile was asked for: the results are the same)
    switch (variant) {
        case kTile256: return launch_gemm_tile_a256(check, want_c, want_q, p, s);
        case kTile128: return launch_gemm_tile_a128(check, want_c, want_q, p, s);
        case kTile64: {
            // The 64x64 kernels are bound by instruction issue and the LDS reads of a wavefront, not by the matrix cores, so they
            // run as four wavefronts of 32x32 on four SIMDs (5-10 % faster than two of 32x64).  Where they are the faster ones their
            // split across workgroups or the kernel that splits K among wavefronts takes the call.
            hipError_t e = launch_gemm_split64(check, want_c, want_q, p, s);
            if (e != hipErrorNotSupported) return e;
            e = launch_gemm_wk(wk_form(p.M, p.N, p.KB2, true), check, want_c, want_q, p, s);
            if (e != hipErrorNotSupported) return e;
            const int64_t tiles = (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64);
            // short K on such a grid: a ring of four stages, all in flight before the first k-step, instead of the
            // double buffer whose every stage waits out a trip to memory (a few tenths of a microsecond at 256x512x1024)
            if (tiles <= 256 && p.K > 256) return launch_gemm_tile_a64r4(check, want_c, want_q, p, s);
            return launch_gemm_tile_a64(check, want_c, want_q, p, s);
        }
        case kTile256w24: return launch_gemm_tile_a256w24(check, want_c, want_q, p, s);
        case kTile256w42: return launch_gemm_tile_a256w42(check, want_c, want_q, p, s);
        default: return hipErrorInvalidValue;
    }
}
}  // namespace abft
