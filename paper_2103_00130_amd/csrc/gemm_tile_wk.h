// Checked u8 x s8 -> s32 GEMM for gfx950 for grids that do not fill the chip: K split among the wavefronts of a workgroup.
//
// The same steps as gemm_tile_async.h (Algorithm 1 of arXiv 2103.00130), in a form for calls of a few microseconds, where the
// chain of dependent waits of one workgroup is what counts.
//  * Small tiles (32x32, 32x64; 64x64 where a long K makes the loads the limit), so that few rows or columns still give many
//    workgroups; the W wavefronts of a workgroup take the stages of 128 k in turn, each for the whole tile and with a part of LDS
//    of its own: nothing is shared until the end, so the K loop has no barrier, and a wavefront waits for its own loads alone.
//  * A stage goes global -> LDS directly (rows of A as whole 128-byte lines, XOR-swizzled; packed B as it lies) and from there into
//    registers all at once; the loads of the next stage go out before the matrix instructions of this one.
//    Rows of any alignment (kAny) come in through registers instead.  (A straight from memory in the order that the matrix
//    instructions want costs 64 cycles a load instead of 24: lanes next to each other hold different rows.)
//  * At the end the wavefronts leave their accumulators in LDS and each of (up to) four adds up and finishes rows of its own: the
//    sums over a row, the arrival at its word, the stores while that comes back.
//  * The checksum product of a row is dealt out over the tile columns of the grid by k-steps of 32, within every wavefront's stages,
//    so that no wavefront has more than its share of it.
//  * kSplit: K split across workgroups as well (few tiles, a long K).  Each finishing wavefront stores its rows' part of the
//    workgroup's sums in the workspace and takes a ticket of those rows; the last one adds the others' parts and goes on.
// Bound: launch and latency below about 6 us; with a long K what a wavefront with one stage in flight gets from its L2: 1024x1024x4096 takes
// 0.85 us for the stages of its four wavefronts, 77 KB/us a compute unit (41 to 44 bytes a cycle at the 1.75 to 1.9 GHz of a counter run),
// six to seven tenths of what such loads reach alone; the matrix pipes are busy 0.17 of the time, the LDS 0.18, wavefronts wait 0.37.
// More in flight is no help: loads alone take 7.2 us of that shape's 11.5, with fragment reads and matrix instructions 8.4, one stage or two in flight,
// and sixteen workgroups draw 151 KB/us each with one, a compute unit's 64 bytes a cycle (99x108x6176: 7.5 us, 8.2 with two).
// Measured, this kernel against the 64x64 tiles of gemm_tile_async.h or the streaming kernel that ran before (us): 64x256x512 4.9 -> 4.0,
// 256x512x1024 requantized 6.8 -> 4.9, 64x1024x1024 5.9 -> 4.5, 130x65x2064 8.8 -> 5.4, 500x500x2000 9.1 -> 6.2, 441x479x1255 8.7 -> 5.2,
// 32x4096x4096 9.4 -> 6.1, 29x9088x1872 10.6 -> 6.1, 64x8192x2048 10.0 -> 8.5, 1024x1024x4096 requantized 13.1 -> 12.1 (11.6 on another
// device).  Of 64x256x512: 0.5 until the first load is out, 0.7 for its only stage, 0.4 until the sums are there, 0.6 for the arrival; an
// empty launch takes 1.6.
#pragma once
#include <type_traits>
#include <utility>

#include "../../include/abft_gemm.h"
#include "abft_internal.h"
#include "gemm_tile_async.h"

namespace abft {
namespace wktile {

using atile::floor_mod127;
using atile::kOutC;
using atile::kOutQ;
using atile::sum32;
using atile::v16i;
using atile::v4i;
using atile::v4i_any;
constexpr int BK = 128;

// LDS of a wavefront: [A rows][B units][1 KiB for the digits of a stage], later its part of the sums
template <int TM, int TN>
constexpr int slot_bytes() { return 32 * TM * BK + 32 * TN * BK + 1024; }
template <int TM, int TN>
constexpr int xch_bytes() { return TM * TN * 4096 + TN * 256 + TM * 512; }
template <int TM, int TN>
constexpr int wave_bytes() { return ((slot_bytes<TM, TN>() > xch_bytes<TM, TN>() ? slot_bytes<TM, TN>() : xch_bytes<TM, TN>()) + 1023) / 1024 * 1024; }

// sixteen bytes per lane from sbase + voff + OFF to LDS address lds + LDS + OFF + lane * 16 (see gemm_tile_async.h); kStream: not kept
// in the caches
template <int LDS, int OFF, bool kStream>
__device__ __attribute__((always_inline)) inline void load_to_lds(uint32_t lds, uint32_t voff, const void* sbase) {
    if constexpr (kStream)
        asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3 nt" ::"s"(lds), "v"(voff), "s"(sbase), "n"(OFF), "n"(LDS) : "m0", "scc", "memory");
    else
        asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" ::"s"(lds), "v"(voff), "s"(sbase), "n"(OFF), "n"(LDS) : "m0", "scc", "memory");
}
// The digit MFMA with its accumulator in ordinary vector registers: left to the compiler, which gives the MFMAs of a function one
// class of registers for their results, the digit accumulators move to accumulation registers and back around every one of them.
// The wait states that a vector write needs before a matrix instruction reads the register are part of the string.
__device__ __attribute__((always_inline)) inline void mfma_digits(v16i& c, v4i a, v4i b) {
    asm volatile("s_nop 1\n\tv_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
template <int N, class Fn, int... I>
__device__ __attribute__((always_inline)) inline void for_each_impl(Fn&& fn, std::integer_sequence<int, I...>) { (fn(std::integral_constant<int, I>{}), ...); }
template <int N, class Fn>
__device__ __attribute__((always_inline)) inline void for_each(Fn&& fn) { for_each_impl<N>(fn, std::make_integer_sequence<int, N>{}); }

// slots: 0, or so many words between the arrivals of many tile columns and a row's word (row_slots)
template <int TM, int TN, int W, bool kCheck, int kOut, bool kAny, bool kSplit>
__global__ __launch_bounds__(W * 64) void gemm_tile_wk_kernel(const GemmParams p, const int tiles_m, const int tiles_n, const uint32_t strip_rcp,
                                                              const int slots, const int slot_rows) {
    constexpr int BM = 32 * TM, BN = 32 * TN;
    constexpr int A_LD = BM / 8, B_LD = BN / 8;   // 1 KiB loads per stage
    constexpr int WAVE = wave_bytes<TM, TN>();
    constexpr bool kWantC = (kOut & kOutC) != 0, kWantQ = (kOut & kOutQ) != 0;
    constexpr int F = W < 4 * TM ? W : 4 * TM;   // wavefronts that finish the tile
    constexpr int PG = 4 * TM / F;               // groups of eight rows that each of them finishes
    constexpr bool kMayStream = W == 8 || TM == 2;   // (the other forms never: of one row of tiles they have few stages, wk_form, and of more, of which 32x64 has any number, none streams)
    static_assert(4 * TM % F == 0 && TM <= 2, "equal shares of the tile; one or two blocks of rows");

    extern __shared__ __align__(1024) uint8_t smem[];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint8_t* const mine = smem + wave * WAVE;
    const uint32_t lds_mine = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)((__attribute__((address_space(3))) uint8_t*)smem) + wave * WAVE);

    // the launch parameters in one go: left to the compiler they are fetched where they are used, a trip to memory each time
    int32_t* C = p.C;
    int64_t ldc = p.ldc, ldcq = p.ldcq;
    uint8_t* Cq = p.Cq;
    int32_t* row_flags = p.row_flags;
    int32_t* err_count = p.err_count;
    int32_t* ws = p.ws;
    int n_inj = p.n_inj, rq_zA = p.rq.zA, rq_zC = p.rq.zC;
    asm volatile("" : "+s"(C), "+s"(ldc), "+s"(row_flags), "+s"(err_count), "+s"(ws), "+s"(n_inj));
    if (kWantQ) asm volatile("" : "+s"(Cq), "+s"(ldcq), "+s"(rq_zA), "+s"(rq_zC));
    int tile_m, tile_n, z = 0;
    {
        // An XCD gets a compact block of tiles, walked in strips of four tile rows (see gemm_tile_async.h), whatever their number: with
        // the tiles of a column spread over the XCDs every L2 fetches it (us, spread / in blocks: 64x5000x12000 23.1 / 18.5,
        // 128x3000x9008 21.9 / 14.9, 100x3000x9001 21.8 / 16.6, 600x3000x250 8.1 / 7.3).  Quotients by multiplication with rounded-up
        // reciprocals, exact for the at most 65535 tiles of a launch.
        const int n_tiles = tiles_m * tiles_n;
        int t = (int)blockIdx.x;
        if (kSplit) {   // slice z, then the tile
            for (; t >= n_tiles; t -= n_tiles) ++z;
        } else {
            const int x = t & 7;
            t = x * (n_tiles >> 3) + (t >> 3);
            // The first n_tiles % 8 XCDs have a tile more.  (The empty asm keeps this a branch of its own: as part of the sum above it moves
            // the loads of the launch parameters apart, 0.1 us a call.)
            if (n_tiles % 8 != 0) {
                int more = min(x, n_tiles & 7);
                asm volatile("" : "+s"(more));
                t += more;
            }
        }
        const int strip = (int)__umulhi((uint32_t)t, strip_rcp), r = t - strip * min(tiles_m, 4) * tiles_n;
        const int h = min(4, tiles_m - strip * 4);
        tile_n = h == 4 ? r >> 2 : h == 3 ? (int)__umulhi((uint32_t)r, 0x55555556u) : r >> (h - 1);
        tile_m = strip * 4 + r - tile_n * h;
    }
    const int row0 = tile_m * BM, col0 = tile_n * BN;
    // this workgroup's run of stages
    const int NS = kSplit ? p.split_q + (z < p.split_r ? 1 : 0) : p.KB2;
    const int s_base = kSplit ? share_begin(z, p.split_q, p.split_r) : 0;
    const int lcol = lane & 31, lhalf = lane >> 5;

    auto wait_lds = []() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
    auto wait_vmem_but = [](auto n_c) __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(n_c)::value) : "memory"); };

    // this wavefront's share of the checksum product: k-steps [u_lo, u_hi) of the 4 * (its stages)
    const int n_mine = (NS + W - 1 - wave) / W;
    const bool longer = n_mine > p.wk_stages;
    const int share_q = longer ? p.wk_share_q1 : p.share_q, share_r = longer ? p.wk_share_r1 : p.share_r;
    const int u_lo = kCheck ? share_begin(tile_n, share_q, share_r) : 0, u_hi = kCheck ? share_begin(tile_n + 1, share_q, share_r) : 0;
    // (of any wavefront of the workgroup: the first has as many stages as any, the last as few)
    const bool any_digits = kCheck && ((NS / W == p.wk_stages && (p.share_q > 0 || tile_n < p.share_r)) ||
                                       ((NS + W - 1) / W > p.wk_stages && (p.wk_share_q1 > 0 || tile_n < p.wk_share_r1)));
    // sum_k S_B[k], which the first tile column needs at the very end; a vector load, for which nothing waits before that
    int32_t total_sb = 0;
    if (kCheck && tile_n == 0) {
        uint32_t zero;
        asm("v_mov_b32 %0, 0" : "=v"(zero));
        total_sb = p.total[zero];
    }
    const bool clears = kCheck && tiles_m == 1 && !p.err_accumulate && err_count != nullptr && tile_n == 0 && z == 0;
    if (clears && tid == 0) __hip_atomic_store(err_count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    int32_t col_sum[TN], col_bias[TN];
    float col_mult[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        col_sum[t] = col_bias[t] = 0;
        col_mult[t] = 0.0f;
        if (kWantQ) {
            const int col = min(col0 + t * 32 + lcol, p.N - 1);
            col_sum[t] = p.colsum[col];
            col_mult[t] = p.rq.mult[p.rq.per_channel ? col : 0];
            if (p.rq.bias) col_bias[t] = p.rq.bias[col];
        }
    }
    uint32_t a_voff[A_LD];
    const uint8_t* a_row[A_LD];
    v4i ra[A_LD] = {};
    // loads whose rows all lie past the last one are left out: what LDS holds there goes into sums that nobody stores or reports
    const int a_loads = min((p.M - row0 + 7) / 8, A_LD);
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
        const int r = i * 8 + (lane >> 3);
        if constexpr (kAny) a_row[i] = p.A + (int64_t)min(row0 + r, p.M - 1) * p.lda;
        else a_voff[i] = (uint32_t)min(row0 + r, p.M - 1) * (uint32_t)p.lda + (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
    }
    constexpr int64_t B_KB_STRIDE = (int64_t)kUnitsPerTile * kUnitBytes;
    const int8_t* const b_base = p.packed + packed_unit_offset(col0 / kTileN, 0, (col0 % kTileN) / kUnitN, p.KB2 * 2);
    const uint32_t b_voff = lane * 16;
    const bool stream = p.wk_stream != 0;

    const bool cut = p.K < p.KB2 * BK;   // the last stage is cut off: a chunk at or past K is re-read from the last whole chunk (it meets zero rows of B)
    const int c16_over = ((lane & 7) ^ ((lane >> 4) & 7)) * 16 - (p.K - 16 - (p.KB2 - 1) * BK);           // of loads of even number ...
    const int c16_over1 = ((lane & 7) ^ (((lane >> 4) & 7) ^ 4)) * 16 - (p.K - 16 - (p.KB2 - 1) * BK);    // ... and of odd number
    // stage number i of this wavefront
    auto issue_stage = [&](int i) __attribute__((always_inline)) {
        const int s = s_base + wave + i * W;
        if (kCheck && u_lo < 4 * i + 4 && u_hi > 4 * i)
            load_to_lds<(BM + BN) * BK, 0, false>(lds_mine, (uint32_t)min(lane * 16, 512 - 16), p.limbs + (int64_t)s * 512);
        if constexpr (!kAny) {
            const uint8_t* const a = p.A + (int64_t)s * BK;
            const bool last = cut && s == p.KB2 - 1;
            const uint32_t over0 = last ? (uint32_t)max(c16_over, 0) : 0u, over1 = last ? (uint32_t)max(c16_over1, 0) : 0u;
            for_each<A_LD>([&](auto n) __attribute__((always_inline)) {
                constexpr int at = n.value;
                if (at < a_loads) load_to_lds<at * 1024, 0, false>(lds_mine, a_voff[at] - (at & 1 ? over1 : over0), a);
            });
        }
        auto load_b = [&](auto stream_c) __attribute__((always_inline)) {
            for_each<B_LD>([&](auto n) __attribute__((always_inline)) {
                constexpr int kbl = n.value / (B_LD / 2), c = n.value % (B_LD / 2);
                load_to_lds<BM * BK + kbl * (BN * 64), c * 1024, decltype(stream_c)::value>(lds_mine, b_voff, b_base + (int64_t)(2 * s + kbl) * B_KB_STRIDE);
            });
        };
        if (kMayStream && stream) load_b(std::true_type{});
        else load_b(std::false_type{});
        if constexpr (kAny) {
            // rows of any alignment come in through registers (behind the loads of B: the wait for them covers those); nothing
            // past the operand is read: a chunk at or past K - 16 is loaded from K - 16
            const int k = min(s * BK + (lane & 7) * 16, p.K - 16);
#pragma unroll
            for (int n = 0; n < A_LD; ++n)
                if (n < a_loads) ra[n] = *reinterpret_cast<const v4i_any*>(a_row[n] + k);
        }
    };
    if (wave < NS) issue_stage(0);
    v16i acc[TM][TN], dacc[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int e = 0; e < 16; ++e) dacc[i][e] = 0;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;
    }
    uint32_t bsum[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) bsum[t] = 0;

    const int a_swz = (lane >> 1) & 7;
    int a_off[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a_off[j] = lcol * BK + (((2 * j + lhalf) ^ a_swz) << 4);

    for (int i = 0; wave + i * W < NS; ++i) {
        if constexpr (kAny) {
            // ... and the one that holds the end of the row is shifted down to its place
            const int over = s_base + wave + i * W == p.KB2 - 1 ? (16 - (p.K & 15)) & 15 : 0;
            const bool end_chunk = (p.KB2 - 1) * BK + (lane & 7) * 16 == (p.K & ~15);
#pragma unroll
            for (int n = 0; n < A_LD; ++n) {
                const int r = n * 8 + (lane >> 3);
                v4i v = ra[n];
                if (over) {
                    const v4i m = shift_down(v, over);
                    v = end_chunk ? m : v;
                }
                *reinterpret_cast<v4i*>(mine + r * BK + (((lane & 7) ^ ((r >> 1) & 7)) << 4)) = v;
            }
        }
        wait_vmem_but(std::integral_constant<int, 0>{});
        v4i fa[4][TM], fb[4][TN], limb[4];
        const uint8_t* const sB = mine + BM * BK;
        const bool dig = kCheck && u_lo < 4 * i + 4 && u_hi > 4 * i;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int m = 0; m < TM; ++m) fa[j][m] = *reinterpret_cast<const v4i*>(mine + a_off[j] + m * 32 * BK);
#pragma unroll
            for (int t = 0; t < TN; ++t) fb[j][t] = *reinterpret_cast<const v4i*>(sB + (j >> 1) * (BN * 64) + t * 2048 + (j & 1) * 1024 + lane * 16);
        }
        if (dig)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                limb[j] = *reinterpret_cast<const v4i*>(sB + BN * BK + ((((j >> 1) * 4 + (j & 1) * 2 + lhalf) * kLimbs + (lane & 3)) << 4));
        if (wave + (i + 1) * W < NS) {
            wait_lds();
            __builtin_amdgcn_sched_barrier(0);
            issue_stage(i + 1);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int m = 0; m < TM; ++m) {
                fa[j][m] ^= (int)0x80808080;
#pragma unroll
                for (int t = 0; t < TN; ++t) acc[m][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[j][m], fb[j][t], acc[m][t], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int d = 0; d < 4; ++d) bsum[t] = (uint32_t)__builtin_amdgcn_sdot4(fb[j][t][d], 0x01010101, (int)bsum[t], false);
        }
#pragma unroll
        for (int x = 0; x < 4 * TM * TN; ++x) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                // an MFMA ...
            __builtin_amdgcn_sched_group_barrier(0x002, (4 * TM + 4 * TN) / (TM * TN), 0);    // ... and its share of the vector work
        }
        if (dig) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (4 * i + j >= u_lo && 4 * i + j < u_hi)
#pragma unroll
                    for (int m = 0; m < TM; ++m) mfma_digits(dacc[m], fa[j][m], limb[j]);
            // the distance from these matrix instructions to whatever reads their results, which go through the string so that nothing that
            // the compiler does with them comes before it
            if constexpr (TM == 1) asm volatile("s_nop 7\n\ts_nop 7" : "+v"(dacc[0]));
            else asm volatile("s_nop 7\n\ts_nop 7" : "+v"(dacc[0]), "+v"(dacc[1]));
        }
    }
    // ---- the partial tiles meet: every wavefront leaves its own in the part of LDS that its stages went through
    {
        v4i* const x = reinterpret_cast<v4i*>(mine);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    x[((i * 4 + g) * TN + t) * 64 + lane] = v4i{acc[i][t][4 * g], acc[i][t][4 * g + 1], acc[i][t][4 * g + 2], acc[i][t][4 * g + 3]};
        int32_t* const xb = reinterpret_cast<int32_t*>(mine + TM * TN * 4096);
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            const auto halves = __builtin_amdgcn_permlane32_swap(bsum[t], bsum[t], false, false);
            xb[t * 64 + lane] = (int32_t)(halves[0] + halves[1]);
        }
        if (any_digits && lcol < 4) {
            v4i* const xd = reinterpret_cast<v4i*>(mine + TM * TN * 4096 + TN * 256);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    xd[(i * 4 + g) * 8 + lhalf * 4 + lcol] = v4i{dacc[i][4 * g], dacc[i][4 * g + 1], dacc[i][4 * g + 2], dacc[i][4 * g + 3]};
        }
    }
    if (clears && wave == 0) wait_vmem_but(std::integral_constant<int, 0>{});
    __syncthreads();
    if (W > F && wave >= F) return;

    RequantCol rqc[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        rqc[t].sub = (uint32_t)rq_zA * (uint32_t)col_sum[t] - (uint32_t)col_bias[t];
        rqc[t].mult = col_mult[t];
    }
    v4i val[PG][TN], ck[PG];
    int32_t cs[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) cs[t] = 0;
#pragma unroll
    for (int q = 0; q < PG; ++q) {
        ck[q] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int t = 0; t < TN; ++t) val[q][t] = v4i{0, 0, 0, 0};
    }
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint8_t* const from = smem + w * WAVE;
#pragma unroll
        for (int q = 0; q < PG; ++q)
#pragma unroll
            for (int t = 0; t < TN; ++t) val[q][t] += reinterpret_cast<const v4i*>(from)[((wave * PG + q) * TN + t) * 64 + lane];
#pragma unroll
        for (int t = 0; t < TN; ++t) cs[t] += reinterpret_cast<const int32_t*>(from + TM * TN * 4096)[t * 64 + lane];
    }
    if (any_digits)
#pragma unroll
        for (int w = 0; w < W; ++w)
#pragma unroll
            for (int q = 0; q < PG; ++q)
                ck[q] += reinterpret_cast<const v4i*>(smem + w * WAVE + TM * TN * 4096 + TN * 256)[(wave * PG + q) * 8 + lhalf * 4 + (lane & 3)];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        cs[t] *= 128;
#pragma unroll
        for (int q = 0; q < PG; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) val[q][t][e] += cs[t];
    }
    // row of group q, element e: rbase + 8 * q + 4 * lhalf + e
    const int rbase = row0 + wave * PG * 8;
    // sums over the lanes of a quad, value number lane & 3 to each
    auto quad_sums = [&](const uint32_t(&v)[4]) __attribute__((always_inline)) {
        const bool b0 = lane & 1, b1 = lane & 2;
        const uint32_t x0 = (b0 ? v[1] : v[0]) + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b0 ? v[0] : v[1]), 0xB1, 0xF, 0xF, true);
        const uint32_t x1 = (b0 ? v[3] : v[2]) + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b0 ? v[2] : v[3]), 0xB1, 0xF, 0xF, true);
        return (b1 ? x1 : x0) + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b1 ? x0 : x1), 0x4E, 0xF, 0xF, true);
    };
    uint32_t chk[PG];   // checksum product of row 8 * q + 4 * lhalf + (lane & 3): digit d, in lane d of every quad, times 256^d
#pragma unroll
    for (int q = 0; q < PG; ++q) {
        chk[q] = 0;
        if (any_digits) {
            uint32_t k[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) k[e] = (uint32_t)ck[q][e] << (8 * (lane & 3));
            chk[q] = quad_sums(k);
        }
    }

    // ---- K split across workgroups: the parts of these rows meet in the last arrival
    if constexpr (kSplit) {
        const int Z = p.ksplit, mine_of = ((tile_m * tiles_n + tile_n) * F + wave);
        constexpr int kInts = PG * (4 * TN + 1) * 64;
        static_assert(F * kInts == kWkPartInts, "layout of a part");
        int32_t* const part = p.ws_part + (size_t)mine_of * Z * kInts + lane;
        {
            // device-scope stores (they pass through the L2, which is not coherent with the other seven): once they are
            // acknowledged the part is in memory
            int32_t* const out = part + (size_t)z * kInts;
            int k = 0;
#pragma unroll
            for (int q = 0; q < PG; ++q) {
#pragma unroll
                for (int t = 0; t < TN; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) __hip_atomic_store(out + (k++) * 64, val[q][t][e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(out + (k++) * 64, (int32_t)chk[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        wait_vmem_but(std::integral_constant<int, 0>{});
        int ticket = 0;
        if (lane == 0) ticket = __hip_atomic_fetch_add(p.ws_tickets + mine_of, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_readfirstlane(ticket) != Z - 1) return;
        if (lane == 0) __hip_atomic_store(p.ws_tickets + mine_of, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // four parts at a time, so that their loads are in flight together (a slice past the last one, or this workgroup's own, is
        // read and not added)
        for (int z0 = 0; z0 < Z; z0 += 4) {
            int32_t v[4][PG * (4 * TN + 1)];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int k = 0; k < PG * (4 * TN + 1); ++k)
                    v[j][k] = __hip_atomic_load(part + (size_t)min(z0 + j, Z - 1) * kInts + k * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int32_t use = (z0 + j < Z && z0 + j != z) ? -1 : 0;
                int k = 0;
#pragma unroll
                for (int q = 0; q < PG; ++q) {
#pragma unroll
                    for (int t = 0; t < TN; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e) val[q][t][e] += v[j][k++] & use;
                    chk[q] += (uint32_t)(v[j][k++] & use);
                }
            }
        }
    }

    if (n_inj > 0) {
        const abft_inject_t* inj = reinterpret_cast<const abft_inject_t*>(p.inj);
        for (int n = 0; n < n_inj; ++n) {
            const int r = inj[n].row - rbase, c = inj[n].col - col0;
            if (r < 0 || r >= 8 * PG || inj[n].row >= p.M || c < 0 || c >= BN || inj[n].col >= p.N) continue;
            const bool hit = lcol == (c & 31) && lhalf == ((r >> 2) & 1);
#pragma unroll
            for (int q = 0; q < PG; ++q)
#pragma unroll
                for (int t = 0; t < TN; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (hit && q == (r >> 3) && t == (c >> 5) && e == (r & 3)) val[q][t][e] ^= (int)inj[n].xor_mask;
        }
    }
    const bool mod127 = kCheck && p.mod127 != 0;
    uint32_t d = 0;   // of the row that this lane reports: group lcol >> 2, element lane & 3
    const int row = rbase + 8 * (lcol >> 2) + 4 * lhalf + (lane & 3);
    const bool reports = kCheck && lcol < 4 * PG && row < p.M;
    // A row's word counts the tile columns that have arrived and adds up their differences (see gemm_tile_async.h).  Where many
    // would arrive at it one after the other, the columns of a slot meet at a word of their own first.
    unsigned long long* const words = reinterpret_cast<unsigned long long*>(ws + kWsHeaderInts);
    const int slot = tile_n & (slots - 1);
    unsigned long long* const w_first = words + (slots > 0 ? slot * slot_rows : 0) + row;
    const uint32_t expected = slots > 0 ? (uint32_t)(tiles_n - slot + slots - 1) >> __builtin_ctz((unsigned)slots) : (uint32_t)tiles_n;
    unsigned long long old = 0;
    if (kCheck) {
        // quad sums over the eight quads that share lane >> 5
        auto half_sum = [&](uint32_t v) __attribute__((always_inline)) {
            v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, true);   // row_ror:4
            v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);   // row_ror:8
            const auto sw = __builtin_amdgcn_permlane16_swap(v, v, false, false);
            return sw[0] + sw[1];
        };
        auto row_sums = [&](auto mod_c) __attribute__((always_inline)) {
            constexpr bool MOD = decltype(mod_c)::value;
#pragma unroll
            for (int q = 0; q < PG; ++q) {
                uint32_t rs[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    rs[e] = 0;
#pragma unroll
                    for (int t = 0; t < TN; ++t) rs[e] += MOD ? (uint32_t)floor_mod127((long long)val[q][t][e]) : (uint32_t)val[q][t][e];
                }
                const uint32_t sum = half_sum(quad_sums(rs));
                const uint32_t x = MOD ? (uint32_t)floor_mod127((long long)sum - (long long)(int32_t)chk[q] - 128ll * (long long)total_sb)
                                       : sum - chk[q] - 128u * (uint32_t)total_sb;
                if (q == 0 || (lcol >> 2) == q) d = x;
            }
        };
        if (mod127) row_sums(std::true_type{});
        else row_sums(std::false_type{});
        // (the stores of the results go out while the word comes back)
        if (reports && tiles_n > 1) old = __hip_atomic_fetch_add(w_first, ((unsigned long long)d << 32) | 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const bool full = row0 + BM <= p.M && col0 + BN <= p.N;
    auto store = [&](auto full_c) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full_c)::value;
        int32_t* c = kWantC ? C + (int64_t)rbase * ldc + col0 + (4 * lhalf * ldc + lcol) : nullptr;
        uint8_t* cq = kWantQ ? Cq + (int64_t)rbase * ldcq + col0 + ((4 * lhalf + (lane & 3)) * ldcq + (lcol & ~3)) : nullptr;
        const int rows = p.M - rbase - 4 * lhalf, cols = p.N - col0 - lcol, left = p.N - col0 - (lcol & ~3);
#pragma unroll
        for (int q = 0; q < PG; ++q) {
            if (kWantC) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
#pragma unroll
                    for (int t = 0; t < TN; ++t)
                        if (FULL || (8 * q + e < rows && t * 32 < cols)) c[t * 32] = val[q][t][e];
                    c += e < 3 ? ldc : 5 * ldc;
                }
            }
            if (kWantQ) {
#pragma unroll
                for (int t = 0; t < TN; ++t) {
                    uint32_t w = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) w = requant_into(w, e, val[q][t][e], rqc[t], rq_zC);
                    w = turn_quad(w, lane);
                    if (FULL) store_quad(cq + t * 32, w, 4);
                    else if (8 * q + (lane & 3) < rows && t * 32 < left) store_quad(cq + t * 32, w, left - t * 32);
                }
                cq += 8 * ldcq;
            }
        }
    };
    if (full) store(std::true_type{});
    else store(std::false_type{});

    if (kCheck) {
        bool fin = false, bad = false;
        if (reports && (uint32_t)old == expected - 1u) {
            uint32_t diff = (uint32_t)(old >> 32) + d;
            fin = true;
            if (tiles_n > 1) __hip_atomic_store(w_first, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (slots > 0) {
                unsigned long long* const w_row = words + slots * slot_rows + row;
                old = __hip_atomic_fetch_add(w_row, ((unsigned long long)diff << 32) | 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                fin = (uint32_t)old == (uint32_t)slots - 1u;
                diff += (uint32_t)(old >> 32);
                if (fin) __hip_atomic_store(w_row, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            bad = fin && (mod127 ? diff % 127u != 0 : diff != 0);
            if (fin) row_flags[row] = bad ? 1 : 0;
        }
        const unsigned long long fin_mask = __ballot(fin), bad_mask = __ballot(fin && bad);
        if (err_count == nullptr) {
            // no count was asked for
        } else if (p.err_accumulate || tiles_m == 1) {
            if (bad_mask != 0ull && lane == __builtin_ctzll(bad_mask))
                __hip_atomic_fetch_add(err_count, (int32_t)__builtin_popcountll(bad_mask), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            // Finished rows are reported, the corrupted ones among them in the high half; the report that brings the count to M writes
            // errCount.  The wavefronts of a workgroup report together (a K split's finish apart), and where there are many
            // tile rows the reports of every sixteenth meet at a word of their own first (2739x80x112, 86 tile rows of 32:
            // 8.4 us with a report per wavefront at one word).
            unsigned long long report = ((unsigned long long)__builtin_popcountll(bad_mask) << 32) | (uint32_t)__builtin_popcountll(fin_mask);
            if constexpr (!kSplit && F > 1) {
                unsigned long long* const s_report = reinterpret_cast<unsigned long long*>(smem + W * WAVE);
                if (lane == 0) s_report[wave] = report;
                __syncthreads();
                report = 0;
#pragma unroll
                for (int w = 0; w < F; ++w) report += s_report[w];
                if (wave != 0) return;
            }
            if (lane == 0 && (uint32_t)report != 0u) {
                unsigned long long* const head = reinterpret_cast<unsigned long long*>(ws);
                bool go = true;
                if (tiles_m > 2 * kWsDoneSlots) {
                    const int slot_m = tile_m & (kWsDoneSlots - 1), last = tiles_m - 1;
                    const int rows = ((last - slot_m) / kWsDoneSlots + 1) * BM - ((last & (kWsDoneSlots - 1)) == slot_m ? tiles_m * BM - p.M : 0);
                    const unsigned long long before = __hip_atomic_fetch_add(head + slot_m, report, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    report += before;
                    go = (uint32_t)report == (uint32_t)rows;
                    if (go) __hip_atomic_store(head + slot_m, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (go) {
                    unsigned long long* const w_done = reinterpret_cast<unsigned long long*>(ws + kWsDoneWord);
                    report += __hip_atomic_fetch_add(w_done, report, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((uint32_t)report == (uint32_t)p.M) {
                        *err_count = (int32_t)(uint32_t)(report >> 32);
                        __hip_atomic_store(w_done, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
        }
    }
}

template <int TM, int TN, int W, bool kAny, bool kSplit>
hipError_t launch_any(bool check, bool want_c, bool want_q, const GemmParams& p_in, hipStream_t s) {
    GemmParams p = p_in;
    const int tiles_m = (p.M + 32 * TM - 1) / (32 * TM), tiles_n = (p.N + 32 * TN - 1) / (32 * TN);
    if ((int64_t)tiles_m * tiles_n > 65535) return hipErrorNotSupported;
    int shortest = p.KB2;   // stages of the shortest run
    if (kSplit) {
        const SplitKPlan pl = splitk_plan(p.M, p.N, p.KB2, !kAny);
        if (pl.z < 2 || p.ws == nullptr || p.ws_ints < pl.total_ints) return hipErrorNotSupported;
        p.ksplit = pl.z;
        p.ws_tickets = p.ws + pl.tickets_off;
        p.ws_part = p.ws + pl.part_off;
        p.split_q = p.KB2 / pl.z;
        p.split_r = p.KB2 % pl.z;
        shortest = p.split_q;
    }
    // k-steps of the checksum product per tile column, of a wavefront with wk_stages stages and of one with a stage more
    p.wk_stages = shortest / W;
    p.share_q = 4 * p.wk_stages / tiles_n;
    p.share_r = 4 * p.wk_stages % tiles_n;
    p.wk_share_q1 = 4 * (p.wk_stages + 1) / tiles_n;
    p.wk_share_r1 = 4 * (p.wk_stages + 1) % tiles_n;
    // A weight of a good part of the 256 MiB memory-side cache, read once, passes through without being kept there: with others of its size
    // in the program it would not be there at the next call (three weights in turn, us, kept / passed through: 16x16384x16384 52.1 / 46.2,
    // 12000x12000 and 8 rows 30.2 / 27.1, 16384x6400 and 32 rows 22.1 / 20.6; but 16x8192x8192 13.9 / 18.7; read by two rows of tiles,
    // 33x8192x12000, 24.6 / 36.4).  Up to 32 rows, which were always read that way; beyond, only what the cache cannot hold at all
    // (60 rows of 12000x12000 alone in a loop 28.6 / 38.3).  With tiles of 32 columns too (8x8192x16384 in a loop 22.0 / 22.6, fresh weights
    // 28.0 / 23.7).
    p.wk_stream = tiles_m == 1 && (int64_t)p.N * p.K >= (int64_t)(p.M <= 32 ? 96 : 224) << 20;
    const uint32_t per_strip = (uint32_t)(tiles_m < 4 ? tiles_m : 4) * (uint32_t)tiles_n;
    const uint32_t strip_rcp = per_strip == 1 ? 0u : (uint32_t)((0x100000000ull + per_strip - 1) / per_strip);
    const RowSlots rs = row_slots(p.M, tiles_n);
    const int slots = rs.slots, slot_rows = rs.rows;
    const dim3 grid((unsigned)(tiles_m * tiles_n * (kSplit ? p.ksplit : 1))), block(W * 64);
    const size_t lds = (size_t)W * wave_bytes<TM, TN>() + 64;   // (the wavefronts' parts, and their reports)
#define ABFT_LAUNCH(CK, OUT)                                                                              \
    do {                                                                                                  \
        auto kern = gemm_tile_wk_kernel<TM, TN, W, CK, OUT, kAny, kSplit>;                                \
        static std::atomic<uint64_t> lds_allowed{0};                                                      \
        const hipError_t e_attr = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds, lds_allowed);\
        if (e_attr != hipSuccess) return e_attr;                                                          \
        kern<<<grid, block, lds, s>>>(p, tiles_m, tiles_n, strip_rcp, slots, slot_rows);                  \
        return hipGetLastError();                                                                         \
    } while (0)
#define ABFT_OUT(CK)                                          \
    do {                                                      \
        if (want_c && want_q) ABFT_LAUNCH(CK, kOutC | kOutQ); \
        if (want_c) ABFT_LAUNCH(CK, kOutC);                   \
        ABFT_LAUNCH(CK, kOutQ);                               \
    } while (0)
    if (check) ABFT_OUT(true);
    ABFT_OUT(false);
#undef ABFT_OUT
#undef ABFT_LAUNCH
}

// (whole_a: A in whole, aligned 16-byte chunks and within 32-bit byte offsets, which the direct loads take)
template <int TM, int TN, int W, bool kSplit>
hipError_t launch_cfg(bool whole_a, bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s) {
    if (whole_a) return launch_any<TM, TN, W, false, kSplit>(check, want_c, want_q, p, s);
    if (p.K < 16) return hipErrorNotSupported;
    return launch_any<TM, TN, W, true, kSplit>(check, want_c, want_q, p, s);
}

}  // namespace wktile
}  // namespace abft
